"""GPU parity of the producer side of the quantizer: moss_swiglu_bf16 (+ backward) against the CPU
oracle's FP64 SwiGLU, and moss_quant_act_2level_given_max (the quantizer of Sec. 3.1, Eq. 2-3 with
the tensor maximum handed in) bit for bit against the oracle.

SwiGLU tolerance: the kernel evaluates in FP32 with hardware exp2 / reciprocal approximations and
rounds once to BF16, so an output is the correctly rounded BF16 value of the exact result except when
the exact result lies closer to a rounding boundary than the FP32 evaluation error (a few times 2^-20
relative): then it is the BF16 neighbour.  The test asserts |gpu - exact| <= (1/2 + 2^-9) BF16 ulp for
every element and that at most 0.5 % of the elements differ from the correctly rounded value.  The
maximum word must be exactly the largest magnitude bit pattern the kernel wrote."""
import numpy as np
import pytest
import torch

import moss_inputs as mi
import paper_2511_05811_amd as moss
from gpu_util import bf16_to_gpu, scalar, u8

pytestmark = pytest.mark.gpu
ROW, COL, CEIL = moss.MOSS_Q_ROW, moss.MOSS_Q_COL, moss.MOSS_EXP_CEIL


def bits_of(t):
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


def check_rounded(got_bits, exact, tag):
    got = mi.bf16_bits_to_f32(got_bits).astype(np.float64)
    ulp = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(exact), 2.0 ** -126))) - 7)      # BF16: 8 significant bits
    err = np.abs(got - exact)
    worst = float((err / ulp).max())
    want_bits = mi.f32_to_bf16_bits(exact.astype(np.float32))     # exact is far from FP32 resolution: good enough a stand-in
    off = float(np.mean(got_bits != want_bits))
    print(f"[swiglu parity] {tag}: max |err| = {worst:.4f} ulp, {off * 100:.4f} % not the nearest BF16", flush=True)
    assert worst <= 0.5 + 2.0 ** -9, tag
    assert off <= 5e-3, tag


def make_inputs(rows, cols, seed):
    rng = np.random.default_rng(seed)
    g = rng.standard_normal((rows, cols)) * 2.5
    g[rng.random((rows, cols)) < 0.01] *= 8.0                # a few far-out gates (sigmoid saturated either way)
    u = rng.standard_normal((rows, cols)) * 1.5
    d = rng.standard_normal((rows, cols)) * 1e-3
    return mi.f32_to_bf16_bits(g.astype(np.float32)), mi.f32_to_bf16_bits(u.astype(np.float32)), mi.f32_to_bf16_bits(d.astype(np.float32))


@pytest.mark.parametrize("shape", [(1, 8), (3, 40), (32, 64), (257, 1000), (1024, 2048 + 8)])
def test_swiglu_forward_and_backward(oracle, shape):
    rows, cols = shape
    gb, ub, db = make_inputs(rows, cols, rows * 31 + cols)
    g, u, d = bf16_to_gpu(gb), bf16_to_gpu(ub), bf16_to_gpu(db)
    h, hmax = moss.swiglu_bf16(g, u)
    dg, du, dgmax, dumax = moss.swiglu_bf16_backward(g, u, d)
    torch.cuda.synchronize()
    hb, dgb, dub = bits_of(h), bits_of(dg), bits_of(du)
    check_rounded(hb, oracle.swiglu(gb, ub), f"h {shape}")
    eg, eu = oracle.swiglu_backward(gb, ub, db)
    check_rounded(dgb, eg, f"d_gate {shape}")
    check_rounded(dub, eu, f"d_up {shape}")
    assert int(hmax.item()) == int((hb & 0x7FFF).max())
    assert int(dgmax.item()) == int((dgb & 0x7FFF).max())
    assert int(dumax.item()) == int((dub & 0x7FFF).max())


@pytest.mark.parametrize("shape", [(3, 43688), (128, 1024), (257, 1032), (129, 4064), (64, 8192)])
def test_swiglu_with_one_two_and_four_chunks_per_thread(oracle, shape):
    # 2^14 and 2^16 chunks are the first tensors with two and four; below and above them, with trips that are not full
    test_swiglu_forward_and_backward(oracle, shape)


def equals_its_parts(rows, cols, cut):
    # the same bits as in two parts, which take other forms.  (A gate below -88.7, which the oracle's tests do not reach,
    # overflows the exponential in FP32: those outputs, of less than 1e-35, are zero, and alike here.)
    g, u, d = (bf16_to_gpu(a) for a in make_inputs(rows, cols, 5))
    h, hmax = moss.swiglu_bf16(g, u)
    dg, du, dgmax, dumax = moss.swiglu_bf16_backward(g, u, d)
    tops = [0, 0, 0]
    for part_rows in (slice(0, cut), slice(cut, rows)):
        ph, pm = moss.swiglu_bf16(g[part_rows], u[part_rows])
        pg, pu, pgm, pum = moss.swiglu_bf16_backward(g[part_rows], u[part_rows], d[part_rows])
        torch.cuda.synchronize()
        for whole, part in ((h, ph), (dg, pg), (du, pu)):
            assert np.array_equal(bits_of(whole[part_rows]), bits_of(part))
        tops = [max(a, int(b.item())) for a, b in zip(tops, (pm, pgm, pum))]
    assert tops == [int(t.item()) for t in (hmax, dgmax, dumax)]


def test_swiglu_of_more_than_32_mib_equals_its_parts():
    equals_its_parts(2049, 8200, 1000)         # above 2^24 elements the outputs are stored through the caches


@pytest.mark.parametrize("rows,cols,cut", [(383, 8192, 100),     # the largest tensor whose workgroups merge without a look, ...
                                           (384, 8200, 20)])     # ... and one whose workgroups look first
def test_swiglu_on_both_sides_of_the_look_equals_its_parts(rows, cols, cut):
    equals_its_parts(rows, cols, cut)


def test_swiglu_on_a_strided_view_and_zero_tensor(oracle):
    rows, cols, ld = 64, 96, 128
    gb, ub, _ = make_inputs(rows, ld, 7)
    g_full, u_full = bf16_to_gpu(gb), bf16_to_gpu(ub)
    g, u = g_full[:, :cols], u_full[:, :cols]
    h_full = torch.full((rows, ld), 3.0, dtype=torch.bfloat16, device=g.device)
    h, hmax = moss.swiglu_bf16(g, u, h=h_full[:, :cols])
    torch.cuda.synchronize()
    check_rounded(bits_of(h), oracle.swiglu(gb[:, :cols], ub[:, :cols]), "strided")
    assert (h_full[:, cols:] == 3.0).all()                   # the padding columns are not touched
    assert int(hmax.item()) == int((bits_of(h) & 0x7FFF).max())
    z = torch.zeros((32, 64), dtype=torch.bfloat16, device=g.device)
    hmax.fill_(12345)                                        # the word is written, not accumulated
    h, hmax = moss.swiglu_bf16(z, u_full[:32, :64].contiguous(), absmax_bits=hmax)
    torch.cuda.synchronize()
    assert int(hmax.item()) == 0 and (bits_of(h) & 0x7FFF).max() == 0


@pytest.mark.parametrize("flag", [0, CEIL])
@pytest.mark.parametrize("shape", [(32, 64), (96, 160), (1056, 2080), (4128, 3104)])
def test_quantizer_with_the_maximum_handed_in(oracle, shape, flag):
    rows, cols = shape
    mode = 1 if flag else 0
    xb = mi.heavy_tailed_activation(rows, cols, seed=rows + cols + mode)
    x = bf16_to_gpu(xb)
    true_bits = int((xb & 0x7FFF).max())
    for given in (true_bits, true_bits + 1, true_bits + 200):
        word = torch.tensor([given], dtype=torch.int32, device=x.device)
        qr, er, s = oracle.quant_act_2level_given_max(xb, given, 0, mode)
        qc, ec, _ = oracle.quant_act_2level_given_max(xb, given, 1, mode)
        for f in (ROW, COL, ROW | COL):
            got = moss.quant_act_2level_given_max(x, word, f | flag)
            torch.cuda.synchronize()
            assert scalar(got["s"]) == s, (shape, given, f)
            if f & ROW:
                assert np.array_equal(u8(got["q_row"]), qr) and np.array_equal(u8(got["e_row"]), er), (shape, given, f)
            if f & COL:
                assert np.array_equal(u8(got["q_col"]), qc) and np.array_equal(u8(got["e_col"]), ec), (shape, given, f)
    # with the true maximum: the searching entry point's outputs, bit for bit
    ref = moss.quant_act_2level(x, ROW | COL | flag)
    got = moss.quant_act_2level_given_max(x, torch.tensor([true_bits], dtype=torch.int32, device=x.device), ROW | COL | flag)
    torch.cuda.synchronize()
    for k in ("q_row", "e_row", "q_col", "e_col", "s"):
        assert torch.equal(ref[k], got[k]), k


def test_quantizer_with_the_maximum_handed_in_on_a_strided_view(oracle):
    rows, cols, ld = 1056, 2080, 2304
    full = mi.heavy_tailed_activation(rows, ld, seed=17)
    xb = np.ascontiguousarray(full[:, :cols])
    x = bf16_to_gpu(full)[:, :cols]
    given = int((xb & 0x7FFF).max())
    got = moss.quant_act_2level_given_max(x, torch.tensor([given], dtype=torch.int32, device=x.device), ROW | COL)
    torch.cuda.synchronize()
    qr, er, s = oracle.quant_act_2level(xb, 0, 0)
    qc, ec, _ = oracle.quant_act_2level(xb, 1, 0)
    assert scalar(got["s"]) == s
    assert np.array_equal(u8(got["q_row"]), qr) and np.array_equal(u8(got["e_row"]), er)
    assert np.array_equal(u8(got["q_col"]), qc) and np.array_equal(u8(got["e_col"]), ec)


def test_swiglu_feeds_the_quantizer_in_one_pass(oracle):
    """The chain the two entry points are for: SwiGLU writes h and its maximum, the quantizer reads h once.
    The codes are those the oracle's quantizer gives for the h the GPU wrote."""
    rows, cols = 2048, 2752
    gb, ub, _ = make_inputs(rows, cols, 99)
    g, u = bf16_to_gpu(gb), bf16_to_gpu(ub)
    h, hmax = moss.swiglu_bf16(g, u)
    got = moss.quant_act_2level_given_max(h, hmax, ROW | COL)
    torch.cuda.synchronize()
    hb = bits_of(h)
    qr, er, s = oracle.quant_act_2level(hb, 0, 0)
    qc, ec, _ = oracle.quant_act_2level(hb, 1, 0)
    assert scalar(got["s"]) == s
    assert np.array_equal(u8(got["q_row"]), qr) and np.array_equal(u8(got["e_row"]), er)
    assert np.array_equal(u8(got["q_col"]), qc) and np.array_equal(u8(got["e_col"]), ec)


@pytest.mark.parametrize("rows,cols,pad", [(1, 8, 0), (32, 256, 8), (640, 1024, 0), (1033, 2056, 64), (4096, 2048, 0), (8192, 4096, 0)])
def test_maximum_words_from_slots_are_those_of_the_atomics(rows, cols, pad):
    """An eager call folds the maxima of up to 2048 workgroups in scratch of its own, a captured one merges them into the
    words: same tensors and same words, twice in a row, and the words are the largest magnitudes written."""
    gen = torch.Generator(device="cuda:0").manual_seed(rows + cols)
    make = lambda: torch.randn(rows, cols + pad, generator=gen, device="cuda:0").bfloat16()[:, :cols]
    a, b, c = make(), make(), make()
    gamma = torch.randn(cols, generator=gen, device="cuda:0").bfloat16()
    calls = (lambda: moss.swiglu_bf16(a, b), lambda: moss.swiglu_bf16_backward(a, b, c), lambda: moss.add_rmsnorm_bf16(a, gamma, 1e-5, delta=b),
             lambda: moss.rmsnorm_bf16_backward(a, gamma, b, 1e-5, d_res=c))
    for k, call in enumerate(calls):
        graph = torch.cuda.CUDAGraph()
        call()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            want = call()
        graph.replay()
        for again in range(2):
            got = call()
            torch.cuda.synchronize()
            for x, y in zip(got, want):
                assert torch.equal(x, y), (k, again)
        tensors = [t for t in got if t.dtype == torch.bfloat16][-2 if k == 1 else -1:]
        words = [t for t in got if t.dtype == torch.int32]
        for t, w in zip(tensors, words):
            assert int(w) == int((t.contiguous().view(torch.int16).int() & 0x7FFF).max()), k


@pytest.mark.parametrize("rows,cols", [(1, 8), (32, 256), (1033, 2056), (8192, 4096)])
def test_maximum_words_of_a_fold_that_is_handed_over(rows, cols):
    """With no look at the others' slots (limit 0) the last workgroup hands the fold over at once, to itself or to whichever
    comes later: the words are the largest magnitudes written, in every one of many calls."""
    gen = torch.Generator(device="cuda:0").manual_seed(rows + cols)
    a, b, c = (torch.randn(rows, cols, generator=gen, device="cuda:0").bfloat16() for _ in range(3))
    gamma = torch.randn(cols, generator=gen, device="cuda:0").bfloat16()
    calls = (lambda w: moss.swiglu_bf16(a, b, absmax_bits=w[0])[:1], lambda w: moss.swiglu_bf16_backward(a, b, c, d_gate_absmax_bits=w[0], d_up_absmax_bits=w[1])[:2],
             lambda w: moss.add_rmsnorm_bf16(a, gamma, 1e-5, delta=b, absmax_bits=w[0])[1:2],
             lambda w: moss.rmsnorm_bf16_backward(a, gamma, b, 1e-5, d_res=c, absmax_bits=w[0])[:1])
    moss.quant_set_poll_limit(0)
    try:
        for k, call in enumerate(calls):
            print(f"[fold handed over] {rows}x{cols} producer {k}", flush=True)
            words = torch.full((50, 2, 1), -1, dtype=torch.int32, device="cuda:0")
            for again in range(50):
                tensors = call(words[again])
            torch.cuda.synchronize()
            for j, t in enumerate(tensors):
                assert bool((words[:, j] == (t.view(torch.int16).int() & 0x7FFF).max()).all()), (k, j)
    finally:
        moss.quant_set_poll_limit(32768)
