// The BF16 producers with a workspace: the entry points of moss.h with the same names take none.  `workspace`: 16-byte aligned
// device memory of any contents, at least kProducerWorkspaceBytes, used by the call alone until it has run (nullptr, fewer bytes,
// and captured calls: as without).  Included by the kernels and by the binding's native calls.
#pragma once
#include <stddef.h>
#include <stdint.h>

constexpr size_t kProducerWorkspaceBytes = (2 * 2048 + 1) * 8;       // two words for each workgroup of the largest grid, one to hand over by

// What the callers of this library's functions were compiled for: the build hands the library and the binding's native calls one number
// made from moss.h and this file (0: built some other way, never the same as anything).
#ifndef MOSS_INTERFACE
#define MOSS_INTERFACE 0
#endif

extern "C" {
uint32_t moss_internal_interface(void);
int moss_internal_swiglu_bf16(const void *gate, const void *up, int64_t rows, int64_t cols, int64_t ld, void *h,
                              uint32_t *h_absmax_bits, void *workspace, size_t workspace_bytes, void *stream);
int moss_internal_swiglu_bf16_backward(const void *gate, const void *up, const void *dh, int64_t rows, int64_t cols, int64_t ld,
                                       void *d_gate, void *d_up, uint32_t *d_gate_absmax_bits, uint32_t *d_up_absmax_bits,
                                       void *workspace, size_t workspace_bytes, void *stream);
int moss_internal_add_rmsnorm_bf16(const void *x, const void *delta, const void *gamma, float eps, int64_t rows, int64_t cols,
                                   int64_t ld, void *h_out, void *y, uint32_t *y_absmax_bits, void *workspace,
                                   size_t workspace_bytes, void *stream);
int moss_internal_rmsnorm_bf16_backward(const void *h, const void *gamma, const void *dy, const void *d_res, float eps, int64_t rows,
                                        int64_t cols, int64_t ld, void *d_h, uint32_t *d_h_absmax_bits, void *workspace,
                                        size_t workspace_bytes, void *stream);
}
