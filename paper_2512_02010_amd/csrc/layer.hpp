// What the Python module runs for paper_2512_02010_amd/linear.py besides the C ABI.  Exported by the library, but no
// part of its interface: the module is built with it and is all that calls it.
#pragma once

#include <cstddef>
#include <cstdint>

extern "C" {

// What linear.py runs where few_rows_in_one_launch() says so.  The same
// codes as nvfp4_46_scale_quantize (rowwise, to nearest, 4/6 by squared error) finds for x [M][K] BF16, their product with B
// as nvfp4_46_gemm takes it, C in BF16; the same checks and statuses, ERR_UNSUPPORTED for any other size.
int nvfp4_46_few_rows(const void *x, float fp8_max, const void *codes_b, const void *scales_b, const float *alpha_b,
                      int64_t M, int64_t N, int64_t K, uint32_t flags, void *out, void *stream);

// Both operands of linear.py's weight gradient, dy [rows][n] rounded
// stochastically and x [rows][k] to nearest, BF16, columnwise with the transform: what two calls of
// nvfp4_46_scale_quantize give, with their checks and statuses, in two launches instead of four where there are scratch words
// for it.
int nvfp4_46_wgrad_operands(const void *dy, const void *x, int64_t rows, int64_t n, int64_t k, uint32_t select,
                            uint64_t sr_seed, uint64_t rht_seed, float *alpha_dy, void *codes_dy, void *scales_dy,
                            float *alpha_x, void *codes_x, void *scales_x, void *workspace, size_t workspace_bytes,
                            void *stream);
}
