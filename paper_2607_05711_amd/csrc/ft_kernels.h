// Internal launch interface between the C ABI (api.hip) and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>

namespace ft {

// 1x32 row quantization with the fused down-projection.  When the columns
// span several chunks, each chunk's fp32 projection partial goes to `ws`
// (quant_rows_workspace bytes) and a reduction kernel sums them into
// proj_out; otherwise proj_out is written directly and ws is unused.
// Numerics variants of the quantizers: the no-clip scale rule, stochastic
// rounding (Philox4x32-10 bits keyed by seed, counter words 2 and 3 = stream),
// and for 32x32 tiles scales written once per row.
struct QuantMode {
  bool no_clip = false;
  bool stochastic = false;
  uint64_t seed = 0, stream = 0;
  int scales_per_row = 0;
};
size_t quant_rows_workspace(int rows, int cols, int R, int layout);
hipError_t launch_quant_rows(const uint16_t* src, int rows, int cols, uint8_t* codes, uint8_t* scales,
                             const uint16_t* proj, int R, int layout, float* proj_out, float* ws, hipStream_t st,
                             const QuantMode& mode = QuantMode{});
// h = bf16(GELU(z)) stored and quantized, with the projection h . proj [cols, R]
// (R = 0: none; R <= 128); ws holds max_groups partials (max_chain: as below).
hipError_t launch_quant_gelu(const uint16_t* z, int rows, int cols, uint16_t* h, uint8_t* codes, uint8_t* scales,
                             const uint16_t* proj, int R, float* proj_out, float* ws, int max_groups, int max_chain,
                             hipStream_t st);
// Streaming form of the row quantization with a projection (nearest-even
// rounding): at most max_groups partials in ws, and no projection sum of more
// roundings than max_groups partials of max_chain each.  gelu_out: src is z, h =
// bf16(GELU(z)) is stored there and quantized (layout 0).
int quant_proj_steps(int rows, int cols, int R, int max_groups, int max_chain);
bool quant_proj_supported(int rows, int cols, int R);
hipError_t launch_quant_proj(const uint16_t* src, int rows, int cols, uint8_t* codes, uint8_t* scales,
                             const uint16_t* proj, int R, int layout, bool no_clip, float* proj_out, float* ws,
                             int max_groups, int max_chain, uint16_t* gelu_out, hipStream_t st);
// Partials that the row quantization's workspace holds, and the products that
// the chunked kernel adds into one of them.
void quant_rows_chain(int rows, int cols, int R, int layout, int& groups, int& chain);
hipError_t launch_quant_tiles(const uint16_t* src, int rows, int cols, uint8_t* codes, uint8_t* scales,
                              hipStream_t st, const QuantMode& mode = QuantMode{});

// out0 (+)= sum of nparts partials [n0 | n1] in ws; likewise out1.  n0, n1 multiples of 4.
hipError_t launch_reduce_parts(const float* ws, int nparts, size_t n0, float* out0, size_t n1, float* out1,
                               bool accumulate, hipStream_t st);

// FP4 GEMM.  bwd = false: out[M, N] = A[M, K] . W[N, K]^T  (+ P . U + bias)
//            bwd = true : out[M, K] = A[M, N] . W[N, K]    (+ P . D^T)
// z (bwd, bf16 out; NULL for none): out = bf16(that result * GELU'(z)), z bf16
// [M, K]; on small tiles only (no gemm_fp4_fuse_mlp).
hipError_t launch_gemm_fp4(bool bwd, const uint8_t* a, const uint8_t* as, const uint8_t* wq, const uint8_t* ws,
                           int M, int N, int K, const float* P, int R, const uint16_t* lr,
                           const uint16_t* bias, void* out, bool out_f32, const uint16_t* z, hipStream_t st);
// The same product on tm x 128 output tiles (tm = 64 or 128), any K and N that are
// multiples of 32; whether its 32-bit offsets and LDS hold this shape.
bool gemm_fp4_tile_supported(bool bwd, int M, int N, int K, int R, bool out_f32);
// LDS ring slots of a workgroup, and whether two workgroups share a CU.
struct TileSlots { bool two_per_cu; int ns; };
TileSlots gemm_fp4_tile_slots(int tm, long tiles, int KR);
hipError_t launch_gemm_fp4_tile(bool bwd, int tm, const uint8_t* a, const uint8_t* as, const uint8_t* wq,
                                const uint8_t* ws, int M, int N, int K, const float* P, int R, const uint16_t* lr,
                                const uint16_t* bias, void* out, bool out_f32, const uint16_t* z, hipStream_t st);
// Which kernel launch_gemm_fp4 takes: 256 (256x256 tiles), 128 or 64 (that many
// rows x 128 columns), 0 (register-staged).
int gemm_fp4_kernel(bool bwd, int M, int N, int K, int R, bool out_f32);

// Epilogues of the 256x256 kernel; GELU and DGELU finish the MLP pair's call
// (the output NO columns feed the next linear).
enum { EPI_PLAIN = 0, EPI_GELU = 1, EPI_DGELU = 2 };
struct GemmEpilogue {
  uint16_t* z_out;        // EPI_GELU: z = bf16(acc) [M, NO]
  const uint16_t* z_in;   // EPI_DGELU: z saved by the forward [M, NO]
  uint16_t* y;            // EPI_GELU: h = bf16(GELU(z));  EPI_DGELU: dz = bf16(acc GELU'(z))  [M, NO]
  uint8_t* q;             // E2M1 codes of y [M, NO/2]
  uint8_t* s;             // E8M0 scales of y [M, NO/32]
  const uint16_t* proj;   // EPI_GELU: D2 [NO, R2];  EPI_DGELU: U1 [R2, NO];  unused when R2 == 0
  int R2;                 // 0, 16, 32, 48 or 64
  float* parts;           // fp32 partials [tiles over NO][M][R2], or the projection when one tile spans NO
};
// Whether the MLP pair's call runs whole in the GEMM's epilogue.
bool gemm_fp4_fuse_mlp(bool bwd, int M, int N, int K, int R, int R2);
hipError_t launch_gemm_fp4_fused(bool bwd, const uint8_t* a, const uint8_t* as, const uint8_t* wq, const uint8_t* ws,
                                 int M, int N, int K, const float* P, int R, const uint16_t* lr, const uint16_t* bias,
                                 const GemmEpilogue& ep, float* proj_out, hipStream_t st);
// Whether the MLP pair's calls take this shape, and the number of projection
// partials that their workspace holds.
bool gemm_fp4_fused_supported(bool bwd, int M, int N, int K, int R, int R2);
int gemm_fp4_col_tiles(int NO);

// Adapter gradients; token chunks leave partials in ws (lora_grads_workspace bytes).
size_t lora_grads_workspace(int M, int K, int N, int ld, int r);
hipError_t launch_lora_grads(const uint16_t* x, int M, int K, const uint16_t* dy, int N, const float* xa,
                             const float* dyb, int ld, int r, float* dA, float* dB, bool accumulate, float* ws,
                             hipStream_t st);

// Size of the static device scratch the allocation-free adapter-gradient entry
// point uses in place of a workspace, and its device address on the current
// device (looked up on the first call per device).  Every call on one device
// shares it.
constexpr size_t kLoraScratchBytes = (size_t)32 << 20;
hipError_t lora_grads_scratch(float** ptr);

// NVFP4 emulation: quantization (1x16 or 16x16 blocks, E4M3 scales, the fp32
// tensor scale left in *tensor_scale) and the dequantizing bf16-MFMA GEMM
// (fp32 output, both tensor scales applied).
hipError_t launch_quant_nvfp4(const uint16_t* src, int rows, int cols, int block_rows, uint8_t* codes,
                              uint8_t* scales, float* tensor_scale, hipStream_t st);
hipError_t launch_gemm_nvfp4(bool bwd, const uint8_t* a, const uint8_t* as, const float* at, const uint8_t* wq,
                             const uint8_t* ws, const float* wt, int M, int N, int K, float* out, hipStream_t st);

}  // namespace ft
