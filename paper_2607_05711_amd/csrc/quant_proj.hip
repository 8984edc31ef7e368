// 1x32 MXFP4 quantization of bf16 rows fused with a low-rank projection of the
// same rows (FourTune Sec. 3.1 and 3.3), streaming form (gfx950), optionally
// with GELU in front (the MLP pair: src is z, h = bf16(GELU(z)) is stored and
// quantized).
//
// Workgroup: 4 waves over 128 rows x a run of 64-column steps.  A step's rows
// (each wave its own 32) and its 64 columns of the projection matrix come by
// buffer loads that write LDS directly, four steps ahead of the one in use
// (three for projections wider than 96),
// so no registers hold data in flight and the loads never wait for
// arithmetic.  A wave reads its rows from LDS in the MFMA operand layout
// (lane = row, lanes l and l + 32 sharing one) and quantizes them there: a
// 32-element block lies in one lane pair, whose block maximum takes one swap
// between half-waves, and two more swaps turn its codes into 16 contiguous
// bytes per lane.  The same registers are the B operand of the projection.
//
// Bound by HBM; one wave per SIMD does a step's arithmetic in about a third of
// the time that its bytes take, so one workgroup with a deep ring per CU is
// enough (two with three slots each: 39 us against 36 at 4608 x 12288).  The
// projection's partial sums, one per run, go to the workspace and are added in
// order by k_reduce_parts.  With that reduction, back to back on one box, against
// the chunked kernel of quantize.hip (nearest-even rounding used it before):
// 4608 x 12288, R = 64 44 -> 36 us ([R, cols]) and 43 -> 36 ([cols, R]); 18432 x
// 21504, R = 96 297 -> 277; 18432 x 15360 227 -> 202; 18432 x 3072, R = 64 43 -> 39;
// 512 x 3072 12.0 -> 10.2; 4608 x 9216 28 either way; of 71 sizes in both layouts
// none more than 4 % slower.  With GELU, the form of the MLP pair's calls on small
// GEMM tiles, 4608 x 12288 takes 65 us (258 MB; the chunked kernel 82).
#include "ft_device.h"
#include "ft_kernels.h"

namespace ft {

namespace {

constexpr int QP_ROWS = 128;                      // rows per workgroup
constexpr int QP_X = QP_ROWS * 128;               // bytes of rows per step

typedef unsigned short v2u16 __attribute__((ext_vector_type(2)));

template <int RT>
struct QpGeom {
  static constexpr int PROJ = RT * 32 * 128;      // bytes of the projection's step
  static constexpr int SLOT = QP_X + PROJ;
  static constexpr int NS = RT == 4 ? 4 : 5;      // ring slots
  // Accumulator sets: a step's four products go round them, so that a sum's
  // fp32 chain is one product a step long (quant_proj_steps bounds it).
  static constexpr int SETS = 4;
  static constexpr int LOADS = 4 + RT;            // per wave and step
};

// XOR of the 16-byte chunk index of row k in the staged [64 k][RT*32 j] tile:
// the four rows of a transposing read fall into different banks.
template <int RT>
__device__ __forceinline__ int qp_swz(int k) { return RT % 2 == 0 ? 2 * (k & 3) : 2 * ((k >> 1) & 1); }

// The pair (lanes l, l + 32): a's upper half and b's lower half change places.
__device__ __forceinline__ void swap_halves(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

}  // namespace

// MODE 1: proj is [cols, R]; MODE 2: proj is [R, cols].
template <int RT, int MODE, int QM, bool GELU>
__global__ __launch_bounds__(256) void k_quant_proj(const uint16_t* __restrict__ src, int rows, int cols,
                                                    uint8_t* __restrict__ codes, uint8_t* __restrict__ scales,
                                                    const uint16_t* __restrict__ proj, int R,
                                                    float* __restrict__ proj_out, float* __restrict__ parts, int spg,
                                                    uint16_t* __restrict__ h_out) {
  using G = QpGeom<RT>;
  __shared__ __attribute__((aligned(16))) uint8_t lds[G::NS * G::SLOT];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, h = lane >> 5, g16 = lane >> 4, t16 = lane & 15, jj = t16 >> 2, qq = t16 & 3;
  const int r8 = lane >> 3, c8 = (lane & 7) ^ r8;
  const int row0 = blockIdx.x * QP_ROWS, nrow = min(QP_ROWS, rows - row0);
  const int nsteps = (cols + 63) >> 6, s0 = blockIdx.y * spg, s1 = min(s0 + spg, nsteps);
  const int nbc = cols >> 5;
  const uint32_t lds0 = lds_addr(lds);

  // Buffers start at the workgroup's first row: offsets stay below 2 GiB for
  // any row count.
  const v4i rx = rsrc_words(src + (size_t)row0 * cols, (uint32_t)nrow * cols * 2);
  const v4i rp = rsrc_words(proj, (uint32_t)R * cols * 2);
  const __amdgpu_buffer_rsrc_t rc = make_rsrc(codes + (size_t)row0 * (cols >> 1), (uint32_t)nrow * (cols >> 1));
  const __amdgpu_buffer_rsrc_t rh = make_rsrc(GELU ? h_out + (size_t)row0 * cols : nullptr, GELU ? (uint32_t)nrow * cols * 2 : 0u);

  // Row load i brings rows 8 i + lane / 8 of the wave's 32; physical chunk
  // lane % 8 holds logical chunk c8 ^ (i & 1).
  uint32_t xoff[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int r = wave * 32 + 8 * i + r8;
    xoff[i] = r < nrow ? (uint32_t)r * cols * 2 + (c8 ^ (i & 1)) * 16 : kOobOffset;
  }
  uint32_t poff[RT];
  int pcol[RT];   // first column (of the step's 64) that the lane's chunk holds
#pragma unroll
  for (int v = 0; v < RT; v++) {
    if constexpr (MODE == 2) {   // rows j of the tile [RT*32 j][64 k]
      const int j = 8 * (wave * RT + v) + r8, c = c8 ^ ((wave * RT + v) & 1);
      poff[v] = j < R ? (uint32_t)j * cols * 2 + c * 16 : kOobOffset;
      pcol[v] = 8 * c;
    } else {                     // [64 k][RT*32 j]
      const int p = (wave * RT + v) * 64 + lane, k = p / (RT * 4), c = (p % (RT * 4)) ^ qp_swz<RT>(k);
      poff[v] = 8 * c < R ? (uint32_t)(k * R + 8 * c) * 2 : kOobOffset;
      pcol[v] = k;
    }
  }
  auto issue = [&](int s, int slot) {
    const uint32_t base = lds0 + (uint32_t)slot * G::SLOT;
    const int left = s < s1 ? cols - 64 * s : 0;   // columns from this step on; none past the run
#pragma unroll
    for (int i = 0; i < 4; i++)
      dma16(rx, base + wave * 4096 + i * 1024, 8 * (c8 ^ (i & 1)) < left ? xoff[i] : kOobOffset, (uint32_t)s * 128);
#pragma unroll
    for (int v = 0; v < RT; v++)
      dma16(rp, base + QP_X + (wave * RT + v) * 1024, pcol[v] < left ? poff[v] : kOobOffset,
            MODE == 2 ? (uint32_t)s * 128 : (uint32_t)s * 128 * R);
  };
#pragma unroll 1
  for (int u = 0; u < G::NS - 1; u++) issue(s0 + u, u);

  v16f acc[RT][G::SETS];
#pragma unroll
  for (int t = 0; t < RT; t++)
#pragma unroll
    for (int e = 0; e < G::SETS; e++) acc[t][e] = v16f{};
  const int sw = swz128(r32);
  const int wrow = wave * 32 + r32;                // this lane's row within the workgroup
  const uint32_t coff = wrow < nrow ? (uint32_t)wrow * (cols >> 1) + 16 * h : kOobOffset;
  uint32_t sword = 0;                              // scale bytes of a pair of steps
  int slot = 0;

#pragma unroll 1
  for (int s = s0; s < s1; s++) {
    // Step s's loads have landed: all but those of the NS - 2 steps behind it
    // and, once NS - 1 steps have run, the stores of those steps (at least
    // STORES each), which were issued after them too.
    constexpr int STORES = GELU ? 5 : 1;
    if (s - s0 >= G::NS - 1) wait_vm<G::LOADS * (G::NS - 2) + STORES * (G::NS - 1)>();
    else wait_vm<G::LOADS * (G::NS - 2)>();
    static_assert(G::LOADS * (G::NS - 2) + STORES * (G::NS - 1) < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt(0xc07f);            // this wave's reads of the previous step are done
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue(s + G::NS - 1, slot == 0 ? G::NS - 1 : slot - 1);
    uint8_t* xb = lds + slot * G::SLOT + wave * 4096;
    const uint8_t* pb = lds + slot * G::SLOT + QP_X;
    if constexpr (GELU) {
      // as stored: eight lanes hold one row's 128 bytes
#pragma unroll
      for (int i = 0; i < 4; i++) {
        v4i z = *(const v4i*)(xb + i * 1024 + lane * 16);
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const v2f hv = {gelu_tanh(bf16_to_f32((uint32_t)z[e] & 0xFFFFu)), gelu_tanh(bf16_to_f32((uint32_t)z[e] >> 16))};
          z[e] = (int)__builtin_bit_cast(uint32_t, __builtin_convertvector(hv, v2bf));
        }
        *(v4i*)(xb + i * 1024 + lane * 16) = z;
        __builtin_amdgcn_raw_buffer_store_b128(z, rh, 64 * s + 8 * (c8 ^ (i & 1)) < cols ? xoff[i] : kOobOffset, s * 128, 0);
      }
    }
    v4i x[4];
#pragma unroll
    for (int kk = 0; kk < 4; kk++) x[kk] = *(const v4i*)(xb + r32 * 128 + (((2 * kk + h) ^ sw) << 4));
    uint32_t o[4], code[2];
#pragma unroll
    for (int b = 0; b < 2; b++) {
      v2u16 p[8];
#pragma unroll
      for (int e = 0; e < 8; e++) p[e] = __builtin_bit_cast(v2u16, (uint32_t)x[2 * b + (e >> 2)][e & 3] & 0x7FFF7FFFu);
#pragma unroll
      for (int n = 4; n > 0; n >>= 1)
#pragma unroll
        for (int e = 0; e < n; e++) p[e] = __builtin_elementwise_max(p[e], p[e + n]);
      uint32_t m = max((uint32_t)p[0][0], (uint32_t)p[0][1]), other = m;
      swap_halves(m, other);
      code[b] = e8m0_of<QM>(max(m, other));
      const float sc = e8m0_to_f32(code[b]);
#pragma unroll
      for (int u = 0; u < 2; u++) {
        const v4i w = x[2 * b + u];
        uint32_t q = 0;
        q = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(q, __builtin_bit_cast(v2bf, (int)w[0]), sc, 0);
        q = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(q, __builtin_bit_cast(v2bf, (int)w[1]), sc, 1);
        q = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(q, __builtin_bit_cast(v2bf, (int)w[2]), sc, 2);
        q = __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(q, __builtin_bit_cast(v2bf, (int)w[3]), sc, 3);
        o[2 * b + u] = q;
      }
    }
    // codes of chunks h, 2 + h, 4 + h, 6 + h -> the lower half-wave's 0..3, the upper's 4..7
    swap_halves(o[0], o[2]);
    swap_halves(o[1], o[3]);
    __builtin_amdgcn_raw_buffer_store_b128(v4i{(int)o[0], (int)o[2], (int)o[1], (int)o[3]}, rc,
                                           64 * s + 32 * h < cols ? coff : kOobOffset, s * 32, 0);
    // scale bytes: a pair of steps (runs begin at even steps) is one dword of the row
    const uint32_t two = code[0] | (code[1] << 8);
    sword = (s & 1) ? sword | (two << 16) : two;
    if (((s & 1) || s + 1 == s1) && h == 0 && wrow < nrow) {
      uint8_t* d = scales + (size_t)(row0 + wrow) * nbc + 2 * (s & ~1);
      const int n = min(4, nbc - 2 * (s & ~1));
      if ((nbc & 3) == 0 && n == 4) *(uint32_t*)d = sword;
      else
        for (int b = 0; b < n; b++) d[b] = (uint8_t)(sword >> (8 * b));
    }
#pragma unroll
    for (int kk = 0; kk < 4; kk++)
#pragma unroll
      for (int t = 0; t < RT; t++) {
        v8bf a;
        if constexpr (MODE == 2) {
          a = __builtin_bit_cast(v8bf, *(const v4i*)(pb + (32 * t + r32) * 128 + (((2 * kk + h) ^ sw) << 4)));
        } else {
          const int k = 16 * kk + 8 * h + jj, ch = 4 * t + 2 * (g16 & 1) + (qq >> 1);
          const uint8_t* p = pb + k * (RT * 64) + ((ch ^ qp_swz<RT>(k)) << 4) + (qq & 1) * 8;   // row k + 4: same swizzle
          a = make_v8bf(lds_read_tr16((const FT_LDS void*)p), lds_read_tr16((const FT_LDS void*)(p + 4 * RT * 64)));
        }
        acc[t][kk % G::SETS] = mfma_bf16_32x32x16(a, __builtin_bit_cast(v8bf, x[kk]), acc[t][kk % G::SETS]);
      }
    slot = slot + 1 == G::NS ? 0 : slot + 1;
  }
  wait_vm<0>();   // the zeros of steps past the run have landed

  // sums: lane = row, element 4 q + e = projection column 32 t + 8 q + 4 h + e
  float* dst = parts ? parts + (size_t)blockIdx.y * rows * R : proj_out;
  if (wrow < nrow) {
#pragma unroll
    for (int t = 0; t < RT; t++) {
      const v16f sum = (acc[t][0] + acc[t][1]) + (acc[t][2] + acc[t][3]);
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int j = 32 * t + 8 * q + 4 * h;
        if (j < R) *(v4f*)(dst + (size_t)(row0 + wrow) * R + j) = v4f{sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]};
      }
    }
  }
}

bool quant_proj_supported(int rows, int cols, int R) {
  // 32-bit offsets within a workgroup's rows and the projection matrix
  return (size_t)QP_ROWS * cols * 2 < ((size_t)1 << 31) && (size_t)cols * R * 2 < ((size_t)1 << 31);
}

// Steps per workgroup so that at most max_groups partials result, by estimated
// time in steps: rounds of workgroups (one per CU) times a run's steps and the
// four that its start and end cost, and what each partial adds in traffic
// (written and read, 4 R bytes a row, where a step of a round moves 20 KB per CU).
// A projection's sum rounds once per step, where the sets meet (their three sums
// weigh as much as four products of a chain) and once per partial; that chain
// stays within max_chain + max_groups, so that long rows over many row blocks,
// which fill the chip without partials, still have some.  32768 x 21504, R = 96,
// [R, cols]: one run of 336 steps takes 446 us with an error of 4.6e-7 (2-norm),
// the bound 466 us and 2.6e-7, the chunked kernel took 533 us and 2.8e-7.
int quant_proj_steps(int rows, int cols, int R, int max_groups, int max_chain) {
  const int nsteps = (cols + 63) / 64;
  const long rb = (rows + QP_ROWS - 1) / QP_ROWS;
  int best = ((nsteps + max_groups - 1) / max_groups + 1) & ~1;
  double best_cost = 1e30;
  for (int g = 1; g <= max_groups && g <= nsteps; g++) {
    const int spg = ((nsteps + g - 1) / g + 1) & ~1;   // even: scale dwords stay whole
    const long groups = (nsteps + spg - 1) / spg;
    if (std::min(spg, nsteps) + 4 + groups > max_chain + max_groups) continue;
    const double cost = (double)((rb * groups + 255) / 256) * (spg + 4) +
                        (groups > 1 ? (double)groups * rows * R * 8.0 / (256 * 20480.0) : 0.0);
    if (cost < best_cost) { best_cost = cost; best = spg; }
  }
  return best;
}

template <int QM, bool GELU>
static hipError_t launch_qp(const uint16_t* src, int rows, int cols, uint8_t* codes, uint8_t* scales, const uint16_t* proj,
                            int R, int layout, float* proj_out, float* ws, int max_groups, int max_chain, uint16_t* h,
                            hipStream_t st) {
  const int spg = quant_proj_steps(rows, cols, R, max_groups, max_chain);
  const int groups = ((cols + 63) / 64 + spg - 1) / spg;
  dim3 grid((rows + QP_ROWS - 1) / QP_ROWS, groups);
  float* parts = groups > 1 ? ws : nullptr;
#define FT_QP(RT_, MODE_) \
  k_quant_proj<RT_, MODE_, QM, GELU><<<grid, 256, 0, st>>>(src, rows, cols, codes, scales, proj, R, proj_out, parts, spg, h)
  const int rt = (R + 31) / 32;
  if (layout == 0) {
    switch (rt) {
      case 1: FT_QP(1, 1); break;
      case 2: FT_QP(2, 1); break;
      case 3: FT_QP(3, 1); break;
      default: FT_QP(4, 1); break;
    }
  } else if constexpr (!GELU) {
    switch (rt) {
      case 1: FT_QP(1, 2); break;
      case 2: FT_QP(2, 2); break;
      case 3: FT_QP(3, 2); break;
      default: FT_QP(4, 2); break;
    }
  }
#undef FT_QP
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !parts) return e;
  return launch_reduce_parts(parts, groups, (size_t)rows * R, proj_out, 0, nullptr, false, st);
}

hipError_t launch_quant_proj(const uint16_t* src, int rows, int cols, uint8_t* codes, uint8_t* scales,
                             const uint16_t* proj, int R, int layout, bool no_clip, float* proj_out, float* ws,
                             int max_groups, int max_chain, uint16_t* gelu_out, hipStream_t st) {
#define FT_QPL(QM_, GELU_, LAYOUT_) \
  launch_qp<QM_, GELU_>(src, rows, cols, codes, scales, proj, R, LAYOUT_, proj_out, ws, max_groups, max_chain, gelu_out, st)
  if (gelu_out) return FT_QPL(0, true, 0);
  if (no_clip) return FT_QPL(QM_NOCLIP, false, layout);
  return FT_QPL(0, false, layout);
#undef FT_QPL
}

}  // namespace ft
