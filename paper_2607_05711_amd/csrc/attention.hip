// Joint attention of a DiT block, head dimension 128 (gfx950): softmax(q k^T /
// sqrt(128)) v over all tokens, forward and backward, bf16 in and out with
// fp32 sums.  Every sum has a fixed order, so results repeat bit for bit.
//
// Forward and dq: a wave owns 32 NI rows of q (NI 32-row MFMA tiles), kept in
// registers as MFMA operands, and walks the keys; dk and dv: a wave owns 32 NI
// keys and walks the rows of q.  The walked tensors pass through LDS in
// 64-row stages, double-buffered, by buffer loads that write LDS directly.
// With NI = 2 each byte read from LDS feeds two MFMAs, 64 bytes a clock and CU
// with the matrix cores busy; with NI = 1 one, 128, but two
// workgroups share a CU (forward and dq) and hide each other's waits: at 4608
// tokens and 24 heads the forward takes 335 us with NI = 1 and 388 with 2.
// The dk/dv kernel's 128 accumulators per tile leave a CU one workgroup either
// way; it takes NI = 2 where that makes fewer rounds.
// Bound by the matrix cores and the vector unit sharing a wave's time (an
// exponential and some ten operations per score beside 64 or more MFMA cycles):
// at 4608 x 24 heads x 128 the forward runs at 780 TFLOP/s and the backward
// (seven products) at 830; the library's attention, whose backward may add
// with atomics, took 505 us and 2460 us (1290 us with atomics), these
// kernels 335 and 1100.
//
// Scores are computed transposed where it saves data movement: a score tile's
// lanes are always the rows that the wave owns and its registers the walked
// rows, so a row's maximum and sum stay in one lane pair, and the tile is,
// after conversion to bf16, the B operand of the next product as it stands.
// (The MFMA's reduction index runs over the walked rows in the order of the
// tile's registers, 4h + {0..3}, 8 + 4h + {0..3} within 16; the other operand
// comes from transposing LDS reads at the same rows.)
#include "../../include/fourtune.h"
#include "ft_device.h"
#include "ft_kernels.h"

namespace ft {

namespace {

constexpr int HD = 128;
constexpr int AROW = HD * 2;                 // bytes per row
constexpr int AST = 64;                      // walked rows per stage
constexpr int ATILE = AST * AROW;            // 16 KB per tensor and stage
template <int NI> constexpr int ablk() { return 128 * NI; }   // rows owned by a workgroup of 4 waves
constexpr float kLog2e = 1.4426950408889634f;

// 16-byte chunk swizzle of a 256-byte row: LDS serves 16 lanes' 16-byte reads
// together, so sixteen rows at one chunk (row reads), and four rows at four
// chunks (transposing reads), fall into the sixteen different places.
// With an eight-place swizzle half of LDS's busy cycles were conflicts (4608 x
// 24 heads, forward: 32.2 of 65.4 million; now 0.3 of 33.5): forward 155 -> 143
// million busy CU cycles, dq 162 -> 154, dk/dv unchanged; in time less, as the
// clock falls with the load (double-stream block forward 1022 -> 1017 us).
__device__ __forceinline__ int aswz(int r) { return ((r & 3) << 2) | (((r >> 2) & 1) << 1) | ((r >> 3) & 1); }

struct Rows {            // element (row, head, d) at row * ts + head * hs + d
  const uint16_t* p;
  int64_t ts, hs;
};

// Larger of the two halves' values of a lane pair (l, l + 32), and their sum.
__device__ __forceinline__ float pair_max(float x) { return fmaxf(x, __shfl_xor(x, 32, 64)); }
__device__ __forceinline__ float pair_sum(float x) { return x + __shfl_xor(x, 32, 64); }

__device__ __forceinline__ v8bf pack_b(const v16f& s, int v) {
  v4i r;
#pragma unroll
  for (int e = 0; e < 4; e++) {
    const v2f x = {s[v + 2 * e], s[v + 2 * e + 1]};
    r[e] = (int)__builtin_bit_cast(uint32_t, __builtin_convertvector(x, v2bf));
  }
  return __builtin_bit_cast(v8bf, r);
}

// Loads of walked rows [64 s, + 64) of one tensor into LDS: wave w fills rows
// 16 w .. + 15, four per instruction; rows past the end read zeros.
struct Walk {
  v4i rs;
  uint32_t off[4], step;
  int row0, L;
  __device__ __forceinline__ Walk(const Rows& t, int head, int rows, int wave, int lane) {
    rs = rsrc_words(t.p + (size_t)head * t.hs, (uint32_t)(((size_t)(rows - 1) * t.ts + HD) * 2));
    row0 = 16 * wave + (lane >> 4);
    L = rows;
    step = (uint32_t)(AST * t.ts * 2);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int r = row0 + 4 * i;
      off[i] = (uint32_t)(r * t.ts * 2) + (((lane & 15) ^ aswz(r)) << 4);
    }
  }
  __device__ __forceinline__ void issue(uint32_t lds, int s, int wave) const {
#pragma unroll
    for (int i = 0; i < 4; i++)
      dma16(rs, lds + wave * 4096 + i * 1024, s * AST + row0 + 4 * i < L ? off[i] : kOobOffset, (uint32_t)s * step);
  }
};

// Operand of the owned rows straight from memory: lane r32 = row, 8
// elements from 16 kk + 8 h; rows past the end repeat the last one.
template <int NI>
__device__ __forceinline__ void load_own(const Rows& t, int head, int row0, int L, int r32, int h, v8bf (&f)[NI][8]) {
#pragma unroll
  for (int i = 0; i < NI; i++) {
    const uint16_t* p = t.p + (size_t)head * t.hs + (size_t)min(row0 + 32 * i + r32, L - 1) * t.ts + 8 * h;
#pragma unroll
    for (int kk = 0; kk < 8; kk++) f[i][kk] = __builtin_bit_cast(v8bf, *(const v4i*)(p + 16 * kk));
  }
}

// Fragments of a staged tile (base: its LDS address, row t0 of 32).
struct Frag {
  int r32, h, jj, byte8, sw_r, ch0;
  __device__ __forceinline__ Frag(int lane) {
    const int g16 = lane >> 4, t16 = lane & 15, qq = t16 & 3;
    r32 = lane & 31;
    h = lane >> 5;
    jj = t16 >> 2;
    ch0 = 2 * (g16 & 1) + (qq >> 1);
    byte8 = (qq & 1) * 8;
    sw_r = aswz(r32);
  }
  // row t0 + r32, elements 16 kk + 8 h ..
  __device__ __forceinline__ v8bf rows(const uint8_t* base, int t0, int kk) const {
    return __builtin_bit_cast(v8bf, *(const v4i*)(base + (t0 + r32) * AROW + (((2 * kk + h) ^ sw_r) << 4)));
  }
  // transposed: column 32 dt + r32, rows t0 + 16 ks + {4h .. + 3, 8 + 4h .. + 3}
  __device__ __forceinline__ v8bf cols(const uint8_t* base, int t0, int ks, int dt) const {
    const int r = t0 + 16 * ks + 4 * h + jj;
    const int at = (((4 * dt + ch0) ^ aswz(r)) << 4) + byte8;   // row + 8 has the neighbouring chunk
    const uint8_t* p = base + r * AROW;
    return make_v8bf(lds_read_tr16((const FT_LDS void*)(p + at)), lds_read_tr16((const FT_LDS void*)(p + 8 * AROW + (at ^ 16))));
  }
};

// Consecutive workgroups go to different XCDs; each XCD takes whole heads, so
// that the blocks that walk a head's rows share an L2.
__device__ __forceinline__ bool att_block(int nblk, int heads, int& head, int& blk) {
  const int T = nblk * heads, per = (T + 7) >> 3;
  const int t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (t >= T) return false;
  head = t / nblk;
  blk = t - head * nblk;
  return true;
}

__device__ __forceinline__ void publish_stage() {
  __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The wave's transposed 128 x 32 NI result to rows of out, 32 rows at a time
// through its own LDS (`scale` per owned row).
template <int NI>
__device__ __forceinline__ void store_own(v16f (&acc)[NI][4], const float (&scale)[NI], uint8_t* stg, uint16_t* out,
                                          int64_t ld, int row0, int L, int lane) {
  const int r32 = lane & 31, h = lane >> 5;
  constexpr int SROW = AROW + 16;
#pragma unroll
  for (int i = 0; i < NI; i++) {
#pragma unroll
    for (int dt = 0; dt < 4; dt++)
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const v2f a = {acc[i][dt][4 * q] * scale[i], acc[i][dt][4 * q + 1] * scale[i]};
        const v2f b = {acc[i][dt][4 * q + 2] * scale[i], acc[i][dt][4 * q + 3] * scale[i]};
        *(v2i*)(stg + r32 * SROW + (32 * dt + 8 * q + 4 * h) * 2) =
            v2i{(int)__builtin_bit_cast(uint32_t, __builtin_convertvector(a, v2bf)),
                (int)__builtin_bit_cast(uint32_t, __builtin_convertvector(b, v2bf))};
      }
    __builtin_amdgcn_s_waitcnt(0xc07f);   // the wave reads back only its own rows
#pragma unroll
    for (int it = 0; it < 8; it++) {
      const int rr = 4 * it + (lane >> 4), row = row0 + 32 * i + rr;
      const v4i v = *(const v4i*)(stg + rr * SROW + (lane & 15) * 16);
      if (row < L) *(v4i*)(out + (size_t)row * ld + (lane & 15) * 8) = v;
    }
  }
}

}  // namespace

// ------------------------------------------------------------------ forward
// Online softmax.  The running maximum follows every larger score: letting it
// lag until a score passes it by 2^8 saves rescaling but rounds the largest
// probability, which is otherwise exactly 1 (2-norm error 2.34e-3 against
// 2.28e-3).
template <int NI>
__global__ __launch_bounds__(256, NI == 1 ? 2 : 1) void k_attn_fwd(Rows q, Rows k, Rows v, uint16_t* __restrict__ o,
                                                                   int64_t ldo, float* __restrict__ lse, int L, int heads,
                                                                   int nblk) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * 2 * ATILE];
  int head, blk;
  if (!att_block(nblk, heads, head, blk)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = blk * ablk<NI>() + wave * 32 * NI;
  const Frag fr(lane);
  const uint32_t lds0 = lds_addr(lds);
  const Walk wk(k, head, L, wave, lane), wv(v, head, L, wave, lane);
  const int nst = (L + AST - 1) / AST;
  wk.issue(lds0, 0, wave);
  wv.issue(lds0 + ATILE, 0, wave);
  v8bf qf[NI][8];
  load_own<NI>(q, head, row0, L, fr.r32, fr.h, qf);
  const float c = 0.08838834764831845f * kLog2e;   // 1/sqrt(128) in powers of two
  v16f acc[NI][4];
  float m[NI], l[NI];
#pragma unroll
  for (int i = 0; i < NI; i++) {
    m[i] = -__builtin_inff();
    l[i] = 0.f;
#pragma unroll
    for (int dt = 0; dt < 4; dt++) acc[i][dt] = v16f{};
  }
#pragma unroll 1
  for (int s = 0; s < nst; s++) {
    publish_stage();
    if (s + 1 < nst) {
      wk.issue(lds0 + ((s + 1) & 1) * 2 * ATILE, s + 1, wave);
      wv.issue(lds0 + ((s + 1) & 1) * 2 * ATILE + ATILE, s + 1, wave);
    }
    const uint8_t* kb = lds + (s & 1) * 2 * ATILE;
    const uint8_t* vb = kb + ATILE;
    v16f sc[2][NI];   // [key tile][q tile]
#pragma unroll
    for (int t = 0; t < 2; t++) {
#pragma unroll
      for (int i = 0; i < NI; i++) sc[t][i] = v16f{};
#pragma unroll
      for (int kk = 0; kk < 8; kk++) {
        const v8bf a = fr.rows(kb, 32 * t, kk);
#pragma unroll
        for (int i = 0; i < NI; i++) sc[t][i] = mfma_bf16_32x32x16(a, qf[i][kk], sc[t][i]);
      }
    }
    if (s == nst - 1 && (L & (AST - 1))) {   // keys past the end
#pragma unroll
      for (int t = 0; t < 2; t++)
#pragma unroll
        for (int e = 0; e < 16; e++)
          if (s * AST + 32 * t + 8 * (e >> 2) + 4 * fr.h + (e & 3) >= L) {
#pragma unroll
            for (int i = 0; i < NI; i++) sc[t][i][e] = -__builtin_inff();
          }
    }
    float mx[NI];
    bool move = false;
#pragma unroll
    for (int i = 0; i < NI; i++) {
      float x = fmaxf(sc[0][i][0], sc[1][i][0]);
#pragma unroll
      for (int e = 1; e < 16; e++) x = fmaxf(x, fmaxf(sc[0][i][e], sc[1][i][e]));
      mx[i] = pair_max(x);
      move |= mx[i] > m[i];
    }
    if (__any(move)) {
#pragma unroll
      for (int i = 0; i < NI; i++) {
        const float mn = fmaxf(m[i], mx[i]);
        const float al = __builtin_amdgcn_exp2f((m[i] - mn) * c);
        m[i] = mn;
        l[i] *= al;
#pragma unroll
        for (int dt = 0; dt < 4; dt++)
#pragma unroll
          for (int e = 0; e < 16; e++) acc[i][dt][e] *= al;
      }
    }
#pragma unroll
    for (int t = 0; t < 2; t++) {
#pragma unroll
      for (int i = 0; i < NI; i++) {
        const float mc = m[i] * c;
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 16; e++) {
          const float p = __builtin_amdgcn_exp2f(fmaf(sc[t][i][e], c, -mc));
          sc[t][i][e] = p;
          sum += p;
        }
        l[i] += sum;
      }
#pragma unroll
      for (int ks = 0; ks < 2; ks++) {
        v8bf p[NI];
#pragma unroll
        for (int i = 0; i < NI; i++) p[i] = pack_b(sc[t][i], 8 * ks);
#pragma unroll
        for (int dt = 0; dt < 4; dt++) {
          const v8bf a = fr.cols(vb, 32 * t, ks, dt);
#pragma unroll
          for (int i = 0; i < NI; i++) acc[i][dt] = mfma_bf16_32x32x16(a, p[i], acc[i][dt]);
        }
      }
    }
  }
  float inv[NI];
#pragma unroll
  for (int i = 0; i < NI; i++) {
    const float sum = pair_sum(l[i]);
    inv[i] = 1.0f / sum;
    const int row = row0 + 32 * i + fr.r32;
    // in powers of two, as the backward uses it
    if (fr.h == 0 && row < L) lse[(size_t)head * L + row] = m[i] * c + __log2f(sum);
  }
  __syncthreads();   // every wave is done with the ring
  store_own<NI>(acc, inv, lds + wave * 32 * (AROW + 16), o + (size_t)head * HD, ldo, row0, L, lane);
}

// ------------------------------------------------------- backward: delta
// delta[head][row] = sum over d of dout o.
__global__ __launch_bounds__(256) void k_attn_delta(Rows dout, Rows o, float* __restrict__ delta, int L, int heads) {
  const int i = blockIdx.x * 16 + (threadIdx.x >> 4), c = threadIdx.x & 15;   // 16 lanes per (row, head)
  const bool live = i < L * heads;
  const int row = live ? i / heads : 0, head = live ? i - row * heads : 0;
  const v4i a = *(const v4i*)(dout.p + (size_t)row * dout.ts + (size_t)head * dout.hs + 8 * c);
  const v4i b = *(const v4i*)(o.p + (size_t)row * o.ts + (size_t)head * o.hs + 8 * c);
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < 4; e++)
    s += bf16_to_f32((uint32_t)a[e] & 0xFFFFu) * bf16_to_f32((uint32_t)b[e] & 0xFFFFu) +
         bf16_to_f32((uint32_t)a[e] >> 16) * bf16_to_f32((uint32_t)b[e] >> 16);
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) s += __shfl_xor(s, off, 64);
  if (live && c == 0) delta[(size_t)head * L + row] = s;
}

// ---------------------------------------------------------- backward: dq
//   p = 2^(s c - lse),  ds = p (dout v^T - delta),  dq = ds k / sqrt(128)
template <int NI>
__global__ __launch_bounds__(256, NI == 1 ? 2 : 1) void k_attn_dq(Rows q, Rows k, Rows v, Rows dout, const float* __restrict__ lse,
                                                    const float* __restrict__ delta, uint16_t* __restrict__ dq, int L,
                                                    int heads, int nblk) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * 2 * ATILE];
  int head, blk;
  if (!att_block(nblk, heads, head, blk)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = blk * ablk<NI>() + wave * 32 * NI;
  const Frag fr(lane);
  const uint32_t lds0 = lds_addr(lds);
  const Walk wk(k, head, L, wave, lane), wv(v, head, L, wave, lane);
  const int nst = (L + AST - 1) / AST;
  wk.issue(lds0, 0, wave);
  wv.issue(lds0 + ATILE, 0, wave);
  v8bf qf[NI][8], gf[NI][8];
  load_own<NI>(q, head, row0, L, fr.r32, fr.h, qf);
  load_own<NI>(dout, head, row0, L, fr.r32, fr.h, gf);
  const float scale = 0.08838834764831845f, c = scale * kLog2e;
  float ls[NI], de[NI];
  v16f acc[NI][4];
#pragma unroll
  for (int i = 0; i < NI; i++) {
    const int row = min(row0 + 32 * i + fr.r32, L - 1);
    ls[i] = lse[(size_t)head * L + row];
    de[i] = delta[(size_t)head * L + row];
#pragma unroll
    for (int dt = 0; dt < 4; dt++) acc[i][dt] = v16f{};
  }
#pragma unroll 1
  for (int s = 0; s < nst; s++) {
    publish_stage();
    if (s + 1 < nst) {
      wk.issue(lds0 + ((s + 1) & 1) * 2 * ATILE, s + 1, wave);
      wv.issue(lds0 + ((s + 1) & 1) * 2 * ATILE + ATILE, s + 1, wave);
    }
    const uint8_t* kb = lds + (s & 1) * 2 * ATILE;
    const uint8_t* vb = kb + ATILE;
#pragma unroll
    for (int t = 0; t < 2; t++) {
      v16f sc[NI], dp[NI];
#pragma unroll
      for (int i = 0; i < NI; i++) sc[i] = dp[i] = v16f{};
#pragma unroll
      for (int kk = 0; kk < 8; kk++) {
        const v8bf a = fr.rows(kb, 32 * t, kk), b = fr.rows(vb, 32 * t, kk);
#pragma unroll
        for (int i = 0; i < NI; i++) {
          sc[i] = mfma_bf16_32x32x16(a, qf[i][kk], sc[i]);
          dp[i] = mfma_bf16_32x32x16(b, gf[i][kk], dp[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < NI; i++)
#pragma unroll
        for (int e = 0; e < 16; e++)
          sc[i][e] = __builtin_amdgcn_exp2f(fmaf(sc[i][e], c, -ls[i])) * (dp[i][e] - de[i]);
      if (s == nst - 1 && (L & (AST - 1))) {
        // keys past the end: their score 0 may lie far above the row's lse, and
        // an overflowed p would not vanish against the zero row of k
#pragma unroll
        for (int e = 0; e < 16; e++)
          if (s * AST + 32 * t + 8 * (e >> 2) + 4 * fr.h + (e & 3) >= L) {
#pragma unroll
            for (int i = 0; i < NI; i++) sc[i][e] = 0.f;
          }
      }
#pragma unroll
      for (int ks = 0; ks < 2; ks++) {
        v8bf p[NI];
#pragma unroll
        for (int i = 0; i < NI; i++) p[i] = pack_b(sc[i], 8 * ks);
#pragma unroll
        for (int dt = 0; dt < 4; dt++) {
          const v8bf a = fr.cols(kb, 32 * t, ks, dt);
#pragma unroll
          for (int i = 0; i < NI; i++) acc[i][dt] = mfma_bf16_32x32x16(a, p[i], acc[i][dt]);
        }
      }
    }
  }
  float sc2[NI];
#pragma unroll
  for (int i = 0; i < NI; i++) sc2[i] = scale;
  __syncthreads();
  store_own<NI>(acc, sc2, lds + wave * 32 * (AROW + 16), dq + (size_t)head * HD, (int64_t)heads * HD, row0, L, lane);
}

// ----------------------------------------------------- backward: dk and dv
//   dv = p^T dout,  dk = ds^T q / sqrt(128): rows of q walked, keys owned.
template <int NI>
__global__ __launch_bounds__(256, 1) void k_attn_dkdv(Rows q, Rows k, Rows v, Rows dout, const float* __restrict__ lse,
                                                      const float* __restrict__ delta, uint16_t* __restrict__ dk,
                                                      uint16_t* __restrict__ dv, int L, int heads, int nblk) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * 2 * ATILE + 2 * 2 * AST * 4];
  int head, blk;
  if (!att_block(nblk, heads, head, blk)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = blk * ablk<NI>() + wave * 32 * NI;
  const Frag fr(lane);
  const uint32_t lds0 = lds_addr(lds);
  const Walk wq(q, head, L, wave, lane), wg(dout, head, L, wave, lane);
  // the stage's lse and delta: waves 0 and 1 bring 64 floats each
  const v4i rst = rsrc_words((wave == 0 ? lse : delta) + (size_t)head * L, (uint32_t)L * 4);
  auto issue = [&](int s) {
    const uint32_t base = lds0 + (s & 1) * 2 * ATILE;
    wq.issue(base, s, wave);
    wg.issue(base + ATILE, s, wave);
    if (wave < 2) dma4(rst, lds0 + 4 * ATILE + ((s & 1) * 2 + wave) * AST * 4, (uint32_t)(s * AST + lane) * 4, 0);
  };
  const int nst = (L + AST - 1) / AST;
  issue(0);
  v8bf kf[NI][8], vf[NI][8];
  load_own<NI>(k, head, row0, L, fr.r32, fr.h, kf);
  load_own<NI>(v, head, row0, L, fr.r32, fr.h, vf);
  const float scale = 0.08838834764831845f, c = scale * kLog2e;
  v16f ak[NI][4], av[NI][4];
#pragma unroll
  for (int i = 0; i < NI; i++)
#pragma unroll
    for (int dt = 0; dt < 4; dt++) ak[i][dt] = av[i][dt] = v16f{};
#pragma unroll 1
  for (int s = 0; s < nst; s++) {
    publish_stage();
    if (s + 1 < nst) issue(s + 1);
    const uint8_t* qb = lds + (s & 1) * 2 * ATILE;
    const uint8_t* gb = qb + ATILE;
    const float* lsb = (const float*)(lds + 4 * ATILE + (s & 1) * 2 * AST * 4);
    const float* deb = lsb + AST;
    // rows of q past the end: q, dout, lse and delta are zeros, so p is 1 but
    // meets a zero row of dout, and ds is 0
#pragma unroll
    for (int t = 0; t < 2; t++) {
      // One key tile at a time: both tiles' scores beside 256 accumulators and
      // 128 registers of k and v would spill.  (The rows are read again for
      // the second tile; the barrier keeps the compiler from holding them.)
      v8bf pb[NI][2], db[NI][2];   // [key tile][k-step]
#pragma unroll
      for (int i = 0; i < NI; i++) {
        v16f sc = v16f{}, dp = v16f{};
#pragma unroll
        for (int kk = 0; kk < 8; kk++) {
          sc = mfma_bf16_32x32x16(fr.rows(qb, 32 * t, kk), kf[i][kk], sc);
          dp = mfma_bf16_32x32x16(fr.rows(gb, 32 * t, kk), vf[i][kk], dp);
        }
#pragma unroll
        for (int g = 0; g < 4; g++) {
          const v4f ls = *(const v4f*)(lsb + 32 * t + 8 * g + 4 * fr.h), de = *(const v4f*)(deb + 32 * t + 8 * g + 4 * fr.h);
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const float p = __builtin_amdgcn_exp2f(fmaf(sc[4 * g + e], c, -ls[e]));
            sc[4 * g + e] = p;
            dp[4 * g + e] = p * (dp[4 * g + e] - de[e]);
          }
        }
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
          pb[i][ks] = pack_b(sc, 8 * ks);
          db[i][ks] = pack_b(dp, 8 * ks);
        }
        asm volatile("" ::: "memory");
      }
#pragma unroll
      for (int ks = 0; ks < 2; ks++)
#pragma unroll
        for (int dt = 0; dt < 4; dt++) {
          const v8bf a = fr.cols(gb, 32 * t, ks, dt), b = fr.cols(qb, 32 * t, ks, dt);
#pragma unroll
          for (int i = 0; i < NI; i++) av[i][dt] = mfma_bf16_32x32x16(a, pb[i][ks], av[i][dt]);
#pragma unroll
          for (int i = 0; i < NI; i++) ak[i][dt] = mfma_bf16_32x32x16(b, db[i][ks], ak[i][dt]);
        }
    }
  }
  float one[NI], sc2[NI];
#pragma unroll
  for (int i = 0; i < NI; i++) {
    one[i] = 1.f;
    sc2[i] = scale;
  }
  __syncthreads();
  uint8_t* stg = lds + wave * 32 * (AROW + 16);
  store_own<NI>(av, one, stg, dv + (size_t)head * HD, (int64_t)heads * HD, row0, L, lane);
  store_own<NI>(ak, sc2, stg, dk + (size_t)head * HD, (int64_t)heads * HD, row0, L, lane);
}

}  // namespace ft

// ------------------------------------------------------------- entry points
// Called by the package's DiT module only, which checks devices and types.
// q, k, v, dout: bf16 [L, heads, 128] with unit stride within a head, strides
// of tokens and heads multiples of 8; o: the same with token stride ot and
// heads side by side; dq, dk, dv: contiguous.  lse (in powers of two) and
// delta: fp32 [heads, L].
namespace {

bool att_rows(const void* p, int64_t ts, int64_t hs, int64_t L, int64_t heads) {
  // 32-bit buffer offsets within a head
  return p && ((uintptr_t)p & 15u) == 0 && ts >= 0 && hs >= 0 && ((ts | hs) & 7) == 0 &&
         (L - 1 + 64) * ts * 2 + 256 < (int64_t)1 << 31;
}

bool al16(const void* p) { return ((uintptr_t)p & 15u) == 0; }
ft_status launched() { return hipGetLastError() == hipSuccess ? FT_OK : FT_ERR_HIP; }
ft::Rows rows_of(const void* p, int64_t ts, int64_t hs) { return ft::Rows{(const uint16_t*)p, ts, hs}; }

// Key tiles per wave of the dk/dv kernel, by rounds of workgroups on the 256
// CUs: one of two tiles (2 x 33 units) takes about 1.65 times one of one tile
// (2 x 20), and a CU holds one workgroup of either.  4608 x 24 heads: 1100 us
// with two tiles, 1178 with one (two rounds against four); 4500 x 16: 972
// against 873 (two against three); 1000 x 8: 111 against 78.
int kv_tiles_per_wave(int64_t L, int64_t heads) {
  const int64_t r1 = ((L + 127) / 128 * heads + 255) / 256, r2 = ((L + 255) / 256 * heads + 255) / 256;
  return 20 * r1 <= 33 * r2 ? 1 : 2;
}
unsigned att_grid(int64_t L, int64_t heads, int ni, int& nblk) {
  nblk = (int)((L + 128 * ni - 1) / (128 * ni));
  return (unsigned)((nblk * heads + 7) / 8 * 8);
}

}  // namespace

extern "C" {

ft_status ftdit_attn_fwd(int64_t L, int64_t heads, const void* q, int64_t qt, int64_t qh, const void* k, int64_t kt,
                         int64_t kh, const void* v, int64_t vt, int64_t vh, void* o, int64_t ot, float* lse,
                         hipStream_t st) {
  if (L <= 0 || heads <= 0 || L * heads >= (int64_t)1 << 27) return FT_ERR_SHAPE;
  if (!att_rows(q, qt, qh, L, heads) || !att_rows(k, kt, kh, L, heads) || !att_rows(v, vt, vh, L, heads) || !o || !lse ||
      !al16(o) || ot < heads * ft::HD || (ot & 7))
    return FT_ERR_ALIGN;
  const ft::Rows Q = rows_of(q, qt, qh), K = rows_of(k, kt, kh), V = rows_of(v, vt, vh);
  int nblk;
  const unsigned grid = att_grid(L, heads, 1, nblk);
  ft::k_attn_fwd<1><<<grid, 256, 0, st>>>(Q, K, V, (uint16_t*)o, ot, lse, (int)L, (int)heads, nblk);
  return launched();
}

ft_status ftdit_attn_bwd(int64_t L, int64_t heads, const void* q, int64_t qt, int64_t qh, const void* k, int64_t kt,
                         int64_t kh, const void* v, int64_t vt, int64_t vh, const void* dout, int64_t gt, int64_t gh,
                         const void* o, int64_t ot, const float* lse, float* delta, void* dq, void* dk, void* dv, hipStream_t st) {
  if (L <= 0 || heads <= 0 || L * heads >= (int64_t)1 << 27) return FT_ERR_SHAPE;
  if (!att_rows(q, qt, qh, L, heads) || !att_rows(k, kt, kh, L, heads) || !att_rows(v, vt, vh, L, heads) ||
      !att_rows(dout, gt, gh, L, heads) || !o || !lse || !delta || !dq || !dk || !dv || !al16(o) || !al16(dq) ||
      !al16(dk) || !al16(dv) || ot < heads * ft::HD || (ot & 7))
    return FT_ERR_ALIGN;
  const ft::Rows Q = rows_of(q, qt, qh), K = rows_of(k, kt, kh), V = rows_of(v, vt, vh), G = rows_of(dout, gt, gh);
  ft::k_attn_delta<<<(unsigned)((L * heads + 15) / 16), 256, 0, st>>>(G, rows_of(o, ot, ft::HD), delta, (int)L,
                                                                    (int)heads);
  int nblk;
  const int ni = kv_tiles_per_wave(L, heads);
  unsigned grid = att_grid(L, heads, ni, nblk);
  if (ni == 2) ft::k_attn_dkdv<2><<<grid, 256, 0, st>>>(Q, K, V, G, lse, delta, (uint16_t*)dk, (uint16_t*)dv, (int)L, (int)heads, nblk);
  else ft::k_attn_dkdv<1><<<grid, 256, 0, st>>>(Q, K, V, G, lse, delta, (uint16_t*)dk, (uint16_t*)dv, (int)L, (int)heads, nblk);
  grid = att_grid(L, heads, 1, nblk);
  ft::k_attn_dq<1><<<grid, 256, 0, st>>>(Q, K, V, G, lse, delta, (uint16_t*)dq, (int)L, (int)heads, nblk);
  return launched();
}

}  // extern "C"
