// Block-scaled FP4 GEMM on small output tiles (gfx950): the same products as
// gemm_fp4.hip (forward, and the backward that reads the weight transposed),
// for outputs that make too few 256x256 tiles to fill the chip, and for
// widths that are not multiples of 128.
//
// Workgroup: 4 waves in a 2x2 grid over a TM x 128 tile (TM = 64 or 128), so
// a wave holds TM/2 x 64 outputs.  Stages of 256 reduction elements (whole
// 128-byte rows of codes) move through an LDS ring of `ns` slots, filled by
// buffer loads that write LDS directly; the low-rank term is extra stages of
// the same ring.  Accumulation order is
// that of the 256x256 kernel: bias, the reduction in 64-element MFMA steps,
// then hi and lo terms of each 16 low-rank columns.
//
// What bounds it: at 512 x 12288 -> 3072 (192 tiles of 64x128, one per CU) a
// stage takes 0.46 us against 0.28 us that its LDS traffic (72 KB at 128
// bytes a clock) needs; the loop is one wave per SIMD, whose waits at the
// stage's barrier nothing covers.  30 us, against 65 us on 24 tiles of
// 256x256; 512 x 3072 -> 3072 12 us against 22.5; 1111 x 2080 -> 3168
// (widths that are no multiple of 128) 14 us forward and 17 us backward,
// against 74 and 121 us in the register-staged kernel.  The first form, whose
// waits, stage kinds and scale alignments were branches of one loop, took
// 0.9 us a stage.
//
// All E8M0 scales of the tile stay in LDS for the whole reduction.  Those of
// the tile's rows are one contiguous run of bytes in memory (TM rows of
// KR/32), so they arrive in 16-byte loads for any width that is a multiple of
// 32, where a load per row and stage would touch a line for every 8 bytes.
#include "ft_device.h"
#include "ft_kernels.h"

namespace ft {

namespace {

constexpr int TN = 128;                   // output columns per workgroup
constexpr int TK = 256;                   // reduction elements per stage
constexpr int TROW = TK / 2;              // bytes per row of a stage
constexpr int TLR = 32;                   // low-rank columns per stage
constexpr int kCuLds = 160 * 1024;

template <int TM>
struct TileGeom {
  static constexpr int OFF_B = TM * TROW;            // W tile, U or D chunk within a slot
  static constexpr int SLOT = (TM + TN) * TROW;
  static constexpr int LOADS = TM / 32 + TN / 32;    // per wave and stage
};

template <int V> struct IC { static constexpr int value = V; };   // a compile-time k-step

__host__ __device__ constexpr int round_up(int v, int m) { return (v + m - 1) / m * m; }

// Bytes of LDS after the ring: A scales, W scales, bias.  Rows of A scales
// that are whole 16-byte chunks get one chunk of padding: without it the 32
// rows that a fragment's lanes read would start in the same few banks (all in
// one at KR = 12288).
__host__ __device__ inline int slab_a_row(int nkb) { return nkb + (nkb % 16 == 0 ? 16 : 0); }
__host__ __device__ inline int slab_a_bytes(int tm, int nkb) { return round_up(tm * slab_a_row(nkb), 1024); }
// Forward [4 column blocks][8 nst bytes]; backward [8 nst reduction blocks][4 bytes].
__host__ __device__ inline int slab_w_bytes(int nst) { return round_up(4 * nst * 8, 256); }
__host__ __device__ inline int slab_bytes(int tm, int nkb, int nst) {
  return slab_a_bytes(tm, nkb) + slab_w_bytes(nst) + TN * 2;
}

}  // namespace

template <bool BWD, int TM, int NS>
__global__ __launch_bounds__(256, 2) void k_gemm_fp4_tile(const uint8_t* __restrict__ A, const uint8_t* __restrict__ As,
                                                          const uint8_t* __restrict__ Wq, const uint8_t* __restrict__ Ws,
                                                          int M, int N, int K, const float* __restrict__ P, int R,
                                                          const uint16_t* __restrict__ LR,
                                                          const uint16_t* __restrict__ bias, void* __restrict__ out,
                                                          int out_f32, int tiles_m, int tiles_n,
                                                          const uint16_t* __restrict__ z) {
  using G = TileGeom<TM>;
  extern __shared__ __attribute__((aligned(16))) uint8_t tlds[];
  constexpr int MT = TM / 64, NT = 2;                // 32x32 MFMA tiles per wave

  // Consecutive workgroup ids go to different XCDs: each XCD takes a
  // contiguous range of tiles, eight tile-rows at a time, so that the
  // workgroups sharing W columns share an L2.
  const int T = tiles_m * tiles_n, per = (T + 7) >> 3;
  const int t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (t >= T || (int)(blockIdx.x >> 3) >= per) return;   // the whole workgroup
  int mt, nt;
  {
    constexpr int GM = 8;
    const int g = t / (GM * tiles_n), first = g * GM;
    const int gm = min(GM, tiles_m - first);
    const int w = t - g * GM * tiles_n;
    mt = first + w % gm;
    nt = w / gm;
  }
  const int m0 = mt * TM, n0 = nt * TN;

  const int NO = BWD ? K : N, KR = BWD ? N : K;
  const int lda = KR >> 1, nkb = KR >> 5, ldw = K >> 1, nwkb = K >> 5;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, h = lane >> 5, g16 = lane >> 4, t16 = lane & 15;
  const int wm = wave >> 1, wn = wave & 1;

  const v4i ra = rsrc_words(A, (uint32_t)M * lda);
  const v4i rw = rsrc_words(Wq, (uint32_t)N * ldw);
  const v4i ras = rsrc_words(As, (uint32_t)M * nkb);
  const v4i rws = rsrc_words(Ws, (uint32_t)(N >> 5) * nwkb);
  const v4i rp = rsrc_words(P, (uint32_t)M * R * 4);
  const v4i rl = rsrc_words(LR, (uint32_t)NO * R * 2);
  const v4i rb = rsrc_words(bias, !BWD && bias ? (uint32_t)N * 2 : 0u);

  const int nst = (KR + TK - 1) / TK, nlr = (R + TLR - 1) / TLR, total = nst + nlr;
  const uint32_t lds0 = lds_addr(tlds);
  const int off_sa = NS * G::SLOT, off_sb = off_sa + slab_a_bytes(TM, nkb);
  const int sas = slab_a_row(nkb), swr = nst * 8, off_bias = off_sb + slab_w_bytes(nst);

  // ---------------- per-lane load geometry (as in the 256x256 kernel)
  const int r8 = lane >> 3, c8 = (lane & 7) ^ r8;
  constexpr int AL = TM / 32, WL = TN / 32;          // loads per wave and stage
  // Byte offsets of each load's lane within a whole stage (rows outside the
  // matrix hold kOobOffset, which reads zeros); the stage adds a uniform
  // offset that stays inside the row of every valid lane.
  uint32_t a_off[AL], w_off[WL];
#pragma unroll
  for (int v = 0; v < AL; v++) {
    const int r = m0 + (wave * AL + v) * 8 + r8;
    a_off[v] = r < M ? (uint32_t)r * lda + (c8 ^ (v & 1)) * 16 : kOobOffset;
  }
#pragma unroll
  for (int v = 0; v < WL; v++) {
    if constexpr (!BWD) {
      const int r = n0 + (wave * WL + v) * 8 + r8;
      w_off[v] = r < N ? (uint32_t)r * ldw + (c8 ^ (v & 1)) * 16 : kOobOffset;
    } else {   // reduction row of the stage, 64 bytes (the tile's 128 columns) of it
      const int r = 16 * (wave * WL + v) + (lane >> 2);
      const int byte = (n0 >> 1) + (((lane & 3) ^ swz64(r)) << 4);
      w_off[v] = byte < ldw ? (uint32_t)r * ldw + byte : kOobOffset;
    }
  }

  // Loads of a whole FP4 stage u into slot `slot`.
  auto issue_full = [&](int u, int slot) {
    const uint32_t base = lds0 + (uint32_t)slot * G::SLOT;
#pragma unroll
    for (int v = 0; v < AL; v++) dma16(ra, base + (wave * AL + v) * 1024, a_off[v], (uint32_t)u * TROW);
#pragma unroll
    for (int v = 0; v < WL; v++)
      dma16(rw, base + G::OFF_B + (wave * WL + v) * 1024, w_off[v], BWD ? (uint32_t)u * TK * ldw : (uint32_t)u * TROW);
  };
  // Loads of any stage: the reduction's last, partial one, a low-rank one, or
  // none (zeros), always G::LOADS of them per wave.
  auto issue_any = [&](int u, int slot) {
    const uint32_t base = lds0 + (uint32_t)slot * G::SLOT;
    if (u < nst) {
      const int nch = (lda >> 4) - u * (TROW / 16);   // 16-byte chunks left in a row of codes
#pragma unroll
      for (int v = 0; v < AL; v++)
        dma16(ra, base + (wave * AL + v) * 1024, (c8 ^ (v & 1)) < nch ? a_off[v] : kOobOffset, (uint32_t)u * TROW);
#pragma unroll
      for (int v = 0; v < WL; v++) {
        const uint32_t dst = base + G::OFF_B + (wave * WL + v) * 1024;
        if constexpr (!BWD)
          dma16(rw, dst, (c8 ^ (v & 1)) < nch ? w_off[v] : kOobOffset, (uint32_t)u * TROW);
        else
          dma16(rw, dst, u * TK + 16 * (wave * WL + v) + (lane >> 2) < N ? w_off[v] : kOobOffset, (uint32_t)u * TK * ldw);
      }
    } else {
      const int q = u - nst, left = u < total ? R - q * TLR : 0;   // low-rank columns from this chunk on
#pragma unroll
      for (int v = 0; v < AL; v++) {
        const int r = m0 + (wave * AL + v) * 8 + r8, c = c8 ^ (v & 1);
        dma16(rp, base + (wave * AL + v) * 1024, 4 * c < left && r < M ? (uint32_t)r * R * 4 + c * 16 : kOobOffset,
              (uint32_t)q * 128);
      }
#pragma unroll
      for (int v = 0; v < WL; v++) {
        // two loads carry the U or D chunk, two read zeros into the rest of the slot
        const int ins = 2 * wave + v;
        uint32_t off = kOobOffset, so = 0;
        if (v < 2) {
          if constexpr (!BWD) {   // [32 j][128 n]: rows 4 ins + lane / 16
            const int j = 4 * ins + (lane >> 4), c = (lane & 15) ^ (2 * (j & 3));
            if (j < left && n0 + c * 8 < N) off = (uint32_t)j * N * 2 + (uint32_t)(n0 + c * 8) * 2;
            so = (uint32_t)q * TLR * N * 2;
          } else {                // [128 k][32 j]: rows 16 ins + lane / 4
            const int k = 16 * ins + (lane >> 2), c = (lane & 3) ^ swz64(k);
            if (n0 + k < K && 8 * c < left) off = (uint32_t)(n0 + k) * R * 2 + c * 16;
            so = (uint32_t)q * 64;
          }
        }
        dma16(rl, base + G::OFF_B + (v < 2 ? ins : 8 + 2 * wave + (v - 2)) * 1024, off, so);
      }
    }
  };

  // ---------------- scales and bias into LDS, then the first NS stages
  const uint32_t end = (uint32_t)M * nkb, beg = (uint32_t)m0 * nkb;   // bytes of As
  {
    // A scales: bytes [m0 nkb, (m0 + TM) nkb) of As in 16-byte chunks, those
    // wholly inside the array.  Chunk p of LDS is chunk p % cpr of row p / cpr
    // (cpr counts the padding chunk; unpadded rows are one run).
    const bool pad = sas != nkb;
    const int nins = slab_a_bytes(TM, nkb) >> 10;
    const int cpr = pad ? sas >> 4 : 1 << 24;
    const int dr = 256 / cpr, dc = 256 - dr * cpr;
    int row = (wave * 64 + lane) / cpr, col = wave * 64 + lane - row * cpr;
    for (int i = wave; i < nins; i += 4) {
      const uint32_t off = beg + (uint32_t)(pad ? row * nkb : 0) + (uint32_t)col * 16;
      const bool ok = off + 16 <= end && !(pad && (col == cpr - 1 || row >= TM));
      dma16(ras, lds0 + off_sa + i * 1024, ok ? off : kOobOffset, 0);
      row += dr;
      col += dc;
      if (col >= cpr) { col -= cpr; row++; }
    }
    if ((nwkb & 3) == 0) {
      for (int i = wave; i < slab_w_bytes(nst) >> 8; i += 4) {
        const int p = i * 64 + lane;      // dword of the slab
        uint32_t off = kOobOffset;
        if constexpr (!BWD) {
          const int j = p / (2 * nst), kb = 4 * (p - j * 2 * nst), nb = (n0 >> 5) + j;
          if (j < 4 && nb < (N >> 5) && kb < nwkb) off = (uint32_t)nb * nwkb + kb;
        } else {
          if (p < nkb) off = (uint32_t)p * nwkb + (n0 >> 5);
        }
        dma4(rws, lds0 + off_sb + i * 256, off, 0);
      }
    } else {                  // rows of scale bytes that are not 4-byte aligned
      for (int i = tid; i < nst * 8; i += 256) {
        uint32_t b[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
          const int nb = (n0 >> 5) + j;
          const bool ok = nb < (NO >> 5) && i < nkb;
          b[j] = ok ? Ws[BWD ? (size_t)i * nwkb + nb : (size_t)nb * nwkb + i] : 0u;
        }
        if constexpr (!BWD) {
#pragma unroll
          for (int j = 0; j < 4; j++) tlds[off_sb + j * swr + i] = (uint8_t)b[j];
        } else {
          *(uint32_t*)(tlds + off_sb + 4 * i) = b[0] | (b[1] << 8) | (b[2] << 16) | (b[3] << 24);
        }
      }
    }
    if (wave == 0) dma4(rb, lds0 + off_bias, (uint32_t)(n0 + 2 * lane) * 2, 0);
    // The array's last, partial 16-byte chunk (only the last tile-row of an
    // array whose size is not a multiple of 16): byte by byte, after the
    // loads above have written their zeros.
    const uint32_t full = end & ~15u;
    if (full != end && full < beg + (uint32_t)TM * nkb && end > beg) {
      wait_vm<0>();
      __syncthreads();
      if (tid < (int)(end - full) && full + tid >= beg) tlds[off_sa + full - beg + tid] = As[full + tid];
    }
  }
#pragma unroll 1
  for (int u = 0; u < NS; u++) issue_any(u, u);

  // ---------------- fragment reads
  const int sw_r = swz128(r32), sw_t = swz64(t16), sw_d = swz64(r32);
  const int jj = t16 >> 2, qq = t16 & 3;
  const uint32_t psel = h ? 0x07050301u : 0x06040200u;   // bytes h, h+2, h+4, h+6 of a dword pair
  v16f acc[MT][NT];

  // Scale operands of stage s: byte kk = k-step kk (64 elements), block 2 kk + h.
  // Row bytes start anywhere within a dword when KR / 32 is no multiple of 4:
  // three dwords hold the eight.  In the last stage, bytes past the row's end
  // (another row's) become neutral scales.
  struct Scales { uint32_t a[MT], b[NT]; };
  uint32_t sa_at[MT];
#pragma unroll
  for (int i = 0; i < MT; i++) sa_at[i] = off_sa + (wm * (TM / 2) + i * 32 + r32) * sas;
  uint32_t keep_last = 0;
#pragma unroll
  for (int kk = 0; kk < 4; kk++)
    if (8 * (nst - 1) + 2 * kk + h < nkb) keep_last |= 0xFFu << (8 * kk);
  auto read_scales = [&](int s, Scales& f) {
    const uint32_t keep = s == nst - 1 ? keep_last : 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < MT; i++) {
      const uint32_t at = sa_at[i] + 8 * s;
      const uint32_t* p = (const uint32_t*)(tlds + (at & ~3u));
      const uint32_t d0 = __builtin_amdgcn_alignbyte(p[1], p[0], at), d1 = __builtin_amdgcn_alignbyte(p[2], p[1], at);
      f.a[i] = (__builtin_amdgcn_perm(d1, d0, psel) & keep) | (0x7F7F7F7Fu & ~keep);
    }
    if constexpr (!BWD) {
#pragma unroll
      for (int j = 0; j < NT; j++) {
        const v2i d = *(const v2i*)(tlds + off_sb + (wn * NT + j) * swr + 8 * s);
        f.b[j] = __builtin_amdgcn_perm((uint32_t)d[1], (uint32_t)d[0], psel);
      }
    } else {
      uint32_t w[4];
#pragma unroll
      for (int kk = 0; kk < 4; kk++) w[kk] = *(const uint32_t*)(tlds + off_sb + (8 * s + 2 * kk + h) * 4) >> (16 * wn);
#pragma unroll
      for (int j = 0; j < NT; j++)
        f.b[j] = __builtin_amdgcn_perm(w[1], w[0], 0x0c0c0400u | (j << 8) | j) |
                 __builtin_amdgcn_perm(w[3], w[2], 0x04000c0cu | (j << 24) | (j << 16));
    }
  };
  // Fragments of k-steps k0 and k0 + 1.
  struct Frags { v4i a[2][MT], b[2][NT]; };
  auto read_frags = [&](int slot, int k0, Frags& f) {
    const uint8_t* base = tlds + slot * G::SLOT;
#pragma unroll
    for (int u = 0; u < 2; u++) {
      const int kk = k0 + u;
#pragma unroll
      for (int i = 0; i < MT; i++)
        f.a[u][i] = *(const v4i*)(base + (wm * (TM / 2) + i * 32 + r32) * TROW + (((2 * kk + h) ^ sw_r) << 4));
#pragma unroll
      for (int j = 0; j < NT; j++) {
        if constexpr (!BWD) {
          f.b[u][j] = *(const v4i*)(base + G::OFF_B + (wn * 64 + j * 32 + r32) * TROW + (((2 * kk + h) ^ sw_r) << 4));
        } else {
          const uint8_t* p = base + G::OFF_B + (kk * 64 + 32 * h + t16) * 64 + (((wn * NT + j) ^ sw_t) << 4) + 8 * (g16 & 1);
          const v2i lo = lds_read_tr4((const FT_LDS void*)p), hi = lds_read_tr4((const FT_LDS void*)(p + 16 * 64));
          f.b[u][j] = v4i{lo[0], lo[1], hi[0], hi[1]};
        }
      }
    }
  };
  auto mfma_step = [&](auto kc, const Frags& f, const Scales& sc) {
    constexpr int KK = decltype(kc)::value;
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
      for (int j = 0; j < NT; j++)
        acc[i][j] = mfma_fp4_32x32x64<KK>(f.b[KK & 1][j], f.a[KK & 1][i], acc[i][j], (int)sc.b[j], (int)sc.a[i]);
  };

  // One 16-column half c of a low-rank stage: P split into bf16 hi + lo.
  auto lr_half = [&](int slot, int c) {
    const uint8_t* base = tlds + slot * G::SLOT;
    v8bf hi[MT], lo[MT], b[NT];
#pragma unroll
    for (int i = 0; i < MT; i++) {
      v4i hp, lp;
#pragma unroll
      for (int e = 0; e < 2; e++) {
        const v4f x = *(const v4f*)(base + (wm * (TM / 2) + i * 32 + r32) * 128 + (((4 * c + 2 * h + e) ^ sw_r) << 4));
        uint32_t a0, l0, a1, l1;
        split_bf16x2(x[0], x[1], a0, l0);
        split_bf16x2(x[2], x[3], a1, l1);
        hp[2 * e] = (int)a0; hp[2 * e + 1] = (int)a1;
        lp[2 * e] = (int)l0; lp[2 * e + 1] = (int)l1;
      }
      hi[i] = __builtin_bit_cast(v8bf, hp);
      lo[i] = __builtin_bit_cast(v8bf, lp);
    }
#pragma unroll
    for (int j = 0; j < NT; j++) {
      if constexpr (!BWD) {
        const int n = wn * 64 + j * 32 + 16 * (g16 & 1) + 4 * qq, row = 16 * c + 8 * h + jj;
        const int ch = (n >> 3) ^ (2 * (row & 3));   // row + 4 has the same swizzle
        const uint8_t* p = base + G::OFF_B + row * 256 + (ch << 4) + ((n >> 2) & 1) * 8;
        b[j] = make_v8bf(lds_read_tr16((const FT_LDS void*)p), lds_read_tr16((const FT_LDS void*)(p + 4 * 256)));
      } else {
        b[j] = __builtin_bit_cast(v8bf, *(const v4i*)(base + G::OFF_B + (wn * 64 + j * 32 + r32) * 64 + (((2 * c + h) ^ sw_d) << 4)));
      }
    }
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
      for (int j = 0; j < NT; j++) acc[i][j] = mfma_bf16_32x32x16(b[j], hi[i], acc[i][j]);
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
      for (int j = 0; j < NT; j++) acc[i][j] = mfma_bf16_32x32x16(b[j], lo[i], acc[i][j]);
  };

  // ---------------- pipeline
  // Stage s + 1 is published in the middle of stage s: by then this wave
  // holds all of stage s in registers, so its slot takes stage s + ns, and
  // the first fragments of stage s + 1 arrive behind the last MFMAs of s.
  auto publish = [&](auto behind) {       // that many stages may stay in flight
    wait_vm<G::LOADS * decltype(behind)::value>();
    __builtin_amdgcn_s_waitcnt(0xc07f);   // this wave's LDS reads are done
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");        // no LDS read moves above the barrier
  };
  publish(IC<NS - 1>{});
  // accumulators start at the bias of their columns (zeros without one)
#pragma unroll
  for (int j = 0; j < NT; j++)
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const v2i bb = *(const v2i*)(tlds + off_bias + (wn * 64 + 32 * j + 8 * q + 4 * h) * 2);
      const float b4[4] = {bf16_to_f32((uint32_t)bb[0] & 0xFFFFu), bf16_to_f32((uint32_t)bb[0] >> 16),
                           bf16_to_f32((uint32_t)bb[1] & 0xFFFFu), bf16_to_f32((uint32_t)bb[1] >> 16)};
#pragma unroll
      for (int i = 0; i < MT; i++)
#pragma unroll
        for (int e = 0; e < 4; e++) acc[i][j][4 * q + e] = b4[e];
    }
  Frags f0, f1;
  Scales sc;
  read_frags(0, 0, f0);
  read_scales(0, sc);
  int slot = 0;
  auto fp4_body = [&](int s, auto fullc) {
    const int next = slot + 1 == NS ? 0 : slot + 1;
    Scales scn;
    read_frags(slot, 2, f1);
    __builtin_amdgcn_sched_barrier(0);
    mfma_step(IC<0>{}, f0, sc);
    mfma_step(IC<1>{}, f0, sc);
    __builtin_amdgcn_sched_barrier(0);
    publish(IC<NS - 2>{});
    // unused when stage s + 1 is a low-rank one
    read_frags(next, 0, f0);
    read_scales(min(s + 1, nst - 1), scn);
    __builtin_amdgcn_sched_barrier(0);
    mfma_step(IC<2>{}, f1, sc);
    mfma_step(IC<3>{}, f1, sc);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(fullc)::value != 0) issue_full(s + NS, slot);
    else issue_any(s + NS, slot);
    sc = scn;
    slot = next;
  };
  const int nfull = KR / TK;
  int s = 0;
#pragma unroll 1
  for (; s + NS < nfull; s++) fp4_body(s, IC<1>{});
#pragma unroll 1
  for (; s < nst; s++) fp4_body(s, IC<0>{});
#pragma unroll 1
  for (; s < total; s++) {
    if (R - (s - nst) * TLR > 16) {
      lr_half(slot, 0);
      lr_half(slot, 1);
    } else {
      lr_half(slot, 0);
    }
    publish(IC<NS - 2>{});
    issue_any(s + NS, slot);
    slot = slot + 1 == NS ? 0 : slot + 1;
  }
  wait_vm<0>();   // zeros of stages past the end must not land in the epilogue's LDS

  // ---------------- epilogue: 32 rows at a time through the wave's own LDS
  __syncthreads();   // all waves are done with the ring
  // OUT: 0 bf16, 1 fp32, 2 bf16(result * GELU'(z)) (staged as fp32).
  auto store = [&](auto outc) {
    constexpr int OUT = decltype(outc)::value;
    constexpr int ES = OUT == 0 ? 2 : 4;               // staged element
    constexpr int SROW = 64 * ES + 16;
    constexpr int CH = 64 * ES / 16, RPI = 64 / CH;    // 16-byte chunks per row, rows per load
    uint8_t* stg = tlds + wave * (32 * SROW);
    const __amdgpu_buffer_rsrc_t ro = make_rsrc(out, (uint32_t)M * NO * (OUT == 1 ? 4 : 2));
    const __amdgpu_buffer_rsrc_t rz = make_rsrc(z, OUT == 2 ? (uint32_t)M * NO * 2 : 0u);
#pragma unroll
    for (int i = 0; i < MT; i++) {
      // element offset of this lane's chunk `it` in the output, or none
      auto at = [&](int it) {
        const int gr = m0 + wm * (TM / 2) + 32 * i + it * RPI + lane / CH, gc = n0 + wn * 64 + (lane % CH) * (16 / ES);
        return gr < M && gc < NO ? (uint32_t)gr * NO + gc : kOobOffset;
      };
      v2i zv[32 / RPI];
      if constexpr (OUT == 2) {
#pragma unroll
        for (int it = 0; it < 32 / RPI; it++)
          zv[it] = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(rz, at(it) == kOobOffset ? kOobOffset : at(it) * 2, 0, 0));
      }
#pragma unroll
      for (int j = 0; j < NT; j++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const int col = 32 * j + 8 * q + 4 * h;
          if constexpr (OUT != 0) {
            *(v4f*)(stg + r32 * SROW + col * 4) =
                v4f{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          } else {
            const v2f x01 = {acc[i][j][4 * q + 0], acc[i][j][4 * q + 1]};
            const v2f x23 = {acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            *(v2i*)(stg + r32 * SROW + col * 2) = v2i{(int)__builtin_bit_cast(uint32_t, __builtin_convertvector(x01, v2bf)),
                                                      (int)__builtin_bit_cast(uint32_t, __builtin_convertvector(x23, v2bf))};
          }
        }
      __builtin_amdgcn_s_waitcnt(0xc07f);  // the wave reads back only its own rows
#pragma unroll
      for (int it = 0; it < 32 / RPI; it++) {
        const v4i seg = *(const v4i*)(stg + (it * RPI + lane / CH) * SROW + (lane % CH) * 16);
        const uint32_t off = at(it);
        if constexpr (OUT == 2) {
          const v4f d = __builtin_bit_cast(v4f, seg);
          v2i w;
#pragma unroll
          for (int e = 0; e < 2; e++) {
            const v2f dv = {d[2 * e] * gelu_tanh_grad(bf16_to_f32((uint32_t)zv[it][e] & 0xFFFFu)),
                            d[2 * e + 1] * gelu_tanh_grad(bf16_to_f32((uint32_t)zv[it][e] >> 16))};
            w[e] = (int)__builtin_bit_cast(uint32_t, __builtin_convertvector(dv, v2bf));
          }
          __builtin_amdgcn_raw_buffer_store_b64(w, ro, off == kOobOffset ? kOobOffset : off * 2, 0, 0);
        } else {
          __builtin_amdgcn_raw_buffer_store_b128(seg, ro, off == kOobOffset ? kOobOffset : off * ES, 0, 0);
        }
      }
    }
  };
  if (z) store(IC<2>{});
  else if (out_f32) store(IC<1>{});
  else store(IC<0>{});
}

bool gemm_fp4_tile_supported(bool bwd, int M, int N, int K, int R, bool out_f32) {
  const int NO = bwd ? K : N, KR = bwd ? N : K;
  const size_t lim = (size_t)1 << 31;   // 32-bit buffer offsets
  if ((size_t)M * KR / 2 >= lim || (size_t)N * K / 2 >= lim || (size_t)M * std::max(R, 1) * 4 >= lim ||
      (size_t)M * NO * (out_f32 ? 4 : 2) >= lim || (size_t)NO * std::max(R, 1) * 2 >= lim || KR > (1 << 16))
    return false;
  return slab_bytes(64, KR >> 5, (KR + TK - 1) / TK) + 2 * TileGeom<64>::SLOT <= kCuLds;
}

// Ring slots: as many as fit, in half of a CU's LDS when there are more
// workgroups than CUs and it holds two, so that two workgroups share one.
TileSlots gemm_fp4_tile_slots(int tm, long tiles, int KR) {
  const int slot = (tm + TN) * TROW, rest = slab_bytes(tm, KR >> 5, (KR + TK - 1) / TK);
  const int half = tiles > 256 ? (kCuLds / 2 - rest) / slot : 0;
  return half >= 2 ? TileSlots{true, half} : TileSlots{false, (kCuLds - rest) / slot};
}

hipError_t launch_gemm_fp4_tile(bool bwd, int tm, const uint8_t* a, const uint8_t* as, const uint8_t* wq,
                                const uint8_t* ws, int M, int N, int K, const float* P, int R, const uint16_t* lr,
                                const uint16_t* bias, void* out, bool out_f32, const uint16_t* z, hipStream_t st) {
  const int NO = bwd ? K : N, KR = bwd ? N : K;
  const int tiles_m = (M + tm - 1) / tm, tiles_n = (NO + TN - 1) / TN, tiles = tiles_m * tiles_n;
  const int slot = (tm + TN) * TROW, rest = slab_bytes(tm, KR >> 5, (KR + TK - 1) / TK);
  const int ns = gemm_fp4_tile_slots(tm, tiles, KR).ns;
  const unsigned grid = (unsigned)((tiles + 7) / 8 * 8);
  // The ring depth is a template argument; depths between the compiled ones
  // (of 64-row tiles 4, of 128-row tiles 3) use the next smaller.
#define FT_TILE(BW, TM_, NS_) \
  k_gemm_fp4_tile<BW, TM_, NS_><<<grid, 256, (size_t)NS_ * slot + rest, st>>>(a, as, wq, ws, M, N, K, P, R, lr, bias, out, \
                                                                          out_f32 ? 1 : 0, tiles_m, tiles_n, z)
  if (tm == 64) {
    if (ns >= 5) { if (!bwd) FT_TILE(false, 64, 5); else FT_TILE(true, 64, 5); }
    else if (ns >= 3) { if (!bwd) FT_TILE(false, 64, 3); else FT_TILE(true, 64, 3); }
    else { if (!bwd) FT_TILE(false, 64, 2); else FT_TILE(true, 64, 2); }
  } else {
    if (ns >= 4) { if (!bwd) FT_TILE(false, 128, 4); else FT_TILE(true, 128, 4); }
    else { if (!bwd) FT_TILE(false, 128, 2); else FT_TILE(true, 128, 2); }
  }
#undef FT_TILE
  return hipGetLastError();
}

}  // namespace ft
