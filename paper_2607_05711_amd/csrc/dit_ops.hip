// The parts of a DiT block between its linears (gfx950): LayerNorm with adaLN
// modulation, RMSNorm of q and k with the rotary embedding, the single-stream
// block's GELU, and the gated residual, forward and backward.  They are not
// part of the paper's method; its timed step (Sec. 4, "Efficiency Results")
// contains them.
//
// Every kernel is bound by HBM: each reads its bf16 inputs once, computes in
// fp32 and writes bf16, where the same chain as separate framework operations
// makes some 80 passes over fp32 intermediates per block.  16-byte accesses,
// 8 elements per lane; a row's or a head's sums go over lanes with shuffles.
// Values are rounded to bf16 where the separate operations stored bf16.
// At 4608 tokens of width 3072 a single-stream block's elementwise work took
// 2.1 ms of its 6.1 ms training pass as separate operations.
#include "../../include/fourtune.h"
#include "ft_device.h"
#include "ft_kernels.h"

namespace ft {

namespace {

struct F8 { float v[8]; };

__device__ __forceinline__ F8 unpack8(v4i x) {
  F8 r;
#pragma unroll
  for (int e = 0; e < 4; e++) {
    r.v[2 * e] = bf16_to_f32((uint32_t)x[e] & 0xFFFFu);
    r.v[2 * e + 1] = bf16_to_f32((uint32_t)x[e] >> 16);
  }
  return r;
}

__device__ __forceinline__ v4i pack8(const F8& f) {
  v4i r;
#pragma unroll
  for (int e = 0; e < 4; e++) {
    const v2f x = {f.v[2 * e], f.v[2 * e + 1]};
    r[e] = (int)__builtin_bit_cast(uint32_t, __builtin_convertvector(x, v2bf));
  }
  return r;
}

__device__ __forceinline__ float bf16_round(float x) {
  const v2f p = {x, x};
  return bf16_to_f32(__builtin_bit_cast(uint32_t, __builtin_convertvector(p, v2bf)) & 0xFFFFu);
}

// Sum over aligned groups of `width` lanes (a power of two up to 64).
__device__ __forceinline__ float group_sum(float x, int width) {
  for (int off = 1; off < width; off <<= 1) x += __shfl_xor(x, off, 64);
  return x;
}

constexpr float kNormEps = 1e-6f;

}  // namespace

// ------------------------------------------------- LayerNorm + modulation
// One wave per row, the row in registers (NC chunks of 8 per lane):
//   out = bf16((x - mean) rstd (1 + scale) + shift)
// BWD: with g = dy (1 + scale), dx = bf16(rstd (g - mean(g) - xh mean(g xh))).
// The moments are recomputed in the backward from the same x.
template <int NC, bool BWD>
__global__ __launch_bounds__(256) void k_dit_modulate(const uint16_t* __restrict__ x, const uint16_t* __restrict__ shift,
                                                      const uint16_t* __restrict__ scale,
                                                      const uint16_t* __restrict__ dy, uint16_t* __restrict__ out,
                                                      int rows, int H) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const size_t base = (size_t)row * H;
  v4i xv[NC], gv[NC];
#pragma unroll
  for (int c = 0; c < NC; c++) {
    const int col = (c * 64 + lane) * 8;
    xv[c] = gv[c] = v4i{0, 0, 0, 0};
    if (col < H) {
      xv[c] = *(const v4i*)(x + base + col);
      if constexpr (BWD) gv[c] = *(const v4i*)(dy + base + col);
    }
  }
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < NC; c++) {
    const F8 f = unpack8(xv[c]);
#pragma unroll
    for (int e = 0; e < 8; e++) s += f.v[e];
  }
  const float inv = 1.0f / (float)H;
  const float mean = group_sum(s, 64) * inv;
  float q = 0.f;
#pragma unroll
  for (int c = 0; c < NC; c++) {
    if ((c * 64 + lane) * 8 < H) {
      const F8 f = unpack8(xv[c]);
#pragma unroll
      for (int e = 0; e < 8; e++) { const float d = f.v[e] - mean; q += d * d; }
    }
  }
  const float rstd = rsqrtf(group_sum(q, 64) * inv + kNormEps);
  if constexpr (!BWD) {
#pragma unroll
    for (int c = 0; c < NC; c++) {
      const int col = (c * 64 + lane) * 8;
      if (col < H) {
        const F8 f = unpack8(xv[c]), sc = unpack8(*(const v4i*)(scale + col)), sh = unpack8(*(const v4i*)(shift + col));
        F8 o;
#pragma unroll
        for (int e = 0; e < 8; e++) o.v[e] = (f.v[e] - mean) * rstd * (1.0f + sc.v[e]) + sh.v[e];
        *(v4i*)(out + base + col) = pack8(o);
      }
    }
  } else {
    float a = 0.f, b = 0.f;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      const int col = (c * 64 + lane) * 8;
      if (col < H) {
        const F8 f = unpack8(xv[c]), g = unpack8(gv[c]), sc = unpack8(*(const v4i*)(scale + col));
#pragma unroll
        for (int e = 0; e < 8; e++) {
          const float t = g.v[e] * (1.0f + sc.v[e]);
          a += t;
          b += t * ((f.v[e] - mean) * rstd);
        }
      }
    }
    a = group_sum(a, 64) * inv;
    b = group_sum(b, 64) * inv;
#pragma unroll
    for (int c = 0; c < NC; c++) {
      const int col = (c * 64 + lane) * 8;
      if (col < H) {
        const F8 f = unpack8(xv[c]), g = unpack8(gv[c]), sc = unpack8(*(const v4i*)(scale + col));
        F8 o;
#pragma unroll
        for (int e = 0; e < 8; e++)
          o.v[e] = rstd * (g.v[e] * (1.0f + sc.v[e]) - a - (f.v[e] - mean) * rstd * b);
        *(v4i*)(out + base + col) = pack8(o);
      }
    }
  }
}

// ------------------------------------------------------- q, k, v and GELU
// One workgroup per token over the row [q | k | v | mlp] of a fused linear's
// output (H, H, H and F wide; F may be 0), in 8-element items; the hd / 8
// lanes of a head are neighbours.
//   q, k:  y = bf16(x rsqrt(mean(x^2) + eps) w), then the rotary embedding of
//          consecutive pairs, to row row0 + token of q_out, k_out
//   v:     copied to row row0 + token of v_out, unless v_out is NULL
//   mlp:   gelu_tanh to columns [H, H + F) of c (row stride H + F)
struct QkvArgs {
  const uint16_t* h;            // [T, ldh]
  int64_t ldh;
  int row0, heads, hd, F;
  const uint16_t *qn, *kn;      // [hd]
  const float *cosv, *sinv;     // [rows, hd / 2]
  uint16_t *q, *k, *v, *c;      // q, k, v: [rows, heads, hd]
};

__global__ __launch_bounds__(256) void k_dit_qkv(QkvArgs a) {
  const int t = blockIdx.x, H = a.heads * a.hd, G = a.hd >> 3, HI = H >> 3;
  const uint16_t* hrow = a.h + (size_t)t * a.ldh;
  const int r = a.row0 + t;
  const int items = 3 * HI + (a.F >> 3);
  for (int i = threadIdx.x; i < items; i += 256) {
    if (i >= 2 * HI && i < 3 * HI && !a.v) continue;
    const v4i raw = *(const v4i*)(hrow + 8 * i);
    if (i < 2 * HI) {
      const bool isk = i >= HI;
      const int col = 8 * (isk ? i - HI : i), d = col % a.hd;
      const F8 x = unpack8(raw), w = unpack8(*(const v4i*)((isk ? a.kn : a.qn) + d));
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < 8; e++) s += x.v[e] * x.v[e];
      const float rs = rsqrtf(group_sum(s, G) / (float)a.hd + kNormEps);
      const v4f c4 = *(const v4f*)(a.cosv + (size_t)r * (a.hd / 2) + d / 2);
      const v4f s4 = *(const v4f*)(a.sinv + (size_t)r * (a.hd / 2) + d / 2);
      F8 o;
#pragma unroll
      for (int p = 0; p < 4; p++) {
        const float y0 = bf16_round(x.v[2 * p] * rs * w.v[2 * p]), y1 = bf16_round(x.v[2 * p + 1] * rs * w.v[2 * p + 1]);
        o.v[2 * p] = y0 * c4[p] - y1 * s4[p];
        o.v[2 * p + 1] = y0 * s4[p] + y1 * c4[p];
      }
      *(v4i*)((isk ? a.k : a.q) + (size_t)r * H + col) = pack8(o);
    } else if (i < 3 * HI) {
      *(v4i*)(a.v + (size_t)r * H + 8 * (i - 2 * HI)) = raw;
    } else {
      F8 x = unpack8(raw);
#pragma unroll
      for (int e = 0; e < 8; e++) x.v[e] = gelu_tanh(x.v[e]);
      *(v4i*)(a.c + (size_t)t * (H + a.F) + H + 8 * (i - 3 * HI)) = pack8(x);
    }
  }
}

// Backward: the whole row of dh from the gradients of q_out, k_out and v
// (strided by token and head) and of c.
struct QkvBwdArgs {
  const uint16_t* h;
  int64_t ldh;
  int row0, heads, hd, F;
  const uint16_t *qn, *kn;
  const float *cosv, *sinv;
  const uint16_t *dq, *dk, *dv, *dc;   // dq, dk, dv: element (row, head, d) at row * ts + head * hs + d
  int64_t qts, qhs, kts, khs, vts, vhs;
  uint16_t* dh;                        // [T, 3H + F]
};

__global__ __launch_bounds__(256) void k_dit_qkv_bwd(QkvBwdArgs a) {
  const int t = blockIdx.x, H = a.heads * a.hd, G = a.hd >> 3, HI = H >> 3;
  const uint16_t* hrow = a.h + (size_t)t * a.ldh;
  uint16_t* drow = a.dh + (size_t)t * (3 * H + a.F);
  const int64_t r = a.row0 + t;
  const int items = 3 * HI + (a.F >> 3);
  for (int i = threadIdx.x; i < items; i += 256) {
    if (i < 2 * HI) {
      const bool isk = i >= HI;
      const int col = 8 * (isk ? i - HI : i), head = col / a.hd, d = col - head * a.hd;
      const F8 x = unpack8(*(const v4i*)(hrow + 8 * i)), w = unpack8(*(const v4i*)((isk ? a.kn : a.qn) + d));
      const F8 g = unpack8(isk ? *(const v4i*)(a.dk + r * a.kts + head * a.khs + d)
                               : *(const v4i*)(a.dq + r * a.qts + head * a.qhs + d));
      const v4f c4 = *(const v4f*)(a.cosv + r * (a.hd / 2) + d / 2);
      const v4f s4 = *(const v4f*)(a.sinv + r * (a.hd / 2) + d / 2);
      float ss = 0.f, sd = 0.f;
      F8 wd;   // w * (gradient of the normalized value)
#pragma unroll
      for (int p = 0; p < 4; p++) {
        const float d0 = bf16_round(g.v[2 * p] * c4[p] + g.v[2 * p + 1] * s4[p]);
        const float d1 = bf16_round(g.v[2 * p + 1] * c4[p] - g.v[2 * p] * s4[p]);
        wd.v[2 * p] = w.v[2 * p] * d0;
        wd.v[2 * p + 1] = w.v[2 * p + 1] * d1;
      }
#pragma unroll
      for (int e = 0; e < 8; e++) { ss += x.v[e] * x.v[e]; sd += x.v[e] * wd.v[e]; }
      const float inv = 1.0f / (float)a.hd;
      const float rs = rsqrtf(group_sum(ss, G) * inv + kNormEps);
      const float m = group_sum(sd, G) * inv * rs * rs;
      F8 o;
#pragma unroll
      for (int e = 0; e < 8; e++) o.v[e] = rs * (wd.v[e] - x.v[e] * m);
      *(v4i*)(drow + 8 * i) = pack8(o);
    } else if (i < 3 * HI) {
      const int col = 8 * (i - 2 * HI), head = col / a.hd, d = col - head * a.hd;
      *(v4i*)(drow + 8 * i) = *(const v4i*)(a.dv + r * a.vts + head * a.vhs + d);
    } else {
      const F8 x = unpack8(*(const v4i*)(hrow + 8 * i));
      F8 g = unpack8(*(const v4i*)(a.dc + (size_t)t * (H + a.F) + H + 8 * (i - 3 * HI)));
#pragma unroll
      for (int e = 0; e < 8; e++) g.v[e] *= gelu_tanh_grad(x.v[e]);
      *(v4i*)(drow + 8 * i) = pack8(g);
    }
  }
}

// ------------------------------------------------------- gated residual
//   forward:  out = bf16(x + bf16(gate y));  backward (x NULL): out = bf16(gate y), y = dout
__global__ __launch_bounds__(256) void k_dit_gate(const uint16_t* __restrict__ x, const uint16_t* __restrict__ gate,
                                                  const uint16_t* __restrict__ y, uint16_t* __restrict__ out,
                                                  size_t n8, int H8) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += (size_t)gridDim.x * 256) {
    F8 o = unpack8(*(const v4i*)(y + 8 * i));
    const F8 g = unpack8(*(const v4i*)(gate + 8 * (i % H8)));
#pragma unroll
    for (int e = 0; e < 8; e++) o.v[e] *= g.v[e];
    if (x) {
      const F8 b = unpack8(*(const v4i*)(x + 8 * i));
#pragma unroll
      for (int e = 0; e < 8; e++) o.v[e] = b.v[e] + bf16_round(o.v[e]);
    }
    *(v4i*)(out + 8 * i) = pack8(o);
  }
}

// ------------------------------------------------- modulation vector
// bf16(silu(vec)) W, W bf16 [K, N] row-major: bound by reading W once.  A
// workgroup of 4 waves takes 128 columns (16 lanes read 256 bytes of a row,
// narrower segments reach half the rate) of `kc` rows, eight loads in flight
// per lane, the first eight issued before silu(vec) is staged; k_dit_mod_sum
// adds the parts in order.  One workgroup for all of K leaves 288 workgroups
// on 256 CUs for 18432 columns, two rounds: 31 us.
// 3072 x 18432 (113 MB): 25 us with both launches, the library's two operations 41;
// 3072 x 9216: 19 against 26, both bound by the host's launches there.
constexpr int kModStep = 128, kModMaxRows = 2048;
__global__ __launch_bounds__(256) void k_dit_mod(const uint16_t* __restrict__ vec, const uint16_t* __restrict__ w,
                                                 float* __restrict__ parts, int K, int N, int kc) {
  constexpr int UN = 8;
  __shared__ float sv[kModMaxRows];
  __shared__ __attribute__((aligned(16))) float part[4][128];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c0 = blockIdx.x * 128, col = c0 + (lane & 15) * 8;
  const int kb = blockIdx.y * kc, ke = min(K, kb + kc), lr = lane >> 4;
  const uint32_t off = (uint32_t)lr * (uint32_t)N + (uint32_t)col;
  v4i buf[UN];
  auto row = [&](int k) {
    const uint16_t* p = w + (size_t)k * N;     // uniform
    return col < N && k + lr < ke ? __builtin_nontemporal_load((const v4i*)(p + off)) : v4i{};
  };
  const int k0 = kb + 4 * wave;
#pragma unroll
  for (int u = 0; u < UN; u++) buf[u] = row(k0 + 16 * u);
  for (int i = tid; i < kc; i += 256) {
    const float x = kb + i < ke ? bf16_to_f32(vec[kb + i]) : 0.f;   // past the end: zeros, as the rows
    sv[i] = bf16_round(x / (1.0f + __expf(-x)));
  }
  __syncthreads();
  float acc[8] = {};
  for (int k = k0; k < kb + kc; k += 16 * UN)
#pragma unroll
    for (int u = 0; u < UN; u++) {
      const float s = sv[k + 16 * u + lr - kb];
#pragma unroll
      for (int e = 0; e < 4; e++) {
        acc[2 * e] = fmaf(s, bf16_to_f32((uint32_t)buf[u][e] & 0xFFFFu), acc[2 * e]);
        acc[2 * e + 1] = fmaf(s, bf16_to_f32((uint32_t)buf[u][e] >> 16), acc[2 * e + 1]);
      }
      buf[u] = row(k + 16 * (u + UN));
    }
#pragma unroll
  for (int d = 16; d < 64; d <<= 1)
#pragma unroll
    for (int e = 0; e < 8; e++) acc[e] += __shfl_xor(acc[e], d, 64);
  if (lane < 16) {
#pragma unroll
    for (int e = 0; e < 8; e++) part[wave][lane * 8 + e] = acc[e];
  }
  __syncthreads();
  if (tid < 128 && c0 + tid < N)
    parts[(size_t)blockIdx.y * N + c0 + tid] = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
}

__global__ __launch_bounds__(256) void k_dit_mod_sum(const float* __restrict__ parts, uint16_t* __restrict__ out, int n,
                                                     int N) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= N) return;
  float s = 0.f;
#pragma unroll 8
  for (int i = 0; i < n; i++) s += parts[(size_t)i * N + c];
  out[c] = (uint16_t)(__float_as_uint(bf16_round(s)) >> 16);
}

}  // namespace ft

// ------------------------------------------------------------- entry points
// Called by the package's DiT module only (not part of the public header):
// it checks devices, types and layouts.  Sizes and alignment are checked here.
namespace {

bool al16(const void* p) { return ((uintptr_t)p & 15u) == 0; }
ft_status launched() { return hipGetLastError() == hipSuccess ? FT_OK : FT_ERR_HIP; }

template <bool BWD>
ft_status modulate(const void* x, const void* shift, const void* scale, const void* dy, void* out, int64_t rows,
                   int64_t H, hipStream_t st) {
  if (rows <= 0 || rows >= (int64_t)1 << 31 || H <= 0 || H > 4096 || H % 8 != 0) return FT_ERR_SHAPE;
  if (!x || !scale || !out || (BWD ? !dy : !shift)) return FT_ERR_NULL;
  if (!al16(x) || !al16(shift) || !al16(scale) || !al16(dy) || !al16(out)) return FT_ERR_ALIGN;
  const unsigned grid = (unsigned)((rows + 3) / 4);
#define FT_MOD(NC) \
  ft::k_dit_modulate<NC, BWD><<<grid, 256, 0, st>>>((const uint16_t*)x, (const uint16_t*)shift, (const uint16_t*)scale, \
                                                    (const uint16_t*)dy, (uint16_t*)out, (int)rows, (int)H)
  const int nc = (int)((H + 511) / 512);
  if (nc <= 2) FT_MOD(2);
  else if (nc <= 4) FT_MOD(4);
  else if (nc <= 6) FT_MOD(6);
  else FT_MOD(8);
#undef FT_MOD
  return launched();
}

// hd / 8 lanes per head, a power of two up to a wave, so that a head's lanes share one
bool qkv_shape(int64_t T, int64_t heads, int64_t hd, int64_t F, int64_t ldh) {
  return T > 0 && T < (int64_t)1 << 31 && heads > 0 && hd >= 8 && hd <= 512 && (hd & (hd - 1)) == 0 && F >= 0 &&
         F % 8 == 0 && heads * hd < (1 << 20) && F < (1 << 24) && ldh >= 3 * heads * hd + F && ldh % 8 == 0;
}

}  // namespace

extern "C" {

ft_status ftdit_modulate(const void* x, const void* shift, const void* scale, void* out, int64_t rows, int64_t H,
                         hipStream_t st) {
  return modulate<false>(x, shift, scale, nullptr, out, rows, H, st);
}

ft_status ftdit_modulate_bwd(const void* x, const void* scale, const void* dy, void* dx, int64_t rows, int64_t H,
                             hipStream_t st) {
  return modulate<true>(x, nullptr, scale, dy, dx, rows, H, st);
}

ft_status ftdit_qkv(const void* h, int64_t T, int64_t ldh, int64_t row0, int64_t heads, int64_t hd, int64_t F,
                    const void* qn, const void* kn, const float* cosv, const float* sinv, void* q, void* k, void* v,
                    void* c, hipStream_t st) {
  if (!qkv_shape(T, heads, hd, F, ldh) || row0 < 0 || row0 + T >= (int64_t)1 << 31) return FT_ERR_SHAPE;
  if (!h || !qn || !kn || !cosv || !sinv || !q || !k || (F > 0 && !c)) return FT_ERR_NULL;
  if (!al16(h) || !al16(qn) || !al16(kn) || !al16(cosv) || !al16(sinv) || !al16(q) || !al16(k) || !al16(v) || !al16(c))
    return FT_ERR_ALIGN;
  const ft::QkvArgs a{(const uint16_t*)h, ldh, (int)row0, (int)heads, (int)hd, (int)F, (const uint16_t*)qn,
                      (const uint16_t*)kn, cosv, sinv, (uint16_t*)q, (uint16_t*)k, (uint16_t*)v, (uint16_t*)c};
  ft::k_dit_qkv<<<(unsigned)T, 256, 0, st>>>(a);
  return launched();
}

ft_status ftdit_qkv_bwd(const void* h, int64_t T, int64_t ldh, int64_t row0, int64_t heads, int64_t hd, int64_t F,
                        const void* qn, const void* kn, const float* cosv, const float* sinv, const void* dq,
                        int64_t qts, int64_t qhs, const void* dk, int64_t kts, int64_t khs, const void* dv, int64_t vts,
                        int64_t vhs, const void* dc, void* dh, hipStream_t st) {
  if (!qkv_shape(T, heads, hd, F, ldh) || row0 < 0 || row0 + T >= (int64_t)1 << 31) return FT_ERR_SHAPE;
  if (!h || !qn || !kn || !cosv || !sinv || !dq || !dk || !dv || !dh || (F > 0 && !dc)) return FT_ERR_NULL;
  if (!al16(h) || !al16(qn) || !al16(kn) || !al16(cosv) || !al16(sinv) || !al16(dq) || !al16(dk) || !al16(dv) ||
      !al16(dc) || !al16(dh) || ((qts | qhs | kts | khs | vts | vhs) & 7))
    return FT_ERR_ALIGN;
  const ft::QkvBwdArgs a{(const uint16_t*)h, ldh, (int)row0, (int)heads, (int)hd, (int)F, (const uint16_t*)qn,
                         (const uint16_t*)kn, cosv, sinv, (const uint16_t*)dq, (const uint16_t*)dk, (const uint16_t*)dv,
                         (const uint16_t*)dc, qts, qhs, kts, khs, vts, vhs, (uint16_t*)dh};
  ft::k_dit_qkv_bwd<<<(unsigned)T, 256, 0, st>>>(a);
  return launched();
}

// x NULL: out = bf16(gate y)
ft_status ftdit_gate(const void* x, const void* gate, const void* y, void* out, int64_t rows, int64_t H,
                     hipStream_t st) {
  if (rows <= 0 || rows >= (int64_t)1 << 31 || H <= 0 || H >= 1 << 24 || H % 8 != 0) return FT_ERR_SHAPE;
  if (!gate || !y || !out) return FT_ERR_NULL;
  if (!al16(x) || !al16(gate) || !al16(y) || !al16(out)) return FT_ERR_ALIGN;
  const size_t n8 = (size_t)rows * (size_t)(H / 8);
  ft::k_dit_gate<<<(unsigned)std::min<size_t>((n8 + 255) / 256, 8192), 256, 0, st>>>(
      (const uint16_t*)x, (const uint16_t*)gate, (const uint16_t*)y, (uint16_t*)out, n8, (int)(H / 8));
  return launched();
}

// Parts of the sum over K: rows in steps of kModStep, at most 2048 workgroups
// (eight a CU, which hold the loads in flight that the memory's latency asks
// for) unless a part would pass kModMaxRows.
int64_t ftdit_mod_parts(int64_t K, int64_t N) {
  if (K <= 0 || K >= 1 << 20 || N <= 0 || N >= 1 << 24 || N % 8 != 0) return 0;
  const int64_t steps = (K + ft::kModStep - 1) / ft::kModStep, groups = (N + 127) / 128;
  const int64_t per = std::min<int64_t>(ft::kModMaxRows / ft::kModStep, (steps * groups + 2047) / 2048);
  return (steps + per - 1) / per;
}

// vec [K], W [K, N], out [N]; parts: fp32 [ftdit_mod_parts(K, N), N].
ft_status ftdit_mod(const void* vec, const void* w, void* out, float* parts, int64_t K, int64_t N, hipStream_t st) {
  const int64_t n = ftdit_mod_parts(K, N);
  if (n <= 0) return FT_ERR_SHAPE;
  if (!vec || !w || !out || !parts) return FT_ERR_NULL;
  if (!al16(vec) || !al16(w) || !al16(out) || !al16(parts)) return FT_ERR_ALIGN;
  const int64_t steps = (K + ft::kModStep - 1) / ft::kModStep, per = (steps + n - 1) / n;
  ft::k_dit_mod<<<dim3((unsigned)((N + 127) / 128), (unsigned)n), 256, 0, st>>>(
      (const uint16_t*)vec, (const uint16_t*)w, parts, (int)K, (int)N, (int)per * ft::kModStep);
  ft::k_dit_mod_sum<<<(unsigned)((N + 255) / 256), 256, 0, st>>>(parts, (uint16_t*)out, (int)n, (int)N);
  return launched();
}

}  // extern "C"
