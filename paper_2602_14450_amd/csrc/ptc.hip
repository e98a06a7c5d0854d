// Gauge-covariant parallel-transport network (learned right preconditioner).
//
// A layer maps C_in spinor fields to C_out fields,
//   out_j(x) = sum_i sum_p W[p][j][i] (T_p psi_i)(x),
// over nine paths p = 0, +x, -x, +y, -y, +z, -z, +t, -t with
//   (T_{+mu} psi)(x) = U_mu(x) psi(x + mu),  (T_{-mu} psi)(x) = U_mu(x - mu)^dag psi(x - mu),
// and W[p][j][i] a complex 4x4 spin matrix; the network composes its layers
// linearly, so it is gauge covariant and a fixed linear operator.
//
// GPU form.  For every (site, colour) column n the transported inputs are a
// real vector X[n][k], k = (re/im, p, i, spin), in BF16.  The channel mixing is
// then the real GEMM
//   [out_re; out_im](16 x N) = A (16 x Kp) X^T,  A = [[Wr, -Wi], [Wi, Wr]],
// run on MFMA 16x16x16 BF16 tiles with FP32 accumulation (rows padded to 16,
// Kp = 2K rounded up to 16).  The backward pass uses A^T for dX (MFMA), the
// adjoint transports (T_{+mu}^dag = T_{-mu} for unitary links) as a gather,
// and an MFMA reduction over columns for dW = dOut X^H.  Activations are
// native FP32 spinor fields; links are the handle's native FP32 copy.  The
// training layers form X in LDS, 64 sites at a time, and never store it; the
// FP32 mixing mode writes X and dX to memory (the two-pass form).  The fused
// inference layer forms X in registers and multiplies on the 16x16x32 BF16
// instruction (K padded to 32).
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstring>
#include <vector>

#include "qcd.h"
#include "internal.h"
#include "half_ops.h"

namespace qcd {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));    // BF16 bits, 8 k of one lane
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));  // the 16x16x32 BF16 operand type
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// FP32 -> BF16 bits, round to nearest even (the hardware's conversion).
__device__ __forceinline__ short to_bf16(float f) { return __builtin_bit_cast(short, (__bf16)f); }
__device__ __forceinline__ float from_bf16(short h) { return __uint_as_float(((unsigned)(unsigned short)h) << 16); }

// Element type E of the training GEMM operands (X, A, dOut): BF16 (as short
// bits) on the 16x16x16 BF16 matrix-core instruction, or FP32 on the 16x16x4
// FP32 one (the network's FP32 mixing mode).  In both a lane supplies four
// consecutive k of its row or column: one BF16 instruction takes all four,
// or four FP32 instructions take one each (the sum over k is the same).
template <typename E> struct Mix;
template <> struct Mix<short> {
  using V4 = bf16x4;
  static __device__ __forceinline__ short cvt(float f) { return to_bf16(f); }
  static __device__ __forceinline__ f32x4 mma(V4 a, V4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
  }
};
template <> struct Mix<float> {
  using V4 = f32x4;
  static __device__ __forceinline__ float cvt(float f) { return f; }
  static __device__ __forceinline__ f32x4 mma(V4 a, V4 b, f32x4 c) {
#pragma unroll
    for (int q = 0; q < 4; q++) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q], b[q], c, 0, 0, 0);
    return c;
  }
};

struct PtcLayerDev {
  int cin, cout, K, M, Kp;  // K = 9*cin*4 complex inputs, M = cout*4 complex outputs, Kp = 2K rounded to 16
};

// neighbour half index of (par, h) one step along +mu (dir > 0) or -mu
__device__ __forceinline__ int nbr(const Geom& g, int h, const Coord& c, int mu, int dir) {
  if (mu == 0) {
    const int base = h - (c.x >> 1);
    const int xn = dir > 0 ? ((c.x + 1 == g.L[0]) ? 0 : c.x + 1) : ((c.x == 0) ? g.L[0] - 1 : c.x - 1);
    return base + (xn >> 1);
  }
  // by masks (at most one is set): a conditional of two members would select an address
  const int my = -(mu == 1), mz = -(mu == 2), mt = -(mu == 3);
  const int cm = (c.y & my) | (c.z & mz) | (c.t & mt);
  const int st = (g.sy & my) | (g.sz & mz) | (g.st & mt);
  const int n = (g.L[1] & my) | (g.L[2] & mz) | (g.L[3] & mt);
  if (dir > 0) return (cm + 1 == n) ? h - (n - 1) * st : h + st;
  return (cm == 0) ? h + (n - 1) * st : h - st;
}

// Entry a of u f for one colour vector f (rows of u): each product one
// multiply and one fused step, the sum over colours by separate adds
// (contraction is off so that every kernel that forms a transport gives the
// same bits).
template <typename F> __device__ __forceinline__ cx<float> link_row(const cx<float> (&u)[9], int a, F&& f) {
#pragma clang fp contract(off)
  cx<float> p[3];
#pragma unroll
  for (int b = 0; b < 3; b++) {
    const cx<float> v = u[3 * a + b], x = f(b);
    p[b] = cx<float>(__builtin_fmaf(v.re, x.re, -(v.im * x.im)), __builtin_fmaf(v.re, x.im, v.im * x.re));
  }
  return cx<float>((p[0].re + p[1].re) + p[2].re, (p[0].im + p[1].im) + p[2].im);
}
// u -> u^dag if dag (a product with the conjugate entry has the rounding of
// the product with its signs flipped, so U^dag f needs no second form)
__device__ __forceinline__ void link_adjoint(cx<float> (&u)[9], bool dag) {
  const uint32_t sign = dag ? 0x80000000u : 0u;
  auto conj = [&](float im) { return __uint_as_float(__float_as_uint(im) ^ sign); };
  auto swap = [&](cx<float>& x, cx<float>& y) {
    const float xr = x.re, xi = conj(x.im), yr = y.re, yi = conj(y.im);
    x.re = dag ? yr : xr;
    x.im = dag ? yi : xi;
    y.re = dag ? xr : yr;
    y.im = dag ? xi : yi;
  };
  u[0].im = conj(u[0].im);
  u[4].im = conj(u[4].im);
  u[8].im = conj(u[8].im);
  swap(u[1], u[3]);
  swap(u[2], u[6]);
  swap(u[5], u[7]);
}
// out = u f for the four spins of f
__device__ __forceinline__ void su3_apply(const cx<float> (&u)[9], const cx<float> (&f)[12], cx<float> (&o)[12]) {
#pragma unroll
  for (int s = 0; s < 4; s++)
#pragma unroll
    for (int a = 0; a < 3; a++) o[3 * s + a] = link_row(u, a, [&](int b) { return f[3 * s + b]; });
}

__device__ __forceinline__ size_t col_of(const Geom& g, int par, int h) { return ((size_t)par * g.nb * 64 + h) * 3; }
__device__ __forceinline__ size_t ncols(const Geom& g) { return (size_t)2 * g.nb * 64 * 3; }
// Element (column n, k) of a column-major operand of the two-pass form (X in
// BF16, DX in FP32), stored k-tile-major: per batch and k-tile the 16 k-values
// of each column are contiguous, so the 16 columns x 16 k of one matrix-core
// tile are one contiguous segment.  nc = columns per batch entry, nk = Kp / 16.
__device__ __forceinline__ size_t xidx(size_t nc, int nk, size_t n, int k) {
  const size_t b = n / nc, col = n - b * nc;
  return ((b * nk + (k >> 4)) * nc + col) * 16 + (k & 15);
}

// ---------------------------------------------------------------------------
// Two-pass form (FP32 mixing): forward transport, X at (n, k), n = b * ncols + column (site, colour),
// k = reim*K + (p*cin + i)*4 + spin; k in [2K, Kp) and padding sites are zero.
__global__ __launch_bounds__(256) void k_ptc_transport(Geom g, PtcLayerDev L, const float2* __restrict__ act,
                                                       const float2* __restrict__ U, int recon, float* __restrict__ X) {
  const int b = blockIdx.y;
  const int i_site = blockIdx.x * 256 + threadIdx.x;  // over 2 * nb * 64 (padding included)
  const int per = g.nb * 64;
  if (i_site >= 2 * per) return;
  const int par = i_site >= per, h = i_site - par * per;
  const size_t nc = ncols(g);
  const int nk = L.Kp / 16;
  const size_t n0 = (size_t)b * nc + col_of(g, par, h);  // column of colour 0
  if (h >= g.Vh) {  // padding site: zero columns
    for (int c = 0; c < 3; c++)
      for (int k = 0; k < L.Kp; k++) X[xidx(nc, nk, n0 + c, k)] = 0;
    return;
  }
  const Coord c = decode(g, par, h);
  const size_t fstride = spinor_elems(g);
  for (int k = 2 * L.K; k < L.Kp; k++)
    for (int cc = 0; cc < 3; cc++) X[xidx(nc, nk, n0 + cc, k)] = 0;
  for (int i = 0; i < L.cin; i++) {
    const float2* f = act + ((size_t)b * L.cin + i) * fstride;
    for (int p = 0; p < 9; p++) {
      cx<float> in[12], t[12];
      if (p == 0) {
        load_site(f, g, par, h, t);
      } else {
        const int mu = (p - 1) >> 1;
        const bool fwd = ((p - 1) & 1) == 0;
        const int hn = nbr(g, h, c, mu, fwd ? 1 : -1);
        load_site(f, g, par ^ 1, hn, in);
        cx<float> u[9];
        if (fwd) load_link_any(g, U, recon, mu, par, h, u);       // U_mu(x)
        else load_link_any(g, U, recon, mu, par ^ 1, hn, u);      // U_mu(x - mu)^dag
        link_adjoint(u, !fwd);
        su3_apply(u, in, t);
      }
      const int k0 = (p * L.cin + i) * 4;
      for (int cc = 0; cc < 3; cc++) {
        f32x4 re, im;
#pragma unroll
        for (int s = 0; s < 4; s++) {
          re[s] = t[3 * s + cc].re;
          im[s] = t[3 * s + cc].im;
        }
        // k0 and K are multiples of 4, so each group of 4 stays in one k-tile
        *reinterpret_cast<f32x4*>(X + xidx(nc, nk, n0 + cc, k0)) = re;
        *reinterpret_cast<f32x4*>(X + xidx(nc, nk, n0 + cc, L.K + k0)) = im;
      }
    }
  }
}

// A[16][Kp] (BF16 or FP32) from the complex weights W[p][j][i][s'][s] of one layer.
template <typename E>
__global__ void k_ptc_prep_A(PtcLayerDev L, const float2* __restrict__ W, E* __restrict__ A) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= 16 * L.Kp) return;
  const int r = idx / L.Kp, k = idx % L.Kp;
  float v = 0.0f;
  const bool rre = r < L.M, rim = r >= L.M && r < 2 * L.M;
  const bool kre = k < L.K, kim = k >= L.K && k < 2 * L.K;
  if ((rre || rim) && (kre || kim)) {
    const int row = rre ? r : r - L.M;       // (j, s')
    const int kk = kre ? k : k - L.K;         // (p, i, s)
    const int j = row >> 2, sp = row & 3;
    const int p = kk / (L.cin * 4), i = (kk / 4) % L.cin, s = kk & 3;
    const float2 w = W[(((size_t)(p * L.cout + j) * L.cin + i) * 4 + sp) * 4 + s];
    if (rre && kre) v = w.x;
    else if (rre && kim) v = -w.y;
    else if (rim && kre) v = w.y;
    else v = w.x;
  }
  A[idx] = Mix<E>::cvt(v);
}

// Channel mixing: out[b][j] (native FP32 fields) = layer(X).  One wave per
// tile of 16 columns; A fragments stay in registers.
__global__ __launch_bounds__(256) void k_ptc_mix(Geom g, PtcLayerDev L, const float* __restrict__ X,
                                                 const float* __restrict__ A, float2* __restrict__ out, int nbatch) {
  const int lane = threadIdx.x & 63;
  const int wave = (blockIdx.x * 256 + threadIdx.x) >> 6, nwaves = gridDim.x * 4;
  const size_t N = ncols(g);
  const size_t ntiles = (N * nbatch) / 16;  // N is a multiple of 192
  const int nk = L.Kp / 16;
  f32x4 af[9];
#pragma unroll
  for (int kt = 0; kt < 9; kt++)
#pragma unroll
    for (int q = 0; q < 4; q++) af[kt][q] = kt < nk ? A[(lane % 16) * L.Kp + kt * 16 + 4 * (lane / 16) + q] : 0;
  const size_t fstride = spinor_elems(g);
  for (size_t tile = wave; tile < ntiles; tile += nwaves) {
    const size_t n = tile * 16 + (lane % 16);
    f32x4 acc = {0, 0, 0, 0};
#pragma unroll
    for (int kt = 0; kt < 9; kt++) {
      if (kt >= nk) break;
      const f32x4 bf = *reinterpret_cast<const f32x4*>(X + xidx(N, nk, n, kt * 16 + 4 * (lane / 16)));
      acc = Mix<float>::mma(af[kt], bf, acc);
    }
    // lane holds rows 4*(lane/16) + q of column n
    const int b = (int)(n / N);
    const size_t nn = n - (size_t)b * N;
    const int site = (int)(nn / 3), cc = (int)(nn % 3);
    const int per = g.nb * 64;
    const int par = site >= per, h = site - par * per;
    if (h >= g.Vh) continue;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int r = 4 * (lane / 16) + q;
      if (r >= 2 * L.M) continue;
      const int row = r < L.M ? r : r - L.M;
      const int j = row >> 2, sp = row & 3;
      float* dst = reinterpret_cast<float*>(out + ((size_t)b * L.cout + j) * fstride + sp_block(g, par, h) +
                                            sp_off<float2>(3 * sp + cc, h & 63));
      dst[r < L.M ? 0 : 1] = acc[q];
    }
  }
}

// ---------------------------------------------------------------------------
// Training layers (BF16 mixing): the operand X of 64 sites is formed in LDS
// and consumed there, by the forward layer and again by the weight gradient,
// so no X or dX crosses memory.  A block of four waves takes 64 sites of one
// parity (one per lane); wave w transports along paths w, w + 4 and w + 8, so a
// path is uniform in a wave, its loads are whole 1 KB segments, and its link
// is loaded and rebuilt once for both input channels.  Bound by FP32 issue
// (2300 multiply-adds per site at C_in = 2) and the latency of the neighbour
// loads at two blocks per CU.  At 16^4 with 16 fields (1.05M sites) a 2 -> 2
// layer takes 207 us; writing X to memory and mixing from there took 1.0 + 1.9
// ms.

// One block's work: 64 sites (block hb of parity par) of batch entry b.
struct TrainItem { int b, par, hb; };
// Work index of XCD-contiguous order: the eight XCDs receive consecutive
// workgroups in turn, and each takes its own contiguous eighth of the
// (entry, site block, parity) list, so the neighbours of its blocks are in its
// own L2.
__device__ __forceinline__ TrainItem train_item(const Geom& g, int idx) {
  const uint32_t r = fdiv((uint32_t)(idx >> 1), g.dnb);
  return {(int)r, idx & 1, (idx >> 1) - (int)r * g.nb};
}

// Two BF16 (round to nearest even) in a word.  The values pass through an empty
// asm first: a vector built from two elements of a local array makes the
// compiler load them as overlapping vectors and keep the array in scratch.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  asm("" : "+v"(lo), "+v"(hi));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// The transported inputs of wave w's paths at site h (this lane's), each
// handed to put(pair p * C_in + i, t).  Paths 4 apart run in the same sense, so
// the odd waves take the forward hops and the even ones the identity and the
// backward hops.
template <int CIN, bool FWD, typename F>
__device__ __forceinline__ void train_hops(const Geom& g, const float2* __restrict__ f, const float2* __restrict__ U,
                                           int recon, int par, int h, int p0, F&& put) {
  const size_t fstride = spinor_elems(g);
  const Coord c = decode(g, par, h);
#pragma unroll 1
  for (int p = p0; p < 9; p += 4) {
    const int mu = (p - 1) >> 1;
    const int hn = nbr(g, h, c, mu, FWD ? 1 : -1);
    cx<float> in[CIN][12], u[9];
#pragma unroll
    for (int i = 0; i < CIN; i++) load_site(f + i * fstride, g, par ^ 1, hn, in[i]);
    // U_mu(x), or U_mu(x - mu) applied as its adjoint
    load_link_any(g, U, recon, mu, FWD ? par : par ^ 1, FWD ? h : hn, u);
    link_adjoint(u, !FWD);
#pragma unroll
    for (int i = 0; i < CIN; i++) {
      cx<float> t[12];
      su3_apply(u, in[i], t);
      put(p * CIN + i, t);
    }
  }
}
template <int CIN, typename F>
__device__ __forceinline__ void train_transport(const Geom& g, const float2* __restrict__ f,
                                                const float2* __restrict__ U, int recon, int par, int h, int w,
                                                F&& put) {
  if (w & 1) {
    train_hops<CIN, true>(g, f, U, recon, par, h, w, put);
    return;
  }
  if (w == 0) {
#pragma unroll 1
    for (int i = 0; i < CIN; i++) {
      cx<float> t[12];
      load_site(f + i * spinor_elems(g), g, par, h, t);
      put(i, t);
    }
  }
  train_hops<CIN, false>(g, f, U, recon, par, h, w ? w : 4, put);
}

// Forward layer.  LDS holds X as 8-byte quads (the four spins of one pair, real
// or imaginary) [quad][colour * 64 + site], rows padded to 208 so that the
// four quads a matrix-core operand reads at once fall on different banks.  The
// products run in the k order of the two-pass GEMM (tile by tile), so the
// activations are those of that form bit for bit.  Each wave mixes its 16
// sites x 3 colours; the real and imaginary rows of an output component lie in
// lanes 32 (C_out = 2) or 16 (C_out = 1) apart and are paired by a row swap, so
// that a lane stores whole 16-byte granules.
constexpr int kXCols = 208;
template <int CIN, int COUT>
__global__ __launch_bounds__(256, 2) void k_ptc_layer(Geom g, const float2* __restrict__ in, float2* __restrict__ out,
                                                      const float2* __restrict__ U, int recon,
                                                      const short* __restrict__ A, int items, int chunk) {
  constexpr int K = 36 * CIN, NK = (2 * K + 15) / 16, Kp = 16 * NK;
  __shared__ u32x2 X[4 * NK * kXCols];
  const int idx = (blockIdx.x & 7) * chunk + (blockIdx.x >> 3);
  if (idx >= items) return;
  const TrainItem it = train_item(g, idx);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const size_t fstride = spinor_elems(g);
  {
    const int h = it.hb * 64 + lane;
    const bool valid = h < g.Vh;  // padding sites mix zeros
    train_transport<CIN>(g, in + (size_t)it.b * CIN * fstride, U, recon, it.par, valid ? h : 0, w,
                         [&](int q, const cx<float>(&t)[12]) {
#pragma unroll
                           for (int c = 0; c < 3; c++) {
                             const u32x2 re = {pack_bf16(t[c].re, t[3 + c].re), pack_bf16(t[6 + c].re, t[9 + c].re)};
                             const u32x2 im = {pack_bf16(t[c].im, t[3 + c].im), pack_bf16(t[6 + c].im, t[9 + c].im)};
                             X[q * kXCols + c * 64 + lane] = valid ? re : u32x2{0, 0};
                             X[(9 * CIN + q) * kXCols + c * 64 + lane] = valid ? im : u32x2{0, 0};
                           }
                         });
  }
  for (int e = threadIdx.x; e < (4 * NK - 18 * CIN) * 192; e += 256)  // k in [2K, Kp)
    X[(18 * CIN + e / 192) * kXCols + e % 192] = u32x2{0, 0};
  const int G = lane >> 4, n = lane & 15;
  bf16x4 af[NK];
#pragma unroll
  for (int kt = 0; kt < NK; kt++) af[kt] = *reinterpret_cast<const bf16x4*>(A + n * Kp + kt * 16 + 4 * G);
  __syncthreads();
  f32x4 acc[3];  // rows 4 G + q of this lane's site, per colour
#pragma unroll
  for (int c = 0; c < 3; c++) {
    acc[c] = (f32x4){0, 0, 0, 0};
#pragma unroll
    for (int kt = 0; kt < NK; kt++) {
      const bf16x4 bf = __builtin_bit_cast(bf16x4, X[(4 * kt + G) * kXCols + c * 64 + 16 * w + n]);
      acc[c] = Mix<short>::mma(af[kt], bf, acc[c]);
    }
  }
  // component k = 3 spin + colour of this lane's rows is acc[k % 3][k / 3]
  const int h = it.hb * 64 + 16 * w + n;
  const int j = COUT == 2 ? (G & 1) : 0, half = COUT == 2 ? G >> 1 : G;
  float2* ob = out + ((size_t)it.b * COUT + j) * fstride + sp_block(g, it.par, h) + (h & 63) * 2;
#pragma unroll
  for (int m = 0; m < 3; m++) {
    float v[4];
#pragma unroll
    for (int e = 0; e < 2; e++) {
      const int a = 4 * m + e, b = a + 2;  // half 0 stores granule 2 m, half 1 granule 2 m + 1
      const uint32_t va = __float_as_uint(acc[a % 3][a / 3]), vb = __float_as_uint(acc[b % 3][b / 3]);
      const u32x2 s = COUT == 2 ? __builtin_amdgcn_permlane32_swap(va, vb, false, false)
                                : __builtin_amdgcn_permlane16_swap(va, vb, false, false);
      v[2 * e] = __uint_as_float(s[0]);
      v[2 * e + 1] = __uint_as_float(s[1]);
    }
    if (h < g.Vh && half < 2) *reinterpret_cast<f32x4*>(ob + (2 * m + half) * 128) = (f32x4){v[0], v[1], v[2], v[3]};
  }
}

// ---------------------------------------------------------------------------
// Fused forward layer (inference): the transported inputs are formed in
// registers and fed to the matrix cores directly, so nothing but the
// activations and links crosses HBM.
//
// Column ordering: a wave takes 16 sites (one per lane % 16) and all three
// colours (three accumulators).  The products run on the 16 x 16 x 32 BF16
// instruction; K is ordered by position q of a (path, input channel) pair,
// 8 k each: k = 8 q + 4 sh + 2 s_lo + re/im for spin s = 2 sh + s_lo.
// Position q holds channel i = q % C_in of path p = (q / C_in + 1) mod 9, so
// the hops come first, the forward and backward hop of one direction side
// by side, and the identity path last.  K-tile kt holds positions 4 kt + G,
// lane group G = lane / 16 supplying all 8 k of its pair: a lane transports
// a whole spinor, loading and rebuilding the link once for both spin halves;
// with C_in = 2 the direction of a k-tile is the same for the whole wave, and
// the last k-tile is the identity path only.  Output rows are
// r = (j * 2 + sh') * 4 + s'_lo * 2 + re/im, so lane group G ends up holding
// channel j = G / 2, spins 2 (G % 2) and 2 (G % 2) + 1 of its site for all
// three colours.

// K of the fused layer's weight operand: 2K rounded up to whole 32-wide k-tiles.
__host__ __device__ inline int fused_kp(const PtcLayerDev& L) { return ((2 * L.K + 31) / 32) * 32; }
// path of pair position q
__host__ __device__ inline int fused_path(int q, int cin) { return (q / cin + 1) % 9; }

// A for the fused ordering, from W[p][j][i][s'][s] of one layer (rows of fused_kp(L)).
__global__ void k_ptc_prep_Af(PtcLayerDev L, const float2* __restrict__ W, short* __restrict__ A) {
  const int kf = fused_kp(L);
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= 16 * kf) return;
  const int r = idx / kf, k = idx % kf;
  const int j = r >> 3, spo = ((r >> 2) & 1) * 2 + ((r >> 1) & 1), ro = r & 1;
  const int q = k >> 3, e = k & 7;
  float v = 0.0f;
  if (j < L.cout && q < 9 * L.cin) {
    const int p = fused_path(q, L.cin), i = q % L.cin, s = (e >> 2) * 2 + ((e >> 1) & 1), ri = e & 1;
    const float2 w = W[(((size_t)(p * L.cout + j) * L.cin + i) * 4 + spo) * 4 + s];
    v = ro == ri ? w.x : (ro == 0 ? -w.y : w.y);
  }
  A[idx] = to_bf16(v);
}

// The transported spinor of one (path, input channel) pair in binary16 form
// (FP16 activations and links): the neighbour's three 16-byte granules, the
// link's row 2 rebuilt in binary16, and U v / U^dag v as exact binary16
// products summed in FP32 (the Wilson operator's FP16 arithmetic).  The lanes
// of a wave take different paths (forward and backward hops), so each lane
// selects its entries and signs into the one forward product form.
template <int CIN>
__device__ __forceinline__ void fused_transport_h(const Geom& g, const __half2* __restrict__ in,
                                                  const __half2* __restrict__ U, int recon, int b, int p, int i,
                                                  int par, int h, const Coord& c, size_t fstride,
                                                  cx<float> (&t)[4][3]) {
  using Gr = typename Lay<__half2>::Gran;  // 4 complex components
  const __half2* f = in + ((size_t)b * CIN + i) * fstride;
  const int mu = (p - 1) >> 1;  // p = 1..8
  const bool fwd = ((p - 1) & 1) == 0;
  const int sh_idx = nbr(g, h, c, mu, fwd ? 1 : -1);
  const __half2* fb = f + sp_block(g, par ^ 1, sh_idx) + (sh_idx & 63) * 4;
  h2v v[4][3];  // v[spin][colour]: component 3 spin + colour
#pragma unroll
  for (int j = 0; j < 3; j++) {
    const Gr q = *reinterpret_cast<const Gr*>(fb + j * 64 * 4);
#pragma unroll
    for (int e = 0; e < 4; e++) v[(4 * j + e) / 3][(4 * j + e) % 3] = h2_of(q.s[e]);
  }
  // U_mu(x) (forward) or U_mu(x - mu) (backward, applied as its adjoint)
  const int lp = fwd ? par : par ^ 1, lh = fwd ? h : sh_idx, lane = lh & 63;
  h2v u[9];
  if (recon) {
    const __half2* lb = U + lk_block<6>(g, mu, lp, lh);
    const Gr q = *reinterpret_cast<const Gr*>(lb + lane * 4);
    const __half2* tl = lb + 4 * 64 + lane * 2;
#pragma unroll
    for (int k = 0; k < 4; k++) u[k] = h2_of(q.s[k]);
    u[4] = h2_of(tl[0]);
    u[5] = h2_of(tl[1]);
    h_third_row(u);
  } else {
    const __half2* lb = U + lk_block<9>(g, mu, lp, lh);
    const Gr q0 = *reinterpret_cast<const Gr*>(lb + lane * 4);
    const Gr q1 = *reinterpret_cast<const Gr*>(lb + 64 * 4 + lane * 4);
#pragma unroll
    for (int k = 0; k < 4; k++) {
      u[k] = h2_of(q0.s[k]);
      u[4 + k] = h2_of(q1.s[k]);
    }
    u[8] = h2_of(lb[8 * 64 + lane]);
  }
  // Entry (r, b) of U, or of U^dag read as conj(u[3b + r]), with the sign
  // flips of each form applied per lane: the same products in the same order
  // as h_mult, without running both forms.
  const uint32_t pm = fwd ? 0x80000000u : 0u;  // (re, -im) forward, (re, im) backward
  const uint32_t qm = fwd ? 0u : 0x8000u;      // (im, re) forward, (-im, re) backward
  HLink<false> L;
#pragma unroll
  for (int r = 0; r < 3; r++)
#pragma unroll
    for (int bb = 0; bb < 3; bb++) {
      // both entries as values first: a conditional of two array elements
      // would select an address and index the array at run time
      const uint32_t ef = __builtin_bit_cast(uint32_t, u[3 * r + bb]);
      const uint32_t eb = __builtin_bit_cast(uint32_t, u[3 * bb + r]);
      const uint32_t a = fwd ? ef : eb;
      L.p[3 * r + bb] = __builtin_bit_cast(h2v, a ^ pm);
      L.q[3 * r + bb] = __builtin_bit_cast(h2v, ((a >> 16) | (a << 16)) ^ qm);
    }
#pragma unroll
  for (int s_ = 0; s_ < 4; s_++) h_mult<false>(L, v[s_], t[s_]);
}

// out[b][j] = oscale * sum_{p,i} W[p][j][i] T_p in[b][i] for batch b = blockIdx.y;
// grid.x = 2 * nb (one 64-site block of one parity per workgroup).  Batches
// whose solver has stopped (scal[b].active == 0) are skipped when scal is given.
template <typename SA, typename SL, int CIN, int COUT>
__global__ __launch_bounds__(256) void k_ptc_fused(Geom g, const SA* __restrict__ in, SA* __restrict__ out,
                                                   const SL* __restrict__ U, int recon, const short* __restrict__ A,
                                                   int Kf, float oscale, const Scalars* __restrict__ scal, int ftz) {
  constexpr int NK = (9 * CIN + 3) / 4;  // 32-wide k-tiles: four (path, channel) pairs each
  const int b = blockIdx.y;
  if (scal && !scal[b].active) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int G = lane >> 4, n = lane & 15;
  const int par = blockIdx.x >= g.nb, hb = blockIdx.x - par * g.nb;
  const int h_raw = hb * 64 + w * 16 + n;
  const bool valid = h_raw < g.Vh;
  const int h = valid ? h_raw : 0;  // padding lanes compute on site 0 and store nothing
  const Coord c = decode(g, par, h);
  const size_t fstride = spinor_elems(g);
  bf16x8 af[NK];
#pragma unroll
  for (int kt = 0; kt < NK; kt++) {
    const s16x8 a8 = *reinterpret_cast<const s16x8*>(A + (lane & 15) * Kf + kt * 32 + 8 * G);
    af[kt] = __builtin_bit_cast(bf16x8, a8);
  }
  f32x4 acc[3];
#pragma unroll
  for (int cc = 0; cc < 3; cc++) acc[cc] = (f32x4){0, 0, 0, 0};
#pragma unroll
  for (int kt = 0; kt < NK; kt++) {
    const int q = 4 * kt + G;  // pair position: channel q % C_in of path fused_path(q, C_in)
    cx<float> t[4][3];         // transported spins 0..3, colours 0..2
#pragma unroll
    for (int s_ = 0; s_ < 4; s_++)
#pragma unroll
      for (int cc = 0; cc < 3; cc++) t[s_][cc] = cx<float>(0, 0);
    if (kt == NK - 1) {  // the identity path (positions past 9 C_in are padding)
      if (q < 9 * CIN) {
        const SA* fb = in + ((size_t)b * CIN + q % CIN) * fstride + sp_block(g, par, h);
#pragma unroll
        for (int s_ = 0; s_ < 4; s_++)
#pragma unroll
          for (int cc = 0; cc < 3; cc++) t[s_][cc] = Traits<SA>::load(fb + sp_off<SA>(3 * s_ + cc, h & 63));
      }
    } else if constexpr (std::is_same<SA, __half2>::value && std::is_same<SL, __half2>::value) {
      fused_transport_h<CIN>(g, in, U, recon, b, q / CIN + 1, q % CIN, par, h, c, fstride, t);
    } else {
      const int p = q / CIN + 1, i = q % CIN;  // a hop, p = 1..8
      const SA* f = in + ((size_t)b * CIN + i) * fstride;
      const int mu = (p - 1) >> 1;
      const bool fwd = ((p - 1) & 1) == 0;
      const int hn = nbr(g, h, c, mu, fwd ? 1 : -1);
      const SA* fb = f + sp_block(g, par ^ 1, hn);
      cx<float> v[4][3], u[9];
#pragma unroll
      for (int s_ = 0; s_ < 4; s_++)
#pragma unroll
        for (int cc = 0; cc < 3; cc++) v[s_][cc] = Traits<SA>::load(fb + sp_off<SA>(3 * s_ + cc, hn & 63));
      const int lp = fwd ? par : par ^ 1, lh = fwd ? h : hn;  // U_mu(x) or U_mu(x - mu)
      load_link_any(g, U, recon, mu, lp, lh, u);
#pragma unroll
      for (int s_ = 0; s_ < 4; s_++)
#pragma unroll
        for (int a = 0; a < 3; a++) {
          cx<float> acc_(0, 0);
#pragma unroll
          for (int bb = 0; bb < 3; bb++)
            acc_ = acc_ + (fwd ? u[3 * a + bb] * v[s_][bb] : cmulc(u[3 * bb + a], v[s_][bb]));
          t[s_][a] = acc_;
        }
    }
#pragma unroll
    for (int cc = 0; cc < 3; cc++) {
      // k = 8 q + 4 sh + 2 s_lo + re/im; the hardware's round-to-nearest-even
      // conversion, two values per instruction
      u32x4 bw;
#pragma unroll
      for (int s_ = 0; s_ < 4; s_++) {
        const f32x2 f = {valid ? t[s_][cc].re : 0.0f, valid ? t[s_][cc].im : 0.0f};
        bw[s_] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
      }
      acc[cc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[kt], __builtin_bit_cast(bf16x8, bw), acc[cc], 0, 0, 0);
    }
  }
  const int j = G >> 1, sh = G & 1;
  if (!valid || j >= COUT) return;
  SA* ob = out + ((size_t)b * COUT + j) * fstride + sp_block(g, par, h);
#pragma unroll
  for (int sl = 0; sl < 2; sl++)
#pragma unroll
    for (int cc = 0; cc < 3; cc++) {
      const cx<float> o(oscale * acc[cc][2 * sl], oscale * acc[cc][2 * sl + 1]);
      ob[sp_off<SA>(3 * (2 * sh + sl) + cc, h & 63)] = Traits<SA>::pack(o, ftz);
    }
}

// ---------------------------------------------------------------------------
// Backward of the training layers (BF16 mixing).  The output gradient of a
// layer is kept as BF16 quads DOq[entry][parity][64-site block][quad][colour *
// 64 + site] (quad j: real parts of channel j's four spins, quad C_out + j:
// imaginary parts), 96 C_out bytes per site.  Padding sites hold anything (the
// blocks of layers with other channel counts lie elsewhere in the same buffer):
// readers take valid sites only.
__device__ __forceinline__ size_t doq_block(const Geom& g, int cout, int b, int par, int hb) {
  return (((size_t)b * 2 + par) * g.nb + hb) * (2 * cout) * 192;
}

// dOut (native FP32 fields of the last layer) -> DOq.
__global__ __launch_bounds__(256) void k_ptc_dout_quads(Geom g, int cout, const float2* __restrict__ dout,
                                                        u32x2* __restrict__ DOq) {
  const int i_site = blockIdx.x * 256 + threadIdx.x;
  if (i_site >= 2 * g.Vh) return;
  const int par = i_site >= g.Vh, h = i_site - par * g.Vh;
  for (int j = 0; j < cout; j++) {
    cx<float> f[12];
    load_site(dout + ((size_t)blockIdx.y * cout + j) * spinor_elems(g), g, par, h, f);
    u32x2* d = DOq + doq_block(g, cout, blockIdx.y, par, h >> 6) + (h & 63);
#pragma unroll
    for (int c = 0; c < 3; c++) {
      d[j * 192 + c * 64] = {pack_bf16(f[c].re, f[3 + c].re), pack_bf16(f[6 + c].re, f[9 + c].re)};
      d[(cout + j) * 192 + c * 64] = {pack_bf16(f[c].im, f[3 + c].im), pack_bf16(f[6 + c].im, f[9 + c].im)};
    }
  }
}

// A^T for the input gradient: Ab[p][row][r] = A[r][k], row = 8 i + 4 re/im +
// spin of input channel i (rows of absent channels are zero).
__global__ void k_ptc_prep_Ab(PtcLayerDev L, const short* __restrict__ A, short* __restrict__ Ab) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= 9 * 256) return;
  const int r = idx & 15, row = (idx >> 4) & 15, p = idx >> 8;
  const int i = row >> 3, k = ((row >> 2) & 1) * L.K + (p * L.cin + i) * 4 + (row & 3);
  Ab[idx] = i < L.cin ? A[r * L.Kp + k] : (short)0;
}

// dIn_i(y) = sum_p (T_p^dag dX_{p,i})(y), dX = A^T dOut: p = 0 identity; +mu:
// U_mu(y - mu)^dag dX(y - mu); -mu: U_mu(y) dX(y + mu).  dX is formed where it
// is used: for each path one 16 x 16 x 16 product per colour gives the 8 C_in
// reals of the path's dX at the neighbours of 16 sites (the sum over the 16
// output rows is a single instruction, so dX is that of the two-pass form bit
// for bit), a row swap pairs real and imaginary parts (lane group G gets channel
// G / 2, spins 2 (G % 2) and 2 (G % 2) + 1), and the lane applies the link in
// FP32.  Bound by FP32 issue: the four lane groups of a site each rebuild the
// link (183 us for 2 -> 2 at 16^4 with 16 fields, against 0.5 + 1.2 ms with dX
// through memory).  The result is what the layer below takes as output gradient, so it is
// rounded to BF16 quads at once and no FP32 field is written.
template <int CIN, int COUT>
__global__ __launch_bounds__(256) void k_ptc_layer_din(Geom g, const u32x2* __restrict__ DOq,
                                                       const short* __restrict__ Ab, const float2* __restrict__ U,
                                                       int recon, u32x2* __restrict__ dinq, int items, int chunk) {
  const int idx = (blockIdx.x & 7) * chunk + (blockIdx.x >> 3);
  if (idx >= items) return;
  const TrainItem it = train_item(g, idx);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int G = lane >> 4, n = lane & 15;
  const int h_raw = it.hb * 64 + 16 * w + n;
  const bool valid = h_raw < g.Vh;
  const int h = valid ? h_raw : 0;  // padding lanes compute on site 0 and store nothing
  const Coord c = decode(g, it.par, h);
  // f = this lane's part of dX of path p at the site (sp, sh)
  auto dx = [&](int p, int sp, int sh, cx<float>(&f)[2][3]) {
    const bf16x4 ab = *reinterpret_cast<const bf16x4*>(Ab + (p * 16 + n) * 16 + 4 * G);
    const u32x2* d = DOq + doq_block(g, COUT, it.b, sp, sh >> 6) + G * 192 + (sh & 63);
#pragma unroll
    for (int a = 0; a < 3; a++) {
      const u32x2 q = G < 2 * COUT ? d[a * 64] : u32x2{0, 0};
      const f32x4 x = Mix<short>::mma(ab, __builtin_bit_cast(bf16x4, q), f32x4{0, 0, 0, 0});
#pragma unroll
      for (int s = 0; s < 2; s++) {
        const u32x2 v = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[s]), __float_as_uint(x[2 + s]), false, false);
        f[s][a] = cx<float>(__uint_as_float(v[0]), __uint_as_float(v[1]));
      }
    }
  };
  cx<float> acc[2][3];
  dx(0, it.par, h, acc);
#pragma unroll 1
  for (int mu = 0; mu < 4; mu++)
#pragma unroll
    for (int k = 0; k < 2; k++) {
      const bool dag = k == 0;  // the +mu path reads y - mu, the -mu path y + mu
      const int sh = nbr(g, h, c, mu, dag ? -1 : 1);
      cx<float> f[2][3], u[9];
      if (dag) load_link_any(g, U, recon, mu, it.par ^ 1, sh, u);  // U_mu(y - mu)^dag
      else load_link_any(g, U, recon, mu, it.par, h, u);           // U_mu(y)
      dx(1 + 2 * mu + k, it.par ^ 1, sh, f);
      link_adjoint(u, dag);
#pragma unroll
      for (int s = 0; s < 2; s++)
#pragma unroll
        for (int a = 0; a < 3; a++) acc[s][a] = acc[s][a] + link_row(u, a, [&](int b) { return f[s][b]; });
    }
  const int i = G >> 1, quad = (G & 1) ? CIN + i : i;
  u32x2* o = dinq + doq_block(g, CIN, it.b, it.par, it.hb) + quad * 192 + 16 * w + n;
#pragma unroll
  for (int a = 0; a < 3; a++) {
    const u32x2 v = __builtin_amdgcn_permlane16_swap(pack_bf16(acc[0][a].re, acc[1][a].re),
                                                     pack_bf16(acc[0][a].im, acc[1][a].im), false, false);
    if (valid && i < CIN) o[a * 64] = {v[0], v[1]};
  }
}

// Weight gradient partials: Gp[block][16][Kp] (FP64) = sum over the block's
// sites of dOut X^T, X formed again from the layer's input (train_transport).
// The sum runs over the columns, so both operands are needed with eight
// consecutive columns of one row per lane: LDS holds them transposed, Xt[k] and
// DOt[r][colour * 64 + site], written two columns at a time (neighbouring
// lanes exchange one BF16 each).  Rows of 200 columns put the sixteen rows an
// operand load touches on different banks.  Wave w owns k-tiles w, w + 4, w + 8
// over all columns, so nothing is reduced between waves; its FP32 sums go to
// FP64 every `hold` products of 32 columns (dw_hold).  Two blocks per CU
// (64 KB of LDS each) walk the site blocks of their XCD's part.  248 us for
// 2 -> 2 at 16^4 with 16 fields (reading a stored X with 2-byte gathers: 0.75
// ms), bound like the forward layer, which it repeats.
constexpr int kTCols = 200;
// (v0, v1) of rows k0, k0 + 1 at this lane's column -> one word of row k0 + (lane & 1), columns lane & ~1 and + 1
__device__ __forceinline__ uint32_t pair_columns(uint32_t v, int lane) {
  const uint32_t o = __builtin_amdgcn_update_dpp(0u, v, 0xB1, 0xf, 0xf, true);  // quad_perm [1, 0, 3, 2]
  return __builtin_amdgcn_perm(o, v, (lane & 1) ? 0x03020706u : 0x05040100u);
}
constexpr int kDwBlocks = 512;
template <int CIN, int COUT>
__global__ __launch_bounds__(256, 2) void k_ptc_layer_dw(Geom g, const float2* __restrict__ in,
                                                         const u32x2* __restrict__ DOq, const float2* __restrict__ U,
                                                         int recon, double* __restrict__ Gp, int items, int chunk,
                                                         int per_xcd, int hold) {
  constexpr int K = 36 * CIN, NK = (2 * K + 15) / 16, Kp = 16 * NK, NT = (NK + 3) / 4;
  alignas(16) __shared__ short Xt[Kp * kTCols];
  alignas(16) __shared__ short DOt[16 * kTCols];
  uint32_t* Xw = reinterpret_cast<uint32_t*>(Xt);
  uint32_t* Dw = reinterpret_cast<uint32_t*>(DOt);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = lane >> 4, n = lane & 15;
  const size_t fstride = spinor_elems(g);
  for (int e = tid; e < (Kp - 2 * K) * kTCols / 2; e += 256) Xw[2 * K * kTCols / 2 + e] = 0;
  for (int e = tid; e < (16 - 8 * COUT) * kTCols / 2; e += 256) Dw[8 * COUT * kTCols / 2 + e] = 0;
  f32x4 acc[NT];
  double sum[NT][4];
#pragma unroll
  for (int m = 0; m < NT; m++) {
    acc[m] = (f32x4){0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < 4; q++) sum[m][q] = 0;
  }
  auto flush = [&]() {
#pragma unroll
    for (int m = 0; m < NT; m++) {
#pragma unroll
      for (int q = 0; q < 4; q++) sum[m][q] += (double)acc[m][q];
      acc[m] = (f32x4){0, 0, 0, 0};
    }
  };
  const int base = (blockIdx.x & 7) * chunk;
  const int end = min(chunk, items - base);
  int held = 0;
  for (int j = blockIdx.x >> 3; j < end; j += per_xcd) {
    const TrainItem it = train_item(g, base + j);
    __syncthreads();  // the previous block's operands have been read
    {
      const int h = it.hb * 64 + lane;
      const bool valid = h < g.Vh;
      const int at = (lane & 1) * kTCols / 2 + (lane >> 1);
      train_transport<CIN>(g, in + (size_t)it.b * CIN * fstride, U, recon, it.par, valid ? h : 0, w,
                           [&](int q, const cx<float>(&t)[12]) {
#pragma unroll
                             for (int ri = 0; ri < 2; ri++)
#pragma unroll
                               for (int c = 0; c < 3; c++)
#pragma unroll
                                 for (int s = 0; s < 4; s += 2) {
                                   const cx<float> t0 = t[3 * s + c], t1 = t[3 * s + 3 + c];
                                   const uint32_t v = ri ? pack_bf16(t0.im, t1.im) : pack_bf16(t0.re, t1.re);
                                   Xw[(ri * K + 4 * q + s) * kTCols / 2 + c * 32 + at] =
                                       pair_columns(valid ? v : 0u, lane);
                                 }
                           });
    }
    const u32x2* d = DOq + doq_block(g, COUT, it.b, it.par, it.hb);
    for (int e = tid; e < 2 * COUT * 192; e += 256) {
      const int quad = e / 192, col = e - quad * 192;  // 192 is a multiple of 64: col has the parity of the lane
      // a padding site's column of X is zero, but what its dOut holds need not be finite
      const u32x2 v = it.hb * 64 + (col & 63) < g.Vh ? d[e] : u32x2{0, 0};
      const int at = (4 * quad + (lane & 1)) * kTCols / 2 + (col >> 1);
      Dw[at] = pair_columns(v.x, lane);
      Dw[at + kTCols] = pair_columns(v.y, lane);
    }
    __syncthreads();
#pragma unroll
    for (int ct = 0; ct < 6; ct++) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, *reinterpret_cast<const s16x8*>(DOt + n * kTCols + ct * 32 + 8 * G));
#pragma unroll
      for (int m = 0; m < NT; m++) {
        const int kt = w + 4 * m;
        if (kt < NK) {
          const bf16x8 x =
              __builtin_bit_cast(bf16x8, *reinterpret_cast<const s16x8*>(Xt + (kt * 16 + n) * kTCols + ct * 32 + 8 * G));
          acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, x, acc[m], 0, 0, 0);
        }
      }
      if (++held == hold) {
        held = 0;
        flush();
      }
    }
  }
  flush();
  // lane holds G[4 G + q][kt * 16 + n]
#pragma unroll
  for (int m = 0; m < NT; m++) {
    const int kt = w + 4 * m;
    if (kt < NK)
#pragma unroll
      for (int q = 0; q < 4; q++) Gp[((size_t)blockIdx.x * 16 + 4 * G + q) * Kp + kt * 16 + n] = sum[m][q];
  }
}

// ---------------------------------------------------------------------------
// Backward of the two-pass form.

// dOut (native FP32 fields) -> DO[b][n][16], real form (re rows, im rows, zeros).
__global__ __launch_bounds__(256) void k_ptc_dout_mix(Geom g, PtcLayerDev L, const float2* __restrict__ dout,
                                                      float* __restrict__ DO) {
  const int b = blockIdx.y;
  const int i_site = blockIdx.x * 256 + threadIdx.x;
  const int per = g.nb * 64;
  if (i_site >= 2 * per) return;
  const int par = i_site >= per, h = i_site - par * per;
  float* d = DO + ((size_t)b * ncols(g) + col_of(g, par, h)) * 16;
  const size_t fstride = spinor_elems(g);
  for (int cc = 0; cc < 3; cc++) {
    float row[16];
#pragma unroll
    for (int r = 0; r < 16; r++) row[r] = 0;
    if (h < g.Vh) {
      for (int j = 0; j < L.cout; j++) {
        cx<float> f[12];
        load_site(dout + ((size_t)b * L.cout + j) * fstride, g, par, h, f);
        for (int sp = 0; sp < 4; sp++) {
          row[4 * j + sp] = f[3 * sp + cc].re;
          row[L.M + 4 * j + sp] = f[3 * sp + cc].im;
        }
      }
    }
    for (int r = 0; r < 16; r += 4) {
      f32x4 v = {row[r], row[r + 1], row[r + 2], row[r + 3]};
      *reinterpret_cast<f32x4*>(d + (size_t)cc * 16 + r) = v;
    }
  }
}

// DX[b][n][k] (FP32) = sum_r A[r][k] DO[b][n][r]: one MFMA per (k tile, column tile).
__global__ __launch_bounds__(256) void k_ptc_mix_dx(Geom g, PtcLayerDev L, const float* __restrict__ DO,
                                                    const float* __restrict__ A, float* __restrict__ DX, int nbatch) {
  const int lane = threadIdx.x & 63;
  const int wave = (blockIdx.x * 256 + threadIdx.x) >> 6, nwaves = gridDim.x * 4;
  const size_t N = ncols(g) * nbatch;
  const size_t ntiles = N / 16;
  const int nk = L.Kp / 16;
  for (size_t tile = wave; tile < ntiles; tile += nwaves) {
    const size_t n = tile * 16 + (lane % 16);
    const size_t nc = ncols(g);
    const f32x4 bf = *reinterpret_cast<const f32x4*>(DO + n * 16 + 4 * (lane / 16));
    for (int kt = 0; kt < nk; kt++) {
      f32x4 at;  // A^T tile: row = k, column = r
#pragma unroll
      for (int q = 0; q < 4; q++) at[q] = A[(4 * (lane / 16) + q) * L.Kp + kt * 16 + (lane % 16)];
      f32x4 acc = {0, 0, 0, 0};
      acc = Mix<float>::mma(at, bf, acc);
      // lane holds rows k = kt*16 + 4*(lane/16) + q of column n
      *reinterpret_cast<f32x4*>(DX + xidx(nc, nk, n, kt * 16 + 4 * (lane / 16))) = acc;
    }
  }
}

// dIn_i(y) = sum_p (T_p^dag dX_{p,i})(y): p = 0 identity; +mu: U_mu(y-mu)^dag dX(y-mu); -mu: U_mu(y) dX(y+mu).
__global__ __launch_bounds__(256) void k_ptc_transport_adj(Geom g, PtcLayerDev L, const float* __restrict__ DX,
                                                           const float2* __restrict__ U, int recon,
                                                           float2* __restrict__ din) {
  const int b = blockIdx.y;
  const int i_site = blockIdx.x * 256 + threadIdx.x;
  if (i_site >= 2 * g.Vh) return;
  const int par = i_site >= g.Vh, h = i_site - par * g.Vh;
  const Coord c = decode(g, par, h);
  const size_t fstride = spinor_elems(g);
  const size_t nc = ncols(g);
  const int nk = L.Kp / 16;
  for (int i = 0; i < L.cin; i++) {
    cx<float> acc[12];
#pragma unroll
    for (int k = 0; k < 12; k++) acc[k] = cx<float>(0, 0);
    for (int p = 0; p < 9; p++) {
      int sp = par, sh = h;  // site whose dX column is read
      bool dag = false;
      int mu = -1;
      if (p > 0) {
        mu = (p - 1) >> 1;
        const bool fwd = ((p - 1) & 1) == 0;
        sp = par ^ 1;
        sh = nbr(g, h, c, mu, fwd ? -1 : 1);  // +mu path reads y - mu, -mu path reads y + mu
        dag = fwd;
      }
      cx<float> f[12];
      const int k0 = (p * L.cin + i) * 4;
      const size_t n0 = (size_t)b * nc + col_of(g, sp, sh);
#pragma unroll
      for (int cc = 0; cc < 3; cc++) {
        const f32x4 re = *reinterpret_cast<const f32x4*>(DX + xidx(nc, nk, n0 + cc, k0));
        const f32x4 im = *reinterpret_cast<const f32x4*>(DX + xidx(nc, nk, n0 + cc, L.K + k0));
#pragma unroll
        for (int s = 0; s < 4; s++) f[3 * s + cc] = cx<float>(re[s], im[s]);
      }
      if (p == 0) {
#pragma unroll
        for (int k = 0; k < 12; k++) acc[k] = acc[k] + f[k];
      } else {
        cx<float> u[9], t[12];
        if (dag) load_link_any(g, U, recon, mu, sp, sh, u);   // U_mu(y - mu)^dag
        else load_link_any(g, U, recon, mu, par, h, u);       // U_mu(y)
        link_adjoint(u, dag);
        su3_apply(u, f, t);
#pragma unroll
        for (int k = 0; k < 12; k++) acc[k] = acc[k] + t[k];
      }
    }
    float2* dst = din + ((size_t)b * L.cin + i) * fstride;
    float2* bb = dst + sp_block(g, par, h);
#pragma unroll
    for (int k = 0; k < 12; k++) bb[sp_off<float2>(k, h & 63)] = make_float2(acc[k].re, acc[k].im);
  }
}

// G partials: Gp[wave][16][Kp] = sum over the wave's columns of DO[n][r] X[n][k].
__global__ __launch_bounds__(256) void k_ptc_mix_dw(Geom g, PtcLayerDev L, const float* __restrict__ DO,
                                                    const float* __restrict__ X, float* __restrict__ Gp, int nbatch) {
  const int lane = threadIdx.x & 63;
  const int wave = (blockIdx.x * 256 + threadIdx.x) >> 6, nwaves = gridDim.x * 4;
  const size_t N = ncols(g) * nbatch;
  const size_t ntiles = N / 16;
  const int nk = L.Kp / 16;
  const size_t nc = ncols(g);
  f32x4 acc[9];
#pragma unroll
  for (int kt = 0; kt < 9; kt++) acc[kt] = (f32x4){0, 0, 0, 0};
  for (size_t tile = wave; tile < ntiles; tile += nwaves) {
    const size_t n0 = tile * 16;
    f32x4 a;  // A[r][nn] = DO[n0 + nn][r]: row r = lane % 16, nn = 4*(lane/16) + q
#pragma unroll
    for (int q = 0; q < 4; q++) a[q] = DO[(n0 + 4 * (lane / 16) + q) * 16 + (lane % 16)];
#pragma unroll
    for (int kt = 0; kt < 9; kt++) {
      if (kt >= nk) break;
      f32x4 bb;  // B[nn][k] = X(n0 + nn, kt*16 + lane % 16)
#pragma unroll
      for (int q = 0; q < 4; q++) bb[q] = X[xidx(nc, nk, n0 + 4 * (lane / 16) + q, kt * 16 + (lane % 16))];
      acc[kt] = Mix<float>::mma(a, bb, acc[kt]);
    }
  }
  // lane holds G[4*(lane/16) + q][kt*16 + lane % 16]
  float* dst = Gp + (size_t)wave * 16 * L.Kp;
#pragma unroll
  for (int kt = 0; kt < 9; kt++) {
    if (kt >= nk) break;
#pragma unroll
    for (int q = 0; q < 4; q++) dst[(size_t)(4 * (lane / 16) + q) * L.Kp + kt * 16 + (lane % 16)] = acc[kt][q];
  }
}

// Sum the partials (FP64 per block, or FP32 per wave in the two-pass form) in
// two fixed-order passes: slice sl adds rows
// sl, sl + kDwSlices, ... for every weight (one thread per weight and slice),
// then the slices are added in order and the complex gradient
// dW = (G00 + G11) + i (G10 - G01) is accumulated into grad in the layout of W.
constexpr int kDwSlices = 64;
template <typename T>
__global__ __launch_bounds__(64) void k_ptc_dw_slices(PtcLayerDev L, const T* __restrict__ Gp, int nrows,
                                                      double* __restrict__ part) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;  // over M*K complex weights
  if (idx >= L.M * L.K) return;
  const int row = idx / L.K, kk = idx % L.K;
  double g00 = 0, g01 = 0, g10 = 0, g11 = 0;
  for (int w = blockIdx.y; w < nrows; w += kDwSlices) {
    const T* G = Gp + (size_t)w * 16 * L.Kp;
    g00 += G[(size_t)row * L.Kp + kk];
    g01 += G[(size_t)row * L.Kp + L.K + kk];
    g10 += G[(size_t)(L.M + row) * L.Kp + kk];
    g11 += G[(size_t)(L.M + row) * L.Kp + L.K + kk];
  }
  double* o = part + ((size_t)blockIdx.y * L.M * L.K + idx) * 4;
  o[0] = g00;
  o[1] = g01;
  o[2] = g10;
  o[3] = g11;
}
__global__ void k_ptc_dw_finish(PtcLayerDev L, const double* __restrict__ part, float2* __restrict__ grad) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= L.M * L.K) return;
  const int row = idx / L.K, kk = idx % L.K;
  double g00 = 0, g01 = 0, g10 = 0, g11 = 0;
  for (int sl = 0; sl < kDwSlices; sl++) {
    const double* q = part + ((size_t)sl * L.M * L.K + idx) * 4;
    g00 += q[0];
    g01 += q[1];
    g10 += q[2];
    g11 += q[3];
  }
  const int j = row >> 2, sp = row & 3;
  const int p = kk / (L.cin * 4), i = (kk / 4) % L.cin, s = kk & 3;
  float2& d = grad[(((size_t)(p * L.cout + j) * L.cin + i) * 4 + sp) * 4 + s];
  d.x += (float)(g00 + g11);
  d.y += (float)(g10 - g01);
}

// ---------------------------------------------------------------------------
// Loss |M(r_b) - e_b|^2 / |e_b|^2 (mean over the batch) and its output gradient.

__global__ __launch_bounds__(256) void k_ptc_loss_parts(Geom g, const float2* __restrict__ out,
                                                        const float2* __restrict__ e, double* __restrict__ partials) {
  const int b = blockIdx.y;
  const int i_site = blockIdx.x * 256 + threadIdx.x;
  double red[2] = {0, 0};
  if (i_site < 2 * g.Vh) {
    const int par = i_site >= g.Vh, h = i_site - par * g.Vh;
    const size_t fo = (size_t)b * spinor_elems(g);
    cx<float> o[12], t[12];
    load_site(out + fo, g, par, h, o);
    load_site(e + fo, g, par, h, t);
    float a = 0, n = 0;
    for (int k = 0; k < 12; k++) {
      a += norm2(o[k] - t[k]);
      n += norm2(t[k]);
    }
    red[0] = a;
    red[1] = n;
  }
  block_reduce_store<2>(red, partials + (size_t)b * gridDim.x * 2, blockIdx.x);
}

__global__ void k_ptc_loss_finish(const double* __restrict__ partials, int nrows, int nbatch, double* __restrict__ sums) {
  // sums[b] = (|out-e|^2, |e|^2) for sample blockIdx.x
  double s[2];
  finish_sum<2>(partials + (size_t)blockIdx.x * nrows * 2, nrows, s);
  if (threadIdx.x == 0) {
    sums[2 * blockIdx.x] = s[0];
    sums[2 * blockIdx.x + 1] = s[1];
  }
}

__global__ __launch_bounds__(256) void k_ptc_dout(Geom g, const float2* __restrict__ out, const float2* __restrict__ e,
                                                  const double* __restrict__ sums, int nbatch,
                                                  float2* __restrict__ dout) {
  const int b = blockIdx.y;
  const int i_site = blockIdx.x * 256 + threadIdx.x;
  if (i_site >= 2 * g.Vh) return;
  const int par = i_site >= g.Vh, h = i_site - par * g.Vh;
  const size_t fo = (size_t)b * spinor_elems(g);
  const float c = (float)(2.0 / (nbatch * sums[2 * b + 1]));
  cx<float> o[12], t[12], d[12];
  load_site(out + fo, g, par, h, o);
  load_site(e + fo, g, par, h, t);
  for (int k = 0; k < 12; k++) d[k] = c * (o[k] - t[k]);
  store_site(dout + fo, g, par, h, d, 0);
}

// Per-field |a|^2 and |b|^2 (for the gain |M(v)| / |v| of the network).
__global__ __launch_bounds__(256) void k_ptc_norms(Geom g, const float2* __restrict__ a, const float2* __restrict__ b,
                                                   double* __restrict__ partials) {
  const int bi = blockIdx.y;
  const int i_site = blockIdx.x * 256 + threadIdx.x;
  double red[2] = {0, 0};
  if (i_site < 2 * g.Vh) {
    const int par = i_site >= g.Vh, h = i_site - par * g.Vh;
    const size_t fo = (size_t)bi * spinor_elems(g);
    cx<float> x[12], y[12];
    load_site(a + fo, g, par, h, x);
    load_site(b + fo, g, par, h, y);
    float na = 0, nb = 0;
    for (int k = 0; k < 12; k++) {
      na += norm2(x[k]);
      nb += norm2(y[k]);
    }
    red[0] = na;
    red[1] = nb;
  }
  block_reduce_store<2>(red, partials + (size_t)bi * gridDim.x * 2, blockIdx.x);
}

// Adam on FP32 weights (Kingma & Ba 2015), bias-corrected.
__global__ void k_adam(float* __restrict__ w, const float* __restrict__ grad, float* __restrict__ m,
                       float* __restrict__ v, int n, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gr = grad[i];
  const float mi = b1 * m[i] + (1 - b1) * gr;
  const float vi = b2 * v[i] + (1 - b2) * gr * gr;
  m[i] = mi;
  v[i] = vi;
  w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// FP16 native -> FP32 native and back (for applying the network inside the FP16 solver).
__global__ __launch_bounds__(256) void k_h2f(Geom g, const __half2* __restrict__ src, float2* __restrict__ dst,
                                             float scale) {
  const int i_site = blockIdx.x * 256 + threadIdx.x;
  if (i_site >= 2 * g.Vh) return;
  const int par = i_site >= g.Vh, h = i_site - par * g.Vh;
  const size_t o = (size_t)blockIdx.y * spinor_elems(g);
  cx<float> f[12];
  load_site(src + o, g, par, h, f);
  for (int k = 0; k < 12; k++) f[k] = scale * f[k];
  store_site(dst + o, g, par, h, f, 0);
}
__global__ __launch_bounds__(256) void k_f2h(Geom g, const float2* __restrict__ src, __half2* __restrict__ dst,
                                             int ftz) {
  const int i_site = blockIdx.x * 256 + threadIdx.x;
  if (i_site >= 2 * g.Vh) return;
  const int par = i_site >= g.Vh, h = i_site - par * g.Vh;
  const size_t o = (size_t)blockIdx.y * spinor_elems(g);
  cx<float> f[12];
  load_site(src + o, g, par, h, f);
  store_site(dst + o, g, par, h, f, ftz);
}

}  // namespace qcd

// ===========================================================================
// Host side: the network handle and its C ABI.

using namespace qcd;

struct qcd_ptc {
  const qcd_gauge* gauge;
  Geom g;
  int nlayers;
  int channels[kPtcMaxLayers + 1];
  PtcLayerDev L[kPtcMaxLayers];
  int max_batch;
  size_t nweights;                  // complex weights in total
  size_t woff[kPtcMaxLayers];       // complex offset of each layer's weights
  float2* w;                        // FP32 master weights
  float2* grad;
  float2* adam_m;
  float2* adam_v;
  int adam_step;
  int mix_fp32;                     // 1: the two-pass GEMMs (A, X, DO) in FP32, else BF16
  void* A[kPtcMaxLayers];           // GEMM operands (training ordering), BF16 or FP32
  short* Ab[kPtcMaxLayers];         // BF16 operands of the input gradient (A^T by path)
  short* Af[kPtcMaxLayers];         // BF16 GEMM operands (fused inference ordering)
  __half2* act16[kPtcMaxLayers + 1];  // FP16 hidden activations of the solver's applications
  float2* act[kPtcMaxLayers + 1];   // activations (batch x channels native FP32 fields)
  // Buffers of training and of the FP32 mixing mode, allocated on first use: a
  // handle that only preconditions never holds them.
  bool train_ready;                 // target, dact
  float2* target;                   // training targets (batch fields)
  float2* dact[2];                  // gradient ping-pong buffers
  bool quads_ready;                 // BF16 mixing: DOq
  u32x2* DOq[2];                    // output gradients in BF16 quads, ping-pong over the layers
  bool two_pass_ready;              // FP32 mixing: X, DO, DX
  float* X[kPtcMaxLayers];          // transported inputs per layer (kept for the backward pass)
  float* DO;                        // output gradient in the real form
  float* DX;
  void* Gp;                         // weight-gradient partials: FP64 per block, or FP32 per wave (two-pass)
  double* dwp;                      // weight-gradient slices [kDwSlices][M*K][4]
  double* partials;
  double* sums;
  int mix_blocks;
  std::vector<void*> allocs;
};

namespace {

template <typename... A> qcd_status pfail(qcd_status code, const char* fmt, A... a) {
  return (qcd_status)set_error((int)code, fmt, a...);
}
#define PTC_TRY(expr)                                                                                   \
  do {                                                                                                  \
    hipError_t e_ = (expr);                                                                             \
    if (e_ != hipSuccess) return pfail(QCD_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_));            \
  } while (0)
#define PTC_LAUNCHED()                                                                                  \
  do {                                                                                                  \
    hipError_t e_ = hipGetLastError();                                                                  \
    if (e_ != hipSuccess) return pfail(QCD_ERR_HIP, "kernel launch: %s", hipGetErrorString(e_));        \
  } while (0)

size_t fields_bytes(const Geom& g, size_t nf) { return nf * spinor_elems(g) * sizeof(float2); }
int site_blocks_pad(const Geom& g) { return (2 * g.nb * 64 + 255) / 256; }
int site_blocks(const Geom& g) { return (2 * g.Vh + 255) / 256; }
const float2* links32(const qcd_ptc* n) { return (const float2*)n->gauge->U[kFP32]; }
int recon_of(const qcd_ptc* n, int prec) { return n->gauge->tune[prec].recon; }

qcd_status alloc(qcd_ptc* n, void** p, size_t bytes) {
  PTC_TRY(hipMalloc(p, bytes ? bytes : 256));
  n->allocs.push_back(*p);
  return QCD_OK;
}

void prep_weights(qcd_ptc* n, hipStream_t st) {
  for (int l = 0; l < n->nlayers; l++) {
    const int cnt = 16 * n->L[l].Kp, cntf = 16 * fused_kp(n->L[l]);
    if (n->mix_fp32)
      hipLaunchKernelGGL(k_ptc_prep_A<float>, dim3((cnt + 255) / 256), dim3(256), 0, st, n->L[l],
                         (const float2*)(n->w + n->woff[l]), (float*)n->A[l]);
    else {
      hipLaunchKernelGGL(k_ptc_prep_A<short>, dim3((cnt + 255) / 256), dim3(256), 0, st, n->L[l],
                         (const float2*)(n->w + n->woff[l]), (short*)n->A[l]);
      hipLaunchKernelGGL(k_ptc_prep_Ab, dim3(9), dim3(256), 0, st, n->L[l], (const short*)n->A[l], n->Ab[l]);
    }
    hipLaunchKernelGGL(k_ptc_prep_Af, dim3((cntf + 255) / 256), dim3(256), 0, st, n->L[l],
                       (const float2*)(n->w + n->woff[l]), n->Af[l]);
  }
}

// Widest GEMM operand row of the network, and the rows of a batch element.
int max_kp(const qcd_ptc* n) {
  int m = 16;
  for (int l = 0; l < n->nlayers; l++) m = std::max(m, n->L[l].Kp);
  return m;
}
size_t gemm_rows(const Geom& g) { return (size_t)2 * g.nb * 64 * 3; }

// The buffers of training and of the FP32 mixing mode (max_batch elements each), on first use.
qcd_status ensure_train(qcd_ptc* n) {
  const Geom& g = n->g;
  int maxc = 1;
  for (int l = 0; l <= n->nlayers; l++) maxc = std::max(maxc, n->channels[l]);
  qcd_status rc = QCD_OK;
  if (!n->train_ready) {
    rc = alloc(n, (void**)&n->target, fields_bytes(g, n->max_batch));
    if (rc == QCD_OK) rc = alloc(n, (void**)&n->dact[0], fields_bytes(g, (size_t)n->max_batch * maxc));
    if (rc == QCD_OK) rc = alloc(n, (void**)&n->dact[1], fields_bytes(g, (size_t)n->max_batch * maxc));
    if (rc) return rc;
    n->train_ready = true;
  }
  if (n->mix_fp32 && !n->two_pass_ready) {
    const size_t N = gemm_rows(g), es = sizeof(float);
    const int maxKp = max_kp(n);
    // the FP32-mixing inference reuses X[0] for every layer: it takes the widest layer's size
    for (int l = 0; l < n->nlayers && rc == QCD_OK; l++)
      rc = alloc(n, (void**)&n->X[l], (size_t)n->max_batch * N * (l == 0 ? maxKp : n->L[l].Kp) * es);
    if (rc == QCD_OK) rc = alloc(n, (void**)&n->DO, (size_t)n->max_batch * N * 16 * es);
    if (rc == QCD_OK) rc = alloc(n, (void**)&n->DX, (size_t)n->max_batch * N * maxKp * es);
    if (rc) return rc;
    n->two_pass_ready = true;
  }
  if (!n->mix_fp32 && !n->quads_ready) {
    const size_t bytes = (size_t)n->max_batch * 2 * g.nb * (2 * maxc) * 192 * sizeof(u32x2);
    for (int k = 0; k < 2 && rc == QCD_OK; k++) rc = alloc(n, (void**)&n->DOq[k], bytes);
    if (rc) return rc;
    n->quads_ready = true;
  }
  return QCD_OK;
}

template <typename SA, typename SL>
void fused_layer(const qcd_ptc* n, int l, int nb, const SA* in, SA* out, const SL* U, float oscale,
                 const Scalars* scal, int ftz, hipStream_t st) {
  const Geom& g = n->g;
  const PtcLayerDev& L = n->L[l];
  const dim3 grid(2 * g.nb, nb), block(256);
  const int recon = recon_of(n, sizeof(SL) == sizeof(float2) ? kFP32 : kFP16);
#define PTC_FUSED(CI, CO)                                                                                          \
  hipLaunchKernelGGL((k_ptc_fused<SA, SL, CI, CO>), grid, block, 0, st, g, in, out, U, recon, (const short*)n->Af[l], \
                     fused_kp(L), oscale, scal, ftz)
  if (L.cin == 1 && L.cout == 1) PTC_FUSED(1, 1);
  else if (L.cin == 1) PTC_FUSED(1, 2);
  else if (L.cout == 1) PTC_FUSED(2, 1);
  else PTC_FUSED(2, 2);
#undef PTC_FUSED
}

// Forward through all layers from act[0].  With train, the layers run in the k
// order that the weight gradient shares, or in FP32 mixing the two-pass form
// keeps the transported inputs of every layer for the backward pass; else
// each layer is one fused kernel.
void two_pass_layer(qcd_ptc* n, int l, int nb, hipStream_t st) {
  const Geom& g = n->g;
  hipLaunchKernelGGL(k_ptc_transport, dim3(site_blocks_pad(g), nb), dim3(256), 0, st, g, n->L[l],
                     (const float2*)n->act[l], links32(n), recon_of(n, kFP32), n->X[l]);
  hipLaunchKernelGGL(k_ptc_mix, dim3(n->mix_blocks), dim3(256), 0, st, g, n->L[l], (const float*)n->X[l],
                     (const float*)n->A[l], n->act[l + 1], nb);
}

// Grid of a training-layer launch: every (batch entry, parity, 64-site block), in eight contiguous parts.
int train_items(const Geom& g, int nb) { return 2 * g.nb * nb; }
int train_chunk(const Geom& g, int nb) { return (train_items(g, nb) + 7) / 8; }
// Products of 32 columns that one FP32 chain of the weight gradient adds up: a
// 4096th of the columns, from 32 on small calls (whose few chains are summed in
// FP64 as well) to 768 at 16^4 with 16 fields.
int dw_hold(const Geom& g, int nb) { return std::min(24, std::max(1, (int)(gemm_rows(g) * nb / 4096 / 32))); }

void train_layer(qcd_ptc* n, int l, int nb, hipStream_t st) {
  const Geom& g = n->g;
  const PtcLayerDev& L = n->L[l];
  const int items = train_items(g, nb), chunk = train_chunk(g, nb);
#define PTC_LAYER(CI, CO)                                                                                            \
  hipLaunchKernelGGL((k_ptc_layer<CI, CO>), dim3(8 * chunk), dim3(256), 0, st, g, (const float2*)n->act[l],            \
                     n->act[l + 1], links32(n), recon_of(n, kFP32), (const short*)n->A[l], items, chunk)
  if (L.cin == 1 && L.cout == 1) PTC_LAYER(1, 1);
  else if (L.cin == 1) PTC_LAYER(1, 2);
  else if (L.cout == 1) PTC_LAYER(2, 1);
  else PTC_LAYER(2, 2);
#undef PTC_LAYER
}

// (the FP32 mixing mode runs every FP32-activation forward in the two-pass form)
qcd_status forward(qcd_ptc* n, int nb, bool train, hipStream_t st) {
  if (train || n->mix_fp32) {
    qcd_status rc = ensure_train(n);
    if (rc) return rc;
  }
  for (int l = 0; l < n->nlayers; l++) {
    if (n->mix_fp32) {
      two_pass_layer(n, l, nb, st);
    } else if (!train) {
      fused_layer<float2, float2>(n, l, nb, n->act[l], n->act[l + 1], links32(n), 1.0f, nullptr, 0, st);
    } else {
      train_layer(n, l, nb, st);
    }
  }
  return QCD_OK;
}

// One layer's backward in the two-pass form from dact[cur]: weight gradient into
// n->grad, and (l > 0) the input gradient into dact[cur ^ 1].
void backward_layer_fp32(qcd_ptc* n, int l, int nb, int cur, hipStream_t st) {
  const Geom& g = n->g;
  const PtcLayerDev& L = n->L[l];
  hipLaunchKernelGGL(k_ptc_dout_mix, dim3(site_blocks_pad(g), nb), dim3(256), 0, st, g, L,
                     (const float2*)n->dact[cur], n->DO);
  hipLaunchKernelGGL(k_ptc_mix_dw, dim3(n->mix_blocks), dim3(256), 0, st, g, L, (const float*)n->DO,
                     (const float*)n->X[l], (float*)n->Gp, nb);
  hipLaunchKernelGGL(k_ptc_dw_slices<float>, dim3((L.M * L.K + 63) / 64, kDwSlices), dim3(64), 0, st, L,
                     (const float*)n->Gp, n->mix_blocks * 4, n->dwp);
  if (l > 0) {
    hipLaunchKernelGGL(k_ptc_mix_dx, dim3(n->mix_blocks), dim3(256), 0, st, g, L, (const float*)n->DO,
                       (const float*)n->A[l], n->DX, nb);
    hipLaunchKernelGGL(k_ptc_transport_adj, dim3(site_blocks(g), nb), dim3(256), 0, st, g, L, (const float*)n->DX,
                       links32(n), recon_of(n, kFP32), n->dact[cur ^ 1]);
  }
}

// The same in BF16 mixing from DOq[cur]; the input gradient goes to DOq[cur ^ 1].
void backward_layer(qcd_ptc* n, int l, int nb, int cur, hipStream_t st) {
  const Geom& g = n->g;
  const PtcLayerDev& L = n->L[l];
  const int items = train_items(g, nb), chunk = train_chunk(g, nb);
  const int per_xcd = std::min(chunk, kDwBlocks / 8), hold = dw_hold(g, nb);
#define PTC_BACK(CI, CO)                                                                                             \
  do {                                                                                                               \
    hipLaunchKernelGGL((k_ptc_layer_dw<CI, CO>), dim3(8 * per_xcd), dim3(256), 0, st, g, (const float2*)n->act[l],     \
                       (const u32x2*)n->DOq[cur], links32(n), recon_of(n, kFP32), (double*)n->Gp, items, chunk,        \
                       per_xcd, hold);                                                                               \
    if (l > 0)                                                                                                       \
      hipLaunchKernelGGL((k_ptc_layer_din<CI, CO>), dim3(8 * chunk), dim3(256), 0, st, g, (const u32x2*)n->DOq[cur],   \
                         (const short*)n->Ab[l], links32(n), recon_of(n, kFP32), n->DOq[cur ^ 1], items, chunk);       \
  } while (0)
  if (L.cin == 1 && L.cout == 1) PTC_BACK(1, 1);
  else if (L.cin == 1) PTC_BACK(1, 2);
  else if (L.cout == 1) PTC_BACK(2, 1);
  else PTC_BACK(2, 2);
#undef PTC_BACK
  hipLaunchKernelGGL(k_ptc_dw_slices<double>, dim3((L.M * L.K + 63) / 64, kDwSlices), dim3(64), 0, st, L,
                     (const double*)n->Gp, 8 * per_xcd, n->dwp);
}

// Weight gradient (into n->grad) from the output gradient in dact[0].
void backward(qcd_ptc* n, int nb, hipStream_t st) {
  if (!n->mix_fp32)
    hipLaunchKernelGGL(k_ptc_dout_quads, dim3(site_blocks(n->g), nb), dim3(256), 0, st, n->g,
                       n->channels[n->nlayers], (const float2*)n->dact[0], n->DOq[0]);
  int cur = 0;
  for (int l = n->nlayers - 1; l >= 0; l--, cur ^= 1) {
    const PtcLayerDev& L = n->L[l];
    if (n->mix_fp32) backward_layer_fp32(n, l, nb, cur, st);
    else backward_layer(n, l, nb, cur, st);
    hipLaunchKernelGGL(k_ptc_dw_finish, dim3((L.M * L.K + 255) / 256), dim3(256), 0, st, L, (const double*)n->dwp,
                       n->grad + n->woff[l]);
  }
}

// mean over the batch of sums[2b] / sums[2b + 1] (synchronises)
qcd_status read_loss(qcd_ptc* n, int nb, double* loss, hipStream_t st) {
  std::vector<double> h(2 * nb);
  PTC_TRY(hipMemcpyAsync(h.data(), n->sums, 2 * nb * sizeof(double), hipMemcpyDeviceToHost, st));
  PTC_TRY(hipStreamSynchronize(st));
  double tot = 0;
  for (int b = 0; b < nb; b++) tot += h[2 * b] / h[2 * b + 1];
  *loss = tot / nb;
  return QCD_OK;
}

// Loss and gradient of the weights (into n->grad) for the batch in act[0] / target.
qcd_status loss_grad(qcd_ptc* n, int nb, double* loss, hipStream_t st) {
  const Geom& g = n->g;
  qcd_status rc = forward(n, nb, true, st);
  if (rc) return rc;
  const int last = n->nlayers;
  hipLaunchKernelGGL(k_ptc_loss_parts, dim3(site_blocks(g), nb), dim3(256), 0, st, g, (const float2*)n->act[last],
                     (const float2*)n->target, n->partials);
  hipLaunchKernelGGL(k_ptc_loss_finish, dim3(nb), dim3(1024), 0, st, (const double*)n->partials, site_blocks(g), nb,
                     n->sums);
  hipLaunchKernelGGL(k_ptc_dout, dim3(site_blocks(g), nb), dim3(256), 0, st, g, (const float2*)n->act[last],
                     (const float2*)n->target, (const double*)n->sums, nb, n->dact[0]);
  PTC_TRY(hipMemsetAsync(n->grad, 0, n->nweights * sizeof(float2), st));
  backward(n, nb, st);
  PTC_LAUNCHED();
  if (loss) return read_loss(n, nb, loss, st);
  return QCD_OK;
}

// The residual loss (1/B) sum_b |D M r_b - r_b|^2 / |r_b|^2 for the batch in
// act[0], D the Wilson matrix of eq. (1) (FP32 operator on the handle's FP32
// links), and its weight gradient: the output gradient is
// 2 / (B |r_b|^2) D^dag (D M r_b - r_b).  target holds D M r, dact[1] the
// scaled residual before D^dag.
qcd_status loss_grad_residual(qcd_ptc* n, double kappa, int nb, double* loss, hipStream_t st) {
  const Geom& g = n->g;
  const qcd_gauge* G = n->gauge;
  qcd_status rc = forward(n, nb, true, st);
  if (rc) return rc;
  const int last = n->nlayers;
  // one thread per site at every size: the small-lattice form adds the hops in
  // another order, and a last-bit change of the residual moves BF16 roundings
  // of the output gradient
  DslashTune tune = G->tune[kFP32];
  tune.split_full = tune.split_eo = 0;
  launch_dslash(kFP32, g, tune, kOpD, kEpiNone, nb, n->target, n->act[last], G->U[kFP32], kappa, nullptr,
                nullptr, nullptr, 0, st);
  hipLaunchKernelGGL(k_ptc_loss_parts, dim3(site_blocks(g), nb), dim3(256), 0, st, g, (const float2*)n->target,
                     (const float2*)n->act[0], n->partials);
  hipLaunchKernelGGL(k_ptc_loss_finish, dim3(nb), dim3(1024), 0, st, (const double*)n->partials, site_blocks(g), nb,
                     n->sums);
  hipLaunchKernelGGL(k_ptc_dout, dim3(site_blocks(g), nb), dim3(256), 0, st, g, (const float2*)n->target,
                     (const float2*)n->act[0], (const double*)n->sums, nb, n->dact[1]);
  launch_dslash(kFP32, g, tune, kOpDdag, kEpiNone, nb, n->dact[0], n->dact[1], G->U[kFP32], kappa, nullptr,
                nullptr, nullptr, 0, st);
  PTC_TRY(hipMemsetAsync(n->grad, 0, n->nweights * sizeof(float2), st));
  backward(n, nb, st);
  PTC_LAUNCHED();
  if (loss) return read_loss(n, nb, loss, st);
  return QCD_OK;
}

// Adam on the FP32 master weights from n->grad, then the GEMM operands.
void adam_step(qcd_ptc* n, double lr, hipStream_t st) {
  n->adam_step++;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.0f - powf(b1, (float)n->adam_step), c2 = 1.0f - powf(b2, (float)n->adam_step);
  const int cnt = (int)(2 * n->nweights);
  hipLaunchKernelGGL(k_adam, dim3((cnt + 255) / 256), dim3(256), 0, st, (float*)n->w, (const float*)n->grad,
                     (float*)n->adam_m, (float*)n->adam_v, cnt, (float)lr, b1, b2, 1e-8f, c1, c2);
  prep_weights(n, st);
}

// Replace one of the handle's buffers by a new one of `bytes`.
qcd_status realloc_buf(qcd_ptc* n, void** p, size_t bytes) {
  void* q = nullptr;
  PTC_TRY(hipMalloc(&q, bytes ? bytes : 256));
  for (auto& a : n->allocs)
    if (a == *p) {
      (void)hipFree(a);
      a = q;
      *p = q;
      return QCD_OK;
    }
  n->allocs.push_back(q);
  *p = q;
  return QCD_OK;
}

// Give one of the handle's buffers back.
template <typename T> void drop_buf(qcd_ptc* n, T** p) {
  const auto at = std::find(n->allocs.begin(), n->allocs.end(), (void*)*p);
  if (at != n->allocs.end()) {
    (void)hipFree(*p);
    n->allocs.erase(at);
  }
  *p = nullptr;
}

qcd_status check_batch(const qcd_ptc* n, int nb) {
  if (!n) return pfail(QCD_ERR_ARG, "null network handle");
  if (nb < 1 || nb > n->max_batch) return pfail(QCD_ERR_ARG, "batch must be in 1..%d", n->max_batch);
  return QCD_OK;
}

}  // namespace

namespace qcd {
// Apply the network to nb native FP16 fields: out = scale * M(in), FP16
// activations and FP16 links (the inner solver's), one fused kernel per
// layer.  Used by the preconditioned inner solver (all launches are
// stream-ordered and capturable); batches whose solver has stopped are
// skipped when scal is given.
// More than max_batch fields are taken max_batch at a time (the hidden
// activations hold max_batch elements).
void ptc_apply_half(qcd_ptc* n, int nb, const void* in, void* out, float scale, int ftz, const Scalars* scal,
                    hipStream_t st) {
  const __half2* U = (const __half2*)n->gauge->U[kFP16];
  const size_t fe = spinor_elems(n->g);
  for (int b0 = 0; b0 < nb; b0 += n->max_batch) {
    const int c = std::min(n->max_batch, nb - b0);
    const __half2* src = (const __half2*)in + b0 * fe;
    for (int l = 0; l < n->nlayers; l++) {
      const bool last = l == n->nlayers - 1;
      __half2* dst = last ? (__half2*)out + b0 * fe : n->act16[l + 1];
      fused_layer<__half2, __half2>(n, l, c, src, dst, U, last ? scale : 1.0f, scal ? scal + b0 : nullptr, ftz, st);
      src = dst;
    }
  }
}
// Largest |M(v_b)| / |v_b| over the nb native FP16 fields v_b (zero fields
// skipped); synchronises.  Returns 0 if every field is zero.
qcd_status ptc_gain(qcd_ptc* n, int nb, const void* in, double* gain, hipStream_t st) {
  const Geom& g = n->g;
  if (!n->gauge->U[kFP16]) return pfail(QCD_ERR_ARG, "the gauge handle holds no FP16 links");
  double best = 0;
  std::vector<double> h(2 * n->max_batch);
  for (int b0 = 0; b0 < nb; b0 += n->max_batch) {  // max_batch fields at a time
    const int c = std::min(n->max_batch, nb - b0);
    hipLaunchKernelGGL(k_h2f, dim3(site_blocks(g), c), dim3(256), 0, st, g,
                       (const __half2*)in + (size_t)b0 * spinor_elems(g), n->act[0], 1.0f);
    qcd_status rc = forward(n, c, false, st);
    if (rc) return rc;
    hipLaunchKernelGGL(k_ptc_norms, dim3(site_blocks(g), c), dim3(256), 0, st, g, (const float2*)n->act[0],
                       (const float2*)n->act[n->nlayers], n->partials);
    hipLaunchKernelGGL(k_ptc_loss_finish, dim3(c), dim3(1024), 0, st, (const double*)n->partials, site_blocks(g), c,
                       n->sums);
    PTC_LAUNCHED();
    PTC_TRY(hipMemcpyAsync(h.data(), n->sums, 2 * c * sizeof(double), hipMemcpyDeviceToHost, st));
    PTC_TRY(hipStreamSynchronize(st));
    for (int b = 0; b < c; b++)
      if (h[2 * b] > 0 && std::isfinite(h[2 * b + 1])) best = std::max(best, std::sqrt(h[2 * b + 1] / h[2 * b]));
      else if (h[2 * b] > 0) return pfail(QCD_ERR_NONFINITE, "network output is not finite");
  }
  *gain = best;
  return QCD_OK;
}
int ptc_max_batch(const qcd_ptc* n) { return n->max_batch; }
const qcd_gauge* ptc_gauge(const qcd_ptc* n) { return n->gauge; }
}  // namespace qcd

extern "C" {

qcd_status qcd_ptc_free(qcd_ptc* n) {
  if (!n) return QCD_OK;
  for (void* p : n->allocs) (void)hipFree(p);
  delete n;
  return QCD_OK;
}

qcd_status qcd_ptc_create(qcd_ptc** out, const qcd_gauge* gauge, int nlayers, const int* channels, int max_batch,
                          void* stream) {
  if (!out || !gauge || !channels) return pfail(QCD_ERR_ARG, "null argument");
  if (nlayers < 1 || nlayers > kPtcMaxLayers) return pfail(QCD_ERR_ARG, "nlayers must be in 1..%d", kPtcMaxLayers);
  if (max_batch < 1 || max_batch > kMaxRhs) return pfail(QCD_ERR_ARG, "max_batch must be in 1..%d", kMaxRhs);
  if (!gauge->U[kFP32]) return pfail(QCD_ERR_ARG, "the network needs the gauge handle's FP32 links");
  for (int l = 0; l <= nlayers; l++)
    if (channels[l] < 1 || channels[l] > 2) return pfail(QCD_ERR_UNSUPPORTED, "channels must be 1 or 2 per layer");
  if (channels[0] != 1 || channels[nlayers] != 1)
    return pfail(QCD_ERR_ARG, "the network maps one spinor field to one spinor field");
  qcd_ptc* n = new qcd_ptc();
  n->gauge = gauge;
  n->g = gauge->g;
  n->nlayers = nlayers;
  n->max_batch = max_batch;
  n->nweights = 0;
  int maxKp = 16;
  for (int l = 0; l <= nlayers; l++) n->channels[l] = channels[l];
  for (int l = 0; l < nlayers; l++) {
    PtcLayerDev& L = n->L[l];
    L.cin = channels[l];
    L.cout = channels[l + 1];
    L.K = 9 * L.cin * 4;
    L.M = L.cout * 4;
    L.Kp = ((2 * L.K + 15) / 16) * 16;
    n->woff[l] = n->nweights;
    n->nweights += (size_t)9 * L.cout * L.cin * 16;
    maxKp = std::max(maxKp, L.Kp);
  }
  const Geom& g = n->g;
  n->mix_blocks = 1024;
  qcd_status rc = QCD_OK;
#define PTC_ALLOC(ptr, bytes) \
  if (rc == QCD_OK) rc = alloc(n, (void**)&(ptr), (bytes))
  PTC_ALLOC(n->w, n->nweights * sizeof(float2));
  PTC_ALLOC(n->grad, n->nweights * sizeof(float2));
  PTC_ALLOC(n->adam_m, n->nweights * sizeof(float2));
  PTC_ALLOC(n->adam_v, n->nweights * sizeof(float2));
  for (int l = 0; l < nlayers; l++) {
    PTC_ALLOC(n->A[l], 16 * (size_t)n->L[l].Kp * sizeof(short));
    PTC_ALLOC(n->Af[l], 16 * (size_t)fused_kp(n->L[l]) * sizeof(short));
    PTC_ALLOC(n->Ab[l], 9 * 256 * sizeof(short));
  }
  for (int l = 0; l <= nlayers; l++) PTC_ALLOC(n->act[l], fields_bytes(g, (size_t)max_batch * channels[l]));
  // act16[0] and act16[nlayers] hold the input and output of qcd_ptc_apply_prec in FP16
  for (int l = 0; l <= nlayers; l++)
    PTC_ALLOC(n->act16[l], (size_t)max_batch * channels[l] * spinor_elems(g) * sizeof(__half2));
  PTC_ALLOC(n->Gp, (size_t)16 * maxKp * std::max(n->mix_blocks * 4 * sizeof(float), kDwBlocks * sizeof(double)));
  size_t max_mk = 0;
  for (int l = 0; l < nlayers; l++) max_mk = std::max(max_mk, (size_t)n->L[l].M * n->L[l].K);
  PTC_ALLOC(n->dwp, (size_t)kDwSlices * max_mk * 4 * sizeof(double));
  PTC_ALLOC(n->partials, (size_t)max_batch * site_blocks(g) * 2 * sizeof(double));
  PTC_ALLOC(n->sums, (size_t)max_batch * 2 * sizeof(double));
#undef PTC_ALLOC
  hipStream_t st = (hipStream_t)stream;
  if (rc == QCD_OK) {
    // activations of padding sites are never written: clear once so they stay finite
    for (int l = 0; l <= nlayers; l++)
      (void)hipMemsetAsync(n->act[l], 0, fields_bytes(g, (size_t)max_batch * channels[l]), st);
    for (int l = 0; l <= nlayers; l++)
      (void)hipMemsetAsync(n->act16[l], 0, (size_t)max_batch * channels[l] * spinor_elems(g) * sizeof(__half2), st);
    (void)hipMemsetAsync(n->w, 0, n->nweights * sizeof(float2), st);
    (void)hipMemsetAsync(n->adam_m, 0, n->nweights * sizeof(float2), st);
    (void)hipMemsetAsync(n->adam_v, 0, n->nweights * sizeof(float2), st);
    prep_weights(n, st);
    if (hipStreamSynchronize(st) != hipSuccess) rc = pfail(QCD_ERR_HIP, "synchronise failed");
  }
  if (rc != QCD_OK) {
    qcd_ptc_free(n);
    return rc;
  }
  *out = n;
  return QCD_OK;
}

size_t qcd_ptc_num_weights(const qcd_ptc* n) { return n ? n->nweights : 0; }

qcd_status qcd_ptc_set_weights(qcd_ptc* n, const double* w_host, void* stream) {
  if (!n || !w_host) return pfail(QCD_ERR_ARG, "null argument");
  std::vector<float2> h(n->nweights);
  for (size_t i = 0; i < n->nweights; i++) h[i] = make_float2((float)w_host[2 * i], (float)w_host[2 * i + 1]);
  hipStream_t st = (hipStream_t)stream;
  PTC_TRY(hipMemcpyAsync(n->w, h.data(), n->nweights * sizeof(float2), hipMemcpyHostToDevice, st));
  PTC_TRY(hipMemsetAsync(n->adam_m, 0, n->nweights * sizeof(float2), st));
  PTC_TRY(hipMemsetAsync(n->adam_v, 0, n->nweights * sizeof(float2), st));
  n->adam_step = 0;
  prep_weights(n, st);
  PTC_LAUNCHED();
  PTC_TRY(hipStreamSynchronize(st));
  return QCD_OK;
}

qcd_status qcd_ptc_get_weights(const qcd_ptc* n, double* w_host, void* stream) {
  if (!n || !w_host) return pfail(QCD_ERR_ARG, "null argument");
  std::vector<float2> h(n->nweights);
  hipStream_t st = (hipStream_t)stream;
  PTC_TRY(hipMemcpyAsync(h.data(), n->w, n->nweights * sizeof(float2), hipMemcpyDeviceToHost, st));
  PTC_TRY(hipStreamSynchronize(st));
  for (size_t i = 0; i < n->nweights; i++) {
    w_host[2 * i] = h[i].x;
    w_host[2 * i + 1] = h[i].y;
  }
  return QCD_OK;
}

qcd_status qcd_ptc_apply(qcd_ptc* n, int nbatch, void* out_dev, const void* in_dev, void* stream) {
  qcd_status rc = check_batch(n, nbatch);
  if (rc) return rc;
  if (!out_dev || !in_dev) return pfail(QCD_ERR_ARG, "null vector");
  hipStream_t st = (hipStream_t)stream;
  launch_pack_spinor(n->g, kFP32, nbatch, n->act[0], (const double*)in_dev, 1.0, 0, nullptr, st);
  if ((rc = forward(n, nbatch, false, st))) return rc;
  launch_unpack_spinor(n->g, kFP32, nbatch, (double*)out_dev, n->act[n->nlayers], nullptr, 1.0, st);
  PTC_LAUNCHED();
  return QCD_OK;
}

qcd_status qcd_ptc_apply_prec(qcd_ptc* n, qcd_prec prec, int nbatch, void* out_dev, const void* in_dev,
                              void* stream) {
  if (prec == QCD_FP32) return qcd_ptc_apply(n, nbatch, out_dev, in_dev, stream);
  if (prec != QCD_FP16) return pfail(QCD_ERR_ARG, "the network applies in FP32 or FP16");
  qcd_status rc = check_batch(n, nbatch);
  if (rc) return rc;
  if (!out_dev || !in_dev) return pfail(QCD_ERR_ARG, "null vector");
  if (!n->gauge->U[kFP16]) return pfail(QCD_ERR_ARG, "the gauge handle holds no FP16 links");
  hipStream_t st = (hipStream_t)stream;
  launch_pack_spinor(n->g, kFP16, nbatch, n->act16[0], (const double*)in_dev, 1.0, 0, nullptr, st);
  ptc_apply_half(n, nbatch, n->act16[0], n->act16[n->nlayers], 1.0f, 0, nullptr, st);
  launch_unpack_spinor(n->g, kFP16, nbatch, (double*)out_dev, n->act16[n->nlayers], nullptr, 1.0, st);
  PTC_LAUNCHED();
  return QCD_OK;
}

qcd_status qcd_ptc_loss_grad(qcd_ptc* n, int nbatch, const void* r_dev, const void* e_dev, double* loss,
                             double* grad_host, void* stream) {
  qcd_status rc = check_batch(n, nbatch);
  if (rc) return rc;
  if (!r_dev || !e_dev) return pfail(QCD_ERR_ARG, "null vector");
  if ((rc = ensure_train(n))) return rc;
  hipStream_t st = (hipStream_t)stream;
  launch_pack_spinor(n->g, kFP32, nbatch, n->act[0], (const double*)r_dev, 1.0, 0, nullptr, st);
  launch_pack_spinor(n->g, kFP32, nbatch, n->target, (const double*)e_dev, 1.0, 0, nullptr, st);
  if ((rc = loss_grad(n, nbatch, loss, st))) return rc;
  if (grad_host) {
    std::vector<float2> h(n->nweights);
    PTC_TRY(hipMemcpyAsync(h.data(), n->grad, n->nweights * sizeof(float2), hipMemcpyDeviceToHost, st));
    PTC_TRY(hipStreamSynchronize(st));
    for (size_t i = 0; i < n->nweights; i++) {
      grad_host[2 * i] = h[i].x;
      grad_host[2 * i + 1] = h[i].y;
    }
  }
  return QCD_OK;
}

qcd_status qcd_ptc_train_step(qcd_ptc* n, int nbatch, const void* r_dev, const void* e_dev, double lr, double* loss,
                              void* stream) {
  qcd_status rc = qcd_ptc_loss_grad(n, nbatch, r_dev, e_dev, loss, nullptr, stream);
  if (rc) return rc;
  adam_step(n, lr, (hipStream_t)stream);
  PTC_LAUNCHED();
  return QCD_OK;
}

qcd_status qcd_ptc_loss_grad_residual(qcd_ptc* n, double kappa, int nbatch, const void* r_dev, double* loss,
                                      double* grad_host, void* stream) {
  qcd_status rc = check_batch(n, nbatch);
  if (rc) return rc;
  if (!r_dev) return pfail(QCD_ERR_ARG, "null vector");
  if (!(kappa > 0) || !std::isfinite(kappa)) return pfail(QCD_ERR_ARG, "kappa must be positive and finite");
  hipStream_t st = (hipStream_t)stream;
  launch_pack_spinor(n->g, kFP32, nbatch, n->act[0], (const double*)r_dev, 1.0, 0, nullptr, st);
  if ((rc = loss_grad_residual(n, kappa, nbatch, loss, st))) return rc;
  if (grad_host) {
    std::vector<float2> h(n->nweights);
    PTC_TRY(hipMemcpyAsync(h.data(), n->grad, n->nweights * sizeof(float2), hipMemcpyDeviceToHost, st));
    PTC_TRY(hipStreamSynchronize(st));
    for (size_t i = 0; i < n->nweights; i++) {
      grad_host[2 * i] = h[i].x;
      grad_host[2 * i + 1] = h[i].y;
    }
  }
  return QCD_OK;
}

qcd_status qcd_ptc_train_step_residual(qcd_ptc* n, double kappa, int nbatch, const void* r_dev, double lr,
                                       double* loss, void* stream) {
  qcd_status rc = qcd_ptc_loss_grad_residual(n, kappa, nbatch, r_dev, loss, nullptr, stream);
  if (rc) return rc;
  adam_step(n, lr, (hipStream_t)stream);
  PTC_LAUNCHED();
  return QCD_OK;
}

qcd_status qcd_ptc_set_mixing(qcd_ptc* n, qcd_prec prec, void* stream) {
  if (!n) return pfail(QCD_ERR_ARG, "null network handle");
  if (prec != QCD_BF16 && prec != QCD_FP32) return pfail(QCD_ERR_ARG, "the mixing runs in BF16 or FP32");
  const int want = prec == QCD_FP32;
  if (want == n->mix_fp32) return QCD_OK;
  hipStream_t st = (hipStream_t)stream;
  PTC_TRY(hipStreamSynchronize(st));  // no launch may still read the old buffers
  const size_t es = want ? sizeof(float) : sizeof(short);
  qcd_status rc = QCD_OK;
  for (int l = 0; l < n->nlayers && rc == QCD_OK; l++) rc = realloc_buf(n, &n->A[l], 16 * (size_t)n->L[l].Kp * es);
  if (rc) return rc;
  // what only the other mode uses (it is made again on that mode's next use)
  if (want) {
    for (auto& p : n->DOq) drop_buf(n, &p);
    n->quads_ready = false;
  } else {
    for (auto& p : n->X) drop_buf(n, &p);
    drop_buf(n, &n->DO);
    drop_buf(n, &n->DX);
    n->two_pass_ready = false;
  }
  n->mix_fp32 = want;
  prep_weights(n, st);
  PTC_LAUNCHED();
  PTC_TRY(hipStreamSynchronize(st));
  return QCD_OK;
}

qcd_status qcd_ptc_set_gauge(qcd_ptc* n, const qcd_gauge* gauge) {
  if (!n || !gauge) return pfail(QCD_ERR_ARG, "null argument");
  if (!gauge->U[kFP32]) return pfail(QCD_ERR_ARG, "the network needs the gauge handle's FP32 links");
  for (int mu = 0; mu < 4; mu++)
    if (gauge->dims[mu] != n->gauge->dims[mu]) return pfail(QCD_ERR_ARG, "lattice extents differ");
  n->gauge = gauge;
  return QCD_OK;
}

qcd_status qcd_ptc_init_neumann(qcd_ptc* n, double kappa, void* stream) {
  if (!n) return pfail(QCD_ERR_ARG, "null network handle");
  const int want[4] = {1, 2, 2, 1};
  if (n->nlayers != 3 || memcmp(n->channels, want, sizeof want) != 0)
    return pfail(QCD_ERR_UNSUPPORTED, "the Neumann form is defined for channels 1, 2, 2, 1");
  // Spin matrices of the hops of kappa H: path +mu carries kappa (1 - gamma_mu),
  // path -mu kappa (1 + gamma_mu), in the Dirac basis of the Wilson kernel
  // (gamma_1 as printed in Sec. 2; gamma_4 = diag(1, 1, -1, -1)).
  typedef std::complex<double> C;
  const C I(0, 1);
  C gam[4][4][4] = {};
  gam[0][0][3] = -I; gam[0][1][2] = -I; gam[0][2][1] = I; gam[0][3][0] = I;
  gam[1][0][3] = -1; gam[1][1][2] = 1;  gam[1][2][1] = 1; gam[1][3][0] = -1;
  gam[2][0][2] = -I; gam[2][1][3] = I;  gam[2][2][0] = I; gam[2][3][1] = -I;
  gam[3][0][0] = 1;  gam[3][1][1] = 1;  gam[3][2][2] = -1; gam[3][3][3] = -1;
  std::vector<double> w(2 * n->nweights, 0.0);
  // weight W[p][j][i][s'][s] of layer l
  auto put = [&](int l, int p, int j, int i, int sp, int sv, C v) {
    const PtcLayerDev& L = n->L[l];
    const size_t k = n->woff[l] + ((((size_t)p * L.cout + j) * L.cin + i) * 4 + sp) * 4 + sv;
    w[2 * k] += v.real();
    w[2 * k + 1] += v.imag();
  };
  auto ident = [&](int l, int j, int i) {
    for (int s = 0; s < 4; s++) put(l, 0, j, i, s, s, 1.0);
  };
  auto hop = [&](int l, int j, int i) {  // out_j += kappa H in_i
    for (int mu = 0; mu < 4; mu++)
      for (int sp = 0; sp < 4; sp++)
        for (int sv = 0; sv < 4; sv++) {
          const C d = sp == sv ? 1.0 : 0.0;
          put(l, 1 + 2 * mu, j, i, sp, sv, kappa * (d - gam[mu][sp][sv]));
          put(l, 2 + 2 * mu, j, i, sp, sv, kappa * (d + gam[mu][sp][sv]));
        }
  };
  // layer 0: (psi, kH psi); layer 1: (c0 + c1, kH (c0 + c1)); layer 2: c0 + kH c1
  // => M = (1 + kH)(1 + (kH)^2) = sum_{k <= 3} (kappa H)^k
  ident(0, 0, 0); hop(0, 1, 0);
  ident(1, 0, 0); ident(1, 0, 1); hop(1, 1, 0); hop(1, 1, 1);
  ident(2, 0, 0); hop(2, 0, 1);
  return qcd_ptc_set_weights(n, w.data(), stream);
}

}  // extern "C"
