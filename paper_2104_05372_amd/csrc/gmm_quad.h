// FP32 GMM units for D <= 32 that do only the products a triangular factor and a
// symmetric moment need. D8: D rounded up to a multiple of 8 (8, 16, 24, 32).
//
// Both are bound by the SIMDs' issue of matrix and vector work: a 16x16x4 FP32 product
// takes 32 cycles and, unlike the 16-bit ones, shares them with no vector instruction
// (4 cycles each), so what counts is the sum. Both cut the products to the triangle
// where 16x16 blocks of one component cannot: D8 (D8 + 4) / 128 products per 16 points
// and component in the forward (2.5, 9 for D8 = 16, 32; with blocks 4, 12), D8 (D8 + 3)
// / 32 per 4 points and 16 components in the reverse (9.5, 35; with blocks 16, 48).
// 512 mixtures, N to 50 000, D in {8, 16, 32}, K to 100 (6.8e8 point-component pairs):
// forward 3.4 ms (blocks, and the vector ALU for D <= 8: 4.57), of which products
// 2.45; reverse 3.8 ms (4.89), of which products 2.75, 16% of them for components that
// pad a group to 16.
#pragma once

#include "gmm_dev.h"

namespace dexk {

// fn(integral_constant D8)
template <typename F>
__host__ __device__ inline void with_d8(int D, F&& fn) {
  if (D <= 8)
    fn(std::integral_constant<int, 8>{});
  else if (D <= 16)
    fn(std::integral_constant<int, 16>{});
  else if (D <= 24)
    fn(std::integral_constant<int, 24>{});
  else
    fn(std::integral_constant<int, 32>{});
}

// ---------------------------------------------------------------------------
// Forward. Four components ("a quad") share the rows of a product: its 16 rows are
// rows 4r .. 4r+3 of the four factors, which are zero past column 4r+3, so row
// group r needs r + 1 of the D8/4 contraction steps. The lane that holds four
// rows of the result then holds them all from one component: squared norms need no
// exchange between lanes, and every lane goes on with a (component, point) of its
// own (a block of one component leaves each lane a quarter of a norm).
__host__ __device__ constexpr int quad_products(int D8) { return D8 / 4 * (D8 / 4 + 1) / 2; }
__host__ __device__ constexpr int quad_groups(int D8) { return (quad_products(D8) + 3) / 4; }
// A quad's record, in floats: the packed factors (product m's operand of lane n at
// (m / 4) 256 + 4 n + m % 4), -Q (mu - shift) [component][D8], kappa [4].
__host__ __device__ constexpr int quad_neg(int D8) { return quad_groups(D8) * 256; }
__host__ __device__ constexpr int quad_floats(int D8) { return quad_neg(D8) + 4 * D8 + 4; }

// Component k's part of its quad's record, and of the tangent record with TAN (dQ,
// exp(qd) dqd on its diagonal; -(dQ (mu - shift) + Q dmu); dkappa). The components that
// fill up the last quad get zero factors, kappa -inf and dkappa 0, so that they add
// nothing. 256 threads; load() issues every load (branch-free, at clamped addresses:
// N = 20000, D = 32, K = 50 prepared both records quad by quad, a load at a time, in 21
// us, this way in 6), store() may come after the block has found the shift.
template <int D8, bool TAN>
struct QuadPrep {
  static constexpr int NL = (D8 * D8 + 255) / 256;
  struct Src {
    const float *al, *mu, *qd, *l;
  };
  float lv[NL], dv[NL], mu, qd, al;
  float tlv[TAN ? NL : 1], tdv[TAN ? NL : 1], tmu, tqd, tal;

  DEX_DEV static void load_one(const Src& s, int D, size_t kc, float (&lv)[NL], float (&dv)[NL],
                               float& mu, float& qd, float& al) {
    const int t = threadIdx.x, L = D * (D - 1) / 2, tc = min(t % D8, D - 1);
    const float* lsrc = L > 0 ? s.l + kc * L : s.qd + kc * D;  // (D = 1: not used)
#pragma unroll
    for (int r = 0; r < NL; ++r) {
      const int e = t + 256 * r, a = e / D8, b = e % D8;
      lv[r] = lsrc[a < D && b < a ? a * (a - 1) / 2 + b : 0];
      dv[r] = s.qd[kc * D + min(a, D - 1)];
    }
    mu = s.mu[kc * D + tc];
    qd = s.qd[kc * D + tc];
    al = s.al[kc];
  }
  DEX_DEV void load(const Src& p, const Src& tp, int D, int K, int k) {
    const size_t kc = min(k, K - 1);
    load_one(p, D, kc, lv, dv, mu, qd, al);
    if constexpr (TAN) load_one(tp, D, kc, tlv, tdv, tmu, tqd, tal);
  }
  DEX_DEV void store(int D, int K, int k, const float* shift, float* rec, float* trec) {
    __shared__ float qs[D8][D8 + 1], ds[TAN ? D8 : 1][D8 + 1];
    __shared__ double mus[D8], dms[D8];
    const int t = threadIdx.x, j = k & 3;
    rec += (size_t)(k >> 2) * quad_floats(D8);
    trec += (size_t)(k >> 2) * quad_floats(D8);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NL; ++r) {
      const int e = t + 256 * r, a = e / D8, b = e % D8;
      const bool in = k < K && a < D && b <= a;
      const float ev = expf(dv[r]);
      if (e < D8 * D8) {
        qs[a][b] = !in ? 0.f : a == b ? ev : lv[r];
        if constexpr (TAN) ds[a][b] = !in ? 0.f : a == b ? ev * tdv[r] : tlv[r];
      }
    }
    const bool own = t < D8 && t < D && k < K;
    if (t < D8) {
      mus[t] = own ? (double)mu - (double)shift[t] : 0.0;
      if constexpr (TAN) dms[t] = own ? (double)tmu : 0.0;
    }
    // What every point of the component shares is summed in FP64 and rounded once: its
    // error would not average out over the points.
    const double s = wave_sum(own ? (double)qd : 0.0);
    if (t == 0) rec[quad_neg(D8) + 4 * D8 + j] = k < K ? (float)((double)al + s) : -INFINITY;
    if constexpr (TAN) {
      const double ts = wave_sum(own ? (double)tqd : 0.0);
      if (t == 0) trec[quad_neg(D8) + 4 * D8 + j] = k < K ? (float)((double)tal + ts) : 0.f;
    }
    __syncthreads();
    // the quad's operands of lanes 16 g + 4 j + i, rows 4 r + i, columns 4 ch + g
    for (int e = t; e < quad_groups(D8) * 64; e += 256) {
      const int m = e / 64 * 4 + e % 4, n = e / 4 % 16, g = n / 4, i = n % 4;
      const int o = e / 64 * 256 + 4 * (16 * g + 4 * j + i) + m % 4;
      int r = (int)((sqrtf(8.f * (float)m + 1.f) - 1.f) * 0.5f);  // (m < 36: exact after this)
      if ((r + 1) * (r + 2) / 2 <= m) ++r;
      if (r * (r + 1) / 2 > m) --r;
      const int ch = m - r * (r + 1) / 2;
      const bool in = m < quad_products(D8);
      const int row = in ? 4 * r + i : 0, col = in ? 4 * ch + g : 0;
      rec[o] = in ? qs[row][col] : 0.f;
      if constexpr (TAN) trec[o] = in ? ds[row][col] : 0.f;
    }
    if (t < D8) {
      double c = 0.0, tc = 0.0;
      for (int b = 0; b <= t; ++b) {
        c = fma((double)qs[t][b], mus[b], c);
        if constexpr (TAN)
          tc = fma((double)ds[t][b], mus[b], fma((double)qs[t][b], dms[b], tc));
      }
      rec[quad_neg(D8) + j * D8 + t] = (float)-c;
      if constexpr (TAN) trec[quad_neg(D8) + j * D8 + t] = (float)-tc;
    }
  }
};

// One block: 64 CB points from the tile's first, quads qa .. qb - 1; wave v takes 16 CB
// points. beta has rows for whole quads (the last may hold values nobody reads, as do
// points N <= p < Npad). Lane 16 g + c holds points CB c .. CB c + CB - 1
// of the wave's and, quad by quad, component 4q + g. A maximum starts at the lowest
// finite number, so that -inf log-weights (a component with alpha = -inf) leave the
// sums as they are. The records go through LDS, QB quads at a time (the four waves
// read the same), so a wave holds few of the operands and four fit a SIMD: 3.4 ms; with
// the operands of two quads in registers (two waves a SIMD) 3.9 ms.
template <int D8>
__host__ __device__ constexpr int quad_batch() { return D8 == 8 ? 8 : D8 == 16 ? 3 : 1; }
constexpr int kQuadLds = 5016;  // floats: the largest 2 quad_batch() quad_floats()

template <int D8, int CB>
DEX_DEV void fwd_quads(const float* __restrict__ x, const float* __restrict__ shift, int N, int D,
                       int Npad, int tile0, const float* __restrict__ rec, int qa, int qb,
                       float* __restrict__ beta, float2* __restrict__ ml, float* lds) {
  constexpr int R = D8 / 4, NG = quad_groups(D8), QB = quad_batch<D8>(), RS = quad_floats(D8);
  constexpr int NL = (QB * RS / 4 + 255) / 256;  // 16-byte loads per thread and batch
  static_assert(2 * QB * RS <= kQuadLds && RS % 4 == 0, "LDS");
  typedef float VC __attribute__((ext_vector_type(CB)));
  int t = threadIdx.x;
  // (opaque: what follows from it is not kept in registers from one item to the next)
  asm volatile("" : "+v"(t));
  const int lane = t & 63, g = lane >> 4, c = lane & 15;
  const int p0 = tile0 + (t >> 6) * 16 * CB;
  f32x4 sv[NL];
  auto fetch = [&](int q) {
    const int last = min(QB, qb - q) * (RS / 4) - 1;
    const f32x4* src = reinterpret_cast<const f32x4*>(rec + (size_t)q * RS);
#pragma unroll
    for (int i = 0; i < NL; ++i) sv[i] = src[min(t + 256 * i, last)];
  };
  auto stage = [&](float* b) {
#pragma unroll
    for (int i = 0; i < NL; ++i)
      if (t + 256 * i < QB * RS / 4) reinterpret_cast<f32x4*>(b)[t + 256 * i] = sv[i];
  };
  fetch(qa);
  float xb[CB][R];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int p = p0 + CB * c + cb;
#pragma unroll
    for (int ch = 0; ch < R; ++ch) xb[cb][ch] = x[(size_t)min(p, N - 1) * D + min(4 * ch + g, D - 1)];
  }
#pragma unroll
  for (int ch = 0; ch < R; ++ch) {
    const float sh = shift[4 * ch + g];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
      xb[cb][ch] = p0 + CB * c + cb < N && 4 * ch + g < D ? xb[cb][ch] - sh : 0.f;
  }
  float m[CB], ls[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    m[cb] = -3.402823466e38f;
    ls[cb] = 0.f;
  }
  auto compute = [&](int q, const float* o) {
    const f32x4* oq = reinterpret_cast<const f32x4*>(o) + lane;
    const float* on = o + quad_neg(D8) + g * D8;
    float s[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) s[cb] = 0.f;
    // operands one group of four products ahead, offsets one row group ahead; the
    // squares of a row group wait until the next one's first products are issued
    f32x4 qv[2], nv[2], acc[2][CB];
    qv[0] = oq[0];
    nv[0] = *reinterpret_cast<const f32x4*>(on);
    const float kap = o[quad_neg(D8) + 4 * D8 + g];
    auto squares = [&](int r) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) s[cb] = fmaf(acc[r & 1][cb][i], acc[r & 1][cb][i], s[cb]);
    };
    int n = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r + 1 < R) nv[(r + 1) & 1] = *reinterpret_cast<const f32x4*>(on + 4 * (r + 1));
#pragma unroll
      for (int ch = 0; ch <= r; ++ch, ++n) {
        if (n % 4 == 0 && n / 4 + 1 < NG) {
          qv[(n / 4 + 1) & 1] = oq[(n / 4 + 1) * 64];
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
          acc[r & 1][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(
              qv[(n / 4) & 1][n % 4], xb[cb][ch], ch == 0 ? nv[r & 1] : acc[r & 1][cb], 0, 0, 0);
        if (ch == 0 && r > 0) squares(r - 1);
        if (n % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
    squares(R - 1);
    VC b;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) b[cb] = kap - 0.5f * s[cb];
    // streams out: read again only by the reverse pass
    __builtin_nontemporal_store(b, reinterpret_cast<VC*>(beta + (size_t)(4 * q + g) * Npad + p0 + CB * c));
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const float d = b[cb] - m[cb];
      const float e = __expf(-fabsf(d));
      ls[cb] = d > 0.f ? fmaf(ls[cb], e, 1.f) : ls[cb] + e;
      m[cb] = fmaxf(m[cb], b[cb]);
    }
  };
  __syncthreads();  // (the item before has left the LDS)
  stage(lds);
  if (qa + QB < qb) fetch(qa + QB);
  for (int q0 = qa, buf = 0; q0 < qb; q0 += QB, buf ^= 1) {
    __syncthreads();
    if (q0 + QB < qb) {
      stage(lds + (buf ^ 1) * QB * RS);
      if (q0 + 2 * QB < qb) fetch(q0 + 2 * QB);
    }
    for (int j = 0; j < QB && q0 + j < qb; ++j) compute(q0 + j, lds + (buf * QB + j) * RS);
  }
  // the four lane groups' sums of a point
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    float mx = fmaxf(m[cb], xor_lane(m[cb], 16));
    mx = fmaxf(mx, xor_lane(mx, 32));
    float v = ls[cb] * __expf(m[cb] - mx);
    v += xor_lane(v, 16);
    v += xor_lane(v, 32);
    if (g == 0) ml[p0 + CB * c + cb] = make_float2(mx, v);
  }
}

// ---------------------------------------------------------------------------
// Forward mode: y and ty = dQ (x - shift) - (dQ (mu - shift) + Q dmu) of four components
// at a time, each row group's products in turn; the derivative of a log-density is
// dkappa - y . ty.
template <int D8>
__host__ __device__ constexpr int quad_tan_batch() { return D8 == 8 ? 4 : D8 == 16 ? 2 : 1; }
constexpr int kQuadTanLds = 9744;  // floats: the largest 4 quad_tan_batch() quad_floats()

// One block: as fwd_quads; the lane's FP64 sum of exp(beta - f) dbeta over its points
// and components.
template <int D8, int CB>
DEX_DEV double jvp_quads(const float* __restrict__ x, const float* __restrict__ shift, int N, int D,
                         int tile0, const float* __restrict__ rec, const float* __restrict__ trec,
                         int qa, int qb, const float* __restrict__ f, float* lds) {
  constexpr int R = D8 / 4, NG = quad_groups(D8), QB = quad_tan_batch<D8>(), RS = quad_floats(D8);
  constexpr int NL = (QB * RS / 4 + 255) / 256;
  static_assert(4 * QB * RS <= kQuadTanLds && RS % 4 == 0, "LDS");
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));  // (as in fwd_quads)
  const int lane = t & 63, g = lane >> 4, c = lane & 15;
  const int p0 = tile0 + (t >> 6) * 16 * CB;
  f32x4 sv[2][NL];
  auto fetch = [&](int q) {
    const int last = min(QB, qb - q) * (RS / 4) - 1;
    const f32x4* a = reinterpret_cast<const f32x4*>(rec + (size_t)q * RS);
    const f32x4* b = reinterpret_cast<const f32x4*>(trec + (size_t)q * RS);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      sv[0][i] = a[min(t + 256 * i, last)];
      sv[1][i] = b[min(t + 256 * i, last)];
    }
  };
  auto stage = [&](float* b) {
#pragma unroll
    for (int i = 0; i < NL; ++i)
      if (t + 256 * i < QB * RS / 4) {
        reinterpret_cast<f32x4*>(b)[t + 256 * i] = sv[0][i];
        reinterpret_cast<f32x4*>(b + QB * RS)[t + 256 * i] = sv[1][i];
      }
  };
  fetch(qa);
  float xb[CB][R], fp[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    const int p = p0 + CB * c + cb;
    fp[cb] = f[min(p, N - 1)];
#pragma unroll
    for (int ch = 0; ch < R; ++ch) xb[cb][ch] = x[(size_t)min(p, N - 1) * D + min(4 * ch + g, D - 1)];
  }
#pragma unroll
  for (int ch = 0; ch < R; ++ch) {
    const float sh = shift[4 * ch + g];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
      xb[cb][ch] = p0 + CB * c + cb < N && 4 * ch + g < D ? xb[cb][ch] - sh : 0.f;
  }
  double sum = 0.0;
  auto compute = [&](const float* o, const float* to) {
    const f32x4 *oq = reinterpret_cast<const f32x4*>(o) + lane,
                *tq = reinterpret_cast<const f32x4*>(to) + lane;
    const int no = quad_neg(D8) + g * D8;
    float s[CB], sd[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) s[cb] = sd[cb] = 0.f;
    f32x4 qv[2], tv[2], nv[2], ntv[2], acc[2][CB], tacc[2][CB];
    qv[0] = oq[0];
    tv[0] = tq[0];
    nv[0] = *reinterpret_cast<const f32x4*>(o + no);
    ntv[0] = *reinterpret_cast<const f32x4*>(to + no);
    const float kap = o[quad_neg(D8) + 4 * D8 + g], dkap = to[quad_neg(D8) + 4 * D8 + g];
    auto squares = [&](int r) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          s[cb] = fmaf(acc[r & 1][cb][i], acc[r & 1][cb][i], s[cb]);
          sd[cb] = fmaf(acc[r & 1][cb][i], tacc[r & 1][cb][i], sd[cb]);
        }
    };
    int n = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r + 1 < R) {
        nv[(r + 1) & 1] = *reinterpret_cast<const f32x4*>(o + no + 4 * (r + 1));
        ntv[(r + 1) & 1] = *reinterpret_cast<const f32x4*>(to + no + 4 * (r + 1));
      }
#pragma unroll
      for (int ch = 0; ch <= r; ++ch, ++n) {
        if (n % 4 == 0 && n / 4 + 1 < NG) {
          qv[(n / 4 + 1) & 1] = oq[(n / 4 + 1) * 64];
          tv[(n / 4 + 1) & 1] = tq[(n / 4 + 1) * 64];
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          acc[r & 1][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(
              qv[(n / 4) & 1][n % 4], xb[cb][ch], ch == 0 ? nv[r & 1] : acc[r & 1][cb], 0, 0, 0);
          tacc[r & 1][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(
              tv[(n / 4) & 1][n % 4], xb[cb][ch], ch == 0 ? ntv[r & 1] : tacc[r & 1][cb], 0, 0, 0);
        }
        if (ch == 0 && r > 0) squares(r - 1);
        if (n % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
    squares(R - 1);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const float v = expf(kap - 0.5f * s[cb] - fp[cb]) * (dkap - sd[cb]);
      if (p0 + CB * c + cb < N) sum += (double)v;
    }
  };
  __syncthreads();  // (the tile before has left the LDS)
  stage(lds);
  if (qa + QB < qb) fetch(qa + QB);
  for (int q0 = qa, buf = 0; q0 < qb; q0 += QB, buf ^= 1) {
    __syncthreads();
    float* cur = lds + buf * 2 * QB * RS;
    if (q0 + QB < qb) {
      stage(lds + (buf ^ 1) * 2 * QB * RS);
      if (q0 + 2 * QB < qb) fetch(q0 + 2 * QB);
    }
    for (int j = 0; j < QB && q0 + j < qb; ++j) compute(cur + j * RS, cur + (QB + j) * RS);
  }
  return sum;
}

// ---------------------------------------------------------------------------
// Reverse. With phi(x) the D8 (D8 + 1) / 2 products x_a x_b and the D8 coordinates
// x_a, the moments of 16 components are one product W^T Phi over the points:
// rows the components' weights, columns 16 features, which no component forms
// again. In MomPack's circulant order the second factor of a feature (a, d) is
// coordinate row a + d of a table whose first D8/2 rows are repeated behind the
// rest, so its address is the lane's own plus a constant, and the first factor
// stays in registers.
constexpr int kMomPackLds = 10960;  // floats: the largest of 2 BUF and RED

// One block: components k0 .. k0 + 15 over the points [pbeg, pend) (multiples of
// 256); slots part[k * pstride]. The cotangent is left to the assembly. Waves split
// the tiles (NH) and the points (NPW), so that the sums leave three waves a SIMD
// room (two, with twice the tiles each: 4.6 ms for 3.85); each weight is formed by one wave and, where several need it, handed over in
// LDS with the coordinates.
template <int D8>
DEX_DEV void mom_pack_unit(const float* __restrict__ x, const float* __restrict__ shift, int N,
                           int D, int Npad, int K, int k0, int pbeg, int pend,
                           const float* __restrict__ beta, const float* __restrict__ f,
                           float* __restrict__ part, size_t pstride, float* lds) {
  using S = MomPack<D8>;
  static_assert(2 * S::BUF <= kMomPackLds && S::RED <= kMomPackLds, "LDS");
  constexpr int ST = S::ST, TQ = S::TH - S::TE, WOFF = S::ROWS * ST;
  int t = threadIdx.x;
  // (opaque: what follows from it is not kept in registers from one item to the next)
  asm volatile("" : "+v"(t));
  const int lane = t & 63, g = lane >> 4, c = lane & 15, wv = t >> 6;
  const int T0 = wv % S::NH * S::TH, ps = wv / S::NH;
  // LDS places of the lane's first factors, of the second ones of its wave's first
  // tiles, and of both factors of the wave's last TE tiles; they change buffers with
  // the tile, so that a read's address is one of them and a constant
  typedef const __attribute__((address_space(3))) float* Lds;
  typedef const __attribute__((address_space(3))) f32x4* Lds4;
  Lds ra[S::P], rb[S::P], ea[S::TE], eb[S::TE];
  Lds wl = (Lds)lds + WOFF + ps * 256 + 4 * lane;  // and of the weights
  const Lds own = (Lds)lds + 16 * ps + 4 * g;
#pragma unroll
  for (int j = 0; j < S::P; ++j) {
    const int e = 16 * (T0 + j) + c;
    ra[j] = own + e % D8 * ST;
    rb[j] = own + (e % D8 + e / D8) * ST;
  }
#pragma unroll
  for (int j = 0; j < S::TE; ++j) {
    const int e = 16 * (T0 + TQ + j) + c, e2 = e - 16 * S::NQ;
    const int one = 3 * D8 / 2, zero = one + 1;
    int a = e % D8, b = e % D8 + e / D8;
    if (e2 >= 0) {
      const int q = e2 - D8 / 2;
      a = q < 0 ? e2 : q < D8 ? q : zero;
      b = q < 0 ? e2 + D8 / 2 : q < D8 ? one : zero;
    }
    ea[j] = own + a * ST;
    eb[j] = own + b * ST;
  }
  // staged element r of the thread: a point of the tile and a coordinate (the same
  // one every time if D8 divides 256)
  constexpr bool kSame = 256 % D8 == 0;
  const unsigned tp = (unsigned)t / D8, td = (unsigned)t % D8;
  auto point = [&](int r) { return kSame ? tp + r * (256 / D8) : ((unsigned)t + 256 * r) / D8; };
  auto coord = [&](int r) { return kSame ? td : ((unsigned)t + 256 * r) % D8; };
  constexpr int NSV = kSame ? 1 : S::NL;
  float xv[S::NL], sv[NSV];
#pragma unroll
  for (int r = 0; r < NSV; ++r) sv[r] = shift[coord(r)];
  // the wave's own weights: 16-point steps wv, wv + 4, ... of a tile (with NH = 1,
  // those it multiplies)
  f32x4 bt[S::SW], ft[S::SW], w[S::SW];
  const float* brow = beta + (size_t)min(k0 + c, K - 1) * Npad + 16 * wv + 4 * g;
  // A tile inside the data: lane offsets that stay the same, scalar steps. The last
  // tile, and D < D8: every address clamped, what it should not have read zeroed.
  const unsigned xlane = 4 * (tp * D + td), flane = 4 * (16 * wv + 4 * g);
  auto fetch = [&](int t0) {
#pragma unroll
    for (int s = 0; s < S::SW; ++s)
      bt[s] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(brow + t0 + 64 * s));
    if (kSame && D == D8 && t0 + S::TP <= N) {
      const char* xt = (const char*)(x + (size_t)t0 * D8);
      const char* ft0 = (const char*)(f + t0);
#pragma unroll
      for (int r = 0; r < S::NL; ++r) xv[r] = *(const float*)(xt + 1024 * r + xlane);
#pragma unroll
      for (int s = 0; s < S::SW; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) ft[s][i] = *(const float*)(ft0 + 256 * s + 4 * i + flane);
    } else {
      const int tb = min(t0, N - 1);
      const unsigned last = N - 1 - tb;
      const float* xt = x + (size_t)tb * D;
      const float* fp = f + tb;
#pragma unroll
      for (int r = 0; r < S::NL; ++r)
        xv[r] = xt[min(point(r), last) * (unsigned)D + min(coord(r), (unsigned)D - 1)];
#pragma unroll
      for (int s = 0; s < S::SW; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          ft[s][i] = fp[min((unsigned)(16 * wv + 64 * s + 4 * g + i), last)];
    }
  };
  float wtot = 0.f;
  auto stage = [&](int t0, float* b) {
#pragma unroll
    for (int r = 0; r < S::NL; ++r) xv[r] -= sv[kSame ? 0 : r];
#pragma unroll
    for (int s = 0; s < S::SW; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) w[s][i] = __expf(bt[s][i] - ft[s][i]);
    if (D < D8 || t0 + S::TP > N) {
      int n = N;
      asm volatile("" : "+s"(n));  // (a branch, not selects in every tile)
#pragma unroll
      for (int r = 0; r < S::NL; ++r)
        if ((int)(t0 + point(r)) >= n || (int)coord(r) >= D) xv[r] = 0.f;
#pragma unroll
      for (int s = 0; s < S::SW; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (t0 + 16 * wv + 64 * s + 4 * g + i >= n) w[s][i] = 0.f;
    }
#pragma unroll
    for (int r = 0; r < S::NL; ++r) {
      float* o = b + coord(r) * ST + point(r);
      o[0] = xv[r];
      if (coord(r) < D8 / 2) o[D8 * ST] = xv[r];
    }
    float ws = 0.f;
#pragma unroll
    for (int s = 0; s < S::SW; ++s) {
#pragma unroll
      for (int i = 0; i < 4; ++i) ws += w[s][i];
      if (S::NH > 1) *reinterpret_cast<f32x4*>(b + WOFF + (wv + 4 * s) * 256 + 4 * lane) = w[s];
    }
    wtot += ws;
  };
  __syncthreads();  // (the item before has left the LDS)
  for (int e = t; e < 2 * S::TP; e += 256) {
    float* b = lds + (e < S::TP ? 0 : S::BUF);
    b[(S::ROWS - 2) * ST + e % S::TP] = 1.f;
    b[(S::ROWS - 1) * ST + e % S::TP] = 0.f;
  }
  // The products of 256 of a wave's points go into sums of their own, which are then
  // added to the totals: no FP32 sum runs through more than 64 products and one
  // addition per 256 points.
  f32x4 tot[S::TH], in[S::TH];
#pragma unroll
  for (int i = 0; i < S::TH; ++i) tot[i] = in[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto fold = [&] {
#pragma unroll
    for (int i = 0; i < S::TH; ++i) {
      tot[i] += in[i];
      in[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  fetch(pbeg);
  stage(pbeg, lds);
  if (pbeg + S::TP < pend) fetch(pbeg + S::TP);
  int buf = 0;
  for (int s0 = pbeg; s0 < pend; s0 += 256 * S::NPW, fold())
    for (int t0 = s0; t0 < min(s0 + 256 * S::NPW, pend); t0 += S::TP, buf ^= 1) {
      __syncthreads();
      auto next = [&] {
        if (t0 + S::TP < pend) {
          stage(t0 + S::TP, lds + (buf ^ 1) * S::BUF);
          if (t0 + 2 * S::TP < pend) fetch(t0 + 2 * S::TP);
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      if (S::NH > 1) next();
#pragma unroll
      for (int s = 0; s < S::SPT; ++s) {
        constexpr int SS = 16 * S::NPW;  // points from one of the wave's steps to the next
        f32x4 wc;
        if constexpr (S::NH > 1)
          wc = *(Lds4)(wl + 16 * SS * s);
        else
          wc = w[s];
        f32x4 xa[S::P];
#pragma unroll
        for (int j = 0; j < S::P; ++j) xa[j] = *(Lds4)(ra[j] + SS * s);
        // the factors of a tile are read while the one before it is multiplied (and no
        // earlier: the registers)
        f32x4 ph[2], pa[2];
        auto read = [&](int i) {
          if (i < TQ) {
            ph[i % 2] =
                *(Lds4)(rb[i % S::P] + (i / S::P * S::M * ST + SS * s));
          } else if (i < S::TH) {
            pa[i % 2] = *(Lds4)(ea[i < TQ ? 0 : i - TQ] + SS * s);
            ph[i % 2] = *(Lds4)(eb[i < TQ ? 0 : i - TQ] + SS * s);
          }
        };
        read(0);
#pragma unroll
        for (int i = 0; i < S::TH; ++i) {
          read(i + 1);
          __builtin_amdgcn_sched_barrier(0);
          const f32x4 v = (i < TQ ? xa[i % S::P] : pa[i % 2]) * ph[i % 2];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            in[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(wc[j], v[j], in[i], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (S::NH == 1) next();  // (replaces the weights)
      const int turn = buf ? -S::BUF : S::BUF;
#pragma unroll
      for (int j = 0; j < S::P; ++j) {
        ra[j] += turn;
        rb[j] += turn;
      }
#pragma unroll
      for (int j = 0; j < S::TE; ++j) {
        ea[j] += turn;
        eb[j] += turn;
      }
      wl += turn;
    }
  wtot += xor_lane(wtot, 16);
  wtot += xor_lane(wtot, 32);
  // the waves that share the points, one after the other
  float* wred = lds + S::TH * S::NH * 256;
  f32x4* red = reinterpret_cast<f32x4*>(lds) + T0 * 64 + lane;
  __syncthreads();
  if (lane < 16) wred[16 * wv + lane] = wtot;
  for (int w = 0; w < S::NPW; ++w) {
    if (w == ps) {
      if (w > 0) {
#pragma unroll
        for (int i = 0; i < S::TH; ++i) tot[i] += red[i * 64];
      }
      if (w + 1 < S::NPW) {
#pragma unroll
        for (int i = 0; i < S::TH; ++i) red[i * 64] = tot[i];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int k = k0 + 4 * g + j;
          if (k < K) {
#pragma unroll
            for (int i = 0; i < S::TH; ++i)
              part[(size_t)k * pstride + 16 * (T0 + i) + c] = tot[i][j];
          }
        }
      }
    }
    __syncthreads();
  }
  if (t < 16 && k0 + t < K)
    part[(size_t)(k0 + t) * pstride + 16 * S::TH * S::NH] =
        (wred[t] + wred[16 + t]) + (wred[32 + t] + wred[48 + t]);
}

}  // namespace dexk
