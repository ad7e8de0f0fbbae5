// GMM log-likelihood in FP64 (one instance): forward and reverse on the FP64
// matrix cores (16x16x4 products; the forward at D <= 4 on the vector ALU).
//
// Forward: y = Q_k (x - mu_k) for 64 points at a time, Q_k's lower-triangular
// chunks as the A operand and x - mu_k, formed per component, as B. Reverse:
// the weighted second moments S_k = sum_i w_ik r_ik r_ik^T (r = x - mu_k), the
// first moments u_k and the weight sums A_k, from which M_k = Q_k S_k and
// b_k = Q_k u_k; so no y is formed again and the per-point work is one product
// per four points and 16x16 block.
//
// The arithmetic is small (N = 20011, D = 16, K = 25: 0.3 GFLOP, 4 us at the
// FP64 peak); what costs is latency, so the work is cut to fill the chip: a wave
// takes 64 points and a share of the components (forward, shares merged in LDS)
// or 64-point tiles of one component (reverse, waves summed in LDS), and a
// problem that fits one block is finished in the same launch.
// Measured (kernel times, against one thread per point and 64 of a block's 256
// threads forming y again in the reverse): N = 20011, D = 16, K = 25: forward 20 us
// and the objective's sum 4 us (128 + 5), reverse 16 + 7 us (139 + 20); N = 1000,
// D = 2, K = 5: forward 9 us (6 + 4), reverse 7 us (6 + 16).
//
// Lane layout of the 16x16x4 FP64 product (lane 16 g + c): A holds row c and
// contraction index g, B column c and contraction index g, the result rows
// g + 4 i (register i) of column c.
#include <algorithm>

#include "gmm_host.h"
#include "internal.h"

namespace dexk {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// ---- FP64 exchanges ----------------------------------------------------------
struct DPair {
  double first, second;  // value at the lower / upper lane of the pair
};
DEX_DEV double join(uint32_t lo, uint32_t hi) {
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
DEX_DEV DPair swap32(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return {join(lo[0], hi[0]), join(lo[1], hi[1])};
}
DEX_DEV DPair swap16(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return {join(lo[0], hi[0]), join(lo[1], hi[1])};
}
DEX_DEV double sum_groups(double v) {  // over the four lane groups
  DPair p = swap32(v, v);
  p = swap16(p.first + p.second, p.first + p.second);
  return p.first + p.second;
}
DEX_DEV double lane_value(double v, int lane) {
  return join(__builtin_amdgcn_readlane(__double2loint(v), lane),
              __builtin_amdgcn_readlane(__double2hiint(v), lane));
}

// One update of a running log-sum-exp (m, s). m starts at the lowest finite number, not
// at -inf: a wave's first component may have beta = -inf (alpha = -inf), and -inf - -inf
// would make its sum NaN.
constexpr double kLowest = -1.7976931348623157e308;
DEX_DEV void lse_add(double& m, double& s, double b) {
  const double d = b - m;
  const double e = exp(-fabs(d));
  s = d > 0 ? s * e + 1.0 : s + e;
  m = fmax(m, b);
}

// ---- forward -------------------------------------------------------------------
// Most waves per block by padded dimension: the operands of larger D need more
// registers than a wave of a 1024-thread block has (128).
constexpr int f64_fwd_waves(int DP) { return DP == 4 ? 16 : 4; }
constexpr int f64_bwd_waves(int DP) { return DP <= 16 ? 16 : DP == 32 ? 8 : 4; }

// Block: blockDim / 64 / KS tiles of 64 points, each shared by KS waves that
// take every KS-th component. The components' operands of the next turn are
// loaded while the current ones are used. gridDim.x == 1: F is finished here.
template <int DP>
__global__ void __launch_bounds__(64 * f64_fwd_waves(DP)) k_f64_fwd(
    const double* __restrict__ alphas, const double* __restrict__ means,
    const double* __restrict__ qd, const double* __restrict__ l, const double* __restrict__ x, int N,
    int D, int K, int KS, double* __restrict__ beta, double* __restrict__ f,
    double* __restrict__ fpart, double* __restrict__ F) {
  __shared__ double ms[f64_fwd_waves(DP)][64], ss[f64_fwd_waves(DP)][64];
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tt = wv / KS, ks = wv - tt * KS, TT = (int)(blockDim.x >> 6) / KS;
  const int p0 = (int)(blockIdx.x * TT + tt) * 64, p = p0 + lane;
  const int64_t L = (int64_t)D * (D - 1) / 2;
  // (one block) logsumexp of alpha, by the last wave while the others begin
  __shared__ double lse_alpha;
  if (gridDim.x == 1 && wv == (int)(blockDim.x >> 6) - 1) {
    double am = -INFINITY, az = 0;
    for (int j = lane; j < K; j += 64) am = fmax(am, alphas[j]);
    am = wave_reduce(am, [](double a, double b) { return fmax(a, b); });
    for (int j = lane; j < K; j += 64) az += exp(alphas[j] - am);
    az = wave_sum(az);
    if (lane == 0) lse_alpha = am + log(az);
  }
  double m = kLowest, s = 0;
  if (p0 < N) {
    if constexpr (DP == 4) {
      double xr[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) xr[b] = b < D ? x[(size_t)min(p, N - 1) * D + b] : 0.0;
      // the operands of sixteen components at a time, read once: lane 4 j + a holds
      // component j's mean and diagonal entry a, kappa, and the lower entries a
      // and 4 + a; a component's are read back as wave-wide values
      const int la = lane & 3, nl = (int)L;
      double mul = 0, ed = 0, kapl = 0, l0 = 0, l1 = 0;
      for (int k = ks, n = 0; k < K; k += KS, ++n) {
        const int j4 = 4 * (n & 15);
        if (j4 == 0) {
          const int kk = min(k + (lane >> 2) * KS, K - 1);
          const double qv = qd[(size_t)kk * D + min(la, D - 1)];
          mul = means[(size_t)kk * D + min(la, D - 1)];
          kapl = alphas[kk];
          if (nl) {
            l0 = l[kk * L + min(la, nl - 1)];
            l1 = l[kk * L + min(la + 4, nl - 1)];
          }
          double sq = la < D ? qv : 0.0;
          sq += butterfly<1>(sq);
          kapl += sq + butterfly<2>(sq);
          ed = exp(qv);
        }
        double r[4], sq = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) r[b] = b < D ? xr[b] - lane_value(mul, j4 + b) : 0.0;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          if (a < D) {
            double y = lane_value(ed, j4 + a) * r[a];
#pragma unroll
            for (int b = 0; b < a; ++b) {
              const int e = a * (a - 1) / 2 + b;
              y += (e < 4 ? lane_value(l0, j4 + e) : lane_value(l1, j4 + e - 4)) * r[b];
            }
            sq += y * y;
          }
        }
        const double bv = lane_value(kapl, j4) - 0.5 * sq;
        if (p < N) beta[(size_t)k * N + p] = bv;
        lse_add(m, s, bv);
      }
    } else {
      // NCHR: chunks of row block rb (DP = 8: the two that hold columns)
      constexpr int NRB = (DP + 15) / 16, NCH = DP / 4, NQ = DP == 8 ? 2 : 2 * NRB * (NRB + 1);
      auto NCHR = [](int rb) { return 4 * (rb + 1) < NCH ? 4 * (rb + 1) : NCH; };
      double xb[4][NCH];
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
          const int col = 4 * ch + g;
          const double v = x[(size_t)min(p0 + 16 * t + c, N - 1) * D + min(col, D - 1)];
          xb[t][ch] = col < D ? v : 0.0;
        }
      struct Ops {
        double q[NQ], mu[NCH], qdr[NRB], al;
      };
      auto load = [&](int k, Ops& o) {
        int n = 0;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
          const int row = 16 * rb + c;
          o.qdr[rb] = qd[(size_t)k * D + min(row, D - 1)];
#pragma unroll
          for (int ch = 0; ch < NCHR(rb); ++ch) {
            const int col = 4 * ch + g;
            const bool in = row < D && col < row;
            o.q[n++] = l[k * L + (in ? row * (row - 1) / 2 + col : 0)];
          }
        }
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) o.mu[ch] = means[(size_t)k * D + min(4 * ch + g, D - 1)];
        o.al = alphas[k];
      };
      auto compute = [&](int k, const Ops& o) {
        double sq[4] = {0, 0, 0, 0}, sqd = 0;
        int n = 0;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
          const int row = 16 * rb + c;
          const bool rin = row < D;
          sqd += rin ? o.qdr[rb] : 0.0;
          const double ed = exp(o.qdr[rb]);
          f64x4 acc[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
          for (int ch = 0; ch < NCHR(rb); ++ch) {
            const int col = 4 * ch + g;
            double q = o.q[n++];
            if (4 * ch >= 16 * rb)  // the chunk meets the diagonal
              q = col < row ? q : col == row ? ed : 0.0;
            q = rin ? q : 0.0;
            const double mu = col < D ? o.mu[ch] : 0.0;
#pragma unroll
            for (int t = 0; t < 4; ++t)
              acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(q, xb[t][ch] - mu, acc[t], 0, 0, 0);
          }
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) sq[t] += acc[t][i] * acc[t][i];
        }
        // sum of qd over the 16 lanes of a group (every group holds the same)
        sqd += butterfly<1>(sqd);
        sqd += butterfly<2>(sqd);
        sqd += butterfly<4>(sqd);
        sqd += butterfly<8>(sqd);
        // tile t's norms summed over the lane groups; group t keeps them: lane
        // 16 t + c holds point 16 t + c
        const DPair a = swap32(sq[0], sq[2]), b = swap32(sq[1], sq[3]);
        const DPair r = swap16(a.first + a.second, b.first + b.second);
        const double bv = o.al + sqd - 0.5 * (r.first + r.second);
        if (p < N) beta[(size_t)k * N + p] = bv;
        lse_add(m, s, bv);
      };
      Ops oa, ob;
      if (ks < K) {
        load(ks, oa);
        int k = ks;
        for (; k + KS < K; k += 2 * KS) {
          load(k + KS, ob);
          compute(k, oa);
          load(min(k + 2 * KS, K - 1), oa);
          compute(k + KS, ob);
        }
        if (k < K) compute(k, oa);
      }
    }
  }
  ms[wv][lane] = m;
  ss[wv][lane] = s;
  __syncthreads();
  double v = 0;
  if (ks == 0 && p < N) {
    for (int q = 1; q < KS; ++q) m = fmax(m, ms[wv + q][lane]);
    s = 0;
    for (int q = 0; q < KS; ++q) s += ss[wv + q][lane] * exp(ms[wv + q][lane] - m);
    v = m + log(s);
    f[p] = v;
  }
  double ps = 0, pe = 0;
  block_comp_sum<double>(v, ps, pe);
  if (gridDim.x == 1) {
    if (threadIdx.x == 0) F[0] = (ps - (double)N * lse_alpha) + pe;
  } else if (threadIdx.x == 0) {
    fpart[2 * blockIdx.x] = ps;
    fpart[2 * blockIdx.x + 1] = pe;
  }
}

// ---- reverse -------------------------------------------------------------------
// A summed slot: DP = 4: S (4x4), u, A; else S's lower 16x16 blocks (block
// ab (ab + 1) / 2 + bb, row-major), u[DP], A.
__host__ __device__ constexpr int f64_nblk(int DP) { return DP / 16 * (DP / 16 + 1) / 2; }
__host__ __device__ constexpr int f64_slot(int DP) {
  return (DP == 4 ? 16 : f64_nblk(DP) * 256) + DP + 1;
}

struct GradPtrs {
  const double *alphas, *means, *qd, *l;
  double *d_alphas, *d_means, *d_qd, *d_l;
};

// What the assembly of component k's gradient needs besides its moments: Q_k and
// softmax(alpha)_k. Every wave takes part; the block meets before they are read.
template <int DP>
struct Assembly {
  double Q[DP][DP + 1], bq[DP], soft;
};

template <int DP>
DEX_DEV void f64_operands(Assembly<DP>& as, const GradPtrs& p, int D, int K, int k) {
  const int t = threadIdx.x, nt = blockDim.x, lane = t & 63;
  const int64_t L = (int64_t)D * (D - 1) / 2;
  for (int e = t; e < DP * DP; e += nt) {
    const int a = e / DP, b = e % DP;
    double q = 0;
    if (a < D && b <= a)
      q = a == b ? exp(p.qd[(size_t)k * D + a]) : p.l[k * L + a * (a - 1) / 2 + b];
    as.Q[a][b] = q;
  }
  if (t >= nt - 64) {  // softmax of alpha, by the last wave
    double am = -INFINITY, az = 0;
    for (int j = lane; j < K; j += 64) am = fmax(am, p.alphas[j]);
    am = wave_reduce(am, [](double a, double b) { return fmax(a, b); });
    for (int j = lane; j < K; j += 64) az += exp(p.alphas[j] - am);
    az = wave_sum(az);
    if (lane == 0) as.soft = exp(p.alphas[k] - am) / az;
  }
}

// Gradient of component k from its summed moments `sm` (LDS); the whole block.
template <int DP>
DEX_DEV void f64_assemble(const double* sm, Assembly<DP>& as, const GradPtrs& p, int64_t N, int D,
                          int k, double ctv, int accumulate) {
  double(&Q)[DP][DP + 1] = as.Q;
  double(&bq)[DP] = as.bq;
  constexpr int kU = f64_slot(DP) - DP - 1;
  const int t = threadIdx.x, nt = blockDim.x;
  const int64_t L = (int64_t)D * (D - 1) / 2;
  auto S = [&](int r, int c) {
    if constexpr (DP == 4) return sm[r * 4 + c];
    const int R = r >> 4, C = c >> 4;
    const int hi = max(R, C), lo = min(R, C);
    const int e = R >= C ? (r & 15) * 16 + (c & 15) : (c & 15) * 16 + (r & 15);
    return sm[(hi * (hi + 1) / 2 + lo) * 256 + e];
  };
  if (t < D) {  // b = Q u
    double v = 0;
    for (int j = 0; j <= t; ++j) v += Q[t][j] * sm[kU + j];
    bq[t] = v;
  }
  __syncthreads();
  const double A = sm[kU + DP];
  for (int e = t; e < D * (D + 1) / 2; e += nt) {
    int a = (int)((sqrtf(8.f * (float)e + 1.f) - 1.f) * 0.5f);
    while (a * (a + 1) / 2 > e) --a;
    while ((a + 1) * (a + 2) / 2 <= e) ++a;
    const int b = e - a * (a + 1) / 2;
    double mv = 0;
    for (int j = 0; j <= a; ++j) mv += Q[a][j] * S(j, b);
    if (a > b) {
      double* o = p.d_l + k * L + a * (a - 1) / 2 + b;
      *o = accumulate ? *o - mv : -mv;
    } else {
      double* o = p.d_qd + (size_t)k * D + a;
      const double gq = A - Q[a][a] * mv;
      *o = accumulate ? *o + gq : gq;
    }
  }
  if (t < D) {
    double gm = 0;
    for (int a = t; a < D; ++a) gm += Q[a][t] * bq[a];
    double* o = p.d_means + (size_t)k * D + t;
    *o = accumulate ? *o + gm : gm;
  }
  if (t == 0) {
    const double ga = A - ctv * (double)N * as.soft;
    p.d_alphas[k] = accumulate ? p.d_alphas[k] + ga : ga;
  }
}

// Block (component k, slot s): the moments of the s-th share of the 64-point
// tiles; wave w takes every blockDim / 64-th of them. The waves' sums are added in
// wave order in LDS. gridDim.y == 1: the gradient is assembled here.
template <int DP>
__global__ void __launch_bounds__(64 * f64_bwd_waves(DP)) k_f64_bwd(
    GradPtrs g_, const double* __restrict__ x, int N, int D, int K,
    const double* __restrict__ beta, const double* __restrict__ f, const double* __restrict__ ct,
    double* __restrict__ part, int accumulate) {
  constexpr int NW = f64_bwd_waves(DP), E = f64_slot(DP), kU = E - DP - 1;
  __shared__ double sm[E];
  __shared__ double buf[NW][DP == 4 ? 16 : 256];
  __shared__ double wsh[NW][64];
  __shared__ Assembly<DP> as;
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int t = threadIdx.x;
  const int k = blockIdx.x;
  const int64_t NT = (N + 63) / 64;
  const int ta = (int)(blockIdx.y * NT / gridDim.y), tb = (int)((blockIdx.y + 1) * NT / gridDim.y);
  const double ctv = ct[0];
  const double* brow = beta + (size_t)k * N;
  double A = 0;
  if (gridDim.y == 1) f64_operands<DP>(as, g_, D, K, k);
  if constexpr (DP == 4) {
    double mu[4], s[10], u[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      mu[b] = b < D ? g_.means[(size_t)k * D + b] : 0.0;
      u[b] = 0;
    }
#pragma unroll
    for (int e = 0; e < 10; ++e) s[e] = 0;
    for (int tile = ta + wv; tile < tb; tile += nw) {
      const int p = tile * 64 + lane, pc = min(p, N - 1);
      const double w = p < N ? exp(brow[pc] - f[pc]) * ctv : 0.0;
      A += w;
      double r[4], wr[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        r[b] = b < D ? x[(size_t)pc * D + b] - mu[b] : 0.0;
        wr[b] = w * r[b];
        u[b] += wr[b];
      }
      int e = 0;
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b) s[e++] += wr[a] * r[b];
    }
    // the wave's 15 sums, halving the values a lane holds at each of the first four
    // steps: lane i ends with value 8 (i/32) + 4 (i/16 % 2) + 2 (i/8 % 2) + i/4 % 2
    double v[16];
#pragma unroll
    for (int e = 0; e < 10; ++e) v[e] = s[e];
#pragma unroll
    for (int b = 0; b < 4; ++b) v[10 + b] = u[b];
    v[14] = A;
    v[15] = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const DPair q = swap32(v[e], v[e + 8]);
      v[e] = q.first + q.second;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const DPair q = swap16(v[e], v[e + 4]);
      v[e] = q.first + q.second;
    }
    auto halve = [&](auto mc, double lo, double hi) {  // lanes with bit M keep hi
      constexpr int M = decltype(mc)::value;
      const bool up = lane & M;
      const double keep = up ? hi : lo, give = up ? lo : hi;
      return keep + __shfl_xor(give, M, 64);
    };
    v[0] = halve(std::integral_constant<int, 8>{}, v[0], v[2]);
    v[1] = halve(std::integral_constant<int, 8>{}, v[1], v[3]);
    v[0] = halve(std::integral_constant<int, 4>{}, v[0], v[1]);
    v[0] += butterfly<1>(v[0]);
    v[0] += butterfly<2>(v[0]);
    if ((lane & 3) == 0)
      buf[wv][8 * (lane >> 5) + 4 * ((lane >> 4) & 1) + 2 * ((lane >> 3) & 1) + ((lane >> 2) & 1)] = v[0];
    __syncthreads();
    if (t < 15) {
      double q = 0;
      for (int w = 0; w < nw; ++w) q += buf[w][t];
      if (t < 10) {
        const int a = t < 1 ? 0 : t < 3 ? 1 : t < 6 ? 2 : 3, b = t - a * (a + 1) / 2;
        sm[a * 4 + b] = q;
        sm[b * 4 + a] = q;
      } else {
        sm[kU + t - 10] = q;
      }
    }
    __syncthreads();
  } else {
    constexpr int NB = DP / 16, NBLK = f64_nblk(DP), BS = DP == 16 ? 16 : DP == 32 ? 8 : 4;
    f64x4 acc[NBLK];
    double u[NB], mu[NB];
#pragma unroll
    for (int q = 0; q < NBLK; ++q) acc[q] = f64x4{0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      u[b] = 0;
      mu[b] = g_.means[(size_t)k * D + min(16 * b + c, D - 1)];
    }
    for (int tile = ta + wv; tile < tb; tile += nw) {
      const int p0 = tile * 64, p = p0 + lane, pc = min(p, N - 1);
      const double w = p < N ? exp(brow[pc] - f[pc]) * ctv : 0.0;
      A += w;
      wsh[wv][lane] = w;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // steps of four points (point 4 s + g of the tile per lane group), the
      // loads of BS steps issued together
#pragma unroll 1
      for (int s0 = 0; s0 < 16; s0 += BS) {
        double xr[BS][NB];
#pragma unroll
        for (int s = 0; s < BS; ++s)
#pragma unroll
          for (int b = 0; b < NB; ++b)
            xr[s][b] = x[(size_t)min(p0 + 4 * (s0 + s) + g, N - 1) * D + min(16 * b + c, D - 1)];
#pragma unroll
        for (int s = 0; s < BS; ++s) {
          const double ws = wsh[wv][4 * (s0 + s) + g];
          double r[NB], wr[NB];
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            r[b] = 16 * b + c < D ? xr[s][b] - mu[b] : 0.0;
            wr[b] = ws * r[b];
            u[b] += wr[b];
          }
#pragma unroll
          for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int b = 0; b <= a; ++b)
              acc[a * (a + 1) / 2 + b] =
                  __builtin_amdgcn_mfma_f64_16x16x4f64(wr[a], r[b], acc[a * (a + 1) / 2 + b], 0, 0, 0);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    // sums over the block's waves, one 16x16 block at a time, then u and A
#pragma unroll
    for (int q = 0; q < NBLK; ++q) {
#pragma unroll
      for (int i = 0; i < 4; ++i) buf[wv][(g + 4 * i) * 16 + c] = acc[q][i];
      __syncthreads();
      if (t < 256) {
        double v = 0;
        for (int w = 0; w < nw; ++w) v += buf[w][t];
        sm[q * 256 + t] = v;
      }
      __syncthreads();
    }
    A = wave_sum(A);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const double v = sum_groups(u[b]);
      if (g == 0) buf[wv][16 * b + c] = v;
    }
    if (lane == 0) buf[wv][DP] = A;
    __syncthreads();
    if (t <= DP) {
      double v = 0;
      for (int w = 0; w < nw; ++w) v += buf[w][t];
      sm[kU + t] = v;
    }
    __syncthreads();
  }
  if (gridDim.y == 1) {
    f64_assemble<DP>(sm, as, g_, N, D, k, ctv, accumulate);
  } else {
    double* P = part + ((size_t)blockIdx.y * K + k) * E;
    for (int e = t; e < E; e += blockDim.x) P[e] = sm[e];
  }
}

// The shares' moments of one component added in order (compensated), then the
// gradient. A thread's loads of 24 shares are issued together.
template <int DP>
__global__ void __launch_bounds__(256) k_f64_bwd_final(GradPtrs g_, const double* __restrict__ part,
                                                       int S, int64_t N, int D, int K,
                                                       const double* __restrict__ ct,
                                                       int accumulate) {
  constexpr int E = f64_slot(DP);
  __shared__ double sm[E];
  __shared__ Assembly<DP> as;
  const int k = blockIdx.x;
  for (int e = threadIdx.x; e < E; e += 256) {
    double s = 0, err = 0;
    for (int s0 = 0; s0 < S; s0 += 24) {
      double v[24];
#pragma unroll
      for (int q = 0; q < 24; ++q)
        v[q] = s0 + q < S ? part[((size_t)(s0 + q) * K + k) * E + e] : 0.0;
#pragma unroll
      for (int q = 0; q < 24; ++q) {
        double ns, ne;
        two_sum<double>(s, v[q], ns, ne);
        s = ns;
        err += ne;
      }
    }
    sm[e] = s + err;
  }
  f64_operands<DP>(as, g_, D, K, k);
  __syncthreads();
  f64_assemble<DP>(sm, as, g_, N, D, k, ct[0], accumulate);
}

__global__ void __launch_bounds__(256) k_f64_finalize_F(const double* __restrict__ fpart, int nparts,
                                                        const double* __restrict__ alphas, int K,
                                                        int64_t N, double* __restrict__ F) {
  finalize_F_block<double>(fpart, nparts, alphas, K, N, F);
}

}  // namespace dexk

namespace dexi {
using namespace dexk;

namespace {
int f64_dp(int64_t D) { return D <= 4 ? 4 : D <= 16 ? 16 : D <= 32 ? 32 : 64; }

// Shares of the points per component in the reverse: about 512 blocks, at
// least a tile per wave.
int f64_shares(int64_t N, int64_t D, int64_t K) {
  const int64_t tiles = (N + 63) / 64, nw = f64_bwd_waves(f64_dp(D));
  return (int)std::max<int64_t>(1, std::min<int64_t>((512 + K - 1) / K, (tiles + nw - 1) / nw));
}
}  // namespace

size_t gmm_f64_fwd_ws(int64_t N) { return align256((size_t)((N + 63) / 64) * 2 * 8); }
// S K slots, and what any smaller N or K may need too (S K is at most 511 + K, and S 1
// from K = 512 on), so that scratch sized for the largest call serves all.
size_t gmm_f64_bwd_ws(int64_t N, int64_t D, int64_t K) {
  const int64_t k = std::min<int64_t>(K, 511), one = f64_shares(N, D, 1);
  if (one == 1) return 0;
  return align256((size_t)std::min(511 + k, one * k) * f64_slot(f64_dp(D)) * 8);
}

#define DEX_F64_DP(DP_, CALL) \
  switch (DP_) {              \
    case 4:                   \
      CALL(4);                \
      break;                  \
    case 16:                  \
      CALL(16);               \
      break;                  \
    case 32:                  \
      CALL(32);               \
      break;                  \
    default:                  \
      CALL(64);               \
  }

void gmm_f64_fwd(int64_t N, int64_t D, int64_t K, const GmmPtrs& in, double* beta, double* f,
                 double* fpart, double* F, hipStream_t st) {
  // (D = 5 .. 8: two chunks of four columns instead of four: N = 1e6, D = 8, K = 3 59 us
  // for 76, with the blocks below 45)
  const int dp = D > 4 && D <= 8 ? 8 : f64_dp(D), maxw = f64_fwd_waves(dp);
  const int64_t tiles = (N + 63) / 64;
  // One block, which also finishes F, where its waves' components take no longer
  // than the launch it saves (about 10 000 cycles; cycles per 64 points and
  // component by padded dimension); else one tile per block and enough waves
  // sharing its components to fill the chip (about four per SIMD).
  const int64_t cost = dp == 4 ? 500 : dp == 8 ? 700 : dp == 16 ? 900 : dp == 32 ? 2200 : 6000;
  int64_t tt = 1, ks;
  if (tiles <= maxw && ((K + maxw / tiles - 1) / (maxw / tiles)) * cost <= 10000) {
    tt = tiles;
    ks = std::min<int64_t>(maxw / tiles, K);
  } else {
    ks = std::min<int64_t>({(4096 + tiles - 1) / tiles, maxw, K});
    // with a wave a tile, four tiles a block, so that starting blocks does not bound the
    // small ones (N = 1e6, D = 1, K = 2 45 us with one tile, 26; D = 16, K = 3 78, 69; D =
    // 32, K = 2 155, 190)
    if (tiles >= 4096 && dp <= 16) tt = 4;
  }
  const unsigned blocks = (unsigned)((tiles + tt - 1) / tt), threads = (unsigned)(64 * tt * ks);
  const double *al = (const double*)in.alphas, *mu = (const double*)in.means,
               *qd = (const double*)in.qd, *l = (const double*)in.l, *x = (const double*)in.x;
#define DEX_F64_FWD(DP_)                                                                    \
  hipLaunchKernelGGL((k_f64_fwd<DP_>), dim3(blocks), dim3(threads), 0, st, al, mu, qd, l, x, \
                     (int)N, (int)D, (int)K, (int)ks, beta, f, fpart, F)
  if (dp == 8)
    DEX_F64_FWD(8);
  else
    DEX_F64_DP(dp, DEX_F64_FWD)
#undef DEX_F64_FWD
  if (blocks > 1)
    hipLaunchKernelGGL(k_f64_finalize_F, dim3(1), dim3(256), 0, st, fpart, (int)blocks, al, (int)K, N,
                       F);
}

void gmm_f64_vjp(int64_t N, int64_t D, int64_t K, const GmmPtrs& in, const double* beta,
                 const double* f, const double* ct, const GmmGrads& out, bool accumulate,
                 double* part, hipStream_t st) {
  const int dp = f64_dp(D), S = f64_shares(N, D, K);
  const int64_t tiles = (N + 63) / 64;
  const int nw = (int)std::min<int64_t>(f64_bwd_waves(dp), std::max<int64_t>(4, tiles));
  const GradPtrs g{(const double*)in.alphas, (const double*)in.means, (const double*)in.qd,
                   (const double*)in.l,      (double*)out.d_alphas,   (double*)out.d_means,
                   (double*)out.d_qd,        (double*)out.d_l};
#define DEX_F64_BWD(DP_)                                                                        \
  hipLaunchKernelGGL((k_f64_bwd<DP_>), dim3((unsigned)K, (unsigned)S), dim3(64 * nw), 0, st, g, \
                     (const double*)in.x, (int)N, (int)D, (int)K, beta, f, ct, part,            \
                     accumulate ? 1 : 0)
  DEX_F64_DP(dp, DEX_F64_BWD)
#undef DEX_F64_BWD
  if (S == 1) return;
#define DEX_F64_FIN(DP_)                                                                     \
  hipLaunchKernelGGL((k_f64_bwd_final<DP_>), dim3((unsigned)K), dim3(256), 0, st, g, part, S, N, \
                     (int)D, (int)K, ct, accumulate ? 1 : 0)
  DEX_F64_DP(dp, DEX_F64_FIN)
#undef DEX_F64_FIN
}

}  // namespace dexi
