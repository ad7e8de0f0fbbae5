// GMM log-likelihood, one instance: host dispatch, the forward mode (but for the
// 16-bit variant's at D = 64 and that on quads of components, gmm_f32.hip) and the
// merge / finalize kernels of the FP32-storage forms (gmm_dev.h, gmm_mfma_inst.hip);
// the FP64 forward and reverse are in gmm_f64.hip.
#include "gmm_host.h"
#include "internal.h"

namespace dexk {

template <typename T>
__global__ void __launch_bounds__(256) k_merge_lse(const float2* __restrict__ ml, int Sk, int N,
                                                   int Npad, T* __restrict__ f,
                                                   T* __restrict__ fpart) {
  T s = 0, e = 0;
  merge_lse_block<T>(ml, Sk, N, Npad, blockIdx.x * 256, f, s, e);
  if (threadIdx.x == 0) {
    fpart[2 * blockIdx.x] = s;
    fpart[2 * blockIdx.x + 1] = e;
  }
}

template <typename T>
__global__ void __launch_bounds__(256) k_merge_lse_quad(const float2* __restrict__ ml, int Sk,
                                                        int N, int Npad, T* __restrict__ f,
                                                        T* __restrict__ fpart) {
  T s = 0, e = 0;
  merge_lse_quad<T>(ml, Sk, N, Npad, blockIdx.x * 64, f, s, e);
  if (threadIdx.x == 0) {
    fpart[2 * blockIdx.x] = s;
    fpart[2 * blockIdx.x + 1] = e;
  }
}

// s + err += a, compensated (two_sum)
DEX_DEV void comp_add(float& s, float& err, float a) {
  float ns, ne;
  two_sum<float>(s, a, ns, ne);
  s = ns;
  err += ne;
}

// Fixed-order compensated sum of each component's partial moment slots (the
// waves that owned part of its group's points), written back into slot 0, so
// the per-component finalize reads a single slot. Slots of component k: on each
// XCD x the waves that owned part of its group's steps, in slots x * SX + rank.
DEX_DEV int mom_slots(int64_t kg, int x, int64_t nkg, int64_t nsteps, int Wx) {
  const int64_t nsx = (x + 1) * nsteps / 8 - x * nsteps / 8;
  return nsx == 0 ? 0 : split_slots(kg * nsx, nsx, nkg * nsx, min<int64_t>(Wx, nkg * nsx));
}

// A block sums 64 consecutive elements, one per lane; its W waves share the
// slots: 8 / W XCDs each in order (W = 4, 1), or every W / 8-th slot of one XCD (W =
// 16), and the waves' sums are added in wave order. Bound by the latency of the
// slot loads, so they are spread over waves as far as there are few elements: with
// few components there are many slots each (N = 1e5, D = 20, K = 5: 340) and one
// thread per element walked them in 190 us. With very many elements one wave takes
// all eight XCDs (reverse pass at N = 100, D = 64, K = 1000: 94 us with W = 4, 82).
template <int W>
__global__ void __launch_bounds__(64 * W) k_mom_reduce(float* __restrict__ part, int64_t E, int K,
                                                       int gw, int64_t nsteps, int Wx, int SX) {
  __shared__ int Ssh[2][8];
  __shared__ float ssh[W][64], esh[W][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t i0 = (int64_t)blockIdx.x * 64, i = i0 + lane;
  const int64_t nkg = (K + gw - 1) / gw;
  // a block meets at most two components (E >= 256): their slot counts
  const int k0 = (int)(i0 / E);
  if (threadIdx.x < 16) {
    const int kk = k0 + (int)(threadIdx.x >> 3);
    Ssh[threadIdx.x >> 3][threadIdx.x & 7] =
        kk < K ? mom_slots(kk / gw, threadIdx.x & 7, nkg, nsteps, Wx) : 0;
  }
  __syncthreads();
  const bool in = i < (int64_t)K * E;
  const int kr = in && i >= (int64_t)(k0 + 1) * E ? 1 : 0;
  const size_t stride = (size_t)K * E;
  constexpr int XW = W < 8 ? 8 / W : 1;   // XCDs of a wave
  constexpr int SH = W < 8 ? 1 : W / 8;   // waves of an XCD
  constexpr int U = 5;                    // slots of an XCD loaded together
  const int xa = W < 8 ? wv * XW : wv / SH, r0 = W < 8 ? 0 : wv % SH;
  float s = 0.f, err = 0.f;
  int S[XW];
  float v[XW][U];
#pragma unroll
  for (int q = 0; q < XW; ++q) {
    S[q] = in ? Ssh[kr][xa + q] : 0;
    const float* base = part + (size_t)(xa + q) * SX * stride + i;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int sp = r0 + u * SH;
      v[q][u] = sp < S[q] ? base[(size_t)sp * stride] : 0.f;
    }
  }
#pragma unroll
  for (int q = 0; q < XW; ++q) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (r0 + u * SH < S[q]) comp_add(s, err, v[q][u]);
    const float* base = part + (size_t)(xa + q) * SX * stride + i;
    for (int sp0 = r0 + U * SH; sp0 < S[q]; sp0 += 8 * SH) {
      float w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int sp = sp0 + u * SH;
        w[u] = sp < S[q] ? base[(size_t)sp * stride] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (sp0 + u * SH < S[q]) comp_add(s, err, w[u]);
    }
  }
  ssh[wv][lane] = s;
  esh[wv][lane] = err;
  __syncthreads();
  if (wv == 0 && in) {
#pragma unroll
    for (int w = 1; w < W; ++w) {
      comp_add(s, err, ssh[w][lane]);
      err += esh[w][lane];
    }
    part[i] = s + err;
  }
}

// Forward mode on the vector ALU: FP64, and FP32 at D <= 4 with few components, where
// quads of components are mostly padding and the start of their blocks (N = 1e6, D = 2, K =
// 5: 27 us, quads 42; K = 64: 217, 153). Block
// (256 points, chunk of kJvpKC components); the components of the chunk are
// staged in LDS in turn. For point i and component k, with r = x_i - mu_k,
//   y = Q_k r, dy = dQ_k r - Q_k dmu_k (dQ: diagonal exp(qd) dqd, strict lower
//   dl), beta = kappa_k - |y|^2 / 2, dbeta = dalpha_k + sum_d dqd_kd - y . dy,
// and the tangent of f_i = LSE_k beta_ik is sum_k exp(beta_ik - f_i) dbeta_ik.
// Each block writes its FP64 sum of these to part[blockIdx.y * gridDim.x +
// blockIdx.x].
constexpr int kJvpKC = 8;

template <typename T, int DB>
__global__ void __launch_bounds__(256) gmm_jvp_valu(
    const T* __restrict__ alphas, const T* __restrict__ means,
    const T* __restrict__ qd, const T* __restrict__ l, const T* __restrict__ x,
    const T* __restrict__ f, int N, int D, int K, const T* __restrict__ da,
    const T* __restrict__ dm, const T* __restrict__ dq, const T* __restrict__ dl,
    double* __restrict__ part) {
  __shared__ T Qs[DB][DB + 1], dQs[DB][DB + 1];
  __shared__ T mus[DB], qdm[DB], kap[2];
  __shared__ double sh[32];
  const int t = threadIdx.x, p = blockIdx.x * 256 + t;
  const bool valid = p < N;
  const int L = D * (D - 1) / 2;
  T xr[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b) xr[b] = (valid && b < D) ? x[(size_t)p * D + b] : T(0);
  const T fp = valid ? f[p] : T(0);
  double acc = 0.0;
  const int k0 = blockIdx.y * kJvpKC, k1 = min(K, k0 + kJvpKC);
  for (int k = k0; k < k1; ++k) {
    __syncthreads();
    for (int e = t; e < DB * DB; e += 256) {
      const int a = e / DB, b = e % DB;
      T q = 0, dqv = 0;
      if (a < D && b < D) {
        if (a == b) {
          const T ev = dexp<T>(qd[(size_t)k * D + a]);
          q = ev;
          dqv = ev * dq[(size_t)k * D + a];
        } else if (a > b) {
          const size_t li = (size_t)k * L + a * (a - 1) / 2 + b;
          q = l[li];
          dqv = dl[li];
        }
      }
      Qs[a][b] = q;
      dQs[a][b] = dqv;
    }
    if (t < DB) mus[t] = t < D ? means[(size_t)k * D + t] : T(0);
    if (t < 64) {
      T s = 0, ds = 0;
      for (int d = t; d < D; d += 64) {
        s += qd[(size_t)k * D + d];
        ds += dq[(size_t)k * D + d];
      }
      s = wave_sum(s);
      ds = wave_sum(ds);
      if (t == 0) {
        kap[0] = alphas[k] + s;
        kap[1] = da[k] + ds;
      }
    }
    __syncthreads();
    if (t < DB) {  // Q_k dmu_k
      T v = 0;
      for (int b = 0; b <= t && b < D; ++b) v += Qs[t][b] * dm[(size_t)k * D + b];
      qdm[t] = v;
    }
    __syncthreads();
    T r[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b) r[b] = b < D ? xr[b] - mus[b] : T(0);
    T s = 0, sd = 0;
#pragma unroll
    for (int a = 0; a < DB; ++a) {
      if (a < D) {
        T y = 0, dy = -qdm[a];
#pragma unroll
        for (int b = 0; b <= a; ++b) {
          y += Qs[a][b] * r[b];
          dy += dQs[a][b] * r[b];
        }
        s += y * y;
        sd += y * dy;
      }
    }
    if (valid) acc += (double)(dexp<T>(kap[0] - T(0.5) * s - fp) * (kap[1] - sd));
  }
  acc = block_sum(acc, sh);
  if (t == 0) part[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = acc;
}

// The same for FP32 storage and D > 32 on the matrix cores (16x16x4 FP32 products;
// smaller D goes on quads of components): a wave takes 64 points and every KS-th
// component. Per component y = Q_k r and dy = dQ_k r - Q_k dmu_k from r = x - mu_k
// (formed per component: the difference of two FP32 values, rounded once), with the
// strict lower parts read as they are stored and the next component's loads issued
// before the current one's products; |y|^2 and y . dy are summed over the lane groups
// so that lane p owns point p. Each wave writes its FP64 sum to part[wave]. (N = 20000,
// D = 32, K = 50: 63 us a launch, 37 on quads; one thread per point and LDS broadcasts
// of Q and dQ 163.) Lane layout: A and B hold row / column c and contraction values
// 16 ch + 4 g + j (element j), the result rows 4 g + i.
__global__ void __launch_bounds__(256) gmm_jvp_mfma(
    const float* __restrict__ alphas, const float* __restrict__ means, const float* __restrict__ qd,
    const float* __restrict__ l, const float* __restrict__ x, const float* __restrict__ f, int N,
    int D, int K, int KS, const float* __restrict__ da, const float* __restrict__ dm,
    const float* __restrict__ dq, const float* __restrict__ dl, double* __restrict__ part) {
  constexpr int NB = 4, NQ = NB * (NB + 1) / 2;
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int wave = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tiles = (N + 63) / 64;
  const int ks = wave / tiles, tile = wave - ks * tiles;
  if (ks >= KS) return;  // (no barrier follows)
  const int p0 = tile * 64, p = p0 + lane;
  const int64_t L = (int64_t)D * (D - 1) / 2;
  f32x4 xb[4][NB];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int ch = 0; ch < NB; ++ch) {
      const float* row = x + (size_t)min(p0 + 16 * t + c, N - 1) * D;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = 16 * ch + 4 * g + j;
        const float v = row[min(col, D - 1)];
        xb[t][ch][j] = col < D ? v : 0.f;
      }
    }
  const float fp = f[min(p, N - 1)];
  // component k's operands as loaded: chunks (rb, ch <= rb) of l and dl, the
  // diagonals of the lane's rows, the means and their tangents at its columns
  struct Ops {
    f32x4 q[NQ], dq[NQ], mu[NB], dmu[NB];
    float qdr[NB], dqr[NB], al, da;
  };
  auto load = [&](int k, Ops& o) {
    int n = 0;
#pragma unroll
    for (int rb = 0; rb < NB; ++rb) {
      const int row = 16 * rb + c, rc = min(row, D - 1);
      o.qdr[rb] = qd[(size_t)k * D + rc];
      o.dqr[rb] = dq[(size_t)k * D + rc];
#pragma unroll
      for (int ch = 0; ch <= rb; ++ch, ++n)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int col = 16 * ch + 4 * g + j;
          const int64_t e = k * L + (row < D && col < row ? row * (row - 1) / 2 + col : 0);
          o.q[n][j] = l[e];
          o.dq[n][j] = dl[e];
        }
    }
#pragma unroll
    for (int ch = 0; ch < NB; ++ch)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const size_t e = (size_t)k * D + min(16 * ch + 4 * g + j, D - 1);
        o.mu[ch][j] = means[e];
        o.dmu[ch][j] = dm[e];
      }
    o.al = alphas[k];
    o.da = da[k];
  };
  double acc = 0.0;
  auto compute = [&](const Ops& o) {
    float s[4] = {0, 0, 0, 0}, sd[4] = {0, 0, 0, 0}, sq = 0.f, sdq = 0.f;
    int n = 0;
#pragma unroll
    for (int rb = 0; rb < NB; ++rb) {
      const int row = 16 * rb + c;
      const bool rin = row < D;
      sq += rin ? o.qdr[rb] : 0.f;
      sdq += rin ? o.dqr[rb] : 0.f;
      const float ed = expf(o.qdr[rb]), ded = ed * o.dqr[rb];
      f32x4 y[4], dy[4], qm = f32x4{0.f, 0.f, 0.f, 0.f};  // qm: Q dmu, the same in every column
#pragma unroll
      for (int t = 0; t < 4; ++t) y[t] = dy[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ch = 0; ch <= rb; ++ch, ++n) {
        f32x4 q = o.q[n], dqv = o.dq[n];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int col = 16 * ch + 4 * g + j;
          if (ch == rb) {
            q[j] = col < row ? q[j] : col == row ? ed : 0.f;
            dqv[j] = col < row ? dqv[j] : col == row ? ded : 0.f;
          }
          q[j] = rin ? q[j] : 0.f;
          dqv[j] = rin ? dqv[j] : 0.f;
          const float mu = col < D ? o.mu[ch][j] : 0.f, dmu = col < D ? o.dmu[ch][j] : 0.f;
          qm = __builtin_amdgcn_mfma_f32_16x16x4f32(q[j], dmu, qm, 0, 0, 0);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const float r = xb[t][ch][j] - mu;
            y[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(q[j], r, y[t], 0, 0, 0);
            dy[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(dqv[j], r, dy[t], 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s[t] = fmaf(y[t][i], y[t][i], s[t]);
          sd[t] = fmaf(y[t][i], dy[t][i] - qm[i], sd[t]);
        }
    }
    treduce_groups<4>(s);   // lane 16 t + c: point 16 t + c
    treduce_groups<4>(sd);
#define DEX_ROW16(v)          \
  v += butterfly<1>(v);       \
  v += butterfly<2>(v);       \
  v += butterfly<4>(v);       \
  v += butterfly<8>(v);
    DEX_ROW16(sq)
    DEX_ROW16(sdq)
#undef DEX_ROW16
    const float w = expf((o.al + sq) - 0.5f * s[0] - fp);
    if (p < N) acc += (double)(w * ((o.da + sdq) - sd[0]));
  };
  Ops oa, ob;
  load(ks, oa);
  int k = ks;
  for (; k + KS < K; k += 2 * KS) {
    load(k + KS, ob);
    compute(oa);
    load(min(k + 2 * KS, K - 1), oa);
    compute(ob);
  }
  if (k < K) compute(oa);
  acc = wave_sum(acc);
  if (lane == 0) part[wave] = acc;
}

// dF = (sum of the partials, fixed order) - N sum_k softmax(alpha)_k dalpha_k,
// in FP64.
template <typename T>
__global__ void __launch_bounds__(256) k_jvp_final(const double* __restrict__ part, int64_t np,
                                                   const T* __restrict__ alphas,
                                                   const T* __restrict__ da, int K, int64_t N,
                                                   T* __restrict__ out) {
  __shared__ double sh[32];
  double s = 0.0, am = -INFINITY;
  for (int64_t i = threadIdx.x; i < np; i += 256) s += part[i];
  for (int k = threadIdx.x; k < K; k += 256) am = fmax(am, (double)alphas[k]);
  s = block_sum(s, sh);
  // max over the block (every thread's am), through the same LDS slots
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = -INFINITY;
  __syncthreads();
  {
    double m = am;
    m = wave_reduce(m, [](double a, double b) { return fmax(a, b); });
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  }
  __syncthreads();
  am = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
  double z = 0.0, zd = 0.0;
  for (int k = threadIdx.x; k < K; k += 256) {
    const double e = exp((double)alphas[k] - am);
    z += e;
    zd += e * (double)da[k];
  }
  z = block_sum(z, sh);
  zd = block_sum(zd, sh);
  if (threadIdx.x == 0) out[0] = (T)(s - (double)N * zd / z);
}

template <typename T>
__global__ void __launch_bounds__(256) k_finalize_F(const T* __restrict__ fpart, int nparts,
                                                    const T* __restrict__ alphas, int K, int64_t N,
                                                    T* __restrict__ F) {
  finalize_F_block<T>(fpart, nparts, alphas, K, N, F);
}

// Component k's moment partials, already summed into slot 0 (S = 1); the
// moments were taken about the origin `shift`.
__global__ void __launch_bounds__(256) k_bwd_finalize_mom(
    const float* __restrict__ part, size_t E, int S, int K, int D, int DP, int64_t N,
    const float* __restrict__ alphas, const float* __restrict__ means, const float* __restrict__ qd,
    const float* __restrict__ l, const float* __restrict__ ct, float* __restrict__ d_alphas,
    float* __restrict__ d_means, float* __restrict__ d_qd, float* __restrict__ d_l, int accumulate,
    const float* __restrict__ shift) {
  const int k = blockIdx.x;
  bwd_finalize_mom(part + (size_t)k * E, (size_t)K * E, S, k, K, D, DP, N, alphas, means, qd, l,
                   ct[0], d_alphas, d_means, d_qd, d_l, accumulate, shift);
}

}  // namespace dexk

// ===========================================================================
namespace dexi {
using namespace dexk;

namespace {

struct Shape {
  GmmGeom g;
  int dtype, variant, prec;
  bool mfma;
  size_t tsize;
};

Shape shape_of(const dex_desc& d) {
  Shape s{};
  s.g.N = d.dims[0];
  s.g.D = d.dims[1];
  s.g.K = d.dims[2];
  s.g.DP = s.g.D <= 16 ? 16 : s.g.D <= 32 ? 32 : 64;
  s.g.Npad = (s.g.N + 255) / 256 * 256;
  s.dtype = d.dtype;
  s.variant = d.variant;
  s.tsize = d.dtype == DEX_F64 ? 8 : 4;
  s.mfma = d.dtype == DEX_F32;
  s.prec = d.variant == DEX_GMM_BF16 ? PREC_BF16 : d.variant == DEX_GMM_BF16X3 ? PREC_BF16X3 : PREC_F32;
  return s;
}

// forward candidates: (components resident per wave, waves per SIMD (0: all
// resident), x~ tiles loaded ahead); BF16 config 0 is the feature-product form
// (D = 64 only; other D run config 1 in its place)
const FwdCfg kFwdBF[] = {{0, 0, 0}, {4, 0, 1}, {4, 0, 2}, {2, 0, 1},
                         {2, 0, 2}, {4, 1, 2}, {2, 2, 2}, {0, 1, 0}};
const FwdCfg kFwdF32[] = {{2, 0, 1}, {2, 0, 2}, {2, 2, 1}, {2, 1, 2}};
// reverse candidates: (components per wave, waves per SIMD (0: all resident),
// FP16 form: scaled rows double-buffered (default) or not)
const BwdCfg kBwdBF[] = {{2, 0}, {3, 0}, {4, 0}, {2, 2}, {3, 2}, {4, 0, 0}, {2, 1}, {4, 1}};
const BwdCfg kBwdF32[] = {{2, 0}, {1, 0}, {4, 0}, {2, 2}, {1, 2}};

int nfwd(const Shape& s) { return s.prec == PREC_BF16 ? 8 : 4; }
int nbwd(const Shape& s) { return s.prec == PREC_F32 ? 5 : 8; }
size_t mom_es(const Shape& s) { return s.prec == PREC_F32 ? 4 : 2; }
FwdCfg fwd_cfg(const Shape& s, int i) { return s.prec == PREC_BF16 ? kFwdBF[i] : kFwdF32[i]; }
BwdCfg bwd_cfg(const Shape& s, int i) { return s.prec == PREC_F32 ? kBwdF32[i] : kBwdBF[i]; }

// FP32 operands and D <= 32: the forward on quads of components
bool quads(const Shape& s) { return s.mfma && s.prec == PREC_F32 && s.g.D <= 32; }

struct CacheLayout {
  size_t xh, xl, xhT, xlT, Qh, Ql, negc, kappa, beta, shift, total;
  // feature-product forward (BF16, D = 64): coefficient operand, kappa',
  // rescale factors, scaled FP16 copy of x, per-tile scale exponents
  size_t W16, kq, isc, x16, texp;
};

CacheLayout cache_layout(const Shape& s) {
  CacheLayout c{};
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o += align256(bytes);
    return at;
  };
  const GmmGeom& g = s.g;
  if (s.mfma) {
    const size_t es = s.prec == PREC_F32 ? 4 : 2;
    const bool lo = s.prec == PREC_BF16X3;
    c.xh = quads(s) ? 0 : take(g.Npad * g.DP * es);
    c.xl = lo ? take(g.Npad * g.DP * es) : 0;
    c.xhT = take(g.Npad * g.DP * mom_es(s));
    c.xlT = lo ? take(g.Npad * g.DP * mom_es(s)) : 0;
    c.Qh = take(quads(s) ? quad_rec_bytes(g) : g.K * g.DP * g.DP * es);
    c.Ql = lo ? take(g.K * g.DP * g.DP * es) : 0;
    c.negc = quads(s) ? 0 : take(g.K * g.DP * 4);  // (quads: in their records)
    c.kappa = quads(s) ? 0 : take(g.K * 4);
    c.shift = take(64 * 4);
    c.beta = take(beta_rows(g.K) * g.Npad * 4);
    if (qf_eligible(g, s.prec)) {
      const size_t Kp = (size_t)beta_rows(g.K);
      c.W16 = take(Kp / 16 * 68 * 64 * 8 * 2);
      c.kq = take(Kp * 4);
      c.isc = take(Kp * 4);
      c.x16 = take((size_t)g.Npad * 64 * 2);
      c.texp = take((size_t)(g.Npad / 64) * 4);
    }
  } else {
    c.beta = take(g.K * g.N * s.tsize);
  }
  c.total = o;
  return c;
}

MfmaOps ops_of(const Shape& s, const CacheLayout& cl, const char* cache) {
  MfmaOps o;
  const bool lo = s.prec == PREC_BF16X3;
  o.xh = cache + cl.xh;
  o.xl = lo ? cache + cl.xl : nullptr;
  o.xhT = cache + cl.xhT;
  o.xlT = lo ? cache + cl.xlT : nullptr;
  o.Qh = cache + cl.Qh;
  o.Ql = lo ? cache + cl.Ql : nullptr;
  o.negc = (const float*)(cache + cl.negc);
  o.kappa = (const float*)(cache + cl.kappa);
  return o;
}

bool valid_shape(const Shape& s) {
  const GmmGeom& g = s.g;
  if (g.N < 1 || g.D < 1 || g.K < 1 || g.D > 64) return false;
  if (s.dtype != DEX_F32 && s.dtype != DEX_F64) return false;
  if (s.variant != DEX_GMM_PLAIN && s.dtype != DEX_F32) return false;
  if (s.variant > DEX_GMM_BF16X3) return false;  // the split-FP16 form is batched only
  return true;
}

}  // namespace

size_t gmm_cache_bytes(const dex_desc& d) {
  Shape s = shape_of(d);
  if (!valid_shape(s)) return 0;
  return cache_layout(s).total;
}

// Forward-mode workspace. Feature-product form (16-bit variant, D = 64): the
// scaled FP16 x~ and its tile exponents, the tangent coefficient operand,
// dkq' and rescale factors, one FP64 partial per (pass, tile). Vector-ALU
// form: one FP64 partial per (point block, component chunk). Quads: both records, the
// origin, one partial per (tile, share).
struct JvpLayout {
  size_t x16, texp, dW16, dkq, disc, rec, trec, shift, part, total;
  int64_t nparts;
  QuadSplit quad;  // quads of components (D <= 32; no tiles: not)
  int ks;  // D > 32: waves sharing a tile's components
};
// Waves that share a 64-point tile's components, for the least rounds of waves
// (one per SIMD) times components each.
static int jvp_shares(const GmmGeom& g) {
  const int64_t tiles = (g.N + 63) / 64, simds = 4 * num_cus();
  int best = 1;
  int64_t cost = INT64_MAX;
  for (int ks = 1; ks <= kMaxShares && ks <= g.K; ++ks) {
    const int64_t c = (tiles * ks + simds - 1) / simds * ((g.K + ks - 1) / ks + 1);
    if (c < cost) {
      cost = c;
      best = ks;
    }
  }
  return best;
}
static int64_t valu_parts(const GmmGeom& g) {
  return (g.N + 255) / 256 * ((g.K + kJvpKC - 1) / kJvpKC);
}
static JvpLayout jvp_layout(const Shape& s) {
  JvpLayout j{};
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o += align256(bytes);
    return at;
  };
  if (s.mfma && qf_eligible(s.g, s.prec)) {
    const size_t Kp = (size_t)beta_rows(s.g.K);
    j.x16 = take((size_t)s.g.Npad * 64 * 2);
    j.texp = take((size_t)(s.g.Npad / 64) * 4);
    j.dW16 = take(Kp / 16 * 68 * 64 * 8 * 2);
    j.dkq = take(Kp * 4);
    j.disc = take(Kp * 4);
    j.nparts = qf_tan_parts(s.g);
  } else if (s.mfma && s.g.D <= 4 && s.g.K <= 10) {
    j.nparts = valu_parts(s.g);
  } else if (s.mfma && s.g.D <= 32) {
    j.quad = quad_jvp_split(s.g);
    j.rec = take(quad_rec_bytes(s.g));
    j.trec = take(quad_rec_bytes(s.g));
    j.shift = take(64 * 4);
    j.nparts = j.quad.tiles * j.quad.ks;
  } else if (s.mfma) {
    j.ks = jvp_shares(s.g);
    j.nparts = (s.g.N + 63) / 64 * j.ks;
  } else {
    j.nparts = valu_parts(s.g);
  }
  // the partials of the most shares any smaller N or K may have, so that scratch sized for
  // the largest call serves all
  const int64_t most = j.quad.tiles ? j.quad.tiles * std::min<int64_t>(kMaxShares, (s.g.K + 3) / 4)
                       : j.ks       ? j.nparts / j.ks * std::min<int64_t>(kMaxShares, s.g.K)
                                    : j.nparts;
  j.part = take((size_t)most * 8);
  j.total = o;
  return j;
}

size_t gmm_ws_bytes(const dex_desc& d, int role) {
  Shape s = shape_of(d);
  if (!valid_shape(s)) return 0;
  if (role == DEX_WS_RESID) return cache_layout(s).total;
  if (role == DEX_WS_JVP) return jvp_layout(s).total;
  if (!s.mfma)
    return role == DEX_WS_FWD ? gmm_f64_fwd_ws(s.g.N) : gmm_f64_bwd_ws(s.g.N, s.g.D, s.g.K);
  const size_t nparts = (size_t)(s.g.Npad / 64);  // objective partials (one per 64 points)
  if (role == DEX_WS_FWD)
    return align256(nparts * 2 * s.tsize) +
           align256((size_t)fwd_max_slots(s.g.K) * s.g.Npad * sizeof(float2));
  return align256((size_t)bwd_max_slots(s.g.Npad, s.g.K) * s.g.K * mom_slot(s.g.DP) * 4);
}

int gmm_num_configs(const dex_desc& d, int role) {
  Shape s = shape_of(d);
  if (!s.mfma) return 1;
  return role == DEX_WS_VJP ? nbwd(s) : nfwd(s);
}

// (Quads have one form: every configuration of the FP32 forward at D <= 32 launches it.)
int gmm_tuned_configs(const dex_desc& d, int role) {
  return role != DEX_WS_VJP && quads(shape_of(d)) ? 1 : gmm_num_configs(d, role);
}

// The configuration of an untuned call, by the form and by N K (the work per
// element of a component's moments). Measured whole calls, us:
//   forward FP32, D > 32 (at D <= 32 every configuration is the quads'): two
//     components a wave, two waves a SIMD; split BF16 at D > 32: one wave a SIMD and two
//     tiles ahead (46 against 50 at N = 1e5, K = 5).
//   reverse 16-bit: below 1.5e6 two components and one wave a SIMD (D = 64, N =
//     10000, K = 37: 37 against 41 with four components); above, four components (D =
//     64, N = 1e5, K = 200: 0.123 ms a call against 0.19 with two), at D <= 16 from 1e7
//     on with all waves resident (N = 1e5, K = 200, D = 8: 44 against 54).
//   reverse FP32: one component and two waves a SIMD below 1.2e6 (D = 20, N = 30011,
//     K = 37: 41 against 45 for two components, all resident), two and two below 5e6
//     (N = 10000, K = 200: 56 against 58), two and all resident above.
//   reverse split BF16: as 16-bit below 1.5e6 (35 against 41); above, three
//     components and two waves a SIMD (D = 20, N = 30011, K = 200: 78 against 82), two
//     at D > 32, where three need too many registers.
int gmm_default_config(const dex_desc& d, int role) {
  const Shape s = shape_of(d);
  if (!s.mfma || !valid_shape(s)) return 0;
  const double nk = (double)s.g.N * (double)s.g.K;
  if (role != DEX_WS_VJP)
    return s.prec == PREC_F32 ? 2 : s.prec == PREC_BF16X3 && s.g.DP == 64 ? 3 : 0;
  if (s.prec == PREC_F32) return nk < 1.2e6 ? 4 : nk < 5e6 ? 3 : 0;
  if (nk < 1.5e6) return 6;
  if (s.prec == PREC_BF16X3) return s.g.DP == 64 ? 3 : 4;
  return s.g.DP == 16 && nk >= 1e7 ? 2 : 7;
}

dex_status gmm_fwd(const dex_desc& d, int cfg, const GmmPtrs& in, void* F, void* f, void* cache,
                   void* ws, hipStream_t st) {
  Shape s = shape_of(d);
  if (!valid_shape(s)) return fail(DEX_ERR_UNSUPPORTED, "GMM shape/dtype/variant not supported");
  CacheLayout cl = cache_layout(s);
  char* cc = (char*)cache;
  const size_t nparts = (size_t)(s.g.Npad / 64);
  if (!s.mfma) {
    gmm_f64_fwd(s.g.N, s.g.D, s.g.K, in, (double*)(cc + cl.beta), (double*)f, (double*)ws,
                (double*)F, st);
    return check_hip(hipGetLastError(), "gmm_fwd (FP64)");
  }
  if (cfg < 0 || cfg >= nfwd(s)) return fail(DEX_ERR_INVALID_ARG, "GMM forward config %d out of range", cfg);
  const FwdCfg c = fwd_cfg(s, cfg);
  float* fpart = (float*)ws;
  float2* ml = (float2*)((char*)ws + align256(nparts * 2 * 4));
  float* beta = (float*)(cc + cl.beta);
  const MfmaOps o = ops_of(s, cl, cc);
  const float* x = (const float*)in.x;
  const float *al = (const float*)in.alphas, *mu = (const float*)in.means,
              *qd = (const float*)in.qd, *l = (const float*)in.l;
  void *xh = cc + cl.xh, *xl = cc + cl.xl, *xhT = cc + cl.xhT, *xlT = cc + cl.xlT, *Qh = cc + cl.Qh,
       *Ql = cc + cl.Ql;
  float *negc = (float*)(cc + cl.negc), *kappa = (float*)(cc + cl.kappa);
  float* shift = (float*)(cc + cl.shift);  // written by the preparation launch
  FlatSplit sp{};
  switch (s.prec) {
    case PREC_BF16:
      if (c.nkq == 0 && qf_eligible(s.g, s.prec)) {
        qf_prep(s.g, x, al, mu, qd, l, xhT, cc + cl.x16, (int*)(cc + cl.texp), cc + cl.W16,
                (float*)(cc + cl.kq), (float*)(cc + cl.isc), shift, st);
        ProfRange pr(DEX_PROF_GMM_FWD, st);
        sp = qf_fwd(s.g, c, cc + cl.x16, cc + cl.W16, (const float*)(cc + cl.kq),
                    (const float*)(cc + cl.isc), (const int*)(cc + cl.texp), beta, ml, st);
        pr.end(1);
      } else {
        const FwdCfg ck = c.nkq == 0 ? kFwdBF[1] : c;
        mfma_prep<PREC_BF16>(s.g, x, al, mu, qd, l, xh, xl, xhT, xlT, Qh, Ql, negc, kappa, shift,
                             st);
        ProfRange pr(DEX_PROF_GMM_FWD, st);
        sp = mfma_fwd<PREC_BF16>(s.g, ck, o, beta, ml, st);
        pr.end(1);
      }
      break;
    case PREC_BF16X3:
      mfma_prep<PREC_BF16X3>(s.g, x, al, mu, qd, l, xh, xl, xhT, xlT, Qh, Ql, negc, kappa, shift,
                             st);
      {
        ProfRange pr(DEX_PROF_GMM_FWD, st);
        sp = mfma_fwd<PREC_BF16X3>(s.g, c, o, beta, ml, st);
        pr.end(1);
      }
      break;
    default:
      if (quads(s)) {
        const QuadSplit q = quad_fwd_split(s.g);
        quad_prep(s.g, in, (float*)xhT, (float*)Qh, shift, st);
        ProfRange pr(DEX_PROF_GMM_FWD, st);
        quad_fwd(s.g, q, x, (const float*)Qh, shift, beta, ml, st);
        sp.sk = q.ks;
        pr.end(1);
        break;
      }
      mfma_prep<PREC_F32>(s.g, x, al, mu, qd, l, xh, xl, xhT, xlT, Qh, Ql, negc, kappa, shift,
                          st);
      {
        ProfRange pr(DEX_PROF_GMM_FWD, st);
        sp = mfma_fwd<PREC_F32>(s.g, c, o, beta, ml, st);
        pr.end(1);
      }
  }
  // few partials per point: one thread per point; many: four
  const bool quad = sp.sk > 16;
  const unsigned nq = (unsigned)(s.g.Npad / (quad ? 64 : 256));
  if (quad)
    hipLaunchKernelGGL((k_merge_lse_quad<float>), dim3(nq), dim3(256), 0, st, ml, sp.sk,
                       (int)s.g.N, (int)s.g.Npad, (float*)f, fpart);
  else
    hipLaunchKernelGGL((k_merge_lse<float>), dim3(nq), dim3(256), 0, st, ml, sp.sk, (int)s.g.N,
                       (int)s.g.Npad, (float*)f, fpart);
  hipLaunchKernelGGL((k_finalize_F<float>), dim3(1), dim3(256), 0, st, fpart, (int)nq, al,
                     (int)s.g.K, s.g.N, (float*)F);
  return check_hip(hipGetLastError(), "gmm_fwd (MFMA)");
}

dex_status gmm_vjp(const dex_desc& d, int cfg, const GmmPtrs& in, const void* f,
                   const void* cache, const void* ct, const GmmGrads& out, bool accumulate,
                   void* ws, hipStream_t st) {
  Shape s = shape_of(d);
  if (!valid_shape(s)) return fail(DEX_ERR_UNSUPPORTED, "GMM shape/dtype/variant not supported");
  CacheLayout cl = cache_layout(s);
  const char* cc = (const char*)cache;
  if (!s.mfma) {
    gmm_f64_vjp(s.g.N, s.g.D, s.g.K, in, (const double*)(cc + cl.beta), (const double*)f,
                (const double*)ct, out, accumulate, (double*)ws, st);
    return check_hip(hipGetLastError(), "gmm_vjp (FP64)");
  }
  if (cfg < 0 || cfg >= nbwd(s)) return fail(DEX_ERR_INVALID_ARG, "GMM reverse config %d out of range", cfg);
  const BwdCfg c = bwd_cfg(s, cfg);
  const MfmaOps o = ops_of(s, cl, cc);
  const float* beta = (const float*)(cc + cl.beta);
  float* part = (float*)ws;
  ProfRange pr(DEX_PROF_GMM_VJP, st);
  FlatSplit sp{};
  switch (s.prec) {
    case PREC_BF16:
      sp = mfma_bwd<PREC_BF16>(s.g, c, o, beta, (const float*)f, (const float*)ct, part, st);
      break;
    case PREC_BF16X3:
      sp = mfma_bwd<PREC_BF16X3>(s.g, c, o, beta, (const float*)f, (const float*)ct, part, st);
      break;
    default:
      sp = mfma_bwd<PREC_F32>(s.g, c, o, beta, (const float*)f, (const float*)ct, part, st);
  }
  pr.end(1);
  const int64_t E = (int64_t)mom_slot(s.g.DP);
  const unsigned nb = (unsigned)((s.g.K * E + 63) / 64);
  if (nb > 16384)
    hipLaunchKernelGGL(k_mom_reduce<1>, dim3(nb), dim3(64), 0, st, part, E, (int)s.g.K, sp.gw,
                       sp.nsteps, sp.W, (int)sp.T);
  else if (nb <= 512)
    hipLaunchKernelGGL(k_mom_reduce<16>, dim3(nb), dim3(1024), 0, st, part, E, (int)s.g.K, sp.gw,
                       sp.nsteps, sp.W, (int)sp.T);
  else
    hipLaunchKernelGGL(k_mom_reduce<4>, dim3(nb), dim3(256), 0, st, part, E, (int)s.g.K, sp.gw,
                       sp.nsteps, sp.W, (int)sp.T);
  hipLaunchKernelGGL(k_bwd_finalize_mom, dim3((unsigned)s.g.K), dim3(256), 0, st, (const float*)part,
                     (size_t)E, 1, (int)s.g.K,
                     (int)s.g.D, s.g.DP, s.g.N, (const float*)in.alphas, (const float*)in.means,
                     (const float*)in.qd, (const float*)in.l, (const float*)ct,
                     (float*)out.d_alphas, (float*)out.d_means, (float*)out.d_qd, (float*)out.d_l,
                     accumulate ? 1 : 0, (const float*)(cc + cl.shift));
  return check_hip(hipGetLastError(), "gmm_vjp (MFMA)");
}

static void launch_jvp_valu(const Shape& s, const GmmPtrs& in, const void* f, const GmmGrads& t,
                            double* part, hipStream_t st) {
  dim3 grid((unsigned)((s.g.N + 255) / 256), (unsigned)((s.g.K + kJvpKC - 1) / kJvpKC));
#define DEX_JV(T, DB)                                                                             \
  hipLaunchKernelGGL((gmm_jvp_valu<T, DB>), grid, dim3(256), 0, st, (const T*)in.alphas,          \
                     (const T*)in.means, (const T*)in.qd, (const T*)in.l, (const T*)in.x,         \
                     (const T*)f, (int)s.g.N, (int)s.g.D, (int)s.g.K, (const T*)t.d_alphas,       \
                     (const T*)t.d_means, (const T*)t.d_qd, (const T*)t.d_l, part)
  if (s.mfma) {
    DEX_JV(float, 4);
  } else if (s.g.D <= 4) {
    DEX_JV(double, 4);
  } else if (s.g.D <= 8) {
    DEX_JV(double, 8);
  } else if (s.g.D <= 16) {
    DEX_JV(double, 16);
  } else if (s.g.D <= 32) {
    DEX_JV(double, 32);
  } else {
    DEX_JV(double, 64);
  }
#undef DEX_JV
}

dex_status gmm_jvp(const dex_desc& d, int cfg, const GmmPtrs& in, const void* f,
                   const void* cache, const GmmGrads& t, void* dF, void* ws, hipStream_t st) {
  (void)cfg;
  Shape s = shape_of(d);
  if (!valid_shape(s)) return fail(DEX_ERR_UNSUPPORTED, "GMM shape/dtype/variant not supported");
  const JvpLayout jl = jvp_layout(s);
  char* w = (char*)ws;
  double* part = (double*)(w + jl.part);
  if (s.mfma && qf_eligible(s.g, s.prec)) {
    // tangent products over the same second-order features as the forward
    const CacheLayout cl = cache_layout(s);
    const char* cc = (const char*)cache;
    const float* shift = (const float*)(cc + cl.shift);
    qf_tan_prep(s.g, (const float*)in.x, (const float*)in.means, (const float*)in.qd,
                (const float*)in.l, (const float*)t.d_alphas, (const float*)t.d_means,
                (const float*)t.d_qd, (const float*)t.d_l, shift, w + jl.x16, (int*)(w + jl.texp),
                w + jl.dW16, (float*)(w + jl.dkq), (float*)(w + jl.disc), st);
    ProfRange pr(DEX_PROF_GMM_JVP, st);
    qf_jvp(s.g, w + jl.x16, w + jl.dW16, (const float*)(w + jl.dkq), (const float*)(w + jl.disc),
           (const int*)(w + jl.texp), (const float*)(cc + cl.beta), (const float*)f, part, st);
    pr.end(1);
  } else if (jl.quad.tiles) {
    ProfRange pr(DEX_PROF_GMM_JVP, st);
    quad_jvp(s.g, jl.quad, in, t, (const float*)f, (float*)(w + jl.rec), (float*)(w + jl.trec),
             (float*)(w + jl.shift), part, st);
    pr.end(1);
  } else if (jl.ks) {
    ProfRange pr(DEX_PROF_GMM_JVP, st);
    const dim3 grid((unsigned)((jl.nparts + 3) / 4));
    hipLaunchKernelGGL(gmm_jvp_mfma, grid, dim3(256), 0, st, (const float*)in.alphas,
                       (const float*)in.means, (const float*)in.qd, (const float*)in.l,
                       (const float*)in.x, (const float*)f, (int)s.g.N, (int)s.g.D, (int)s.g.K,
                       jl.ks, (const float*)t.d_alphas, (const float*)t.d_means,
                       (const float*)t.d_qd, (const float*)t.d_l, part);
    pr.end(1);
  } else {
    ProfRange pr(DEX_PROF_GMM_JVP, st);
    launch_jvp_valu(s, in, f, t, part, st);
    pr.end(1);
  }
  if (s.tsize == 8)
    hipLaunchKernelGGL((k_jvp_final<double>), dim3(1), dim3(256), 0, st, (const double*)part,
                       jl.nparts, (const double*)in.alphas, (const double*)t.d_alphas, (int)s.g.K,
                       s.g.N, (double*)dF);
  else
    hipLaunchKernelGGL((k_jvp_final<float>), dim3(1), dim3(256), 0, st, (const double*)part,
                       jl.nparts, (const float*)in.alphas, (const float*)t.d_alphas, (int)s.g.K,
                       s.g.N, (float*)dF);
  return check_hip(hipGetLastError(), "gmm_jvp");
}

}  // namespace dexi
