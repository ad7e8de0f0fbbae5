// Many independent GMM instances of uneven size, FP32 matrix-core form.
//
// The nested parallel loop `for b. for i k. ...` is flattened into work items
// (Sec. 6.1.1: parallelism is allocated at the top level only). A host-side
// plan lists, per phase, the items (instance, point block[, component group])
// ordered longest first; the forward and reverse phases each run as one
// persistent launch whose blocks take items from an atomic counter until the
// list is exhausted, so the smallest instances do not pay a launch each.
// FP32 units: gmm_quad.h, D padded to a multiple of 8; the moments of instances that
// fill few quads go component by component, D padded to 16 or 32 (blocks_pay).
// Split-FP16 forward (D > 8): tiles of 16-deep contraction chunks, D padded likewise.
#include <string.h>

#include <algorithm>
#include <numeric>
#include <vector>

#include "gmm_host.h"
#include "gmm_quad.h"
#include "internal.h"

namespace dexk {

struct BInst {
  int32_t N, D, K, DP;
  int64_t Npad;
  int64_t a_off, m_off, l_off, x_off, f_off;       // packed inputs / f (elements)
  // cache (bytes); xhT_off: of instances whose moments go component by component
  // (blocks_pay), else 0
  int64_t xh_off, xhT_off, Q_off, negc_off, kappa_off, beta_off;
  int64_t ml_off;     // ws float2 elements
  int64_t fpart_off;  // ws float pairs
  int64_t part_off;   // ws floats
  int32_t nblk;       // Npad / 256
  int32_t split;      // forward operands in split FP16 (variant DEX_GMM_F16X3, D > 8):
                      // x~ and per-component Q~, negc, kappa; else records of component quads at Q_off
  int64_t xl_off, ts_off, Ql_off;  // cache (bytes): split form: low parts, per-tile x scales
  int64_t sh_off;     // cache (bytes): origin shift[DP], the factor scale, max |mu - shift|
};

struct BItem {
  int32_t inst, a, b, c;
};

constexpr int kBFwdCfgs = 2;
constexpr int kBBwdCfgs = 4;
// Points per reverse work item (a block, 16 components). Configuration 0: 4096, halved
// down to 512 while the batch has fewer than kBItems items, so that a small batch still
// fills the chip (64 mixtures of 10000 points, chunks of 512, 1024, 2048, 8192: 238,
// 222, 253, 690 us; 12 of 2000: 73, 116, 193, 230), and no instance more than kBChunks
// chunks, whose moments one block adds up (1e6 points, D = 2, K = 3: 141, 93, 76, 134).
// The plan says what was chosen.
inline int64_t bbwd_chunk(int i) {
  const int64_t t[kBBwdCfgs] = {4096, 1024, 2048, 8192};
  return t[i];
}
constexpr int64_t kBItems = 2048, kBChunks = 512;
__host__ __device__ inline int bfwd_cb(int i) { return i == 0 ? 4 : 2; }

struct PlanHeader {
  int64_t B;
  int64_t inst_off;
  int64_t prepx_off, n_prepx;
  int64_t prepq_off, n_prepq;  // (instance, component), those that fill up a quad too
  int64_t merge_off, n_merge;
  int64_t fwd_off[kBFwdCfgs], n_fwd[kBFwdCfgs];
  int64_t bwd_off[kBBwdCfgs], n_bwd[kBBwdCfgs];
  int64_t nch_off;  // int32 [kBBwdCfgs][B]: point chunks per instance
  int64_t cache_bytes, ws_bytes;
  int64_t ws_ml, ws_fpart, ws_counter, ws_part;  // byte offsets into ws
  int64_t comp_off, n_comp;      // (instance, component)
  int64_t bwd_chunk[kBBwdCfgs];  // points per reverse item
  int64_t blk_off[kBBwdCfgs], n_blk[kBBwdCfgs];  // items of 8 components, one by one
};

__device__ inline const PlanHeader* hdr(const char* plan) { return (const PlanHeader*)plan; }

// (split instances)
__device__ inline MfmaOps bops(const BInst& I, const char* cache) {
  MfmaOps o;
  o.xh = cache + I.xh_off;
  o.xl = cache + I.xl_off;
  o.xhT = o.xlT = nullptr;
  o.Qh = cache + I.Q_off;
  o.Ql = cache + I.Ql_off;
  o.negc = (const float*)(cache + I.negc_off);
  o.kappa = (const float*)(cache + I.kappa_off);
  return o;
}

// One block per instance: the origin shift, the mean of the first min(K, 16)
// means (every operand is taken about it, so data far from the origin loses
// nothing to cancellation: only x - mu enters). Split instances also get the
// power of two that brings the largest factor entry (exp(qd) or |l|) to
// [2^13, 2^14), and the largest |mu_k - shift|, which bounds every tile's
// point scale (the points are scaled per 64-point tile in the preparation):
// scaled means then stay inside the FP16 range in every tile.
__global__ void __launch_bounds__(256) k_bscale(const char* __restrict__ plan,
                                                const float* __restrict__ means,
                                                const float* __restrict__ qd,
                                                const float* __restrict__ l, char* cache) {
  const PlanHeader* h = hdr(plan);
  const BInst I = ((const BInst*)(plan + h->inst_off))[blockIdx.x];
  __shared__ float csh[64];
  __shared__ float red[8];
  block_shift(means + I.m_off, I.K, I.D, csh);
  const int t = threadIdx.x;
  float* sh = (float*)(cache + I.sh_off);
  if (t < I.DP) sh[t] = csh[t];
  if (!I.split) {
    if (t == 0) sh[I.DP] = sh[I.DP + 1] = 1.f;
    return;
  }
  float mq = 0.f, mm = 0.f;
  const int64_t nd = (int64_t)I.K * I.D, nl = (int64_t)I.K * I.D * (I.D - 1) / 2;
  for (int64_t e = t; e < nd; e += 256) {
    mq = fmaxf(mq, expf(qd[I.m_off + e]));
    mm = fmaxf(mm, fabsf(means[I.m_off + e] - csh[(int)(e % I.D)]));
  }
  for (int64_t e = t; e < nl; e += 256) mq = fmaxf(mq, fabsf(l[I.l_off + e]));
  mq = wave_max(mq);
  mm = wave_max(mm);
  if ((t & 63) == 0) {
    red[t >> 6] = mq;
    red[4 + (t >> 6)] = mm;
  }
  __syncthreads();
  if (t == 0) {
    mq = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    int eq = 0;
    if (mq > 0.f && mq <= 3.0e38f) (void)frexpf(mq, &eq);
    sh[I.DP] = ldexpf(1.f, 14 - eq);
    sh[I.DP + 1] = fmaxf(fmaxf(red[4], red[5]), fmaxf(red[6], red[7]));
  }
}

// Split form, one 64-point tile: x - shift scaled by the power of two that brings the larger of the
// tile's largest |x - shift| and the instance's largest |mu - shift| (shift[DP
// + 1]) to [2^13, 2^14), in split FP16 for the forward (row layout); the tile's
// scale goes to ts[p0 / 64]. (256 threads; the loads are all issued before the
// first is used.)
template <int DP>
DEX_DEV void prep_x_tile_split(const float* __restrict__ x, int N, int D, int Npad, int p0,
                               const float* __restrict__ shift, _Float16* xh, _Float16* xl,
                               float* ts) {
  constexpr int NL = 64 * DP / 256;
  __shared__ float tile[64][DP + 1];
  __shared__ float red[4];
  __syncthreads();
  float v[NL], mx = 0.f;
  // branch-free loads at clamped addresses, selected afterwards
  float sv[NL];  // (the shift has DP entries, zero past D)
#pragma unroll
  for (int r = 0; r < NL; ++r) {
    const int e = threadIdx.x + 256 * r, pp = e / DP, b = e % DP, p = p0 + pp;
    v[r] = x[(size_t)min(p, N - 1) * D + min(b, D - 1)];
    sv[r] = shift[b];
  }
#pragma unroll
  for (int r = 0; r < NL; ++r) {
    const int e = threadIdx.x + 256 * r, pp = e / DP, b = e % DP, p = p0 + pp;
    v[r] = p < N && b < D ? v[r] - sv[r] : 0.f;
  }
#pragma unroll
  for (int r = 0; r < NL; ++r) {
    const int e = threadIdx.x + 256 * r;
    tile[e / DP][e % DP] = v[r];
    mx = fmaxf(mx, fabsf(v[r]));
  }
  mx = wave_max(mx);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])), shift[DP + 1]);
  int ex = 0;
  if (mx > 0.f && mx <= 3.0e38f) (void)frexpf(mx, &ex);
  const float sc = ldexpf(1.f, 14 - ex);
  if (threadIdx.x == 0) ts[p0 / 64] = sc;
  for (int e = threadIdx.x; e < 8 * DP; e += blockDim.x) {
    const int pp = e / (DP / 8), b0 = 8 * (e % (DP / 8));
    float w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = tile[pp][b0 + i] * sc;
    store8_split<PREC_F16X3>(xh, xl, (size_t)(p0 + pp) * DP + b0, w);
  }
}

__global__ void __launch_bounds__(256) k_bprep_x(const char* __restrict__ plan,
                                                 const float* __restrict__ x, char* cache) {
  const PlanHeader* h = hdr(plan);
  const BItem w = ((const BItem*)(plan + h->prepx_off))[blockIdx.x];
  const BInst I = ((const BInst*)(plan + h->inst_off))[w.inst];
  const float* sh = (const float*)(cache + I.sh_off);
  if (I.xhT_off) {
    float* xhT = (float*)(cache + I.xhT_off);
    if (I.DP == 16)
      prep_x_tile<PREC_F32, 16>(x + I.x_off, I.N, I.D, (int)I.Npad, w.a * 64, nullptr, nullptr, xhT,
                                nullptr, nullptr, sh);
    else
      prep_x_tile<PREC_F32, 32>(x + I.x_off, I.N, I.D, (int)I.Npad, w.a * 64, nullptr, nullptr, xhT,
                                nullptr, nullptr, sh);
  }
  if (!I.split) return;
  _Float16* xh = (_Float16*)(cache + I.xh_off);
  _Float16* xl = (_Float16*)(cache + I.xl_off);
  float* ts = (float*)(cache + I.ts_off);
  if (I.DP == 16)
    prep_x_tile_split<16>(x + I.x_off, I.N, I.D, (int)I.Npad, w.a * 64, sh, xh, xl, ts);
  else
    prep_x_tile_split<32>(x + I.x_off, I.N, I.D, (int)I.Npad, w.a * 64, sh, xh, xl, ts);
}

__global__ void __launch_bounds__(256) k_bprep_q(const char* __restrict__ plan,
                                                 const float* __restrict__ alphas,
                                                 const float* __restrict__ means,
                                                 const float* __restrict__ qd,
                                                 const float* __restrict__ l, char* cache) {
  const PlanHeader* h = hdr(plan);
  const BItem w = ((const BItem*)(plan + h->prepq_off))[blockIdx.x];
  const BInst I = ((const BInst*)(plan + h->inst_off))[w.inst];
  if (I.split) {
    float* negc = (float*)(cache + I.negc_off);
    float* kappa = (float*)(cache + I.kappa_off);
    using H = Store<PREC_F16X3>::S;
    const float* sh = (const float*)(cache + I.sh_off);
    H* Qh = (H*)(cache + I.Q_off);
    H* Ql = (H*)(cache + I.Ql_off);
    if (I.DP == 16)
      prep_q_comp<PREC_F16X3, 16>(alphas + I.a_off, means + I.m_off, qd + I.m_off, l + I.l_off, I.D,
                                  w.a, Qh, Ql, negc, kappa, sh, sh[I.DP]);
    else
      prep_q_comp<PREC_F16X3, 32>(alphas + I.a_off, means + I.m_off, qd + I.m_off, l + I.l_off, I.D,
                                  w.a, Qh, Ql, negc, kappa, sh, sh[I.DP]);
    return;
  }
  float* Q = (float*)(cache + I.Q_off);
  const float* sh = (const float*)(cache + I.sh_off);
  with_d8(I.D, [&](auto d8) {
    QuadPrep<decltype(d8)::value, false> p;
    const typename decltype(p)::Src src{alphas + I.a_off, means + I.m_off, qd + I.m_off,
                                        l + I.l_off};
    p.load(src, src, I.D, I.K, w.a);
    p.store(I.D, I.K, w.a, sh, Q, Q);
  });
}

__global__ void fill_counters(int* c, int n) {
  if ((int)threadIdx.x < n) c[threadIdx.x] = 0;
}

// Take the next item index for the whole block.
DEX_DEV int next_item(int* counter) {
  __shared__ int cur;
  __syncthreads();
  if (threadIdx.x == 0) cur = atomicAdd(counter, 1);
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(cur);
}

// SPLIT: the plan's instances with D > 8 carry split FP16 operands.
template <int CB, bool SPLIT>
__global__ void __launch_bounds__(256, SPLIT ? 3 : 4) k_bgmm_fwd(const char* __restrict__ plan, int cfg,
                                                  const float* __restrict__ x, const char* cache,
                                                  char* ws) {
  __shared__ __attribute__((aligned(16))) float lds[kQuadLds];
  const PlanHeader* h = hdr(plan);
  const BInst* inst = (const BInst*)(plan + h->inst_off);
  const BItem* items = (const BItem*)(plan + h->fwd_off[cfg]);
  const int n = (int)h->n_fwd[cfg];
  int* counter = (int*)(ws + h->ws_counter);
  float2* ml = (float2*)(ws + h->ws_ml);
  for (;;) {
    const int it = next_item(counter);
    if (it >= n) break;
    const BItem w = items[it];
    const BInst I = inst[w.inst];
    float* beta = (float*)(cache + I.beta_off);
    if constexpr (SPLIT) {
      if (I.split) {
        // the wave's points lie in one 64-point tile, whose x scale applies
        const int p0 = w.a * 64 * CB + (threadIdx.x >> 6) * 16 * CB;
        const MfmaOps o = bops(I, cache);
        const float xs = ((const float*)(cache + I.ts_off))[p0 / 64];
        const float sc = xs * ((const float*)(cache + I.sh_off))[I.DP], sfac = 1.f / (sc * sc);
        if (I.DP == 16)
          fwd_unit<16, PREC_F16X3, CB, 16>(o, I.N, (int)I.Npad, p0, 0, I.K, beta, ml + I.ml_off, sfac,
                                           xs);
        else
          fwd_unit<32, PREC_F16X3, CB, 16>(o, I.N, (int)I.Npad, p0, 0, I.K, beta, ml + I.ml_off, sfac,
                                           xs);
        continue;
      }
    }
    auto quads = [&](auto d8) {
      fwd_quads<decltype(d8)::value, CB>(x + I.x_off, (const float*)(cache + I.sh_off), I.N, I.D,
                                         (int)I.Npad, w.a * 64 * CB, (const float*)(cache + I.Q_off),
                                         0, (I.K + 3) / 4, beta, ml + I.ml_off, lds);
    };
    if constexpr (SPLIT)
      quads(std::integral_constant<int, 8>{});  // (D <= 8: the others are split)
    else
      with_d8(I.D, quads);
  }
}

__global__ void __launch_bounds__(256) k_bmerge(const char* __restrict__ plan, float* __restrict__ f,
                                                char* ws) {
  const PlanHeader* h = hdr(plan);
  const BItem w = ((const BItem*)(plan + h->merge_off))[blockIdx.x];
  const BInst I = ((const BInst*)(plan + h->inst_off))[w.inst];
  const float2* ml = (const float2*)(ws + h->ws_ml) + I.ml_off;
  float* fpart = (float*)(ws + h->ws_fpart) + 2 * I.fpart_off;
  float s = 0.f, e = 0.f;
  merge_lse_block<float>(ml, 1, I.N, (int)I.Npad, w.a * 256, f + I.f_off, s, e);
  if (threadIdx.x == 0) {
    fpart[2 * w.a] = s;
    fpart[2 * w.a + 1] = e;
  }
}

__global__ void __launch_bounds__(256) k_bfinalize_F(const char* __restrict__ plan,
                                                     const float* __restrict__ alphas,
                                                     const char* ws, float* __restrict__ F) {
  const PlanHeader* h = hdr(plan);
  const BInst I = ((const BInst*)(plan + h->inst_off))[blockIdx.x];
  const float* fpart = (const float*)(ws + h->ws_fpart) + 2 * I.fpart_off;
  finalize_F_block<float>(fpart, I.nblk, alphas + I.a_off, I.K, I.N, F + blockIdx.x);
}

__global__ void __launch_bounds__(256, 3) k_bgmm_bwd(const char* __restrict__ plan, int cfg,
                                                     const float* __restrict__ x,
                                                     const char* cache,
                                                     const float* __restrict__ f, char* ws) {
  __shared__ __attribute__((aligned(16))) float lds[kMomPackLds];
  const PlanHeader* h = hdr(plan);
  const BInst* inst = (const BInst*)(plan + h->inst_off);
  const BItem* items = (const BItem*)(plan + h->bwd_off[cfg]);
  const int n = (int)h->n_bwd[cfg];
  const int64_t chunk = h->bwd_chunk[cfg];
  int* counter = (int*)(ws + h->ws_counter) + 1;
  float* part = (float*)(ws + h->ws_part);
  for (;;) {
    const int it = next_item(counter);
    if (it >= n) break;
    const BItem w = items[it];
    const BInst I = inst[w.inst];
    const int pbeg = (int)(w.b * chunk);
    const int pend = (int)std::min<int64_t>(I.Npad, pbeg + chunk);
    with_d8(I.D, [&](auto d8) {
      constexpr int D8 = decltype(d8)::value;
      const size_t E = mom_pack_slot(D8);
      mom_pack_unit<D8>(x + I.x_off, (const float*)(cache + I.sh_off), I.N, I.D, (int)I.Npad, I.K,
                        16 * w.a, pbeg, pend, (const float*)(cache + I.beta_off), f + I.f_off,
                        part + I.part_off + (size_t)w.b * I.K * E, E, lds);
    });
  }
}

// The items of instances whose moments go component by component: eight components, two
// a wave, from x~^T.
__global__ void __launch_bounds__(256) k_bgmm_bwd_blocks(const char* __restrict__ plan, int cfg,
                                                         const char* cache,
                                                         const float* __restrict__ f, char* ws) {
  const PlanHeader* h = hdr(plan);
  const BInst* inst = (const BInst*)(plan + h->inst_off);
  const BItem* items = (const BItem*)(plan + h->blk_off[cfg]);
  const int n = (int)h->n_blk[cfg];
  const int64_t chunk = h->bwd_chunk[cfg];
  int* counter = (int*)(ws + h->ws_counter) + 2;
  for (;;) {
    const int it = next_item(counter);
    if (it >= n) break;
    const BItem w = items[it];
    const BInst I = inst[w.inst];
    const int pbeg = (int)(w.b * chunk);
    const int pend = (int)std::min<int64_t>(I.Npad, pbeg + chunk);
    const size_t E = mom_slot(I.DP);
    float* P = (float*)(ws + h->ws_part) + I.part_off + (size_t)w.b * I.K * E;
    const float* beta = (const float*)(cache + I.beta_off);
    const int kw = w.a * 8 + (threadIdx.x >> 6) * 2;
    if (I.DP == 16)
      bwd_mom_unit<16, MP_F32, 2>(cache + I.xhT_off, nullptr, I.N, (int)I.Npad, I.K, kw, pbeg, pend,
                                  beta, f + I.f_off, 1.f, P, E);
    else
      bwd_mom_unit<32, MP_F32, 2>(cache + I.xhT_off, nullptr, I.N, (int)I.Npad, I.K, kw, pbeg, pend,
                                  beta, f + I.f_off, 1.f, P, E);
  }
}

// PACK: the instances of the packed moments, else the others.
template <bool PACK>
__global__ void __launch_bounds__(256) k_bbwd_finalize(const char* __restrict__ plan, int cfg,
                                                       const char* ws, const char* cache,
                                                       const float* __restrict__ alphas,
                                                       const float* __restrict__ qd,
                                                       const float* __restrict__ l,
                                                       const float* __restrict__ means,
                                                       const float* __restrict__ ct,
                                                       float* __restrict__ d_alphas,
                                                       float* __restrict__ d_means,
                                                       float* __restrict__ d_qd,
                                                       float* __restrict__ d_l, int accumulate) {
  const PlanHeader* h = hdr(plan);
  const BItem w = ((const BItem*)(plan + h->comp_off))[blockIdx.x];
  const BInst I = ((const BInst*)(plan + h->inst_off))[w.inst];
  if (PACK == (I.xhT_off != 0)) return;
  const int nch = ((const int32_t*)(plan + h->nch_off))[cfg * h->B + w.inst];
  const size_t E = PACK ? mom_pack_slot((I.D + 7) & ~7) : mom_slot(I.DP);
  const float* part = (const float*)(ws + h->ws_part) + I.part_off + (size_t)w.a * E;
  // moments of x - shift without the cotangent
  const float c = ct[w.inst];
  bwd_finalize_mom<32, PACK>(part, (size_t)I.K * E, nch, w.a, I.K, I.D, I.DP, I.N, alphas + I.a_off,
                             means + I.m_off, qd + I.m_off, l + I.l_off, c, d_alphas + I.a_off,
                             d_means + I.m_off, d_qd + I.m_off, d_l + I.l_off, accumulate,
                             (const float*)(cache + I.sh_off), c, c, c);
}

}  // namespace dexk

// ===========================================================================
namespace dexi {
using namespace dexk;

namespace {

struct PlanBuild {
  PlanHeader h{};
  std::vector<BInst> inst;
  std::vector<BItem> prepx, prepq, comp, merge;
  std::vector<BItem> fwd[kBFwdCfgs], bwd[kBBwdCfgs], blk[kBBwdCfgs];
  std::vector<int32_t> nch;  // [cfg][B]
  size_t bytes = 0;
};

// Matrix products per 4 points of an instance's moments: packed, 16 components at a time
// however many there are; and component by component, the 16x16 blocks of each (a third
// dearer apiece) with the weights and, in the forward, x~^T to prepare. 100 mixtures of
// 20000 points, forward and reverse, us: D = 25, K = 3 155 + 390 packed, 246 + 172; D = 32,
// K = 5 250 + 373, 341 + 223; D = 24, K = 3 145 + 267, 227 + 172; D = 16, K = 3 134 + 135,
// 177 + 104.
double packed_cost(const BInst& I) {
  return (double)(mom_pack_slot((I.D + 7) & ~7) / 16) * ((I.K + 15) / 16);
}
double blocks_cost(const BInst& I) {
  return I.DP == 16 ? 1.34 * I.K + 7.7 : 1.34 * 3 * I.K + 12.2;
}
bool blocks_pay(const BInst& I) { return I.D > 8 && blocks_cost(I) < packed_cost(I); }

PlanBuild build_plan(const int64_t* shapes, int64_t B, int32_t variant) {
  PlanBuild p;
  p.h.B = B;
  p.inst.resize(B);
  int64_t a = 0, m = 0, lo = 0, xo = 0, fo = 0, ml = 0, fp = 0, cache = 0, part = 0;
  auto take = [&](int64_t bytes) {
    int64_t at = cache;
    cache += (int64_t)align256((size_t)bytes);
    return at;
  };
  // A second kind of launch for some instances is worth it where it saves a tenth of all.
  double packed = 0.0, best = 0.0;
  for (int64_t b = 0; b < B; ++b) {
    BInst& I = p.inst[b];
    I.N = (int32_t)shapes[3 * b];
    I.D = (int32_t)shapes[3 * b + 1];
    I.K = (int32_t)shapes[3 * b + 2];
    I.DP = I.D <= 16 ? 16 : 32;
    I.Npad = (I.N + 255) / 256 * 256;
    packed += I.Npad * packed_cost(I);
    best += I.Npad * (blocks_pay(I) ? blocks_cost(I) : packed_cost(I));
  }
  const bool some_blocks = best < 0.9 * packed;
  for (int64_t b = 0; b < B; ++b) {
    BInst& I = p.inst[b];
    I.nblk = (int32_t)(I.Npad / 256);
    I.a_off = a;
    I.m_off = m;
    I.l_off = lo;
    I.x_off = xo;
    I.f_off = fo;
    a += I.K;
    m += (int64_t)I.K * I.D;
    lo += (int64_t)I.K * I.D * (I.D - 1) / 2;
    xo += (int64_t)I.N * I.D;
    fo += I.N;
    I.split = variant == DEX_GMM_F16X3 && I.D > 8;
    const int D8 = (I.D + 7) & ~7;
    const int64_t nq = (I.K + 3) / 4;  // component quads
    if (I.split) {
      I.xh_off = take(I.Npad * I.DP * 2);
      I.xl_off = take(I.Npad * I.DP * 2);
      I.Q_off = take((int64_t)I.K * I.DP * I.DP * 2);
      I.Ql_off = take((int64_t)I.K * I.DP * I.DP * 2);
      I.ts_off = take(I.Npad / 64 * 4);
    } else {
      I.Q_off = take(nq * quad_floats(D8) * 4);
    }
    I.sh_off = take((int64_t)(I.DP + 2) * 4);
    if (I.split) {
      I.negc_off = take((int64_t)I.K * I.DP * 4);
      I.kappa_off = take((int64_t)I.K * 4);
    }
    I.beta_off = take(4 * nq * I.Npad * 4);
    if (some_blocks && blocks_pay(I)) I.xhT_off = take(I.Npad * I.DP * 4);  // (never at 0)
    I.ml_off = ml;
    ml += I.Npad;
    I.fpart_off = fp;
    fp += I.nblk;
    for (int t = 0; (I.split || I.xhT_off) && t < I.Npad / 64; ++t) p.prepx.push_back({(int32_t)b, t, 0, 0});
    for (int k = 0; k < (I.split ? I.K : 4 * nq); ++k) p.prepq.push_back({(int32_t)b, k, 0, 0});
    for (int k = 0; k < I.K; ++k) p.comp.push_back({(int32_t)b, k, 0, 0});
    for (int t = 0; t < I.nblk; ++t) p.merge.push_back({(int32_t)b, t, 0, 0});
  }
  int64_t minch = INT64_MAX;
  for (int c = 0; c < kBBwdCfgs; ++c) {
    int64_t ch = bbwd_chunk(c);
    for (; c == 0 && ch > 512; ch /= 2) {
      int64_t items = 0, most = 0;
      for (const BInst& I : p.inst) {
        items += (I.K + 15) / 16 * ((I.Npad + ch - 1) / ch);
        most = std::max(most, (I.Npad + ch / 2 - 1) / (ch / 2));
      }
      if (items >= kBItems || most > kBChunks) break;
    }
    p.h.bwd_chunk[c] = ch;
    minch = std::min(minch, ch);
  }
  for (BInst& I : p.inst) {
    I.part_off = part;
    part += (I.Npad + minch - 1) / minch * I.K *
            (int64_t)(I.xhT_off ? mom_slot(I.DP) : mom_pack_slot((I.D + 7) & ~7));
    part = (part + 63) / 64 * 64;
  }
  // forward work lists, longest first
  for (int c = 0; c < kBFwdCfgs; ++c) {
    const int pts = 64 * bfwd_cb(c);
    std::vector<std::pair<int64_t, BItem>> v;
    for (int64_t b = 0; b < B; ++b) {
      const BInst& I = p.inst[b];
      for (int t = 0; t < I.Npad / pts; ++t)
        v.push_back({(I.K + 3) / 4 * (int64_t)quad_products((I.D + 7) & ~7) * pts,
                     BItem{(int32_t)b, t, 0, 0}});
    }
    std::stable_sort(v.begin(), v.end(), [](auto& x, auto& y) { return x.first > y.first; });
    for (auto& e : v) p.fwd[c].push_back(e.second);
  }
  p.nch.assign((size_t)kBBwdCfgs * B, 0);
  for (int c = 0; c < kBBwdCfgs; ++c) {
    const int64_t chunk = p.h.bwd_chunk[c];
    std::vector<std::pair<int64_t, BItem>> v, vb;
    for (int64_t b = 0; b < B; ++b) {
      const BInst& I = p.inst[b];
      const int nch = (int)((I.Npad + chunk - 1) / chunk);
      p.nch[(size_t)c * B + b] = nch;
      const int per = I.xhT_off ? 8 : 16;
      for (int g = 0; g < (I.K + per - 1) / per; ++g)
        for (int s = 0; s < nch; ++s) {
          const int64_t pts = std::min<int64_t>(chunk, I.Npad - s * chunk);
          const BItem it{(int32_t)b, g, s, 0};
          if (I.xhT_off)
            vb.push_back({std::min(2, I.K - 8 * g) * pts * (I.DP == 16 ? 1 : 3), it});
          else
            v.push_back({pts * mom_pack_slot((I.D + 7) & ~7), it});
        }
    }
    for (auto* l : {&v, &vb})
      std::stable_sort(l->begin(), l->end(), [](auto& x, auto& y) { return x.first > y.first; });
    for (auto& e : v) p.bwd[c].push_back(e.second);
    for (auto& e : vb) p.blk[c].push_back(e.second);
  }
  // layout of the plan bytes
  size_t o = align256(sizeof(PlanHeader));
  auto place = [&](size_t bytes) {
    size_t at = o;
    o += align256(bytes);
    return (int64_t)at;
  };
  p.h.inst_off = place(p.inst.size() * sizeof(BInst));
  p.h.prepx_off = place(p.prepx.size() * sizeof(BItem));
  p.h.n_prepx = (int64_t)p.prepx.size();
  p.h.prepq_off = place(p.prepq.size() * sizeof(BItem));
  p.h.n_prepq = (int64_t)p.prepq.size();
  p.h.comp_off = place(p.comp.size() * sizeof(BItem));
  p.h.n_comp = (int64_t)p.comp.size();
  p.h.merge_off = place(p.merge.size() * sizeof(BItem));
  p.h.n_merge = (int64_t)p.merge.size();
  for (int c = 0; c < kBFwdCfgs; ++c) {
    p.h.fwd_off[c] = place(p.fwd[c].size() * sizeof(BItem));
    p.h.n_fwd[c] = (int64_t)p.fwd[c].size();
  }
  for (int c = 0; c < kBBwdCfgs; ++c) {
    p.h.bwd_off[c] = place(p.bwd[c].size() * sizeof(BItem));
    p.h.n_bwd[c] = (int64_t)p.bwd[c].size();
    p.h.blk_off[c] = place(p.blk[c].size() * sizeof(BItem));
    p.h.n_blk[c] = (int64_t)p.blk[c].size();
  }
  p.h.nch_off = place(p.nch.size() * sizeof(int32_t));
  p.bytes = o;
  p.h.cache_bytes = cache;
  size_t w = 0;
  p.h.ws_counter = (int64_t)w;  // fixed at offset 0: the host clears it before each phase
  w += 256;
  p.h.ws_ml = (int64_t)w;
  w += align256((size_t)ml * sizeof(float2));
  p.h.ws_fpart = (int64_t)w;
  w += align256((size_t)fp * 2 * sizeof(float));
  p.h.ws_part = (int64_t)w;
  w += align256((size_t)part * sizeof(float));
  p.h.ws_bytes = (int64_t)w;
  return p;
}

}  // namespace

size_t gmm_batched_plan_bytes(int64_t B, const int64_t* shapes, int32_t variant) {
  return build_plan(shapes, B, variant).bytes;
}

// Descriptor dims: {B, sum N, sum K, sum K*D, sum K*L, sum N*D, plan bytes, cache bytes}.
// The item counts and workspace size are recovered from the plan header on
// the host by dex_gmm_batched_plan only; launches use the counts stored in
// fparams (exact integers below 2^53).
dex_status gmm_batched_plan(const int64_t* shapes, int64_t B, int32_t variant, dex_desc* d,
                            void* plan, size_t plan_bytes) {
  PlanBuild p = build_plan(shapes, B, variant);
  int64_t sumN = 0, sumK = 0, sumKD = 0, sumKL = 0, sumND = 0;
  for (int64_t b = 0; b < B; ++b) {
    const int64_t N = shapes[3 * b], D = shapes[3 * b + 1], K = shapes[3 * b + 2];
    sumN += N;
    sumK += K;
    sumKD += K * D;
    sumKL += K * D * (D - 1) / 2;
    sumND += N * D;
  }
  memset(d, 0, sizeof(*d));
  d->kind = DEX_GMM_BATCHED;
  d->dtype = DEX_F32;
  d->variant = variant;
  d->dims[0] = B;
  d->dims[1] = sumN;
  d->dims[2] = sumK;
  d->dims[3] = sumKD;
  d->dims[4] = sumKL;
  d->dims[5] = sumND;
  d->dims[6] = (int64_t)p.bytes;
  d->dims[7] = p.h.cache_bytes;
  // item counts for the launches: prepx (negative where some moments go component by
  // component), merge, ws bytes, prepq; the persistent lists' lengths are read on the
  // device
  d->fparams[0] = p.h.n_blk[0] ? -(double)p.h.n_prepx : (double)p.h.n_prepx;
  d->fparams[1] = (double)p.h.n_merge;
  d->fparams[2] = (double)p.h.ws_bytes;
  d->fparams[3] = (double)p.h.n_prepq;
  if (!plan) return DEX_OK;
  if (plan_bytes < p.bytes) return fail(DEX_ERR_INVALID_ARG, "plan buffer too small");
  char* o = (char*)plan;
  memset(o, 0, p.bytes);
  memcpy(o, &p.h, sizeof(PlanHeader));
  memcpy(o + p.h.inst_off, p.inst.data(), p.inst.size() * sizeof(BInst));
  memcpy(o + p.h.prepx_off, p.prepx.data(), p.prepx.size() * sizeof(BItem));
  memcpy(o + p.h.prepq_off, p.prepq.data(), p.prepq.size() * sizeof(BItem));
  memcpy(o + p.h.comp_off, p.comp.data(), p.comp.size() * sizeof(BItem));
  memcpy(o + p.h.merge_off, p.merge.data(), p.merge.size() * sizeof(BItem));
  for (int c = 0; c < kBFwdCfgs; ++c)
    memcpy(o + p.h.fwd_off[c], p.fwd[c].data(), p.fwd[c].size() * sizeof(BItem));
  for (int c = 0; c < kBBwdCfgs; ++c) {
    memcpy(o + p.h.bwd_off[c], p.bwd[c].data(), p.bwd[c].size() * sizeof(BItem));
    memcpy(o + p.h.blk_off[c], p.blk[c].data(), p.blk[c].size() * sizeof(BItem));
  }
  memcpy(o + p.h.nch_off, p.nch.data(), p.nch.size() * sizeof(int32_t));
  return DEX_OK;
}

size_t gmm_batched_ws_bytes(const dex_desc& d, int role) {
  if (role == DEX_WS_RESID) return (size_t)d.dims[7];
  return (size_t)d.fparams[2];
}

int gmm_batched_num_configs(const dex_desc& d, int role) {
  (void)d;
  return role == DEX_WS_VJP ? kBBwdCfgs : kBFwdCfgs;
}

// FP32 forward of an untuned call: 256 points a block, which reads its records and its
// item once for more of them (100 mixtures of 20000 points, 256 and 128, us: D = 8, K = 2
// 130, 218; D = 16, K = 30 253, 268; D = 24, K = 17 303, 311; D = 32, K = 10 329, 309), but
// 128 where the batch is small and each point's products are many, for an even end (12
// mixtures of 2000, D to 32, K to 100: 99, 75; 64 of 10000: 204, 196; 512 of 25000: 3.39
// ms, 3.53), and where it is smaller still (10 of 300, D = 9, K = 5: 29.2, 27.5).
int gmm_batched_default_config(const dex_desc& d, int role) {
  if (role == DEX_WS_VJP || d.variant != DEX_GMM_PLAIN) return 0;
  const int64_t B = d.dims[0], sumN = d.dims[1], sumK = d.dims[2], sumKD = d.dims[3];
  const int D8 = (int)((sumKD / std::max<int64_t>(sumK, 1) + 7) / 8 * 8);
  const bool heavy = (double)sumK / (4.0 * B) * quad_products(D8) >= 88.0;
  return sumN < (int64_t(1) << 17) || (sumN < (int64_t(1) << 21) && heavy) ? 1 : 0;
}

// Blocks of the persistent launches: as many as a CU holds.
static int persistent_blocks(int per_cu) { return num_cus() * per_cu; }

dex_status gmm_batched_fwd(const dex_desc& d, int cfg, const void* plan, const GmmPtrs& in,
                           void* F, void* f, void* cache, void* ws, hipStream_t st) {
  if (cfg < 0 || cfg >= kBFwdCfgs) return fail(DEX_ERR_INVALID_ARG, "batched forward config");
  const int64_t B = d.dims[0];
  const int64_t n_prepx = std::abs((int64_t)d.fparams[0]), n_merge = (int64_t)d.fparams[1];
  const int64_t n_prepq = (int64_t)d.fparams[3];
  if (n_prepq < 1) return fail(DEX_ERR_INVALID_ARG, "batched GMM: plan of another library version");
  const char* pl = (const char*)plan;
  char* cc = (char*)cache;
  char* w = (char*)ws;
  const bool split = d.variant == DEX_GMM_F16X3;
  hipLaunchKernelGGL(k_bscale, dim3((unsigned)B), dim3(256), 0, st, pl, (const float*)in.means,
                     (const float*)in.qd, (const float*)in.l, cc);
  if (n_prepx > 0)
    hipLaunchKernelGGL(k_bprep_x, dim3((unsigned)n_prepx), dim3(256), 0, st, pl, (const float*)in.x, cc);
  hipLaunchKernelGGL(k_bprep_q, dim3((unsigned)n_prepq), dim3(256), 0, st, pl, (const float*)in.alphas,
                     (const float*)in.means, (const float*)in.qd, (const float*)in.l, cc);
  hipLaunchKernelGGL(fill_counters, dim3(1), dim3(64), 0, st, (int*)w, 64);
  ProfRange pr(DEX_PROF_BGMM_FWD, st);
#define DEX_BF(CB_, S_)                                                                    \
  hipLaunchKernelGGL((k_bgmm_fwd<CB_, S_>), dim3(persistent_blocks(S_ ? 3 : 4)), dim3(256), 0, st, pl, \
                     cfg, (const float*)in.x, (const char*)cc, w)
  if (bfwd_cb(cfg) == 4) {
    if (split)
      DEX_BF(4, true);
    else
      DEX_BF(4, false);
  } else {
    if (split)
      DEX_BF(2, true);
    else
      DEX_BF(2, false);
  }
#undef DEX_BF
  pr.end(1);
  hipLaunchKernelGGL(k_bmerge, dim3((unsigned)n_merge), dim3(256), 0, st, pl, (float*)f, w);
  hipLaunchKernelGGL(k_bfinalize_F, dim3((unsigned)B), dim3(256), 0, st, pl, (const float*)in.alphas,
                     (const char*)w, (float*)F);
  return check_hip(hipGetLastError(), "gmm_batched_fwd");
}

dex_status gmm_batched_vjp(const dex_desc& d, int cfg, const void* plan, const GmmPtrs& in,
                           const void* f, const void* cache, const void* ct, const GmmGrads& out,
                           bool accumulate, void* ws, hipStream_t st) {
  if (cfg < 0 || cfg >= kBBwdCfgs) return fail(DEX_ERR_INVALID_ARG, "batched reverse config");
  if (d.fparams[3] < 1) return fail(DEX_ERR_INVALID_ARG, "batched GMM: plan of another library version");
  const int64_t sumK = d.dims[2];
  const char* pl = (const char*)plan;
  char* w = (char*)ws;
  hipLaunchKernelGGL(fill_counters, dim3(1), dim3(64), 0, st, (int*)w, 64);
  ProfRange pr(DEX_PROF_BGMM_VJP, st);
  hipLaunchKernelGGL(k_bgmm_bwd, dim3(persistent_blocks(3)), dim3(256), 0, st, pl, cfg,
                     (const float*)in.x, (const char*)cache, (const float*)f, w);
  const bool blocks = d.fparams[0] < 0;
  if (blocks)
    hipLaunchKernelGGL(k_bgmm_bwd_blocks, dim3(persistent_blocks(4)), dim3(256), 0, st, pl, cfg,
                       (const char*)cache, (const float*)f, w);
  pr.end(blocks ? 2 : 1);
#define DEX_BFIN(PACK_)                                                                           \
  hipLaunchKernelGGL(k_bbwd_finalize<PACK_>, dim3((unsigned)sumK), dim3(256), 0, st, pl, cfg,     \
                     (const char*)w, (const char*)cache, (const float*)in.alphas,                 \
                     (const float*)in.qd, (const float*)in.l, (const float*)in.means,             \
                     (const float*)ct, (float*)out.d_alphas, (float*)out.d_means,                 \
                     (float*)out.d_qd, (float*)out.d_l, accumulate ? 1 : 0)
  DEX_BFIN(true);
  if (blocks) DEX_BFIN(false);
#undef DEX_BFIN
  return check_hip(hipGetLastError(), "gmm_batched_vjp");
}

}  // namespace dexi
