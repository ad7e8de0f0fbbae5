// Grid kernels of the single-instance FP32 GMM, D <= 32, on quads of components
// (gmm_quad.h): the forward of the PLAIN variant and the forward mode of every variant
// with FP32 storage. N = 20000, D = 32, K = 50: forward 19 us (16x16 blocks of one
// component: 23.6), of which products and vector instructions 10; forward mode 32 us and
// 6 for the records (blocks: 63), of which 18. The rest is the start of a block (records
// and points from memory, then LDS) and uneven rounds.
#include <algorithm>

#include "gmm_host.h"
#include "gmm_quad.h"

namespace dexk {

// Blocks 0 .. 4 ceil(K/4) - 1 prepare a component each, the others a 64-point tile of
// x~^T (the reverse's operand). Every block finds the origin itself (one launch less);
// block 0 keeps it.
template <int D8>
__global__ void __launch_bounds__(256) k_quad_prep(const float* __restrict__ x, int N, int D,
                                                   int Npad, int K,
                                                   const float* __restrict__ alphas,
                                                   const float* __restrict__ means,
                                                   const float* __restrict__ qd,
                                                   const float* __restrict__ l, float* xhT,
                                                   float* __restrict__ rec,
                                                   float* __restrict__ shift) {
  __shared__ float csh[64];
  const int nk = (K + 3) / 4 * 4, b = blockIdx.x;
  QuadPrep<D8, false> p;
  if (b < nk) p.load({alphas, means, qd, l}, {}, D, K, b);
  block_shift(means, K, D, csh);
  if (b == 0 && threadIdx.x < 64) shift[threadIdx.x] = csh[threadIdx.x];
  if (b < nk)
    p.store(D, K, b, csh, rec, rec);
  else
    prep_x_tile<PREC_F32, (D8 + 15) / 16 * 16>(x, N, D, Npad, (b - nk) * 64, nullptr, nullptr, xhT,
                                               nullptr, nullptr, csh);
}

// Block (tile, share): 64 points, the share's quads; one log-sum-exp partial per share
// and point.
template <int D8>
__global__ void __launch_bounds__(256, 4) k_quad_fwd(const float* __restrict__ x,
                                                     const float* __restrict__ shift, int N, int D,
                                                     int Npad, int K,
                                                     const float* __restrict__ rec,
                                                     float* __restrict__ beta,
                                                     float2* __restrict__ ml) {
  __shared__ __attribute__((aligned(16))) float lds[2 * quad_batch<D8>() * quad_floats(D8)];
  const int ks = blockIdx.y, KS = gridDim.y, nq = (K + 3) / 4;
  fwd_quads<D8, 1>(x, shift, N, D, Npad, blockIdx.x * 64, rec, (int)split_lo(ks, nq, KS),
                   (int)split_lo(ks + 1, nq, KS), beta, ml + (size_t)ks * Npad, lds);
}

// A block per component: its parts of both records.
template <int D8>
__global__ void __launch_bounds__(256) k_quad_tan_prep(
    int D, int K, const float* __restrict__ alphas, const float* __restrict__ means,
    const float* __restrict__ qd, const float* __restrict__ l, const float* __restrict__ da,
    const float* __restrict__ dm, const float* __restrict__ dq, const float* __restrict__ dl,
    float* __restrict__ rec, float* __restrict__ trec, float* __restrict__ shift) {
  __shared__ float csh[64];
  QuadPrep<D8, true> p;
  p.load({alphas, means, qd, l}, {da, dm, dq, dl}, D, K, blockIdx.x);
  block_shift(means, K, D, csh);
  if (blockIdx.x == 0 && threadIdx.x < 64) shift[threadIdx.x] = csh[threadIdx.x];
  p.store(D, K, blockIdx.x, csh, rec, trec);
}

// 128 points, two blocks a CU: the lanes of a wave then have two products of their own
// for every operand read (with 64 and four blocks: 73 us for 69, see quad_split).
constexpr int kJvpCB = 2;
template <int D8>
__global__ void __launch_bounds__(256, 2) k_quad_jvp(
    const float* __restrict__ x, const float* __restrict__ shift, int N, int D, int K,
    const float* __restrict__ rec, const float* __restrict__ trec, const float* __restrict__ f,
    double* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) float lds[4 * quad_tan_batch<D8>() * quad_floats(D8)];
  __shared__ double sh[16];
  const int ks = blockIdx.y, KS = gridDim.y, nq = (K + 3) / 4;
  double s = jvp_quads<D8, kJvpCB>(x, shift, N, D, blockIdx.x * 64 * kJvpCB, rec, trec,
                               (int)split_lo(ks, nq, KS), (int)split_lo(ks + 1, nq, KS), f, lds);
  s = block_sum(s, sh);
  if (threadIdx.x == 0) part[(size_t)ks * gridDim.x + blockIdx.x] = s;
}

}  // namespace dexk

namespace dexi {
using namespace dexk;

// Shares for the least modelled time: rounds of resident blocks, each its quads and
// the worth of one for its start. N = 20000, D = 32, K = 50 (one round of 3 shares in the
// forward, 471 blocks in the forward mode): objective and derivative 69 us; N = 1e5, K =
// 200: 617 (with the fewest shares that fill the chip 77 and 715).
static QuadSplit quad_split(const GmmGeom& g, int cb, int per_cu) {
  QuadSplit q;
  const int64_t nq = (g.K + 3) / 4, resident = (int64_t)per_cu * num_cus();
  q.tiles = (g.N + 64 * cb - 1) / (64 * cb);
  int64_t best = INT64_MAX;
  for (int64_t ks = 1; ks <= nq && ks <= kMaxShares; ++ks) {
    const int64_t t = (q.tiles * ks + resident - 1) / resident * ((nq + ks - 1) / ks + 1);
    if (t < best) {
      best = t;
      q.ks = (int)ks;
    }
  }
  return q;
}
QuadSplit quad_fwd_split(const GmmGeom& g) {
  GmmGeom p = g;
  p.N = g.Npad;  // (the merge reads a partial of every padded point)
  return quad_split(p, 1, 4);  // (four blocks of 64 points a CU)
}
QuadSplit quad_jvp_split(const GmmGeom& g) { return quad_split(g, kJvpCB, 2); }

size_t quad_rec_bytes(const GmmGeom& g) {
  return (size_t)((g.K + 3) / 4) * quad_floats((int)(g.D + 7) / 8 * 8) * 4;
}

void quad_prep(const GmmGeom& g, const GmmPtrs& in, float* xhT, float* rec, float* shift,
               hipStream_t st) {
  const dim3 grid((unsigned)((g.K + 3) / 4 * 4 + g.Npad / 64));
  with_d8((int)g.D, [&](auto d8) {
    hipLaunchKernelGGL((k_quad_prep<decltype(d8)::value>), grid, dim3(256), 0, st,
                       (const float*)in.x, (int)g.N, (int)g.D, (int)g.Npad, (int)g.K,
                       (const float*)in.alphas, (const float*)in.means, (const float*)in.qd,
                       (const float*)in.l, xhT, rec, shift);
  });
}

void quad_fwd(const GmmGeom& g, const QuadSplit& q, const float* x, const float* rec,
              const float* shift, float* beta, float2* ml, hipStream_t st) {
  with_d8((int)g.D, [&](auto d8) {
    hipLaunchKernelGGL((k_quad_fwd<decltype(d8)::value>), dim3((unsigned)q.tiles, (unsigned)q.ks),
                       dim3(256), 0, st, x, shift, (int)g.N, (int)g.D, (int)g.Npad, (int)g.K, rec,
                       beta, ml);
  });
}

void quad_jvp(const GmmGeom& g, const QuadSplit& q, const GmmPtrs& in, const GmmGrads& t,
              const float* f, float* rec, float* trec, float* shift, double* part,
              hipStream_t st) {
  with_d8((int)g.D, [&](auto d8) {
    constexpr int D8 = decltype(d8)::value;
    hipLaunchKernelGGL((k_quad_tan_prep<D8>), dim3((unsigned)((g.K + 3) / 4 * 4)), dim3(256), 0, st,
                       (int)g.D, (int)g.K, (const float*)in.alphas, (const float*)in.means,
                       (const float*)in.qd, (const float*)in.l, (const float*)t.d_alphas,
                       (const float*)t.d_means, (const float*)t.d_qd, (const float*)t.d_l, rec,
                       trec, shift);
    hipLaunchKernelGGL((k_quad_jvp<D8>), dim3((unsigned)q.tiles, (unsigned)q.ks), dim3(256), 0, st,
                       (const float*)in.x, shift, (int)g.N, (int)g.D, (int)g.K, rec, trec, f, part);
  });
}

}  // namespace dexi
