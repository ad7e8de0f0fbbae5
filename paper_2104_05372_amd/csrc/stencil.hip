// In-place periodic five-point diffusion loop and its reverse pass, gfx950.
//
// Forward (a State loop, Sec. 2.3.1): for t in 0..T-1,
//   u <- u + c (u[y+1,x] + u[y-1,x] + u[y,x+1] + u[y,x-1] - 4u) + rho sin(u)
// where every read is of the previous field (`get` yields a value, Sec. 5.3.2),
// so each step is a Jacobi sweep into a second buffer. Every `every`-th state
// (t = 0, every, 2 every, ...) is a checkpoint. By default up to eight steps run
// per launch, the levels in between held in registers (stencil_tb); on grids of a few
// columns or rows one step does (TbPlan::one_step).
// Loss L = 1/2 ||u_T - target||^2.
//
// Reverse (ForTranspose runs the loop backwards; GetTranspose/PutTranspose carry
// the cotangent of the state): lam_T = dL (u_T - target), then for t = T-1..0
//   lam_t = S^T lam_{t+1} + rho cos(u_t) lam_{t+1},
// S being the linear diffusion step. The gather form computes S^T lam at each
// cell from its neighbours (S is symmetric); the scatter form is the literal
// transposed loop body, in which every cell adds its weighted cotangent into the
// cells it read (LetIndexingTranspose), with atomics. With the recompute
// variant the states of a checkpoint segment are rebuilt before its adjoint
// steps; only the non-linear term reads them (Sec. 5.3.2).
#include "common.h"
#include "internal.h"

namespace dexk {

// Sine and cosine of the non-linear term, for a row of VW cells per lane.
// x = k pi/2 + r, |r| <= pi/4; sin r and cos r are polynomials in t = r^2
// (minimax fits of the Remez exchange, coefficients rounded to FP32 one after the
// other; 4.0e-9 relative for the sine, 1.2e-10 for the cosine), and k's low bits
// pick one and its sign. Three ways to (k, r), taken by the whole wave:
//   every |x| <= 0.785   k = 0, r = x: six operations a sine instead of about 22
//                        (with the reduction); where the field has been
//                        smoothed, most rows take it
//   |x| <= 2^14          k = rint(2x/pi), r = x - k pi/2 by three fused
//                        multiply-adds (pi/2 in three FP32 parts, Cody and Waite)
//   larger               by lane, Payne and Hanek's way: x = m 2^e with a 24-bit m,
//                        and kTurn[e + 9] holds 2^e (2/pi) modulo 4 in two doubles
// Lanes with the same x get the same bits whichever way their wave goes.
struct Turn {
  double hi, lo;
};
__device__ const Turn kTurn[114] = {
    {0x1.45f306dc9c883p-10, -0x1.6b01ec5417056p-64},
    {0x1.45f306dc9c883p-9, -0x1.6b01ec5417056p-63},
    {0x1.45f306dc9c883p-8, -0x1.6b01ec5417056p-62},
    {0x1.45f306dc9c883p-7, -0x1.6b01ec5417056p-61},
    {0x1.45f306dc9c883p-6, -0x1.6b01ec5417056p-60},
    {0x1.45f306dc9c883p-5, -0x1.6b01ec5417056p-59},
    {0x1.45f306dc9c883p-4, -0x1.6b01ec5417056p-58},
    {0x1.45f306dc9c883p-3, -0x1.6b01ec5417056p-57},
    {0x1.45f306dc9c883p-2, -0x1.6b01ec5417056p-56},
    {0x1.45f306dc9c883p-1, -0x1.6b01ec5417056p-55},
    {0x1.45f306dc9c883p+0, -0x1.6b01ec5417056p-54},
    {-0x1.7419f246c6efbp+0, 0x1.29fc2757d1f53p-54},
    {0x1.17cc1b727220bp+0, -0x1.ac07b1505c159p-54},
    {-0x1.d067c91b1bbebp+0, 0x1.4fe13abe8fa9ap-55}, {0x1.7cc1b727220a9p-2, 0x1.3f84eafa3ea6ap-56},
    {0x1.7cc1b727220a9p-1, 0x1.3f84eafa3ea6ap-55}, {0x1.7cc1b727220a9p+0, 0x1.3f84eafa3ea6ap-54},
    {-0x1.067c91b1bbeadp+0, -0x1.80f62a0b82b2dp-54},
    {0x1.f306dc9c882a5p+0, 0x1.fc2757d1f534ep-55},
    {-0x1.9f246c6efab58p-4, -0x1.ec54170565912p-61},
    {-0x1.9f246c6efab58p-3, -0x1.ec54170565912p-60},
    {-0x1.9f246c6efab58p-2, -0x1.ec54170565912p-59},
    {-0x1.9f246c6efab58p-1, -0x1.ec54170565912p-58},
    {-0x1.9f246c6efab58p+0, -0x1.ec54170565912p-57},
    {0x1.836e4e44152a0p-1, -0x1.ec54170565912p-56},
    {0x1.836e4e44152a0p+0, -0x1.ec54170565912p-55},
    {-0x1.f246c6efab581p-1, 0x1.3abe8fa9a6ee0p-58},
    {-0x1.f246c6efab581p+0, 0x1.3abe8fa9a6ee0p-57}, {0x1.b727220a94fe1p-4, 0x1.d5f47d4d37703p-59},
    {0x1.b727220a94fe1p-3, 0x1.d5f47d4d37703p-58}, {0x1.b727220a94fe1p-2, 0x1.d5f47d4d37703p-57},
    {0x1.b727220a94fe1p-1, 0x1.d5f47d4d37703p-56}, {0x1.b727220a94fe1p+0, 0x1.d5f47d4d37703p-55},
    {-0x1.236377d5ac07bp-1, -0x1.505c1596447e5p-57},
    {-0x1.236377d5ac07bp+0, -0x1.505c1596447e5p-56},
    {0x1.b9391054a7f0ap+0, -0x1.505c1596447e5p-55},
    {-0x1.1b1bbead603d9p-1, 0x1.5f47d4d377037p-55},
    {-0x1.1b1bbead603d9p+0, 0x1.5f47d4d377037p-54},
    {0x1.c9c882a53f84fp+0, -0x1.4170565911f92p-54},
    {-0x1.b1bbead603d8bp-2, 0x1.f47d4d377036ep-56},
    {-0x1.b1bbead603d8bp-1, 0x1.f47d4d377036ep-55},
    {-0x1.b1bbead603d8bp+0, 0x1.f47d4d377036ep-54},
    {0x1.391054a7f09d6p-1, -0x1.70565911f924fp-58},
    {0x1.391054a7f09d6p+0, -0x1.70565911f924fp-57},
    {-0x1.8ddf56b01ec54p+0, -0x1.70565911f924fp-56},
    {0x1.c882a53f84eb0p-1, -0x1.70565911f924fp-55},
    {0x1.c882a53f84eb0p+0, -0x1.70565911f924fp-54},
    {-0x1.bbead603d8a83p-2, 0x1.f534ddc0db629p-58},
    {-0x1.bbead603d8a83p-1, 0x1.f534ddc0db629p-57},
    {-0x1.bbead603d8a83p+0, 0x1.f534ddc0db629p-56}, {0x1.1054a7f09d5f4p-1, 0x1.f534ddc0db629p-55},
    {0x1.1054a7f09d5f4p+0, 0x1.f534ddc0db629p-54},
    {-0x1.df56b01ec5417p+0, -0x1.596447e493ad5p-58},
    {0x1.054a7f09d5f48p-2, -0x1.596447e493ad5p-57},
    {0x1.054a7f09d5f48p-1, -0x1.596447e493ad5p-56},
    {0x1.054a7f09d5f48p+0, -0x1.596447e493ad5p-55},
    {-0x1.f56b01ec54170p+0, -0x1.596447e493ad5p-54},
    {0x1.529fc2757d1f5p-4, 0x1.a6ee06db14acdp-59}, {0x1.529fc2757d1f5p-3, 0x1.a6ee06db14acdp-58},
    {0x1.529fc2757d1f5p-2, 0x1.a6ee06db14acdp-57}, {0x1.529fc2757d1f5p-1, 0x1.a6ee06db14acdp-56},
    {0x1.529fc2757d1f5p+0, 0x1.a6ee06db14acdp-55}, {-0x1.5ac07b1505c16p+0, 0x1.a6ee06db14acdp-54},
    {0x1.4a7f09d5f47d5p+0, -0x1.6447e493ad4cep-55},
    {-0x1.6b01ec5417056p+0, -0x1.6447e493ad4cep-54},
    {0x1.29fc2757d1f53p+0, 0x1.377036d8a5665p-54},
    {-0x1.ac07b1505c159p+0, -0x1.911f924eb5336p-54},
    {0x1.4fe13abe8fa9ap-1, 0x1.bb81b6c52b328p-55}, {0x1.4fe13abe8fa9ap+0, 0x1.bb81b6c52b328p-54},
    {-0x1.603d8a82e0acbp+0, -0x1.11f924eb53362p-55},
    {0x1.3f84eafa3ea6ap+0, -0x1.11f924eb53362p-54},
    {-0x1.80f62a0b82b2dp+0, 0x1.dc0db6295993cp-54},
    {0x1.fc2757d1f534ep-1, -0x1.1f924eb53361ep-56},
    {0x1.fc2757d1f534ep+0, -0x1.1f924eb53361ep-55},
    {-0x1.ec54170565912p-6, 0x1.b6c52b3278872p-64},
    {-0x1.ec54170565912p-5, 0x1.b6c52b3278872p-63},
    {-0x1.ec54170565912p-4, 0x1.b6c52b3278872p-62},
    {-0x1.ec54170565912p-3, 0x1.b6c52b3278872p-61},
    {-0x1.ec54170565912p-2, 0x1.b6c52b3278872p-60},
    {-0x1.ec54170565912p-1, 0x1.b6c52b3278872p-59},
    {-0x1.ec54170565912p+0, 0x1.b6c52b3278872p-58}, {0x1.3abe8fa9a6ee0p-3, 0x1.b6c52b3278872p-57},
    {0x1.3abe8fa9a6ee0p-2, 0x1.b6c52b3278872p-56}, {0x1.3abe8fa9a6ee0p-1, 0x1.b6c52b3278872p-55},
    {0x1.3abe8fa9a6ee0p+0, 0x1.b6c52b3278872p-54},
    {-0x1.8a82e0acb223fp+0, -0x1.24eb53361de38p-55},
    {0x1.d5f47d4d37703p-1, 0x1.b6295993c4390p-55}, {0x1.d5f47d4d37703p+0, 0x1.b6295993c4390p-54},
    {-0x1.505c1596447e5p-2, 0x1.b14acc9e21c82p-56},
    {-0x1.505c1596447e5p-1, 0x1.b14acc9e21c82p-55},
    {-0x1.505c1596447e5p+0, 0x1.b14acc9e21c82p-54},
    {0x1.5f47d4d377037p+0, -0x1.3ad4cd8778df8p-55},
    {-0x1.4170565911f92p+0, -0x1.3ad4cd8778df8p-54},
    {0x1.7d1f534ddc0dbp+0, 0x1.8a5664f10e410p-54},
    {-0x1.05c1596447e49p+0, -0x1.d6a66c3bc6fbep-55},
    {0x1.f47d4d377036ep+0, -0x1.d6a66c3bc6fbep-54},
    {-0x1.70565911f924fp-4, 0x1.2b32788720840p-58},
    {-0x1.70565911f924fp-3, 0x1.2b32788720840p-57},
    {-0x1.70565911f924fp-2, 0x1.2b32788720840p-56},
    {-0x1.70565911f924fp-1, 0x1.2b32788720840p-55},
    {-0x1.70565911f924fp+0, 0x1.2b32788720840p-54},
    {0x1.1f534ddc0db63p+0, -0x1.a99b0ef1bef80p-54},
    {-0x1.c1596447e493bp+0, 0x1.5993c439041fep-55}, {0x1.f534ddc0db629p-2, 0x1.664f10e4107f9p-56},
    {0x1.f534ddc0db629p-1, 0x1.664f10e4107f9p-55}, {0x1.f534ddc0db629p+0, 0x1.664f10e4107f9p-54},
    {-0x1.596447e493ad5p-4, 0x1.93c439041fe51p-59},
    {-0x1.596447e493ad5p-3, 0x1.93c439041fe51p-58},
    {-0x1.596447e493ad5p-2, 0x1.93c439041fe51p-57},
    {-0x1.596447e493ad5p-1, 0x1.93c439041fe51p-56},
    {-0x1.596447e493ad5p+0, 0x1.93c439041fe51p-55}, {0x1.4d377036d8a56p+0, 0x1.93c439041fe51p-54},
    {-0x1.65911f924eb53p+0, -0x1.b0ef1bef806bap-55},
    {0x1.34ddc0db6295ap+0, -0x1.b0ef1bef806bap-54},
};

template <int VW>
struct Cells {
  float v[VW];
};

template <bool SIN, bool COS, int VW>
DEX_DEV void trig(const Cells<VW>& x, Cells<VW>& s, Cells<VW>& c) {
  auto poly = [](float r, float& sn, float& cs) {
    const float t = r * r;
    sn = fmaf(r * t, fmaf(t, fmaf(t, -0x1.9952fap-13f, 0x1.110776p-7f), -0x1.555546p-3f), r);
    cs = fmaf(t, fmaf(t, fmaf(t, fmaf(t, 0x1.99e80cp-16f, -0x1.6c0c28p-10f), 0x1.55554ap-5f), -0.5f), 1.f);
  };
  float m = 0.f;
#pragma unroll
  for (int e = 0; e < VW; ++e) m = fmaxf(m, fabsf(x.v[e]));
  if (__all(m <= 0.785f)) {
#pragma unroll
    for (int e = 0; e < VW; ++e) poly(x.v[e], s.v[e], c.v[e]);
    return;
  }
  const bool huge = !__all(m <= 16384.f);
#pragma unroll
  for (int e = 0; e < VW; ++e) {
    const float xe = x.v[e], kf = rintf(xe * 0x1.45f306p-1f);
    int k = (int)kf;
    float r = fmaf(-kf, 0x1.921fb6p0f, xe);
    r = fmaf(-kf, -0x1.777a5cp-25f, r);
    r = fmaf(-kf, -0x1.ee59dap-50f, r);
    if (huge) {
      if (!(fabsf(xe) <= 16384.f)) {
        const uint32_t b = __float_as_uint(xe);
        const int ex = (int)((b >> 23) & 255u);
        const Turn tn = kTurn[min(ex - 141, 113)];
        const double md = (double)(int)((b & 0x7FFFFFu) | 0x800000u);
        double p = md * tn.hi;
        const double err = fma(md, tn.hi, -p) + md * tn.lo;
        p -= 4.0 * rint(0.25 * p);
        const double kd = rint(p);
        float rr = (float)(((p - kd) + err) * 1.57079632679489661923);
        int kk = (int)kd;
        if (b >> 31) {
          rr = -rr;
          kk = -kk;
        }
        r = rr + (xe - xe);  // an infinity or NaN gives NaN
        k = kk;
      }
    }
    float sn, cs;
    poly(r, sn, cs);
    const bool odd = k & 1;
    if constexpr (SIN)
      s.v[e] = __uint_as_float(__float_as_uint(odd ? cs : sn) ^ ((uint32_t)(k & 2) << 30));
    if constexpr (COS)
      c.v[e] = __uint_as_float(__float_as_uint(odd ? sn : cs) ^ ((uint32_t)((k + 1) & 2) << 30));
  }
}

// rho * sin / cos of one value (the one-step kernels; rows of one cell)
DEX_DEV float sin1(float x) {
  Cells<1> s, c;
  trig<true, false, 1>(Cells<1>{{x}}, s, c);
  return s.v[0];
}
DEX_DEV float cos1(float x) {
  Cells<1> s, c;
  trig<false, true, 1>(Cells<1>{{x}}, s, c);
  return c.v[0];
}

// One step of a cell from the sum of its neighbours, and its adjoint; the fused
// multiply-adds are written out, so that every kernel rounds alike.
DEX_DEV float step1(float u, float sum, float c) { return fmaf(c, fmaf(-4.f, u, sum), u); }
DEX_DEV float adj1(float g, float sum, float c) { return fmaf(1.f - 4.f * c, g, c * sum); }

// Which 256 of a one-step launch's threads a block is. Blocks go to the XCDs in turn; of
// every 512 among the first `runs` an XCD takes 64 that follow each other, so that a row's
// neighbours come from its own L2. Non-linear adjoint, a checkpoint every step, 24 steps,
// in turn / runs of 16 / 64 / 128 / an eighth of the grid: 4096^2 1042 / 899 / 849 / 905 /
// 1019 us, 2048^2 344 / 268 / 259 / 269 / 266.
constexpr unsigned kRun = 64;
DEX_DEV int64_t own_block(unsigned runs) {
  const unsigned b = blockIdx.x, in = b % (8 * kRun);
  return b < runs ? b - in + (in & 7) * kRun + (in >> 3) : b;
}

// One forward step, 4 cells per thread (W % 4 == 0, W >= 8).
__global__ void __launch_bounds__(256) stencil_step_vec(const float* __restrict__ u,
                                                        float* __restrict__ un,
                                                        float* __restrict__ snap, int H, int W,
                                                        float c, float rho, unsigned runs) {
  const int W4 = W >> 2;
  const int64_t t = own_block(runs) * 256 + threadIdx.x;
  if (t >= (int64_t)H * W4) return;
  const int y = (int)(t / W4), x4 = (int)(t % W4);
  const int yn = y == 0 ? H - 1 : y - 1, ys = y == H - 1 ? 0 : y + 1;
  const int x0 = 4 * x4;
  const float4 cc = *reinterpret_cast<const float4*>(u + (int64_t)y * W + x0);
  const float4 nn = *reinterpret_cast<const float4*>(u + (int64_t)yn * W + x0);
  const float4 ss = *reinterpret_cast<const float4*>(u + (int64_t)ys * W + x0);
  const float lf = u[(int64_t)y * W + (x0 == 0 ? W - 1 : x0 - 1)];
  const float rt = u[(int64_t)y * W + (x0 + 4 == W ? 0 : x0 + 4)];
  float4 o;
  o.x = step1(cc.x, ((ss.x + nn.x) + cc.y) + lf, c);
  o.y = step1(cc.y, ((ss.y + nn.y) + cc.z) + cc.x, c);
  o.z = step1(cc.z, ((ss.z + nn.z) + cc.w) + cc.y, c);
  o.w = step1(cc.w, ((ss.w + nn.w) + rt) + cc.z, c);
  if (rho != 0.f) {
    Cells<4> sn, cs;
    trig<true, false, 4>(Cells<4>{{cc.x, cc.y, cc.z, cc.w}}, sn, cs);
    o.x = fmaf(rho, sn.v[0], o.x);
    o.y = fmaf(rho, sn.v[1], o.y);
    o.z = fmaf(rho, sn.v[2], o.z);
    o.w = fmaf(rho, sn.v[3], o.w);
  }
  *reinterpret_cast<float4*>(un + (int64_t)y * W + x0) = o;
  if (snap) *reinterpret_cast<float4*>(snap + (int64_t)y * W + x0) = cc;
}

// ---------------------------------------------------------------------------
// Time-blocked steps: one launch advances the field TB steps.
//
// A step alone is bound by memory (the field read and written, 8 bytes per
// cell, against 5 vector instructions), so TB steps per pass divide the traffic
// by TB. Each wave owns a strip of 64 VW columns (VW per lane) and streams down
// a chunk of rows, keeping the last two rows of every intermediate time level
// in registers: when row i of level 0 arrives, level 1 forms its row i - 1, level
// 2 its row i - 2, ..., level TB its row i - TB, which is stored. Horizontal
// neighbours are the adjacent lanes' registers (wave shifts folded into the
// additions), so there is no LDS, no barrier and no exchange between waves; the
// price is a halo of TB columns on either side of a strip (whole lanes: HL) and
// 2 TB rows read ahead of a chunk's first output row. All indices are periodic,
// so any H, W >= 1 is accepted. Measured per step, 4096^2, against one step per
// launch: forward 6.5 us (24.0), adjoint 6.2 us (23.3); with the non-linear term
// forward 10.6 us (25.8), adjoint 27.6 us (62; stencil_fused); 601 x 333:
// 0.77 us (3.0). Bound by issuing the vector instructions (5 a cell, halo and
// row overlap on top: 1.75 times the cells are computed at 4096^2).
//
// MODE   FWD   u -> u after TB steps; `snap` (if given) receives the input rows,
//              `mid` (TB = 8) the state after four
//        ADJ   cotangent back through TB linear steps
//        ADJI  ADJ, the first cotangent dL (u_T - target) formed on the fly
//        TAN   a state and its tangent together (forward mode)
// NL: rho != 0 (its adjoint is stencil_fused). Products and sums are written as
// explicit fused multiply-adds in the order of the one-step kernels, so every TB, VW
// and MODE rounds alike and results do not depend on how the steps are grouped.
enum { TB_FWD = 0, TB_ADJ = 1, TB_ADJI = 2, TB_TAN = 3 };

struct TbArgs {
  const float* in;    // level 0 (ADJI: u_T; TAN: the state; stencil_fused: the cotangent or u_T)
  const float* in2;   // ADJI: target; TAN: the tangent; stencil_fused: the state TB steps back
  const float* in3;   // stencil_fused, first cotangent: target
  float* out;         // level TB
  float* out2;        // TAN: the tangent's
  float* snap;        // FWD: copy of level 0, or null
  float* mid;         // FWD, TB = 8: level 4, or null
  const float* dL;    // first cotangent
  int H, W, RB, strips, accumulate;
  float c, rho;
};

// Value of the lane below (left neighbour) / above; lanes 0 / 63 get zero.
DEX_DEV float from_left(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, true));
}
DEX_DEV float from_right(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xF, 0xF, true));
}

// Sum of the four neighbours in the order ((south + north) + east) + west.
template <int VW>
DEX_DEV Cells<VW> neighbours(const Cells<VW>& n, const Cells<VW>& c, const Cells<VW>& s) {
  Cells<VW> o;
  const float lf = from_left(c.v[VW - 1]), rt = from_right(c.v[0]);
#pragma unroll
  for (int e = 0; e < VW; ++e)
    o.v[e] = ((s.v[e] + n.v[e]) + (e + 1 < VW ? c.v[(e + 1) % VW] : rt)) +
             (e > 0 ? c.v[(e + VW - 1) % VW] : lf);
  return o;
}

// 4-byte aligned vectors: a strip may start at any column
template <int VW>
struct UVec {
  typedef float T __attribute__((ext_vector_type(VW), aligned(4)));
};
template <>
struct UVec<1> {
  typedef float T;
};

// A wave's strip of columns: x0 + VW (lane - HL) onwards, taken modulo W for the
// loads; lanes HL .. 63 - HL store theirs where they lie inside the grid.
template <int VW>
struct Strip {
  using C = Cells<VW>;
  using U = typename UVec<VW>::T;
  int W, xc, col[VW], nmine;  // nmine: columns this lane stores
  bool whole, even;           // no lane straddles the wrap; every lane stores all or none
  // (x0 + 64 VW may pass 2^31 where W is just below it: unsigned, and compared with W - x0)
  DEX_DEV Strip(int lane, int x0, int HL, int W_) : W(W_) {
    const int off = VW * (lane - HL);
    xc = (int)((uint32_t)x0 + (uint32_t)off);
#pragma unroll
    for (int e = 0; e < VW; ++e) {
      const bool below = off + e < 0 && x0 + off + e < 0;
      const uint32_t a = (uint32_t)x0 + (uint32_t)(off + e), m = (below ? 0u - a : a) % (uint32_t)W;
      col[e] = below && m ? W - (int)m : (int)m;
    }
    whole = __all(col[VW - 1] - col[0] == VW - 1);
    nmine = lane >= HL && lane < 64 - HL && off < W - x0 ? min(VW, W - x0 - off) : 0;
    even = __all(nmine == 0 || nmine == VW);
  }
  DEX_DEV C load(const float* f, int y) const {
    C r;
    const float* row = f + (int64_t)y * W;
    if (VW == 1 || whole) {
      const U v = *reinterpret_cast<const U*>(row + col[0]);
      if constexpr (VW == 1) {
        r.v[0] = v;
      } else {
#pragma unroll
        for (int e = 0; e < VW; ++e) r.v[e] = v[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < VW; ++e) r.v[e] = row[col[e]];
    }
    return r;
  }
  DEX_DEV void store(float* f, int y, const C& r) const {
    float* row = f + (int64_t)y * W + xc;
    if (VW == 1 || even) {
      if (nmine) {
        U v;
        if constexpr (VW == 1) {
          v = r.v[0];
        } else {
#pragma unroll
          for (int e = 0; e < VW; ++e) v[e] = r.v[e];
        }
        *reinterpret_cast<U*>(row) = v;
      }
    } else {
#pragma unroll
      for (int e = 0; e < VW; ++e)
        if (e < nmine) row[e] = r.v[e];
    }
  }
  // r += the row's present values
  DEX_DEV void add(const float* f, int y, C& r) const {
    const float* row = f + (int64_t)y * W + xc;
#pragma unroll
    for (int e = 0; e < VW; ++e)
      if (e < nmine) r.v[e] += row[e];
  }
};

template <int TB, int VW, int MODE, bool NL>
__global__ void __launch_bounds__(256) stencil_tb(TbArgs a) {
  constexpr bool kAdj = MODE == TB_ADJ || MODE == TB_ADJI;
  constexpr bool kTwo = MODE == TB_TAN || MODE == TB_ADJI;  // a second input field
  constexpr bool kTan = MODE == TB_TAN;
  static_assert(!(kAdj && NL), "the non-linear adjoint is stencil_fused");
  constexpr int HL = (TB + VW - 1) / VW;
  using C = Cells<VW>;
  const int lane = threadIdx.x & 63;
  const int wave = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int chunk = wave / a.strips, strip = wave - chunk * a.strips;
  const int y0 = chunk * a.RB;
  if (y0 >= a.H) return;  // (no barrier follows)
  const Strip<VW> sp(lane, strip * VW * (64 - 2 * HL), HL, a.W);
  const int H = a.H;
  const int total = min(a.RB, H - y0) + 2 * TB;  // level-0 rows this wave needs
  const float cw = a.c, rho = a.rho, ac = 1.f - 4.f * a.c;
  const float dL = MODE == TB_ADJI ? a.dL[0] : 0.f;
  int yl = (y0 - TB) % H;  // row of the next load, modulo H
  if (yl < 0) yl += H;
  auto next = [&](int y) { return y + 1 == H ? 0 : y + 1; };

  C sl[2][TB], sl2[2][TB];     // the last two rows of every level (sl2: the tangent's)
  C pf[2], pf2[2];             // rows loaded two ahead
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int e = 0; e < VW; ++e) sl[q][t].v[e] = sl2[q][t].v[e] = 0.f;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    pf[q] = sp.load(a.in, yl);
    if constexpr (kTwo) pf2[q] = sp.load(a.in2, yl);
    yl = next(yl);
  }

  // row i of level 0: P = i % 2; FULL: every level has its rows
  auto advance = [&](auto pc, auto fullc, int i) {
    constexpr int P = decltype(pc)::value;
    constexpr bool FULL = decltype(fullc)::value;
    C s = pf[P], s2;
    pf[P] = sp.load(a.in, yl);
    if constexpr (kTwo) {
      s2 = pf2[P];
      pf2[P] = sp.load(a.in2, yl);
    }
    yl = next(yl);
    if constexpr (MODE == TB_ADJI) {
#pragma unroll
      for (int e = 0; e < VW; ++e) s.v[e] = dL * (s.v[e] - s2.v[e]);
    }
    if constexpr (MODE == TB_FWD) {
      if (a.snap && i >= TB && i < total - TB) sp.store(a.snap, y0 + i - TB, s);
    }
    static_for<TB>([&](auto tc) {
      constexpr int t = decltype(tc)::value;
      if constexpr (MODE == TB_FWD && TB == 8 && t == 4) {  // s: row i - 4 of level 4
        if (a.mid && i - 4 >= TB && i - 4 < total - TB) sp.store(a.mid, y0 + i - 4 - TB, s);
      }
      if (!FULL && i < 2 * (t + 1)) {  // (uniform) level t + 1 has no complete row yet
        if (i >= 2 * t) {
          sl[P][t] = s;
          if constexpr (kTan) sl2[P][t] = s2;
        }
        return;
      }
      const C c = sl[P ^ 1][t];
      C o = neighbours<VW>(sl[P][t], c, s), o2;
      if constexpr (kAdj) {
#pragma unroll
        for (int e = 0; e < VW; ++e) o.v[e] = fmaf(ac, c.v[e], cw * o.v[e]);
      } else {
        C sn, cs;
        if constexpr (NL) trig<true, kTan, VW>(c, sn, cs);
        if constexpr (kTan) {
          const C c2 = sl2[P ^ 1][t];
          o2 = neighbours<VW>(sl2[P][t], c2, s2);
#pragma unroll
          for (int e = 0; e < VW; ++e) o2.v[e] = fmaf(cw, fmaf(-4.f, c2.v[e], o2.v[e]), c2.v[e]);
        }
#pragma unroll
        for (int e = 0; e < VW; ++e) {
          o.v[e] = fmaf(cw, fmaf(-4.f, c.v[e], o.v[e]), c.v[e]);
          if constexpr (NL) {
            o.v[e] = fmaf(rho, sn.v[e], o.v[e]);
            if constexpr (kTan) o2.v[e] = fmaf(rho * cs.v[e], sl2[P ^ 1][t].v[e], o2.v[e]);
          }
        }
      }
      sl[P][t] = s;
      s = o;
      if constexpr (kTan) {
        sl2[P][t] = s2;
        s2 = o2;
      }
    });
    if constexpr (FULL) {
      const int y = y0 + i - 2 * TB;
      if (kAdj && a.accumulate) sp.add(a.out, y, s);
      sp.store(a.out, y, s);
      if constexpr (kTan) sp.store(a.out2, y, s2);
    }
  };
  using F = std::integral_constant<bool, false>;
  using T = std::integral_constant<bool, true>;
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  for (int i = 0; i < 2 * TB; i += 2) {
    advance(P0{}, F{}, i);
    advance(P1{}, F{}, i + 1);
  }
  for (int i = 2 * TB; i < total; i += 2) {
    advance(P0{}, T{}, i);
    if (i + 1 < total) advance(P1{}, T{}, i + 1);
  }
}

// The non-linear adjoint through TB steps, the states it linearizes about rebuilt
// in the same pass from the state TB steps back: nothing but that state and the two
// cotangents crosses memory (storing rho cos(u) of every step cost 2 fields a step,
// 49 us at 4096^2 against 27.6). Forward levels as in stencil_tb; when the centre
// row of level t is complete its sine carries the state on and rho cos(u_t) waits
// in registers for the adjoint level j = TB - 1 - t, which reaches that row 2 j
// row-times later (chains of two-row delays, so that a loop of two rows needs a
// move only between links). Row i of the state, row i - TB + 1 of the first
// cotangent and row i - 2 TB + 1 of the last belong together. Halo: 2 (TB - 1)
// columns, U rows ahead of the first output row. TB = 4: at 8 the delays take 112
// registers and the halo a quarter of the columns.
template <int TB, int VW, bool INIT>
__global__ void __launch_bounds__(256) stencil_fused(TbArgs a) {
  constexpr int U = 2 * (TB - 1) > TB ? 2 * (TB - 1) : TB;
  constexpr int HL = (U + VW - 1) / VW;
  using C = Cells<VW>;
  const int lane = threadIdx.x & 63;
  const int wave = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int chunk = wave / a.strips, strip = wave - chunk * a.strips;
  const int y0 = chunk * a.RB;
  if (y0 >= a.H) return;  // (no barrier follows)
  const Strip<VW> sp(lane, strip * VW * (64 - 2 * HL), HL, a.W);
  const int H = a.H;
  const int total = U + 2 * TB - 1 + min(a.RB, H - y0);
  const float cw = a.c, rho = a.rho, ac = 1.f - 4.f * a.c;
  const float dL = INIT ? a.dL[0] : 0.f;
  auto wrap = [&](int y) {
    y %= H;
    return y < 0 ? y + H : y;
  };
  auto next = [&](int y) { return y + 1 == H ? 0 : y + 1; };
  int yu = wrap(y0 - U), yl = wrap(y0 - U - TB + 1);  // rows of the next loads
  C us[2][TB], ls[2][TB];           // the last two rows of every level
  C dl[2][TB * (TB - 1) / 2 + 1];   // delays: level j's links at j (j - 1) / 2 ...
  C pu[2], pl[2], pt[2];            // rows loaded two ahead
#pragma unroll
  for (int q = 0; q < 2; ++q) {
#pragma unroll
    for (int e = 0; e < VW; ++e) {
#pragma unroll
      for (int t = 0; t < TB; ++t) us[q][t].v[e] = ls[q][t].v[e] = 0.f;
#pragma unroll
      for (int t = 0; t <= TB * (TB - 1) / 2; ++t) dl[q][t].v[e] = 0.f;
    }
    pu[q] = sp.load(a.in2, yu);
    pl[q] = sp.load(a.in, yl);
    if constexpr (INIT) pt[q] = sp.load(a.in3, yl);
    yu = next(yu);
    yl = next(yl);
  }
  auto advance = [&](auto pc, int i) {
    constexpr int P = decltype(pc)::value;
    C s = pu[P], g = pl[P];
    if constexpr (INIT) {
#pragma unroll
      for (int e = 0; e < VW; ++e) g.v[e] = dL * (g.v[e] - pt[P].v[e]);
      pt[P] = sp.load(a.in3, yl);
    }
    pu[P] = sp.load(a.in2, yu);
    pl[P] = sp.load(a.in, yl);
    yu = next(yu);
    yl = next(yl);
    C rc[TB];  // rho cos(u) of level t at its centre row
    static_for<TB>([&](auto tc) {
      constexpr int t = decltype(tc)::value;
      const C c = us[P ^ 1][t];
      C sn, o;
      trig<(t < TB - 1), true, VW>(c, sn, rc[t]);
#pragma unroll
      for (int e = 0; e < VW; ++e) rc[t].v[e] *= rho;
      if constexpr (t < TB - 1) {
        o = neighbours<VW>(us[P][t], c, s);
#pragma unroll
        for (int e = 0; e < VW; ++e)
          o.v[e] = fmaf(rho, sn.v[e], fmaf(cw, fmaf(-4.f, c.v[e], o.v[e]), c.v[e]));
      }
      us[P][t] = s;
      s = o;
    });
    static_for<TB>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      C r = rc[TB - 1 - j];
#pragma unroll
      for (int q = 0; q < j; ++q) {  // two row-times per link
        const C old = dl[P][j * (j - 1) / 2 + q];
        dl[P][j * (j - 1) / 2 + q] = r;
        r = old;
      }
      const C c = ls[P ^ 1][j];
      C o = neighbours<VW>(ls[P][j], c, g);
#pragma unroll
      for (int e = 0; e < VW; ++e)
        o.v[e] = fmaf(r.v[e], c.v[e], fmaf(ac, c.v[e], cw * o.v[e]));
      ls[P][j] = g;
      g = o;
    });
    const int y = y0 + i - (U + 2 * TB - 1);
    if (y >= y0) {
      if (a.accumulate) sp.add(a.out, y, g);
      sp.store(a.out, y, g);
    }
  };
  for (int i = 0; i < total; i += 2) {
    advance(std::integral_constant<int, 0>{}, i);
    if (i + 1 < total) advance(std::integral_constant<int, 1>{}, i + 1);
  }
}

__global__ void __launch_bounds__(256) stencil_step_scalar(const float* __restrict__ u,
                                                           float* __restrict__ un,
                                                           float* __restrict__ snap, int H,
                                                           int W, float c, float rho,
                                                           unsigned runs) {
  const int64_t t = own_block(runs) * 256 + threadIdx.x;
  if (t >= (int64_t)H * W) return;
  const int y = (int)(t / W), x = (int)(t % W);
  const int yn = y == 0 ? H - 1 : y - 1, ys = y == H - 1 ? 0 : y + 1;
  const int xl = x == 0 ? W - 1 : x - 1, xr = x == W - 1 ? 0 : x + 1;
  const float cc = u[t];
  float o = step1(cc, ((u[(int64_t)ys * W + x] + u[(int64_t)yn * W + x]) + u[(int64_t)y * W + xr]) +
                          u[(int64_t)y * W + xl], c);
  if (rho != 0.f) o = fmaf(rho, sin1(cc), o);
  un[t] = o;
  if (snap) snap[t] = cc;
}

// Forward mode, one step of the state and its tangent; one cell per thread.
__global__ void __launch_bounds__(256) stencil_tan_step(const float* __restrict__ u,
                                                        const float* __restrict__ du,
                                                        float* __restrict__ un,
                                                        float* __restrict__ dun, int H, int W,
                                                        float c, float rho, unsigned runs) {
  const int64_t t = own_block(runs) * 256 + threadIdx.x;
  if (t >= (int64_t)H * W) return;
  const int y = (int)(t / W), x = (int)(t % W);
  const int yn = y == 0 ? H - 1 : y - 1, ys = y == H - 1 ? 0 : y + 1;
  const int xl = x == 0 ? W - 1 : x - 1, xr = x == W - 1 ? 0 : x + 1;
  const int64_t is = (int64_t)ys * W + x, in = (int64_t)yn * W + x;
  const int64_t ir = (int64_t)y * W + xr, il = (int64_t)y * W + xl;
  const float cc = u[t], dc = du[t];
  float o = step1(cc, ((u[is] + u[in]) + u[ir]) + u[il], c);
  float d = step1(dc, ((du[is] + du[in]) + du[ir]) + du[il], c);
  if (rho != 0.f) {
    Cells<1> sn, cs;
    trig<true, true, 1>(Cells<1>{{cc}}, sn, cs);
    o = fmaf(rho, sn.v[0], o);
    d = fmaf(rho * cs.v[0], dc, d);
  }
  un[t] = o;
  dun[t] = d;
}

// Adjoint step, gather form: lam = S^T g + rho cos(u) g  (=|+= into out).
__global__ void __launch_bounds__(256) stencil_adj_gather(const float* __restrict__ g,
                                                          const float* __restrict__ u,
                                                          float* __restrict__ out, int H, int W,
                                                          float c, float rho, int accumulate,
                                                          unsigned runs) {
  const int64_t t = own_block(runs) * 256 + threadIdx.x;
  if (t >= (int64_t)H * W) return;
  const int y = (int)(t / W), x = (int)(t % W);
  const int yn = y == 0 ? H - 1 : y - 1, ys = y == H - 1 ? 0 : y + 1;
  const int xl = x == 0 ? W - 1 : x - 1, xr = x == W - 1 ? 0 : x + 1;
  const float gc = g[t];
  // cell (y+1, x) read u[y, x] as its north neighbour, etc.
  float v = adj1(gc, ((g[(int64_t)ys * W + x] + g[(int64_t)yn * W + x]) + g[(int64_t)y * W + xr]) +
                         g[(int64_t)y * W + xl], c);
  if (rho != 0.f) v = fmaf(rho * cos1(u[t]), gc, v);
  out[t] = accumulate ? out[t] + v : v;
}

// Vectorised gather-form adjoint (W % 4 == 0, W >= 8); same arithmetic order.
__global__ void __launch_bounds__(256) stencil_adj_gather_vec(const float* __restrict__ g,
                                                              const float* __restrict__ u,
                                                              float* __restrict__ out, int H,
                                                              int W, float c, float rho,
                                                              int accumulate, unsigned runs) {
  const int W4 = W >> 2;
  const int64_t t = own_block(runs) * 256 + threadIdx.x;
  if (t >= (int64_t)H * W4) return;
  const int y = (int)(t / W4), x4 = (int)(t % W4);
  const int yn = y == 0 ? H - 1 : y - 1, ys = y == H - 1 ? 0 : y + 1;
  const int x0 = 4 * x4;
  const float4 cc = *reinterpret_cast<const float4*>(g + (int64_t)y * W + x0);
  const float4 nn = *reinterpret_cast<const float4*>(g + (int64_t)yn * W + x0);
  const float4 ss = *reinterpret_cast<const float4*>(g + (int64_t)ys * W + x0);
  const float lf = g[(int64_t)y * W + (x0 == 0 ? W - 1 : x0 - 1)];
  const float rt = g[(int64_t)y * W + (x0 + 4 == W ? 0 : x0 + 4)];
  float4 v;
  v.x = adj1(cc.x, ((ss.x + nn.x) + cc.y) + lf, c);
  v.y = adj1(cc.y, ((ss.y + nn.y) + cc.z) + cc.x, c);
  v.z = adj1(cc.z, ((ss.z + nn.z) + cc.w) + cc.y, c);
  v.w = adj1(cc.w, ((ss.w + nn.w) + rt) + cc.z, c);
  if (rho != 0.f) {
    const float4 uu = *reinterpret_cast<const float4*>(u + (int64_t)y * W + x0);
    Cells<4> sn, cs;
    trig<false, true, 4>(Cells<4>{{uu.x, uu.y, uu.z, uu.w}}, sn, cs);
    v.x = fmaf(rho * cs.v[0], cc.x, v.x);
    v.y = fmaf(rho * cs.v[1], cc.y, v.y);
    v.z = fmaf(rho * cs.v[2], cc.z, v.z);
    v.w = fmaf(rho * cs.v[3], cc.w, v.w);
  }
  float4* o = reinterpret_cast<float4*>(out + (int64_t)y * W + x0);
  if (accumulate) {
    float4 p = *o;
    v.x += p.x;
    v.y += p.y;
    v.z += p.z;
    v.w += p.w;
  }
  *o = v;
}

// Adjoint step, scatter form: the transposed loop body literally, each cell
// accumulating its weighted cotangent into the five cells it read. `out`
// must hold zero (or the value to accumulate onto) on entry.
__global__ void __launch_bounds__(256) stencil_adj_scatter(const float* __restrict__ g,
                                                           const float* __restrict__ u,
                                                           float* __restrict__ out, int H,
                                                           int W, float c, float rho) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)H * W) return;
  const int y = (int)(t / W), x = (int)(t % W);
  const int yn = y == 0 ? H - 1 : y - 1, ys = y == H - 1 ? 0 : y + 1;
  const int xl = x == 0 ? W - 1 : x - 1, xr = x == W - 1 ? 0 : x + 1;
  const float gc = g[t];
  float self = (1.f - 4.f * c) * gc;
  if (rho != 0.f) self += rho * cos1(u[t]) * gc;
  atomicAdd(&out[t], self);
  atomicAdd(&out[(int64_t)ys * W + x], c * gc);
  atomicAdd(&out[(int64_t)yn * W + x], c * gc);
  atomicAdd(&out[(int64_t)y * W + xr], c * gc);
  atomicAdd(&out[(int64_t)y * W + xl], c * gc);
}

// Per-block partial sums of (u - target)(du - dtarget) in FP64: the tangent of
// L = 1/2 ||u - target||^2.
__global__ void __launch_bounds__(256) stencil_tan_loss_partial(const float* __restrict__ u,
                                                                const float* __restrict__ tg,
                                                                const float* __restrict__ du,
                                                                const float* __restrict__ dtg,
                                                                int64_t n,
                                                                double* __restrict__ part) {
  __shared__ double sh[16];
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    s += ((double)u[i] - (double)tg[i]) * ((double)du[i] - (double)dtg[i]);
  s = block_sum(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ void stencil_sum_final(const double* __restrict__ part, int nb, float* __restrict__ out) {
  __shared__ double sh[16];
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) s += part[i];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) out[0] = (float)s;
}

// Per-block partial sums of (u - target)^2 in FP64.
__global__ void __launch_bounds__(256) stencil_loss_partial(const float* __restrict__ u,
                                                            const float* __restrict__ tg,
                                                            int64_t n, double* __restrict__ part) {
  __shared__ double sh[16];
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const double d = (double)u[i] - (double)tg[i];
    s += d * d;
  }
  s = block_sum(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ void stencil_loss_final(const double* __restrict__ part, int nb, float* __restrict__ L) {
  __shared__ double sh[16];
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) s += part[i];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) L[0] = (float)(0.5 * s);
}

// lam = dL * (u - target)
__global__ void __launch_bounds__(256) stencil_lam_init(const float* __restrict__ u,
                                                        const float* __restrict__ tg,
                                                        const float* __restrict__ dL, int64_t n,
                                                        float* __restrict__ lam) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) lam[i] = dL[0] * (u[i] - tg[i]);
}

__global__ void __launch_bounds__(256) copy_f32(const float* __restrict__ a, float* __restrict__ b,
                                                int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) b[i] = a[i];
}

__global__ void __launch_bounds__(256) add_f32(const float* __restrict__ a, float* __restrict__ b,
                                               int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) b[i] += a[i];
}

}  // namespace dexk

// ===========================================================================
namespace dexi {
using namespace dexk;

namespace {
constexpr int kLossBlocks = 1024;

struct St {
  int H, W, T, every, nck;
  float c, rho;
  int64_t n;
  bool vec;
};

St st_of(const dex_desc& d) {
  St s;
  s.H = (int)d.dims[0];
  s.W = (int)d.dims[1];
  s.T = (int)d.dims[2];
  s.every = (int)d.dims[3];
  s.nck = s.every > 0 ? (s.T + s.every - 1) / s.every : 0;
  s.c = (float)d.fparams[0];
  s.rho = (float)d.fparams[1];
  s.n = (int64_t)s.H * s.W;
  s.vec = (s.W % 4) == 0 && s.W >= 8;
  return s;
}

// Steps per launch are powers of two up to kTB: a stretch of n steps runs as
// n / kTB launches of kTB steps and the binary digits of the rest.
constexpr int kTB = 8, kFused = 4;  // (kFused: the non-linear adjoint)
int tb_of(int left) {
  int tb = kTB;
  while (tb > left) tb >>= 1;
  return tb;
}
int tb_pieces(int n) { return n / kTB + __builtin_popcount(n % kTB); }

template <int MODE, int TB, int VW>
void tb_launch(const TbArgs& a, bool nl, int blocks, hipStream_t st) {
  if constexpr (MODE == TB_ADJ || MODE == TB_ADJI) {
    hipLaunchKernelGGL((stencil_tb<TB, VW, MODE, false>), dim3(blocks), dim3(256), 0, st, a);
  } else {
    if (nl)
      hipLaunchKernelGGL((stencil_tb<TB, VW, MODE, true>), dim3(blocks), dim3(256), 0, st, a);
    else
      hipLaunchKernelGGL((stencil_tb<TB, VW, MODE, false>), dim3(blocks), dim3(256), 0, st, a);
  }
}

template <int TB, int VW>
void fused_launch(const TbArgs& a, int blocks, hipStream_t st) {
  if (a.in3)
    hipLaunchKernelGGL((stencil_fused<TB, VW, true>), dim3(blocks), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((stencil_fused<TB, VW, false>), dim3(blocks), dim3(256), 0, st, a);
}

// Launch shape of a tb-step launch on a grid: columns per lane, rows per wave,
// strips; and the modelled time of one of its steps. row: the least cycles that a wave
// spends on a row, whatever its levels.
struct TbShape {
  int vw, rb, strips;
  double us;
};
TbShape tb_shape(const St& s, int tb, bool fused, double row) {
  const bool nl = s.rho != 0.f;
  const int halo = fused ? std::max(2 * (tb - 1), tb) : tb;
  const double warm = fused ? halo + 2.0 * tb - 1.0 : 1.5 * tb;
  // Columns per lane (1 or 2) and rows per wave: the least modelled time, over the
  // heights that give every SIMD the same whole number n of waves. A wave takes rb +
  // warm row-times, tb levels each; a level is about ins vector instructions, which
  // several waves of a SIMD issue every 4.4 cycles and one wave by itself (a dependent
  // chain, nothing to hide its loads) every 14 or so. Wide lanes waste fewer halo
  // columns (112 of 128 kept against 48 of 64 at tb = 8), narrow ones give small grids
  // more waves. Measured per step (forward rho = 0; rho != 0; adjoint rho != 0), for
  // the lone wave's interval taken as 7, 14 +- 2 and 22: 4096^2 7.6, 6.5, 6.3; 11.9,
  // 10.7, 10.2; 31.5, 27.6, 29.7 us; 1024^2 1.30, 1.30, 1.39; 2.60, 2.54, 2.78; 5.77,
  // 5.57, 6.35 us; 601 x 333 within 2% throughout. Heights from a fixed list, which
  // leave the last waves of a SIMD alone: 4096^2 6.3, 10.5 and 32.7 us.
  const int simds = 4 * num_cus();
  TbShape g{2, 32, 0, 0.0};
  double best = 1e300;
  for (int v = 1; v <= 2; ++v) {
    const int wv = v * (64 - 2 * ((halo + v - 1) / v));
    const int64_t strips = ((int64_t)s.W + wv - 1) / wv;
    // (a launch of 2^31 threads and more runs only in part; wide lanes stay below)
    if (v == 1 && strips * 64 > (int64_t(1) << 30)) continue;
    const double ins = fused ? 27.0 * v + 8.0 : nl ? 14.0 * v + 6.0 : 5.5 * v + 2.5;
    for (int n = 1; n <= 16; ++n) {  // waves per SIMD
      const int64_t chunks = std::max<int64_t>(1, (int64_t)n * simds / strips);
      const int r = (int)std::max<int64_t>(4, (s.H + chunks - 1) / chunks);
      const int64_t per_simd = (strips * ((s.H + r - 1) / r) + simds - 1) / simds;
      const double t =
          (r + warm) * std::max(row, tb * ins * std::max(14.0, 4.4 * (double)per_simd));
      if (t < best) {
        best = t;
        // (what the levels compute: the forward ones skip the rows they do not have yet)
        const double rows = std::min(r, s.H) + (fused ? warm : tb - 1.0);
        g = {v, r, (int)strips, rows * ins * std::max(14.0, 4.4 * (double)per_simd) / 2800.0};
      }
    }
  }
  return g;
}

// The shapes of one call's launches, found once per number of steps.
struct TbPlan {
  // A wave of the forward kernel is taken to need 900 cycles for a row, as long as its
  // load and its store (with one or two levels there is no more to do meanwhile), so that
  // short stretches get more waves: a checkpoint every step, 24 steps of 4096 x 4095 794 us
  // (0: 921), 8192 x 2047 798 (906), 1536 x 1535 182 (174); every 5th, 2048^2 139 (151); every
  // 2nd, 2048^2 132 (122), 1024^2 68 (71). The adjoint reads a row as far ahead as its levels
  // let it and loses by it.
  static constexpr double kFwdRow = 900.0;
  const St& s;
  TbShape shape[3][4];
  explicit TbPlan(const St& s_) : s(s_), shape{} {}
  const TbShape& at(int tb, bool fused) {
    TbShape& g = shape[fused][__builtin_ctz(tb)];
    if (!g.vw) g = tb_shape(s, tb, fused, 0.0);
    return g;
  }
  const TbShape& fwd_at(int tb) {
    TbShape& g = shape[2][__builtin_ctz(tb)];
    if (!g.vw) g = tb_shape(s, tb, false, kFwdRow);
    return g;
  }
  // Whether a call whose stretches are of `len` steps goes one step a launch. A strip is
  // 48 or 112 columns and a halo, and a chunk some rows and 2 tb more, so on columns or
  // rows by themselves the time-blocked kernels compute many times their cells: 1.6e7 x 1
  // cells 196 us a step (one-step kernel 34), 4e6 x 4 with the sine 107 (35), 1 x 1.6e7
  // with the sine 55 (22). Modelled, us a step: one-step kernels by a launch and what they
  // read and write (four cells a thread, or one), the others by their instructions; the
  // factors are those of measured grids from 1 x 1e6 to 4096^2. The sine's adjoint of one
  // step by itself only loses by the blocked form (a checkpoint every step, 24 steps of
  // 601 x 333: 69 us, 93).
  enum Pass { FWD, TAN, ADJ };
  bool one_step(int len, Pass pass) {
    const int tb = tb_of(len);
    const bool nl = s.rho != 0.f;
    if (tb <= 1) return pass == ADJ && nl;
    auto one = [&](double fields, bool vec) {
      return std::max(3.0, 2.2 + (double)s.n * fields * (vec ? 0.72e-6 : 1.05e-6));
    };
    const double blocked = at(tb, false).us;
    if (pass == TAN) return blocked * (nl ? 1.5 : 2.1) > one(nl ? 3.1 : 2.7, false);
    if (pass == FWD || !nl) return blocked > one(2.0, s.vec);
    // the sine's adjoint, with the states it rebuilds
    const int tf = std::min(tb, kFused);
    const double again = (double)((len + tf - 1) / tf - 1) * tf / len;
    return at(tf, true).us + again * blocked >
           one(3.0, s.vec) + (len - 1.0) / len * one(2.0, s.vec);
  }
  // The launch's arguments from its shape; returns its blocks.
  int fill(const TbShape& g, TbArgs& a) const {
    a.H = s.H;
    a.W = s.W;
    a.c = s.c;
    a.rho = s.rho;
    a.RB = g.rb;
    a.strips = g.strips;
    return (int)(((int64_t)g.strips * ((s.H + g.rb - 1) / g.rb) + 3) / 4);
  }
};

// One launch of tb steps (a power of two up to kTB).
template <int MODE>
void tb_steps(TbPlan& plan, int tb, TbArgs a, hipStream_t st) {
  const TbShape& g = MODE == TB_FWD ? plan.fwd_at(tb) : plan.at(tb, false);
  const bool nl = plan.s.rho != 0.f;
  const int vw = g.vw, blocks = plan.fill(g, a);
#define DEX_TB(T_)                                     \
  (vw == 2 ? tb_launch<MODE, T_, 2>(a, nl, blocks, st) \
           : tb_launch<MODE, T_, 1>(a, nl, blocks, st))
  switch (tb) {
    case 8:
      DEX_TB(8);
      break;
    case 4:
      DEX_TB(4);
      break;
    case 2:
      DEX_TB(2);
      break;
    default:
      DEX_TB(1);
  }
#undef DEX_TB
}

// One launch of the non-linear adjoint through tb steps (up to kFused).
void fused_steps(TbPlan& plan, int tb, TbArgs a, hipStream_t st) {
  const TbShape& g = plan.at(tb, true);
  const int blocks = plan.fill(g, a);
#define DEX_FU(T_) \
  (g.vw == 2 ? fused_launch<T_, 2>(a, blocks, st) : fused_launch<T_, 1>(a, blocks, st))
  if (tb == 4)
    DEX_FU(4);
  else if (tb == 2)
    DEX_FU(2);
  else
    DEX_FU(1);
#undef DEX_FU
}

// Blocks of a one-step launch that go in runs (own_block): whole groups of runs; none where
// a block holds a row's neighbours itself or a run holds no two rows (1e6 x 1 with the sine
// 138 us, 144 in runs; 2 x 500000 back 229, 265).
unsigned run_blocks(const St& s, bool vec) {
  const int64_t row = vec ? s.W / 4 : s.W, nb = ((int64_t)s.H * row + 255) / 256;
  return row >= 64 && row <= 128 * kRun ? (unsigned)(nb / (8 * kRun) * (8 * kRun)) : 0u;
}

// One step by itself.
void step(const St& s, const float* u, float* un, float* snap, hipStream_t st) {
  if (s.vec) {
    const int64_t nt = s.n / 4;
    hipLaunchKernelGGL(stencil_step_vec, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, st, u,
                       un, snap, s.H, s.W, s.c, s.rho, run_blocks(s, true));
  } else {
    hipLaunchKernelGGL(stencil_step_scalar, dim3((unsigned)((s.n + 255) / 256)), dim3(256), 0, st,
                       u, un, snap, s.H, s.W, s.c, s.rho, run_blocks(s, false));
  }
}

// One adjoint step; form: 1 scatter, else gather.
void adj(const St& s, int form, const float* g, const float* u, float* out, bool accumulate,
         hipStream_t st) {
  const unsigned nb = (unsigned)((s.n + 255) / 256);
  if (form == 1) {
    if (!accumulate) fill_zero(out, (size_t)s.n * 4, st);
    hipLaunchKernelGGL(stencil_adj_scatter, dim3(nb), dim3(256), 0, st, g, u, out, s.H, s.W, s.c,
                       s.rho);
  } else if (s.vec) {
    hipLaunchKernelGGL(stencil_adj_gather_vec, dim3((unsigned)((s.n / 4 + 255) / 256)), dim3(256),
                       0, st, g, u, out, s.H, s.W, s.c, s.rho, accumulate ? 1 : 0,
                       run_blocks(s, true));
  } else {
    hipLaunchKernelGGL(stencil_adj_gather, dim3(nb), dim3(256), 0, st, g, u, out, s.H, s.W, s.c,
                       s.rho, accumulate ? 1 : 0, run_blocks(s, false));
  }
}
}  // namespace

size_t stencil_ws_bytes(const dex_desc& d, int role) {
  St s = st_of(d);
  const size_t fb = align256((size_t)s.n * 4);
  if (role == DEX_WS_FWD) return fb + align256(kLossBlocks * 8);
  if (role == DEX_WS_JVP) return 4 * fb + align256(kLossBlocks * 8);  // (u, du) ping-pong
  if (role == DEX_WS_VJP) {
    size_t b = 2 * fb;  // cotangent ping-pong
    if (d.variant == DEX_STENCIL_RECOMPUTE) b += (size_t)(s.every > 1 ? s.every - 1 : 0) * fb + fb;
    return b;
  }
  return 0;
}

int stencil_num_configs(const dex_desc& d, int role) {
  (void)d;
  // fwd: 0 time-blocked kernel, 1 vector kernel; vjp: 0 gather form,
  // time-blocked, 1 scatter form, 2 gather form with vector kernels
  return role == DEX_WS_VJP ? 3 : 2;
}

dex_status stencil_fwd(const dex_desc& d, int cfg, const float* u0, const float* target, float* L,
                       float* uT, float* ckpt, void* ws, hipStream_t st) {
  St s = st_of(d);
  float* other = (float*)ws;
  double* part = (double*)((char*)ws + align256((size_t)s.n * 4));
  const float* cur = u0;
  ProfRange pr(DEX_PROF_STENCIL_FWD, st);
  TbPlan plan(s);
  const bool one = cfg != 0 || plan.one_step(std::min(s.every, s.T), TbPlan::FWD);
  // each stretch between checkpoints ends in the next one's storage (the last
  // in uT); its inner launches alternate between uT and the workspace field,
  // the one before uT's writing the workspace. The first launch also copies
  // u0 to its checkpoint.
  for (int sg = 0; sg < s.nck; ++sg) {
    const int len = std::min(s.every, s.T - sg * s.every);
    const bool last = sg == s.nck - 1;
    int pieces = one ? len : tb_pieces(len);
    for (int left = len; left > 0; --pieces) {
      const int tb = one ? 1 : tb_of(left);
      left -= tb;
      TbArgs a{};
      a.in = cur;
      a.out = left == 0 ? (last ? uT : ckpt + (int64_t)(sg + 1) * s.n)
                        : (pieces % 2 == 0 ? other : uT);
      if (sg == 0 && left + tb == len) a.snap = ckpt;
      // (one step by itself: 2048^2, a checkpoint every step, 24 steps 193 us, blocked 266)
      if (one || (tb == 1 && s.vec))
        step(s, a.in, a.out, a.snap, st);
      else
        tb_steps<TB_FWD>(plan, tb, a, st);
      cur = a.out;
    }
  }
  pr.end(s.T);
  if (s.T == 0) {
    hipLaunchKernelGGL(copy_f32, dim3((unsigned)((s.n + 255) / 256)), dim3(256), 0, st, u0, uT, s.n);
  }
  hipLaunchKernelGGL(stencil_loss_partial, dim3(kLossBlocks), dim3(256), 0, st, uT, target, s.n, part);
  hipLaunchKernelGGL(stencil_loss_final, dim3(1), dim3(256), 0, st, part, kLossBlocks, L);
  return check_hip(hipGetLastError(), "stencil_fwd");
}

// Forward mode: tL = <u_T - target, du_T - dtarget>, the primal and tangent
// states stepped together through the workspace ping-pong buffers.
dex_status stencil_jvp(const dex_desc& d, const float* u0, const float* target, const float* du0,
                       const float* dtarget, float* tL, void* ws, hipStream_t st) {
  St s = st_of(d);
  const size_t fb = align256((size_t)s.n * 4);
  float* buf[2][2] = {{(float*)ws, (float*)((char*)ws + fb)},
                      {(float*)((char*)ws + 2 * fb), (float*)((char*)ws + 3 * fb)}};
  double* part = (double*)((char*)ws + 4 * fb);
  const float *u = u0, *du = du0;
  TbPlan plan(s);
  const bool one = plan.one_step(s.T, TbPlan::TAN);
  for (int left = s.T, q = 0; left > 0; q ^= 1) {
    const int tb = one ? 1 : tb_of(left);
    left -= tb;
    TbArgs a{};
    a.in = u;
    a.in2 = du;
    a.out = buf[q][0];
    a.out2 = buf[q][1];
    if (one)
      hipLaunchKernelGGL(stencil_tan_step, dim3((unsigned)((s.n + 255) / 256)), dim3(256), 0, st, u,
                         du, a.out, a.out2, s.H, s.W, s.c, s.rho, run_blocks(s, false));
    else
      tb_steps<TB_TAN>(plan, tb, a, st);
    u = a.out;
    du = a.out2;
  }
  hipLaunchKernelGGL(stencil_tan_loss_partial, dim3(kLossBlocks), dim3(256), 0, st, u, target, du,
                     dtarget, s.n, part);
  hipLaunchKernelGGL(stencil_sum_final, dim3(1), dim3(256), 0, st, part, kLossBlocks, tL);
  return check_hip(hipGetLastError(), "stencil_jvp");
}

// [a, a + na) and [b, b + nb) do not meet.
static bool apart_from(const float* a, int64_t na, const float* b, int64_t nb) {
  return (uintptr_t)(a + na) <= (uintptr_t)b || (uintptr_t)(b + nb) <= (uintptr_t)a;
}

// uT_in: the forward's final state (second residual).
dex_status stencil_vjp(const dex_desc& d, int cfg, const float* u0, const float* target,
                       const float* ckpt, const float* uT_in, const float* dL, float* du0,
                       bool accumulate, void* ws, hipStream_t st) {
  (void)u0;
  St s = st_of(d);
  const int form = cfg;
  const size_t fb = align256((size_t)s.n * 4);
  float* lamA = (float*)ws;
  float* lamB = (float*)((char*)ws + fb);
  // recompute: a segment's states u_{s0+1} .. u_{s0+len-1} (vector and scatter
  // forms), or those its pieces start from (time-blocked form)
  float* seg = (float*)((char*)ws + 2 * fb);
  const unsigned nb = (unsigned)((s.n + 255) / 256);
  if (s.T == 0) {
    if (accumulate) {
      // du0 += dL (u0 - target)
      hipLaunchKernelGGL(stencil_lam_init, dim3(nb), dim3(256), 0, st, uT_in, target, dL, s.n, lamA);
      hipLaunchKernelGGL(stencil_adj_gather, dim3(nb), dim3(256), 0, st, lamA, nullptr, du0, s.H,
                         s.W, 0.f, 0.f, 1, 0u);
    } else {
      hipLaunchKernelGGL(stencil_lam_init, dim3(nb), dim3(256), 0, st, uT_in, target, dL, s.n, du0);
    }
    return check_hip(hipGetLastError(), "stencil_vjp");
  }
  const bool recompute = d.variant == DEX_STENCIL_RECOMPUTE;
  // du0 over a buffer that the last time-blocked launch reads (its rows feed other waves'
  // cells): that launch writes scratch, from where the field is copied or added
  const bool apart = apart_from(du0, s.n, uT_in, s.n) && apart_from(du0, s.n, target, s.n) &&
                     apart_from(du0, s.n, ckpt, (int64_t)s.nck * s.n);
  if (!recompute && s.rho != 0.f)
    return fail(DEX_ERR_INVALID_ARG, "the no-recompute reverse pass needs rho == 0");
  float* g = lamA;
  float* o = lamB;
  int64_t launches = 0;
  TbPlan plan(s);
  const bool nl = s.rho != 0.f;
  // With rho = 0 the adjoint steps read no state: they go through all steps as one
  // stretch, whatever the checkpoints (one every step, 32 steps of 2048^2: 293 us when it
  // ended at each).
  const int stretch = nl ? std::min(s.every, s.T) : s.T;
  if (form == 0 && !plan.one_step(stretch, TbPlan::ADJ)) {
    ProfRange pr(DEX_PROF_STENCIL_VJP, st);
    const int64_t fe = (int64_t)(fb / 4);
    bool first = true;
    for (int sg = nl ? s.nck - 1 : 0; sg >= 0; --sg) {
      const int s0 = sg * s.every;
      const int len = std::min(stretch, s.T - s0);
      const float* ck = ckpt + (int64_t)sg * s.n;
      // rho != 0: the segment goes in pieces of kFused steps and the binary digits of
      // the rest; the states they start from (the first is the checkpoint, the m-th
      // seg + (m - 1) fe) are rebuilt first, two pieces a launch where they can.
      const int lim = nl ? kFused : kTB;
      if (nl) {
        const int full = len / kFused;  // pieces of kFused steps
        const int starts = full + __builtin_popcount(len % kFused);
        for (int m = 1; m < starts;) {
          TbArgs a{};
          a.in = m == 1 ? ck : seg + (m - 2) * fe;
          int tb = kFused;
          if (m + 1 < starts && m + 1 <= full) {
            tb = 2 * kFused;
            a.mid = seg + (m - 1) * fe;
            ++m;
          } else if (m > full) {
            tb = 1 << (31 - __builtin_clz(len % kFused));
          }
          a.out = seg + (m - 1) * fe;
          ++m;
          tb_steps<TB_FWD>(plan, tb, a, st);
          launches += tb;
        }
      }
      // pieces from the segment's end: the smallest digit of the rest first
      for (int left = len, m = nl ? len / kFused + __builtin_popcount(len % kFused) - 1 : 0; left > 0; --m) {
        int tb;
        if (nl)
          tb = left % lim ? left & -left : lim;
        else
          tb = tb_of(left);
        left -= tb;
        const bool last = sg == 0 && left == 0;
        TbArgs a{};
        a.in = first ? uT_in : g;
        a.out = last && apart ? du0 : o;
        a.accumulate = last && apart && accumulate;
        a.dL = dL;
        if (nl) {
          a.in2 = m == 0 ? ck : seg + (m - 1) * fe;
          a.in3 = first ? target : nullptr;
          fused_steps(plan, tb, a, st);
        } else if (first) {
          a.in2 = target;
          tb_steps<TB_ADJI>(plan, tb, a, st);
        } else {
          tb_steps<TB_ADJ>(plan, tb, a, st);
        }
        first = false;
        launches += tb;
        std::swap(g, o);
      }
    }
    if (!apart) {  // (g: the last launch's field)
      if (accumulate)
        hipLaunchKernelGGL(add_f32, dim3(nb), dim3(256), 0, st, g, du0, s.n);
      else
        hipLaunchKernelGGL(copy_f32, dim3(nb), dim3(256), 0, st, g, du0, s.n);
    }
    pr.end(launches);
    return check_hip(hipGetLastError(), "stencil_vjp");
  }
  hipLaunchKernelGGL(stencil_lam_init, dim3(nb), dim3(256), 0, st, uT_in, target, dL, s.n, lamA);
  ProfRange pr(DEX_PROF_STENCIL_VJP, st);
  for (int sg = s.nck - 1; sg >= 0; --sg) {
    const int s0 = sg * s.every;
    const int len = std::min(s.every, s.T - s0);
    const float* ck = ckpt + (int64_t)sg * s.n;
    const bool rebuild = recompute && (nl || form != 0);
    if (rebuild) {
      // rebuild u_{s0+1} .. u_{s0+len-1} from the checkpoint
      const float* cur = ck;
      for (int q = 1; q < len; ++q) {
        float* dst = seg + (int64_t)(q - 1) * (fb / 4);
        step(s, cur, dst, nullptr, st);
        cur = dst;
        ++launches;
      }
    }
    for (int q = len - 1; q >= 0; --q) {
      const int t = s0 + q;
      const float* ut = nullptr;
      if (rebuild) ut = q == 0 ? ck : seg + (int64_t)(q - 1) * (fb / 4);
      const bool last = (t == 0);
      float* dst = last ? du0 : o;
      adj(s, form, g, ut, dst, last && accumulate, st);
      ++launches;
      if (!last) std::swap(g, o);
    }
  }
  pr.end(launches);
  return check_hip(hipGetLastError(), "stencil_vjp");
}

}  // namespace dexi
