// Path-replay backward of the render (models 0..4) and of the projection.
//
// composite_bwd: each wave re-walks its 8x8 block's splats front to back
// exactly as the forward did (the same records staged in LDS in the same
// order, the same float32 decisions), rebuilding each pixel's state from the start instead of
// storing anything per splat.  The adjoint of every composited splat comes
// from quantities the forward left per pixel:
//   exponential   dL/dalpha_i = T_i E_i - R_{i+1} / (1 - alpha_i), with the
//                 radiance behind the splat R_{i+1} = L - sum_{j<=i} E_j p_j
//                 (the last composited splat uses T_k (E_k - L_b));
//   linear and    dL/dalpha_i = (E_i - E_k)(1 + c tau_i) + c Theta_i,
//   quadratic     Theta_i = sum_{i<j<k} (E_j - E_k) alpha_j, rebuilt from its
//                 total U - E_k tau_k; dL/dalpha_k = 0 for the saturating
//                 splat (appendix "Adjoints": eq. generalized_gaussians_gen
//                 and the two recursions that follow it);
//   every model   dL/dE_i = p_i.
// The final transmittance rides along as a fourth channel with emission 0 and
// background 1, so dLoss/dtrans needs no separate code.  Each splat's
// per-pixel moments alpha dL/dalpha (1, dx, dy, dx^2, dx dy, dy^2) and
// p (dL/dL_rgb) are summed over the wave and added once per wave into its
// slot (dx, dy: the pixel centre relative to the splat's).
//
// project_bwd: one thread per Gaussian turns each view's slot moments into
// dL/d(opacity, centre, conic, colour) (written back to the slot) and chains
// them through the conic inverse, the EWA covariance, the perspective
// Jacobian, the rotation and scales, and the SH emission.
#include "nxs_internal.h"
#include "nxs_ops.h"
#include "nxs_stage.h"

namespace nxs {

namespace {

// x + the y of another lane of the row of 16 (CTRL; 0 where there is none).
// (no contraction: an add of the moved value folds into one DPP add, which a
// product of the caller fused into an FMA with it would prevent)
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x, float y) {
#pragma clang fp contract(off)
  const int m = __builtin_amdgcn_update_dpp(0, __float_as_int(y), CTRL, 0xF, 0xF, true);
  return x + __int_as_float(m);
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor8 = 0x128;   // quad_perm, quad_perm, row_ror:8
constexpr int kFrom4 = 0x104;                              // row_shl:4, lane j reads j + 4
constexpr int kRor4 = 0x124;                               // row_ror:4

// Per-wave sums over the 64 pixels of the 9 fields da (1, dx, dy, dx^2, dx dy,
// dy^2) and p g_rgb.  Of each contributing splat every lane leaves only da and p
// in two rows of the wave's table; a flush gives each of the kRedSplats pending
// splats a row of 16 lanes, a lane four pixels of one image row, over which it
// forms the sums in registers (dy is one number for them), and folds the 16
// lanes, each fold halving the fields that a lane still carries.  The kernel is
// bound by VALU issue (88% busy): this takes about 18 instructions a splat,
// where forming nine products in every lane and adding them over lane quads
// took 32 and nine LDS writes (8 views of 720p, 500k splats: 910 -> 770 us;
// 1080p, 1M, quadratic: 132 -> 115 us).  Six work-groups of four waves fit a CU by
// their registers (77 to 80), eight by 20 KB of LDS; with eight splats a flush, 2 KB
// more a wave and 28 KB a work-group, five fit, and that loses although it needs
// fewer instructions (1013 us).
constexpr int kRedSplats = 4;
constexpr int kRedF4 = 2 * kRedSplats * 64 / 4;  // float4 per wave

// (six waves a SIMD: left to itself the compiler takes 82 registers for the
// quadratic operators, two more than six waves leave each)
template <int MODEL, int TW, int TH>
__global__ __launch_bounds__(TW* TH, 6) void composite_bwd_kernel(
    const ViewDev* __restrict__ views, int n_views, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ inst_val, const float4* __restrict__ rec, CompositeParams prm,
    const float4* __restrict__ pstate, float* __restrict__ gslot, uint32_t n_tiles,
    uint32_t per_xcd, const uint32_t* __restrict__ order) {
  __shared__ float4 stage[(TW / 8) * (TH / 8) * kStageF4];
  __shared__ float4 rsum[(TW / 8) * (TH / 8) * kRedF4];   // per wave: pending da and p
  // the forward's order (longest tile lists first) when it made one, else
  // each XCD a contiguous band of tiles
  const uint32_t w = order ? blockIdx.x : xcd_banded(blockIdx.x, per_xcd);
  if (w >= n_tiles) return;
  const uint32_t tile = order ? order[w] : w;
  int vi = 0;
  {
    int lo = 0, hi = n_views - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if ((uint32_t)views[mid].tile_off <= tile) lo = mid; else hi = mid - 1;
    }
    vi = lo;
  }
  const ViewDev& v = views[vi];
  const int lt = (int)(tile - (uint32_t)v.tile_off);
  const int tx = lt % v.tiles_x, ty = lt / v.tiles_x;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int bx = (wid % (TW / 8)) * 8, by = (wid / (TW / 8)) * 8;
  const int lx = bx + (lane & 7), ly = by + (lane >> 3);
  const int px = tx * TW + lx, py = ty * TH + ly;
  const bool inside = px < v.width && py < v.height;
  const float fx = (float)lx + 0.5f, fy = (float)ly + 0.5f;
  const StageBlock sb = stage_block<TW>(tx, ty, TH, wid, prm.log2_alpha_min);
  float4* wlds = stage + wid * kStageF4;
  float* wred = reinterpret_cast<float*>(rsum + wid * kRedF4);
  const uint2 rg = ranges[tile];
  const float amin = prm.log2_alpha_min;
  const float t_eps = prm.t_eps;
  const float param = prm.param;
  constexpr float kc = MODEL == 2 ? -0.5f : MODEL == 3 ? 0.5f : 0.0f;
  const float c = MODEL == 4 ? param : kc;

  // upstream gradient (g0, g1, g2, gT) and what the forward left per pixel
  float g0 = 0.f, g1 = 0.f, g2 = 0.f, gT = 0.f;
  float4 s0 = make_float4(0.f, 0.f, 0.f, 1.f), s1 = make_float4(0.f, 0.f, 0.f, 0.f),
         s2 = s1;
  if (inside) {
    const int64_t pix = (int64_t)py * v.width + px;
    g0 = v.g_rgb[3 * pix + 0];
    g1 = v.g_rgb[3 * pix + 1];
    g2 = v.g_rgb[3 * pix + 2];
    gT = v.g_trans ? v.g_trans[pix] : 0.0f;
    const float4* st = pstate + 3 * (v.pix_off + pix);
    s0 = st[0];
    s1 = st[1];
    s2 = st[2];
  }
  // (the fourth channel is T, whose emission is 0 and background 1)
  // exponential: the radiance not yet attributed
  float R0 = s0.x, R1 = s0.y, R2 = s0.z;
  const float RT = gT * s0.w;
  // linear / quadratic: E_k, and g . Theta.  (Emissions are subtracted channel by
  // channel before they meet g: splats of one surface have nearly equal ones, and
  // g . E - g . E_k would keep the rounding of two large numbers.  In float32, of
  // emissions within 0.001 of each other, the linear operator's da is 5e-8 off
  // this way, as with all in four channels, and 3.5e-5 off that way.)
  const float k0 = s1.x, k1 = s1.y, k2 = s1.z;
  const float k3 = s0.w == 0.0f ? 0.0f : 1.0f;   // (saturated: 0)
  const float kT = gT * k3;
  float thg = g0 * (s2.x - k0 * s1.w) + g1 * (s2.y - k1 * s1.w) + g2 * (s2.z - k2 * s1.w) -
              kT * s1.w;

  Op<MODEL> op;
  // running lanes; each batch is staged against the rows and columns that
  // still hold one
  // (none where t_eps > 1, as in the forward)
  uint64_t act = __builtin_amdgcn_ballot_w64(inside && !op.stopped(t_eps));
  // (an empty tile fetches nothing: its range is [0, 0) or [x, x))
  StageSlot slots{0u, false};
  StageFetch fetched{};
  if (rg.x < rg.y) {
    slots = stage_slot(inst_val, rg.x, rg.y, lane);
    fetched = stage_records(slots, rec, prm.slot_mask, wid);
    slots = stage_slot(inst_val, (uint64_t)rg.x + 64, rg.y, lane);
  }
  // The flush's view of the block: lane 16 s + j has splat s and pixels 4 j .. 4 j
  // + 3, that is columns 4 (j & 1) + 0 .. 3 of row j >> 1, and their g_rgb.
  const int fs = lane >> 4, fj = lane & 15;
  const float fcx = (float)(bx + 4 * (fj & 1)) + 0.5f, fcy = (float)(by + (fj >> 1)) + 0.5f;
  float4 h0, h1, h2;
  {
    wred[lane] = g0;
    wred[64 + lane] = g1;
    wred[128 + lane] = g2;
    wave_lds_order();
    const float4* q = reinterpret_cast<const float4*>(wred) + fj;
    h0 = q[0];
    h1 = q[16];
    h2 = q[32];
    wave_lds_order();
  }
  // the field that lane j of a row ends with (below), 9: none
  const bool b0 = (lane & 1) != 0, b1 = (lane & 2) != 0, b3 = (lane & 8) != 0;
  const int field = (lane & 4) == 0 ? (b0 ? 4 : 0) + (b1 ? 2 : 0) + (b3 ? 1 : 0)
                                    : fj == 4 ? 8 : 9;
  float fu = 0.0f, fv = 0.0f;   // the lane's pending splat: its centre and slot
  uint32_t fslot = 0, pend = 0;
  auto flush = [&]() {
    wave_lds_order();
    const float4 d = reinterpret_cast<const float4*>(wred)[lane];
    const float4 q = reinterpret_cast<const float4*>(wred)[64 + lane];
    const float x0 = fcx - fu, x1 = fcx + 1.0f - fu, x2 = fcx + 2.0f - fu,
                x3 = fcx + 3.0f - fu, y = fcy - fv;
    const float d0 = d.x * x0, d1 = d.y * x1, d2 = d.z * x2, d3 = d.w * x3;
    const float m0 = (d.x + d.y) + (d.z + d.w);
    const float mx = (d0 + d1) + (d2 + d3);
    const float mxx = fmaf(d3, x3, fmaf(d2, x2, fmaf(d1, x1, d0 * x0)));
    const float my = m0 * y, mxy = mx * y, myy = my * y;
    const float c0 = fmaf(q.w, h0.w, fmaf(q.z, h0.z, fmaf(q.y, h0.y, q.x * h0.x)));
    const float c1 = fmaf(q.w, h1.w, fmaf(q.z, h1.z, fmaf(q.y, h1.y, q.x * h1.x)));
    float c2 = fmaf(q.w, h2.w, fmaf(q.z, h2.z, fmaf(q.y, h2.y, q.x * h2.x)));
    // fields 0..7: m0, mx, my, mxx | mxy, myy, c0, c1.  Across bit 0 a lane keeps
    // one half of them, then one quarter across bit 1, one across bit 3
    const float u0 = dpp_add<kXor1>(b0 ? mxy : m0, b0 ? m0 : mxy);
    const float u1 = dpp_add<kXor1>(b0 ? myy : mx, b0 ? mx : myy);
    const float u2 = dpp_add<kXor1>(b0 ? c0 : my, b0 ? my : c0);
    const float u3 = dpp_add<kXor1>(b0 ? c1 : mxx, b0 ? mxx : c1);
    const float w0 = dpp_add<kXor2>(b1 ? u2 : u0, b1 ? u0 : u2);
    const float w1 = dpp_add<kXor2>(b1 ? u3 : u1, b1 ? u1 : u3);
    float sum = dpp_add<kXor8>(b3 ? w1 : w0, b3 ? w0 : w1);
    sum = dpp_add<kFrom4>(sum, sum);
    c2 = dpp_add<kXor1>(c2, c2);
    c2 = dpp_add<kXor2>(c2, c2);
    c2 = dpp_add<kXor8>(c2, c2);
    c2 = dpp_add<kRor4>(c2, c2);
    if (field == 8) sum = c2;
    if (field < 9 && fs < (int)pend) atomicAdd(gslot + 9 * (size_t)fslot + field, sum);
    wave_lds_order();
    pend = 0;
  };
  for (uint32_t base = rg.x; base < rg.y && act != 0; base += 64) {
    const uint32_t n = stage_batch(fetched, stage_shrink(sb, act), wlds);
    fetched = stage_records(slots, rec, prm.slot_mask, wid);          // batch base + 64
    slots = stage_slot(inst_val, (uint64_t)base + 128, rg.y, lane);   // batch base + 128
    for (uint32_t k = 0; k < n && act != 0; ++k) {
      const float4 q0 = wlds[3 * k + 0], q1 = wlds[3 * k + 1], q2 = wlds[3 * k + 2];
      float r[10] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w, q2.x, q2.y};
      // (an empty statement that keeps the whole record's reads here, in flight
      // together, instead of half of them after the branch below)
      __asm__ volatile("" : "+v"(r[6]), "+v"(r[7]), "+v"(r[8]), "+v"(r[9]));
      const float dx = fx - r[0], dy = fy - r[1];
      const float e = fmaf(dx, fmaf(r[2], dx, r[3] * dy), fmaf(r[4] * dy, dy, r[5]));
      // The lanes that composite this splat, and those still running, are kept
      // as scalar masks: no lane instructions for them, and a splat that no lane
      // takes ends here (780 -> 728 us, 112 -> 103 us, in the cases above)
      const uint64_t hit = __builtin_amdgcn_ballot_w64(e >= amin) & act;
      if (hit == 0) continue;
      // Every lane runs the same arithmetic: a lane that has stopped, or
      // whose alpha is below alpha_min, takes a = 0 and dL/dalpha = 0, which
      // leaves its state unchanged and makes each of its terms an exact zero.
      const bool contrib = __builtin_amdgcn_inverse_ballot_w64(hit);
      const float a = contrib ? __builtin_amdgcn_exp2f(e) : 0.0f;
      const float T_before = op.T, tau_before = op.tau;
      bool stops;
      const float p = op.step(a, param, t_eps, stops);
      const uint64_t ends = __builtin_amdgcn_ballot_w64(stops);
      float dalpha;
      bool adds = contrib;
      if (MODEL == 0) {
        const float G = fmaf(g0, r[6], fmaf(g1, r[7], g2 * r[8]));   // g . E
        R0 = fmaf(-r[6], p, R0);
        R1 = fmaf(-r[7], p, R1);
        R2 = fmaf(-r[8], p, R2);
        const float Rg = fmaf(g0, R0, fmaf(g1, R1, fmaf(g2, R2, RT)));
        // (1 - a > 0 unless the splat stops the pixel: one with a = 1 leaves T = 0)
        dalpha = fmaf(T_before, G, -(__builtin_amdgcn_rcpf(1.0f - a) * Rg));
        if (ends & hit) {   // (uniform; once a pixel) only the background lies behind
          const float e0 = r[6] - prm.bg[0], e1 = r[7] - prm.bg[1], e2 = r[8] - prm.bg[2];
          const float last = T_before * fmaf(g0, e0, fmaf(g1, e1, fmaf(g2, e2, -gT)));
          dalpha = stops ? last : dalpha;
        }
      } else {
        const float e0 = r[6] - k0, e1 = r[7] - k1, e2 = r[8] - k2;
        const float G = fmaf(g0, e0, fmaf(g1, e1, fmaf(g2, e2, -kT)));   // g . (E - E_k)
        thg = fmaf(-G, a, thg);
        dalpha = fmaf(c, fmaf(G, tau_before, thg), G);
        adds = contrib && !stops;   // the saturating splat takes the remainder: 0
      }
      // alpha = aleph exp(-q/2), q = A dx^2 + 2 B dx dy + C dy^2: with
      // da = alpha dL/dalpha a pixel adds dL/daleph = da / aleph,
      // dL/du = da (A dx + B dy), dL/dv = da (B dx + C dy) and
      // dL/d(A, B, C) = -da (dx^2 / 2, dx dy, dy^2 / 2), all linear in the
      // moments da (1, dx, dy, dx^2, dx dy, dy^2): the wave sums those, and
      // project_bwd applies the slot's aleph and conic once per slot
      wred[64 * pend + lane] = adds ? dalpha * a : 0.0f;
      wred[64 * (kRedSplats + pend) + lane] = p;
      const bool mine = fs == (int)pend;
      fu = mine ? r[0] : fu;
      fv = mine ? r[1] : fv;
      fslot = mine ? __float_as_uint(r[9]) : fslot;
      if (++pend == kRedSplats) flush();
      act &= ~ends;
    }
  }
  if (pend) flush();
}

// ------------------------------------------------------------ projection

constexpr int kBlock = 256;

// gradient of the real SH basis value Y_k at (x, y, z), as a polynomial in
// x, y, z (the caller projects it onto the sphere's tangent plane)
template <int DEG>
__device__ __forceinline__ void sh_basis_grad(float x, float y, float z, float* Y,
                                              float* gx, float* gy, float* gz) {
  constexpr int K = (DEG + 1) * (DEG + 1);
#pragma unroll
  for (int k = 0; k < K; ++k) gx[k] = gy[k] = gz[k] = 0.0f;
  Y[0] = 0.28209479177387814f;
  if (DEG >= 1) {
    const float c1 = 0.4886025119029199f;
    Y[1] = c1 * y; gy[1] = c1;
    Y[2] = c1 * z; gz[2] = c1;
    Y[3] = c1 * x; gx[3] = c1;
  }
  if (DEG >= 2) {
    const float a = 1.0925484305920792f, b = 0.31539156525252005f, cc = 0.5462742152960396f;
    Y[4] = a * x * y; gx[4] = a * y; gy[4] = a * x;
    Y[5] = a * y * z; gy[5] = a * z; gz[5] = a * y;
    Y[6] = b * (3.0f * z * z - 1.0f); gz[6] = 6.0f * b * z;
    Y[7] = a * x * z; gx[7] = a * z; gz[7] = a * x;
    Y[8] = cc * (x * x - y * y); gx[8] = 2.0f * cc * x; gy[8] = -2.0f * cc * y;
  }
  if (DEG >= 3) {
    const float c3a = 0.5900435899266435f, c3b = 2.890611442640554f,
                c3c = 0.4570457994644658f, c3d = 0.3731763325901154f,
                c3e = 1.445305721320277f;
    Y[9] = c3a * y * (3.0f * x * x - y * y);
    gx[9] = 6.0f * c3a * x * y; gy[9] = 3.0f * c3a * (x * x - y * y);
    Y[10] = c3b * x * y * z;
    gx[10] = c3b * y * z; gy[10] = c3b * x * z; gz[10] = c3b * x * y;
    Y[11] = c3c * y * (5.0f * z * z - 1.0f);
    gy[11] = c3c * (5.0f * z * z - 1.0f); gz[11] = 10.0f * c3c * y * z;
    Y[12] = c3d * z * (5.0f * z * z - 3.0f);
    gz[12] = c3d * (15.0f * z * z - 3.0f);
    Y[13] = c3c * x * (5.0f * z * z - 1.0f);
    gx[13] = c3c * (5.0f * z * z - 1.0f); gz[13] = 10.0f * c3c * x * z;
    Y[14] = c3e * z * (x * x - y * y);
    gx[14] = 2.0f * c3e * x * z; gy[14] = -2.0f * c3e * y * z; gz[14] = c3e * (x * x - y * y);
    Y[15] = c3a * x * (x * x - 3.0f * y * y);
    gx[15] = 3.0f * c3a * (x * x - y * y); gy[15] = -6.0f * c3a * x * y;
  }
}

// Gaussian i's gradients; those of its coefficients `coef` into gcoef.
template <int DEG>
__device__ __forceinline__ void project_bwd_one(const GaussDev& g,
                                                const ViewDev* __restrict__ views, int n_views,
                                                float* __restrict__ gslot,
                                                const GaussGradDev& out, int i,
                                                const float* coef, float* gcoef) {
  constexpr int K = (DEG + 1) * (DEG + 1);
  const float m[3] = {g.means[3 * i], g.means[3 * i + 1], g.means[3 * i + 2]};
  const float s[3] = {g.scales[3 * i], g.scales[3 * i + 1], g.scales[3 * i + 2]};
  const float q[4] = {g.quats[4 * i], g.quats[4 * i + 1], g.quats[4 * i + 2],
                      g.quats[4 * i + 3]};
  // rotation of the normalised quaternion
  const float qn = sqrtf(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
  float gm[3] = {0.f, 0.f, 0.f}, gs[3] = {0.f, 0.f, 0.f}, gq[4] = {0.f, 0.f, 0.f, 0.f};
  float gop = 0.f;
#pragma unroll
  for (int k = 0; k < K * 3; ++k) gcoef[k] = 0.f;
  if (!(qn > 0.0f)) {
    // culled in every view: no gradient
  } else {
    const float w = q[0] / qn, x = q[1] / qn, y = q[2] / qn, z = q[3] / qn;
    const float Rq[3][3] = {{1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)},
                            {2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)},
                            {2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)}};
    float M[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) M[a][b] = Rq[a][b] * s[b];
    float gRq[3][3] = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
    for (int vi = 0; vi < n_views; ++vi) {
      float* gsl = gslot + 9 * ((size_t)vi * g.n + i);
      // the slot's moments: alpha dL/dalpha (1, dx, dy, dx^2, dx dy, dy^2), colour
      const float m0 = gsl[0], m1 = gsl[1], m2 = gsl[2], m3 = gsl[3], m4 = gsl[4],
                  m5 = gsl[5];
      const float g_rgb[3] = {gsl[6], gsl[7], gsl[8]};
      if (m0 == 0.f && m1 == 0.f && m2 == 0.f && m3 == 0.f && m4 == 0.f && m5 == 0.f &&
          g_rgb[0] == 0.f && g_rgb[1] == 0.f && g_rgb[2] == 0.f)
        continue;   // no pixel of this view saw the Gaussian
      const ViewDev& v = views[vi];
      const float* R = v.R;
      const float pxc = R[0] * m[0] + R[1] * m[1] + R[2] * m[2] + v.t[0];
      const float pyc = R[3] * m[0] + R[4] * m[1] + R[5] * m[2] + v.t[1];
      const float pzc = R[6] * m[0] + R[7] * m[1] + R[8] * m[2] + v.t[2];
      const float iz = 1.0f / pzc, iz2 = iz * iz;
      const float j00 = v.fx * iz, j02 = -v.fx * pxc * iz2;
      const float j11 = v.fy * iz, j12 = -v.fy * pyc * iz2;
      float T[2][3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        T[0][k] = j00 * R[k] + j02 * R[6 + k];
        T[1][k] = j11 * R[3 + k] + j12 * R[6 + k];
      }
      float A[2][3];
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int b = 0; b < 3; ++b)
          A[r][b] = T[r][0] * M[0][b] + T[r][1] * M[1][b] + T[r][2] * M[2][b];
      const float a = A[0][0] * A[0][0] + A[0][1] * A[0][1] + A[0][2] * A[0][2] + 0.3f;
      const float b = A[0][0] * A[1][0] + A[0][1] * A[1][1] + A[0][2] * A[1][2];
      const float cc = A[1][0] * A[1][0] + A[1][1] * A[1][1] + A[1][2] * A[1][2] + 0.3f;
      const float idet = 1.0f / (a * cc - b * b);
      // conic K = Sigma2D^-1; dL/dSigma = -K G_K K with G_K = [[gA, gB/2], [gB/2, gC]]
      const float K00 = cc * idet, K01 = -b * idet, K11 = a * idet;
      // dL/d(opacity, u, v) and dL/d(A, B, C) of the conic q = A dx^2 + 2 B dx dy + C dy^2
      const float g_op = m0 / g.opac[i];
      const float g_u = K00 * m1 + K01 * m2, g_v = K01 * m1 + K11 * m2;
      const float gA = -0.5f * m3, gB = -m4, gC = -0.5f * m5;
      gsl[0] = g_op;
      gsl[1] = g_u;
      gsl[2] = g_v;
      gsl[3] = gA;
      gsl[4] = gB;
      gsl[5] = gC;
      const float G00 = gA, G01 = 0.5f * gB, G11 = gC;
      // (K G K) entries
      const float KG00 = K00 * G00 + K01 * G01, KG01 = K00 * G01 + K01 * G11;
      const float KG10 = K01 * G00 + K11 * G01, KG11 = K01 * G01 + K11 * G11;
      const float S00 = -(KG00 * K00 + KG01 * K01);
      const float S01 = -(KG00 * K01 + KG01 * K11);
      const float S11 = -(KG10 * K01 + KG11 * K11);
      const float ga = S00, gb = 2.0f * S01, gc = S11;
      // A rows: a = A0.A0, b = A0.A1, c = A1.A1
      float gAm[2][3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        gAm[0][k] = 2.0f * ga * A[0][k] + gb * A[1][k];
        gAm[1][k] = gb * A[0][k] + 2.0f * gc * A[1][k];
      }
      // A = T M
      float gT[2][3];
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k)
          gT[r][k] = gAm[r][0] * M[k][0] + gAm[r][1] * M[k][1] + gAm[r][2] * M[k][2];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int b2 = 0; b2 < 3; ++b2) {
          const float gM = T[0][k] * gAm[0][b2] + T[1][k] * gAm[1][b2];
          gs[b2] += gM * Rq[k][b2];
          gRq[k][b2] += gM * s[b2];
        }
      // T = J R_cam
      float gj00 = 0.f, gj02 = 0.f, gj11 = 0.f, gj12 = 0.f;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        gj00 += gT[0][k] * R[k];
        gj02 += gT[0][k] * R[6 + k];
        gj11 += gT[1][k] * R[3 + k];
        gj12 += gT[1][k] * R[6 + k];
      }
      // J and the centre as functions of the camera-space mean
      const float gpx = gj02 * (-v.fx * iz2) + g_u * v.fx * iz;
      const float gpy = gj12 * (-v.fy * iz2) + g_v * v.fy * iz;
      const float gpz = gj00 * (-v.fx * iz2) + gj02 * (2.0f * v.fx * pxc * iz2 * iz) +
                        gj11 * (-v.fy * iz2) + gj12 * (2.0f * v.fy * pyc * iz2 * iz) +
                        g_u * (-v.fx * pxc * iz2) + g_v * (-v.fy * pyc * iz2);
#pragma unroll
      for (int k = 0; k < 3; ++k) gm[k] += R[k] * gpx + R[3 + k] * gpy + R[6 + k] * gpz;
      gop += g_op;
      // emission
      const float dxw = m[0] - v.campos[0], dyw = m[1] - v.campos[1], dzw = m[2] - v.campos[2];
      const float dn = sqrtf(dxw * dxw + dyw * dyw + dzw * dzw);
      const float ux = dxw / dn, uy = dyw / dn, uz = dzw / dn;
      float Y[K], Gx[K], Gy[K], Gz[K];
      sh_basis_grad<DEG>(ux, uy, uz, Y, Gx, Gy, Gz);
      float gdx = 0.f, gdy = 0.f, gdz = 0.f;
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        float val = 0.5f;
#pragma unroll
        for (int k = 0; k < K; ++k) val += Y[k] * coef[3 * k + ch];
        if (!(val > 0.0f)) continue;   // clamped at 0
        const float gch = g_rgb[ch];
#pragma unroll
        for (int k = 0; k < K; ++k) {
          gcoef[3 * k + ch] += Y[k] * gch;
          gdx += gch * coef[3 * k + ch] * Gx[k];
          gdy += gch * coef[3 * k + ch] * Gy[k];
          gdz += gch * coef[3 * k + ch] * Gz[k];
        }
      }
      const float dot = ux * gdx + uy * gdy + uz * gdz;
      gm[0] += (gdx - ux * dot) / dn;
      gm[1] += (gdy - uy * dot) / dn;
      gm[2] += (gdz - uz * dot) / dn;
    }
    // rotation entries -> normalised quaternion (w, x, y, z)
    float gw = 0.f, gx = 0.f, gy = 0.f, gz = 0.f;
    gw += gRq[0][1] * (-2 * z) + gRq[0][2] * (2 * y) + gRq[1][0] * (2 * z) +
          gRq[1][2] * (-2 * x) + gRq[2][0] * (-2 * y) + gRq[2][1] * (2 * x);
    gx += gRq[0][1] * (2 * y) + gRq[0][2] * (2 * z) + gRq[1][0] * (2 * y) +
          gRq[1][1] * (-4 * x) + gRq[1][2] * (-2 * w) + gRq[2][0] * (2 * z) +
          gRq[2][1] * (2 * w) + gRq[2][2] * (-4 * x);
    gy += gRq[0][0] * (-4 * y) + gRq[0][1] * (2 * x) + gRq[0][2] * (2 * w) +
          gRq[1][0] * (2 * x) + gRq[1][2] * (2 * z) + gRq[2][0] * (-2 * w) +
          gRq[2][1] * (2 * z) + gRq[2][2] * (-4 * y);
    gz += gRq[0][0] * (-4 * z) + gRq[0][1] * (-2 * w) + gRq[0][2] * (2 * x) +
          gRq[1][0] * (2 * w) + gRq[1][1] * (-4 * z) + gRq[1][2] * (2 * y) +
          gRq[2][0] * (2 * x) + gRq[2][1] * (2 * y);
    const float qh[4] = {w, x, y, z}, gqh[4] = {gw, gx, gy, gz};
    const float dqh = qh[0] * gqh[0] + qh[1] * gqh[1] + qh[2] * gqh[2] + qh[3] * gqh[3];
#pragma unroll
    for (int k = 0; k < 4; ++k) gq[k] = (gqh[k] - qh[k] * dqh) / qn;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    out.means[3 * i + k] = gm[k];
    out.scales[3 * i + k] = gs[k];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) out.quats[4 * i + k] = gq[k];
  out.opac[i] = gop;
}

// A Gaussian's coefficients and their gradients are each a row of 12 K bytes.
// When a row is whole float4s (degrees 1 and 3) and both arrays are 16-byte
// aligned, the work-group's rows pass through LDS, so that global memory is
// read and written in address order; rows are an odd number of float4s apart,
// which spreads the lanes' accesses over all banks (1M Gaussians of degree 3,
// 516 MB in all: 117 -> 100 us; below two waves a SIMD of 214 registers each,
// the latency of the chain through one Gaussian is what remains).
template <int DEG>
__global__ __launch_bounds__(kBlock) void project_bwd_kernel(
    GaussDev g, const ViewDev* __restrict__ views, int n_views,
    float* __restrict__ gslot, GaussGradDev out) {
  constexpr int K = (DEG + 1) * (DEG + 1);
  constexpr int NC = 3 * K, NC4 = NC / 4;
  constexpr bool kVec = NC % 4 == 0;
  constexpr int STRIDE4 = NC4 % 2 == 1 ? NC4 : NC4 + 1;   // float4s per row
  __shared__ float4 s_row[kVec ? kBlock * STRIDE4 : 1];
  const int i = blockIdx.x * kBlock + threadIdx.x;
  const bool rows = kVec && ((reinterpret_cast<uintptr_t>(g.sh) |
                              reinterpret_cast<uintptr_t>(out.sh)) & 15u) == 0;   // (uniform)
  const size_t row4 = (size_t)blockIdx.x * kBlock * NC4;   // the work-group's first float4
  const int n4 = min(kBlock, g.n - (int)blockIdx.x * kBlock) * NC4;
  if (rows) {
    // (every load issued before any is used)
    const float4* src = reinterpret_cast<const float4*>(g.sh) + row4;
    float4 buf[NC4 > 0 ? NC4 : 1];
#pragma unroll
    for (int r = 0; r < NC4; ++r) {
      const int f = r * kBlock + threadIdx.x;
      buf[r] = f < n4 ? src[f] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
#pragma unroll
    for (int r = 0; r < NC4; ++r) {
      const int f = r * kBlock + threadIdx.x;
      s_row[(f / NC4) * STRIDE4 + f % NC4] = buf[r];
    }
    __syncthreads();
  }
  float gcoef[NC];
  if (!rows) {
    if (i >= g.n) return;
    project_bwd_one<DEG>(g, views, n_views, gslot, out, i, g.sh + (size_t)i * NC, gcoef);
#pragma unroll
    for (int k = 0; k < NC; ++k) out.sh[(size_t)i * NC + k] = gcoef[k];
    return;
  }
  float4* mine = s_row + threadIdx.x * STRIDE4;
  if (i < g.n) {
    project_bwd_one<DEG>(g, views, n_views, gslot, out, i, reinterpret_cast<const float*>(mine),
                         gcoef);
    // (over its own row, the only one it read)
#pragma unroll
    for (int r = 0; r < NC4; ++r)
      mine[r] = make_float4(gcoef[4 * r], gcoef[4 * r + 1], gcoef[4 * r + 2], gcoef[4 * r + 3]);
  }
  __syncthreads();
  float4* dst = reinterpret_cast<float4*>(out.sh) + row4;
#pragma unroll
  for (int r = 0; r < NC4; ++r) {
    const int f = r * kBlock + threadIdx.x;
    if (f < n4) dst[f] = s_row[(f / NC4) * STRIDE4 + f % NC4];
  }
}

template <int MODEL, int TW, int TH>
void bwd_t(int64_t n_tiles, const ViewDev* views, int n_views, const uint2* ranges,
           const uint32_t* inst_val, const float4* rec, const CompositeParams& p,
           const float4* pstate, float* gslot, const uint32_t* order, hipStream_t s) {
  const uint32_t per = (uint32_t)((n_tiles + 7) / 8);
  hipLaunchKernelGGL((composite_bwd_kernel<MODEL, TW, TH>), dim3(per * 8), dim3(TW * TH), 0, s,
                     views, n_views, ranges, inst_val, rec, p, pstate, gslot,
                     (uint32_t)n_tiles, per, order);
}

template <int MODEL>
void bwd_m(int tile_w, int tile_h, int64_t n_tiles, const ViewDev* views, int n_views,
           const uint2* ranges, const uint32_t* inst_val, const float4* rec,
           const CompositeParams& p, const float4* pstate, float* gslot, const uint32_t* order,
           hipStream_t s) {
  if (tile_w == 8 && tile_h == 8)
    bwd_t<MODEL, 8, 8>(n_tiles, views, n_views, ranges, inst_val, rec, p, pstate, gslot, order,
                       s);
  else if (tile_w == 32 && tile_h == 8)
    bwd_t<MODEL, 32, 8>(n_tiles, views, n_views, ranges, inst_val, rec, p, pstate, gslot, order,
                        s);
  else
    bwd_t<MODEL, 16, 16>(n_tiles, views, n_views, ranges, inst_val, rec, p, pstate, gslot,
                         order, s);
}

}  // namespace

void launch_composite_bwd(int model, int tile_w, int tile_h, int64_t n_tiles,
                          const ViewDev* views, int n_views, const uint2* ranges,
                          const uint32_t* inst_val, const float4* rec, const CompositeParams& p,
                          const float4* pstate, float* gslot, const uint32_t* order,
                          hipStream_t s) {
  if (n_tiles <= 0) return;
  switch (model) {
#define NXS_B(M)                                                                        \
  case M:                                                                               \
    bwd_m<M>(tile_w, tile_h, n_tiles, views, n_views, ranges, inst_val, rec, p, pstate, \
             gslot, order, s);                                                          \
    break;
    NXS_B(0) NXS_B(1) NXS_B(2) NXS_B(3) NXS_B(4)
#undef NXS_B
    default: break;
  }
}

void launch_project_bwd(const GaussDev& g, const ViewDev* views, int n_views,
                        float* gslot, const GaussGradDev& out, hipStream_t s) {
  if (g.n <= 0) return;
  dim3 grid((g.n + kBlock - 1) / kBlock);
  switch (g.sh_degree) {
    case 0: hipLaunchKernelGGL(project_bwd_kernel<0>, grid, dim3(kBlock), 0, s, g, views, n_views, gslot, out); break;
    case 1: hipLaunchKernelGGL(project_bwd_kernel<1>, grid, dim3(kBlock), 0, s, g, views, n_views, gslot, out); break;
    case 2: hipLaunchKernelGGL(project_bwd_kernel<2>, grid, dim3(kBlock), 0, s, g, views, n_views, gslot, out); break;
    default: hipLaunchKernelGGL(project_bwd_kernel<3>, grid, dim3(kBlock), 0, s, g, views, n_views, gslot, out); break;
  }
}

}  // namespace nxs
