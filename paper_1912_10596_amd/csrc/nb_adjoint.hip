// nb_adjoint.hip -- reverse-mode adjoint of the two-flavour radial integration.
//
// Forward step (state P_n, Bloch vector of one beam; f_i = (h/c_i) B(r_i, J^(i))):
//   Y2 = R(f1/2) P,  Y3 = R(Om) P with Om = f2/2 - (f1 x f2)/8,  Y4 = R(f3) P,
//   Theta = (f1 + 2 f2 + 2 f3 + f4)/6 - (f1 x f4)/12,  P_{n+1} = R(Theta) P / |.|,
// with J^(1) = M(P), J^(2) = M(Y2), J^(3) = M(Y3), J^(4) = M(Y4) the moment sums
// J0 = sum g S y / c, J1 = sum g S y (S = diag(s, 1, s), s = -1 for antineutrinos).
// Its reverse, per step and beam, runs the stages backwards; every moment adjoint is a
// grid-wide sum, so a reverse step has the forward step's four grid barriers:
//   A: renormalisation and final rotation -> Theta-bar -> f4-bar -> sum (J^(4)-bar)
//   B: Y4 broadcast of J^(4)-bar -> f3-bar -> sum (J^(3)-bar)
//   C: Y3 broadcast -> Om-bar -> f2-bar (and part of f1-bar) -> sum (J^(2)-bar)
//   D: Y2 broadcast -> f1-bar -> sum (J^(1)-bar); then the J^(1)-bar broadcast onto P_n.
// For y = R(x) p: p-bar = R(-x) y-bar and x-bar = Jl(x)^T (y x y-bar) with the left
// Jacobian Jl(x) = I + a [x]x + b [x]x^2, a = (1 - cos t)/t^2, b = (t - sin t)/t^3.
// The parameters enter through the weights g (luminosities), B_vac (theta_v) and the
// matter term lambda = sqrt2 G_F n0 (R/r)^p (n0); their adjoints are accumulated per
// thread and summed once at the end.
//
// Memory: the forward pass (nb_adjoint) keeps the state at the start of every segment of
// `ckpt` steps and records all stage moments; a segment is recomputed beam by beam from
// its checkpoint with the recorded moments (no grid synchronisation, the same arithmetic
// as the stepping kernel, hence the same bits) into a tape of `ckpt` states, which the
// reverse steps then read backwards.  Each beam's adjoint state lives in registers of
// the thread that owns it for the whole launch.
#include "nb_device.h"
#include "nb_internal.h"
#include "nb_stage.h"

namespace nb {

// Rotation by the angle vector x (angle |x| about x/|x|, as rotate2) with what its adjoint
// needs: the half-angle quaternion and the left-Jacobian coefficients a, b.
struct Rot {
  double x0, x1, x2;
  double v0, v1, v2, c;  // sin(t/2) x/t, cos(t/2)
  double ja, jb;
};
// SK: as sincos_nb.
template <bool SK>
__device__ __forceinline__ Rot make_rot(double x0, double x1, double x2) {
  Rot r;
  r.x0 = x0;
  r.x1 = x1;
  r.x2 = x2;
  const double t2 = (x0 * x0 + x1 * x1) + x2 * x2;
  double ih, s, c;
  double t = sqrt_in_range(t2, ih);
  if (!(t2 >= 0x1p-767)) {   // tiny or zero (rare)
    t = sqrt(t2);
    ih = (t > 0.0) ? 0.5 / t : 0.0;
  }
  sincos_nb<SK>(0.5 * t, s, c);
  const double k = div_by_sqrt(s, t, ih);   // 0 for t = 0
  r.v0 = x0 * k;
  r.v1 = x1 * k;
  r.v2 = x2 * k;
  r.c = c;
  // (1 - cos t) / t^2 and (t - sin t) / t^3; below 0.05 their series, free of cancellation
  const double it = rcp_step(t, ih + ih);
  const double ja = 2.0 * (k * k), jb = (t - 2.0 * (s * c)) * (it * (it * it));
  const double sa = (0.5 - t2 * (1.0 / 24.0)) + (t2 * t2) * (1.0 / 720.0);
  const double sb = (1.0 / 6.0 - t2 * (1.0 / 120.0)) + (t2 * t2) * (1.0 / 5040.0);
  r.ja = (t < 0.05) ? sa : ja;
  r.jb = (t < 0.05) ? sb : jb;
  return r;
}
// y = R(x) p  (quaternion form: t = 2 v x p, y = p + c t + v x t)
__device__ __forceinline__ void rot_fwd(const Rot& r, double p0, double p1, double p2, double& y0,
                                        double& y1, double& y2) {
  double t0 = r.v1 * p2 - r.v2 * p1;
  double t1 = r.v2 * p0 - r.v0 * p2;
  double t2 = r.v0 * p1 - r.v1 * p0;
  t0 = t0 + t0;
  t1 = t1 + t1;
  t2 = t2 + t2;
  y0 = (p0 + r.c * t0) + (r.v1 * t2 - r.v2 * t1);
  y1 = (p1 + r.c * t1) + (r.v2 * t0 - r.v0 * t2);
  y2 = (p2 + r.c * t2) + (r.v0 * t1 - r.v1 * t0);
}
// p-bar += R(-x) y-bar
__device__ __forceinline__ void rot_inv_add(const Rot& r, double y0, double y1, double y2, double* pb) {
  double t0 = r.v2 * y1 - r.v1 * y2;
  double t1 = r.v0 * y2 - r.v2 * y0;
  double t2 = r.v1 * y0 - r.v0 * y1;
  t0 = t0 + t0;
  t1 = t1 + t1;
  t2 = t2 + t2;
  pb[0] += (y0 + r.c * t0) + (r.v2 * t1 - r.v1 * t2);
  pb[1] += (y1 + r.c * t1) + (r.v0 * t2 - r.v2 * t0);
  pb[2] += (y2 + r.c * t2) + (r.v1 * t0 - r.v0 * t1);
}
__device__ __forceinline__ void cross(const double* a, const double* b, double* o) {
  o[0] = a[1] * b[2] - a[2] * b[1];
  o[1] = a[2] * b[0] - a[0] * b[2];
  o[2] = a[0] * b[1] - a[1] * b[0];
}
// x-bar = Jl(x)^T w = w - a (x x w) + b x x (x x w)
__device__ __forceinline__ void jl_t(const Rot& r, const double* w, double* o) {
  const double x[3] = {r.x0, r.x1, r.x2};
  double c1[3], c2[3];
  cross(x, w, c1);
  cross(x, c1, c2);
#pragma unroll
  for (int i = 0; i < 3; ++i) o[i] = (w[i] - r.ja * c1[i]) + r.jb * c2[i];
}

// Sums of the lanes' NV <= 8 values over the wavefront, in a fixed order: value lane / 8 in
// every lane (halving steps that add pairs of lanes for two values at once).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) { return as_double(dpp_u64<CTRL>(as_bits(x))); }
__device__ __forceinline__ double swap_add32_f64(double a, double b) {
  const unsigned long long x = as_bits(a), y = as_bits(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  return as_double(((unsigned long long)hi[0] << 32) | lo[0]) + as_double(((unsigned long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double swap_add16_f64(double a, double b) {
  const unsigned long long x = as_bits(a), y = as_bits(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  return as_double(((unsigned long long)hi[0] << 32) | lo[0]) + as_double(((unsigned long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double sum8_f64(double x) {
  x += dpp_f64<kDppXor1>(x);
  x += dpp_f64<kDppXor2>(x);
  x += dpp_f64<kDppHalfMirror>(x);
  return x;
}
template <int NV>
__device__ __forceinline__ double wave_sums_f64(const double (&v)[NV], int lane) {
  const auto at = [&](int i) { return i < NV ? v[i < NV ? i : 0] : 0.0; };
  const double z0 = swap_add16_f64(swap_add32_f64(at(0), at(4)), swap_add32_f64(at(2), at(6)));
  const double z1 = swap_add16_f64(swap_add32_f64(at(1), at(5)), swap_add32_f64(at(3), at(7)));
  const bool up = lane & 8;
  return sum8_f64((up ? z1 : z0) + dpp_f64<kDppRor8>(up ? z0 : z1));
}

// Deterministic grid sum of NV per-thread values: lanes of a wavefront, the block's waves in
// order, the blocks of a die (blockIdx % 8) in eight interleaved ascending chains, the dies
// -- every order fixed by the grid.  Partials and sums travel as tagged words (a 32-bit
// barrier epoch and a 32-bit half of the double): block b > 7 publishes its 2 NV words in its
// slot, block b mod 8 gathers its die's slots and publishes the die's sum, and every block
// polls the 8 dies' words.  A slot is rewritten at epoch e + 1 after its block has read the
// dies' sums of e, which its die's gathering block published after reading the slot; the
// dies' words alternate between two regions (a gathering block that publishes e + 2 has read
// every die's e + 1, so every block has read all of e).  A grid of one block adds in LDS.
// One block gathering all partials and publishing the result in 8 copies cost about 2 us
// more at 196 blocks (four sums a reverse step).
// overlap: work of every thread that needs no sum, run between publication and poll.
// The result lands in res[0..NV) of every block.  Returns false if the barrier was abandoned
// (time limit or abort).
struct NoOverlap {
  __device__ __forceinline__ void operator()() const {}
};
struct SumLds {
  double sw[kBlock / 64][8];
  unsigned half[kAdjDieBlocks * 12];
  double res[8];
  int bad;
};
template <int NV, int BS, typename OV = NoOverlap>
__device__ __forceinline__ bool grid_sum(const AdjArgs& a, unsigned epoch, const double (&v)[NV], SumLds& L,
                                         OV overlap = OV{}) {
  constexpr int W = 2 * NV;        // words per partial
  static_assert(W <= 12 && 8 * W <= BS, "too many words");
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const unsigned want = epoch + 1u;
  const unsigned long long tg = (unsigned long long)want << 32;
  const unsigned die = blockIdx.x % 8u, slot = blockIdx.x / 8u, nd = (gridDim.x + 7u - die) / 8u;
  unsigned long long* part = reinterpret_cast<unsigned long long*>(a.sync + kSyncPart);
  unsigned long long* dw = reinterpret_cast<unsigned long long*>(a.sync + kSyncJTag) + (size_t)(epoch & 1u) * 8 * kTagWords64;
  const double t = wave_sums_f64<NV>(v, lane);
  if ((lane & 7) == 0 && (lane >> 3) < NV) L.sw[wid][lane >> 3] = t;
  __syncthreads();
  const unsigned long long t0 = wall_clock64();
  int ok = 1;
  // a word of a slot or of a die's sum, once it carries the epoch
  const auto poll = [&](const unsigned long long* w) {
    unsigned long long x = 0;
    for (unsigned it = 1; ok; ++it) {
      x = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((unsigned)(x >> 32) == want) break;
      if ((it & 31u) == 0u && give_up(a.sync, a.cancel, t0, a.timeout_ticks, it)) ok = 0;
      __builtin_amdgcn_s_sleep(1);
    }
    return (unsigned)x;
  };
  if (tid < W) {   // half tid % 2 of block sum tid / 2
    double blk = 0.0;
#pragma unroll
    for (int w = 0; w < BS / 64; ++w) blk += L.sw[w][tid >> 1];
    const unsigned long long bits = as_bits(blk);
    const unsigned half = (tid & 1) ? (unsigned)(bits >> 32) : (unsigned)bits;
    if (gridDim.x == 1) {
      if (tid & 1) L.res[tid >> 1] = blk;
    } else if (slot == 0) {
      L.half[tid] = half;
    } else {
      __hip_atomic_store(part + (size_t)blockIdx.x * kTagWords64 + tid, tg | half, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  overlap();
  if (gridDim.x > 1) {
    if (slot == 0) {   // this block gathers its die
      for (unsigned i = tid + W; i < nd * W; i += BS)
        L.half[i] = poll(part + (size_t)(die + 8u * (i / W)) * kTagWords64 + i % W);
      __syncthreads();
      const int val = tid >> 3;
      if (val < NV) {
        double s = 0.0;
        for (unsigned j = tid & 7; j < nd; j += 8)
          s += as_double(((unsigned long long)L.half[j * W + 2 * val + 1] << 32) | L.half[j * W + 2 * val]);
        s = sum8_f64(s);
        if ((tid & 7) < 2 && !__any(!ok)) {
          const unsigned long long bits = as_bits(s);
          __hip_atomic_store(dw + (size_t)die * kTagWords64 + 2 * val + (tid & 1),
                             tg | ((tid & 1) ? (bits >> 32) : (bits & 0xffffffffull)), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    // thread (word, die): the 8 dies of a word in 8 consecutive lanes, the halves of a value
    // in 16
    if (tid < 8 * W) {
      const unsigned c = tid & 7, w = tid >> 3;
      const unsigned x = (c < gridDim.x) ? poll(dw + (size_t)c * kTagWords64 + w) : 0u;
      const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, kDppRor8, 0xf, 0xf, true);
      const double s = sum8_f64(as_double((w & 1) ? ((unsigned long long)x << 32) | o : ((unsigned long long)o << 32) | x));
      if ((tid & 15) == 0) L.res[w >> 1] = s;
    }
  }
  if (!ok) L.bad = 1;
  __syncthreads();
  return L.bad == 0;
}

// Per-beam constants and adjoint registers.
struct AdjBeam {
  double P[3];      // state at the start of the step being reversed
  double Pb[3];     // adjoint of the state
  double F1[3];     // adjoint of f1 (accumulated over phases A, C, D)
  double Tb[3];     // Theta-bar (enters f2-bar and f3-bar)
  double c0, cm, c1, hc0, hcm, hc1;
  double u;
  double bx, bz, w; // vacuum terms and weight of the beam's energy
  // sums over the reverse steps of the adjoints of B_x, B_z and w, whose derivatives with
  // respect to theta_v and the luminosities are the same at every step
  double gx, gz, gw;
  int s, k;
  bool on;
};

// Adjoint of B at one stage: moment-adjoint contributions S B-bar and c S B-bar of the
// beam, and the direct parameter terms (theta_v through B_vac, n0 through lambda).
__device__ __forceinline__ void b_bar(AdjBeam& q, const double* Bb, double c, const Radial& g, double (&red)[6],
                                      double& gn0) {
  const double sg = q.s ? -1.0 : 1.0;
  const double S0 = sg * Bb[0], S1 = Bb[1], S2 = sg * Bb[2];
  red[0] += S0;
  red[1] += S1;
  red[2] += S2;
  red[3] += c * S0;
  red[4] += c * S1;
  red[5] += c * S2;
  q.gx += Bb[0];
  q.gz += Bb[2];
  gn0 += S2 * g.qp;
}

// Broadcast of a moment adjoint (J0-bar | J1-bar) onto a stage state y at cos c:
// y-bar = g S (J0-bar/c + J1-bar); the weight adjoint (S y).(J0-bar/c + J1-bar) feeds the
// luminosity gradients.  Far out the two terms nearly cancel, so J0-bar/c is divided exactly
// (a factor 1/c doubles the gradients' error), its three quotients from one reciprocal (0 < c <= 1;
// below 2^-960, moment adjoints of cotangents that small, they are within two ulp).
__device__ __forceinline__ void m_bar(AdjBeam& q, const double* Jb, double c, const double* y, double* yb) {
  const double sg = q.s ? -1.0 : 1.0;
  const double r = rcp_step(c, rcp_step(c, __builtin_amdgcn_rcp(c)));
  const double v0 = div_by_rcp(Jb[0], c, r) + Jb[3], v1 = div_by_rcp(Jb[1], c, r) + Jb[4],
               v2 = div_by_rcp(Jb[2], c, r) + Jb[5];
  yb[0] = q.w * (sg * v0);
  yb[1] = q.w * v1;
  yb[2] = q.w * (sg * v2);
  q.gw += ((sg * y[0]) * v0 + y[1] * v1) + (sg * y[2]) * v2;
}

__device__ __forceinline__ void stage_f(const AdjBeam& q, const double* J, const Radial& g, double c, double hc,
                                        double* f) {
  double nn[3];
  nunu<3>(J, g.mu, c, nn);
  gen2(q.s, q.bx, q.bz, g.lam, nn, hc, f);
}

// Beam b's fixed labels, its adjoint initialised from the cotangent (L = sum_b c_b Pee_b,
// Pee = (1 + P_z)/2).
__device__ __forceinline__ void beam_init(const AdjArgs& a, long long b, bool on, AdjBeam& q) {
  q.on = on;
  const long long bb = on ? b : 0;
  const long long row = bb / a.NE;
  q.k = (int)(bb - row * a.NE);
  q.s = (int)(row / a.NU);
  q.u = u_of((int)(row - (long long)q.s * a.NU), a.NU);
  q.bx = a.tab[q.k];
  q.bz = a.tab[a.NE + q.k];
  q.w = a.tab[(size_t)(2 + q.s) * a.NE + q.k];
  const double cb = on ? (a.cot ? a.cot[b] : a.cot_const) : 0.0;
  q.Pb[0] = 0.0;
  q.Pb[1] = 0.0;
  q.Pb[2] = 0.5 * cb;
  q.gx = q.gz = q.gw = 0.0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    q.F1[c] = 0.0;
    q.Tb[c] = 0.0;
    q.P[c] = 0.0;
  }
  q.c0 = q.cm = q.c1 = 1.0;
  q.hc0 = q.hcm = q.hc1 = 0.0;
}
// The beam's sums onto the thread's parameter gradients (L_e, L_ebar, L_x, theta_v).
__device__ __forceinline__ void beam_grads(const AdjArgs& a, AdjBeam& q, double (&gacc)[5]) {
  const double* d = a.dtab + q.k;
  const size_t NE = (size_t)a.NE;
  const double gl = q.gw * d[q.s * NE];
  if (q.s) gacc[1] += gl;
  else gacc[0] += gl;
  gacc[2] += q.gw * d[2 * NE];
  gacc[3] += q.gx * d[3 * NE] + q.gz * d[4 * NE];
  q.gx = q.gz = q.gw = 0.0;
}

// Recompute beam b's states over a segment of len steps from its checkpoint with the
// recorded moments (the stepping kernel's arithmetic, hence its bits) into the tape.
template <bool SK>
__device__ __forceinline__ void recompute_segment(const AdjArgs& a, const AdjBeam& q, long long b, long long seg,
                                                  long long s0, long long len) {
  const long long plane = a.plane;
  const double* ck = a.ck + (size_t)seg * 3 * plane;
  double P0 = ck[b], P1 = ck[b + plane], P2 = ck[b + 2 * plane];
  for (long long t = 0; t < len; ++t) {
    double* tp = a.tape + (size_t)t * 3 * plane;
    tp[b] = P0;
    tp[b + plane] = P1;
    tp[b + 2 * plane] = P2;
    if (t + 1 == len) break;
    const long long n = s0 + t;
    const double r0 = a.rs + (double)n * a.h;
    const double rm = r0 + 0.5 * a.h;
    const double r1 = a.rs + (double)(n + 1) * a.h;
    const Radial g0 = radial(a.R, a.ne_power, a.lam0, r0), gm = radial(a.R, a.ne_power, a.lam0, rm),
                 g1 = radial(a.R, a.ne_power, a.lam0, r1);
    const RowGeo rg = row_geo_in_range(q.u, a.h, g0, gm, g1);
    const double* J = a.Jhist + (size_t)n * 24;
    double n1[3], n2[3], n3[3], n4[3], f1[3], f2[3], f3[3], f4[3];
    nunu<3>(J, g0.mu, rg.c0, n1);
    nunu<3>(J + 6, gm.mu, rg.cm, n2);
    nunu<3>(J + 12, gm.mu, rg.cm, n3);
    nunu<3>(J + 18, g1.mu, rg.c1, n4);
    const double bx = q.bx, bz = q.bz;
    gen2(q.s, bx, bz, g0.lam, n1, rg.hc0, f1);
    gen2(q.s, bx, bz, gm.lam, n2, rg.hcm, f2);
    gen2(q.s, bx, bz, gm.lam, n3, rg.hcm, f3);
    gen2(q.s, bx, bz, g1.lam, n4, rg.hc1, f4);
    const double cr0 = f1[1] * f4[2] - f1[2] * f4[1];
    const double cr1 = f1[2] * f4[0] - f1[0] * f4[2];
    const double cr2 = f1[0] * f4[1] - f1[1] * f4[0];
    const double t0 = (((f1[0] + 2.0 * f2[0]) + 2.0 * f3[0]) + f4[0]) * (1.0 / 6.0) - cr0 * (1.0 / 12.0);
    const double t1 = (((f1[1] + 2.0 * f2[1]) + 2.0 * f3[1]) + f4[1]) * (1.0 / 6.0) - cr1 * (1.0 / 12.0);
    const double t2 = (((f1[2] + 2.0 * f2[2]) + 2.0 * f3[2]) + f4[2]) * (1.0 / 6.0) - cr2 * (1.0 / 12.0);
    rotate2<false, SK>(t0, t1, t2, P0, P1, P2);
    if (a.renorm) {   // as the forward stepper: one Newton step for 1/sqrt from 1
      const double nrm2 = (P0 * P0 + P1 * P1) + P2 * P2;
      const double inv = fma(-0.5, nrm2, 1.5);
      P0 = P0 * inv;
      P1 = P1 * inv;
      P2 = P2 * inv;
    }
  }
}

// The state at the start of the step being reversed (tape slot t) and the beam's geometry
// at the step's three stage radii.
__device__ __forceinline__ void load_step(const AdjArgs& a, AdjBeam& B, long long b, long long t,
                                          const Radial& g0, const Radial& gm, const Radial& g1) {
  const double* tp = a.tape + (size_t)t * 3 * a.plane;
  B.P[0] = tp[b];
  B.P[1] = tp[b + a.plane];
  B.P[2] = tp[b + 2 * a.plane];
  const RowGeo rg = row_geo_in_range(B.u, a.h, g0, gm, g1);
  B.c0 = rg.c0; B.cm = rg.cm; B.c1 = rg.c1;
  B.hc0 = rg.hc0; B.hcm = rg.hcm; B.hc1 = rg.hc1;
}

// A: P_{n+1} = R(Theta) P_n / |.|  ->  Theta-bar, f4-bar
template <bool SK>
__device__ __forceinline__ void phase_a(int renorm, AdjBeam& B, const double (*sJ)[6], const Radial& g0,
                                        const Radial& gm, const Radial& g1, double (&red)[6], double& gn0) {
  double f1[3], f2[3], f3[3], f4[3], cr[3];
  stage_f(B, sJ[0], g0, B.c0, B.hc0, f1);
  stage_f(B, sJ[1], gm, B.cm, B.hcm, f2);
  stage_f(B, sJ[2], gm, B.cm, B.hcm, f3);
  stage_f(B, sJ[3], g1, B.c1, B.hc1, f4);
  cross(f1, f4, cr);
  double th[3];
#pragma unroll
  for (int c = 0; c < 3; ++c)
    th[c] = (((f1[c] + 2.0 * f2[c]) + 2.0 * f3[c]) + f4[c]) * (1.0 / 6.0) - cr[c] * (1.0 / 12.0);
  const Rot R = make_rot<SK>(th[0], th[1], th[2]);
  double Pp[3];
  rot_fwd(R, B.P[0], B.P[1], B.P[2], Pp[0], Pp[1], Pp[2]);
  double Ppb[3] = {B.Pb[0], B.Pb[1], B.Pb[2]};
  if (renorm) {
    // y = P (1.5 - |P|^2 / 2): P-bar = (1.5 - |P|^2 / 2) y-bar - P (P . y-bar)
    const double sf = fma(-0.5, (Pp[0] * Pp[0] + Pp[1] * Pp[1]) + Pp[2] * Pp[2], 1.5);
    const double d = (Pp[0] * Ppb[0] + Pp[1] * Ppb[1]) + Pp[2] * Ppb[2];
    Ppb[0] = sf * Ppb[0] - Pp[0] * d;
    Ppb[1] = sf * Ppb[1] - Pp[1] * d;
    Ppb[2] = sf * Ppb[2] - Pp[2] * d;
  }
  B.Pb[0] = B.Pb[1] = B.Pb[2] = 0.0;
  rot_inv_add(R, Ppb[0], Ppb[1], Ppb[2], B.Pb);
  double om[3], tb[3], c4[3], c1v[3], f4b[3];
  cross(Pp, Ppb, om);
  jl_t(R, om, tb);
  cross(f4, tb, c4);
  cross(tb, f1, c1v);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    B.F1[c] = tb[c] * (1.0 / 6.0) - c4[c] * (1.0 / 12.0);
    f4b[c] = tb[c] * (1.0 / 6.0) - c1v[c] * (1.0 / 12.0);
    B.Tb[c] = tb[c];
  }
  const double Bb[3] = {B.hc1 * f4b[0], B.hc1 * f4b[1], B.hc1 * f4b[2]};
  b_bar(B, Bb, B.c1, g1, red, gn0);
}
// B: Y4 = R(f3) P  ->  f3-bar
template <bool SK>
__device__ __forceinline__ void phase_b(AdjBeam& B, const double (*sJ)[6], const double* Jb,
                                        const Radial& gm, double (&red)[6], double& gn0) {
  double f3[3], Y[3], Yb[3], om[3], f3b[3];
  stage_f(B, sJ[2], gm, B.cm, B.hcm, f3);
  const Rot R = make_rot<SK>(f3[0], f3[1], f3[2]);
  rot_fwd(R, B.P[0], B.P[1], B.P[2], Y[0], Y[1], Y[2]);
  m_bar(B, Jb, B.c1, Y, Yb);
  rot_inv_add(R, Yb[0], Yb[1], Yb[2], B.Pb);
  cross(Y, Yb, om);
  jl_t(R, om, f3b);
#pragma unroll
  for (int c = 0; c < 3; ++c) f3b[c] += B.Tb[c] * (1.0 / 3.0);
  const double Bb[3] = {B.hcm * f3b[0], B.hcm * f3b[1], B.hcm * f3b[2]};
  b_bar(B, Bb, B.cm, gm, red, gn0);
}
// C: Y3 = R(Om) P, Om = f2/2 - (f1 x f2)/8  ->  f2-bar, f1-bar
template <bool SK>
__device__ __forceinline__ void phase_c(AdjBeam& B, const double (*sJ)[6], const double* Jb,
                                        const Radial& g0, const Radial& gm, double (&red)[6], double& gn0) {
  double f1[3], f2[3], cr[3], Y[3], Yb[3], om[3], ob[3], a1[3], a2[3], f2b[3];
  stage_f(B, sJ[0], g0, B.c0, B.hc0, f1);
  stage_f(B, sJ[1], gm, B.cm, B.hcm, f2);
  cross(f1, f2, cr);
  const Rot R = make_rot<SK>(0.5 * f2[0] - 0.125 * cr[0], 0.5 * f2[1] - 0.125 * cr[1],
                         0.5 * f2[2] - 0.125 * cr[2]);
  rot_fwd(R, B.P[0], B.P[1], B.P[2], Y[0], Y[1], Y[2]);
  m_bar(B, Jb, B.cm, Y, Yb);
  rot_inv_add(R, Yb[0], Yb[1], Yb[2], B.Pb);
  cross(Y, Yb, om);
  jl_t(R, om, ob);
  cross(ob, f1, a1);
  cross(f2, ob, a2);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    f2b[c] = (0.5 * ob[c] - a1[c] * 0.125) + B.Tb[c] * (1.0 / 3.0);
    B.F1[c] -= a2[c] * 0.125;
  }
  const double Bb[3] = {B.hcm * f2b[0], B.hcm * f2b[1], B.hcm * f2b[2]};
  b_bar(B, Bb, B.cm, gm, red, gn0);
}
// D: Y2 = R(f1/2) P  ->  f1-bar complete
template <bool SK>
__device__ __forceinline__ void phase_d(AdjBeam& B, const double (*sJ)[6], const double* Jb,
                                        const Radial& g0, double (&red)[6], double& gn0) {
  double f1[3], Y[3], Yb[3], om[3], ob[3];
  stage_f(B, sJ[0], g0, B.c0, B.hc0, f1);
  const Rot R = make_rot<SK>(0.5 * f1[0], 0.5 * f1[1], 0.5 * f1[2]);
  rot_fwd(R, B.P[0], B.P[1], B.P[2], Y[0], Y[1], Y[2]);
  m_bar(B, Jb, B.cm, Y, Yb);
  rot_inv_add(R, Yb[0], Yb[1], Yb[2], B.Pb);
  cross(Y, Yb, om);
  jl_t(R, om, ob);
#pragma unroll
  for (int c = 0; c < 3; ++c) B.F1[c] += 0.5 * ob[c];
  const double Bb[3] = {B.hc0 * B.F1[0], B.hc0 * B.F1[1], B.hc0 * B.F1[2]};
  b_bar(B, Bb, B.c0, g0, red, gn0);
}
// J^(1) = M(P_n): the moment adjoint broadcast onto the state itself
__device__ __forceinline__ void phase_e(AdjBeam& B, const double* Jb) {
  double Yb[3];
  m_bar(B, Jb, B.c0, B.P, Yb);
  B.Pb[0] += Yb[0];
  B.Pb[1] += Yb[1];
  B.Pb[2] += Yb[2];
}

// Adjoint registers of beam b kept in the workspace between phases (spill mode): P-bar,
// f1-bar, Theta-bar as nine planes of a.plane doubles.
__device__ __forceinline__ void adj_load(const AdjArgs& a, AdjBeam& B, long long b) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    B.Pb[c] = a.spill[(size_t)c * a.plane + b];
    B.F1[c] = a.spill[(size_t)(3 + c) * a.plane + b];
    B.Tb[c] = a.spill[(size_t)(6 + c) * a.plane + b];
  }
}
__device__ __forceinline__ void adj_store(const AdjArgs& a, const AdjBeam& B, long long b) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    a.spill[(size_t)c * a.plane + b] = B.Pb[c];
    a.spill[(size_t)(3 + c) * a.plane + b] = B.F1[c];
    a.spill[(size_t)(6 + c) * a.plane + b] = B.Tb[c];
  }
}

// BPT > 0: thread gt owns beams gt + i nthr (i < BPT) and keeps their adjoint state in its
// registers, or what the compiler spills of it (at 256 VGPRs 104 bytes of scratch per lane for
// two beams, 768 for four; none for one), for the whole launch.  BPT = 0 (spill mode, any number of beams): each phase loops over the
// thread's beams gt, gt + nthr, ..., reading and writing their adjoint registers in the
// workspace and recomputing the state and geometry from the tape.  Reverse pass of 24 steps, four beams
// per thread against spill mode: 300k beams 1.62 and 1.38 ms, 400k 1.76 and 1.83, 520k 1.92 and 2.13.
// Bound: VALU issue and the latency of a phase's chain (one rotation with its Jacobian) plus
// the grid sums.  Between the publication of a step's last sum and the poll for it every
// thread loads its next step's states and computes that step's geometry (one radius of three:
// r0 of step n is r1 of step n - 1), and the recorded moments of the step go to LDS.
template <int BPT, int BS>
__global__ void __launch_bounds__(BS) k_adjoint2(AdjArgs a) {
  // one wavefront per SIMD has registers for the literals and no other wavefront's vector
  // instructions to issue the moves beside
  constexpr bool kSK = BPT != 1 || BS != kBlockSmall;
  __shared__ double sJ[2][24];
  __shared__ SumLds L;
  constexpr int NQ = BPT > 0 ? BPT : 1;
  if (launch_aborted(a.sync)) return;
  const int tid = threadIdx.x;
  const long long nthr = (long long)gridDim.x * BS;
  const long long gt = (long long)blockIdx.x * BS + tid;
  const int renorm = a.renorm;
  if (tid == 0) L.bad = 0;
  AdjBeam q[NQ];
  if constexpr (BPT > 0) {
#pragma unroll
    for (int i = 0; i < BPT; ++i) beam_init(a, gt + i * nthr, gt + i * nthr < a.nb, q[i]);
  } else {
    for (long long b = gt; b < a.nb; b += nthr) {
      beam_init(a, b, true, q[0]);
      adj_store(a, q[0], b);
    }
  }
  double gacc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  // every beam of this thread (register mode: its BPT slots; spill mode: all of them, each
  // loaded and stored around fn)
  auto each = [&](auto fn, long long t, const Radial& g0, const Radial& gm, const Radial& g1) {
    if constexpr (BPT > 0) {
#pragma unroll
      for (int i = 0; i < BPT; ++i)
        if (q[i].on) fn(q[i]);
    } else {
      for (long long b = gt; b < a.nb; b += nthr) {
        beam_init(a, b, true, q[0]);
        adj_load(a, q[0], b);
        load_step(a, q[0], b, t, g0, gm, g1);
        fn(q[0]);
        adj_store(a, q[0], b);
        beam_grads(a, q[0], gacc);
      }
    }
  };
  double gn0 = 0.0;   // sum of S B_z-bar (R/r)^p
  unsigned epoch = 0;
  bool ok = true;
  for (long long seg = a.nseg - 1; ok && seg >= 0; --seg) {
    const long long s0 = a.n0 + seg * a.ckpt;
    const long long len = min(a.ckpt, a.n0 + a.nsteps - s0);
    // -- recompute the segment's states from its checkpoint with the recorded moments
    if constexpr (BPT > 0) {
#pragma unroll
      for (int i = 0; i < BPT; ++i)
        if (q[i].on) recompute_segment<kSK>(a, q[i], gt + i * nthr, seg, s0, len);
    } else {
      for (long long b = gt; b < a.nb; b += nthr) {
        beam_init(a, b, true, q[0]);
        recompute_segment<kSK>(a, q[0], b, seg, s0, len);
      }
    }
    // -- reverse steps of the segment
    const auto rad = [&](double r) { return radial(a.R, a.ne_power, a.lam0, r); };
    const auto at = [&](long long n) { return a.rs + (double)n * a.h; };
    Radial g0 = rad(at(s0 + len - 1)), gm = rad(at(s0 + len - 1) + 0.5 * a.h), g1 = rad(at(s0 + len));
    if constexpr (BPT > 0) {
#pragma unroll
      for (int i = 0; i < BPT; ++i)
        if (q[i].on) load_step(a, q[i], gt + i * nthr, len - 1, g0, gm, g1);
    }
    __syncthreads();   // the last segment's moments have been read
    if (tid < 24) sJ[0][tid] = a.Jhist[(size_t)(s0 + len - 1) * 24 + tid];
    __syncthreads();
    int cur = 0;
    for (long long t = len - 1; ok && t >= 0; --t) {
      const long long n = s0 + t;
      const double (*J)[6] = reinterpret_cast<const double (*)[6]>(sJ[cur]);
      double red[6];
      double Jb[6];
      // the adjoints of the moments from their sums
      const auto moments = [&](double mu) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          Jb[c] = mu * L.res[c];
          Jb[3 + c] = -(mu * L.res[3 + c]);
        }
#pragma unroll
        for (int c = 0; c < 6; ++c) red[c] = 0.0;
      };
#pragma unroll
      for (int c = 0; c < 6; ++c) red[c] = 0.0;
      each([&](AdjBeam& B) { phase_a<kSK>(renorm, B, J, g0, gm, g1, red, gn0); }, t, g0, gm, g1);
      if (!(ok = grid_sum<6, BS>(a, epoch++, red, L))) break;
      moments(g1.mu);
      each([&](AdjBeam& B) { phase_b<kSK>(B, J, Jb, gm, red, gn0); }, t, g0, gm, g1);
      if (!(ok = grid_sum<6, BS>(a, epoch++, red, L))) break;
      moments(gm.mu);
      each([&](AdjBeam& B) { phase_c<kSK>(B, J, Jb, g0, gm, red, gn0); }, t, g0, gm, g1);
      if (!(ok = grid_sum<6, BS>(a, epoch++, red, L))) break;
      moments(gm.mu);
      each([&](AdjBeam& B) { phase_d<kSK>(B, J, Jb, g0, red, gn0); }, t, g0, gm, g1);
      double PN[NQ][3], c0n[NQ], cmn[NQ], h0n[NQ], hmn[NQ];
      Radial gn = g0, gnm = g0;
      ok = grid_sum<6, BS>(a, epoch++, red, L, [&] {
        if (t == 0) return;
        if (tid < 24) sJ[cur ^ 1][tid] = a.Jhist[(size_t)(n - 1) * 24 + tid];
        gn = rad(at(n - 1));
        gnm = rad(at(n - 1) + 0.5 * a.h);
        if constexpr (BPT > 0) {
          const double* tp = a.tape + (size_t)(t - 1) * 3 * a.plane;
#pragma unroll
          for (int i = 0; i < BPT; ++i) {
            if (!q[i].on) continue;
#pragma unroll
            for (int c = 0; c < 3; ++c) PN[i][c] = tp[gt + i * nthr + c * a.plane];
            row_cos(q[i].u, a.h, gn.q2, c0n[i], h0n[i]);
            row_cos(q[i].u, a.h, gnm.q2, cmn[i], hmn[i]);
          }
        }
      });
      if (!ok) break;
      moments(g0.mu);
      each([&](AdjBeam& B) { phase_e(B, Jb); }, t, g0, gm, g1);
      if constexpr (BPT > 0) {
        if (t > 0) {
#pragma unroll
          for (int i = 0; i < BPT; ++i) {
            if (!q[i].on) continue;
#pragma unroll
            for (int c = 0; c < 3; ++c) q[i].P[c] = PN[i][c];
            q[i].c1 = q[i].c0; q[i].hc1 = q[i].hc0;
            q[i].c0 = c0n[i]; q[i].hc0 = h0n[i];
            q[i].cm = cmn[i]; q[i].hcm = hmn[i];
          }
        }
      }
      g1 = g0;
      g0 = gn;
      gm = gnm;
      cur ^= 1;
    }
  }
  if (!ok) return;
  if (a.state_bar) {
    if constexpr (BPT > 0) {
#pragma unroll
      for (int i = 0; i < BPT; ++i) {
        if (!q[i].on) continue;
        const long long b = gt + i * nthr;
        a.state_bar[b] = q[i].Pb[0];
        a.state_bar[b + a.nb] = q[i].Pb[1];
        a.state_bar[b + 2 * a.nb] = q[i].Pb[2];
      }
    } else {
      for (long long b = gt; b < a.nb; b += nthr)
#pragma unroll
        for (int c = 0; c < 3; ++c) a.state_bar[b + c * a.nb] = a.spill[(size_t)c * a.plane + b];
    }
  }
  if constexpr (BPT > 0) {
#pragma unroll
    for (int i = 0; i < BPT; ++i)
      if (q[i].on) beam_grads(a, q[i], gacc);
  }
  gacc[4] = gn0 * a.s2gf;
  if (grid_sum<5, BS>(a, epoch++, gacc, L) && blockIdx.x == 0 && tid < 5) a.out[tid] = L.res[tid];
}

template __global__ void k_adjoint2<0, kBlock>(AdjArgs);
template __global__ void k_adjoint2<1, kBlock>(AdjArgs);
template __global__ void k_adjoint2<2, kBlock>(AdjArgs);
template __global__ void k_adjoint2<4, kBlock>(AdjArgs);
template __global__ void k_adjoint2<1, kBlockSmall>(AdjArgs);

}  // namespace nb
