// nb_kernels.hip -- persistent CDNA4 kernels of the bulb-model radial stepper.
//
// One persistent launch advances every beam by `nsteps` radial steps.  Work unit: one
// (species, emission-bin) row of N_E beams per wavefront -- the paper's NBeam with its
// SIMD loop over energy bins (Sec. 3.3) mapped onto 64 lanes.  Per RK stage each wave
//   1. streams its rows' state planes (SoA, coalesced 64 x 8 B per load),
//   2. rebuilds every beam's stage generator from the global stage moments (no per-beam
//      stage storage: F_1..F_{i-1} are recomputed from J^(1..i-1)),
//   3. applies the exact exponential to get the stage state Y_i (Eq. U),
//   4. accumulates the beam's moment contribution as a 64-bit fixed-point integer; the
//      lanes' sums fold to the row's exact energy sum (wave_fold), then the angle sum (1/cos
//      weighting for J0) is added to per-lane 128-bit totals,
// then the block folds its waves through LDS and adds its partial to counted accumulators,
// whose published totals every block reads as J^(i) (agent-scope atomics).
// Four barriers per step; the final pass writes rho_{n+1} and also produces the next
// step's stage-1 moments.
#include "nb_device.h"
#include "nb_device32.h"
#include "nb_internal.h"
#include "nb_stage.h"
#include <type_traits>

namespace nb {

__device__ __forceinline__ Radial radial_at(const StepArgs& a, double r) {
  return radial(a.R, a.ne_power, a.lam0, r);
}

// Grid-wide reduction of the stage moments: counted accumulators, one copy per die, whose
// totals are published and read by every block.
//  * A block's partial is NV 128-bit sums, each below 2^93 in magnitude (a row's term is
//    below 2^62), as 2 NV chunks: bits 0..46 and bits 47..93 (biased by 2^46).  A 64-bit
//    accumulator holds the sum of chunks in its upper 55 bits and the count of adds, modulo
//    512, in its lower 9, so one atomic add both delivers a chunk and announces it.  Block b
//    adds to copy b % 8, n_c <= 256 blocks to a copy.
//  * Accumulators are never cleared during a launch.  The block whose add completes the
//    count (e + 1) n_c of epoch e knows it from the value the add returned, and stores the
//    word's running sum, modulo 2^55, under a 9-bit epoch tag into the published words of
//    the epoch's parity.  (A copy of one block needs no accumulator: its block keeps the
//    running sum itself.)
//  * Every block polls the 8 copies of the 2 NV published words for the epoch's tag, takes
//    the differences from the previous epoch's running sums (below 2^55, at most 256 chunks
//    below 2^47), adds the copies in 64-bit integers and combines the chunks to the exact
//    128-bit totals: the same integers in every block, whatever the order.
// A published word of parity e % 2 is overwritten at epoch e by a block that has passed
// barrier e - 1, so every block has added for e - 1 and hence has read all of e - 2.  All
// words are zeroed before each launch and tags start at 1; a polled word holds tag e - 1 or
// e + 1 (modulo 512), never an older one.
// A grid of one block keeps its moments in LDS.
// Bound: two trips beyond the die (the add within it, then store to poll) of about 0.8 us
// together with the skew of the blocks.  Measured per barrier in a loop of nothing else, 250
// blocks, 12 / 32 words: 2.2 / 2.7 us, and 3.6 / 3.8 us with arrivals spread over 2 us,
// against 3.1 / 3.6 and 4.9 / 5.3 us for slots of tagged words that every block gathers from
// every other (64 KB per block and poll round).  Polling the accumulators themselves saves
// a trip (1.65 / 1.76 us) but every early poll delays the adds that it waits for: 5.6 / 7.3
// us with the spread arrivals, and the 200k-beam step 33 against 26 us.
// Returns false if the barrier was abandoned (time limit or abort).
constexpr unsigned long long kMask47 = (1ull << 47) - 1ull;
constexpr unsigned long long kTag9 = 511ull;
// 47-bit chunk k of a 128-bit value below 2^93 in magnitude: k = 0 the unsigned bits
// 0..46, k = 1 the signed bits 47..93 plus 2^46.
__device__ __forceinline__ unsigned long long chunk_field(const I128& x, int k) {
  const unsigned long long hi = (x.lo >> 47) | ((unsigned long long)x.hi << 17);
  return (k ? hi + (1ull << 46) : x.lo) & kMask47;
}
template <int NC>
__device__ __forceinline__ int fold_comp(int lane);     // lane layout of the moment totals, below
template <int NC>
__device__ __forceinline__ int fold_moment(int lane);

// LDS words of the reduction: the waves' partials, the running sums (read: those of the
// previous epoch, by polling thread; own: this block's, in a copy of one block), the block's
// abandoned flag and, for adaptive runs, the waves' error words.
template <int NV, int BS, bool MAXE = false>
struct RedLds {
  I128 sw[BS / 64][NV];
  unsigned long long read[2 * NV * kRedCopies], own[2 * NV];
  unsigned long long swm[MAXE ? BS / 64 : 1];
  int bad;
};
template <int NV, int BS, bool MAXE>
__device__ __forceinline__ void red_init(RedLds<NV, BS, MAXE>& R) {   // then a block barrier
  for (int i = threadIdx.x; i < 2 * NV * kRedCopies; i += BS) R.read[i] = 0ull;
  if (threadIdx.x < 2 * NV) R.own[threadIdx.x] = 0ull;
  if (threadIdx.x == 0) R.bad = 0;
}

// Fold the waves' per-lane totals (in the lanes of fold_comp, fold_moment) and run the grid
// reduction; the moments land in sJ.  NM moment groups of NV / NM components: J0 | J1 (| J_sc | J_ss); J1 is
// at scale 2^e1, the others at 2^e0.
// MAXE: also the largest of the lanes' error estimates emax, into *sE: every block stores
// its largest as the top 48 bits of the binary form (a non-negative double, so the integer
// order of the fields is the order of the values) under a 16-bit epoch tag in a word of its
// own, of the region of the epoch's parity, and takes the maximum over all blocks' words
// (block b writes its word of parity e % 2 at epoch e only after barrier e - 1, when every
// block has read all words of epoch e - 2).
// overlap: work of every thread that does not need the moments, run between the publication
// and the poll.
// BS: threads per block (the launch's block size).
// (always inlined: a call would take the address of the launch arguments and make the
// compiler keep a private copy of them)
struct NoOverlap {
  __device__ __forceinline__ void operator()() const {}
};
template <bool MAXE, int NM, int NV, int BS, bool RM, typename OV = NoOverlap>
__device__ __forceinline__ bool finish_stage(const StepArgs& a, unsigned epoch, I128 T, RedLds<NV, BS, RM>& R,
                                             double* sJ, OV overlap = OV{}, double emax = 0.0,
                                             double* sE = nullptr) {
  constexpr int WPB = BS / 64;
  constexpr int W = 2 * NV;   // words per copy
  static_assert(W <= kRedStride && W <= BS, "too many words");
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  constexpr int NC = NV / NM;
  const auto scale = [&](int v) { return (v / NC) == 1 ? a.p2e1 : a.p2e0; };
  if (fold_moment<NC>(lane) < NM && fold_comp<NC>(lane) < NC)
    R.sw[wid][fold_moment<NC>(lane) * NC + fold_comp<NC>(lane)] = T;
  if constexpr (MAXE) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const double o = __shfl_xor(emax, off, 64);
      emax = (o > emax) ? o : emax;
    }
    if (lane == 0) R.swm[wid] = as_bits(emax) >> 16;
  }
  __syncthreads();
  I128 blk{0ull, 0ll};
  unsigned long long f = 0;   // MAXE: the block's error field
  if (tid < W) {
    blk = R.sw[0][tid >> 1];
#pragma unroll
    for (int w = 1; w < WPB; ++w) blk = i128_add(blk, R.sw[w][tid >> 1]);
  }
  if constexpr (MAXE) {
    f = R.swm[0];
#pragma unroll
    for (int w = 1; w < WPB; ++w) f = max(f, R.swm[w]);
  }
  unsigned long long* red = reinterpret_cast<unsigned long long*>(a.sync + kSyncRed);
  unsigned long long* pub =
      reinterpret_cast<unsigned long long*>(a.sync + kSyncPub) + (size_t)(epoch & 1u) * kRedCopies * kRedStride;
  const unsigned long long tag = (epoch + 1u) & 511u;
  const unsigned long long tag16 = (epoch + 1u) & 0xffffu;
  unsigned long long* ew =
      reinterpret_cast<unsigned long long*>(a.sync + kSyncErr) + (size_t)(epoch & 1u) * kMaxBlocks;
  if (tid < W && gridDim.x > 1) {
    const unsigned me = blockIdx.x % kRedCopies;
    const unsigned nc = (gridDim.x + (kRedCopies - 1) - me) / kRedCopies;   // blocks of the copy
    const unsigned long long add = chunk_field(blk, tid & 1) << 9;
    unsigned long long sum;
    bool last = true;
    if (nc == 1) {
      sum = R.own[tid] + add;
      R.own[tid] = sum;
    } else {
      const unsigned long long n0 = (unsigned long long)epoch * nc;   // adds before this epoch
      sum = __hip_atomic_fetch_add(red + me * kRedStride + tid, add + 1ull, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT) + add + 1ull;
      last = (((unsigned)sum - (unsigned)n0) & 511u) == (nc & 511u);
      sum -= n0 + nc;
    }
    if (last)
      __hip_atomic_store(pub + me * kRedStride + tid, (sum & ~kTag9) | tag, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  }
  if (MAXE && tid == 0 && gridDim.x > 1)
    __hip_atomic_store(ew + blockIdx.x, (tag16 << 48) | f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  overlap();
  if (gridDim.x == 1) {
    if (tid < W && !(tid & 1)) sJ[tid >> 1] = i128_to_double(blk) * scale(tid >> 1);
    if (MAXE && tid == 0) *sE = as_double(f << 16);
    __syncthreads();
    return true;
  }
  int ok = 1;
  const unsigned long long t0 = wall_clock64();
  // thread i: copy i % 8 of word i / 8 (the 8 copies of a word in 8 consecutive lanes, the
  // two words of a value in 16)
  for (int i = tid; i < W * kRedCopies; i += BS) {
    const unsigned c = i % kRedCopies;
    const unsigned long long* w = pub + c * kRedStride + i / kRedCopies;
    const unsigned long long prev = R.read[i];
    unsigned long long x = prev | tag;   // a copy without blocks
    for (unsigned it = 1; c < gridDim.x; ++it) {
      x = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((x & kTag9) == tag) break;
      if ((it & 31u) == 0u && give_up(a.sync, a.cancel, t0, a.timeout_ticks, it)) {
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    x &= ~kTag9;
    R.read[i] = x;
    const int k = (i / kRedCopies) & 1;
    const unsigned long long mine = sum8((x - prev) >> 9) - (k ? (unsigned long long)gridDim.x << 46 : 0ull);
    const unsigned long long other = dpp_u64<kDppRor8>(mine);
    const unsigned long long c0 = k ? other : mine, c1 = k ? mine : other;
    const I128 tot = i128_add(I128{c0, 0ll}, I128{c1 << 47, (long long)c1 >> 17});
    const int v = i / (2 * kRedCopies);
    const double J = i128_to_double(tot) * scale(v);
    if (i % (2 * kRedCopies) == 0) sJ[v] = J;
  }
  if constexpr (MAXE) {
    f = 0;
    for (unsigned b = tid; b < gridDim.x; b += BS) {
      unsigned long long x = 0;
      for (unsigned it = 1; ok; ++it) {
        x = __hip_atomic_load(ew + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((x >> 48) == tag16) break;
        if ((it & 31u) == 0u && give_up(a.sync, a.cancel, t0, a.timeout_ticks, it)) ok = 0;
        __builtin_amdgcn_s_sleep(1);
      }
      f = max(f, x & ((1ull << 48) - 1ull));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) f = max(f, (unsigned long long)__shfl_xor(f, off, 64));
    __syncthreads();   // every thread has read the waves' words above
    if (lane == 0) R.swm[wid] = f;
  }
  if (!ok) R.bad = 1;
  __syncthreads();
  if constexpr (MAXE) {
    f = R.swm[0];
#pragma unroll
    for (int w = 1; w < WPB; ++w) f = max(f, R.swm[w]);
    if (tid == 0) *sE = as_double(f << 16);
    __syncthreads();
  }
  return R.bad == 0;
}

// Radii and length of one step: stage radii r0, rm = r0 + h/2 and r1.  On the fixed grid
// r1 = r_start + (n + 1) h (not r0 + h), as in the serial definition.
struct StepGeo {
  double r0, rm, r1, h;
};
__device__ __forceinline__ StepGeo geo_fixed(const StepArgs& a, long long n) {
  StepGeo g;
  g.r0 = a.rs + (double)n * a.h;
  g.rm = g.r0 + 0.5 * a.h;
  g.r1 = a.rs + (double)(n + 1) * a.h;
  g.h = a.h;
  return g;
}

// ------------------------------------------------------------- row helpers
// Fixed-point scales of one model: 2^e1, 2^e0, 2^-e1, 2^-e0.
struct Scales {
  double s1, s0, p2e1, p2e0;
};
// Energies of one row segment (32 of a lane's beams): longer rows add several segments' sums.
constexpr int kSegNE = 64 * 32;
// Start value of a lane's 64-bit sums over the segment k0, k0 + 64, ... < kend: minus
// kFixMagic once per contribution (modulo 2^64), so that adding the contributions' bit
// patterns leaves the sum of their integers.
__device__ __forceinline__ unsigned long long fix_base(int k0, int kend) {
  const unsigned long long n = (kend > k0) ? (unsigned long long)((kend - k0 + 63) >> 6) : 0ull;
  return 0ull - n * kFixMagic;
}
// Lane layout of a wavefront's moment totals: component c of moment m (J0, J1, J_sc, J_ss)
// sits in lane c * (64 / (NC rounded up to a power of two)) + m.
template <int NC>
__device__ __forceinline__ int fold_comp(int lane) { return lane >> (NC == 3 ? 4 : 3); }
template <int NC>
__device__ __forceinline__ int fold_moment(int lane) { return lane & (NC == 3 ? 15 : 7); }

// a over the lower, b over the upper half of the wavefront (of each 32 lanes), every lane
// adding the value of the lane 32 (16) further: two components' sums in one register pair.
__device__ __forceinline__ unsigned long long swap_add32(unsigned long long a, unsigned long long b) {
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
  return (((unsigned long long)hi[0] << 32) | lo[0]) + (((unsigned long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ unsigned long long swap_add16(unsigned long long a, unsigned long long b) {
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)a, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
  return (((unsigned long long)hi[0] << 32) | lo[0]) + (((unsigned long long)hi[1] << 32) | lo[1]);
}
// Exact sums of the lanes' NC 64-bit values over the wavefront (all lanes active): component
// fold_comp(lane) in every lane of its group.  Halving steps: each step adds pairs of lanes
// for two components at once, so NC components need about 2 NC + 8 adds instead of 6 NC, and
// no LDS trip (through LDS, with one lane per partial sum, a fold of 3 components took 1340
// cycles and one of 8 took 780-950; this one about 250).
// Every lane value is below 2^56 in magnitude (at most 32 contributions below 2^51, or a
// mixed-precision lane sum converted below 2^56), so the sums stay below 2^62.
template <int NC>
__device__ __forceinline__ long long wave_fold(const unsigned long long (&x)[NC], int lane) {
  unsigned long long t;
  if constexpr (NC == 3) {
    t = swap_add16(swap_add32(x[0], x[2]), swap_add32(x[1], 0ull));
    t += dpp_u64<kDppRor8>(t);
  } else {
    static_assert(NC == 8, "3 or 8 components");
    const unsigned long long z0 = swap_add16(swap_add32(x[0], x[4]), swap_add32(x[2], x[6]));
    const unsigned long long z1 = swap_add16(swap_add32(x[1], x[5]), swap_add32(x[3], x[7]));
    const bool up = lane & 8;
    t = (up ? z1 : z0) + dpp_u64<kDppRor8>(up ? z0 : z1);
  }
  return (long long)sum8(t);
}
// End of a row: the lanes of moment 0 add the J0 angle term (energy sum / cos), those of
// moment 1 the J1 energy sum, to their running totals; with NM = 4 (extended model) those of
// moments 2 and 3 the J_sc term (energy sum sin(theta) cos(phi) / cos: asc = (sin(theta) /
// cos) cos(phi)) and the J_ss term (ass, sin(phi)).  mine: the row's sum of the lane's
// component, v the same as a double.
template <int NC, int NM = 2>
__device__ __forceinline__ void close_row(const Scales& sc, int lane, const I128& mine, double v, double icmom,
                                          I128& T, int& err, double asc = 0.0, double ass = 0.0) {
  const int m = fold_moment<NC>(lane);
  if (m == 1) {
    T = i128_add(T, mine);
  } else if (m < NM && fold_comp<NC>(lane) < NC) {
    const double f = (m == 0) ? icmom : ((m == 2) ? asc : ass);
    T = i128_add(T, i128_from(to_fix(f * (v * sc.p2e1), sc.s0, kTwo62, err)));
  }
}

// Row geometry of a stage: cos(theta) and h / cos(theta) at the three stage radii, 1/cos at
// the radius of the stage's moments, and (extended model) sin(theta) at the three radii.
template <int KIND, bool EXT>
__device__ __forceinline__ void stage_geo(double u, double h, const Radial& g0, const Radial& gm,
                                          const Radial& g1, RowGeo& rg, double& icmom, double& sn0, double& snm,
                                          double& sn1) {
  rg = row_geo(u, h, g0, gm, g1);
  icmom = 1.0 / ((KIND == 0) ? rg.c0 : ((KIND <= 2) ? rg.cm : rg.c1));
  // sin(theta) at the three stage radii (sin(theta) r = sin(theta_R) R)
  sn0 = EXT ? sqrt(u * g0.q2) : 0.0;
  snm = EXT ? sqrt(u * gm.q2) : 0.0;
  sn1 = EXT ? sqrt(u * g1.q2) : 0.0;
}

// ----------------------------------------------------------------- two flavours
// Every two-flavour step keeps its radial profiles and scales in a per-wavefront LDS block, and
// its rows' constants in a per-wavefront LDS table, re-read where they are used, so that
// the beam loop holds only per-beam values in registers:
constexpr int kC2Rad = 0;    // q2, lam, mu at the stage radii r0, rm, r1 (9)
constexpr int kC2Sc = 9;     // fixed-point scales s1, s0, p2e1, p2e0 (4)
constexpr int kC2Size = 14;
__device__ __forceinline__ void put_stage2(double* cb, int lane, const Radial& g0, const Radial& gm,
                                           const Radial& g1, const Scales& sc) {
  if (lane == 0) {
    cb[kC2Rad + 0] = g0.q2; cb[kC2Rad + 1] = g0.lam; cb[kC2Rad + 2] = g0.mu;
    cb[kC2Rad + 3] = gm.q2; cb[kC2Rad + 4] = gm.lam; cb[kC2Rad + 5] = gm.mu;
    cb[kC2Rad + 6] = g1.q2; cb[kC2Rad + 7] = g1.lam; cb[kC2Rad + 8] = g1.mu;
    cb[kC2Sc + 0] = sc.s1; cb[kC2Sc + 1] = sc.s0; cb[kC2Sc + 2] = sc.p2e1; cb[kC2Sc + 3] = sc.p2e0;
  }
  __asm__ volatile("" ::: "memory");   // the wave's LDS operations complete in program order
}
// A row's constants rc, the same for every beam of the row:
//   rc[5 (i - 1) ...]  stage generator i = 1..4: h/cos, sg lam, and the nu-nu term (sg n_x,
//                      n_y, sg n_z), with sg = -1 for antineutrino rows (B_vac - lam e_z -
//                      nn^*), so that the generator needs no selection by species
//   rc[20]             1/cos at the moments' radius; rc[21..22] the extended model's
//                      azimuthal factors
//   rc[kRowS], rc[kRowA]  species row, sg
constexpr int kRowS = 23, kRowA = 24;
constexpr int kRowC = 26;    // doubles per block of a row group's table (25 used)
// Rows whose constants a wavefront of the bulb model keeps through a step (kRowP doubles
// each, an even number, so that pairs are read together): also cos at the three stage radii,
// 1/cos at rm and r1, and u.
constexpr int kRowCos = 25, kRowIcm = 28, kRowIc1 = 29, kRowU = 30, kRowP = 34, kRowKeep = kBatchKeep;
// Stage generator of beam (bx, bz) from its block c = [h/cos, sg lam, nu-nu term] (the
// arithmetic of gen2: subtracting a term is adding its negative).
__device__ __forceinline__ void gen2c(double bx, double bz, const double* c, double f[3]) {
  const double B0 = bx + c[2], B1 = c[3], B2 = (bz + c[1]) + c[4];
  f[0] = c[0] * B0;
  f[1] = c[0] * B1;
  f[2] = c[0] * B2;
}
__device__ __forceinline__ void put_gen2(double* c, double hc, double sg, double lam, const double* n) {
  c[0] = hc; c[1] = sg * lam; c[2] = sg * n[0]; c[3] = n[1]; c[4] = sg * n[2];
}

// All the constants of one row for a stage (a wavefront with more rows than it keeps, the
// extended model and batches: lane l of a row group computes row l's).
template <int KIND, bool EXT>
__device__ __forceinline__ void row_setup2(double u, double h, const double* cb, const double* const* J,
                                           double cp, double sp, int s, double sg, double* rc) {
  const Radial g0{cb[kC2Rad + 0], cb[kC2Rad + 1], cb[kC2Rad + 2], 0.0};
  const Radial gm{cb[kC2Rad + 3], cb[kC2Rad + 4], cb[kC2Rad + 5], 0.0};
  const Radial g1{cb[kC2Rad + 6], cb[kC2Rad + 7], cb[kC2Rad + 8], 0.0};
  RowGeo rg;
  double icmom, sn0, snm, sn1;
  stage_geo<KIND, EXT>(u, h, g0, gm, g1, rg, icmom, sn0, snm, sn1);
  double n[3];
  if (KIND == 1 || KIND == 2 || KIND == 4) {
    nunu_row<3, EXT>(J[0], g0.mu, rg.c0, sn0, cp, sp, n);
    put_gen2(rc, rg.hc0, sg, g0.lam, n);
  }
  if (KIND == 2 || KIND == 4) {
    nunu_row<3, EXT>(J[1], gm.mu, rg.cm, snm, cp, sp, n);
    put_gen2(rc + 5, rg.hcm, sg, gm.lam, n);
  }
  if (KIND >= 3) {
    nunu_row<3, EXT>(J[2], gm.mu, rg.cm, snm, cp, sp, n);
    put_gen2(rc + 10, rg.hcm, sg, gm.lam, n);
  }
  if (KIND == 4) {
    nunu_row<3, EXT>(J[3], g1.mu, rg.c1, sn1, cp, sp, n);
    put_gen2(rc + 15, rg.hc1, sg, g1.lam, n);
  }
  const double snmom = (KIND == 0) ? sn0 : ((KIND <= 2) ? snm : sn1);
  rc[20] = icmom; rc[21] = (snmom * icmom) * cp; rc[22] = (snmom * icmom) * sp;
  rc[kRowS] = (double)s;
  rc[kRowA] = sg;
}

// Kept rows (bulb model, at most kRowKeep rows per wavefront): the step's geometry, the same
// for its four stages, is computed lane-parallel (lane l: the wavefront's row l) while the
// wavefront waits at the barrier before the step, and each stage adds only the nu-nu term of
// the newest moments.  Every value is the one row_setup2 computes.  (The set-up of a stage,
// radial profiles included, was 1800-3200 cycles between the barrier and the first beam, of
// about 13000 per stage for a model of one block; it is now the nu-nu term, about 350.)
__device__ __forceinline__ void keep_geo2(const double* cb, double h, int lane, int nrw, double* rt) {
  if (lane < nrw) {
    double* rc = rt + lane * kRowP;
    const Radial g0{cb[kC2Rad + 0], 0.0, 0.0, 0.0}, gm{cb[kC2Rad + 3], 0.0, 0.0, 0.0}, g1{cb[kC2Rad + 6], 0.0, 0.0, 0.0};
    const RowGeo rg = row_geo(rc[kRowU], h, g0, gm, g1);
    const double sg = rc[kRowA];
    rc[0] = rg.hc0; rc[1] = sg * cb[kC2Rad + 1];
    rc[5] = rg.hcm; rc[6] = sg * cb[kC2Rad + 4];
    rc[10] = rg.hcm; rc[11] = sg * cb[kC2Rad + 4];
    rc[15] = rg.hc1; rc[16] = sg * cb[kC2Rad + 7];
    rc[kRowCos] = rg.c0; rc[kRowCos + 1] = rg.cm; rc[kRowCos + 2] = rg.c1;
    rc[kRowIcm] = 1.0 / rg.cm;
    rc[kRowIc1] = 1.0 / rg.c1;
  }
  __asm__ volatile("" ::: "memory");
}
template <int KIND>
__device__ __forceinline__ void keep_nunu2(const double* cb, const double (*sJ)[6], int lane, int nrw, double* rt) {
  if (lane < nrw) {
    double* rc = rt + lane * kRowP;
    if (KIND == 0) {
      rc[20] = 1.0 / rc[kRowCos];
    } else {
      constexpr int at = (KIND == 1) ? 0 : ((KIND == 4) ? 2 : 1);   // the newest moments' radius
      const double* J = sJ[KIND == 0 ? 0 : KIND - 1];
      double n[3];
      nunu<3>(J, cb[kC2Rad + 3 * at + 2], rc[kRowCos + at], n);
      double* c = rc + 5 * (KIND == 0 ? 0 : KIND - 1);
      const double sg = rc[kRowA];
      c[2] = sg * n[0]; c[3] = n[1]; c[4] = sg * n[2];
      if (KIND == 1) rc[20] = rc[kRowIcm];
      if (KIND == 3) rc[20] = rc[kRowIc1];
    }
  }
  __asm__ volatile("" ::: "memory");
}

// Stage stencil for one row of NE beams starting at beam rb, with its constants at rc.
// KIND: 0 moments of rho_n at r_n; 1 stage Y2 (moments at r_n + h/2); 2 stage Y3
// (r_n + h/2); 3 stage Y4 (r_{n+1}); 4 final update, store and moments at r_{n+1}.
// A lane adds the fixed-point contributions of up to 32 of its beams in 64-bit integers
// (each below 2^51) before they are folded into exact 128-bit wave sums; a beam whose state
// has squared norm 2 or more (NaN included) sets err.
// ADAPT (final update only): the new state goes to Xo instead of X, and emax keeps the
// largest embedded error estimate |Theta - f2|^2 of the lane's beams.
// EXT: extended bulb model.  pre: the lane's first beam, if it was loaded before.
// TAB: sin/cos constants from sct, the block's table in LDS (sincos_coefs).
template <int KIND, bool TAB, bool ADAPT = false, bool EXT = false>
__device__ __forceinline__ void row2(const double* X, double* Xo, long long plane, long long rb, int NE,
                                     const double* tab, const double* cb, const double* rc, int renorm, int lane,
                                     I128& T, int& err, double& emax, const double* sct,
                                     const double* pre = nullptr) {
  constexpr int NM = EXT ? 4 : 2;
  double q0 = 0.0, q1 = 0.0, q2 = 0.0;
  if (pre) {
    q0 = pre[0]; q1 = pre[1]; q2 = pre[2];
  } else if (lane < NE) {
    q0 = X[rb + lane]; q1 = X[rb + lane + plane]; q2 = X[rb + lane + 2 * plane];
  }
  const double* G = tab + (size_t)(2 + (int)rc[kRowS]) * NE;
  const double sg = rc[kRowA];
  I128 mine = i128_zero();
  for (int k0 = lane; k0 - lane < NE; k0 += 64 * 32) {
    const int kend = min(NE, k0 + 64 * 32);
    const unsigned long long base = fix_base(k0, kend);
    unsigned long long acc[3] = {base, base, base};
    if (k0 != lane && k0 < kend) {   // a later segment's first beam
      q0 = X[rb + k0]; q1 = X[rb + k0 + plane]; q2 = X[rb + k0 + 2 * plane];
    }
    for (int k = k0; k < kend; k += 64) {
      double P0 = q0, P1 = q1, P2 = q2;
      if (k + 64 < kend) {    // prefetch the lane's next beam
        q0 = X[rb + k + 64]; q1 = X[rb + k + 64 + plane]; q2 = X[rb + k + 64 + 2 * plane];
      }
      __asm__ volatile("" ::: "memory");   // the row constants are re-read from LDS per beam
      if (KIND >= 1) {
        const double bx = tab[k], bz = tab[NE + k];
        double f1[3], f2[3], f3[3], f4[3];
        if (KIND != 3) gen2c(bx, bz, rc + 0, f1);
        if (KIND == 1) {
          rotate2<TAB>(0.5 * f1[0], 0.5 * f1[1], 0.5 * f1[2], P0, P1, P2, sct);
        } else if (KIND == 2) {
          gen2c(bx, bz, rc + 5, f2);
          const double cr0 = f1[1] * f2[2] - f1[2] * f2[1];
          const double cr1 = f1[2] * f2[0] - f1[0] * f2[2];
          const double cr2 = f1[0] * f2[1] - f1[1] * f2[0];
          rotate2<TAB>(0.5 * f2[0] - 0.125 * cr0, 0.5 * f2[1] - 0.125 * cr1, 0.5 * f2[2] - 0.125 * cr2,
                  P0, P1, P2, sct);
        } else if (KIND == 3) {
          gen2c(bx, bz, rc + 10, f3);
          rotate2<TAB>(f3[0], f3[1], f3[2], P0, P1, P2, sct);
        } else {
          gen2c(bx, bz, rc + 5, f2);
          gen2c(bx, bz, rc + 10, f3);
          gen2c(bx, bz, rc + 15, f4);
          const double cr0 = f1[1] * f4[2] - f1[2] * f4[1];
          const double cr1 = f1[2] * f4[0] - f1[0] * f4[2];
          const double cr2 = f1[0] * f4[1] - f1[1] * f4[0];
          const double t0 = (((f1[0] + 2.0 * f2[0]) + 2.0 * f3[0]) + f4[0]) * (1.0 / 6.0) - cr0 * (1.0 / 12.0);
          const double t1 = (((f1[1] + 2.0 * f2[1]) + 2.0 * f3[1]) + f4[1]) * (1.0 / 6.0) - cr1 * (1.0 / 12.0);
          const double t2 = (((f1[2] + 2.0 * f2[2]) + 2.0 * f3[2]) + f4[2]) * (1.0 / 6.0) - cr2 * (1.0 / 12.0);
          if (ADAPT) {
            const double d0 = t0 - f2[0], d1 = t1 - f2[1], d2 = t2 - f2[2];
            const double e = (d0 * d0 + d1 * d1) + d2 * d2;
            emax = (e > emax) ? e : emax;
          }
          rotate2<TAB>(t0, t1, t2, P0, P1, P2, sct);
          if (renorm) {
            const double nrm2 = (P0 * P0 + P1 * P1) + P2 * P2;
            if (!(fabs(nrm2 - 1.0) <= kRenormTol)) err |= 8;
            const double inv = fma(-0.5, nrm2, 1.5);   // one Newton step for 1/sqrt from 1
            P0 = P0 * inv;
            P1 = P1 * inv;
            P2 = P2 * inv;
          }
          Xo[rb + k] = P0;
          Xo[rb + k + plane] = P1;
          Xo[rb + k + 2 * plane] = P2;
        }
      }
      // rho~: rho for neutrinos, -rho^* (Bloch (-x, y, -z)) for antineutrinos
      if (!(fma(P0, P0, fma(P1, P1, P2 * P2)) < 2.0)) err |= 1;
      const double ws = G[k] * cb[kC2Sc + 0];
      const double wa = sg * ws;
      acc[0] += fix_bits(P0, wa);
      acc[1] += fix_bits(P1, ws);
      acc[2] += fix_bits(P2, wa);
    }
    mine = i128_add(mine, i128_from(wave_fold<3>(acc, lane)));
  }
  __asm__ volatile("" ::: "memory");
  const double v = (NE <= kSegNE) ? (double)(long long)mine.lo : i128_to_double(mine);
  close_row<3, NM>(Scales{cb[kC2Sc + 0], cb[kC2Sc + 1], cb[kC2Sc + 2], cb[kC2Sc + 3]}, lane, mine, v, rc[20], T,
                   err, rc[21], rc[22]);
}

// A group of gn rows of one model whose beams are contiguous from beam gb0 (NE energies a
// row), streamed as full 64-lane chunks: lane l of chunk c takes the group's beam
// f = 64 c + l, row i = f / NE, energy k = f - i NE, and reads its row's constants from the
// group table rt (row i's block).  The
// last chunk of one row and the first of the next share a wavefront instead of leaving
// lanes idle.  A row's exact sum is folded in the chunk where the row ends (its lanes fold,
// the others go on with the next row), so every row adds the same integer sum as in row2
// and the moments keep their bits.  A lane adds at most ceil(NE / 64) + 1 contributions
// to a row, so with NE <= kGroupMaxNE its 64-bit sums stay below 2^56 as wave_fold needs.
constexpr int kGroupMaxNE = 64 * 31;
// Rows folded together by group2.  The extended model's rows (100 energies) end in most
// chunks, so its wavefront stages ended rows in LDS and folds and closes four at a time (20M
// beams, 31 energies: 351 us per step against 366 with one row at a time; 100 energies: 771
// against 782).  The batch kernel folds each row as it ends (wave_fold): its rows are longer
// (50-400 energies) and at 128 VGPRs staged totals spill (two rows at a time: 2.88 -> 4.63 ms).
constexpr int kFoldRowsExt = 4, kFoldRowsBatch = 1;
// A wavefront's fold scratch for group2 with R > 1 rows per fold: 3 R staged components, each
// in a run of fold2_stride(R) words, then the 3 R G partial sums (G = 64 / 3 R per
// component).  A run is 64 + G words and lane g of component c adds words g, g + G, ...: the
// padding puts component c's run G banks after component c - 1's, so these reads meet no
// bank conflicts (the extended model's 12 components would otherwise read one bank 12-fold;
// 60M beams 2.43 -> 2.35 ms per step).
__host__ __device__ constexpr int fold2_stride(int R) { return 64 + 64 / (3 * R); }
__host__ __device__ constexpr int fold2_words(int R) { return 3 * R * fold2_stride(R) + 64; }

// Fold of up to R rows whose lane sums were staged as they ended: component c of slot q in
// fl[(q * 3 + c) * S + lane], q < nrows, S = fold2_stride(R).  G partial sums per component,
// each over every G-th word, then lane v adds the G partial sums of its component.  Lane
// m * 3 R + q * 3 + c then closes moment m, component c of the row in slot q (its row
// constants at rr0 + q * kRowC) exactly as close_row does, into Tq.  One set of
// instructions folds and closes R rows, instead of one per row.
template <int R, int NM>
__device__ __forceinline__ void fold_rows2(int lane, long long* fl, int nrows, const double* rr0,
                                           const Scales& sc, I128& Tq, int& err) {
  constexpr int NCR = 3 * R, G = 64 / NCR, L = (64 + G - 1) / G, S = fold2_stride(R);
  long long* gs = fl + NCR * S;
  __asm__ volatile("" ::: "memory");   // the wave's LDS operations complete in program order
  // lane (cc, g): partial sum g of component cc, stored at gs[cc * G + g]
  const int cc = lane / G, g = lane - cc * G;
  if (cc < NCR) {
    long long part = 0;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const int src = i * G + g;
      if (src < 64) part += fl[cc * S + src];
    }
    gs[cc * G + g] = part;
  }
  __asm__ volatile("" ::: "memory");
  if (lane < NM * NCR) {
    const int m = lane / NCR, qc = lane - m * NCR, q = qc / 3;
    if (q < nrows) {
      long long t = 0;
#pragma unroll
      for (int gg = 0; gg < G; ++gg) t += gs[qc * G + gg];
      const double* rr = rr0 + q * kRowC;
      if (m == 1) {
        Tq = i128_add(Tq, i128_from(t));
      } else {
        const double f = (m == 0) ? rr[20] : ((m == 2) ? rr[21] : rr[22]);
        Tq = i128_add(Tq, i128_from(to_fix(f * (i128_to_double(i128_from(t)) * sc.p2e1), sc.s0, kTwo62, err)));
      }
    }
  }
  __asm__ volatile("" ::: "memory");
}

// RS: doubles per block of the table rt.
template <int KIND, bool EXT, int R, int RS>
__device__ __forceinline__ void group2(double* X, long long plane, long long gb0, int NE, int gn,
                                       const double* tab, const double* cb, const double* rt, int renorm,
                                       int lane, long long* fl, I128& T, int& err) {
  constexpr int NM = EXT ? 4 : 2;
  constexpr int NCR = 3 * R, S = fold2_stride(R);   // R > 1
  const Scales sc{cb[kC2Sc + 0], cb[kC2Sc + 1], cb[kC2Sc + 2], cb[kC2Sc + 3]};
  const int nbeam = gn * NE;
  const int nchunk = (nbeam + 63) >> 6;
  int i = lane / NE;                 // the lane's row and energy in the current chunk
  int k = lane - i * NE;
  const int irow = 64 / NE, krow = 64 - irow * NE;   // a chunk further: irow rows, krow energies
  // a plane's base is uniform and the group's byte offsets fit 32 bits (at most kGroup rows of
  // kGroupMaxNE energies): one offset register serves all planes, and the next beam is found
  // without a loop over lanes (passes of 4 steps with the state set and read back, with the
  // sin/cos constants from scalar registers in both: 256-model batch 11.7 -> 11.0 ms, extended
  // 20M beams 3.43 -> 3.37 ms, against 64-bit addresses and a loop that stepped k row by row)
  char *X0 = reinterpret_cast<char*>(X + gb0), *X1 = reinterpret_cast<char*>(X + gb0 + plane),
       *X2 = reinterpret_cast<char*>(X + gb0 + 2 * plane);
  const auto at = [](char* base, unsigned off) -> double& { return *reinterpret_cast<double*>(base + off); };
  // (PF: two species, so row 2 or 3 of the tables)
  const auto load_tab = [&](int row, int e, double& x, double& z, double& w) {
    const unsigned off = 8u * (unsigned)e;
    const unsigned woff = off + (rt[row * RS + kRowS] != 0.0 ? 8u * (unsigned)NE : 0u);
    char* t = reinterpret_cast<char*>(const_cast<double*>(tab));
    x = at(t, off);
    z = at(t + 8 * (size_t)NE, off);
    w = at(t + 16 * (size_t)NE, woff);
  };
  double q0 = 0.0, q1 = 0.0, q2 = 0.0;
  // PF (batches): the energy tables of a batch's models stay in HBM, so the lane's table
  // values (vacuum terms and weight) for its beam in the next chunk are loaded with that
  // beam's state, instead of at their use (256-model batch 2.90 -> 2.53 ms per step).  The
  // extended model reads its tables from LDS.
  constexpr bool PF = !EXT;
  double tx = 0.0, tz = 0.0, tw = 0.0;
  if (lane < nbeam) {
    const unsigned off = 8u * (unsigned)lane;
    q0 = at(X0, off); q1 = at(X1, off); q2 = at(X2, off);
    if (PF) load_tab(i, k, tx, tz, tw);
  }
  unsigned long long acc[3] = {0ull, 0ull, 0ull};
  unsigned long long cnt = 0;        // contributions in acc (each carries kFixMagic)
  int r = 0;                         // the oldest unfinished row (wave-uniform)
  int ns = 0;                        // ended rows staged for the next fold (wave-uniform)
  I128 Tq = i128_zero();             // closed rows, lane m * 3 R + q * 3 + c (fold_rows2)
  for (int c = 0; c < nchunk; ++c) {
    const int f = (c << 6) + lane;
    const bool on = f < nbeam;
    double P0 = q0, P1 = q1, P2 = q2;
    const double bxc = tx, bzc = tz, wsc = tw;
    const unsigned off = 8u * (unsigned)f;
    int kn = k + krow, in = i + irow;   // the lane's beam in the next chunk
    if (kn >= NE) {
      kn -= NE;
      ++in;
    }
    if (f + 64 < nbeam) {    // prefetch it
      q0 = at(X0 + 512, off); q1 = at(X1 + 512, off); q2 = at(X2 + 512, off);
      if (PF) load_tab(in, kn, tx, tz, tw);
    }
    __asm__ volatile("" ::: "memory");   // the row constants are re-read from LDS per beam
    unsigned long long x0 = 0ull, x1 = 0ull, x2 = 0ull;
    if (on) {
      const double* rc = rt + i * RS;
      const int sr = (int)rc[kRowS];
      if (KIND >= 1) {
        const double bx = PF ? bxc : tab[k], bz = PF ? bzc : tab[NE + k];
        double f1[3], f2[3], f3[3], f4[3];
        if (KIND != 3) gen2c(bx, bz, rc + 0, f1);
        if (KIND == 1) {
          rotate2(0.5 * f1[0], 0.5 * f1[1], 0.5 * f1[2], P0, P1, P2);
        } else if (KIND == 2) {
          gen2c(bx, bz, rc + 5, f2);
          const double cr0 = f1[1] * f2[2] - f1[2] * f2[1];
          const double cr1 = f1[2] * f2[0] - f1[0] * f2[2];
          const double cr2 = f1[0] * f2[1] - f1[1] * f2[0];
          rotate2(0.5 * f2[0] - 0.125 * cr0, 0.5 * f2[1] - 0.125 * cr1, 0.5 * f2[2] - 0.125 * cr2,
                        P0, P1, P2);
        } else if (KIND == 3) {
          gen2c(bx, bz, rc + 10, f3);
          rotate2(f3[0], f3[1], f3[2], P0, P1, P2);
        } else {
          gen2c(bx, bz, rc + 5, f2);
          gen2c(bx, bz, rc + 10, f3);
          gen2c(bx, bz, rc + 15, f4);
          const double cr0 = f1[1] * f4[2] - f1[2] * f4[1];
          const double cr1 = f1[2] * f4[0] - f1[0] * f4[2];
          const double cr2 = f1[0] * f4[1] - f1[1] * f4[0];
          const double t0 = (((f1[0] + 2.0 * f2[0]) + 2.0 * f3[0]) + f4[0]) * (1.0 / 6.0) - cr0 * (1.0 / 12.0);
          const double t1 = (((f1[1] + 2.0 * f2[1]) + 2.0 * f3[1]) + f4[1]) * (1.0 / 6.0) - cr1 * (1.0 / 12.0);
          const double t2 = (((f1[2] + 2.0 * f2[2]) + 2.0 * f3[2]) + f4[2]) * (1.0 / 6.0) - cr2 * (1.0 / 12.0);
          rotate2(t0, t1, t2, P0, P1, P2);
          if (renorm) {
            const double nrm2 = (P0 * P0 + P1 * P1) + P2 * P2;
            if (!(fabs(nrm2 - 1.0) <= kRenormTol)) err |= 8;
            const double inv = fma(-0.5, nrm2, 1.5);   // one Newton step for 1/sqrt from 1
            P0 = P0 * inv;
            P1 = P1 * inv;
            P2 = P2 * inv;
          }
          at(X0, off) = P0;
          at(X1, off) = P1;
          at(X2, off) = P2;
        }
      }
      // rho~: rho for neutrinos, -rho^* (Bloch (-x, y, -z)) for antineutrinos
      if (!(fma(P0, P0, fma(P1, P1, P2 * P2)) < 2.0)) err |= 1;
      const double ws = (PF ? wsc : tab[(size_t)(2 + sr) * NE + k]) * cb[kC2Sc + 0];
      const double wa = rc[kRowA] * ws;
      x0 = fix_bits(P0, wa);
      x1 = fix_bits(P1, ws);
      x2 = fix_bits(P2, wa);
    }
    // stage every row that ends in this chunk (its lanes add their contribution first);
    // fold R staged rows at a time
    const int fend = min(nbeam, (c + 1) << 6);
    while (r < gn && (r + 1) * NE <= fend) {
      if (on && i == r) {
        acc[0] += x0; acc[1] += x1; acc[2] += x2;
        ++cnt;
      }
      const unsigned long long bias = cnt * kFixMagic;
      const unsigned long long ended[3] = {acc[0] - bias, acc[1] - bias, acc[2] - bias};
      acc[0] = acc[1] = acc[2] = 0ull;
      cnt = 0;
      if constexpr (R == 1) {
        const long long t = wave_fold<3>(ended, lane);
        const double* rr = rt + r * RS;
        close_row<3, NM>(sc, lane, i128_from(t), (double)t, rr[20], T, err, rr[21], rr[22]);
        ++r;
      } else {
        long long* slot = fl + ns * 3 * S + lane;
        slot[0] = (long long)ended[0];
        slot[S] = (long long)ended[1];
        slot[2 * S] = (long long)ended[2];
        ++r;
        if (++ns == R) {
          fold_rows2<R, NM>(lane, fl, R, rt + (r - R) * kRowC, sc, Tq, err);
          ns = 0;
        }
      }
    }
    if (on && i == r) {      // the row that goes on into the next chunk
      acc[0] += x0; acc[1] += x1; acc[2] += x2;
      ++cnt;
    }
    k = kn;
    i = in;
  }
  if constexpr (R == 1) return;
  if (ns) fold_rows2<R, NM>(lane, fl, ns, rt + (r - ns) * kRowC, sc, Tq, err);
  // the closed rows' totals (lane m * 3 R + q * 3 + c) into T (lane m * 3 + c): integer sums
  __asm__ volatile("" ::: "memory");
  if (lane < NM * NCR) {
    fl[2 * lane] = (long long)Tq.lo;
    fl[2 * lane + 1] = Tq.hi;
  }
  __asm__ volatile("" ::: "memory");
  const int m = fold_moment<3>(lane);
  if (m < NM && fold_comp<3>(lane) < 3) {
    const int c = fold_comp<3>(lane);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int src = m * NCR + q * 3 + c;
      T = i128_add(T, I128{(unsigned long long)fl[2 * src], fl[2 * src + 1]});
    }
  }
  __asm__ volatile("" ::: "memory");
}

// rt: the wavefront's row-constant table, kGroup2 blocks of kRowC doubles (extended model) or
// kRowKeep of kRowP (bulb model, which keeps up to kRowKeep rows through a step; 17 KB of a
// block of 256 threads, so that of energy tables of 1064-1215 energies two blocks fit a CU
// where three would without it: the kept rows gain more, 1120 x 2000 bins 161 -> 135 us per step).
constexpr int kGroup2 = 16;
constexpr int row_table2(bool ext) { return ext ? kGroup2 * kRowC : kRowKeep * kRowP; }
// Rows gw, gw + nw, ... of nrow.
__device__ __forceinline__ int wave_rows(long long gw, long long nw, long long nrow) {
  return gw < nrow ? (int)((nrow - 1 - gw) / nw + 1) : 0;
}
// Once per launch: the labels of the bulb model's kept rows.
__device__ __forceinline__ void keep_rows2(const StepArgs& a, long long gw, long long nw, int lane, int nrw, double* rt) {
  if (nrw <= kRowKeep && lane < nrw) {
    const long long row = gw + lane * nw;
    const int s = (int)(row / a.NU);
    rt[lane * kRowP + kRowU] = u_of((int)(row - (long long)s * a.NU), a.NU);
    rt[lane * kRowP + kRowS] = (double)s;
    rt[lane * kRowP + kRowA] = (s >= (a.NS >> 1)) ? -1.0 : 1.0;
  }
  __asm__ volatile("" ::: "memory");
}
// Before every step: its radial profiles, and the kept rows' geometry.
template <bool EXT>
__device__ __forceinline__ void prep2(const StepArgs& a, const StepGeo& G, int lane, int nrw, double* cb, double* rt) {
  __asm__ volatile("" ::: "memory");
  put_stage2(cb, lane, radial_at(a, G.r0), radial_at(a, G.rm), radial_at(a, G.r1),
             Scales{a.s1, a.s0, a.p2e1, a.p2e0});
  if (!EXT && nrw <= kRowKeep) keep_geo2(cb, G.h, lane, nrw, rt);
}
// Every other stage of the extended model takes a wavefront's row groups in reverse order, so that
// it begins with the beams the stage before it touched last: of a state beyond the 256 MB
// last-level cache the part that is still there is read from it, where a sweep in the same
// direction each time finds none (passes of 4 steps with the state set and read back: 20M beams,
// 480 MB, 3.46 -> 3.37 ms; the 256-model batch, 1.5 GB, gains nothing, 11.14 against 11.18 ms, so
// its sweeps keep one direction).  The moments are integer sums, so the order does not change
// their bits.
__device__ constexpr bool backwards(int kind) { return (kind & 1) == 0; }

template <int KIND, bool ADAPT = false, bool EXT = false>
__device__ __forceinline__ void stage2(const StepArgs& a, double h, const double* X, double* Xo,
                                       const double (*sJ)[EXT ? 12 : 6], const double* tab, long long gw,
                                       long long nw, int nrw, int lane, long long* fl, I128& T, int& err,
                                       double& emax, const double* cb, const double* sct, double* rt,
                                       const double* pre = nullptr) {
  const double* J[4] = {sJ[0], sJ[1], sJ[2], sJ[3]};
  // (the launch arguments are read into locals first: the LDS-order barriers below would
  // otherwise make the compiler re-read them from a private copy of the argument block)
  const int NE = a.NE, NU = a.NU, NS = a.NS, renorm = a.renorm;
  const long long plane = a.plane;
  if constexpr (EXT) {
    // rows (s, j, p): species, emission bin, azimuthal bin.  Each wavefront takes a
    // contiguous range of rows, in groups of up to kGroup2: lane l computes the constants of
    // the group's row l (row_setup2: geometry, nu-nu terms with the row's azimuth) into the
    // table rt, then the rows run one after the other.
    const int NP = a.NP;
    const double* phi = a.tab + (size_t)(2 + NS) * NE;
    const long long nrow = (long long)NS * NU * NP;
    const long long per = (nrow + nw - 1) / nw;
    const long long rbeg = gw * per, rend = min(nrow, rbeg + per);
    const int ng = rend > rbeg ? (int)((rend - rbeg + kGroup2 - 1) / kGroup2) : 0;
    for (int g = 0; g < ng; ++g) {
      long long row = rbeg + (long long)(backwards(KIND) ? ng - 1 - g : g) * kGroup2;
      const int gn = (int)min(rend - row, (long long)kGroup2);
      __asm__ volatile("" ::: "memory");   // the previous group's rows have read their blocks
      if (lane < gn) {
        const long long r = row + lane;
        const long long sj = r / NP;
        const int p = (int)(r - sj * NP);
        const int s = (int)(sj / NU);
        const int j = (int)(sj - (long long)s * NU);
        row_setup2<KIND, true>(u_of(j, NU), h, cb, J, phi[p], phi[NP + p], s, (s >= (NS >> 1)) ? -1.0 : 1.0,
                               rt + lane * kRowC);
      }
      __asm__ volatile("" ::: "memory");
      if (!ADAPT && NE <= kGroupMaxNE) {
        group2<KIND, true, kFoldRowsExt, kRowC>(Xo, plane, row * NE, NE, gn, tab, cb, rt, renorm, lane, fl, T, err);
      } else {
        for (int i = 0; i < gn; ++i, ++row)
          row2<KIND, false, ADAPT, true>(X, Xo, plane, row * NE, NE, tab, cb, rt + i * kRowC, renorm, lane, T, err, emax,
                                         nullptr);
      }
    }
  } else if (nrw <= kRowKeep) {
    keep_nunu2<KIND>(cb, sJ, lane, nrw, rt);
    for (int i = 0; i < nrw; ++i)
      row2<KIND, true, ADAPT>(X, Xo, plane, (gw + i * nw) * NE, NE, tab, cb, rt + i * kRowP, renorm, lane, T, err, emax,
                        sct, i == 0 ? pre : nullptr);
  } else {
    for (int r0 = 0; r0 < nrw; r0 += kRowKeep) {
      const int gn = min(nrw - r0, kRowKeep);
      __asm__ volatile("" ::: "memory");   // the previous group's rows have read their blocks
      if (lane < gn) {
        const long long row = gw + (r0 + lane) * nw;
        const int s = (int)(row / NU);
        row_setup2<KIND, false>(u_of((int)(row - (long long)s * NU), NU), h, cb, J, 0.0, 0.0, s,
                                (s >= (NS >> 1)) ? -1.0 : 1.0, rt + lane * kRowP);
      }
      __asm__ volatile("" ::: "memory");
      for (int i = 0; i < gn; ++i)
        row2<KIND, true, ADAPT>(X, Xo, plane, (gw + (r0 + i) * nw) * NE, NE, tab, cb, rt + i * kRowP, renorm, lane, T, err,
                          emax, sct, r0 + i == 0 ? pre : nullptr);
    }
  }
}

// --------------------------------------------------------------- three flavours
// Stage generators by linearity.  Stage i's generator of a beam of energy bin k is
// K_i = a_i (V_k + M_i): a_i = h / cos(theta) at the stage radius, V_k = e_k V0 the vacuum
// Hamiltonian of the bin (e_k = 1 / E_k), M_i the matter and nu-nu part, the same for
// every energy of a (species, angle) row.  Every generator the step exponentiates is
// affine in V_k; with i[K_1, K_i] = a_1 a_i (e_k i[V0, D] + i[M_1, D]), D = M_i - M_1, each
// is G = alpha V_k + e_k P + Q with alpha, P, Q fixed per row:
//   K1/2               alpha = a1/2, P = 0, Q = (a1/2) M1
//   K3                 alpha = am,   P = 0, Q = am M3
//   K2/2 + i[K1,K2]/8  alpha = am/2, P = c i[V0, D], Q = (am/2) M2 + c i[M1, D], c = a1 am/8
//   Theta              alpha = (a1 + 2 am + 2 am + a4)/6, P = c i[V0, D],
//                      Q = S/6 + c i[M1, D], c = a1 a4/12, S = a1 M1 + 2 am M2 + 2 am M3 + a4 M4
// and the error estimate Theta - K2 = (alpha - am) V_k + e_k P + (Q - am M2).  Per beam that
// is 6 (no P) or 15 fma.  Hermitian matrices as 9 reals: d0 d1 d2, re/im of (0,1), (0,2),
// (1,2).
// alpha V_k + Q
__device__ __forceinline__ Herm3 lin3q(double alpha, const double* Q, const double* v) {
  return Herm3{fma(alpha, v[0], Q[0]), fma(alpha, v[1], Q[1]), fma(alpha, v[2], Q[2]),
               mk(fma(alpha, v[3], Q[3]), Q[4]), mk(fma(alpha, v[4], Q[5]), Q[6]),
               mk(fma(alpha, v[5], Q[7]), Q[8])};
}
// alpha V_k + e_k P + Q
__device__ __forceinline__ Herm3 lin3p(double alpha, const double* P, const double* Q, const double* v,
                                       double ek) {
  return Herm3{fma(alpha, v[0], fma(ek, P[0], Q[0])), fma(alpha, v[1], fma(ek, P[1], Q[1])),
               fma(alpha, v[2], fma(ek, P[2], Q[2])),
               mk(fma(alpha, v[3], fma(ek, P[3], Q[3])), fma(ek, P[4], Q[4])),
               mk(fma(alpha, v[4], fma(ek, P[5], Q[5])), fma(ek, P[6], Q[6])),
               mk(fma(alpha, v[5], fma(ek, P[7], Q[7])), fma(ek, P[8], Q[8]))};
}

// A three-flavour wavefront's LDS block (doubles): row constants Q, P and the error estimate's
// Q (27), for packed tails alpha and the species row; FP32 copies of Q and P (18 floats); M1
// and D as full complex matrices (18 each, the diagonal's imaginary parts zero for the whole
// launch); the step's q2, lam, mu at the three stage radii.
constexpr int kL3Alpha = 28, kL3S = 29, kL3F32 = 32, kL3FM = 42, kL3FD = 60, kL3Rad = 78, kL3Size = 88;
// Kept rows: constants of up to kKeep3 rows that hold for a whole step, kRow3 doubles each:
// cos(theta) and h / cos(theta) at the three stage radii, 1/cos at rm and r1, sin(theta) at the
// three radii (extended model); then the row's labels: u, species row, sg, cos and sin of
// its azimuth.
constexpr int kKeep3 = 8, kRow3 = 17;
constexpr int kR3C = 0, kR3H = 3, kR3Icm = 6, kR3Ic1 = 7, kR3Sn = 8, kR3U = 11, kR3S = 12, kR3Sg = 13, kR3Cp = 14,
              kR3Sp = 15;
// Labels of rows row0, row0 + nw, ... (gn <= kKeep3 of them, lane l row l).
template <bool EXT>
__device__ __forceinline__ void keep_labels3(const StepArgs& a, long long row0, long long nw, int gn, int lane, double* kr) {
  if (lane < gn) {
    const long long row = row0 + lane * nw;
    const long long sj = EXT ? row / a.NP : row;
    const int s = (int)(sj / a.NU);
    double* g = kr + lane * kRow3;
    g[kR3U] = u_of((int)(sj - (long long)s * a.NU), a.NU);
    g[kR3S] = (double)s;
    g[kR3Sg] = (s >= (a.NS >> 1)) ? -1.0 : 1.0;
    if (EXT) {
      const double* phi = a.tab + (size_t)(kVacRows3 + a.NS) * a.NE;
      const int p = (int)(row - sj * a.NP);
      g[kR3Cp] = phi[p];
      g[kR3Sp] = phi[a.NP + p];
    }
  }
  __asm__ volatile("" ::: "memory");   // the wave's LDS operations complete in program order
}
template <bool EXT>
__device__ __forceinline__ void keep_geo3(const double* rad, double h, int gn, int lane, double* kr) {
  if (lane < gn) {
    double* g = kr + lane * kRow3;
    const Radial g0{rad[0], 0.0, 0.0, 0.0}, gm{rad[3], 0.0, 0.0, 0.0}, g1{rad[6], 0.0, 0.0, 0.0};
    const double u = g[kR3U];
    const RowGeo rg = row_geo(u, h, g0, gm, g1);
    g[kR3C] = rg.c0; g[kR3C + 1] = rg.cm; g[kR3C + 2] = rg.c1;
    g[kR3H] = rg.hc0; g[kR3H + 1] = rg.hcm; g[kR3H + 2] = rg.hc1;
    g[kR3Icm] = 1.0 / rg.cm;
    g[kR3Ic1] = 1.0 / rg.c1;
    if (EXT) {   // sin(theta) r = sin(theta_R) R
      g[kR3Sn] = sqrt(u * rad[0]); g[kR3Sn + 1] = sqrt(u * rad[3]); g[kR3Sn + 2] = sqrt(u * rad[6]);
    }
  }
  __asm__ volatile("" ::: "memory");
}
// Before every step: its radial profiles and, if the wavefront's nrw rows are all kept, their
// geometry (run behind the barrier before the step).
template <bool EXT>
__device__ __forceinline__ void prep3(const StepArgs& a, const StepGeo& G, int lane, int nrw, double* snn, double* kr) {
  __asm__ volatile("" ::: "memory");
  const Radial r[3] = {radial_at(a, G.r0), radial_at(a, G.rm), radial_at(a, G.r1)};
  double* rad = snn + kL3Rad;
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      rad[3 * q] = r[q].q2; rad[3 * q + 1] = r[q].lam; rad[3 * q + 2] = r[q].mu;
    }
  __asm__ volatile("" ::: "memory");
  if (nrw <= kKeep3) keep_geo3<EXT>(rad, G.h, nrw, lane, kr);
}
// The matrix V0 (vacuum Hamiltonian times E) in full, for the block, and the zero imaginary
// parts of the wavefront's matrices (then a block barrier).
__device__ __forceinline__ void put_full(double* F, int a, int b, bool im, double v) {
  F[(a * 3 + b) * 2 + (im ? 1 : 0)] = v;
  F[(b * 3 + a) * 2 + (im ? 1 : 0)] = im ? -v : v;
}
__device__ __forceinline__ void init3(const StepArgs& a, int lane, double* fv, double* snn) {
  if (threadIdx.x < 6) {
    const int q = (int)threadIdx.x - 3;
    const int ra = (q < 0) ? (int)threadIdx.x : (q == 2 ? 1 : 0), rb = (q < 0) ? (int)threadIdx.x : (q == 0 ? 1 : 2);
    put_full(fv, ra, rb, true, 0.0);
    put_full(fv, ra, rb, false, a.v0[threadIdx.x]);
  }
  if (lane < 3) {
    snn[kL3FM + (lane * 3 + lane) * 2 + 1] = 0.0;
    snn[kL3FD + (lane * 3 + lane) * 2 + 1] = 0.0;
  }
}

// Row constants of stage KIND's generator (KIND >= 1): Q to snn[0..8], P to snn[9..17]
// and, with ADAPT (KIND 4), the error estimate's Q to snn[18..26]; returns alpha (and the
// error estimate's alpha in alphaE).  J0..J3: the stage moments; g: the row's kept constants;
// fv: V0 in full.  Lanes i < 9 of each half of the wavefront compute component i of every
// 9-real matrix (the same operations as a matrix-at-a-time evaluation, component by
// component), the lower half's the commutator with V0 (P), the upper half's the one with M1
// (Q); the commutators read their operands as full complex 3x3 matrices from LDS, where
// each lane writes its component and its mirror.  No lane branches: written with a branch per
// kind of component and both commutators in the same lanes, the stages with commutators took
// 2800-3400 cycles here.
// Component i of the 9-real form: 0..2 the diagonal, 3 + 2t / 4 + 2t re / im of entry t of
// (0,1), (0,2), (1,2).  nn component of M's component i (the matter part sits on i = 0):
__device__ __forceinline__ int nn_index(int i) { return (i <= 1) ? i : i - 1; }
// nu-nu component j of a row (as nunu_row)
template <int NC, bool EXT>
__device__ __forceinline__ double nunu_comp(const double* J, double mu, double c, double sn, double cp,
                                            double sp, int j) {
  if constexpr (EXT) return mu * ((J[j] - c * J[NC + j]) - sn * (cp * J[2 * NC + j] + sp * J[3 * NC + j]));
  else return mu * (J[j] - c * J[NC + j]);
}
template <int KIND, bool ADAPT, bool EXT>
__device__ __forceinline__ double row_lin3(const double* g, const double* fv, const double* J0, const double* J1,
                                           const double* J2, const double* J3, double* snn, double& alphaE, int lane) {
  constexpr int NC = 8;
  const int i = min(lane & 31, 8);
  const bool act = (lane & 31) < 9, upper = lane >= 32;   // other lanes repeat component 8 and write nothing
  const int q = (i - 3) >> 1;
  const int ra = (i < 3) ? i : (q == 2 ? 1 : 0), rb = (i < 3) ? i : (q == 0 ? 1 : 2);
  const bool im = i >= 4 && (i & 1) == 0;
  const int jn = nn_index(i);
  const double* rad = snn + kL3Rad;
  const double sg = g[kR3Sg];
  const double sgi = im ? 1.0 : sg;
  const double cp = EXT ? g[kR3Cp] : 0.0, sp = EXT ? g[kR3Sp] : 0.0;
  // component i of M = lam E_ee + nn (neutrinos) or -(lam E_ee + nn^*) (antineutrinos)
  const auto matter = [&](const double* J, int at) {
    const double nn = nunu_comp<NC, EXT>(J, rad[3 * at + 2], g[kR3C + at], EXT ? g[kR3Sn + at] : 0.0, cp, sp, jn);
    const double x = sgi * ((i == 0) ? rad[3 * at + 1] + nn : nn);
    return (i == 2) ? 0.0 : x;
  };
  double M1 = 0.0, M2 = 0.0, M3 = 0.0, M4 = 0.0;
  if (KIND != 3) M1 = matter(J0, 0);
  if (KIND == 2 || KIND == 4) M2 = matter(J1, 1);
  if (KIND >= 3) M3 = matter(J2, 1);
  if (KIND == 4) M4 = matter(J3, 2);
  double alpha;
  if (KIND == 1 || KIND == 3) {
    alpha = (KIND == 1) ? 0.5 * g[kR3H] : g[kR3H + 1];
    if (lane < 9) snn[i] = alpha * ((KIND == 1) ? M1 : M3);
  } else {
    const double D = ((KIND == 2) ? M2 : M4) - M1;
    double* FM = snn + kL3FM;
    double* FD = snn + kL3FD;
    if (act) put_full(upper ? FM : FD, ra, rb, im, upper ? M1 : D);
    __asm__ volatile("" ::: "memory");   // the wave's LDS operations complete in program order
    // component i of i[A, D] (X = A D; C_aa = -2 Im X_aa, C_ab = (-(Im X_ab + Im X_ba),
    // Re X_ab - Re X_ba)), A = V0 or M1
    const double* A = upper ? FM : fv;
    const auto at = [](const double* F, int r, int c) { return mk(F[(r * 3 + c) * 2], F[(r * 3 + c) * 2 + 1]); };
    const cplx xab = dot3_mul(at(A, ra, 0), at(FD, 0, rb), at(A, ra, 1), at(FD, 1, rb), at(A, ra, 2), at(FD, 2, rb));
    const cplx xba = dot3_mul(at(A, rb, 0), at(FD, 0, ra), at(A, rb, 1), at(FD, 1, ra), at(A, rb, 2), at(FD, 2, ra));
    const double R = im ? xab.re - xba.re : -(xab.im + xba.im);
    const double hc0 = g[kR3H], hcm = g[kR3H + 1], hc1 = g[kR3H + 2];
    __asm__ volatile("" ::: "memory");
    if (KIND == 2) {
      const double c = (hc0 * hcm) * 0.125;
      alpha = 0.5 * hcm;
      const double P = c * R, Q = fma(alpha, M2, c * R);
      if (act) snn[upper ? i : 9 + i] = upper ? Q : P;
    } else {
      const double c = (hc0 * hc1) * (1.0 / 12.0), a2 = 2.0 * hcm;
      alpha = (((hc0 + a2) + a2) + hc1) * (1.0 / 6.0);
      alphaE = alpha - hcm;
      const double S = fma(hc1, M4, fma(a2, M3, fma(a2, M2, hc0 * M1)));
      const double P = c * R, Q = fma(S, 1.0 / 6.0, c * R);
      if (act) snn[upper ? i : 9 + i] = upper ? Q : P;
      if (ADAPT && act && upper) snn[18 + i] = fma(-hcm, M2, Q);
    }
  }
  __asm__ volatile("" ::: "memory");
  return alpha;
}

// The row constants Q, P (and the error estimate's Q) live in LDS (one 32-double block per
// wave) and are re-read per beam, so the compiler does not keep all of them in registers.
// One (species, emission bin) row of the three-flavour stage, FP64 arithmetic.
// ADAPT (final update only): the new state goes to Xo instead of X, and emax keeps the
// largest embedded error estimate |Theta - K2|^2 (traceless part, Frobenius norm).
// EXT: extended bulb model; rows are (s, j, p) with the azimuth table of the tables.
//
// PK (packed row tails; three flavours, FP64 fixed steps, stages 1-4, one row per
// wavefront, 512-thread blocks, N_E = 64 m + t with 1 <= t <= 32 and N_E <= 2048): a row
// takes m full passes and one pass with t busy lanes.  Wavefronts w and w + 4 of a block
// share a SIMD (the placement measured on this device), so wavefront w < 4 (the owner) also
// runs its partner's tail: after its m passes it runs one pass with lanes 0-31 on its own
// beams 64 m + l and lanes 32-63 on the partner's beams 64 m + l - 32 (with the partner's
// row constants), and the SIMD issues 2 m + 1 passes instead of 2 m + 2.  The owner adds its
// tail's contributions to its own lane sums and hands the partner's over through the
// partner's fold scratch flp as exact integers, so every row adds the same integer sum and
// the moments keep their bits.  Block barriers: after the row constants (the owner reads
// its partner's, snp) and before the partner's fold (the handed-over sums).
template <typename ST, int KIND, bool ADAPT = false, bool EXT = false, bool PK = false>
__device__ __forceinline__ void row3(const StepArgs& a, const ST* X, ST* Xo, long long row, const double* g,
                                     const double* fv, const double (*sJ)[EXT ? 32 : 16], const double* tab,
                                     double* snn, int lane, I128& T, int& err, double& emax,
                                     const ST* pre = nullptr, const double* snp = nullptr, long long* fl = nullptr,
                                     long long* flp = nullptr, bool owner = false) {
  static_assert(!PK || (!ADAPT && !EXT && sizeof(ST) == 8 && KIND >= 1), "packed tails: FP64 fixed steps");
  constexpr int NM = EXT ? 4 : 2;
  const long long plane = a.plane;
  const int NE = a.NE;
  const int s = __builtin_amdgcn_readfirstlane((int)g[kR3S]);
  const int an = (s >= (a.NS >> 1)) ? 1 : 0;   // antiparticle row
  double alpha = 0.0, alphaE = 0.0;
  if constexpr (KIND >= 1)
    alpha = row_lin3<KIND, ADAPT, EXT>(g, fv, sJ[0], sJ[1], sJ[2], sJ[3], snn, alphaE, lane);
  if constexpr (PK) {
    if (lane == 0) {
      snn[kL3Alpha] = alpha;
      snn[kL3S] = (double)s;
    }
    __syncthreads();   // every row's constants are in place (the owner reads its partner's)
  }
  const double* G = tab + (size_t)(kVacRows3 + s) * NE;
  const long long rb = row * NE;
  // PK: the full passes end at kmain; the owner's packed pass takes lane l to beam
  // kmain + (l & 31) of its own row (l < 32) or its partner's (row + 4)
  const int kmain = NE & ~63;
  const bool ton = PK && owner && (lane & 31) < NE - kmain;
  const long long rbt = (lane >> 5) ? rb + 4LL * NE : rb;
  I128 mine = i128_zero();
  for (int k0 = lane; k0 - lane < NE; k0 += 64 * 32) {
    const int kend = PK ? kmain : min(NE, k0 + 64 * 32);
    const unsigned long long base = fix_base(k0, kend);
    unsigned long long acc[8] = {base, base, base, base, base, base, base, base};
    ST q[6];
    if (k0 < kend) {
      if (pre && k0 == lane) {   // the lane's first beam, loaded before the last barrier
#pragma unroll
        for (int c = 0; c < 6; ++c) q[c] = pre[c];
      } else {
#pragma unroll
        for (int c = 0; c < 6; ++c) q[c] = X[rb + k0 + c * plane];
      }
    }
    for (int k = k0; k < kend; k += 64) {
      cplx ps[3] = {mk((double)q[0], (double)q[1]), mk((double)q[2], (double)q[3]),
                    mk((double)q[4], (double)q[5])};
      if (k + 64 < kend) {    // prefetch the lane's next beam
#pragma unroll
        for (int c = 0; c < 6; ++c) q[c] = X[rb + k + 64 + c * plane];
      } else if (PK && ton) {   // the lane's beam of the packed pass
#pragma unroll
        for (int c = 0; c < 6; ++c) q[c] = X[rbt + kmain + (lane & 31) + c * plane];
      }
      __asm__ volatile("" ::: "memory");   // re-read the row's nn terms from LDS per beam
      if (KIND >= 1) {
        double v[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) v[c] = tab[c * NE + k];
        if (KIND == 1 || KIND == 3) {
          exp3_apply(lin3q(alpha, snn, v), ps);
        } else if (KIND == 2) {
          exp3_apply(lin3p(alpha, snn + 9, snn, v, tab[6 * NE + k]), ps);
        } else {
          const double ek = tab[6 * NE + k];
          const Herm3 Th = lin3p(alpha, snn + 9, snn, v, ek);
          if (ADAPT) {
            // |Theta - K2|^2: traceless part, Frobenius norm
            const Herm3 Ed = lin3p(alphaE, snn + 9, snn + 18, v, ek);
            const double tr = ((Ed.d0 + Ed.d1) + Ed.d2) * (1.0 / 3.0);
            const double a0 = Ed.d0 - tr, a1 = Ed.d1 - tr, a2 = Ed.d2 - tr;
            const double o0 = Ed.o01.re * Ed.o01.re + Ed.o01.im * Ed.o01.im;
            const double o1 = Ed.o02.re * Ed.o02.re + Ed.o02.im * Ed.o02.im;
            const double o2 = Ed.o12.re * Ed.o12.re + Ed.o12.im * Ed.o12.im;
            const double e = ((a0 * a0 + a1 * a1) + a2 * a2) + 2.0 * ((o0 + o1) + o2);
            emax = (e > emax) ? e : emax;
          }
          exp3_apply(Th, ps);
          if (a.renorm) {
            const double nrm2 = (norm2(ps[0]) + norm2(ps[1])) + norm2(ps[2]);
            if (!(fabs(nrm2 - 1.0) <= (sizeof(ST) == 8 ? kRenormTol : kRenormTol32))) err |= 8;
            const double inv = fma(-0.5, nrm2, 1.5);   // one Newton step for 1/sqrt from 1
#pragma unroll
            for (int c = 0; c < 3; ++c) ps[c] = mk(ps[c].re * inv, ps[c].im * inv);
          }
          // store, and take the next step's moments from exactly what was stored
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const ST re = (ST)ps[c].re, im = (ST)ps[c].im;
            Xo[rb + k + (2 * c) * plane] = re;
            Xo[rb + k + (2 * c + 1) * plane] = im;
            ps[c] = mk((double)re, (double)im);
          }
        }
      }
      // rho~ components: rho_ee-rho_tt, rho_mm-rho_tt, Re/Im rho_em, rho_et, rho_mt;
      // antineutrinos: -rho^* (real parts and diagonal negated)
      const double n0 = norm2(ps[0]), nm = norm2(ps[1]), nt = norm2(ps[2]);
      const cplx em = cmul_conjb(ps[0], ps[1]), et = cmul_conjb(ps[0], ps[2]), mt = cmul_conjb(ps[1], ps[2]);
      const double v8[8] = {n0 - nt, nm - nt, em.re, em.im, et.re, et.im, mt.re, mt.im};
      if (!((n0 + nm) + nt < 2.0)) err |= 1;
      const double ws = G[k] * a.s1;
      const double wa = an ? -ws : ws;    // the negated components of -rho^*
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += fix_bits(v8[i], (i < 3 || i == 4 || i == 6) ? wa : ws);
    }
    if constexpr (PK) {
      if (owner) {
        // the packed pass: the same arithmetic as a full pass, with each lane's row constants
        __asm__ volatile("" ::: "memory");
        unsigned long long x[8] = {kFixMagic, kFixMagic, kFixMagic, kFixMagic,
                                   kFixMagic, kFixMagic, kFixMagic, kFixMagic};
        if (ton) {
          const int hf = lane >> 5, k = kmain + (lane & 31);
          const double* sl = hf ? snp : snn;
          const double al = hf ? snp[kL3Alpha] : alpha;
          const int sh = hf ? (int)snp[kL3S] : s;
          const int anl = (sh >= (a.NS >> 1)) ? 1 : 0;
          cplx ps[3] = {mk((double)q[0], (double)q[1]), mk((double)q[2], (double)q[3]),
                        mk((double)q[4], (double)q[5])};
          double v[6];
#pragma unroll
          for (int c = 0; c < 6; ++c) v[c] = tab[c * NE + k];
          if (KIND == 1 || KIND == 3) {
            exp3_apply(lin3q(al, sl, v), ps);
          } else if (KIND == 2) {
            exp3_apply(lin3p(al, sl + 9, sl, v, tab[6 * NE + k]), ps);
          } else {
            const double ek = tab[6 * NE + k];
            exp3_apply(lin3p(al, sl + 9, sl, v, ek), ps);
            if (a.renorm) {
              const double nrm2 = (norm2(ps[0]) + norm2(ps[1])) + norm2(ps[2]);
              if (!(fabs(nrm2 - 1.0) <= kRenormTol)) err |= 8;
              const double inv = fma(-0.5, nrm2, 1.5);   // one Newton step for 1/sqrt from 1
#pragma unroll
              for (int c = 0; c < 3; ++c) ps[c] = mk(ps[c].re * inv, ps[c].im * inv);
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              Xo[rbt + k + (2 * c) * plane] = (ST)ps[c].re;
              Xo[rbt + k + (2 * c + 1) * plane] = (ST)ps[c].im;
            }
          }
          const double n0 = norm2(ps[0]), nm = norm2(ps[1]), nt = norm2(ps[2]);
          const cplx em = cmul_conjb(ps[0], ps[1]), et = cmul_conjb(ps[0], ps[2]), mt = cmul_conjb(ps[1], ps[2]);
          const double v8[8] = {n0 - nt, nm - nt, em.re, em.im, et.re, et.im, mt.re, mt.im};
          if (!((n0 + nm) + nt < 2.0)) err |= 1;
          const double ws = tab[(size_t)(kVacRows3 + sh) * NE + k] * a.s1;
          const double wa = anl ? -ws : ws;
#pragma unroll
          for (int i = 0; i < 8; ++i) x[i] = fix_bits(v8[i], (i < 3 || i == 4 || i == 6) ? wa : ws);
        }
        // contributions as integers (less the kFixMagic each carries); idle lanes give 0
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const unsigned long long xv = x[i] - kFixMagic;
          if (lane >> 5) flp[i * 32 + (lane & 31)] = (long long)xv;
          else acc[i] += xv;
        }
        mine = i128_add(mine, i128_from(wave_fold<8>(acc, lane)));
      }
      __syncthreads();   // the owner's handed-over contributions are in the partner's scratch
      if (!owner) {
        if (lane < 32) {
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[i] += (unsigned long long)fl[i * 32 + lane];
        }
        mine = i128_add(mine, i128_from(wave_fold<8>(acc, lane)));
      }
    } else {
      mine = i128_add(mine, i128_from(wave_fold<8>(acc, lane)));
    }
  }
  const double v = (NE <= kSegNE) ? (double)(long long)mine.lo : i128_to_double(mine);
  const double icmom = (KIND == 0) ? 1.0 / g[kR3C] : ((KIND <= 2) ? g[kR3Icm] : g[kR3Ic1]);
  double asc = 0.0, ass = 0.0;
  if constexpr (EXT) {
    const double t = g[kR3Sn + ((KIND == 0) ? 0 : ((KIND <= 2) ? 1 : 2))] * icmom;
    asc = t * g[kR3Cp];
    ass = t * g[kR3Sp];
  }
  close_row<8, NM>(Scales{a.s1, a.s0, a.p2e1, a.p2e0}, lane, mine, v, icmom, T, err, asc, ass);
}

// Rows gw, gw + nw, ... (nrw of them): kept ones from the table kr, more in groups of kKeep3
// whose labels and geometry are computed (lane-parallel) in every stage.
template <bool EXT, typename F>
__device__ __forceinline__ void each_row3(const StepArgs& a, double h, long long gw, long long nw, int nrw, int lane,
                                          const double* snn, double* kr, F fn) {
  for (int r0 = 0; r0 < nrw; r0 += kKeep3) {
    const int gn = min(nrw - r0, kKeep3);
    if (nrw > kKeep3) {
      __asm__ volatile("" ::: "memory");   // the previous group's rows have read their blocks
      keep_labels3<EXT>(a, gw + r0 * nw, nw, gn, lane, kr);
      keep_geo3<EXT>(snn + kL3Rad, h, gn, lane, kr);
    }
    for (int i = 0; i < gn; ++i) fn(gw + (r0 + i) * nw, kr + i * kRow3, r0 + i == 0);
  }
}
template <typename ST, int KIND, bool ADAPT = false, bool EXT = false, bool PK = false>
__device__ __forceinline__ void stage3(const StepArgs& a, double h, const ST* X, ST* Xo,
                                       const double (*sJ)[EXT ? 32 : 16], const double* tab, double* snn, double* kr,
                                       const double* fv, long long gw, long long nw, int nrw, int lane, I128& T,
                                       int& err, double& emax, const ST* pre = nullptr, const double* snp = nullptr,
                                       long long* fl = nullptr, long long* flp = nullptr, bool owner = false) {
  if constexpr (PK) {   // one row per wavefront
    row3<ST, KIND, false, false, true>(a, X, Xo, gw, kr, fv, sJ, tab, snn, lane, T, err, emax, pre, snp, fl, flp, owner);
  } else {
    each_row3<EXT>(a, h, gw, nw, nrw, lane, snn, kr, [&](long long row, const double* g, bool first) {
      row3<ST, KIND, ADAPT, EXT>(a, X, Xo, row, g, fv, sJ, tab, snn, lane, T, err, emax, first ? pre : nullptr);
    });
  }
}
// Load the lane's first beam of the wavefront's first row (the next stage starts there),
// so that the load completes while the wavefront waits at the grid barrier.
template <int NSC, typename ST>
__device__ __forceinline__ void prefetch_first(const StepArgs& a, const ST* X, long long gw, long long nrow, int lane,
                                               ST* pre) {
  if (gw < nrow && lane < a.NE) {
#pragma unroll
    for (int c = 0; c < NSC; ++c) pre[c] = X[gw * a.NE + lane + c * a.plane];
  }
}

// ------------------------------------------------------- three flavours, mixed precision
// NB_FP32_STATE: psi stored in FP32 and the per-beam exponentials in FP32; the generators
// come from the FP64 row constants (stages 1-3 rounded to FP32 once per row, the final
// update's Theta summed per beam in FP64 and rounded), the moment contributions, their
// reduction and the renormalisation of the updated state are FP64, and the next moments
// are taken from the rounded stored state.

// One row of the mixed-precision stage with FP32 per-beam arithmetic.
// The moment contributions of a lane's beams (k = lane mod 64 within a segment of 64 x 16
// beams) are summed in FP64 and converted to fixed point once per segment, so the total
// does not depend on the launch shape; 16 contributions below 2^51 each stay below the
// 2^56 that the fold's 64-bit lane sums allow.
// FT: ftab (LDS) holds the vacuum rows and e_k as FP32, eight floats per energy
// (H_ee, H_mumu, H_tautau, H_emu, H_etau, H_mutau, e_k, 0), read by stages 1-3.
template <int KIND, bool FT>
__device__ __forceinline__ void row3m(const StepArgs& a, long long row, const double* g, const double* fv,
                                      const double (*sJ)[16], const double* tab, const float* ftab, double* snd,
                                      int lane, I128& T, int& err) {
#pragma clang fp contract(fast)
  constexpr int kSeg = 64 * 16;
  const long long plane = a.plane;
  const int NE = a.NE;
  // per-plane bases (uniform) and one 32-bit byte offset per lane: the FP32 planes are
  // below 2^32 bytes (checked at model creation)
  char* Xp[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) Xp[c] = (char*)((float*)a.X + c * plane);
  const int s = __builtin_amdgcn_readfirstlane((int)g[kR3S]);
  const int an = (s >= (a.NS >> 1)) ? 1 : 0;   // antiparticle row
  // generator row constants (FP64, as in the FP64 stepper): snd[0..8] Q, snd[9..17] P;
  // stages 1-3 use FP32 copies in snn, the final update's Theta is summed in FP64
  double alphaE = 0.0;
  const double alpha = (KIND >= 1) ? row_lin3<(KIND >= 1 ? KIND : 1), false, false>(g, fv, sJ[0], sJ[1], sJ[2], sJ[3],
                                                                                     snd, alphaE, lane)
                                   : 0.0;
  const float alphaf = (float)alpha;
  float* snn = (float*)(snd + kL3F32);
  if (KIND >= 1 && KIND <= 3) {
    if (lane < 18) snn[lane] = (float)snd[lane];
    __asm__ volatile("" ::: "memory");
  }
  const double* G = tab + (size_t)(kVacRows3 + s) * NE;
  const long long rb = row * NE;
  I128 mine = i128_zero();
  for (int k0 = lane; k0 - lane < NE; k0 += kSeg) {
    const int kend = min(NE, k0 + kSeg);
    double dacc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float q[6];
    if (k0 < kend) {
#pragma unroll
      for (int c = 0; c < 6; ++c) q[c] = *(const float*)(Xp[c] + (unsigned)(rb + k0) * 4u);
    }
    for (int k = k0; k < kend; k += 64) {
      cplxf ps[3] = {mkf(q[0], q[1]), mkf(q[2], q[3]), mkf(q[4], q[5])};
      if (k + 64 < kend) {
#pragma unroll
        for (int c = 0; c < 6; ++c) q[c] = *(const float*)(Xp[c] + (unsigned)(rb + k + 64) * 4u);
      }
      __asm__ volatile("" ::: "memory");
      double pd[6];
      if (KIND >= 1) {
        float v[6], ekf = 0.0f;
        double vd[6];
        if constexpr (KIND <= 3 && FT) {
          const float4 f0 = *reinterpret_cast<const float4*>(ftab + 8 * k);
          const float4 f1 = *reinterpret_cast<const float4*>(ftab + 8 * k + 4);
          v[0] = f0.x; v[1] = f0.y; v[2] = f0.z; v[3] = f0.w; v[4] = f1.x; v[5] = f1.y;
          ekf = f1.z;
        } else {
#pragma unroll
          for (int c = 0; c < 6; ++c) {
            vd[c] = tab[c * NE + k];
            v[c] = (float)vd[c];
          }
          if (KIND == 2) ekf = (float)tab[6 * NE + k];
        }
        if (KIND == 1 || KIND == 3) {
          exp3_apply_f(Herm3f{fmaf(alphaf, v[0], snn[0]), fmaf(alphaf, v[1], snn[1]), fmaf(alphaf, v[2], snn[2]),
                              mkf(fmaf(alphaf, v[3], snn[3]), snn[4]), mkf(fmaf(alphaf, v[4], snn[5]), snn[6]),
                              mkf(fmaf(alphaf, v[5], snn[7]), snn[8])},
                       ps);
        } else if (KIND == 2) {
          const float ek = ekf;
          const float* P = snn + 9;
          exp3_apply_f(Herm3f{fmaf(alphaf, v[0], fmaf(ek, P[0], snn[0])), fmaf(alphaf, v[1], fmaf(ek, P[1], snn[1])),
                              fmaf(alphaf, v[2], fmaf(ek, P[2], snn[2])),
                              mkf(fmaf(alphaf, v[3], fmaf(ek, P[3], snn[3])), fmaf(ek, P[4], snn[4])),
                              mkf(fmaf(alphaf, v[4], fmaf(ek, P[5], snn[5])), fmaf(ek, P[6], snn[6])),
                              mkf(fmaf(alphaf, v[5], fmaf(ek, P[7], snn[7])), fmaf(ek, P[8], snn[8]))},
                       ps);
        } else {
          // Theta = alpha V_k + e_k P + Q.  The generators are nearly constant from step to
          // step (the vacuum term is), so rounding their parts to FP32 would repeat the same
          // phase error every step; Theta is formed in FP64 and rounded once.
          const Herm3 Td = lin3p(alpha, snd + 9, snd, vd, tab[6 * NE + k]);
          const Herm3f Th{(float)Td.d0, (float)Td.d1, (float)Td.d2, mkf((float)Td.o01.re, (float)Td.o01.im),
                          mkf((float)Td.o02.re, (float)Td.o02.im), mkf((float)Td.o12.re, (float)Td.o12.im)};
          // psi + (exp(-i Theta) - 1) psi formed in FP64 from the FP32 increment, then
          // renormalised in FP64, stored rounded to FP32; moments from the stored values
          cplxf dl[3];
          exp3_incr_f(Th, ps, dl);
          const double re0 = (double)ps[0].re + (double)dl[0].re, im0 = (double)ps[0].im + (double)dl[0].im;
          const double re1 = (double)ps[1].re + (double)dl[1].re, im1 = (double)ps[1].im + (double)dl[1].im;
          const double re2 = (double)ps[2].re + (double)dl[2].re, im2 = (double)ps[2].im + (double)dl[2].im;
          const double nrm2 = (fma(re0, re0, im0 * im0) + fma(re1, re1, im1 * im1)) + fma(re2, re2, im2 * im2);
          // 1/sqrt(nrm2) by one Newton step from 1: nrm2 = 1 + d with |d| ~ 1e-7 (a unit
          // FP32-stored state and an increment accurate to FP32), so the error 3 d^2 / 8 is
          // far below FP32 storage precision
          if (a.renorm && !(fabs(nrm2 - 1.0) <= kRenormTol32)) err |= 8;
          const double inv = fma(-0.5, nrm2, 1.5);
          const float o[6] = {(float)(re0 * inv), (float)(im0 * inv), (float)(re1 * inv),
                              (float)(im1 * inv), (float)(re2 * inv), (float)(im2 * inv)};
#pragma unroll
          for (int c = 0; c < 6; ++c) *(float*)(Xp[c] + (unsigned)(rb + k) * 4u) = o[c];
          ps[0] = mkf(o[0], o[1]);
          ps[1] = mkf(o[2], o[3]);
          ps[2] = mkf(o[4], o[5]);
        }
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        pd[2 * c] = (double)ps[c].re;
        pd[2 * c + 1] = (double)ps[c].im;
      }
      const cplx p0 = mk(pd[0], pd[1]), p1 = mk(pd[2], pd[3]), p2 = mk(pd[4], pd[5]);
      const double n0 = norm2(p0), nm = norm2(p1), nt = norm2(p2);
      const cplx em = cmul_conjb(p0, p1), et = cmul_conjb(p0, p2), mt = cmul_conjb(p1, p2);
      const double v8[8] = {n0 - nt, nm - nt, em.re, em.im, et.re, et.im, mt.re, mt.im};
      const double w = G[k];
      const double wa = an ? -w : w;   // the negated components of -rho^*
#pragma unroll
      for (int i = 0; i < 8; ++i) dacc[i] = fma((i < 3 || i == 4 || i == 6) ? wa : w, v8[i], dacc[i]);
    }
    unsigned long long acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = (unsigned long long)to_fix(dacc[i], a.s1, kTwo56, err);
    mine = i128_add(mine, i128_from(wave_fold<8>(acc, lane)));
  }
  const double v = (NE <= kSeg) ? (double)(long long)mine.lo : i128_to_double(mine);
  const double icmom = (KIND == 0) ? 1.0 / g[kR3C] : ((KIND <= 2) ? g[kR3Icm] : g[kR3Ic1]);
  close_row<8>(Scales{a.s1, a.s0, a.p2e1, a.p2e0}, lane, mine, v, icmom, T, err);
}

// Mixed-precision stage: every row with FP32 per-beam arithmetic.  The host runs these
// launches only over steps whose stage generators rotate a beam by at most one radian per
// step (a bound computed from the model's parameters); nearer the neutrinosphere FP32
// cannot hold the per-step phase and the FP64-arithmetic launch on the FP32 state is used.
template <int KIND, bool FT>
__device__ __forceinline__ void stage3m(const StepArgs& a, const double (*sJ)[16], const double* tab, const float* ftab,
                                        double* snn, double* kr, const double* fv, long long gw, long long nw, int nrw,
                                        int lane, I128& T, int& err) {
  each_row3<false>(a, a.h, gw, nw, nrw, lane, snn, kr, [&](long long row, const double* g, bool) {
    row3m<KIND, FT>(a, row, g, fv, sJ, tab, ftab, snn, lane, T, err);
  });
}

// --------------------------------------------------------------- the stepper
// The energy tables (vacuum terms and weights) are staged into LDS once per launch
// when TLDS (they are read by every row).
// EXT: the extended bulb model (azimuthal bins, four moments); FP64 only.
// BS: threads per block (512 or 256; every array and loop bound below is a constant).
// PK: packed row tails (row3); the host launches this variant only when every wavefront of
// the grid owns exactly one row and the row length qualifies.
template <int NF, typename ST, bool TLDS, bool F32, bool EXT, int BS, bool PK = false>
// Register budget: the two-flavour instantiations at 256 threads per block are held to 168
// VGPRs (three wavefronts per SIMD, three blocks per CU); the others keep the compiler's
// choice under the 512-thread bound (two wavefronts per SIMD).
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu((NF == 2 && BS == 256) ? 3 : 1)))
k_advance(StepArgs a) {
  constexpr int NC = (NF == 2) ? 3 : 8;
  constexpr int NM = EXT ? 4 : 2;
  constexpr int NV = NM * NC;
  constexpr int WPB = BS / 64;
  __shared__ double sJ[4][NV];
  __shared__ RedLds<NV, BS> R;
  // per wavefront: stage constants
  __shared__ double snn_all[WPB][NF == 2 ? kC2Size : kL3Size];
  // three flavours: each wave's kept rows, and V0
  __shared__ double skr[NF == 3 ? WPB : 1][NF == 3 ? kKeep3 * kRow3 : 1];
  __shared__ double sfv[NF == 3 ? 18 : 1];
  // the two-flavour extended model's rows fold kFoldRowsExt at a time (group2); packed tails
  // hand sums over
  __shared__ long long sfold[WPB][(NF == 2) ? (EXT ? fold2_words(kFoldRowsExt) : 1) : (PK ? 256 : 1)];
  __shared__ double s_sct[kSinCosTab];   // sin/cos constants of the two-flavour rotations
  // two flavours: each wave's row-constant table
  __shared__ double srt[NF == 2 ? WPB : 1][NF == 2 ? row_table2(EXT) : 1];
  extern __shared__ __align__(16) double dyn_tab[];
  // the wavefront index as a wave-uniform (scalar) value: the row indices, their divisions
  // and the row base offsets derived from it then live in scalar registers
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long gw = (long long)blockIdx.x * WPB + wid;
  const long long nw = (long long)gridDim.x * WPB;
  const double* tab = a.tab;
  const float* ftab = nullptr;
  if (launch_aborted(a.sync, a.cancel)) return;
  red_init(R);
  if (NF == 2 && threadIdx.x == 0) sincos_coefs(s_sct);
  __syncthreads();
  if constexpr (TLDS) {
    const int ntab = ((NF == 2) ? 2 : kVacRows3) * a.NE + a.NS * a.NE;
    for (int i = threadIdx.x; i < ntab; i += BS) dyn_tab[i] = a.tab[i];
    if constexpr (F32) {
      // the FP32 copy of the vacuum rows and e_k, eight floats per energy, after the table
      // (at a 16-byte boundary)
      float* ft = reinterpret_cast<float*>(dyn_tab + ((ntab + 1) & ~1));
      for (int i = threadIdx.x; i < 8 * a.NE; i += BS) {
        const int k = i >> 3, c = i & 7;
        ft[i] = (c < 7) ? (float)a.tab[c * a.NE + k] : 0.0f;
      }
      ftab = ft;
    }
    __syncthreads();
    tab = dyn_tab;
  }
  double* snn = snn_all[wid];
  long long* fl = sfold[wid];
  const long long step0 = a.step_ctl[0];
  long long nsteps;
  if (a.use_window) {
    // steps [step0, min(target, win_hi)) if step0 lies in the window [win_lo, win_hi)
    nsteps = (step0 < a.win_lo) ? 0LL : max(0LL, min(a.step_ctl[1], a.win_hi) - step0);
  } else {
    nsteps = max(0LL, min(a.nsteps, a.total_steps - step0));
  }
  if (a.use_window && nsteps == 0) {   // uniform over the grid: nothing to do
    if (a.host && blockIdx.x == 0 && threadIdx.x == 0) put_host(a.host, a.sync, step0);
    return;
  }
  unsigned epoch = 0;
  int err = 0;
  bool ok = true;
  double enone = 0.0;   // error estimate (adaptive runs only)
  I128 T = i128_zero();
  // FP64 arithmetic, bulb model and 3f: each stage's first beam is loaded before the preceding barrier
  ST pre[6] = {};
  const long long nrow3 = (long long)a.NS * a.NU * (EXT ? a.NP : 1);
  if constexpr (PK) {
    // the packed variant's block barriers need one row per wavefront (uniform over the grid):
    // a launch that breaks it ends at once with a range error instead of waiting
    if (!(nrow3 == nw && a.NE > 64 && a.NE <= 64 * 32 && (a.NE & 63) <= 32 && (a.NE & 63) != 0)) {
      if (threadIdx.x == 0)
        __hip_atomic_fetch_or(a.sync + kSyncStatus, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
  }
  const int nrw = wave_rows(gw, nw, nrow3);
  double* rt = srt[NF == 2 ? wid : 0];
  double* kr = skr[NF == 3 ? wid : 0];
  if constexpr (NF == 3) {
    init3(a, lane, sfv, snn);
    if (nrw <= kKeep3) keep_labels3<EXT>(a, gw, nw, nrw, lane, kr);
    prep3<EXT>(a, geo_fixed(a, step0), lane, nrw, snn, kr);
    __syncthreads();
  }
  if constexpr (NF == 2) {
    if (!EXT) keep_rows2(a, gw, nw, lane, nrw, rt);
    prep2<EXT>(a, geo_fixed(a, step0), lane, nrw, snn, rt);
  }
  // the partner wavefront's constant block and fold scratch (packed tails)
  const double* snp = snn_all[wid ^ (WPB / 2)];
  long long* flp = sfold[wid ^ (WPB / 2)];
  const bool owner = wid < WPB / 2;
  // the stage-1 moments of the current state: left by the previous launch of this variant
  // if it ended at this step (the same values the initial pass would compute), else the
  // initial moment pass
  const long long kind = NF * 16 + (sizeof(ST) == 4 ? 8 : 0) + (F32 ? 4 : 0) + (EXT ? 2 : 0);
  if (a.step_ctl[kCtlMTag] == step0 && a.step_ctl[kCtlMKind] == kind) {
    if constexpr (NF == 3 && !F32) prefetch_first<6>(a, (const ST*)a.X, gw, nrow3, lane, pre);
    if constexpr (NF == 2 && !EXT) prefetch_first<3>(a, (const ST*)a.X, gw, nrow3, lane, pre);
    if (threadIdx.x < NV) sJ[0][threadIdx.x] = as_double((unsigned long long)a.step_ctl[kCtlMom + threadIdx.x]);
    __syncthreads();
  } else {
    if constexpr (NF == 2) { stage2<0, false, EXT>(a, a.h, (const double*)a.X, (double*)a.X, sJ, tab, gw, nw, nrw, lane, fl, T, err, enone, snn, s_sct, rt); if (!EXT) prefetch_first<3>(a, (const ST*)a.X, gw, nrow3, lane, pre); }
    else if constexpr (F32) stage3m<0, TLDS>(a, sJ, tab, ftab, snn, kr, sfv, gw, nw, nrw, lane, T, err);
    else { stage3<ST, 0, false, EXT>(a, a.h, (const ST*)a.X, (ST*)a.X, sJ, tab, snn, kr, sfv, gw, nw, nrw, lane, T, err, enone); prefetch_first<6>(a, (const ST*)a.X, gw, nrow3, lane, pre); }
    ok = finish_stage<false, NM>(a, epoch++, T, R, sJ[0]);
  }
  // the adjoint's forward pass records every stage's moments: [step][slot][NV]
  auto record = [&](long long step, int slot) {
    if (a.Jhist && ok && blockIdx.x == 0 && threadIdx.x < NV)
      a.Jhist[((size_t)step * 4 + slot) * NV + threadIdx.x] = sJ[slot][threadIdx.x];
  };
  record(step0, 0);
  for (long long n = step0; ok && n < step0 + nsteps; ++n) {
    T = i128_zero();
    if constexpr (NF == 2) { stage2<1, false, EXT>(a, a.h, (const double*)a.X, (double*)a.X, sJ, tab, gw, nw, nrw, lane, fl, T, err, enone, snn, s_sct, rt, EXT ? nullptr : pre); if (!EXT) prefetch_first<3>(a, (const ST*)a.X, gw, nrow3, lane, pre); }
    else if constexpr (F32) stage3m<1, TLDS>(a, sJ, tab, ftab, snn, kr, sfv, gw, nw, nrw, lane, T, err);
    else { stage3<ST, 1, false, EXT, PK>(a, a.h, (const ST*)a.X, (ST*)a.X, sJ, tab, snn, kr, sfv, gw, nw, nrw, lane, T, err, enone, pre, snp, fl, flp, owner); prefetch_first<6>(a, (const ST*)a.X, gw, nrow3, lane, pre); }
    if (!(ok = finish_stage<false, NM>(a, epoch++, T, R, sJ[1]))) break;
    record(n, 1);
    T = i128_zero();
    if constexpr (NF == 2) { stage2<2, false, EXT>(a, a.h, (const double*)a.X, (double*)a.X, sJ, tab, gw, nw, nrw, lane, fl, T, err, enone, snn, s_sct, rt, EXT ? nullptr : pre); if (!EXT) prefetch_first<3>(a, (const ST*)a.X, gw, nrow3, lane, pre); }
    else if constexpr (F32) stage3m<2, TLDS>(a, sJ, tab, ftab, snn, kr, sfv, gw, nw, nrw, lane, T, err);
    else { stage3<ST, 2, false, EXT, PK>(a, a.h, (const ST*)a.X, (ST*)a.X, sJ, tab, snn, kr, sfv, gw, nw, nrw, lane, T, err, enone, pre, snp, fl, flp, owner); prefetch_first<6>(a, (const ST*)a.X, gw, nrow3, lane, pre); }
    if (!(ok = finish_stage<false, NM>(a, epoch++, T, R, sJ[2]))) break;
    record(n, 2);
    T = i128_zero();
    if constexpr (NF == 2) { stage2<3, false, EXT>(a, a.h, (const double*)a.X, (double*)a.X, sJ, tab, gw, nw, nrw, lane, fl, T, err, enone, snn, s_sct, rt, EXT ? nullptr : pre); if (!EXT) prefetch_first<3>(a, (const ST*)a.X, gw, nrow3, lane, pre); }
    else if constexpr (F32) stage3m<3, TLDS>(a, sJ, tab, ftab, snn, kr, sfv, gw, nw, nrw, lane, T, err);
    else { stage3<ST, 3, false, EXT, PK>(a, a.h, (const ST*)a.X, (ST*)a.X, sJ, tab, snn, kr, sfv, gw, nw, nrw, lane, T, err, enone, pre, snp, fl, flp, owner); prefetch_first<6>(a, (const ST*)a.X, gw, nrow3, lane, pre); }
    if (!(ok = finish_stage<false, NM>(a, epoch++, T, R, sJ[3]))) break;
    record(n, 3);
    T = i128_zero();
    if constexpr (NF == 2) { stage2<4, false, EXT>(a, a.h, (const double*)a.X, (double*)a.X, sJ, tab, gw, nw, nrw, lane, fl, T, err, enone, snn, s_sct, rt, EXT ? nullptr : pre); if (!EXT) prefetch_first<3>(a, (const ST*)a.X, gw, nrow3, lane, pre); }
    else if constexpr (F32) stage3m<4, TLDS>(a, sJ, tab, ftab, snn, kr, sfv, gw, nw, nrw, lane, T, err);
    else { stage3<ST, 4, false, EXT, PK>(a, a.h, (const ST*)a.X, (ST*)a.X, sJ, tab, snn, kr, sfv, gw, nw, nrw, lane, T, err, enone, pre, snp, fl, flp, owner); prefetch_first<6>(a, (const ST*)a.X, gw, nrow3, lane, pre); }
    ok = finish_stage<false, NM>(a, epoch++, T, R, sJ[0], [&] {
      if constexpr (NF == 2) prep2<EXT>(a, geo_fixed(a, n + 1), lane, nrw, snn, rt);
      else prep3<EXT>(a, geo_fixed(a, n + 1), lane, nrw, snn, kr);
    });
    record(n + 1, 0);
  }
  // the block that ends last (all have passed the last barrier and read its sums, and read
  // the start step before the first) moves the step counter, leaves the moments of the new
  // state for the next launch, clears the reduction words for it (so that no clear need
  // precede it) and reports to the host
  if (launch_ends(a.sync, err, ok)) {
    if (threadIdx.x < NV) a.step_ctl[kCtlMom + threadIdx.x] = (long long)as_bits(sJ[0][threadIdx.x]);
    for (int i = threadIdx.x; i < kSyncRedEnd - kSyncRed; i += BS) a.sync[kSyncRed + i] = 0u;
    if (threadIdx.x == 0) {
      a.sync[kSyncDone] = 0u;
      a.step_ctl[0] = step0 + nsteps;
      a.step_ctl[kCtlMTag] = step0 + nsteps;
      a.step_ctl[kCtlMKind] = kind;
      if (a.host) put_host(a.host, a.sync, step0 + nsteps);
    }
  }
}

template __global__ void k_advance<2, double, true, false, false, kBlock>(StepArgs);
template __global__ void k_advance<2, double, false, false, false, kBlock>(StepArgs);
template __global__ void k_advance<3, double, true, false, false, kBlock>(StepArgs);
template __global__ void k_advance<3, double, false, false, false, kBlock>(StepArgs);
template __global__ void k_advance<3, float, true, false, false, kBlock>(StepArgs);
template __global__ void k_advance<3, float, false, false, false, kBlock>(StepArgs);
template __global__ void k_advance<3, float, true, true, false, kBlock>(StepArgs);
template __global__ void k_advance<3, float, false, true, false, kBlock>(StepArgs);
template __global__ void k_advance<2, double, true, false, true, kBlock>(StepArgs);
template __global__ void k_advance<2, double, false, false, true, kBlock>(StepArgs);
template __global__ void k_advance<3, double, true, false, true, kBlock>(StepArgs);
template __global__ void k_advance<3, double, false, false, true, kBlock>(StepArgs);
template __global__ void k_advance<2, double, true, false, false, kBlockSmall>(StepArgs);
template __global__ void k_advance<2, double, false, false, false, kBlockSmall>(StepArgs);
template __global__ void k_advance<3, double, true, false, false, kBlockSmall>(StepArgs);
template __global__ void k_advance<3, double, false, false, false, kBlockSmall>(StepArgs);
template __global__ void k_advance<3, float, true, false, false, kBlockSmall>(StepArgs);
template __global__ void k_advance<3, float, false, false, false, kBlockSmall>(StepArgs);
template __global__ void k_advance<3, float, true, true, false, kBlockSmall>(StepArgs);
template __global__ void k_advance<3, float, false, true, false, kBlockSmall>(StepArgs);
template __global__ void k_advance<2, double, true, false, true, kBlockSmall>(StepArgs);
template __global__ void k_advance<2, double, false, false, true, kBlockSmall>(StepArgs);
template __global__ void k_advance<3, double, true, false, true, kBlockSmall>(StepArgs);
template __global__ void k_advance<3, double, false, false, true, kBlockSmall>(StepArgs);
template __global__ void k_advance<3, double, true, false, false, kBlock, true>(StepArgs);
template __global__ void k_advance<3, double, false, false, false, kBlock, true>(StepArgs);

// --------------------------------------------------------------- adaptive step control
// One persistent launch integrates from r (step_ctl[kCtlR]) with the step length
// step_ctl[kCtlH] to r_end.  Each attempt is a full RKMK4 step from the current state X
// into the other buffer Xn; the final update's barrier also reduces the largest error
// estimate E, from which every block takes the same decision: accept (swap buffers,
// advance r, double h if E <= tol^2/128 and 2h <= h_max) or reject (keep X and the saved
// moments of X, halve h).  The last step is shortened to end at r_end.  At the end each
// wavefront copies its rows back to X if the result sits in the second buffer.
template <int NF, bool TLDS, int BS>
__global__ void __launch_bounds__(BS) k_adaptive(StepArgs a) {
  constexpr int NC = (NF == 2) ? 3 : 8;
  constexpr int NV = 2 * NC;
  __shared__ double sJ[4][NV];
  __shared__ double sJsave[NV];
  __shared__ double sE[1];
  __shared__ RedLds<NV, BS, true> R;
  __shared__ double snn_all[BS / 64][NF == 2 ? kC2Size : kL3Size];   // stage constants
  __shared__ double skr[NF == 3 ? BS / 64 : 1][NF == 3 ? kKeep3 * kRow3 : 1];
  __shared__ double sfv[NF == 3 ? 18 : 1];
  __shared__ double s_sct[kSinCosTab];   // sin/cos constants of the two-flavour rotations
  extern __shared__ __align__(16) double dyn_tab[];
  // the wavefront index as a wave-uniform (scalar) value: the row indices, their divisions
  // and the row base offsets derived from it then live in scalar registers
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long gw = (long long)blockIdx.x * (BS / 64) + wid;
  const long long nw = (long long)gridDim.x * (BS / 64);
  if (launch_aborted(a.sync)) return;
  const double* tab = a.tab;
  red_init(R);
  if (NF == 2 && threadIdx.x == 0) sincos_coefs(s_sct);
  __syncthreads();
  if constexpr (TLDS) {
    const int ntab = ((NF == 2) ? 2 : kVacRows3) * a.NE + a.NS * a.NE;
    for (int i = threadIdx.x; i < ntab; i += BS) dyn_tab[i] = a.tab[i];
    __syncthreads();
    tab = dyn_tab;
  }
  double* snn = snn_all[wid];
  double* kr = skr[NF == 3 ? wid : 0];
  long long* ctl = a.step_ctl;
  double r = as_double((unsigned long long)ctl[kCtlR]);
  double h = as_double((unsigned long long)ctl[kCtlH]);
  double* X = (double*)a.X;
  double* Xn = (double*)a.X2;
  unsigned epoch = 0;
  int err = 0, fail = 0;
  long long nacc = 0, nrej = 0, natt = 0;
  double emax = 0.0;
  I128 T = i128_zero();
  const int nrw = wave_rows(gw, nw, (long long)a.NS * a.NU);
  __shared__ double srt[NF == 2 ? BS / 64 : 1][NF == 2 ? row_table2(false) : 1];
  double* rt = srt[NF == 2 ? wid : 0];
  auto stage = [&](auto kind, const StepGeo& G) {
    constexpr int K = decltype(kind)::value;
    if constexpr (NF == 2) stage2<K, K == 4>(a, G.h, X, Xn, sJ, tab, gw, nw, nrw, lane, nullptr, T, err, emax, snn, s_sct, rt);
    else stage3<double, K, K == 4>(a, G.h, X, Xn, sJ, tab, snn, kr, sfv, gw, nw, nrw, lane, T, err, emax);
  };
  using K0 = std::integral_constant<int, 0>;
  using K1 = std::integral_constant<int, 1>;
  using K2 = std::integral_constant<int, 2>;
  using K3 = std::integral_constant<int, 3>;
  using K4 = std::integral_constant<int, 4>;
  if constexpr (NF == 2) {
    keep_rows2(a, gw, nw, lane, nrw, rt);
    prep2<false>(a, StepGeo{r, r, r, 0.0}, lane, nrw, snn, rt);
  } else {
    init3(a, lane, sfv, snn);
    if (nrw <= kKeep3) keep_labels3<false>(a, gw, nw, nrw, lane, kr);
    prep3<false>(a, StepGeo{r, r, r, 0.0}, lane, nrw, snn, kr);
    __syncthreads();
  }
  stage(K0{}, StepGeo{r, r, r, 0.0});
  bool ok = finish_stage<false, 2>(a, epoch++, T, R, sJ[0]);
  if (threadIdx.x < NV) sJsave[threadIdx.x] = sJ[0][threadIdx.x];
  while (ok) {
    const bool last = (r + h >= a.r_end);
    const double hs = last ? a.r_end - r : h;
    const StepGeo G{r, r + 0.5 * hs, last ? a.r_end : r + hs, hs};
    if constexpr (NF == 2) prep2<false>(a, G, lane, nrw, snn, rt);
    else prep3<false>(a, G, lane, nrw, snn, kr);
    T = i128_zero();
    stage(K1{}, G);
    if (!(ok = finish_stage<false, 2>(a, epoch++, T, R, sJ[1]))) break;
    T = i128_zero();
    stage(K2{}, G);
    if (!(ok = finish_stage<false, 2>(a, epoch++, T, R, sJ[2]))) break;
    T = i128_zero();
    stage(K3{}, G);
    if (!(ok = finish_stage<false, 2>(a, epoch++, T, R, sJ[3]))) break;
    T = i128_zero();
    emax = 0.0;
    stage(K4{}, G);
    if (!(ok = finish_stage<true, 2>(a, epoch++, T, R, sJ[0], NoOverlap{}, emax, sE))) break;
    ++natt;
    const double E = *sE;
    if (E <= a.tol2) {
      ++nacc;
      r = G.r1;
      double* t = X;
      X = Xn;
      Xn = t;
      if (E <= a.tol2 * (1.0 / 128.0) && 2.0 * h <= a.hmax) h = 2.0 * h;
      if (threadIdx.x < NV) sJsave[threadIdx.x] = sJ[0][threadIdx.x];
      if (last) break;
    } else {
      ++nrej;
      h = 0.5 * h;
      if (threadIdx.x < NV) sJ[0][threadIdx.x] = sJsave[threadIdx.x];
      if (h < a.hmin) {
        fail = 1;
        break;
      }
    }
    if (natt >= a.max_attempts) {
      fail = 1;
      break;
    }
    __syncthreads();
  }
  if (ok && X != (double*)a.X) {
    // the accepted state sits in the second buffer: copy this wavefront's rows back
    constexpr int nsc = (NF == 2) ? 3 : 6;
    double* D = (double*)a.X;
    for (long long row = gw; row < (long long)a.NS * a.NU; row += nw)
      for (int k = lane; k < a.NE; k += 64)
#pragma unroll
        for (int c = 0; c < nsc; ++c) D[row * a.NE + k + c * a.plane] = X[row * a.NE + k + c * a.plane];
  }
  if (err) __hip_atomic_fetch_or(a.sync + kSyncStatus, (unsigned)err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (ok && blockIdx.x == 0 && threadIdx.x == 0) {
    ctl[kCtlR] = (long long)as_bits(r);
    ctl[kCtlH] = (long long)as_bits(h);
    ctl[kCtlAcc] = nacc;
    ctl[kCtlRej] = nrej;
    ctl[kCtlAtt] = natt;
    ctl[kCtlFail] = fail;
    ctl[kCtlMTag] = -1;   // the state changed outside the fixed-step launches
    if (!fail) ctl[0] = a.total_steps;
  }
}

template __global__ void k_adaptive<2, true, kBlock>(StepArgs);
template __global__ void k_adaptive<2, false, kBlock>(StepArgs);
template __global__ void k_adaptive<3, true, kBlock>(StepArgs);
template __global__ void k_adaptive<3, false, kBlock>(StepArgs);
template __global__ void k_adaptive<2, true, kBlockSmall>(StepArgs);
template __global__ void k_adaptive<2, false, kBlockSmall>(StepArgs);
template __global__ void k_adaptive<3, true, kBlockSmall>(StepArgs);
template __global__ void k_adaptive<3, false, kBlockSmall>(StepArgs);

// --------------------------------------------------------------- batched models
// Many independent two-flavour models in one persistent launch (shared step grid).
// Each wavefront owns a contiguous, cost-balanced range of the concatenated rows, so it
// meets only a few models per stage.  Models are independent, so there is no grid barrier:
// a stage of a model waits only for the wavefronts that own rows of that model.
//
// Per model and epoch (barrier index) the wavefronts' exact 128-bit totals meet as in the
// single-model reduction, one level up: 6 sums of 3 chunks of 32 bits (the last signed and
// biased by 2^31; a total is below 2^93), each added with one atomic to a counted word (50
// bits of running sum, 14 bits of count: at most 2^14 wavefronts); the wavefront whose add
// completes the model's count publishes the running sum under a 14-bit epoch tag, and readers
// take differences of consecutive epochs.  Six published sets rotate: the final update of a
// step still reads the sums of stage 1 and those before it, five epochs back, and set
// e % 6 is rewritten at epoch e only after every wavefront of the model has added for e, that
// is after all it read up to its stage e.  A wavefront's add for e follows its reads for e - 1
// of every model, and waits point only to earlier epochs, so they cannot form a cycle.
// A grid barrier with arrival lines gathered by one block, a release flag and a read of
// the accumulators took 14 us per stage for 16 small models, of which the beams are 1 us.
constexpr unsigned long long kTag14 = 16383ull;

__device__ __forceinline__ unsigned long long* batch_pub(const BatchArgs& a, unsigned epoch, int m) {
  return a.acc + (size_t)a.nmodels * kAccWords + ((size_t)(epoch % kAccSets) * a.nmodels + m) * kPubWords;
}
// Add this wavefront's totals T of model m (lanes of fold_comp, fold_moment) for the epoch;
// n: the model's wavefronts.  sx: 12 words of the wavefront's LDS.
__device__ __forceinline__ void batch_publish(const BatchArgs& a, int m, unsigned n, unsigned epoch, const I128& T,
                                              int lane, unsigned long long* sx) {
  const int mo = fold_moment<3>(lane), co = fold_comp<3>(lane);
  __asm__ volatile("" ::: "memory");   // the wave's LDS operations complete in program order
  if (mo < 2 && co < 3) {
    sx[2 * (mo * 3 + co)] = T.lo;
    sx[2 * (mo * 3 + co) + 1] = (unsigned long long)T.hi;
  }
  __asm__ volatile("" ::: "memory");
  const int v = lane >> 2, l = lane & 3;
  if (lane < 24 && l < 3) {
    const unsigned long long w = sx[2 * v + (l == 2 ? 1 : 0)];
    const unsigned c = (l == 1) ? (unsigned)(w >> 32) : ((l == 2) ? (unsigned)w + 0x80000000u : (unsigned)w);
    const unsigned long long add = ((unsigned long long)c << 14) + 1ull, n0 = (unsigned long long)epoch * n;
    const unsigned long long sum = __hip_atomic_fetch_add(a.acc + (size_t)m * kAccWords + lane, add, __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT) + add;
    if ((((unsigned)sum - (unsigned)n0) & (unsigned)kTag14) == (n & (unsigned)kTag14))
      __hip_atomic_store(batch_pub(a, epoch, m) + lane, ((sum - n0 - n) & ~kTag14) | ((epoch + 1u) & kTag14),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}
// The moments J^(1..KIND) of model m for stage KIND of epoch `epoch` (NEWEST: only the last)
// into Jv.  Returns false if the wait was abandoned (time limit or abort).
template <int KIND, bool NEWEST>
__device__ __forceinline__ bool batch_moments(const BatchArgs& a, int m, unsigned n, unsigned epoch, double p2e0,
                                              double p2e1, int lane, double (*Jv)[6]) {
  constexpr int J0 = NEWEST ? KIND - 1 : 0;
  const int v = lane >> 2, l = lane & 3;
  const bool on = lane < 24 && l < 3;
  // words of the sums of epochs epoch - KIND - 1 + J0 (the difference's base; before epoch 0
  // a set not yet written), ..., epoch - 1
  unsigned long long w[KIND + 1 - J0];
#pragma unroll
  for (int i = 0; i <= KIND - J0; ++i) w[i] = 0ull;
  if (on)
#pragma unroll
    for (int i = 0; i < KIND - J0; ++i)
      w[i] = __hip_atomic_load(batch_pub(a, epoch + (unsigned)(kAccSets - (KIND + 1 - J0 - i)), m) + lane, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
  int ok = 1;
  if (on) {
    const unsigned long long* q = batch_pub(a, epoch - 1u, m) + lane;
    const unsigned long long tag = epoch & kTag14, t0 = wall_clock64();
    for (unsigned it = 1;; ++it) {
      const unsigned long long x = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      w[KIND - J0] = x;
      if ((x & kTag14) == tag) break;
      if ((it & 31u) == 0u && give_up(a.sync, a.cancel, t0, a.timeout_ticks, it)) {
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  if (__any(!ok)) return false;
  __asm__ volatile("" ::: "memory");
#pragma unroll
  for (int i = J0; i < KIND; ++i) {
    // (the fields are differences modulo 2^50; the last chunk less its bias is signed)
    unsigned long long d = ((w[i + 1 - J0] & ~kTag14) - (w[i - J0] & ~kTag14)) >> 14;
    if (l == 2) d -= (unsigned long long)n << 31;
    const unsigned long long c1 = dpp_u64<0x55>(d), c2 = dpp_u64<0xAA>(d);   // lanes 1, 2 of each four
    const I128 tot = i128_add(i128_add(I128{d, 0ll}, I128{c1 << 32, (long long)(c1 >> 32)}), I128{0ull, (long long)c2});
    if (on && l == 0) Jv[i][v] = i128_to_double(tot) * (v < 3 ? p2e0 : p2e1);
  }
  __asm__ volatile("" ::: "memory");
  return true;
}

// All blocks meet (a.lockstep): counted arrivals per die, published by the block that
// completes them, polled by every block.  i: the number of earlier meetings of the launch.
__device__ __forceinline__ bool batch_meet(const BatchArgs& a, unsigned i) {
  const int tid = threadIdx.x;
  int ok = 1;
  __syncthreads();
  if (tid == 0) {
    const unsigned c = blockIdx.x % kRedCopies, n = (gridDim.x + (kRedCopies - 1) - c) / kRedCopies;
    if (__hip_atomic_fetch_add(a.sync + kSyncStep + c * kLineWords, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u ==
        (i + 1u) * n)
      __hip_atomic_store(a.sync + kSyncStepPub + c * kLineWords, i + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (tid < kRedCopies && tid < (int)gridDim.x) {
    const unsigned long long t0 = wall_clock64();
    for (unsigned it = 1;; ++it) {
      if (__hip_atomic_load(a.sync + kSyncStepPub + tid * kLineWords, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= i + 1u)
        break;
      if ((it & 31u) == 0u && give_up(a.sync, a.cancel, t0, a.timeout_ticks, it)) {
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  return !__syncthreads_or(!ok);
}

// A wavefront's part of the batch: its rows, the first model it meets and, where all its rows
// are of that model and at most kRowKeep, kept = their number: such a wavefront keeps its
// rows' constants (keep_geo2, keep_nunu2) like those of the bulb model.
struct BatchWave {
  long long r0, r1;
  int m0, kept;
};
// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ long long uni(long long x) {
  return (long long)(((unsigned long long)(unsigned)uni((int)(x >> 32)) << 32) | (unsigned)uni((int)x));
}
// Rows are taken in groups of up to kGroup rows of one model: lane l first computes the
// constants of the group's row l (row_setup2, the arithmetic every lane of the row would
// otherwise repeat) into the wave's table rt, then the group's beams are streamed (group2).
constexpr int kGroup = 16;
__device__ __forceinline__ void batch_radii(const BatchArgs& a, long long n, const BatchModel* md, int lane, double* cb) {
  const double r0 = a.rs + (double)n * a.h;
  const double rm = r0 + 0.5 * a.h;
  const double r1 = a.rs + (double)(n + 1) * a.h;
  const double lam0 = md->lam0;
  __asm__ volatile("" ::: "memory");
  put_stage2(cb, lane, radial(a.R, a.ne_power, lam0, r0), radial(a.R, a.ne_power, lam0, rm),
             radial(a.R, a.ne_power, lam0, r1), Scales{md->s1, md->s0, md->p2e1, md->p2e0});
}
// Before a step: radial profiles and geometry of a keeping wavefront.
__device__ __forceinline__ void batch_prep(const BatchArgs& a, long long n, const BatchWave& W, int lane, double* cb,
                                           double* rt) {
  if (!W.kept) return;
  batch_radii(a, n, a.models + W.m0, lane, cb);
  keep_geo2(cb, a.h, lane, W.kept, rt);
}
template <int KIND>
__device__ __forceinline__ bool batch_stage(const BatchArgs& a, long long n, unsigned epoch, const BatchWave& W, int lane,
                                            double (*Jv)[6], double* cb, double* rt, unsigned long long* sx, int& err) {
  const double* J[4] = {Jv[0], Jv[1], Jv[2], Jv[3]};   // this wave's LDS block
  double enone = 0.0;
  int m = W.m0;
  for (long long row = W.r0; row < W.r1; ++m) {   // the models the range meets
    const BatchModel* md = a.models + m;
    const long long mrow0 = uni(md->row0), mbeam0 = uni(md->beam0);
    const int mNE = uni(md->NE), mNU = uni(md->NU);
    const unsigned nw = (unsigned)uni(a.wave_count[m]);
    const long long mend = min(W.r1, mrow0 + 2LL * mNU);
    const double* tab = a.tab + uni(md->tab0);
    I128 T = i128_zero();
    if (W.kept) {
      if constexpr (KIND >= 1)
        if (!batch_moments<KIND, true>(a, m, nw, epoch, cb[kC2Sc + 3], cb[kC2Sc + 2], lane, Jv)) return false;
      keep_nunu2<KIND>(cb, Jv, lane, W.kept, rt);
    } else {
      batch_radii(a, n, md, lane, cb);
      if constexpr (KIND >= 1)
        if (!batch_moments<KIND, false>(a, m, nw, epoch, cb[kC2Sc + 3], cb[kC2Sc + 2], lane, Jv)) return false;
    }
    while (row < mend) {
      const int gn = (int)min(mend - row, (long long)kGroup);
      if (!W.kept) {
        __asm__ volatile("" ::: "memory");   // the previous group's rows have read their blocks
        if (lane < gn) {
          const int lr = (int)(row + lane - mrow0);
          const int s = lr / mNU;
          const int j = lr - s * mNU;
          row_setup2<KIND, false>(u_of(j, mNU), a.h, cb, J, 0.0, 0.0, s, s ? -1.0 : 1.0, rt + lane * kRowP);
        }
        __asm__ volatile("" ::: "memory");
      }
      const long long gb0 = mbeam0 + (row - mrow0) * mNE;
      if (mNE <= kGroupMaxNE) {
        group2<KIND, false, kFoldRowsBatch, kRowP>(a.X, a.plane, gb0, mNE, gn, tab, cb, rt, a.renorm, lane, nullptr, T,
                                                   err);
      } else {
        for (int i = 0; i < gn; ++i)
          row2<KIND, false>(a.X, a.X, a.plane, gb0 + (long long)i * mNE, mNE, tab, cb, rt + i * kRowP, a.renorm, lane, T, err,
                            enone, nullptr);
      }
      row += gn;
    }
    batch_publish(a, m, nw, epoch, T, lane, sx);
  }
  return true;
}

// Four wavefronts per SIMD (128 VGPRs; the row groups' set-up spills, 264 bytes of scratch per
// lane, outside the chunk loop): the rows of a batch are short (50-400 energies), so a wave
// spends much of its time on row set-up and the first load of each row, which more
// wavefronts hide.  Measured on the 256-model batch before the chunks were streamed across
// rows: 4.35 ms per step at two wavefronts per SIMD, 3.52 at three, 3.19 at four; after it
// 2.65 at three and 2.53 at four.
template <int BS>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) k_batch2(BatchArgs a) {
  __shared__ double sJw[BS / 64][4][6];
  __shared__ double scb[BS / 64][kC2Size];
  __shared__ unsigned long long sxw[BS / 64][12];
  __shared__ double srt[BS / 64][kRowKeep * kRowP];   // each wave's row-constant table
  static_assert(kGroup <= kRowKeep, "one table for kept rows and groups");
  if (launch_aborted(a.sync)) return;
  // the wavefront index as a wave-uniform (scalar) value: the row indices, their divisions
  // and the row base offsets derived from it then live in scalar registers
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double (*Jv)[6] = sJw[wid];
  double *cb = scb[wid], *rt = srt[wid];
  unsigned long long* sx = sxw[wid];
  const long long w = (long long)blockIdx.x * (BS / 64) + wid;
  BatchWave W;
  W.r0 = min(max(uni(a.wave_row0[w]), 0LL), a.total_rows);
  W.r1 = min(max(uni(a.wave_row0[w + 1]), W.r0), a.total_rows);
  W.m0 = 0;
  W.kept = 0;
  if (W.r0 < W.r1) {
    int lo = 0, hi = a.nmodels - 1;   // the first row's model
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (a.models[mid].row0 <= W.r0) lo = mid; else hi = mid - 1;
    }
    W.m0 = uni(lo);
    const BatchModel* md = a.models + W.m0;
    if (W.r1 <= uni(md->row0) + 2LL * uni(md->NU) && W.r1 - W.r0 <= kRowKeep) {
      W.kept = (int)(W.r1 - W.r0);
      if (lane < W.kept) {
        const int lr = (int)(W.r0 + lane - md->row0), s = lr / md->NU;
        rt[lane * kRowP + kRowU] = u_of(lr - s * md->NU, md->NU);
        rt[lane * kRowP + kRowS] = (double)s;
        rt[lane * kRowP + kRowA] = s ? -1.0 : 1.0;   // two tracked species: row s is anti iff s = 1
      }
    }
  }
  const long long step0 = uni(*a.step_ctl);
  const long long nsteps = max(0LL, min(a.nsteps, a.total_steps - step0));
  unsigned epoch = 0;
  int err = 0;
  batch_prep(a, step0, W, lane, cb, rt);
  bool ok = batch_stage<0>(a, step0, epoch++, W, lane, Jv, cb, rt, sx, err);
  for (long long n = step0; ok && n < step0 + nsteps; ++n) {
    ok = batch_stage<1>(a, n, epoch++, W, lane, Jv, cb, rt, sx, err) &&
         batch_stage<2>(a, n, epoch++, W, lane, Jv, cb, rt, sx, err) &&
         batch_stage<3>(a, n, epoch++, W, lane, Jv, cb, rt, sx, err) &&
         batch_stage<4>(a, n, epoch++, W, lane, Jv, cb, rt, sx, err);
    // (a.lockstep is uniform over the grid, ok is not: a wavefront that gave up still meets the
    // others of its block, which read the abort word at their next wait)
    if (a.lockstep) {
      const bool met = batch_meet(a, (unsigned)(n - step0));
      ok = ok && met;
      if (__syncthreads_or(!ok)) ok = false;
    }
    batch_prep(a, n + 1, W, lane, cb, rt);   // while the models' other wavefronts finish
  }
  // the block that ends last moves the step counter (every block read it at its start)
  if (launch_ends(a.sync, err, ok) && threadIdx.x == 0) {
    *a.step_ctl = step0 + nsteps;
    if (a.host) put_host(a.host, a.sync, step0 + nsteps);
  }
}
template __global__ void k_batch2<kBlock>(BatchArgs);
template __global__ void k_batch2<kBlockSmall>(BatchArgs);

// ----------------------------------------------------------------- small kernels
// The state was set or reset: the step, and no moments left for the next launch.
__global__ void k_set_step(long long* step_ctl, long long step) {
  step_ctl[0] = step;
  step_ctl[kCtlMTag] = -1;
}
// The status word and the device step counter into host memory (one small write the host
// reads after synchronising, instead of two copies).
__global__ void k_status_out(const unsigned int* sync, const long long* step_ctl, long long* host) {
  __hip_atomic_store(host, (long long)sync[kSyncStatus], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(host + 1, step_ctl[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// Target of a group of windowed launches: k more steps from the device step counter.
__global__ void k_set_target(long long* step_ctl, long long k, long long total) {
  step_ctl[1] = min(step_ctl[0] + k, total);
}

// Clear the first `words` barrier and reduction words (those the launch uses), and nacc
// accumulators at acc (batches), before a persistent launch (keep_status: keep the status bits of earlier launches of the same call).  If the host has set the model's
// cancel word (fine-grained host memory; nullptr: none), the abort word is set instead of
// cleared, with status bit 2, so that the next persistent launch returns at once.
__global__ void k_zero_sync(unsigned int* sync, int keep_status, const unsigned* cancel, int words,
                            unsigned long long* acc, long long nacc) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nacc; i += (long long)gridDim.x * blockDim.x)
    acc[i] = 0ull;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < words; i += gridDim.x * blockDim.x) {
    if (i == kSyncStatus) continue;   // written with the abort word
    if (i == kSyncAbort) {
      const unsigned c =
          cancel ? __hip_atomic_load(cancel, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) : 0u;
      const unsigned st = keep_status ? sync[kSyncStatus] : 0u;
      sync[kSyncAbort] = c ? 1u : 0u;
      sync[kSyncStatus] = st | (c ? 4u : 0u);
      continue;
    }
    sync[i] = 0u;
  }
}

// Initial flavour eigenstates (Sec. 3.4): species row s = b / per_species is born in
// flavour s % nfl (nfl = 1 when only electron-born beams are tracked); 2f: P = (0, 0, +-1),
// 3f: psi = the unit vector of that flavour.
template <typename ST>
__global__ void k_init(ST* X, long long nb, long long plane, int nsc, long long per_species, int nfl,
                       long long* step_ctl) {
  const long long b = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (b == 0) {   // step 0, no moments left for the next launch
    step_ctl[0] = 0;
    step_ctl[kCtlMTag] = -1;
  }
  if (b >= nb) return;
  const int fl = (int)((b / per_species) % nfl);
  for (int c = 0; c < nsc; ++c) {
    ST v = (ST)0;
    if (nsc == 3) v = (c == 2) ? (ST)(fl == 0 ? 1 : -1) : (ST)0;
    else v = (c == 2 * fl) ? (ST)1 : (ST)0;
    X[b + c * plane] = v;
  }
}
template __global__ void k_init<double>(double*, long long, long long, int, long long, int, long long*);
template __global__ void k_init<float>(float*, long long, long long, int, long long, int, long long*);

template <typename ST>
__global__ void k_read_pee(const ST* X, long long nb, long long plane, int nsc, double* out) {
  const long long b = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nb) return;
  if (nsc == 3) {
    out[b] = 0.5 * (1.0 + (double)X[b + 2 * plane]);
  } else {
    const double re = (double)X[b], im = (double)X[b + plane];
    out[b] = fma(re, re, im * im);
  }
}
template __global__ void k_read_pee<double>(const double*, long long, long long, int, double*);
template __global__ void k_read_pee<float>(const float*, long long, long long, int, double*);

// State exchange with FP64 [comp][beam] planes (dir 0: state -> out, 1: in -> state, and the
// step counter, as k_set_step).
template <typename ST>
__global__ void k_state_xfer(ST* X, long long nb, long long plane, int nsc, double* buf, int dir, long long* step_ctl,
                             long long step) {
  const long long b = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (dir == 1 && b == 0) {
    step_ctl[0] = step;
    step_ctl[kCtlMTag] = -1;
  }
  if (b >= nb) return;
  for (int c = 0; c < nsc; ++c) {
    if (dir == 0) buf[c * nb + b] = (double)X[b + c * plane];
    else X[b + c * plane] = (ST)buf[c * nb + b];
  }
}
template __global__ void k_state_xfer<double>(double*, long long, long long, int, double*, int, long long*, long long);
template __global__ void k_state_xfer<float>(float*, long long, long long, int, double*, int, long long*, long long);

}  // namespace nb
