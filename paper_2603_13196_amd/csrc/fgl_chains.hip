// Device-resident slice-sampling chains for batched nested sampling.
//
// One call advances n hit-and-run slice chains, each by `steps` steps under
// the constraint lnL > lnL* inside the prior box (the replacement step of
// nested slice sampling, Tutt et al. Sec. 3.1.2 and 3.1.3).  A round is the
// model's row preparation and likelihood kernel over the n proposal rows,
// then k_chain_step, one wavefront per chain, which
//   * forms each row's lnL from the likelihood kernel's partial sums, in the
//     order and arithmetic of the library's finalize (so it equals what
//     fgl_loglike_batch returns for that row, bit for bit),
//   * advances the chain's state machine:
//       stepping out:  the interval ends move out by one unit (in the
//                      geometry whitened by the caller's Cholesky factor)
//                      while they are inside the constrained region;
//       shrinking:     a uniform point of the interval is accepted if
//                      inside, otherwise the interval is cut at it,
//   * and writes the chain's next proposal row.
// The lanes of a chain's wavefront share its coordinates (directions,
// Cholesky product, proposal) and its lnL reduction.  A chain that has
// finished its steps keeps its point and proposes nothing new.  Rounds are
// captured once into a hipGraph (R rounds per graph) and replayed; the host
// reads the chains' stages after each replay and stops when every chain is
// done.
//
// Small models (the thin form) leave that scheme: k_chain_run keeps a chain in
// one workgroup for all its rounds, so a round costs no launch.
//
// Coordinates: the sampler works in z = [beta.., A, nu21, w, log sigma] (or
// [beta.., log sigma] without the 21-cm term), uniform over the box; the
// likelihood row is z with its last entry exponentiated.
//
// Random numbers: Philox4x32-10 (Salmon, Moraes, Dror and Shaw, "Parallel
// random numbers: as easy as 1, 2, 3", SC 2011), keyed by the seed, with the
// chain index and a per-chain counter as the counter block; the counters
// start at zero when the engine is created and keep counting across calls,
// so no draw is ever repeated.  Uniforms take 53 bits, normals come from the
// Box-Muller transform.
#include "fgl_host.h"
#include "fgl_philox.h"
#include "fgl_pow2.h"
#include "fgl_wave.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

namespace fgl {

namespace {

constexpr int kLeft = 0, kRight = 1, kShrink = 2, kDone = 3;
constexpr int kMaxExpand = 64;
constexpr int kRoundsPerGraph = 32;

struct ChainState {
  int n, P;
  double* x;        // [n][P] current points (sampler coordinates)
  double* dir;      // [n][P] step directions
  double* a;        // [n] interval, in units of dir
  double* b;
  double* t;        // [n] last proposal's position
  double* lx;       // [n] lnL at x
  int* stage;       // [n]
  int* done;        // [n] finished steps
  int* expand;      // [n] expansions of the current side
  int* evals;       // [n] in-box proposals evaluated
  long long* rounds;   // [n] rounds taken (k_chain_run)
  unsigned long long* ctr;   // [n] Philox counter
  double* theta;    // [n][P] likelihood rows of the proposals
  int* inbox;       // [n]
  double* lnl;      // [n] likelihood of the proposals
  const double* chol;  // [P][P] lower-triangular whitening factor
  const double* lo;    // [P]
  const double* hi;    // [P]
  const double* lstar; // the constraint lnL > *lstar (device memory, so a
                       // captured graph stays valid across iterations)
  unsigned long long seed;
  int steps;
  // the likelihood's row records and transposed indices of the proposals,
  // written by the chain kernels themselves (the model's N = NA' NB regions,
  // NA' = max(NA, 1), betaRows = 32 KC transposed rows)
  RowParams* rows;
  double* betaT;
  double* offT;
  int Bpad, N, NA, NB, betaRows;
  unsigned flags;
};

// Two uniforms in [0, 1) with 53 random bits each, from Philox block c of
// chain i.
__device__ __forceinline__ void uniform2(const ChainState& s, int i, unsigned long long c, double& u0,
                                double& u1) {
  uint32_t v[4] = {(uint32_t)c, (uint32_t)(c >> 32), (uint32_t)i, 0x5eed5eedu};
  philox4x32(v, (uint32_t)s.seed, (uint32_t)(s.seed >> 32));
  const uint64_t a = ((uint64_t)v[0] << 32 | v[1]) >> 11;
  const uint64_t b = ((uint64_t)v[2] << 32 | v[3]) >> 11;
  u0 = (double)a * 0x1.0p-53;
  u1 = (double)b * 0x1.0p-53;
}

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
  return v;
}

constexpr int kMaxP = 160;            // parameters a chain's LDS direction holds
constexpr int kWaves = 4;             // chains (wavefronts) per workgroup

// Per-chain scalars, held in registers (uniform across the wavefront) while a
// kernel works on the chain and written back by lane 0.
struct Scal {
  double a, b, t, lx;
  int stage, done, expand, evals;
  unsigned long long ctr;
};

__device__ inline Scal load_scal(const ChainState& s, int i) {
  return Scal{s.a[i], s.b[i], s.t[i], s.lx[i], s.stage[i], s.done[i], s.expand[i], s.evals[i],
              s.ctr[i]};
}

__device__ inline void store_scal(const ChainState& s, int i, const Scal& c, int lane) {
  if (lane != 0) return;
  s.a[i] = c.a;
  s.b[i] = c.b;
  s.t[i] = c.t;
  s.lx[i] = c.lx;
  s.stage[i] = c.stage;
  s.done[i] = c.done;
  s.expand[i] = c.expand;
  s.evals[i] = c.evals;
  s.ctr[i] = c.ctr;
}

// A chain's coordinates: the lane holds entries lane + 64 q, q < Q, of the
// point and of the step's direction.
template <int Q>
struct Coord {
  double x[Q], d[Q];
};
constexpr int kQ = 3;
static_assert(kMaxP <= kQ * 64, "three entries per lane");

template <int Q>
__device__ inline void load_coord(Coord<Q>& v, const double* x, const double* d, int P, int lane) {
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int k = lane + 64 * q;
    v.x[q] = k < P ? x[k] : 0.0;
    v.d[q] = k < P && d ? d[k] : 0.0;
  }
}

template <int Q>
__device__ inline void store_coord(const double (&v)[Q], double* to, int P, int lane) {
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (lane + 64 * q < P) to[lane + 64 * q] = v[q];
}

// A new slice step: direction uniform on the unit sphere in whitened
// coordinates, mapped by the Cholesky factor; unit interval at a random
// offset around the current point.  Lane k/2 draws the normal pair of
// coordinates k, k + 1 (Philox block ctr + k/2); the pairs go through LDS (u)
// so that lane j can form row j of the Cholesky product.
template <int Q>
__device__ __forceinline__ void new_step(const ChainState& s, int i, Scal& c, int lane, double* u,
                                         Coord<Q>& v) {
  const int P = s.P, np = (P + 1) / 2;
  double nrm = 0.0;
  // the direction needs randomness, not precision: the Box-Muller pairs are
  // formed with the FP32 hardware transcendentals
  for (int pr = lane; pr < np; pr += 64) {
    double u0, u1;
    uniform2(s, i, c.ctr + pr, u0, u1);
    const float w = (float)(1.0 - u0);                  // in (0, 1]
    const float rad = __builtin_sqrtf(-2.0f * __logf(w));
    const float ang = 6.2831853f * (float)u1;
    const double z0 = (double)(rad * __cosf(ang)), z1 = (double)(rad * __sinf(ang));
    u[2 * pr] = z0;
    nrm += z0 * z0;
    if (2 * pr + 1 < P) {
      u[2 * pr + 1] = z1;
      nrm += z1 * z1;
    }
  }
  nrm = wave_sum(nrm);
  wave_sync();                                          // u written by all lanes
  const double inv = 1.0 / sqrt(nrm);
#pragma unroll
  for (int q = 0; q < Q; ++q) {                         // dir = L u, L lower triangular
    const int j = lane + 64 * q;
    if (j >= P) continue;
    double acc = 0.0;
    for (int k = 0; k <= j; ++k) acc += s.chol[(size_t)j * P + k] * u[k];
    v.d[q] = acc * inv;
  }
  wave_sync();                                          // u read by all lanes
  double r, unused;
  uniform2(s, i, c.ctr + np, r, unused);
  c.ctr += np + 1;
  c.a = -r;
  c.b = 1.0 - r;
}

// The row record and the transposed spectral indices (and log2 alpha) of
// likelihood row i, from the row's entries held by the chain's wavefront
// (v[q] is entry lane + 64 q), with the row-preparation kernel's rules:
// finite entries, |beta| <= 64, alpha in [2^-32, 2^32], sigma > 0 and
// w > 0; extremes of beta and log2 alpha; fills of the row's minimum for
// padded regions (zero for an invalid row).
__device__ void prep_row(const ChainState& s, int i, int lane, const double (&v)[3]) {
  const int P = s.P, NB = s.NB, NA = s.NA;
  const bool no21 = s.flags & 1u;
  int ok = 1;
  double bmin = INFINITY, bmax = -INFINITY, omin = INFINITY, omax = -INFINITY;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int k = lane + 64 * q;
    if (k < P) {
      const double x = v[q];
      ok = ok && isfinite(x);
      if (k < NB) {
        ok = ok && fabs(x) <= 64.0;
        bmin = fmin(bmin, x);
        bmax = fmax(bmax, x);
      } else if (k < NB + NA) {
        ok = ok && x >= 0x1p-32 && x <= 0x1p32;
        const double o = log2(x);
        omin = fmin(omin, o);
        omax = fmax(omax, o);
      }
    }
  }
  ok = __builtin_amdgcn_ballot_w64(!ok) == 0;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    bmin = fmin(bmin, __shfl_xor(bmin, m));
    bmax = fmax(bmax, __shfl_xor(bmax, m));
    omin = fmin(omin, __shfl_xor(omin, m));
    omax = fmax(omax, __shfl_xor(omax, m));
  }
  // entry k of the row (k may differ between lanes; every lane takes part)
  auto entry = [&](int k) {
    const double a0 = __shfl(v[0], k & 63), a1 = __shfl(v[1], k & 63);
    const double a2 = __shfl(v[2], k & 63);
    return k < 64 ? a0 : (k < 128 ? a1 : a2);
  };
  const double sig = entry(P - 1);
  const double wd = entry(no21 ? P - 1 : P - 2);
  const double amp = entry(no21 ? P - 1 : P - 4);
  const double nu0 = entry(no21 ? P - 1 : P - 3);
  if (ok) {
    ok = sig > 0.0;
    if (!no21) ok = ok && wd > 0.0;
  }
  if (!ok) bmin = bmax = 0.0;
  if (!ok || NA == 0) omin = omax = 0.0;
  if (lane == 0) {
    RowParams rp;
    rp.valid = ok ? 1 : 0;
    rp.pad = 0;
    rp.A = 0.0;
    rp.nu0 = 0.0;
    rp.inv_w = 1.0;
    rp.sigma = 1.0;
    rp.t21 = no21 ? 0.0 : 1.0;
    if (ok) {
      rp.sigma = sig;
      if (!no21) {
        rp.A = amp;
        rp.nu0 = nu0;
        rp.inv_w = 1.0 / wd;
      }
    }
    rp.bmin = bmin;
    rp.bmax = bmax;
    rp.omin = omin;
    rp.omax = omax;
    s.rows[i] = rp;
  }
  const int nq = (s.betaRows + 63) / 64;
  for (int q = 0; q < nq; ++q) {
    const int r = lane + 64 * q;
    const int ia = r / NB, jb = r - ia * NB;
    const bool real = ok && r < s.N;
    const double bv = entry(min(jb, P - 1));
    const double av = NA > 0 ? entry(min(NB + ia, P - 1)) : 1.0;
    if (r < s.betaRows) {
      s.betaT[(size_t)r * s.Bpad + i] = real ? bv : bmin;
      if (NA > 0) s.offT[(size_t)r * s.Bpad + i] = real ? log2(av) : omin;
    }
  }
}

// The chain's next likelihood row: the proposal x + t dir when it is inside
// the box, else (and for a finished chain) the chain's point itself, whose
// result is ignored.  The last coordinate is log sigma.  The row's record
// and transposed indices are prepared here too.
__device__ void propose(const ChainState& s, int i, Scal& c, int lane, const Coord<kQ>& y) {
  const int P = s.P;
  double* th = s.theta + (size_t)i * P;
  double v[3] = {0.0, 0.0, 0.0};
  if (c.stage == kDone) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int k = lane + 64 * q;
      if (k < P) {
        v[q] = k == P - 1 ? exp(y.x[q]) : y.x[q];
        th[k] = v[q];
      }
    }
    if (lane == 0) s.inbox[i] = 0;
    prep_row(s, i, lane, v);
    return;
  }
  double t;
  if (c.stage == kShrink) {
    double u, unused;
    uniform2(s, i, c.ctr, u, unused);
    c.ctr += 1;
    t = c.a + (c.b - c.a) * u;
  } else {
    t = c.stage == kLeft ? c.a : c.b;
  }
  c.t = t;
  int out = 0;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int k = lane + 64 * q;
    if (k >= P) continue;
    const double p = y.x[q] + t * y.d[q];
    out |= !((p >= s.lo[k]) & (p <= s.hi[k]));
  }
  const bool in = __builtin_amdgcn_ballot_w64(out != 0) == 0;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int k = lane + 64 * q;
    if (k < P) {
      const double p = in ? y.x[q] + t * y.d[q] : y.x[q];
      v[q] = k == P - 1 ? exp(p) : p;
      th[k] = v[q];
    }
  }
  if (lane == 0) s.inbox[i] = in ? 1 : 0;
  prep_row(s, i, lane, v);
}

template <int Q>
__device__ __forceinline__ void finish_step(const ChainState& s, int i, Scal& c, int lane,
                                            double* u, Coord<Q>& y) {
  c.done += 1;
  const bool end = c.done >= s.steps;
  if (!end) new_step(s, i, c, lane, u, y);
  c.stage = end ? kDone : kLeft;
  c.expand = 0;
}

// One transition of the state machine after the last proposal, x + t d
// (inside the box or not), evaluated to lp; true when it ends the step.
template <int Q>
__device__ __forceinline__ bool advance(Scal& c, double lp, bool in, double lstar, Coord<Q>& y) {
  // NaN and -inf are outside (ballots keep the state's branches scalar, selects
  // keep the state in registers)
  const bool inside = in && __builtin_amdgcn_ballot_w64(lp > lstar) != 0;
  const bool left = c.stage == kLeft, out = c.stage != kShrink;   // stepping out
  const bool grow = out && inside && c.expand < kMaxExpand;
  const bool take = !out && inside;                // shrinking: accepted
  const bool cut = !out && !inside, below = c.t < 0.0;
  c.evals = in ? c.evals + 1 : c.evals;
  c.a = grow && left ? c.a - 1.0 : cut && below ? c.t : c.a;
  c.b = grow && !left ? c.b + 1.0 : cut && !below ? c.t : c.b;
  c.expand = grow ? c.expand + 1 : 0;
  c.stage = out && !grow ? (left ? kRight : kShrink) : c.stage;
  c.lx = take ? lp : c.lx;
  if (take) {
#pragma unroll
    for (int q = 0; q < Q; ++q) y.x[q] = y.x[q] + c.t * y.d[q];   // the proposal, exactly
  }
  // an interval shrunk to nothing (a likelihood plateau at lnL*): keep the point
  return take || (cut && __builtin_amdgcn_ballot_w64(c.b - c.a < 1e-12) != 0);
}

// The likelihood kernel's partial sums of row b, reduced as the library's
// finalize does (sixteen strided sums, then an xor tree).
struct RowSums {
  const double* partial;
  const RowParams* rows;
  int ngroup, Bpad;
  double nFT, chi0;
};

__device__ inline double sum16(double acc) {
  acc += __shfl_xor(acc, 8);
  acc += __shfl_xor(acc, 4);
  acc += __shfl_xor(acc, 2);
  acc += __shfl_xor(acc, 1);
  return __shfl(acc, 0);
}

__device__ inline double row_lnl(const RowSums& r, int b, int lane) {
  double acc = 0.0;
  if (lane < 16)
    for (int c = lane; c < r.ngroup; c += 16) acc += r.partial[(size_t)c * r.Bpad + b];
  acc = sum16(acc);
  const RowParams rp = r.rows[b];
  if (!rp.valid) return -INFINITY;
  const double s2 = rp.sigma * rp.sigma;
  return -0.5 * (acc + r.chi0) / s2 - 0.5 * r.nFT * log(2.0 * M_PI * s2);
}

// Start: copy the starting points, draw every chain's first step and write
// its first proposal.
__global__ __launch_bounds__(64 * kWaves) void k_chain_start(ChainState s, const double* x0,
                                                             const double* l0) {
  __shared__ double s_u[kWaves][kMaxP];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i = blockIdx.x * kWaves + wv;
  if (i >= s.n) return;
  const int P = s.P;
  Coord<kQ> y;
  load_coord(y, x0 + (size_t)i * P, nullptr, P, lane);
  store_coord(y.x, s.x + (size_t)i * P, P, lane);
  Scal c = load_scal(s, i);             // ctr keeps counting across calls: fresh numbers
  c.lx = l0[i];
  c.done = -1;                          // the first step starts as any other
  c.evals = 0;
  c.t = 0.0;
  finish_step(s, i, c, lane, s_u[wv], y);
  store_coord(y.d, s.dir + (size_t)i * P, P, lane);
  propose(s, i, c, lane, y);
  store_scal(s, i, c, lane);
}

// One round's update from the likelihood of the last proposals, then the
// next proposal.
__global__ __launch_bounds__(64 * kWaves) void k_chain_step(ChainState s, RowSums rs) {
  __shared__ double s_u[kWaves][kMaxP];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i = blockIdx.x * kWaves + wv;
  if (i >= s.n) return;
  const double lstar = *s.lstar;
  Scal c = load_scal(s, i);
  if (c.stage == kDone) return;
  const double lp = row_lnl(rs, i, lane);
  if (lane == 0) s.lnl[i] = lp;
  Coord<kQ> y;
  load_coord(y, s.x + (size_t)i * s.P, s.dir + (size_t)i * s.P, s.P, lane);
  if (advance(c, lp, s.inbox[i] != 0, lstar, y)) {
    finish_step(s, i, c, lane, s_u[wv], y);
    store_coord(y.x, s.x + (size_t)i * s.P, s.P, lane);
    store_coord(y.d, s.dir + (size_t)i * s.P, s.P, lane);
  }
  propose(s, i, c, lane, y);
  store_scal(s, i, c, lane);
}

// ---------------------------------------------------------------------------
// small models: a chain's rounds inside one workgroup
//
// A round of the launches above is two dependent kernels over a few dozen
// rows, so a call of 70 chains (14 parameters, 70 steps, ~2200 rounds) is
// launch latency: 12.5 us a round.  Chains never exchange anything, so here
// one workgroup owns a chain and runs its rounds in a loop.  What bounds a
// round is then the latency of its serial chain, and the waves split it:
//   wave 0       the state machine (the code above), its coordinates in
//                registers, and sigma = exp(log sigma) with ln(2 pi sigma^2)
//                while the channels are evaluated;
//   wave 1       the uniform a following shrink step would draw;
//   waves 2 ..   one channel per lane of the thin kernel's model, the same
//                operations in the same order, so lnL is bitwise what the
//                library returns.
// Proposals outside the box or invalid cost no evaluation.  Two barriers a
// round; a launch ends after kRunRounds rounds (state saved) so that no
// launch lasts long.

constexpr int kRunRounds = 4096;        // rounds of one k_chain_run launch (5-10 ms)
constexpr int kRunMaxThreads = 512;
constexpr int kRunHelpers = 128;        // threads of waves 0 and 1
constexpr int kRunMaxP = 64;            // one coordinate per lane (thin models have at most 37)

// The thin model laid out for one lane per channel: K as [T][NT/4][Fp] quads
// of regions and D as [T][Fp], Fp = F rounded up to 64.
struct RunModel {
  const float4* k;
  const double* d;
  int Fp;
};

// k and d of a RunModel from the thin kernel's K [F][T][NT] and D [F][TT 32].
__global__ __launch_bounds__(256) void k_run_layout(DevModel m, int Fp, float4* __restrict__ k,
                                                    double* __restrict__ d) {
  const int f = blockIdx.x * blockDim.x + threadIdx.x, t = blockIdx.y, nq = m.NT / 4;
  if (f >= Fp) return;
  for (int q = 0; q < nq; ++q)
    k[((size_t)t * nq + q) * Fp + f] =
        f < m.F ? reinterpret_cast<const float4*>(m.kthin)[((size_t)f * m.T + t) * nq + q]
                : make_float4(0.f, 0.f, 0.f, 0.f);
  d[(size_t)t * Fp + f] = f < m.F ? m.D[(size_t)f * m.TT * 32 + t] : 0.0;
}

// Partials per row, padded so that sixteen lanes read four each at a time.
__host__ __device__ inline int run_parts(int F) { return ((F + 3) / 4 + 63) / 64 * 64; }

// dynamic LDS of k_chain_run: the partials, residuals [T][E]
inline size_t run_lds(int T, int E, int F) {
  return ((size_t)T * E + run_parts(F)) * sizeof(double);
}

// v of the lane `by` above, within rows of sixteen lanes (0 past the row)
template <int by>
__device__ inline double row_down(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x100 | by, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x100 | by, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// v of one lane (the same in every lane's call)
__device__ inline double any_lane(double v, int of) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, of);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), of);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// ONE: one time bin and a lane for every channel, whose constants then stay in
// registers over the rounds.
template <int NT, bool AB, bool ONE>
__global__ __launch_bounds__(kRunMaxThreads) void k_chain_run(ChainState s, DevModel m,
                                                              RunModel rm, double nFT, int first,
                                                              const double* __restrict__ x0,
                                                              const double* __restrict__ l0,
                                                              long long limit) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double s_u[64], s_v[64], s_t64[64];
  __shared__ double s_unif;
  __shared__ unsigned long long s_ctr;
  __shared__ int s_go;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, E = blockDim.x - kRunHelpers;
  const int i = blockIdx.x, P = s.P, F = m.F, T = m.T;
  const int nparts = run_parts(F);
  double* s_part = reinterpret_cast<double*>(smem);
  double* s_r = s_part + nparts;                    // [T][E]
  const bool no21 = s.flags & 1u;
  init_t64(s_t64);
  for (int k = tid; k < nparts; k += blockDim.x) s_part[k] = 0.0;

  if (wave == 0) {
    const double lstar = *s.lstar;
    const double lo = lane < P ? s.lo[lane] : -1.0, hi = lane < P ? s.hi[lane] : 1.0;
    const bool is_beta = lane < s.NB, is_alpha = !is_beta && lane < s.NB + s.NA;
    const bool is_width = !no21 && lane == P - 2;
    Coord<1> y;
    Scal c = load_scal(s, i);
    long long rounds = 0;
    bool over = first != 0;                         // a step is to begin
    if (first) {
      load_coord(y, x0 + (size_t)i * P, nullptr, P, lane);
      c.lx = l0[i];
      c.done = -1;                                  // the first step starts as any other
      c.evals = 0;
      c.t = 0.0;
    } else {
      load_coord(y, s.x + (size_t)i * P, s.dir + (size_t)i * P, P, lane);
      rounds = s.rounds[i];
    }
    unsigned long long drawn = ~0ull;               // counter whose uniform wave 1 formed
    double lp = -INFINITY;
    bool in = false, made = false;                  // made: a proposal has its lp
    for (;;) {
      if (made) {
        over = advance(c, lp, in, lstar, y);
        ++rounds;
      }
      if (over) finish_step(s, i, c, lane, s_u, y);
      over = false;
      if (c.stage == kDone || rounds >= limit) break;
      made = true;
      // the next proposal's position, as propose() draws it
      if (c.stage == kShrink) {
        double u = s_unif, unused;
        if (drawn != c.ctr) uniform2(s, i, c.ctr, u, unused);
        c.ctr += 1;
        c.t = c.a + (c.b - c.a) * u;
      } else {
        c.t = c.stage == kLeft ? c.a : c.b;
      }
      // its row, but for sigma, into LDS (entries past P are 0, inside their
      // box of -1 .. 1; inside the box entries are finite)
      const double p = y.x[0] + c.t * y.d[0];
      const bool out = !((p >= lo) & (p <= hi));
      const bool bad = (is_beta & !(fabs(p) <= 64.0)) | (is_width & !(p > 0.0)) |
                       (is_alpha & !(p >= 0x1p-32 && p <= 0x1p32));
      // amplitude scales as the exponents they add: 64 log2 alpha
      if (lane < P) s_v[lane] = AB && is_alpha ? 64.0 * log2(p) : p;
      in = __builtin_amdgcn_ballot_w64(out) == 0;
      lp = -INFINITY;
      if (!in || __builtin_amdgcn_ballot_w64(bad) != 0) continue;   // nothing to evaluate
      const double last = any_lane(p, P - 1);
      drawn = c.ctr;
      if (lane == 0) {
        s_ctr = drawn;
        s_go = 1;
      }
      __syncthreads();
      const double sigma = exp(last), s2 = sigma * sigma;
      const double ln = log(2.0 * M_PI * s2);
      __syncthreads();
      double acc = 0.0;
      for (int g = 0; g < nparts; g += 64) {        // group order within a sum; padding is 0
        const double* at = s_part + g + (lane & 15);
        const double v0 = at[0], v1 = at[16], v2 = at[32], v3 = at[48];
        acc += v0;
        acc += v1;
        acc += v2;
        acc += v3;
      }
      acc += row_down<8>(acc);
      acc += row_down<4>(acc);
      acc += row_down<2>(acc);
      acc += row_down<1>(acc);
      acc = any_lane(acc, 0);
      if (isfinite(sigma) && sigma > 0.0) lp = -0.5 * (acc + 0.0) / s2 - 0.5 * nFT * ln;
    }
    if (lane == 0) s_go = 0;
    __syncthreads();
    store_coord(y.x, s.x + (size_t)i * P, P, lane);
    store_coord(y.d, s.dir + (size_t)i * P, P, lane);
    store_scal(s, i, c, lane);
    if (lane == 0) s.rounds[i] = rounds;
    return;
  }

  if (wave == 1) {
    for (;;) {
      __syncthreads();
      if (!s_go) return;
      double u, unused;
      uniform2(s, i, s_ctr, u, unused);
      s_unif = u;
      __syncthreads();
    }
  }

  const int id = tid - kRunHelpers;                 // channel f0 + id of every pass
  const int own = min(id, F - 1);
  const double nl0 = m.nl64[own], nu0 = m.nu[own], d0 = rm.d[own];
  float k0[NT];
  if constexpr (ONE) {
#pragma unroll
    for (int q = 0; q < NT / 4; ++q) {
      const float4 k = rm.k[(size_t)q * rm.Fp + own];
      k0[4 * q] = k.x;
      k0[4 * q + 1] = k.y;
      k0[4 * q + 2] = k.z;
      k0[4 * q + 3] = k.w;
    }
  }
  for (;;) {
    __syncthreads();
    if (!s_go) return;
    const double A = no21 ? 0.0 : s_v[P - 4], c21 = no21 ? 0.0 : s_v[P - 3];
    const double inv_w = no21 ? 1.0 : 1.0 / s_v[P - 2];
    for (int f0 = 0; f0 < F; f0 += E) {
      const int f = f0 + id;
      if (f < F) {
        const double nl = ONE ? nl0 : m.nl64[f];
        const double z = ((ONE ? nu0 : m.nu[f]) - c21) * inv_w;
        const double cc = m.t_cmb + A * exp(-0.5 * z * z);
        double Pw[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          // regions past N have K = 0: any finite power will do
          const int jr = min(j, s.N - 1), ia = AB ? jr / s.NB : 0, jb = AB ? jr - ia * s.NB : jr;
          const double b = s_v[jb];
          Pw[j] = pow2_64(AB ? fma(b, nl, s_v[s.NB + ia]) : b * nl, s_t64, m);
        }
        if constexpr (ONE) {
          double msum = 0.0;
#pragma unroll
          for (int j = 0; j < NT; ++j) msum = fma((double)k0[j], Pw[j], msum);
          s_r[id] = (d0 - cc) - msum;
        } else {
          // U bins at a time, so that their loads and chains overlap
          constexpr int U = NT <= 8 ? 8 : NT <= 12 ? 4 : 2;
          for (int t0 = 0; t0 < T; t0 += U) {
            float4 k[U][NT / 4];
            double dv[U], ms[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const size_t t = min(t0 + u, T - 1);
#pragma unroll
              for (int q = 0; q < NT / 4; ++q) k[u][q] = rm.k[(t * (NT / 4) + q) * rm.Fp + f];
              dv[u] = rm.d[t * rm.Fp + f];
              ms[u] = 0.0;
            }
#pragma unroll
            for (int q = 0; q < NT / 4; ++q)
#pragma unroll
              for (int u = 0; u < U; ++u) {
                ms[u] = fma((double)k[u][q].x, Pw[4 * q], ms[u]);
                ms[u] = fma((double)k[u][q].y, Pw[4 * q + 1], ms[u]);
                ms[u] = fma((double)k[u][q].z, Pw[4 * q + 2], ms[u]);
                ms[u] = fma((double)k[u][q].w, Pw[4 * q + 3], ms[u]);
              }
#pragma unroll
            for (int u = 0; u < U; ++u)
              if (t0 + u < T) s_r[(size_t)(t0 + u) * E + id] = (dv[u] - cc) - ms[u];
          }
        }
      }
      wave_sync();                                  // a group's four lanes are in one wave
      if (f < F && (id & 3) == 0) {
        // channels in order, time bins in order: one chain of fmas, its
        // residuals read eight ahead
        double acc = 0.0;
        const int nq = min(4, F - f);
        if constexpr (ONE) {
          for (int q = 0; q < nq; ++q) acc = fma(s_r[id + q], s_r[id + q], acc);
        } else {
          for (int q = 0; q < nq; ++q) {
            const double* r = s_r + id + q;
            int t = 0;
            for (; t + 8 <= T; t += 8) {
              double v[8];
#pragma unroll
              for (int u = 0; u < 8; ++u) v[u] = r[(size_t)(t + u) * E];
#pragma unroll
              for (int u = 0; u < 8; ++u) acc = fma(v[u], v[u], acc);
            }
            for (; t < T; ++t) acc = fma(r[(size_t)t * E], r[(size_t)t * E], acc);
          }
        }
        s_part[f >> 2] = acc;
      }
      wave_sync();                                  // s_r is free for the next channels
    }
    __syncthreads();
  }
}

using RunKernel = void (*)(ChainState, DevModel, RunModel, double, int, const double*,
                           const double*, long long);

template <bool AB, bool ONE>
RunKernel run_kernel(int NT) {
  switch (NT) {
    case 4: return k_chain_run<4, AB, ONE>;
    case 8: return k_chain_run<8, AB, ONE>;
    case 12: return k_chain_run<12, AB, ONE>;
    case 16: return k_chain_run<16, AB, ONE>;
    case 24: return k_chain_run<24, AB, ONE>;
    case 32: return k_chain_run<32, AB, ONE>;
    default: return nullptr;
  }
}

// Evaluation lanes of k_chain_run: a lane per channel (a channel loop past
// 384), with the residuals of all lanes within 96 KB of LDS (T <= 64).
int run_lanes(const DevModel& m) {
  const int most = 96 * 1024 / (8 * m.T) / 64 * 64;
  return std::min({(m.F + 63) / 64 * 64, kRunMaxThreads - kRunHelpers, most});
}

}  // namespace

// ---------------------------------------------------------------------------
// host engine

struct Chains {
  Model* m = nullptr;
  int cap = 0, P = 0;
  ChainState st{};
  double *d_x0 = nullptr, *d_l0 = nullptr, *d_chol = nullptr, *d_lo = nullptr, *d_hi = nullptr;
  double* d_lstar = nullptr;
  int* h_stage = nullptr;                       // pinned
  float4* d_rk = nullptr;                       // the model laid out for k_chain_run
  double* d_rd = nullptr;
  std::vector<double> lo, hi;
  unsigned long long seed = 0;
  unsigned long long calls = 0;
  hipStream_t s = nullptr;
  // graph of kRoundsPerGraph rounds; rebuilt when the chain count, the
  // precision, the steps or any buffer it captured changes
  hipGraphExec_t graph = nullptr;
  int g_n = -1, g_prec = -1, g_steps = -1;
  const void* g_model = nullptr;      // model buffers at capture (eviction moves them)
  const void* g_work = nullptr;       // likelihood workspace at capture
  Tile g_tile{};
};

static void chains_free(Chains* c) {
  void* ps[] = {c->st.x, c->st.dir, c->st.a, c->st.b, c->st.t, c->st.lx, c->st.stage,
                c->st.done, c->st.expand, c->st.evals, c->st.ctr, c->st.theta, c->st.inbox,
                c->st.lnl, c->st.rounds, c->d_x0, c->d_l0, c->d_chol, c->d_lo, c->d_hi, c->d_lstar,
                c->d_rk, c->d_rd};
  for (void* p : ps)
    if (p) (void)hipFree(p);
  if (c->h_stage) (void)hipHostFree(c->h_stage);
  if (c->graph) (void)hipGraphExecDestroy(c->graph);
  if (c->s) (void)hipStreamDestroy(c->s);
}

template <typename T>
static hipError_t dalloc(T** p, size_t n) {
  return hipMalloc(reinterpret_cast<void**>(p), std::max<size_t>(n * sizeof(T), 16));
}

// The chains' generator on its own: one thread per counter block.
__global__ void k_philox(const uint32_t* __restrict__ ctr, int n, uint32_t k0, uint32_t k1,
                         uint32_t* __restrict__ out) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  uint32_t c[4] = {ctr[4 * j], ctr[4 * j + 1], ctr[4 * j + 2], ctr[4 * j + 3]};
  philox4x32(c, k0, k1);
#pragma unroll
  for (int q = 0; q < 4; ++q) out[4 * j + q] = c[q];
}

constexpr int kPhiloxMaxBlocks = 1 << 24;

// Whether a call's rounds run in place (k_chain_run): the model's thin form
// for this precision, no kernel timing (whose events bracket the likelihood
// kernel of the launched rounds), and few enough chains.  A launched round costs
// 11-13 us plus the batch's throughput; a round in place costs its latency
// (passes over the channels, each with a serial chain over the time bins), once
// per generation of resident workgroups.  Both measured per call (ms, launched
// and in place; one card, 301 channels but for N10's 151):
//   N10 T1  n 70: 28.1, 3.9    n 1000: 11.1, 3.3    n 4000: 10.0, 5.4
//   N16 T20 n 100: 22.4, 6.4   n 1000: 28.0, 15.1   n 4000: 32.0, 26.7-43
//   N8 T40  n 100: 17.4, 9.5   n 1000: 21.8, 32.0   N4 T64 n 400: 12.1, 16.4
// so the line lies at 96 channel passes x bins (at least 8) x generations.
constexpr int kRunCost = 96;
static bool run_takes(const Model* m, int prec, int n) {
  const DevModel& d = m->dm;
  if (kind_of(prec, d) != kThin || group_of(kThin, d) != 4 || m->timing || m->P > kRunMaxP ||
      run_parts(d.F) > 2048)
    return false;
  const int E = run_lanes(d), passes = (d.F + E - 1) / E;
  const int by_lds = (int)(max_lds_bytes() / (run_lds(d.T, E, d.F) + 2048));
  const int per_cu = std::max(1, std::min(by_lds, 16 / (E / 64 + 2)));
  const int64_t gens = ((int64_t)n + kCUs * per_cu - 1) / (kCUs * per_cu);
  return gens * passes * std::max(d.T, 8) <= kRunCost;
}

// The call's rounds by k_chain_run, from the inputs already queued on the
// engine's stream.  The counts reported are those of the launched rounds: one,
// then batches of kRoundsPerGraph until every chain is done.
static int run_in_place(Chains* c, ChainState st, long long max_rounds, double* x_out,
                        double* l_out, int64_t* evals, int64_t* rounds) {
  Model* m = c->m;
  const DevModel& d = m->dm;
  hipStream_t s = c->s;
  const int n = st.n, P = c->P, Fp = (d.F + 63) / 64 * 64;
  hipError_t e = hipSuccess;
  if (!c->d_rd) {
    if ((e = dalloc(&c->d_rk, (size_t)d.T * (d.NT / 4) * Fp)) == hipSuccess &&
        (e = dalloc(&c->d_rd, (size_t)d.T * Fp)) == hipSuccess) {
      hipLaunchKernelGGL(k_run_layout, dim3((Fp + 255) / 256, d.T), dim3(256), 0, s, d, Fp,
                         c->d_rk, c->d_rd);
      e = hipGetLastError();
    }
    if (e != hipSuccess) {
      (void)hipStreamSynchronize(s);
      if (c->d_rk) (void)hipFree(c->d_rk);
      if (c->d_rd) (void)hipFree(c->d_rd);
      c->d_rk = nullptr;
      c->d_rd = nullptr;
      return hip_err(e, "laying out the model for the chains");
    }
  }
  const int E = run_lanes(d);
  const bool one = d.T == 1 && d.F <= E;
  const RunKernel kern = d.NA > 0 ? (one ? run_kernel<true, true>(d.NT) : run_kernel<true, false>(d.NT))
                                  : (one ? run_kernel<false, true>(d.NT) : run_kernel<false, false>(d.NT));
  if (!kern) return set_err(FGL_EINVAL, "NT=%d has no chain kernel", d.NT);
  const size_t lds = run_lds(d.T, E, d.F);
  if ((e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                               hipFuncAttributeMaxDynamicSharedMemorySize, 120 * 1024)) != hipSuccess)
    return hip_err(e, "chain kernel LDS");
  const long long cap = 1 + (max_rounds - 1 + kRoundsPerGraph - 1) / kRoundsPerGraph * kRoundsPerGraph;
  std::vector<int> ev(n);
  std::vector<long long> nr(n);
  bool all = false;
  long long limit = 0;
  for (int first = 1; !all && limit < cap; first = 0) {
    limit = std::min<long long>(cap, limit + kRunRounds);
    hipLaunchKernelGGL(kern, dim3(n), dim3(E + kRunHelpers), lds, s, st, d, RunModel{c->d_rk, c->d_rd, Fp},
                       (double)d.F * (double)d.T, first, c->d_x0, c->d_l0, limit);
    if ((e = hipGetLastError()) != hipSuccess) return hip_err(e, "chain rounds");
    if ((e = hipMemcpyAsync(c->h_stage, st.stage, (size_t)n * sizeof(int), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipMemcpyAsync(x_out, st.x, (size_t)n * P * 8, hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipMemcpyAsync(l_out, st.lx, (size_t)n * 8, hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipMemcpyAsync(ev.data(), st.evals, (size_t)n * sizeof(int), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipMemcpyAsync(nr.data(), st.rounds, (size_t)n * sizeof(long long), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
      return hip_err(e, "copy chain results");
    all = true;
    for (int i = 0; i < n && all; ++i) all = c->h_stage[i] == kDone;
  }
  if (!all) return set_err(FGL_EAGAIN, "chains did not finish within %lld rounds", max_rounds);
  if (evals) {
    int64_t sum = 0;
    for (int v : ev) sum += v;
    *evals = sum;
  }
  if (rounds) {
    const int64_t most = (int64_t)*std::max_element(nr.begin(), nr.end());
    *rounds = 1 + std::max<int64_t>(1, (most - 1 + kRoundsPerGraph - 1) / kRoundsPerGraph) * kRoundsPerGraph;
  }
  c->calls++;
  return FGL_OK;
}

}  // namespace fgl

using namespace fgl;

extern "C" {

int fgl_chains_create(fgl_model* mh, int max_chains, const double* lo, const double* hi,
                      uint64_t seed, fgl_chains** out) {
  if (!out) return set_err(FGL_EINVAL, "out is NULL");
  *out = nullptr;
  Model* m = reinterpret_cast<Model*>(mh);
  if (!m || !lo || !hi) return set_err(FGL_EINVAL, "model, lo and hi must be non-NULL");
  if (max_chains < 1 || max_chains > kMaxRows)
    return set_err(FGL_EINVAL, "max_chains=%d outside 1..2^26", max_chains);
  const int P = m->P;
  if (P > kMaxP) return set_err(FGL_EINVAL, "P=%d exceeds the chains' %d parameters", P, kMaxP);
  for (int k = 0; k < P; ++k)
    if (!std::isfinite(lo[k]) || !std::isfinite(hi[k]) || !(lo[k] < hi[k]))
      return set_err(FGL_EINVAL, "box coordinate %d: need finite lo < hi", k);
  Chains* c = new (std::nothrow) Chains();
  if (!c) return set_err(FGL_ENOMEM, "host allocation");
  c->m = m;
  c->cap = max_chains;
  c->P = P;
  c->lo.assign(lo, lo + P);
  c->hi.assign(hi, hi + P);
  c->seed = seed;
  hipError_t e = hipSetDevice(m->dev);
  const size_t n = (size_t)max_chains;
  ChainState& s = c->st;
  if (e == hipSuccess) e = hipStreamCreateWithFlags(&c->s, hipStreamNonBlocking);
  if (e == hipSuccess) e = dalloc(&s.x, n * P);
  if (e == hipSuccess) e = dalloc(&s.dir, n * P);
  if (e == hipSuccess) e = dalloc(&s.a, n);
  if (e == hipSuccess) e = dalloc(&s.b, n);
  if (e == hipSuccess) e = dalloc(&s.t, n);
  if (e == hipSuccess) e = dalloc(&s.lx, n);
  if (e == hipSuccess) e = dalloc(&s.stage, n);
  if (e == hipSuccess) e = dalloc(&s.done, n);
  if (e == hipSuccess) e = dalloc(&s.expand, n);
  if (e == hipSuccess) e = dalloc(&s.evals, n);
  if (e == hipSuccess) e = dalloc(&s.rounds, n);
  if (e == hipSuccess) e = dalloc(&s.ctr, n);
  if (e == hipSuccess) e = dalloc(&s.theta, n * P);
  if (e == hipSuccess) e = dalloc(&s.inbox, n);
  if (e == hipSuccess) e = dalloc(&s.lnl, n);
  if (e == hipSuccess) e = dalloc(&c->d_x0, n * P);
  if (e == hipSuccess) e = dalloc(&c->d_l0, n);
  if (e == hipSuccess) e = dalloc(&c->d_chol, (size_t)P * P);
  if (e == hipSuccess) e = dalloc(&c->d_lo, (size_t)P);
  if (e == hipSuccess) e = dalloc(&c->d_hi, (size_t)P);
  if (e == hipSuccess) e = dalloc(&c->d_lstar, 1);
  if (e == hipSuccess)
    e = hipHostMalloc(reinterpret_cast<void**>(&c->h_stage), n * sizeof(int), hipHostMallocDefault);
  if (e == hipSuccess) e = hipMemset(s.ctr, 0, n * sizeof(unsigned long long));
  if (e == hipSuccess) e = hipMemcpy(c->d_lo, lo, P * 8, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(c->d_hi, hi, P * 8, hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    chains_free(c);
    delete c;
    return hip_err(e, "allocating chain state");
  }
  s.P = P;
  s.chol = c->d_chol;
  s.lo = c->d_lo;
  s.hi = c->d_hi;
  s.lstar = c->d_lstar;
  s.seed = seed;
  m->served.fetch_add(1);       // the model stays alive while the engine exists
  *out = reinterpret_cast<fgl_chains*>(c);
  return FGL_OK;
}

int fgl_chains_run(fgl_chains* ch, const double* x0, const double* l0, int n, double lstar,
                   const double* chol, int steps, int prec, double* x_out, double* l_out,
                   int64_t* evals, int64_t* rounds) {
  TraceRange tr("fgl_chains_run n=%d steps=%d prec=%d", n, steps, prec);
  Chains* c = reinterpret_cast<Chains*>(ch);
  if (!c || !x0 || !l0 || !chol || !x_out || !l_out)
    return set_err(FGL_EINVAL, "NULL argument");
  if (n < 1 || n > c->cap) return set_err(FGL_EINVAL, "n=%d outside 1..%d", n, c->cap);
  if (steps < 0) return set_err(FGL_EINVAL, "steps=%d < 0", steps);
  if (prec != FGL_PREC_MIXED && prec != FGL_PREC_FP32 && prec != FGL_PREC_FP64)
    return set_err(FGL_EINVAL, "unknown precision %d", prec);
  if (std::isnan(lstar)) return set_err(FGL_EINVAL, "lstar is NaN");
  Model* m = c->m;
  const int P = c->P;
  for (int i = 0; i < n; ++i)
    for (int k = 0; k < P; ++k) {
      const double v = x0[(size_t)i * P + k];
      if (!(v >= c->lo[k] && v <= c->hi[k]))
        return set_err(FGL_EINVAL, "start point %d is outside the box (coordinate %d)", i, k);
    }
  InflightGuard guard(m);
  std::lock_guard<std::mutex> lk(m->mu);
  hipError_t e = hipSetDevice(m->dev);
  if (e != hipSuccess) return hip_err(e, "hipSetDevice");
  int rc = make_resident(m);
  if (rc != FGL_OK) return rc;
  hipStream_t s = c->s;
  ChainState st = c->st;
  st.n = n;
  st.steps = steps;
  if ((e = hipMemcpyAsync(c->d_x0, x0, (size_t)n * P * 8, hipMemcpyHostToDevice, s)) != hipSuccess ||
      (e = hipMemcpyAsync(c->d_l0, l0, (size_t)n * 8, hipMemcpyHostToDevice, s)) != hipSuccess ||
      (e = hipMemcpyAsync(c->d_chol, chol, (size_t)P * P * 8, hipMemcpyHostToDevice, s)) != hipSuccess ||
      (e = hipMemcpyAsync(c->d_lstar, &lstar, 8, hipMemcpyHostToDevice, s)) != hipSuccess)
    return hip_err(e, "copy chain inputs");
  if (P > kMaxP) return set_err(FGL_EINVAL, "P=%d exceeds the chains' %d parameters", P, kMaxP);
  st.N = m->dm.N;
  st.NA = m->dm.NA;
  st.NB = m->dm.NB;
  st.betaRows = m->dm.KC * 32;
  st.flags = m->dm.flags;
  // the bound covers steps of at most 2 kMaxExpand + 64 rounds each
  const long long max_rounds = (long long)std::max(steps, 1) * (2 * kMaxExpand + 66);
  if (run_takes(m, prec, n)) return run_in_place(c, st, max_rounds, x_out, l_out, evals, rounds);
  const int blocks = (n + kWaves - 1) / kWaves;
  // the likelihood's workspace for n rows on this stream, fixed before the
  // start kernel (which writes the first proposals' row records into it)
  // and before capture
  const Kind k = kind_of(prec, m->dm);
  const Tile tile = tile_for(m, k, n);
  WorkBuf& wb = m->work[s];
  wb.stream_synced_free = true;
  if ((rc = ensure_work(m, wb, n, n_groups(m->dm, tile), false)) != FGL_OK) return rc;
  st.rows = wb.w.rows;
  st.betaT = wb.w.betaT;
  st.offT = wb.w.offT;
  st.Bpad = wb.w.Bpad;
  hipLaunchKernelGGL(k_chain_start, dim3(blocks), dim3(64 * kWaves), 0, s, st, c->d_x0, c->d_l0);
  if ((e = hipGetLastError()) != hipSuccess) return hip_err(e, "chain start");
  // the padding rows up to Bpad (and the first proposals again, with the
  // same result) by the row-preparation kernel, once per call; later rounds
  // take the records the step kernel writes with each proposal
  if ((e = launch_prep(m->dm, st.theta, n, wb.w, m->dm.KC * 32, s)) != hipSuccess)
    return hip_err(e, "prep kernel");
  RowSums rs{wb.w.partial, wb.w.rows, n_groups(m->dm, tile), wb.w.Bpad,
             (double)m->dm.F * (double)m->dm.T,
             chi0_of(k, m->dm)};
  auto round = [&]() -> int {
    int rc2 = enqueue_main(m, k, tile, wb, s);
    if (rc2 != FGL_OK) return rc2;
    hipLaunchKernelGGL(k_chain_step, dim3(blocks), dim3(64 * kWaves), 0, s, st, rs);
    hipError_t e2 = hipGetLastError();
    return e2 == hipSuccess ? FGL_OK : hip_err(e2, "chain step");
  };
  // one eager round (it also sets the kernels' launch attributes outside
  // any capture), then kRoundsPerGraph rounds captured once and replayed
  if ((rc = round()) != FGL_OK) return rc;
  long long done_rounds = 1;
  const void* model_buf = m->dm.proj ? (const void*)m->dm.rd : (const void*)m->dm.kd;
  if (c->graph && (c->g_n != n || c->g_prec != prec || c->g_steps != steps ||
                   c->g_model != model_buf || c->g_work != (const void*)wb.w.partial ||
                   c->g_tile.waves != tile.waves || c->g_tile.fc != tile.fc ||
                   c->g_tile.occ != tile.occ)) {
    (void)hipGraphExecDestroy(c->graph);
    c->graph = nullptr;
  }
  const bool timing = m->timing;
  if (!c->graph && !timing) {
    hipGraph_t g = nullptr;
    if ((e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal)) != hipSuccess)
      return hip_err(e, "begin capture");
    int crc = FGL_OK;
    for (int r = 0; r < kRoundsPerGraph && crc == FGL_OK; ++r) crc = round();
    e = hipStreamEndCapture(s, &g);
    if (crc != FGL_OK) {
      if (g) (void)hipGraphDestroy(g);
      return crc;
    }
    if (e != hipSuccess) return hip_err(e, "end capture");
    e = hipGraphInstantiate(&c->graph, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
      c->graph = nullptr;
      return hip_err(e, "graph instantiate");
    }
    c->g_n = n;
    c->g_prec = prec;
    c->g_steps = steps;
    c->g_model = model_buf;
    c->g_work = wb.w.partial;
    c->g_tile = tile;
  }
  // replay until every chain is done
  while (done_rounds < max_rounds) {
    if (c->graph) {
      if ((e = hipGraphLaunch(c->graph, s)) != hipSuccess) return hip_err(e, "graph launch");
    } else {
      for (int r = 0; r < kRoundsPerGraph; ++r)
        if ((rc = round()) != FGL_OK) return rc;
    }
    done_rounds += kRoundsPerGraph;
    if ((e = hipMemcpyAsync(c->h_stage, st.stage, (size_t)n * sizeof(int), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
      return hip_err(e, "chain progress");
    bool all = true;
    for (int i = 0; i < n && all; ++i) all = c->h_stage[i] == kDone;
    if (all) break;
  }
  std::vector<int> ev(n);
  if ((e = hipMemcpyAsync(x_out, st.x, (size_t)n * P * 8, hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipMemcpyAsync(l_out, st.lx, (size_t)n * 8, hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipMemcpyAsync(ev.data(), st.evals, (size_t)n * sizeof(int), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return hip_err(e, "copy chain results");
  bool all = true;
  for (int i = 0; i < n && all; ++i) all = c->h_stage[i] == kDone;
  if (!all) return set_err(FGL_EAGAIN, "chains did not finish within %lld rounds", max_rounds);
  if (evals) {
    int64_t sum = 0;
    for (int v : ev) sum += v;
    *evals = sum;
  }
  if (rounds) *rounds = done_rounds;
  c->calls++;
  return FGL_OK;
}

int fgl_chains_philox(const uint32_t* ctr, int n, uint32_t k0, uint32_t k1, uint32_t* out) {
  if (!ctr || !out) return set_err(FGL_EINVAL, "ctr and out must be non-NULL");
  if (n < 1 || n > kPhiloxMaxBlocks)
    return set_err(FGL_EINVAL, "n=%d outside 1..%d", n, kPhiloxMaxBlocks);
  int dev = 0;
  int rc = check_device(&dev);
  if (rc != FGL_OK) return rc;
  const size_t bytes = (size_t)n * 16;
  uint32_t *d_in = nullptr, *d_out = nullptr;
  hipStream_t s = nullptr;
  hipError_t e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
  if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&d_in), bytes);
  if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&d_out), bytes);
  if (e == hipSuccess) e = hipMemcpyAsync(d_in, ctr, bytes, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_philox, dim3((n + 255) / 256), dim3(256), 0, s, d_in, n, k0, k1, d_out);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(out, d_out, bytes, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (s) (void)hipStreamSynchronize(s);
  if (d_in) (void)hipFree(d_in);
  if (d_out) (void)hipFree(d_out);
  if (s) (void)hipStreamDestroy(s);
  return e == hipSuccess ? FGL_OK : hip_err(e, "Philox kernel");
}

int fgl_chains_destroy(fgl_chains* ch) {
  Chains* c = reinterpret_cast<Chains*>(ch);
  if (!c) return set_err(FGL_EINVAL, "chains is NULL");
  (void)hipSetDevice(c->m->dev);
  if (c->s) (void)hipStreamSynchronize(c->s);
  if (c->s) drop_stream_work(c->s);
  chains_free(c);
  c->m->served.fetch_sub(1);
  delete c;
  return FGL_OK;
}

}  // extern "C"
