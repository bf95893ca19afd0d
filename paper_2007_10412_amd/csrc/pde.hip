// Reaction-diffusion PDE-constrained optimisation with a sampled adjoint (Section 5, Appendix B).
// phi lives on the nodes (i, j), 0 <= i, j <= n <= 32, of the unit square, zero on the boundary; one explicit
// step is phi += r (4-neighbour sum - 4 phi) + dt C phi with r = D dt / dx^2 and C the seven-term series in x and
// t.  The steps depend on each other, so one problem is one workgroup (one barrier per step) and the launch runs
// many problems (control vectors, sampling streams) side by side, one per CU.  All arithmetic is fp64.
//
// What is kept of phi_t for the backward pass: the interior entries whose key is below p 2^32 (entry
// c = (i-1)(n-1) + (j-1) of step t takes word c mod 4 of the Philox call c / 4 with (stream, step = t)).  The
// backward pass draws the same keys again and walks the kept entries back.
//
// What bounds it: instruction issue, vector instructions above all (a wave alone issues one every four to six clocks),
// and the chain read - compute - write - barrier of a step.  So a third of the waves does nothing but the stencil,
// four cells of the linear order to a lane: the cells' values stay in registers, the ten around them come from LDS,
// neighbours across a row's end are masked by a factor.  The other waves sample from the state that the stencil waves
// publish: the lane of a quad of cells makes its one Philox call and has the keys in registers.  They come in two
// sets, for even and for odd steps, so that a wave has two steps' time for one draw: its latency (46 clocks a round)
// is off the chain.  Backward the sampling waves also form what kept entries add to lambda (a dense array in LDS that
// the stencil adds) and the weighted sums of the gradient, without branches on which lanes kept something: a taken
// branch costs as much as ten instructions.
// 256 problems of 32 x 32, 4096 steps, microseconds, with a node a lane in sixteen waves that do everything / this:
// p = 0.01 4790 / 3290, 0.05 4900 / 3280, 0.5 5225 / 3650, 1 5300 / 3960 (forward at the HBM's write rate); 512
// problems 9500 / 6260; one problem 4690 / 3100; one of 8 x 8 3570 / 2100.  40960 steps: 22.0 + 25.3 / 12.5 + 18.5 ms.
// Slower: sampling waves that draw every step (18.0 + 31.2); three sets (13.2 + 33.1, registers spill); skipping the
// places of a quad that no lane of the wave kept (12.6 + 22.6); the stencil waves sampling for themselves (43 in all).
#include <cmath>

#include "kernels.hpp"
#include "pde_layout.hpp"
#include "philox.hpp"

namespace rad {

namespace {

constexpr int kPdeLanes = 64 * kPdeWaves;                      // lanes of the stencil waves (four cells each)
constexpr int kPdePad = 32;                                    // zeros before the first cell: a grid row and more
constexpr int kPdePlane = 320;                                 // pitch of the planes; a multiple of 64: paired LDS writes
constexpr int kPdeBuf = 4 * kPdePlane;
constexpr int kPdeTab = 64;                                    // time points per refill of half the table
constexpr int kPdeUnit = 256, kPdeRing = 2 * kPdeUnit;         // kept values per load, in a wave's LDS ring
static_assert(4 * kPdePlane >= 4 * kPdeLanes + 2 * kPdePad, "a grid row of zeros on either side of the cells");

// place of cell c >= -kPdePad in a buffer: cells e, e + 4, e + 8, ... form plane e, so that the lanes of a wave, with
// four cells in a row each, read and write consecutive doubles
__device__ __forceinline__ int pde_slot(int c) {
  c += kPdePad;
  return (c & 3) * kPdePlane + (c >> 2);
}

// Fixed values of cell c (0 where there is none).
struct PdeCell {
  bool in;
  int i, j;
  double s2x, c2x, phi0, tgt;
  __device__ __forceinline__ PdeCell(int n, int c) {
    const int m = n - 1;
    in = c < m * m;
    i = c / m + 1; j = c - (i - 1) * m + 1;
    const double x = (double)i / n, y = (double)j / n;
    s2x = in ? sinpi(2.0 * x) : 0.0;
    c2x = in ? cospi(2.0 * x) : 0.0;
    phi0 = in ? sinpi(x) * sinpi(y) : 0.0;
    tgt = in ? sinpi(2.0 * x) * sinpi(y) : 0.0;
  }
};

// LDS written before is seen after; global accesses stay in flight
__device__ __forceinline__ void pde_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

struct PdeArgs {
  int n; int64_t steps; double r, dt, p;
  uint32_t thr;                               // keep iff key < thr; kernels of their own keep everything (p = 1)
  uint32_t seed_lo, seed_hi, stream_id;
  const double* theta;                        // [problems][7]
  double* vals; int64_t per_problem;          // [problems][per_problem] kept entries, a run for each sampling wave
  PdeRunLayout runs;                          // of even and of odd steps
  uint32_t* wave_end;                         // [problems][kPdeRuns] entries each wave kept in all
  int* overflow;                              // [problems]
  double* loss; double* grad; int64_t* stored;
};

// a time point: dt C - 4 r = ka + sin(2 pi x) kb + cos(2 pi x) kc, and the sine and cosine of pi t
struct __align__(16) PdePoint { double ka, kb, kc, s, c, unused; };

struct PdeShared {
  double f[2][kPdeBuf];                       // phi (forward) or lambda (backward) of this step and the next
  PdePoint tab[2][kPdeTab];
  double red[3 * kPdeWaves];
  double theta[7];
  __device__ __forceinline__ const PdePoint& point(uint32_t i) const {
    return tab[(i / kPdeTab) & 1u][i & (kPdeTab - 1)];
  }
};

// A stencil lane: its four cells' values stay in registers, those around them come from LDS.
struct PdeStencil {
  double s2x[4], c2x[4];
  double bond[3];                  // 1 if cells e and e + 1 are neighbours in a row, else 0
  int up[4], down[4], left, right, own;
  double x[4];
  __device__ __forceinline__ void init(int n, int q) {
    const int m = n - 1, zero = pde_slot(-kPdePad);
    own = pde_slot(4 * q);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const PdeCell cell(n, 4 * q + e);
      const int c = 4 * q + e;
      s2x[e] = cell.s2x; c2x[e] = cell.c2x;
      if (e < 3) bond[e] = cell.in && cell.j < m ? 1.0 : 0.0;
      up[e] = cell.in ? pde_slot(c - m) : zero;
      down[e] = cell.in ? pde_slot(c + m) : zero;
      if (e == 0) left = cell.in && cell.j > 1 ? pde_slot(c - 1) : zero;
      if (e == 3) right = cell.in && cell.j < m ? pde_slot(c + 1) : zero;
    }
  }
  struct Around { double up[4], down[4], left, right; };
  __device__ __forceinline__ Around read(const double* f) const {
    Around a;
#pragma unroll
    for (int e = 0; e < 4; ++e) { a.up[e] = f[up[e]]; a.down[e] = f[down[e]]; }
    a.left = f[left]; a.right = f[right];
    return a;
  }
  // x <- x + r (neighbours) + (dt C - 4 r) x; places past the last cell see zeros only and stay zero
  __device__ __forceinline__ void step(const Around& a, double r, double ka, double kb, double kc) {
    double nw[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double nb = a.up[e] + a.down[e];
      nb = e == 0 ? nb + a.left : fma(bond[e - 1], x[e - 1], nb);
      nb = e == 3 ? nb + a.right : fma(bond[e], x[e + 1], nb);
      const double k = fma(s2x[e], kb, fma(c2x[e], kc, ka));
      nw[e] = x[e] + fma(k, x[e], r * nb);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = nw[e];
  }
  __device__ __forceinline__ void write(double* f) const {
#pragma unroll
    for (int e = 0; e < 4; ++e) f[own + e * kPdePlane] = x[e];
  }
};

// A sampling lane: draws for the cells of the stencil lane of the same number.  A draw is made in two halves of five
// Philox rounds, so that both of the steps that a sampling wave has for one of its times carry one.
template <bool kAll>
struct PdeSampler {
  uint32_t q, stream;
  int own;
  uint32_t thr[4];                 // 0 where there is no cell
  u32x4 half;
  __device__ __forceinline__ void init(const PdeArgs& a, int lane_q, int pb) {
    const int cells = (a.n - 1) * (a.n - 1);
    q = (uint32_t)lane_q;
    stream = a.stream_id + (uint32_t)pb;
    own = pde_slot(4 * lane_q);
#pragma unroll
    for (int e = 0; e < 4; ++e) thr[e] = 4 * lane_q + e < cells ? a.thr : 0u;
  }
  __device__ __forceinline__ void draw_first(const PdeArgs& a, uint32_t t) {
    if (!kAll) half = philox4x32_rounds<5>(q, 0u, stream, t, a.seed_lo, a.seed_hi);
  }
  // the kept cells of the step that draw_first was given, as masks over the wave
  __device__ __forceinline__ void draw_second(const PdeArgs& a, uint64_t (&m)[4]) const {
    if (kAll) {
#pragma unroll
      for (int e = 0; e < 4; ++e) m[e] = __ballot(thr[e] != 0u);
      return;
    }
    const u32x4 k4 = philox4x32_rounds<5>(half[0], half[1], half[2], half[3], a.seed_lo + 5u * kPhiloxW0,
                                          a.seed_hi + 5u * kPhiloxW1);
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = __ballot(k4[e] < thr[e]);
  }
  // time point `t` (of a lane) into place `lane` of a half of the table
  __device__ __forceinline__ void table(const PdeArgs& a, const double* th, PdePoint* half_tab, double t) const {
    double sn, cs;
    sincospi(t * a.dt, &sn, &cs);
    PdePoint o;
    o.ka = a.dt * (th[0] + th[1] * sn + th[2] * cs) - 4.0 * a.r;
    o.kb = a.dt * (th[3] * sn + th[4] * cs);
    o.kc = a.dt * (th[5] * sn + th[6] * cs);
    o.s = sn; o.c = cs; o.unused = 0.0;
    half_tab[q & 63u] = o;
  }
};

__device__ __forceinline__ int pde_count(const uint64_t (&m)[4]) {
  return (__popcll(m[0]) + __popcll(m[1])) + (__popcll(m[2]) + __popcll(m[3]));
}

__device__ __forceinline__ uint32_t pde_lanes_below(uint64_t m, uint32_t plus = 0u) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, plus));
}

__device__ __forceinline__ bool pde_bit(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// sum over the workgroup in a fixed order; every thread gets the result
__device__ __forceinline__ double pde_sum(double v, double* red) {
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) v += __shfl_down(v, s);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
  return t;
}

template <bool kAll>
__global__ __launch_bounds__(3 * kPdeLanes) void pde_forward_kernel(PdeArgs a) {
  __shared__ PdeShared sh;
  const int pb = blockIdx.x;
  const int waves = (int)blockDim.x / 192;                      // stencil waves; twice as many sample
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t steps = (uint32_t)a.steps;
  for (int k = threadIdx.x; k < 2 * kPdeBuf; k += blockDim.x) (&sh.f[0][0])[k] = 0.0;
  if (threadIdx.x < 7) sh.theta[threadIdx.x] = a.theta[(size_t)pb * 7 + threadIdx.x];
  __syncthreads();
  double loss = 0.0, over = 0.0, kept = 0.0;
  if (wave < waves) {
    const int q = (int)threadIdx.x;
    PdeStencil me; me.init(a.n, q);
    double phi0[4], tgt[4], sum[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const PdeCell cell(a.n, 4 * q + e);
      phi0[e] = me.x[e] = cell.phi0; tgt[e] = cell.tgt; sum[e] = 0.0;
    }
    me.write(sh.f[0]);
    auto add_loss = [&](double s) {                             // nothing at t = 0, where phi_0 is the target
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double d = me.x[e] - fma(0.25 * s, tgt[e], phi0[e]);
        sum[e] = fma(d, d, sum[e]);
      }
    };
    __builtin_amdgcn_s_setprio(3);
    pde_barrier();
    auto step = [&](uint32_t t, int cur) {
      const PdeStencil::Around nb = me.read(sh.f[cur]);
      const PdePoint& pt = sh.point(t);
      const double ka = pt.ka, kb = pt.kb, kc = pt.kc;
      add_loss(pt.s);
      me.step(nb, a.r, ka, kb, kc);
      me.write(sh.f[cur ^ 1]);
      pde_barrier();
    };
    uint32_t t = 0;
    for (; pde_pair_left(t, steps); t += 2) { step(t, 0); step(t + 1, 1); }
    if (t < steps) step(t, 0);
    add_loss(sh.point(steps).s);
    loss = (sum[0] + sum[1]) + (sum[2] + sum[3]);
  } else {
    const int sw = wave - waves, odd = sw >= waves ? 1 : 0;     // even or odd steps
    PdeSampler<kAll> me; me.init(a, (int)threadIdx.x - 64 * waves * (1 + odd), pb);
    const bool filler = sw == 0;                                // fills the table
    double* at = a.vals + (size_t)pb * a.per_problem + a.runs.at[odd][sw - odd * waves];
    const int64_t cap = a.runs.cap[odd][sw - odd * waves];
    int64_t offset = 0;                                         // entries this wave has kept so far
    uint64_t m[4];
    double x[4];
    auto read = [&]() {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = sh.f[odd][me.own + e * kPdePlane];
    };
    auto append = [&]() {
      offset += pde_count(m);
      if (offset > cap) { over = 1.0; return; }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (pde_bit(m[e])) at[pde_lanes_below(m[e])] = x[e];
        at += __popcll(m[e]);
      }
    };
    me.draw_first(a, (uint32_t)odd);
    me.draw_second(a, m);
    if (filler) me.table(a, sh.theta, sh.tab[0], (double)(me.q & 63u));
    pde_barrier();
    if (odd) pde_barrier();
    // phi_t is read in step t and appended in step t + 1
    for (uint32_t t = (uint32_t)odd;; t += 2) {
      read();
      if (t == steps) { append(); break; }
      if (filler && (t & (kPdeTab - 1)) == 0)
        me.table(a, sh.theta, sh.tab[(t / kPdeTab + 1) & 1u], (double)t + (double)(kPdeTab + (me.q & 63u)));
      me.draw_first(a, t + 2);
      pde_barrier();
      append();
      if (t + 1 == steps) break;
      me.draw_second(a, m);
      pde_barrier();
    }
    if ((threadIdx.x & 63) == 0) {
      a.wave_end[(size_t)pb * kPdeRuns + sw] = (uint32_t)(offset < cap ? offset : cap);
      kept = (double)offset;
    }
  }
  const double total_loss = pde_sum(loss, sh.red);
  const double any_over = pde_sum(over, sh.red);
  const double all_kept = pde_sum(kept, sh.red);
  if (threadIdx.x == 0) {
    a.loss[pb] = total_loss / (double)a.steps;
    a.overflow[pb] = any_over > 0.0 ? 1 : 0;
    if (a.stored) a.stored[pb] = (int64_t)all_kept;
  }
}

template <bool kAll>
__global__ __launch_bounds__(3 * kPdeLanes) void pde_backward_kernel(PdeArgs a) {
  __shared__ PdeShared sh;
  __shared__ double source[2][4 * kPdeLanes];                   // what the kept entries add to lambda, 0 elsewhere
  __shared__ double rings[2 * kPdeWaves][kPdeRing + 1];          // a zero at the end
  const int pb = blockIdx.x;
  const int waves = (int)blockDim.x / 192;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t steps = (uint32_t)a.steps;
  for (int k = threadIdx.x; k < 2 * kPdeBuf; k += blockDim.x) (&sh.f[0][0])[k] = 0.0;
  if (threadIdx.x < 7) sh.theta[threadIdx.x] = a.theta[(size_t)pb * 7 + threadIdx.x];
  __syncthreads();
  // dL/dC of a cell summed over time with the weights 1, sin(pi t), cos(pi t): the cell's factors
  // sin(2 pi x), cos(2 pi x) of the seven basis functions are applied once at the end
  double g[7] = {0, 0, 0, 0, 0, 0, 0};
  // step i turns lambda of time steps - i + 1 into that of u = steps - i; table entry i is for time u
  if (wave < waves) {
    const int q = (int)threadIdx.x;
    PdeStencil me; me.init(a.n, q);
#pragma unroll
    for (int e = 0; e < 4; ++e) me.x[e] = 0.0;
    __builtin_amdgcn_s_setprio(3);
    pde_barrier();
    auto step = [&](uint32_t i, int cur) {
      const PdeStencil::Around nb = me.read(sh.f[cur]);
      const PdePoint& pt = sh.point(i);
      const double ka = pt.ka, kb = pt.kb, kc = pt.kc;
      double add[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) add[e] = source[cur][e * kPdeLanes + q];
      me.step(nb, a.r, ka, kb, kc);
#pragma unroll
      for (int e = 0; e < 4; ++e) me.x[e] += add[e];
      me.write(sh.f[cur ^ 1]);
      pde_barrier();
    };
    uint32_t i = 0;
    for (; i + 1 <= steps; i += 2) { step(i, 0); step(i + 1, 1); }
    if (i <= steps) step(i, 0);
  } else {
    const int sw = wave - waves, odd = sw >= waves ? 1 : 0, lane = (int)threadIdx.x & 63;
    PdeSampler<kAll> me; me.init(a, (int)threadIdx.x - 64 * waves * (1 + odd), pb);
    const uint32_t i0 = (steps - (uint32_t)odd) & 1u;           // the first step whose u this wave sampled
    const bool filler = i0 == 0 && sw == odd * waves;
    double phi0[4], tgt[4], w1[4], ws[4], wc[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const PdeCell cell(a.n, 4 * (int)me.q + e);
      phi0[e] = cell.phi0; tgt[e] = cell.tgt; w1[e] = ws[e] = wc[e] = 0.0;
    }
    const double* const run = a.vals + (size_t)pb * a.per_problem + a.runs.at[odd][sw - odd * waves];
    double* const ring = rings[sw];
    const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.wave_end[(size_t)pb * kPdeRuns + sw]);
    int64_t offset = (int64_t)end;                              // walks back one step's count at a time
    uint32_t unit = (uint32_t)((offset + kPdeUnit - 1) / kPdeUnit);   // entries from unit * kPdeUnit on are in the ring
    double pending[4] = {0, 0, 0, 0};                           // the unit below, on its way
    auto load_unit = [&]() {
      if (unit == 0) return;
      const uint32_t lo = (unit - 1) * kPdeUnit, last = end - 1 - lo;
      const double* from = run + lo;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t k = (uint32_t)(e * 64 + lane);
        pending[e] = from[k < last ? k : last];
      }
    };
    const double inv_p = 1.0 / a.p, wl = 2.0 / (double)a.steps * inv_p;
    uint64_t m[4], next_m[4];                                   // kept cells of the wave's time and of its next
    double v[4] = {0, 0, 0, 0}, next_v[4] = {0, 0, 0, 0};       // their values, 0 elsewhere
    // reads the kept values of the wave's next time from the ring
    auto fetch = [&](const uint64_t (&mask)[4], double (&val)[4]) {
      offset -= pde_count(mask);
      while (unit > 0 && offset < (int64_t)unit * kPdeUnit) {
        --unit;
#pragma unroll
        for (int e = 0; e < 4; ++e) ring[((unit * kPdeUnit) & (kPdeRing - 1)) + e * 64 + lane] = pending[e];
        load_unit();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
      }
      uint32_t at = (uint32_t)offset;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t place = pde_lanes_below(mask[e], at) & (kPdeRing - 1);
        val[e] = ring[pde_bit(mask[e]) ? place : kPdeRing];     // 0 there
        at += (uint32_t)__popcll(mask[e]);
      }
    };
    auto write_source = [&](const uint64_t (&mask)[4], const double (&val)[4], double s) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double d = wl * (val[e] - fma(0.25 * s, tgt[e], phi0[e]));
        source[i0][e * kPdeLanes + (int)me.q] = pde_bit(mask[e]) ? d : 0.0;
      }
    };
    if (lane == 0) ring[kPdeRing] = 0.0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    load_unit();
    me.draw_first(a, steps - i0);
    me.draw_second(a, m);
    me.draw_first(a, steps - i0 - 2);                           // past time 0: not used
    me.draw_second(a, next_m);
    if (filler) me.table(a, sh.theta, sh.tab[0], (double)steps - (double)lane);
    fetch(m, v);
    write_source(m, v, sinpi((double)(steps - i0) * a.dt));
    pde_barrier();
    if (i0) pde_barrier();
    // Step i takes the weights of time u and reads the values of the wave's next time, step i + 1 writes what they
    // add; the time after that is drawn meanwhile.
    for (uint32_t i = i0; i <= steps; i += 2) {
      const bool more = i + 1 < steps;
      double lam[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) lam[e] = sh.f[i0][me.own + e * kPdePlane];
      const PdePoint& pt = sh.point(i);
      const double s = pt.s, c = pt.c, next_s = sh.point(i + 2).s;
      if (more) fetch(next_m, next_v);
      if (filler && (i & (kPdeTab - 1)) == 0)                   // the half that the step before has left
        me.table(a, sh.theta, sh.tab[(i / kPdeTab + 1) & 1u], (double)steps - (double)i - (double)(kPdeTab + lane));
      me.draw_first(a, steps - i - 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double w = v[e] * lam[e];                         // times dt / p at the end
        w1[e] += w; ws[e] = fma(s, w, ws[e]); wc[e] = fma(c, w, wc[e]);
      }
      pde_barrier();
      if (i == steps) break;
      if (more) write_source(next_m, next_v, next_s);
#pragma unroll
      for (int e = 0; e < 4; ++e) { m[e] = next_m[e]; v[e] = next_v[e]; }
      me.draw_second(a, next_m);
      pde_barrier();
    }
    const double sc = a.dt * inv_p;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const PdeCell cell(a.n, 4 * (int)me.q + e);
      g[0] += w1[e] * sc; g[1] += ws[e] * sc; g[2] += wc[e] * sc;
      g[3] += cell.s2x * ws[e] * sc; g[4] += cell.s2x * wc[e] * sc;
      g[5] += cell.c2x * ws[e] * sc; g[6] += cell.c2x * wc[e] * sc;
    }
  }
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    const double tot = pde_sum(g[k], sh.red);
    if (threadIdx.x == 0) a.grad[(size_t)pb * 7 + k] = tot;
  }
}

}  // namespace

hipError_t launch_pde(int problems, int n, int64_t steps, double D, double dt, double p, uint32_t seed_lo,
                      uint32_t seed_hi, uint32_t stream_id, const double* theta, double* vals, int64_t cap,
                      uint32_t* wave_end, int* overflow, double* loss, double* grad, int64_t* stored, hipStream_t st) {
  PdeArgs a;
  a.n = n; a.steps = steps; a.r = D * dt * (double)n * (double)n; a.dt = dt; a.p = p;
  const double thr = std::floor(p * 4294967296.0 + 0.5);
  const bool all = thr >= 4294967296.0;
  a.thr = all ? 0xffffffffu : (uint32_t)thr;
  a.seed_lo = seed_lo; a.seed_hi = seed_hi; a.stream_id = stream_id;
  a.theta = theta; a.vals = vals; a.wave_end = wave_end; a.overflow = overflow;
  a.loss = loss; a.grad = grad; a.stored = stored;
  const int cells = (n - 1) * (n - 1), waves = (cells + kPdeCells - 1) / kPdeCells;
  a.runs = pde_run_layout(cells, steps, p);
  a.per_problem = kPdeRuns * cap;
  if (waves > kPdeWaves || a.runs.total > a.per_problem) return hipErrorInvalidValue;
  const dim3 grid((unsigned)problems), block((unsigned)(192 * waves));
  hipLaunchKernelGGL(all ? pde_forward_kernel<true> : pde_forward_kernel<false>, grid, block, 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(all ? pde_backward_kernel<true> : pde_backward_kernel<false>, grid, block, 0, st, a);
  return hipGetLastError();
}

}  // namespace rad
