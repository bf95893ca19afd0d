// The recurrent model with a small hidden state (Appendix A: hidden 100, batch 150, 784 steps): the whole chain of
// time steps in one launch per direction.
//
// An example's chain h_t = ReLU(x_t W_ih + h_{t-1} W_hh + b) depends on no other example, so a workgroup takes one
// example and keeps all of W_hh in registers (lane: columns lane + 64 c, wave: a range of k).  A step is then a
// vector-matrix product from LDS-broadcast h, a sum of the waves' partial vectors through LDS and two barriers; the
// sample of h_t is packed where it is formed.  The backward chain is the same with W_hh transposed, and as every lane
// already holds the g values of its range it adds the outer product x~_{t-1}^T g_t to registers too (the sampled row
// is fetched two steps ahead by keep bitmap): dW_hh, db and dW_ih leave the launch as one partial array per workgroup.
// What bounds a step is the latency of LDS, barriers and the dependent adds, not arithmetic, so what the chain does not
// wait for is on waves of its own, a column a lane: forward they work out where the entries of the next sample go while
// h_t is formed, store them, the ReLU bits and the dense h; backward they bring the sampled rows into LDS and sum db and
// dW_ih.  Hidden 100, batch 150: 0.62 us a step forward and 0.56 backward (a training step, plan and output layer included, per
// time step: 1.28, with all of it on the waves that sum the products 2.04).
// The outer product reads g from LDS again: held from the vector product on, its registers spilled (batch 4096: 793 us
// with it held, 647 with it read again).
// A training step, fraction 0.1, us, all on one set of waves / this: hidden 100, batch 150, T = 784 1597 / 1005;
// T = 49, batch 256: hidden 64 141 / 102, 100 172 / 120, 128 183 / 132; batch 4096: 64 598 / 530, 100 946 / 647,
// 128 970 / 673, 192 1993 / 1501; a launch per step and product took 17137 in the first case.
// Hidden 192 is where the two arrays fill the registers of a workgroup of 16 waves; wider states are in rnn_wide.hip.
#include "gemm.hpp"

namespace rad {

namespace {

constexpr int kComputeUnits = 256;
constexpr int kMaxIn = 8;                    // input width of the model (kernels for a width of 1, its usual value, and for up to 8)

// Registers hold W_hh (and the sums of dW_hh): 64 CPL columns by NW KPW rows.  CPL more waves, a column a lane, do what is off
// the chain of steps.
template <int NW_, int CPL_, int KPW_> struct RnnShape {
  static constexpr int NW = NW_, CPL = CPL_, KPW = KPW_, COLS = 64 * CPL_, ROWS = NW_ * KPW_, THREADS = 64 * (NW_ + CPL_);
  static_assert(KPW_ % 4 == 0 && NW_ * KPW_ >= COLS && NW_ % 2 == 0 && CPL_ <= NW_ && THREADS <= 1024, "whole vectors of h, a thread per column");
};

// a zero the compiler does not see through: keeps loads of uniform addresses on the vector path, whose counter is
// not the one LDS waits on
__device__ __forceinline__ int opaque_zero() {
  int z;
  asm volatile("v_mov_b32 %0, 0" : "=v"(z));
  return z;
}

// where the kept entries of one store row lie: entries start at `first`, keep word j is in lane j of `words`
struct RowPlan { uint32_t words, first; };

__device__ __forceinline__ RowPlan row_plan(const RnnStore& s, int slot, int row, int B, int lane, int z) {
  RowPlan p;
  p.words = 0u; p.first = 0u;
  if (s.exact) return p;
  const size_t prow = (size_t)slot * s.plan_rows + (size_t)row * s.v.plan_row_stride;
  if (lane < s.v.bm_pitch) p.words = s.v.bitmap[prow * s.v.bm_pitch + lane];
  p.first = s.v.row_ptr[(size_t)slot * B + row + z];
  return p;
}

// keep mask of columns 64 c .. 64 c + 63 and the number of entries before them
__device__ __forceinline__ uint64_t keep_mask(uint32_t words, int c, uint32_t* before) {
  uint32_t n = 0u;
  for (int j = 0; j < 2 * c; ++j) n += __popc(__builtin_amdgcn_readlane(words, j));
  *before = n;
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane(words, 2 * c) |
         ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(words, 2 * c + 1) << 32);
}

// (eight waves to a SIMD where that costs no more than a few registers: batch 4096, hidden 128, 188 us of forward to 152)
template <class S, int IN>
__global__ __launch_bounds__(S::THREADS, S::KPW == 24 && IN == 1 ? 8 : 4) void rnn_forward_kernel(RnnArgs a) {
  constexpr int NW = S::NW, CPL = S::CPL, KPW = S::KPW, COLS = S::COLS, ROWS = S::ROWS;
  __shared__ __align__(16) float hs[2][ROWS];
  __shared__ float part[NW][COLS];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int row = blockIdx.x, H = a.H, z = opaque_zero();
  for (int i = threadIdx.x; i < 2 * ROWS; i += S::THREADS) (&hs[0][0])[i] = 0.f;
  __syncthreads();
  if (w >= NW) {
    // the waves off the chain: ReLU bits, the sample of h_t, the dense h_T, of columns 64 (w - NW) + lane.  Where the
    // entry goes is worked out while h_t is formed; after the step's second barrier there are its value and the stores.
    const int cw = w - NW, n = cw * 64 + lane;
    RowPlan plan = row_plan(a.T > 1 ? a.hh : a.ho, 0, row, a.B, lane, z);
    for (int t = 1; t <= a.T; ++t) {
      const RnnStore& st = t < a.T ? a.hh : a.ho;
      const int slot = t < a.T ? t - 1 : 0;
      uint32_t before;
      const uint64_t keep = keep_mask(plan.words, cw, &before);
      const uint32_t rank = before + (uint32_t)lanes_below(keep), pos = plan.first + rank;
      const bool kept = !st.exact && n < H && ((keep >> lane) & 1u) && (int64_t)pos < st.v.capacity;
      float wgt = st.v.scale;
      if (st.v.mult && kept)
        wgt *= (float)st.v.mult[((size_t)slot * st.plan_rows + (size_t)row * st.v.plan_row_stride) * st.v.mult_pitch + rank];
      if (t + 1 < a.T) plan = row_plan(a.hh, t, row, a.B, lane, z);
      else if (t + 1 == a.T) plan = row_plan(a.ho, 0, row, a.B, lane, z);
      __syncthreads();
      __syncthreads();
      const float h = hs[t & 1][n];
      const uint64_t on = __ballot(h > 0.f);
      if ((lane & 31) == 0 && 2 * cw + (lane >> 5) < a.bp)
        a.bits[((size_t)(t - 1) * a.B + row) * a.bp + 2 * cw + (lane >> 5)] = (uint32_t)(on >> lane);
      if (n < H && t == a.T) a.hT[(size_t)row * H + n] = h;
      if (st.exact && n < H && t < a.T) static_cast<float*>(st.v.values)[((size_t)slot * a.B + row) * H + n] = h;
      if (kept) {
        static_cast<float*>(st.v.values)[pos] = h * wgt;
        if (!st.v.indices) {}
        else if (!st.v.idx_shared) st.v.indices[pos] = (uint16_t)n;
        else if (row == 0) st.v.indices[(size_t)slot * st.v.shared_k + rank] = (uint16_t)n;
      }
    }
    return;
  }
  float wr[CPL][KPW];
#pragma unroll
  for (int c = 0; c < CPL; ++c)
#pragma unroll
    for (int q = 0; q < KPW; ++q) {
      const int k = w * KPW + q, n = c * 64 + lane;
      wr[c][q] = (k < H && n < H) ? a.W_hh[(size_t)k * H + n] : 0.f;
    }
  const bool sums = w < CPL;                 // this wave adds the partial vectors of columns 64 w + lane
  const int n = w * 64 + lane;
  float bias = 0.f, V[IN], u[IN];
#pragma unroll
  for (int i = 0; i < IN; ++i) V[i] = u[i] = 0.f;
  auto prefetch = [&](int t) {               // input of step t
#pragma unroll
    for (int i = 0; i < IN; ++i) if (IN == 1 || i < a.I) u[i] = a.xs[((size_t)row * a.T + (t - 1)) * a.I + i + z];
  };
  if (sums) {
    if (n < H) {
      bias = a.b[n];
#pragma unroll
      for (int i = 0; i < IN; ++i) if (IN == 1 || i < a.I) V[i] = a.W_ih[(size_t)i * H + n];
    }
    prefetch(1);
  }
  for (int t = 1; t <= a.T; ++t) {
    float acc[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) acc[c] = 0.f;
    const float* const hv = &hs[(t - 1) & 1][w * KPW];
#pragma unroll
    for (int q4 = 0; q4 < KPW; q4 += 4) {
      const floatx4 h4 = *reinterpret_cast<const floatx4*>(hv + q4);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int c = 0; c < CPL; ++c) acc[c] = fmaf(h4[e], wr[c][q4 + e], acc[c]);
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c) part[w][c * 64 + lane] = acc[c];
    __syncthreads();
    if (sums) {
      float p0 = part[0][n], p1 = part[1][n];
#pragma unroll
      for (int q = 2; q < NW; q += 2) { p0 += part[q][n]; p1 += part[q + 1][n]; }
      float s = (p0 + p1) + bias;
#pragma unroll
      for (int i = 0; i < IN; ++i) if (IN == 1 || i < a.I) s = fmaf(u[i], V[i], s);
      hs[t & 1][n] = (n < H && s > 0.f) ? s : 0.f;
      if (t < a.T) prefetch(t + 1);
    }
    __syncthreads();
  }
}

template <class S, int IN>
__global__ __launch_bounds__(S::THREADS, 4) void rnn_backward_kernel(RnnArgs a) {
  constexpr int NW = S::NW, CPL = S::CPL, KPW = S::KPW, COLS = S::COLS, ROWS = S::ROWS;
  __shared__ __align__(16) float gl[2][ROWS];
  __shared__ float xl[2][COLS];              // sampled h that step t multiplies g_t with, in half t mod 2
  __shared__ float part[NW][COLS];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int H = a.H, z = opaque_zero();
  const size_t total = (size_t)H * H + (size_t)(1 + a.I) * H;
  float* const out = a.part + (size_t)blockIdx.x * total;
  for (int i = COLS + (int)threadIdx.x; i < ROWS; i += S::THREADS) gl[0][i] = gl[1][i] = 0.f;   // (the first barrier below)

  if (w >= NW) {
    // the waves off the chain, a column a lane: they bring the sampled rows in and sum db and dW_ih
    const int cw = w - NW, n = cw * 64 + lane;
    // (db and dW_ih are sums of every step: 8 steps at a time, so that hundreds of steps do not cost them digits)
    float db = 0.f, dV[IN], u[IN], db8 = 0.f, dV8[IN];
#pragma unroll
    for (int i = 0; i < IN; ++i) dV[i] = dV8[i] = u[i] = 0.f;
    for (int row = blockIdx.x; row < a.B; row += gridDim.x) {
      // sampled h of slot s (what step s + 2 multiplies g with), this lane's column; p: the row's plan
      auto fetch = [&](const RowPlan& p, int slot) {
        if (a.hh.exact) return n < H ? static_cast<const float*>(a.hh.v.values)[((size_t)slot * a.B + row) * H + n] : 0.f;
        uint32_t before;
        const uint64_t keep = keep_mask(p.words, cw, &before);
        const uint32_t pos = p.first + before + (uint32_t)lanes_below(keep);
        return ((keep >> lane) & 1u) && (int64_t)pos < a.hh.v.capacity ? static_cast<const float*>(a.hh.v.values)[pos] : 0.f;
      };
      auto prefetch = [&](int t) {           // input of step t
#pragma unroll
        for (int i = 0; i < IN; ++i) if (IN == 1 || i < a.I) u[i] = a.xs[((size_t)row * a.T + (t - 1)) * a.I + i + z];
      };
      RowPlan plan = {0u, 0u};
      float x = 0.f;                         // of slot t - 3, for step t - 1
      if (a.T >= 2) xl[a.T & 1][n] = fetch(row_plan(a.hh, a.T - 2, row, a.B, lane, z), a.T - 2);
      if (a.T >= 3) x = fetch(row_plan(a.hh, a.T - 3, row, a.B, lane, z), a.T - 3);
      if (a.T >= 4) plan = row_plan(a.hh, a.T - 4, row, a.B, lane, z);
      prefetch(a.T);
      __syncthreads();
      for (int t = a.T; t >= 1; --t) {
        const float g = gl[t & 1][n];
        db8 += g;
#pragma unroll
        for (int i = 0; i < IN; ++i) if (IN == 1 || i < a.I) dV8[i] = fmaf(u[i], g, dV8[i]);
        if ((t & 7) == 1) {                  // (t = 1, the last one, too)
          db += db8; db8 = 0.f;
#pragma unroll
          for (int i = 0; i < IN; ++i) { dV[i] += dV8[i]; dV8[i] = 0.f; }
        }
        if (t >= 2) prefetch(t - 1);
        __syncthreads();
        if (t >= 3) xl[(t - 1) & 1][n] = x;
        if (t >= 4) x = fetch(plan, t - 4);
        if (t >= 5) plan = row_plan(a.hh, t - 5, row, a.B, lane, z);
        __syncthreads();
      }
    }
    if (n < H) {
      out[(size_t)H * H + n] = db;
#pragma unroll
      for (int i = 0; i < IN; ++i) if (IN == 1 || i < a.I) out[(size_t)H * H + (size_t)(1 + i) * H + n] = dV[i];
    }
    return;
  }

  float wr[CPL][KPW], dw[CPL][KPW];          // W_hh[k][n] and dW_hh[k][n], k = lane + 64 c, n = w KPW + q
#pragma unroll
  for (int c = 0; c < CPL; ++c)
#pragma unroll
    for (int q = 0; q < KPW; ++q) {
      const int k = c * 64 + lane, n = w * KPW + q;
      wr[c][q] = (k < H && n < H) ? a.W_hh[(size_t)k * H + n] : 0.f;
      dw[c][q] = 0.f;
    }
  const bool sums = w < CPL;
  const int n = w * 64 + lane;
  for (int row = blockIdx.x; row < a.B; row += gridDim.x) {
    uint32_t mask = 0u;
    auto prefetch = [&](int t) {             // ReLU bits of step t - 1
      if (t >= 2 && (n >> 5) < a.bp) mask = a.bits[((size_t)(t - 2) * a.B + row) * a.bp + (n >> 5)];
    };
    if (sums) {
      gl[a.T & 1][n] = n < H ? a.gT[(size_t)row * H + n] : 0.f;
      prefetch(a.T);
    }
    __syncthreads();
    for (int t = a.T; t >= 1; --t) {
      const float* const gp = &gl[t & 1][w * KPW];
      float acc[CPL];
#pragma unroll
      for (int c = 0; c < CPL; ++c) acc[c] = 0.f;
#pragma unroll
      for (int q4 = 0; q4 < KPW; q4 += 4) {
        const floatx4 g4 = *reinterpret_cast<const floatx4*>(gp + q4);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int c = 0; c < CPL; ++c) acc[c] = fmaf(g4[e], wr[c][q4 + e], acc[c]);
      }
#pragma unroll
      for (int c = 0; c < CPL; ++c) part[w][c * 64 + lane] = acc[c];
      __syncthreads();
      if (sums) {
        float p0 = part[0][n], p1 = part[1][n];
#pragma unroll
        for (int q = 2; q < NW; q += 2) { p0 += part[q][n]; p1 += part[q + 1][n]; }
        gl[(t & 1) ^ 1][n] = ((mask >> (n & 31)) & 1u) ? p0 + p1 : 0.f;
        if (t >= 2) prefetch(t - 1);
      }
      if (t >= 2) {
        float x[CPL];
#pragma unroll
        for (int c = 0; c < CPL; ++c) x[c] = xl[t & 1][c * 64 + lane];
#pragma unroll
        for (int q4 = 0; q4 < KPW; q4 += 4) {
          const floatx4 g4 = *reinterpret_cast<const floatx4*>(gp + q4);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int c = 0; c < CPL; ++c) dw[c][q4 + e] = fmaf(x[c], g4[e], dw[c][q4 + e]);
        }
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int c = 0; c < CPL; ++c)
#pragma unroll
    for (int q = 0; q < KPW; ++q) {
      const int k = c * 64 + lane, nn = w * KPW + q;
      if (k < H && nn < H) out[(size_t)k * H + nn] = dw[c][q];
    }
}

// adds the workgroups' partial arrays, each output's in four interleaved sums (a fixed order)
__global__ __launch_bounds__(256) void rnn_reduce_kernel(const float* part, int groups, int H, int I, float* dW, float* db,
                                                         float* dV) {
  __shared__ float red[4][64];
  const int total = H * H + (1 + I) * H, e = blockIdx.x * 64 + (threadIdx.x & 63), w = threadIdx.x >> 6;
  float s = 0.f;
  if (e < total) {
#pragma unroll 8
    for (int g = w; g < groups; g += 4) s += part[(size_t)g * total + e];
  }
  red[w][threadIdx.x & 63] = s;
  __syncthreads();
  if (w != 0 || e >= total) return;
  s = (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
  if (e < H * H) dW[e] = s;
  else if (e < H * H + H) db[e - H * H] = s;
  else dV[e - H * H - H] = s;
}

// Up to 128 columns there are two shapes.  Ten waves make the shorter step while every example has a compute unit to
// itself, but two such workgroups do not run side by side on one; two of eight waves do.  A training step, T = 49,
// hidden 100, us, ten / eight waves: batch 16 101 / 115, 150 113 / 132, 256 124 / 142; 300 163 / 151, 1024 302 / 221,
// 4096 1072 / 647.
typedef RnnShape<4, 1, 16> Rnn64;
typedef RnnShape<8, 2, 16> Rnn128;
typedef RnnShape<6, 2, 24> Rnn128Pair;       // eight waves with the two off the chain: two workgroups on a compute unit
typedef RnnShape<12, 3, 16> Rnn192;

}  // namespace

int rnn_fused_max_hidden() { return Rnn192::COLS; }
int rnn_fused_groups(int B) { return B < 512 ? B : 512; }
int64_t rnn_fused_part_floats(int B, int H, int I) { return (int64_t)rnn_fused_groups(B) * ((int64_t)H * H + (int64_t)(1 + I) * H); }

template <class S> static void start(bool forward, dim3 grid, const RnnArgs& a, hipStream_t st) {
  auto kern = a.I == 1 ? (forward ? rnn_forward_kernel<S, 1> : rnn_backward_kernel<S, 1>)
                       : (forward ? rnn_forward_kernel<S, kMaxIn> : rnn_backward_kernel<S, kMaxIn>);
  hipLaunchKernelGGL(kern, grid, dim3(S::THREADS), 0, st, a);
}
static hipError_t start_for(bool forward, dim3 grid, const RnnArgs& a, hipStream_t st) {
  if (a.H < 1 || a.H > rnn_fused_max_hidden() || a.I < 1 || a.I > kMaxIn || a.B < 1 || a.T < 1) return hipErrorInvalidValue;
  if (a.H <= Rnn64::COLS) start<Rnn64>(forward, grid, a, st);
  else if (a.H <= Rnn128::COLS) a.B <= kComputeUnits ? start<Rnn128>(forward, grid, a, st) : start<Rnn128Pair>(forward, grid, a, st);
  else start<Rnn192>(forward, grid, a, st);
  return hipGetLastError();
}

hipError_t launch_rnn_forward(const RnnArgs& a, hipStream_t st) { return start_for(true, dim3(a.B), a, st); }

hipError_t launch_rnn_backward(const RnnArgs& a, float* dW_hh, float* db, float* dW_ih, hipStream_t st) {
  const dim3 grid(rnn_fused_groups(a.B));
  const hipError_t e = start_for(false, grid, a, st);
  if (e != hipSuccess) return e;
  const int total = a.H * a.H + (1 + a.I) * a.H;
  hipLaunchKernelGGL(rnn_reduce_kernel, dim3((total + 63) / 64), dim3(256), 0, st, a.part, (int)grid.x, a.H, a.I, dW_hh, db, dW_ih);
  return hipGetLastError();
}

}  // namespace rad
