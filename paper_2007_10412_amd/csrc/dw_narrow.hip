// dW of a narrow layer (class scores: few output columns) from a compressed store, fp32 sums.
//
// dW[j][n] = sum over rows b of x~[b][j] g[b][n] with N around ten: a 16- or 32-wide matrix-core tile would be filled to a
// part and its output gives a handful of tiles, so the work is split over rows instead.  A wave takes one 256-column bucket
// and eight store rows at a time: it scatters their entries into a zeroed 8 x 256 LDS stage of its own (eight lanes per
// row), reads them back as four consecutive columns per lane and adds 4 x NT products per row to registers with 4x4x1
// matrix instructions, g broadcast by them (zeros included: at the usual fractions the dense form is as fast as
// read-modify-write of the sums in LDS and does not depend on the fraction).  The rows are split until the chip is full;
// the partial sums of a workgroup's four waves are added in LDS and those of the splits by the reduction kernel, both in a
// fixed order.
// 65536 x 4096 fp32, 10 outputs, fraction 0.1: 110 us, about 41 each of matrix instructions, LDS and address arithmetic; 158
// with loads under conditions, which the wave waited for one by one, vector-ALU products and buckets of the same rows on
// different XCDs (matrix instructions alone 153, the regrouping 145).
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

#include "gemm.hpp"

namespace rad {

namespace {

constexpr int kRows = 8, kWaves = 4;         // store rows of a wave at a time, waves of a workgroup
constexpr int kLanes = 64 / kRows;           // lanes that share a store row

struct NarrowArgs {
  StoreView s;
  int rows, N, M;
  const void* dy; int64_t ldy;
  const uint32_t* bits; int bits_pitch;
  float* out; int64_t split_stride;          // > 0: partial sums [split][M][N]; 0: out itself
  int beta, rows_per_split;
};

// An entry as it is loaded (nothing is computed from it until it is scattered: arithmetic at the load would wait for it).
template <typename T> struct Entry;
template <> struct Entry<float> {
  float v; uint32_t c;
  __device__ __forceinline__ void load(const StoreView& s, uint32_t e) {
    c = s.indices[e];
    v = reinterpret_cast<const float*>(s.values)[e];
  }
  __device__ __forceinline__ int col() const { return c & (kBucket - 1); }          // inside its bucket
  __device__ __forceinline__ float value() const { return v; }
};
template <> struct Entry<uint16_t> {         // paired entries
  uint32_t u;
  __device__ __forceinline__ void load(const StoreView& s, uint32_t e) { u = reinterpret_cast<const uint32_t*>(s.values)[e]; }
  __device__ __forceinline__ int col() const { return pair_col(u, 0); }
  __device__ __forceinline__ float value() const { return __uint_as_float(u & 0xFFFF0000u); }
};

__device__ __forceinline__ float raw_value(float v) { return v; }
__device__ __forceinline__ float raw_value(uint32_t bf16) { return __uint_as_float(bf16 << 16); }

// row Q of the group: acc[j][n4] += g[row][4 n4 ..] x~[row][4 lane + j].  A 4x4x1 matrix instruction is sixteen outer
// products of four values each; the broadcast controls hand block ABID of the register that holds g (four of a row's
// values) to all sixteen, so g is never staged, and the second operand is the lane's column.
template <int NT, int Q, int... N4>
__device__ __forceinline__ void row_products(const float* gc, floatx4* mine, floatx4 (&acc)[4][NT / 4],
                                             std::integer_sequence<int, N4...>) {
  const floatx4 x = mine[Q * (kBucket / 4)];
  mine[Q * (kBucket / 4)] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 4; ++j)
    ((acc[j][N4] = __builtin_amdgcn_mfma_f32_4x4x1f32(gc[(Q * NT / 4 + N4) / 16], x[j], acc[j][N4], 4, (Q * NT / 4 + N4) % 16, 0)), ...);
}
template <int NT, int... Q>
__device__ __forceinline__ void products(const float* gc, floatx4* mine, floatx4 (&acc)[4][NT / 4], std::integer_sequence<int, Q...>) {
  (row_products<NT, Q>(gc, mine, acc, std::make_integer_sequence<int, NT / 4>()), ...);
}

// HELD: entries per lane and row group that are in flight in registers; what a row has beyond them is loaded when it is
// needed, a whole memory latency each time, so they cover a row's bucket nearly always.
// Loads are unconditional, at addresses clamped into the arrays, and what they bring is judged when it is used: a condition
// around a load, or arithmetic on its result beside it, made the wave wait for each load in turn.
template <typename T, int NT, int HELD, bool MASKED>
__global__ __launch_bounds__(64 * kWaves, NT == 16 || HELD > 5 ? 3 : 4) void dw_narrow_kernel(NarrowArgs a) {
  constexpr int NG = (kRows * NT + 63) / 64;             // values of g per lane and row group
  __shared__ __align__(16) float stage[kWaves][kRows * kBucket];
  __shared__ float spare[kWaves][64];                    // where slots without an entry go
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // Workgroups go round-robin over the eight XCDs: all buckets of a range of rows on one of them, whose L2 then holds the
  // cache lines that the segments of neighbouring buckets share.
  const int id = blockIdx.x + a.s.nb * blockIdx.y, whole = (int)gridDim.y / 8 * 8;
  const bool regroup = id < whole * a.s.nb;
  const int bucket = regroup ? id / 8 % a.s.nb : (int)blockIdx.x;
  const int split = regroup ? id / 8 / a.s.nb * 8 + id % 8 : (int)blockIdx.y;
  const int n0 = blockIdx.z * NT;
  const int rbeg = split * a.rows_per_split, rend = min(a.rows, rbeg + a.rows_per_split);
  const int rr = lane / kLanes, sub = lane % kLanes;
  float* const st = stage[w];
  float* const none = spare[w] + lane;
  floatx4* const mine = reinterpret_cast<floatx4*>(st + lane * 4);       // this lane's columns of stage row 0
  const floatx4 z4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < kRows; ++q) mine[q * (kBucket / 4)] = z4;

  floatx4 acc[4][NT / 4];                    // dW of column 4 lane + j, outputs 4 n4 .. 4 n4 + 3
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int n4 = 0; n4 < NT / 4; ++n4) acc[j][n4] = z4;

  // g value c = lane + 64 q of a row group: row c / NT of the group, output n0 + c % NT
  int g_row[NG], g_n[NG]; bool g_ok[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    const int c = min(lane + 64 * q, kRows * NT - 1);
    g_row[q] = c / NT;
    g_ok[q] = lane + 64 * q < kRows * NT && n0 + c % NT < a.N;
    g_n[q] = min(n0 + c % NT, a.N - 1);
  }
  struct Bounds { uint32_t base, b0, b1; };     // of a row's segment, as loaded
  const uint32_t last = (uint32_t)(a.s.capacity - 1);
  Entry<T> ent[HELD];
  typedef typename std::conditional<sizeof(T) == 2, uint32_t, float>::type Raw;
  Raw gv[NG];
  uint32_t gm[MASKED ? NG : 1];
  uint32_t beg, end;                                     // segment of the row in flight
  auto load_bounds = [&](int r0) {
    const int row = min(r0 + rr, rend - 1);
    const uint16_t* const bo = a.s.bucket_off + (size_t)(row * a.s.plan_row_stride) * (a.s.nb + 1) + bucket;
    return Bounds{a.s.row_ptr[row], bo[0], bo[1]};
  };
  auto load_rows = [&](int r0, Bounds b) {               // entries and g of a row group
    const uint32_t cap = (uint32_t)a.s.capacity;         // (an overflowed draw never reads past the arrays)
    end = min(b.base + b.b1, cap);
    beg = r0 + rr < rend ? min(b.base + b.b0, end) : end;
#pragma unroll
    for (int i = 0; i < HELD; ++i) ent[i].load(a.s, min(beg + sub + i * kLanes, last));
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int row = min(r0 + g_row[q], rend - 1);
      gv[q] = static_cast<const T*>(a.dy)[(size_t)row * a.ldy + g_n[q]];
      if (MASKED) gm[MASKED ? q : 0] = a.bits[(size_t)row * a.bits_pitch + (g_n[q] >> 5)];
    }
  };

  constexpr int kStep = kRows * kWaves;
  const int r_first = rbeg + w * kRows;
  load_rows(r_first, load_bounds(r_first));
  Bounds next = load_bounds(r_first + kStep);
  for (int r0 = r_first; r0 < rend; r0 += kStep) {
    // scatter the held entries and whatever a row has beyond them; then the loads of the group after those in flight
    // start, and these rows are multiplied
#pragma unroll
    for (int i = 0; i < HELD; ++i) {
      float* const at = st + rr * kBucket + ent[i].col();
      *(beg + sub + i * kLanes < end ? at : none) = ent[i].value();
    }
    for (uint32_t e = beg + sub + HELD * kLanes; e < end; e += kLanes) {
      Entry<T> x;
      x.load(a.s, e);
      st[rr * kBucket + x.col()] = x.value();
    }
    float gc[NG];                          // g of these rows: value q NT + n of the group in lane (q NT + n) % 64
#pragma unroll
    for (int q = 0; q < NG; ++q)
      gc[q] = g_ok[q] && r0 + g_row[q] < rend && (!MASKED || ((gm[MASKED ? q : 0] >> (g_n[q] & 31)) & 1u)) ? raw_value(gv[q]) : 0.f;
    load_rows(r0 + kStep, next);
    next = load_bounds(r0 + 2 * kStep);
    __builtin_amdgcn_wave_barrier();       // the stage belongs to this wave: its LDS accesses complete in order
    products<NT>(gc, mine, acc, std::make_integer_sequence<int, kRows>());
    __builtin_amdgcn_wave_barrier();
  }

  // (0 + 2) + (1 + 3): half of the stage holds one wave's sums
  float* const all = &stage[0][0];
  static_assert(2 * kBucket * NT <= kWaves * kRows * kBucket, "two waves' sums fit the stage");
  auto put = [&](float* p) {
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) p[(n * 4 + j) * 64 + lane] = acc[j][n / 4][n % 4];
  };
  auto add = [&](const float* p) {
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j][n / 4][n % 4] += p[(n * 4 + j) * 64 + lane];
  };
  __syncthreads();
  if (w >= 2) put(all + (w - 2) * kBucket * NT);
  __syncthreads();
  if (w < 2) add(all + w * kBucket * NT);
  __syncthreads();
  if (w == 1) put(all);
  __syncthreads();
  if (w != 0) return;
  add(all);
  float* const out = a.out + (int64_t)split * a.split_stride;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int m = bucket * kBucket + lane * 4 + j;
    if (m >= a.M) continue;
#pragma unroll
    for (int n = 0; n < NT; ++n)
      if (n0 + n < a.N) {
        float* dst = out + (size_t)m * a.N + n0 + n;
        *dst = a.beta ? *dst + acc[j][n / 4][n % 4] : acc[j][n / 4][n % 4];
      }
  }
}

template <typename T, int NT, int HELD> hipError_t launch_held(const NarrowArgs& a, int splits, hipStream_t st) {
  auto kern = a.bits ? dw_narrow_kernel<T, NT, HELD, true> : dw_narrow_kernel<T, NT, HELD, false>;
  hipLaunchKernelGGL(kern, dim3((unsigned)a.s.nb, (unsigned)splits, (unsigned)((a.N + NT - 1) / NT)), dim3(64 * kWaves), 0, st, a);
  return hipGetLastError();
}
template <typename T, int NT> hipError_t launch_nt(const NarrowArgs& a, int entries, int splits, hipStream_t st) {
  if (entries <= 3 * kLanes) return launch_held<T, NT, 3>(a, splits, st);
  if (entries <= 5 * kLanes) return launch_held<T, NT, 5>(a, splits, st);
  return launch_held<T, NT, 10>(a, splits, st);
}
template <typename T> hipError_t launch_t(const NarrowArgs& a, int nt, int entries, int splits, hipStream_t st) {
  switch (nt) {
    case 4: return launch_nt<T, 4>(a, entries, splits, st);
    case 8: return launch_nt<T, 8>(a, entries, splits, st);
    case 12: return launch_nt<T, 12>(a, entries, splits, st);
    default: return launch_nt<T, 16>(a, entries, splits, st);
  }
}

// ---------------------------------------------------------------------------------------------------- few rows, fp32
// dW of a layer with up to 256 rows: bound by latencies, of which the tile kernel has one chain per 16 rows (bounds, entries,
// scatter, barrier).  Here the rows of a 32 x 32 output tile are shared out to eight waves, at most 32 to each: a wave loads
// all of its bounds, entries and g at once, scatters the entries into an LDS stage of its own, multiplies 32x32x2 and the
// eight sums meet in LDS: one barrier.
// rad_backward_dW with 10 % of the columns and no mask, us, tile kernel / this: 150 x 784 x 300 11.8 / 5.5, 64 x 784 x 300 6.5 /
// 5.4, 256 x 784 x 300 17.3 / 5.7, 256 x 1024 x 1024 17.9 / 14.5; row split / this: 150 x 300 x 300 11.7 / 5.2.  Every workgroup
// reads the whole bucket's entries for its 32 columns, so it loses with many tiles: 150 x 2048 x 1024 15.7 / 25.4.
constexpr int kSmallWaves = 8, kSmallTile = 32, kSmallRows = 32;       // rows of a wave at most
constexpr int kSmallPasses = kSmallRows / kRows, kSmallHeld = 10;      // entries a lane of a row holds at most

template <int HELD, bool MASKED>
__global__ __launch_bounds__(64 * kSmallWaves) void dw_small_kernel(NarrowArgs a) {
  __shared__ __align__(16) float stage[kSmallWaves][kSmallRows * kSmallTile];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int m0 = (int)blockIdx.x * kSmallTile, n0 = (int)blockIdx.y * kSmallTile, bucket = m0 / kBucket;
  const int r0 = w * a.rows_per_split, rend = min(a.rows, r0 + a.rows_per_split);      // an even number of rows a wave
  float* const st = stage[w];
  const uint32_t cap = (uint32_t)a.s.capacity;             // (an overflowed draw never reads past the arrays)

  // g of the wave's rows in the order of the B operand; loads are unconditional at clamped addresses
  const int n = min(n0 + (lane & 31), a.N - 1), hi = lane >> 5;
  float gv[kSmallRows / 2];
  uint32_t gm[MASKED ? kSmallRows / 2 : 1];
#pragma unroll
  for (int j = 0; j < kSmallRows / 2; ++j) {
    const int row = min(r0 + 2 * j + hi, a.rows - 1);
    gv[j] = static_cast<const float*>(a.dy)[(size_t)row * a.ldy + n];
    if (MASKED) gm[MASKED ? j : 0] = a.bits[(size_t)row * a.bits_pitch + (n >> 5)];
  }
  uint32_t beg[kSmallPasses], end[kSmallPasses];           // segment of row r0 + 8 q + lane / 8 in this bucket
  {
    uint32_t base[kSmallPasses], b0[kSmallPasses], b1[kSmallPasses];
#pragma unroll
    for (int q = 0; q < kSmallPasses; ++q) {
      const int row = min(r0 + q * kRows + lane / kLanes, a.rows - 1);
      const uint16_t* const bo = a.s.bucket_off + (size_t)(row * a.s.plan_row_stride) * (a.s.nb + 1) + bucket;
      base[q] = a.s.row_ptr[row]; b0[q] = bo[0]; b1[q] = bo[1];
    }
#pragma unroll
    for (int q = 0; q < kSmallPasses; ++q) {
      end[q] = min(base[q] + b1[q], cap);
      beg[q] = (r0 + q * kRows + lane / kLanes < rend ? min(base[q] + b0[q], end[q]) : end[q]) + lane % kLanes;
    }
  }
  const float* const vals = reinterpret_cast<const float*>(a.s.values);
  float val[kSmallPasses][HELD];
  uint32_t col[kSmallPasses][HELD];
#pragma unroll
  for (int q = 0; q < kSmallPasses; ++q)
#pragma unroll
    for (int i = 0; i < HELD; ++i) {
      const uint32_t e = min(beg[q] + i * kLanes, cap - 1u);
      col[q][i] = a.s.indices[e]; val[q][i] = vals[e];
    }
  const floatx4 z4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < kSmallRows * kSmallTile / 256; ++q) reinterpret_cast<floatx4*>(st)[q * 64 + lane] = z4;
  __builtin_amdgcn_wave_barrier();                         // the stage belongs to this wave: its accesses complete in order
#pragma unroll
  for (int q = 0; q < kSmallPasses; ++q) {
    float* const at = st + (q * kRows + lane / kLanes) * kSmallTile;
#pragma unroll
    for (int i = 0; i < HELD; ++i) {
      const uint32_t c = col[q][i] - (uint32_t)m0;
      if (beg[q] + i * kLanes < end[q] && c < (uint32_t)kSmallTile) at[c] = val[q][i];
    }
    for (uint32_t e = beg[q] + HELD * kLanes; e < end[q]; e += kLanes) {
      const uint32_t c = a.s.indices[e] - (uint32_t)m0;
      if (c < (uint32_t)kSmallTile) at[c] = vals[e];
    }
  }
  __builtin_amdgcn_wave_barrier();
  floatx16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  const bool n_ok = n0 + (lane & 31) < a.N;
#pragma unroll
  for (int j = 0; j < kSmallRows / 2; ++j) {
    const bool ok = n_ok && r0 + 2 * j + hi < rend && (!MASKED || ((gm[MASKED ? j : 0] >> (n & 31)) & 1u));
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(st[(2 * j + hi) * kSmallTile + (lane & 31)], ok ? gv[j] : 0.f, acc, 0, 0, 0);
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int e = 0; e < 16; ++e) st[e * 64 + lane] = acc[e];
  __syncthreads();
  // wave w adds accumulator elements 2 w and 2 w + 1 of all waves
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int e = 2 * w + u, m = m0 + acc_row(e, lane);
    float v = stage[0][e * 64 + lane];
#pragma unroll
    for (int q = 1; q < kSmallWaves; ++q) v += stage[q][e * 64 + lane];
    if (m < a.M && n_ok) {
      float* const dst = a.out + (size_t)m * a.N + n;
      *dst = a.beta ? *dst + v : v;
    }
  }
}

template <int HELD> hipError_t launch_small_held(const NarrowArgs& a, hipStream_t st) {
  auto kern = a.bits ? dw_small_kernel<HELD, true> : dw_small_kernel<HELD, false>;
  hipLaunchKernelGGL(kern, dim3((unsigned)((a.M + kSmallTile - 1) / kSmallTile), (unsigned)((a.N + kSmallTile - 1) / kSmallTile)),
                     dim3(64 * kSmallWaves), 0, st, a);
  return hipGetLastError();
}

}  // namespace

// entries of a row's bucket that a kernel is chosen for (a row with more: one in a hundred)
static int bucket_entries(int cols, double kept) {
  const double mean = kept * std::min(cols, kBucket);
  return (int)(mean + 2.5 * std::sqrt(mean));
}

// rows of a wave of dw_small_kernel
static int small_rows_per_wave(int rows) { return ((rows + kSmallWaves - 1) / kSmallWaves + 1) / 2 * 2; }

hipError_t launch_dw_small(const StoreView& s, int rows, const void* dy, int64_t ldy, int N, const uint32_t* bits, int bits_pitch,
                           float* out, int beta, double kept, hipStream_t st) {
  if (rows < 1 || rows > kSmallWaves * kSmallRows) return hipErrorInvalidValue;
  NarrowArgs a;
  a.s = s; a.rows = rows; a.N = N; a.M = s.cols; a.dy = dy; a.ldy = ldy; a.bits = bits; a.bits_pitch = bits_pitch;
  a.out = out; a.split_stride = 0; a.beta = beta;
  a.rows_per_split = small_rows_per_wave(rows);
  const int entries = bucket_entries(s.cols, kept);
  if (entries <= 3 * kLanes) return launch_small_held<3>(a, st);
  if (entries <= 5 * kLanes) return launch_small_held<5>(a, st);
  return launch_small_held<kSmallHeld>(a, st);
}

// columns per workgroup: the output width in equal parts of at most 16, rounded up to whole vectors
static int narrow_nt(int N) {
  const int parts = (N + 15) / 16;
  return ((N + parts - 1) / parts + 3) / 4 * 4;
}

static int64_t narrow_blocks(int cols, int N) {             // workgroups of one split
  const int nt = narrow_nt(N);
  return (int64_t)((cols + kBucket - 1) / kBucket) * ((N + nt - 1) / nt);
}
static int narrow_groups(int rows) { return (rows + kRows * kWaves - 1) / (kRows * kWaves); }

// four workgroups per CU fit; a split takes whole groups of the workgroup's 32 rows
int dw_narrow_splits(int rows, int cols, int N) {
  const int64_t blocks = narrow_blocks(cols, N);
  int64_t splits = blocks < 1024 ? 1024 / blocks : 1;       // rounded down: one wave of workgroups and no remainder
  const int groups = narrow_groups(rows);
  if (splits > groups) splits = groups;
  if (splits > 128) splits = 128;
  const int per = (int)((groups + splits - 1) / splits);
  return (groups + per - 1) / per;
}

// us of the fp32 tile kernel, which walks all rows as one chain (see dw_narrow_pays)
static double dw_tile_estimate(int rows, int cols, int N, int sparse_prefetch, bool masked) {
  const bool wide = f32_sparse_wide(sparse_prefetch);
  const double tiles128 = ((cols + 127) / 128) * (double)((N + 127) / 128), tiles64 = ((cols + 63) / 64) * (double)((N + 63) / 64);
  const double load = tiles128 >= 192 ? tiles128 / 256 : tiles64 / 512;
  const double row = (wide ? 0.095 : 0.056) * std::max(1.0, load) + (wide ? 0.023 : 0.018) * std::min(1.0, load) + (masked ? 0.009 : 0.0);
  const double edge = tiles128 >= 192 && (cols % 128 || N % 128) ? 1.33 : 1.0;         // guarded loads on a full chip
  return 3.7 + rows * row * edge;
}

// us of dw_narrow_kernel and the reduction behind it (see dw_narrow_pays)
static double dw_narrow_estimate(int rows, int cols, int N, double kept) {
  const double out = (double)cols * N / 1e6, blocks = (double)narrow_blocks(cols, N);
  const int splits = dw_narrow_splits(rows, cols, N), per = (narrow_groups(rows) + splits - 1) / splits;
  const double group = 0.5 + (1.6 + 0.030 * kept * std::min(cols, kBucket)) * std::min(1.0, blocks * splits / 1024);
  return 3.4 * narrow_nt(N) / 16 + per * std::max(1.0, blocks / 1024) * group + (splits > 1 ? 4.7 + 6.3 * splits * out : 24.7);
}

// Whether this kernel is faster than the tile kernels, both sides measured (us of rad_backward_dW, tile kernel / here).
// bf16, whose tile kernel runs at 16 times the matrix rate with a split K, up to 12 columns: 65536 x 4096 x 10 792 / 130,
// 4096 x 1000 x 10 28 / 17, 150 x 784 x 10 12.8 / 9.2; with the sampling 16 columns 582 / 535 and 45 / 47, 32 582 / 647.
// Not 64 rows or fewer, a short contraction there and a pass of mostly latency here: 16 rows 3.8 / 5.6.
// fp32 up to 12 columns (100 x 4096 x 10 12.5 / 8.8, 65536 x 4096 x 10 7318 / 110), and wider where an estimate of each
// side says so.  The tile kernel walks all rows as one chain, 0.056 us a row and more with the tiles a CU has, nearly
// twice that where a bucket's entries take its wide loader, so the fraction counts; here a round of up to 1024 workgroups
// takes 2 us and 0.03 an entry of a row's bucket per group of 32 rows, and every split writes and adds an array of partial
// sums.  Fitted to 908 pairs of calls (65 to 8192 rows, 64 to 65535 columns, 10 to 8000 outputs, fractions 0.02 to 0.5): the
// estimates are within 15 and 10 % of nine tenths of them, the choice within 10 % of the better side in all but one
// (by 14 %).  At fraction 0.1 100 x 1024 x 128 9.1 / 10.8,
// 65 x 4096 x 128 7.5 / 17, 200 x 4096 x 128 15 / 31, 150 x 784 x 300 12 / 18, 300 x 784 x 300 20 / 25, 512 x 784 x 300
// 32 / 26, 512 x 1024 x 1024 32 / 44, 1024 x 1024 x 1024 61 / 54, 8192 x 1100 x 1000 599 / 270; at 0.5 300 x 784 x 300
// 31 / 27, 512 x 1024 x 1024 51 / 56, 1024 x 2048 x 1024 125 / 130.  Above 2.2 million outputs with more than 128 columns
// nothing is measured.
// kept: the fraction of a row's columns that the store holds
bool dw_narrow_pays(int dtype, int rows, int cols, int N, int sparse_prefetch, bool masked, double kept) {
  if (rows <= 64) return false;
  if (dtype == kBF16 || N <= 12) return N <= 12;
  if (N > 128 && (N > 16384 || (int64_t)cols * N > 2200000)) return false;
  // (the factor that loses least over the pairs)
  return dw_narrow_estimate(rows, cols, N, kept) < 1.04 * dw_tile_estimate(rows, cols, N, sparse_prefetch, masked);
}

// us of dw_small_kernel: its start and 2.6 (5.6 where its lanes hold ten entries of a row, which leaves two waves a SIMD) for
// every workgroup a CU takes one after the other, more under a mask; entries beyond those held cost 0.2 a round of eight lanes.
static double dw_small_estimate(int rows, int cols, int N, bool masked, double kept) {
  const int entries = bucket_entries(cols, kept);
  const double round = entries <= 5 * kLanes ? 2.6 : 5.6, start = entries <= 3 * kLanes ? 2.2 : entries <= 5 * kLanes ? 2.6 : 0.9;
  const double tiles = ((cols + kSmallTile - 1) / kSmallTile) * (double)((N + kSmallTile - 1) / kSmallTile) / 256;
  const int passes = (small_rows_per_wave(rows) + kRows - 1) / kRows;
  const double beyond = passes * std::max(0.0, kept * std::min(cols, kBucket) - kSmallHeld * kLanes) / kLanes;
  return start + round * (tiles > 1 ? tiles + 0.6 : 1.0) * (masked ? 1.15 : 1.0) + (masked ? 0.5 : 0.0) + 0.2 * beyond * std::max(1.0, tiles);
}

// Whether it is faster than the tile kernel and, where that one is, than dw_narrow_kernel (see dw_narrow_pays): estimates of
// both sides.  Fitted to 1088 pairs of calls (1 to 256 rows, 32 to 5800 columns, 14 to 4000 outputs, fractions 0.01 to 0.8, with
// and without a mask): nine tenths of the estimates are within 12 %, and with the factor the choice is behind the other side by
// more than 3 % in one pair (12 %), in none of 1400 further ones.  us, the other side / here: at fraction 0.1 256 x 512 x 2048
// 17.9 / 13.6; at 0.25 105 x 141 x 3927 under a mask 16.4 / 19.9; at 0.6 235 x 230 x 2396 25.8 / 34.0; at 0.8 145 x 3087 x 90
// 21.8 / 29.4.  Rows with more entries in a bucket than the registers hold keep the row split where that is ahead of the tiles,
// though it is often the slower one (175 x 701 x 347 at 0.35 19.0 / 9.5).  Up to twelve outputs dw_narrow_kernel and the tiles stay.
bool dw_small_pays(int dtype, int rows, int cols, int N, int sparse_prefetch, bool masked, double kept) {
  if (dtype != kF32 || rows > kSmallWaves * kSmallRows || N <= 12) return false;
  if (N > 65535 * kSmallTile) return false;                    // the grid's second axis
  double other = dw_tile_estimate(rows, cols, N, sparse_prefetch, masked);
  if (dw_narrow_pays(dtype, rows, cols, N, sparse_prefetch, masked, kept)) {
    if (bucket_entries(cols, kept) > kSmallHeld * kLanes) return false;
    other = dw_narrow_estimate(rows, cols, N, kept);
  }
  return dw_small_estimate(rows, cols, N, masked, kept) < 0.85 * other;
}

hipError_t launch_dw_narrow(const StoreView& s, int dtype, int rows, const void* dy, int64_t ldy, int N,
                            const uint32_t* bits, int bits_pitch, float* out, int beta, int splits, int64_t split_stride,
                            double kept, hipStream_t st) {
  if (splits < 1 || splits > 128) return hipErrorInvalidValue;
  NarrowArgs a;
  a.s = s; a.rows = rows; a.N = N; a.M = s.cols; a.dy = dy; a.ldy = ldy; a.bits = bits; a.bits_pitch = bits_pitch;
  a.out = out; a.split_stride = split_stride; a.beta = beta;
  a.rows_per_split = (narrow_groups(rows) + splits - 1) / splits * (kRows * kWaves);
  const int entries = bucket_entries(s.cols, kept);
  return dtype == kBF16 ? launch_t<uint16_t>(a, narrow_nt(N), entries, splits, st)
                        : launch_t<float>(a, narrow_nt(N), entries, splits, st);
}

}  // namespace rad
