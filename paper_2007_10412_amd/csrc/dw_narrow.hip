// dW of a narrow layer (class scores: few output columns) from a compressed store, fp32 sums.
//
// dW[j][n] = sum over rows b of x~[b][j] g[b][n] with N around ten: a matrix-core tile would be filled to a sixth and
// its output gives a handful of tiles, so the work is split over rows instead.  A wave takes one 256-column bucket and
// eight store rows at a time: it scatters their entries into a zeroed 8 x 256 LDS stage of its own (eight lanes per
// row), reads them back as four consecutive columns per lane and adds 4 x NT products per row to registers with g
// broadcast from LDS.  What bounds it is the vector ALU, 4 NT multiply-adds per row and wave (zeros included: at the
// usual fractions the dense form is as fast as read-modify-write of the sums in LDS and does not depend on the
// fraction), so the rows are split until the chip is full; the partial sums of a workgroup's four waves are added in
// LDS and those of the splits by the reduction kernel, both in a fixed order.
#include <algorithm>

#include "gemm.hpp"

namespace rad {

namespace {

constexpr int kRows = 8, kWaves = 4;         // store rows of a wave at a time, waves of a workgroup
constexpr int kLanes = 64 / kRows;           // lanes that share a store row
constexpr int kHeld = 4;                     // entries per lane in flight in registers (32 of a row's bucket)

struct NarrowArgs {
  StoreView s;
  int rows, N, M;
  const void* dy; int64_t ldy;
  const uint32_t* bits; int bits_pitch;
  float* out; int64_t split_stride;          // > 0: partial sums [split][M][N]; 0: out itself
  int beta, rows_per_split;
};

template <typename T> struct Entry;
template <> struct Entry<float> {
  static __device__ __forceinline__ void get(const StoreView& s, uint32_t e, int bucket, int* col, float* v) {
    *col = (int)s.indices[e] - bucket * kBucket;
    *v = reinterpret_cast<const float*>(s.values)[e];
  }
};
template <> struct Entry<uint16_t> {         // paired entries
  static __device__ __forceinline__ void get(const StoreView& s, uint32_t e, int, int* col, float* v) {
    const uint32_t u = reinterpret_cast<const uint32_t*>(s.values)[e];
    *col = pair_col(u, 0);
    *v = __uint_as_float(u & 0xFFFF0000u);
  }
};

template <typename T, int NT>
__global__ __launch_bounds__(64 * kWaves, 4) void dw_narrow_kernel(NarrowArgs a) {
  constexpr int NG = (kRows * NT + 63) / 64;             // values of g per lane and row group
  __shared__ __align__(16) float stage[kWaves][kRows * kBucket];
  __shared__ __align__(16) float gs[kWaves][kRows * NT];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int bucket = blockIdx.x, n0 = blockIdx.z * NT;
  const int rbeg = blockIdx.y * a.rows_per_split, rend = min(a.rows, rbeg + a.rows_per_split);
  const int rr = lane / kLanes, sub = lane % kLanes;
  float* const st = stage[w];
  float* const gw = gs[w];
  floatx4* const mine = reinterpret_cast<floatx4*>(st + lane * 4);       // this lane's columns of stage row 0
  const floatx4 z4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < kRows; ++q) mine[q * (kBucket / 4)] = z4;

  float acc[4][NT];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[j][n] = 0.f;

  uint32_t beg = 0, end = 0;
  int col[kHeld]; float val[kHeld]; float gv[NG];
  auto load_segment = [&](int r0) {
    const int row = r0 + rr;
    beg = end = 0u;
    if (row < rend) store_segment(a.s, row, bucket, &beg, &end);
  };
  auto load_rows = [&](int r0) {             // entries and g of the rows whose segment was loaded last
#pragma unroll
    for (int i = 0; i < kHeld; ++i) {
      const uint32_t e = beg + sub + i * kLanes;
      col[i] = -1; val[i] = 0.f;
      if (e < end) Entry<T>::get(a.s, e, bucket, &col[i], &val[i]);
    }
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int c = lane + 64 * q, row = r0 + c / NT, n = n0 + c % NT;
      gv[q] = 0.f;
      if ((kRows * NT % 64 == 0 || c < kRows * NT) && row < rend && n < a.N) {
        const float v = get_elem(static_cast<const T*>(a.dy) + (size_t)row * a.ldy + n);
        gv[q] = !a.bits || (mask_bits(a.bits, a.bits_pitch, row, n) & 1u) ? v : 0.f;
      }
    }
  };

  constexpr int kStep = kRows * kWaves;
  int r0 = rbeg + w * kRows;
  load_segment(r0);
  load_rows(r0);
  uint32_t cbeg = beg, cend = end;
  load_segment(r0 + kStep);
  for (; r0 < rend; r0 += kStep) {
    // scatter the held entries and whatever a row has beyond them; then the loads of the next rows are in flight
    // while these are multiplied
#pragma unroll
    for (int i = 0; i < kHeld; ++i) if (col[i] >= 0) st[rr * kBucket + col[i]] = val[i];
    for (uint32_t e = cbeg + sub + kHeld * kLanes; e < cend; e += kLanes) {
      int c; float v;
      Entry<T>::get(a.s, e, bucket, &c, &v);
      st[rr * kBucket + c] = v;
    }
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int c = lane + 64 * q;
      if (kRows * NT % 64 == 0 || c < kRows * NT) gw[c] = gv[q];
    }
    load_rows(r0 + kStep);
    cbeg = beg; cend = end;
    load_segment(r0 + 2 * kStep);
    __builtin_amdgcn_wave_barrier();         // the stage belongs to this wave: its LDS accesses complete in order
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const floatx4 x = mine[q * (kBucket / 4)];
      mine[q * (kBucket / 4)] = z4;
#pragma unroll
      for (int n4 = 0; n4 < NT / 4; ++n4) {
        const floatx4 g = *reinterpret_cast<const floatx4*>(&gw[q * NT + n4 * 4]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[j][n4 * 4 + e] = fmaf(x[j], g[e], acc[j][n4 * 4 + e]);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }

  // (0 + 2) + (1 + 3): half of the stage holds one wave's sums
  float* const all = &stage[0][0];
  static_assert(2 * kBucket * NT <= kWaves * kRows * kBucket, "two waves' sums fit the stage");
  auto put = [&](float* p) {
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) p[(n * 4 + j) * 64 + lane] = acc[j][n];
  };
  auto add = [&](const float* p) {
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j][n] += p[(n * 4 + j) * 64 + lane];
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
  float* const out = a.out + (int64_t)blockIdx.y * a.split_stride;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int m = bucket * kBucket + lane * 4 + j;
    if (m >= a.M) continue;
#pragma unroll
    for (int n = 0; n < NT; ++n)
      if (n0 + n < a.N) {
        float* dst = out + (size_t)m * a.N + n0 + n;
        *dst = a.beta ? *dst + acc[j][n] : acc[j][n];
      }
  }
}

template <typename T, int NT> hipError_t launch_nt(const NarrowArgs& a, int splits, hipStream_t st) {
  hipLaunchKernelGGL((dw_narrow_kernel<T, NT>), dim3((unsigned)a.s.nb, (unsigned)splits, (unsigned)((a.N + NT - 1) / NT)),
                     dim3(64 * kWaves), 0, st, a);
  return hipGetLastError();
}

template <typename T> hipError_t launch_t(const NarrowArgs& a, int nt, int splits, hipStream_t st) {
  switch (nt) {
    case 4: return launch_nt<T, 4>(a, splits, st);
    case 8: return launch_nt<T, 8>(a, splits, st);
    case 12: return launch_nt<T, 12>(a, splits, st);
    default: return launch_nt<T, 16>(a, splits, st);
  }
}

}  // namespace

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

// Whether this kernel is faster than the tile kernels, both sides measured (us of rad_backward_dW, tile kernel / here).
// bf16, whose tile kernel runs at 16 times the matrix rate with a split K, up to 12 columns: 65536 x 4096 x 10 792 / 130,
// 4096 x 1000 x 10 28 / 17, 150 x 784 x 10 12.8 / 9.2; with the sampling 16 columns 582 / 535 and 45 / 47, 32 582 / 647.
// Not 64 rows or fewer, a short contraction there and a pass of mostly latency here: 16 rows 3.8 / 5.6.
// fp32 up to 12 columns (100 x 4096 x 10 12.5 / 8.8, 65536 x 4096 x 10 7318 / 132), and wider where an estimate of each
// side says so.  The tile kernel walks all rows as one chain, 0.07 us a row and more with the tiles a CU has, nearly
// twice that where a bucket's entries take its wide loader, so the fraction counts; here a round of up to 1024 workgroups
// takes 3 to 5 us per group of 32 rows and every split writes and adds an array of partial sums.  The estimates are
// within 15 % of nine tenths of 1650 calls (65 to 8192 rows, 64 to 65535 columns, 4 to 8000 outputs, fractions 0.02 to
// 0.5), the choice within 11 % of the better side in all but five: at fraction 0.1 100 x 1024 x 100 12 / 13,
// 65 x 4096 x 128 8.8 / 19, 200 x 4096 x 128 19 / 32, 1000 x 65535 x 128 217 / 258, 4096 x 1000 x 128 306 / 47,
// 150 x 784 x 300 15 / 19, 300 x 784 x 300 25 / 28, 512 x 784 x 300 40 / 27, 512 x 1024 x 1024 41 / 48, 1024 x 1024 x 1024
// 79 / 64; at 0.5 300 x 784 x 300 47 / 30, 512 x 1024 x 1024 78 / 57.  Above a million outputs with more than 128 columns
// the two are close or unmeasured, and a grid's third axis holds 65535 parts.
bool dw_narrow_pays(int dtype, int rows, int cols, int N, int sparse_prefetch, bool masked) {
  if (rows <= 64) return false;
  if (dtype == kBF16 || N <= 12) return N <= 12;
  if (N > 128 && (N > 16384 || (int64_t)cols * N > (1 << 20))) return false;
  const bool wide = f32_sparse_wide(sparse_prefetch);
  const double out = (double)cols * N / 1e6, blocks = (double)narrow_blocks(cols, N);
  const int splits = dw_narrow_splits(rows, cols, N), per = (narrow_groups(rows) + splits - 1) / splits;
  const double group = 2.8 + (wide ? 2.0 : 0.4) * std::min(1.0, blocks * splits / 1024);
  const double here = 3.0 + 4.5 * narrow_nt(N) / 16 + per * std::max(1.0, blocks / 1024) * group + (splits > 1 ? 6.4 * splits * out : 0.0);
  const double tiles128 = ((cols + 127) / 128) * (double)((N + 127) / 128), tiles64 = ((cols + 63) / 64) * (double)((N + 63) / 64);
  const double load = tiles128 >= 192 ? tiles128 / 256 : tiles64 / 512;
  const double row = (wide ? 0.126 : 0.069) * std::max(1.0, load) + (wide ? 0.030 : 0.019) * std::min(1.0, load) + (masked ? 0.010 : 0.0);
  return here < 3.5 + rows * row;
}

hipError_t launch_dw_narrow(const StoreView& s, int dtype, int rows, const void* dy, int64_t ldy, int N,
                            const uint32_t* bits, int bits_pitch, float* out, int beta, int splits, int64_t split_stride,
                            hipStream_t st) {
  if (splits < 1 || splits > 128) return hipErrorInvalidValue;
  NarrowArgs a;
  a.s = s; a.rows = rows; a.N = N; a.M = s.cols; a.dy = dy; a.ldy = ldy; a.bits = bits; a.bits_pitch = bits_pitch;
  a.out = out; a.split_stride = split_stride; a.beta = beta;
  a.rows_per_split = (narrow_groups(rows) + splits - 1) / splits * (kRows * kWaves);
  return dtype == kBF16 ? launch_t<uint16_t>(a, narrow_nt(N), splits, st) : launch_t<float>(a, narrow_nt(N), splits, st);
}

}  // namespace rad
