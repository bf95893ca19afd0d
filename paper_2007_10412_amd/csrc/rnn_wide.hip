// The recurrent model with a hidden state of 193 to 1024 units: a chunk of time steps in one launch per direction.
//
// h_t = ReLU(x_t W_ih + h_{t-1} W_hh + b) and g_{t-1} = (g_t W_hh^T) under the ReLU bits are chains of small products
// (128 x 1024 x 1024: 1.9 us at the fp32 matrix rate) whose operand W_hh is the same at every step.  A launch per step
// pays the launch and reads W_hh again (7.6 us).  Here W_hh stays in the registers of the chip: the 32 CUs of one XCD hold
// it once, 32 columns each, and the eight XCDs take an eighth of the batch each.  Examples do not depend on each other,
// so the only exchange is that of a step's h (or g) among the workgroups of one XCD, through that XCD's L2.
//
// A workgroup of eight waves owns 16 NC columns; wave w multiplies k in [16 J w, 16 J (w + 1)) (16x16x4 matrix
// instructions), the waves' partial sums meet in LDS, the finished 16-column blocks go to the exchange buffer in the order
// in which the waves' A fragments are loaded (1 KB runs), and a flag per (block, accumulator element) says that a step's
// piece is there.  A wave waits only for the flags of its own k range (one 128-byte line), so a step has one workgroup
// barrier.  Two exchange buffers suffice: who publishes step s has read step s - 1 of everybody.
//
// A step takes 3.2 us forward and 3.6 backward at batch 128, hidden 1024, T = 784, its share of the launch included (3.6 and
// 4.1 with launches of 32 steps; 1.7 us of matrix instructions, then the
// latencies of the flags, of the fragments from L2 and of the sum through LDS).  A training step with fraction 0.1, a launch per
// step / this, us: batch 128, hidden 1024, T = 784 14757 / 8264 (9310 with chunks of 32 steps); T = 200: batch 192, hidden 1000 14777 / 4024, 192 x 640
// 3932 / 2545, 16 x 700 4153 / 1507; batch 40, hidden 300, T = 300 4806 / 1505.  A hidden state that does not fit 32 columns
// a CU keeps a launch per step, and so does a batch above 192 (rnn_wide_ok; the kernels for two row tiles hold up to 256).
//
// The workgroups find their XCD in the hardware register and take a place in it from a counter; the loads of flags and
// exchanged values pass by the L1 (agent scope, sc1), which is all the coherence that sharers of one L2 need.
// What has to hold and is not the library's to decide is that the workgroups of a group run side by side on one XCD (another
// kernel on some CUs, another partition mode).  Every wait is bounded: a workgroup that waited too long gives up and sets the
// launch's abort word.  A group that too few workgroups reached shows in its counter, also where nobody waits for it.
// rnn_wide_redo_kernel follows every launch, looks at both and, unless all is there, computes the chunk again without any
// exchange.  It also counts the launches that failed in a row and has the next ones come to it at once.
// Models of several contexts on streams of their own share the chip: a launch waits for the CUs that another one holds, and
// where the workgroups of two arrive together and each holds a part of an XCD, the one with the lower bound gives up and the
// other goes on (the bounds differ from context to context).  Steps of T = 200, ms for one of each context, a launch per step /
// this: three contexts 128 x 1024 9.4 / 7.9 (one launch in 35 computed again), two 192 x 1000 30.2 / 8.0, two 160 x 600 6.0 / 4.0
// (none).
// A launch of a long chunk that gives up costs its whole chunk on the stand-in (98 steps of 128 x 1024 8.4 ms forward, 12.3
// backward), but its waits are longer and fewer give up.  T = 784, ms for one step of each, chunks of 32 / of 98: three contexts
// 128 x 1024 28.0 / 26.1, two 192 x 1000 57.7 (one in 15 computed again) / 26.5 to 46.5 (none), three 160 x 600 23.1 / 21.7, 128
// x 1024 beside twenty bf16 products of 8192 49.8 (one in 100) / 47.3 to 51.8 (none); slower only 128 x 1024 beside 192 x 1000 of T = 300:
// 15.0 (none) / 15.4 to 16.4 (one in 35).
#include <algorithm>

#include "gemm.hpp"
#include "rnn_chunk.hpp"

namespace rad {

namespace {

constexpr int kWaves = 8, kGroups = kRnnWideGroups, kFlagsPerGroup = 256;     // flags: 64 blocks x 4 accumulator elements
constexpr int kXccIdReg = 20;                                                 // HW_REG_XCC_ID

__host__ __device__ constexpr int rows_per_group(int B) { return (B + kGroups - 1) / kGroups; }
constexpr int columns_per_member(int H) { return (H + 127) / 128 <= 4 ? 16 : 32; }
constexpr int members_of(int H) { return (H + columns_per_member(H) - 1) / columns_per_member(H); }

__device__ __forceinline__ float load_or_zero(const float* p, bool ok) { return ok ? *p : 0.f; }

template <int J, int NC, int R, bool FWD>
__global__ __launch_bounds__(64 * kWaves, R == 1 ? 4 : 2) void rnn_wide_kernel(RnnWideArgs a) {
  __shared__ float part[2][kWaves][R][NC][4][64];
  __shared__ float s_V[kRnnWideMaxIn + 1][16 * NC];       // W_ih and the bias of this workgroup's columns
  __shared__ int s_member, s_dead;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int r = lane & 15, kq = lane >> 4, H = a.H, B = a.B;
  const int xcc = (int)(__builtin_amdgcn_s_getreg((3 << 11) | kXccIdReg) & 15u);
  uint32_t* const abort_word = a.abort_words + a.launch;
  if (threadIdx.x == 0) {
    s_dead = 0;
    const bool counts = xcc < kGroups && !((a.absent >> xcc) & 1u);
    const uint32_t resume = a.backoff[1];
    s_member = counts ? (int)atomicAdd(a.tickets + a.launch * kGroups + xcc, 1u) : 0x7fffffff;
    if ((uint32_t)a.launch < resume) {                 // launches gave up just now: not yet again
      s_member = 0x7fffffff;
      __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();
  const int member = __builtin_amdgcn_readfirstlane(s_member), nblk = (H + 15) / 16;
  const int rg = rows_per_group(B), row0 = xcc * rg, row_end = min(B, row0 + rg);
  if (member >= a.members || row0 >= row_end) return;
  const int n0 = member * 16 * NC;

  float wr[J][4][NC];                        // W_hh[k][n] (forward) or W_hh[n][k], k = 16 (J w + j) + 4 kq + e
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int k = 16 * (J * w + j) + 4 * kq + e, n = n0 + 16 * c + r;
        const size_t at = FWD ? (size_t)k * H + n : (size_t)n * H + k;
        wr[j][e][c] = load_or_zero(a.W_hh + at, k < H && n < H);
      }

  // this wave finishes accumulator element fe of column block fc
  const int fc = NC == 2 ? w >> 2 : 0, fe = w & 3, blk = n0 / 16 + fc, col = 16 * blk + r;
  const bool finishes = (NC == 2 || w < 4) && blk < nblk, col_ok = col < H;
  if (FWD) {
    for (int q = threadIdx.x; q < (a.I + 1) * 16 * NC; q += 64 * kWaves) {
      const int i = q / (16 * NC), n = n0 + q % (16 * NC);
      s_V[i][q % (16 * NC)] = load_or_zero((i < a.I ? a.W_ih + (size_t)i * H : a.b) + n, n < H);
    }
    __syncthreads();
  }

  const size_t area = (size_t)kWaves * R * J * 256;            // floats of one exchange buffer of a group
  float* const xch[2] = {a.xch + (size_t)xcc * area, a.xch + (size_t)(kGroups + xcc) * area};
  uint32_t* const flags = a.flags + (size_t)xcc * kFlagsPerGroup;
  const int wait_flags = 4 * min(J, nblk - J * w);             // flags of this wave's k range; <= 0: all of it is padding
  uint16_t* const bits16 = reinterpret_cast<uint16_t*>(a.bits);

  for (int i = 0; i < a.n; ++i) {
    const int t = FWD ? a.t0 + i : a.t0 - i;                   // the step whose h_t or g_t is formed
    // what the epilogue adds or masks with, fetched now so that it has arrived by then
    float addend[R];
    uint32_t keep[R];
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
      const int row = min(row0 + 16 * rt + 4 * kq + fe, row_end - 1);
      addend[rt] = 0.f; keep[rt] = 0u;
      if (!finishes) continue;
      if (FWD) {
        addend[rt] = s_V[a.I][16 * fc + r];
        for (int q = 0; q < a.I; ++q)
          addend[rt] = fmaf(a.xs[((size_t)row * a.T + (t - 1)) * a.I + q], s_V[q][16 * fc + r], addend[rt]);
      } else {
        keep[rt] = bits16[((size_t)(t - 1) * B + row) * (2 * a.bp) + blk];
      }
    }
    floatx4 av[R][J], acc[R][NC];
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[rt][c] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < J; ++j) av[rt][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    if (i == 0) {
      if (a.src) {
#pragma unroll
        for (int rt = 0; rt < R; ++rt) {
          const int row = row0 + 16 * rt + r;
#pragma unroll
          for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int k = 16 * (J * w + j) + 4 * kq + e;
              av[rt][j][e] = load_or_zero(a.src + (size_t)row * H + k, row < row_end && k < H);
            }
        }
      }
    } else if (wait_flags > 0) {
      const uint32_t need = a.seq0 + (uint32_t)i - 1u;
      const uint32_t* const fl = flags + 4 * J * w + lane;
      uint32_t polls = 0;
      for (;;) {
        const uint32_t v = lane < wait_flags ? __hip_atomic_load(fl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : need;
        if (__all((int)(v - need) >= 0)) break;
        ++polls;
        if (polls >= a.poll_limit ||
            (polls % 64u == 0 && __hip_atomic_load(abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
          s_dead = 1;                        // seen by the whole workgroup at the barrier below
          if (lane == 0) __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
      }
      asm volatile("" ::: "memory");
      auto rsrc = __builtin_amdgcn_make_buffer_rsrc(xch[(i - 1) & 1] + (size_t)w * R * J * 256, 0, R * J * 1024, 0x00020000);
#pragma unroll
      for (int rt = 0; rt < R; ++rt)
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, (rt * J + j) * 1024, 16);     // sc1
          av[rt][j] = __builtin_bit_cast(floatx4, v);
        }
    }
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int rt = 0; rt < R; ++rt)
#pragma unroll
          for (int c = 0; c < NC; ++c)
            acc[rt][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[rt][j][e], wr[j][e][c], acc[rt][c], 0, 0, 0);
#pragma unroll
    for (int rt = 0; rt < R; ++rt)
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[i & 1][w][rt][c][e][lane] = acc[rt][c][e];
    __syncthreads();
    if (s_dead) return;
    if (finishes) {
      float v[R];
#pragma unroll
      for (int rt = 0; rt < R; ++rt) {
        const float* const p = &part[i & 1][0][rt][fc][fe][lane];
        constexpr int kStep = R * NC * 4 * 64;
        float s0 = p[0], s1 = p[kStep];
#pragma unroll
        for (int q = 2; q < kWaves; q += 2) { s0 += p[q * kStep]; s1 += p[(q + 1) * kStep]; }
        v[rt] = s0 + s1;
        if (FWD) { v[rt] += addend[rt]; v[rt] = v[rt] > 0.f ? v[rt] : 0.f; }
        else if (!((keep[rt] >> r) & 1u)) v[rt] = 0.f;
        if (!col_ok) v[rt] = 0.f;
        // element (row, column) of the block: fragment lane 16 (column / 4) + row, component column % 4
        float* const x = xch[i & 1] + ((size_t)(blk / J * R + rt) * J + blk % J) * 256;
        x[((r >> 2) * 16 + 4 * kq + fe) * 4 + (r & 3)] = v[rt];
      }
      if (i + 1 < a.n) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // the values are in L2
        if (lane == 0)
          __hip_atomic_store(flags + 4 * blk + fe, a.seq0 + (uint32_t)i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      // off the chain: dense output, ReLU bits
#pragma unroll
      for (int rt = 0; rt < R; ++rt) {
        const int row = row0 + 16 * rt + 4 * kq + fe;
        const bool row_ok = row < row_end;
        if (row_ok && col_ok) {
          if (t <= a.t_out) a.out[((size_t)(t - a.t_lo) * B + row) * H + col] = v[rt];
          if (i + 1 == a.n && a.carry) a.carry[(size_t)row * H + col] = v[rt];
        }
        if (FWD) {
          const uint64_t on = __ballot(v[rt] > 0.f);
          if (r == 0 && row_ok) {
            uint16_t* const word = bits16 + ((size_t)(t - 1) * B + row) * (2 * a.bp) + blk;
            word[0] = (uint16_t)(on >> (16 * kq));
            if (blk == nblk - 1 && (nblk & 1)) word[1] = 0;      // the padding half of the last word
          }
        }
      }
    }
  }
}

// Whether the launch before left anything out: a wait that ran out, or a group of examples that fewer workgroups reached
// than its columns take.  (The second does not follow from the first: a chunk of one step has no waits, and a group that
// nobody reached has nobody to wait.)
__device__ __forceinline__ bool left_out(const RnnWideArgs& a) {
  const int g = threadIdx.x & 63;
  const bool short_group = g < kGroups && g * rows_per_group(a.B) < a.B && a.tickets[a.launch * kGroups + min(g, kGroups - 1)] < (uint32_t)a.members;
  return __any(short_group) || a.abort_words[a.launch] != 0u;
}

// four consecutive numbers at element alignment, those past `n` zero
__device__ __forceinline__ floatx4 load4_or_zero(const float* p, int n) {
  floatx4 v = {0.f, 0.f, 0.f, 0.f};
  if (n >= 4) __builtin_memcpy(&v, p, 16);
  else {
#pragma unroll
    for (int e = 0; e < 3; ++e) if (e < n) v[e] = p[e];
  }
  return v;
}

// The chunk again if the launch before left something out (normally it returns at once).  A workgroup takes sixteen examples
// and all columns, so nothing is exchanged: h or g is in LDS in the order of the A fragments, and two groups of eight waves
// take the 16-column blocks in turn, with the products, the split of k over the waves and the order of every sum of
// rnn_wide_kernel, so that a step's numbers do not depend on which of the two computed it.  W_hh is read from L2 again every
// step by the few CUs that run, and sixteen rows are 55 us of matrix instructions for one of them at hidden 1024.  A step, us,
// forward / backward: 128 x 1024 86 / 125 (with an example at a time on the vector ALU 650 for either), 192 x 1000 93 / 98,
// 16 x 700 44 / 46, 40 x 300 13 / 14.  (The next block's columns loaded a block ahead: 116 / 150 in the first case.)
template <int J, bool FWD>
__global__ __launch_bounds__(128 * kWaves) void rnn_wide_redo_kernel(RnnWideArgs a) {
  const bool again = left_out(a);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    // [0] launches in a row that gave up, [1] the next one that tries: a wait that runs out costs a quarter of a chunk here, so
    // the first failure costs no launch and further ones more and more time steps (rnn_wide_skip)
    const uint32_t fails = a.backoff[0];
    if ((uint32_t)a.launch >= a.backoff[1]) {
      if (again) { a.backoff[0] = fails + 1u; a.backoff[1] = (uint32_t)a.launch + 1u + rnn_wide_skip(fails, a.chunk); }
      else if (fails) a.backoff[0] = 0u;
    }
    if (again) a.redone[a.launch] = 1u;
  }
  if (!again) return;
  __shared__ __align__(16) float state[kWaves * J * 256];
  __shared__ float part[2][2][kWaves][4][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int grp = wave / kWaves, w = wave % kWaves, r = lane & 15, kq = lane >> 4;
  const int H = a.H, B = a.B, nblk = (H + 15) / 16, row0 = 16 * (int)blockIdx.x;
  uint16_t* const bits16 = reinterpret_cast<uint16_t*>(a.bits);
  for (int q = threadIdx.x; q < kWaves * J * 64; q += 128 * kWaves) {       // fragment lane q % 64 of block q / 64
    const int row = row0 + (q & 15), k = q / 64 * 16 + (q % 64) / 16 * 4;
    const bool any = a.src && row < B && k < H;
    reinterpret_cast<floatx4*>(state)[q] = load4_or_zero(a.src + (any ? (size_t)row * H + k : 0), any ? H - k : 0);
  }
  auto W = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.W_hh), 0, H * H * 4, 0x00020000);
  // W_hh of this lane's column of a block, in the wave's range of k (what lies past the matrix reads as zero: rows k >= H are behind its
  // end, and so is a column that does not exist)
  floatx4 wr[J];
  auto load_columns = [&](int col) {
    const int k = 16 * J * w + 4 * kq;
    const uint32_t at = col >= H ? 0x40000000u : 4u * (uint32_t)(FWD ? k * H + col : col * H + k);
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if (FWD) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          wr[j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(W, at + 4u * (uint32_t)((16 * j + e) * H), 0, 0));
      } else {
        wr[j] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(W, at + 64u * (uint32_t)j, 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) wr[j][e] = k + 16 * j + e < H ? wr[j][e] : 0.f;
      }
    }
  };
  const int fe = w & 3, row = row0 + 4 * kq + fe;       // what a finishing wave (w < 4) adds up: element fe of each block
  const bool row_ok = row < B;
  for (int i = 0; i < a.n; ++i) {
    const int t = FWD ? a.t0 + i : a.t0 - i;
    __syncthreads();
    floatx4 av[J];
#pragma unroll
    for (int j = 0; j < J; ++j) av[j] = reinterpret_cast<const floatx4*>(state)[(J * w + j) * 64 + lane];
    for (int b0 = 0, par = 0; b0 < nblk; b0 += 2, par ^= 1) {
      const int blk = b0 + grp, col = 16 * blk + r;
      const bool col_ok = col < H, finishes = w < 4 && blk < nblk;
      float addend = 0.f;
      uint32_t keep = 0u;
      if (finishes && row_ok) {
        if (FWD) {
          addend = load_or_zero(a.b + col, col_ok);
          for (int q = 0; q < a.I; ++q)
            addend = fmaf(a.xs[((size_t)row * a.T + (t - 1)) * a.I + q], load_or_zero(a.W_ih + (size_t)q * H + col, col_ok), addend);
        } else {
          keep = bits16[((size_t)(t - 1) * B + row) * (2 * a.bp) + blk];
        }
      }
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
      load_columns(col);
#pragma unroll
      for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[j][e], wr[j][e], acc, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) part[par][grp][w][e][lane] = acc[e];
      __syncthreads();                       // (all waves hold av since the first of these: state may change)
      if (!finishes) continue;
      const float* const p = &part[par][grp][0][fe][lane];
      float s0 = p[0], s1 = p[4 * 64];
#pragma unroll
      for (int q = 2; q < kWaves; q += 2) { s0 += p[q * 4 * 64]; s1 += p[(q + 1) * 4 * 64]; }
      float v = s0 + s1;
      if (FWD) { v += addend; v = v > 0.f ? v : 0.f; }
      else if (!((keep >> r) & 1u)) v = 0.f;
      if (!col_ok) v = 0.f;
      state[blk * 256 + ((r >> 2) * 16 + 4 * kq + fe) * 4 + (r & 3)] = v;
      if (row_ok && col_ok) {
        if (t <= a.t_out) a.out[((size_t)(t - a.t_lo) * B + row) * H + col] = v;
        if (i + 1 == a.n && a.carry) a.carry[(size_t)row * H + col] = v;
      }
      if (FWD) {
        const uint64_t on = __ballot(v > 0.f);
        if (r == 0 && row_ok) {
          uint16_t* const word = bits16 + ((size_t)(t - 1) * B + row) * (2 * a.bp) + blk;
          word[0] = (uint16_t)(on >> (16 * kq));
          if (blk == nblk - 1 && (nblk & 1)) word[1] = 0;
        }
      }
    }
  }
}

template <int J, int NC> hipError_t start(bool forward, const RnnWideArgs& a, hipStream_t st) {
  static_assert(columns_per_member(128 * J) == 16 * NC, "members_of counts this kernel's workgroups");
  const bool two = a.B > 16 * kGroups;
  auto kern = two ? (forward ? rnn_wide_kernel<J, NC, 2, true> : rnn_wide_kernel<J, NC, 2, false>)
                  : (forward ? rnn_wide_kernel<J, NC, 1, true> : rnn_wide_kernel<J, NC, 1, false>);
  hipLaunchKernelGGL(kern, dim3(a.members * kGroups), dim3(64 * kWaves), 0, st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto redo = forward ? rnn_wide_redo_kernel<J, true> : rnn_wide_redo_kernel<J, false>;
  hipLaunchKernelGGL(redo, dim3((a.B + 15) / 16), dim3(128 * kWaves), 0, st, a);
  return hipGetLastError();
}

}  // namespace

// The batch: two row tiles a group are 256 examples, but those above 192 are still on the launch per step, though it is the slower
// one: T = 100, fraction 0.1, us, a launch per step / these kernels, 193 x 1000 7428 / 2032, 256 x 1000 7654 / 2221, 256 x 1024
// 3472 / 2146, 193 x 600 2334 / 1327, 256 x 600 4364 / 1435, 256 x 300 2174 / 893, 224 x 200 2015 / 1346.
bool rnn_wide_ok(int64_t B, int64_t H, int64_t I, int compute_units) {
  return H > rnn_fused_max_hidden() && H <= 1024 && B <= 24 * kGroups && I <= kRnnWideMaxIn && compute_units == 32 * kGroups;
}

size_t rnn_wide_sync_bytes(int B, int H, int launches) {
  const size_t J = (size_t)(H + 127) / 128, R = B > 16 * kGroups ? 2 : 1;
  return ((size_t)2 * kGroups * kWaves * R * J * 256 + (size_t)kGroups * kFlagsPerGroup + (size_t)launches * (kGroups + 2) + 2) * 4;
}

void rnn_wide_sync_layout(RnnWideArgs* a, void* ws, int launches) {
  const size_t J = (size_t)(a->H + 127) / 128, R = a->B > 16 * kGroups ? 2 : 1;
  a->xch = static_cast<float*>(ws);
  a->flags = reinterpret_cast<uint32_t*>(a->xch + (size_t)2 * kGroups * kWaves * R * J * 256);
  a->tickets = a->flags + (size_t)kGroups * kFlagsPerGroup;
  a->abort_words = a->tickets + (size_t)launches * kGroups;
  a->redone = a->abort_words + launches;
  a->backoff = a->redone + launches;
}

hipError_t launch_rnn_wide(bool forward, const RnnWideArgs& args, hipStream_t st) {
  RnnWideArgs a = args;
  if (!rnn_wide_ok(a.B, a.H, a.I, 32 * kGroups) || a.n < 1) return hipErrorInvalidValue;
  a.members = members_of(a.H);
  switch ((a.H + 127) / 128) {
    case 2: return start<2, 1>(forward, a, st);
    case 3: return start<3, 1>(forward, a, st);
    case 4: return start<4, 1>(forward, a, st);
    case 5: return start<5, 2>(forward, a, st);
    case 6: return start<6, 2>(forward, a, st);
    case 7: return start<7, 2>(forward, a, st);
    case 8: return start<8, 2>(forward, a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace rad
