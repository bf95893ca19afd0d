// fp32 GEMM for few output tiles (a time step of the recurrent model, Appendix A: 128 x 1024 x 1024; the layers of small
// networks): one launch, no partial sums through memory.  A workgroup of eight waves owns a 16 x 32
// output tile (256 workgroups for the recurrent step: one per CU); every wave takes a share of K, brings its own
// operand slices in through a private LDS area and runs two chains of v_mfma_f32_16x16x4_f32 (the tile's two
// 16-column halves); the waves' accumulators meet in LDS, are added in wave order, and the tile's epilogue
// runs in the same kernel: forward (bias, low-rank input term, ReLU, bits) or dX (output mask of the layer
// below).  Splitting K over workgroups instead needs a second launch to add the splits (the time steps are a
// chain of dependent launches, so a launch is what a step costs), and adding them in the same kernel needs
// device-coherent traffic between XCDs, which measured slower than the second launch.
#include "gemm.hpp"

namespace rad {

namespace {

// Workgroups of eight waves, or of four (half the LDS, so that three share a CU) where there are more tiles than CUs.
constexpr int kKsWavesMax = 8;

// A wave's operand slices reach the MFMA through its own LDS area, 64 k at a time.  K-contiguous operands (A; for
// dX also B) are loaded with whole 256-byte rows per 16 lanes and stored [rows][64 k] at a pitch of 65 floats, so
// that lane (r = lane % 16, kq = lane / 16) reads element [r][4s + kq] of step s without bank conflicts between
// rows.  An N-contiguous B (forward) is kept as it lies in memory, [64 k][32 n].  Only the wave itself touches its
// area, so there is no workgroup barrier before the final sum.
// BK_CONTIG: B is K-contiguous (B[n * ldb + k], dX) or N-contiguous (B[k * ldb + n], forward).
constexpr int kKsPitch = 65, kKsHalf = 64;
constexpr int kKsAreaA = 16 * kKsPitch, kKsAreaB = 32 * kKsPitch;       // floats (B: the larger of the two layouts)

// EDGE: any M, N, K and alignment: rows past the edge read the last row, columns and k past the end are zeros, 16-byte
// loads at element alignment, guarded stores.
__device__ __forceinline__ floatx4 load4_any(const float* p, int n) {        // the first n elements, zeros after them
  floatx4 t = {0.f, 0.f, 0.f, 0.f};
  if (n >= 4) __builtin_memcpy(&t, p, 16);
  else {
#pragma unroll
    for (int e = 0; e < 3; ++e) if (e < n) t[e] = p[e];
  }
  return t;
}

template <bool BK_CONTIG, int FINISH, bool EDGE, int kKsWaves>
__global__ __launch_bounds__(64 * kKsWaves) void gemm_f32_ks_kernel(GemmArgs g) {
  extern __shared__ __align__(16) float smem_ks[];
  float (*s_acc)[2][4][64] = reinterpret_cast<float (*)[2][4][64]>(smem_ks);     // [waves][half][elem][lane], at the end
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int tiles_n = (g.N + 31) / 32;
  const int m0 = ((int)blockIdx.x / tiles_n) * 16, n0 = ((int)blockIdx.x % tiles_n) * 32;
  // K per wave: a multiple of 8 that covers K with EDGE, an exact share without
  const int kshare = EDGE ? (g.K + kKsWaves * 8 - 1) / (kKsWaves * 8) * 8 : g.K / kKsWaves;
  const int kbeg = w * kshare;
  const int kw = EDGE ? min(kshare, g.K - kbeg) : kshare;          // (may be negative for the last waves: no pass)
  float* As = smem_ks + w * (kKsAreaA + kKsAreaB);          // (the accumulators take this space over at the end)
  float* Bs = As + kKsAreaA;
  const float* Ag = static_cast<const float*>(g.A);
  const float* Bg = static_cast<const float*>(g.B);
  floatx4 acc[2];
#pragma unroll
  for (int jn = 0; jn < 2; ++jn) acc[jn] = floatx4{0.f, 0.f, 0.f, 0.f};

  // what the epilogue adds or masks with, fetched now so that it has arrived by then: waves 0 .. 3 finish
  // accumulator element w of every lane, for both column halves
  float addend[2] = {0.f, 0.f};
  uint32_t keepw = ~0u;
  if (w < 4) {
    const int row = EDGE ? min(m0 + 4 * kq + w, g.M - 1) : m0 + 4 * kq + w;
#pragma unroll
    for (int jn = 0; jn < 2; ++jn) {
      const int col = EDGE ? min(n0 + 16 * jn + r, g.N - 1) : n0 + 16 * jn + r;
      if (FINISH == 1) {
        if (g.bias) addend[jn] = g.bias[col];
        for (int q = 0; q < g.u_n; ++q) addend[jn] += g.u[(size_t)row * g.u_ld + q] * g.V[(size_t)q * g.N + col];
      }
    }
    if (FINISH == 2 && g.c_mask) keepw = g.c_mask[(size_t)row * g.c_mask_pitch + (n0 >> 5)];
  }

  // One pass = 64 k.  The loads of pass p + 1 are issued before the LDS stores and MFMAs of pass p.
  // A: [16 rows][64 k], piece f = lane + 64 i (i < 4) is row f / 16, k 4 (f % 16).  K-contiguous B: [32 rows][64 k],
  // pieces f = lane + 64 i (i < 8).  N-contiguous B: [64 k][32 n], piece f is k f / 8, n 4 (f % 8).
  // (EDGE, dX: A may come with ReLU bits, element (row, k) is zeroed where its bit is 0)
  constexpr bool kMaskA = EDGE && FINISH == 2;
  floatx4 av[4], bv4[8];
  uint32_t am[kMaskA ? 4 : 1];
  auto load_pass = [&](int k0) {
    const int kn = min(kKsHalf, kw - k0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int f = lane + 64 * i;
      const int row = f >> 4, c4 = (f & 15) * 4;
      if constexpr (EDGE) {
        if (i < 4) {
          const int arow = min(m0 + row, g.M - 1);
          av[i] = load4_any(Ag + (size_t)arow * g.lda + kbeg + k0 + c4, kn - c4);
          if constexpr (kMaskA) {
            am[i] = ~0u;
            if (g.a_mask && c4 < kn) am[i] = mask_bits(g.a_mask, g.a_mask_pitch, arow, kbeg + k0 + c4);
          }
        }
        if constexpr (BK_CONTIG) {
          bv4[i] = load4_any(Bg + (size_t)min(n0 + row, g.N - 1) * g.ldb + kbeg + k0 + c4, kn - c4);
        } else {
          const int kk = f >> 3, n4 = (f & 7) * 4;
          bv4[i] = load4_any(Bg + (size_t)(kbeg + k0 + kk) * g.ldb + n0 + n4, kk < kn ? g.N - n0 - n4 : 0);
        }
        continue;
      }
      if (i < 4) {
        av[i] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (c4 < kn) av[i] = *reinterpret_cast<const floatx4*>(Ag + (size_t)(m0 + row) * g.lda + kbeg + k0 + c4);
      }
      bv4[i] = floatx4{0.f, 0.f, 0.f, 0.f};
      if constexpr (BK_CONTIG) {
        if (c4 < kn) bv4[i] = *reinterpret_cast<const floatx4*>(Bg + (size_t)(n0 + row) * g.ldb + kbeg + k0 + c4);
      } else {
        const int kk = f >> 3, n4 = (f & 7) * 4;
        if (kk < kn) bv4[i] = *reinterpret_cast<const floatx4*>(Bg + (size_t)(kbeg + k0 + kk) * g.ldb + n0 + n4);
      }
    }
  };
  if (!EDGE || kw > 0) load_pass(0);
  for (int k0 = 0; k0 < kw; k0 += kKsHalf) {
    const int kn = min(kKsHalf, kw - k0);      // k in this pass
    __builtin_amdgcn_wave_barrier();           // the reads of the previous pass are done (same wave, in order)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int f = lane + 64 * i, row = f >> 4, c4 = (f & 15) * 4;
      if (i < 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) As[row * kKsPitch + c4 + e] = (!kMaskA || ((am[i] >> e) & 1u)) ? av[i][e] : 0.f;
      }
      if constexpr (BK_CONTIG) {
#pragma unroll
        for (int e = 0; e < 4; ++e) Bs[row * kKsPitch + c4 + e] = bv4[i][e];
      } else {
        *reinterpret_cast<floatx4*>(Bs + (f >> 3) * 32 + (f & 7) * 4) = bv4[i];
      }
    }
    if (k0 + kKsHalf < kw) load_pass(k0 + kKsHalf);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int s0 = 0; s0 < kKsHalf / 4; s0 += 8) {
      float a[8], b[8][2];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int kk = 4 * (s0 + u) + kq;
        a[u] = As[r * kKsPitch + kk];
#pragma unroll
        for (int jn = 0; jn < 2; ++jn) b[u][jn] = BK_CONTIG ? Bs[(16 * jn + r) * kKsPitch + kk] : Bs[kk * 32 + 16 * jn + r];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (4 * (s0 + u) < kn) {
#pragma unroll
          for (int jn = 0; jn < 2; ++jn) acc[jn] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], b[u][jn], acc[jn], 0, 0, 0);
        }
    }
  }
  __syncthreads();                             // every wave is through with its operand area: the accumulators go there
#pragma unroll
  for (int jn = 0; jn < 2; ++jn)
#pragma unroll
    for (int e = 0; e < 4; ++e) s_acc[w][jn][e][lane] = acc[jn][e];
  __syncthreads();
  if (w >= 4) return;
  // accumulator element e of a 16 x 16 block sits at row 4 (lane / 16) + e, column lane % 16
  const int row = m0 + 4 * kq + w;
  float v[2];
#pragma unroll
  for (int jn = 0; jn < 2; ++jn) {
    v[jn] = s_acc[0][jn][w][lane];
#pragma unroll
    for (int q = 1; q < kKsWaves; ++q) v[jn] += s_acc[q][jn][w][lane];
    const int col = n0 + 16 * jn + r;
    if (FINISH == 1) {
      v[jn] += addend[jn];
      if (g.relu) v[jn] = v[jn] > 0.f ? v[jn] : 0.f;
    } else if (!((keepw >> (col & 31)) & 1u)) {
      v[jn] = 0.f;
    }
    if (EDGE && (row >= g.M || col >= g.N)) v[jn] = 0.f;
    else static_cast<float*>(g.y)[(size_t)row * g.ldy + col] = v[jn];
  }
  if (FINISH == 1 && g.bits) {
    // a ballot holds 16 columns of each of four rows: row lane / 16 in bits 16 (lane / 16) ..
    const uint64_t b0 = __ballot(v[0] > 0.f), b1 = __ballot(v[1] > 0.f);
    const uint32_t word = (uint32_t)((b0 >> (16 * kq)) & 0xFFFFu) | ((uint32_t)((b1 >> (16 * kq)) & 0xFFFFu) << 16);
    if (r == 0 && (!EDGE || row < g.M)) g.bits[(size_t)row * g.bits_pitch + (n0 >> 5)] = word;
  }
}

}  // namespace

// A whole 16 x 32 tile grid with K a multiple of 64 and operand rows that are whole 16-byte vectors needs no guards.
static bool ks_whole(const GemmArgs& g) {
  if (g.M % 16 || g.N % 32 || g.K % 64 || g.K < 512 || g.a_mask) return false;
  return !(g.lda % 4 || (reinterpret_cast<uintptr_t>(g.A) & 15) || g.ldb % 4 || (reinterpret_cast<uintptr_t>(g.B) & 15));
}

// Which products run here instead of on 64 x 64 tiles (32 x 32 x 2 matrix instructions, a serial K, element loads of
// ragged rows), measured in us, 64 x 64 tiles / here:
//  - few tiles: forward 150 x 784 x 300 19.7 (two launches) / 8, dX 16.8 / 8; up to 128 of the 64 x 64 tiles, where those
//    still leave half the chip idle: step of 900-600-300-50, batch 400, 229 / 203 against a limit of 64 tiles; at 256
//    tiles (1024 x 1024 x 1024) the larger tiles are ahead, 213 / 233 for a layer;
//  - not a contraction of a few slices, which 64 x 64 tiles finish before the waves here have added up: dX with K = 10
//    2.6 / 5.0, 64 4.0 / 7.0; forward with K = 64 5.3 / 5.2, 128 7.0 / 6.1, many tiles 512 x 1000 x 64 80 / 83 a layer;
//  - ragged, more tiles than CUs and a long K: split over workgroups there (300 x 700 x 2000 22.8 / 31.2); so is a very
//    long K over a handful of tiles (class scores of a wide input: 150 x 10 x 4096 19 / 29, step of a network with
//    64 x 10 x 8192 104 / 128);
//  - whole tiles (M x K x N, K split over workgroups / here) keep a K of any length here while there is at most one of
//    them a CU: dX 16 x 1536 x 512 12.6 / 8.7, 16 x 4096 x 4096 32.9 / 19.6, 64 x 4096 x 512 20.6 / 18.9, 64 x 8192 x 512
//    33.3 / 34.2; with two a CU and K above 2048 not, 64 x 4096 x 4096 31.3 / 37.5.  Forward the same, 16 x 2048 x 512
//    14.7 / 12.0, 16 x 4096 x 4096 33.3 / 20.8, 64 x 4096 x 2048 22.2 / 21.0, but for a K above 3072 over fewer than 32 of
//    the 64 x 64 tiles, or above 2048 over fewer than eight here, which is split up to 32 ways there: 16 x 3072 x 512
//    17.0 / 16.0 and x 64 14.9 / 15.7, 64 x 4096 x 512 18.6 / 20.1, 64 x 8192 x 512 21.8 / 35.4.
bool gemm_f32_ks_ok(const GemmArgs& g, int finish) {
  if (g.b_mask || (g.a_mask && finish != 2) || g.M < 1 || g.N < 1) return false;
  const int64_t tiles64 = (int64_t)((g.M + 63) / 64) * ((g.N + 63) / 64);
  const int64_t tiles = (int64_t)((g.M + 15) / 16) * ((g.N + 31) / 32);
  if (tiles64 > 128 || g.K < (tiles64 > 64 ? 128 : finish == 2 ? 112 : 64)) return false;
  if (tiles64 > 64) return true;
  if (ks_whole(g)) return tiles > 256 ? g.K <= 2048 : finish == 2 || g.K <= (tiles < 8 ? 2048 : 3072) || tiles64 >= 32;
  if (g.K > (tiles < 32 ? 1024 : 2048)) return false;
  return tiles <= 256 || g.K < 512;
}

template <bool EDGE, int WAVES> static hipError_t launch_ks(const GemmArgs& g, int finish, hipStream_t st) {
  const dim3 grid(((g.M + 15) / 16) * ((g.N + 31) / 32)), block(64 * WAVES);
  // every wave's private operand areas; the accumulators (2 KB a wave) take the same space over at the end
  constexpr size_t smem = (size_t)(WAVES * (kKsAreaA + kKsAreaB)) * 4;
  auto kern = finish == 1 ? gemm_f32_ks_kernel<false, 1, EDGE, WAVES> : gemm_f32_ks_kernel<true, 2, EDGE, WAVES>;
  static bool prepared[2] = {false, false};   // one host thread drives a context
  if (!prepared[finish - 1]) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    prepared[finish - 1] = true;
  }
  hipLaunchKernelGGL(kern, grid, block, smem, st, g);
  return hipGetLastError();
}

// finish 1: y = act(A B + bias + u V) with ReLU bits (forward); finish 2: y = (A B^T) under c_mask (dX)
hipError_t launch_gemm_f32_ks(const GemmArgs& g, int finish, hipStream_t st) {
  if (!gemm_f32_ks_ok(g, finish)) return hipErrorInvalidValue;
  if (ks_whole(g)) return launch_ks<false, kKsWavesMax>(g, finish, st);
  const int64_t tiles = (int64_t)((g.M + 15) / 16) * ((g.N + 31) / 32);
  return tiles > 256 ? launch_ks<true, 4>(g, finish, st) : launch_ks<true, 8>(g, finish, st);
}

}  // namespace rad
