// FP32 GEMM on the gfx950 FP32 matrix cores (v_mfma_f32_32x32x2_f32).  Two kernels:
//   gemm_f32_kernel: one workgroup per BM x BN output tile, tiles visited in an
//     XCD-contiguous, grouped order so that concurrently running tiles share A and
//     B panels in their XCD's L2; the K loop (reduceSeq over split(BK) slabs, each
//     staged in LDS: toMem(Local), paper Sec. V-B/C) is tiles::gemm_ring_tile;
//   gemm_f32_split_kernel: one workgroup per 32 x 32 output tile whose waves take
//     alternate slabs of K and add their sums at the end, for small products.
#include <algorithm>

#include "common.h"
#include "tiles.h"

namespace rise {
namespace {

using tiles::kThreads;

// How slabs reach LDS: 16-byte copies (rows of whole aligned chunks), through
// registers, or 4-byte copies.
enum Fill { CHUNKS, STAGED, VALUES };

// Two waves to a SIMD, if by two workgroups of four waves: while one waits for its
// ring to fill or stores its tile the other computes.  (256 x 128, left to take more
// than half of the registers, ran 4096^3 in 972 us instead of 933 and, with three slabs
// of 4-byte copies to a tile, 6681 x 6656 x 83 in 160 instead of 119.)
template <typename T, bool TA, bool TB, Fill FILL>
__global__ __launch_bounds__(T::THREADS, T::WAVES < 8 ? 2 : T::WAVES / 4) void gemm_f32_kernel(
    float* __restrict__ C, int64_t ldc, const float* __restrict__ A, int64_t lda,
    const float* __restrict__ B, int64_t ldb, int M, int N, int K, int tiles_m, int tiles_n) {
  __shared__ f32x4 lds[T::LDS_CHUNKS];
  int tm, tn;
  grouped_tile(xcd_contiguous(blockIdx.x, gridDim.x), tiles_m, tiles_n, 8, tm, tn);
  tiles::gemm_ring_tile<T, TA, TB, FILL != VALUES, false, 1, FILL == STAGED>(
      C, ldc, A, lda, B, ldb, M, N, K, tm * T::BM, tn * T::BN, lds);
}

// Few output tiles: a workgroup of NW waves owns a 32 x 32 tile, and wave w sums
// the 32-k slabs w, w + NW, ... of it, loading its MFMA fragments straight from
// global memory into registers one slab ahead (no LDS and no barrier until the
// NW partial tiles are added, in wave order).  What bounds such a product is the
// chain of slabs, one memory latency each: with NW waves it is NW times shorter,
// and 32 x 32 tiles are four times as many workgroups as 64 x 64 (128^3: one slab
// per wave on 16 workgroups, kernel 6.6 -> 4.1 us; 512^3 13.1 -> 7.7).
//   rows along k: a lane reads 16 bytes (4 k of its row, at the row's own 4-byte
//     alignment; gfx950 runs global memory in unaligned-access mode);
//   rows along m or n: a lane reads one value per k, 32 lanes 128 contiguous bytes.
// Rows past the edge repeat the last one and feed outputs that are not stored;
// k past the end reads as zero.

template <bool ALONG_K>
struct SplitFrag {
  f32x4 v[4];  // v[s][t]: k = 8 s + 4 kl + t of the slab
  __device__ void load(const float* X, int64_t ld, int mn, int k0, int K, int kl) {
    if (k0 + 32 <= K) {
#pragma unroll
      for (int s = 0; s < 4; s++) {
        const int k = k0 + 8 * s + 4 * kl;
        if (ALONG_K) {
          v[s] = *reinterpret_cast<const tiles::f32x4u*>(X + (int64_t)mn * ld + k);
        } else {
#pragma unroll
          for (int t = 0; t < 4; t++) v[s][t] = X[(int64_t)(k + t) * ld + mn];
        }
      }
      return;
    }
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
      for (int t = 0; t < 4; t++) {
        const int k = k0 + 8 * s + 4 * kl + t, kc = min(k, K - 1);
        const float x = ALONG_K ? X[(int64_t)mn * ld + kc] : X[(int64_t)kc * ld + mn];
        v[s][t] = k < K ? x : 0.f;
      }
  }
};

template <int NW, bool TA, bool TB>
__global__ __launch_bounds__(64 * NW) void gemm_f32_split_kernel(
    float* __restrict__ C, int64_t ldc, const float* __restrict__ A, int64_t lda,
    const float* __restrict__ B, int64_t ldb, int M, int N, int K, int tiles_m, int tiles_n) {
  __shared__ float part[NW][32 * 32];
  int tm, tn;
  grouped_tile(xcd_contiguous(blockIdx.x, gridDim.x), tiles_m, tiles_n, 8, tm, tn);
  const int m0 = tm * 32, n0 = tn * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kl = lane >> 5, il = lane & 31;
  const int m = min(m0 + il, M - 1), n = min(n0 + il, N - 1);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; r++) acc[r] = 0.f;
  SplitFrag<!TA> a[2];
  SplitFrag<TB> b[2];
  auto mfmas = [&](const SplitFrag<!TA>& x, const SplitFrag<TB>& y) {
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
      for (int t = 0; t < 4; t++)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.v[s][t], y.v[s][t], acc, 0, 0, 0);
  };
  int k0 = 32 * wave;
  if (k0 < K) {
    a[0].load(A, lda, m, k0, K, kl);
    b[0].load(B, ldb, n, k0, K, kl);
  }
  for (; k0 < K; k0 += 64 * NW) {  // two slabs a round, so the register sets alternate
    const int k1 = k0 + 32 * NW, k2 = k1 + 32 * NW;
    if (k1 < K) {
      a[1].load(A, lda, m, k1, K, kl);
      b[1].load(B, ldb, n, k1, K, kl);
    }
    mfmas(a[0], b[0]);
    if (k1 >= K) break;
    if (k2 < K) {
      a[0].load(A, lda, m, k2, K, kl);
      b[0].load(B, ldb, n, k2, K, kl);
    }
    mfmas(a[1], b[1]);
  }
#pragma unroll
  for (int r = 0; r < 16; r++) part[wave][(8 * (r >> 2) + 4 * kl + (r & 3)) * 32 + il] = acc[r];
  __syncthreads();
#pragma unroll
  for (int o = tid; o < 32 * 32; o += 64 * NW) {
    float s = part[0][o];
#pragma unroll
    for (int w = 1; w < NW; w++) s += part[w][o];
    const int row = m0 + o / 32, col = n0 + o % 32;
    if (row < M && col < N) C[(int64_t)row * ldc + col] = s;
  }
}

template <typename T, Fill FILL>
rise_status launch_fill(const GemmF32Args& a, hipStream_t s) {
  const int tiles_m = (a.M + T::BM - 1) / T::BM, tiles_n = (a.N + T::BN - 1) / T::BN;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(tiles_m * tiles_n), dim3(T::THREADS), 0, s, a.C, a.ldc, a.A,
                       a.lda, a.B, a.ldb, a.M, a.N, a.K, tiles_m, tiles_n);
  };
  if (!a.ta && !a.tb) go(gemm_f32_kernel<T, false, false, FILL>);
  else if (!a.ta) go(gemm_f32_kernel<T, false, true, FILL>);
  else if (!a.tb) go(gemm_f32_kernel<T, true, false, FILL>);
  else go(gemm_f32_kernel<T, true, true, FILL>);
  return check_launch("gemm_f32_kernel");
}

// Rows that are not whole aligned chunks go through registers while K is short: a
// ring fills with a quarter of the instructions, and its first three slabs in one
// memory latency (64 x 64 tiles, by values and staged: 1664 x 903 x 79 14.2 and 11.6 us, 5001 x
// 5003 x 101 125 and 101, x 301 198 and 190).  Over a longer K copies that need no
// registers run further ahead (1000 x 1531 x 777 32.2 and 35.5 us, 3001^3 479 and
// 516), and 256 x 128 tiles gain nothing (6681 x 6656 x 83 119 us either way).
constexpr int kStagedMaxK = 320;

template <typename T>
rise_status launch_tile(const GemmF32Args& a, bool vec, hipStream_t s) {
  if (vec) return launch_fill<T, CHUNKS>(a, s);
  if constexpr (T::BM * T::BN < 128 * 128)
    if (a.K <= kStagedMaxK) return launch_fill<T, STAGED>(a, s);
  return launch_fill<T, VALUES>(a, s);
}

template <int NW>
rise_status launch_split(const GemmF32Args& a, hipStream_t s) {
  const int tiles_m = (a.M + 31) / 32, tiles_n = (a.N + 31) / 32;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(tiles_m * tiles_n), dim3(64 * NW), 0, s, a.C, a.ldc, a.A,
                       a.lda, a.B, a.ldb, a.M, a.N, a.K, tiles_m, tiles_n);
  };
  if (!a.ta && !a.tb) go(gemm_f32_split_kernel<NW, false, false>);
  else if (!a.ta) go(gemm_f32_split_kernel<NW, false, true>);
  else if (!a.tb) go(gemm_f32_split_kernel<NW, true, false>);
  else go(gemm_f32_split_kernel<NW, true, true>);
  return check_launch("gemm_f32_split_kernel");
}

// The tiles, and nanoseconds per 64 x 64 outputs and k that one CU takes on them
// (measured: 256 x 128 at 4096^3, 32 x 32 x 32 at 512^3, 32 x 32 x 128 at 64 x 64 x
// 4096, the others at 1024^3, 1000 x 1531 x 777 and 1500 x 300 x 6000; the matrix
// cores alone need 13.6 at 2.3 GHz), where rows are whole aligned chunks and where
// they are not (what differs is how the two kinds of 32 x 32 tiles compare with the
// rest, as the split kernel's loads keep their width, and 256 x 128 of a longer K, whose
// 4-byte copies are then more of its time: 5189 x 5376 x 1940 916 us, 64 x 64 860).  0: only
// where asked for.
struct TileCost {
  rise_tile t;
  double ns, ns_values;
};
const TileCost kTiles[] = {{{128, 128, 32}, 0, 0},        {{128, 64, 32}, 16.0, 16.0},
                           {{64, 128, 32}, 16.0, 16.0},   {{64, 64, 32}, 16.5, 16.5},
                           {{256, 128, 16}, 14.6, 15.4},  {{64, 96, 32}, 17.0, 17.0},
                           {{96, 64, 32}, 16.5, 16.5},    {{64, 32, 64}, 19.5, 19.5},
                           {{32, 64, 64}, 19.5, 19.5},    {{32, 32, 32}, 36.0, 26.0},
                           {{32, 32, 128}, 18.5, 22.0}};

}  // namespace

bool gemm_f32_tile_supported(const rise_tile& t) {
  for (const auto& k : kTiles)
    if (k.t.bm == t.bm && k.t.bn == t.bn && k.t.bk == t.bk) return true;
  return false;
}

int gemm_f32_tiles(rise_tile* out, int cap) {
  int n = (int)(sizeof(kTiles) / sizeof(kTiles[0]));
  for (int i = 0; out && i < n && i < cap; i++) out[i] = kTiles[i].t;
  return n;
}

rise_tile gemm_f32_best_tile(int M, int N, int K, bool chunks) {
  // The tile with the shortest time for the CU that gets the most tiles: what the
  // shapes differ in is mainly how evenly they cover 256 CUs (1000 x 1531: 384
  // tiles of 64 x 64, two on half of the CUs, 36 us; 256 of 64 x 96, one each, 31
  // us; 512 x 512 x 512: 64 of 64 x 64, 14 us, 256 of 32 x 32, 8 us).
  // 32 x 32 tiles of a short K run gemm_f32_split_kernel, whose waves wait out
  // one memory latency per 32 k but need no ring to fill (128^3: 4.1 against 4.9
  // us); of a longer K the ring (814 x 200 x 1024, rows of whole chunks: 8.9 against
  // 11.3 us; 64 x 64 x 4096: 22 against 38 us).  Where rows are not whole chunks the
  // ring's copies go value by value and the crossing lies further out (130 x 333 x
  // 1601 16.7 against 20.2 us, 555 x 85 x 3001 27.4 and 26.4), and so is the time of
  // the split kernel lower beside them.
  // That holds while the split kernel's tiles are few; many of them read each row
  // of A and B too often (5755 x 6140 x 112: 216 us, 256 x 128 102).
  // Every round also pays for the stages a ring starts with and for the store of
  // the tile, as K grows short most of its time: counted as four stages and 128 k,
  // and a last round that is not full runs somewhat faster than a full one (without
  // these 1664 x 903 x 79 took 64 x 32 tiles, 23.9 us, 32 x 32 11.0).  256 x 128 tiles
  // are resident in pairs, and the last ones can go in pairs to some CUs while others
  // are idle, which counts where rows are whole chunks (5968 x 2961 x 1128, 576 tiles,
  // takes 1.5 times as long as in 64 x 64; by 4-byte copies the fill hides more of it).
  // `chunks` has to be how the operands are stored: M says nothing about the rows of
  // A as stored, nor N about those of B read through transpose, and a padded row can
  // break the alignment of sizes that are whole chunks.  Over 1500 random shapes up to
  // 7000 x 7000 x 3000 of which every tile was timed, the choice is 1.3 to 1.8 %
  // above the best tile of each by class, 1.6 where taken from the three sizes it was 5.0
  // (170 x 1020 x 2304 23.1 us instead of 15.8, 480 x 447 x 2388 21.4 and 16.0).
  const int split_max_k = chunks ? 768 : 2560;
  rise_tile best{64, 64, 32};
  double least = 0;
  for (const auto& c : kTiles) {
    if (c.ns == 0) continue;
    if (c.t.bm == 32 && c.t.bn == 32 && (c.t.bk == 128) != (K > split_max_k)) continue;
    const bool split = c.t.bm == 32 && c.t.bn == 32 && c.t.bk == 32;
    const int64_t tiles = (((int64_t)M + c.t.bm - 1) / c.t.bm) * (((int64_t)N + c.t.bn - 1) / c.t.bn);
    const bool as_chunks = chunks || (split && tiles > 2048) || (c.t.bm == 256 && K <= 512);
    const double ns = as_chunks ? c.ns : c.ns_values;
    const double k = (double)K + 128 + (split ? 0 : 4 * c.t.bk);
    double rounds = 0.85 * (double)((tiles + 255) / 256) + 0.15 * (double)tiles / 256;
    if (c.t.bm == 256 && chunks)
      rounds += 0.2 * (double)(2 * ((tiles + 511) / 512) - (tiles + 255) / 256);
    const double t = rounds * c.t.bm * c.t.bn * ns * k;
    if (least == 0 || t < least) least = t, best = c.t;
  }
  return best;
}

rise_tile gemm_f32_default_tile(int M, int N, int K) {
  return gemm_f32_best_tile(M, N, K, N % 4 == 0 && K % 4 == 0);
}

rise_tile gemm_f32_default_tile(const GemmF32Args& a) {
  return gemm_f32_best_tile(
      a.M, a.N, a.K, tiles::whole_chunks(a.A, a.lda, a.B, a.ldb, a.M, a.N, a.K, a.ta, a.tb));
}

rise_status launch_gemm_f32(const GemmF32Args& a, const rise_tile& t, hipStream_t s) {
  const bool vec = tiles::whole_chunks(a.A, a.lda, a.B, a.ldb, a.M, a.N, a.K, a.ta, a.tb);
#define RISE_F32_TILE(BM, BN, BK, ...)                                         \
  if (t.bm == BM && t.bn == BN && t.bk == BK) {                                \
    using T = tiles::F32Cfg<BM, BN, BK, __VA_ARGS__>;                          \
    return launch_tile<T>(a, vec, s);                                          \
  }
  RISE_F32_TILE(256, 128, 16, 3, 2, 2, 1)
  RISE_F32_TILE(128, 128, 32, 3, 2, 2, 2)
  RISE_F32_TILE(128, 64, 32, 3, 2, 2, 2)
  RISE_F32_TILE(64, 128, 32, 3, 2, 2, 2)
  RISE_F32_TILE(64, 64, 32, 3, 2, 2, 2)
  RISE_F32_TILE(64, 96, 32, 3, 2, 3, 2)
  RISE_F32_TILE(96, 64, 32, 3, 3, 2, 2)
  RISE_F32_TILE(64, 32, 64, 3, 2, 1, 4)
  RISE_F32_TILE(32, 64, 64, 3, 1, 2, 4)
  RISE_F32_TILE(32, 32, 128, 3, 1, 1, 8)
#undef RISE_F32_TILE
  if (t.bm == 32 && t.bn == 32 && t.bk == 32)
    return a.K <= 512 ? launch_split<4>(a, s) : launch_split<8>(a, s);
  return fail(RISE_ERR_UNSUPPORTED, "gemm_f32: unsupported tile");
}

}  // namespace rise
