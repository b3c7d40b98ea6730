// Matrix-vector product, the paper's running example (Sec. IV):
//
//   y = A |> map(row => zip(row, x) |> map(*) |> reduce(+, 0))
//
// It reads every element of A once and does one multiply-add per element, so it
// is bound by HBM bandwidth (0.5 flop per byte), not by arithmetic: the kernels
// are organised around coalesced 16-byte loads and enough loads in flight.
//
//   A row-major (the paper's layout, RISE_OP_N): a wavefront owns rows (map over
//     rows -> waves, as the generated kernel's work-items own rows), up to four at a
//     time when there are plenty; its lanes stride along the rows in 16-byte chunks
//     (split of the row into lane-sized pieces), and the per-lane partial sums are
//     combined across the wavefront (the reduce, as a tree over the 64 lanes).
//     Unless rows are short or very many, several waves share them;
//   A read through transpose (RISE_OP_T, A stored K x M): a lane owns 4
//     consecutive outputs and sweeps rows of the stored A with 16-byte loads;
//     K is split over waves and workgroups when there are too few column blocks
//     to fill the GPU, and a second kernel sums the split-K partials in a fixed
//     order.
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <mutex>

#include "common.h"

namespace rise {
namespace {

constexpr int kThreads = 256;
constexpr int kCols = 256, kWideCols = 1024;  // outputs per workgroup (RISE_OP_T)

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// a 16-byte load from any 4-byte boundary (gfx950 runs global memory in
// unaligned-access mode)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// RPW rows per wave; WAVES waves of a workgroup share a row group's K (1: a wave
// owns its rows), each taking every WAVES-th run of UN 16-byte chunks per lane.
template <int RPW, int WAVES, int UN>
__global__ __launch_bounds__(WAVES == 1 ? kThreads : 64 * WAVES) void gemv_rows(
    float* __restrict__ y, const float* __restrict__ A, int64_t lda, const float* __restrict__ x,
    int M, int K, int64_t row_groups) {
  __shared__ float part[WAVES][RPW];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t step = WAVES == 1 ? (int64_t)gridDim.x * (kThreads / 64) : gridDim.x;
  for (int64_t g = WAVES == 1 ? (int64_t)blockIdx.x * (kThreads / 64) + wave : blockIdx.x;
       g < row_groups; g += step) {
    const int r0 = (int)(g * RPW);
    const float* rows[RPW];
#pragma unroll
    for (int j = 0; j < RPW; j++)  // rows past M repeat the last row; never stored
      rows[j] = A + (int64_t)min(r0 + j, M - 1) * lda;
    f32x4 a4[RPW];
#pragma unroll
    for (int j = 0; j < RPW; j++) a4[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nchunk = K / 4, kw = WAVES == 1 ? 0 : wave;
    auto fma4 = [&](f32x4& acc, const f32x4& v, const f32x4& w) {
      acc.x = fmaf(v.x, w.x, acc.x);
      acc.y = fmaf(v.y, w.y, acc.y);
      acc.z = fmaf(v.z, w.z, acc.z);
      acc.w = fmaf(v.w, w.w, acc.w);
    };
    int c = 64 * UN * kw + lane;
    for (; c + 64 * (UN - 1) < nchunk; c += 64 * UN * WAVES) {  // all loads of a run in flight
      f32x4 xv[UN], v[UN][RPW];
#pragma unroll
      for (int u = 0; u < UN; u++) {
        xv[u] = reinterpret_cast<const f32x4u*>(x)[c + 64 * u];
#pragma unroll
        for (int j = 0; j < RPW; j++) v[u][j] = reinterpret_cast<const f32x4u*>(rows[j])[c + 64 * u];
      }
#pragma unroll
      for (int u = 0; u < UN; u++)
#pragma unroll
        for (int j = 0; j < RPW; j++) fma4(a4[j], v[u][j], xv[u]);
    }
#pragma unroll
    for (int u = 0; u < UN; u++)  // this lane's chunks of the last, shorter run
      if (c + 64 * u < nchunk) {
        const f32x4 xv = reinterpret_cast<const f32x4u*>(x)[c + 64 * u];
#pragma unroll
        for (int j = 0; j < RPW; j++)
          fma4(a4[j], f32x4(reinterpret_cast<const f32x4u*>(rows[j])[c + 64 * u]), xv);
      }
    float acc[RPW];
#pragma unroll
    for (int j = 0; j < RPW; j++) acc[j] = (a4[j].x + a4[j].y) + (a4[j].z + a4[j].w);
    if (kw == 0 && nchunk * 4 + lane < K) {  // up to 3 values past the last chunk
      const int k = nchunk * 4 + lane;
#pragma unroll
      for (int j = 0; j < RPW; j++) acc[j] = fmaf(rows[j][k], x[k], acc[j]);
    }
#pragma unroll
    for (int j = 0; j < RPW; j++) {
      const float s = wave_sum(acc[j]);
      if (WAVES == 1) {
        if (lane == 0 && r0 + j < M) y[r0 + j] = s;
      } else if (lane == 0) {
        part[wave][j] = s;
      }
    }
    if (WAVES > 1) {
      __syncthreads();
      if (threadIdx.x < RPW && r0 + (int)threadIdx.x < M) {
        float s = part[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < WAVES; w++) s += part[w][threadIdx.x];
        y[r0 + threadIdx.x] = s;
      }
      __syncthreads();
    }
  }
}

// out[kc * ldo + m] = sum over k in chunk kc of A[k][m] * x[k].  A lane owns four
// columns; KS of the workgroup's four waves share the chunk's rows (their sums are
// added in wave order), the others stand side by side, and 16-byte loads of UN
// rows are in flight per lane.
//   KS = 4, UN = 8: 256 columns a workgroup.  The split over waves inside the
//     workgroup quarters the partial sums that a split over workgroups alone
//     writes for the same number of waves (4096^2 with the reduction: 18.5 -> 15.3
//     us, 512 x 16384 19.5 -> 10.3 us).
//   KS = 1, UN = 2: 1024 columns a workgroup, for large matrices: one row of a
//     workgroup is 4 KB of consecutive memory (16384^2: 162 us against 198).
// Lanes at the right edge load the last four columns instead (their sums are
// written by column, so nothing is counted twice).
template <int KS, int UN>
__global__ __launch_bounds__(kThreads) void gemv_cols(float* __restrict__ out, int64_t ldo,
                                                      const float* __restrict__ A, int64_t lda,
                                                      const float* __restrict__ x, int M, int K,
                                                      int mblocks, int kchunk) {
  constexpr int COLS = kThreads * 4 / KS;
  __shared__ float part[KS][COLS];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int side = wave % (4 / KS), kw = wave / (4 / KS);
  const int mb = blockIdx.x % mblocks, kc = blockIdx.x / mblocks;
  const int m0 = mb * COLS, m = min(m0 + 256 * side + 4 * lane, M - 4);
  const int c0 = kc * kchunk, c1 = min(K, c0 + kchunk), share = (c1 - c0 + KS - 1) / KS;
  int k = c0 + kw * share;
  const int k1 = min(c1, k + share);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (M >= 4) {
    const float* p = A + (int64_t)k * lda + m;
    for (; k + UN <= k1; k += UN, p += UN * lda) {
      f32x4 v[UN];
#pragma unroll
      for (int u = 0; u < UN; u++) v[u] = *reinterpret_cast<const f32x4u*>(p + u * lda);
#pragma unroll
      for (int u = 0; u < UN; u++) {
        const float xv = x[k + u];
        acc.x = fmaf(v[u].x, xv, acc.x); acc.y = fmaf(v[u].y, xv, acc.y);
        acc.z = fmaf(v[u].z, xv, acc.z); acc.w = fmaf(v[u].w, xv, acc.w);
      }
    }
    for (; k < k1; k++, p += lda) {
      const f32x4 v = *reinterpret_cast<const f32x4u*>(p);
      const float xv = x[k];
      acc.x = fmaf(v.x, xv, acc.x); acc.y = fmaf(v.y, xv, acc.y);
      acc.z = fmaf(v.z, xv, acc.z); acc.w = fmaf(v.w, xv, acc.w);
    }
#pragma unroll
    for (int q = 0; q < 4; q++)
      if (m + q >= m0) part[kw][m + q - m0] = acc[q];
  } else if (side == 0) {  // fewer than four columns: one lane each
    float a = 0.f;
    if (lane < M)
      for (; k < k1; k++) a = fmaf(A[(int64_t)k * lda + lane], x[k], a);
    part[kw][lane] = a;
  }
  __syncthreads();
#pragma unroll
  for (int c = threadIdx.x; c < COLS; c += kThreads) {
    float s = part[0][c];
#pragma unroll
    for (int q = 1; q < KS; q++) s += part[q][c];
    if (m0 + c < M) out[(int64_t)kc * ldo + m0 + c] = s;
  }
}

// y[m] = sum of the parts in a fixed order: a workgroup owns 64 outputs, its four
// waves a quarter of the parts each, added in wave order.  Bound by the latency of
// its loads, so 16 are in flight, and 8 of what is left: one at a time the fewer than
// 64 parts of wide and short matrices were a serial chain (outputs x K, both kernels: 7104
// x 3566 20.6 -> 18.9 us, 5184 x 2593 13.9 -> 12.0, 8192 x 3000 20.5 -> 18.7).
__global__ __launch_bounds__(kThreads) void gemv_reduce(float* __restrict__ y,
                                                        const float* __restrict__ part, int M,
                                                        int nparts) {
  __shared__ float sums[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t m = (int64_t)blockIdx.x * 64 + lane, mc = m < M ? m : M - 1;
  const int share = (nparts + 3) / 4, p1 = min(nparts, (wave + 1) * share);
  float s = 0.f;
  int p = wave * share;
  for (; p + 16 <= p1; p += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; u++) v[u] = part[(int64_t)(p + u) * M + mc];
#pragma unroll
    for (int u = 0; u < 16; u++) s += v[u];
  }
  for (; p < p1; p += 8) {  // past the end the last part is loaded again and not added
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; u++) v[u] = part[(int64_t)min(p + u, p1 - 1) * M + mc];
#pragma unroll
    for (int u = 0; u < 8; u++) s += p + u < p1 ? v[u] : 0.f;
  }
  sums[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && m < M)
    y[m] = (sums[0][lane] + sums[1][lane]) + (sums[2][lane] + sums[3][lane]);
}

struct ColSplit {
  bool wide;  // 1024 columns a workgroup, else 256
  int mblocks, kchunks, kchunk;
};
ColSplit col_split(int64_t M, int64_t K) {
  ColSplit c;
  // Wide workgroups, where there are enough chunks of 64 rows for them: about 400,
  // whichever way they lie (outputs x K, wide and narrow: 16278 x 1029 15.4 and
  // 14.8 us, 12584 x 1588 16.3 and 16.1, 8192 x 3000 18.4 both, 7060 x 3920 19.6 and 21.6,
  // 2000 x 14000 20.4 and 21.6, 1000 x 40000 29.5 and 30.1, 3000 x 12000 24.8 and 26.3,
  // 6000^2 24.2 and 26.8, 16384^2 162 and 198); few outputs leave most of its columns
  // empty (64 x 200000 41.2 and 17.3, 300 x 60000 22.0 and 21.2).
  const int64_t wide_blocks = (M + kWideCols - 1) / kWideCols;
  c.wide = M >= 512 && wide_blocks * ((K + 63) / 64) >= 400;
  const int cols = c.wide ? kWideCols : kCols;
  c.mblocks = (int)((M + cols - 1) / cols);
  // about 1024 workgroups in all, four per compute unit, and chunks of at least 64 rows
  // of A (with 2048, 16384^2 took 202 us; narrow ones with 2176, 500 x 100000 40.9 us
  // and 36.8, 300 x 60000 23.6 and 21.2, 3000 x 10000 22.9 and 22.6)
  int64_t want = std::min<int64_t>(1024, (1024 + c.mblocks - 1) / c.mblocks);
  int64_t most = std::max<int64_t>(1, (K + 63) / 64);
  c.kchunks = (int)std::max<int64_t>(1, std::min(want, most));
  c.kchunk = (int)((K + c.kchunks - 1) / c.kchunks);
  if (c.kchunk == 0) c.kchunk = 1;
  c.kchunks = (int)std::max<int64_t>(1, (K + c.kchunk - 1) / c.kchunk);
  return c;
}

}  // namespace

size_t gemv_workspace(int64_t M, int64_t K, bool trans) {
  if (!trans || M == 0 || K == 0) return 0;
  const ColSplit c = col_split(M, K);
  return c.kchunks > 1 ? (size_t)c.kchunks * M * 4 : 0;
}

int gemv_parts(int64_t M, int64_t K, bool trans) {
  if (!trans || M == 0 || K == 0) return 1;
  return col_split(M, K).kchunks;
}

rise_status launch_gemv(const GemvArgs& a, void* ws, hipStream_t s) {
  // K = 0 needs no special case: the kernels reduce over an empty range and
  // store the initial value 0
  if (!a.trans) {
    const int64_t cus = device_cu_count();
    auto go = [&](auto kernel, int rpw, int waves) {
      const int64_t groups = (a.M + rpw - 1) / rpw;
      const int64_t blocks = std::min<int64_t>(waves == 1 ? (groups + 3) / 4 : groups, cus * 32);
      hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(waves == 1 ? kThreads : 64 * waves), 0,
                         s, a.y, a.A, a.lda, a.x, a.M, a.K, groups);
    };
    // two rows to four waves: 2048 rows are four waves per SIMD,
    // and each value of x feeds two.  8192^2 38.3 us (7.0 TB/s, some of it from the
    // last-level cache) where one wave for four rows took 48.9; 16384^2 162.3 against
    // 171.8 and 3566 x 7104 16.0 against 16.5 with four rows a wave.  The grid holds four
    // times what is resident, as far as there are rows: with no more than is resident,
    // each walking through the rows, the last ones end unevenly (11344 x 8448 66.3 us,
    // 63.8 so).  Short rows do not feed four waves: of many, four rows go to one wave
    // (100000 x 64 13.5 against 36.1 us, 15993 x 868 10.3 and 12.1, 14486 x 1151 12.2 and
    // 12.7; but 12584 x 1588 14.7 and 13.1, 16000 x 1600 16.6 and 15.8).  Fewer rows go
    // one to four and to sixteen waves.  Before, all went four to a wave: 4096^2 17.0 ->
    // 13.0 us, 1000 x 40000 60 -> 30, 64 x 16384 14.4 -> 5.0; 1500 x 12345, whose rows
    // are not 16-byte aligned and went value by value, 96.9 -> 15.4
    if (a.M >= 10240 && a.K < 1400) go(gemv_rows<4, 1, 2>, 4, 1);
    else if (a.M >= 2048) go(gemv_rows<2, 4, 2>, 2, 4);
    else if (a.M >= 256) go(gemv_rows<1, 4, 4>, 1, 4);
    else go(gemv_rows<1, 16, 4>, 1, 16);
    return check_launch("gemv_rows");
  }
  const ColSplit c = col_split(a.M, a.K);
  float* out = c.kchunks > 1 ? (float*)ws : a.y;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((int64_t)c.mblocks * c.kchunks)), dim3(kThreads), 0, s,
                       out, (int64_t)a.M, a.A, a.lda, a.x, a.M, a.K, c.mblocks, c.kchunk);
  };
  if (c.wide)
    go(gemv_cols<1, 2>);
  else
    go(gemv_cols<4, 8>);
  rise_status st = check_launch("gemv_cols");
  if (st != RISE_OK || c.kchunks == 1) return st;
  hipLaunchKernelGGL(gemv_reduce, dim3((unsigned)((a.M + 63) / 64)), dim3(kThreads), 0,
                     s, a.y, (const float*)ws, a.M, c.kchunks);
  return check_launch("gemv_reduce");
}


// ---------------------------------------------------------------------------
// Fixed scratch for the entry point that allocates nothing (rise_gemv_noalloc).
// The split-K partials of the transposed product go to this file-scope device
// array instead of a caller workspace.  Its size covers every split col_split
// picks: kchunks > 1 only when there are fewer column blocks than workgroups
// wanted, and then kchunks * M <= ceil(1024 / mblocks) * mblocks * 1024 <= 2046 *
// 1024 floats (wide; a quarter of that narrow).
// Each device holds its own copy for the life of the process; its device
// address is looked up once per device (hipGetSymbolAddress with that device
// current) and only that address is handed to kernels.
// ---------------------------------------------------------------------------
constexpr size_t kGemvScratchBytes = RISE_GEMV_NOALLOC_SCRATCH_BYTES;
static_assert(kGemvScratchBytes >= (size_t)2046 * kWideCols * 4, "scratch below the largest split");
static __device__ __align__(256) unsigned char scratch[kGemvScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];
std::mutex g_scratch_mu;
}  // namespace

size_t gemv_scratch_bytes() { return kGemvScratchBytes; }

rise_status gemv_scratch(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return fail(RISE_ERR_HIP, "rise_gemv_noalloc: hipGetDevice failed");
  if (dev < 0 || dev >= kMaxDevices) return fail(RISE_ERR_HIP, "rise_gemv_noalloc: device index above 63");
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    p = g_scratch_ptr[dev].load(std::memory_order_relaxed);
    if (!p) {
      const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !p)
        return fail(RISE_ERR_HIP, std::string("rise_gemv_noalloc: hipGetSymbolAddress(scratch): ") +
                                      hipGetErrorString(e));
      g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
  }
  *out = p;
  return RISE_OK;
}

}  // namespace rise
