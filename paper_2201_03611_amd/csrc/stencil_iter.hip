// iterate with a size-preserving body (Sec. VI): `steps` applications of the
// 2D stencil, pad2D |> slide2D |> weighted reduce, each reading the image the
// previous one wrote (a Jacobi-style iteration).
//
// The paper's translation is a double buffer in memory and one loop round per
// application.  That is the fuse = 1 schedule here: one stencil launch per
// step, ping-ponging between two images in the caller's workspace; the first
// launch reads the input and the last writes the output.
//
// fuse = T > 1 runs T steps per launch (temporal blocking), in registers: a wave
// walks down a strip of 128 columns, two to a lane, and every row it loads passes
// through the T steps at once.  HBM then carries the image once per T steps.
//
// Every output is the sum over dy (outer) and dx (inner) of fma(x, w, acc)
// from 0, the order of the single-step kernels, so fused and unfused
// schedules give identical bits.
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "common.h"

namespace rise {
namespace {

constexpr int kThreads = 256;
constexpr int kItTMax = 4;  // most steps per launch

// Strips and segments of the fused kernel: a strip has C columns to a lane, of which
// HALO on each side are only read, and a segment `rows` output rows; one wave each.
// (Four columns to a lane halve the share of the halo but also the waves: as fast at
// 4096^2, 10 to 40 % slower below 1500^2.)
constexpr int C = 2;
template <int K, int T>
struct ItCfg {
  static constexpr int R = (K - 1) / 2;
  static constexpr int HALO = (R * T + C - 1) / C * C;
  static constexpr int USE = 64 * C - 2 * HALO;
  static_assert(C >= R, "windows reach into the neighbouring lanes only");
  static constexpr int PF = K;  // rows loaded ahead (a multiple of K)
};

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

typedef float V __attribute__((ext_vector_type(C)));
typedef float VU __attribute__((ext_vector_type(C), aligned(4)));

// the value of the lane before (UP) or after, by a DPP move over the whole wave
template <bool UP>
__device__ __forceinline__ float neighbour(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v),
                                                            UP ? 0x138 : 0x130, 0xf, 0xf, true));
}

// One wave's segment.  Level t holds the image after t steps.  In every tick the next
// row of level 0 is loaded, and level t = 1 .. T finishes row i - R t: a row that
// arrives at a level is added to the K output rows of the next level whose windows
// it is in (dy = 0 opens an accumulator, dy = K - 1 closes one), so each level keeps
// K accumulators per column and no rows.
// EX, EY (a strip or a segment that reaches past the image): a level's columns and
// rows outside the image are what pad2D reads there, the level's own edge (clamp) or
// zeros.  Outside columns are rewritten in each finished row.  Rows above row 0 are
// not processed; when row 0 arrives, it is first added for the rows above it.  Past
// the last row the row before arrives again.
template <int K, int T, bool EX, bool EY>
__device__ __forceinline__ void iterate_segment(float* __restrict__ out, int64_t ld_out,
                                                const float* __restrict__ in, int64_t ld_in, int H,
                                                int W, const float (&wt)[K][K], int zero_pad,
                                                int xs, int y0, int y1, int keep_out) {
  using Cfg = ItCfg<K, T>;
  constexpr int R = Cfg::R, PF = Cfg::PF, HALO = Cfg::HALO;
  const int lane = threadIdx.x & 63, x = xs + C * lane;
  const int first = y0 - R * T, ticks = y1 - y0 + 2 * R * T;
  auto load = [&](int i) {  // row first + i, inside the image
    const float* row = in + (int64_t)clampi(first + i, 0, H - 1) * ld_in;
    if (!EX) return V(*reinterpret_cast<const VU*>(row + x));
    V v;
#pragma unroll
    for (int q = 0; q < C; q++) v[q] = row[clampi(x + q, 0, W - 1)];
    return v;
  };
  // columns of a level's row outside the image; the column W - 1 is lane `le`'s
  // element `ee` (when the strip reaches past it)
  const int cr = W - 1 - xs, le = cr / C & 63, ee = cr % C;
  const bool left = xs < 0, right = xs + 64 * C > W;
  auto pad_columns = [&](V& v) {
    if (left) {
      const float e = __builtin_bit_cast(
          float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v.x), HALO / C));
#pragma unroll
      for (int q = 0; q < C; q++) v[q] = x < 0 ? (zero_pad ? 0.f : e) : v[q];
    }
    if (right) {
      float pick = v[0];
#pragma unroll
      for (int q = 1; q < C; q++) pick = ee == q ? v[q] : pick;
      const float e =
          __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, pick), le));
#pragma unroll
      for (int q = 0; q < C; q++) v[q] = x + q >= W ? (zero_pad ? 0.f : e) : v[q];
    }
  };

  float acc[T][K][C] = {};  // [level - 1][output row modulo K][column]
  V last[EY ? T : 1] = {};
  V ahead[PF];
#pragma unroll
  for (int i = 0; i < PF; i++) ahead[i] = load(i);

  auto tick = [&](auto phase, int i) {
    constexpr int P = decltype(phase)::value;
    V v = ahead[P];
    ahead[P] = load(min(i + PF, ticks - 1));
#pragma unroll
    for (int t = 0; t < T; t++) {  // v: row y of level t, which makes one of level t + 1
      const int y = first + i - R * t;
      if (EY && y < 0) return;  // (the next levels are further up still)
      if (EX) pad_columns(v);
      if (EY) {
        if (y >= H) v = zero_pad ? V(0.f) : last[t];
        last[t] = v;
      }
      float win[C + 2 * R];
#pragma unroll
      for (int q = 0; q < R; q++) {
        win[q] = neighbour<true>(v[C - R + q]);
        win[C + R + q] = neighbour<false>(v[q]);
      }
#pragma unroll
      for (int q = 0; q < C; q++) win[R + q] = v[q];
      auto add = [&](float (&a)[C], int dy, bool pad_row) {
#pragma unroll
        for (int q = 0; q < C; q++)
#pragma unroll
          for (int dx = 0; dx < K; dx++)
            a[q] = fmaf(pad_row && zero_pad ? 0.f : win[q + dx], wt[dy][dx], a[q]);
      };
      if (EY && y == 0) {  // output rows j < R start with the rows above the image
#pragma unroll
        for (int j = 0; j < R; j++) {
          float(&a)[C] = acc[t][(P + K - (R - j)) % K];
#pragma unroll
          for (int q = 0; q < C; q++) a[q] = 0.f;
#pragma unroll
          for (int dy = 0; dy < R - j; dy++) add(a, dy, true);
        }
      }
#pragma unroll
      for (int dy = K - 1; dy >= 0; dy--) {
        float(&a)[C] = acc[t][(P + K - dy) % K];
        if (dy == 0) {
#pragma unroll
          for (int q = 0; q < C; q++) a[q] = 0.f;
        }
        add(a, dy, false);
      }
#pragma unroll
      for (int q = 0; q < C; q++) v[q] = acc[t][(P + 1) % K][q];
    }
    const int y = first + i - R * T;
    if (y < y0) return;
    // (rows y0 .. y1 - 1, columns HALO .. of the strip inside the image)
    if (lane >= HALO / C && lane < 64 - HALO / C) {
      float* dst = out + (int64_t)y * ld_out + x;
      if (!EX || x + C <= W) {
        if (keep_out)  // the next launch reads it: leave it in the caches
          *reinterpret_cast<VU*>(dst) = VU(v);
        else
          __builtin_nontemporal_store(VU(v), reinterpret_cast<VU*>(dst));
      } else {
#pragma unroll
        for (int q = 0; q < C; q++)
          if (x + q < W) dst[q] = v[q];
      }
    }
  };
  auto ticks_from = [&](auto self, auto phase, int i) {
    constexpr int P = decltype(phase)::value;
    if constexpr (P < PF) {
      if (i + P >= ticks) return;
      tick(phase, i + P);
      self(self, std::integral_constant<int, P + 1>{}, i);
    }
  };
  for (int i = 0; i < ticks; i += PF) ticks_from(ticks_from, std::integral_constant<int, 0>{}, i);
}

// Bound by vector issue where there are several waves to a SIMD, and by a wave's own
// latency on small images: HALO columns and 2 R T rows of every strip and segment are
// computed again (4096^2, 5 x 5, four steps: 26.2 M FMAs needed, 44.4 M vector
// instructions issued, which fill 69 % of the launch; the three waves of a SIMD wait out
// their loads and shifts in the rest).  It replaced LDS tiles of 32
// rows by 128 columns, which read 96 bytes of LDS per eight outputs and step: 4096^2,
// 3 x 3, four steps a launch 18.5 -> 9.9 us per step, 256^2 3.9 -> 1.9; 5 x 5 35.5 ->
// 24 and 5.0 -> 4.0.
template <int K, int T>
__global__ __launch_bounds__(kThreads) void stencil_iter_fused(
    float* __restrict__ out, int64_t ld_out, const float* __restrict__ in, int64_t ld_in, int H,
    int W, const float* __restrict__ w, int zero_pad, int strips, int rows, int segments,
    int keep_out) {
  using Cfg = ItCfg<K, T>;
  const int64_t g =
      (int64_t)blockIdx.x * (kThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (g >= (int64_t)strips * segments) return;
  const int seg = (int)(g / strips), strip = (int)(g - (int64_t)seg * strips);
  const int xs = strip * Cfg::USE - Cfg::HALO, y0 = seg * rows, y1 = min(H, y0 + rows);
  float wt[K][K];
#pragma unroll
  for (int dy = 0; dy < K; dy++)
#pragma unroll
    for (int dx = 0; dx < K; dx++) wt[dy][dx] = w[dy * K + dx];
  constexpr int RT = Cfg::R * T;
  const bool inside_x = xs >= 0 && xs + 64 * C <= W, inside_y = y0 >= RT && y1 + RT <= H;
  auto run = [&](auto ex, auto ey) {
    iterate_segment<K, T, decltype(ex)::value, decltype(ey)::value>(
        out, ld_out, in, ld_in, H, W, wt, zero_pad, xs, y0, y1, keep_out);
  };
  if (!inside_y)
    run(std::true_type{}, std::true_type{});
  else if (!inside_x)
    run(std::true_type{}, std::false_type{});
  else
    run(std::false_type{}, std::false_type{});
}

template <int K, int T>
rise_status launch_fused_steps(const StencilArgs& a, hipStream_t s) {
  using Cfg = ItCfg<K, T>;
  const int64_t strips = ((int64_t)a.W + Cfg::USE - 1) / Cfg::USE;
  const int64_t simds = 4 * (int64_t)device_cu_count();
  // rows of a segment: the least time of the SIMD that gets the most waves.  A row of
  // four 3 x 3 steps takes one wave 0.61 us and two 0.59, six 1.18, eight 1.42; of
  // 5 x 5 steps one wave 0.7, two 1.1, three 1.4, nine 3.3
  double least = 0;
  int rows = 0;
  for (int r = 2; r <= 256; r += 1 + r / 16) {
    const int64_t per = (strips * (((int64_t)a.H + r - 1) / r) + simds - 1) / simds;
    const double cost =
        (K == 3 ? std::max(3.5, per + 1.2) : per + 1.4) * (r + 2 * Cfg::R * T);
    if (least == 0 || cost < least) least = cost, rows = r;
  }
  const int64_t segments = ((int64_t)a.H + rows - 1) / rows, blocks = (strips * segments + 3) / 4;
  if (blocks > INT32_MAX) return fail(RISE_ERR_SHAPE, "rise_stencil2d_iterate: too many tiles");
  hipLaunchKernelGGL((stencil_iter_fused<K, T>), dim3((unsigned)blocks), dim3(kThreads), 0, s,
                     a.out, a.ld_out, a.in, a.ld_in, a.H, a.W, a.w, (int)(a.pad == RISE_PAD_ZERO),
                     (int)strips, rows, (int)segments, (int)a.keep_out);
  return check_launch("stencil_iter_fused");
}
template <int K>
rise_status launch_fused(const StencilArgs& a, int steps, hipStream_t s) {
  switch (steps) {
    case 2: return launch_fused_steps<K, 2>(a, s);
    case 3: return launch_fused_steps<K, 3>(a, s);
    default: return launch_fused_steps<K, kItTMax>(a, s);
  }
}

int launches(int64_t steps, int fuse) { return (int)((steps + fuse - 1) / fuse); }

}  // namespace

bool stencil_iterate_fusable(int kh, int kw) { return kh == kw && (kh == 3 || kh == 5); }
int stencil_iterate_max_fuse() { return kItTMax; }

// Measured at 4096^2: for 3x3 four fused steps beat one launch per step (9.9 against
// 20 us per step).  For 5x5, whose recomputed halo costs up to half as much again as the
// steps, one launch per step and two, three and four steps fused take 94, 69, 70 and 71 us
// per step at 8192^2, past the last-level cache, 24.8, 21.9, 22.9 and 23.9 at 4096^2, 7.9,
// 8.4, 8.0 and 9.4 at 2047 x 1531, and 4.8, 5.3, 5.2 and 5.4 at 1000^2.
int stencil_iterate_default_fuse(int kh, int kw) {
  return kh == 3 && kw == 3 ? kItTMax : 1;
}

size_t stencil_iterate_workspace(int64_t H, int64_t W, int64_t steps, int fuse) {
  if (steps <= 1 || fuse < 1) return 0;
  const int L = launches(steps, fuse);
  const size_t img = ((size_t)H * W * 4 + 255) / 256 * 256;
  return L >= 3 ? 2 * img : L == 2 ? img : 0;
}

rise_status launch_stencil_iterate(const StencilArgs& a, int64_t steps, int fuse, void* ws,
                                   hipStream_t s) {
  if (steps == 0) {
    const hipError_t e = hipMemcpy2DAsync(a.out, a.ld_out * 4, a.in, a.ld_in * 4,
                                          (size_t)a.W * 4, a.H, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess)
      return fail(RISE_ERR_HIP, std::string("rise_stencil2d_iterate: copy: ") + hipGetErrorString(e));
    return RISE_OK;
  }
  const int L = launches(steps, fuse);
  const size_t img = ((size_t)a.H * a.W * 4 + 255) / 256 * 256;
  float* buf[2] = {(float*)ws, (float*)((char*)ws + img)};
  const float* src = a.in;
  int64_t ld_src = a.ld_in;
  for (int i = 0; i < L; i++) {
    const bool last = i == L - 1;
    StencilArgs b = a;
    b.in = src;
    b.ld_in = ld_src;
    b.out = last ? a.out : buf[i & 1];
    b.ld_out = last ? a.ld_out : a.W;
    b.keep_out = !last;  // the next launch reads it
    const int n = (int)std::min<int64_t>(fuse, steps - (int64_t)i * fuse);
    rise_status st;
    if (n == 1)
      st = launch_stencil2d(b, stencil_default_schedule(a.H, a.W, a.kh, a.kw), s);
    else if (a.kh == 3)
      st = launch_fused<3>(b, n, s);
    else
      st = launch_fused<5>(b, n, s);
    if (st != RISE_OK) return st;
    src = b.out;
    ld_src = b.ld_out;
  }
  return RISE_OK;
}

}  // namespace rise
