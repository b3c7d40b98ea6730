// Multi-channel stencil layer (a "convolution" layer): NHWC bfloat16 activations,
// FP32 weights rounded to bfloat16 for the matrix cores, FP32 accumulation.
//
//   out[b][y][x][co] = reduce(+, 0) over ci of
//                      stencil(pad2D(in[b][.][.][ci]), w[co][ci])     (3 x 3 window)
//
// is a contraction over K = (tap, ci) = 9 * Cin for every output pixel, i.e. an
// implicit GEMM with M = pixels and N = Cout: the window gather (pad2D |>
// slide2D) is an index view into an LDS halo tile, never materialised in HBM.
//
// Forward (and dIn, which is the same kernel on dOut with the window rotated by
// 180 degrees and the channel roles swapped): out^T = W' X with the prepared
// weights as the A operand, held in registers, and pixels as the B operand.
// dW (the gradient of the weights) contracts over pixels instead, with fragments
// read from LDS by the transpose read; a fixed-order reduction over workgroups
// finishes it.
// Both walk down strips of 64 pixel columns a row at a time, copy rows
// asynchronously several rows ahead, and use what a row brings (a pixel fragment
// forward, the input fragments of dW) for the three tap rows at once, so every
// row is fetched and read from LDS once.
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "async_copy.h"
#include "common.h"
#include "conv.h"

namespace rise {
namespace {

constexpr int kThreads = 256;
constexpr int TXP = 64;              // output pixels per row of a tile
constexpr int HC = TXP + 2;          // halo columns
constexpr int TAPS = 9;

// where the asynchronous copies take out-of-image pixels from
__device__ const i32x4 zero_page[16] = {};

__device__ __forceinline__ uint16_t f32_to_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Two floats to two bf16 (round to nearest even) in one 32-bit word, low half
// first: one v_cvt_pk_bf16_f32 on gfx950.
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}

// dst[o][tap * I + i] = bf16(weight), with
//   forward : o = co, i = ci, weight = w[co][ci][tap]
//   adjoint : o = ci, i = co, weight = w[co][ci][8 - tap]   (180-degree rotation)
__global__ void conv_prep_weights(uint16_t* __restrict__ dst, const float* __restrict__ w, int Cout,
                                  int Cin, int adjoint) {
  const int e = blockIdx.x * kThreads + threadIdx.x;
  if (e >= Cout * Cin * TAPS) return;
  const int co = e / (Cin * TAPS), rem = e - co * Cin * TAPS, ci = rem / TAPS, tap = rem % TAPS;
  const uint16_t v = f32_to_bf16(w[e]);
  if (!adjoint)
    dst[(int64_t)co * TAPS * Cin + tap * Cin + ci] = v;
  else
    dst[(int64_t)ci * TAPS * Cout + (TAPS - 1 - tap) * Cout + co] = v;
}

// Forward layer (and dIn with the adjoint weights): out^T = W' . X as an
// implicit GEMM with M = Cout (the prepared weights, A operand), N = pixels
// (B operand, gathered from LDS: pad2D |> slide2D as an index view) and
// K = 9 * Cin.
//   * a workgroup walks down a strip of 64 pixel columns; its waves own 32 output
//     channels x 32 columns each, and the weight fragments for every k-step stay
//     in registers (36 x 16 bytes per lane for 64 input channels), so only pixels
//     are read from LDS;
//   * an input row feeds three output rows (its taps dy = 0, 1, 2), whose
//     accumulators are open at the same time: a pixel fragment is read once for
//     three MFMAs and an input row is fetched once per strip.  One fragment per
//     MFMA, with tiles of two output rows, kept the LDS port busy as long as the
//     matrix cores and ran at 0.71 ms (64 -> 64 channels, 32 x 512 x 512);
//   * rows of 66 pixels are copied global -> LDS asynchronously into a ring of
//     NBUF rows, NBUF - 1 rows ahead; out-of-image pixels come from a page of zeros
//     (zero padding) or from the clamped pixel;
//   * the waits count instructions: every row issues the same copies (the tail
//     re-copies the strip's last row into a free buffer) and the same stores
//     (outputs that do not exist go to a 256-byte dump page), so "the copies of
//     the next row have landed" is a fixed vmcnt;
//   * pixels sit at an odd pitch of CH + 1 16-byte chunks, so the 16 pixels a
//     lane group reads at one chunk hit 16 distinct bank slots, and every
//     fragment read of a row is one base register plus an immediate offset;
//   * the weight rows are permuted so that the D layout gives each lane 16
//     consecutive output channels of its pixel: two 16-byte stores of bf16.
// The order of every output's sum is (tap, ci), as stored in the weights.
template <int CI, int CO>
struct FwdCfg {
  static constexpr int CH = CI / 8;                 // 16-byte chunks per pixel
  static constexpr int NCB = CO / 32;               // cout blocks
  static constexpr int WAVES = 2 * NCB;             // x two blocks of 32 pixels
  static constexpr int KC = CI / 16;                // k-steps of 16 per tap
  static constexpr int PITCH = CH + 1;              // chunks per halo pixel (odd)
  static constexpr int SLOTS = HC * PITCH;          // chunks of a row
  static constexpr int NQ = (SLOTS + 63) / 64;      // wave-sized copies per row
  static constexpr int QPW = (NQ + WAVES - 1) / WAVES;  // copies per wave (at most)
  // two waves per SIMD (the weights take 144 of 256 registers): 8 / WAVES
  // workgroups share the LDS
  static constexpr int FIT = 19 * WAVES / NQ;
  static constexpr int NBUF = FIT > 8 ? 8 : FIT;
  static constexpr int XPF = CI == 64 ? 3 : 2;      // fragment lookahead (k-steps); the
                                                    // register ring divides a row's steps
  static constexpr int AHEAD = NBUF >= 5;           // rows visible before they are needed
  static_assert(NBUF >= 3, "ring");
};

template <int CI, int CO>
__global__ __launch_bounds__((64 * FwdCfg<CI, CO>::WAVES), 2) void conv3x3_fwd(
    uint16_t* __restrict__ out, const uint16_t* __restrict__ in,
    const uint16_t* __restrict__ wp, uint16_t* __restrict__ dump_page, int H, int W, int zero_pad,
    int tiles_x, int segs, int rows) {
  using F = FwdCfg<CI, CO>;
  constexpr int CH = F::CH, NCB = F::NCB, KC = F::KC, NQ = F::NQ, QPW = F::QPW, WAVES = F::WAVES;
  constexpr int NBUF = F::NBUF, DIST = NBUF - 1, XPF = F::XPF, AHEAD = F::AHEAD;
  constexpr int NST = 2;  // stores per wave per row
  __shared__ i32x4 halo[NBUF][NQ * 64];  // padded to whole copies; the tail is never read
  __shared__ i32x4 turn[WAVES][128];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int il = lane & 31, kh = lane >> 5;
  const int wcb = wave % NCB, wpb = wave / NCB;
  const int tx = blockIdx.x % tiles_x, sy = (blockIdx.x / tiles_x) % segs,
            b = blockIdx.x / tiles_x / segs;
  const int x0 = tx * TXP, y0 = sy * rows, R = min(rows, H - y0);  // output rows y0 .. y0 + R - 1

  // copies of this lane: copy q of this wave fills slot (wave + WAVES q) * 64 +
  // lane = pixel p, chunk c; byte offset from the strip's first pixel, or from the
  // zero page for out-of-image pixels, padding chunks and the tail
  int off[QPW];
  uint32_t inside = 0;
#pragma unroll
  for (int q = 0; q < QPW; q++) {
    const int sl = (wave + WAVES * q) * 64 + lane, p = sl / F::PITCH, c = sl - p * F::PITCH;
    const int gx = x0 - 1 + p, gxc = gx < 0 ? 0 : (gx >= W ? W - 1 : gx);
    off[q] = (gxc - x0) * (CI * 2) + c * 16;
    if (p < HC && c < CH && (gx == gxc || (!zero_pad && gx <= W))) inside |= 1u << q;
  }
  const int64_t row_bytes = (int64_t)W * CI * 2;
  const char* strip = (const char*)in + ((int64_t)b * H * W + x0) * (CI * 2);
  // input row i of the segment (image row y0 - 1 + i) into ring buffer buf
  auto issue = [&](int i, int buf) {
    const int r = y0 - 1 + min(i, R + 1), rc = r < 0 ? 0 : (r >= H ? H - 1 : r);
    const bool row_ok = r == rc || !zero_pad;
    const char* row = strip + rc * row_bytes;
#pragma unroll
    for (int q = 0; q < QPW; q++)
      if (q + 1 < QPW || wave + WAVES * q < NQ)
        async::copy16(row_ok && (inside >> q & 1u) ? (const void*)(row + off[q])
                                                   : zero_page + (lane & 15),
                      &halo[buf][(wave + WAVES * q) * 64]);
  };

  // weight fragments: lane (il, kh) holds w'[co][16 ks + 8 kh .. +8] of the output
  // channel that makes D row il the lane's channel 4 (il / 8) + il % 4 of 16
  bf16x8 wf[TAPS * KC];
  {
    const int co = wcb * 32 + 16 * ((il >> 2) & 1) + 4 * (il >> 3) + (il & 3);
    const uint16_t* wr = wp + (int64_t)co * (TAPS * CI) + 8 * kh;
#pragma unroll
    for (int ks = 0; ks < TAPS * KC; ks++)
      wf[ks] = *reinterpret_cast<const bf16x8*>(wr + 16 * ks);
  }
  const bool full_copies = wave + WAVES * (QPW - 1) < NQ;  // wave-uniform
  for (int d = 0; d < DIST; d++) issue(d, d);
  async::wait_vmcnt<0>();  // the first rows' copies (and the weight loads) have landed

  const int xs = x0 + 32 * wpb + (lane >> 2);  // this lane's pixel and chunk in a store
  uint16_t* const out_px = out + (((int64_t)b * H + y0) * W + xs) * CO + wcb * 32 + 8 * (lane & 3);
  f32x16 acc[3] = {};
  int buf = 0;
  constexpr int STEPS = 3 * KC;  // (dx, 16 channels)
  static_assert(STEPS % (XPF + 1) == 0, "fragment ring");
  bf16x8 xf[XPF + 1];
  auto read_x = [&](int st, int from) {
    xf[st % (XPF + 1)] = __builtin_bit_cast(
        bf16x8, halo[from][(32 * wpb + il + st / KC) * F::PITCH + kh + 2 * (st % KC)]);
  };
  if (AHEAD) {
    async::barrier();
#pragma unroll
    for (int st = 0; st < XPF; st++) read_x(st, 0);
  }
  // input row i: opens the accumulator of output row i, adds to that of row i - 1
  // and closes that of row i - 2 (slots modulo 3; P = i % 3)
  auto row_step = [&](auto phase, int i) {
    constexpr int P = decltype(phase)::value, S0 = P, S1 = (P + 2) % 3, S2 = (P + 1) % 3;
    async::wait_lgkmcnt0();  // this wave's reads of the previous row are done
    async::barrier();        // every wave's copies into halo[buf] are visible
    const int next = buf + 1 == NBUF ? 0 : buf + 1;
    if (!AHEAD)
#pragma unroll
      for (int st = 0; st < XPF; st++) read_x(st, buf);
#pragma unroll
    for (int st = 0; st < STEPS; st++) {
      if (st + XPF < STEPS)
        read_x(st + XPF, buf);
      else if (AHEAD)
        read_x(st + XPF - STEPS, next);  // the next row's first fragments
      const bf16x8 v = xf[st % (XPF + 1)];
      const f32x16 zero = {};
      acc[S2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[2 * STEPS + st], v, acc[S2], 0, 0, 0);
      acc[S1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[STEPS + st], v, acc[S1], 0, 0, 0);
      acc[S0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[st], v, st ? acc[S0] : zero, 0, 0, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one LDS read
      __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);  // three MFMAs
      if (st == 0) issue(i + DIST, buf == 0 ? NBUF - 1 : buf - 1);  // the previous row's buffer
    }
    // the wave's 32 pixels x 4 chunks, turned so that four lanes store the 64
    // consecutive bytes of a pixel
#pragma unroll
    for (int h = 0; h < 2; h++) {
      i32x4 v;
#pragma unroll
      for (int e = 0; e < 4; e++)
        v[e] = (int)pack_bf16x2(acc[S2][8 * h + 2 * e], acc[S2][8 * h + 2 * e + 1]);
      turn[wave][il * 4 + ((2 * kh + h) ^ ((il >> 1) & 3))] = v;
    }
#pragma unroll
    for (int h = 0; h < 2; h++) {
      const int pl = 16 * h + (lane >> 2);
      const i32x4 v = turn[wave][pl * 4 + ((lane & 3) ^ ((pl >> 1) & 3))];
      uint16_t* dst = i >= 2 && xs + 16 * h < W ? out_px + ((int64_t)(i - 2) * W + 16 * h) * CO
                                                : dump_page + 8 * (lane & 3);
      *reinterpret_cast<i32x4*>(dst) = v;
    }
    buf = next;
    // the copies of row i + 1 + AHEAD have landed: younger than them are the copies
    // of the rows up to i + DIST and the stores of the DIST - AHEAD latest rows
    // (this one's included)
    constexpr int ROWS = DIST - AHEAD;
    if (full_copies)
      async::wait_vmcnt<ROWS * NST + (ROWS - 1) * QPW>();
    else
      async::wait_vmcnt<ROWS * NST + (ROWS - 1) * (QPW - 1)>();
  };
  for (int i = 0;;) {
    row_step(std::integral_constant<int, 0>{}, i);
    if (++i == R + 2) break;
    row_step(std::integral_constant<int, 1>{}, i);
    if (++i == R + 2) break;
    row_step(std::integral_constant<int, 2>{}, i);
    if (++i == R + 2) break;
  }
  async::wait_vmcnt<0>();  // no copy outlives the workgroup's LDS
}

// ---------------------------------------------------------------------------
// dW: each workgroup accumulates dW^T restricted to its pixels.
//   dWt[o][tap * CI + ci] = sum over pixels of dOut[px][o] * in[px shifted by tap][ci]
// M = output channels (A operand: dOut), N = input channels of one tap (B operand:
// in), K = pixels, 16 of one row per MFMA, 8 per lane.
//   * a workgroup walks down strips of 64 pixel columns; a wave owns 32 output
//     channels x 32 input channels of all nine taps (9 accumulators) and KXS of
//     the four 16-pixel groups of a row;
//   * rows of dOut and of the input are copied global -> LDS asynchronously into
//     a ring of NBUF row pairs, NBUF - 2 pairs ahead, as stored (NHWC), and the
//     fragments, which need 8 pixels of one channel per lane, are read with the
//     gfx950 LDS transpose read ds_read_b64_tr_b16.  Within each group of 16 lanes
//     it takes the 16 addresses as a 16 x 4 block of 16-bit values M[s][e] (lane s
//     supplies the 4 values at its address) and returns M[4 j + i / 4][i % 4] as
//     element j of lane i.  With source lane s = 4 j + q pointing at channels
//     c0 + 4 q .. + 3 of pixel p(j), lane i receives channel c0 + i of the pixels
//     p(0) .. p(3);
//   * which pixel sits where in K is free as long as both operands agree: register
//     j of a fragment holds pixels (j, j + 4) of the lane's run, so the fragment
//     of the next tap column is the same registers shifted by one.  Three reads
//     of one row serve its three tap columns, and the registers of the last three
//     input rows are kept, so they serve the three tap rows as well: five reads
//     (two for dOut) per nine MFMAs.  One read pair per tap, staged through
//     registers one tile ahead, took 1.02 ms (64 -> 64 channels, 32 x 512 x 512);
//   * 32 lanes read 64 bytes of four pixels (0, 4, 1, 5) at a time, which have to
//     lie in different banks: with 64 channels the 64-byte halves of a pixel are
//     exchanged by bit 2 of its index, with 32 channels bits 1 and 2 of the index
//     are exchanged (px_slot, px_half);
//   * the next row's fragments are read while this row's MFMAs run.
// ---------------------------------------------------------------------------
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// 4 pixels of one channel per lane (see above); p points at the four values this
// lane supplies as a source.
__device__ __forceinline__ s16x4 read_tr16(const char* p) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
#else
  return s16x4{0, 0, 0, 0};
#endif
}

// place of pixel p (C channels of 2 bytes) in its row, and which 64-byte half
// comes first (see above); px_slot is its own inverse
template <int C>
__device__ __forceinline__ int px_slot(int p) {
  return C == 64 ? p : (p & ~6) | (p >> 1 & 2) | (p << 1 & 4);
}
template <int C>
__device__ __forceinline__ int px_half(int p) {
  return C == 64 ? p >> 2 & 1 : 0;
}

template <int CI, int CO>
struct DwCfg {
  static constexpr int NH = CI / 32, MB = CO / 32, UNITS = NH * MB;  // 32 x 32 blocks per tap
  static constexpr int KXW = UNITS == 4 ? 2 : 4;    // waves along the row's pixels
  static constexpr int KXS = 4 / KXW;               // groups of 16 pixels per wave
  static constexpr int WAVES = UNITS * KXW;
  static constexpr int CH = CI / 8, OH = CO / 8;    // 16-byte chunks per pixel
  static constexpr int XQ = (68 * CH + 63) / 64;    // copies of an input row: 66 pixels,
                                                    // and 2 read but never used
  static constexpr int GQ = OH;                     // copies of a dOut row: 64 pixels
  static constexpr int NQ = XQ + GQ;
  static constexpr int QPW = (NQ + WAVES - 1) / WAVES;
  static constexpr int NBUF = 8;                    // ring of row pairs
  static constexpr int WGS = 8 / WAVES;             // workgroups per CU: two waves per SIMD
  static_assert(NBUF * NQ * 1024 * WGS <= 160 * 1024, "LDS");
};

template <int CI, int CO>
__global__ __launch_bounds__((64 * DwCfg<CI, CO>::WAVES), 2) void conv3x3_dw(
    float* __restrict__ partial, const uint16_t* __restrict__ dout,
    const uint16_t* __restrict__ in, int H, int W, int zero_pad, int tiles_x, int segs, int rows,
    int nseg) {
  using D = DwCfg<CI, CO>;
  constexpr int CH = D::CH, OH = D::OH, XQ = D::XQ, NQ = D::NQ, QPW = D::QPW, WAVES = D::WAVES;
  constexpr int KXS = D::KXS, NBUF = D::NBUF;
  __shared__ i32x4 ring[NBUF][NQ * 64];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int il = lane & 31, kh = lane >> 5;
  const int unit = wave % D::UNITS, kxw = wave / D::UNITS;
  const int nh = unit % D::NH, mb = unit / D::NH;
  // this lane's source addresses: pixel 8 kh + {0, 4, 1, 5}[j] (+ 2, + 4), 8 bytes of
  // the 32 of its 16 channels
  const int j = (lane & 15) >> 2, ch = 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
  const int px = 16 * KXS * kxw + 8 * kh + (j >> 1) + 4 * (j & 1);
  auto x_at = [&](int p) { return px_slot<CI>(p) * (CI * 2) + 64 * (nh ^ px_half<CI>(p)) + ch; };
  auto g_at = [&](int p) {
    return XQ * 1024 + px_slot<CO>(p) * (CO * 2) + 64 * (mb ^ px_half<CO>(p)) + ch;
  };
  const int xa[3] = {x_at(px), x_at(px + 2), x_at(px + 4)}, ga[2] = {g_at(px), g_at(px + 2)};

  f32x16 acc[TAPS] = {};
  const char* const lds = (const char*)&ring[0][0];
  for (int seg = blockIdx.x; seg < nseg; seg += gridDim.x) {
    const int tx = seg % tiles_x, sy = (seg / tiles_x) % segs, b = seg / tiles_x / segs;
    const int x0 = tx * TXP, y0 = sy * rows, R = min(rows, H - y0);  // dOut rows y0 .. y0 + R - 1
    // copies of this lane: copy q of this wave is row copy g = wave + WAVES q, of
    // the input (g < XQ) or of dOut; slot 64 g + lane = pixel p, chunk c
    int off[QPW];
    uint32_t inside = 0;
#pragma unroll
    for (int q = 0; q < QPW; q++) {
      const int g = wave + WAVES * q;
      if (g < XQ) {
        const int sl = g * 64 + lane, p = px_slot<CI>(sl / CH);
        const int c = (sl % CH) ^ 4 * px_half<CI>(p);
        const int gx = x0 - 1 + p, gxc = gx < 0 ? 0 : (gx >= W ? W - 1 : gx);
        off[q] = (gxc - x0) * (CI * 2) + c * 16;
        if (p < HC && (gx == gxc || (!zero_pad && gx <= W))) inside |= 1u << q;
      } else {
        const int sl = (g - XQ) * 64 + lane, p = px_slot<CO>(sl / OH);
        const int c = (sl % OH) ^ 4 * px_half<CO>(p);
        off[q] = p * (CO * 2) + c * 16;
        if (x0 + p < W) inside |= 1u << q;  // outputs outside the image do not exist
      }
    }
    const int64_t xrow = (int64_t)W * CI * 2, grow = (int64_t)W * CO * 2;
    const char* xs = (const char*)in + ((int64_t)b * H * W + x0) * (CI * 2);
    const char* gs = (const char*)dout + ((int64_t)b * H * W + x0) * (CO * 2);
    // row pair i: input row y0 - 1 + i and dOut row y0 + i - 2 (for i >= 2)
    auto issue = [&](int i, int buf) {
      const int ic = min(i, R + 1), r = y0 - 1 + ic, rc = r < 0 ? 0 : (r >= H ? H - 1 : r);
      const bool row_ok = r == rc || !zero_pad;
      const char* xp = xs + rc * xrow;
      const char* gp = gs + (y0 + max(ic - 2, 0)) * grow;
#pragma unroll
      for (int q = 0; q < QPW; q++) {
        const int g = wave + WAVES * q;
        if (q + 1 < QPW || g < NQ) {
          const bool ok = (inside >> q & 1u) && (g >= XQ || row_ok);
          async::copy16(ok ? (const void*)((g < XQ ? xp : gp) + off[q])
                           : zero_page + (lane & 15),
                        &ring[buf][g * 64]);
        }
      }
    };
    const bool full_copies = wave + WAVES * (QPW - 1) < NQ;

    s16x4 bv[3][KXS][3], av[KXS][2], an[KXS][2];
    auto read_b = [&](s16x4* v, int kx, int at) {
      const char* p = lds + at * (NQ * 1024) + kx * (16 * CI * 2);
#pragma unroll
      for (int u = 0; u < 3; u++) v[u] = read_tr16(p + xa[u]);
    };
    auto read_a = [&](s16x4* v, int kx, int at) {
      const char* p = lds + at * (NQ * 1024) + kx * (16 * CO * 2);
#pragma unroll
      for (int u = 0; u < 2; u++) v[u] = read_tr16(p + ga[u]);
    };
    auto frag = [](s16x4 lo, s16x4 hi) {
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // one tap row: accumulators 3 dy .. 3 dy + 2
    auto taps = [&](int dy, const s16x4* a, const s16x4* v) {
      const bf16x8 af = frag(a[0], a[1]);
      const bf16x8 b[3] = {frag(v[0], v[1]),
                           frag(__builtin_shufflevector(v[0], v[1], 2, 3, 4, 5),
                                __builtin_shufflevector(v[1], v[2], 2, 3, 4, 5)),
                           frag(v[1], v[2])};
#pragma unroll
      for (int dx = 0; dx < 3; dx++)
        acc[3 * dy + dx] =
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, b[dx], acc[3 * dy + dx], 0, 0, 0);
    };

    async::wait_lgkmcnt0();
    async::barrier();  // every wave is done with the previous segment's rows
#pragma unroll
    for (int d = 0; d < NBUF; d++) issue(d, d);
    if (full_copies)  // rows 0, 1 and 2 (at least three exist: R >= 1)
      async::wait_vmcnt<(NBUF - 3) * QPW>();
    else
      async::wait_vmcnt<(NBUF - 3) * (QPW - 1)>();
    async::barrier();
#pragma unroll
    for (int kx = 0; kx < KXS; kx++) {
      read_b(bv[0][kx], kx, 0);
      read_b(bv[1][kx], kx, 1);
      read_b(bv[2][kx], kx, 2);
      read_a(av[kx], kx, 2);
    }
    async::wait_lgkmcnt0();
    async::barrier();  // rows 0 and 1 have been read
    issue(NBUF, 0);
    issue(NBUF + 1, 1);
    // dOut row i - 2 against the input rows i - 2, i - 1 and i (slots modulo 3, P =
    // i % 3); reads row i + 1 into the slot of row i - 2 when that is done
    auto row_step = [&](auto phase, int i) {
      constexpr int P = decltype(phase)::value, S0 = (P + 1) % 3, S1 = (P + 2) % 3, S2 = P;
      const int nb = (i + 1) % NBUF;
      // this wave's copies of row i + 1 have landed (those of rows i + 2 .. i + NBUF
      // - 1 are younger) and its reads of row i are done
      if (full_copies)
        async::wait_vmcnt<(NBUF - 2) * QPW>();
      else
        async::wait_vmcnt<(NBUF - 2) * (QPW - 1)>();
      async::wait_lgkmcnt0();
      async::barrier();
#pragma unroll
      for (int kx = 0; kx < KXS; kx++) {
        taps(0, av[kx], bv[S0][kx]);
        read_b(bv[S0][kx], kx, nb);
        read_a(an[kx], kx, nb);
        taps(1, av[kx], bv[S1][kx]);
        if (kx == 0) issue(i + NBUF, i % NBUF);
        taps(2, av[kx], bv[S2][kx]);
        __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 5, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
        av[kx][0] = an[kx][0];
        av[kx][1] = an[kx][1];
      }
    };
    for (int i = 2;;) {
      row_step(std::integral_constant<int, 2>{}, i);
      if (++i == R + 2) break;
      row_step(std::integral_constant<int, 0>{}, i);
      if (++i == R + 2) break;
      row_step(std::integral_constant<int, 1>{}, i);
      if (++i == R + 2) break;
    }
    async::wait_vmcnt<0>();  // no copy outlives its segment
  }
  // partial[block][o][n] of dW^T: the KXW waves of a 32 x 32 block add their sums
  // through LDS, a tap row at a time, each an equal part of it
  constexpr int PART = 48 / D::KXW;
  float* const sum = (float*)&ring[0][0];  // [wave][48][64]
  static_assert(WAVES * 48 * 64 * 4 <= (int)sizeof(ring), "sums in the ring");
  float* const dst = partial + (int64_t)blockIdx.x * CO * TAPS * CI;
#pragma unroll
  for (int dy = 0; dy < 3; dy++) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < D::KXW; k++)
      if (k != kxw)
#pragma unroll
        for (int e = PART * k; e < PART * (k + 1); e++)
          sum[(wave * 48 + e) * 64 + lane] = acc[3 * dy + e / 16][e % 16];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < D::KXW; k++)
      if (k == kxw)
#pragma unroll
        for (int e = PART * k; e < PART * (k + 1); e++) {
          const int t = 3 * dy + e / 16, r = e % 16, o = 32 * mb + 8 * (r >> 2) + 4 * kh + (r & 3);
          float v = 0.f;
#pragma unroll
          for (int w = 0; w < D::KXW; w++)
            v += w == k ? acc[t][r] : sum[((unit + D::UNITS * w) * 48 + e) * 64 + lane];
          dst[(int64_t)o * TAPS * CI + t * CI + 32 * nh + il] = v;
        }
  }
}

// dW[co][ci][tap] = sum over blocks of partial[block][co][tap * CI + ci] (fixed
// order: each wave of a workgroup sums a quarter of the blocks, 16 loads in
// flight; one thread per element over all of them was a serial chain of loads, 30
// us for 512 blocks)
__global__ __launch_bounds__(kThreads) void conv_dw_reduce(float* __restrict__ dw,
                                                           const float* __restrict__ partial,
                                                           int blocks, int CO, int CI) {
  __shared__ float part[kThreads / 64][64];
  const int n = CO * TAPS * CI;  // a multiple of 64
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + lane, share = (blocks + 3) / 4;
  int q = wave * share;
  const int q1 = min(blocks, q + share);
  float s = 0.f;
  for (; q + 16 <= q1; q += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; u++) v[u] = partial[(int64_t)(q + u) * n + e];
#pragma unroll
    for (int u = 0; u < 16; u++) s += v[u];
  }
  for (; q < q1; q++) s += partial[(int64_t)q * n + e];
  part[wave][lane] = s;
  __syncthreads();
  if (wave) return;
  s = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
  const int o = e / (TAPS * CI), rem = e - o * TAPS * CI, tap = rem / CI, ci = rem - tap * CI;
  dw[((int64_t)o * CI + ci) * TAPS + tap] = s;
}

// Rows of a segment (a strip of 64 columns is cut into segments of whole rows, one
// workgroup each): the cheapest by cost(segments of all strips, rows), over counts
// per strip in steps of an eighth and those that fill `slots` workgroups evenly.
template <typename Cost>
int segment_rows(int64_t strips, int H, int64_t slots, int min_rows, Cost cost) {
  int best = std::max(H, 1);
  if (strips < 1 || H < 1) return best;
  double best_cost = cost(strips, H);
  const int64_t most = std::min<int64_t>((H + min_rows - 1) / min_rows, 8 * slots / strips);
  auto look = [&](int64_t n) {
    if (n < 2 || n > most) return;
    const int rows = (int)((H + n - 1) / n);
    const double c = cost(strips * ((H + rows - 1) / rows), rows);
    if (c < best_cost) best_cost = c, best = rows;
  };
  for (int64_t n = 2; n <= most; n += std::max<int64_t>(1, n / 8)) look(n);
  for (int k = 1; k <= 8; k++) look(k * slots / strips);
  return best;
}

// The dW kernel's segments and workgroups (each sums its segments in registers).
struct DwSplit {
  int tiles_x, segs, rows, nseg, blocks;
};
DwSplit dw_split(int B, int CI, int CO, int H, int W) {
  const int64_t slots = 256 * ((CI / 32) * (CO / 32) == 1 ? 2 : 1);  // on 256 CUs
  DwSplit d;
  d.tiles_x = (W + TXP - 1) / TXP;
  const int64_t strips = (int64_t)B * d.tiles_x;
  // in rows: a workgroup's rounds of rows plus its start and end, and writing and
  // reading its partial sums (128 x 128 x 2 images of 64 -> 64 channels: 256
  // segments of 2 rows 30 us, 64 of 8 rows 20 us)
  d.rows = segment_rows(strips, H, slots, 2, [&](int64_t segs, int rows) {
    return (double)((segs + slots - 1) / slots) * (rows + 10) + std::min(segs, slots) * 0.1;
  });
  d.segs = (H + d.rows - 1) / d.rows;
  d.nseg = (int)(strips * d.segs);
  d.blocks = (int)std::min<int64_t>(d.nseg, slots);
  return d;
}

template <int CI, int CO>
rise_status launch_fwd(uint16_t* out, const uint16_t* in, const uint16_t* wp,
                       uint16_t* dump_page, int B, int H, int W, int zero, hipStream_t s) {
  constexpr int WAVES = FwdCfg<CI, CO>::WAVES;
  const int tiles_x = (W + TXP - 1) / TXP;
  if ((int64_t)B * tiles_x * ((H + 1) / 2) > INT32_MAX)
    return fail(RISE_ERR_SHAPE, "conv: too many tiles");
  // in rows per CU: two halo rows, the weights and the first copies cost about six;
  // a CU whose two waves per SIMD are not there runs at two thirds
  const int64_t cus = device_cu_count(), per_cu = 8 / WAVES;
  const int rows = segment_rows((int64_t)B * tiles_x, H, cus, 1, [&](int64_t segs, int rows) {
    const int64_t k = (segs + cus - 1) / cus;
    return (k < per_cu ? 1.5 * per_cu / 2 : (double)k) * (rows + 6);
  });
  const int segs = (H + rows - 1) / rows;
  hipLaunchKernelGGL((conv3x3_fwd<CI, CO>), dim3((unsigned)(B * tiles_x * segs)), dim3(64 * WAVES),
                     0, s, out, in, wp, dump_page, H, W, zero, tiles_x, segs, rows);
  return check_launch("conv3x3_fwd");
}

template <int CI, int CO>
rise_status launch_dw(float* partial, const uint16_t* dout, const uint16_t* in,
                      int B, int H, int W, int zero, hipStream_t s) {
  const DwSplit d = dw_split(B, CI, CO, H, W);
  hipLaunchKernelGGL((conv3x3_dw<CI, CO>), dim3(d.blocks), dim3(64 * DwCfg<CI, CO>::WAVES), 0, s,
                     partial, dout, in, H, W, zero, d.tiles_x, d.segs, d.rows, d.nseg);
  return check_launch("conv3x3_dw");
}

rise_status fwd_dispatch(uint16_t* out, const uint16_t* in, const uint16_t* wp,
                         uint16_t* dump_page, int B, int CI, int CO, int H, int W, int zero,
                         hipStream_t s) {
#define RISE_CONV_CASE(I, O) \
  if (CI == I && CO == O)    \
    return launch_fwd<I, O>(out, in, wp, dump_page, B, H, W, zero, s);
  RISE_CONV_CASE(16, 32) RISE_CONV_CASE(16, 64) RISE_CONV_CASE(32, 32)
  RISE_CONV_CASE(32, 64) RISE_CONV_CASE(64, 32) RISE_CONV_CASE(64, 64)
#undef RISE_CONV_CASE
  return fail(RISE_ERR_UNSUPPORTED, "conv: channel counts");
}

rise_status dw_dispatch(float* partial, const uint16_t* dout, const uint16_t* in, int B, int CI,
                        int CO, int H, int W, int zero, hipStream_t s) {
  if (CI == 32 && CO == 32) return launch_dw<32, 32>(partial, dout, in, B, H, W, zero, s);
  if (CI == 32 && CO == 64) return launch_dw<32, 64>(partial, dout, in, B, H, W, zero, s);
  if (CI == 64 && CO == 32) return launch_dw<64, 32>(partial, dout, in, B, H, W, zero, s);
  if (CI == 64 && CO == 64) return launch_dw<64, 64>(partial, dout, in, B, H, W, zero, s);
  return fail(RISE_ERR_UNSUPPORTED, "conv backward: channel counts");
}

rise_status prep_weights(uint16_t* dst, const float* w, int Cout, int Cin, int adjoint,
                         hipStream_t s) {
  hipLaunchKernelGGL(conv_prep_weights, dim3((Cout * Cin * TAPS + kThreads - 1) / kThreads),
                     dim3(kThreads), 0, s, dst, w, Cout, Cin, adjoint);
  return check_launch("conv_prep_weights");
}

size_t round256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

bool conv_supported(int Cin, int Cout, int kh, int kw, bool backward) {
  if (kh != 3 || kw != 3) return false;
  bool fwd_ok = (Cin == 16 || Cin == 32 || Cin == 64) && (Cout == 32 || Cout == 64);
  if (!backward) return fwd_ok;
  // backward runs the forward kernel with the roles of Cin and Cout swapped (dIn) and the
  // dW kernel
  bool din_ok = (Cout == 16 || Cout == 32 || Cout == 64) && (Cin == 32 || Cin == 64);
  bool dw_ok = (Cin == 32 || Cin == 64) && (Cout == 32 || Cout == 64);
  return din_ok && dw_ok;
}

// workspace: [prepared bf16 weights | 256-byte dump page | dW partials (backward)]
size_t conv_forward_workspace(int Cin, int Cout) {
  return round256((size_t)Cout * TAPS * Cin * 2) + 256;
}

size_t conv_backward_workspace(int B, int Cin, int Cout, int H, int W) {
  return conv_forward_workspace(Cin, Cout) +
         (size_t)dw_split(B, Cin, Cout, H, W).blocks * Cout * TAPS * Cin * 4;
}

rise_status launch_conv2d(const ConvArgs& a, void* ws, hipStream_t s) {
  uint16_t* wp = (uint16_t*)ws;
  uint16_t* dump_page = (uint16_t*)((char*)ws + round256((size_t)a.Cout * TAPS * a.Cin * 2));
  rise_status st = prep_weights(wp, a.w, a.Cout, a.Cin, 0, s);
  if (st != RISE_OK) return st;
  return fwd_dispatch(a.out, a.in, wp, dump_page, a.B, a.Cin, a.Cout, a.H, a.W, a.zero_pad, s);
}

rise_status launch_conv2d_backward(const ConvBwdArgs& a, void* ws, hipStream_t s) {
  uint16_t* wp = (uint16_t*)ws;
  uint16_t* dump_page = (uint16_t*)((char*)ws + round256((size_t)a.Cout * TAPS * a.Cin * 2));
  float* partial = (float*)((char*)ws + conv_forward_workspace(a.Cin, a.Cout));
  rise_status st = RISE_OK;
  if (a.din) {
    // dIn = the layer with dOut as input, channel roles swapped and the window rotated
    if ((st = prep_weights(wp, a.w, a.Cout, a.Cin, 1, s)) != RISE_OK) return st;
    st = fwd_dispatch(a.din, a.dout, wp, dump_page, a.B, a.Cout, a.Cin, a.H, a.W, 1, s);
    if (st != RISE_OK) return st;
  }
  if (a.dw) {
    st = dw_dispatch(partial, a.dout, a.in, a.B, a.Cin, a.Cout, a.H, a.W, a.zero_pad, s);
    if (st != RISE_OK) return st;
    const int n = a.Cout * TAPS * a.Cin;
    hipLaunchKernelGGL(conv_dw_reduce, dim3(n / 64), dim3(kThreads), 0, s,
                       a.dw, partial, dw_split(a.B, a.Cin, a.Cout, a.H, a.W).blocks, a.Cout, a.Cin);
    if ((st = check_launch("conv_dw_reduce")) != RISE_OK) return st;
  }
  return RISE_OK;
}

}  // namespace rise
