// Tile-level device functions shared by the one-problem kernels and the
// persistent batched kernel.  Each function computes one output tile with the
// whole workgroup (256 threads for a stencil tile, RingCfg::THREADS for a GEMM tile)
// and takes its LDS through a pointer, so a kernel that runs several kinds of tiles
// can overlay them in one buffer.
#pragma once

#include <type_traits>

#include "async_copy.h"
#include "common.h"

namespace rise {
namespace tiles {

constexpr int kThreads = 256;

// a 16-byte vector of floats that may sit at any 4-byte boundary (gfx950 runs
// global memory in unaligned-access mode: one dwordx4 access either way)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ int clampi(int v, int lo, int hi) {
  return v < lo ? lo : (v > hi ? hi : v);
}

// Four bf16 values of one column from four consecutive LDS rows (gfx950
// ds_read_b64_tr_b16).  Within each group of 16 lanes, lane s supplies the
// address of 4 consecutive 16-bit values M[s][0..3] and lane i receives
// M[4 j + i / 4][i % 4] as element j: with lane s = 4 j + q pointing at
// columns c0 + 4 q .. c0 + 4 q + 3 of row r0 + j, lane i receives column
// c0 + i of rows r0 .. r0 + 3.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ s16x4_t lds_read_tr16(const void* p) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)p);
#else
  (void)p;
  return s16x4_t{0, 0, 0, 0};
#endif
}

// ===========================================================================
// GEMM tile: C[m0:m0+BM, n0:n0+BN] = A B, FP32 (v_mfma_f32_32x32x2_f32) or bf16
// operands with FP32 accumulation (v_mfma_f32_32x32x16_bf16)
//
// Pattern -> hardware mapping (paper Sec. IV-B/C: splitJoinMap, the map lowerings
// and fuseReduceMap; Sec. V-C: toMem and reduceSeq): the workgroup owns one
// split(BM) x split(BN) tile (mapWorkGroup); its 2 x 2 sub-tiles go to the four
// waves (mapLocal); split(BK) + reduceSeq(Private) is the K loop with register
// accumulators; each slab is staged in LDS (toMem(Local)); zip |> map(*) |>
// reduce(+) is the matrix instruction; join . join is the guarded row-major
// store.  Operands may be read through transpose (TA, TB) without copies.
//
// Slabs flow global -> LDS through a ring of STAGES buffers by asynchronous
// copies (global_load_lds: lane i's bytes land at the wave-uniform base + its
// size * i; no registers hold data in flight), STAGES - 1 slabs ahead.  Each
// operand's slab (BK values of k by BM or BN values of m or n) is staged in the
// orientation it is stored in:
//   rows along k (A as stored, B read through transpose): MN rows of BK/4
//     16-byte chunks; the chunks of a row are XOR-swizzled by a key of the row, so
//     the 16 rows one 16-lane group reads at one logical chunk fall in 16
//     distinct 16-byte slots of a 256-byte (64-bank) LDS line;
//   rows along m or n (A read through transpose, B as stored): BK rows of MN/4
//     chunks; with whole 256-byte lines (MN a multiple of 64), chunk p of row k
//     holds logical chunk p ^ (8 ((k >> 3) & 1)), so rows k and k + 8, which the
//     two halves of a wave read together, use different banks.  bf16: the four rows
//     that one transposed read touches (lds_read_tr16) fall in four different
//     quarters of a 256-byte line.
// The swizzles are applied on the global side, by choosing what each lane
// fetches.  VEC copies move 16 bytes per lane and need 16-byte aligned rows of
// whole chunks; otherwise each lane copies one value (4 bytes, any alignment)
// to the same place: four times the copies and the same MFMAs and LDS reads.
// FP32 slabs can also pass through registers (STAGED): unaligned 16-byte loads and
// LDS writes to the same place, faster while K is a few slabs.
// Register staging through guarded value-by-value loads, which such storage took
// before, ran 1000 x 1531 x 777 in 58 us and 3001^3 in 1188 us, where an aligned
// neighbour took 45 and 839.
// The FP32 MFMA's k pair is (k, k + 8) at step t = 0..7 of 16 values of k (lane
// half kl supplies k = 8 kl + t): the sum over a slab is the same, and a lane
// of a rows-along-k operand then reads its values of four steps with one
// 16-byte LDS read.
// Ragged M and N: rows (chunks, values) past the edge are fetched from the last
// valid one and only feed outputs that are not stored.  Ragged K: in the last
// slab, what lies beyond K is copied from a page of zeros, for both operands.
// ===========================================================================
__device__ __align__(16) static float g_zero_chunk[4];  // never written: zeros

// Element types of the ring: what a 16-byte chunk holds, the k of one step (one
// fragment per 32 rows or columns) and its matrix instructions.
struct F32Elem {
  typedef float Value;
  typedef f32x4 Frag;  // k = 8 kl + 4 (step % 2) + s of 16 values of k, s = 0..3
  static constexpr int PER_CHUNK = 4, KSTEP = 8, SUBSTEPS = 4;
  __device__ static f32x16 mfma(const Frag& a, const Frag& b, const f32x16& c, int s) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], b[s], c, 0, 0, 0);
  }
};
struct Bf16Elem {
  typedef uint16_t Value;
  typedef bf16x8 Frag;  // k = 16 step + 8 kl + 0..7
  static constexpr int PER_CHUNK = 8, KSTEP = 16, SUBSTEPS = 1;
  __device__ static f32x16 mfma(const Frag& a, const Frag& b, const f32x16& c, int) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};

template <typename E, int MN, bool ALONG_K, int BK, bool VEC>
struct AsyncSlab {
  typedef typename E::Value Value;
  typedef typename E::Frag Frag;
  static constexpr bool F32 = sizeof(Value) == 4;
  static constexpr int PC = E::PER_CHUNK;
  static constexpr int CHUNKS = MN * BK / PC;                 // 16-byte chunks of a slab
  static constexpr int COPIES = CHUNKS * (VEC ? 1 : 4) / 64;  // wave copies of a slab
  static constexpr int COPY_BYTES = VEC ? 1024 : 256;
  static constexpr int CPR = BK / PC;  // chunks per row along k
  static constexpr int CPM = MN / PC;  // chunks per row along m or n
  static_assert((CPR == 4 || CPR == 8 || CPR == 16 || CPR == 32) && MN % 32 == 0, "slab shape");
  static_assert(VEC || F32, "value-by-value copies move 4 bytes");
  __device__ static int key(int r) {
    return CPR == 4 ? (r >> 2) & 3 : CPR == 8 ? (r >> 1) & 7 : r & 15;
  }
  __device__ static int key_mn(int k) {
    if (F32) return MN % 64 == 0 ? 8 * ((k >> 3) & 1) : 0;
    return CPM % 16 == 0 ? 4 * (k & 3) : CPM == 8 ? 4 * ((k >> 1) & 1) : 0;
  }
  // index of this lane's source in wave copy i of a slab, from the slab's first
  // value of the tile (row or column mn0), and the (first) k it holds
  __device__ static int64_t index(int64_t ld, int mn0, int mn_total, int i, int lane, int& k) {
    const int d = i * 64 + lane, ch = VEC ? d : d >> 2, e = VEC ? 0 : d & 3;
    if (ALONG_K) {
      const int r = ch / CPR;
      k = PC * ((ch % CPR) ^ key(r)) + e;
      return min(r, mn_total - 1 - mn0) * ld + k;
    }
    k = ch / CPM;
    const int col = PC * ((ch % CPM) ^ key_mn(k)) + e;
    return k * ld + min(col, mn_total - mn0 - (VEC ? PC : 1));
  }
  // Staged through registers: the chunk of lane `lane` in wave copy i (its row or
  // column in the tile and its first k), and where it is loaded from, any 4-byte
  // alignment.  base_mn is the row or column that the slab's pointer stands at.  A
  // chunk that would pass the end of a row along m or n is loaded `shift` values
  // further left.
  __device__ static void place(int i, int lane, int& mn, int& k) {
    const int ch = i * 64 + lane;
    if (ALONG_K) {
      mn = ch / CPR;
      k = PC * ((ch % CPR) ^ key(mn));
    } else {
      k = ch / CPM;
      mn = PC * ((ch % CPM) ^ key_mn(k));
    }
  }
  __device__ static int base_mn(int mn0, int mn_total) {
    return ALONG_K ? mn0 : min(mn0, max(mn_total - PC, 0));
  }
  __device__ static int64_t staged_index(int64_t ld, int mn0, int mn_total, int i, int lane, int& shift) {
    int mn, k;
    place(i, lane, mn, k);
    shift = 0;
    if (ALONG_K) return min(mn, mn_total - 1 - mn0) * ld + k;
    const int col = min(mn0 + mn, mn_total - PC);
    shift = min(mn0 + mn - col, PC - 1);
    return k * ld + (col - base_mn(mn0, mn_total));
  }
  // a 16-byte load from any 4-byte boundary (gfx950 runs global memory in
  // unaligned-access mode)
  __device__ static f32x4 load_any(const void* from) {
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    return f32x4(*reinterpret_cast<const f32x4u*>(from));
  }
  // a chunk of the last slab, zeros from k = kend on (and of any slab, by 64-bit
  // address).  A chunk along k that would pass kend is loaded further left, from the
  // slab before where this one is shorter than a chunk, and shifted.
  __device__ static f32x4 staged_tail(const float* base, int64_t ld, int mn0, int mn_total, int kend,
                                      int i, int lane) {
    int mn, k;
    place(i, lane, mn, k);
    if (ALONG_K) {
      const int from = min(k, kend - 4), s = k - from;
      f32x4 v = load_any(base + (min(mn, mn_total - 1 - mn0) * ld + from));
      if (s & 1) v = f32x4{v.y, v.z, v.w, 0.f};
      if (s & 2) v = f32x4{v.z, v.w, 0.f, 0.f};
      return s >= 4 ? f32x4{0.f, 0.f, 0.f, 0.f} : v;
    }
    const int col = min(mn0 + mn, mn_total - PC) - base_mn(mn0, mn_total);
    const f32x4 v = load_any(base + (min(k, kend - 1) * ld + col));
    return k >= kend ? f32x4{0.f, 0.f, 0.f, 0.f} : v;
  }
  // the same chunk value by value
  __device__ static f32x4 staged_values(const float* base, int64_t ld, int mn0, int mn_total, int kend,
                                        int i, int lane) {
    int mn, k;
    place(i, lane, mn, k);
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int ke = ALONG_K ? k + e : k;
      const int64_t at = ALONG_K ? min(mn, mn_total - 1 - mn0) * ld + ke
                                 : k * ld + (min(mn0 + mn + e, mn_total - 1) - base_mn(mn0, mn_total));
      v[e] = ke < kend ? base[at] : 0.f;
    }
    return v;
  }
  __device__ static void copy(const Value* base, uint32_t off, uint32_t to) {
    if (VEC)
      async::copy16_at(base, off, to);
    else
      async::copy4_at(base, off, to);
  }
  // by 64-bit address, zeros when !valid
  __device__ static void copy_any(const Value* from, bool valid, uint32_t to) {
    const void* src = valid ? (const void*)from : (const void*)g_zero_chunk;
    if (VEC)
      async::copy16_from(src, to);
    else
      async::copy4_from(src, to);
  }
  // fragment of step `st` of the slab for rows/columns r0 .. r0 + 31
  __device__ static Frag frag(const f32x4* slab, int r0, int lane, int st) {
    const int kl = lane >> 5, r = r0 + (lane & 31);
    if constexpr (F32) {
      const int u = st >> 1, h = st & 1;
      if (ALONG_K) return slab[r * CPR + ((4 * u + 2 * kl + h) ^ key(r))];
      const float* f = reinterpret_cast<const float*>(slab);
      f32x4 v;
#pragma unroll
      for (int s = 0; s < 4; s++) {
        const int k = 16 * u + 8 * kl + 4 * h + s;
        v[s] = f[k * MN + 4 * ((r >> 2) ^ key_mn(k)) + (r & 3)];
      }
      return v;
    } else {
      if (ALONG_K) return __builtin_bit_cast(bf16x8, slab[r * CPR + ((2 * st + kl) ^ key(r))]);
      // two transposed reads of four rows of k each (see lds_read_tr16)
      const int i16 = lane & 15, col = r0 + 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
      const char* p = reinterpret_cast<const char*>(slab);
      s16x4_t part[2];
#pragma unroll
      for (int q = 0; q < 2; q++) {
        const int k = 16 * st + 8 * kl + 4 * q + (i16 >> 2);
        part[q] = lds_read_tr16(p + k * MN * 2 + (((col >> 3) ^ key_mn(k)) * 16) + (col & 4) * 2);
      }
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7));
    }
  }
};

// A tile: BM x BN outputs in GM x GN waves, slabs of BK values of k in a ring of
// STAGES, KG groups of waves that share every slab's k.
template <typename E, int BM_, int BN_, int BK_, int STAGES_, int GM_, int GN_, int KG_>
struct RingCfg {
  typedef E Elem;
  static constexpr int BM = BM_, BN = BN_, BK = BK_, STAGES = STAGES_, GM = GM_, GN = GN_, KG = KG_;
  static constexpr int WAVES = GM * GN * KG, THREADS = 64 * WAVES;
  static constexpr int TM = BM / GM / 32, TN = BN / GN / 32;  // 32 x 32 blocks of a wave
  static_assert(TM * GM * 32 == BM && TN * GN * 32 == BN, "whole blocks per wave");
  static constexpr int SL = (BM + BN) * BK / E::PER_CHUNK;  // chunks per stage: A slab, then B slab
  static constexpr int LDS_CHUNKS = STAGES * SL;
};
template <int... Shape>
using F32Cfg = RingCfg<F32Elem, Shape...>;
template <int... Shape>
using Bf16Cfg = RingCfg<Bf16Elem, Shape...>;

// Below this leading dimension a copy's byte offset in a slab (up to 255 rows) fits
// 32 bits, and copies take a uniform base and that offset; longer rows are
// addressed with 64 bits, lane by lane.
constexpr int64_t kF32OffsetLd = (int64_t)1 << 22;

// The operands' storage allows 16-byte copies: 16-byte aligned rows that are
// whole chunks.
template <typename V>
__host__ __device__ inline bool whole_chunks(const V* A, int64_t lda, const V* B, int64_t ldb, int M,
                                             int N, int K, bool ta, bool tb) {
  constexpr int q = 16 / sizeof(V);
  return ((uintptr_t)A & 15) == 0 && ((uintptr_t)B & 15) == 0 && lda % q == 0 && ldb % q == 0 &&
         (ta ? M : K) % q == 0 && (tb ? K : N) % q == 0;
}

// C[m0:m0+BM, n0:n0+BN] = A B with the whole workgroup of T::THREADS: KG groups
// of GM x GN waves, each group summing its share of every slab's k (the groups'
// tiles are added at the end, group 0 first).  lds holds T::LDS_CHUNKS 16-byte
// chunks.  No copy is in flight into lds when it returns.
// KBLOCKED: both operands prepared K-blocked (K block b of row r holds BK values
// at (b * rows + r) * BK, zero padded to whole tiles): lda and ldb are then the
// operands' row counts.
// PARTS > 1: the operands are prepared as that many planes (plane_a and plane_b values
// apart, K whole slabs) whose sum they are, and C is the sum of the products of parts
// i, j with i + j < PARTS, each over all k, small products first.
// STAGED (FP32, VEC's layout): rows of any alignment and length.  Slabs pass through
// registers instead, a 16-byte load and an LDS write per chunk: what is loaded
// during one slab is written during the next, a ring's length before it is read.
template <typename T, bool TA, bool TB, bool VEC, bool KBLOCKED = false, int PARTS = 1,
          bool STAGED = false, typename V = typename T::Elem::Value>
__device__ __forceinline__ void gemm_ring_tile(float* __restrict__ C, int64_t ldc,
                                               const V* __restrict__ A, int64_t lda,
                                               const V* __restrict__ B, int64_t ldb, int M, int N,
                                               int K, int m0, int n0, f32x4* lds_base,
                                               int64_t plane_a = 0, int64_t plane_b = 0) {
  typedef typename T::Elem E;
  constexpr int BM = T::BM, BN = T::BN, BK = T::BK, STAGES = T::STAGES, KG = T::KG;
  constexpr int TM = T::TM, TN = T::TN, SL = T::SL, NW = T::WAVES;
  using SA = AsyncSlab<E, BM, !TA, BK, VEC>;
  using SB = AsyncSlab<E, BN, TB, BK, VEC>;
  // copies of a slab, A's then B's; copy j of wave w is number j NW + w, or the
  // last one again where the waves do not share them evenly
  constexpr int COPIES = SA::COPIES + SB::COPIES, NCP = (COPIES + NW - 1) / NW;
  static_assert(BK % (2 * E::KSTEP * KG) == 0, "the groups share the k evenly, in even steps");
  static_assert(KG == 1 || (KG - 1) * BM * BN / 4 <= T::LDS_CHUNKS, "the groups' tiles fit the ring");
  static_assert(STAGES >= 2 && (STAGES - 1) * NCP < 64, "ring and its vmcnt");
  auto lds = reinterpret_cast<f32x4(*)[SL]>(lds_base);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave / (T::GM * T::GN), wing = wave % (T::GM * T::GN);
  const int wm0 = wing / T::GN * (32 * TM), wn0 = wing % T::GN * (32 * TN);

  // wave-uniform for the compiler too (in a batch they come from memory)
  lda = async::uniform(lda);
  ldb = async::uniform(ldb);
  K = __builtin_amdgcn_readfirstlane(K);
  static_assert(!KBLOCKED || (!TA && TB && VEC), "prepared operands are rows along k");
  const int64_t step_a = TA || KBLOCKED ? (int64_t)BK * lda : BK;
  const int64_t step_b = TB && !KBLOCKED ? BK : (int64_t)BK * ldb;
  if (KBLOCKED) lda = ldb = BK;
  auto number = [&](int j) { return min(j * NW + wave, COPIES - 1); };
  auto is_a = [&](int j) {  // known at compile time where the waves share A's copies evenly
    return (j + 1) * NW <= SA::COPIES || (j * NW < SA::COPIES && number(j) < SA::COPIES);
  };
  auto index = [&](int j, int ln, int& k) {
    return is_a(j) ? SA::index(lda, m0, M, number(j), ln, k)
                   : SB::index(ldb, n0, N, number(j) - SA::COPIES, ln, k);
  };
  static_assert(!STAGED || (E::PER_CHUNK == 4 && VEC && !KBLOCKED && PARTS == 1 && NCP <= 16),
                "staged slabs are FP32 operands as stored");
  uint32_t off[NCP], shifts = 0;  // (STAGED) two bits a chunk
#pragma unroll
  for (int j = 0; j < NCP; j++) {
    int k;
    if constexpr (STAGED) {
      const int64_t at = is_a(j) ? SA::staged_index(lda, m0, M, number(j), lane, k)
                                 : SB::staged_index(ldb, n0, N, number(j) - SA::COPIES, lane, k);
      off[j] = 4 * (uint32_t)at;
      shifts |= (uint32_t)k << 2 * j;
    } else {
      off[j] = (uint32_t)sizeof(V) * (uint32_t)index(j, lane, k);
    }
  }
  constexpr int PRODUCTS = PARTS * (PARTS + 1) / 2;
  static_assert(PARTS == 1 || (!TA && TB && VEC && !KBLOCKED && PARTS <= 3), "prepared planes");
  const int nk1 = (K + BK - 1) / BK, krem = K - (nk1 - 1) * BK, nk = PRODUCTS * nk1;
  // (STAGED) an operand has rows shorter than a chunk
  const bool tiny = STAGED && ((TA ? M : K) < 4 || (TB ? K : N) < 4);
  const bool wide = lda >= kF32OffsetLd || ldb >= kF32OffsetLd || tiny;
  // the next slab to copy (its first value in the tile's first row or column);
  // past the last slab the last one is copied again, into a stage nothing reads
  const V* pa = async::uniform(A + (!TA ? (int64_t)m0 * lda : STAGED ? SA::base_mn(m0, M) : m0));
  const V* pb = async::uniform(B + (TB ? (int64_t)n0 * ldb : STAGED ? SB::base_mn(n0, N) : n0));
  constexpr uint32_t STAGE_BYTES = SL * 16;
  const uint32_t lds0 = async::lds_address(lds_base);
  // parts of product q (as in the packed kernels), two bits each
  constexpr uint32_t PART_A = 2 << 10 | 1 << 8 | 0 << 6 | 1 << 4 | 0 << 2 | 0;
  constexpr uint32_t PART_B = 0 << 10 | 1 << 8 | 2 << 6 | 0 << 4 | 1 << 2 | 0;
  const V *pa0 = pa, *pb0 = pb;
  int product = PRODUCTS - 1, left = nk1;  // (PARTS > 1) the slab's product, its slabs to come
  if (PARTS > 1) {
    pa += (PART_A >> 2 * product & 3) * plane_a;
    pb += (PART_B >> 2 * product & 3) * plane_b;
  }
  int next = 0;      // that slab
  uint32_t put = 0;  // and the byte offset of its ring stage
  // copy j of that slab.  careful: it may be the last slab of a ragged K, or rows
  // may be too long for 32-bit offsets
  auto copy = [&](int j, auto careful) {
    const uint32_t to = lds0 + put + (COPIES % NW == 0 ? j * NW + wave : number(j)) * SA::COPY_BYTES;
    if (decltype(careful)::value && (wide || (next >= nk - 1 && krem < BK))) {
      const int kend = next >= nk - 1 ? krem : BK;
      int ln = lane, k;  // opaque: what this computes stays out of the loop's registers
      asm volatile("" : "+v"(ln));
      const int64_t at = index(j, ln, k);
      SA::copy_any((is_a(j) ? pa : pb) + at, k < kend, to);
    } else if (is_a(j)) {  // wave-uniform
      SA::copy(pa, off[j], to);
    } else {
      SB::copy(pb, off[j], to);
    }
  };
  // (STAGED) chunk j of the slab in flight, its load from slab `next` and its write
  // to the stage at `put`
  f32x4 held[STAGED ? NCP : 1];
  const bool shifted = STAGED && ((TA && m0 + BM > M) || (!TB && n0 + BN > N));
  auto load = [&](int j, auto careful) -> f32x4 {
    if (decltype(careful)::value && (wide || (next >= nk - 1 && krem < BK))) {
      const int kend = next >= nk - 1 ? krem : BK;
      const float *fa = (const float*)pa, *fb = (const float*)pb;
      int ln = lane;
      asm volatile("" : "+v"(ln));
      if (tiny)
        return is_a(j) ? SA::staged_values(fa, lda, m0, M, kend, number(j), ln)
                       : SB::staged_values(fb, ldb, n0, N, kend, number(j) - SA::COPIES, ln);
      return is_a(j) ? SA::staged_tail(fa, lda, m0, M, kend, number(j), ln)
                     : SB::staged_tail(fb, ldb, n0, N, kend, number(j) - SA::COPIES, ln);
    }
    return SA::load_any((is_a(j) ? (const char*)pa : (const char*)pb) + off[j]);
  };
  auto store = [&](int j, f32x4 v, uint32_t at) {
    if (shifted && !tiny) {  // a shifted chunk's values move to their columns
      const uint32_t sh = shifts >> 2 * j;
      if (sh & 1) v = f32x4{v.y, v.z, v.w, v.w};
      if (sh & 2) v = f32x4{v.z, v.w, v.w, v.w};
    }
    char* to = reinterpret_cast<char*>(lds_base) + at;
    reinterpret_cast<f32x4*>(to)[number(j) * 64 + lane] = v;
  };
  auto advance = [&] {
    if (PARTS > 1 && --left == 0 && product > 0) {
      product--;
      left = nk1;
      pa = pa0 + (PART_A >> 2 * product & 3) * plane_a;
      pb = pb0 + (PART_B >> 2 * product & 3) * plane_b;
    } else {
      pa += next < nk - 1 ? step_a : 0;
      pb += next < nk - 1 ? step_b : 0;
    }
    next++;
    put = put == (STAGES - 1) * STAGE_BYTES ? 0 : put + STAGE_BYTES;
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

  const int kl = lane >> 5, il = lane & 31;
  // A group's share of a slab is NS steps.  A step's fragments are read
  // while the step before runs its MFMAs, across slabs too: the barrier that
  // publishes slab kt + 1 stands in the last step of slab kt, whose
  // fragments are in registers by then, so it also frees the stage of slab kt for
  // the copies of slab kt + STAGES, which the next slab's steps issue.  (With
  // the barrier at the start of a slab every wave waited out an LDS latency
  // there: FP32 64 x 64 tiles took 1700 cycles for the 1024 of a slab's MFMAs.)
  // Reads and copies are placed one by one between the MFMAs: a wave issues in
  // order, and as a block in front of a step's MFMAs they left the matrix cores
  // idle for about as long as the MFMAs run.
  constexpr int NS = BK / E::KSTEP / KG;  // even: the fragment sets alternate by step
  typename E::Frag a[2][TM], b[2][TN];
  int buf = 0;
  // fragment r of step st of the slab in stage `at`, in the order the MFMAs need
  // them: A's first, B's, the rest of A's
  auto read = [&](int at, int st, int r) {
    const f32x4* slab = &lds[at][0];
    if (r == 0 || r > TN) {
      const int i = r == 0 ? 0 : r - TN;
      a[st & 1][i] = SA::frag(slab, wm0 + 32 * i, lane, group * NS + st);
    } else {
      b[st & 1][r - 1] = SB::frag(slab + SA::CHUNKS, wn0 + 32 * (r - 1), lane, group * NS + st);
    }
  };
  constexpr int NR = TM + TN;
  if constexpr (STAGED) {
    if (nk > 0) {
      f32x4 first[STAGES - 1][NCP];
#pragma unroll
      for (int st = 0; st < STAGES - 1; st++) {
#pragma unroll
        for (int j = 0; j < NCP; j++) first[st][j] = load(j, std::true_type{});
        advance();
      }
#pragma unroll
      for (int st = 0; st < STAGES - 1; st++)
#pragma unroll
        for (int j = 0; j < NCP; j++) store(j, first[st][j], st * STAGE_BYTES);
#pragma unroll
      for (int j = 0; j < NCP; j++) held[j] = load(j, std::true_type{});
      advance();
      put = (STAGES - 1) * STAGE_BYTES;
      async::wait_lgkmcnt0();
      async::barrier();
#pragma unroll
      for (int r = 0; r < NR; r++) read(0, 0, r);
    }
  } else if (nk > 0) {
#pragma unroll
    for (int st = 0; st < STAGES - 1; st++) {
#pragma unroll
      for (int j = 0; j < NCP; j++) copy(j, std::true_type{});
      advance();
    }
    async::wait_vmcnt<(STAGES - 2) * NCP>();  // slab 0 has landed
    async::barrier();
#pragma unroll
    for (int r = 0; r < NR; r++) read(0, 0, r);
  }
  auto slab = [&](auto careful) {
    const int after = buf == STAGES - 1 ? 0 : buf + 1;
    auto steps = [&](auto self, auto st_tag) {
      constexpr int st = decltype(st_tag)::value;
      if constexpr (st < NS) {
        constexpr bool last = st == NS - 1;
        constexpr int c0 = last ? 0 : NCP * st / (NS - 1), c1 = last ? 0 : NCP * (st + 1) / (NS - 1);
        constexpr int NM = E::SUBSTEPS * TM * TN, OPS = NR + c1 - c0;  // MFMAs, other operations
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < NM; m++) {
          const int s = m / (TM * TN), i = m / TN % TM, j = m % TN;
          acc[i][j] = E::mfma(a[st & 1][i], b[st & 1][j], acc[i][j], s);
          __builtin_amdgcn_sched_barrier(0);
          if (last && m == 0) {
            if (!STAGED) async::wait_vmcnt<(STAGES - 2) * NCP>();  // copies of slab kt + 1 landed
            async::wait_lgkmcnt0();  // and this wave has read all of slab kt (STAGED: written kt + 2)
            async::barrier();
          }
#pragma unroll
          for (int o = OPS * m / NM; o < OPS * (m + 1) / NM; o++) {
            if (o < NR)
              read(last ? after : buf, last ? 0 : st + 1, o);
            else if constexpr (STAGED) {
              store(c0 + o - NR, held[c0 + o - NR], put);
              held[c0 + o - NR] = load(c0 + o - NR, careful);
            } else
              copy(c0 + o - NR, careful);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        self(self, std::integral_constant<int, st + 1>{});
      }
    };
    steps(steps, std::integral_constant<int, 0>{});
    advance();
    buf = after;
  };
  int kt = 0;
  if (!wide)
    for (; kt < nk - STAGES - STAGED; kt++) slab(std::false_type{});
  for (; kt < nk; kt++) slab(std::true_type{});
  async::wait_vmcnt<0>();  // the copies past the last slab land before the exit

  if constexpr (KG > 1) {
    async::wait_lgkmcnt0();
    __syncthreads();  // every wave is done with the ring
    constexpr int TILE = TM * TN * 16 * 64;  // values of a wave's tile
    constexpr int GROUP = T::GM * T::GN * TILE;
    float* part = reinterpret_cast<float*>(lds_base) + wing * TILE + lane;
    if (group > 0) {
#pragma unroll
      for (int e = 0; e < TM * TN * 16; e++)
        part[(group - 1) * GROUP + e * 64] = acc[e / 16 / TN][e / 16 % TN][e % 16];
    }
    __syncthreads();
    if (group > 0) return;
#pragma unroll
    for (int g = 1; g < KG; g++)
#pragma unroll
      for (int e = 0; e < TM * TN * 16; e++)
        acc[e / 16 / TN][e / 16 % TN][e % 16] += part[(g - 1) * GROUP + e * 64];
  }

  // join . join: D layout of a 32x32 block, lane l holds column l % 32 and rows
  // 8 (r / 4) + 4 (l / 32) + r % 4; stores guarded on edge tiles only
  const bool full = m0 + BM <= M && n0 + BN <= N;
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const int col = n0 + wn0 + j * 32 + il;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int row = m0 + wm0 + i * 32 + 8 * (r >> 2) + 4 * kl + (r & 3);
        if (full || (row < M && col < N)) C[(int64_t)row * ldc + col] = acc[i][j][r];
      }
    }
}

// ===========================================================================
// Stencil tile, LDS halo schedule: out rows [y0, y0+TY) x columns [x0, x0+256)
//   pad2D (clamp/zero)     -> index remapping while the halo tile is fetched;
//   slide2D                -> one (TY + 2R) x (256 + 8) halo tile staged in LDS
//                             (toMem(Local), paper Sec. V-B/C) with coalesced
//                             16-byte loads;
//   map(map(...))          -> each lane owns 4 adjacent outputs of a row and walks
//                             down TY / 4 rows, keeping the k rows of its window
//                             in registers;
//   zip |> map(*) |> reduce -> k*k FMAs per output (fuseReduceMap, Sec. IV-B),
//                             weights in scalar registers;
//   join                   -> 16-byte coalesced stores.
// ===========================================================================
constexpr int kStencilTX = 256;   // columns per tile (64 lanes x 4)
constexpr int kHalo = 4;          // LDS columns left and right of the tile
constexpr int kLChunks = (kStencilTX + 2 * kHalo) / 4;  // 16-byte chunks per LDS row

template <int K, int TY>
struct StencilCfg {
  static constexpr int R = (K - 1) / 2;
  static constexpr int ROWS = TY + 2 * R;
  static constexpr int LDS_CHUNKS = ROWS * kLChunks;
  static constexpr int PER = (LDS_CHUNKS + kThreads - 1) / kThreads;  // chunks per thread
};
template <int K, int TY>
using StencilRegs = f32x4[StencilCfg<K, TY>::PER];  // one thread's share of a halo tile


// Global -> registers: the (TY + 2R) x (256 + 8) halo tile of output rows
// [y0, y0 + TY), columns [x0, x0 + 256), with pad2D applied as index remapping.
// Chunks wholly inside the image row are one 16-byte load (aligned when VEC,
// otherwise at the row's own 4-byte alignment); edge chunks go element-wise.
template <int K, bool VEC, int TY>
__device__ __forceinline__ void stencil_fetch(StencilRegs<K, TY>& st,
                                              const float* __restrict__ in, int64_t ld_in,
                                              int H, int W, int zero_pad, int y0, int x0) {
  using Cfg = StencilCfg<K, TY>;
  const int tid = threadIdx.x;
#pragma unroll
  for (int p = 0; p < Cfg::PER; p++) {
    const int c = tid + p * kThreads;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (c < Cfg::LDS_CHUNKS) {
      const int lr = c / kLChunks, cc = c - lr * kLChunks;
      int gy = y0 - Cfg::R + lr;
      const int gx = x0 - kHalo + cc * 4;
      bool row_ok = true;
      if (gy < 0 || gy >= H) {
        if (zero_pad) row_ok = false;
        gy = clampi(gy, 0, H - 1);
      }
      if (row_ok) {
        const float* rp = in + (int64_t)gy * ld_in;
        if (gx >= 0 && gx + 3 < W) {
          if (VEC)
            v = *reinterpret_cast<const f32x4*>(rp + gx);
          else
            v = *reinterpret_cast<const f32x4u*>(rp + gx);
        } else {
          float e[4];
#pragma unroll
          for (int q = 0; q < 4; q++) {
            const int xx = gx + q;
            if (xx < 0 || xx >= W)
              e[q] = zero_pad ? 0.f : rp[clampi(xx, 0, W - 1)];
            else
              e[q] = rp[xx];
          }
          v = f32x4{e[0], e[1], e[2], e[3]};
        }
      }
    }
    st[p] = v;
  }
}

// Registers -> LDS (row-major (TY + 2R) x 66 chunks of 16 bytes).
template <int K, int TY>
__device__ __forceinline__ void stencil_stash(const StencilRegs<K, TY>& st,
                                              f32x4* lds) {
  using Cfg = StencilCfg<K, TY>;
#pragma unroll
  for (int p = 0; p < Cfg::PER; p++) {
    const int c = threadIdx.x + p * kThreads;
    if (c < Cfg::LDS_CHUNKS) lds[c] = st[p];
  }
}

// Rows of any width >= 4 and any alignment, without branches between the
// loads: each chunk is one 16-byte load from the nearest position that lies
// wholly inside its (clamped) row, and what pad2D makes of it is decided when
// the chunk is written to LDS (stencil_stash_any), so all loads of an edge tile
// are in flight together.  Element-wise loads under per-chunk branches instead
// waited out one memory latency per chunk: the 7 x 7 stencil of a 1531 x 2047
// image, a third of whose tiles touch an edge, ran 11.6 us with them.
template <int K, int TY>
__device__ __forceinline__ void stencil_fetch_any(StencilRegs<K, TY>& st,
                                                  const float* __restrict__ in, int64_t ld_in,
                                                  int H, int W, int y0, int x0) {
  using Cfg = StencilCfg<K, TY>;
#pragma unroll
  for (int p = 0; p < Cfg::PER; p++) {
    const int c = min((int)threadIdx.x + p * kThreads, Cfg::LDS_CHUNKS - 1);
    const int lr = c / kLChunks, cc = c - lr * kLChunks;
    const int gy = clampi(y0 - Cfg::R + lr, 0, H - 1), gx = clampi(x0 - kHalo + cc * 4, 0, W - 4);
    st[p] = *reinterpret_cast<const f32x4u*>(in + (int64_t)gy * ld_in + gx);
  }
}

// Columns gx .. gx + 3 under pad2D from the chunk loaded at clamp(gx, 0, W - 4).
__device__ __forceinline__ f32x4 chunk_any(f32x4 v, int gx, int W, int zero_pad) {
  if (gx < 0 || gx > W - 4) {
    const int at = clampi(gx, 0, W - 4);
    f32x4 u;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int i = clampi(gx + q, 0, W - 1) - at;
      const float lo = i == 0 ? v.x : v.y, hi = i == 2 ? v.z : v.w;
      u[q] = zero_pad && (gx + q < 0 || gx + q >= W) ? 0.f : i < 2 ? lo : hi;
    }
    v = u;
  }
  return v;
}

template <int K, int TY>
__device__ __forceinline__ void stencil_stash_any(const StencilRegs<K, TY>& st, f32x4* lds, int H,
                                                  int W, int zero_pad, int y0, int x0) {
  using Cfg = StencilCfg<K, TY>;
#pragma unroll
  for (int p = 0; p < Cfg::PER; p++) {
    const int c = threadIdx.x + p * kThreads;
    if (c < Cfg::LDS_CHUNKS) {
      const int lr = c / kLChunks, cc = c - lr * kLChunks;
      const int gy = y0 - Cfg::R + lr, gx = x0 - kHalo + cc * 4;
      f32x4 v = chunk_any(st[p], gx, W, zero_pad);
      if (zero_pad && (gy < 0 || gy >= H)) v = f32x4{0.f, 0.f, 0.f, 0.f};
      lds[c] = v;
    }
  }
}

// The loads of a halo tile (returned: whether it lies wholly inside the image)
// and its place in LDS with pad2D applied, for any alignment and width.
template <int K, bool VEC, int TY>
__device__ __forceinline__ bool stencil_load_tile(StencilRegs<K, TY>& st,
                                                  const float* __restrict__ in, int64_t ld_in,
                                                  int H, int W, int zero_pad, int y0, int x0) {
  using Cfg = StencilCfg<K, TY>;
  if (y0 >= Cfg::R && y0 + TY + Cfg::R <= H && x0 >= kHalo && x0 + kStencilTX + kHalo <= W) {
    // interior tile: no padding, every chunk at a fixed offset from the corner
    // (16-byte aligned when VEC, otherwise at the rows' own 4-byte alignment)
    const float* corner = in + (int64_t)(y0 - Cfg::R) * ld_in + (x0 - kHalo);
#pragma unroll
    for (int p = 0; p < Cfg::PER; p++) {
      const int c = min((int)threadIdx.x + p * kThreads, Cfg::LDS_CHUNKS - 1);
      const int lr = c / kLChunks, cc = c - lr * kLChunks;
      const float* q = corner + (int64_t)lr * ld_in + 4 * cc;
      st[p] = VEC ? *reinterpret_cast<const f32x4*>(q) : f32x4(*reinterpret_cast<const f32x4u*>(q));
    }
    return true;
  }
  if (W >= 4)
    stencil_fetch_any<K, TY>(st, in, ld_in, H, W, y0, x0);
  else
    stencil_fetch<K, VEC, TY>(st, in, ld_in, H, W, zero_pad, y0, x0);
  return false;
}
template <int K, int TY>
__device__ __forceinline__ void stencil_put_tile(const StencilRegs<K, TY>& st, f32x4* lds, int H,
                                                 int W, int zero_pad, int y0, int x0,
                                                 bool inside) {
  if (inside || W < 4)
    stencil_stash<K, TY>(st, lds);
  else
    stencil_stash_any<K, TY>(st, lds, H, W, zero_pad, y0, x0);
}

// Aligned rows (VEC and W % 4 == 0, which the callers check): every 16-byte
// chunk of the halo tile is either wholly inside or wholly outside the image
// (its columns start at a multiple of 4), so the fetch can be branch-free: each chunk is loaded from a clamped,
// always valid address, and a 2-bit mode per chunk says what pad2D makes of
// it (0 as loaded, 1 zero, 2 the first element repeated, 3 the last element
// repeated); the mode is applied when the chunk is written to LDS, so the
// loads stay in flight until then.
template <int K, int TY>
__device__ __forceinline__ void stencil_fetch_aligned(StencilRegs<K, TY>& st, uint32_t& mode,
                                                      const float* __restrict__ in, int64_t ld_in,
                                                      int H, int W, int zero_pad, int y0, int x0) {
  using Cfg = StencilCfg<K, TY>;
  static_assert(2 * Cfg::PER <= 32, "mode bits");
  uint32_t m_all = 0;
#pragma unroll
  for (int p = 0; p < Cfg::PER; p++) {
    const int c = min((int)threadIdx.x + p * kThreads, Cfg::LDS_CHUNKS - 1);
    const int lr = c / kLChunks, cc = c - lr * kLChunks;
    const int gy = y0 - Cfg::R + lr, gx = x0 - kHalo + cc * 4;
    uint32_t m = 0;
    if (gx < 0) m = 2;
    if (gx >= W) m = 3;
    if (zero_pad && (m != 0 || gy < 0 || gy >= H)) m = 1;
    const int gyc = clampi(gy, 0, H - 1), gxc = clampi(gx, 0, W - 4);
    st[p] = *reinterpret_cast<const f32x4*>(in + (int64_t)gyc * ld_in + gxc);
    m_all |= m << (2 * p);
  }
  mode = m_all;
}

template <int K, int TY>
__device__ __forceinline__ void stencil_stash_aligned(const StencilRegs<K, TY>& st, uint32_t mode,
                                                      f32x4* lds) {
  using Cfg = StencilCfg<K, TY>;
#pragma unroll
  for (int p = 0; p < Cfg::PER; p++) {
    const int c = threadIdx.x + p * kThreads;
    if (c < Cfg::LDS_CHUNKS) {
      const uint32_t m = (mode >> (2 * p)) & 3u;
      f32x4 v = st[p];
      if (m == 1) v = f32x4{0.f, 0.f, 0.f, 0.f};
      if (m == 2) v = f32x4{v.x, v.x, v.x, v.x};
      if (m == 3) v = f32x4{v.w, v.w, v.w, v.w};
      lds[c] = v;
    }
  }
}

// LDS -> k*k weighted sums.  Wave v computes output rows [y0 + v*TY/4,
// y0 + (v+1)*TY/4); lane l owns columns x0 + 4l .. x0 + 4l + 3.
// The window rows stream through registers: row j feeds every output row o
// with 0 <= j - o < k, so each output takes its k*k products in the order dy
// outer, dx inner.  ROWWISE (the default for k >= 7; the batched kernels take
// it from k = 5, to fit eight workgroups per CU) keeps that streaming in
// the schedule: the next row's LDS reads are issued before this row's FMAs,
// and empty asm statements after the FMAs take the accumulators and the LDS
// row index as operands they may change, so the FMAs must be done before them
// and the reads two rows on cannot be hoisted above them; two window rows and
// the accumulators are live instead of the whole window (k = 7 on 16-row
// tiles: 43 VGPRs instead of 124).
// EDGES (clamp padding with whole 16-byte chunks): the chunk left of column 0
// (lane 0 when `left`) and every chunk right of column lim - 1 (lim is the
// image width on the right-edge tile) read as the edge element, whatever the
// LDS tile holds there.
template <int K, int TY, bool EDGES = false, bool ROWWISE = (K >= 7)>
__device__ __forceinline__ void stencil_compute(float (&res)[TY / 4][4], const float (&wt)[K][K],
                                                const f32x4* lds, bool left = false,
                                                int lim = 0, int x = 0) {
  constexpr int R = (K - 1) / 2;
  constexpr int RW = TY / 4;      // output rows per wave
  constexpr int NR = RW + 2 * R;  // window rows
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // this lane's chunk of window row 0 (an index, so the pin below leaves the
  // pointer's LDS address space known); row j is kLChunks * j chunks further
  int base = wave * RW * kLChunks + lane;
  // LDS chunk `lane` = columns x-4..x-1, lane+1 = x..x+3, lane+2 = x+4..x+7
  auto load_row = [&](int j, f32x4 (&c)[3]) {
    const f32x4* row = lds + base + j * kLChunks;
    c[1] = row[1];
    if (R > 0) {
      c[0] = row[0];
      c[2] = row[2];
      if (EDGES) {
        if (left && lane == 0) c[0] = f32x4{c[1].x, c[1].x, c[1].x, c[1].x};
        if (x + 4 >= lim) c[2] = f32x4{c[1].w, c[1].w, c[1].w, c[1].w};
      }
    } else {
      c[0] = c[2] = c[1];
    }
  };
#pragma unroll
  for (int o = 0; o < RW; o++)
#pragma unroll
    for (int q = 0; q < 4; q++) res[o][q] = 0.f;
  f32x4 cur[3], nxt[3];
  load_row(0, cur);
#pragma unroll
  for (int j = 0; j < NR; j++) {
    if (j + 1 < NR) load_row(j + 1, nxt);
    float win[12];
#pragma unroll
    for (int c = 0; c < 3; c++) {
      win[4 * c] = cur[c].x; win[4 * c + 1] = cur[c].y;
      win[4 * c + 2] = cur[c].z; win[4 * c + 3] = cur[c].w;
    }
#pragma unroll
    for (int o = 0; o < RW; o++) {
      const int dy = j - o;
      if (dy < 0 || dy >= K) continue;
#pragma unroll
      for (int q = 0; q < 4; q++)
#pragma unroll
        for (int dx = 0; dx < K; dx++)
          res[o][q] = fmaf(win[4 + q + dx - R], wt[dy][dx], res[o][q]);
    }
    if (ROWWISE) {  // volatile asm statements keep their order: accumulators, then the index
#pragma unroll
      for (int o = 0; o < RW; o++)
        asm volatile("" : "+v"(res[o][0]), "+v"(res[o][1]), "+v"(res[o][2]), "+v"(res[o][3]));
      asm volatile("" : "+v"(base));
    }
#pragma unroll
    for (int c = 0; c < 3; c++) cur[c] = nxt[c];
  }
}

// join: 16-byte row stores of the wave's outputs (guarded at the image edge;
// rows that are not 16-byte aligned use unaligned 16-byte stores).
// NT selects non-temporal stores (the output is not read again by this pass).
template <bool VEC, int TY, bool NT>
__device__ __forceinline__ void stencil_store(float* __restrict__ out, int64_t ld_out, int H,
                                              int W, const float (&res)[TY / 4][4], int y0,
                                              int x0) {
  constexpr int RW = TY / 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int x = x0 + lane * 4;
#pragma unroll
  for (int o = 0; o < RW; o++) {
    const int y = y0 + wave * RW + o;
    if (y < H) {
      float* op = out + (int64_t)y * ld_out;
      if (x + 3 < W) {
        if (VEC) {
          const f32x4 v = f32x4{res[o][0], res[o][1], res[o][2], res[o][3]};
          if (NT)
            __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(op + x));
          else
            *reinterpret_cast<f32x4*>(op + x) = v;
        } else {
          const f32x4u v = f32x4u{res[o][0], res[o][1], res[o][2], res[o][3]};
          if (NT)
            __builtin_nontemporal_store(v, reinterpret_cast<f32x4u*>(op + x));
          else
            *reinterpret_cast<f32x4u*>(op + x) = v;
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; q++)
          if (x + q < W) op[x + q] = res[o][q];
      }
    }
  }
}

template <int K, bool VEC, int TY, bool NT, bool ROWWISE = (K >= 7)>
__device__ __forceinline__ void stencil_compute_store(float* __restrict__ out, int64_t ld_out,
                                                      int H, int W, const float (&wt)[K][K],
                                                      int y0, int x0, const f32x4* lds) {
  float res[TY / 4][4];
  stencil_compute<K, TY, false, ROWWISE>(res, wt, lds);
  stencil_store<VEC, TY, NT>(out, ld_out, H, W, res, y0, x0);
}

// SCALAR: the weight pointer is read from memory (not a kernel argument), so
// the compiler cannot tell that the loads are uniform and not overwritten while
// the kernel runs; it would read them with vector loads.  They are read through
// the constant address space instead: scalar loads straight into scalar
// registers (the weights are the same for every lane and only read).
template <int K, bool SCALAR = false>
__device__ __forceinline__ void stencil_weights(float (&wt)[K][K], const float* __restrict__ w) {
  typedef const __attribute__((address_space(4))) float cfloat;
  cfloat* cw = (cfloat*)(uintptr_t)w;
#pragma unroll
  for (int dy = 0; dy < K; dy++)
#pragma unroll
    for (int dx = 0; dx < K; dx++) wt[dy][dx] = SCALAR ? cw[dy * K + dx] : w[dy * K + dx];
}

// One tile, start to finish (fetch, stage, barrier, compute, store).
// NT: non-temporal output stores (the output is not read again soon); without
// it the output stays in the caches for a consumer that reads it next.
template <int K, bool VEC, int TY, bool NT = true, bool SCALAR_W = false,
          bool ROWWISE = (K >= 7)>
__device__ __forceinline__ void stencil_lds_tile(float* __restrict__ out, int64_t ld_out,
                                                 const float* __restrict__ in, int64_t ld_in,
                                                 int H, int W, const float* __restrict__ w,
                                                 int zero_pad, int y0, int x0, f32x4* lds) {
  StencilRegs<K, TY> st;
  using Cfg = StencilCfg<K, TY>;
  float wt[K][K];
  if (SCALAR_W) stencil_weights<K, true>(wt, w);  // scalar loads, in flight during the fetch
  const bool interior =
      y0 >= Cfg::R && y0 + TY + Cfg::R <= H && x0 >= kHalo && x0 + kStencilTX + kHalo <= W;
  if (VEC && !interior && (W & 3) == 0) {
    uint32_t mode;
    stencil_fetch_aligned<K, TY>(st, mode, in, ld_in, H, W, zero_pad, y0, x0);
    stencil_stash_aligned<K, TY>(st, mode, lds);
  } else {
    stencil_load_tile<K, VEC, TY>(st, in, ld_in, H, W, zero_pad, y0, x0);
    stencil_put_tile<K, TY>(st, lds, H, W, zero_pad, y0, x0, interior);
  }
  __syncthreads();
  if (!SCALAR_W) stencil_weights<K, false>(wt, w);
  stencil_compute_store<K, VEC, TY, NT, ROWWISE>(out, ld_out, H, W, wt, y0, x0, lds);
}

}  // namespace tiles
}  // namespace rise
