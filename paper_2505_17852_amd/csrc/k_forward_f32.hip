// Kernels of the batched perturbed forward for fp32 weights: fp32 products as
// sums of bf16 matrix products.
//
// The fp32 matrix instructions reach 157 TFLOP/s, the bf16 ones sixteen times
// that. An fp32 value is the exact sum of three bf16 values (8 significant
// bits each, the remainder of every rounding to nearest representable), so a
// product of two fp32 operands a = a0 + a1 + a2, b = b0 + b1 + b2 is
//     a0 b0 + (a0 b1 + a1 b0) + (a0 b2 + a1 b1 + a2 b0) + the rest:
// six bf16 products, each exact in fp32, accumulated in fp32 smallest first.
// The three terms left out are 2^-27.5 of a b in the root mean square and at
// most 2^-24.2 of it (one rounding of an fp32 product: 2^-25.2 and 2^-24), and a
// sum of K products takes 6 K / 32 roundings instead of the K / 4 of
// v_mfma_f32_16x16x4_f32. bf16 has fp32's exponent range, so nothing is
// scaled; at its ends, an infinite weight or activation gives NaN (its remainder
// is inf - inf), and so does a finite one from 0x7F7F8000 (3.3961775e38) on,
// whose first part rounds to infinity, while the lowest parts of values below
// 2^-109 flush.
//
// Operands.
// - Activations (the perturbed embeddings x0 and the states h) are stored
//   split and fragment-packed: 16-row tile rt, 32-k tile kt and part p of a
//   state with K values per row is 1 KB at ((rt (K / 32) + kt) 3 + p) 1024,
//   lane L = row % 16 + 16 (k % 32) / 8 holding the 8 values k % 8, which is
//   the v_mfma_f32_16x16x32_bf16 operand. A workgroup copies the tiles of its
//   rows into LDS (1 KB per wave instruction, linear, no bank conflicts), one
//   stage of 8 (row tile, k tile) pairs ahead.
// - Weights (and cached eps z of normal probes) are read in fp32, 8
//   consecutive k per lane, PD k tiles ahead into registers, from copies packed
//   so that a wave instruction covers 1 KB of consecutive memory (row_piece;
//   read in place the 64 lanes fall on 16 rows, which the address unit takes
//   one by one: 256 normal probes of a 512-unit model 137 -> 117 ms). Each wave
//   adds the probe term (w + eps z for the rows of the + pass, w - eps z for
//   the - pass, one fp32 rounding) and splits the sum in registers: a
//   workgroup's rows are RT row tiles of the + pass and the same RT tiles of
//   the - pass of one probe, and its waves own different columns, so each
//   perturbed weight is formed once per workgroup and used for 16 RT rows.
//
// Measured against v_mfma_f32_16x16x4_f32 on the same rows (64 x 128 and 128 x
// 128 tiles through LDS): the two-layer gate launch of a 256-unit model with
// 4,096 rows 83.8 -> 47.5 us, with 128 rows 36 -> 10 us; losses against 64 bits
// with weights scaled up until the products' own error shows: 2.1e-7 against
// 2.9e-7, 2.2e-7 against 3.0e-7, 2.6e-7 against 3.5e-7 (three models).
//
// What bounds them: forming a pair of perturbed fragments costs ~120 VALU
// instructions (480 cycles) per 16 columns x 32 k, against 2 RT x 6 MFMAs of
// 16 cycles; at RT = 4 (B >= 49) the two are close to balanced and overlap
// across the two waves of a SIMD, at RT = 2 the VALU bounds.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "zo_cell.hpp"
#include "zo_kernels.hpp"
#include "zo_pack.hpp"
#include "zo_profile.hpp"
#include "zo_rng.hpp"

namespace zo {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __amdgpu_buffer_rsrc_t Rsrc;

constexpr int NT = 256;     // threads per workgroup: 4 waves, each with its own columns
constexpr int kPart = 1024; // bytes of one (row tile, k tile, part) fragment
constexpr int kFrag = 3 * kPart;

// The epilogue's LDS buffer: 32 rows of up to 128 columns, padded.
constexpr int kEpRow = kVocabTile + 4;
constexpr int kStageBytes = 8 * kFrag;  // 8 (row tile, k tile) pairs
static_assert(32 * kEpRow * 4 <= kStageBytes, "the epilogue's rows fit one stage");

__device__ __forceinline__ Rsrc make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// As in the bf16 path: wait until at most VM vector memory loads of this
// thread are outstanding and its LDS accesses are done, then a barrier.
template <int VM>
__device__ __forceinline__ void wait_and_barrier() {
  static_assert(VM >= 0 && VM < 64, "vmcnt");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | 0x70);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void issue_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Two fp32 values to packed bf16, round to nearest even, low half first.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){lo, hi}, bf2));
}

// The magnitude bits m with a sign from bit 31 of x (set: plus), in one
// instruction: (~x & 0x80000000) ^ m.
__device__ __forceinline__ uint32_t sign_of(uint32_t x, uint32_t m) {
  uint32_t d;
  asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0xa6" : "=v"(d) : "v"(x), "s"(0x80000000u), "v"(m));
  return d;
}

// (a, b) = sum of the three packed bf16 pairs p[0] + p[1] + p[2] (exact: 24
// bits in three parts of 8; the lowest parts of values below 2^-109 flush).
__device__ __forceinline__ void split3(float a, float b, uint32_t (&p)[3]) {
  p[0] = pack_bf16x2(a, b);
  const float a1 = a - __uint_as_float(p[0] << 16), b1 = b - __uint_as_float(p[0] & 0xFFFF0000u);
  p[1] = pack_bf16x2(a1, b1);
  p[2] = pack_bf16x2(a1 - __uint_as_float(p[1] << 16), b1 - __uint_as_float(p[1] & 0xFFFF0000u));
}

// ---------------------------------------------------------------------------
// x0[tt][r][e] = EMB[tok][e] + s eps z_n[emb + tok E + e] for the input token
// of row r at time t0 + tt, tt < Tc, split and packed; zeros for padding
// rows, NaN for a token outside [0, V) (never read). One thread per 8
// elements; one launch per time chunk.
template <int kind>
__global__ __launch_bounds__(256) void embed_f32_kernel(const float* theta, uint64_t emb_off, int E, int V,
                                                        const int32_t* tokens, int C, int t0, int Tc, int B,
                                                        RowMap rm, int64_t M, Key key, uint32_t i0,
                                                        float eps, char* x0) {
  const int E8 = E >> 3;
  const int64_t total = (int64_t)Tc * M * E8;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    // consecutive threads fill consecutive lanes of a fragment: 16 rows, then k
    const int64_t rt = idx / (16 * E8);  // row tile of the chunk: tt M / 16 + r / 16
    const int rem = (int)(idx - rt * 16 * E8);
    const int64_t rr = rt * 16 + (rem & 15);
    const int e = (rem >> 4) * 8;
    const int tt = (int)(rr / M);
    const int64_t r = rr - (int64_t)tt * M;
    const PassOf ps = pass_of(rm, r);
    const int pair = ps.probe, b = ps.b;
    float out[8] = {};
    const int tok = b < B ? tokens[(int64_t)b * (C + 1) + t0 + tt] : 0;
    if (b < B && (uint32_t)tok >= (uint32_t)V) {
#pragma unroll
      for (int q = 0; q < 8; ++q) out[q] = __builtin_nanf("");
    } else if (b < B) {
      const uint64_t j = emb_off + (uint64_t)tok * E + e;
      float w[8], z[8];
      *(f4*)w = *(const f4*)(theta + j);
      *(f4*)(w + 4) = *(const f4*)(theta + j + 4);
      if constexpr (kind == ZO_RADEMACHER) {
        const uint32_t word = rademacher_word(key, i0 + pair, j >> 5) >> (uint32_t)(j & 31u);
#pragma unroll
        for (int q = 0; q < 8; ++q) z[q] = ((word >> q) & 1u) ? 1.0f : -1.0f;
      } else {
        gauss_block(key, i0 + pair, j >> 2, z);
        gauss_block(key, i0 + pair, (j >> 2) + 1, z + 4);
      }
      const float se = (float)ps.sign * eps;  // 0 for the clean pass: out = w
#pragma unroll
      for (int q = 0; q < 8; ++q) out[q] = w[q] + fmul(se, z[q]);
    }
    u4 part[3];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      uint32_t p[3];
      split3(out[2 * d], out[2 * d + 1], p);
#pragma unroll
      for (int q = 0; q < 3; ++q) part[q][d] = p[q];
    }
    char* dst = x0 + split_offset(rt, rem & 15, e, E);
#pragma unroll
    for (int q = 0; q < 3; ++q) *(u4*)(dst + q * kPart) = part[q];
  }
}

// ---------------------------------------------------------------------------
// Tile shape. NS: signs of a workgroup's rows (2: RT row tiles of each pass of
// a probe, central differences; 1: 2 RT row tiles of one pass, forward
// differences). CT: 16-column tiles per wave.
template <int kind_, int NS_, int RT_, int CT_>
struct Shape {
  static constexpr int kind = kind_, NS = NS_, RT = RT_, CT = CT_;
  static constexpr int RTT = 2 * RT;               // row tiles of the workgroup
  static constexpr int S = RT == 3 ? 1 : 4 / RT;   // k tiles per stage
  static constexpr int NB = S == 4 ? 4 : 2;        // weight buffers: k tiles g .. g + NB - 1
  static constexpr int PD = NB - 1;                // k tiles loaded ahead
  static constexpr bool kZ = kind == kGaussCached;  // cached eps z beside the weights
  static constexpr bool kBits = kind == kSignsCached;
  static constexpr int LPT = CT * (2 + (kZ ? 2 : kBits ? 1 : 0));  // register loads per k tile
  static_assert(RT >= 1 && RT <= 4 && (CT == 1 || CT == 2), "shape");
  static_assert(S * RTT * kFrag <= kStageBytes, "stage");
  static_assert((2 * S) % NB == 0, "the weight buffers repeat every two stages");
  static_assert(RT * S <= 4, "each wave copies one (row tile, k tile) of a half");
};

// The rows of a workgroup: up to RTT row tiles of 16 rows. Tiles past the end
// of a pass repeat its last one and are not stored.
struct RowTiles {
  int64_t base0, base1;  // row tile 0 of the first and second half of the workgroup's tiles
  int last0, last1;      // tiles i of a half past last.. repeat it
  int probe;
  int sign0, sign1;      // the sign of eps of each half's rows (+1, -1, 0)
};
template <int NS, int RT>
__device__ __forceinline__ RowTiles row_tiles(const RowMap& rm, int blk) {
  const int q = rm.Bp >> 4;
  RowTiles r;
  if constexpr (NS == 2) {
    const int nblk = (q + RT - 1) / RT;
    const int n = blk / nblk;
    const int j = (blk - n * nblk) * RT;
    r.base0 = (int64_t)(2 * n) * q + j;
    r.base1 = r.base0 + q;
    r.last0 = r.last1 = min(RT, q - j) - 1;
    r.probe = n;
    r.sign0 = 1;
    r.sign1 = -1;
  } else {
    const int nblk = (q + 2 * RT - 1) / (2 * RT);
    const int p = blk / nblk;
    const int j = (blk - p * nblk) * 2 * RT;
    r.base0 = (int64_t)p * q + j;
    r.base1 = r.base0 + RT;
    r.last0 = min(RT, q - j) - 1;
    r.last1 = min(RT, q - j - RT) - 1;  // may be negative: the second half repeats the last tile of the first
    r.probe = min(p, rm.N - 1);  // as pass_of: the clean pass reports the last probe with sign 0
    r.sign0 = r.sign1 = p < rm.N ? 1 : 0;
  }
  return r;
}
// Row tile of tile i < 2 RT, and whether it is the workgroup's own.
template <int RT>
__device__ __forceinline__ int64_t row_tile(const RowTiles& r, int i, bool& own) {
  if (i < RT) {
    own = i <= r.last0;
    return r.base0 + min(i, r.last0);
  }
  own = i - RT <= r.last1;
  return r.base1 + min(i - RT, r.last1);
}
// Workgroup x of a grid of row blocks x column blocks. Workgroups go to the 8
// XCDs in turn, each with its own L2: XCD i takes the i-th eighth of the tiles
// in row-major order, so the column blocks of a row block share its
// activations (written by the previous launch, 6 bytes a value, more than the
// weights they meet) in one L2 instead of fetching them into all eight.
__device__ __forceinline__ void tile_of(int x, int total, int ncol, int& row, int& col) {
  const int i = x & 7, q = total >> 3, r = total & 7;
  const int t = i * q + min(i, r) + (x >> 3);
  row = t / ncol;
  col = t - row * ncol;
}

// One K segment: packed activations, the weight matrix and its place in theta.
struct Seg {
  const char* A;   // packed activations (K values per row), row tile 0
  int64_t step;    // bytes between row tiles: K / 32 kFrag, or 0 (one tile for all rows)
  const float* W;  // [rows][K], packed (row_piece) or row-major
  uint64_t zoff;   // offset of W inside theta (probe coordinates)
  int K;
  const float* Z;  // kGaussCached: eps z of this probe and matrix, packed
};

// acc[row tile][column tile] of this wave: 16x16 fp32, lane = column lane % 16,
// rows 4 (lane / 16) + v. rows: of the weight matrices; row0: the wave's first one
// (uniform, a multiple of 16); col(ct): this lane's weight row of column tile
// ct, from row0. split: the two products W.h and (s eps z).h one after the other into
// one accumulator (twice the matrix work, for measurement).
template <typename T, bool kSplit, typename Col, typename Init>
__device__ __forceinline__ void mainloop(f4 (&acc)[T::RTT][T::CT], const Seg s0, const Seg s1, int nseg,
                                         const RowTiles& rt, int rows, int row0, Col col, bool packed, Key key,
                                         uint32_t probe, float eps,
                                         const uint32_t* bits, uint8_t* st0, uint8_t* st1, Init init) {
  constexpr int NS = T::NS, RT = T::RT, CT = T::CT, S = T::S, NB = T::NB, PD = T::PD;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = lane >> 4;
  const int kt0 = s0.K >> 5, ntiles = kt0 + (nseg > 1 ? s1.K >> 5 : 0);

  struct Buf {
    f4 w[CT][2];
    f4 z[T::kZ ? CT : 1][2];
    uint32_t word[CT];
    int g;
  };
  Buf buf[NB];
  // Addresses of the weights. Packed, a wave's column tile c is one block of R
  // rows (16; fewer at the end of the head matrix), a k tile of it 128 R
  // consecutive bytes: two halves of 64 R, this lane's piece at (kg R + row)
  // 16. In place (a workspace without the packed copy), this lane's row with
  // 128 bytes per k tile, its halves 16 bytes apart. Sign words: 32 values per
  // 4-byte word (K is a multiple of 32).
  int rel[CT];               // this lane's row of column tile c, from row0
  uint32_t lp[CT], tp[CT];   // packed: lane offset, bytes per k tile
  uint32_t lw[2][CT];
  int64_t blk[CT];           // first row of column tile c's block
  uint32_t lo[2][CT];        // in place: lane offset from the block
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    rel[c] = col(c);
    const int b0 = min(16 * c, (rows - 1 - row0) & ~15);  // column tiles past the matrix repeat its last block
    const int R = min(16, rows - row0 - b0);
    blk[c] = (int64_t)row0 + b0;
    lp[c] = (uint32_t)((kg * R + rel[c] - b0) * 16);
    tp[c] = (uint32_t)R * 128u;
    lo[0][c] = (uint32_t)((rel[c] - b0) * s0.K + 8 * kg) * 4u;
    lo[1][c] = (uint32_t)((rel[c] - b0) * s1.K + 8 * kg) * 4u;
    lw[0][c] = (uint32_t)(rel[c] * (s0.K >> 5)) * 4u;
    lw[1][c] = (uint32_t)(rel[c] * (s1.K >> 5)) * 4u;
  }
  const int64_t r0 = (int64_t)row0 * s0.K, r1 = (int64_t)row0 * s1.K;
  const char* wbase[2][CT];
  const char* zbase[2][T::kZ ? CT : 1];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    wbase[0][c] = (const char*)(s0.W + blk[c] * s0.K);
    wbase[1][c] = (const char*)(s1.W + blk[c] * s1.K);
    if constexpr (T::kZ) {
      zbase[0][c] = (const char*)(s0.Z + blk[c] * s0.K);
      zbase[1][c] = (const char*)(s1.Z + blk[c] * s1.K);
    }
  }
  const char* bbase[2] = {(const char*)(bits + ((s0.zoff + (uint64_t)r0) >> 5)),
                          (const char*)(bits + ((s1.zoff + (uint64_t)r1) >> 5))};
  // weights (and probe values or sign words) of k tile g, the last tile past the end
  auto load_b = [&](Buf& b, int g) {
    g = min(g, ntiles - 1);
    const bool second = g >= kt0;
    const uint32_t kt = (uint32_t)(second ? g - kt0 : g);
    const char* wd = (second ? bbase[1] : bbase[0]) + kt * 4u;
    b.g = g;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const char* W = (second ? wbase[1][c] : wbase[0][c]) + kt * (packed ? tp[c] : 128u);
      const uint32_t v = packed ? lp[c] : second ? lo[1][c] : lo[0][c];
      b.w[c][0] = *(const f4*)(W + v);
      b.w[c][1] = *(const f4*)(W + (packed ? tp[c] / 2 : 16u) + v);
      if constexpr (T::kZ) {
        const char* Z = (second ? zbase[1][c] : zbase[0][c]) + kt * tp[c];
        b.z[c][0] = *(const f4*)(Z + lp[c]);
        b.z[c][1] = *(const f4*)(Z + tp[c] / 2 + lp[c]);
      }
      if constexpr (T::kBits) b.word[c] = *(const uint32_t*)(wd + (second ? lw[1][c] : lw[0][c]));
    }
  };
  // The activation tiles of stage s (S k tiles of every row tile) into st:
  // wave w copies row tile w / S of each half and k tile w % S, part by part
  // (the instruction's offset moves both the source and the LDS address). A
  // half's row tiles follow one another in memory, so one resource per
  // segment and half reaches them (offsets below RT K 96).
  const int ck = wave % S;
  const char* abase[2][2];
  uint32_t co[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int last = h ? rt.last1 : rt.last0;
    const int64_t first = (h ? rt.base1 : rt.base0) + min(0, last);
    const uint32_t i = (uint32_t)min(min(wave / S, RT - 1), max(0, last));
    abase[0][h] = s0.A + first * s0.step;
    abase[1][h] = s1.A + first * s1.step;
    co[0][h] = i * (uint32_t)s0.step;
    co[1][h] = i * (uint32_t)s1.step;
  }
  const uint32_t abytes[2] = {(uint32_t)((RT - 1) * s0.step) + (uint32_t)(kt0 * kFrag),
                              (uint32_t)((RT - 1) * s1.step) + (uint32_t)((s1.K >> 5) * kFrag)};
  const int cdst = (min(wave / S, RT - 1) * S + ck) * kFrag;
  auto copy_a = [&](uint8_t* st, int s) {
    const int g = min(s * S + ck, ntiles - 1);
    const bool second = g >= kt0;
    const uint32_t kt = (uint32_t)(second ? g - kt0 : g) * kFrag;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const Rsrc r = make_rsrc(second ? abase[1][h] : abase[0][h], second ? abytes[1] : abytes[0]);
      const uint32_t off = (second ? co[1][h] : co[0][h]) + kt;
      auto* dst = (__attribute__((address_space(3))) void*)(st + h * RT * S * kFrag + cdst);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, lane * 16, off, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, lane * 16, off, kPart, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, lane * 16, off, 2 * kPart, 0);
    }
  };

  const uint32_t epsb = __float_as_uint(rt.sign0 == 0 ? 0.f : eps);  // the clean pass of forward differences adds +-0
  Words zc[CT];  // regenerated signs: the Philox block of the column's current 128 k
  // eps z of column tile c of buffer b: 8 consecutive k from 8 kg
  auto probe_values = [&](const Buf& b, int c, float (&ez)[8]) {
    if constexpr (T::kZ) {
#pragma unroll
      for (int e = 0; e < 8; ++e) ez[e] = NS == 1 && rt.sign0 == 0 ? 0.f : b.z[c][e >> 2][e & 3];
    } else if constexpr (T::kind == ZO_GAUSSIAN) {
      const bool second = b.g >= kt0;
      const uint64_t j = (second ? s1.zoff : s0.zoff) + (uint64_t)(row0 + rel[c]) * (uint64_t)(second ? s1.K : s0.K) +
                         (uint64_t)((second ? b.g - kt0 : b.g) * 32 + 8 * kg);
      float z[8];
      gauss_block(key, probe, j >> 2, z);
      gauss_block(key, probe, (j >> 2) + 1, z + 4);
#pragma unroll
      for (int e = 0; e < 8; ++e) ez[e] = fmul(__uint_as_float(epsb), z[e]);
    } else {
      // flag pair d of this lane's 8: bits 4 kg + d and 16 + 4 kg + d of the unshuffled word
      uint32_t word;
      if constexpr (T::kBits) {
        word = b.word[c];
      } else {
        const bool second = b.g >= kt0;
        const uint64_t zoff = second ? s1.zoff : s0.zoff;
        const int K = second ? s1.K : s0.K;
        const int k0 = (second ? b.g - kt0 : b.g) * 32;
        const uint64_t j = zoff + (uint64_t)(row0 + rel[c]) * (uint64_t)K + (uint64_t)k0;
        const bool aligned = (zoff % 128u) == 0 && (K % 128) == 0;
        if (!aligned || (k0 & 127) == 0) zc[c] = stream_block(key, j >> 7, probe, kTagRademacher);
        const uint32_t q = (uint32_t)(j >> 5) & 3u;
        word = sign_word_unshuffle(q == 0 ? zc[c].w[0] : q == 1 ? zc[c].w[1] : q == 2 ? zc[c].w[2] : zc[c].w[3]);
      }
      const uint32_t u = word >> (4 * kg);  // bit set: z = +1
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        ez[2 * d] = __uint_as_float(sign_of(u << (31 - d), epsb));
        ez[2 * d + 1] = __uint_as_float(sign_of(u << (15 - d), epsb));
      }
    }
  };
  auto form = [&](const float (&t)[8], b8 (&B)[3]) {
    u4 q[3];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      uint32_t p[3];
      split3(t[2 * d], t[2 * d + 1], p);
      q[0][d] = p[0];
      q[1][d] = p[1];
      q[2][d] = p[2];
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) B[p] = __builtin_bit_cast(b8, q[p]);
  };
  // rows of half h times the fragment B of column tile c: smallest products first
  constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};
  auto mma = [&](const b8 (&A)[RT][3], const b8 (&B)[3], int h, int c) {
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int i = 0; i < RT; ++i)
        acc[h * RT + i][c] =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[i][PA[q]], B[PB[q]], acc[h * RT + i][c], 0, 0, 0);
  };
  auto compute = [&](const Buf& b, const uint8_t* st, int ks) {
    auto load_a = [&](b8 (&A)[RT][3], int h) {
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int p = 0; p < 3; ++p)
          A[i][p] = __builtin_bit_cast(b8, *(const u4*)(st + (((h * RT + i) * S + ks) * 3 + p) * kPart + lane * 16));
    };
    float ez[CT][8];
#pragma unroll
    for (int c = 0; c < CT; ++c) probe_values(b, c, ez[c]);
    auto weight = [&](int c, int h, float (&t)[8]) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float w = b.w[c][e >> 2][e & 3];
        t[e] = NS == 2 && h == 1 ? fadd(w, -ez[c][e]) : fadd(w, ez[c][e]);
      }
    };
    if constexpr (kSplit) {
      static_assert(!kSplit || NS == 2, "the two-stream form is central differences only");
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        b8 A[RT][3];
        load_a(A, h);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          float t[8];
          b8 B[3];
#pragma unroll
          for (int e = 0; e < 8; ++e) t[e] = b.w[c][e >> 2][e & 3];
          form(t, B);
          mma(A, B, h, c);
#pragma unroll
          for (int e = 0; e < 8; ++e) t[e] = h == 1 ? -ez[c][e] : ez[c][e];
          form(t, B);
          mma(A, B, h, c);
        }
      }
    } else if constexpr (NS == 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        b8 A[RT][3];
        load_a(A, h);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          float t[8];
          b8 B[3];
          weight(c, h, t);
          form(t, B);
          mma(A, B, h, c);
        }
      }
    } else {
      b8 B[CT][3], A[2][RT][3];
      if constexpr (RT <= 2) {  // (more row tiles: too many registers)
        load_a(A[0], 0);
        load_a(A[1], 1);
        __builtin_amdgcn_sched_barrier(0x7);  // arithmetic may move across, LDS reads may not
      }
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        float t[8];
        weight(c, 0, t);
        form(t, B[c]);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if constexpr (RT > 2) load_a(A[h], h);
#pragma unroll
        for (int c = 0; c < CT; ++c) mma(A[h], B[c], h, c);
      }
    }
  };

  // Stage s lives in st0 / st1 by parity. Before it is read: its copies have
  // landed (every load after them may stay in flight: a fixed number, since
  // all loads are issued unconditionally) and every wave has passed the
  // barrier; while it is read the next stage's copies fly into the other.
  const int nst = (ntiles + S - 1) / S;
  copy_a(st0, 0);
  issue_fence();
#pragma unroll
  for (int g = 0; g < PD; ++g) load_b(buf[g], g);
  asm volatile("" ::: "memory");
  init();  // waits for loads older than these only
  wait_and_barrier<PD * T::LPT>();
  auto stage = [&](auto parity, int s) {
    constexpr int P = decltype(parity)::value;
    copy_a(P ? st0 : st1, s + 1);
    issue_fence();
#pragma unroll
    for (int ks = 0; ks < S; ++ks) {
      const int g = s * S + ks;
      load_b(buf[(P * S + ks + PD) % NB], g + PD);
      asm volatile("" ::: "memory");  // the loads stay here: wait_and_barrier counts them
      if (S == 1 || g < ntiles) compute(buf[(P * S + ks) % NB], P ? st1 : st0, ks);
    }
    wait_and_barrier<S * T::LPT>();
  };
  for (int s = 0; s < nst; s += 2) {
    stage(std::integral_constant<int, 0>{}, s);
    if (s + 1 < nst) stage(std::integral_constant<int, 1>{}, s + 1);
  }
  wait_and_barrier<0>();  // the copies past the last stage have landed: the stages are free
}

// acc = bias + s eps z of each column, for the rows of each sign.
template <typename T>
__device__ __forceinline__ void bias_init(f4 (&acc)[T::RTT][T::CT], const float (&bias)[T::CT], const float (&zb)[T::CT],
                                          int sign0) {
#pragma unroll
  for (int ct = 0; ct < T::CT; ++ct) {
    const float v0 = sign0 == 0 ? bias[ct] : bias[ct] + zb[ct], v1 = T::NS == 2 ? bias[ct] - zb[ct] : v0;
#pragma unroll
    for (int i = 0; i < T::RTT; ++i) acc[i][ct] = i < T::RT ? f4{v0, v0, v0, v0} : f4{v1, v1, v1, v1};
  }
}

// 32 rows (row tiles 2 c, 2 c + 1) of the accumulators into ep[32][kEpRow],
// column 16 CT wave + 16 ct + lane % 16.
template <typename T>
__device__ __forceinline__ void put_rows(const f4 (&acc)[T::RTT][T::CT], int c, float* ep) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int ct = 0; ct < T::CT; ++ct)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        ep[(16 * i + 4 * (lane >> 4) + v) * kEpRow + 16 * T::CT * wave + 16 * ct + (lane & 15)] = acc[2 * c + i][ct][v];
}

// ---------------------------------------------------------------------------
// One LSTM layer at one timestep for all rows:
//   a = (W_ih + s eps Z_ih) x + (W_hh + s eps Z_hh) h + b + s eps z_b
//   i, f, o = sigmoid, g = tanh; c <- f c + i g; h <- o tanh(c)
// Workgroup: RTT row tiles x 16 CT hidden units, wave w the units' gate w
// (i, f, g, o). One launch runs up to kLaunchLayers layers, each at its own
// timestep (blockIdx.y picks the layer): the step is a wavefront over (layer,
// timestep) in which layer l at time t and layer l + 1 at time t - 1 are
// independent.
struct GateArgs {
  GateLayerF32 layer[kLaunchLayers];
  const float* theta;
  int H;
  int hstep;  // bytes between row tiles of the layers' hprev (0: one tile for all)
  Key key;
  uint32_t i0;
  float eps;
  RowMap rm;
  uint64_t zc_stride;
  const uint32_t* bits;  // sign-probe cache: probe 0's words; probe n at + n * bits_stride
  uint64_t bits_stride;
  int ncol;              // column blocks
  bool packed;           // the layers' weights are packed copies
};

template <typename T, bool kSplit>
__global__ __launch_bounds__(NT, 2) void gate_f32_kernel(GateArgs g) {
  __shared__ __align__(16) uint8_t st0[kStageBytes];
  __shared__ __align__(16) uint8_t st1[kStageBytes];
  constexpr int RT = T::RT, RTT = T::RTT, CT = T::CT, U = 16 * CT, UPT = U / 8;
  const GateLayerF32& gl = g.layer[blockIdx.y];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int mb, nb;
  tile_of(blockIdx.x, gridDim.x, g.ncol, mb, nb);
  const int u0 = nb * U, H = g.H;
  const RowTiles rt = row_tiles<T::NS, RT>(g.rm, mb);
  // this thread's cells in the epilogue: row t / 8 of each 32 rows, UPT units
  const int er = t >> 3, eu = (t & 7) * UPT;
  float cprev[RTT / 2][UPT];
  int64_t crow[RTT / 2];
  bool cown[RTT / 2];
#pragma unroll
  for (int c = 0; c < RTT / 2; ++c) {
    crow[c] = row_tile<RT>(rt, 2 * c + (er >> 4), cown[c]) * 16 + (er & 15);
    const float* cp = gl.cst + crow[c] * H + u0 + eu;
#pragma unroll
    for (int e = 0; e < UPT; ++e) cprev[c][e] = cp[e];
  }
  f4 acc[RTT][CT];
  // the bias (with its probe term) of this lane's columns, into the
  // accumulators once the main loop's first loads are on their way
  float bias[CT], zb[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const int64_t u = u0 + 16 * ct + (lane & 15);
    bias[ct] = g.theta[gl.off_b + (int64_t)wave * H + u];
    zb[ct] = gl.zb[((int64_t)rt.probe * 4 + wave) * H + u];
  }
  auto init = [&]() { bias_init<T>(acc, bias, zb, rt.sign0); };
  const uint64_t zpos = (uint64_t)rt.probe * g.zc_stride;
  const Seg s0{gl.x, (gl.El >> 5) * kFrag, gl.w_ih, gl.off_ih, gl.El, T::kZ ? gl.zc_ih + zpos : nullptr};
  const Seg s1{gl.hprev, g.hstep, gl.w_hh, gl.off_hh, H, T::kZ ? gl.zc_hh + zpos : nullptr};
  mainloop<T, kSplit>(
      acc, s0, s1, 2, rt, 4 * H, __builtin_amdgcn_readfirstlane(wave * H + u0),
      [&](int ct) { return 16 * ct + (lane & 15); }, g.packed, g.key, g.i0 + (uint32_t)rt.probe, g.eps, T::kBits ? g.bits + (uint64_t)rt.probe * g.bits_stride : nullptr, st0, st1, init);
#pragma unroll
  for (int c = 0; c < RTT / 2; ++c) {
    float* ep = (float*)(c & 1 ? st1 : st0);
    put_rows<T>(acc, c, ep);
    __syncthreads();
    float a[4][UPT], h[UPT], cn[UPT];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < UPT; ++e) a[q][e] = ep[er * kEpRow + q * U + eu + e];
#pragma unroll
    for (int e = 0; e < UPT; ++e) {
      cn[e] = cprev[c][e];
      h[e] = lstm_cell(a[0][e], a[1][e], a[2][e], a[3][e], cn[e]);
    }
    if (cown[c]) {
      float* cp = gl.cst + crow[c] * H + u0 + eu;
#pragma unroll
      for (int e = 0; e < UPT; ++e) cp[e] = cn[e];
      char* hp = gl.hout + split_offset(crow[c] >> 4, (int)(crow[c] & 15), u0 + eu, H);
      uint32_t part[3][UPT / 2];
#pragma unroll
      for (int d = 0; d < UPT / 2; ++d) {
        uint32_t p[3];
        split3(h[2 * d], h[2 * d + 1], p);
#pragma unroll
        for (int q = 0; q < 3; ++q) part[q][d] = p[q];
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        if constexpr (UPT == 4) *(uint2*)(hp + q * kPart) = uint2{part[q][0], part[q][UPT / 2 - 1]};
        else *(uint32_t*)(hp + q * kPart) = part[q][0];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Output head over a chunk of timesteps: row tiles tt M / 16 + r / 16 of the
// chunk's top-layer states. Logits y = W_out h + b_out (+ s eps (Z_out h +
// z_bout)) for a 128-wide vocabulary tile; the tile's maximum and sum of
// exp(y - max) per row go to pmax/psum, and the logit of the target token is
// written by the tile that holds it.
struct HeadArgs {
  const char* h;  // packed states, [Tc][M / 16] row tiles
  const float* theta;
  uint64_t off_w, off_b;
  int H, V;
  const float* zbo;  // [N][V]
  Key key;
  uint32_t i0;
  float eps;
  RowMap rm;
  int64_t M;
  int64_t rows;    // Tc M
  int blocks;        // workgroups (block_id may run past them)
  int blocks_per_t;  // row blocks of one timestep
  int nvt;             // vocabulary tiles
  const float* w_out;  // W_out: packed copy, or theta's own
  bool packed;
  const int32_t* tokens;
  int C, t0, B;
  float* pmax;  // [nvt][rows]
  float* psum;
  float* ptgt;  // [rows]
  const float* zc_out;  // probe cache: W_out's values of probe 0; probe n at + n * zc_stride
  uint64_t zc_stride;
  const uint32_t* bits;
  uint64_t bits_stride;
};

template <typename T, bool kSplit>
__global__ __launch_bounds__(NT, 2) void head_f32_kernel(HeadArgs g) {
  __shared__ __align__(16) uint8_t st0[kStageBytes];
  __shared__ __align__(16) uint8_t st1[kStageBytes];
  constexpr int RT = T::RT, RTT = T::RTT, CT = T::CT;
  static_assert(64 * CT == kVocabTile, "head vocabulary tile");
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int mb, vt;
  const int id = (int)block_id();
  if (id >= g.blocks) return;
  tile_of(id, g.blocks, g.nvt, mb, vt);
  const int v0 = vt * kVocabTile, V = g.V;
  const int tt = mb / g.blocks_per_t;
  RowTiles rt = row_tiles<T::NS, RT>(g.rm, mb - tt * g.blocks_per_t);
  const int64_t tile0 = (int64_t)tt * (g.M >> 4);
  rt.base0 += tile0;
  rt.base1 += tile0;
  // this thread's cells in the epilogue: row t / 8 of each 32 rows, columns t % 8 + 8 j
  const int er = t >> 3, ec = t & 7;
  int64_t erow[RTT / 2];
  bool eown[RTT / 2];
  int tgt[RTT / 2];
#pragma unroll
  for (int c = 0; c < RTT / 2; ++c) {
    erow[c] = row_tile<RT>(rt, 2 * c + (er >> 4), eown[c]) * 16 + (er & 15);
    const int b = pass_of(g.rm, erow[c] - (int64_t)tt * g.M).b;
    tgt[c] = b < g.B ? g.tokens[(int64_t)b * (g.C + 1) + g.t0 + tt + 1] - v0 : -1;
  }
  f4 acc[RTT][CT];
  const int row0 = __builtin_amdgcn_readfirstlane(min(v0 + 16 * CT * wave, (V - 1) & ~15));
  auto col = [&](int ct) { return min(16 * ct + (lane & 15), V - 1 - row0); };
  float bias[CT], zb[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    bias[ct] = g.theta[g.off_b + (uint64_t)(row0 + col(ct))];
    zb[ct] = g.zbo[(int64_t)rt.probe * V + row0 + col(ct)];
  }
  auto init = [&]() { bias_init<T>(acc, bias, zb, rt.sign0); };
  const Seg s0{g.h, (g.H >> 5) * kFrag, g.w_out, g.off_w, g.H,
               T::kZ ? g.zc_out + (uint64_t)rt.probe * g.zc_stride : nullptr};
  mainloop<T, kSplit>(acc, s0, s0, 1, rt, V, row0, col, g.packed, g.key, g.i0 + (uint32_t)rt.probe, g.eps,
                      T::kBits ? g.bits + (uint64_t)rt.probe * g.bits_stride : nullptr, st0, st1, init);
#pragma unroll
  for (int c = 0; c < RTT / 2; ++c) {
    float* ep = (float*)(c & 1 ? st1 : st0);
    put_rows<T>(acc, c, ep);
    __syncthreads();
    float y[kVocabTile / 8];
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < kVocabTile / 8; ++j) {
      y[j] = v0 + ec + 8 * j < V ? ep[er * kEpRow + ec + 8 * j] : -INFINITY;
      mx = max_or_nan(mx, y[j]);
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) mx = max_or_nan(mx, __shfl_xor(mx, off, 64));
    float se = 0.f;
#pragma unroll
    for (int j = 0; j < kVocabTile / 8; ++j) se += v0 + ec + 8 * j < V ? __expf(y[j] - mx) : 0.f;
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) se += __shfl_xor(se, off, 64);
    if (eown[c] && ec == 0) {
      g.pmax[(int64_t)vt * g.rows + erow[c]] = mx;
      g.psum[(int64_t)vt * g.rows + erow[c]] = se;
      // a target outside [0, V) is never looked up: its position's loss is NaN
      if (tgt[c] >= 0 && tgt[c] < kVocabTile && v0 + tgt[c] < V) g.ptgt[erow[c]] = ep[er * kEpRow + tgt[c]];
    }
  }
}

// Calls go(kind, split) with the compile-time probe kind of this call.
template <typename Go>
hipError_t by_kind(const ForwardArgs& a, Go&& go) {
  using std::integral_constant;
  if (a.cfg.probe == ZO_RADEMACHER) {
    if (a.bits) return go(integral_constant<int, kSignsCached>{});
    return go(integral_constant<int, ZO_RADEMACHER>{});
  }
  if (a.zc) return go(integral_constant<int, kGaussCached>{});
  return go(integral_constant<int, ZO_GAUSSIAN>{});
}
template <typename Go>
hipError_t by_rt(int rt, Go&& go) {
  using std::integral_constant;
  switch (rt) {
    case 1: return go(integral_constant<int, 1>{});
    case 2: return go(integral_constant<int, 2>{});
    case 3: return go(integral_constant<int, 3>{});
    default: return go(integral_constant<int, 4>{});
  }
}

}  // namespace

hipError_t launch_embed_f32(const ForwardArgs& a, int t0, int Tc, void* x0, hipStream_t st) {
  const Rows& R = a.rows;
  const int E = a.cfg.embed;
  const RowMap rm = row_map(R);
  const int64_t n = (int64_t)Tc * R.M * (E / 8);
  const unsigned grid = (unsigned)std::min<int64_t>((n + 255) / 256, (int64_t)1 << 20);
  const Key key = make_key(a.seed);
  ProfScope ps(kKEmbed, st);
  if (a.cfg.probe == ZO_RADEMACHER)
    embed_f32_kernel<ZO_RADEMACHER><<<grid, 256, 0, st>>>((const float*)a.theta, a.lay.emb, E, a.cfg.vocab, a.tokens,
                                                          a.C, t0, Tc, R.B, rm, R.M, key, a.i0, a.eps, (char*)x0);
  else
    embed_f32_kernel<ZO_GAUSSIAN><<<grid, 256, 0, st>>>((const float*)a.theta, a.lay.emb, E, a.cfg.vocab, a.tokens,
                                                        a.C, t0, Tc, R.B, rm, R.M, key, a.i0, a.eps, (char*)x0);
  return hipGetLastError();
}

hipError_t launch_gates_f32(const ForwardArgs& a, const GateLayerF32* ls, int n, hipStream_t st) {
  if (n < 1 || n > kLaunchLayers) return hipErrorInvalidValue;
  const Rows& R = a.rows;
  GateArgs g{};
  for (int i = 0; i < n; ++i) g.layer[i] = ls[i];
  g.theta = (const float*)a.theta;
  g.H = a.cfg.hidden;
  // (a call with a zero tile has one position: its launches have one layer each)
  g.hstep = a.ws.T == 1 && ls[0].hprev == a.work + a.ws.hzero ? 0 : g.H / 32 * kFrag;
  g.key = make_key(a.seed);
  g.i0 = a.i0;
  g.eps = a.eps;
  g.rm = row_map(R);
  g.zc_stride = a.zmap.pg;
  g.bits = a.bits;
  g.bits_stride = bit_words(a.lay.total);
  const int ns = R.fd ? 1 : 2;
  const Pick pk = pick_shape(g.rm, R.M, ns, 4 * (int64_t)g.H, n, !a.split);
  g.ncol = g.H / (16 * pk.ct);
  g.packed = a.wpack != nullptr;
  const int64_t blocks = row_blocks(g.rm, R.M, ns, pk.rt) * g.ncol;
  if (blocks * NT > 0xFFFFFFFFll) return hipErrorInvalidValue;  // (states of over 200 GB)
  const dim3 grid((unsigned)blocks, (unsigned)n);
  ProfScope ps(kKGate, st);
  return by_kind(a, [&](auto k) {
    return by_rt(pk.rt, [&](auto r) {
      constexpr int kind = decltype(k)::value, RT = decltype(r)::value;
      if (a.split) gate_f32_kernel<Shape<kind, 2, RT, 2>, true><<<grid, NT, 0, st>>>(g);
      else if (ns == 2 && pk.ct == 2) gate_f32_kernel<Shape<kind, 2, RT, 2>, false><<<grid, NT, 0, st>>>(g);
      else if (ns == 2) gate_f32_kernel<Shape<kind, 2, RT, 1>, false><<<grid, NT, 0, st>>>(g);
      else if (pk.ct == 2) gate_f32_kernel<Shape<kind, 1, RT, 2>, false><<<grid, NT, 0, st>>>(g);
      else gate_f32_kernel<Shape<kind, 1, RT, 1>, false><<<grid, NT, 0, st>>>(g);
      return hipGetLastError();
    });
  });
}

hipError_t launch_head_f32(const ForwardArgs& a, const void* hist, int t0, int Tc, const float* zbo,
                           float* pmax, float* psum, float* ptgt, hipStream_t st) {
  const Rows& R = a.rows;
  HeadArgs h{};
  h.h = (const char*)hist;
  h.theta = (const float*)a.theta;
  h.off_w = a.lay.w_out;
  h.off_b = a.lay.b_out;
  h.H = a.cfg.hidden;
  h.V = a.cfg.vocab;
  h.zbo = zbo;
  h.key = make_key(a.seed);
  h.i0 = a.i0;
  h.eps = a.eps;
  h.rm = row_map(R);
  h.M = R.M;
  h.rows = (int64_t)Tc * R.M;
  h.tokens = a.tokens;
  h.C = a.C;
  h.t0 = t0;
  h.B = R.B;
  h.pmax = pmax;
  h.psum = psum;
  h.ptgt = ptgt;
  h.zc_out = a.zc ? (const float*)a.zc + a.zmap.out : nullptr;
  h.zc_stride = a.zmap.pg;
  h.bits = a.bits;
  h.bits_stride = bit_words(a.lay.total);
  const int ns = R.fd ? 1 : 2;
  const Pick pk = pick_shape(h.rm, R.M, ns, (int64_t)a.ws.nvt * kVocabTile, Tc, false);
  h.blocks_per_t = (int)row_blocks(h.rm, R.M, ns, pk.rt);
  h.nvt = a.ws.nvt;
  h.packed = a.wpack != nullptr;
  h.w_out = a.wpack ? a.wpack + a.zmap.out : (const float*)a.theta + a.lay.w_out;
  const int64_t blocks = (int64_t)h.blocks_per_t * Tc * h.nvt;
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  h.blocks = (int)blocks;
  const dim3 grid = wide_grid(blocks);
  ProfScope ps(kKHead, st);
  return by_kind(a, [&](auto k) {
    return by_rt(pk.rt, [&](auto r) {
      constexpr int kind = decltype(k)::value, RT = decltype(r)::value;
      if (a.split) head_f32_kernel<Shape<kind, 2, RT, 2>, true><<<grid, NT, 0, st>>>(h);
      else if (ns == 2) head_f32_kernel<Shape<kind, 2, RT, 2>, false><<<grid, NT, 0, st>>>(h);
      else head_f32_kernel<Shape<kind, 1, RT, 2>, false><<<grid, NT, 0, st>>>(h);
      return hipGetLastError();
    });
  });
}

}  // namespace zo
