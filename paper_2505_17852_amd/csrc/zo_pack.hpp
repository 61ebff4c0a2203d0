// Address arithmetic of the bf16 path's matrix operands, shared by the
// kernels and the host-side bounds checks (every function here is plain
// integer arithmetic, callable on the host and on the device).
//
// Fragment-packed fp16 matrices. The products of the bf16 path read their B
// operand (the fp16 copy of a weight matrix, and the cached fp16(eps z) of
// normal probes) straight from global memory into registers, one 16-byte
// piece per lane. So that one wave instruction reads 1 KB of consecutive
// memory, the call writes those matrices in the order the v_mfma_f32_32x32x16
// fragments are consumed: the matrix's columns, in the kernels' column
// order, are cut into blocks of 32 and its K dimension into steps of 16;
// block (cb, ks) is 1 KB at ((cb * KS + ks) * 64) * 8 values, and its lane
// L = lr + 32 lg holds the 8 values (column 32 cb + lr, k = 16 ks + 8 lg ..
// 16 ks + 8 lg + 7).
//
// Column order: a gate matrix (4H weight rows, K = E_l or H) takes column
// rho = 64 ug + c to weight row (c / 16) H + 16 ug + c % 16, i.e. gate c / 16
// (i, f, g, o) of hidden unit 16 ug + c % 16, so that one 64-column wave tile
// holds all four gates of 16 units. The head (V rows, K = H) takes column rho
// to vocabulary row rho, padded with zero rows up to out_rows (a whole number
// of 256-wide vocabulary tiles).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zo {

constexpr int kPackBlockCols = 32;  // columns per packed block
constexpr int kPackKStep = 16;      // k per packed block
constexpr int kPackBlockBytes = 1024;

// Weight row of gate-matrix column rho (H hidden units).
__host__ __device__ inline int64_t gate_row_of_column(int64_t rho, int64_t H) {
  const int64_t c = rho & 63, ug = rho >> 6;
  return (c >> 4) * H + 16 * ug + (c & 15);
}

// Source of lane `lane`'s 16 bytes of 1 KB block `blk` of a packed matrix with K
// columns of k: the column (in the kernels' order) and the first k of its 8
// values. (32 bits: a matrix has at most 2^31 values, 2^22 blocks.)
struct PackedPos {
  int64_t col;
  int64_t k;
};
__host__ __device__ inline PackedPos packed_position(uint32_t blk, int lane, uint32_t K) {
  const uint32_t KS = K / kPackKStep, cb = blk / KS, ks = blk - cb * KS;
  return PackedPos{kPackBlockCols * (int64_t)cb + (lane & 31), kPackKStep * (int64_t)ks + 8 * (lane >> 5)};
}

// Byte offset, inside a packed matrix with K columns of k, of the 16 bytes
// lane `lane` reads for the fragment of column block cb at k step ks.
__host__ __device__ inline uint64_t packed_lane_offset(int64_t cb, int64_t K, int lane) {
  return ((uint64_t)cb * (uint64_t)(K / kPackKStep) * 64u + (uint64_t)lane) * 16u;
}
__host__ __device__ inline uint32_t packed_step_offset(int64_t ks) { return (uint32_t)ks * kPackBlockBytes; }

// Packed column block of column tile nt (of 2) of wave column wn (64
// columns each) in workgroup column block nb of tn columns: the same for the
// gate (nb = block of tn / 4 hidden units) and the head (nb = vocabulary tile
// of tn).
__host__ __device__ inline int64_t packed_block_of(int64_t nb, int wn, int nt, int tn) {
  return (int64_t)(tn / kPackBlockCols) * nb + 2 * wn + nt;
}

// Activation tile copies (global -> LDS, 1 KB per wave instruction): copy q
// of wave w fills LDS rows 8 (q NW + w) .. + 7 of the workgroup's tile (128-byte
// rows of 64 fp16 k, 16-byte chunks XOR-swizzled by row so that the 16 rows
// of one fragment read cover all banks). Lane L writes row 8 (q NW + w) +
// L / 8, slot L % 8, which must hold chunk (L % 8) ^ swz(row); this is the
// byte offset of that chunk from the tile's first row at k0 = 0 (lda: the
// row stride in elements); the K tile adds 2 k0 bytes.
__host__ __device__ inline int act_row_of_copy(int q, int w, int lane, int nwaves) {
  return 8 * (q * nwaves + w) + lane / 8;
}
__host__ __device__ inline int act_swizzle(int row) { return (row >> 1) & 7; }
__host__ __device__ inline uint64_t act_copy_offset(int q, int w, int lane, int nwaves, int64_t lda) {
  const int r = act_row_of_copy(q, w, lane, nwaves);
  return (uint64_t)r * (uint64_t)lda * 2u + 16u * (uint64_t)((lane % 8) ^ act_swizzle(r));
}

// Byte offset, in the sign-probe cache of one probe, of the word holding the
// sign of parameter j (32 per word).
__host__ __device__ inline uint32_t sign_word_offset(uint64_t j) { return (uint32_t)(j >> 5) * 4u; }

// The gate's cell-state tile (the workgroup's rows x `cols` hidden units, 64
// or 32, fp32, row stride H in global memory, 4 cols bytes per row in LDS):
// copies of 1 KB, 256 / cols rows each; lane L of copy cp writes row (256 /
// cols) cp + L / (cols / 4), units u0 + 4 (L % (cols / 4)) .. + 3, at LDS byte
// 1024 cp + 16 L. Byte offset from the tile's first row:
__host__ __device__ inline int cell_row_of_copy(int cp, int lane, int cols = 64) {
  return 256 / cols * cp + lane / (cols / 4);
}
__host__ __device__ inline uint32_t cell_copy_offset(int cp, int lane, int64_t H, int64_t u0, int cols = 64) {
  return ((uint32_t)cell_row_of_copy(cp, lane, cols) * (uint32_t)H + (uint32_t)u0) * 4u +
         16u * (uint32_t)(lane % (cols / 4));
}

// The head's bias values of vocabulary tile v0 .. v0 + 255: the bias probe
// values (fp32) one column per lane, lane L of copy q < 4 reading column
// v0 + 64 q + L; the bf16 bias as 4-byte words from the 4-byte boundary at
// or below its first element (lead: 0 or 2 bytes before it), word d < 256 of
// the tile at this offset from that boundary. Column c's bias is then at
// byte lead + 2 (c - v0) of the tile's words.
__host__ __device__ inline uint32_t head_probe_offset(int64_t v0, int q, int lane) {
  return 4u * (uint32_t)(v0 + 64 * q + lane);
}
__host__ __device__ inline uint32_t head_bias_word_offset(int64_t v0, int d) {
  return 2u * (uint32_t)v0 + 4u * (uint32_t)d;
}
__host__ __device__ inline uint32_t head_bias_bytes(uint32_t lead, int64_t V) {
  return (lead + 2u * (uint32_t)V + 3u) & ~3u;
}

// fp32 path: activations split into three bf16 parts and packed in the order
// the v_mfma_f32_16x16x32_bf16 operands are read: part p of 16-row tile rt and
// 32-k tile kt of a state with K values per row (a multiple of 32) is 1 KB at
// ((rt (K / 32) + kt) 3 + p) 1024, lane L = row + 16 (k % 32) / 8 holding the 8
// values k % 8. Byte offset of part 0 of element k of row `row` of tile rt (parts 1 and
// 2 are 1024 and 2048 bytes further).
constexpr int kSplitParts = 3;
__host__ __device__ inline size_t split_offset(int64_t rt, int row, int k, int K) {
  return (size_t)(rt * (K >> 5) + (k >> 5)) * (kSplitParts * 1024) + (size_t)((row + 16 * ((k & 31) >> 3)) * 16 + (k & 7) * 2);
}

// fp32 path: weight matrices (and cached eps z) packed in the order the gate and
// head kernels read them, so that a wave instruction covers consecutive
// memory: rows in blocks of 16 (the last block may have fewer, R), K in tiles
// of 32; block b starts at value 16 b K and holds, per k tile, the 16-byte
// pieces [half][kg][row] of the R rows: values k = 32 kt + 8 kg + 4 half .. + 3
// of row 16 b + row. (rows, k) of 16-byte piece u of a matrix of n rows of K:
struct RowPiece {
  int64_t row;
  int k;
};
__host__ __device__ inline int64_t block_rows(int64_t b, int64_t n) { return n - 16 * b < 16 ? n - 16 * b : 16; }
__host__ __device__ inline RowPiece row_piece(uint64_t u, int64_t n, int64_t K) {
  const int64_t b = (int64_t)(u / (uint64_t)(4 * K));  // 16 rows of K / 4 pieces
  uint32_t rem = (uint32_t)(u - (uint64_t)b * (uint64_t)(4 * K));
  const uint32_t R = (uint32_t)block_rows(b, n);
  const uint32_t kt = rem / (8 * R);
  rem -= kt * 8 * R;
  const uint32_t half = rem / (4 * R);
  rem -= half * 4 * R;
  const uint32_t kg = rem / R;
  return RowPiece{16 * b + (rem - kg * R), (int)(32 * kt + 8 * kg + 4 * half)};
}

}  // namespace zo
