// Shapes, parameter layout, pass/row numbering and workspace plan of the
// CD-RGE step, shared by the host launchers and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <initializer_list>

#include "../../include/zo.h"

namespace zo {

constexpr int kMaxLayers = 64;

// Flat parameter layout (the model as one vector, every element perturbed):
// EMB[V][E]; per layer W_ih[4H][E_l], W_hh[4H][H], b[4H]; W_out[V][H]; b_out[V].
struct Layout {
  uint64_t emb;
  uint64_t w_ih[kMaxLayers];
  uint64_t w_hh[kMaxLayers];
  uint64_t bias[kMaxLayers];
  uint64_t w_out;
  uint64_t b_out;
  uint64_t total;
};

inline bool config_valid(const zo_config* c) {
  return c && c->n_layers >= 1 && c->n_layers <= kMaxLayers && c->vocab >= 1 && c->embed >= 1 &&
         c->hidden >= 1 && (c->wdtype == ZO_WFP32 || c->wdtype == ZO_WBF16) &&
         (c->probe == ZO_RADEMACHER || c->probe == ZO_GAUSSIAN);
}

inline Layout make_layout(const zo_config& c) {
  Layout L{};
  const uint64_t V = (uint64_t)c.vocab, E = (uint64_t)c.embed, H = (uint64_t)c.hidden;
  uint64_t p = 0;
  L.emb = p;
  p += V * E;
  for (int l = 0; l < c.n_layers; ++l) {
    const uint64_t El = l == 0 ? E : H;
    L.w_ih[l] = p;
    p += 4 * H * El;
    L.w_hh[l] = p;
    p += 4 * H * H;
    L.bias[l] = p;
    p += 4 * H;
  }
  L.w_out = p;
  p += V * H;
  L.b_out = p;
  p += V;
  L.total = p;
  return L;
}

// Rows of the batched forward. The passes each run the B sequences; every
// matrix product of a timestep covers all of them at once. B is padded to Bp
// (a multiple of the path's row granule) so that every row tile of a kernel
// lies inside one pass (and, for central differences, one probe). Padded
// rows (b >= B) carry zeros in, are computed like the others and never
// scored.
//   central differences (2N passes): row r = (2 n + sidx) Bp + b with sidx 0
//     for theta + eps z_n and 1 for theta - eps z_n;
//   forward differences (N + 1 passes): row r = p Bp + b, pass p < N at
//     theta + eps z_p, pass N at theta itself (the clean pass).
constexpr int kRowGranuleF32 = 16;   // fp32 path: the row tile of its MFMAs and of the packed states

// Workgroup tiles of the bf16 path: 256, 128 or 64 rows (two wave rows of half
// as many), 256 columns; the gate's 64-row tile has 128 columns. Every wave
// row lies inside one sign's rows and every tile inside one probe's, so the
// batch is padded to half the tile's rows (central differences) or to all of
// them (forward differences).
constexpr int kTileRows[3] = {256, 128, 64};

// Cost of wgs workgroups of a tile, in units of one round of 256-row tiles (a
// workgroup per CU). Measured with one shape forced at a time over models of
// 512 to 4,096 units and 256 to 16,384 rows: a round of 128-row tiles takes
// 0.62 of one of 256-row tiles, the gate's 64 x 128 tiles 0.32 for the first
// 256 and 0.25 per 256 when three share a CU, the head's 64 x 256 ones 0.45.
// (Every tile reads the same weight fragments per column, so smaller tiles
// cost more per row; they win where 256-row tiles would leave CUs idle or
// compute padding.)
inline double tile_cost(int64_t wgs, int tm, bool gate) {
  const double rounds = (double)((wgs + 255) / 256);
  if (tm == 256) return rounds;
  if (tm == 128) return 0.62 * rounds;
  if (!gate) return 0.45 * rounds;
  return wgs == 0 ? 0 : 0.25 * rounds > 0.32 ? 0.25 * rounds : 0.32;
}
inline int64_t tile_cols(int tm, bool gate) { return gate && tm == 64 ? 128 : 256; }

// The tiles of a launch over `rows` rows and `cols` columns, at most max_tm
// rows each: the first `rows` of the plan in tiles of tm rows and (gate) the
// rest in 64-row tiles, where that fills a last round that tiles of tm rows
// would leave nearly empty. Every tile shape gives the same bits.
struct TilePlan {
  int tm;
  int64_t rows;
};
inline TilePlan pick_tiles(int64_t rows, int64_t cols, bool gate, int max_tm, double* cost = nullptr) {
  TilePlan best{64, rows};
  double least = 0;
  for (int tm : kTileRows) {
    if (tm > max_tm) continue;
    const int64_t tn = tile_cols(tm, gate), nn = (cols + tn - 1) / tn, nm = rows / tm;
    double c = tile_cost(nm * nn, tm, gate);
    int64_t whole = nm;
    if (gate && tm > 64) {
      // whole rounds of tm-row tiles, the rest (64-row tiles) after them
      const int64_t n1 = nm * nn / 256 * 256 / nn;
      const int64_t rest = (rows - n1 * tm) / 64 * ((cols + 127) / 128);
      const double split = tile_cost(n1 * nn, tm, true) + tile_cost(rest, 64, true) + 0.05;
      if (n1 > 0 && n1 < nm && split < 0.97 * c) {
        c = split;
        whole = n1;
      }
    }
    if (least == 0 || c < 0.97 * least) {
      least = c;
      best = TilePlan{tm, whole * tm};
    }
  }
  if (cost) *cost = least;
  return best;
}

// The multiple that batches are padded to. bf16 path: the one whose launches
// cost least (per timestep: L gate launches of K = 2 H and a share of the
// head's, K = H), the largest of equals.
inline int row_granule(const zo_config& c, int32_t N, int32_t B, bool fd = false) {
  if (c.wdtype != ZO_WBF16) return kRowGranuleF32;
  int best = 0;
  double least = 0;
  for (int tm : kTileRows) {
    const int g = fd ? tm : tm / 2;
    const int64_t Bp = ((int64_t)B + g - 1) / g * g;
    const int64_t M = (fd ? (int64_t)N + 1 : 2 * (int64_t)N) * Bp;
    double gate, head;
    pick_tiles(M, 4 * (int64_t)c.hidden, true, tm, &gate);
    pick_tiles(16 * M, c.vocab, false, tm, &head);
    const double cost = c.n_layers * gate * 2 + head / 16;
    if (best == 0 || cost < 0.97 * least) {
      least = cost;
      best = g;
    }
  }
  return best;
}
// The multiple that the reported workspace sizes count with. The bf16 granule
// above turns with N and B, so the rows of a call are not monotone in them
// (N = 32 and 33 of a batch of 160 take 12,288 and 10,560 rows); a workspace of a
// reported size also holds every call with fewer probes, sequences or positions.
// Every granule divides this one, so no call has more rows than it counts.
inline int size_granule(const zo_config& c, bool fd) {
  if (c.wdtype != ZO_WBF16) return kRowGranuleF32;
  return fd ? kTileRows[0] : kTileRows[0] / 2;
}
// Bytes of one activation value: fp16 (bf16 weights), three bf16 parts (fp32 weights).
inline size_t act_bytes(const zo_config& c) { return c.wdtype == ZO_WBF16 ? 2 : 6; }

struct Rows {
  int32_t B, Bp, N;
  int64_t pair_rows;  // rows of one probe: 2 Bp (central) or Bp (forward)
  int64_t M;          // all rows: 2 N Bp (central) or (N + 1) Bp (forward)
  int fd;
};

// Grids that may have more workgroups than one dimension takes: a dimension's
// workgroups times their threads (up to 1,024) must stay below 2^32, and the
// runtime cuts a larger product to 32 bits without an error. x takes up to kGridX
// workgroups (a multiple of 8, so that workgroup i stays on XCD i % 8), y the
// rest; block_id() (zo_rng.hpp) counts them, in the last row past their number.
constexpr int64_t kGridX = (int64_t)1 << 21;
inline dim3 wide_grid(int64_t blocks) {
  return blocks <= kGridX ? dim3((unsigned)blocks) : dim3((unsigned)kGridX, (unsigned)((blocks + kGridX - 1) / kGridX));
}

// The most rows of a bf16 tile: a tile lies inside one probe's rows, a wave row
// (half of it) inside one sign's.
inline int largest_tile(const Rows& r) {
  for (int tm : kTileRows)
    if (r.pair_rows % tm == 0) return tm;
  return 0;
}

struct RowMap {
  int Bp;
  int64_t pair_rows;
  int fd;  // forward differences
  int N;
};

inline Rows make_rows(int32_t N, int32_t B, int granule, bool fd = false) {
  Rows r;
  r.B = B;
  r.N = N;
  r.fd = fd ? 1 : 0;
  r.Bp = (B + granule - 1) / granule * granule;
  r.pair_rows = fd ? (int64_t)r.Bp : 2 * (int64_t)r.Bp;
  r.M = fd ? (int64_t)(N + 1) * r.Bp : (int64_t)N * r.pair_rows;
  return r;
}

inline RowMap row_map(const Rows& r) { return RowMap{r.Bp, r.pair_rows, r.fd, r.N}; }

// The pass of row r: its probe (relative index; the clean pass reports
// probe N - 1, whose values it multiplies by 0), the sign of eps (+1, -1, or
// 0 for the clean pass) and its sequence b.
struct PassOf {
  int probe;
  int sign;
  int b;
};
__host__ __device__ inline PassOf pass_of(const RowMap& m, int64_t r) {
  const int64_t p = r / m.pair_rows;
  const int loc = (int)(r - p * m.pair_rows);
  if (m.fd) return PassOf{p < m.N ? (int)p : m.N - 1, p < m.N ? 1 : 0, loc};
  return loc >= m.Bp ? PassOf{(int)p, -1, loc - m.Bp} : PassOf{(int)p, 1, loc};
}

// Workgroup tiles of the fp32 path: 2 rt row tiles of 16 rows (rt of each pass of
// a probe, central differences; 2 rt of one pass, forward differences), 64 ct
// columns. ns: the signs of a workgroup's rows, 2 or 1.
inline int64_t row_blocks(const RowMap& rm, int64_t M, int NS, int RT) {
  const int q = rm.Bp >> 4;
  return NS == 2 ? M / (2 * rm.Bp) * ((q + RT - 1) / RT) : M / rm.Bp * ((q + 2 * RT - 1) / (2 * RT));
}
// The tile shape of a launch: the cheapest by the time a compute unit spends
// on its workgroups. A workgroup of RT and CT takes, per k tile and wave, CT x
// (forming its weights: 480 cycles, 270 for one sign, and 12 RT MFMAs of 16
// cycles) plus a fixed part; the chip takes ceil(workgroups / CUs) of them.
// Every shape sums in the same order, so the choice never changes a result. (The
// forming time is that of sign words read as bits; reading eps z takes about as
// long, regenerating normals several times it. The rule does not tell them
// apart: no other shape was measured for regenerated probes.)
struct Pick {
  int rt, ct;
};
inline Pick pick_shape(const RowMap& rm, int64_t M, int NS, int64_t cols, int64_t groups, bool ct1) {
  constexpr int kCus = 256;
  Pick best{4, 2};
  double cost = 0;
  for (int ct = 2; ct >= (ct1 ? 1 : 2); --ct) {
    for (int rt = 4; rt >= 1; --rt) {
      const int64_t wgs = row_blocks(rm, M, NS, rt) * ((cols + 64 * ct - 1) / (64 * ct)) * groups;
      const double one = ct * ((NS == 2 ? 480 : 270) + 192.0 * rt) + 150;
      const double c = (double)((wgs + kCus - 1) / kCus) * one;
      if (cost == 0 || c < 0.97 * cost) {
        cost = c;
        best = Pick{rt, ct};
      }
    }
  }
  return best;
}

// Time steps whose top-layer states are kept for one batched output-head pass
// (fp32 path: see time_chunk).
constexpr int kTimeChunk = 16;

// Output-head vocabulary tile (columns per workgroup): 256 on the bf16 path,
// 128 on the fp32 path.
constexpr int kVocabTile = 128;
// Columns per workgroup of the bf16 products (gate columns or vocabulary
// rows; the gate's 64-row tiles have 128). (128 x 512 workgroups, which load
// each weight fragment once, measured slower than 256 x 256.)
constexpr int kVocabTileWide = 256;
inline int vocab_tile(const zo_config& c) { return c.wdtype == ZO_WBF16 ? kVocabTileWide : kVocabTile; }

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Probe cache (normal probes only): the 2N forward passes read the probe
// terms of every weight matrix (W_ih, W_hh of each layer and W_out) at every
// timestep and row tile, while each value is the same for the whole call.
// With a large enough workspace the call first writes, once, the values the
// kernels would otherwise regenerate: eps z in fp32 (fp32 weights) or
// fp16(eps z) (bf16 weights), for probes i0 .. i0+N-1. Layout: probe n's
// block of P_g values (the matrices in theta order) at n * P_g; each matrix
// packed like the weight copy the kernels read: row_piece (fp32 weights) or
// fragment-packed fp16 (bf16 weights), both in zo_pack.hpp. Sign
// probes are cached as bits instead (below). The same map places the matrices of the
// bf16 path's fp16 weight copy; there the head matrix is padded with zero
// rows to a whole number of 256-wide vocabulary tiles.
struct ZCacheMap {
  uint64_t pg;              // values per probe: the matrices' total size
  uint64_t ih[kMaxLayers];  // offsets of each matrix inside a probe's block
  uint64_t hh[kMaxLayers];
  uint64_t out;
  uint64_t out_rows;        // rows of the head matrix as stored (V, or padded on the bf16 path)
};

inline ZCacheMap make_zcache_map(const zo_config& c) {
  ZCacheMap m{};
  const uint64_t E = (uint64_t)c.embed, H = (uint64_t)c.hidden, V = (uint64_t)c.vocab;
  uint64_t p = 0;
  for (int l = 0; l < c.n_layers; ++l) {
    m.ih[l] = p;
    p += 4 * H * (l == 0 ? E : H);
    m.hh[l] = p;
    p += 4 * H * H;
  }
  m.out = p;
  m.out_rows = c.wdtype == ZO_WBF16 ? (V + kVocabTileWide - 1) / kVocabTileWide * kVocabTileWide : V;
  p += m.out_rows * H;
  m.pg = p;
  return m;
}

// The bf16 kernels reach a packed matrix through one buffer resource with 32-bit
// offsets.
inline bool bf16_matrices_fit(const zo_config& c) {
  const uint64_t H = (uint64_t)c.hidden, K = std::max(H, (uint64_t)c.embed);
  return 4 * H * K * 2 < 1ull << 32 && make_zcache_map(c).out_rows * H * 2 < 1ull << 32;
}

// Bit-packed sign-probe cache (sign probes): the sign words of probes i0 ..
// i0+N-1 over the whole parameter vector, written once per call (one Philox
// block per 128 parameters and probe) and read by the forward kernels in place of regenerating them in every K tile: probe n's word w, the
// signs of parameters 32 w .. 32 w + 31 (a set bit for z = +1), at
// n * bit_words(P) + w, unshuffled: parameter 32 w + 2 i at bit i and
// 32 w + 2 i + 1 at bit 16 + i (sign_word_unshuffle of the generator's word),
// the order in which the bf16 products turn a pair of flags into a packed
// fp16 pair with one shift. The update can read the same words
// (zo_update_cached) instead of regenerating them.
// With fp32 weights the words are for the forward's own use; only the bf16
// ones are offered to callers (bit_cache_kind). The bf16 kernels reach a probe's
// words with 32-bit offsets too: from 2^35 parameters on they are regenerated.
inline bool cacheable_probes(const zo_config& c) {
  return c.probe != ZO_RADEMACHER || c.wdtype != ZO_WBF16 || make_layout(c).total < 1ull << 35;
}
inline bool bit_cache_kind(const zo_config& c) {
  return c.probe == ZO_RADEMACHER && c.wdtype == ZO_WBF16 && cacheable_probes(c);
}
__host__ __device__ inline uint64_t bit_words(uint64_t P) { return (P + 127) / 128 * 4; }

// A word of 32 flags with the even-indexed flags moved to bits 0..15 and the
// odd-indexed ones to bits 16..31, each half in order (four delta swaps);
// sign_word_shuffle is its inverse (the same swaps in reverse order).
__host__ __device__ inline uint32_t sign_word_unshuffle(uint32_t x) {
  uint32_t t;
  t = (x ^ (x >> 1)) & 0x22222222u;
  x = x ^ t ^ (t << 1);
  t = (x ^ (x >> 2)) & 0x0C0C0C0Cu;
  x = x ^ t ^ (t << 2);
  t = (x ^ (x >> 4)) & 0x00F000F0u;
  x = x ^ t ^ (t << 4);
  t = (x ^ (x >> 8)) & 0x0000FF00u;
  x = x ^ t ^ (t << 8);
  return x;
}
__host__ __device__ inline uint32_t sign_word_shuffle(uint32_t x) {
  uint32_t t;
  t = (x ^ (x >> 8)) & 0x0000FF00u;
  x = x ^ t ^ (t << 8);
  t = (x ^ (x >> 4)) & 0x00F000F0u;
  x = x ^ t ^ (t << 4);
  t = (x ^ (x >> 2)) & 0x0C0C0C0Cu;
  x = x ^ t ^ (t << 2);
  t = (x ^ (x >> 1)) & 0x22222222u;
  x = x ^ t ^ (t << 1);
  return x;
}

// Kernel variants for normal probes read from the probe cache (fp16(eps z)
// as a second operand stream; or, bf16 weights with fused products, the
// perturbed weights fp16(w +- fp16(eps z)) as the B operand itself) and for
// sign probes read from the sign-probe cache (next to the probe kinds
// ZO_RADEMACHER and ZO_GAUSSIAN, which regenerate them).
constexpr int kGaussCached = 2;
constexpr int kSignsCached = 3;
constexpr int kGaussPerturbed = 4;

// Workspace plan (byte offsets from the workspace base, 256-aligned). An
// activation value takes act_bytes: fp16, or three bf16 parts (split_offset).
struct WsPlan {
  size_t x0;         // [M][E] perturbed embeddings of one timestep (bf16 path), [T][M][E] of a chunk (fp32)
  size_t hbuf;       // [L-1][2][M][H]     double-buffered states of the lower layers
  size_t hist;       // [T][M][H]          top-layer states of the current time chunk
  size_t hzero;      // the top layer's state before the first timestep where the chunk has one slot (C = 1):
                     // [M][H] (bf16 path), one packed row tile of zeros for all rows (fp32)
  size_t cbuf;       // f32 [L][M][H]      cell states
  size_t zb;         // f32 [L][N][4H]     eps * z of the gate biases, per probe
  size_t zbo;        // f32 [N][V]         eps * z of the head bias, per probe
  size_t pmax;       // f32 [nvt][T*M]     per vocabulary tile: running max
  size_t psum;       // f32 [nvt][T*M]     per vocabulary tile: sum of exp(y - max)
  size_t ptgt;       // f32 [T*M]          target logit
  size_t row_loss;   // f64 [M]            masked loss sum of each row
  size_t w16;        // f16 [P_g]          bf16 weights: the product matrices in fp16 (ZCacheMap layout)
  // what the plan's Caches ask for; everything else is needed
  size_t wpack;      // f32 [P_g]          fp32 weights: the product matrices packed (row_piece)
  size_t zcache;     // probe cache (normal probes; see ZCacheMap): fp32 weights [N][P_g] eps z;
                     // bf16 weights [N][2][P_g] fp16: probe n's perturbed weights
                     // fp16(w + fp16(eps z)) and fp16(w - fp16(eps z)) (fused products), or
                     // fp16(eps z) in the first N P_g values (two-stream products)
  size_t bits;       // sign words [N][bit_words(P)] u32 (sign probes)
  size_t total;      // bytes of the plan
  int nvt;           // vocabulary tiles
  int T;             // time chunk
};

// The parts of a plan that save work where there is room for them.
struct Caches {
  bool probes;  // normal probes: zcache; sign probes: bits
  bool wpack;   // fp32 weights: the packed copy
};

// Time steps per chunk. bf16 path: kTimeChunk. fp32 path: as many (8 to 64) as
// keep the chunk's buffers below 16 MiB: small models then take few head
// launches, and the states of large ones stay near the caches. A workspace
// without room for that takes fewer (plan_for_bytes), down to
// least_time_chunk: two, which keeps the state being written apart from the
// one before it.
constexpr size_t kChunkBytes = (size_t)16 << 20;
inline size_t chunk_step_bytes(const zo_config& c, int64_t M, int nvt) {
  return (size_t)M * (((size_t)c.embed + (size_t)c.hidden) * act_bytes(c) + 8 * (size_t)nvt + 4);
}
inline int time_chunk(const zo_config& c, int64_t M, int nvt, int32_t C) {
  if (c.wdtype == ZO_WBF16) return C < kTimeChunk ? C : kTimeChunk;
  const size_t n = kChunkBytes / chunk_step_bytes(c, M, nvt);
  const int T = n < 8 ? 8 : n > 64 ? 64 : (int)n;
  return C < T ? C : T;
}
inline int least_time_chunk(const zo_config& c, int32_t C) {
  const int least = c.wdtype == ZO_WBF16 ? kTimeChunk : 2;
  return C < least ? C : least;
}

// Bytes of the zero state of a one-slot chunk. (bf16 path: all rows; with one
// row for all, the row stride became a value of its own in the gate kernel,
// which cost the large model's losses 0.2%.)
inline size_t zero_state_bytes(const zo_config& c, int64_t M) {
  return (size_t)c.hidden * act_bytes(c) * (c.wdtype == ZO_WBF16 ? (size_t)M : 16);
}

inline int vocab_tiles(const zo_config& c) { return (int)(((int64_t)c.vocab + vocab_tile(c) - 1) / vocab_tile(c)); }
inline size_t probe_cache_bytes(const zo_config& c, int32_t N) {
  if (c.probe == ZO_RADEMACHER) return (size_t)N * bit_words(make_layout(c).total) * 4;
  return (size_t)N * make_zcache_map(c).pg * (c.wdtype == ZO_WBF16 ? 2 * 2 : 4);
}
inline size_t wpack_bytes(const zo_config& c) { return (size_t)make_zcache_map(c).pg * 4; }
// The packed weight copy costs one launch more, made up for after a few hundred
// k tiles per column (c1, 96 of them: 232 us per step without it, 238 with;
// c2's evaluation, 3,600: 2.75 against 2.62 ms).
inline bool wpack_pays(const zo_config& c, int32_t C) {
  return c.wdtype == ZO_WFP32 && (int64_t)C * ((int64_t)c.embed + c.hidden) / 32 >= 256;
}

inline WsPlan plan_workspace(const zo_config& c, const Rows& r, int T, Caches caches) {
  WsPlan w{};
  const size_t M = (size_t)r.M, E = (size_t)c.embed, H = (size_t)c.hidden, V = (size_t)c.vocab;
  const size_t L = (size_t)c.n_layers;
  const size_t el = act_bytes(c);
  w.nvt = vocab_tiles(c);
  w.T = T;
  size_t p = 0;
  auto take = [&](size_t bytes) {
    size_t o = p;
    p = align_up(p + bytes, 256);
    return o;
  };
  w.x0 = take((c.wdtype == ZO_WBF16 ? 1 : (size_t)w.T) * M * E * el);
  w.hbuf = take((L - 1) * 2 * M * H * el);
  w.hist = take((size_t)w.T * M * H * el);
  w.hzero = p;
  if (w.T == 1) take(zero_state_bytes(c, r.M));
  w.cbuf = take(L * M * H * 4);
  w.zb = take(L * (size_t)r.N * 4 * H * 4);
  w.zbo = take((size_t)r.N * V * 4);
  w.pmax = take((size_t)w.nvt * w.T * M * 4);
  w.psum = take((size_t)w.nvt * w.T * M * 4);
  w.ptgt = take((size_t)w.T * M * 4);
  w.row_loss = take(M * 8);
  w.w16 = p;
  if (c.wdtype == ZO_WBF16) take((size_t)make_zcache_map(c).pg * 2);
  w.wpack = p;
  if (caches.wpack) take(wpack_bytes(c));
  w.zcache = w.bits = p;
  if (caches.probes) take(probe_cache_bytes(c, r.N));
  w.total = p;
  return w;
}

// The plan of a call in a workspace of ws_bytes: the caches that fit beside a
// chunk of at least 8 timesteps (the probes' first: a regenerated probe costs
// more than a weight read in place), then the longest chunk up to the preferred
// one. total > ws_bytes: the workspace holds no plan, and total is what the
// smallest takes.
inline WsPlan plan_for_bytes(const zo_config& c, const Rows& r, int32_t C, size_t ws_bytes, Caches* used) {
  const int most = time_chunk(c, r.M, vocab_tiles(c), C), least = least_time_chunk(c, C);
  const int mid = most < 8 || c.wdtype == ZO_WBF16 ? most : 8;
  WsPlan w{};
  auto fits = [&](int T, Caches k) {
    w = plan_workspace(c, r, T, k);
    *used = k;
    return w.total <= ws_bytes;
  };
  const bool pack = wpack_pays(c, C), probes = cacheable_probes(c);
  for (Caches k : {Caches{true, true}, Caches{true, false}, Caches{false, true}, Caches{false, false}}) {
    if ((k.wpack && !pack) || (k.probes && !probes)) continue;
    if (!fits(mid, k)) continue;
    for (int T = most; T > mid; --T)
      if (fits(T, k)) return w;
    fits(mid, k);
    return w;
  }
  for (int T = mid; T > least; --T)
    if (fits(T, Caches{false, false})) return w;
  fits(least, Caches{false, false});
  return w;
}

// A fixed account of the bytes of a call with N probes and B x C positions:
// batches padded to 128 or 256 sequences with bf16 weights, to 32 or 64 with
// fp32 ones, 2 or 4 bytes per activation, chunks of kTimeChunk timesteps. It
// grows with N, B and C and does not follow how the forward lays out its
// buffers; zo_perturbed_losses_noalloc holds it against its fixed size (so the
// shapes it takes stay the same), and the smallest fp32 workspace is at least
// as large (fp32 states take 6 bytes, in fewer rows and timesteps).
inline size_t account_bytes(const zo_config& c, int32_t N, int32_t B, int32_t C, bool fd) {
  const bool b16 = c.wdtype == ZO_WBF16;
  const int g = (b16 ? 128 : 32) * (fd ? 2 : 1);
  const size_t M = (size_t)make_rows(N, B, g, fd).M, T = (size_t)(C < kTimeChunk ? C : kTimeChunk);
  const size_t E = (size_t)c.embed, H = (size_t)c.hidden, V = (size_t)c.vocab, L = (size_t)c.n_layers;
  const size_t nvt = (V + (size_t)vocab_tile(c) - 1) / (size_t)vocab_tile(c), el = b16 ? 2 : 4;
  size_t p = 0;
  for (size_t bytes : {(b16 ? 1 : T) * M * E * el, (L - 1) * 2 * M * H * el, T * M * H * el, L * M * H * 4,
                       L * (size_t)N * 4 * H * 4, (size_t)N * V * 4, nvt * T * M * 4, nvt * T * M * 4, T * M * 4, M * 8,
                       b16 ? (size_t)make_zcache_map(c).pg * 2 : (size_t)0})
    p = align_up(p + bytes, 256);
  return p;
}

// Reported workspace sizes. A workspace of the size of (N, B, C) holds every call
// with at most as many probes, sequences and positions, so each part grows with
// them: rows by size_granule, and for the fp32 chunk, whose length falls with
// the rows, the bound min(min(C, 64) steps, max(16 MiB, min(C, 8) steps)) of
// time_chunk's bytes.
//   full      every cache, except sign words or packed weights (fp32) beyond
//             kExtraCap each: a call that fills the device's memory without
//             them still fits, and takes them where a workspace has the room
//   smallest  no caches beyond kSmallExtras of them and of longer chunks (a small
//             model's smallest workspace then has what its full one has; 3
//             layers of 160 units, 8 probes, a batch of 16: 668 us with the
//             whole sequence in one chunk, 696 us with one timestep left over),
//             and at least account_bytes
constexpr size_t kExtraCap = (size_t)8 << 30, kSmallExtras = (size_t)32 << 20;
struct WsSizes {
  size_t full, smallest;
};
inline WsSizes workspace_sizes(const zo_config& c, int32_t N, int32_t B, int32_t C, bool fd) {
  const Rows r = make_rows(N, B, size_granule(c, fd), fd);
  const int least = least_time_chunk(c, C);
  if (c.wdtype == ZO_WBF16)
    return WsSizes{plan_workspace(c, r, least, Caches{cacheable_probes(c), false}).total,
                   plan_workspace(c, r, least, Caches{false, false}).total};
  // a plan without its chunk's buffers and with room for the zero state and each buffer's alignment
  const size_t step = chunk_step_bytes(c, r.M, vocab_tiles(c));
  const size_t fixed = plan_workspace(c, r, 0, Caches{false, false}).total + zero_state_bytes(c, r.M) + 8 * 256;
  const size_t need = fixed + (size_t)least * step;
  size_t want = fixed + std::min((size_t)std::min(C, 64) * step, std::max(kChunkBytes, (size_t)std::min(C, 8) * step));
  if (wpack_pays(c, C) && wpack_bytes(c) <= kExtraCap) want += align_up(wpack_bytes(c), 256);
  size_t zc = 0;
  if (c.probe == ZO_RADEMACHER) want += align_up(std::min(probe_cache_bytes(c, N), kExtraCap), 256);
  else zc = align_up(probe_cache_bytes(c, N), 256);
  const size_t smallest = std::max(account_bytes(c, N, B, C, fd), std::min(want, need + kSmallExtras));
  return WsSizes{std::max(smallest, want) + zc, smallest};
}

}  // namespace zo
