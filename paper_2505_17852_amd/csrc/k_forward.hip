// The 2N perturbed forward passes of one CD-RGE step (Algorithm 1's probe
// loop; Eq. 2's two loss queries per probe), batched over all passes.
//
// Every pass (probe n, sign s) runs the same LSTM on the same B sequences
// with weights theta + s eps z_n. A matrix product of a timestep is computed
// for all 2N*B rows at once as
//     a[r] = sum_k A[r][k] (W[c][k] + s_r eps z_n[c][k])
// with the perturbed weight formed from the shared weight and the probe where
// the kernel reads it; theta + s eps z_n as a whole is never formed in memory.
//
// Per timestep: embed (perturbed embedding rows) -> one gate kernel per
// layer (both input products, bias, gate nonlinearities and the cell update
// fused). Every time chunk: one output-head kernel over the chunk's top-layer
// states (vocabulary-tiled, online logsumexp partials), then a combine kernel
// that adds each position's cross-entropy to its row.
// At the end a reduction turns row sums into the 2N losses.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <optional>
#include <type_traits>

#include "zo_kernels.hpp"
#include "zo_pack.hpp"
#include "zo_profile.hpp"
#include "zo_rng.hpp"

namespace zo {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// What a call writes before its first timestep, in one launch (each launch of
// a small model costs more than its work). First the zeros: every pass starts
// from h = c = 0 and empty row sums (the state slots that timestep 0 reads, the
// cell states, the row sums), n16 16-byte words per range; a kernel rather
// than a memset, so that a caller can capture the forward into a graph and
// replay it. Then the bias probes (the biases' perturbation is the same for
// every timestep): zb[l][n][c] = eps z_{i0+n}[bias_l + c], zbo[n][v] = eps
// z_{i0+n}[b_out + v].
struct ZeroRanges {
  uint4* slots;  // `n_slots` state slots of n_state words, `stride` words apart
  int64_t n_slots, n_state, stride;
  uint4* p[3];   // three more ranges
  int64_t n[3];
};
struct BiasOffsets {
  uint64_t layer[kMaxLayers];
};

__global__ __launch_bounds__(256) void prepare_kernel(ZeroRanges zr, int kind, Key key, uint32_t i0, float eps, int N,
                                                      int L, int H4, int V, BiasOffsets bias_off, uint64_t bout_off,
                                                      float* zb, float* zbo) {
  const int64_t per_layer = (int64_t)N * H4, biases = per_layer * L + (int64_t)N * V;
  const int64_t slots = zr.n_slots * zr.n_state;
  const int64_t zeros = slots + zr.n[0] + zr.n[1] + zr.n[2];
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < zeros + biases; i += (int64_t)gridDim.x * 256) {
    if (i < zeros) {
      uint4* q;
      int64_t j = i - slots;
      if (j < 0) {
        const int64_t k = i / zr.n_state;
        q = zr.slots + k * zr.stride + (i - k * zr.n_state);
      } else if (j < zr.n[0]) {
        q = zr.p[0] + j;
      } else if ((j -= zr.n[0]) < zr.n[1]) {
        q = zr.p[1] + j;
      } else {
        q = zr.p[2] + (j - zr.n[1]);
      }
      *q = uint4{0u, 0u, 0u, 0u};
      continue;
    }
    const int64_t t = i - zeros;
    if (t < per_layer * L) {
      const int l = (int)(t / per_layer);
      const int64_t rem = t - l * per_layer;
      const int n = (int)(rem / H4);
      const int c = (int)(rem - (int64_t)n * H4);
      zb[t] = fmul(eps, probe_value(kind, key, i0 + n, bias_off.layer[l] + c));
    } else {
      const int64_t rem = t - per_layer * L;
      const int n = (int)(rem / V);
      const int v = (int)(rem - (int64_t)n * V);
      zbo[rem] = fmul(eps, probe_value(kind, key, i0 + n, bout_off + v));
    }
  }
}

// ---------------------------------------------------------------------------
// Cross-entropy of every position of the chunk: logsumexp over the
// vocabulary tiles' (max, sum of exp) partials, merged online in tile order,
// minus the target logit (0 for unscored positions and padding rows, NaN for
// a scored position whose target token lies outside [0, V)); then added to
// each row's running sum in time order (a fixed summation order: the result
// does not depend on scheduling). A workgroup takes 64 rows, thread (step,
// row) one position of 16 timesteps at a time.
constexpr int kCombineRows = 64, kCombineSteps = 16;
__global__ __launch_bounds__(kCombineRows* kCombineSteps) void combine_kernel(
    const float* pmax, const float* psum, const float* ptgt, int nvt, int64_t rows, int64_t M, int t0, int Tc, int C,
    int B, RowMap rm, const uint8_t* mask, const int32_t* tokens, int V, double* row_loss) {
  __shared__ float ell[kCombineSteps][kCombineRows];
  const int lr = threadIdx.x % kCombineRows, step = threadIdx.x / kCombineRows;
  const int64_t r = block_id() * kCombineRows + lr;
  const int b = r < M ? pass_of(rm, r).b : B;
  double acc = step == 0 && r < M ? row_loss[r] : 0.0;
  for (int c0 = 0; c0 < Tc; c0 += kCombineSteps) {
    const int tt = c0 + step;
    float loss = 0.f;
    if (tt < Tc && b < B && !(mask && !mask[(int64_t)b * C + t0 + tt])) {
      if ((uint32_t)tokens[(int64_t)b * (C + 1) + t0 + tt + 1] >= (uint32_t)V) {
        loss = __builtin_nanf("");
      } else {
        const int64_t rr = (int64_t)tt * M + r;
        float mx = -INFINITY, s = 0.f;
        for (int v = 0; v < nvt; ++v) {
          const float m = pmax[(int64_t)v * rows + rr];
          const float e = psum[(int64_t)v * rows + rr];
          if (m == -INFINITY) continue;
          if (m > mx) {
            s = s * expf(mx - m) + e;
            mx = m;
          } else {
            s += e * expf(m - mx);
          }
        }
        loss = mx + logf(s) - ptgt[rr];
      }
    }
    ell[step][lr] = loss;
    __syncthreads();
    if (step == 0)
      for (int k = 0; k < kCombineSteps && c0 + k < Tc; ++k) acc += (double)ell[k][lr];
    __syncthreads();
  }
  if (step == 0 && r < M) row_loss[r] = acc;
}

// Loss of each pass = (sum over the pass's sequences of their row sums) /
// (scored positions). Central differences: pass 2n -> Lp[n], 2n+1 -> Lm[n];
// forward differences: pass p < N -> Lp[p], the clean pass N -> Lm[0]. One
// wave per pass; every workgroup counts the scored positions.
__global__ __launch_bounds__(256) void reduce_kernel(const double* row_loss, int N, int B, int C,
                                                     RowMap rm, const uint8_t* mask, float* Lp,
                                                     float* Lm) {
  __shared__ int64_t part[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t positions = (int64_t)B * C;
  int64_t total = positions;
  if (mask) {
    int64_t cnt = 0;
    const int64_t whole = ((uintptr_t)mask & 15u) == 0 ? positions / 16 : 0;
    for (int64_t k = threadIdx.x; k < whole; k += 256) {
      const uint4 v = ((const uint4*)mask)[k];
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const uint32_t x = d == 0 ? v.x : d == 1 ? v.y : d == 2 ? v.z : v.w;
        // bit 7 of each byte: the byte is not zero
        cnt += __popc((x | ((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu)) & 0x80808080u);
      }
    }
    for (int64_t k = whole * 16 + threadIdx.x; k < positions; k += 256) cnt += mask[k] ? 1 : 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, 64);
    if (lane == 0) part[wave] = cnt;
    __syncthreads();
    total = part[0] + part[1] + part[2] + part[3];
  }
  const int npass = rm.fd ? N + 1 : 2 * N;
  const int p = (int)blockIdx.x * 4 + wave;
  if (p >= npass) return;
  double s = 0.0;
  const double* rl = row_loss + (int64_t)p * rm.Bp;
  for (int b = lane; b < B; b += 64) s += rl[b];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane != 0) return;
  const float L = total > 0 ? (float)(s / (double)total) : 0.0f;
  if (rm.fd) {
    if (p < N) Lp[p] = L;
    else Lm[0] = L;
  } else if (p & 1) {
    Lm[p >> 1] = L;
  } else {
    Lp[p >> 1] = L;
  }
}

// The fp32 path's product matrices, packed (row_piece), for the gate and head
// kernels: in place their rows lie K values apart, a wave instruction's 64
// lanes fall on 16 rows, and the address unit takes them one row at a time.
// kProbe: instead of the weights, probes i0 .. i0 + N - 1's cached eps z
// (ZCacheMap), the values the kernels compute when they regenerate the
// probe, fp32(eps * z). One thread per 16-byte piece (one
// Philox block).
struct RowSegs {
  int n;
  uint64_t cstart[2 * kMaxLayers + 2];  // start of matrix m in a block of P_g values; cstart[n] = P_g
  uint64_t toff[2 * kMaxLayers + 1];    // offset of matrix m in theta
  int64_t rows[2 * kMaxLayers + 1], K[2 * kMaxLayers + 1];
};

template <bool kProbe>
__global__ __launch_bounds__(256) void row_pack_kernel(const float* theta, float* out, RowSegs segs, Key key,
                                                       uint32_t i0, int N, float eps) {
  const uint64_t pg = segs.cstart[segs.n];
  const uint64_t np = pg >> 2;
  for (int n = blockIdx.y; n < N; n += gridDim.y) {
    float* dst = out + (uint64_t)n * pg;
    for (uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; u < np; u += (uint64_t)gridDim.x * blockDim.x) {
      int m = 0;
      while (m + 1 < segs.n && 4 * u >= segs.cstart[m + 1]) ++m;
      const RowPiece rp = row_piece(u - (segs.cstart[m] >> 2), segs.rows[m], segs.K[m]);
      const uint64_t j = segs.toff[m] + (uint64_t)rp.row * (uint64_t)segs.K[m] + (uint64_t)rp.k;
      if constexpr (kProbe) {
        float z[4];
        gauss_block(key, i0 + (uint32_t)n, j >> 2, z);
        *(f4*)(dst + 4 * u) = f4{fmul(eps, z[0]), fmul(eps, z[1]), fmul(eps, z[2]), fmul(eps, z[3])};
      } else {
        *(f4*)(dst + 4 * u) = *(const f4*)(theta + j);
      }
    }
  }
}

// The bf16 path's product matrices in fragment-packed order (zo_pack.hpp):
// their packed start (ZCacheMap offsets, in values), their offset in theta,
// K, and whether the matrix is the head (vocabulary rows, zero-padded) or a
// gate matrix (4H rows in the gate column order).
struct PackSegs {
  int n;
  int64_t H, V;
  uint64_t cstart[2 * kMaxLayers + 2];  // cstart[n] = P_g (padded)
  uint64_t toff[2 * kMaxLayers + 1];
  int64_t K[2 * kMaxLayers + 1];
  int head[2 * kMaxLayers + 1];
};

// Theta row and first k of lane `lane`'s 8 values of packed block blk (the 1 KB
// blocks of all matrices, counted from the first; the same for a whole wave,
// so its matrix and place are worked out once per wave in 32 bits, not by a
// 64-bit division per chunk: c3's probe cache 8.8 -> 7.7 ms); row < 0 for the head's padding
// rows.
__device__ __forceinline__ void packed_source(const PackSegs& segs, uint32_t blk, int lane, int& m, int64_t& row,
                                              int64_t& k) {
  m = 0;
  while (m + 1 < segs.n && blk >= (uint32_t)(segs.cstart[m + 1] >> 9)) ++m;
  const PackedPos p = packed_position(blk - (uint32_t)(segs.cstart[m] >> 9), lane, (uint32_t)segs.K[m]);
  k = p.k;
  row = segs.head[m] ? (p.col < segs.V ? p.col : -1) : gate_row_of_column(p.col, segs.H);
}

// fp16 copy of the bf16 weight matrices, fragment-packed, read by the bf16
// path's products in place of theta: bf16 -> fp32 is exact and fp32 -> fp16
// rounds to nearest even, exact for every bf16 weight in [2^-14, 65504)
// (smaller ones keep an absolute error below 2^-25). One thread per packed
// 16-byte chunk (8 consecutive k of one row, 16 bytes of theta).
__global__ __launch_bounds__(256) void w16_pack_kernel(const uint16_t* theta, uint16_t* w16, PackSegs segs) {
  const uint64_t nchunks = segs.cstart[segs.n] >> 3;
  for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nchunks;
       q += (uint64_t)gridDim.x * blockDim.x) {
    int m;
    int64_t row, k;
    packed_source(segs, __builtin_amdgcn_readfirstlane((uint32_t)(q >> 6)), (int)(threadIdx.x & 63), m, row, k);
    uint32_t o[4] = {0u, 0u, 0u, 0u};
    if (row >= 0) {
      const uint4 v = *(const uint4*)(theta + segs.toff[m] + (uint64_t)row * (uint64_t)segs.K[m] + (uint64_t)k);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int d = 0; d < 4; ++d)
        o[d] = pack_f16x2(bf16_to_f32((uint16_t)w[d]), bf16_to_f32((uint16_t)(w[d] >> 16)));
    }
    *(uint4*)(w16 + (q << 3)) = uint4{o[0], o[1], o[2], o[3]};
  }
}

// Probe cache of the bf16 path: fp16(eps z) of every product matrix,
// fragment-packed like the weight copy, for probes i0 .. i0 + N - 1. One
// thread per packed chunk: 8 consecutive elements j (a multiple of 8), two
// Philox blocks; zeros for the head's padding rows. The values are those the
// kernels compute when they regenerate the probe.
// w +- z for two packed fp16 pairs, each rounded once to nearest even (the
// value the products' fused form computes in registers from w and z).
__device__ __forceinline__ uint32_t add_f16x2(uint32_t w, uint32_t z, bool minus) {
  typedef _Float16 h2 __attribute__((ext_vector_type(2)));
  const h2 a = __builtin_bit_cast(h2, w), b = __builtin_bit_cast(h2, z);
  return __builtin_bit_cast(uint32_t, minus ? a - b : a + b);
}

// bf16 weights: the probe cache in the packed order of the fp16 weight copy.
// perturbed = false: probe n's fp16(eps z) at n pg. perturbed = true: probe
// n's perturbed weights fp16(w + fp16(eps z)) at 2n pg and fp16(w - fp16(eps
// z)) at (2n + 1) pg, from the packed fp16 weights w16 (written before).
__global__ __launch_bounds__(256) void zcache_pack_kernel(uint16_t* zc, const uint16_t* w16, PackSegs segs, Key key,
                                                          uint32_t i0, int N, float eps, bool perturbed) {
  const uint64_t pg = segs.cstart[segs.n];
  const uint64_t nchunks = pg >> 3;
  for (int n = blockIdx.y; n < N; n += gridDim.y) {
    for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nchunks;
         q += (uint64_t)gridDim.x * blockDim.x) {
      int m;
      int64_t row, k;
      packed_source(segs, __builtin_amdgcn_readfirstlane((uint32_t)(q >> 6)), (int)(threadIdx.x & 63), m, row, k);
      uint32_t o[4] = {0u, 0u, 0u, 0u};
      if (row >= 0) {
        const uint64_t j = segs.toff[m] + (uint64_t)row * (uint64_t)segs.K[m] + (uint64_t)k;
        float za[4], zb[4];
        gauss_block(key, i0 + (uint32_t)n, j >> 2, za);
        gauss_block(key, i0 + (uint32_t)n, (j >> 2) + 1, zb);
        o[0] = pack_f16x2(fmul(eps, za[0]), fmul(eps, za[1]));
        o[1] = pack_f16x2(fmul(eps, za[2]), fmul(eps, za[3]));
        o[2] = pack_f16x2(fmul(eps, zb[0]), fmul(eps, zb[1]));
        o[3] = pack_f16x2(fmul(eps, zb[2]), fmul(eps, zb[3]));
      }
      if (!perturbed) {
        *(uint4*)(zc + (uint64_t)n * pg + (q << 3)) = uint4{o[0], o[1], o[2], o[3]};
      } else {
        // padding rows: w = 0 and z = 0
        const uint4 w = *(const uint4*)(w16 + (q << 3));
        *(uint4*)(zc + (uint64_t)(2 * n) * pg + (q << 3)) =
            uint4{add_f16x2(w.x, o[0], false), add_f16x2(w.y, o[1], false), add_f16x2(w.z, o[2], false),
                  add_f16x2(w.w, o[3], false)};
        *(uint4*)(zc + (uint64_t)(2 * n + 1) * pg + (q << 3)) =
            uint4{add_f16x2(w.x, o[0], true), add_f16x2(w.y, o[1], true), add_f16x2(w.z, o[2], true),
                  add_f16x2(w.w, o[3], true)};
      }
    }
  }
}

}  // namespace

namespace {

// The product matrices in theta order (fp32 path).
RowSegs matrix_segments(const ForwardArgs& a) {
  const zo_config& c = a.cfg;
  RowSegs segs{};
  int m = 0;
  auto add = [&](uint64_t cstart, uint64_t toff, int64_t rows, int64_t K) {
    segs.cstart[m] = cstart;
    segs.toff[m] = toff;
    segs.rows[m] = rows;
    segs.K[m++] = K;
  };
  for (int l = 0; l < c.n_layers; ++l) {
    add(a.zmap.ih[l], a.lay.w_ih[l], 4 * (int64_t)c.hidden, l == 0 ? c.embed : c.hidden);
    add(a.zmap.hh[l], a.lay.w_hh[l], 4 * (int64_t)c.hidden, c.hidden);
  }
  add(a.zmap.out, a.lay.w_out, c.vocab, c.hidden);
  segs.n = m;
  segs.cstart[m] = a.zmap.pg;
  return segs;
}

// The same matrices for the bf16 path's packed fp16 weight copy and probe
// cache.
PackSegs packed_segments(const ForwardArgs& a) {
  const zo_config& c = a.cfg;
  PackSegs segs{};
  segs.H = c.hidden;
  segs.V = c.vocab;
  int m = 0;
  for (int l = 0; l < c.n_layers; ++l) {
    segs.cstart[m] = a.zmap.ih[l];
    segs.toff[m] = a.lay.w_ih[l];
    segs.K[m] = l == 0 ? c.embed : c.hidden;
    segs.head[m++] = 0;
    segs.cstart[m] = a.zmap.hh[l];
    segs.toff[m] = a.lay.w_hh[l];
    segs.K[m] = c.hidden;
    segs.head[m++] = 0;
  }
  segs.cstart[m] = a.zmap.out;
  segs.toff[m] = a.lay.w_out;
  segs.K[m] = c.hidden;
  segs.head[m++] = 1;
  segs.n = m;
  segs.cstart[m] = a.zmap.pg;
  return segs;
}

hipError_t launch_w16_fill(const ForwardArgs& a, hipStream_t st) {
  const PackSegs segs = packed_segments(a);
  uint64_t grid = (a.zmap.pg / 8 + 255) / 256;
  if (grid > 16384) grid = 16384;
  ProfScope ps(kKWeights16, st);
  w16_pack_kernel<<<dim3((unsigned)grid), 256, 0, st>>>((const uint16_t*)a.theta, (uint16_t*)a.w16, segs);
  return hipGetLastError();
}

// The fp32 path's packed weight copy.
hipError_t launch_wpack(const ForwardArgs& a, hipStream_t st) {
  const uint64_t grid = std::min<uint64_t>((a.zmap.pg / 4 + 255) / 256, 16384);
  ProfScope ps(kKWeights16, st);
  row_pack_kernel<false><<<dim3((unsigned)grid), 256, 0, st>>>((const float*)a.theta, const_cast<float*>(a.wpack),
                                                               matrix_segments(a), Key{}, 0, 1, 0.f);
  return hipGetLastError();
}

hipError_t launch_zcache_fill(const ForwardArgs& a, hipStream_t st) {
  const zo_config& c = a.cfg;
  const unsigned gy = (unsigned)(a.rows.N < 65535 ? a.rows.N : 65535);
  const Key key = make_key(a.seed);
  ProfScope ps(kKProbeCache, st);
  if (c.wdtype == ZO_WBF16) {
    const PackSegs segs = packed_segments(a);
    uint64_t gx = (a.zmap.pg / 8 + 255) / 256;
    if (gx > 4096) gx = 4096;
    // fused products read the perturbed weights; two-stream ones fp16(eps z)
    zcache_pack_kernel<<<dim3((unsigned)gx, gy), 256, 0, st>>>((uint16_t*)a.zc, (const uint16_t*)a.w16, segs, key,
                                                                a.i0, a.rows.N, a.eps, !a.split);
  } else {
    uint64_t gx = (a.zmap.pg / 4 + 255) / 256;
    if (gx > 4096) gx = 4096;
    row_pack_kernel<true><<<dim3((unsigned)gx, gy), 256, 0, st>>>((const float*)a.theta, (float*)a.zc, matrix_segments(a),
                                                                  key, a.i0, a.rows.N, a.eps);
  }
  return hipGetLastError();
}

}  // namespace

// The step driver: per timestep the perturbed embedding and one gate launch
// per layer; per time chunk one head launch and one combine; then the
// per-pass reduction. The fp32 and bf16 paths differ only in their embed,
// gate and head kernels.
hipError_t launch_forward(const ForwardArgs& a, hipStream_t st) {
  const zo_config& c = a.cfg;
  const bool bf16 = c.wdtype == ZO_WBF16;
  const int L = c.n_layers, H = c.hidden, V = c.vocab;
  const Rows& R = a.rows;
  const WsPlan& W = a.ws;
  const int64_t M = R.M;
  const size_t el = act_bytes(c);  // bytes of an activation element
  const size_t state = (size_t)M * H * el;
  const RowMap rm = row_map(R);
  char* ws = a.work;
  char* x0 = ws + W.x0;
  char* hbuf = ws + W.hbuf;
  char* hist = ws + W.hist;
  float* cbuf = (float*)(ws + W.cbuf);
  float* zb = (float*)(ws + W.zb);
  float* zbo = (float*)(ws + W.zbo);
  float* pmax = (float*)(ws + W.pmax);
  float* psum = (float*)(ws + W.psum);
  float* ptgt = (float*)(ws + W.ptgt);
  double* row_loss = (double*)(ws + W.row_loss);
  auto head = bf16 ? launch_head_bf16 : launch_head_f32;
  hipError_t e;
#define ZO_TRY(x)                          \
  do {                                     \
    if ((e = (x)) != hipSuccess) return e; \
  } while (0)

  const int T = W.T;
  std::optional<PhaseRange> phase;
  phase.emplace("forward: prepare");
  {
    ZeroRanges zr{};
    zr.slots = (uint4*)(hbuf + state);  // slot 1 of every lower layer
    zr.n_slots = L - 1;
    zr.n_state = (int64_t)(state / 16);
    zr.stride = 2 * zr.n_state;
    zr.p[0] = (uint4*)(T > 1 ? hist + (size_t)(T - 1) * state : ws + W.hzero);
    zr.n[0] = T > 1 ? zr.n_state : (int64_t)(zero_state_bytes(c, M) / 16);
    zr.p[1] = (uint4*)cbuf;
    zr.n[1] = (int64_t)((size_t)L * M * H / 4);
    zr.p[2] = (uint4*)row_loss;
    zr.n[2] = M / 2;
    BiasOffsets boff{};
    for (int l = 0; l < L; ++l) boff.layer[l] = a.lay.bias[l];
    const int64_t total = zr.n_slots * zr.n_state + zr.n[0] + zr.n[1] + zr.n[2] + (int64_t)R.N * 4 * H * L + (int64_t)R.N * V;
    const unsigned grid = (unsigned)std::min<int64_t>((total + 255) / 256, 65536);
    prepare_kernel<<<dim3(grid), dim3(256), 0, st>>>(zr, c.probe, make_key(a.seed), a.i0, a.eps, R.N, L, 4 * H, V, boff,
                                                     a.lay.b_out, zb, zbo);
    ZO_TRY(hipGetLastError());
  }

  // bf16 weights: the fp16 copy of the product matrices; probe cache (normal
  // probes, when the workspace holds it)
  if (bf16) ZO_TRY(launch_w16_fill(a, st));
  if (a.wpack) ZO_TRY(launch_wpack(a, st));
  if (a.zc) ZO_TRY(launch_zcache_fill(a, st));
  if (a.bits) ZO_TRY(launch_bits_fill(a.bits, a.lay.total, a.seed, a.i0, R.N, st));

  // states of layer l at time t: lower layers alternate between two slots
  // (time t in slot t & 1), the top layer writes the time-chunk ring. A ring of
  // one slot (C = 1) holds only the state being written, while other
  // workgroups still read the one before it: that one has memory of its own
  auto state_in = [&](int l, int t) -> char* {  // h of layer l at time t - 1
    if (l < L - 1) return hbuf + (size_t)l * 2 * state + (size_t)((t + 1) & 1) * state;
    return T > 1 ? hist + (size_t)((t + T - 1) % T) * state : ws + W.hzero;
  };
  auto state_out = [&](int l, int t) -> char* {  // h of layer l at time t
    if (l < L - 1) return hbuf + (size_t)l * 2 * state + (size_t)(t & 1) * state;
    return hist + (size_t)(t % T) * state;
  };
  // Launch order. bf16: per timestep the embedding and one gate launch per
  // layer. fp32: a wavefront, launch d running layer l at time d - l for every
  // layer with 0 <= d - l < C, in one launch (layer l reads layer l - 1's state
  // of time d - l, written by launch d - 1, while layer l - 1 writes its other
  // slot); the embeddings of a whole time chunk [d, d + T) are written in one
  // launch before launch d, after launch d - 1 read the last of the previous
  // chunk's.
  const int ndiag = bf16 ? a.C : a.C + L - 1;
  const size_t x0_step = (size_t)M * c.embed * el;  // one timestep of embeddings
  phase.reset();
  for (int d = 0; d < ndiag; ++d) {
    PhaseRange step_range("forward: layer steps of one timestep");
    if (bf16) ZO_TRY(launch_embed_bf16(a, d, x0, st));
    else if (d < a.C && d % T == 0) ZO_TRY(launch_embed_f32(a, d, std::min(T, a.C - d), x0, st));
    if (bf16) {
      for (int l = 0; l < L; ++l) {
        const char* xin = l == 0 ? x0 : state_out(l - 1, d);
        ZO_TRY(launch_gate_bf16(a, l, xin, state_in(l, d), state_out(l, d), cbuf + (size_t)l * M * H,
                                zb + (size_t)l * R.N * 4 * H, st));
      }
    } else {
      GateLayerF32 ls[kLaunchLayers];
      int n = 0;
      for (int l = 0; l < L; ++l) {
        const int t = d - l;
        if (t < 0 || t >= a.C) continue;
        GateLayerF32& g = ls[n++];
        g.x = l == 0 ? x0 + (size_t)(t % T) * x0_step : state_out(l - 1, t);
        g.hprev = state_in(l, t);
        g.hout = state_out(l, t);
        g.cst = cbuf + (size_t)l * M * H;
        g.off_ih = a.lay.w_ih[l];
        g.off_hh = a.lay.w_hh[l];
        g.off_b = a.lay.bias[l];
        g.El = l == 0 ? c.embed : c.hidden;
        g.w_ih = a.wpack ? a.wpack + a.zmap.ih[l] : (const float*)a.theta + g.off_ih;
        g.w_hh = a.wpack ? a.wpack + a.zmap.hh[l] : (const float*)a.theta + g.off_hh;
        g.zb = zb + (size_t)l * R.N * 4 * H;
        g.zc_ih = a.zc ? (const float*)a.zc + a.zmap.ih[l] : nullptr;
        g.zc_hh = a.zc ? (const float*)a.zc + a.zmap.hh[l] : nullptr;
        if (n == kLaunchLayers) {
          ZO_TRY(launch_gates_f32(a, ls, n, st));
          n = 0;
        }
      }
      if (n) ZO_TRY(launch_gates_f32(a, ls, n, st));
    }
    // the top layer has finished time t: the head runs over each completed time chunk
    const int t = bf16 ? d : d - (L - 1);
    if (t >= 0 && (t % T == T - 1 || t == a.C - 1)) {
      const int t0 = t - t % T;
      const int Tc = t - t0 + 1;
      PhaseRange head_range("forward: head and cross entropy of a time chunk");
      ZO_TRY(head(a, hist, t0, Tc, zbo, pmax, psum, ptgt, st));
      ProfScope ps(kKCombine, st);
      combine_kernel<<<wide_grid((M + kCombineRows - 1) / kCombineRows), kCombineRows * kCombineSteps, 0, st>>>(
          pmax, psum, ptgt, W.nvt, (int64_t)Tc * M, M, t0, Tc, a.C, R.B, rm, a.mask, a.tokens, a.cfg.vocab, row_loss);
      ZO_TRY(hipGetLastError());
    }
  }
  PhaseRange reduce_range("forward: loss reduction");
  const unsigned npass = R.fd ? (unsigned)R.N + 1u : 2u * (unsigned)R.N;
  reduce_kernel<<<(npass + 3) / 4, 256, 0, st>>>(row_loss, R.N, R.B, a.C, rm, a.mask, a.Lplus, a.Lminus);
  ZO_TRY(hipGetLastError());
#undef ZO_TRY
  return hipSuccess;
}

}  // namespace zo
