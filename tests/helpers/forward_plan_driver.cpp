// Runs the host side of a forward call (zo_api.hip and k_forward.hip, as
// built for the host) with its kernel launchers replaced by checks: no GPU is
// touched. Every buffer that a launch is given must lie inside the workspace,
// apart from the others, and no launch may write memory that it also reads as
// another workgroup's input (a layer's new state over the state before it or
// over its input). One call per input line,
//     L V E H wdtype probe fd N B C ws_bytes
// (fd 2: the no-alloc entry point, which ignores ws_bytes); one output line per
// call: status, last byte used, steps per chunk, which caches were used (sign
// words, probe cache, packed weights) and the number of violations.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <vector>

#include "../../include/zo.h"
#include "../../paper_2505_17852_amd/csrc/zo_kernels.hpp"

namespace {

struct Range {
  const char* name;
  const char* p;
  size_t n;
};
char* const kWork = (char*)0x100000000000ull;  // never dereferenced
char* const kTheta = (char*)0x200000000000ull;
size_t ws_bytes, used;
int violations, steps, caches;

void bad(const char* what, const char* a, const char* b = "") {
  if (violations++ < 5) std::fprintf(stderr, "violation: %s %s %s\n", what, a, b);
}
void inside(const Range& r) {
  if (r.p < kWork || r.p + r.n > kWork + ws_bytes) bad("outside the workspace:", r.name);
  else if ((size_t)(r.p - kWork) + r.n > used) used = (size_t)(r.p - kWork) + r.n;
}
void apart(const Range& a, const Range& b) {
  if (a.n && b.n && a.p < b.p + b.n && b.p < a.p + a.n) bad("overlap:", a.name, b.name);
}
// the buffers that live for the whole call, against one another and against r
std::vector<Range> lasting(const zo::ForwardArgs& a) {
  std::vector<Range> v;
  const zo::WsPlan& w = a.ws;
  const size_t M = (size_t)a.rows.M, N = (size_t)a.rows.N, L = (size_t)a.cfg.n_layers, H = (size_t)a.cfg.hidden;
  const size_t V = (size_t)a.cfg.vocab, rows = (size_t)w.T * M, pg = (size_t)a.zmap.pg;
  const bool b16 = a.cfg.wdtype == ZO_WBF16;
  v.push_back({"c", a.work + w.cbuf, L * M * H * 4});
  v.push_back({"zb", a.work + w.zb, L * N * 4 * H * 4});
  v.push_back({"zbo", a.work + w.zbo, N * V * 4});
  v.push_back({"pmax", a.work + w.pmax, (size_t)w.nvt * rows * 4});
  v.push_back({"psum", a.work + w.psum, (size_t)w.nvt * rows * 4});
  v.push_back({"ptgt", a.work + w.ptgt, rows * 4});
  v.push_back({"row_loss", a.work + w.row_loss, M * 8});
  if (a.w16) v.push_back({"w16", (const char*)a.w16, pg * 2});
  if (a.wpack) v.push_back({"wpack", (const char*)a.wpack, pg * 4});
  if (a.bits) v.push_back({"bits", (const char*)a.bits, N * zo::bit_words(a.lay.total) * 4});
  if (a.zc) v.push_back({"zc", (const char*)a.zc, N * pg * (b16 ? 4 : 4)});
  return v;
}
void check_state(const zo::ForwardArgs& a, const Range& r) {
  inside(r);
  for (const Range& q : lasting(a)) apart(r, q);
}
// activations: M rows of K values, t timesteps
Range acts(const zo::ForwardArgs& a, const char* name, const void* p, size_t K, size_t t = 1) {
  return {name, (const char*)p, t * (size_t)a.rows.M * K * zo::act_bytes(a.cfg)};
}
size_t zero_tile(const zo::ForwardArgs& a) { return zo::zero_state_bytes(a.cfg, a.rows.M); }

}  // namespace

// the runtime, as far as the launching code calls it
extern "C" {
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = kWork;
  return hipSuccess;
}
}

namespace zo {
hipError_t launch_debug_probe(int, uint64_t, uint32_t, uint64_t, uint64_t, float*, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_debug_gauss_pairs(const uint32_t*, uint64_t, float*, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_init(int, void*, uint64_t, uint64_t, float, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_update(int, int, void*, uint64_t, uint64_t, float, float, int32_t, uint32_t, const float*, const float*,
                         int32_t*, hipStream_t, int, const uint32_t*) {
  return hipErrorInvalidValue;
}
hipError_t launch_bits_fill(uint32_t*, uint64_t, uint64_t, uint32_t, int32_t, hipStream_t) { return hipSuccess; }

static void begin(const ForwardArgs& a) {
  if (steps) return;
  steps = a.ws.T;
  caches = (a.bits ? 1 : 0) + (a.zc ? 2 : 0) + (a.wpack ? 4 : 0);
  const std::vector<Range> v = lasting(a);
  for (size_t i = 0; i < v.size(); ++i) {
    inside(v[i]);
    for (size_t j = 0; j < i; ++j) apart(v[i], v[j]);
  }
}
hipError_t launch_embed_f32(const ForwardArgs& a, int, int Tc, void* x0, hipStream_t) {
  begin(a);
  check_state(a, acts(a, "x0", x0, (size_t)a.cfg.embed, (size_t)Tc));
  return hipSuccess;
}
hipError_t launch_embed_bf16(const ForwardArgs& a, int, void* x0, hipStream_t) {
  begin(a);
  check_state(a, acts(a, "x0", x0, (size_t)a.cfg.embed));
  return hipSuccess;
}
hipError_t launch_gates_f32(const ForwardArgs& a, const GateLayerF32* ls, int n, hipStream_t) {
  std::vector<Range> reads, writes;
  for (int i = 0; i < n; ++i) {
    const GateLayerF32& g = ls[i];
    reads.push_back(acts(a, "x", g.x, (size_t)g.El));
    reads.push_back(acts(a, "h before", g.hprev, (size_t)a.cfg.hidden));
    if (a.ws.T == 1 && g.hprev == a.work + a.ws.hzero) {
      reads.back().n = zero_tile(a);
      if (n != 1) bad("more than one layer beside the zero tile:", "h before");
    }
    writes.push_back(acts(a, "h", g.hout, (size_t)a.cfg.hidden));
    writes.push_back({"c", (const char*)g.cst, (size_t)a.rows.M * (size_t)a.cfg.hidden * 4});
    inside(writes.back());
    inside({"zb", (const char*)g.zb, (size_t)a.rows.N * 16 * (size_t)a.cfg.hidden});
    check_state(a, writes[writes.size() - 2]);
  }
  for (size_t i = 0; i < writes.size(); ++i) {
    for (const Range& r : reads) apart(writes[i], r);
    for (size_t j = 0; j < i; ++j) apart(writes[i], writes[j]);
  }
  for (const Range& r : reads) check_state(a, r);
  return hipSuccess;
}
hipError_t launch_gate_bf16(const ForwardArgs& a, int l, const void* x, const void* hprev, void* hout, float* cst,
                            const float* zb, hipStream_t) {
  const Range rx = acts(a, "x", x, (size_t)(l == 0 ? a.cfg.embed : a.cfg.hidden));
  const Range rh = acts(a, "h before", hprev, (size_t)a.cfg.hidden);
  const Range wh = acts(a, "h", hout, (size_t)a.cfg.hidden);
  const Range wc{"c", (const char*)cst, (size_t)a.rows.M * (size_t)a.cfg.hidden * 4};
  inside({"zb", (const char*)zb, (size_t)a.rows.N * 16 * (size_t)a.cfg.hidden});
  for (const Range& r : {rx, rh}) {
    check_state(a, r);
    apart(r, wh);
    apart(r, wc);
  }
  check_state(a, wh);
  inside(wc);
  return hipSuccess;
}
static hipError_t head(const ForwardArgs& a, const void* hist, int Tc, const float* pmax, const float* psum,
                       const float* ptgt) {
  check_state(a, acts(a, "states", hist, (size_t)a.cfg.hidden, (size_t)Tc));
  const size_t rows = (size_t)Tc * (size_t)a.rows.M;
  inside({"pmax", (const char*)pmax, (size_t)a.ws.nvt * rows * 4});
  inside({"psum", (const char*)psum, (size_t)a.ws.nvt * rows * 4});
  inside({"ptgt", (const char*)ptgt, rows * 4});
  return hipSuccess;
}
hipError_t launch_head_f32(const ForwardArgs& a, const void* hist, int, int Tc, const float*, float* pmax, float* psum,
                           float* ptgt, hipStream_t) {
  return head(a, hist, Tc, pmax, psum, ptgt);
}
hipError_t launch_head_bf16(const ForwardArgs& a, const void* hist, int, int Tc, const float*, float* pmax, float* psum,
                            float* ptgt, hipStream_t) {
  return head(a, hist, Tc, pmax, psum, ptgt);
}
}  // namespace zo

int main() {
  const int32_t* tok = (const int32_t*)kTheta;
  float* out = (float*)kTheta;
  zo_config c;
  int fd, N, B, C;
  while (std::scanf("%d %d %d %d %d %d %d %d %d %d %zu", &c.n_layers, &c.vocab, &c.embed, &c.hidden, &c.wdtype, &c.probe,
                    &fd, &N, &B, &C, &ws_bytes) == 11) {
    used = 0;
    violations = steps = caches = 0;
    int st;
    if (fd == 2) {
      ws_bytes = (size_t)ZO_NOALLOC_WORKSPACE_BYTES / 2 * 3 + (1u << 16);  // the library's array
      st = zo_perturbed_losses_noalloc(&c, kTheta, 1, 1e-2f, N, 0, tok, nullptr, B, C, out, out, nullptr);
    } else {
      auto f = fd ? zo_fd_losses : zo_perturbed_losses;
      st = f(&c, kTheta, 1, 1e-2f, N, 0, tok, nullptr, B, C, out, out, kWork, ws_bytes, nullptr);
    }
    std::printf("%d %zu %d %d %d\n", st, used, steps, caches, violations);
  }
  return 0;
}
