// The stage runtime on a simulated device: stage.cpp is compiled into this program as it is, with the HIP calls and the
// kernel launches it makes replaced by a model that keeps a vector clock per stream and remembers which bytes every launch
// reads and writes.  Two accesses to a byte, one of them a write, that no event, stream order or host wait puts in order are
// reported: what a schedule leaves to chance shows here, whatever the kernels' durations are.  No memory is allocated.
//   clang++ -std=c++17 -D__HIP_PLATFORM_AMD__ -I<rocm>/include tests/host/stage_runtime_test.cpp
#include <hip/hip_runtime.h>
#define __device__
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) (&(x))
#include "../../paper_2110_13005_amd/csrc/stage.cpp"

#include <cstdlib>
#include <map>
#include <unordered_map>

#define CHECK(cond)                                                            \
  do {                                                                         \
    if (!(cond)) { std::printf("%s:%d: %s\n", __FILE__, __LINE__, #cond); std::exit(1); } \
  } while (0)

namespace sim {
typedef std::map<int, uint32_t> Clock;                       // stream -> launches of it that are in the past
void merge(Clock& a, const Clock& b) {
  for (const auto& p : b) a[p.first] = std::max(a[p.first], p.second);
}
struct Access { uint64_t lo, hi; int stream; uint32_t time; bool write; const char* what; };
struct Range { const void* p; uint64_t bytes; };

uint64_t next_address = 1 << 20;
int mallocs_until_failure = -1;
std::map<hipStream_t, int> stream_ids;
std::map<int, Clock> clocks;
std::map<hipEvent_t, Clock> events;                          // recorded ones
Clock host;
constexpr uint64_t kPage = 4096;
std::unordered_map<uint64_t, std::vector<Access>> accesses;   // by page
std::vector<std::string> races;
std::map<std::string, int> launches;
std::vector<int> wgrad_segments;                             // microbatches of each weight-gradient launch, in order

int id(hipStream_t s) { return stream_ids.emplace(s, (int)stream_ids.size()).first->second; }
Clock& clock(hipStream_t s) {
  Clock& c = clocks[id(s)];
  merge(c, host);
  return c;
}
void access(hipStream_t s, const char* what, Range r, bool write) {
  if (!r.p || !r.bytes) return;
  const Clock& c = clock(s);
  const int stream = id(s);
  const auto past = [&c](const Access& b) { const auto t = c.find(b.stream); return t != c.end() && b.time <= t->second; };
  const uint64_t lo = (uint64_t)(uintptr_t)r.p, hi = lo + r.bytes;
  for (uint64_t page = lo / kPage; page * kPage < hi; ++page) {
    const Access a = {std::max(lo, page * kPage), std::min(hi, (page + 1) * kPage), stream, c.at(stream), write, what};
    std::vector<Access>& here = accesses[page];
    size_t kept = 0;
    for (const Access& b : here) {
      const bool apart = a.hi <= b.lo || b.hi <= a.lo, before = apart || past(b);
      if (!apart && (write || b.write) && !before && races.size() < 8)
        races.push_back(std::string(b.what) + (b.write ? " (write)" : " (read)") + " and " + what + (write ? " (write)" : " (read)"));
      // who comes after a write, or a read on the same stream, comes after what that covers
      const bool covered = a.lo <= b.lo && b.hi <= a.hi && before && !apart && (write || (!b.write && b.stream == stream));
      if (!covered) here[kept++] = b;
    }
    here.resize(kept);
    here.push_back(a);
  }
}
hipError_t launch(hipStream_t s, const char* what, std::initializer_list<Range> reads, std::initializer_list<Range> writes) {
  ++clock(s)[id(s)];
  ++launches[what];
  for (Range r : reads) access(s, what, r, false);
  for (Range r : writes) access(s, what, r, true);
  return hipSuccess;
}
void forget() {                                              // a fresh start, everything before is in the past
  stream_ids.clear(); clocks.clear(); events.clear(); host.clear();
  accesses.clear(); races.clear(); launches.clear(); wgrad_segments.clear();
}
Range elems(const void* p, int64_t n) { return {p, (uint64_t)n * sizeof(axonn::elem_t)}; }
Range floats(const void* p, int64_t n) { return {p, (uint64_t)n * 4}; }
Range matrix(const void* p, int64_t rows, int64_t cols, int64_t ld) { return elems(p, p ? (rows - 1) * ld + cols : 0); }
}  // namespace sim

// ------------------------------------------------------------------------------------------------------- the HIP calls
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  if (sim::mallocs_until_failure == 0) { sim::mallocs_until_failure = -1; *p = nullptr; return hipErrorOutOfMemory; }
  if (sim::mallocs_until_failure > 0) --sim::mallocs_until_failure;
  *p = (void*)(uintptr_t)sim::next_address;
  sim::next_address += (n + 511) / 256 * 256;
  return hipSuccess;
}
hipError_t hipFree(void*) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void*) { return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "simulated error"; }
hipError_t hipDeviceSynchronize() {
  for (const auto& c : sim::clocks) sim::merge(sim::host, c.second);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) { sim::merge(sim::host, sim::clock(s)); return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) { return hipDeviceSynchronize(); }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return hipMalloc((void**)s, 1); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return hipMalloc((void**)e, 1); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { sim::events.erase(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { sim::events[e] = sim::clock(s); ++sim::launches["event record"]; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  if (sim::events.count(e)) sim::merge(sim::clock(s), sim::events[e]);
  ++sim::launches["event wait"];
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) { if (sim::events.count(e)) sim::merge(sim::host, sim::events[e]); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { return hipEventQuery(e); }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t s) {
  return sim::launch(s, "copy", {{src, n}}, {{dst, n}});
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t*, const void*) { return hipErrorInvalidValue; }
hipError_t hipMemGetAddressRange(hipDeviceptr_t*, size_t*, hipDeviceptr_t) { return hipErrorInvalidValue; }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidValue; }
}

// ------------------------------------------------------------------------------------------------ the kernel launchers
namespace axonn {
using namespace sim;
static void gemm_accesses(const char* what, bool a_kc, bool b_kc, int epi, const GemmArgs& g, hipStream_t s) {
  (void)launch(s, what, {}, {});
  for (int i = 0; i < g.n_seg; ++i) {
    sim::access(s, what, a_kc ? matrix(g.A_seg[i], g.M, g.K, g.lda) : matrix(g.A_seg[i], g.K, g.M, g.lda), false);
    sim::access(s, what, b_kc ? matrix(g.B_seg[i], g.N, g.K, g.ldb) : matrix(g.B_seg[i], g.K, g.N, g.ldb), false);
  }
  const bool f32 = epi == EPI_ACC_F32;
  sim::access(s, what, elems(g.bias, g.N), false);
  sim::access(s, what, matrix(g.res, g.M, g.N, g.ld_res), false);
  sim::access(s, what, matrix(g.aux, g.M, g.N, g.ld_aux), epi == EPI_BIAS_GELU);
  // one row at a time: the columns between the rows of a part of a matrix belong to somebody else
  if (g.ldc == g.N) sim::access(s, what, f32 ? floats(g.C, (int64_t)g.M * g.N) : elems(g.C, (int64_t)g.M * g.N), true);
  else
    for (int64_t r = 0; r < g.M; ++r) sim::access(s, what, elems((elem_t*)g.C + r * g.ldc, g.N), true);
  sim::access(s, what, f32 ? floats(g.colsum, g.N) : elems(g.colsum, g.N), true);
  sim::access(s, what, floats(g.colsum_ws, (int64_t)((g.K + 63) / 64) * g.N), true);
  sim::access(s, what, floats(g.split_ws, g.split_floats), true);
}
hipError_t launch_gemm(bool a_kc, bool b_kc, int epi, const GemmArgs& g, hipStream_t s) {
  gemm_accesses(a_kc ? (b_kc ? "input gradient" : "forward gemm") : "head weight gradient", a_kc, b_kc, epi, g, s);
  return hipSuccess;
}
hipError_t launch_wgrad_group(int epi, GemmGroup& grp, hipStream_t s) {
  wgrad_segments.push_back(grp.g[0].n_seg);
  for (int i = 0; i < grp.n; ++i) gemm_accesses("weight gradients", false, false, epi, grp.g[i], s);
  return hipSuccess;
}
int64_t gemm_split_ws_floats(int64_t, int64_t, int64_t) { return 0; }
bool set_gemm_tuning(int, int64_t) { return false; }
hipError_t launch_layernorm_fwd(int64_t T, int64_t h, const void* x, const void* gamma, const void* beta, float, void* out,
                                void* out_lo, float* stats, hipStream_t s) {
  return launch(s, "layernorm", {elems(x, T * h), elems(gamma, h), elems(beta, h)},
                {elems(out, T * h), elems(out_lo, out_lo ? T * h : 0), floats(stats, 2 * T)});
}
int layernorm_bwd_slices(int64_t T, int64_t) { return (int)std::min<int64_t>(256, (T + 3) / 4); }
hipError_t launch_layernorm_bwd_partial(int64_t T, int64_t h, const void* dout, const void* x, const float* stats, const void* gamma,
                                        const void* res, void* dx, float* partial, int slices, bool, hipStream_t s) {
  return launch(s, "layernorm backward", {elems(dout, T * h), elems(x, T * h), floats(stats, 2 * T), elems(gamma, h), elems(res, res ? T * h : 0)},
                {elems(dx, T * h), floats(partial, 2 * h * slices)});
}
static hipError_t param_grads(int slices, int64_t h, const float* partial, void* dgamma, void* dbeta, bool f32, hipStream_t s) {
  return launch(s, "layernorm sums", {floats(partial, 2 * h * slices)}, {f32 ? floats(dgamma, h) : elems(dgamma, h), f32 ? floats(dbeta, h) : elems(dbeta, h)});
}
hipError_t launch_layernorm_param_grads(int slices, int64_t h, const float* partial, void* dgamma, void* dbeta, bool f32, hipStream_t s) {
  return param_grads(slices, h, partial, dgamma, dbeta, f32, s);
}
hipError_t launch_layernorm_param_grads_all(int slices, int64_t h, int n_layers, const float* partial, void* dgamma,
                                            int64_t layer_stride, int64_t second, hipStream_t s) {
  for (int i = 0; i < 2 * n_layers; ++i) {
    elem_t* const g = (elem_t*)dgamma + i / 2 * layer_stride + i % 2 * second;
    (void)param_grads(slices, h, partial + (int64_t)i * 2 * h * slices, g, g + h, false, s);
  }
  return hipSuccess;
}
hipError_t launch_layernorm_bwd(int64_t, int64_t, const void*, const void*, const float*, const void*, const void*, void*, void*,
                                void*, int, bool, float*, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_colsum(int64_t, int64_t, const void*, int64_t, void*, int, bool, float*, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_copies(int n, uint64_t bytes, const Copies& c, hipStream_t s) {
  (void)launch(s, "copies", {}, {});
  for (int i = 0; i < n; ++i) { sim::access(s, "copies", {c.src[i], bytes}, false); sim::access(s, "copies", {c.dst[i], bytes}, true); }
  return hipSuccess;
}
hipError_t launch_f32_to_elem(uint64_t n, const float* src, void* dst, hipStream_t s) {
  return launch(s, "rounding", {floats(src, n)}, {elems(dst, n)});
}
hipError_t launch_fill_elem(uint64_t n, void* dst, float, hipStream_t s) { return launch(s, "fill", {}, {elems(dst, n)}); }
hipError_t launch_count_nonfinite(uint64_t n, const void* x, uint64_t* ws, hipStream_t s) {
  return launch(s, "count", {elems(x, n)}, {{ws, 8}});
}
hipError_t launch_attention_fwd(int b, int s, int a, int d, const void* qkv, void* o, float* lse, hipStream_t st) {
  const int64_t n = (int64_t)b * s * a;
  return launch(st, "attention", {elems(qkv, 3 * n * d)}, {elems(o, n * d), floats(lse, n)});
}
hipError_t launch_attention_bwd(int b, int s, int a, int d, const void* qkv, const void* o, const float* lse, const void* dout,
                                void* dqkv, float* delta, hipStream_t st, int) {
  const int64_t n = (int64_t)b * s * a;
  return launch(st, "attention backward", {elems(qkv, 3 * n * d), elems(o, n * d), floats(lse, n), elems(dout, n * d)},
                {elems(dqkv, 3 * n * d), floats(delta, n)});
}
hipError_t launch_embed_fwd(int T, int h, int s, int vocab, const int* tokens, const void* wte, const void* wpe, void* x, hipStream_t st) {
  return launch(st, "embedding", {{tokens, (uint64_t)T * 4}, elems(wte, (int64_t)vocab * h), elems(wpe, (int64_t)s * h)}, {elems(x, (int64_t)T * h)});
}
hipError_t launch_embed_bwd(int b, int s, int h, int vocab, const int* tokens, const void* dx, void* dwte, void* dwpe, int, hipStream_t st) {
  return launch(st, "embedding backward", {{tokens, (uint64_t)b * s * 4}, elems(dx, (int64_t)b * s * h)},
                {elems(dwte, (int64_t)vocab * h), elems(dwpe, (int64_t)s * h)});
}
hipError_t launch_xent(int T, int V, void* logits, const int* targets, int, float, float* token_loss, float* loss, hipStream_t st) {
  return launch(st, "cross-entropy", {{targets, (uint64_t)T * 4}}, {elems(logits, (int64_t)T * V), floats(token_loss, T), floats(loss, 1)});
}
hipError_t launch_adam(uint64_t, float*, float*, float*, const void*, void*, double, double, double, double, double, int64_t, double,
                       hipStream_t) { return hipSuccess; }
hipError_t launch_adam_host(uint64_t, float*, float*, float*, const void*, void*, double, double, double, double, double, int64_t,
                            double, hipStream_t) { return hipSuccess; }
}  // namespace axonn

namespace {
struct Shape { int layers, h, heads, f, s, b, M, limit, group, stride, accum, vocab; bool embed, head; };
void* device(uint64_t bytes) { void* p; CHECK(hipMalloc(&p, bytes) == hipSuccess); return p; }
hipStream_t stream() { return (hipStream_t)device(1); }
hipEvent_t event() { return (hipEvent_t)device(1); }

// A stage with what its user holds: buffers for every microbatch, and streams of the user's own.
struct Program {
  Shape c;
  axonn_stage_t* st = nullptr;
  axonn_embed_t* embed = nullptr;
  axonn_head_t* head = nullptr;
  std::vector<void*> x, y, dy, dx, targets, loss;
  std::vector<hipEvent_t> done;

  explicit Program(const Shape& shape) : c(shape) {
    forget();
    axonn_stage_config cfg;
    memset(&cfg, 0, sizeof cfg);
    cfg.n_layers = c.layers; cfg.hidden = c.h; cfg.n_heads = c.heads; cfg.ffn_hidden = c.f; cfg.seq_len = c.s;
    cfg.microbatch_size = c.b; cfg.n_microbatches = c.M; cfg.pipeline_limit = c.limit; cfg.ln_eps = 1e-5f;
    cfg.wgrad_group = c.group; cfg.ckpt_stride = c.stride; cfg.grad_accum_fp32 = c.accum;
    CHECK(axonn_stage_create(&cfg, &st) == AXONN_OK);
    if (c.embed) CHECK(axonn_embed_create(0, c.vocab, c.h, c.s, c.b, &embed) == AXONN_OK);
    if (c.head) CHECK(axonn_head_create(0, c.vocab, c.h, c.b * c.s, c.M, 1e-5f, &head) == AXONN_OK);
    if (embed || head) CHECK(axonn_stage_attach_ends(st, embed, head) == AXONN_OK);
    new_buffers();
    forget();
  }
  ~Program() {
    axonn_stage_destroy(st);
    if (head) axonn_head_destroy(head);
    if (embed) axonn_embed_destroy(embed);
  }
  void new_buffers() {
    const uint64_t act = (uint64_t)c.b * c.s * c.h * 2, ids = (uint64_t)c.b * c.s * 4;
    for (auto* v : {&x, &y, &dy, &dx, &targets, &loss}) v->assign(c.M, nullptr);
    done.assign(c.M * 2, nullptr);
    for (int i = 0; i < c.M; ++i) {
      x[i] = device(c.embed ? ids : act); y[i] = device(act); dy[i] = device(act); dx[i] = device(act);
      targets[i] = device(ids); loss[i] = device(4);
      done[2 * i] = event(); done[2 * i + 1] = event();
    }
  }
  void post(int kind, int i, bool with_event = false) {
    axonn_msg m;
    memset(&m, 0, sizeof m);
    m.kind = kind; m.mb_id = i;
    m.payload_dev = kind == 0 ? x[i] : dy[i];
    m.result_dev = c.head ? (c.embed ? nullptr : dx[i]) : kind == 0 ? y[i] : c.embed ? nullptr : dx[i];
    if (c.head) { m.targets_dev = targets[i]; m.loss_dev = loss[i]; }
    if (with_event) m.done_event = done[2 * i + kind];
    CHECK(axonn_stage_post(st, &m) == AXONN_OK);
  }
  // a middle stage's order: `limit` forwards, then a backward and a forward in turn; a last stage's: its forwards
  void post_batch(bool with_events = false) {
    for (int i = 0; i < c.M; ++i)
      if (c.head || i < c.limit) post(0, i, with_events);
    for (int i = 0; !c.head && i < c.M; ++i) {
      post(1, i, with_events);
      if (c.limit + i < c.M) post(0, c.limit + i, with_events);
    }
  }
  // everything the batch has written, read on `s`
  void read_results(hipStream_t s) {
    (void)launch(s, "user", {}, {});
    const int64_t act = (int64_t)c.b * c.s * c.h;
    for (int i = 0; i < c.M; ++i) {
      if (c.head) sim::access(s, "user", floats(loss[i], 1), false);
      else sim::access(s, "user", elems(y[i], act), false);
      if (!c.embed) sim::access(s, "user", elems(dx[i], act), false);
    }
    sim::access(s, "user", elems(st->grads, st->n_params), false);
    if (embed) sim::access(s, "user", elems(embed->grads, embed->n_params), false);
    if (head) sim::access(s, "user", elems(head->grads, head->n_params), false);
  }
  std::vector<int> log() {
    std::vector<int32_t> out(4096);
    int32_t n = 0;
    CHECK(axonn_stage_dispatch_log(st, out.data(), 4096, &n) == AXONN_OK);
    return std::vector<int>(out.begin(), out.begin() + n);
  }
};

void expect_ordered(const Shape& c, int n_streams, const char* how) {
  for (const std::string& r : races)
    std::printf("layers %d h %d f %d s %d b %d M %d limit %d group %d stride %d fp32 %d embed %d head %d, %d streams, %s: not ordered: %s\n",
                c.layers, c.h, c.f, c.s, c.b, c.M, c.limit, c.group, c.stride, c.accum, c.embed, c.head, n_streams, how, r.c_str());
  CHECK(races.empty());
}

// Weight-gradient passes close after the same microbatches whether these come one by one or several at a time.
void test_weight_gradient_groups() {
  const auto segments = [](int M, int limit, int group, int n_streams, bool events) {
    Program p({1, 256, 4, 1024, 64, 1, M, limit, group, 0, 0, 0, false, false});
    hipStream_t u = stream();
    CHECK(axonn_stage_zero_grad(p.st, u) == AXONN_OK);
    p.post_batch(events);
    CHECK(axonn_stage_run(p.st, n_streams, u) == AXONN_OK && axonn_stage_join(p.st, u) == AXONN_OK);
    p.read_results(u);
    expect_ordered(p.c, n_streams, "groups");
    CHECK(events ? launches["layernorm"] == 2 * M : launches["layernorm"] < 2 * M);        // two of each pass over the layer
    return wgrad_segments;
  };
  for (int n_streams = 1; n_streams <= 3; ++n_streams) {
    CHECK((segments(8, 8, 3, n_streams, false) == std::vector<int>{3, 3, 2}));
    // where slots run out a forward closes a group: here after each of the first five
    CHECK((segments(8, 3, 0, n_streams, false) == std::vector<int>{1, 1, 1, 1, 1, 3}));
    for (int M = 2; M <= 9; ++M)
      for (int limit = 2; limit <= M; ++limit)
        for (int group = 0; group <= 4; ++group)
          CHECK(segments(M, limit, group, n_streams, false) == segments(M, limit, group, n_streams, true));
  }

  // a batch cut short is accepted or refused by what a run one by one leaves pending
  for (int limit = 1; limit <= 4; ++limit)
    for (int group = 0; group <= 3; ++group)
      for (int cut = 1; cut < 8; ++cut)
        for (int n_streams = 1; n_streams <= 2; ++n_streams) {
          int status[2];
          for (bool events : {false, true}) {
            Program p({1, 256, 4, 1024, 64, 1, 8, limit, group, 0, 0, 0, false, false});
            hipStream_t u = stream();
            CHECK(axonn_stage_zero_grad(p.st, u) == AXONN_OK);
            for (int i = 0; i < std::min(limit, cut); ++i) p.post(0, i, events);
            for (int i = 0; i < cut; ++i) {
              p.post(1, i, events);
              if (limit + i < cut) p.post(0, limit + i, events);
            }
            int32_t n = 0, left = 0;
            CHECK(axonn_stage_poll(p.st, n_streams, u, &n, &left) == AXONN_OK && n == 2 * cut);
            uint64_t bad = 0;
            status[events] = axonn_stage_count_nonfinite_grads(p.st, u, &bad);
            expect_ordered(p.c, n_streams, "cut short");
          }
          if (status[0] != status[1]) std::printf("limit %d group %d cut %d: %d, one by one %d\n", limit, group, cut, status[0], status[1]);
          CHECK(status[0] == status[1]);
        }
  // a batch cut short at a multiple of the group: no weight gradients are pending, and the optimizer's calls accept it
  for (int n_streams = 1; n_streams <= 3; ++n_streams) {
    Program p({1, 256, 4, 1024, 64, 1, 8, 4, 3, 0, 0, 0, false, false});
    hipStream_t u = stream();
    CHECK(axonn_stage_zero_grad(p.st, u) == AXONN_OK);
    for (int i = 0; i < 6; ++i) { p.post(0, i); p.post(1, i); }
    int32_t n = 0, left = 0;
    CHECK(axonn_stage_poll(p.st, n_streams, u, &n, &left) == AXONN_OK && n == 12 && left == 4);
    uint64_t bad = 0;
    CHECK(axonn_stage_count_nonfinite_grads(p.st, u, &bad) == AXONN_OK);
    expect_ordered(p.c, n_streams, "cut short");
  }
}

// Nothing a batch reads or writes is left to chance, nor what its user reads behind the join; two batches, so that every
// slot is used again.  `apart`: the second batch gets buffers and streams of its own, in no order with the first one's; what
// the stage itself holds is in order all the same.
void test_order_of_accesses() {
  for (int ends = 0; ends < 4; ++ends)
    for (int M : {1, 2, 3, 5})
      for (int limit : {1, 2, 3, 4, 5})
        for (int group : {0, 1, 3})
          for (int mode = 0; mode < 3 && limit <= M; ++mode)           // 16-bit, fp32 sums, checkpointing
            for (int n_streams = 1; n_streams <= 3; ++n_streams)
              for (int how = 0; how < 4; ++how) {
                const bool events = how & 1, apart = how & 2;
                Program p({2, 64, 2, 256, 16, 1, M, limit, group, mode == 2 ? 1 : 0, mode == 1, 512, ends % 2 == 1, ends >= 2});
                hipStream_t u = stream();
                for (int batch = 0; batch < 2; ++batch) {
                  CHECK(axonn_stage_zero_grad(p.st, u) == AXONN_OK);
                  if (apart) { p.new_buffers(); u = stream(); }
                  p.post_batch(events);
                  CHECK(axonn_stage_run(p.st, n_streams, u) == AXONN_OK && axonn_stage_join(p.st, u) == AXONN_OK);
                  if (!apart) p.read_results(u);
                }
                expect_ordered(p.c, n_streams, events ? "done events" : apart ? "merged, two users" : "merged");
              }
}

// A batch given up with weight gradients pending: the next one's forwards take the slots behind its chains, whatever streams
// its caller uses.
void test_dropped_microbatches() {
  for (int n_streams = 1; n_streams <= 3; ++n_streams)
    for (bool events : {false, true}) {
      Program p({2, 64, 2, 256, 16, 1, 5, 3, 0, 0, 0, 0, false, false});
      hipStream_t u = stream();
      CHECK(axonn_stage_zero_grad(p.st, u) == AXONN_OK);
      for (int i = 0; i < 2; ++i) { p.post(0, i, events); p.post(1, i, events); }
      int32_t n = 0, left = 0;
      CHECK(axonn_stage_poll(p.st, n_streams, u, &n, &left) == AXONN_OK && n == 4);
      CHECK(axonn_stage_zero_grad(p.st, u) == AXONN_OK);
      p.new_buffers();
      u = stream();
      p.post_batch(events);
      CHECK(axonn_stage_run(p.st, n_streams, u) == AXONN_OK && axonn_stage_join(p.st, u) == AXONN_OK);
      expect_ordered(p.c, n_streams, "given up");
    }
}

// How many passes the microbatches of a batch make, forward and backward.
void test_passes() {
  const auto passes = [](int s, int M, int limit, int group, int n_streams, bool events) {
    Program p({1, 256, 4, 1024, s, 1, M, limit, group, 0, 0, 0, false, false});
    hipStream_t u = stream();
    CHECK(axonn_stage_zero_grad(p.st, u) == AXONN_OK);
    p.post_batch(events);
    CHECK(axonn_stage_run(p.st, n_streams, u) == AXONN_OK && axonn_stage_join(p.st, u) == AXONN_OK);
    CHECK((int)p.log().size() == 2 * M);
    return std::make_pair(launches["attention"], launches["attention backward"]);
  };
  typedef std::pair<int, int> Passes;
  for (int n_streams = 1; n_streams <= 3; ++n_streams) {
    CHECK(passes(64, 8, 8, 0, n_streams, false) == Passes(1, 1) && passes(64, 8, 8, 0, n_streams, true) == Passes(8, 8));
    CHECK(passes(64, 8, 4, 0, n_streams, false) == Passes(2, 2) && passes(64, 4, 2, 0, n_streams, false) == Passes(2, 2));
    // two slots: together on one stream, on several only small ones
    CHECK(passes(512, 3, 2, 0, n_streams, false) == Passes(2, 2) && passes(4096, 4, 2, 1, n_streams, false) == Passes(2, 2));
    CHECK(passes(576, 3, 2, 0, n_streams, false) == (n_streams == 1 ? Passes(2, 2) : Passes(3, 3)));
    CHECK(passes(4160, 4, 2, 1, n_streams, false) == (n_streams == 1 ? Passes(2, 2) : Passes(4, 4)));
  }
}

// attach_ends after an allocation of it has failed: the next call makes what is missing.
void test_attach_after_failed_allocation() {
  for (int stride : {0, 1})
    for (int fails = 0; fails < 4; ++fails) {
      Program p({2, 64, 2, 256, 16, 1, 2, 2, 0, stride, 0, 512, false, false});
      CHECK(axonn_embed_create(0, 512, 64, 16, 1, &p.embed) == AXONN_OK && axonn_head_create(0, 512, 64, 16, 2, 1e-5f, &p.head) == AXONN_OK);
      mallocs_until_failure = fails;
      const int needed = stride ? 3 : 2;                     // one for the embedding, one or two for the head
      CHECK((axonn_stage_attach_ends(p.st, p.embed, p.head) == AXONN_OK) == (fails >= needed));
      mallocs_until_failure = -1;
      CHECK(axonn_stage_attach_ends(p.st, p.embed, p.head) == AXONN_OK);
      CHECK(p.st->embed_dx && p.st->head_y_base && (p.st->head_dx != nullptr) == (stride > 0));
      for (const Slot& slot : p.st->slots) CHECK(slot.head_y);
    }
}
}  // namespace

int main() {
  test_order_of_accesses();
  test_weight_gradient_groups();
  test_dropped_microbatches();
  test_passes();
  test_attach_after_failed_allocation();
  std::puts("stage runtime: all checks passed");
  return 0;
}
