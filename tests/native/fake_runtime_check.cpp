// Drives the library's host code on a machine without a GPU.  This file defines the HIP functions that the library's objects
// call: memory is address ranges without backing, streams and events are tokens, a launch is written down with its arguments
// and runs nothing.  Like the HIP runtime (7.0 on) it keeps the last error of a failed call until hipGetLastError reads it.
// Every attention launch is checked against the allocations alive: scratch that a kernel would write outside of them fails.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "../../include/tkv.h"
#include "../../paper_2605_09490_amd/csrc/tkv_internal.h"

#define CHECK(cond)                                                                                        \
  do {                                                                                                     \
    if (!(cond)) { std::printf("FAILED %s (line %d)\n", #cond, __LINE__); std::fflush(stdout); std::exit(1); } \
  } while (0)
#define OK(call)                                                                                              \
  do {                                                                                                        \
    tkv_status s_ = (call);                                                                                   \
    if (s_ != TKV_OK) { std::printf("FAILED %s -> %d: %s (line %d)\n", #call, s_, tkv_last_error(c), __LINE__); std::exit(1); } \
  } while (0)

// ---- the runtime ---------------------------------------------------------------------------------------------------
struct Launch { std::string kernel; dim3 grid; tkv::AttnArgs a; hipStream_t st; size_t lds; };
static std::map<const void*, std::string> g_kernels;
static std::map<uintptr_t, size_t> g_mem;           // live device ranges
static uintptr_t g_next = (uintptr_t)1 << 40;
static hipError_t g_last = hipSuccess;
static std::vector<Launch> g_launches;
static std::string g_log;                           // A: device allocation, S: device synchronised, M: memset, L: launch
static int g_allocs = 0, g_fail_at = -1, g_fail_from = 1 << 30, g_cus = 256;
static int g_last_host_alloc = 0;                   // the number of the last pinned one
static size_t g_fail_above = SIZE_MAX, g_fail_size = SIZE_MAX;
static hipStream_t g_capturing = nullptr;
static std::set<hipEvent_t> g_recorded;
static dim3 g_cfg_grid, g_cfg_block;
static size_t g_cfg_lds;
static hipStream_t g_cfg_stream;

static hipError_t err(hipError_t e) { if (e != hipSuccess) g_last = e; return e; }
static void* range(size_t n) { void* p = (void*)g_next; g_mem[g_next] = n; g_next += (n + 511) / 256 * 256; return p; }
static bool inside(const void* p, size_t n) {
  auto it = g_mem.upper_bound((uintptr_t)p);
  if (it == g_mem.begin()) return false;
  --it;
  return (uintptr_t)p + n <= it->first + it->second;
}
static bool refused(size_t n) { const int k = g_allocs++; return k == g_fail_at || k >= g_fail_from || n > g_fail_above || n == g_fail_size; }

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  g_log += 'A';
  if (refused(n)) return err(hipErrorOutOfMemory);
  *p = range(n);
  return hipSuccess;
}
hipError_t hipFree(void* p) { CHECK(g_mem.erase((uintptr_t)p) == 1); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  g_last_host_alloc = g_allocs;
  if (refused(n)) return err(hipErrorOutOfMemory);
  *p = std::calloc(n, 1);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = g_cus; return hipSuccess; }
hipError_t hipDeviceSynchronize() { g_log += 'S'; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* s = range((size_t)16 << 20);
  *p = s;
  return hipSuccess;
}
hipError_t hipMemset(void* p, int, size_t n) { CHECK(inside(p, n)); g_log += 'M'; return hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)std::malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { std::free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) {
  *c = g_capturing && s == g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { g_recorded.erase(e); std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { g_recorded.insert(e); return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {   // 1 ms between a kernel's two events
  if (!g_recorded.count(a) || !g_recorded.count(b)) return err(hipErrorInvalidHandle);
  *ms = 1.f;
  return hipSuccess;
}

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { g_kernels[host] = name; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) { g_cfg_grid = g; g_cfg_block = b; g_cfg_lds = lds; g_cfg_stream = s; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) { *g = g_cfg_grid; *b = g_cfg_block; *lds = g_cfg_lds; *s = g_cfg_stream; return hipSuccess; }

hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t lds, hipStream_t st) {
  Launch l{g_kernels.at(f), grid, {}, st, lds};
  g_log += 'L';
  const auto is = [&](const char* n) { return l.kernel.find(n) != std::string::npos; };
  if (is("k_attn") || is("k_step_scores") || is("k_call_scores")) {
    const tkv::AttnArgs& a = l.a = *(const tkv::AttnArgs*)args[0];
    CHECK(grid.x >= 1 && grid.y >= 1 && grid.y <= 65535 && grid.z >= 1 && grid.z <= 65535);
    const size_t seqs = (size_t)a.nl * a.B * a.n_q * a.cq, G = a.Hq / a.Hkv;
    const size_t D = l.kernel.find("ILi128E") != std::string::npos ? 128 : 64;
    CHECK(a.xs_stride == 0 || a.sc || inside(a.xs, seqs * a.Hq * a.xs_stride * 4));
    // a chunk whose logits are not written keeps its packed query vectors there
    if (a.groups && a.xs_stride == 0) CHECK(inside(a.xs, (size_t)a.B * a.Hkv * ((a.cq * G + 15) / 16) * (D / 32) * 64 * 16));
    if (a.sc) {
      // whole pairs: a row's weights, and the logits beyond the LDS; pairs in parts: their logits and the parts' partials
      const size_t rows = a.whole_rows, split = seqs - rows, first = (size_t)(a.whole_rows * a.Hkv + a.tail0);
      const size_t sc = rows * a.Hkv * a.sc_stride * 4, xs = rows * a.Hq * a.xs_stride * 4, xt = split * a.Hq * a.sc_stride * 4;
      const char *sc0 = (char*)a.sc, *xs0 = (char*)a.xs, *xt0 = (char*)(a.xt + first * G * a.sc_stride);
      CHECK(a.whole_rows >= 0 && rows <= seqs && inside(sc0, sc) && inside(xs0, xs));
      CHECK(xs == 0 || xs0 >= sc0 + sc || xs0 + xs <= sc0);
      if (split > 0) {
        CHECK(a.whole_rows * a.Hkv + a.tail0 >= 0 && a.S >= 2 && a.S <= 8 && inside(xt0, xt));
        CHECK(inside(a.part_ml + first * a.S * 2 * G, split * a.Hkv * a.S * 2 * G * 4) && inside(a.part_o + first * a.S * G * D, split * a.Hkv * a.S * G * D * 4));
        CHECK((xt0 >= sc0 + sc || xt0 + xt <= sc0) && (xs == 0 || xt0 >= xs0 + xs || xt0 + xt <= xs0));
        if (is("k_attn_step")) CHECK(grid.y == rows + split * a.S);
      }
    } else {
      CHECK(inside(a.part_ml, seqs * a.Hkv * a.S_total * 2 * G * 4) && inside(a.part_o, seqs * a.Hkv * a.S_total * G * D * 4));
    }
    g_launches.push_back(l);
  }
  return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, hipStream_t st, hipEvent_t e0, hipEvent_t e1, int) {
  for (hipEvent_t e : {e0, e1}) if (e) g_recorded.insert(e);
  return hipLaunchKernel(f, g, b, args, lds, st);
}
}

// ---- scenarios -------------------------------------------------------------------------------------------------------
static tkv_config config(int L, int B, int Hq, int Hkv, int D, int n) {
  tkv_config cfg;
  std::memset(&cfg, 0, sizeof cfg);
  cfg.n_layers = L; cfg.batch = B; cfg.n_q_heads = Hq; cfg.n_kv_heads = Hkv; cfg.head_dim = D; cfg.max_tokens = n;
  cfg.kv_dtype = TKV_BF16; cfg.staging_rows = 64; cfg.t2_rows = 64; cfg.host_rows = 64; cfg.prefetch_mode = TKV_PREFETCH_LAZY;
  return cfg;
}
static char* const DATA = (char*)0x1000;            // stands for the caller's tensors, never read
static hipStream_t const STREAM = (hipStream_t)0x2000;

static void fill(tkv_cache* c, const tkv_config& cfg, int n) {
  for (int l = 0; l < cfg.n_layers; ++l) OK(tkv_append(c, l, DATA, DATA, n, STREAM));
}
static int count(const char* kernel) {
  int n = 0;
  for (auto& l : g_launches) n += l.kernel.find(kernel) != std::string::npos;
  return n;
}
// one decode step; its attention launches must cover every layer once, in order
static std::vector<Launch> step(tkv_cache* c, const tkv_config& cfg, hipStream_t st = STREAM) {
  g_launches.clear();
  OK(tkv_decode_step(c, DATA, DATA, DATA, DATA, st));
  size_t out = (size_t)DATA;
  std::vector<Launch> attn;
  for (auto& l : g_launches)
    if (l.kernel.find("k_attn_step") != std::string::npos || l.kernel.find("k_attn_tiered") != std::string::npos) {
      CHECK((size_t)l.a.out == out && l.st == st);
      out += (size_t)l.a.nl * cfg.batch * cfg.n_q_heads * cfg.head_dim * 4;
      attn.push_back(l);
    }
  CHECK(out == (size_t)DATA + (size_t)cfg.n_layers * cfg.batch * cfg.n_q_heads * cfg.head_dim * 4);
  CHECK(count("k_attn_step") + count("k_attn_tiered") == count("k_attn_finish") + count("scores"));
  return attn;
}

static const int SHAPES[][6] = {   // layers, sequences, query heads, kv heads, head_dim, max_tokens
    {28, 1, 28, 4, 128, 1500}, {5, 3, 10, 2, 128, 700}, {48, 8, 40, 8, 128, 4200}, {1, 64, 28, 4, 128, 16500}, {70, 1, 6, 2, 64, 100},
    {2, 130, 4, 2, 64, 200}, {12, 1, 40, 8, 128, 70000}, {28, 16, 64, 8, 64, 3000}};

// A refused allocation leaves no error behind for the next launch to report, and a cache that could be created works.
static void refused_allocations() {
  for (auto& s : SHAPES) {
    tkv_config cfg = config(s[0], s[1], s[2], s[3], s[4], s[5]);
    tkv_cache* c = nullptr;
    g_fail_at = -1; g_allocs = 0;
    CHECK(tkv_create(&cfg, &c) == TKV_OK);
    const int total = g_allocs;
    fill(c, cfg, 60);
    g_fail_above = 0;                               // nothing more is to be had
    step(c, cfg);
    CHECK(hipGetLastError() == hipSuccess);
    for (int l = 0; l < cfg.n_layers; ++l) OK(tkv_append(c, l, DATA, DATA, 3, STREAM));
    CHECK(tkv_attend_and_score_chunk(c, 0, DATA, DATA, 3, STREAM) == TKV_ENOMEM);
    OK(tkv_attend_and_score(c, 0, DATA, DATA, STREAM));
    g_fail_above = SIZE_MAX;
    OK(tkv_attend_and_score_chunk(c, 0, DATA, DATA, 3, STREAM));
    tkv_destroy(c);
    for (int k = 0; k < total; ++k) {
      g_fail_at = k; g_allocs = 0;
      const tkv_status st = tkv_create(&cfg, &c);
      g_fail_at = -1;
      CHECK(hipGetLastError() == hipSuccess);
      CHECK((st == TKV_OK) == (c != nullptr) && (st == TKV_OK || st == TKV_ENOMEM));
      if (!c) continue;
      fill(c, cfg, 60);
      step(c, cfg);
      tkv_destroy(c);
    }
    CHECK(g_mem.size() == 1);                       // the library's own array; everything else was given back
  }
}

// Device memory is taken by tkv_create (and by the first chunk) only, and nothing of it is used before the device has been
// synchronised: a block may come from an allocator whose last owner's work is still queued on another stream.
static void allocations_before_use() {
  for (auto& s : SHAPES)
    for (int mode : {TKV_PREFETCH_WAIT, TKV_PREFETCH_LAZY, TKV_PREFETCH_STREAM}) {
      tkv_config cfg = config(s[0], s[1], s[2], s[3], s[4], s[5]);
      cfg.prefetch_mode = mode;
      tkv_cache* c = nullptr;
      g_log.clear();
      CHECK(tkv_create(&cfg, &c) == TKV_OK);
      const size_t used = g_log.find_first_of("LM"), synced = g_log.rfind('S', used);
      CHECK(used != std::string::npos && synced != std::string::npos && g_log.find('A', synced) == std::string::npos);
      fill(c, cfg, 60);
      g_log.clear();
      const auto first = step(c, cfg), second = step(c, cfg);
      CHECK(g_log.find('A') == std::string::npos);
      // a step that is being captured is launched like any other, the first one included
      tkv_cache* d = nullptr;
      CHECK(tkv_create(&cfg, &d) == TKV_OK);
      fill(d, cfg, 60);
      g_capturing = STREAM;
      const auto captured = step(d, cfg);
      g_capturing = nullptr;
      CHECK(captured.size() == first.size() && first.size() == second.size());
      for (size_t i = 0; i < first.size(); ++i) CHECK(captured[i].kernel == first[i].kernel && captured[i].a.nl == first[i].a.nl && captured[i].a.S == first[i].a.S);
      tkv_destroy(c);
      tkv_destroy(d);
    }
}

// The kind of launch that serves a decode step (whole pairs or split ones: two orders of addition) and the splits of a pair
// follow from the cache's shape.  However little memory there is beyond what tkv_create must have, and in whatever prefetch
// mode, only the number of layers per launch may change.
static void route_follows_from_the_shape() {
  for (auto& s : SHAPES) {
    std::string kernel;
    int S = 0, fewest = 1 << 30, most = 0;
    for (int mode : {TKV_PREFETCH_WAIT, TKV_PREFETCH_LAZY})
      for (int from = 1 << 30, total = 0; from > 0; from = from == 1 << 30 ? total - 1 : from - 1) {
        tkv_config cfg = config(s[0], s[1], s[2], s[3], s[4], s[5]);
        cfg.prefetch_mode = mode;
        tkv_cache* c = nullptr;
        g_fail_from = from; g_allocs = 0;
        const tkv_status st = tkv_create(&cfg, &c);
        if (from == 1 << 30) total = g_allocs;
        if (st == TKV_ENOMEM && from < total) break;      // now it is memory that the cache must have
        CHECK(st == TKV_OK);
        fill(c, cfg, 60);
        for (auto& l : step(c, cfg)) {
          if (kernel.empty()) { kernel = l.kernel; S = l.a.S; }
          CHECK(l.kernel == kernel && l.a.S == S);
          fewest = std::min(fewest, l.a.nl); most = std::max(most, l.a.nl);
        }
        tkv_destroy(c);
        g_fail_from = 1 << 30;
      }
    CHECK(most == 1 || fewest < most);                    // the refusals did bite
  }
}

// Pairs in parts: which, and in how many, follows from the shape as well, whatever groups the layers go in.  A cache is created
// with the memory it needs without parts but for their partials: with no more than that its steps go layer by layer.
static const int PARTS[][8] = {   // layers, sequences, query heads, kv heads, head_dim, max_tokens; parts, pairs that go in parts
    {4, 70, 5, 1, 128, 2048, 8, 24}, {4, 70, 5, 1, 128, 1792, 7, 24}, {20, 7, 8, 2, 64, 3072, 6, 24}, {28, 5, 28, 4, 128, 2500, 5, 48},
    {9, 4, 8, 8, 64, 2048, 4, 32}, {28, 3, 28, 4, 128, 2904, 3, 80}, {28, 1, 28, 4, 128, 1500, 2, 112}, {48, 8, 40, 8, 128, 4200, 1, 0}};
static void parts_of_pairs() {
  for (auto& s : PARTS)
    for (int mode : {TKV_PREFETCH_WAIT, TKV_PREFETCH_LAZY}) {
      tkv_config cfg = config(s[0], s[1], s[2], s[3], s[4], s[5]);
      cfg.prefetch_mode = mode;
      const size_t columns = (s[5] + 127) / 64 * 64, G = s[2] / s[3], scratch = (size_t)s[7] * G * (columns + s[6] * (2 + s[4])) * 4;
      int nl[3];                                    // layers of the first launch
      for (int refuse = 0; refuse < 3; ++refuse) {  // nothing, the parts' scratch, everything behind the pinned store
        tkv_cache* c = nullptr;
        g_allocs = 0;
        if (refuse == 1) g_fail_size = scratch;
        if (refuse == 2) g_fail_from = g_last_host_alloc + 1;
        CHECK(tkv_create(&cfg, &c) == TKV_OK);
        CHECK(refuse != 2 || g_allocs > g_fail_from);
        g_fail_from = 1 << 30; g_fail_size = SIZE_MAX;
        fill(c, cfg, 60);
        const auto launches = step(c, cfg);
        int pairs = 0;
        for (auto& l : launches) {
          const int split = (l.a.nl * s[1] - l.a.whole_rows) * s[3];
          CHECK(l.kernel.find("k_attn_step") != std::string::npos);
          CHECK(split == 0 || l.a.S == s[6]);
          CHECK(pairs == 0 || split == l.a.nl * s[1] * s[3]);     // the last ones of the step
          pairs += split;
        }
        CHECK(pairs == s[7]);
        nl[refuse] = launches[0].a.nl;
        tkv_destroy(c);
      }
      CHECK(nl[0] > 1 && nl[1] == (s[7] ? 1 : nl[0]) && nl[2] == 1);
    }
}

// Whole pairs where they fill the chip, their lists are short or a layer has few; with other compute unit counts too.
static void long_lists_fill_the_chip() {
  const struct { int L, Hq, Hkv, n, cus; bool whole; } cases[] = {
      {12, 40, 8, 16400, 256, true}, {12, 40, 8, 33000, 256, false}, {12, 40, 8, 20480, 256, true}, {12, 40, 8, 20481, 256, false},
      {28, 28, 4, 33000, 256, true}, {28, 28, 4, 65600, 256, true}, {28, 28, 4, 131100, 256, false},
      {20, 40, 8, 33000, 256, true}, {33, 32, 8, 33000, 256, false}, {48, 40, 8, 33000, 256, true}, {48, 40, 8, 65600, 256, false},
      {32, 32, 8, 33000, 256, true}, {12, 40, 8, 33000, 128, true}, {32, 32, 8, 33000, 192, true}, {11, 40, 8, 1000, 256, false}};
  for (auto& t : cases) {
    tkv_config cfg = config(t.L, 1, t.Hq, t.Hkv, 128, t.n);
    g_cus = t.cus;
    tkv_cache* c = nullptr;
    CHECK(tkv_create(&cfg, &c) == TKV_OK);
    fill(c, cfg, 60);
    step(c, cfg);
    if ((count("k_attn_step") > 0) != t.whole) std::printf("%d layers, %d/%d heads, %d tokens, %d units\n", t.L, t.Hq, t.Hkv, t.n, t.cus);
    CHECK((count("k_attn_step") > 0) == t.whole);
    tkv_destroy(c);
  }
  g_cus = 256;
}

// A chunk's workgroups leave a partial per query token and head behind, which the second launch merges one by one: no more of
// them than have a tile (8 KB of rows) for each of their eight waves, but for lists of up to eight 64-row tiles, and no more
// than the compute units hold at once.  The second launch is the one that goes with written logits or the one that does
// without, and what it asks of the LDS is there beside its tile buffers.
static void chunk_splits() {
  const struct { int B, Hq, Hkv, D; } shapes[] = {{1, 28, 4, 128}, {8, 28, 4, 128}, {1, 8, 8, 64}, {3, 40, 8, 64}, {64, 28, 4, 128}, {2, 128, 128, 64}, {70, 6, 2, 64}};
  for (auto& t : shapes)
    for (int n : {300, 700, 2000, 9000, 16384})
      for (int m : {2, 3, 4, 5, 9, 16, 17, 32, 33}) {
        tkv_config cfg = config(1, t.B, t.Hq, t.Hkv, t.D, n + m);
        tkv_cache* c = nullptr;
        CHECK(tkv_create(&cfg, &c) == TKV_OK);
        fill(c, cfg, n + m);
        g_launches.clear();
        OK(tkv_attend_and_score_chunk(c, 0, DATA, DATA, m, STREAM));
        const int G = t.Hq / t.Hkv, first = m < 32 ? m : 32, cols = first * G;
        const bool logits = cols <= 32 && first <= 16;
        CHECK(g_launches.size() == (m > 32 ? 4u : 2u) && g_launches[0].kernel.find("k_attn_tiered_mc") != std::string::npos);
        CHECK(g_launches[1].kernel.find(logits ? "k_attn_finish_chunk" : "k_attn_chunk_scores") != std::string::npos);
        const Launch &l = g_launches[0], &l2 = g_launches[1];
        const int rows = 4096 / t.D, tiles = (n + first + rows - 1) / rows, groups = (cols + 31) / 32;
        CHECK(l.a.S == (int)l.grid.x && l.a.cq == first && (int)l.grid.y == t.Hkv && (int)l.grid.z == t.B * groups);
        CHECK(l.a.S == 1 || l.a.S * t.B * t.Hkv * groups <= g_cus);
        CHECK((tiles * rows <= 512 && t.D == 64) || (l.a.S - 1) * 8 < tiles);
        if (!logits) CHECK(l2.lds + (size_t)8 * 2 * 32 * 2 * t.D <= 163840);   // two tiles of 32 rows for each of eight waves
        tkv_destroy(c);
      }
}

// A cache with a pair for every compute unit, few heads a group, head_dim 64 and short lists has its whole-pair launches on the
// vector ALUs, single calls and steps alike; others do not, nor do steps over pairs of several layers.
static void few_heads_on_the_vector_alus() {
  const struct { int L, B, Hq, Hkv, D, n; bool vec; } cases[] = {
      {2, 64, 8, 8, 64, 700, true}, {1, 86, 6, 3, 64, 1024, true}, {1, 86, 6, 3, 64, 1025, false}, {1, 86, 9, 3, 64, 700, false},
      {1, 64, 4, 4, 128, 700, false}, {70, 130, 4, 2, 64, 100, true}, {50, 2, 8, 8, 64, 700, false}};
  for (auto& t : cases) {
    tkv_config cfg = config(t.L, t.B, t.Hq, t.Hkv, t.D, t.n);
    tkv_cache* c = nullptr;
    CHECK(tkv_create(&cfg, &c) == TKV_OK);
    fill(c, cfg, 60);
    for (auto& l : step(c, cfg)) CHECK(l.kernel.find("k_attn_step") != std::string::npos && (l.a.vec != 0) == t.vec && (l.kernel.find("Lb1E") != std::string::npos) == t.vec);
    g_launches.clear();
    OK(tkv_attend_and_score(c, 0, DATA, DATA, STREAM));
    CHECK((g_launches[0].a.vec != 0) == t.vec);
    tkv_destroy(c);
  }
}

// Chunks whose logits are written (up to 32 columns and 16 tokens) go in one launch pair whatever the number of heads; longer
// ones in as many as the score launch's LDS makes of them, each with a sensible share.
static void chunk_tokens_per_launch() {
  const struct { int Hq, Hkv, D, m, launches; } cases[] = {
      {128, 128, 128, 16, 1}, {128, 128, 128, 12, 1}, {128, 128, 128, 20, 2}, {128, 128, 64, 16, 1}, {128, 128, 64, 32, 1},
      {96, 96, 128, 16, 1}, {128, 64, 128, 16, 1}, {28, 4, 128, 32, 1}, {28, 4, 128, 33, 2}, {128, 16, 128, 4, 1}};
  for (auto& t : cases) {
    tkv_config cfg = config(1, 2, t.Hq, t.Hkv, t.D, 400);
    tkv_cache* c = nullptr;
    CHECK(tkv_create(&cfg, &c) == TKV_OK);
    fill(c, cfg, 100);
    g_launches.clear();
    OK(tkv_attend_and_score_chunk(c, 0, DATA, DATA, t.m, STREAM));
    if (count("k_attn_tiered") != t.launches) std::printf("%d/%d heads, head_dim %d, %d tokens: %d launches\n", t.Hq, t.Hkv, t.D, t.m, count("k_attn_tiered"));
    CHECK(count("k_attn_tiered") == t.launches);
    tkv_destroy(c);
  }
}

// Kernel times count what was launched since they were last read: single calls their two launches, a chunk its first.
static void kernel_times() {
  tkv_config cfg = config(2, 2, 28, 4, 128, 400);
  cfg.profile = 1;
  tkv_cache* c = nullptr;
  CHECK(tkv_create(&cfg, &c) == TKV_OK);
  fill(c, cfg, 100);
  tkv_stats st;
  const auto read = [&](double kernel, double finish, double call) {
    OK(tkv_get_stats(c, &st));
    CHECK(st.attn_kernel_ms == kernel && st.attn_finish_ms == finish && st.attn_call_ms == call);
  };
  for (int i = 0; i < 6; ++i) OK(tkv_attend_and_score(c, i & 1, DATA, DATA, STREAM));
  read(6, 6, 6);
  for (int m : {4, 9, 33}) OK(tkv_attend_and_score_chunk(c, 0, DATA, DATA, m, STREAM));   // 33 tokens: 32 and a single call
  read(10, 7, 7);
  tkv_destroy(c);
}

// What a decode step of a cache of the given shape (layers, sequences, query heads, kv heads, head_dim, max_tokens; 16-bit rows) does:
// the pairs that go whole, those in parts and in how many, and the entries of a whole pair whose logits the LDS holds; the same
// of a single call.
static void print_route(char** v) {
  int s[6];
  for (int i = 0; i < 6; ++i) s[i] = std::atoi(v[i]);
  tkv_config cfg = config(s[0], s[1], s[2], s[3], s[4], s[5]);
  tkv_cache* c = nullptr;
  CHECK(tkv_create(&cfg, &c) == TKV_OK);
  fill(c, cfg, 1);
  const auto launches = step(c, cfg);
  int whole = 0, parts = 0, S = 1;
  for (auto& l : launches)
    if (l.a.sc) {
      whole += l.a.whole_rows * s[3];
      parts += (l.a.nl * s[1] - l.a.whole_rows) * s[3];
      if (l.a.whole_rows < l.a.nl * s[1]) S = l.a.S;
    }
  g_launches.clear();
  OK(tkv_attend_and_score(c, 0, DATA, DATA, STREAM));
  std::printf("step %d whole %d in %d parts; call %d whole; lds %d\n", whole, parts, S, g_launches[0].a.sc ? s[1] * s[3] : 0, tkv::attn_step_lds_entries(s[4], s[2] / s[3]));
  tkv_destroy(c);
}

int main(int argc, char** argv) {
  if (argc == 8 && std::string(argv[1]) == "route") { print_route(argv + 2); return 0; }
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "refused_allocations") refused_allocations();
  else if (what == "allocations_before_use") allocations_before_use();
  else if (what == "route_follows_from_the_shape") route_follows_from_the_shape();
  else if (what == "parts_of_pairs") parts_of_pairs();
  else if (what == "few_heads_on_the_vector_alus") few_heads_on_the_vector_alus();
  else if (what == "long_lists_fill_the_chip") long_lists_fill_the_chip();
  else if (what == "chunk_splits") chunk_splits();
  else if (what == "chunk_tokens_per_launch") chunk_tokens_per_launch();
  else if (what == "kernel_times") kernel_times();
  else { std::printf("no scenario %s\n", what.c_str()); return 2; }
  std::printf("%s: ok\n", what.c_str());
  return 0;
}
