// The library's runtime (csrc/runtime.cpp, whole) on the CPU, against a model
// of streams, events and device memory in place of HIP and of the kernels.
//
// Every kernel launch is an operation ordered after what its stream has
// enqueued or waited for and after what the host has waited for.  Nothing
// finishes by itself: an operation is complete only once the host has waited
// for it, so a query answers "not ready" until then, and every wait of the
// host for unfinished work is counted.  Two calls whose operations use one
// workspace block without being ordered are a race; so is any use of a block
// that a captured graph refers to.
#include <cstdio>
#include <cstdlib>
#include <set>

#define __HIP_PLATFORM_AMD__ 1
#define __align__(n)
#define HIP_SYMBOL(x) (&x)
#include "../paper_2301_06763_amd/csrc/runtime.cpp"

namespace {

using Ops = std::set<int>;
struct Stream {
  Ops before;  // operations the next one is ordered after
  bool capturing = false;
};
struct Event {
  Ops marks;
  hipStream_t s = nullptr;
};
struct Mem {
  size_t bytes;
  std::vector<std::pair<int, int>> uses;  // (operation, call)
  bool in_graph = false;
  bool table = false, read = false;  // a table of the plane passes, and one that a launch has read
};
std::map<hipStream_t, Stream> g_streams;
std::map<hipEvent_t, Event> g_events;
std::map<char*, Mem> g_mem;
Ops g_done;            // what the host knows to be complete
char* g_next = (char*)0x100000000;
size_t g_held = 0, g_capacity = ~size_t(0);
int g_ops = 0, g_call = 0, g_races = 0, g_waits = 0, g_streams_made = 0;
int g_fail_at = -1;    // launch number (from now) that fails
int g_mallocs = 0, g_launches = 0;

bool g_ended = false;  // a call that ends a capture
void wait_for(const Ops& o) {
  for (const auto& s : g_streams) g_ended |= s.second.capturing;
  if (!std::includes(g_done.begin(), g_done.end(), o.begin(), o.end())) ++g_waits;
  g_done.insert(o.begin(), o.end());
}
Ops all_ops() {
  Ops o;
  for (int i = 0; i < g_ops; ++i) o.insert(i);
  return o;
}
Mem* block_of(const void* p) {
  auto it = g_mem.upper_bound((char*)p);
  if (it == g_mem.begin()) return nullptr;
  --it;
  return (char*)p < it->first + it->second.bytes ? &it->second : nullptr;
}
void use(const void* p, hipStream_t s, int op) {
  Mem* m = block_of(p);
  if (!m) {
    if (p) return;  // the caller's, or the static scratch
    ++g_races;
    std::printf("null buffer\n");
    return;
  }
  const Stream& st = g_streams[s];
  for (auto [o, call] : m->uses)
    if (call != g_call && !st.before.count(o) && !g_done.count(o)) {
      ++g_races;
      std::printf("race: operation %d of call %d and %d of call %d\n", o, call, op, g_call);
      break;
    }
  if (m->in_graph && !(m->uses.size() && m->uses.back().second == g_call)) {
    ++g_races;
    std::printf("call %d uses a captured graph's block\n", g_call);
  }
  m->uses.push_back({op, g_call});
  if (st.capturing) m->in_graph = true;
}
hipError_t op_on(hipStream_t s, std::initializer_list<const void*> bufs) {
  ++g_launches;
  if (g_fail_at >= 0 && g_fail_at-- == 0) return hipErrorLaunchFailure;
  const int op = g_ops++;
  for (const void* p : bufs) use(p, s, op);
  g_streams[s].before.insert(op);
  return hipSuccess;
}
std::map<std::string, int> g_passes;  // grids per pass
hipError_t grids(const char* pass, const nmc::FieldTable& ft, int n, hipStream_t s) {
  ++g_launches;
  g_passes[pass] += n;
  if (g_fail_at >= 0 && g_fail_at-- == 0) return hipErrorLaunchFailure;
  const int op = g_ops++;
  for (int i = 0; i < n; ++i) use(ft.f[i].A, s, op), use(ft.f[i].B, s, op);
  g_streams[s].before.insert(op);
  return hipSuccess;
}
int g_no_table = 0;
void table(const void* p, size_t bytes, hipStream_t s) {  // a Green table of this size
  Mem* m = block_of(p);
  if (!m || m->bytes < bytes) ++g_no_table, std::printf("table missing or of another size (%zu)\n", bytes);
  else {
    m->read = true;
    if (g_streams[s].capturing) m->in_graph = true;
  }
}
hipError_t build_table(const void* p) {
  if (Mem* m = block_of(p)) m->table = true;
  return hipSuccess;
}
size_t cube(int P, size_t r) { return (size_t)(P / 2 + 1) * (P / 2 + 1) * (P / 2 + 1) * r; }

}  // namespace

// --- HIP ----------------------------------------------------------------------
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  ++g_mallocs;
  if (g_held + n > g_capacity) return hipErrorOutOfMemory;
  g_held += n;
  *p = g_next;
  g_mem[g_next] = Mem{n, {}};
  g_next += (n + 4095) / 4096 * 4096 + 4096;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  wait_for(all_ops());
  auto it = g_mem.find((char*)p);
  if (it == g_mem.end()) std::printf("free of an unknown block\n"), std::abort();
  if (it->second.in_graph) ++g_races, std::printf("a captured graph's block freed\n");
  g_held -= it->second.bytes;
  g_mem.erase(it);
  return hipSuccess;
}
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t)(uintptr_t)(0x1000 + 16 * ++g_streams_made);
  g_streams[*s] = Stream{};
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return g_streams.erase(s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return wait_for(g_streams[s].before), hipSuccess; }
hipError_t hipDeviceSynchronize() { return wait_for(all_ops()), hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  const Ops& m = g_events[e].marks;
  g_streams[s].before.insert(m.begin(), m.end());
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = g_streams[s].capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  static uintptr_t n = 0x900000;
  *e = (hipEvent_t)(n += 16);
  g_events[*e] = Event{};
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  if (!g_events.erase(e)) std::printf("event destroyed twice\n"), std::abort();
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  g_events[e] = Event{g_streams[s].before, s};
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  const Event& v = g_events[e];
  if (g_streams[v.s].capturing) return g_ended = true, hipErrorCapturedEvent;  // even if recorded before
  return std::includes(g_done.begin(), g_done.end(), v.marks.begin(), v.marks.end()) ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t e) { return wait_for(g_events[e].marks), hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { return *t = 0, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error of the model"; }
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { return *p = const_cast<void*>(s), hipSuccess; }
}

// --- kernels --------------------------------------------------------------------
namespace nmc {
void set_next_launch_events(hipEvent_t, hipEvent_t) {}
bool take_next_launch_events() { return false; }
#define PASS(name)                                                                              \
  template <class R>                                                                            \
  hipError_t name(const FieldTable& ft, PassGeom g, Tables<R> t, hipStream_t s) {               \
    if (!t.tw) ++g_no_table;                                                                    \
    return grids(#name, ft, g.nf, s);                                                           \
  }
PASS(launch_fwd_x) PASS(launch_fwd_y) PASS(launch_inv_y) PASS(launch_inv_x) PASS(launch_inv_y_fold)
PASS(launch_inv_x_fold) PASS(launch_fwd_xy) PASS(launch_inv_yx)
template <class R>
hipError_t launch_z(const FieldTable& ft, PassGeom g, Tables<R> t, hipStream_t s) {
  table(t.gz, cube(g.P, sizeof(R)), s);
  table(t.gn, sizeof(R), s);
  return grids("launch_z", ft, g.nf, s);
}
template <class R> bool plane_passes_fit(int P) { return P <= 64; }
#define PLANE(name)                                                                             \
  template <class R>                                                                            \
  hipError_t name(const FieldTable& ft, PlaneGeom g, PlaneTables<R> t, hipStream_t s) {         \
    const int PL = g.plan.C * g.plan.NP;                                                        \
    if (g.nfull) table(t.gp, cube(PL, sizeof(R)), s), table(t.tw, PL * 2 * sizeof(R), s);             \
    if (g.nbox) {                                                                               \
      const int PB = g.joint ? PL / 2 : PL;                                                     \
      table(t.gpb, cube(PB, sizeof(R)), s), table(t.twb, PB * 2 * sizeof(R), s);                      \
    }                                                                                           \
    return grids(#name, ft, g.nfull + g.nbox, s);                                               \
  }
PLANE(launch_plane_x) PLANE(launch_plane_yz) PLANE(launch_plane_ix) PLANE(launch_plane_ix_box)
#define SCALED(name)                                                                            \
  template <class R>                                                                            \
  hipError_t name(const FieldTable& ft, PlaneGeom g, int S, PlaneTables<R> t, hipStream_t s) {  \
    const int P = (S + 1) * scaled_points<R>(g.N);                                              \
    table(t.gp, cube(P, sizeof(R)), s), table(t.tw, P * 2 * sizeof(R), s);                            \
    return grids(#name, ft, g.nfull, s);                                                        \
  }
SCALED(launch_scaled_x) SCALED(launch_scaled_yz) SCALED(launch_scaled_ix)
template <class R>
hipError_t launch_restrict(const R*, const R*, R* out, int, hipStream_t s) { return op_on(s, {out}); }
template <class R>
hipError_t launch_pyramid(const PyramidTable& t, int, int, int, hipStream_t s) { return op_on(s, {t.r[0].pyr}); }
template <class R>
hipError_t launch_restrict_cascade(const PyramidTable& t, int, int, int, hipStream_t s) { return op_on(s, {t.r[0].pyr}); }
template <class R>
hipError_t launch_carry(const CarryTable& t, int, int, int, hipStream_t s) { return op_on(s, {t.r[0].S}); }
template <class R>
hipError_t launch_carry_tri(const CarryTable& t, int, int, int, hipStream_t s) { return op_on(s, {t.r[0].S}); }
template <class R>
hipError_t launch_accel(const R*, R*, int, int, double, hipStream_t s) { return op_on(s, {}); }
template <class R>
hipError_t launch_fft_lines(const void*, void*, int, int, int, const void*, hipStream_t s) { return op_on(s, {}); }
// tables are read by every later call: only their existence and size is modelled
hipError_t launch_green(int, double, const double2*, double*, double*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_green_sums(int, double, const double2*, double*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_round_f32(const double*, float*, size_t, hipStream_t) { return hipSuccess; }
template <class R>
hipError_t launch_green_layout(int, const double*, R*, R*, hipStream_t) { return hipSuccess; }
template <class R>
hipError_t launch_plane_spectrum(int, int, const double*, R* gp, hipStream_t) { return build_table(gp); }
}  // namespace nmc

// --- cases ----------------------------------------------------------------------
namespace {

int g_failed = 0;
#define CHECK(c) \
  do { \
    if (!(c)) ++g_failed, std::printf("line %d: %s\n", __LINE__, #c); \
  } while (0)

char* const kRho = (char*)0x10;       // the caller's arrays, outside the model's memory
char* const kPhi = (char*)(1ull << 40);

hipStream_t stream() {
  hipStream_t s;
  (void)hipStreamCreateWithFlags(&s, 0);
  return s;
}
int solve(nmc_ctx* c, int N, int L, hipStream_t s, unsigned flags = 0, nmc_precision p = NMC_F64) {
  ++g_call;
  return nmc_solve(c, kRho, kPhi, N, L, 0.1, 2, 1.0, p, flags, s);
}
nmc_ctx* context(size_t budget = 0) {
  nmc_ctx* c = nullptr;
  if (g_mem.empty()) {  // nothing is left of earlier contexts
    g_ops = 0;
    g_done.clear();
    g_streams.clear();
  }
  CHECK(nmc_create(&c, 0, budget) == NMC_OK);
  return c;
}
void close(nmc_ctx* c) {
  for (auto& m : g_mem) m.second.in_graph = false;  // the caller's graphs go first
  nmc_destroy(c);
  CHECK(g_mem.empty());
  CHECK(g_races == 0);
  CHECK(g_no_table == 0);
}

// A stream's block grows when the stream's handle names another queue than
// the one whose work still uses it: nobody may get the old block before.
void outgrown_block() {
  nmc_ctx* c = context();
  hipStream_t s = stream();
  CHECK(solve(c, 64, 1, stream()) == NMC_OK);  // tables
  CHECK(solve(c, 64, 2, s) == NMC_OK);
  g_streams[s] = Stream{};                     // destroyed, and given out again
  CHECK(solve(c, 64, 5, s) == NMC_OK);
  CHECK(solve(c, 64, 2, stream()) == NMC_OK);
  close(c);
}

// More streams than the context keeps workspace for: a solve only enqueues,
// whatever the streams are still waiting for.
void many_streams() {
  nmc_ctx* c = context();
  CHECK(solve(c, 64, 2, nullptr) == NMC_OK);  // tables; the null stream's block
  g_waits = 0;
  std::vector<hipStream_t> s;
  for (int i = 0; i < 12; ++i) s.push_back(stream());
  for (int k = 0; k < 36; ++k) CHECK(solve(c, 64, 2, s[k % 12]) == NMC_OK);
  CHECK(solve(c, 64, 2, nullptr) == NMC_OK);
  CHECK(g_waits == 0);
  close(c);
}

// A captured call's workspace and tables are the graph's: nobody else gets the
// block and nothing of it is freed, whatever is solved afterwards.
void captured() {
  for (size_t budget : {size_t(0), size_t(24) << 20}) {
    nmc_ctx* c = context(budget);
    hipStream_t s = stream();
    CHECK(solve(c, 16, 3, s) == NMC_OK);
    (void)hipDeviceSynchronize();
    for (int graph = 0; graph < 2; ++graph) {
      if (graph) CHECK(solve(c, 20, 4, s) == NMC_OK);  // the stream's block grows: the old one is still in use
      g_streams[s].capturing = true;
      CHECK(solve(c, 16, 3, s) == NMC_OK);
      if (budget == 0) {  // the call for callers that cannot allocate
        ++g_call;
        CHECK(nmc_solve_noalloc(c, kRho, kPhi, 16, 3, 0.1, 2, 1.0, NMC_F32, 0, s) == NMC_OK);
      }
      if (budget == 0) CHECK(solve(c, 64, 1, s) == NMC_EDEVICE);  // tables not resident
      g_streams[s].capturing = false;
      CHECK(!g_ended);
    }
    for (int N : {16, 8, 32, 64, 16, 4, 12, 64, 16})
      for (int i = 0; i < 3; ++i) {
        (void)hipDeviceSynchronize();
        CHECK(solve(c, N, N == 64 ? 1 : 3, i ? stream() : s) == NMC_OK);
      }
    close(c);
  }
}

// A launch fails at any point of a solve, also after the second stream has been
// forked: the next solve is not beside what that one left behind.
void failed_launch() {
  struct { int N, L; unsigned flags; } const shapes[] = {{128, 3, 0}, {64, 3, NMC_MODIFIED3}, {256, 2, NMC_MODIFIED}};
  nmc_ctx* c = context();
  for (auto q : shapes) {
    hipStream_t s = stream();
    CHECK(solve(c, q.N, q.L, s, q.flags) == NMC_OK);
    const int before = g_launches;
    CHECK(solve(c, q.N, q.L, s, q.flags) == NMC_OK);
    const int n = g_launches - before;
    for (int k = 0; k < n; ++k) {
      g_fail_at = k;
      CHECK(solve(c, q.N, q.L, s, q.flags) == NMC_EDEVICE);
      CHECK(g_fail_at == -1);
      CHECK(solve(c, q.N, q.L, s, q.flags) == NMC_OK);
    }
  }
  close(c);
}

// The device has room for one large workspace: a call that needs it waits for
// every lease and takes back what is kept for other streams.
void device_full() {
  nmc_ctx* c = context();
  CHECK(solve(c, 64, 5, stream()) == NMC_OK);  // tables
  std::vector<hipStream_t> s;
  for (int i = 0; i < 4; ++i) s.push_back(stream());
  for (int L : {1, 2, 4})  // outgrown blocks: leases; and one kept for each stream
    for (hipStream_t q : s) CHECK(solve(c, 64, L, q) == NMC_OK);
  g_capacity = g_held;
  size_t tables = 0;
  for (const auto& m : g_mem)
    if (m.second.uses.empty()) tables += m.second.bytes;
  size_t ws = 0;
  CHECK(nmc_footprint_bytes(64, 16, NMC_F64, &ws) == NMC_OK);
  CHECK(ws + tables + (4 << 20) < g_capacity);  // it fits, alone
  CHECK(solve(c, 64, 16, stream()) == NMC_OK);
  g_capacity = ~size_t(0);
  close(c);
}

int submit(nmc_ctx* c, int N, int L, hipStream_t s) {
  const nmc_request q{kRho, kPhi, N, L, 0.1, 1.0, NMC_F64, 0};
  uint64_t t;
  ++g_call;
  return nmc_serve_submit(c, &q, s, &t);
}

// Solves beside batches in flight under a budget: the stream's workspace is
// still there, unless the serving arena would get less than it.
void beside_serving() {
  for (bool large : {false, true}) {
    nmc_ctx* c = context((large ? 300 : 800) << 20ull);
    hipStream_t s = stream();
    for (int k = 0; k < 2; ++k) CHECK(solve(c, 64, 6, s) == NMC_OK);  // 140 MB
    CHECK(submit(c, 64, 3, s) == NMC_OK);
    int launched = 0;
    CHECK(nmc_serve_tick(c, &launched) == NMC_OK && launched == 1);
    nmc_serve_stats st;
    CHECK(nmc_serve_stats_get(c, &st) == NMC_OK && st.inflight == 1);
    if (!large) CHECK(solve(c, 64, 6, s) == NMC_OK);
    else CHECK(st.arena_bytes > 250u << 20);
    CHECK(nmc_serve_drain(c) == NMC_OK);
    CHECK(solve(c, 64, 6, s) == NMC_OK);
    close(c);
  }
}

// Requests of one call take the passes that each takes alone, whichever comes
// first (results are bitwise those of the solve alone).
void mixed_batch() {
  nmc_ctx* c = context();
  hipStream_t s = stream();
  for (unsigned method : {0u, (unsigned)NMC_MODIFIED})
    for (int N : {16, 64, 128}) {
      const unsigned flags[2] = {method, method | NMC_NO_FUSED_PLANES};
      g_passes.clear();
      for (unsigned f : flags) CHECK(solve(c, N, 2, s, f) == NMC_OK);
      const auto alone = g_passes;
      for (int first : {0, 1}) {
        nmc_request q[2];
        for (int i = 0; i < 2; ++i) q[i] = {kRho, kPhi, N, 2, 0.1, 1.0, NMC_F64, flags[i ^ first]};
        g_passes.clear();
        ++g_call;
        CHECK(nmc_solve_batch(c, q, 2, s) == NMC_OK);
        CHECK(g_passes == alone);
        uint64_t t;
        g_passes.clear();
        for (auto& r : q) CHECK(nmc_serve_submit(c, &r, s, &t) == NMC_OK);
        ++g_call;
        CHECK(nmc_serve_drain(c) == NMC_OK);
        CHECK(g_passes == alone);
      }
    }
  close(c);
}

// Every size, method and choice of passes finds the tables that its launches
// read, in both precisions, and no plane table is built that none of them reads.
void tables() {
  for (int N = 4; N <= 256; N += 4)
    for (unsigned method : {0u, (unsigned)NMC_MODIFIED, (unsigned)NMC_MODIFIED3})
      for (unsigned f : {method, method | NMC_NO_FUSED_PLANES, method | NMC_NO_RESTRICT}) {
        if (method == NMC_MODIFIED3 && N > 128) continue;
        nmc_ctx* c = context();
        for (nmc_precision p : {NMC_F64, NMC_F32}) CHECK(solve(c, N, 3, nullptr, f, p) == NMC_OK);
        bool all = true;
        for (const auto& m : g_mem) all = all && (!m.second.table || m.second.read);
        // (kept coarse densities: the boxes' tables serve the other meshes of a batch)
        if (!all && !(f & NMC_NO_RESTRICT)) ++g_failed, std::printf("N %d flags %u: a table nobody reads\n", N, f);
        close(c);
      }
}

// nmc_solve_noalloc of a mesh finds its tables after any call that leaves
// those of its periods (P, and 2P and 4P of the modified methods): a solve of
// another size, method, precision or choice of passes, or nmc_green_spectrum.
void noalloc_tables() {
  struct Call { int N; unsigned flags; bool spectrum; };
  const unsigned M = NMC_MODIFIED, M3 = NMC_MODIFIED3, S = NMC_NO_FUSED_PLANES;
  std::vector<Call> calls;
  for (int N : {8, 16, 20, 32, 36, 48, 64, 68, 96, 100, 124, 128, 256}) {
    for (unsigned f : {0u, S, M, M | S, M3, M3 | S})
      if (N <= 128 || !is_modified(f)) calls.push_back({N, f, false});
    calls.push_back({N, 0, true});
  }
  auto periods = [](int N, unsigned f, bool m3) {
    const int P = period_of(N);
    std::set<int> o{P};
    if (is_modified(f)) o.insert(2 * P);
    if (m3) o.insert(4 * P);
    return o;
  };
  int accepted = 0;
  for (const Call& x : calls) {
    nmc_ctx* c = context();
    if (x.spectrum) CHECK(nmc_green_spectrum(c, x.N, NMC_F32, kPhi, nullptr) == NMC_OK);
    else CHECK(solve(c, x.N, 3, nullptr, x.flags) == NMC_OK);
    const auto left = periods(x.N, x.flags, (x.flags & M3) != 0);
    for (const Call& y : calls)
      for (int L : {1, 2, 3})
        for (nmc_precision p : {NMC_F64, NMC_F32}) {
          if (y.spectrum) continue;
          size_t ws = 0;
          if (nmc_footprint_bytes_flags(y.N, L, p, y.flags, &ws) != NMC_OK || ws > NMC_SCRATCH_BYTES) continue;
          const auto need = periods(y.N, y.flags, is_modified3(y.flags, L));
          if (!std::includes(left.begin(), left.end(), need.begin(), need.end())) continue;
          ++g_call;
          ++accepted;
          const int mallocs = g_mallocs;
          if (nmc_solve_noalloc(c, kRho, kPhi, y.N, L, 0.1, 2, 1.0, p, y.flags, nullptr) != NMC_OK)
            ++g_failed, std::printf("after %s %d flags %u: N %d L %d flags %u precision %d refused\n",
                                    x.spectrum ? "spectrum" : "solve", x.N, x.flags, y.N, L, y.flags, (int)p);
          CHECK(mallocs == g_mallocs);
        }
    close(c);
  }
  CHECK(accepted > 500);
}

// A budget of the workspace and of what the tables of the periods took when
// every size of a period shared them (24 bytes a point) is enough, for one size
// after another.
void tight_budget() {
  for (int first : {16, 32, 48, 64, 96, 100, 128, 200, 256})
    for (unsigned f : {0u, (unsigned)NMC_NO_FUSED_PLANES, (unsigned)NMC_MODIFIED, (unsigned)NMC_MODIFIED3}) {
      if (f == NMC_MODIFIED3 && first > 128) continue;
      const int P = period_of(first), other = first == P / 2 ? P / 4 + 4 : P / 2;
      size_t ws = 0, more = 0;
      CHECK(nmc_footprint_bytes_flags(first, 3, NMC_F64, f, &ws) == NMC_OK);
      CHECK(nmc_footprint_bytes_flags(other, 3, NMC_F64, f, &more) == NMC_OK);
      size_t budget = align_up(std::max(ws, more), 2u << 20) + cube(P, 24);
      if (is_modified(f)) budget += cube(2 * P, 24);
      if (f == NMC_MODIFIED3) budget += cube(4 * P, 24);
      nmc_ctx* c = context(budget);
      for (int N : {first, first, other, first}) {
        for (nmc_precision p : {NMC_F64, NMC_F32})
          if (solve(c, N, 3, nullptr, f, p) != NMC_OK) ++g_failed, std::printf("N %d flags %u refused\n", N, f);
        CHECK(g_held <= budget + (8 << 20));  // the twiddles are not counted
      }
      close(c);
    }
}

}  // namespace

int main(int argc, char** argv) {
  const std::map<std::string, void (*)()> cases = {
      {"outgrown_block", outgrown_block}, {"many_streams", many_streams}, {"captured", captured},
      {"failed_launch", failed_launch}, {"device_full", device_full},
      {"beside_serving", beside_serving}, {"mixed_batch", mixed_batch},
      {"tables", tables}, {"tight_budget", tight_budget},
      {"noalloc_tables", noalloc_tables},
  };
  if (argc != 2 || !cases.count(argv[1])) return 2;
  cases.at(argv[1])();
  std::printf("%s: %s\n", argv[1], g_failed ? "FAILED" : "OK");
  return g_failed ? 1 : 0;
}
