// The host layer's launch sequence with recording stand-ins for the runtime and
// the kernels' launchers (no GPU, no memory behind the pointers): every tile
// table of a search lies inside the workspace, apart from the moments and the
// grids, whatever the granularity of the table, the curves per wave and the
// periods it covers, on one stream and with the waves overlapped on two.
// Tables in use on different streams are apart from each other.
#include <cstdint>

#include "../../paper_0901_1913_amd/csrc/host.hip"

// ---- the runtime -------------------------------------------------------------
namespace {
uintptr_t g_next = (uintptr_t)1 << 40;
void* fake() { return (void*)(g_next += 4096); }
}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  *p = (void*)(g_next += 4096);
  g_next += (n + 4095) & ~(size_t)4095;
  return hipSuccess;
}
hipError_t hipFree(void*) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = fake();
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t)fake();
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t)fake();
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}

// ---- the launchers -----------------------------------------------------------
struct Use {  // bytes a launch reads or writes
  const char* what;
  uintptr_t lo, hi;
  hipStream_t st;
};
static std::vector<Use> g_tables, g_rest;
static int g_ls = 5;          // granularity the spreading takes
static size_t g_elem = 0;

static void use(std::vector<Use>& v, const char* what, const void* p, size_t n, hipStream_t st) {
  v.push_back(Use{what, (uintptr_t)p, (uintptr_t)p + n, st});
}

namespace fchi2 {
size_t tile_bounds_bytes(const Geom& g, int log_tile, int n) {
  return sizeof(int32_t) * (size_t)n * (size_t)(2 * g.H) * (size_t)((g.L >> log_tile) * g.laps + 2);
}
int spread_table_log(const Geom&, int, int64_t, int64_t) { return g_ls; }
int persist_table_log() { return 7; }
hipError_t persist_occupancy(int, int* n) {
  *n = 0;  // staged searches only
  return hipSuccess;
}
hipError_t launch_moments(const double*, const double*, const double*, const int64_t*, int n, int bpc,
                          const Geom&, MomPart* part, Moments* mom, double*, hipStream_t st, bool,
                          const double*) {
  use(g_rest, "moments", mom, sizeof(Moments) * (size_t)n, st);
  use(g_rest, "partial moments", part, sizeof(MomPart) * (size_t)n * bpc, st);
  return hipSuccess;
}
hipError_t launch_tile_bounds(const double*, const Moments*, const Geom& g, int, int n, int64_t, int32_t* tb,
                              int log_tile, hipStream_t st) {
  use(g_tables, "table", tb, tile_bounds_bytes(g, log_tile, n), st);
  return hipSuccess;
}
hipError_t launch_spread(bool, const double*, const double*, const double*, const Moments*, const Geom& g, int,
                         int n, int64_t, int32_t* tb, int ls, void* grid, hipStream_t st, bool share) {
  use(g_tables, "table", tb, tile_bounds_bytes(g, ls, share ? 1 : n), st);
  use(g_rest, "spread grids", grid, (size_t)n * g.P * (size_t)g.L * g_elem, st);
  return hipSuccess;
}
hipError_t launch_fft_pass(bool, const FftPassArgs& a, int, int, const void* in, void* out, const Moments*,
                           const Geom& g, const void*, int n, int64_t, hipStream_t st) {
  if (!a.fused) use(g_rest, "pass input", in, (size_t)n * g.P * (size_t)g.L * g_elem, st);
  if (a.kind == PASS_FIRST || a.kind == PASS_MID)
    use(g_rest, "pass output", out, (size_t)n * g.P * (size_t)g.L * g_elem, st);
  else
    use(g_rest, "spectra", a.zc, (size_t)n * g.P * 2 * (size_t)g.n_freq * g_elem, st);
  return hipSuccess;
}
hipError_t launch_pass2_tw(const void*, int, int, void*, void*, hipStream_t) { return hipSuccess; }
hipError_t launch_deconv_init(void*, const Geom&, const double*, const double*, int, hipStream_t) {
  return hipSuccess;
}
hipError_t launch_solve(bool, const void*, const void*, const Moments*, const Geom&, int, int, double, void*,
                        uint8_t*, hipStream_t, void*, bool) { return hipSuccess; }
hipError_t launch_solve_multi(bool, const void*, const void*, const void*, const Moments*, const Moments*,
                              const double*, const Geom&, int, int, double, void*, uint8_t*, hipStream_t) {
  return hipSuccess;
}
hipError_t launch_persistent(const PersistArgs&, int, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_fine(const double*, const double*, const double*, const Moments*, int, int, int64_t,
                       const double*, int, int, double, double*, int, const FineOut&, hipStream_t) {
  return hipErrorInvalidValue;
}
size_t fine_part_bytes(int, int, int64_t, int, int) { return 0; }
hipError_t launch_peaks(bool, const void*, int64_t, int, int, int, int64_t, int, void*, int64_t*, hipStream_t) {
  return hipErrorInvalidValue;
}
size_t peaks_scratch_bytes(int64_t, int, int) { return 0; }
hipError_t launch_gather(bool, const double*, const Moments*, const Geom&, int, int, const void*, double*,
                         double*, int64_t, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_detrend(const double*, const double*, const double*, const int64_t*, int, int, int64_t,
                          double*, double*, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_finalize(const double*, const double*, const Moments*, const Geom&, int, int, const double*,
                           int, const double*, const double*, double*, double*, double*, int, hipStream_t) {
  return hipErrorInvalidValue;
}
hipError_t launch_adjoint_solve(bool, const void*, const void*, const Moments*, const Geom&, int, int, double,
                                const void*, void*, double*, int, hipStream_t) { return hipErrorInvalidValue; }
size_t top_scratch_bytes(int64_t, int, int, int) { return 256; }
TopScratch top_scratch_carve(void*, int64_t, int, int, int) { return TopScratch{}; }
hipError_t launch_solve_top(bool, const void*, const void*, const Moments*, const Geom&, int, int, double, int,
                            int64_t, int, const TopScratch&, hipStream_t) { return hipSuccess; }
hipError_t launch_top_merge(const Moments*, const Geom&, int, int, int, int, const TopScratch&, const TopOut&,
                            hipStream_t) { return hipSuccess; }
}  // namespace fchi2

// ---- the checks --------------------------------------------------------------
static int g_fail = 0;
static bool meet(const Use& a, const Use& b) { return a.lo < b.hi && b.lo < a.hi; }

static void check(const char* call, int H, int wave, int laps, uintptr_t ws, size_t bytes) {
  if (g_tables.empty() || g_rest.empty()) {
    std::printf("FAIL %s: nothing launched\n", call);
    ++g_fail;
  }
  for (const Use& t : g_tables) {
    bool bad = t.lo < ws || t.hi > ws + bytes;
    const char* with = "the end of the workspace";
    for (const Use& r : g_rest)
      if (meet(t, r)) {
        bad = true;
        with = r.what;
      }
    for (const Use& u : g_tables)
      if (u.st != t.st && meet(t, u)) {
        bad = true;
        with = "a table of the other stream";
      }
    if (bad && ++g_fail <= 20)
      std::printf("FAIL %s: table meets %s (H %d, waves of %d, %d laps, strips of 2^%d)\n", call, with, H, wave,
                  laps, g_ls);
  }
  g_tables.clear();
  g_rest.clear();
}

#define OK(expr)                                                                    \
  do {                                                                              \
    if ((expr) != FCHI2_OK) {                                                       \
      std::printf("FAIL %s: %s\n", #expr, fchi2_last_error());                      \
      return 1;                                                                     \
    }                                                                               \
  } while (0)

int main() {
  const double* pts = (const double*)fake();
  void* rows = fake();
  hipStream_t st = (hipStream_t)fake();
  const fchi2_top_out_t top{(int64_t*)rows, (double*)rows, nullptr, nullptr, nullptr, nullptr, nullptr};
  for (int H = 1; H <= 16; ++H)
    for (int laps : {1, 2, 3, 8})
      for (int wave_max = 1; wave_max <= 64; wave_max += wave_max < 40 ? 1 : 8) {
        std::vector<int64_t> off(wave_max + 1);
        for (int c = 0; c <= wave_max; ++c) off[c] = 40 * c;
        std::vector<double> span(wave_max, 1.0);
        fchi2_plan_desc_t d{};
        d.n_curves = wave_max;
        d.offsets = off.data();
        d.H = H;
        d.n_freq = 1 << (wave_max % 2 ? 10 : 11);
        d.f_max = (laps - 0.5) * (double)d.n_freq / (2.0 * H);
        d.precision = H % 2 ? FCHI2_MIXED : FCHI2_FP64;
        d.t_span = span.data();
        d.flags = FCHI2_TWO_STREAMS;
        fchi2_plan_t plan = nullptr;
        OK(fchi2_plan(&d, nullptr, &plan));
        g_elem = d.precision == FCHI2_FP64 ? 16 : 8;
        const size_t bytes = fchi2_search_top_workspace_bytes(plan, 4);
        void* ws = (void*)((uintptr_t)1 << 44);
        for (int wave : {wave_max, (wave_max + 1) / 2, wave_max / 2, wave_max / 3}) {
          if (wave < 1) continue;
          int32_t info[15];
          OK(fchi2_plan_info(plan, info, 15));
          info[6] = wave;
          OK(fchi2_plan_set_schedule(plan, info, 15));
          for (int ls : {5, 7}) {
            g_ls = ls;
            OK(fchi2_search(plan, pts, pts, pts, ws, bytes, rows, nullptr, nullptr, st));
            check("search", H, wave, laps, (uintptr_t)ws, bytes);
            if (H <= 8) {
              OK(fchi2_search_top(plan, pts, pts, pts, ws, bytes, 0, 1, 4, nullptr, &top, st));
              check("search_top", H, wave, laps, (uintptr_t)ws, bytes);
            }
          }
          if (info[0] > 1) {  // the table of the fused first pass
            info[12] = 1;
            OK(fchi2_plan_set_schedule(plan, info, 15));
            OK(fchi2_search(plan, pts, pts, pts, ws, bytes, rows, nullptr, nullptr, st));
            check("fused search", H, wave, laps, (uintptr_t)ws, bytes);
            info[12] = 0;
            OK(fchi2_plan_set_schedule(plan, info, 15));
          }
        }
        if (wave_max == 1 && H <= 5)
          for (int ls : {5, 7})
            for (int sources : {1, 2, 3, 50}) {
              g_ls = ls;
              const size_t need = fchi2_search_multi_workspace_bytes(plan, sources);
              OK(fchi2_search_multi(plan, pts, pts, pts, pts, sources, ws, need, rows, nullptr, nullptr, st));
              check("search_multi", H, sources, laps, (uintptr_t)ws, need);
            }
        fchi2_destroy(plan);
      }
  if (g_fail) {
    std::printf("%d FAILED\n", g_fail);
    return 1;
  }
  std::printf("ALL OK\n");
  return 0;
}
