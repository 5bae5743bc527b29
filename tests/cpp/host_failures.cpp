// The entry points that share pinned memory with kernels, built for the host alone over a stand-in of the HIP runtime
// (fake_hip/) whose calls can be made to fail: whatever fails, memory that a kernel may still use is not handed to
// another call, written again or freed, and once nothing fails any more the calls succeed.
// Prints "ok <runs>" or the first violation.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <string>
#include <vector>

#include "lc_api.hip"

// ---- the stand-in runtime: kernels stay in flight until an event behind them or their stream has been waited for
struct FakeStream {};
struct FakeEvent { FakeStream* stream = nullptr; long long seq = 0; };
namespace {
struct Flight { const char *lo, *hi; FakeStream* stream; long long seq; };
std::vector<Flight> g_flights;
long long g_seq = 0;
std::string g_violation, g_fail_name;
int g_fail_from = 0, g_fail_count = 0, g_seen = 0;     // calls [from, from + count) of one function fail

bool fails(const char* name) {
    if (g_fail_name != name && g_fail_name != "all") return false;
    const int i = g_seen++;
    return i >= g_fail_from && i < g_fail_from + g_fail_count;
}
void land(FakeStream* stream, long long upto) {
    std::vector<Flight> left;
    for (const Flight& f : g_flights)
        if (f.stream != stream || f.seq > upto) left.push_back(f);
    g_flights.swap(left);
}
// (an event that fails to be waited for does not say that its kernels are done)
int launch(const void* p, size_t bytes, FakeStream* stream) {
    const char *lo = static_cast<const char*>(p), *hi = lo + bytes;
    for (const Flight& f : g_flights)
        if (lo < f.hi && f.lo < hi) g_violation = "memory of a kernel in flight is used again";
    g_flights.push_back({lo, hi, stream, ++g_seq});
    return fails("launch") ? LC_ERR_HIP : LC_OK;       // (an error reported behind a launch may be an older one's)
}
}  // namespace

hipError_t hipGetDevice(int* dev) { *dev = 0; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = new FakeEvent; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    if (fails("hipEventRecord")) return hipErrorUnknown;
    e->stream = s;
    e->seq = g_seq;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    if (fails("hipEventSynchronize")) return hipErrorUnknown;
    land(e->stream, e->seq);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    if (fails("hipStreamSynchronize")) return hipErrorUnknown;
    land(s, g_seq);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
    if (fails("hipHostMalloc")) return hipErrorUnknown;
    *p = std::malloc(bytes);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    for (const Flight& f : g_flights)
        if (static_cast<const char*>(p) >= f.lo && static_cast<const char*>(p) < f.hi) g_violation = "memory of a kernel in flight is freed";
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in"; }

// ---- the launchers that lc_api.hip calls
int lc_walk_max_internal_nodes() { return 0; }
int lc_beam_max_level_nodes() { return 0; }
int lc_launch_build(const lc_index*, const LcWs&, const void*, const int64_t*, int, hipStream_t) { return LC_OK; }
int lc_launch_retrieve(const lc_index*, const LcWs&, const void*, int, int, int32_t*, int32_t*, float*, int, int, int, int,
                       hipStream_t) { return LC_OK; }
int lc_launch_decode(const lc_index*, const LcWs&, const void*, const void*, const void*, const int64_t*, const int32_t*,
                     const int32_t*, int, int, int, float*, float*, hipStream_t) { return LC_OK; }
bool lc_decode_fused_fits(int, int) { return false; }
int lc_launch_decode_fused(const lc_index*, const LcWs&, const void*, const void*, const void*, const int64_t*, int, int, int,
                           int32_t*, int32_t*, int, int, bool, float*, float*, hipStream_t) { return LC_OK; }
int lc_launch_append(const lc_index*, void*, void*, const int64_t*, const void*, const void*, const uint8_t*, uint32_t,
                     hipStream_t) { return LC_OK; }
int lc_launch_drift(const lc_index* idx, int, float* out, hipStream_t s) {
    return launch(out, (size_t)idx->B * idx->H_kv * 16, s);
}
int lc_launch_place_state(const lc_index* idx, const int32_t* staged, int, hipStream_t s) {
    return launch(staged, ((size_t)idx->B * idx->H_kv * 4 + idx->B * (LC_MAX_LEVELS + 1)) * 4, s);
}
int lc_launch_place_counts(const lc_index* idx, const int32_t* staged, hipStream_t s) {
    return launch(staged, (size_t)idx->B * LC_MAX_LEVELS * 4, s);
}
int lc_launch_blob_export(const LcDev&, const LcBlobMap&, const long long*, unsigned long long, unsigned n, uint32_t* window,
                          hipStream_t s) { return launch(window, (size_t)n * 4, s); }
int lc_launch_blob_import(const LcDev&, const LcBlobMap&, const long long*, unsigned long long, unsigned n,
                          const uint32_t* window, hipStream_t s) { return launch(window, (size_t)n * 4, s); }

int main() {
    const int M = 2000, H = 8;                         // a blob of more windows than there are slots
    lc_config cfg;
    lc_config_default(&cfg);
    cfg.levels = 2;
    cfg.max_chunks = M;
    cfg.max_tokens = 4 * M;
    const int64_t strides[3] = {(int64_t)H * 4 * M * 128, (int64_t)4 * M * 128, 128};
    std::vector<int32_t> bounds(M + 1);
    for (int i = 0; i <= M; ++i) bounds[i] = 3 * i;
    const int32_t T = 3 * M, count = M;
    const size_t ib = lc_index_bytes(&cfg, 1, H, 128), wb = lc_workspace_bytes(&cfg, 1, H, H, 128);
    void* const buf = aligned_alloc(256, ib);
    void* const ws = aligned_alloc(256, wb);
    FakeStream streams[2];
    FakeStream* s = &streams[0];                       // the failing call's stream; later calls go to another one
    auto build = [&](lc_index** out) {
        return lc_build_index(out, &cfg, ws, strides, &T, bounds.data(), &count, 1, H, 128, buf, ib, ws, wb, s);
    };
    lc_index* idx = nullptr;
    if (build(&idx) != LC_OK) { std::printf("FAIL build\n"); return 1; }
    size_t bytes = 0;
    lc_index_export(idx, nullptr, &bytes, nullptr);
    std::vector<char> blob(bytes, 0), copy(bytes);
    const int32_t hdr[9] = {0x5849434C, 1, 1, H, 128, cfg.levels, cfg.fanout, cfg.geometry, cfg.center_dtype};
    std::memcpy(blob.data(), hdr, sizeof(hdr));
    const int32_t rec[3] = {T, M, (M + cfg.fanout - 1) / cfg.fanout};
    std::memcpy(blob.data() + 64, rec, sizeof(rec));
    std::memcpy(blob.data() + 76, bounds.data(), bounds.size() * 4);
    std::vector<float> drift(H * 4);

    struct Call { const char* name; std::function<int()> run; };
    const std::vector<Call> calls = {
        {"build", [&] { lc_index* i = nullptr; const int rc = build(&i); lc_index_destroy(i); return rc; }},
        {"recluster", [&] { return lc_recluster(idx, ws, wb, s); }},
        {"drift", [&] { return lc_index_drift(idx, 1, drift.data(), ws, wb, s); }},
        {"export", [&] { size_t n = bytes; return lc_index_export(idx, copy.data(), &n, s); }},
        {"import", [&] {
            lc_index* i = nullptr;
            const int rc = lc_index_import(&i, &cfg, blob.data(), blob.size(), buf, ib, s);
            lc_index_destroy(i);
            return rc;
        }},
    };
    long runs = 0;
    for (const char* what : {"launch", "hipEventRecord", "hipEventSynchronize", "hipStreamSynchronize", "hipHostMalloc", "all"})
        for (const Call& c : calls)
            for (int from = 0; from < 12; ++from)
                for (int many : {1, 1000}) {
                    // the failing call, then (nothing failing any more) every call several times
                    g_fail_name = what; g_fail_from = from; g_fail_count = many; g_seen = 0;
                    s = &streams[0];
                    const int rc = c.run();
                    g_fail_name.clear();
                    s = &streams[1];
                    if (rc != LC_OK && rc != LC_ERR_HIP) g_violation = "unexpected code";
                    for (int r = 0; r < 5 && g_violation.empty(); ++r)
                        for (const Call& d : calls)
                            if (d.run() != LC_OK) g_violation = std::string("a later call fails: ") + d.name;
                    if (!g_violation.empty()) {
                        std::printf("FAIL %s after %s fails from call %d on (%d times): %s\n", c.name, what, from, many, g_violation.c_str());
                        return 1;
                    }
                    ++runs;
                }
    std::printf("ok %ld\n", runs);
    return 0;
}
