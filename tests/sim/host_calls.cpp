// Host side of libgpusparse.so over a stand-in for the device (built and run by
// tests/test_host_calls_sim.py on the CPU, one case per run). Device memory is host memory,
// copies are done at once, and kernel launches are only recorded, with the device that was
// current and the stream they went to. So a case can check what the host code asks of the
// device - which allocations, on which device it waits, which launches with which
// arguments - where a GPU could not show it: two devices, memory that runs out, a call that
// fails, a stream under capture, sizes past any memory.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <random>
#include <set>
#include <string>
#include <utility>
#include <vector>

#include "../../include/gpusparse.h"
#include "../../paper_2606_26441_amd/csrc/gs_internal.h"

// ------------------------------------------------------------- the device --

struct Launch {
    std::string kernel;
    int device;
    hipStream_t stream;
    int tile_shift = 0, chunk = 0;
    bool wide = false, from_row = false;
};

static int g_device = 0;
static std::vector<Launch> g_launches;
static std::set<std::pair<int, hipStream_t>> g_pending;  // (device, stream) with work not waited for
static std::map<void*, size_t> g_live;                   // device allocations
static size_t g_room = (size_t)1 << 40, g_used = 0;
static int g_fail_event_record = -1;                     // calls left before one fails
static hipStream_t g_capturing = nullptr;
static hipError_t g_last = hipSuccess;
static gs::DevBatch g_batch{};                           // of the last doc-tiled launch
static int32_t g_rows = 0;                               // rows of its index

static Launch& launch(const char* kernel, hipStream_t s) {
    g_launches.push_back(Launch{kernel, g_device, s});
    g_pending.insert({g_device, s});
    return g_launches.back();
}
static void wait_device() {
    for (auto it = g_pending.begin(); it != g_pending.end();)
        it = it->first == g_device ? g_pending.erase(it) : std::next(it);
}

extern "C" {
hipError_t hipGetDevice(int* d) { *d = g_device; return hipSuccess; }
hipError_t hipSetDevice(int d) { g_device = d; return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMalloc(void** p, size_t n) {
    if (g_used + n > g_room) { *p = nullptr; return g_last = hipErrorOutOfMemory; }
    *p = std::malloc(n ? n : 1);
    g_live[*p] = n;
    g_used += n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    wait_device();
    g_used -= g_live[p];
    g_live.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::malloc(n ? n : 1); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = g_room - g_used; *t = g_room; return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { wait_device(); std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    std::memcpy(d, s, n);
    g_pending.insert({g_device, st});
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
    std::memset(d, v, n);
    g_pending.insert({g_device, st});
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) {
    if (g_fail_event_record == 0) { g_fail_event_record = -1; return hipErrorUnknown; }
    if (g_fail_event_record > 0) g_fail_event_record--;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { g_pending.erase({g_device, s}); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
    *st = s && s == g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)std::malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { std::free(s); return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = nullptr; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) { *e = nullptr; return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
}

namespace gs {
hipError_t launch_fill_rows(const DevIndex&, const int32_t*, void*, hipStream_t s) { launch("fill_rows", s); return hipSuccess; }
hipError_t launch_narrow(const int32_t* src, uint16_t* dst, int64_t n, hipStream_t s) {
    for (int64_t i = 0; i < n; i++) dst[i] = (uint16_t)src[i];
    launch("narrow", s);
    return hipSuccess;
}
hipError_t launch_clear(const Workspace&, int32_t, hipStream_t s) { launch("clear", s); return hipSuccess; }
hipError_t launch_score_tiled(const DevIndex& ix, const DevBatch& qb, int32_t, int32_t, const ScoreOpts& o,
                              const Workspace&, hipStream_t s, int) {
    Launch& l = launch("score_tiled", s);
    g_batch = qb;
    g_rows = ix.n_rows;
    l.tile_shift = o.tile_shift;
    l.chunk = o.chunk;
    return hipSuccess;
}
hipError_t launch_score_group(const DevIndex&, const DevBatch&, const ScoreOpts&, const Workspace&, hipStream_t s, int) {
    launch("score_group", s);
    return hipSuccess;
}
hipError_t launch_score_atomic(const DevIndex&, const DevBatch&, int32_t, int32_t, const ScoreOpts& o, const Workspace&,
                               hipStream_t s) {
    launch("score_atomic", s).chunk = o.chunk;
    return hipSuccess;
}
hipError_t launch_score_docpar(const DevIndex&, const DevBatch&, int32_t, int32_t, const ScoreOpts&, const Workspace&,
                               hipStream_t s) {
    launch("score_docpar", s);
    return hipSuccess;
}
hipError_t launch_select(const DevIndex&, const DevBatch&, int32_t, int32_t, const Workspace&, int32_t*, void*, int32_t*,
                         hipStream_t s, int, int, int, const ScoreOpts*, bool wide, bool from_row) {
    Launch& l = launch("select", s);
    l.wide = wide;
    l.from_row = from_row;
    return hipSuccess;
}
hipError_t launch_seed_bound(const DevIndex&, const DevBatch&, int32_t, int32_t, const Workspace&, hipStream_t s, int, int) {
    launch("seed_bound", s);
    return hipSuccess;
}
hipError_t launch_upload(void* d, const void* h, const UploadRanges& r, hipStream_t s) {
    for (int i = 0; i < r.n; i++)
        std::memcpy((uint8_t*)d + (size_t)r.at[i] * 16, (const uint8_t*)h + (size_t)r.at[i] * 16, (size_t)r.len[i] * 16);
    launch("upload", s);
    return hipSuccess;
}
hipError_t launch_copy16(void*, const void*, int64_t, hipStream_t s) { launch("copy16", s); return hipSuccess; }
hipError_t launch_lds_atomic(int, int, int, int, void*, hipStream_t s) { launch("lds_atomic", s); return hipSuccess; }
hipError_t launch_fill(void*, int64_t, uint32_t, hipStream_t s) { launch("fill", s); return hipSuccess; }
hipError_t scratch_address(int, void** out) {
    static std::vector<uint8_t> scratch(256);  // only its address is used: launches do nothing here
    *out = scratch.data();
    return hipSuccess;
}
}  // namespace gs

// -------------------------------------------------------------- the cases --

static int failures = 0;
static void expect(bool ok, const char* what) {
    if (!ok) {
        std::fprintf(stderr, "FAILED: %s (%s)\n", what, gs_last_error());
        failures++;
    }
}

// n documents: term 0 in all of them, term 1 in every other one, term 2 + d % 20 in document d.
static gs_index make_index(int n, int precision, uint32_t flags = 0) {
    std::vector<int64_t> rp{0};
    std::vector<int32_t> t;
    std::vector<float> w;
    for (int d = 0; d < n; d++) {
        t.push_back(0);
        if (d % 2) t.push_back(1);
        t.push_back(2 + d % 20);
        while (w.size() < t.size()) w.push_back(0.5f + (float)(w.size() % 7) / 4.0f);
        rp.push_back((int64_t)t.size());
    }
    gs_index ix = nullptr;
    gs_build_index(rp.data(), n, t.data(), w.data(), (int64_t)t.size(), 22, precision, flags, nullptr, &ix);
    return ix;
}

struct Query {
    std::vector<int64_t> rp{0, 3};
    std::vector<int32_t> term{0, 1, 5};
    std::vector<float> w{1.0f, 0.75f, 1.5f};
    std::vector<int32_t> k{10};
    std::vector<uint8_t> ws;
    std::vector<int32_t> ids = std::vector<int32_t>(10);
    std::vector<double> sc = std::vector<double>(10);
    explicit Query(gs_index ix) {
        size_t bytes = 0;
        gs_workspace_size(ix, 1, nullptr, &bytes);
        ws.resize(bytes);
    }
    int32_t search(gs_index ix, hipStream_t s = nullptr, const gs_search_opts* o = nullptr) {
        return gs_search(ix, rp.data(), 1, term.data(), w.data(), 3, k.data(), 10, ws.data(), ws.size(), ids.data(),
                         sc.data(), o, s);
    }
};

static int count(const char* kernel) {
    int n = 0;
    for (const Launch& l : g_launches) n += l.kernel == kernel;
    return n;
}

// The rows of the commonest terms: their number keeps the 32-bit byte offsets that the scoring
// kernel forms inside its largest tile (2 grains of fp32, 4 of the other forms) below 2^31.
static void row_limit() {
    struct { int precision; int64_t w, grains; } form[3] = {{GS_FP32, 4, 2}, {GS_BF16, 2, 4}, {GS_U8, 1, 4}};
    for (const auto& f : form)
        for (int64_t n_grains : {1, 2, 3, 4, 100, 262144})
            for (int64_t padded : {(int64_t)64, (int64_t)1 << 24, (int64_t)1 << 30, (int64_t)1 << 36}) {
                const int64_t n = gs::row_limit(f.precision, n_grains, padded);
                expect(n >= 0, "a limit");
                expect(n << gs::kGrainShift < (int64_t)1 << 31, "a grain's rows");
                expect((((f.grains - 1) * n + 1) << gs::kGrainShift) * f.w < (int64_t)1 << 31, "a tile's bytes");
                const int64_t row = (n_grains << gs::kGrainShift) * f.w;
                expect(n * row <= std::max((int64_t)64 << 20, 3 * (2 + f.w) * padded), "a limit on the rows' bytes");
            }
    // 16,384 documents, 262,144 terms in a quarter of them each
    expect(gs::row_limit(GS_FP32, 2, 262144ll * 4096) > 0, "rows in a large index");
}

// A synchronous search of an index on another device than the current one, on the default
// stream: its work, on the index's device, is done when the call returns.
static void search_waits_on_the_index_device() {
    for (int precision : {GS_FP32, GS_BF16, GS_U8}) {
        g_device = 1;
        gs_index ix = make_index(40000, precision);
        wait_device();
        g_device = 0;
        Query q(ix);
        expect(q.search(ix) == GS_OK, "search");
        for (const Launch& l : g_launches) expect(l.device == 1, "launched on the index's device");
        expect(g_pending.empty(), "waited for");
        expect(g_device == 0, "the caller's device is current again");
        gs_free_index(ix);
    }
}

// An update that fails after its upload was enqueued: the batch's memory is still being read, so
// it is freed (which waits for the device) and not kept for the next call.
static void failed_upload_keeps_no_batch() {
    gs_index ix = make_index(40000, GS_FP32);
    wait_device();
    Query q(ix);
    const size_t before = g_live.size();
    g_fail_event_record = 0;
    expect(q.search(ix) == GS_EHIP, "the update fails");
    expect(g_pending.empty() && g_live.size() == before, "nothing is kept while work is under way");
    expect(q.search(ix) == GS_OK && g_live.size() == before + 1, "the next call keeps its batch");
    q.term[0] = -1;
    expect(q.search(ix) == GS_EINVAL && g_live.size() == before + 1, "a refused call keeps it too");
    gs_free_index(ix);
    expect(g_live.empty(), "all of it is freed with the index");
}

// A search that its caller captures is replayed after updates with any queries, wide-range ones
// among them: the launches hold the wide-range pass whatever the batch holds at capture.
static void captured_search_has_the_wide_pass() {
    for (int precision : {GS_FP32, GS_BF16, GS_U8})
        for (int docs : {20000, 40000})
            for (bool captured : {false, true}) {
                gs_index ix = make_index(docs, precision);
                Query q(ix);
                gs_batch b = nullptr;
                expect(gs_batch_create(ix, q.rp.data(), 1, q.term.data(), q.w.data(), 3, q.k.data(), 10, nullptr, &b) == GS_OK,
                       "batch");
                int mine = 0;
                const hipStream_t s = (hipStream_t)&mine;
                g_capturing = captured ? s : nullptr;
                for (int noalloc = 0; noalloc < 2; noalloc++) {
                    g_launches.clear();
                    expect((noalloc ? gs_search_batch_noalloc(ix, b, q.ids.data(), q.sc.data(), nullptr, s)
                                    : gs_search_batch(ix, b, q.ws.data(), q.ws.size(), q.ids.data(), q.sc.data(), nullptr, s)) == GS_OK,
                           "search");
                    expect(count("select") == 1, "one selection");
                    const Launch& l = g_launches.back();
                    // these weights give an fp32 query no wide-range limit, a bf16 one neither
                    expect(l.wide == (captured && precision != GS_U8), "the wide-range pass");
                    expect(l.from_row == (docs <= gs::kCandCap && precision != GS_BF16 && !l.wide), "rows as candidates");
                }
                g_capturing = nullptr;
                gs_batch_free(b);
                gs_free_index(ix);
            }
}

// Rows are optional: where their memory cannot be had the index is built without them, and it
// takes no memory that the rest of the index needs.
static void index_without_room_for_rows() {
    for (int precision : {GS_FP32, GS_BF16, GS_U8}) {
        const int n = 200000;
        const uint32_t flags = GS_KEEP_FORWARD | GS_KEEP_DOC_IDS;
        gs_index ix = make_index(n, precision, flags);
        expect(ix && count("fill_rows") == 1, "rows where there is room");
        gs_index_info_t with{}, without{};
        gs_index_info(ix, &with);
        gs_free_index(ix);
        expect(g_live.empty(), "freed");
        // the least memory that the index can be built in, to 1 MiB
        size_t lo = 0, hi = (size_t)with.device_bytes + (64 << 20);
        while (hi - lo > (1 << 20)) {
            g_room = (lo + hi) / 2;
            g_launches.clear();
            gs_index t = make_index(n, precision, flags);
            if (t) {
                hi = g_room;
                if (count("fill_rows") == 0) gs_index_info(t, &without);
                gs_free_index(t);
            } else {
                lo = g_room;
            }
            expect(g_used == 0, "nothing is left of a failed build");
        }
        const int64_t row = ((n + 8191) / 8192) * 8192ll * (precision == GS_FP32 ? 4 : precision == GS_BF16 ? 2 : 1);
        expect(with.device_bytes - without.device_bytes == 2 * row, "two rows");
        // the forward terms pass through a stage of four bytes each while the index is built
        expect((int64_t)hi <= without.device_bytes + 4 * with.nnz + (2 << 20), "no memory of the rows is needed");
        g_room = (size_t)1 << 40;
        // their allocation fails, whatever the free memory says: no rows, and a search that works
        g_launches.clear();
        int64_t allocs = 0;
        for (;; allocs++) {
            gs_debug_fail_alloc(allocs);
            ix = make_index(n, precision, flags);
            gs_debug_fail_alloc(-1);
            if (ix) break;
        }
        gs_index_info(ix, &without);
        expect(count("fill_rows") == 0 && with.device_bytes - without.device_bytes == 2 * row, "built without rows");
        uint8_t has[22];
        expect(gs_index_row_terms(ix, has, 22) == GS_OK && std::count(has, has + 22, 0) == 22, "no term has a row");
        Query q(ix);
        expect(q.search(ix) == GS_OK, "searched without rows");
        gs_free_index(ix);
    }
}

// The autotuner times each different launch once: the per-query and the shared-traversal kernel are
// one, and chunks below 256 run as 256.
static void autotune_times_each_launch_once() {
    for (int precision : {GS_FP32, GS_U8}) {
        gs_index ix = make_index(40000, precision);
        Query q(ix);
        gs_batch b = nullptr;
        gs_batch_create(ix, q.rp.data(), 1, q.term.data(), q.w.data(), 3, q.k.data(), 10, nullptr, &b);
        g_launches.clear();
        gs_search_opts best{}, cands[64];
        float ms[64] = {};
        int32_t n = 0;
        const int reps = 3, tiles = precision == GS_FP32 ? 2 : 3;
        expect(gs_autotune(ix, b, q.ws.data(), q.ws.size(), q.ids.data(), q.sc.data(), reps, nullptr, &best, cands, ms, 64,
                           &n) == GS_OK, "autotune");
        expect(n == 2 * tiles * 4 + 3, "every option set is listed");
        std::map<std::pair<int, int>, int> runs;
        for (const Launch& l : g_launches)
            if (l.kernel == "score_tiled") runs[{l.tile_shift, std::max(l.chunk, 256)}]++;
        int total = 0;
        for (const auto& r : runs) total += r.second;
        expect((int)runs.size() == tiles * 3, "different doc-tiled launches");
        expect(total == tiles * 3 * (1 + reps) + 1, "each timed once, and the best run at the end");
        for (int i = 0; i < n; i++) expect(ms[i] > 0.0f, "a time for every option set");
        gs_batch_free(b);
        gs_free_index(ix);
    }
}

// Workgroups per tile of a pass over listed queries: the chip is full where the work allows it,
// and no workgroup is without a query that could be listed.
static void listed_queries_fill_the_chip() {
    for (int64_t tiles : {1, 2, 17, 28, 62, 511, 512, 513, 1075, 262144})
        for (int64_t qt : {1, 2, 32, 500, 4096}) {
            const int64_t w = gs::listed_ways(tiles, qt);
            expect(w >= 1 && w <= qt, "at most one workgroup per query and tile");
            expect(tiles * w >= std::min<int64_t>(512, tiles * qt), "two workgroups per CU");
            expect(w == 1 || tiles * (w - 1) < 512, "no more than that");
        }
}

// The first selection digit of float scores: bins in the order of the scores, each score between
// its bin's edges, and an edge close below it: within 0.4 % in the seven octaves below the query's
// largest possible score, within 12.5 % in the 32 below those.
static void first_digit_bounds_the_score() {
    auto bits = [](float f) { uint32_t b; std::memcpy(&b, &f, 4); return b; };
    auto value = [](unsigned long long c) { const uint32_t b = (uint32_t)(c >> 32); float f; std::memcpy(&f, &b, 4); return f; };
    for (float w : {1.0f, 3.0f, 1e-30f, 3e-38f, 1e-44f, 1e30f, 3e38f, 0.0f})
        for (float t : {1.0f, 2.9f, 1e-6f, 3e38f, 0.0f}) {
            const gs::FirstDigit f = gs::float_digit(1, &w, &t, 0.0);
            const double top = (double)w * (double)t;
            uint32_t last = 0;
            int zero_bin = (int)gs::first_digit<true>(f, 0u);
            expect(gs::first_edge(f, zero_bin) == 0ull, "the edge of score 0's bin");
            for (int e = 400; e >= 0; e--) {  // ascending scores
                const float s = (float)(top * std::pow(2.0, -e / 8.0) * 0.999);
                const uint32_t d = gs::first_digit<true>(f, bits(s));
                expect(d >= last && d < (uint32_t)gs::kHistBins, "ascending bins");
                last = d;
                const unsigned long long c = (unsigned long long)bits(s) << 32;
                expect(gs::first_edge(f, (int)d) <= c && c < gs::first_edge(f, (int)d + 1), "between the bin's edges");
                if (s >= 1.2e-38f && std::isfinite(s) && e < 38 * 8) {
                    const double rel = 1.0 - (double)value(gs::first_edge(f, (int)d)) / (double)s;
                    expect(rel <= (e < 6 * 8 ? 0.004 : 0.125), "an edge close below the score");
                }
            }
            expect(gs::first_digit<true>(f, 0x7f800000u) < (uint32_t)gs::kHistBins, "infinity");
        }
}

// Which terms have rows: held by at least a quarter of the documents.
static void row_terms_at_the_threshold() {
    const int n = 10000;
    std::vector<int64_t> rp{0};
    std::vector<int32_t> t;
    for (int d = 0; d < n; d++) {
        if (d < n / 4) t.push_back(0);      // exactly a quarter
        if (d < n / 4 - 1) t.push_back(1);  // one less
        t.push_back(3);                     // every document; none holds terms 2 and 4
        rp.push_back((int64_t)t.size());
    }
    const std::vector<float> w(t.size(), 1.0f);
    for (int precision : {GS_FP32, GS_BF16, GS_U8}) {
        gs_index ix = nullptr;
        expect(gs_build_index(rp.data(), n, t.data(), w.data(), (int64_t)t.size(), 5, precision, 0, nullptr, &ix) == GS_OK,
               "build");
        uint8_t row[5] = {9, 9, 9, 9, 9};
        expect(gs_index_row_terms(ix, row, 5) == GS_OK, "flags");
        expect(row[0] == 1 && row[1] == 0 && row[2] == 0 && row[3] == 1 && row[4] == 0, "the terms with rows");
        expect(gs_index_row_terms(ix, row, 4) == GS_EINVAL && gs_index_row_terms(ix, nullptr, 5) == GS_EINVAL &&
                   gs_index_row_terms(nullptr, row, 5) == GS_EINVAL, "bad arguments");
        gs_free_index(ix);
    }
}

// What a batch update leaves on the device of a query's terms: the scoring records (terms with rows
// first, by row, the commonest first; then the others, ascending) and the cumulative bounds of pruning (per
// term, the sum of the bounds of the terms up to it in ascending order of bound, ties by position).
static void update_records() {
    std::mt19937_64 rng(11);
    const int n = 3000, vocab = 400;
    std::vector<int64_t> rp{0};
    std::vector<int32_t> t;
    std::vector<float> w;
    for (int d = 0; d < n; d++) {
        for (int v = 0; v < vocab; v++)
            if (rng() % 400 < (v < 150 ? 90u + v : 10u)) {  // some of the first 150 terms in a quarter of the documents
                t.push_back(v);
                w.push_back((float)(1 + rng() % 255) / 85.0f);
            }
        rp.push_back((int64_t)t.size());
    }
    std::vector<int64_t> df(vocab, 0);
    std::vector<float> top(vocab, 0.0f);
    for (size_t i = 0; i < t.size(); i++) {
        df[t[i]]++;
        top[t[i]] = std::max(top[t[i]], w[i]);
    }
    for (int precision : {GS_FP32, GS_BF16, GS_U8}) {
        gs_index ix = nullptr;
        gs_build_index(rp.data(), n, t.data(), w.data(), (int64_t)t.size(), vocab, precision, 0, nullptr, &ix);
        std::vector<uint8_t> row(vocab);
        gs_index_row_terms(ix, row.data(), vocab);
        std::vector<int64_t> qp{0};
        std::vector<int32_t> qt, k;
        std::vector<float> qw;
        for (int m : {0, 1, 2, 9, 34, 64, 65, 200, 256}) {
            std::vector<int32_t> all(vocab);
            for (int v = 0; v < vocab; v++) all[v] = v;
            std::shuffle(all.begin(), all.end(), rng);
            std::sort(all.begin(), all.begin() + m);
            for (int j = 0; j < m; j++) {
                qt.push_back(all[j]);
                qw.push_back((float)(rng() % 20) / 10.0f);  // zeros and equal ones among them
            }
            qp.push_back((int64_t)qt.size());
            k.push_back(5);
        }
        const int nq = (int)k.size();
        gs_batch b = nullptr;
        expect(gs_batch_create(ix, qp.data(), nq, qt.data(), qw.data(), (int64_t)qt.size(), k.data(), 5, nullptr, &b) == GS_OK,
               "batch");
        size_t bytes = 0;
        gs_workspace_size(ix, nq, nullptr, &bytes);
        std::vector<uint8_t> ws(bytes);
        std::vector<int32_t> ids(nq * 5);
        std::vector<double> sc(nq * 5);
        expect(gs_search_batch(ix, b, ws.data(), bytes, ids.data(), sc.data(), nullptr, nullptr) == GS_OK, "search");
        expect(g_rows > 10 && g_rows < 150, "some terms have rows");
        auto impact = [](float x) { return (int64_t)std::nearbyint((double)x * 85.0); };
        for (int q = 0; q < nq; q++) {
            std::vector<int32_t> want, rest;
            for (int64_t j = qp[q]; j < qp[q + 1]; j++)
                if (qw[j] > 0.0f) (row[qt[j]] ? want : rest).push_back(qt[j]);
            std::sort(want.begin(), want.end(), [&](int a, int c) { return df[a] > df[c] || (df[a] == df[c] && a < c); });
            const size_t n_row = want.size();
            want.insert(want.end(), rest.begin(), rest.end());
            const gs::ScoreItem it = g_batch.s_item[q];
            expect(it.q == q && (size_t)(it.n & 1023) == want.size() && (size_t)(it.n >> 10) == n_row, "a query's item");
            for (size_t i = 0; i < want.size(); i++) {
                const gs::ScoreTerm& r = g_batch.s_term[it.start + (int64_t)i];
                expect(r.term == want[i] && (r.row >= 0) == (i < n_row), "the order of the records");
                expect(i == 0 || i >= n_row || r.row > g_batch.s_term[it.start + (int64_t)i - 1].row, "ascending rows");
                const int64_t j = std::lower_bound(qt.begin() + qp[q], qt.begin() + qp[q + 1], r.term) - qt.begin();
                double fx;
                std::memcpy(&fx, &r.q, 8);
                expect(precision == GS_U8 ? (int64_t)r.q == impact(qw[j]) : fx == (double)qw[j] / g_batch.q_scale[q], "the weight");
            }
            if (precision == GS_BF16) continue;
            const int64_t m = qp[q + 1] - qp[q];
            std::vector<std::pair<uint64_t, int64_t>> u;
            for (int64_t j = 0; j < m; j++) {
                const float x = qw[qp[q] + j], y = top[qt[qp[q] + j]];
                u.push_back({precision == GS_U8 ? (uint64_t)(impact(x) * impact(y))
                                                : (uint64_t)std::ceil((double)x / g_batch.q_scale[q] * (double)y) + 1, j});
            }
            std::sort(u.begin(), u.end());
            uint64_t run = 0;
            for (const auto& e : u) {
                run += e.first;
                expect(g_batch.q_ub_cum[qp[q] + e.second] == run, "a cumulative bound");
            }
        }
        gs_batch_free(b);
        gs_free_index(ix);
    }
}

int main(int argc, char** argv) {
    const std::string name = argc > 1 ? argv[1] : "";
    if (name == "row_limit") row_limit();
    else if (name == "search_waits_on_the_index_device") search_waits_on_the_index_device();
    else if (name == "failed_upload_keeps_no_batch") failed_upload_keeps_no_batch();
    else if (name == "captured_search_has_the_wide_pass") captured_search_has_the_wide_pass();
    else if (name == "index_without_room_for_rows") index_without_room_for_rows();
    else if (name == "autotune_times_each_launch_once") autotune_times_each_launch_once();
    else if (name == "listed_queries_fill_the_chip") listed_queries_fill_the_chip();
    else if (name == "first_digit_bounds_the_score") first_digit_bounds_the_score();
    else if (name == "row_terms_at_the_threshold") row_terms_at_the_threshold();
    else if (name == "update_records") update_records();
    else expect(false, "unknown case");
    std::printf("%s: %d failures\n", name.c_str(), failures);
    return failures == 0 ? 0 : 1;
}
