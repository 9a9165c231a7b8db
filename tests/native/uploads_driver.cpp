// Test infrastructure: when the library copies a plan's tables into its workspace, on a runtime of the driver's own: streams are queues of host functions that run at once or,
// while the stream is held, when the test says so; a captured stream records them in a graph.  "Device" memory is host memory, and a launch looks the tables up when it runs.
// Built with g++, no device code, no HIP runtime.  The first argument names the check; the exit status is 0 if it holds, and the text says what does not.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <ctime>
#include <deque>
#include <functional>
#include <string>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "../../include/packinfer.h"
#include "../../paper_2602_06072_amd/csrc/kernels.h"
#include "../../paper_2602_06072_amd/csrc/plan.h"

// ---- the runtime -----------------------------------------------------------
using Work = std::function<void()>;
struct Graph { std::vector<Work> nodes; int copies = 0; };
struct Stream {
    bool held = false;
    std::deque<Work> queue;
    Graph* graph = nullptr;                        // not null: being captured
    unsigned long long capture = 0;
    void add(Work w) {
        if (graph) graph->nodes.push_back(std::move(w));
        else if (held) queue.push_back(std::move(w));
        else w();
    }
    void run(size_t most = ~size_t{0}) {
        for (; most > 0 && !queue.empty(); --most) {
            queue.front()();
            queue.pop_front();
        }
    }
};
struct Event { bool reached = true; };
static unsigned long long captures = 0;
static int pageable = 0, waits = 0;               // copies from pageable memory outside of captures; turns of waiting
static Work on_wait;
static std::vector<std::pair<char*, size_t>> pinned;
static Stream* of(void* s) { return static_cast<Stream*>(s); }
static Stream* of(hipStream_t s) { return reinterpret_cast<Stream*>(s); }
static void begin(Stream& s, Graph& g) { s.graph = &g; s.capture = ++captures; }
static void end(Stream& s) { s.graph = nullptr; s.capture = 0; }
static void replay(Graph& g) { for (Work& w : g.nodes) w(); }

extern "C" {
int nanosleep(const timespec*, timespec*) { ++waits; if (on_wait) on_wait(); return 0; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::malloc(n);
    pinned.emplace_back(static_cast<char*>(*p), n);
    return hipSuccess;
}
hipError_t hipHostFree(void*) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(new Event); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    Event* ev = reinterpret_cast<Event*>(e);
    ev->reached = false;
    of(s)->add([ev] { ev->reached = true; });
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) { return reinterpret_cast<Event*>(e)->reached ? hipSuccess : hipErrorNotReady; }
hipError_t hipStreamSynchronize(hipStream_t s) { of(s)->run(); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* status) {
    *status = of(s)->graph ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamGetCaptureInfo(hipStream_t s, hipStreamCaptureStatus* status, unsigned long long* id) {
    *id = of(s)->capture;
    return hipStreamIsCapturing(s, status);
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) { *m = hipStreamCaptureModeGlobal; return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t s) {
    const char* p = static_cast<const char*>(src);
    bool own = false;
    for (const auto& [at, size] : pinned) own = own || (p >= at && p < at + size);
    if (of(s)->graph) ++of(s)->graph->copies;
    else if (!own) { ++pageable; of(s)->run(); }   // (the host waits for the stream)
    of(s)->add([=] { std::memcpy(dst, src, n); });
    return hipSuccess;
}
}  // extern "C"

// ---- launches: what they find in the workspace when they run ----------------
static const pk_plan* current = nullptr;           // the plan that the next launch belongs to
static int launches = 0, wrong = 0;
static void expects(void* stream, const void* at, const std::vector<int32_t>& host, const pk::TableRef& r) {
    const auto* first = host.data() + r.offset / sizeof(int32_t);
    std::vector<int32_t> words(first, first + r.count);
    of(stream)->add([=] {
        ++launches;
        wrong += words.empty() || std::memcmp(at, words.data(), words.size() * sizeof(int32_t)) != 0;
    });
}
alignas(256) static char scratch[PK_STATIC_SCRATCH_BYTES];

namespace pk {
int launch_upload(const void* src, void* dst, int64_t bytes, uint32_t* done, uint32_t stamp, void* stream) {
    of(stream)->add([=] { std::memcpy(dst, src, static_cast<size_t>(bytes)); *done = stamp; });
    return 0;
}
int launch_reorg_bf16(const ReorgArgs& a, void* s) { expects(s, a.seg, current->tables.host, current->tables.reorg_seg); return 0; }
int launch_append_bf16(const AppendArgs& a, void* s) { expects(s, a.req_seg, current->tables.host, current->tables.dec_req_seg); return 0; }
int launch_decode_bf16(const DecodeArgs& a, void* s) { expects(s, a.items, current->tables.host, current->tables.dec.items); return 0; }
int launch_prefill_bf16(const PrefillArgs& a, void* s) {
    const DeviceTables& t = current->tables;
    const char* tiles = reinterpret_cast<const char*>(a.tiles);
    const char* packed = static_cast<const char*>(current->bound_ws) + (current->decode_only ? t.packed_offset : 0) + t.packed.tiles.offset;
    if (tiles == packed) expects(s, a.tiles, current->decode_only ? t.host_packed : t.host, t.packed.tiles);
    else expects(s, a.tiles, t.host_padded, t.padded.tiles);
    return 0;
}
int launch_mixed_step_bf16(const PrefillArgs& a, const DecodeArgs&, void* s) { return launch_prefill_bf16(a, s); }
int static_scratch_address(void** p) { *p = scratch; return 0; }
int launch_padded_decode_bf16(const PagedDecodeArgs&, void*) { std::abort(); }
int launch_decode_merge_bf16(const DecodeArgs&, void*) { std::abort(); }
int launch_reorg_f32(const ReorgArgs&, void*) { std::abort(); }
int launch_append_f32(const AppendArgs&, void*) { std::abort(); }
int launch_decode_f32(const DecodeArgs&, void*) { std::abort(); }
int launch_prefill_f32(const PrefillArgs&, void*) { std::abort(); }
}  // namespace pk

// ---- a plan and its calls ---------------------------------------------------
constexpr int HQ = 8, HKV = 2, D = 128;
alignas(16) static char tensor[16];                // (nothing reads the tensors)
struct Batch {
    pk_plan* plan = nullptr;
    std::vector<char> memory;
    char* ws = nullptr;
    size_t bytes = 0;
    Batch(int n, int q_len, int first = 5) {
        std::vector<int32_t> kv, q;
        for (int i = 0; i < n; ++i) { kv.push_back(q_len + first + 37 * i % 400); q.push_back(q_len); }
        if (pk_pack_plan(kv.data(), q.data(), nullptr, nullptr, n, 2048, 4, &plan) != PK_OK) std::abort();
        bytes = pk_workspace_bytes(plan, HQ, HKV, D, PK_BF16);
        memory.assign(bytes + 256, '\xEE');
        ws = memory.data() + (256 - reinterpret_cast<uintptr_t>(memory.data()) % 256) % 256;
    }
    Batch(const Batch&) = delete;
    ~Batch() { pk_plan_destroy(plan); }
    int call(const std::string& what, Stream& s) {
        current = plan;
        void* const t = tensor;
        if (what == "bind") return pk_plan_bind(plan, HQ, HKV, D, PK_BF16, ws, bytes, &s);
        if (what == "prefill") return pk_packed_prefill_attn(plan, t, t, t, t, 1.f, HQ, HKV, D, PK_BF16, PK_BF16, ws, bytes, &s);
        if (what == "padded") return pk_padded_prefill_attn(plan, t, t, t, t, 1.f, HQ, HKV, D, PK_BF16, PK_BF16, ws, bytes, &s);
        if (what == "reorganize") return pk_kv_reorganize(plan, t, t, reinterpret_cast<int32_t*>(tensor), 1, 1 << 20, 1, HKV, D, PK_BF16, t, ws, bytes, &s);
        if (what == "append") return pk_kv_append(plan, t, t, t, 0, HKV, D, PK_BF16, ws, bytes, &s);
        if (what == "decode") return pk_packed_decode_attn(plan, t, t, t, 1.f, HQ, HKV, D, PK_BF16, PK_BF16, ws, bytes, &s);
        if (what == "static") return pk_packed_decode_attn_static(plan, t, t, t, 1.f, HQ, HKV, D, PK_BF16, PK_BF16, &s);
        std::abort();
    }
};
static int failures = 0;
#define CHECK(COND, ...) do { if (!(COND)) { ++failures; std::printf("line %d: ", __LINE__); std::printf(__VA_ARGS__); std::printf("\n"); } } while (0)

// A table copy that a capture has recorded is no copy yet: a call outside of it, or in another capture, makes its own.
static void captured() {
    struct { int q_len; const char *before, *inside; } cases[] = {
        {1, "bind", "prefill"}, {1, "bind", "padded"}, {3, "bind", "padded"}, {3, "", "prefill"}, {3, "bind", "bind"}, {3, "", "bind"}, {1, "", "bind"},
        {1, "", "reorganize"}, {1, "", "append"}, {1, "", "decode"}, {1, "decode", "prefill"}, {1, "", "static"}};
    for (const auto& c : cases) {
        const std::string inside = c.inside, after = inside != "bind" ? inside : c.q_len == 1 ? "decode" : "prefill";
        for (const bool again_captured : {false, true}) {
            std::memset(scratch, 0x11, sizeof(scratch));
            Batch b(40, c.q_len);
            Stream s;
            Graph dropped, g;
            if (*c.before) b.call(c.before, s);
            begin(s, dropped);
            CHECK(b.call(inside, s) == PK_OK, "%s captured", c.inside);
            CHECK(dropped.copies == 1, "%s captured: %d copies", c.inside, dropped.copies);
            if (inside != "bind") {                // the same capture needs it once
                CHECK(b.call(inside, s) == PK_OK && dropped.copies == 1, "%s twice in a capture: %d copies", c.inside, dropped.copies);
            }
            end(s);                                // never replayed
            launches = wrong = 0;
            if (again_captured) begin(s, g);
            CHECK(b.call(after, s) == PK_OK, "%s", after.c_str());
            if (again_captured) { end(s); replay(g); }
            CHECK(launches == 1 && wrong == 0, "%s behind a capture of %s that never ran%s: %d launches, %d of them without their tables", after.c_str(), c.inside,
                  again_captured ? " (captured too)" : "", launches, wrong);
            if (!again_captured) {                 // from here on a captured call is its launch alone
                Graph h;
                begin(s, h);
                CHECK(b.call(after, s) == PK_OK, "%s", after.c_str());
                end(s);
                CHECK(h.nodes.size() == 1 && h.copies == 0, "%s with its tables in place: %zu nodes, %d copies", after.c_str(), h.nodes.size(), h.copies);
                launches = wrong = 0;
                replay(h);
                replay(dropped);
                CHECK(wrong == 0, "replays of %s: %d without their tables", c.inside, wrong);
            }
        }
    }
}

// Buffers that graphs read from for good are no part of the pool: they neither use it up nor are they waited for.
static void graphs() {
    Batch b(6, 3);
    Stream s;
    Graph g;
    int copies = 0;
    auto capture = [&](int n) {
        for (int x = 0; x < n; ++x) {
            begin(s, g);
            CHECK(b.call("bind", s) == PK_OK, "captured bind %d", x);
            end(s);
            ++copies;
        }
        CHECK(g.copies == copies, "%d copies of %d captured", g.copies, copies);
    };
    capture(20);
    s.held = true;
    for (int x = 0; x < 10; ++x) CHECK(b.call("bind", s) == PK_OK, "bind %d", x);
    CHECK(waits == 0, "%d turns of waiting for buffers of graphs", waits);
    s.run();
    capture(100);
    for (int x = 0; x < 10; ++x) CHECK(b.call("bind", s) == PK_OK, "bind %d", x);
    CHECK(waits == 0 && pageable == 0, "behind 120 captured uploads: %d turns of waiting, %d copies from pageable memory", waits, pageable);
    s.run();
    s.held = false;
    const std::vector<int32_t> host = b.plan->tables.host;
    const pk::TableRef tiles = b.plan->tables.packed.tiles;
    if (pk_workspace_bytes(b.plan, 64, 8, 64, PK_BF16) == 0) std::abort();         // (the plan's own memory has other tables)
    launches = wrong = 0;
    for (Work& w : g.nodes) {                      // every graph its own tables, whatever has gone through the pool since
        std::memset(b.ws, 0xEE, b.bytes);
        w();
        expects(&s, b.ws + tiles.offset, host, tiles);
    }
    CHECK(launches == 120 && wrong == 0, "%d of %d replays without their tables", wrong, launches);
}

// A host far ahead of the GPU: no upload waits while the pool may grow; then one waits for a buffer behind uploads of its own stream, in place of a copy from pageable
// memory, for which the host would wait until the stream has drained; and never because of another stream.
static void ahead() {
    constexpr int POOL = 64;
    Batch b(6, 3), c(6, 1);
    Stream s, other;
    s.held = true;
    for (int x = 0; x < POOL; ++x) CHECK(b.call("bind", s) == PK_OK, "bind %d", x);
    CHECK(waits == 0 && pageable == 0 && pinned.size() == POOL, "%d uploads: %d turns of waiting, %d copies from pageable memory, %zu buffers", POOL, waits, pageable, pinned.size());
    int turns = 0;
    on_wait = [&] { if (++turns % 3 == 0) s.run(1); };
    for (int x = 0; x < 20; ++x) CHECK(b.call("bind", s) == PK_OK, "bind %d", POOL + x);
    CHECK(turns == 60 && pageable == 0 && s.queue.size() == POOL && pinned.size() == POOL, "with buffers that come back: %d turns of waiting, %d copies from pageable memory, %zu uploads in "
          "flight, %zu buffers", turns, pageable, s.queue.size(), pinned.size());
    on_wait = nullptr;
    waits = 0;
    CHECK(b.call("bind", other) == PK_OK, "bind on an idle stream");
    CHECK(waits == 0 && pageable == 1 && s.queue.size() == POOL, "an idle stream: %d turns of waiting, %d copies from pageable memory, %zu uploads left", waits, pageable, s.queue.size());
    CHECK(c.call("static", s) == PK_OK, "static");
    CHECK(waits == 0 && pageable == 2, "the fixed scratch: %d turns of waiting, %d copies from pageable memory", waits, pageable);
    s.run();
    for (int x = 0; x < POOL; ++x) CHECK(b.call("bind", s) == PK_OK, "bind %d", x);
    CHECK(waits == 0 && pageable == 2 && s.queue.size() == POOL, "again: %d turns of waiting, %d copies from pageable memory", waits, pageable);
    CHECK(b.call("bind", s) == PK_OK, "bind on a stream that stands still");
    CHECK(waits > 0 && pageable == 3, "a stream that stands still: %d turns of waiting, %d copies from pageable memory", waits, pageable);
    Graph g;
    s.run();
    for (int x = 0; x < POOL; ++x) CHECK(b.call("bind", s) == PK_OK, "bind %d", x);
    waits = 0;
    begin(s, g);
    CHECK(b.call("bind", s) == PK_OK && g.copies == 1, "captured bind");
    end(s);
    CHECK(waits == 0, "captured: %d turns of waiting", waits);
    s.run();
}

int main(int, char** argv) {
    const std::string check = argv[1];
    if (check == "captured") captured();
    else if (check == "graphs") graphs();
    else if (check == "ahead") ahead();
    else return 2;
    return failures ? 1 : 0;
}
