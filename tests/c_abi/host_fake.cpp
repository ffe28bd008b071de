// Host runtime of libes on a device made of host memory: the HIP calls it uses are defined here and
// the kernel launchers record what they were given, so a handle's life (tables, options, waits,
// allocations) can be followed without a GPU.  Test program: argv[1] names the check, exit status 0 = passed.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <vector>

#include "es.h"
#include "es_internal.h"

static std::map<char*, size_t> g_live;          // what the handle holds of the caller's allocator
static int g_allocs = 0, g_frees = 0, g_waits = 0;

static void* dev_alloc(size_t bytes, void*)
{
    void* p = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
    g_live[(char*)p] = bytes;
    ++g_allocs;
    return p;
}
static void dev_free(void* p, void*)
{
    g_live.erase((char*)p);
    ++g_frees;
    std::free(p);
}

// Host memory: no single allocation above the limit.
static size_t g_host_limit = ~(size_t)0;
#ifndef __SANITIZE_ADDRESS__                     // which has an operator new of its own
void* operator new(size_t n)
{
    void* p = n > g_host_limit ? nullptr : std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
#endif

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::aligned_alloc(256, (n + 255) / 256 * 256); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { ++g_waits; return hipSuccess; }
// what is asked about any stream: 0 = runs, 1 = is captured, -1 = cannot be said
static int g_capturing = 0;
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st)
{
    *st = g_capturing == 1 ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return g_capturing < 0 ? hipErrorStreamCaptureImplicit : hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}

namespace es {
// What the last reduce was launched with, and a copy of its tiles.
static const Tile* l_tiles;
static uint32_t l_n, l_big;
static ReduceShape l_shape;
static std::vector<Tile> l_copy;

hipError_t launch_ring_reduce(hipStream_t, const Tile* t, uint32_t n, uint32_t n_big, const float* const*, uint32_t,
                              float*, float*, float*, float, float, ReduceShape sh)
{
    l_tiles = t; l_n = n; l_big = n_big; l_shape = sh;
    l_copy.assign(t, t + n);
    return hipSuccess;
}
hipError_t launch_sgd(hipStream_t, float*, float*, const float*, uint64_t, float, float, bool) { return hipSuccess; }
hipError_t launch_copy_f32(hipStream_t, float*, const float*, uint64_t) { return hipSuccess; }
hipError_t launch_copy_runs(hipStream_t, const CopyRuns&) { return hipSuccess; }
hipError_t launch_patch_slots(hipStream_t, const float**, const InPlace&) { return hipSuccess; }
hipError_t launch_ctx(hipStream_t, const Piece*, uint32_t, uint8_t*, const uint8_t*, CtxDir) { return hipSuccess; }
hipError_t launch_est_boundary(hipStream_t, const CopyRuns&, const Piece*, uint32_t, uint8_t*, const uint8_t*, CtxDir) { return hipSuccess; }
hipError_t launch_sgd_clip(hipStream_t, float*, float*, const float*, uint64_t, const float*, float, float, float, float, bool) { return hipSuccess; }
hipError_t launch_bn_batch_stats(hipStream_t, const float*, uint32_t, uint32_t, uint32_t, float*, float*, float*) { return hipSuccess; }
hipError_t launch_copy_bytes(hipStream_t, uint8_t*, const uint8_t*, uint64_t) { return hipSuccess; }
// The last norm: its partials and, in the form that has them, its counters.
static float* n_part;
static uint32_t* n_counters;
hipError_t launch_sq_norm(hipStream_t, const float*, uint64_t, float* part, float*)
{
    n_part = part; n_counters = nullptr;
    return hipSuccess;
}
hipError_t launch_sq_norm_counted(hipStream_t, const float*, uint64_t, float* part, float*, uint32_t* counters)
{
    n_part = part; n_counters = counters;
    return hipSuccess;
}
hipError_t launch_sq_norm_static(hipStream_t, const float*, uint64_t, float*) { return hipSuccess; }

// The last mask: which launcher drew it, from which state, with which counters.
enum { kNone, kShort, kLong, kCaptured };
static int m_form;
static uint64_t* m_state;
static uint32_t* m_counters;
static hipError_t drew(int form, uint64_t* state, uint32_t* counters)
{
    m_form = form; m_state = state; m_counters = counters;
    return hipSuccess;
}
hipError_t launch_dropout_mask(hipStream_t, uint64_t* st, uint8_t*, uint64_t, uint64_t) { return drew(kShort, st, nullptr); }
hipError_t launch_dropout_mask_captured(hipStream_t, uint64_t* st, uint8_t*, uint64_t, uint64_t) { return drew(kCaptured, st, nullptr); }
hipError_t launch_dropout_mask_long(hipStream_t, uint64_t* st, uint8_t*, uint64_t, uint64_t, uint32_t* c) { return drew(kLong, st, c); }
}  // namespace es
using namespace es;

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); return 1; } } while (0)

struct Job {
    es_handle* h = nullptr;
    uint32_t N, A;
    uint64_t P;
    std::vector<float> avg;
    Job(uint32_t n, uint64_t p, uint32_t a = 1) : N(n), A(a), P(p), avg(p + 64)
    {
        es_bucket b[2] = {{0, p / 3}, {p / 3, p - p / 3}};
        es_bucket_layout lay = {p, 2, b, a, 0, nullptr, dev_alloc, dev_free, nullptr};
        if (es_init(&h, n, &lay) != ES_OK) h = nullptr;
    }
    ~Job() { if (h) es_destroy(h); }
    int reduce()
    {
        for (uint32_t e = 0; e < N; ++e) {
            const float* g = es_grad_slot(h, e, 0);
            const int rc = es_accumulate_many(h, 1, &e, &g);
            if (rc != ES_OK) return rc;
        }
        return es_ring_order_reduce(h, (float*)(((uintptr_t)avg.data() + 15) & ~(uintptr_t)15));
    }
};

// Whether `n` tiles from `t` on lie in memory the handle still holds.
static bool held(const Tile* t, size_t n)
{
    for (const auto& m : g_live)
        if ((const char*)t >= m.first && (const char*)(t + n) <= m.first + m.second) return true;
    return false;
}

// A launch captured into a graph keeps its tables: the options that name a launch shape without
// changing the decomposition neither wait, allocate nor free, and no option gives the first table back.
static int check_options()
{
    for (uint32_t N : {4u, 9u, 48u}) {
        Job j(N, 70001);
        CHECK(j.h && j.reduce() == ES_OK && l_n > 0 && l_shape.wave_width != 0);
        const Tile* tiles = l_tiles;
        const std::vector<Tile> wave = l_copy;
        const struct { const char* name; int64_t value; } fields[] = {
            {"reduce_unroll", 4}, {"reduce_rank_batch", 2}, {"reduce_lds_pad_kib", 16}, {"nontemporal", 0}, {"nontemporal_pv", 1}};
        for (const auto& f : fields) {
            const int a = g_allocs, fr = g_frees, w = g_waits;
            CHECK(es_set_option(j.h, f.name, f.value) == ES_OK);
            CHECK(g_allocs == a && g_frees == fr && g_waits == w);
        }
        CHECK(j.reduce() == ES_OK && l_shape.wave_width == 0 && l_shape.unroll == 4 && l_shape.rank_batch == 2 && l_shape.lds_pad_kib == 16 && !l_shape.nontemporal);
        const std::vector<Tile> tiled = l_copy;
        const Tile* tiled_at = l_tiles;
        for (int64_t v : {512, 1024, 2048}) CHECK(es_set_option(j.h, "reduce_tile_elems", v) == ES_OK && j.reduce() == ES_OK);
        CHECK(l_n == tiled.size() && std::memcmp(l_copy.data(), tiled.data(), l_n * sizeof(Tile)) == 0);
        CHECK(held(tiles, wave.size()) && std::memcmp(tiles, wave.data(), wave.size() * sizeof(Tile)) == 0);
        CHECK(held(tiled_at, tiled.size()) && std::memcmp(tiled_at, tiled.data(), tiled.size() * sizeof(Tile)) == 0);
    }
    CHECK(g_live.empty());                      // es_destroy has given everything back
    return 0;
}

static int64_t option(es_handle* h, const char* name)
{
    int64_t v = -99;
    return es_get_option(h, name, &v) == ES_OK ? v : -98;
}

// The automatic launch shape can be seen, left and taken up again, and gives the same launch as before.
static int check_auto()
{
    for (uint32_t N : {1u, 9u, 64u, 65u}) {
        Job j(N, 70001);
        CHECK(j.h && option(j.h, "reduce_auto") == 1 && j.reduce() == ES_OK);
        const int width = l_shape.wave_width;
        const std::vector<Tile> tiles = l_copy;
        CHECK((width != 0) == (N <= 64) && option(j.h, "reduce_wave_width") == width);
        CHECK(es_set_option(j.h, "reduce_lds_pad_kib", -1) == ES_OK && es_set_option(j.h, "nontemporal", 1) == ES_OK);
        CHECK(option(j.h, "reduce_auto") == 1);
        const char* leave[] = {"reduce_unroll", "reduce_rank_batch", "reduce_tile_elems", "reduce_big_unroll", "reduce_big_rank_batch", "nontemporal"};
        for (const char* name : leave) {
            const int64_t was = option(j.h, name);
            CHECK(es_set_option(j.h, name, std::strcmp(name, "nontemporal") ? was : 0) == ES_OK);
            CHECK(option(j.h, "reduce_auto") == 0 && option(j.h, "reduce_wave_width") == 0);
            CHECK(j.reduce() == ES_OK && l_shape.wave_width == 0);
            CHECK(es_set_option(j.h, name, was) == ES_OK && es_set_option(j.h, "reduce_auto", 1) == ES_OK);
            CHECK(option(j.h, "reduce_wave_width") == width && j.reduce() == ES_OK && l_shape.wave_width == width);
            CHECK(l_copy.size() == tiles.size() && std::memcmp(l_copy.data(), tiles.data(), tiles.size() * sizeof(Tile)) == 0);
        }
        CHECK(es_set_option(j.h, "reduce_auto", 2) == ES_EINVAL && es_set_option(j.h, "reduce_wave_width", 4) == ES_EINVAL);
    }
    return 0;
}

// Gradients in host memory, all of them or some, are not for the wave-tile form.
static int check_host_slots()
{
    Job j(4, 70001);
    const uint32_t one[4] = {0, 0, 0, 0}, slots[4] = {0, 1, 2, 3}, two[4] = {0, 0, 1, 1}, slots2[4] = {0, 1, 0, 1};
    CHECK(j.h && j.reduce() == ES_OK && l_shape.wave_width);
    CHECK(es_set_option(j.h, "host_slots", 1) == ES_OK && j.reduce() == ES_OK && l_shape.wave_width);   // from the next grouping on
    CHECK(es_set_grouping(j.h, 1, one, slots) == ES_OK && option(j.h, "slots_on_host") == 4);
    CHECK(option(j.h, "reduce_wave_width") == 0 && j.reduce() == ES_OK && !l_shape.wave_width && option(j.h, "reduce_auto") == 1);
    CHECK(es_set_option(j.h, "host_slots", 0) == ES_OK && es_set_option(j.h, "hbm_slot_budget_mib", 1) == ES_OK);
    CHECK(es_set_grouping(j.h, 2, two, slots2) == ES_OK && option(j.h, "slots_on_host") == 2);
    CHECK(option(j.h, "reduce_wave_width") == 0 && j.reduce() == ES_OK && !l_shape.wave_width);
    CHECK(es_set_option(j.h, "hbm_slot_budget_mib", -1) == ES_OK && es_set_grouping(j.h, 2, two, slots2) == ES_OK);
    CHECK(option(j.h, "slots_on_host") == 0 && option(j.h, "reduce_wave_width") && j.reduce() == ES_OK && l_shape.wave_width);
    return 0;
}

// The tiles of the last launch against the ring's chunks: each in one chunk of one bucket, opened by the
// rank of the chunk, and all of them [0, P) without a gap.
static bool tiles_follow_the_ring(const Job& j)
{
    const uint64_t start[3] = {0, j.P / 3, j.P};
    uint64_t next = 0;
    std::vector<Tile> t = l_copy;               // big tiles are listed first
    std::sort(t.begin(), t.end(), [](const Tile& x, const Tile& y) { return x.off < y.off; });
    for (const Tile& x : t) {
        const int b = x.off >= start[1] ? 1 : 0;
        const uint64_t len = start[b + 1] - start[b], chunk = ((len + j.N - 1) / j.N + j.A - 1) / j.A * j.A;
        const uint64_t lo = x.off - start[b], hi = lo + x.len;
        if (x.off != next || x.len == 0 || hi > len || lo / chunk != x.rank0 || (hi - 1) / chunk != x.rank0) return false;
        next += x.len;
    }
    return next == j.P;
}

// Which form a job's size chooses, on both sides of every line.
static int check_rule()
{
    const struct { uint32_t n; uint64_t p; int width, batch, pad; } lines[] = {
        {1, 1499999, 4, 1, 32}, {1, 1500000, 4, 1, 0}, {2, 1500000, 4, 2, 0}, {7, 1499999, 4, 4, 32}, {7, 1500000, 4, 4, 0},
        {7, 7999999, 4, 4, 0}, {7, 8000000, 0, 0, 0}, {8, 4999999, 4, 8, 32}, {8, 5000000, 0, 0, 0}, {24, 4999999, 4, 4, 64}, {64, 5000000, 0, 0, 0}, {10, 8000001, 0, 0, 0}, {8, 299999, 1, 8, 0}, {8, 300000, 4, 8, 32}, {64, 131072, 1, 64, 0},
        {64, 131073, 1, 16, 0}, {23, 2000000, 4, 8, 32}, {24, 1999999, 4, 4, 32}, {24, 2000000, 4, 4, 64}, {65, 100000, 0, 0, 0}};
    for (const auto& l : lines) {
        Job j(l.n, l.p);
        CHECK(j.h && j.reduce() == ES_OK && l_shape.wave_width == l.width);
        if (l.width) CHECK(l_shape.wave_batch == l.batch && l_shape.wave_pad_kib == l.pad);
        for (const Tile& t : l_copy) CHECK(!l.width || t.len <= 64u * l.width);
        CHECK(tiles_follow_the_ring(j));
        CHECK(es_set_option(j.h, "reduce_auto", 0) == ES_OK && j.reduce() == ES_OK && tiles_follow_the_ring(j));
    }
    for (uint32_t a : {1u, 3u, 4u, 64u})
        for (uint64_t p : {1ull, 5ull, 63ull, 64ull, 200ull, 1001ull, 70001ull, 300007ull, 2000003ull})
            for (uint32_t n : {1u, 2u, 7u, 8u, 33u, 64u}) {
                Job j(n, p, a);
                CHECK(j.h && j.reduce() == ES_OK && l_shape.wave_width && tiles_follow_the_ring(j));
                for (const Tile& t : l_copy) CHECK(t.len <= 64u * l_shape.wave_width);
            }
    const struct { uint32_t n; uint64_t p; int streamed; } policy[] = {
        {1, 13999999, 0}, {1, 14000000, 1}, {31, 4999999, 0}, {32, 999999, 0}, {32, 1000000, 1}, {64, 4999999, 1}, {64, 5000000, 0}};
    for (const auto& l : policy) {
        Job j(l.n, l.p);
        CHECK(j.h && j.reduce() == ES_OK && l_shape.nontemporal_pv == l.streamed && option(j.h, "nontemporal_pv") == l.streamed);
        const ReduceShape chosen = l_shape;     // the option set to what it is: the same launch
        CHECK(es_set_option(j.h, "nontemporal_pv", l.streamed) == ES_OK && j.reduce() == ES_OK);
        CHECK(std::memcmp(&chosen, &l_shape, sizeof(chosen)) == 0);
    }
    return 0;
}

// Words the handle holds, all zero.
static bool zeros_held(const uint32_t* w, size_t n)
{
    for (const auto& m : g_live)
        if ((const char*)w >= m.first && (const char*)(w + n) <= m.first + m.second)
            return std::all_of(w, w + n, [](uint32_t v) { return v == 0; });
    return false;
}

// A long mask counts its workgroups on words of the handle; one that is recorded into a graph, which can be replayed
// when the handle has regrouped its ESTs or is gone, and beside other draws, gets none.
static int check_masks()
{
    const uint64_t segs[5] = {24, 16, 7, 16, 40};
    es_bucket b = {0, 4};
    es_bucket_layout lay = {4, 1, &b, 4, 5, segs, dev_alloc, dev_free, nullptr};
    es_handle* h = nullptr;
    CHECK(es_init(&h, 3, &lay) == ES_OK);
    alignas(16) static uint64_t live[2][5][8];
    static uint8_t mask[kShortMask + 1];
    const uint32_t workers[3] = {0, 1, 1}, slots[3] = {0, 0, 1};
    void* ptrs[2][5];
    for (int w = 0; w < 2; ++w)
        for (int j = 0; j < 5; ++j) ptrs[w][j] = live[w][j];
    const uint32_t* counters = nullptr;
    for (int round = 0; round < 3; ++round) {
        if (round == 1) CHECK(es_set_grouping(h, 2, workers, slots) == ES_OK);
        for (uint32_t w = 0; w < (round ? 2u : 1u); ++w)        // in the last round the same states, the other way round
            CHECK(es_bind_live_state(h, w, ptrs[round == 2 ? 1 - w : w]) == ES_OK);
        for (uint32_t e = 0; e < 3; ++e)
            for (uint32_t seg : {1u, 3u}) {
                uint64_t* state = live[round == 0 ? 0 : round == 1 ? workers[e] : 1 - workers[e]][seg];
                for (int capturing : {1, -1, 0}) {
                    g_capturing = capturing;
                    CHECK(es_dropout_mask(h, e, seg, mask, kShortMask + 1, 0.5) == ES_OK && m_state == state);
                    CHECK(m_form == (capturing ? kCaptured : kLong));
                    if (!capturing) {
                        CHECK(zeros_held(m_counters, kArrivalWords) && (!counters || m_counters == counters));
                        counters = m_counters;                  // not the regrouping's to free
                    }
                    CHECK(es_dropout_mask(h, e, seg, mask, kShortMask, 0.5) == ES_OK && m_form == kShort && m_state == state);
                }
            }
        alignas(16) float x[4] = {}, out[2];    // the norm has words of its own
        CHECK(es_grad_sq_norm(h, x, out) == ES_OK && zeros_held(n_counters, kArrivalWords));
        CHECK(n_counters + kArrivalWords <= counters || counters + kArrivalWords <= n_counters);
        m_form = kNone;
        CHECK(es_dropout_mask(h, 0, 0, mask, kShortMask + 1, 0.5) == ES_EINVAL && m_form == kNone);
    }
    CHECK(es_destroy(h) == ES_OK && g_live.empty());
    return 0;
}

// The norm's partials, and the counters of its one-launch form on lines of their own.
static int check_norms()
{
    const uint64_t block = 4096;
    for (uint64_t blocks : {1ull, 2ull, 31ull, 32ull, 33ull, 2047ull, 2048ull, 2049ull})
        for (uint64_t n : {blocks * block, (blocks - 1) * block + 1}) {
            Job j(1, n);
            float* x = (float*)(((uintptr_t)j.avg.data() + 15) & ~(uintptr_t)15);
            float out[2];
            CHECK(j.h && es_grad_sq_norm(j.h, x, out) == ES_OK && (n_counters != nullptr) == (blocks <= kCountedBlocks));
            std::fill(n_part, n_part + blocks, 1.0f);           // all of them, and no counter
            if (!n_counters) continue;
            CHECK(zeros_held(n_counters, kArrivalWords) && (uintptr_t)n_counters % 128 == 0);
            CHECK(j.reduce() == ES_OK && (const char*)(l_tiles + l_n) <= (const char*)n_counters);
        }
    CHECK(g_live.empty());
    return 0;
}

// An EST is named once per es_accumulate_many call, and once per step; a call that is refused leaves nothing behind.
static int check_many()
{
    Job j(5, 4001);
    const float* g[6];
    for (uint32_t e = 0; e < 5; ++e) g[e] = es_grad_slot(j.h, e, 0);
    g[5] = g[0];
    const uint32_t all[6] = {0, 1, 2, 3, 4, 0}, far[2] = {3, 5};
    for (int step = 0; step < 3; ++step) {
        CHECK(es_accumulate_many(j.h, 6, all, g) == ES_ESTATE && es_accumulate_many(j.h, 2, far, g + 3) == ES_EINVAL);
        CHECK(es_accumulate_many(j.h, 3, all, g) == ES_OK && es_accumulate_many(j.h, 3, all + 2, g + 2) == ES_ESTATE);
        CHECK(es_accumulate_many(j.h, 2, all + 3, g + 3) == ES_OK && es_accumulate_many(j.h, 1, all + 4, g + 4) == ES_ESTATE);
        CHECK(es_accumulate_many(j.h, 0, nullptr, nullptr) == ES_OK);
        CHECK(es_ring_order_reduce(j.h, (float*)(((uintptr_t)j.avg.data() + 15) & ~(uintptr_t)15)) == ES_OK);
    }
    return 0;
}

// Where the host's memory does not suffice for the tile tables, es_init says so and holds nothing.
static int check_no_memory()
{
    es_bucket b = {0, 1u << 22};
    es_bucket_layout lay = {1u << 22, 1, &b, 4, 0, nullptr, dev_alloc, dev_free, nullptr};
    for (size_t limit : {(size_t)1 << 15, (size_t)1 << 16}) {
        es_handle* h = nullptr;
        g_host_limit = limit;
        const int rc = es_init(&h, 4, &lay);
        g_host_limit = ~(size_t)0;
        CHECK(rc == ES_ENOMEM && !h && g_live.empty());
    }
    return 0;
}

int main(int argc, char** argv)
{
    const char* what = argc > 1 ? argv[1] : "";
    int rc = 2;
    if (!std::strcmp(what, "options")) rc = check_options();
    if (!std::strcmp(what, "auto")) rc = check_auto();
    if (!std::strcmp(what, "host slots")) rc = check_host_slots();
    if (!std::strcmp(what, "rule")) rc = check_rule();
    if (!std::strcmp(what, "masks")) rc = check_masks();
    if (!std::strcmp(what, "norms")) rc = check_norms();
    if (!std::strcmp(what, "many")) rc = check_many();
    if (!std::strcmp(what, "no memory")) rc = check_no_memory();
    if (rc == 0) std::printf("%s: passed\n", what);
    return rc;
}
