// When a staging copy goes behind main by an event and when main is known to be idle, on a device made of host memory (the
// doubles of host_fake.cpp) whose streams answer what this program says.  Exit status 0 = passed.
#define hipEventRecord fake_hipEventRecord
#define main fake_main
#include "host_fake.cpp"
#undef main
#undef hipEventRecord

static int g_records = 0, g_asked_idle = 0, g_asked_done = 0;
static bool g_idle = false, g_done = true;
extern "C" hipError_t hipEventRecord(hipEvent_t, hipStream_t) { ++g_records; return hipSuccess; }
static bool idle(hipStream_t) { ++g_asked_idle; return g_idle; }
static bool done(hipEvent_t) { ++g_asked_done; return g_done; }

// n hand-offs: how many went by an event
static int hand_offs(Job& j, int n)
{
    std::vector<float> g(j.P);
    const int before = g_records;
    for (int k = 0; k < n; ++k) {
        // a step of one copy: the second bucket's gradient is in its slot already
        if (es_accumulate(j.h, 0, 0, g.data()) != ES_OK) return -1;
        const int mine = g_records;
        const float* slot = es_grad_slot(j.h, 0, 1);
        if (es_accumulate(j.h, 0, 1, slot) != ES_OK || g_records != mine) return -1;
        if (es_ring_order_reduce(j.h, (float*)(((uintptr_t)j.avg.data() + 15) & ~(uintptr_t)15)) != ES_OK) return -1;
        g_records = mine;                        // the reduce's own hand-off back to main is not counted
    }
    return g_records - before;
}

// The calls beside staging record the same event on main: into a capture it is not asked afterwards, else it is.
static int other_calls()
{
    const uint64_t seg = 16;
    es_bucket b[2] = {{0, 64}, {64, 64}};
    es_bucket_layout lay = {128, 2, b, 4, 1, &seg, dev_alloc, dev_free, nullptr};
    es_handle* h = nullptr;
    alignas(16) static uint64_t live[2];
    alignas(16) static float g[128];
    void* ptrs[1] = {live};
    const uint32_t ids[2] = {0, 1};
    const float* grads[2] = {g, g + 64};
    CHECK(es_init(&h, 2, &lay) == ES_OK && es_bind_live_state(h, 0, ptrs) == ES_OK);
    CHECK(es_set_streams(h, (void*)48, (void*)64, (void*)32) == ES_OK);
    g_idle = false;
    for (int call = 0; call < 4; ++call)
        for (int c : {0, 1, -1}) {
            // a record outside any capture, by staging, and the ladder back at its start
            CHECK(es_set_streams(h, (void*)48, (void*)64, (void*)32) == ES_OK);
            CHECK(es_accumulate(h, 0, 0, g) == ES_OK && es_accumulate(h, 0, 1, g + 64) == ES_OK);
            for (int k = 0; k < 2; ++k) CHECK(es_accumulate(h, 1, k, g + 64 * k) == ES_OK);
            CHECK(es_ring_order_reduce(h, g) == ES_OK);
            g_capturing = c;
            if (call == 0) CHECK(es_ctx_restore(h, 0) == ES_OK);
            if (call == 1) CHECK(es_ctx_save(h, 0) == ES_OK);
            if (call == 2) CHECK(es_ctx_switch(h, 0, 1) == ES_OK);
            if (call == 3) CHECK(es_est_boundary(h, 0, 1, 0, nullptr, nullptr) == ES_OK);
            g_capturing = 0;
            g_asked_done = g_asked_idle = 0;
            CHECK(es_accumulate_batch(h, 0, 2, ids, grads) == ES_OK);
            CHECK(g_asked_done == (c == 0) && g_asked_idle == 1);
            for (int k = 0; k < 2; ++k) CHECK(es_accumulate(h, 1, k, g + 64 * k) == ES_OK);
            CHECK(es_ring_order_reduce(h, g) == ES_OK);
        }
    return es_destroy(h) == ES_OK ? 0 : 1;
}

int main()
{
    Job j(1, 4096);
    CHECK(j.h && es_set_streams(j.h, (void*)16, (void*)16, (void*)32) == ES_OK);
    // no answers at all: always an event
    CHECK(!stream_probe.idle && hand_offs(j, 5) == 5);
    stream_probe = StreamProbe{idle, done};
    // idle: never
    g_idle = true;
    CHECK(hand_offs(j, 5) == 0 && g_asked_idle == 5 && g_asked_done == 0);
    // busy: always, asked ever more seldom (after 3, 15 and 63 hand-offs)
    g_idle = false;
    g_asked_idle = 0;
    CHECK(hand_offs(j, 1) == 1 && g_asked_idle == 1);
    CHECK(hand_offs(j, 3) == 3 && g_asked_idle == 1);
    CHECK(hand_offs(j, 16) == 16 && g_asked_idle == 2);
    CHECK(hand_offs(j, 64) == 64 && g_asked_idle == 3 && g_asked_done == 2);
    CHECK(hand_offs(j, 640) == 640 && g_asked_idle == 13);
    // an event of ours that is still ahead: nothing else is asked, and that is no refusal
    CHECK(hand_offs(j, 63) == 63);
    g_done = false;
    g_asked_idle = g_asked_done = 0;
    CHECK(hand_offs(j, 8) == 8 && g_asked_idle == 0 && g_asked_done > 0);
    // idle again: the first answer is used at once, and after six of them every hand-off is asked for
    g_done = g_idle = true;
    CHECK(hand_offs(j, 400) < 130);
    g_asked_idle = 0;
    CHECK(hand_offs(j, 10) == 0 && g_asked_idle == 10);
    // captured, or not to be said: an event, and nothing is asked, nor is that event afterwards
    for (int c : {1, -1}) {
        g_capturing = c;
        g_asked_idle = g_asked_done = 0;
        CHECK(hand_offs(j, 4) == 4 && g_asked_idle == 0 && g_asked_done == 0);
        g_capturing = 0;
        CHECK(hand_offs(j, 1) == 0 && g_asked_idle == 1 && g_asked_done == 0);
    }
    // another main: what was learned of the one before says nothing, and its event is not asked
    g_idle = false;
    CHECK(hand_offs(j, 100) == 100);
    CHECK(es_set_streams(j.h, (void*)48, (void*)48, (void*)32) == ES_OK);
    g_idle = true;
    g_asked_idle = g_asked_done = 0;
    CHECK(hand_offs(j, 1) == 0 && g_asked_idle == 1 && g_asked_done == 0);
    CHECK(hand_offs(j, 20) == 0 && g_asked_idle == 21);
    if (other_calls() != 0) return 1;
    // one stream for both: neither
    CHECK(es_set_streams(j.h, (void*)16, (void*)16, (void*)16) == ES_OK);
    g_asked_idle = 0;
    CHECK(hand_offs(j, 4) == 0 && g_asked_idle == 0);
    std::printf("passed\n");
    return 0;
}
