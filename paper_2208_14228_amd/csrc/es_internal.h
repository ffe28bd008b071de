// Internal interface between the host runtime (es_api.cpp) and the gfx950
// kernels (es_kernels.hip).  Not part of the public boundary.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace es {

// One workgroup's share of the ring-ordered reduction: a contiguous range of
// the flat parameter space that lies inside a single ring chunk, so the rank
// the fold starts at is the same for every element of the tile.
struct Tile {
    uint64_t off;      // first element (flat parameter space)
    uint32_t len;      // elements
    uint32_t rank0;    // virtual rank whose gradient opens the fold (= chunk index)
};
static_assert(sizeof(Tile) == 16, "Tile is read with one 16-byte scalar load");

// One workgroup's share of a small-state context copy.
struct Piece {
    void*    live;       // device address inside a live state tensor
    uint64_t slot_off;   // byte offset inside the EST's context slot
    uint32_t nbytes;     // <= kPieceBytes
    uint32_t width;      // 16, 4 or 1: widest access both sides are aligned for
};
static_assert(sizeof(Piece) == 24, "Piece layout");

constexpr uint32_t kPieceBytes = 4096;
constexpr uint32_t kBlock = 256;
#ifndef ES_REDUCE_BLOCK
#define ES_REDUCE_BLOCK 256
#endif
constexpr uint32_t kReduceBlock = ES_REDUCE_BLOCK;   // lanes per workgroup of the ring-ordered reduce
constexpr int kBigEpilogue = 16;                     // vectors per lane per pass of a big tile's update epilogue

// Occupancy caps.  Measured on MI355X: the streaming kernels reach more of the HBM rate with few
// workgroups resident per CU (more resident workgroups = more DRAM regions open at once), as long
// as each has a few tens of KiB of loads in flight.  A launch reserves LDS it never touches so that
// only 160 KiB / reserve workgroups fit a CU.  Small-tile reduce: 2 per CU (3 below 4 ranks, where a
// workgroup has fewer loads in flight): +4-8 % at N = 2..10 on 26 M and 109 M parameters with
// nothing cache-resident; 1 per CU when every batch of the fold is full or nearly so (N = 8,
// N >= 10) and parameters and momentum stream (another +3-7 %; with parameters and momentum coming
// from the Infinity Cache one workgroup per CU is 7 % slower than two).  Update and norm kernels:
// 2 per CU, +4 % at 355 M parameters.
constexpr uint32_t kAuxLdsPad = 64u << 10;
inline uint32_t reduce_lds_pad(int option_kib, uint32_t n_ranks, bool streaming_pv, bool fused)
{
    if (option_kib >= 0) return (uint32_t)option_kib << 10;
    // below 4 ranks the unfused reduce is close to a copy and wants more waves still (5 per CU:
    // 57 -> 77 % of the HBM peak at N = 1, 70 -> 80 % at N = 3 on 109 M parameters)
    if (n_ranks < 4) return fused ? 53u << 10 : 32u << 10;
    if (streaming_pv && (n_ranks == 8 || n_ranks >= 10)) return 160u << 10;
    return 64u << 10;
}
// Lanes per workgroup of the staging copies: one wave for long ones, two for short ones, which the
// rate of starting workgroups bounds as much as memory (0.5 M floats 2.49 -> 2.32 us, 1 M 3.40 -> 3.06,
// 2 M 4.56 -> 3.87 together with plain loads; 4.2 M 7.03 -> 6.35, but from 7 M on 3-10 % worse).  In a staged
// step the plain loads also fill the caches that the reduce reads from: at 2.9 M floats per copy the short
// form gains 3-5 % up to 4 ranks, nothing at 5, and loses 5 % at 7, so the line is not drawn higher.
constexpr uint32_t kCopyBlock = 64;
constexpr uint32_t kCopyBlockShort = 128;
constexpr uint64_t kShortCopy = 3ull << 20;      // floats of one call
inline uint32_t copy_block(uint64_t floats) { return floats < kShortCopy ? kCopyBlockShort : kCopyBlock; }

// Entries of the rank -> gradient-base table that are redirected for one reduce
// (gradients taken in place from caller memory, no staging copy).
constexpr uint32_t kMaxInPlace = 16;            // entries one patch launch carries
struct InPlace {
    uint32_t     n;
    uint32_t     rank[kMaxInPlace];
    const float* ptr[kMaxInPlace];      // flat parameter order, 16-byte aligned
};
// table[patch.rank[k]] <- patch.ptr[k], stream-ordered (the values travel as a kernel argument)
hipError_t launch_patch_slots(hipStream_t s, const float** table, const InPlace& patch);

struct ReduceShape {
    int unroll;        // 16-byte vectors per lane per rank
    int rank_batch;    // ranks loaded before adds are issued
    int nontemporal;   // streaming hint on gradient loads
    int big_unroll;    // 0, or vectors per lane of a big tile (8, 16, 32): see k_ring_reduce_big
    int big_rank_batch;
    int nontemporal_pv; // streaming hint on parameter / momentum traffic of the update and on the store of the
                        // averaged gradient
    int lds_pad_kib = -1; // KiB of LDS reserved (and never touched) per workgroup of the small-tile kernel, to cap the
                          // workgroups resident per CU; -1 = default for the rank count (see reduce_lds_pad)
    // wave-tile form (k_ring_reduce_wave): floats per lane (1 or 4; 0 = the other kernels), ranks
    // loaded before adds are issued, KiB of LDS reserved per workgroup
    int wave_width = 0, wave_batch = 0, wave_pad_kib = 0;
};

// Whether parameters, momentum and the averaged gradient are streamed by default.  Cacheable over
// streaming time of a zero-copy step, fused / with clipping (reduce, norm and update kernel):
//
//                             1 to 5 M, 32 ranks +   8 to 10 M                12 M                    14 to 25 M
//  caches swept before        1.04-1.10 / 1.00-1.11  0.96-1.11 / 0.99-1.07  0.97-1.12 / 0.99-1.06  0.98-1.14 / 0.98-1.09
//  three jobs on one stream   0.99-1.08 / 0.98-1.03  0.86-1.00 / 0.98-1.04  0.93-1.03 / 1.00-1.07  1.00-1.11 / 0.99-1.08
//  three, on a stream each    0.94-1.05 / 0.92-1.11  0.87-0.99 / 0.92-1.02  0.91-1.06 / 0.93-1.05  0.93-1.10 / 0.95-1.10
//  one job, nothing else      0.95-1.09 / 0.97-1.05  0.88-1.04 / 0.96-1.03  0.91-0.99 / 0.97-1.02  0.88-1.05 / 0.95-1.04
//
// The first is a training job, whose model uses the caches between two reduces; in the others parameters
// and momentum can come back from the Infinity Cache, up to 37 M for one job and 12 M for three, unless the
// gradients push them out (32 ranks or more, wave tiles).  The line lies where streaming wins or ties in the
// first two and for the most part in the third.  One bit rules the update kernel as well, which alone in a
// loop takes 0.0893 ms for 0.0817 at 25.6 M; above 37 M streaming wins in every loop.
inline bool stream_pv(uint32_t N, uint64_t P)
{
    return P >= 14000000 || (N >= 32 && P >= 1000000 && P < 5000000);
}

// The wave-tile form where it is the faster one, by the rank count N and the parameter count P;
// returns false (and leaves the shape alone) where the other kernels are.  Measured on 13 rank counts
// x 9 sizes, fused, three jobs in turn (time of the other kernels over this one's):
//  - N <= 64: the slot table is one pointer per lane.
//  - P < 8 M, from 8 ranks on 5 M: 1.0-1.3 at 4 M, 1.0-2.2 at 1 M, 1.05-3.4 at 20 k.  Above, a wave's 1 KiB per
//    stream costs what the saved round trips gain.  On one stream / three jobs on a stream each:
//      12 ranks and more, zero-copy  1.05-1.12 / 0.92-0.97 at 4.5 M, 0.94-1.03 / 0.87-0.93 at 5.5 M, 0.90-0.98 /
//                                    0.93-0.99 at 6.5 M
//      the same, clipped             1.11-1.13 / 0.94-1.0, 0.98-1.03 / 0.90-1.0, 0.94-1.0 / 0.93-0.99
//      the same, staged              1.05-1.09 / 1.06-1.11, 1.02-1.05 / 1.0-1.16, 1.0-1.04 / 1.01-1.11
//      8 to 10 ranks, zero-copy      1.02-1.05 / 0.95-1.06 at 3.3 M, 0.96-0.99 / 0.94-0.99 at 5.5 M
//      8 to 10 ranks at 25.6 M, both with parameters and momentum streamed: fused 0.98-1.03 / 0.96-0.98,
//                                    staged and hooked 1.0, unfused 0.92-0.97
//    Where three zero-copy jobs fill the chip together the other kernels' long reads win from 2 M and 12 ranks
//    on, by 3-14 %; a job that has the GPU to itself is 1.05-1.75 times as fast by this form there, and the
//    line follows that.
//  - one float per lane below 300 k elements and from 8 ranks on, where four leave SIMDs without a wave
//    (1.1-1.7 x slower at 100 k, 1.0-1.1 x faster at 500 k); then as many ranks per batch as there are,
//    up to 64, while a SIMD has at most two waves (P <= 128 k), else 16.
//  - four floats per lane: batches of 4, of 8 from 8 to 23 ranks (a second round trip less: 1.0-1.1).
//  - 5 workgroups per CU, or 2 where there are many streams (1.01-1.04 from 24 ranks and 2 M on); no cap with
//    fewer than 8 ranks from 1.5 M elements on, where 5 per CU reach 0.86-0.98 of the other kernels' rate in
//    zero-copy steps of one to three ranks and no cap costs nothing: staged steps 1.0-1.2 on one stream and, as
//    three jobs on a stream each, 21.0 us for 21.2 at 2 ranks and 3.3 M, 38.1 for 39.1 at 4 and 4 M, 69.8 for
//    70.7 at 4 and 7.6 M.  (One wave per workgroup is 2-4 % faster alone, and slower than the other kernels
//    beside other jobs' copies: 22.2, 41.3 and 73.6 us.)
inline bool wave_shape(uint32_t N, uint64_t P, ReduceShape& sh)
{
    if (N == 0 || N > 64 || P >= (N < 8 ? 8000000u : 5000000u)) return false;
    auto pow2_up_to = [N](int b) {
        while (b > 1 && (uint32_t)b > N) b /= 2;
        return b;
    };
    if (N >= 8 && P < 300000) {
        sh.wave_width = 1;
        sh.wave_batch = pow2_up_to(P <= (128u << 10) ? 64 : 16);
        sh.wave_pad_kib = 0;
        return true;
    }
    sh.wave_width = 4;
    sh.wave_batch = pow2_up_to(N >= 8 && N < 24 ? 8 : 4);
    sh.wave_pad_kib = N >= 24 && P >= 2000000 ? 64 : 32;
    if (N < 8 && P >= 1500000) sh.wave_pad_kib = 0;
    return true;
}

// ring-ordered N-way reduce (+ optional fused SGD-momentum).
//  slots: device table of N slot base pointers indexed by virtual rank.
//  avg may be null only when p and v are given.
//  With shape.wave_width != 0 every tile holds at most 64 * wave_width elements, and N <= 64.
//  With shape.big_unroll != 0 the first n_big tiles must be full big tiles
//  (kBlock * big_unroll * 4 elements, offset a multiple of 4) and all others
//  at most 2048 elements.
hipError_t launch_ring_reduce(hipStream_t s, const Tile* tiles, uint32_t n_tiles, uint32_t n_big,
                              const float* const* slots, uint32_t N,
                              float* avg, float* p, float* v, float lr, float mu,
                              ReduceShape shape);

// stream_pv: streaming accesses to p and v (vectors too large to stay in the caches between steps)
hipError_t launch_sgd(hipStream_t s, float* p, float* v, const float* g, uint64_t n,
                      float lr, float mu, bool stream_pv);

// dst[0..n) <- src[0..n) floats (any 4-byte alignment)
hipError_t launch_copy_f32(hipStream_t s, float* dst, const float* src, uint64_t n);

// Several contiguous runs copied by one launch (batched gradient staging).
constexpr int kMaxRuns = 16;                // the prefix sums then travel in one 64-byte scalar load
struct CopyRuns {
    float*       dst[kMaxRuns];
    const float* src[kMaxRuns];
    uint64_t     n[kMaxRuns];               // floats; dst and src 4-byte aligned
    uint32_t     first_block[kMaxRuns + 1]; // prefix sums of workgroups per run; [n_runs] = total,
                                            // entries after it 0xFFFFFFFF
    uint32_t     n_runs;
    uint32_t     block;                     // lanes per workgroup the prefix sums count (kCopyBlock or kCopyBlockShort)
};
struct CopyRun {                            // the same for a single run
    float*       dst;
    const float* src;
    uint64_t     n;
};
hipError_t launch_copy_runs(hipStream_t s, const CopyRuns& runs);

enum CtxDir { kSave = 0, kRestore = 1, kSwitch = 2 };
// kSave:    slot_a <- live;  kRestore: live <- slot_a;
// kSwitch:  slot_a <- live, then live <- slot_b (per byte, same lane)
hipError_t launch_ctx(hipStream_t s, const Piece* pieces, uint32_t n_pieces,
                      uint8_t* slot_a, const uint8_t* slot_b, CtxDir dir);

// One launch for an EST boundary: the small-state pieces (kSave or kSwitch) and the staging
// copy of the outgoing EST's runs.  runs.n_runs may be 0, n_pieces may be 0.  The unused
// prefix-sum entries of `runs` must hold 0xFFFFFFFF as for launch_copy_runs.
hipError_t launch_est_boundary(hipStream_t s, const CopyRuns& runs, const Piece* pieces, uint32_t n_pieces,
                               uint8_t* slot_a, const uint8_t* slot_b, CtxDir dir);

// generic byte copy used when contexts move between arenas
hipError_t launch_copy_bytes(hipStream_t s, uint8_t* dst, const uint8_t* src, uint64_t n);

// out[0] = fixed-tree sum of squares of x[0..n), out[1] = its square root;
// part: scratch of ceil(n / 4096) floats.  Leaves the front of x in the caches for the update that follows.
hipError_t launch_sq_norm(hipStream_t s, const float* x, uint64_t n, float* part, float* out);

// The same in one launch up to kCountedBlocks blocks, given kArrivalWords counters that are zero before
// the first launch and left at zero by every one; launches that share them run one after the other.
constexpr uint64_t kCountedBlocks = 2048;
hipError_t launch_sq_norm_counted(hipStream_t s, const float* x, uint64_t n, float* part, float* out, uint32_t* arrivals);

// The same (but all of x streamed) with the block partials in a file-scope device array of kStaticPartials floats
// (1 MiB per GPU): no allocation; n <= kStaticPartials * 4096, else hipErrorInvalidValue.
// Runs on the current device.
constexpr uint64_t kStaticPartials = 1ull << 18;
hipError_t launch_sq_norm_static(hipStream_t s, const float* x, uint64_t n, float* out);

// v <- mu*v + coef*g ; p <- p - lr*v with coef = min(1, max_norm / (norm2[1] + eps)) formed on the device
hipError_t launch_sgd_clip(hipStream_t s, float* p, float* v, const float* g, uint64_t n,
                           const float* norm2, float max_norm, float eps, float lr, float mu, bool stream_pv);

// Per-channel mean and biased variance of x[B][C][HW] along the fixed tree; B * HW < 2^31,
// C <= 65535; part: scratch of C * ceil(B * HW / 4096) floats
hipError_t launch_bn_batch_stats(hipStream_t s, const float* x, uint32_t B, uint32_t C, uint32_t HW,
                                 float* mean, float* var, float* part);

// The same; where workgroups wait for each other's sums, each looks for them `polls` times and then reads
// what it needs for itself.
hipError_t launch_bn_batch_stats_polls(hipStream_t s, const float* x, uint32_t B, uint32_t C, uint32_t HW,
                                       float* mean, float* var, float* part, uint32_t polls);

// mask[0..n) from state = {seed, offset}, offset += ceil(n / 4); n <= kShortMask, threshold <= 2^32
constexpr uint32_t kMaskGroup = 1024;            // lanes of the one workgroup
constexpr uint64_t kShortMask = 16 * kMaskGroup;
hipError_t launch_dropout_mask(hipStream_t s, uint64_t* state, uint8_t* mask, uint64_t n,
                               uint64_t threshold);

// The same for any n, given counters of the workgroups that have read the state: 32-bit words a line apart,
// zero before the first launch and left at zero by every one; launches that share them run one after the other.
constexpr uint32_t kOneCounter = 64;             // workgroups that share one counter
constexpr uint32_t kCounters = 16;               // counters beyond that, and one more
constexpr uint32_t kCounterStep = 32;            // words between two counters
constexpr uint32_t kArrivalWords = (kCounters + 1) * kCounterStep;
hipError_t launch_dropout_mask_long(hipStream_t s, uint64_t* state, uint8_t* mask, uint64_t n, uint64_t threshold,
                                    uint32_t* arrivals);

// The same for any n without counters, in two launches: for launches that a caller captures, which can be replayed
// after the handle is gone and beside its other draws.
hipError_t launch_dropout_mask_captured(hipStream_t s, uint64_t* state, uint8_t* mask, uint64_t n, uint64_t threshold);

// Whether a launch on the stream would be recorded instead of run.
inline bool stream_captured(hipStream_t s)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();                            // the legacy stream while another one is captured, say
    return true;
}

// What the runtime knows of a stream without enqueuing on it.  Set by the file that holds the kernels when the library is
// loaded; null in a program that has the host side alone, whose streams are always handed over by events.
struct StreamProbe {
    bool (*idle)(hipStream_t);          // everything that was enqueued has finished: what follows on any stream sees it
    bool (*done)(hipEvent_t);           // the event has been reached
};
extern StreamProbe stream_probe;

}  // namespace es
