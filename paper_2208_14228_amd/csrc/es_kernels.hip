// gfx950 (CDNA4) kernels of the EST step.  Wave size 64; 256-lane workgroups except
// the staging copies, which run one wave per workgroup.
//
// Bit-exactness rules that hold for every kernel in this file:
//  - fp32 IEEE arithmetic, denormals kept, no fused multiply-add (the file is
//    compiled with -ffp-contract=off), division correctly rounded;
//  - a sum over N ranks is a chain of N-1 adds in one lane in program order, and sums
//    across lanes follow a fixed tree, so neither the grid shape nor the order in which
//    loads return can change a bit; no atomic does arithmetic on a floating-point value
//    (they count workgroups, or carry a finished sum from one to another);
//  - loads may be issued early and in any order, only the add chain is ordered.
#include "es_internal.h"

#include <unistd.h>

#include <atomic>
#include <chrono>
#include <mutex>
#include <tuple>
#include <type_traits>

namespace es {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// Tables that every lane of a workgroup reads at the same index live in the
// constant address space so the reads are scalar loads shared by the wave.
#define ES_CONST_AS __attribute__((address_space(4)))
// A base put together from registers: without the address space its loads would be flat ones.
#define ES_GLOBAL_AS __attribute__((address_space(1)))
#pragma clang diagnostic ignored "-Wold-style-cast"

// A launch in one call of the runtime.  (kernel<<<>>> makes three and the query of the last error is a fourth: 2.48 us a launch
// on three streams in turn, 2.28 so; a hipFunction_t in the place of the kernel's address saves nothing more.)
template <typename... P, typename... A>
static hipError_t run_kernel(void (*kernel)(P...), dim3 grid, dim3 block, uint32_t lds, hipStream_t s, const A&... a)
{
    std::tuple<P...> args(static_cast<P>(a)...);
    const hipError_t e = std::apply(
        [&](P&... v) {
            void* at[] = {&v...};
            return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, at, lds, s);
        },
        args);
    if (e != hipSuccess) (void)hipGetLastError();       // the caller has it: no later call is to find it
    return e;
}
#define ES_RUN(kernel, grid, block, lds, s, ...)                                                                      \
    do {                                                                                                              \
        const hipError_t e__ = run_kernel(kernel, grid, block, lds, s, __VA_ARGS__);                                  \
        if (e__ != hipSuccess) return e__;                                                                            \
    } while (0)

template <bool NT>
__device__ __forceinline__ f4 ld4(const float* p)
{
    const f4* q = reinterpret_cast<const f4*>(p);
    if constexpr (NT)
        return __builtin_nontemporal_load(q);
    else
        return *q;
}

__device__ __forceinline__ void st4(float* p, f4 x) { *reinterpret_cast<f4*>(p) = x; }

// Parameter / momentum traffic of the update, and the store of the averaged
// gradient.  Touched once per global step: streamed where stream_pv says so
// (fused: +6 % at P = 109 M; the unfused reduce: +11 % at P = 109 M, N = 16 and
// +13 % at P = 355 M, N = 64 from the store of the averaged gradient alone).
template <bool NTPV>
__device__ __forceinline__ f4 ld4_pv(const float* p)
{
    if constexpr (NTPV) return __builtin_nontemporal_load(reinterpret_cast<const f4*>(p));
    else return *reinterpret_cast<const f4*>(p);
}
template <bool NTPV>
__device__ __forceinline__ void st4_pv(float* p, f4 x)
{
    if constexpr (NTPV) __builtin_nontemporal_store(x, reinterpret_cast<f4*>(p));
    else *reinterpret_cast<f4*>(p) = x;
}

// ---------------------------------------------------------------------------
// Ring-ordered N-way reduce (paper §3.3 D1: aggregation order fixed by the
// ESTs' constant virtual ranks), optionally fused with the SGD-momentum update
// of the shared replica (paper §3.2).
//
// One workgroup = one Tile (a range inside one ring chunk).  Chunk c's sum is
// the left fold over ranks c, c+1, ..., c+N-1 (mod N): what the reduce-scatter
// of an N-rank ring computes when rank r sends to r+1 and first sends its own
// chunk.  Each lane keeps U independent 16-byte accumulators and loads NB ranks
// ahead of the adds.
// ---------------------------------------------------------------------------
template <int U, int NB, int NT, bool FIRST>
__device__ __forceinline__ void fold_batch(const float* const ES_CONST_AS* slots, uint32_t N,
                                           uint32_t r0, const uint64_t (&e)[U], f4 (&acc)[U])
{
    // ranks r0 .. r0+NB-1 (mod N): all loads first, then the adds in rank order
    f4 x[NB][U];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        uint32_t r = r0 + j;
        if (r >= N) r -= N;
        const float* g = slots[r];
#pragma unroll
        for (int u = 0; u < U; ++u) x[j][u] = ld4<(NT & 1) != 0>(g + e[u]);
    }
    // keep every load of the batch ahead of the first add: the batch is the
    // wave's bytes in flight
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (FIRST && j == 0)
                acc[u] = x[0][u];                          // the fold opens with rank c itself
            else
                acc[u] = acc[u] + x[j][u];
        }
    }
}

// The last N - k < 2*NBX ranks of a fold, in batches of NBX, NBX/2, .. 1 (same order of adds).
template <int U, int NBX, int NT>
__device__ __forceinline__ void fold_rest(const float* const ES_CONST_AS* slots, uint32_t N, uint32_t rank0,
                                          uint32_t& k, const uint64_t (&e)[U], f4 (&acc)[U])
{
    if constexpr (NBX >= 1) {
        if (k + NBX <= N) {
            uint32_t r0 = rank0 + k;
            if (r0 >= N) r0 -= N;
            fold_batch<U, NBX, NT, false>(slots, N, r0, e, acc);
            k += NBX;
        }
        fold_rest<U, NBX / 2, NT>(slots, N, rank0, k, e, acc);
    }
}

template <bool SGD>
__device__ __forceinline__ void finish_scalar(float acc, float fN, uint64_t e, float* avg,
                                              float* p, float* v, float lr, float mu)
{
    const float a = acc / fN;
    if (avg) avg[e] = a;
    if constexpr (SGD) {
        const float mv = mu * v[e];
        const float vn = mv + a;
        const float st = lr * vn;
        v[e] = vn;
        p[e] = p[e] - st;
    }
}

template <bool SGD>
__device__ __forceinline__ void fold_scalar(const float* const ES_CONST_AS* slots, uint32_t N,
                                            uint32_t rank0, float fN, uint64_t e, float* avg,
                                            float* p, float* v, float lr, float mu)
{
    uint32_t r = rank0;
    float acc = slots[r][e];
    for (uint32_t k = 1; k < N; ++k) {
        r = (r + 1 == N) ? 0 : r + 1;
        acc = acc + slots[r][e];
    }
    finish_scalar<SGD>(acc, fN, e, avg, p, v, lr, mu);
}

template <int U, int NB, int NT, bool SGD>
__device__ __forceinline__ void small_tile(const float* const ES_CONST_AS* slots, uint32_t N,
                                           uint64_t off, uint32_t len, uint32_t rank0,
                                           float* __restrict__ avg, float* __restrict__ p,
                                           float* __restrict__ v, float lr, float mu)
{
    const float fN = (float)N;

    // 16-byte vectors need element offsets that are multiples of 4 (all slot,
    // avg, p and v bases are 16-byte aligned): up to 3 leading and 3 trailing
    // elements of a tile take the scalar path.
    uint32_t head = (uint32_t)((4 - (off & 3)) & 3);
    if (head > len) head = len;
    const uint32_t nvec = (len - head) >> 2;
    const uint64_t vbase = off + head;
    const uint32_t tail = len - head - 4 * nvec;

    for (uint32_t i0 = threadIdx.x; i0 < nvec; i0 += kReduceBlock * U) {
        uint64_t e[U];
        bool ok[U];
        f4 acc[U], pp[U], vv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = i0 + u * kReduceBlock;
            ok[u] = i < nvec;
            // a lane without work in this pass re-reads the tile's last vector
            // (in bounds, result dropped) so that no load needs a predicate
            e[u] = vbase + 4ull * (ok[u] ? i : nvec - 1);
        }
        if constexpr (SGD) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                pp[u] = ld4_pv<(NT & 2) != 0>(p + e[u]);
                vv[u] = ld4_pv<(NT & 2) != 0>(v + e[u]);
            }
        }
        // N = q*NB + rem ranks: q full batches, then the rest in batches of NB/2, NB/4, .. 1
        // (a remainder taken one rank at a time leaves the wave with a single rank's loads in
        // flight: measured -10 % at N = 12 when one workgroup has a CU to itself)
        uint32_t k;
        if (N >= (uint32_t)NB) {
            fold_batch<U, NB, NT, true>(slots, N, rank0, e, acc);
            k = NB;
        } else {
            fold_batch<U, 1, NT, true>(slots, N, rank0, e, acc);
            k = 1;
        }
        for (; k + NB <= N; k += NB) {
            uint32_t r0 = rank0 + k;
            if (r0 >= N) r0 -= N;
            fold_batch<U, NB, NT, false>(slots, N, r0, e, acc);
        }
        fold_rest<U, NB / 2, NT>(slots, N, rank0, k, e, acc);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!ok[u]) continue;
            const f4 a = acc[u] / fN;
            if (avg) st4_pv<(NT & 2) != 0>(avg + e[u], a);
            if constexpr (SGD) {
                const f4 mv = mu * vv[u];
                const f4 vn = mv + a;
                const f4 st = lr * vn;
                st4_pv<(NT & 2) != 0>(v + e[u], vn);
                st4_pv<(NT & 2) != 0>(p + e[u], pp[u] - st);
            }
        }
    }
    if (threadIdx.x < head)
        fold_scalar<SGD>(slots, N, rank0, fN, off + threadIdx.x, avg, p, v, lr, mu);
    if (threadIdx.x < tail)
        fold_scalar<SGD>(slots, N, rank0, fN, vbase + 4ull * nvec + threadIdx.x, avg, p, v, lr, mu);
}

template <int U, int NB, int NT, bool SGD>
__global__ __launch_bounds__(kReduceBlock) void k_ring_reduce(const Tile* tiles_g,
                                                        const float* const* slots_g, uint32_t N,
                                                        float* __restrict__ avg,
                                                        float* __restrict__ p,
                                                        float* __restrict__ v, float lr, float mu)
{
    const Tile ES_CONST_AS* tiles = (const Tile ES_CONST_AS*)tiles_g;
    const float* const ES_CONST_AS* slots = (const float* const ES_CONST_AS*)slots_g;
    small_tile<U, NB, NT, SGD>(slots, N, tiles[blockIdx.x].off, tiles[blockIdx.x].len,
                               tiles[blockIdx.x].rank0, avg, p, v, lr, mu);
}

// ---------------------------------------------------------------------------
// Big-tile form of the same kernel for large N.  Measured on MI355X: with many
// concurrent gradient streams HBM delivers more when each workgroup reads a long
// contiguous span per stream (128 KiB at UB = 32: 6.2 TB/s at N = 64 against
// 5.4 TB/s for 8 KiB spans).  A big tile is always full and 16-byte aligned, so
// addresses are base + constants and nothing is predicated; each wave owns UB
// consecutive KiB of every stream.  The first n_big workgroups take big tiles,
// the rest run the small-tile path (chunk remainders, ragged and unaligned
// pieces) with U = 2, NB = 8.
// ---------------------------------------------------------------------------
template <int UB, int NB, int NT, bool FIRST>
__device__ __forceinline__ void fold_batch_lin(const float* const ES_CONST_AS* slots, uint32_t N,
                                               uint32_t r0, uint64_t e0, f4 (&acc)[UB])
{
    f4 x[NB][UB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        uint32_t r = r0 + j;
        if (r >= N) r -= N;
        const float* g = slots[r] + e0;
#pragma unroll
        for (int u = 0; u < UB; ++u) x[j][u] = ld4<(NT & 1) != 0>(g + 256 * u);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            if (FIRST && j == 0)
                acc[u] = x[0][u];
            else
                acc[u] = acc[u] + x[j][u];
        }
    }
}

template <int UB, int NBB, int NT, bool SGD>
__global__ __launch_bounds__(kReduceBlock) void k_ring_reduce_big(const Tile* tiles_g, uint32_t n_big,
                                                            const float* const* slots_g, uint32_t N,
                                                            float* __restrict__ avg,
                                                            float* __restrict__ p,
                                                            float* __restrict__ v, float lr, float mu)
{
    const Tile ES_CONST_AS* tiles = (const Tile ES_CONST_AS*)tiles_g;
    const float* const ES_CONST_AS* slots = (const float* const ES_CONST_AS*)slots_g;
    const uint64_t off = tiles[blockIdx.x].off;
    const uint32_t len = tiles[blockIdx.x].len;
    const uint32_t rank0 = tiles[blockIdx.x].rank0;
    if (blockIdx.x >= n_big) {
        small_tile<2, 8, NT, SGD>(slots, N, off, len, rank0, avg, p, v, lr, mu);
        return;
    }
    const float fN = (float)N;
    const uint32_t w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const uint64_t e0 = off + 4ull * ((uint64_t)(w * UB) * 64 + l);
    f4 acc[UB];
    uint32_t k;
    if (N >= (uint32_t)NBB) {
        fold_batch_lin<UB, NBB, NT, true>(slots, N, rank0, e0, acc);
        k = NBB;
    } else {
        fold_batch_lin<UB, 1, NT, true>(slots, N, rank0, e0, acc);
        k = 1;
    }
    for (; k + NBB <= N; k += NBB) {
        uint32_t r0 = rank0 + k;
        if (r0 >= N) r0 -= N;
        fold_batch_lin<UB, NBB, NT, false>(slots, N, r0, e0, acc);
    }
    for (; k < N; ++k) {
        uint32_t r0 = rank0 + k;
        if (r0 >= N) r0 -= N;
        fold_batch_lin<UB, 1, NT, false>(slots, N, r0, e0, acc);
    }
    // Epilogue kBigEpilogue vectors at a time, in the registers the rank loads have left free:
    // 2 * 16 loads of parameters and momentum in flight, then their stores (measured against
    // groups of 4: +3 % at N = 16, +2 % at N = 64; parameter and momentum accesses alternating
    // as here beat all of one, then all of the other).
    constexpr int EG = (kBigEpilogue < UB) ? kBigEpilogue : UB;
#pragma unroll
    for (int u0 = 0; u0 < UB; u0 += EG) {
        f4 pp[EG], vv[EG];
        if constexpr (SGD) {
#pragma unroll
            for (int q = 0; q < EG; ++q) {
                pp[q] = ld4_pv<(NT & 2) != 0>(p + e0 + 256 * (u0 + q));
                vv[q] = ld4_pv<(NT & 2) != 0>(v + e0 + 256 * (u0 + q));
            }
        }
#pragma unroll
        for (int q = 0; q < EG; ++q) {
            const uint64_t e = e0 + 256 * (u0 + q);
            const f4 a = acc[u0 + q] / fN;
            if (avg) st4_pv<(NT & 2) != 0>(avg + e, a);
            if constexpr (SGD) {
                const f4 mv = mu * vv[q];
                const f4 vn = mv + a;
                const f4 st = lr * vn;
                st4_pv<(NT & 2) != 0>(v + e, vn);
                st4_pv<(NT & 2) != 0>(p + e, pp[q] - st);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int U, int NB>
static hipError_t launch_reduce_unb(hipStream_t s, const Tile* tiles, uint32_t n_tiles,
                                    const float* const* slots, uint32_t N, float* avg, float* p,
                                    float* v, float lr, float mu, int nt, uint32_t lds_pad)
{
    const bool sgd = p != nullptr;
    dim3 grid(n_tiles), block(kReduceBlock);
#define ES_LAUNCH(NTV, SGDV) \
    ES_RUN((k_ring_reduce<U, NB, NTV, SGDV>), grid, block, lds_pad, s, tiles, slots, N, avg, p, v, lr, mu)
    if (!sgd) {
        switch (nt & 3) {
        case 0: ES_LAUNCH(0, false); break;
        case 1: ES_LAUNCH(1, false); break;
        case 2: ES_LAUNCH(2, false); break;
        default: ES_LAUNCH(3, false); break;
        }
    } else {
        switch (nt & 3) {
        case 0: ES_LAUNCH(0, true); break;
        case 1: ES_LAUNCH(1, true); break;
        case 2: ES_LAUNCH(2, true); break;
        default: ES_LAUNCH(3, true); break;
        }
    }
#undef ES_LAUNCH
    return hipSuccess;
}

template <int U>
static hipError_t launch_reduce_u(hipStream_t s, const Tile* tiles, uint32_t n_tiles,
                                  const float* const* slots, uint32_t N, float* avg, float* p,
                                  float* v, float lr, float mu, ReduceShape sh)
{
    const int nt = (sh.nontemporal ? 1 : 0) | (sh.nontemporal_pv ? 2 : 0);
    switch (sh.rank_batch) {
    case 1:  return launch_reduce_unb<U, 1>(s, tiles, n_tiles, slots, N, avg, p, v, lr, mu, nt, reduce_lds_pad(sh.lds_pad_kib, N, sh.nontemporal_pv != 0 && p != nullptr, p != nullptr));
    case 2:  return launch_reduce_unb<U, 2>(s, tiles, n_tiles, slots, N, avg, p, v, lr, mu, nt, reduce_lds_pad(sh.lds_pad_kib, N, sh.nontemporal_pv != 0 && p != nullptr, p != nullptr));
    case 4:  return launch_reduce_unb<U, 4>(s, tiles, n_tiles, slots, N, avg, p, v, lr, mu, nt, reduce_lds_pad(sh.lds_pad_kib, N, sh.nontemporal_pv != 0 && p != nullptr, p != nullptr));
    case 8:  return launch_reduce_unb<U, 8>(s, tiles, n_tiles, slots, N, avg, p, v, lr, mu, nt, reduce_lds_pad(sh.lds_pad_kib, N, sh.nontemporal_pv != 0 && p != nullptr, p != nullptr));
    case 16: return launch_reduce_unb<U, 16>(s, tiles, n_tiles, slots, N, avg, p, v, lr, mu, nt, reduce_lds_pad(sh.lds_pad_kib, N, sh.nontemporal_pv != 0 && p != nullptr, p != nullptr));
    default: return hipErrorInvalidValue;
    }
}

template <int UB, int NBB>
static hipError_t launch_reduce_big(hipStream_t s, const Tile* tiles, uint32_t n_tiles, uint32_t n_big,
                                    const float* const* slots, uint32_t N, float* avg, float* p,
                                    float* v, float lr, float mu, int nt)
{
    const bool sgd = p != nullptr;
    dim3 grid(n_tiles), block(kReduceBlock);
#define ES_LAUNCH(NTV, SGDV) \
    ES_RUN((k_ring_reduce_big<UB, NBB, NTV, SGDV>), grid, block, 0, s, tiles, n_big, slots, N, avg, p, v, lr, mu)
    if (!sgd) {
        switch (nt & 3) {
        case 0: ES_LAUNCH(0, false); break;
        case 1: ES_LAUNCH(1, false); break;
        case 2: ES_LAUNCH(2, false); break;
        default: ES_LAUNCH(3, false); break;
        }
    } else {
        switch (nt & 3) {
        case 0: ES_LAUNCH(0, true); break;
        case 1: ES_LAUNCH(1, true); break;
        case 2: ES_LAUNCH(2, true); break;
        default: ES_LAUNCH(3, true); break;
        }
    }
#undef ES_LAUNCH
    return hipSuccess;
}

template <int UB>
static hipError_t launch_reduce_big_u(hipStream_t s, const Tile* tiles, uint32_t n_tiles, uint32_t n_big,
                                      const float* const* slots, uint32_t N, float* avg, float* p,
                                      float* v, float lr, float mu, ReduceShape sh)
{
    const int nt = (sh.nontemporal ? 1 : 0) | (sh.nontemporal_pv ? 2 : 0);
    // only shapes whose loads in flight fit the register file exist: UB * batch <= 32
    if (sh.big_rank_batch == 1)
        return launch_reduce_big<UB, 1>(s, tiles, n_tiles, n_big, slots, N, avg, p, v, lr, mu, nt);
    if constexpr (UB <= 16) {
        if (sh.big_rank_batch == 2)
            return launch_reduce_big<UB, 2>(s, tiles, n_tiles, n_big, slots, N, avg, p, v, lr, mu, nt);
    }
    if constexpr (UB <= 8) {
        if (sh.big_rank_batch == 4)
            return launch_reduce_big<UB, 4>(s, tiles, n_tiles, n_big, slots, N, avg, p, v, lr, mu, nt);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Wave-tile form of the same kernel for short vectors and at most 64 ranks: one WAVE
// per tile of 64 * W elements, W floats per lane.
//
// What bounds a short reduce is the number of dependent round trips to memory in one
// wave's life and the number of waves, not bytes.  So: the rank -> slot table is read
// with one vector load (lane r holds rank r's base) that does not wait for the tile, and
// a rank's base then comes out of a register (v_readlane) instead of a scalar load in
// front of every batch; tiles are small enough that every CU has some; a batch is as
// many ranks as the registers hold when few waves share a SIMD.  Vectors may start at
// any 4-byte address, and the last one of a tile is shifted back over its neighbour's
// elements (both lanes of the wave have loaded before either stores, and store the same
// values), so ragged chunks have no element-wise path; only a tile shorter than a vector
// is read one float per lane.
//
// Fused, default options, three jobs in turn: N = 64, P = 20 k 16.8 -> 4.9 us, P = 200 k
// 19.0 -> 10.6 us; N = 16, P = 500 k 14.1 -> 7.9 us, P = 4 M 67 -> 53 us; N = 8, P = 1 M
// 11.4 -> 9.2 us; N = 4, P = 1 M 7.6 -> 6.8 us (4.9 TB/s).
// ---------------------------------------------------------------------------
template <int W> struct WaveVec;
template <> struct WaveVec<1> { typedef float T; };
template <> struct WaveVec<4> { typedef float T __attribute__((ext_vector_type(4), aligned(4))); };

template <int W, int NB, int NT, bool SGD>
__device__ __forceinline__ void wave_tile(uint64_t off, uint32_t len, uint32_t rank0, uint32_t base_lo,
                                          uint32_t base_hi, uint32_t lane, uint32_t N, float* __restrict__ avg,
                                          float* __restrict__ p, float* __restrict__ v, float lr, float mu)
{
    typedef typename WaveVec<W>::T T;
    const uint32_t i = W * lane;
    const bool ok = i < len;
    const uint32_t e = 4u * (i + W <= len ? i : len - W);       // bytes; W <= len
    auto at = [&](float* base) { return reinterpret_cast<T*>(reinterpret_cast<char*>(base + off) + e); };
    T pp, vv;
    if constexpr (SGD) {
        if constexpr ((NT & 2) != 0) {
            pp = __builtin_nontemporal_load(at(p));
            vv = __builtin_nontemporal_load(at(v));
        } else {
            pp = *at(p);
            vv = *at(v);
        }
    }
    T acc;
    uint32_t k = 0, r = rank0;
    auto batch = [&](auto count, bool first) {
        constexpr int C = decltype(count)::value;
        T x[C];
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const uint32_t lo = __builtin_amdgcn_readlane(base_lo, r), hi = __builtin_amdgcn_readlane(base_hi, r);
            const ES_GLOBAL_AS T* g = (const ES_GLOBAL_AS T*)(((uint64_t)hi << 32 | lo) + 4 * off + e);
            x[j] = (NT & 1) ? __builtin_nontemporal_load(g) : *g;
            r = r + 1 == N ? 0 : r + 1;
        }
        __builtin_amdgcn_sched_barrier(0);              // all loads of the batch ahead of its adds
#pragma unroll
        for (int j = 0; j < C; ++j) acc = (j == 0 && first) ? x[0] : acc + x[j];
        k += C;
    };
    auto rest = [&](auto self, auto count) {            // batches of NB/2, NB/4, .. 1
        constexpr int C = decltype(count)::value;
        if (k + C <= N) batch(count, false);
        if constexpr (C > 1) self(self, std::integral_constant<int, C / 2>{});
    };
    if (N >= (uint32_t)NB) batch(std::integral_constant<int, NB>{}, true);
    else batch(std::integral_constant<int, 1>{}, true);
    while (k + NB <= N) batch(std::integral_constant<int, NB>{}, false);
    if constexpr (NB > 1) rest(rest, std::integral_constant<int, NB / 2>{});
    if (!ok) return;
    const T a = acc / (float)N;
    if (avg) {
        if constexpr ((NT & 2) != 0) __builtin_nontemporal_store(a, at(avg));
        else *at(avg) = a;
    }
    if constexpr (SGD) {
        const T mv = mu * vv;
        const T vn = mv + a;
        const T st = lr * vn;
        if constexpr ((NT & 2) != 0) {
            __builtin_nontemporal_store(vn, at(v));
            __builtin_nontemporal_store(pp - st, at(p));
        } else {
            *at(v) = vn;
            *at(p) = pp - st;
        }
    }
}

template <int W, int NB, int NT, bool SGD>
__global__ __launch_bounds__(kReduceBlock) void k_ring_reduce_wave(const Tile* tiles_g, uint32_t n_tiles,
                                                             const float* const* slots, uint32_t N,
                                                             float* __restrict__ avg, float* __restrict__ p,
                                                             float* __restrict__ v, float lr, float mu)
{
    const uint32_t lane = threadIdx.x & 63;
    // (blockDim for the constant would make the runtime write the hidden arguments with every launch:
    // 5.4 -> 5.7 us per call in a loop of small steps)
    const uint32_t t = __builtin_amdgcn_readfirstlane(blockIdx.x * (kReduceBlock / 64) + (threadIdx.x >> 6));
    if (t >= n_tiles) return;
    const uint64_t base = reinterpret_cast<uint64_t>(slots[lane < N ? lane : N - 1]);
    const uint32_t lo = (uint32_t)base, hi = (uint32_t)(base >> 32);
    const Tile ES_CONST_AS* tiles = (const Tile ES_CONST_AS*)tiles_g;
    const uint64_t off = tiles[t].off;
    const uint32_t len = tiles[t].len;
    const uint32_t rank0 = tiles[t].rank0;
    if (len >= W) wave_tile<W, NB, NT, SGD>(off, len, rank0, lo, hi, lane, N, avg, p, v, lr, mu);
    else wave_tile<1, 8, NT, SGD>(off, len, rank0, lo, hi, lane, N, avg, p, v, lr, mu);
}

template <int W, int NB>
static hipError_t launch_reduce_wave(hipStream_t s, const Tile* tiles, uint32_t n_tiles, const float* const* slots,
                                     uint32_t N, float* avg, float* p, float* v, float lr, float mu, ReduceShape sh)
{
    constexpr uint32_t per = kReduceBlock / 64;
    const dim3 grid((uint32_t)(((uint64_t)n_tiles + per - 1) / per)), block(kReduceBlock);
#define ES_LAUNCH(NTV, SGDV)                                                                                      \
    ES_RUN((k_ring_reduce_wave<W, NB, NTV, SGDV>), grid, block, (uint32_t)sh.wave_pad_kib << 10, s, tiles, \
                       n_tiles, slots, N, avg, p, v, lr, mu)
    if (p) {
        if (sh.nontemporal_pv) ES_LAUNCH(3, true);
        else ES_LAUNCH(1, true);
    } else {
        if (sh.nontemporal_pv) ES_LAUNCH(3, false);
        else ES_LAUNCH(1, false);
    }
#undef ES_LAUNCH
    return hipSuccess;
}

static hipError_t launch_reduce_wave_any(hipStream_t s, const Tile* tiles, uint32_t n_tiles, const float* const* slots,
                                         uint32_t N, float* avg, float* p, float* v, float lr, float mu, ReduceShape sh)
{
    if (N > 64) return hipErrorInvalidValue;            // the table is one pointer per lane
#define ES_WAVE(W, NB)                                   \
    if (sh.wave_width == W && sh.wave_batch == NB)      \
        return launch_reduce_wave<W, NB>(s, tiles, n_tiles, slots, N, avg, p, v, lr, mu, sh)
    ES_WAVE(1, 8);
    ES_WAVE(1, 16);
    ES_WAVE(1, 32);
    ES_WAVE(1, 64);
    ES_WAVE(4, 1);
    ES_WAVE(4, 2);
    ES_WAVE(4, 4);
    ES_WAVE(4, 8);
#undef ES_WAVE
    return hipErrorInvalidValue;
}

hipError_t launch_ring_reduce(hipStream_t s, const Tile* tiles, uint32_t n_tiles, uint32_t n_big,
                              const float* const* slots, uint32_t N, float* avg, float* p,
                              float* v, float lr, float mu, ReduceShape sh)
{
    if (n_tiles == 0) return hipSuccess;
    if (sh.wave_width) return launch_reduce_wave_any(s, tiles, n_tiles, slots, N, avg, p, v, lr, mu, sh);
    if (sh.big_unroll) {
        switch (sh.big_unroll) {
        case 8:  return launch_reduce_big_u<8>(s, tiles, n_tiles, n_big, slots, N, avg, p, v, lr, mu, sh);
        case 16: return launch_reduce_big_u<16>(s, tiles, n_tiles, n_big, slots, N, avg, p, v, lr, mu, sh);
        case 32: return launch_reduce_big_u<32>(s, tiles, n_tiles, n_big, slots, N, avg, p, v, lr, mu, sh);
        default: return hipErrorInvalidValue;
        }
    }
    switch (sh.unroll) {
    case 1: return launch_reduce_u<1>(s, tiles, n_tiles, slots, N, avg, p, v, lr, mu, sh);
    case 2: return launch_reduce_u<2>(s, tiles, n_tiles, slots, N, avg, p, v, lr, mu, sh);
    case 4: return launch_reduce_u<4>(s, tiles, n_tiles, slots, N, avg, p, v, lr, mu, sh);
    default: return hipErrorInvalidValue;
    }
}

// Redirect a few entries of the rank -> gradient-base table in stream order.
__global__ void k_patch_slots(const float** table, const InPlace patch)
{
    if (blockIdx.x == 0 && threadIdx.x < patch.n) table[patch.rank[threadIdx.x]] = patch.ptr[threadIdx.x];
}

hipError_t launch_patch_slots(hipStream_t s, const float** table, const InPlace& patch)
{
    if (patch.n == 0) return hipSuccess;
    ES_RUN(k_patch_slots, dim3(1), dim3(64), 0, s, table, patch);
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// SGD with momentum on the shared replica (paper §3.2), unfused form.
// ---------------------------------------------------------------------------
constexpr int kSgdU = 4;

template <bool NTPV>
__global__ __launch_bounds__(kBlock) void k_sgd(float* __restrict__ p, float* __restrict__ v,
                                                const float* __restrict__ g, uint64_t n,
                                                float lr, float mu)
{
    const uint64_t nvec = n >> 2;
    const uint64_t base = (uint64_t)blockIdx.x * (kBlock * kSgdU) + threadIdx.x;
    f4 pp[kSgdU], vv[kSgdU], gg[kSgdU];
#pragma unroll
    for (int u = 0; u < kSgdU; ++u) {
        const uint64_t i = base + (uint64_t)u * kBlock;
        if (i < nvec) {
            gg[u] = ld4<true>(g + 4 * i);
            pp[u] = ld4_pv<NTPV>(p + 4 * i);
            vv[u] = ld4_pv<NTPV>(v + 4 * i);
        }
    }
#pragma unroll
    for (int u = 0; u < kSgdU; ++u) {
        const uint64_t i = base + (uint64_t)u * kBlock;
        if (i < nvec) {
            const f4 mv = mu * vv[u];
            const f4 vn = mv + gg[u];
            const f4 st = lr * vn;
            st4_pv<NTPV>(v + 4 * i, vn);
            st4_pv<NTPV>(p + 4 * i, pp[u] - st);
        }
    }
    if (blockIdx.x == 0) {
        const uint64_t e = 4 * nvec + threadIdx.x;
        if (e < n) {
            const float mv = mu * v[e];
            const float vn = mv + g[e];
            const float st = lr * vn;
            v[e] = vn;
            p[e] = p[e] - st;
        }
    }
}

hipError_t launch_sgd(hipStream_t s, float* p, float* v, const float* g, uint64_t n, float lr,
                      float mu, bool stream_pv)
{
    if (n == 0) return hipSuccess;
    const uint64_t nvec = n >> 2;
    uint64_t blocks = (nvec + kBlock * kSgdU - 1) / (kBlock * kSgdU);
    if (blocks == 0) blocks = 1;
    if (stream_pv)
        ES_RUN(k_sgd<true>, dim3((uint32_t)blocks), dim3(kBlock), kAuxLdsPad, s, p, v, g, n, lr, mu);
    else
        ES_RUN(k_sgd<false>, dim3((uint32_t)blocks), dim3(kBlock), kAuxLdsPad, s, p, v, g, n, lr, mu);
    return hipSuccess;
}

// The same update with the gradient clipped by its global norm first: every lane forms
//     coef = min(1, max_norm / (norm + eps))
// from the norm es_grad_sq_norm left in device memory (no host round trip) and scales its
// gradient elements by it; coef * g is rounded on its own before it enters the momentum.
template <bool NTPV>
__global__ __launch_bounds__(kBlock) void k_sgd_clip(float* __restrict__ p, float* __restrict__ v,
                                                     const float* __restrict__ g, uint64_t n,
                                                     const float* __restrict__ norm2, float max_norm,
                                                     float eps, float lr, float mu)
{
    const float d = norm2[1] + eps;
    const float q = max_norm / d;
    const float coef = q < 1.0f ? q : 1.0f;
    const uint64_t nvec = n >> 2;
    const uint64_t base = (uint64_t)blockIdx.x * (kBlock * kSgdU) + threadIdx.x;
    f4 pp[kSgdU], vv[kSgdU], gg[kSgdU];
#pragma unroll
    for (int u = 0; u < kSgdU; ++u) {
        const uint64_t i = base + (uint64_t)u * kBlock;
        if (i < nvec) {
            gg[u] = ld4<true>(g + 4 * i);
            pp[u] = ld4_pv<NTPV>(p + 4 * i);
            vv[u] = ld4_pv<NTPV>(v + 4 * i);
        }
    }
#pragma unroll
    for (int u = 0; u < kSgdU; ++u) {
        const uint64_t i = base + (uint64_t)u * kBlock;
        if (i < nvec) {
            const f4 gs = coef * gg[u];
            const f4 mv = mu * vv[u];
            const f4 vn = mv + gs;
            const f4 st = lr * vn;
            st4_pv<NTPV>(v + 4 * i, vn);
            st4_pv<NTPV>(p + 4 * i, pp[u] - st);
        }
    }
    if (blockIdx.x == 0) {
        const uint64_t e = 4 * nvec + threadIdx.x;
        if (e < n) {
            const float gs = coef * g[e];
            const float mv = mu * v[e];
            const float vn = mv + gs;
            const float st = lr * vn;
            v[e] = vn;
            p[e] = p[e] - st;
        }
    }
}

hipError_t launch_sgd_clip(hipStream_t s, float* p, float* v, const float* g, uint64_t n,
                           const float* norm2, float max_norm, float eps, float lr, float mu, bool stream_pv)
{
    if (n == 0) return hipSuccess;
    const uint64_t nvec = n >> 2;
    uint64_t blocks = (nvec + kBlock * kSgdU - 1) / (kBlock * kSgdU);
    if (blocks == 0) blocks = 1;
    if (stream_pv)
        ES_RUN(k_sgd_clip<true>, dim3((uint32_t)blocks), dim3(kBlock), kAuxLdsPad, s, p, v, g, n, norm2,
                           max_norm, eps, lr, mu);
    else
        ES_RUN(k_sgd_clip<false>, dim3((uint32_t)blocks), dim3(kBlock), kAuxLdsPad, s, p, v, g, n, norm2,
                           max_norm, eps, lr, mu);
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Fixed-tree sum of squares of a flat vector (global gradient norm).  In the
// spirit of the paper's level D2 (section 3.3: reductions must not depend on
// the GPU they run on) the summation tree is a function of the vector length
// alone: blocks of 4096 elements; lane t adds the squares of elements
// 4*(256*q + t) + c, q = 0..3 outer, c = 0..3 inner, starting from +0; the 256
// lane sums combine as v[t] += v[t+s], s = 128 .. 1; block partials combine the
// same way in one more workgroup (lane t adds partials t, t+256, ... first).
// Lane exchanges (and LDS in the last stage) carry the tree; no atomic adds to a sum.
// ---------------------------------------------------------------------------
// The strides 32 .. 1 of a stride-halving tree (v[t] += v[t + s]) over the wave; the sum is valid in lane 0.
// Lane exchanges of the vector ALU only: a permutation through LDS in each of six steps in a row was
// most of what a wave did between its loads and its result (BatchNorm statistics 32x2048x7x7 6.5 -> 6.1 us,
// 4x375x13788 17.8 -> 16.6).
template <uint32_t ROW_SHIFT>
__device__ __forceinline__ float add_shifted(float r)       // lane t: r + lane t + ROW_SHIFT of its row of 16
{
    return r + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(r), 0x100 | ROW_SHIFT, 0xF, 0xF, true));
}

__device__ __forceinline__ float tree16(float r)
{
    return add_shifted<1>(add_shifted<2>(add_shifted<4>(add_shifted<8>(r))));
}

__device__ __forceinline__ float tree32(float r)
{
    const auto rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(r), __float_as_uint(r), false, false);
    return tree16(__uint_as_float(rows[0]) + __uint_as_float(rows[1]));
}

__device__ __forceinline__ float tree64(float r)
{
    const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(r), __float_as_uint(r), false, false);
    return tree32(__uint_as_float(halves[0]) + __uint_as_float(halves[1]));
}

__device__ __forceinline__ float lane0(float r)
{
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(r)));
}

__device__ __forceinline__ float tree256(float s, float* lds)
{
    const uint32_t t = threadIdx.x;
    lds[t] = s;
    __syncthreads();
    if (t < 128) {
        s = s + lds[t + 128];
        lds[t] = s;
    }
    __syncthreads();
    if (t < 64) {
        s = tree64(s + lds[t + 64]);
    }
    return s;                                           // valid in lane 0
}

// One WAVE per 4096-element block: hardware lane h plays the tree's lanes h, h+64,
// h+128 and h+192, so the strides 128 and 64 are adds between its own registers,
// 32 .. 1 are lane exchanges, and no LDS or barrier is needed; all 16 loads of a
// lane are in flight before the first add.
//
// Bound by reading x.  What follows the norm of a job's average is the clipped update, which reads the same vector from
// its start: the first kNormKept blocks are read last and without the streaming hint (kSqFrontKept), so that the Infinity
// Cache (256 MB) still has them.  Kept blocks of 64, 128, 192 and 256 MB: 50 M and 2 ranks 284, 281, 288, 290 us (299
// without); whether the others are read forwards or backwards makes no difference.  Reduce, norm and update in us, all of x
// streamed / so, by what ran before them:
//
//                    writes of all gradients  staging copies   nothing else     reads of 1 GiB   a 1 GiB fill
//   11 M x  8 ranks      116 /  113             120 /  117       117 /  111       121 /  118       131 /  128
//   25.6 M x 8           253 /  242             252 /  243       252 /  243       251 /  244       250 /  262
//   50 M x   2           293 /  279             295 /  283       292 /  281       298 /  281       297 /  312
//   100 M x  8           984 /  946             981 /  949       996 /  971       977 /  955       979 /  987
//   109 M x 16          1612 / 1599            1616 / 1595      1613 / 1599      1620 / 1596      1616 / 1634
//
// What loses is a cacheable read behind a fill, which has to write the fill's lines back first, and any cacheable read that
// nothing follows.  The norm alone, cacheable over streamed, 8.5 / 15 / 25.6 / 41.9 / 150 M: behind a fill 1.50 / 1.75 /
// 1.84 / 2.09 / 1.35, behind reads 1.01 / 1.03 / 1.06 / 1.08 / 1.02, of a vector just written 1.00-1.02.  So the norm that
// belongs to no job (kSqStreamed) does without, and reads forwards: 110 M and 150 M just written 71.5 and 100 us, backwards
// 75.4 and 105.
constexpr uint64_t kNormKept = 10240;                   // 168 MB
enum { kSqStreamed = 0, kSqFrontKept = 1, kSqKept = 2 };

template <bool STREAM>
__device__ __forceinline__ void load_block(const float* __restrict__ x, uint32_t h, f4 (&v)[4][4])
{
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j][q] = ld4<STREAM>(x + 4ull * (256 * q + 64 * j + h));
}

// The sum of squares of block `blk` (the same in the whole wave), valid in lane 0.
template <int READ>
__device__ __forceinline__ float sq_block_sum(const float* __restrict__ x, uint64_t n, uint64_t blk, uint32_t h)
{
    const uint64_t base = blk * 4096;
    f4 v[4][4];                                         // [tree lane h + 64 j][q]
    if (base + 4096 <= n) {
        if constexpr (READ != kSqFrontKept) {
            load_block<READ == kSqStreamed>(x + base, h, v);
        } else if (blk >= kNormKept) {
            asm volatile("" ::: "memory");              // (and behind the loads: or the compiler makes one
            load_block<true>(x + base, h, v);           // branch of the two, without the hint)
            asm volatile("" ::: "memory");
        } else {
            load_block<false>(x + base, h, v);
        }
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint64_t i = base + 4ull * (256 * q + 64 * j + h);
                f4 e;
                e.x = (i + 0 < n) ? x[i + 0] : 0.0f;
                e.y = (i + 1 < n) ? x[i + 1] : 0.0f;
                e.z = (i + 2 < n) ? x[i + 2] : 0.0f;
                e.w = (i + 3 < n) ? x[i + 3] : 0.0f;
                v[j][q] = e;
            }
    }
    __builtin_amdgcn_sched_barrier(0);
    float s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float a = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f4 e = v[j][q];
            a = a + e.x * e.x;
            a = a + e.y * e.y;
            a = a + e.z * e.z;
            a = a + e.w * e.w;
        }
        s[j] = a;
    }
    float r0 = s[0] + s[2];                             // stride 128: lanes h and h+64
    float r1 = s[1] + s[3];
    return tree64(r0 + r1);                             // stride 64 and the rest
}

template <int READ>
__global__ __launch_bounds__(kBlock) void k_sq_partials(const float* __restrict__ x, uint64_t n,
                                                        uint64_t nblk, float* __restrict__ part)
{
    const uint32_t h = threadIdx.x & 63;
    const uint64_t k = (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (k >= nblk) return;                              // whole wave leaves together
    const uint64_t blk = READ == kSqStreamed ? k : nblk - 1 - k;
    const float r = sq_block_sum<READ>(x, n, blk, h);
    if (h == 0) part[blk] = r;
}

// Lane t's share of the partials' tree: partials t, t+256, ... added in that order from +0.  One
// workgroup does this while the GPU waits, so what counts is the number of round trips to memory:
// 32 loads are issued ahead of their adds while that many are left (without the clamp of the
// last round: it kept the loads from going out together), then 8.  The norm of 355 M values
// (86,627 partials) went from 224.7 to 216.2 us, of 109 M from 72.9 to 70.3 us.
__device__ __forceinline__ float lane_partials(const float* __restrict__ part, uint64_t nblk)
{
    float s = 0.0f;
    uint64_t k0 = threadIdx.x;
    for (uint64_t left = nblk; left >= 32 * kBlock; left -= 32 * kBlock, k0 += 32 * kBlock) {
        float v[32];
#pragma unroll
        for (int j = 0; j < 32; ++j) v[j] = part[k0 + j * kBlock];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 32; ++j) s = s + v[j];
    }
    for (; k0 < nblk; k0 += 8 * kBlock) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint64_t k = k0 + (uint64_t)j * kBlock;
            v[j] = part[k < nblk ? k : nblk - 1];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (k0 + (uint64_t)j * kBlock < nblk) s = s + v[j];
    }
    return s;
}

__global__ __launch_bounds__(kBlock) void k_sq_final(const float* __restrict__ part, uint64_t nblk,
                                                     float* __restrict__ out)
{
    __shared__ float lds[kBlock];
    const float s = tree256(lane_partials(part, nblk), lds);
    if (threadIdx.x == 0) {
        out[0] = s;
        out[1] = sqrtf(s);
    }
}

template <int READ>
static hipError_t launch_sq_pair(hipStream_t s, const float* x, uint64_t n, float* part, float* out)
{
    const uint64_t nblk = (n + 4095) / 4096;
    if (nblk)
        ES_RUN(k_sq_partials<READ>, dim3((uint32_t)((nblk + 3) / 4)), dim3(kBlock), kAuxLdsPad, s, x, n, nblk, part);
    ES_RUN(k_sq_final, dim3(1), dim3(kBlock), 0, s, part, nblk, out);
    return hipSuccess;
}

hipError_t launch_sq_norm(hipStream_t s, const float* x, uint64_t n, float* part, float* out)
{
    return launch_sq_pair<kSqFrontKept>(s, x, n, part, out);
}

// Counts a workgroup in (one lane of it calls) and says whether it was the last of all: on one word up to
// kOneCounter workgroups, beyond in kCounters groups whose last members meet on one more, because an addition to
// a word that others add to as well takes 12 ns.  The words are left at zero.
__device__ __forceinline__ bool arrived_last(uint32_t* arrivals, uint32_t groups)
{
    const uint32_t counters = groups > kOneCounter ? kCounters : 1;
    const uint32_t mine = blockIdx.x % counters;
    uint32_t* word = arrivals + mine * kCounterStep;
    if (__hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 !=
        (groups - mine + counters - 1) / counters)
        return false;
    __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (counters == 1) return true;
    word = arrivals + kCounters * kCounterStep;
    if (__hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 != counters) return false;
    __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// The norm of a short vector in one launch: the workgroup whose partials come last adds them all up, with the lanes
// and in the order of k_sq_final; no workgroup waits.
//
// Partials are stored and loaded at agent scope, past the L2 that each compute die has to itself; the one lane
// that stores a workgroup's waits until its stores have been acknowledged before it counts the workgroup in.  The
// language's memory model would ask for a release and an acquire around the count; that these accesses in this order are
// enough is a property of this target, where an agent-scope store is acknowledged at the memory all dies share.  (A
// release fence writes back the whole L2, of the reduce's average too: 4 M 5.7 -> 7.9 us, 8 M 5.9 -> 16.)
//
// Bound by the launch and two round trips.  Against two launches, called from Python one after the other (0.4 us of it the
// binding): 4 k 6.3 -> 3.6 us, 200 k 6.3 -> 4.7, 1 M 6.4 -> 4.9, 4 M 6.4 -> 5.1, 8 M 7.4 -> 5.6; reduce, norm and update of 20 k and
// 4 ranks 15.4 -> 12.2, 200 k and 16 ranks 16.2 -> 13.4, 1 M and 8 ranks 18.5 -> 17.9.  Beyond 2,048 blocks a launch is less than
// a hundredth of such a step.
__global__ __launch_bounds__(kBlock) void k_sq_norm(const float* __restrict__ x, uint64_t n, uint32_t nblk,
                                                    float* part, float* __restrict__ out,
                                                    uint32_t* __restrict__ arrivals, uint32_t groups)
{
    __shared__ float lds[kBlock];
    __shared__ bool last;
    const uint32_t h = threadIdx.x & 63;
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t k = blockIdx.x * 4 + w;
    const float r = k < nblk ? sq_block_sum<kSqKept>(x, n, nblk - 1 - k, h) : 0.0f;
    if (h == 0) lds[w] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
            if (blockIdx.x * 4 + j < nblk)
                __hip_atomic_store(part + (nblk - 1 - (blockIdx.x * 4 + j)), lds[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        last = arrived_last(arrivals, groups);
    }
    __syncthreads();
    if (!last) return;
    float s = 0.0f;
    constexpr uint32_t kMost = kCountedBlocks / kBlock;
    float v[kMost];
#pragma unroll
    for (uint32_t j = 0; j < kMost; ++j) {
        const uint32_t i = threadIdx.x + j * kBlock;
        v[j] = __hip_atomic_load(part + (i < nblk ? i : nblk - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (uint32_t j = 0; j < kMost; ++j)
        if (threadIdx.x + j * kBlock < nblk) s = s + v[j];
    s = tree256(s, lds);
    if (threadIdx.x == 0) {
        out[0] = s;
        out[1] = sqrtf(s);
    }
}

hipError_t launch_sq_norm_counted(hipStream_t s, const float* x, uint64_t n, float* part, float* out, uint32_t* arrivals)
{
    const uint64_t nblk = (n + 4095) / 4096;
    static_assert(kCountedBlocks <= kNormKept, "k_sq_norm reads every block without the hint");
    if (nblk == 0 || nblk > kCountedBlocks) return hipErrorInvalidValue;
    const uint32_t groups = (uint32_t)((nblk + 3) / 4);
    ES_RUN(k_sq_norm, dim3(groups), dim3(kBlock), 0, s, x, n, (uint32_t)nblk, part, out, arrivals, groups);
    return hipSuccess;
}

// Block partials of the allocation-free norm: one array per GPU, part of the code
// object, held until the process ends.  `scratch` is a host-side stand-in for the
// symbol, not a device address: host code only ever uses the address that
// hipGetSymbolAddress returned for the device in question.
static __device__ __align__(256) float scratch[kStaticPartials];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
float* g_scratch_ptr[kMaxDevices] = {};          // per device: where that GPU's copy of `scratch` lives
}

// Device address of the current device's `scratch` (looked up once per device).
static hipError_t static_partials(float** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        float* p = nullptr;
        e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

hipError_t launch_sq_norm_static(hipStream_t s, const float* x, uint64_t n, float* out)
{
    if ((n + 4095) / 4096 > kStaticPartials) return hipErrorInvalidValue;
    float* part = nullptr;
    const hipError_t e = static_partials(&part);
    if (e != hipSuccess) return e;
    // k_sq_partials writes partials [0, nblk) before k_sq_final reads exactly those, so what
    // an earlier call left in the array is never read and nothing has to be cleared
    return launch_sq_pair<kSqStreamed>(s, x, n, part, out);
}

// ---------------------------------------------------------------------------
// Gradient staging: copy one bucket into an EST's context slot (paper §3.2).
// ---------------------------------------------------------------------------
// One 16-byte vector per lane and streaming hints on both sides measured fastest
// on MI355X (about 6.5 TB/s read+write; four vectors per lane: 4.6 TB/s).
//
// Neither side needs 16-byte alignment.  Each wave moves 1 KiB that starts on a 128-byte
// line of the destination (a piece that starts inside a line shares that line with the
// neighbouring workgroup on another compute die, and the line travels twice: measured
// -13 % for buckets at offsets that are not multiples of 128 bytes).  The elements up to
// the first such line and the 0-3 after the last whole vector are copied one by one by the
// first workgroup.  Loads are 16 bytes wide at whatever 4-byte-aligned address that gives
// on the source side (global memory needs dword alignment only): when source and
// destination are equally far off a line - the usual case, a bucket at the same offset in
// a flat gradient and in the slot - they are aligned alike.
typedef float f4_dword_aligned __attribute__((ext_vector_type(4), aligned(4)));

// Short copies (two waves per workgroup) load without the hint: the source has just been written
// and is likely to sit in a cache.
template <uint32_t lanes>
__device__ __forceinline__ void copy_span(float* __restrict__ dst, const float* __restrict__ src,
                                          uint64_t n, uint32_t block, uint32_t lane)
{
    constexpr uintptr_t kAlign = 128;                    // 1 KiB alignment measured no better
    uint64_t head = ((kAlign - (reinterpret_cast<uintptr_t>(dst) & (kAlign - 1))) & (kAlign - 1)) >> 2;
    if (head > n) head = n;
    const float* __restrict__ sb = src + head;
    float* __restrict__ db = dst + head;
    const uint64_t nb = n - head;
    const uint64_t nvec = nb >> 2;
    const uint64_t i = (uint64_t)block * lanes + lane;
    if (i < nvec) {
        const f4_dword_aligned* from = reinterpret_cast<const f4_dword_aligned*>(sb + 4 * i);
        const f4 x = lanes == kCopyBlockShort ? *from : __builtin_nontemporal_load(from);
        __builtin_nontemporal_store(x, reinterpret_cast<f4*>(db + 4 * i));
    }
    if (block == 0) {
        for (uint64_t e = lane; e < head; e += lanes) dst[e] = src[e];
        const uint64_t e = 4 * nvec + lane;
        if (lane < 4 && e < nb) db[e] = sb[e];
    }
}

template <uint32_t BS>
__global__ __launch_bounds__(BS) void k_copy_f4(float* __restrict__ dst, const float* __restrict__ src, uint64_t n)
{
    copy_span<BS>(dst, src, n, blockIdx.x, threadIdx.x);
}

static hipError_t launch_copy(hipStream_t s, float* dst, const float* src, uint64_t n, uint32_t bs)
{
    uint64_t blocks = ((n >> 2) + bs - 1) / bs;
    if (blocks == 0) blocks = 1;
    if (bs == kCopyBlockShort)
        ES_RUN(k_copy_f4<kCopyBlockShort>, dim3((uint32_t)blocks), dim3(bs), 0, s, dst, src, n);
    else
        ES_RUN(k_copy_f4<kCopyBlock>, dim3((uint32_t)blocks), dim3(bs), 0, s, dst, src, n);
    return hipSuccess;
}

hipError_t launch_copy_f32(hipStream_t s, float* dst, const float* src, uint64_t n)
{
    return n ? launch_copy(s, dst, src, n, copy_block(n)) : hipSuccess;
}

// Batched staging: the runs arrive as a kernel argument (no table upload); a
// workgroup finds its run from the prefix sums (wave-uniform, scalar).
template <uint32_t BS>
__global__ __launch_bounds__(BS) void k_copy_runs(const CopyRuns runs)
{
    // the run of this workgroup = how many later runs start at or before it.  All prefix sums
    // are fetched at once (independent scalar loads of the kernel argument) and compared in
    // registers: a dependent load per run would be most of this short workgroup's life.
    // (Entries past the last run hold 0xFFFFFFFF, so the count needs no bound.)  A single run -
    // one flat gradient vector, the common case - goes to k_copy_f4: the lookup costs 2.7 % there,
    // and its 24 bytes of arguments are a twentieth of these.
    uint32_t r = 0;
#pragma unroll
    for (int k = 1; k < kMaxRuns; ++k) r += blockIdx.x >= runs.first_block[k] ? 1u : 0u;
    copy_span<BS>(runs.dst[r], runs.src[r], runs.n[r], blockIdx.x - runs.first_block[r], threadIdx.x);
}

hipError_t launch_copy_runs(hipStream_t s, const CopyRuns& runs)
{
    if (runs.n_runs == 0) return hipSuccess;
    if (runs.n_runs == 1) return launch_copy(s, runs.dst[0], runs.src[0], runs.n[0], runs.block);
    const uint32_t blocks = runs.first_block[runs.n_runs];
    if (blocks == 0) return hipSuccess;
    if (runs.block == kCopyBlockShort)
        ES_RUN(k_copy_runs<kCopyBlockShort>, dim3(blocks), dim3(kCopyBlockShort), 0, s, runs);
    else
        ES_RUN(k_copy_runs<kCopyBlock>, dim3(blocks), dim3(kCopyBlock), 0, s, runs);
    return hipSuccess;
}

__global__ __launch_bounds__(kBlock) void k_copy_bytes(uint8_t* __restrict__ dst,
                                                       const uint8_t* __restrict__ src, uint64_t n16)
{
    const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n16) reinterpret_cast<u4*>(dst)[i] = reinterpret_cast<const u4*>(src)[i];
}

// dst, src 16-byte aligned, n a multiple of 16
hipError_t launch_copy_bytes(hipStream_t s, uint8_t* dst, const uint8_t* src, uint64_t n)
{
    if (n == 0) return hipSuccess;
    const uint64_t n16 = n >> 4;
    const uint64_t blocks = (n16 + kBlock - 1) / kBlock;
    ES_RUN(k_copy_bytes, dim3((uint32_t)blocks), dim3(kBlock), 0, s, dst, src, n16);
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Small-state context switch (paper §3.2): scattered live tensors <-> one
// contiguous slot, all segments in one launch.  One workgroup per Piece.
// In kSwitch every lane reads its live bytes, then overwrites them with the
// incoming EST's bytes: outgoing and incoming state never meet across lanes.
// ---------------------------------------------------------------------------
template <typename T, uint32_t BS = kBlock>
__device__ __forceinline__ void ctx_move(T* live, T* sa, const T* sb, uint32_t n, int dir)
{
    for (uint32_t i = threadIdx.x; i < n; i += BS) {
        if (dir == kSave) {
            sa[i] = live[i];
        } else if (dir == kRestore) {
            live[i] = sa[i];
        } else {
            const T out = live[i];
            const T in = sb[i];
            sa[i] = out;
            live[i] = in;
        }
    }
}

template <uint32_t BS>
__device__ __forceinline__ void ctx_piece(const Piece ES_CONST_AS* pieces, uint32_t k, uint8_t* slot_a,
                                          const uint8_t* slot_b, int dir)
{
    uint8_t* live = (uint8_t*)pieces[k].live;
    const uint64_t so = pieces[k].slot_off;
    const uint32_t nb = pieces[k].nbytes;
    const uint32_t w = pieces[k].width;
    uint8_t* sa = slot_a + so;
    const uint8_t* sb = slot_b ? slot_b + so : nullptr;
    if (w == 16)
        ctx_move<u4, BS>((u4*)live, (u4*)sa, (const u4*)sb, nb >> 4, dir);
    else if (w == 4)
        ctx_move<uint32_t, BS>((uint32_t*)live, (uint32_t*)sa, (const uint32_t*)sb, nb >> 2, dir);
    else
        ctx_move<uint8_t, BS>(live, sa, sb, nb, dir);
}

__global__ __launch_bounds__(kBlock) void k_ctx(const Piece* pieces_g, uint8_t* slot_a,
                                                const uint8_t* slot_b, int dir)
{
    ctx_piece<kBlock>((const Piece ES_CONST_AS*)pieces_g, blockIdx.x, slot_a, slot_b, dir);
}

// An EST boundary in one launch (paper section 3.2: at a mini-batch boundary the outgoing EST's
// context is saved, its gradients are copied aside, and the incoming EST's context is restored):
// the first n_pieces workgroups move small-state pieces (save, or save + restore per byte in one
// lane), all others are the staging copy of the outgoing EST's gradient runs.  The two parts touch
// disjoint memory, so no ordering between them is needed inside the launch.
// RUNS is CopyRuns, or CopyRun where the gradients are one run (the common case: no lookup, and 24
// instead of 464 bytes of a table, 60 instead of 500 of arguments in all, for the host to write and every
// workgroup to fetch).
template <uint32_t BS, typename RUNS>
__global__ __launch_bounds__(BS) void k_est_boundary(const RUNS runs, const Piece* pieces_g,
                                                     uint32_t n_pieces, uint8_t* slot_a,
                                                     const uint8_t* slot_b, int dir)
{
    if (blockIdx.x < n_pieces) {
        ctx_piece<BS>((const Piece ES_CONST_AS*)pieces_g, blockIdx.x, slot_a, slot_b, dir);
        return;
    }
    const uint32_t blk = blockIdx.x - n_pieces;
    if constexpr (std::is_same_v<RUNS, CopyRun>) {
        copy_span<BS>(runs.dst, runs.src, runs.n, blk, threadIdx.x);
    } else {
        uint32_t r = 0;
#pragma unroll
        for (int k = 1; k < kMaxRuns; ++k) r += blk >= runs.first_block[k] ? 1u : 0u;
        copy_span<BS>(runs.dst[r], runs.src[r], runs.n[r], blk - runs.first_block[r], threadIdx.x);
    }
}

hipError_t launch_est_boundary(hipStream_t s, const CopyRuns& runs, const Piece* pieces, uint32_t n_pieces,
                               uint8_t* slot_a, const uint8_t* slot_b, CtxDir dir)
{
    const uint32_t copy_blocks = runs.n_runs ? runs.first_block[runs.n_runs] : 0;
    if (n_pieces + copy_blocks == 0) return hipSuccess;
    const dim3 grid(n_pieces + copy_blocks), block(runs.block);
#define ES_BOUNDARY(BS, RUNS, R) \
    ES_RUN((k_est_boundary<BS, RUNS>), grid, block, 0, s, R, pieces, n_pieces, slot_a, slot_b, (int)dir)
    if (runs.n_runs <= 1) {
        const CopyRun one{runs.dst[0], runs.src[0], runs.n[0]};   // n_runs = 0: no workgroup gets that far
        if (runs.block == kCopyBlockShort) ES_BOUNDARY(kCopyBlockShort, CopyRun, one);
        else ES_BOUNDARY(kCopyBlock, CopyRun, one);
    } else {
        if (runs.block == kCopyBlockShort) ES_BOUNDARY(kCopyBlockShort, CopyRuns, runs);
        else ES_BOUNDARY(kCopyBlock, CopyRuns, runs);
    }
#undef ES_BOUNDARY
    return hipSuccess;
}

hipError_t launch_ctx(hipStream_t s, const Piece* pieces, uint32_t n_pieces, uint8_t* slot_a,
                      const uint8_t* slot_b, CtxDir dir)
{
    if (n_pieces == 0) return hipSuccess;
    ES_RUN(k_ctx, dim3(n_pieces), dim3(kBlock), 0, s, pieces, slot_a, slot_b, (int)dir);
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Dropout keep-mask from an EST's live RNG state (paper §3.3: Dropout depends
// on RNG state, which is therefore EST context).  Philox4x32-10 after Salmon,
// Moraes, Dror, Shaw (SC'11): ten rounds of two 32x32->64 multiplies whose
// high halves are mixed with the other two counter words and the key; the key
// advances by two Weyl constants per round.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t (&out)[4])
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t a = (uint64_t)0xD2511F53u * c0;
        const uint64_t b = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = (uint32_t)(b >> 32) ^ c1 ^ k0;
        const uint32_t n2 = (uint32_t)(a >> 32) ^ c3 ^ k1;
        c1 = (uint32_t)b;
        c3 = (uint32_t)a;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// a ^ b ^ c in one instruction (the compiler leaves two)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// The same ten rounds for a counter (c0, hi, 0, 0) whose second word is the same in the whole wave:
// the first product with c2 = 0 vanishes, the second round's product of (hi ^ k0) is a scalar one, and
// the words they would have fed drop out of the exclusive ors.  18 vector products instead of 20 (two
// of them scalar) and 19 exclusive ors instead of 40.
__device__ __forceinline__ void philox4x32_10_uniform_hi(uint32_t c0, uint32_t hi, uint32_t k0, uint32_t k1,
                                                         uint32_t (&out)[4])
{
    constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
    const uint64_t a0 = (uint64_t)M0 * c0;
    const uint64_t a1 = (uint64_t)M0 * (hi ^ k0);       // uniform
    uint32_t c2 = (uint32_t)(a0 >> 32) ^ k1;
    const uint64_t b1 = (uint64_t)M1 * c2;
    k0 += W0;
    k1 += W1;
    c0 = (uint32_t)(b1 >> 32) ^ k0;
    c2 = (uint32_t)a0 ^ ((uint32_t)(a1 >> 32) ^ k1);
    uint32_t c1 = (uint32_t)b1, c3 = (uint32_t)a1;      // c3 uniform here
#pragma unroll
    for (int round = 2; round < 10; ++round) {
        k0 += W0;
        k1 += W1;
        const uint64_t a = (uint64_t)M0 * c0;
        const uint64_t b = (uint64_t)M1 * c2;
        c0 = xor3((uint32_t)(b >> 32), c1, k0);
        c2 = round == 2 ? (uint32_t)(a >> 32) ^ (c3 ^ k1) : xor3((uint32_t)(a >> 32), c3, k1);
        c1 = (uint32_t)b;
        c3 = (uint32_t)a;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// 1 if w >= threshold, else 0, for keep = 2^32 - threshold: the carry of a 64-bit sum.  (A comparison and a
// selection through a mask register take 12.7 cycles of a SIMD, this product by one 4.6; 2^32 and 0 are
// thresholds like any other.)
__device__ __forceinline__ uint32_t kept(uint32_t w, uint64_t keep)
{
    uint64_t sum, carry;
    asm("v_mad_u64_u32 %0, %1, %2, 1, %3" : "=v"(sum), "=s"(carry) : "v"(w), "s"(keep));
    return (uint32_t)(sum >> 32);
}

// bytes << 8 | kept(w, keep) in one instruction more (the compiler, which cannot know that the second is 0 or 1,
// makes two or three of it)
__device__ __forceinline__ uint32_t push_kept(uint32_t bytes, uint32_t w, uint64_t keep)
{
    uint32_t r;
    asm("v_lshl_or_b32 %0, %1, 8, %2" : "=v"(r) : "v"(bytes), "v"(kept(w, keep)));
    return r;
}

// The 16 mask bytes (4 counter values) of a lane of the wave that starts at the 16 bytes number `first`:
// byte j is 1 iff its word reaches the threshold.  All arguments but the lane are uniform.
__device__ __forceinline__ void mask_bytes(uint32_t lane, uint64_t first, uint64_t offset, uint32_t k0, uint32_t k1,
                                           uint64_t keep, uint32_t (&packed)[4])
{
    const uint64_t base = offset + 4 * first;           // the wave's counters are base .. base + 255
    auto pack = [&](const uint32_t (&w)[4]) {
        return push_kept(push_kept(push_kept(kept(w[3], keep), w[2], keep), w[1], keep), w[0], keep);
    };
    if ((uint32_t)base <= 0xFFFFFFFFu - 255u) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t w[4];
            philox4x32_10_uniform_hi((uint32_t)base + (4 * lane + q), (uint32_t)(base >> 32), k0, k1, w);
            packed[q] = pack(w);
        }
    } else {                                            // a carry into the second word inside the wave
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t w[4];
            const uint64_t pos = base + (4 * lane + q);
            philox4x32_10((uint32_t)pos, (uint32_t)(pos >> 32), 0u, 0u, k0, k1, w);
            packed[q] = pack(w);
        }
    }
}

// Bytes j0 .. j0 + 15 of a mask of which n bytes are left; none beyond.
__device__ __forceinline__ void store_mask(uint8_t* __restrict__ mask, uint32_t j0, uint64_t n, int aligned16,
                                           const uint32_t (&packed)[4])
{
    if (aligned16 && j0 + 16 <= n) {
        u4 o = {packed[0], packed[1], packed[2], packed[3]};
        *reinterpret_cast<u4*>(mask + j0) = o;
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (j0 + i < n) mask[j0 + i] = (uint8_t)((packed[i >> 2] >> (8 * (i & 3))) & 0xFF);
    }
}

// The wave-uniform 64-bit value of a lane's v.
__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    return (uint64_t)hi << 32 | lo;
}

constexpr uint64_t kMaskGroups = 2048;                  // 8 workgroups of 4 waves per CU: all that are resident

// Each lane draws 4 counter values = 16 mask bytes at a time.  Whichever workgroup is the last to have
// read the state advances the offset, so no second launch is needed; no workgroup waits for another.
// `arrivals` (one line per counter, zero between launches) counts them: on one counter up to kOneCounter
// workgroups, beyond in kCounters groups whose last members meet on one more (an addition to a word
// that others add to as well takes 12 ns: 1,024 of them 13 us on one word, nothing to be seen on 16).  That is
// what arrived_last does, written out: the draw lies between the count and its evaluation here, and
// with the helper called after it 16x12x512x512 bytes took 16.6 us for 15.2.
//
// Integer-ALU bound: per four bytes 18 products, 19 exclusive ors and 7 instructions to compare and pack.
// One launch instead of two, called from Python one after the other (0.7 us of it the binding): 16 KiB to 1 MB 6.5 ->
// 3.5 us a mask (that is what a launch costs the host), 3.7 MB 6.8 -> 4.5, 10 MB 8.0 -> 7.1, 16x12x512x512 bytes 22.6 -> 20.9,
// 143 MB 52.1 -> 49.6; 16x12x512x512 where passes overlap 16.9 -> 15.5 (3.2 TB/s of stores).
//
// A draw that is captured into a graph can be replayed when the counters are gone, or beside another draw that uses
// them: it only reads the state (COUNTED = false), and k_philox_advance follows it (in a graph 4.2 us up to 1 MB, 5.5 for
// 3.7 MB).
template <bool COUNTED>
__global__ __launch_bounds__(kBlock) void k_dropout_mask(uint64_t* __restrict__ state, uint8_t* __restrict__ mask,
                                                         uint64_t n, uint64_t keep, int aligned16,
                                                         uint32_t* __restrict__ arrivals, uint32_t groups)
{
    const uint64_t seed = uniform64(state[0]);
    const uint64_t offset = uniform64(state[1]);
    __syncthreads();                                    // every wave has its copy of the state
    const uint32_t counters = groups > kOneCounter ? kCounters : 1;
    const uint32_t mine = blockIdx.x % counters;
    uint32_t before = 0;
    if (COUNTED && threadIdx.x == 0)
        before = __hip_atomic_fetch_add(arrivals + mine * kCounterStep, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t lane = threadIdx.x & 63;
    uint64_t first = (uint64_t)blockIdx.x * kBlock + __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
    for (; 16 * first < n; first += groups * kBlock) {  // `first` and the bounds stay in scalar registers
        uint32_t packed[4];
        mask_bytes(lane, first, offset, (uint32_t)seed, (uint32_t)(seed >> 32), keep, packed);
        store_mask(mask + 16 * first, 16 * lane, n - 16 * first, aligned16, packed);
    }
    if (!COUNTED || threadIdx.x != 0 || before + 1 != (groups - mine + counters - 1) / counters) return;
    __hip_atomic_store(arrivals + mine * kCounterStep, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (counters > 1) {
        uint32_t* last = arrivals + kCounters * kCounterStep;
        if (__hip_atomic_fetch_add(last, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 != counters) return;
        __hip_atomic_store(last, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    state[1] = offset + (n + 3) / 4;
}

__global__ void k_philox_advance(uint64_t* state, uint64_t blocks)
{
    if (threadIdx.x == 0) state[1] = state[1] + blocks;
}

// A short mask: one workgroup of up to 16 waves draws all of it and advances the offset it has read.
__global__ __launch_bounds__(kMaskGroup) void k_dropout_mask_short(uint64_t* __restrict__ state,
                                                                   uint8_t* __restrict__ mask, uint64_t n,
                                                                   uint64_t keep, int aligned16)
{
    const uint64_t seed = uniform64(state[0]);
    const uint64_t offset = uniform64(state[1]);
    __syncthreads();                                    // every wave has its copy of the state
    if (threadIdx.x == 0) state[1] = offset + (n + 3) / 4;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t first = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
    uint32_t packed[4];
    mask_bytes(lane, first, offset, (uint32_t)seed, (uint32_t)(seed >> 32), keep, packed);
    store_mask(mask + 16 * first, 16 * lane, n - 16 * first, aligned16, packed);
}

hipError_t launch_dropout_mask(hipStream_t s, uint64_t* state, uint8_t* mask, uint64_t n, uint64_t threshold)
{
    if (n == 0) return hipSuccess;
    if (n > kShortMask) return hipErrorInvalidValue;
    const uint32_t block = (uint32_t)(((n + 15) / 16 + 63) / 64 * 64);
    ES_RUN(k_dropout_mask_short, dim3(1), dim3(block), 0, s, state, mask, n, (1ull << 32) - threshold,
                       ((uintptr_t)mask & 15) == 0);
    return hipSuccess;
}

static uint32_t mask_groups(uint64_t n)
{
    const uint64_t all = ((n + 15) / 16 + kBlock - 1) / kBlock;
    return (uint32_t)(all < kMaskGroups ? all : kMaskGroups);
}

hipError_t launch_dropout_mask_captured(hipStream_t s, uint64_t* state, uint8_t* mask, uint64_t n, uint64_t threshold)
{
    if (n == 0) return hipSuccess;
    const uint32_t groups = mask_groups(n);
    ES_RUN(k_dropout_mask<false>, dim3(groups), dim3(kBlock), 0, s, state, mask, n, (1ull << 32) - threshold,
                       ((uintptr_t)mask & 15) == 0, nullptr, groups);
    ES_RUN(k_philox_advance, dim3(1), dim3(64), 0, s, state, (n + 3) / 4);
    return hipSuccess;
}

hipError_t launch_dropout_mask_long(hipStream_t s, uint64_t* state, uint8_t* mask, uint64_t n, uint64_t threshold,
                                    uint32_t* arrivals)
{
    if (n == 0) return hipSuccess;
    const uint32_t groups = mask_groups(n);
    ES_RUN(k_dropout_mask<true>, dim3(groups), dim3(kBlock), 0, s, state, mask, n, (1ull << 32) - threshold,
                       ((uintptr_t)mask & 15) == 0, arrivals, groups);
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// BatchNorm batch statistics along the fixed tree (the paper's level D2, section 3.3: a
// reduce whose result does not depend on the GPU; BatchNorm is the operator whose statistics
// every EST tracks).  x is [B][C][HW].  For channel ch the M = B*HW values in the order
// (image, position) form a vector y; its terms f(y[m]) are summed along the tree of the norm
// (blocks of 4096 terms; lane t adds terms 4*(256*q + t) + c, q outer, c inner, from +0;
// stride halving over 256 lanes; block partials combined the same way, lane t first adding
// partials t, t+256, ...).  mean = T(y) / M, var = T((y - mean)^2) / M.
//
// One WAVE per block of one channel; hardware lane h plays tree lanes h, h+64, h+128, h+192
// (strides 128 and 64 are adds between its own registers, 32..1 lane exchanges).
// ---------------------------------------------------------------------------
struct BnGeom {
    uint32_t C, HW, M, nblk;
    uint64_t magic;                                     // m / HW = (m * magic) >> shift for m < 2^31
    uint32_t shift;
    uint32_t step_img, step_pos;                        // 256 = step_img * HW + step_pos
};

// The same as kernel arguments: single words in front of all others, so that they are in registers when a wave
// starts (a structure never is; fetching it was one or two round trips before the first load's address).  One layer after
// the other, without and with the arguments in registers: 32x2048x7x7 6.15 -> 5.92 us, 32x512x7x7 4.62 -> 4.23, 32x256x9x9
// 5.48 -> 5.06, 8x192x35x35 4.44 -> 4.17, 32x64x112x112 21.0 -> 20.6.
#define ES_BN_GEOM_PARAMS uint64_t magic, uint32_t C, uint32_t HW, uint32_t M, uint32_t shift_step
#define ES_BN_GEOM_ARGS(g) (g).magic, (g).C, (g).HW, (g).M, (g).shift | (g).step_img << 8
#define ES_BN_GEOM                                                                                                    \
    BnGeom { C, HW, M, (M + 4095) >> 12, magic, shift_step & 0xFF, shift_step >> 8, 256 - (shift_step >> 8) * HW }

// How four consecutive terms lie in memory.
enum { kBnVector = 0, kBnLong = 1, kBnWrap = 2, kBnAny = 3 };
// kBnVector: HW is a multiple of 4, so they are one 16-byte vector of one image.
// kBnWrap:   4 <= HW, any remainder: the image can end once inside them.  One vector all the same; where the image ends, the
//            values behind its end are loaded over it one by one (a vector and at most three loads of a few lanes each, for
//            four loads of all lanes 16 bytes apart, which fetch every line four times: 32x2048x7x7 5.42 -> 3.86 us,
//            200x64x11x11 7.74 -> 4.89, 158x134x13x13 7.74 -> 4.69, 256x512x3x3 4.89 -> 3.69; from two
//            blocks of up to 9 positions on 0.9-1.27 of the time, 2000x256x7 7.8 and 9.9, so those keep single loads).
// kBnLong:   long images, HW >= kBnLongHW: a plain vector if no image (nor the channel) ends inside the wave's 256 terms,
//            else four single loads.  Fewer instructions where images seldom end.  kBnWrap over it, up to 25 blocks a
//            channel: 0.65 at 289 positions, 0.74 at 625, 0.81-0.98 at 841, 0.77-0.97 at 961 to 1,369, 0.98-1.0 at 2,025, 0.97-1.02
//            at 3,025; where workgroups share a channel, which then is read at the rate of the HBM, 1.06 at 841
//            and 1.03 at 2,809.
// kBnAny:    HW < 4.
constexpr uint32_t kBnLongHW = 2560, kBnLongSharedHW = 128;

// The 16 vectors of lane h of block `blk`, [tree lane h + 64 j][q].  Where a term lies beyond M
// some value of the channel is loaded instead; bn_block_sum drops it.
// A lane's vectors are 256 terms apart, so (image, position) is divided out once and then
// stepped: a division per vector was most of the kernel's instructions.  OFF is the type of a
// byte offset into x (32 bits where x is small enough: one scalar base, one register per lane).
template <int MODE, typename OFF>
__device__ __forceinline__ void bn_load(const float* __restrict__ x, const BnGeom& g, uint32_t ch, uint32_t blk,
                                        uint32_t h, f4 (&t)[4][4])
{
    const char* xb = reinterpret_cast<const char*>(x);
    const OFF image = (OFF)4 * g.C * g.HW;              // bytes between images
    const OFF wrap = image - (OFF)4 * g.HW;             // what an image's end adds to the offset
    const OFF first = (OFF)4 * ch * g.HW;               // the channel's first value: always readable
    const OFF step = image * g.step_img + 4u * g.step_pos;
    uint32_t m = blk * 4096u + 4u * h;
    uint32_t img = (uint32_t)(((uint64_t)m * g.magic) >> g.shift);
    uint32_t pos = m - img * g.HW;
    OFF off = first + image * img + (OFF)4 * pos;
    // Single loads for all terms even so: the end of the last channel where it fills no vector (there may be nothing to read
    // behind it), and longer channels of tiny images, where a wave's 256 terms end an image in every second or third lane.
    const bool end = ch + 1 == g.C && (g.M & 3) != 0 && g.M >> 12 == blk;
    const bool tiny = g.HW < 10 && g.M > 4096;
    if (MODE == kBnWrap && !end && !tiny) {
        uint32_t left = g.HW - 1 - pos;                 // values of the image behind the vector's first
        const int at = 4 * (int)h;
        const int ends = (int)(g.M - blk * 4096u);      // terms from the block's first to the channel's end
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            f4& e = t[i & 3][i >> 2];
            if (256 * i >= ends) {                      // the whole wave is beyond M: no loads
                e = f4{0.0f, 0.0f, 0.0f, 0.0f};
            } else {
                e = *reinterpret_cast<const f4_dword_aligned*>(xb + (at < ends - 256 * i ? off : first));
                if (left < 3 && at < ends - 256 * i - 3) {
                    OFF next = off + wrap;
                    asm volatile("" : "+v"(next));      // the branches below need no address of their own
                    e.w = *reinterpret_cast<const float*>(xb + next + 12);
                    if (left < 2) {
                        e.z = *reinterpret_cast<const float*>(xb + next + 8);
                        if (left < 1) e.y = *reinterpret_cast<const float*>(xb + next + 4);
                    }
                }
            }
            off += step + (left < g.step_pos ? wrap : (OFF)0);
            const uint32_t down = left - g.step_pos, over = down + g.HW;
            left = down < over ? down : over;           // whichever has not passed 2^32
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        f4& e = t[i & 3][i >> 2];
        auto singles = [&] {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                OFF o;
                if constexpr (MODE != kBnAny) {
                    o = off + 4u * c + (pos + c >= g.HW ? wrap : (OFF)0);
                } else {
                    const uint32_t im = (uint32_t)(((uint64_t)(m + c) * g.magic) >> g.shift);
                    o = first + image * im + (OFF)4 * (m + c - im * g.HW);
                }
                e[c] = *reinterpret_cast<const float*>(xb + (m + c < g.M ? o : first));
            }
        };
        if constexpr (MODE == kBnVector) {              // M is a multiple of 4 too
            e = *reinterpret_cast<const f4_dword_aligned*>(xb + (m < g.M ? off : first));
        } else if constexpr (MODE == kBnLong) {
            if (blk * 4096u + 256u * i >= g.M) e = f4{0.0f, 0.0f, 0.0f, 0.0f};
            else if (__any(pos + 3 >= g.HW || m + 3 >= g.M)) singles();
            else e = *reinterpret_cast<const f4_dword_aligned*>(xb + off);
        } else {
            // the whole wave is beyond M: no loads (four of them can cost more than this branch: 500x256x3 4.9 -> 3.9 us,
            // 1000x256x7 4.8 -> 4.5, but 1600x256x3 5.4 -> 5.7; the one load of kBnVector does not: 32x512x28x28 8.9 -> 9.8)
            if (blk * 4096u + 256u * i < g.M) singles();
            else e = f4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        m += 256;
        pos += g.step_pos;
        off += step;
        if (pos >= g.HW) {
            pos -= g.HW;
            off += wrap;
        }
    }
}

// The block's partial sum (valid in lane 0): of the terms, or of their squared distance to
// `mean`; terms beyond M count as +0.
//
// With a wave or two per SIMD what counts here is the number of instructions.  A channel's last block is mostly empty (49
// positions of 32 images are 1,568 terms of 4,096): its quarters behind M are left out, and only the one that M lies in is
// masked term by term.  All 64 terms masked -> so: 32x2048x7x7 5.93 -> 5.44 us, 8x2048x7x7 4.30 -> 3.32, 13x500x59x59 17.8 ->
// 15.5, 32x512x14x14 4.92 -> 4.46.
template <bool SQDEV, bool FULL>
__device__ __forceinline__ float bn_block_sum_of(const f4 (&t)[4][4], uint32_t blk, uint32_t h, uint32_t M, float mean)
{
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        auto add = [&](auto whole) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f4 e = t[j][q];
                if constexpr (SQDEV) {
                    const f4 d = e - mean;
                    e = d * d;
                }
                if constexpr (!decltype(whole)::value) {
                    const uint32_t m = blk * 4096u + 4u * (256 * q + 64 * j + h);
#pragma unroll
                    for (int c = 0; c < 4; ++c) e[c] = m + c < M ? e[c] : 0.0f;
                }
                s[j] = s[j] + e.x;
                s[j] = s[j] + e.y;
                s[j] = s[j] + e.z;
                s[j] = s[j] + e.w;
            }
        };
        // a sum is never -0, so +0 need not be added
        if (FULL || blk * 4096u + 1024u * (q + 1) <= M) add(std::true_type{});
        else if (blk * 4096u + 1024u * q < M) add(std::false_type{});
    }
    const float r0 = s[0] + s[2];                       // stride 128
    const float r1 = s[1] + s[3];
    return tree64(r0 + r1);                             // stride 64 and the rest
}

template <bool SQDEV>
__device__ __forceinline__ float bn_block_sum(const f4 (&t)[4][4], uint32_t blk, uint32_t h, uint32_t M, float mean)
{
    return (uint64_t)blk * 4096 + 4096 <= M ? bn_block_sum_of<SQDEV, true>(t, blk, h, M, mean)
                                            : bn_block_sum_of<SQDEV, false>(t, blk, h, M, mean);
}

// A channel of at most kBnWaves + kBnExtra blocks: one workgroup, everything in one launch, x
// read once.  Each wave keeps one block in registers (64 per lane) and, in the EXTRA form, the
// first waves park a second one in LDS; the second pass costs no memory traffic.  The block
// partials meet in LDS, where every wave sums them for itself: at most 64 partials are lanes
// 0..63 of the tree, and its strides 128 and 64 only add +0.  With one block per channel a
// workgroup takes one channel per wave instead and needs no LDS.
// Bound by the launch and one round trip to memory for small layers, by HBM for large ones.
// Two passes of two launches each, and this as it is now: 32x2048x7x7 27.2 and 3.9 us, 32x512x28x28
// 23.8 and 8.9, 32x256x56x56 (25 blocks, parked) 46.7 and 18.0 = 5.7 TB/s.
constexpr uint32_t kBnWaves = 16;                       // 1024 lanes: the registers of a CU hold 16 blocks
constexpr uint32_t kBnExtra = 9;                        // 16 KiB each: what fits in 160 KiB beside the partials
constexpr uint32_t kBnSingles = 4;                      // channels per workgroup when a channel is one block
enum { kBnSingle = 0, kBnRegs = 1, kBnParked = 2 };

// Workgroups that follow each other go to the eight compute dies in turn, each with an L2 of its own; this is the piece of
// work, of n, for workgroup b, such that the pieces a die has follow each other.  A permutation of 0 .. n - 1 wherever the
// workgroups run.  Channels that follow each other share lines of memory: always where an image's positions fill less
// than a line, at both ends otherwise.  In the order of dispatch every die that has one of them fetches the line.  So, against
// that: 900x2048x5 56.4 -> 16.2 us, 512x1024x9 17.4 -> 8.0, 256x2048x25 20.2 -> 15.7, 128x512x7x7 6.03 -> 5.56, 32x512x14x14 4.39 ->
// 3.77; where images are whole lines (32x512x28x28 9.21 -> 8.93, 64x256x56x56) nothing is lost.  Long channels of images of
// one position lose, where they are many: 25 blocks, 160, 256, 300, 512 and 1,000 channels 140 -> 125, 221 -> 244, 320 -> 285,
// 412 -> 417 and 674 -> 705.
__device__ __forceinline__ uint32_t die_contiguous(uint32_t b, uint32_t n)
{
    const uint32_t die = b & 7, each = n >> 3, more = n & 7;
    return die * each + (die < more ? die : more) + (b >> 3);
}

template <int MODE, typename OFF, int FORM>
__global__ __launch_bounds__(FORM == kBnSingle ? 64 * kBnSingles : 64 * kBnWaves)
void k_bn_channel(const float* __restrict__ x, float* __restrict__ mean, float* __restrict__ var, ES_BN_GEOM_PARAMS)
{
    const BnGeom g = ES_BN_GEOM;
    const float fM = (float)M;
    extern __shared__ __align__(16) float park[];       // kBnParked: [extra block][vector][lane]
    __shared__ float part[2][kBnWaves + kBnExtra];
    const uint32_t h = threadIdx.x & 63;
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t pieces = FORM == kBnSingle ? (C + kBnSingles - 1) / kBnSingles : C;
    const uint32_t ch = die_contiguous(blockIdx.x, pieces) * (FORM == kBnSingle ? kBnSingles : 1) + (FORM == kBnSingle ? w : 0);
    const uint32_t blk = FORM == kBnSingle ? 0 : w;
    if (FORM == kBnSingle && ch >= g.C) return;         // whole wave; no barrier in this form
    const uint32_t blk2 = kBnWaves + w;
    const bool two = FORM == kBnParked && blk2 < g.nblk;
    f4* mine = reinterpret_cast<f4*>(park) + (w * 16) * 64 + h;
    f4 t[4][4];
    if (two) {                                          // what a lane parks only that lane reads back
        bn_load<MODE, OFF>(x, g, ch, blk2, h, t);
#pragma unroll
        for (int i = 0; i < 16; ++i) mine[64 * i] = t[i & 3][i >> 2];
        const float s = bn_block_sum<false>(t, blk2, h, g.M, 0.0f);
        if (h == 0) part[0][blk2] = s;
    }
    bn_load<MODE, OFF>(x, g, ch, blk, h, t);
    __builtin_amdgcn_sched_barrier(0);
    auto combine = [&](float s, int pass) {
        if constexpr (FORM == kBnSingle) {
            return lane0(s) / fM;
        } else {
            if (h == 0) part[pass][w] = s;
            __syncthreads();
            return lane0(tree64(h < g.nblk ? 0.0f + part[pass][h] : 0.0f)) / fM;
        }
    };
    const float mu = combine(bn_block_sum<false>(t, blk, h, g.M, 0.0f), 0);
    const float s = bn_block_sum<true>(t, blk, h, g.M, mu);
    if (two) {
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i & 3][i >> 2] = mine[64 * i];
        const float s2 = bn_block_sum<true>(t, blk2, h, g.M, mu);
        if (h == 0) part[1][blk2] = s2;
    }
    const float va = combine(s, 1);
    if (h == 0 && (FORM == kBnSingle || w == 0)) {
        mean[ch] = mu;
        var[ch] = va;
    }
}

// A channel of 26 to 1,024 blocks, x read once all the same: several workgroups hold its blocks, three per
// wave in registers and one in LDS (32 per CU: 134 MB on the chip), and wait for each other's sums of the first
// pass.  Workgroup g of G (a power of two) has the blocks g, g + G, g + 2G, ..: tree lanes t and t + 256 and the
// strides down to G stay inside it, and its one sum is lane g of the tree's last levels.
//
// The sums travel through the workspace, whose contents are not known beforehand, so every one carries the launch's
// tag: 64 bits that no other launch of the process has and that other contents hold with a probability of
// 2^-64.  (A launch before this one could clear the workspace instead, at 3 us; a captured launch, whose tag comes
// back with every replay, has that.)  Nothing depends on all workgroups of a channel being resident at once: one that has
// looked for the others' sums `polls` times computes them from memory and goes on.
//
// Bound by reading x (6.4 TB/s), then by the second pass over what is held (three operations per value: 1.9 of 20.7 us on
// 32x64x112x112) and the exchange of sums (0.8 us of them).  Reading x twice in three launches, and this: 32x64x112x112 37.6 and
// 20.6 us (captured, with the clearing launch, 38.7 and 24.5), 144x51x53x53 30.3 and 18.9, 64x512x56x56 (411 MB, several rounds of
// workgroups) 138 and 72, 26x4x64x64 8.4 and 5.6, 256x3x120x120 19.1 and 12.9.
constexpr uint32_t kBnPerWave = 3;
constexpr uint32_t kBnHeld = kBnPerWave + 1;            // blocks per wave
constexpr uint32_t kBnMostGroups = 64;                  // one per lane

// How often a workgroup looks for the others' sums before it computes the missing ones.  A look takes 0.165 us, so it gives
// up after 17 us (a workgroup alone in its grid: 400 looks in each of two passes 131 us more than none).  No layer measured
// needs more than 30, neither on an idle card nor beside a 1 GiB copy on another stream; with 10, a large layer takes 1.5 times
// as long.  Giving up too early is the dearer mistake: a sum of 16 blocks takes 4.7 us from memory, and a workgroup of 64 that
// misses them all 300 us.  Beside a kernel that holds all but 128 / 64 / 32 CUs, reading x twice over this: 32x64x112x112 42.6 /
// 54 / 91 over 30 / 43 / 73 us, 144x51x53x53 40 / 57 / 94 over 33 / 54 / 88, but 256x3x120x120, which reads little and waits
// most, 24 / 24 / 24 over 21 / 27 / 40.
constexpr uint32_t kBnPolls = 100;

// A sum s under a tag: s, s ^ low half, s ^ high half.  Three words that were not all written together pass
// for a sum only where they hold the right one.
struct BnSum {
    uint32_t word[3];
};

__device__ __forceinline__ void bn_publish(BnSum* to, float sum, uint64_t tag, uint32_t h)
{
    const uint32_t key = h == 0 ? 0 : (uint32_t)(h == 1 ? tag : tag >> 32);
    if (h < 3) __hip_atomic_store(&to->word[h], __float_as_uint(sum) ^ key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Lane g of `sum`: what workgroup g has published at from[g]; lanes in `have` hold theirs already.  Returns the lanes
// whose sum has not come.
__device__ __forceinline__ unsigned long long bn_collect(BnSum* from, uint32_t groups, uint64_t tag, uint32_t polls,
                                                         uint32_t h, bool have, float& sum)
{
    bool wanted = h < groups && !have;
    for (uint32_t k = 0;; ++k) {
        if (wanted) {
            uint32_t v[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) v[i] = __hip_atomic_load(&from[h].word[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((v[0] ^ v[1]) == (uint32_t)tag && (v[0] ^ v[2]) == (uint32_t)(tag >> 32)) {
                sum = __uint_as_float(v[0]);
                wanted = false;
            }
        }
        const unsigned long long missing = __ballot(wanted);
        if (missing == 0 || k >= polls) return missing;
        __builtin_amdgcn_s_sleep(1);
    }
}

__global__ __launch_bounds__(kBlock) void k_bn_clear(uint32_t* __restrict__ words, uint32_t n)
{
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) words[i] = 0;
}

// The sums part[0 .. n-1] of one workgroup's blocks, as the tree over its 256 / groups lanes combines them
// (what further lanes and strides add is +0, and no sum is -0).
template <uint32_t WAVES>
__device__ __forceinline__ float bn_group_sum(const float* part, uint32_t n, uint32_t groups, uint32_t h)
{
    static_assert(WAVES * kBnHeld == 16 || WAVES * kBnHeld == 32, "the sums lie in one or two rows of lanes");
    const uint32_t lanes = 256 / groups;
    float r = 0.0f;
    if (h < lanes)
        for (uint32_t j = h; j < n; j += lanes) r = r + part[j];
    return lane0(WAVES * kBnHeld == 16 ? tree16(r) : tree32(r));
}

// The sums of the workgroups in `missing` from memory into other[]; every wave of the workgroup calls it.
template <bool SQDEV, int MODE, typename OFF, uint32_t WAVES>
__device__ __forceinline__ void bn_recompute(const float* __restrict__ x, const BnGeom& g, uint32_t ch, uint32_t groups,
                                             unsigned long long missing, float center, float* part, float* other,
                                             uint32_t w, uint32_t h)
{
    for (; missing != 0; missing &= missing - 1) {
        const uint32_t from = __builtin_ctzll(missing);
        const uint32_t n = (g.nblk - from + groups - 1) / groups;
        for (uint32_t j = w; j < n; j += WAVES) {
            f4 t[4][4];
            bn_load<MODE, OFF>(x, g, ch, from + j * groups, h, t);
            const float s = bn_block_sum<SQDEV>(t, from + j * groups, h, g.M, center);
            if (h == 0) part[j] = s;
        }
        __syncthreads();
        if (w == 0) {
            const float s = bn_group_sum<WAVES>(part, n, groups, h);
            if (h == 0) other[from] = s;
        }
        __syncthreads();
    }
}

template <int MODE, typename OFF, uint32_t WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_bn_shared(const float* __restrict__ x, ES_BN_GEOM_PARAMS, uint32_t groups, uint32_t polls, BnSum* __restrict__ sums,
                 uint64_t tag, float* __restrict__ mean, float* __restrict__ var)
{
    const BnGeom g = ES_BN_GEOM;
    const float fM = (float)M;
    extern __shared__ __align__(16) float park[];       // [wave][vector][lane], if any wave has a fourth block
    __shared__ float part[2][WAVES * kBnHeld];
    __shared__ float other[kBnMostGroups];
    __shared__ unsigned long long s_missing;
    const uint32_t h = threadIdx.x & 63;
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t ch = blockIdx.x / groups;
    const uint32_t grp = blockIdx.x % groups;
    const uint32_t n = (g.nblk - grp + groups - 1) / groups;
    auto block = [&](uint32_t j) { return grp + j * groups; };
    auto load = [&](uint32_t j, f4 (&r)[4][4]) {
        if (j < n) {
            bn_load<MODE, OFF>(x, g, ch, block(j), h, r);
        } else {                                        // not used, but no old value has to be kept for it either
#pragma unroll
            for (int i = 0; i < 16; ++i) r[i & 3][i >> 2] = f4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    };
    f4* mine = reinterpret_cast<f4*>(park) + w * 16 * 64 + h;
    BnSum* first = sums + (uint64_t)ch * 2 * groups;
    BnSum* second = first + groups;
    f4 t[kBnPerWave][4][4];
    const uint32_t parked = WAVES * kBnPerWave + w;
    constexpr uint32_t kLast = kBnPerWave - 1;
    // the parked block passes through the registers of the last one, behind the loads of the others
    if (parked < n) bn_load<MODE, OFF>(x, g, ch, block(parked), h, t[kLast]);
#pragma unroll
    for (uint32_t k = 0; k < kLast; ++k) {
        __builtin_amdgcn_sched_barrier(0);              // one block's addresses at a time
        load(WAVES * k + w, t[k]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (parked < n) {
#pragma unroll
        for (int i = 0; i < 16; ++i) mine[64 * i] = t[kLast][i & 3][i >> 2];
        const float s = bn_block_sum<false>(t[kLast], block(parked), h, g.M, 0.0f);
        if (h == 0) part[0][parked] = s;
    }
    __builtin_amdgcn_sched_barrier(0);
    load(WAVES * kLast + w, t[kLast]);
#pragma unroll
    for (uint32_t k = 0; k < kBnPerWave; ++k) {
        __builtin_amdgcn_sched_barrier(0);
        if (WAVES * k + w < n) {
            const float s = bn_block_sum<false>(t[k], block(WAVES * k + w), h, g.M, 0.0f);
            if (h == 0) part[0][WAVES * k + w] = s;
        }
    }
    __syncthreads();
    if (w == 0) {
        float sum = bn_group_sum<WAVES>(part[0], n, groups, h);
        bn_publish(first + grp, sum, tag, h);
        const unsigned long long missing = bn_collect(first, groups, tag, polls, h, h == grp, sum);
        if (h < groups) other[h] = sum;
        if (h == 0) s_missing = missing;
    }
    __syncthreads();
    unsigned long long missing = uniform64(s_missing);
    if (missing != 0) {                                 // at the cost of this workgroup's own blocks, which are read again
        bn_recompute<false, MODE, OFF, WAVES>(x, g, ch, groups, missing, 0.0f, part[0], other, w, h);
        uint32_t zero = 0;
        asm volatile("" : "+s"(zero));                  // no address is kept from above for this
#pragma unroll
        for (uint32_t k = 0; k < kBnPerWave; ++k) {
            __builtin_amdgcn_sched_barrier(0);
            load(WAVES * k + w + zero, t[k]);
        }
    }
    const float mu = lane0(tree64(h < groups ? other[h] : 0.0f)) / fM;
#pragma unroll
    for (uint32_t k = 0; k < kBnPerWave; ++k) {
        __builtin_amdgcn_sched_barrier(0);
        if (WAVES * k + w < n) {
            const float s = bn_block_sum<true>(t[k], block(WAVES * k + w), h, g.M, mu);
            if (h == 0) part[1][WAVES * k + w] = s;
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (parked < n) {                                   // what a lane parks only that lane reads back
#pragma unroll
        for (int i = 0; i < 16; ++i) t[0][i & 3][i >> 2] = mine[64 * i];
        const float s = bn_block_sum<true>(t[0], block(parked), h, g.M, mu);
        if (h == 0) part[1][parked] = s;
    }
    __syncthreads();
    if (grp != 0) {
        if (w == 0) bn_publish(second + grp, bn_group_sum<WAVES>(part[1], n, groups, h), tag, h);
        return;
    }
    if (w == 0) {
        float sum = bn_group_sum<WAVES>(part[1], n, groups, h);
        missing = bn_collect(second, groups, tag, polls, h, h == 0, sum);
        if (h < groups) other[h] = sum;
        if (h == 0) s_missing = missing;
    }
    __syncthreads();
    bn_recompute<true, MODE, OFF, WAVES>(x, g, ch, groups, uniform64(s_missing), mu, part[1], other, w, h);
    const float va = lane0(tree64(h < groups ? other[h] : 0.0f)) / fM;
    if (threadIdx.x == 0) {
        mean[ch] = mu;
        var[ch] = va;
    }
}

// The number of workgroups per channel: as few as hold it, more while they are all resident at once (eight waves on each
// of the 256 CUs; with fewer CUs to be had, some wait for the others in vain, see kBnPolls) and their sums fit the workspace of
// nblk floats per channel.
static uint32_t bn_groups(uint32_t C, uint32_t nblk, uint32_t waves)
{
    constexpr uint32_t floats = 2 * sizeof(BnSum) / sizeof(float);
    uint32_t n = 2;
    while (n * waves * kBnHeld < nblk) n *= 2;
    while (n < kBnMostGroups && 2ull * n * C <= 2048 / waves && 2 * n * floats <= nblk) n *= 2;
    return n;
}

// 64 bits that differ from launch to launch (the mixing steps are invertible), and from process to process.
static uint64_t bn_tag()
{
    static const uint64_t seed = [] {
        uint64_t s = 0;
        if (getentropy(&s, sizeof(s)) != 0) s = (uint64_t)std::chrono::steady_clock::now().time_since_epoch().count();
        return s;
    }();
    static std::atomic<uint64_t> launches{0};
    uint64_t z = seed + 0x9E3779B97F4A7C15ull * ++launches;
    z = (z ^ z >> 30) * 0xBF58476D1CE4E5B9ull;          // splitmix64
    z = (z ^ z >> 27) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z ? z : 1;                                   // a cleared workspace has no tag
}

// part: C * nblk floats, nblk >= 26; polls: see k_bn_shared
template <int MODE, typename OFF, uint32_t WAVES>
static hipError_t launch_bn_shared(hipStream_t s, const float* x, const BnGeom& g, float* mean, float* var, float* part, uint32_t polls,
                             bool captured)
{
    const uint32_t n = bn_groups(g.C, g.nblk, WAVES);
    BnSum* sums = reinterpret_cast<BnSum*>(part);
    if (captured) {
        const uint32_t clear = (uint32_t)(2ull * g.C * n * (sizeof(BnSum) / sizeof(uint32_t)));
        ES_RUN(k_bn_clear, dim3((clear + kBlock - 1) / kBlock), dim3(kBlock), 0, s, (uint32_t*)sums, clear);
    }
    const uint32_t most = (g.nblk + n - 1) / n;
    const uint32_t parked = most > WAVES * kBnPerWave ? most - WAVES * kBnPerWave : 0;
    ES_RUN((k_bn_shared<MODE, OFF, WAVES>), dim3(g.C * n), dim3(64 * WAVES), parked * 4096 * sizeof(float), s, x,
                       ES_BN_GEOM_ARGS(g), n, polls, sums, bn_tag(), mean, var);
    return hipSuccess;
}

// Longer channels, short images and little captured work read x twice (second pass over blocks in reverse:
// what the first read last may still be in the L2s).
//
// Up to 256 blocks, and few channels of tiny images from 8 on (WIDE): the four waves of a workgroup take the blocks b, b + W/4,
// b + W/2 and b + 3W/4, W being the number of blocks rounded up to a power of two, so the first
// two levels of the partials' tree (strides W/2 and W/4) happen in the workgroup: W/4 sums per
// channel are left, few enough for both passes' to fit in the workspace side by side and for one
// wave to add up.  Every wave of the second pass forms the mean for itself while its terms are on
// their way; three launches.  (A read that hits the Infinity Cache is no faster than one that does not.)
// Beyond that: one partial per block, and a launch after each pass that combines them.
template <bool SQDEV, bool WIDE, int MODE, typename OFF>
__device__ __forceinline__ void bn_partials(const float* __restrict__ x, const BnGeom& g, uint32_t groups, float fM,
                                            float* __restrict__ mean, float* __restrict__ part)
{
    const uint32_t h = threadIdx.x & 63;
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t bx = SQDEV ? groups - 1 - blockIdx.x : blockIdx.x;
    const uint32_t ch = SQDEV ? g.C - 1 - blockIdx.y : blockIdx.y;
    const uint32_t blk = WIDE ? bx + w * groups : bx * 4 + w;
    if (!WIDE && blk >= g.nblk) return;                 // whole wave leaves together
    f4 t[4][4];
    if (blk < g.nblk) bn_load<MODE, OFF>(x, g, ch, blk, h, t);
    __builtin_amdgcn_sched_barrier(0);
    float center = 0.0f;
    if constexpr (SQDEV) {
        if constexpr (WIDE) {
            center = lane0(tree64(h < groups ? part[(uint64_t)ch * groups + h] : 0.0f)) / fM;
            if (bx == 0 && threadIdx.x == 0) mean[ch] = center;
        } else {
            center = mean[ch];
        }
    }
    if constexpr (WIDE) {
        __shared__ float sums[4];
        const float r = blk < g.nblk ? bn_block_sum<SQDEV>(t, blk, h, g.M, center) : 0.0f;
        if (h == 0) sums[w] = r;
        __syncthreads();
        if (threadIdx.x == 0) {
            float* out = part + (SQDEV ? (uint64_t)g.C * groups : 0);
            out[(uint64_t)ch * groups + bx] = (sums[0] + sums[2]) + (sums[1] + sums[3]);
        }
    } else {
        const float r = bn_block_sum<SQDEV>(t, blk, h, g.M, center);
        if (h == 0) part[(uint64_t)ch * g.nblk + blk] = r;
    }
}

template <bool SQDEV, bool WIDE, int MODE, typename OFF>
__global__ __launch_bounds__(kBlock) void k_bn_partials(const float* __restrict__ x, ES_BN_GEOM_PARAMS, uint32_t groups,
                                                        float* __restrict__ mean, float* __restrict__ part)
{
    bn_partials<SQDEV, WIDE, MODE, OFF>(x, ES_BN_GEOM, groups, (float)M, mean, part);
}

// The same for images of up to kBnFetchedHW positions that are no vector, whose lines of memory are shared by many waves that
// run at about the same time, with its arguments in a structure: fetched by each wave, not in registers when it starts.  The
// wait costs a launch 0.15 us, but without it the layers take longer; the fetch is the only difference in the code, so it is
// when the waves reach their loads.  All launches of a layer, arguments in registers and so: 64 channels of 30 blocks of 1,
// 2, 3 positions 75.8 / 73.7, 63.2 / 59.9 and 67.6 / 66.5 us, 256 of them 430 / 396, 324 / 294 and 334 / 309, 256 of 64
// blocks 758 / 677, 672 / 572 and 587 / 536, of 64 blocks of 5 positions 275 / 266; 8 channels of 30 blocks 20.1 / 20.3.  7
// and 9 positions: 25.0 / 25.4 and 24.9 / 25.3 (64 channels of 30 blocks), 190.4 / 190.1 and 176.5 / 176.4 (256 of 64), so
// those have them in registers.
constexpr uint32_t kBnFetchedHW = 6;

template <bool SQDEV, bool WIDE, int MODE, typename OFF>
__global__ __launch_bounds__(kBlock) void k_bn_partials_fetched(const float* __restrict__ x, const BnGeom g, uint32_t groups,
                                                               float fM, float* __restrict__ mean, float* __restrict__ part)
{
    bn_partials<SQDEV, WIDE, MODE, OFF>(x, g, groups, fM, mean, part);
}

template <bool SQDEV, bool WIDE, int MODE, typename OFF>
static hipError_t launch_bn_partials(hipStream_t s, dim3 grid, const float* x, const BnGeom& g, float fM, float* mean, float* part)
{
    if constexpr (MODE == kBnWrap || MODE == kBnAny) {
        if (g.HW <= kBnFetchedHW) {
            ES_RUN((k_bn_partials_fetched<SQDEV, WIDE, MODE, OFF>), grid, dim3(kBlock), 0, s, x, g, grid.x, fM, mean, part);
            return hipSuccess;
        }
    }
    if constexpr (MODE != kBnAny)
        ES_RUN((k_bn_partials<SQDEV, WIDE, MODE, OFF>), grid, dim3(kBlock), 0, s, x, ES_BN_GEOM_ARGS(g), grid.x, mean, part);
    return hipSuccess;
}

// out[ch] = the tree over the last `n` <= 64 sums of channel ch / M; one wave per channel.
__global__ __launch_bounds__(kBlock) void k_bn_final_wave(const float* __restrict__ part, uint32_t n, uint32_t C,
                                                          float fM, float* __restrict__ out)
{
    const uint32_t h = threadIdx.x & 63;
    const uint32_t ch = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (ch >= C) return;
    const float r = tree64(h < n ? part[(uint64_t)ch * n + h] : 0.0f);
    if (h == 0) out[ch] = r / fM;
}

__global__ __launch_bounds__(kBlock) void k_bn_final(const float* __restrict__ part, uint32_t nblk, float fM,
                                                     float* __restrict__ out)
{
    __shared__ float lds[kBlock];
    const float* pc = part + (uint64_t)blockIdx.x * nblk;
    const float s = tree256(lane_partials(pc, nblk), lds);
    if (threadIdx.x == 0) out[blockIdx.x] = s / fM;
}

// Whether several workgroups share a channel (k_bn_shared).  Up to 25 blocks one workgroup is 1.2-1.5 times as fast.  Images
// of up to 127 positions that are no whole vectors keep the forms below because they were read in single loads when the line
// was drawn.  It has not been moved since they are read as vectors (from 10 positions on), though three launches and a shared
// channel now take, for 64 channels of 30 blocks of 17, 49 and 121 positions, 17.8 / 14.2, 15.5 / 12.4 and 14.9 / 10.9 us,
// for 16 of 300 blocks 66 / 21, 42 / 19 and 36 / 19, for 200 of 26 blocks 42 / 41, 33 / 27 and 33 / 23. Captured, with the
// clearing launch before it, little work takes longer so.  The line was drawn with workgroups of four waves (26 blocks: 4
// channels 7.2 in three launches and 10.4 us so, 20 channels 9.1 / 9.6, 40 11.9 / 10.7; 120 blocks: 8 channels 11.1 / 11.3,
// 10 12.3 / 12.2).  With those of eight, which work below it now has, the two meet earlier: 26 blocks: 3 channels 7.0 / 8.0,
// 19 8.5 / 8.1, 34 10.7 / 9.2; 64 blocks: 4 channels 7.3 / 8.3, 7 8.4 / 8.3, 14 10.2 / 9.5; 120 blocks: 4 channels 8.4 / 8.4,
// 8 10.3 / 9.9; 240 blocks: 4 channels 10.3 / 10.7, 5 11.6 / 10.8.  Enqueued, with no other launch than itself, it is ahead
// everywhere (1 to 8 channels of 26 to 1,000 blocks 1.2-1.5).
template <int MODE>
static bool bn_shares(const BnGeom& g, hipStream_t s, bool& captured)
{
    if ((MODE != kBnVector && MODE != kBnLong) || g.HW < 16) return false;
    if (g.nblk <= kBnWaves + kBnExtra || g.nblk > kBnMostGroups * 4 * kBnHeld) return false;
    captured = stream_captured(s);
    return !captured || (uint64_t)g.C * g.nblk >= (g.nblk <= 64 ? 1000 : 1300);
}

template <int MODE, typename OFF>
static hipError_t launch_bn(hipStream_t s, const float* x, const BnGeom& g, float* mean, float* var, float* part, uint32_t polls)
{
    const float fM = (float)g.M;
    // Few channels of many tiny images (a line of memory holds an image's few values of a channel, the rest belongs to
    // others): a channel's loads queue in the L1 of the one CU that has it, and most CUs have none.  Three launches spread a
    // channel over several workgroups instead.  16 blocks in one launch and in three: 16 channels of 1, 3, 5 and 7 positions
    // 59 / 31, 64 / 30, 36 / 16 and 27 / 16 us, 64 channels 72 / 44, 63 / 38, 33 / 19 and 24 / 16; 160 channels take one
    // launch.  Vectors of one image each (4 positions) need it least: 40 channels of 10, 12 and 16 blocks 16.0 / 13.3, 18.8 /
    // 13.5 and 24.3 / 15.9 us, 64 channels of 8, 10, 14 and 16 blocks 6.3 / 12.9, 7.6 / 15.9, 16.2 / 18.4 and 21.9 / 19.6, 96
    // channels of 10 and 25 blocks 14.9 / 23.0 and 35 / 37, 160 of 16 24.9 / 43.4. 8 to 15 positions, 16 and 64 channels: 10
    // blocks of 9 positions 12.4 / 11.6 and 16.1 / 13.6, of 15 6.7 / 10.0 and 12.5 / 12.4, 14 blocks of 9 18.4 / 14.1 and
    // 21.6 / 16.0, of 13 13.7 / 11.4 and 17.7 / 15.5, 25 of 11 27 / 11 and 33 / 19; 96 channels of 14 blocks of 9 and 13 26.3
    // / 26.0 and 17.9 / 23.8.  The line is theirs.  Whole vectors share it, though they change sides with the number of
    // channels: 16 blocks of 8 positions, 16, 32, 48 and 64 channels 6.5 / 11.9, 6.4 / 13.9, 15.2 / 13.2 and 13.5 / 17.1, of
    // 12 15.2 / 9.8, 11.4 / 11.0, 15.6 / 12.6 and 13.1 / 16.0; 25 blocks of 8 22 / 11, 21 / 13, 22 / 17 and 24 / 19, of 12 23
    // / 10, 17 / 11, 23 / 14 and 20 / 16.  From 16 positions on one launch is everywhere as fast as two per pass.
    const bool spread = g.HW == 4  ? (g.nblk > 14 ? g.C <= 64 : g.nblk > 9 && g.C <= 48)
                        : g.HW < 8 ? g.nblk >= 8 && g.C <= 128
                                   : g.HW < 16 && g.nblk > 12 && g.C <= 64;
    bool captured = false;
    hipError_t e;
    if (g.nblk == 1) {                                  // at most 65,535 x 4096 values: 32-bit offsets always
        ES_RUN((k_bn_channel<MODE, uint32_t, kBnSingle>), dim3((g.C + kBnSingles - 1) / kBnSingles),
                           dim3(64 * kBnSingles), 0, s, x, mean, var, ES_BN_GEOM_ARGS(g));
    } else if (g.nblk <= kBnWaves && !spread) {
        ES_RUN((k_bn_channel<MODE, OFF, kBnRegs>), dim3(g.C), dim3(64 * g.nblk), 0, s, x, mean, var, ES_BN_GEOM_ARGS(g));
    } else if (g.nblk <= kBnWaves + kBnExtra && !spread) {
        ES_RUN((k_bn_channel<MODE, OFF, kBnParked>), dim3(g.C), dim3(64 * kBnWaves),
                           (g.nblk - kBnWaves) * 4096 * sizeof(float), s, x, mean, var, ES_BN_GEOM_ARGS(g));
    } else if (bn_shares<MODE>(g, s, captured)) {
        if constexpr (MODE == kBnVector || MODE == kBnLong) {
            // Little work (25 MB; 32-bit offsets therefore): workgroups of eight waves, half as many sums to wait for.  26x4x64x64
            // 6.2 -> 5.6 us, 250x20x31x31 9.0 -> 7.9, 256x8x50x50 8.9 -> 8.2, 1x1x4190208 10.6 -> 9.6; beside a staging copy on another
            // stream 22.9 -> 21.2, 28.7 -> 27.4, 28.3 -> 25.6.  The line lies where that copy's waves begin to keep a CU from being
            // free for so large a workgroup: 1,664 blocks (26x64x64x64) 9.5 -> 9.1 us alone, but 25.3 -> 33.8 beside it, 5,100
            // (144x51x53x53) 19.1 -> 17.6 and 39 -> 47.  (In several rounds eight waves lose alone, too: 64x512x56x56 72 -> 79.)
            if constexpr (sizeof(OFF) == 4) {
                if ((uint64_t)g.C * g.nblk <= 1500)
                    return launch_bn_shared<MODE, OFF, 8>(s, x, g, mean, var, part, polls, captured);
            }
            return launch_bn_shared<MODE, OFF, 4>(s, x, g, mean, var, part, polls, captured);
        }
    } else if (g.nblk <= 256) {
        uint32_t n = 4;                                 // sums per channel: a quarter of the blocks' power of two
        while (4 * n < g.nblk) n *= 2;
        const dim3 grid(n, g.C);
        if ((e = launch_bn_partials<false, true, MODE, OFF>(s, grid, x, g, fM, mean, part)) != hipSuccess) return e;
        if ((e = launch_bn_partials<true, true, MODE, OFF>(s, grid, x, g, fM, mean, part)) != hipSuccess) return e;
        ES_RUN(k_bn_final_wave, dim3((g.C + 3) / 4), dim3(kBlock), 0, s, part + (uint64_t)g.C * n, n, g.C,
                           fM, var);
    } else {
        const dim3 grid((g.nblk + 3) / 4, g.C);
        if ((e = launch_bn_partials<false, false, MODE, OFF>(s, grid, x, g, fM, mean, part)) != hipSuccess) return e;
        ES_RUN(k_bn_final, dim3(g.C), dim3(kBlock), 0, s, part, g.nblk, fM, mean);
        if ((e = launch_bn_partials<true, false, MODE, OFF>(s, grid, x, g, fM, mean, part)) != hipSuccess) return e;
        ES_RUN(k_bn_final, dim3(g.C), dim3(kBlock), 0, s, part, g.nblk, fM, var);
    }
    return hipSuccess;
}

hipError_t launch_bn_batch_stats(hipStream_t s, const float* x, uint32_t B, uint32_t C, uint32_t HW,
                                 float* mean, float* var, float* part)
{
    return launch_bn_batch_stats_polls(s, x, B, C, HW, mean, var, part, kBnPolls);
}

hipError_t launch_bn_batch_stats_polls(hipStream_t s, const float* x, uint32_t B, uint32_t C, uint32_t HW,
                                       float* mean, float* var, float* part, uint32_t polls)
{
    if (C == 0) return hipSuccess;
    BnGeom g;
    g.C = C;
    g.HW = HW;
    g.M = B * HW;
    g.nblk = (g.M + 4095) / 4096;
    // 2^l >= HW: magic * HW exceeds 2^(31+l) by at most HW <= 2^l, which m < 2^31 cannot carry into the quotient
    uint32_t l = 0;
    while ((1ull << l) < HW) ++l;
    g.magic = (1ull << (31 + l)) / HW + 1;
    g.shift = 31 + l;
    g.step_img = 256 / HW;
    g.step_pos = 256 % HW;
    const bool small = (uint64_t)B * C * HW * sizeof(float) <= 0xFFFFFFFFull;
#define ES_BN(MODE)                                                              \
    do {                                                                         \
        if (small) return launch_bn<MODE, uint32_t>(s, x, g, mean, var, part, polls);   \
        return launch_bn<MODE, uint64_t>(s, x, g, mean, var, part, polls);              \
    } while (0)
    if (HW % 4 == 0) ES_BN(kBnVector);
    else if (HW >= (g.nblk > kBnWaves + kBnExtra ? kBnLongSharedHW : kBnLongHW)) ES_BN(kBnLong);
    else if (HW >= 4) ES_BN(kBnWrap);
    else ES_BN(kBnAny);
#undef ES_BN
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// What the runtime knows of a stream (StreamProbe).
// ---------------------------------------------------------------------------
namespace {

// A query is not allowed while another thread captures in the global mode, unless this thread says that it does not mind.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    bool set = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    ~RelaxedCapture()
    {
        if (set) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
};

bool answered_yes(hipError_t e)
{
    // "Not ready" is no error to the runtime: it leaves the thread's last one as it is, which may be another library's.
    if (e != hipSuccess && e != hipErrorNotReady) (void)hipGetLastError();
    return e == hipSuccess;
}

// Only of streams that are not ordered with the null stream: an idle one of the others may still have to wait for it.
bool stream_idle(hipStream_t s)
{
    unsigned flags = 0;
    if (reinterpret_cast<uintptr_t>(s) <= 2) return false;                    // the null stream and the named ones
    if (!answered_yes(hipStreamGetFlags(s, &flags)) || !(flags & hipStreamNonBlocking) || stream_captured(s)) return false;
    RelaxedCapture relaxed;
    return relaxed.set && answered_yes(hipStreamQuery(s));
}

bool event_done(hipEvent_t e)
{
    RelaxedCapture relaxed;
    return relaxed.set && answered_yes(hipEventQuery(e));
}

const bool g_probe_set = (stream_probe = StreamProbe{stream_idle, event_done}, true);

}  // namespace

}  // namespace es
