// HIP kernels of the SparkCL map -> reduce hot path, written for gfx950.
//
// A partition task (a MapCL / MapCLPartition / ReduceCL application, paper
// sec. 3.1.3) is cut into tiles of `tile_elems` elements.  One 256-thread
// block turns one tile into one partial:
//   1. streaming loop: coalesced 128-bit loads (float4), U quads per input
//      in flight per thread (2, 4 or 8, from the tuning table), the registry kernel's map applied per
//      element, each value added to a per-thread FP64 sum, a running max, or
//      a hit counter;
//   2. the per-thread values are combined across the wave with cross-lane
//      shuffles and across the block's waves through LDS in a fixed tree;
//   3. the partial is published and an arrival ticket taken; the block that
//      takes the last ticket combines the task's partials in FP64 in a fixed
//      order and writes the partition result (the tree-reduce of ReduceCL,
//      sec. 3.1.3 and 3.2.2); a task of one tile is finished by its block
//      directly.  The block that finishes the last task of a launch folds
//      the partition results into the RDD-level total.
// Tiles of at least one chunk (B threads x U quads, B the block size and U
// the quads each thread has in flight per input) deal a task's chunks
// round-robin to its tiles, so the tiles that run together read one sliding
// window of the task; smaller tiles are contiguous ranges.  Every element's
// owner thread and every combine order depend only on the tile size, the
// block size, U and x's 16-byte alignment, so results are identical run to
// run and across execution modes with the same tiles, block size and U.
//
// Compiled with -ffp-contract=off: the maps are the binary32 definition
// operation by operation.  No MFMA: nothing on this path is a contraction.

#include <hip/hip_runtime.h>

#include <cstddef>

#include "launches.h"
#include "philox_dev.h"
#include "sparkcl_dev.h"

namespace sparkcl {

namespace {

constexpr float kNegInf = -__builtin_huge_valf();

__device__ __forceinline__ uint32_t uni(uint32_t v)
{
    return __builtin_amdgcn_readfirstlane(v);
}

__device__ __forceinline__ uint64_t uni64(uint64_t v)
{
    uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// ---- agent-scope atomics used by the last-block combine -----------------
__device__ __forceinline__ void st_agent(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_agent(const uint64_t *p)
{
    return __hip_atomic_load(const_cast<uint64_t *>(p), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void store_partial(Partial *p, double s, float m,
                                              uint64_t h, uint64_t n)
{
    uint64_t *w = reinterpret_cast<uint64_t *>(p);
    st_agent(w + 0, __double_as_longlong(s));
    st_agent(w + 1, (uint64_t)__float_as_uint(m));
    st_agent(w + 2, h);
    st_agent(w + 3, n);
}

__device__ __forceinline__ void load_partial(const Partial *p, double &s,
                                             float &m, uint64_t &h, uint64_t &n)
{
    const uint64_t *w = reinterpret_cast<const uint64_t *>(p);
    s = __longlong_as_double(ld_agent(w + 0));
    m = __uint_as_float((uint32_t)ld_agent(w + 1));
    h = ld_agent(w + 2);
    n = ld_agent(w + 3);
}

__device__ __forceinline__ uint64_t device_ns(uint32_t ns_per_tick)
{
    return (uint64_t)wall_clock64() * ns_per_tick;
}

// ---- streaming loads and stores -------------------------------------------
// The task's arrays arrive as generic pointers read from the task table; the
// casts below tell the compiler they are global memory, so it emits
// global_load/global_store instead of flat ones (flat accesses also count
// against the LDS/scalar counter and stall behind unrelated waits).  Every
// element is touched once, so the loads and stores are nontemporal.
typedef float f4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const f4v gf4;
typedef __attribute__((address_space(1))) f4v gf4w;
typedef __attribute__((address_space(1))) const float gf1;
typedef __attribute__((address_space(1))) float gf1w;

__device__ __forceinline__ float4 ld4(const float *p)
{
    const f4v v = __builtin_nontemporal_load((gf4 *)p);
    return make_float4(v.x, v.y, v.z, v.w);
}
// y and out need only 4-byte alignment: a 16-byte access at a 4-byte-aligned
// address is still one dwordx4 instruction (the memory pipeline splits it
// over the two 16-byte segments it touches), so arrays whose misalignments
// differ from x's stream as quads too.
typedef float f4a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef __attribute__((address_space(1))) const f4a4 gf4u;
typedef __attribute__((address_space(1))) f4a4 gf4uw;
__device__ __forceinline__ float4 ld4u(const float *p)
{
    const f4a4 v = __builtin_nontemporal_load((gf4u *)p);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st4u(float *p, const float4 &v)
{
    const f4a4 w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, (gf4uw *)p);
}
__device__ __forceinline__ float ld1(const float *p)
{
    return __builtin_nontemporal_load((gf1 *)p);
}
__device__ __forceinline__ void st4(float *p, const float4 &v)
{
    const f4v w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, (gf4w *)p);
}
__device__ __forceinline__ void st1(float *p, float v)
{
    __builtin_nontemporal_store(v, (gf1w *)p);
}

// Publication order without cache maintenance: the partials and results are
// written with agent-scope atomic stores, which write through the per-XCD L2
// to the device coherence point, and read back with agent-scope atomic loads,
// which bypass it.  Waiting for this thread's stores to complete before the
// arrival ticket is taken therefore makes them visible to the block that
// takes the last ticket, without the L2 write-back of a release fence (which
// costs half the streaming bandwidth when paid once per tile).
__device__ __forceinline__ void own_stores_complete()
{
    __builtin_amdgcn_s_waitcnt(0);
}

// ---- registry maps (one binary32 operation per step, in order) -----------
template <int D> struct PolyMap {
    static constexpr bool kTwo = false;
    static constexpr bool kGroup = false;
    float k[8];
    __device__ __forceinline__ float operator()(float x, float) const
    {
        float t = k[D];
#pragma unroll
        for (int i = D - 1; i >= 0; --i) {
            float p = t * x;
            t = p + k[i];
        }
        return t;
    }
};

struct FmulMap {
    static constexpr bool kTwo = true;
    static constexpr bool kGroup = false;
    float c;
    __device__ __forceinline__ float operator()(float x, float y) const
    {
        float xy = x * y;
        float cx = c * x;
        return xy + cx;
    }
};

// Per-thread accumulator of one tile.  The sum is carried in FP64: on
// gfx950 a vector FP64 add issues at the full 32-bit rate, so converting and
// adding (two instructions) is cheaper than binary32 Neumaier compensation
// (seven), and a recursive FP64 sum of m terms is within (m-1) 2^-53 of the
// sum of magnitudes -- far inside the binary32 result's own resolution.
struct Acc {
    double s = 0.0;
    float m = kNegInf;
    uint32_t hits = 0;
    __device__ __forceinline__ void add(float v)
    {
        s += (double)v;
        m = fmaxf(m, v);
    }
};

// ---- elementwise tiles ------------------------------------------------------
// One quad of the map: four results, optionally stored, folded into the
// thread's accumulator in element order.
template <class M, bool W>
__device__ __forceinline__ void map_quad(const M &f, const float4 &xv,
                                         const float4 &yv, float *o, Acc &a)
{
    float4 v;
    v.x = f(xv.x, yv.x);
    v.y = f(xv.y, yv.y);
    v.z = f(xv.z, yv.z);
    v.w = f(xv.w, yv.w);
    if (W)
        st4u(o, v);
    a.add(v.x);
    a.add(v.y);
    a.add(v.z);
    a.add(v.w);
}

// Stream `ng` groups of the calling thread.  Group g is the U quads
// base(g) + u * B (u = 0..U-1, B the block size), in quads from x4/y4/o4: all the
// group's loads are issued, then the group is folded in order.  (Measured on
// MI355X: keeping a second group in flight while folding -- a register double
// buffer -- streams slower than this at every tile size and occupancy; the
// extra requests in flight cost more at the HBM than the overlap gains.)
//
// A map with run-time steps (kGroup: a fused chain) maps the whole group at
// once, so each step's uniform test and coefficient is paid once per group
// of 4 U elements per thread rather than once per element.
template <class M, bool W, int U, class Base>
__device__ __forceinline__ void stream_groups(const M &f, const float *x4,
                                              const float *y4, float *o4,
                                              uint64_t ng, Base base, Acc &a)
{
    const uint32_t B = blockDim.x;
    constexpr int NY = M::kTwo ? U : 1; // one-input maps carry no y buffer
    for (uint64_t g = 0; g < ng; ++g) {
        const uint64_t q0 = base(g);
        float4 xv[U], yv[NY];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            xv[u] = ld4(x4 + 4 * (q0 + u * B));
            if (M::kTwo)
                yv[u] = ld4u(y4 + 4 * (q0 + u * B));
        }
        if constexpr (M::kGroup) {
            float v[4 * U];
            f.template group<U>(xv, M::kTwo ? yv : xv, v);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (W)
                    st4u(o4 + 4 * (q0 + u * B),
                         make_float4(v[4 * u], v[4 * u + 1], v[4 * u + 2], v[4 * u + 3]));
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    a.add(v[4 * u + e]);
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
                map_quad<M, W>(f, xv[u], M::kTwo ? yv[u] : xv[u],
                               W ? o4 + 4 * (q0 + u * B) : nullptr, a);
        }
    }
}

// Scalar elements [i0, i1) of an elementwise task, strided over the block.
template <class M, bool W>
__device__ __forceinline__ void map_scalar(const M &f, const float *x,
                                           const float *y, float *out,
                                           uint64_t i0, uint64_t i1, Acc &a)
{
    for (uint64_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
        float v = f(ld1(x + i), M::kTwo ? ld1(y + i) : 0.0f);
        if (W)
            st1(out + i, v);
        a.add(v);
    }
}

// The scalar head of a task's range: the elements before x reaches a 16-byte
// boundary.  The quads after it are aligned for x; y and out, at any 4-byte
// alignment, are read and written with the same quad indices.
__device__ __forceinline__ uint32_t quad_head(const float *x, uint64_t n)
{
    const uint32_t mis = (uint32_t)(((uintptr_t)x & 15u) >> 2);
    return (uint32_t)min((uint64_t)((4u - mis) & 3u), n);
}

// Contiguous tile [begin, end): the middle in float4 quads (thread t owns
// quads t, t+B, t+2B, ...), the head before x's first 16-byte boundary and
// the ragged tail as single elements owned by threads 0..2.
template <class M, bool W, int U>
__device__ __forceinline__ void tile_contiguous(const M &f,
                                                const float *__restrict__ x,
                                                const float *__restrict__ y,
                                                float *__restrict__ out,
                                                uint64_t begin, uint64_t end,
                                                Acc &a)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t len = (uint32_t)(end - begin);
    const float *xb = x + begin;
    const float *yb = M::kTwo ? y + begin : nullptr;
    float *ob = W ? out + begin : nullptr;
    const uint32_t head = quad_head(xb, len);
    map_scalar<M, W>(f, xb, yb, ob, 0, head, a);

    const uint32_t B = blockDim.x;
    const uint32_t kStep = U * B;
    const uint32_t nq = (len - head) >> 2;
    const float *x4 = xb + head;
    const float *y4 = M::kTwo ? yb + head : nullptr;
    float *o4 = W ? ob + head : nullptr;
    // full groups of U quads owned by this thread
    const uint32_t full = (tid + (U - 1) * B < nq)
                              ? (nq - tid - (U - 1) * B + kStep - 1) / kStep
                              : 0u;
    stream_groups<M, W, U>(f, x4, y4, o4, full,
                           [&](uint64_t g) { return (uint64_t)tid + g * kStep; }, a);
    for (uint32_t q = tid + full * kStep; q < nq; q += B)
        map_quad<M, W>(f, ld4(x4 + 4u * q), M::kTwo ? ld4u(y4 + 4u * q) : float4{},
                       W ? o4 + 4u * q : nullptr, a);
    map_scalar<M, W>(f, xb, yb, ob, head + 4u * nq, len, a);
}

// Interleaved layout of a whole task (tiles of at least one chunk, 4 U B
// elements): the task's quad-aligned
// middle is cut into chunks of U * B quads, and tile j of nt owns
// chunks j, j + nt, j + 2 nt, ...; tile 0 also owns the unaligned head and
// the ragged tail.  Tiles that run at the same time (the queue hands out a
// task's tiles in order) then read neighbouring chunks, one sliding window
// per task instead of one stream per tile, which HBM serves at a higher rate.
// Returns the number of elements the tile covers.
template <class M, bool W, int U>
__device__ __forceinline__ uint64_t tile_interleaved(const M &f,
                                                     const float *__restrict__ x,
                                                     const float *__restrict__ y,
                                                     float *__restrict__ out,
                                                     uint64_t n, uint32_t head,
                                                     uint32_t nt, uint32_t j,
                                                     Acc &a)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t B = blockDim.x;
    const uint32_t kChunkQuads = U * B;
    const uint64_t nq = (n - head) >> 2;
    const uint64_t nfull = nq / kChunkQuads;
    const uint32_t rem = (uint32_t)(nq % kChunkQuads);
    const float *x4 = x + head;
    const float *y4 = M::kTwo ? y + head : nullptr;
    float *o4 = W ? out + head : nullptr;
    const uint64_t ng = nfull > j ? (nfull - j + nt - 1) / nt : 0;
    stream_groups<M, W, U>(f, x4, y4, o4, ng,
                           [&](uint64_t g) { return (j + g * nt) * kChunkQuads + tid; }, a);
    uint64_t count = 4 * ng * kChunkQuads;
    if (rem != 0 && nfull % nt == j) {
        const uint64_t q0 = nfull * kChunkQuads;
        for (uint32_t q = tid; q < rem; q += B)
            map_quad<M, W>(f, ld4(x4 + 4 * (q0 + q)),
                           M::kTwo ? ld4u(y4 + 4 * (q0 + q)) : float4{},
                           W ? o4 + 4 * (q0 + q) : nullptr, a);
        count += 4 * rem;
    }
    if (j == 0) {
        map_scalar<M, W>(f, x, y, out, 0, head, a);
        map_scalar<M, W>(f, x, y, out, head + 4 * nq, n, a);
        count += n - 4 * nq;
    }
    return count;
}

// Tile j of an elementwise task: interleaved when the tile size allows,
// else the contiguous range [jT, jT + T).  Returns the number of elements
// covered.
template <class M, bool W, int U>
__device__ __forceinline__ uint64_t tile_map(const M &f, const float *x,
                                             const float *y, float *out,
                                             uint64_t n, uint32_t T, uint32_t nt,
                                             uint32_t j, Acc &a)
{
    if (T >= 4u * U * blockDim.x)
        return tile_interleaved<M, W, U>(f, x, y, out, n, quad_head(x, n), nt, j, a);
    const uint64_t begin = (uint64_t)j * T;
    const uint64_t end = min(n, begin + T);
    if (begin < end)
        tile_contiguous<M, W, U>(f, x, y, out, begin, end, a);
    return begin < end ? end - begin : 0;
}

// MapCLPartition Monte-Carlo tile: samples [begin, end), begin even.  Pair p
// is the Philox block with counter (p lo, p hi, partition id, 0); sample 2p
// takes words (0, 1), sample 2p+1 words (2, 3).
__device__ __forceinline__ void tile_mc(uint64_t seed, uint32_t pid,
                                        uint64_t begin, uint64_t end, Acc &a)
{
    const uint64_t p0 = begin >> 1;
    const uint32_t npairs = (uint32_t)(((end + 1) >> 1) - p0);
    const bool odd_tail = (end & 1u) != 0;
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    uint32_t hits = 0;
    for (uint32_t i = threadIdx.x; i < npairs; i += blockDim.x) {
        const uint64_t p = p0 + i;
        const U4 r = philox10(U4{(uint32_t)p, (uint32_t)(p >> 32), pid, 0u}, k0, k1);
        const uint32_t second = (odd_tail && i == npairs - 1) ? 0u : 1u;
        hits += disc_hit(r.x, r.y) + (disc_hit(r.z, r.w) & second);
    }
    a.hits += hits;
}

// The same tile for the Monte-Carlo-only executor, which is bound by VALU
// issue: the counter's high word is the same for a whole tile (tiles are
// powers of two, at most 2^22 samples, and start at multiples of their
// size), so the rounds it makes uniform run once per tile, and the wave counts
// its misses in scalar registers (wave_misses).  (Mixed batches keep the body
// above: there the loop runs beside streaming tiles, which bound the time.)
// Measured on MI355X, 256 partitions of 2^24 samples: 2440 us, 43 vector
// instructions per pair of samples at 0.99 per CU and clock, against 2975 us
// and 57 with the body above (2600 us and 47 with the words masked first).
__device__ __forceinline__ void tile_mc_uniform(uint64_t seed, uint32_t pid, uint64_t begin,
                                                uint64_t end, Acc &a)
{
    const uint64_t p0 = begin >> 1;
    const uint32_t npairs = (uint32_t)(((end + 1) >> 1) - p0);
    const PhiloxTile ph((uint32_t)(p0 >> 32), pid, (uint32_t)seed, (uint32_t)(seed >> 32));
    const uint32_t B = blockDim.x;
    // whole iterations of the block, every lane active
    const uint32_t iters = (npairs - (uint32_t)(end & 1u)) / (kMcPairs * B);
    uint32_t lo = (uint32_t)p0 + threadIdx.x;
    uint32_t misses = 0;
    for (uint32_t it = 0; it < iters; ++it) {
        misses += wave_misses(ph, lo, B);
        lo += kMcPairs * B;
    }
    if ((threadIdx.x & 63u) == 0)
        a.hits += 64u * 2u * kMcPairs * iters - misses;
    // the rest, pair by pair; the last sample of an odd count has no second
    const bool odd_tail = (end & 1u) != 0;
    for (uint32_t i = iters * kMcPairs * B + threadIdx.x; i < npairs; i += B) {
        const U4 r = ph.block((uint32_t)p0 + i);
        const uint32_t second = (odd_tail && i == npairs - 1) ? 0u : 1u;
        a.hits += disc_hit(r.x, r.y) + (disc_hit(r.z, r.w) & second);
    }
}

// ---- wave and block combines --------------------------------------------
struct Red {
    double s;
    float m;
    uint64_t h, n;
};

__device__ __forceinline__ void wave_reduce(Red &r)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        r.s += __shfl_xor(r.s, o);
        r.m = fmaxf(r.m, __shfl_xor(r.m, o));
        r.h += __shfl_xor(r.h, o);
        r.n += __shfl_xor(r.n, o);
    }
}

// Block-wide combine; the result is valid in thread 0.  Waves are combined
// as a fixed pairwise tree ((w0 + w1) + (w2 + w3)) + ... over the block's
// B / 64 waves (4, 8 or 16).
__device__ __forceinline__ Red block_reduce(Red r)
{
    __shared__ double sh_s[kMaxWaves];
    __shared__ float sh_m[kMaxWaves];
    __shared__ uint64_t sh_h[kMaxWaves], sh_n[kMaxWaves];
    const uint32_t nw = blockDim.x >> 6;
    wave_reduce(r);
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    if (lane == 0) {
        sh_s[w] = r.s;
        sh_m[w] = r.m;
        sh_h[w] = r.h;
        sh_n[w] = r.n;
    }
    __syncthreads();
    Red out = r;
    if (threadIdx.x == 0) {
        // in place in LDS (thread 0 alone): the pairwise tree over nw waves
        for (uint32_t step = 1; step < nw; step <<= 1)
            for (uint32_t i = 0; i + step < nw; i += 2 * step) {
                sh_s[i] = sh_s[i] + sh_s[i + step];
                sh_m[i] = fmaxf(sh_m[i], sh_m[i + step]);
                sh_h[i] += sh_h[i + step];
                sh_n[i] += sh_n[i + step];
            }
        out = Red{sh_s[0], sh_m[0], sh_h[0], sh_n[0]};
    }
    __syncthreads();
    return out;
}

// Fold the strided slice of `count` partials owned by this thread (in index
// order), then combine across the block.  Thread 0 holds the result.
template <class Load>
__device__ __forceinline__ Red combine_ordered(uint32_t count, Load load)
{
    Red r{0.0, kNegInf, 0, 0};
    for (uint32_t k = threadIdx.x; k < count; k += blockDim.x) {
        double s;
        float m;
        uint64_t h, n;
        load(k, s, m, h, n);
        r.s += s;
        r.m = fmaxf(r.m, m);
        r.h += h;
        r.n += n;
    }
    return block_reduce(r);
}

__device__ __forceinline__ void write_result(sparkcl_result *dst, uint32_t ops,
                                             const Red &r, uint64_t t_start,
                                             uint64_t t_done, int32_t status = SPARKCL_OK)
{
    sparkcl_result v;
    v.sum = (ops & SPARKCL_SUM) ? r.s : 0.0;
    v.max = (ops & SPARKCL_MAX) ? r.m : kNegInf;
    v.status = status;
    v.count = (ops & SPARKCL_COUNT) ? r.h : 0;
    v.n = r.n;
    v.t_arrive_ns = 0;
    v.t_admit_ns = 0;
    v.t_start_ns = t_start;
    v.t_done_ns = t_done;
    const uint64_t *src = reinterpret_cast<const uint64_t *>(&v);
    uint64_t *d = reinterpret_cast<uint64_t *>(dst);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(v) / 8); ++i)
        st_agent(d + i, src[i]);
}

__device__ __forceinline__ void read_result(const sparkcl_result *p, double &s,
                                            float &m, uint64_t &h, uint64_t &n)
{
    const uint64_t *w = reinterpret_cast<const uint64_t *>(p);
    s = __longlong_as_double(ld_agent(w + 0));
    m = __uint_as_float((uint32_t)ld_agent(w + 1));
    h = ld_agent(w + 2);
    n = ld_agent(w + 3);
}

// ---- one tile, start to finish ------------------------------------------
// Thread 0 of the block that completes a task: write its result and, when
// serving, publish the completion word.  With `wait` false the result stores
// are left to complete while the block goes on: the persistent executor waits
// for all of a block's stores once, before the block counts itself out, and
// only then is any result read on the device (the RDD total).
__device__ __forceinline__ void finish_task(const TaskDev *__restrict__ tp, const LaunchOut &L,
                                            const Red &t, uint64_t t_start, uint32_t variant,
                                            uint32_t idx, bool wait = true)
{
    write_result(L.results + idx, uni(tp->ops), t, t_start, device_ns(L.ns_per_tick),
                 variant == V_DECLINED ? SPARKCL_EDECLINED : SPARKCL_OK);
    if (L.done) {
        // Serving: the result lives in host memory; publish it with a
        // system-scope release so the host sees the result before the word.
        __threadfence_system();
        __hip_atomic_store(L.done + idx, uni64(tp->seq) + 1, __ATOMIC_RELEASE,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    } else if (wait) {
        own_stores_complete();
    }
}

// Returns true in the block that completed the task (after writing its
// result); callers use it only for the RDD-level step.  kExec: called by the
// persistent executor, which waits for the result stores at its exit.
template <bool kExec = false, class Body>
__device__ __forceinline__ bool run_tile_with(const TaskDev *__restrict__ tp, uint32_t j,
                                              const LaunchOut &L, Body body)
{
    __shared__ uint32_t sh_last;
    TaskSync *__restrict__ sync = L.sync;
    const uint64_t t0 = device_ns(L.ns_per_tick);

    const uint32_t variant = uni(tp->variant);
    const uint32_t ntiles = uni(tp->ntiles);

    Acc a;
    const uint64_t count = body(a);

    Red r{a.s, a.m, a.hits, 0};
    r = block_reduce(r);

    const uint32_t idx = uni(tp->index);
    if (ntiles == 1) {
        // A task of one tile: its block finishes the task by construction,
        // so the partial, the start-time word and the arrival ticket (three
        // round trips to memory-side atomics) are skipped.  The ordered
        // combine of a single partial is the partial itself, except that its
        // FP64 sum starts from +0.0, which the + 0.0 below reproduces.
        if (threadIdx.x == 0)
            finish_task(tp, L, Red{r.s + 0.0, r.m, r.h, count}, t0, variant, idx, !kExec);
        __syncthreads();
        return true;
    }
    if (threadIdx.x == 0) {
        store_partial(tp->partials + j, r.s, r.m, r.h, count);
        // t_start keeps the bitwise complement of the earliest tile start, so
        // its cleared state (0) is the identity of the max below.
        __hip_atomic_fetch_max(&sync[idx].t_start, ~t0, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        own_stores_complete();
        const uint32_t prev = __hip_atomic_fetch_add(&sync[idx].ticket, 1u, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
        sh_last = (prev == ntiles - 1) ? 1u : 0u;
    }
    __syncthreads();
    // Every branch that guards a barrier must be provably uniform (a scalar
    // value): a condition read from LDS looks divergent to the compiler, and
    // its control-flow structurizer may then send some threads around a loop
    // latch without the others.
    const bool last = uni(sh_last) != 0;
    __syncthreads();
    if (!last)
        return false;

    // Last tile of the task: combine its partials in index order (agent-scope
    // atomic loads, issued only after the last ticket was observed).
    const Partial *parts = tp->partials;
    Red t = combine_ordered(ntiles, [&](uint32_t k, double &s, float &m,
                                        uint64_t &h, uint64_t &nn) {
        load_partial(parts + k, s, m, h, nn);
    });
    if (threadIdx.x == 0) {
        const uint64_t t_start = ~ld_agent(&sync[idx].t_start);
        __hip_atomic_store(&sync[idx].t_start, 0ull, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&sync[idx].ticket, 0u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        finish_task(tp, L, t, t_start, variant, idx, !kExec);
    }
    // A barrier closes every thread-0 region that ends a loop iteration of the
    // callers: without it the compiler may sink the region past the loop
    // latch and let the other threads start the next iteration early.
    __syncthreads();
    return true;
}

// The registry kernels' tile body (maps fused with their reductions, or the
// Monte-Carlo count) run through the common tile epilogue.
template <bool kExec = false>
__device__ __forceinline__ bool run_tile(const TaskDev *__restrict__ tp, uint32_t j,
                                         const LaunchOut &L)
{
    return run_tile_with<kExec>(tp, j, L, [&](Acc &a) -> uint64_t {
        const uint32_t variant = uni(tp->variant);
        const uint32_t T = uni(tp->tile_elems);
        const uint32_t ntiles = uni(tp->ntiles);
        const uint64_t n = uni64(tp->n);
        uint64_t count = 0;
        const float *x = tp->in0;
        const float *y = tp->in1;
        float *o = tp->out;
        const uint32_t U = uni(tp->unroll);
        // the tile loop for map f with U quads in flight per thread
#define SPARKCL_TILE_U(MAP, WR, f)                                             \
    (U == 2   ? tile_map<MAP, WR, 2>(f, x, y, o, n, T, ntiles, j, a)               \
     : U == 8 ? tile_map<MAP, WR, 8>(f, x, y, o, n, T, ntiles, j, a)               \
              : tile_map<MAP, WR, 4>(f, x, y, o, n, T, ntiles, j, a))
        if (variant < V_FMUL) {
            const bool w = variant >= V_POLYW;
            const uint32_t d = variant & 7u;
            float k[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                k[i] = tp->coef[i];
#define SPARKCL_POLY_CASE(D)                                                   \
        case D: {                                                                  \
            PolyMap<D> f;                                                          \
            for (int i = 0; i < 8; ++i)                                            \
                f.k[i] = k[i];                                                     \
            count = w ? SPARKCL_TILE_U(PolyMap<D>, true, f)                        \
                      : SPARKCL_TILE_U(PolyMap<D>, false, f);                      \
        } break;
            switch (d) {
                SPARKCL_POLY_CASE(0)
                SPARKCL_POLY_CASE(1)
                SPARKCL_POLY_CASE(2)
                SPARKCL_POLY_CASE(3)
                SPARKCL_POLY_CASE(4)
                SPARKCL_POLY_CASE(5)
                SPARKCL_POLY_CASE(6)
                SPARKCL_POLY_CASE(7)
            }
#undef SPARKCL_POLY_CASE
        } else if (variant == V_FMUL || variant == V_FMULW) {
            FmulMap f{tp->c};
            count = variant == V_FMULW ? SPARKCL_TILE_U(FmulMap, true, f)
                                       : SPARKCL_TILE_U(FmulMap, false, f);
        } else if (variant == V_MC) {
            const uint64_t begin = (uint64_t)j * T;
            const uint64_t end = min(n, begin + T);
            if (begin < end) {
                tile_mc(uni64(tp->seed), uni(tp->pid), begin, end, a);
                count = end - begin;
            }
        } // V_DECLINED: nothing to do; the empty partial leaves the total as is
#undef SPARKCL_TILE_U
        return count;
    });
}

// The RDD-level total: all partition results folded in task order (run by
// one block once every task of the launch has its result).
__device__ __forceinline__ void rdd_total(const LaunchOut &L)
{
    const sparkcl_result *res = L.results;
    Red t = combine_ordered(L.ntasks, [&](uint32_t k, double &s, float &m,
                                          uint64_t &h, uint64_t &n) {
        read_result(res + k, s, m, h, n);
    });
    if (threadIdx.x == 0 && L.total) {
        write_result(L.total, SPARKCL_SUM | SPARKCL_MAX | SPARKCL_COUNT, t, 0,
                     device_ns(L.ns_per_tick));
        own_stores_complete();
    }
    __syncthreads();
    if (L.host) {
        // A blocking call: its results go to the host from here, 64 bytes a
        // task over the link, instead of by a copy after the launch, which
        // waited for it, took as long again and was waited for (one task of
        // 1000 elements, whole call: 29.1 us with the copy, 22.6 without).
        constexpr uint32_t kWords = sizeof(sparkcl_result) / 8;
        uint64_t *to = reinterpret_cast<uint64_t *>(L.host);
        const uint64_t *res = reinterpret_cast<const uint64_t *>(L.results);
        const uint64_t *tot = reinterpret_cast<const uint64_t *>(L.total);
        const uint32_t n = L.ntasks * kWords;
        for (uint32_t i = threadIdx.x; i < n + kWords; i += blockDim.x)
            __hip_atomic_store(to + i, ld_agent(i < n ? res + i : tot + (i - n)),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        own_stores_complete();
        __syncthreads();
    }
}

// RDD-level step of the per-partition launches, run by the block that
// completed a task: the block that completes the last task of the sequence
// folds all partition results.
__device__ __forceinline__ void rdd_step(const LaunchOut &L)
{
    __shared__ uint32_t sh_last;
    if (L.ntasks == 0)
        return;
    if (threadIdx.x == 0) {
        const uint32_t prev = __hip_atomic_fetch_add(&L.ctl->rdd_ticket, 1u, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
        sh_last = (prev == L.ntasks - 1) ? 1u : 0u;
    }
    __syncthreads();
    const bool last = uni(sh_last) != 0;
    __syncthreads();
    if (!last)
        return;
    rdd_total(L);
    if (threadIdx.x == 0) {
        __hip_atomic_store(&L.ctl->rdd_ticket, 0u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        own_stores_complete();
    }
    __syncthreads();
}

// ---- fused map chains ------------------------------------------------------
// A task's registry map followed by up to kMaxPost POLY stages on the running
// binary32 value (map -> map -> ... -> reduce in one pass).  Every Horner step
// is one binary32 multiply and one add in the written order.  Degrees are
// run-time values: a stage's eight coefficients are loaded (scalar loads from
// the uniform task or chain table) into registers at the stage's start, and
// its steps are unrolled to degree 7, each taken under a uniform test, so the
// coefficients are indexed by constants and the tests cost one scalar branch
// per group of values.

// t[e] <- p(x[e]) for the degree-d polynomial with coefficients kp[0..d].
template <int NV>
__device__ __forceinline__ void horner_group(const float *__restrict__ kp, uint32_t d,
                                             const float *x, float *t)
{
    float k[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
        k[i] = kp[i];
    float top = k[7];
#pragma unroll
    for (int i = 0; i < 7; ++i)
        top = d == (uint32_t)i ? k[i] : top;
#pragma unroll
    for (int e = 0; e < NV; ++e)
        t[e] = top;
#pragma unroll
    for (int i = 6; i >= 0; --i) {
        if ((uint32_t)i < d) {
#pragma unroll
            for (int e = 0; e < NV; ++e) {
                const float p = t[e] * x[e];
                t[e] = p + k[i];
            }
        }
    }
}

template <bool TWO> struct ChainMap {
    static constexpr bool kTwo = TWO;
    static constexpr bool kGroup = true;
    const float *k0; // the task's own POLY coefficients
    uint32_t d0;
    float c;
    const ChainDev *ch;
    uint32_t npost;

    // v[0..NV) <- the chain over x[0..NV) (and y), in element order
    template <int NV>
    __device__ __forceinline__ void apply(float *x, const float *y, float *v) const
    {
        if (TWO) {
#pragma unroll
            for (int e = 0; e < NV; ++e) {
                const float xy = x[e] * y[e];
                const float cx = c * x[e];
                v[e] = xy + cx;
            }
        } else {
            horner_group<NV>(k0, d0, x, v);
        }
        for (uint32_t s = 0; s < npost; ++s) {
#pragma unroll
            for (int e = 0; e < NV; ++e)
                x[e] = v[e];
            horner_group<NV>(ch->coef[s], uni(ch->deg[s]), x, v);
        }
    }
    template <int U>
    __device__ __forceinline__ void group(const float4 *xv, const float4 *yv, float *v) const
    {
        constexpr int NV = 4 * U;
        float x[NV], y[TWO ? NV : 1];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[4 * u] = xv[u].x;
            x[4 * u + 1] = xv[u].y;
            x[4 * u + 2] = xv[u].z;
            x[4 * u + 3] = xv[u].w;
            if (TWO) {
                y[4 * u] = yv[u].x;
                y[4 * u + 1] = yv[u].y;
                y[4 * u + 2] = yv[u].z;
                y[4 * u + 3] = yv[u].w;
            }
        }
        apply<NV>(x, y, v);
    }
    __device__ __forceinline__ float operator()(float x, float y) const
    {
        float v;
        apply<1>(&x, &y, &v);
        return v;
    }
};

template <bool TWO>
__device__ __forceinline__ ChainMap<TWO> chain_map(const TaskDev *tp, const ChainDev *ch)
{
    return ChainMap<TWO>{tp->coef, uni(tp->variant) & 7u, tp->c, ch, uni(ch->npost)};
}

// Tile j of a task with a map chain, through the common tile epilogue.
template <int UC>
__device__ __forceinline__ bool chain_tile(const TaskDev *__restrict__ tp,
                                           const ChainDev *__restrict__ chain, uint32_t j,
                                           const LaunchOut &L)
{
    return run_tile_with<true>(tp, j, L, [&](Acc &a) -> uint64_t {
        const uint32_t variant = uni(tp->variant);
        if (variant == V_DECLINED)
            return 0;
        const uint32_t T = uni(tp->tile_elems);
        const uint32_t nt = uni(tp->ntiles);
        const uint64_t n = uni64(tp->n);
        const float *x = tp->in0;
        const float *y = tp->in1;
        float *o = tp->out;
        const bool two = variant == V_FMUL || variant == V_FMULW;
        const bool w = variant == V_FMULW || (variant >= V_POLYW && variant < V_FMUL);
        if (two) {
            const ChainMap<true> f = chain_map<true>(tp, chain);
            return w ? tile_map<ChainMap<true>, true, UC>(f, x, y, o, n, T, nt, j, a)
                     : tile_map<ChainMap<true>, false, UC>(f, x, y, o, n, T, nt, j, a);
        }
        const ChainMap<false> f = chain_map<false>(tp, chain);
        return w ? tile_map<ChainMap<false>, true, UC>(f, x, y, o, n, T, nt, j, a)
                 : tile_map<ChainMap<false>, false, UC>(f, x, y, o, n, T, nt, j, a);
    });
}

// ---- kernels --------------------------------------------------------------

// One partition per launch: blocks stride over the task's tiles.
__global__ __launch_bounds__(kMaxBlock) void k_task(const TaskDev *__restrict__ task,
                                                 LaunchOut L)
{
    const uint32_t ntiles = uni(task->ntiles);
    for (uint32_t j = blockIdx.x; j < ntiles; j += gridDim.x)
        if (run_tile(task, j, L))
            rdd_step(L);
}

// Persistent executor: a fixed grid of blocks; block b starts with tile b of
// the queue and takes the others with one atomic each until the queue is
// empty; thread 0 asks for the next tile while the current one streams, so the
// queue round trip is hidden.  (All blocks' atomics meet on one address, about
// 60 a microsecond: 16384 tiles of 4096 elements took 255 us whatever they
// hold, so tiles of a small call are cut larger than that.)  The last block to
// leave resets the queue head, so the next launch of the same plan needs no
// clearing.
template <class Tile>
__device__ __forceinline__ void executor(const TaskDev *__restrict__ tasks,
                                         const TileRef *__restrict__ tiles, uint32_t ntiles,
                                         const LaunchOut &L, Tile tile)
{
    __shared__ uint32_t sh_tile;
    uint32_t t = blockIdx.x;
    while (t < ntiles) {
        uint32_t next = 0;
        if (threadIdx.x == 0)
            next = gridDim.x + __hip_atomic_fetch_add(&L.ctl->head, 1u, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
        const TileRef tr = tiles[t];
        const TaskDev *tp = tasks + uni(tr.task);
        tile(tp, uni(tr.tile));
        if (threadIdx.x == 0)
            sh_tile = next;
        __syncthreads();
        t = uni(sh_tile);
        __syncthreads();
    }
    // The last block to leave has every task's result (each block waited for
    // its own stores before it counted itself out): it folds the RDD total,
    // once per launch instead of one contended ticket per task, and resets
    // the queue for the next launch.
    __shared__ uint32_t sh_out;
    if (threadIdx.x == 0) {
        own_stores_complete();
        sh_out = __hip_atomic_fetch_add(&L.ctl->exited, 1u, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1
                     ? 1u
                     : 0u;
    }
    __syncthreads();
    if (uni(sh_out) != 0) {
        if (L.ntasks != 0)
            rdd_total(L);
        if (threadIdx.x == 0) {
            __hip_atomic_store(&L.ctl->head, 0u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&L.ctl->exited, 0u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

__global__ __launch_bounds__(kMaxBlock) void k_batch(const TaskDev *__restrict__ tasks,
                                                  const TileRef *__restrict__ tiles,
                                                  uint32_t ntiles, LaunchOut L)
{
    executor(tasks, tiles, ntiles, L,
             [&](const TaskDev *tp, uint32_t j) { return run_tile<true>(tp, j, L); });
}

// The persistent executor for batches whose tasks are all Monte-Carlo ones:
// the same queue and tile epilogue around the Philox tile body alone.  The
// streaming bodies set k_batch's register count (and so its waves per CU);
// without them this kernel holds half the registers and fits twice the
// waves, which the VALU-bound loop needs to issue near its rate (measured on
// MI355X: 0.95 wave-instructions per CU per clock at 3 blocks per CU, 1.04
// at 8).  A declined task (empty partial) runs no body.
__global__ __launch_bounds__(kMaxBlock) void k_batch_mc(const TaskDev *__restrict__ tasks,
                                                     const TileRef *__restrict__ tiles,
                                                     uint32_t ntiles, LaunchOut L)
{
    executor(tasks, tiles, ntiles, L, [&](const TaskDev *tp, uint32_t j) {
        return run_tile_with<true>(tp, j, L, [&](Acc &a) -> uint64_t {
            if (uni(tp->variant) != V_MC)
                return 0;
            const uint32_t T = uni(tp->tile_elems);
            const uint64_t n = uni64(tp->n);
            const uint64_t begin = (uint64_t)j * T;
            const uint64_t end = min(n, begin + T);
            if (begin >= end)
                return 0;
            tile_mc_uniform(uni64(tp->seed), uni(tp->pid), begin, end, a);
            return end - begin;
        });
    });
}

// The persistent executor over tasks that share one map chain, with UC float4
// loads in flight per thread and input (4, or 8 for short chains run at one
// block per CU, where the deeper stream hides the Horner steps' latency that
// more blocks would otherwise have to).
template <int UC>
__global__ __launch_bounds__(kBlock) void k_chain(const TaskDev *__restrict__ tasks,
                                                  const TileRef *__restrict__ tiles,
                                                  uint32_t ntiles,
                                                  const ChainDev *__restrict__ chain,
                                                  LaunchOut L)
{
    executor(tasks, tiles, ntiles, L,
             [&](const TaskDev *tp, uint32_t j) { return chain_tile<UC>(tp, chain, j, L); });
}

// MapCL materialisation only (no reduction): out[i] = map(x[i] [, y[i]]) for
// the tasks of a call, all in one launch.  Block b runs tile b: kMapUnroll
// quads per thread, all loads issued before the first store, and ends; a
// launch has one block per tile rather than a loop over few blocks.  The map
// is bound by HBM (and below a few MB by the launch), and short blocks of
// plain stores behind nontemporal loads keep both directions busiest
// (measured on MI355X, x*y + c*x over 2^26 elements: 105.7 us, 7.6 TB/s;
// nontemporal stores 123 us; one quad per thread in a loop over 768 blocks,
// the earlier kernel, 129 us; 2^28 elements: 530 us against 557).  Calls:
// 64 FMUL tasks of 2^20 elements 133 us (one launch per task: 230 us), 256
// POLY tasks of 20001 elements 10.4 us (774 us).
template <class M>
__device__ __forceinline__ void map_tile(const M &f, const float *__restrict__ x,
                                         const float *__restrict__ y,
                                         float *__restrict__ out, uint64_t n, uint64_t j)
{
    constexpr int NY = M::kTwo ? kMapUnroll : 1;
    const uint32_t tid = threadIdx.x;
    const uint32_t head = quad_head(x, n);
    const uint64_t nq = (n - head) >> 2;
    const float *x4 = x + head;
    const float *y4 = M::kTwo ? y + head : nullptr;
    float *o4 = out + head;
    auto quad = [&](uint64_t q, const float4 &xv, const float4 &yv) {
        float4 v;
        v.x = f(xv.x, yv.x);
        v.y = f(xv.y, yv.y);
        v.z = f(xv.z, yv.z);
        v.w = f(xv.w, yv.w);
        *(gf4uw *)(o4 + 4 * q) = f4a4{v.x, v.y, v.z, v.w};
    };
    const uint64_t q0 = j * (kMapUnroll * kBlock) + tid;
    if ((j + 1) * (kMapUnroll * kBlock) <= nq) {
        float4 xv[kMapUnroll], yv[NY];
#pragma unroll
        for (int u = 0; u < kMapUnroll; ++u) {
            xv[u] = ld4(x4 + 4 * (q0 + u * kBlock));
            if (M::kTwo)
                yv[u] = ld4u(y4 + 4 * (q0 + u * kBlock));
        }
#pragma unroll
        for (int u = 0; u < kMapUnroll; ++u)
            quad(q0 + u * kBlock, xv[u], M::kTwo ? yv[u] : xv[u]);
    } else {
        for (uint64_t q = q0; q < nq; q += kBlock) {
            const float4 xv = ld4(x4 + 4 * q);
            quad(q, xv, M::kTwo ? ld4u(y4 + 4 * q) : xv);
        }
    }
    if (j == 0) { // the unaligned head and the ragged tail: at most 3 each
        const uint64_t t0 = head + 4 * nq;
        if (tid < head)
            st1(out + tid, f(ld1(x + tid), M::kTwo ? ld1(y + tid) : 0.0f));
        if (tid < n - t0)
            st1(out + t0 + tid, f(ld1(x + t0 + tid), M::kTwo ? ld1(y + t0 + tid) : 0.0f));
    }
}

// The task of tile t among `count` tasks whose first tiles ascend from
// tasks[0].tile_first <= t: the last one with tile_first <= t (tasks without
// tiles share the next one's, and so are passed over).  A wave reads 64
// candidates at a time, so 4096 tasks take two rounds of loads.
__device__ __forceinline__ uint32_t task_of_tile(const TaskDev *__restrict__ tasks,
                                                 uint32_t count, uint64_t t)
{
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t lo = 0;
    while (count > 1) {
        const uint32_t step = (count + 63) / 64;
        const uint32_t at = lane * step;
        const bool le = at < count && tasks[lo + at].tile_first <= t;
        const uint32_t k = (uint32_t)__popcll(__ballot(le)) - 1u; // lane 0 always holds
        lo += k * step;
        count = min(step, count - k * step);
    }
    return uni(lo);
}

__global__ __launch_bounds__(kBlock) void k_map(const TaskDev *__restrict__ tasks,
                                                uint32_t ntasks, uint64_t tile0)
{
    const uint64_t t = tile0 + blockIdx.x;
    const TaskDev *tp = tasks + task_of_tile(tasks, ntasks, t);
    const uint64_t j = t - uni64(tp->tile_first);
    const uint64_t n = uni64(tp->n);
    const uint32_t variant = uni(tp->variant);
    const float *x = tp->in0;
    const float *y = tp->in1;
    float *o = tp->out;
    if (variant < V_FMUL) {
        float k[8];
        for (int i = 0; i < 8; ++i)
            k[i] = tp->coef[i];
#define SPARKCL_MAP_CASE(D)                                                    \
    case D: {                                                                  \
        PolyMap<D> f;                                                          \
        for (int i = 0; i < 8; ++i)                                            \
            f.k[i] = k[i];                                                     \
        map_tile(f, x, y, o, n, j);                                            \
    } break;
        switch (variant & 7u) {
            SPARKCL_MAP_CASE(0)
            SPARKCL_MAP_CASE(1)
            SPARKCL_MAP_CASE(2)
            SPARKCL_MAP_CASE(3)
            SPARKCL_MAP_CASE(4)
            SPARKCL_MAP_CASE(5)
            SPARKCL_MAP_CASE(6)
            SPARKCL_MAP_CASE(7)
        }
#undef SPARKCL_MAP_CASE
    } else {
        FmulMap f{tp->c};
        map_tile(f, x, y, o, n, j);
    }
}

// ---- array-valued ReduceCL ----------------------------------------------------
// The RDD's elements are float arrays of one length; the two-input combiner
// (Fig 3 adds two arrays elementwise) folds them pairwise along a fixed
// tree: over elements [k0, k1) the tree splits at k0 + the largest power of
// two below the count, left part first.  Each thread owns V columns and
// walks the leaves in order with a binary counter of partial results: slot j
// holds the finished perfect subtree of 2^j leaves, a new leaf merges with
// the full slots of the counter's carry chain, and at the end the occupied
// slots are merged from the smallest (rightmost) up.  That is exactly the
// tree above, so every position sees the same sequence of binary32
// combines as the definition.  Eight aligned leaves are combined as a perfect
// tree first and enter the counter at level 3.
//
// A pass reduces chunks of S leaves (S a power of two unless the pass has a
// single chunk); chunk c writes its tree to row c of the output.  Full chunks
// are aligned perfect subtrees and the last chunk is the tree of the
// remaining suffix, so a later pass over the chunk rows, with the same rule,
// rebuilds the tree over all elements.
constexpr int kTreeSlots = 13; // up to 2^12 leaves per chunk

// Float4 columns cover any length of at least 4: the last quad of a length
// that is no multiple of 4 is moved back to end at the array's end, and its
// thread stores only the columns that the quad before does not own (so a
// column is stored by one thread, and read before by no other that keeps it).
template <int V> struct TreeVec;
template <> struct TreeVec<1> {
    typedef float T;
    static __device__ __forceinline__ T ld(const float *p) { return ld1(p); }
    static __device__ __forceinline__ void st(float *p, T v, uint32_t) { st1(p, v); }
};
template <> struct TreeVec<4> {
    typedef float4 T;
    static __device__ __forceinline__ T ld(const float *p) { return ld4u(p); }
    // columns skip..3 of the quad at p
    static __device__ __forceinline__ void st(float *p, const T &v, uint32_t skip)
    {
        if (skip == 0) {
            st4u(p, v);
            return;
        }
        if (skip <= 1)
            st1(p + 1, v.y);
        if (skip <= 2)
            st1(p + 2, v.z);
        st1(p + 3, v.w);
    }
};
// First column of vector column q of arrays of len floats (len >= V), and how
// many of its columns belong to the vector before.
template <int V>
__device__ __forceinline__ uint64_t tree_col(uint64_t q, uint64_t len, uint32_t &skip)
{
    const uint64_t at = min(q * V, len - V);
    skip = (uint32_t)(q * V - at);
    return at;
}

template <uint32_t COMB>
__device__ __forceinline__ float comb1(float a, float b)
{
    if (COMB == SPARKCL_VADD)
        return a + b;
    return (b > a) ? b : a;
}
template <uint32_t COMB>
__device__ __forceinline__ float comb(float a, float b)
{
    return comb1<COMB>(a, b);
}
template <uint32_t COMB>
__device__ __forceinline__ float4 comb(const float4 &a, const float4 &b)
{
    return make_float4(comb1<COMB>(a.x, b.x), comb1<COMB>(a.y, b.y),
                       comb1<COMB>(a.z, b.z), comb1<COMB>(a.w, b.w));
}

// Insert a perfect subtree of 2^L leaves that starts at leaf `pos` (a
// multiple of 2^L) into the counter.  `pos` is wave-uniform, so every branch
// here is a scalar branch and every slot index is a compile-time constant.
template <int L, uint32_t COMB, class T, int N>
__device__ __forceinline__ void tree_insert(T (&slot)[N], uint32_t pos, T v)
{
    // the carry chain: the full slots L, L+1, ... below the first empty one
    const uint32_t full = (uint32_t)__builtin_ctz(~(pos >> L));
#pragma unroll
    for (int j = L; j < N; ++j) {
        if ((uint32_t)j < L + full)
            v = comb<COMB>(slot[j], v);
        else if ((uint32_t)j == L + full)
            slot[j] = v;
    }
}

// The tree over leaves [0, m) of one vector column, each read with leaf(i).
template <uint32_t COMB, int N, class T, class Leaf>
__device__ __forceinline__ T tree_fold(uint32_t m, Leaf leaf)
{
    T slot[N];
    uint32_t i = 0;
    for (; i + 8 <= m; i += 8) {
        T v[8];
#pragma unroll
        for (int b = 0; b < 8; ++b)
            v[b] = leaf(i + b);
        const T l = comb<COMB>(comb<COMB>(v[0], v[1]), comb<COMB>(v[2], v[3]));
        const T r = comb<COMB>(comb<COMB>(v[4], v[5]), comb<COMB>(v[6], v[7]));
        tree_insert<3, COMB>(slot, i, comb<COMB>(l, r));
    }
    for (; i < m; ++i)
        tree_insert<0, COMB>(slot, i, leaf(i));
    // merge the occupied slots, smallest (rightmost) first
    T acc{};
    bool have = false;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (m & (1u << j)) {
            acc = have ? comb<COMB>(slot[j], acc) : slot[j];
            have = true;
        }
    }
    return acc;
}

// The same over [0, m), m < 2^N, in fewer registers: the eights enter a counter
// of N - 3 slots, the last m % 8 leaves are combined as subtrees of 4, 2 and 1,
// and LOADS leaves (4 or 8) are in flight.
template <uint32_t COMB, int N, int LOADS, class T, class Leaf>
__device__ __forceinline__ T tree_fold_short(uint32_t m, Leaf leaf)
{
    T slot[N - 3];
    auto half = [&](uint32_t i) -> T { // the subtree of 4 leaves
        T v[4];
#pragma unroll
        for (int b = 0; b < 4; ++b)
            v[b] = leaf(i + b);
        return comb<COMB>(comb<COMB>(v[0], v[1]), comb<COMB>(v[2], v[3]));
    };
    uint32_t i = 0;
    for (; i + 8 <= m; i += 8) {
        const T l = half(i);
        if constexpr (LOADS == 4)
            __asm__ volatile("" ::: "memory"); // the second half's loads after the first's
        tree_insert<0, COMB>(slot, i >> 3, comb<COMB>(l, half(i + 4)));
    }
    T four{}, two{}, acc{};
    bool have = false;
    if (m & 4u) {
        four = half(i);
        i += 4;
    }
    if (m & 2u) {
        const T a = leaf(i), b = leaf(i + 1);
        two = comb<COMB>(a, b);
        i += 2;
    }
    // smallest (rightmost) first
    auto merge = [&](const T &left) {
        acc = have ? comb<COMB>(left, acc) : left;
        have = true;
    };
    if (m & 1u)
        merge(leaf(i));
    if (m & 2u)
        merge(two);
    if (m & 4u)
        merge(four);
#pragma unroll
    for (int j = 0; j < N - 3; ++j)
        if (m & (8u << j))
            merge(slot[j]);
    return acc;
}

template <uint32_t COMB>
__global__ __launch_bounds__(kBlock) void k_tree(TreeArgs a)
{
    typedef TreeVec<4> TV;
    const uint64_t q = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (4 * q >= a.len)
        return; // no barriers below
    uint32_t skip;
    const uint64_t col = tree_col<4>(q, a.len, skip);
    const uint32_t c = blockIdx.y;
    const uint32_t k0 = c * a.chunk;
    const uint32_t m = min(a.count - k0, a.chunk);
    const float4 acc = tree_fold<COMB, kTreeSlots, float4>(m, [&](uint32_t i) {
        const uint32_t kk = k0 + i;
        return TV::ld((a.ptrs ? a.ptrs[kk] : a.base + (uint64_t)kk * a.stride) + col);
    });
    TV::st(a.out + (uint64_t)c * a.len + col, acc, skip);
}

// Short arrays (at most kTreeFlatThreads vector columns): the threads of a
// block are `groups` groups (a power of two) of one thread per vector column
// of the block's `cols`, group g folds leaves [g * per, (g + 1) * per) of the
// block's chunk, and the groups' trees are combined pairwise through LDS.
// With one thread per column alone, arrays shorter than a block's threads
// leave most lanes idle and give each live one a long serial chain.  Bound by
// HBM or the memory-side cache for large inputs, by the launches and the last
// pass (one block) below some 20 MB.  At 64 registers two blocks of 1024
// threads fit a CU, or one beside two blocks of the resident serving executor;
// so the eights' counter is kept short (tree_fold_short), and a pointer table,
// whose pointers take registers of their own, has 4 loads in flight (8 for
// rows).  Measured on MI355X, in columns, with 80 registers and with 64: 2^20
// rows of 255 floats 260, 254 and 216 us; 5.6 10^6 rows of 24 722, 172 and
// 120; 268435 rows of 1000 211, 225 and 195; 2048 rows of 4096 18.3, 9.9 and
// 9.4.  The rows of a group are neighbours, so the loads of its 8 steps share
// cache lines and repeated inputs stay in the memory-side cache: plain loads,
// except NT, for inputs that exceed that cache (2^20 rows of 64 floats, 256
// MiB: 57 us plain, 68 nontemporal; 131072 rows of 2047, 1 GiB: 217 and 206;
// both with 80 registers).
constexpr int kTreeFlatSlots = 7; // up to 2^6 leaves per group
static_assert(kTreeFlatPer == 1u << (kTreeFlatSlots - 1), "a group's leaves fit the counter");

template <int V, uint32_t COMB, bool NT, bool PTRS>
__global__ __launch_bounds__(kTreeFlatThreads, 8) void k_tree_flat(TreeArgs a)
{
    typedef TreeVec<V> TV;
    typedef typename TV::T T;
    __shared__ T part[kTreeFlatThreads];
    const uint32_t tid = threadIdx.x;
    const uint32_t g = tid / a.cols;
    const uint32_t q = blockIdx.y * a.cols + (tid - g * a.cols);
    // the block is rounded up to whole waves, the last column tile is ragged
    const bool live = g < a.groups && (uint64_t)q * V < a.len;
    uint32_t skip;
    const uint64_t col = tree_col<V>(live ? q : 0, a.len, skip);
    const uint32_t per = a.chunk / a.groups;
    const uint32_t k0 = blockIdx.x * a.chunk;
    const uint32_t mb = min(a.count - k0, a.chunk);
    const uint32_t g0 = g * per;
    const uint32_t m = live && g0 < mb ? min(per, mb - g0) : 0;
    T acc = tree_fold_short<COMB, kTreeFlatSlots, PTRS ? 4 : 8, T>(m, [&](uint32_t i) -> T {
        const uint32_t kk = k0 + g0 + i;
        const float *p = (PTRS ? a.ptrs[kk] : a.base + (uint64_t)kk * a.stride) + col;
        if constexpr (NT) {
            return TV::ld(p);
        } else if constexpr (V == 4) {
            const f4a4 v = *(gf4u *)p;
            return make_float4(v.x, v.y, v.z, v.w);
        } else {
            return *(gf1 *)p;
        }
    });
    part[tid] = acc;
    const uint32_t used = (mb + per - 1) / per; // groups that hold leaves
    for (uint32_t s = 1; s < a.groups; s <<= 1) {
        __syncthreads();
        if (live && (g & (2 * s - 1)) == 0 && g + s < used) {
            acc = comb<COMB>(acc, part[tid + s * a.cols]);
            part[tid] = acc;
        }
    }
    if (live && g == 0)
        TV::st(a.out + (uint64_t)blockIdx.x * a.len + col, acc, skip);
}

// Wide variant (float4 columns only): a thread owns CPT float4 columns BT
// quads apart, so a block of BT threads reads CPT * BT * 16 bytes of one leaf
// contiguously, and the leaves are walked two at a time: each pair is a
// perfect subtree that enters the counter at level 1.  Fewer leaves and
// longer runs of each leaf in flight keep the HBM row buffers open (measured
// on MI355X over 64 arrays of 2^22 floats: 32 KiB per leaf per block, as 512
// threads of 4 columns, streams at 6.7 TB/s; 16 KiB per leaf per block in
// 256 threads at 6.4; eight leaves of 4 KiB at 5.3).  The counter holds
// kTreeWideSlots levels per column, so a chunk has at most 64 leaves.
constexpr int kTreeWideSlots = 7;
static_assert(kTreeWideChunk == 1u << (kTreeWideSlots - 1), "chunk fits the counter");

template <int L, uint32_t COMB, int CPT>
__device__ __forceinline__ void tree_insert_cols(float4 (&slot)[kTreeWideSlots][CPT],
                                                 uint32_t pos, float4 (&v)[CPT])
{
    const uint32_t full = (uint32_t)__builtin_ctz(~(pos >> L));
#pragma unroll
    for (int j = L; j < kTreeWideSlots; ++j) {
        if ((uint32_t)j < L + full) {
#pragma unroll
            for (int c = 0; c < CPT; ++c)
                v[c] = comb<COMB>(slot[j][c], v[c]);
        } else if ((uint32_t)j == L + full) {
#pragma unroll
            for (int c = 0; c < CPT; ++c)
                slot[j][c] = v[c];
        }
    }
}

template <uint32_t COMB, int CPT, int BT>
__global__ __launch_bounds__(BT) void k_tree_wide(TreeArgs a)
{
    const uint64_t nq = (a.len + 3) >> 2;
    const uint64_t q0 = (uint64_t)blockIdx.x * BT * CPT + threadIdx.x;
    if (q0 >= nq)
        return; // no barriers below
    // the array's last quad may start up to 3 floats early
    bool ok[CPT];
    uint32_t skip[CPT];
    uint64_t col[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const uint64_t q = q0 + (uint64_t)c * BT;
        ok[c] = q < nq;
        col[c] = tree_col<4>(min(q, nq - 1), a.len, skip[c]);
    }
    const uint32_t ch = blockIdx.y;
    const uint32_t k0 = ch * a.chunk;
    const uint32_t m = min(a.count - k0, a.chunk);
    auto load = [&](uint32_t i, float4 (&v)[CPT]) {
        const uint32_t kk = k0 + i;
        const float *p = a.ptrs ? a.ptrs[kk] : a.base + (uint64_t)kk * a.stride;
#pragma unroll
        for (int c = 0; c < CPT; ++c)
            v[c] = ok[c] ? ld4u(p + col[c]) : float4{};
    };
    float4 slot[kTreeWideSlots][CPT];
    uint32_t i = 0;
    for (; i + 2 <= m; i += 2) {
        float4 l[CPT], r[CPT];
        load(i, l);
        load(i + 1, r);
#pragma unroll
        for (int c = 0; c < CPT; ++c)
            l[c] = comb<COMB>(l[c], r[c]);
        tree_insert_cols<1, COMB, CPT>(slot, i, l);
    }
    if (i < m) {
        float4 v[CPT];
        load(i, v);
        tree_insert_cols<0, COMB, CPT>(slot, i, v);
    }
    float4 acc[CPT];
    bool have = false;
#pragma unroll
    for (int j = 0; j < kTreeWideSlots; ++j) {
        if (m & (1u << j)) {
#pragma unroll
            for (int c = 0; c < CPT; ++c)
                acc[c] = have ? comb<COMB>(slot[j][c], acc[c]) : slot[j][c];
            have = true;
        }
    }
    float *o = a.out + (uint64_t)ch * a.len;
#pragma unroll
    for (int c = 0; c < CPT; ++c)
        if (ok[c])
            TreeVec<4>::st(o + col[c], acc[c], skip[c]);
}

// Clears library workspaces with a kernel (no memset nodes in captured work),
// 16 bytes per store from the first 16-byte boundary on: 16 MiB in 8.2 us, in
// single words 9.2.
__global__ __launch_bounds__(kBlock) void k_zero(uint32_t *p, uint64_t words)
{
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    const uint64_t at = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    const uint64_t head = min((uint64_t)((0u - (uint32_t)((uintptr_t)p >> 2)) & 3u), words);
    const uint64_t quads = (words - head) / 4, tail = head + 4 * quads;
    uint4 *q = reinterpret_cast<uint4 *>(p + head);
    for (uint64_t i = at; i < quads; i += stride)
        q[i] = make_uint4(0u, 0u, 0u, 0u);
    if (at < head)
        p[at] = 0u;
    if (at < words - tail)
        p[tail + at] = 0u;
}

// ---- WordCount --------------------------------------------------------------
// The word-count demo (sec. 3.2.3) as a partition kernel over a byte stream:
// a word is a maximal run of non-whitespace bytes, counted under the 64-bit
// FNV-1a hash of its bytes (Fowler, Noll, Vo: xor the byte in, multiply by
// the 64-bit FNV prime).  Every lane walks a span of the text, all lanes in
// step, and keeps the running hash in registers; a word belongs to the lane
// whose span holds its first byte, which follows it past the span's end.  The
// words that end at a step go to a queue of the wave in LDS, which is emptied
// 64 words at a time, all lanes busy, into the block's LDS hash table (the
// paper's "local data").  The table absorbs the frequent words of a skewed
// vocabulary; a word that finds no place in its set is appended to the
// block's spill region of its key's partition (a plain store at an
// LDS-counted position), and the table itself is written out whole at the end;
// a merge kernel then counts each partition's keys, spilled and from the
// tables, in LDS and adds each distinct key once to the global open-addressing
// table.  (Adding every such word to the global table with a device-scope
// atomic cost more than the scan: those atomics are carried out at the memory
// side, one round trip each.)  Words that overflow a spill region go to the
// global table with atomics, and without spill regions every miss and every
// block's table.  Counts are integers, so the result does not depend on which
// block counts which word.
//
// Two blocks of 8 waves per CU with tables of 4096 keys: smaller ones hold the
// same few frequent words several times over (four of 2048 keys), and one of 16
// waves and 8192 keys, 1 to 5% faster on 16 MiB and more (512 MiB, 10^5 words:
// 544 us against 558 a call; first occurrences in 256 MiB 463 and 489), can't
// start on a CU that holds a block of the resident serving executor, whose
// registers leave room for one of 8 waves.
//
// Measured on MI355X, 512 MiB of Zipf text (10^5 words), whole call with its
// sort of the keys: 1440-1575 us with one word per lane hashed byte by byte
// from LDS and the tables added to the global one by atomics, 634 us so; 128
// MiB of 2 10^5 words, without the sort, 2155 and 250 us.  Of the scan's 435 us
// (one block of 16 waves) its walk took 320 without a word kept; places 55; the
// second queue and the tables written out whole took 150 off what misses and
// atomics cost.
constexpr int kWcScanBlock = (int)kWcWaves * 64;
constexpr int kWcBlock = 1024; // of the merge and the compaction
constexpr uint32_t kWcBlockWaves = kWcBlock / 64;
constexpr uint32_t kWcQueue = 64 + 4 * 64; // a wave's waiting words: 8 steps end
                                           // at most 4 per lane
constexpr uint32_t kWcCompact = 4 * kWcBlock; // table slots of a compaction block
constexpr uint32_t kWcMissed = 2 * 64;     // those that found no place in the table
constexpr uint32_t kWcPartSets = kWcSets >> kWcPartBits;
// Locating keeps offsets beside the words, so its table is smaller.
constexpr uint32_t kWlSets = 1760;
constexpr uint32_t kWlFew = 512;

__device__ __forceinline__ bool wc_space(uint32_t b)
{
    return b == 0x20u || (b - 0x09u) <= 4u; // space, tab, LF, VT, FF, CR
}

// Add c to key h in the global table (keys 0 = empty; a word whose hash is 0
// is counted in ctl[1] instead).
__device__ void wc_global_add(const WcArgs &a, uint64_t h, uint64_t c)
{
    if (h == 0) {
        atomicAdd((unsigned long long *)&a.ctl[1], (unsigned long long)c);
        return;
    }
    // Probe sequences are bounded: at the load factor of 1/2 that a table
    // within capacity keeps, a run of 2^16 occupied slots does not happen, so
    // only an overflowing table reaches the bound.  Every 64 probes the
    // table-full flag is checked, so once the table is full the remaining
    // words stop early (the call fails with ETOOBIG).
    uint64_t s = h & a.mask;
    const uint64_t probes = min(a.mask, (uint64_t)0xFFFF);
    for (uint64_t probe = 0; probe <= probes; ++probe) {
        if ((probe & 63) == 63 &&
            __hip_atomic_load(&a.ctl[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            return;
        const uint64_t k = a.keys[s];
        if (k == h) {
            atomicAdd((unsigned long long *)&a.counts[s], (unsigned long long)c);
            return;
        }
        if (k == 0) {
            const uint64_t old =
                atomicCAS((unsigned long long *)&a.keys[s], 0ull, (unsigned long long)h);
            if (old == 0 || old == h) {
                atomicAdd((unsigned long long *)&a.counts[s], (unsigned long long)c);
                return;
            }
        }
        s = (s + 1) & a.mask;
    }
    atomicOr((unsigned long long *)&a.ctl[2], 1ull); // table full
}

// A word that found no LDS slot: appended to this block's spill region of
// its partition, or, when the region is full (or there are none, or its key
// is 0), added to the table directly.  scnt: the block's per-partition
// append counters in LDS.
__device__ __forceinline__ void wc_spill(uint32_t *scnt, const WcArgs &a, uint64_t h)
{
    if (a.spill_cap != 0 && h != 0) {
        const uint32_t p = ((uint32_t)h & (kWcSets - 1)) / kWcPartSets;
        const uint32_t pos = atomicAdd(&scnt[p], 1u);
        if (pos < a.spill_cap) {
            a.spill[((uint64_t)blockIdx.x << kWcPartBits | p) * a.spill_cap + pos] = h;
            return;
        }
    }
    wc_global_add(a, h, 1);
}

// The place of key h in an LDS table of two-key sets: the slot that holds it
// or, if a way of its set is free, takes it; else kNoSlot.  Keys are only ever
// added, so a key read as equal stays.
constexpr uint32_t kNoSlot = ~0u;
__device__ __forceinline__ uint32_t wc_place(uint64_t *sk, uint32_t set, uint64_t h)
{
    const uint32_t s = 2 * set;
    const ulonglong2 k = *reinterpret_cast<const ulonglong2 *>(sk + s);
    const bool second = k.y == h;
    uint32_t at = k.x == h || second ? s + (second ? 1u : 0u) : kNoSlot;
    if (at == kNoSlot && (k.x == 0 || k.y == 0)) {
        // a free way, seldom once the table has filled
        for (uint32_t w = 0; w < 2 && at == kNoSlot; ++w) {
            const uint64_t old =
                atomicCAS((unsigned long long *)&sk[s + w], 0ull, (unsigned long long)h);
            if (old == 0 || old == h)
                at = s + w;
        }
    }
    return at;
}

// 16 bytes of text at byte `pos`, whatever its alignment (the memory pipeline
// takes unaligned 16-byte loads).
// Kept as vectors, and not as structs of four words, so that a load's result
// stays where it arrives.
typedef uint32_t wc_u4 __attribute__((ext_vector_type(4)));
typedef uint32_t wc_u4a1 __attribute__((ext_vector_type(4), aligned(1)));
typedef __attribute__((address_space(1))) const wc_u4a1 wc_gu4;
typedef __attribute__((address_space(1))) const uint8_t wc_gu1;
__device__ __forceinline__ wc_u4 wc_span(const uint8_t *text, uint64_t pos)
{
    return *(wc_gu4 *)(text + pos);
}
// The bytes of the 16 at `pos` of a text of n >= 16 that lie before n, the
// others spaces, so that no word starts or goes on there: v is what stands at
// min(pos, n - 16), moved down as differences from spaces.
__device__ __forceinline__ wc_u4 wc_span_end(const wc_u4 &v, uint64_t n, uint64_t pos)
{
    constexpr uint64_t kSpaces = 0x2020202020202020ull;
    uint64_t lo = ((uint64_t)v.y << 32 | v.x) ^ kSpaces;
    uint64_t hi = ((uint64_t)v.w << 32 | v.z) ^ kSpaces;
    uint32_t by = pos > n - 16 ? (uint32_t)min(pos - (n - 16), (uint64_t)16) : 0u;
    if (by >= 8) {
        lo = hi;
        hi = 0;
        by -= 8;
    }
    if (by >= 8) {
        lo = 0;
    } else if (by > 0) {
        lo = lo >> (8 * by) | hi << (64 - 8 * by);
        hi >>= 8 * by;
    }
    lo ^= kSpaces;
    hi ^= kSpaces;
    return wc_u4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

// The top bit of every byte of w that is whitespace (wc_space), the other bits
// clear: with each byte's top bit forced to 1, the per-byte subtractions
// cannot borrow across bytes, so the top bit of each byte of
// (w | 0x80..) - c tells whether its low 7 bits are >= c; bytes of 0x80 and
// above are never whitespace.
__device__ __forceinline__ uint32_t wc_space_tops(uint32_t w)
{
    const uint32_t top = 0x80808080u;
    const uint32_t up = w | top;
    const uint32_t ge09 = up - 0x09090909u;
    const uint32_t ge0e = up - 0x0E0E0E0Eu;
    const uint32_t ne20 = ((w ^ 0x20202020u) & 0x7F7F7F7Fu) + 0x7F7F7F7Fu;
    return ((ge09 & ~ge0e) | ~ne20) & ~w & top;
}

// Byte K of w: the mask of lanes in which it is not 0 / a ^ it.  One vector
// instruction each (the byte select is an operand modifier).  The first needs
// every lane active; a vector instruction may read its scalar result no
// earlier than two wait states on, which the compiler cannot see to here:
// masks_ready() stands between.
template <int K> __device__ __forceinline__ uint64_t byte_mask(uint32_t w, uint32_t zero)
{
    uint64_t r;
#define SPARKCL_BYTE_MASK(B)                                                   \
    __asm__ volatile("v_cmp_ne_u32_sdwa %0, %1, %2 src0_sel:" B " src1_sel:DWORD" \
                     : "=s"(r) : "v"(w), "v"(zero))
    if constexpr (K == 0)
        SPARKCL_BYTE_MASK("BYTE_0");
    else if constexpr (K == 1)
        SPARKCL_BYTE_MASK("BYTE_1");
    else if constexpr (K == 2)
        SPARKCL_BYTE_MASK("BYTE_2");
    else
        SPARKCL_BYTE_MASK("BYTE_3");
#undef SPARKCL_BYTE_MASK
    return r;
}
__device__ __forceinline__ void masks_ready(uint64_t (&m)[8])
{
    __asm__ volatile("s_nop 1" : "+s"(m[0]), "+s"(m[1]), "+s"(m[2]), "+s"(m[3]), "+s"(m[4]),
                                 "+s"(m[5]), "+s"(m[6]), "+s"(m[7]));
}
template <int K> __device__ __forceinline__ uint32_t xor_byte(uint32_t a, uint32_t w)
{
    uint32_t r;
    if constexpr (K == 0)
        __asm__("v_xor_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD "
                "src0_sel:DWORD src1_sel:BYTE_0" : "=v"(r) : "v"(a), "v"(w));
    else if constexpr (K == 1)
        __asm__("v_xor_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD "
                "src0_sel:DWORD src1_sel:BYTE_1" : "=v"(r) : "v"(a), "v"(w));
    else if constexpr (K == 2)
        __asm__("v_xor_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD "
                "src0_sel:DWORD src1_sel:BYTE_2" : "=v"(r) : "v"(a), "v"(w));
    else
        __asm__("v_xor_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD "
                "src0_sel:DWORD src1_sel:BYTE_3" : "=v"(r) : "v"(a), "v"(w));
    return r;
}

// to <- from before any load that follows.  Left to itself the compiler issues
// the loads that refill `from` first, into other registers, and then waits for
// them to copy them into place.
__device__ __forceinline__ void wc_take(wc_u4 (&to)[4], const wc_u4 (&from)[4])
{
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        to[u] = from[u];
        __asm__ volatile("" : "+v"(to[u]) : : "memory");
    }
}

// a in the lanes of the mask, b in the others.
__device__ __forceinline__ uint32_t lanes_select(uint64_t mask, uint32_t a, uint32_t b)
{
    uint32_t r;
    __asm__("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(b), "v"(a), "s"(mask));
    return r;
}

// A wave's walk: the lanes' running hashes, and for all lanes at once whether
// a word of the lane's is open and whether the lane may not start one: before
// its span's first whitespace, in a word of the lane before, and past its
// span's end.
template <bool kOff> struct WcWalk {
    uint32_t lo, hi;
    uint32_t start;  // kOff: where the open word starts, from the chunk's start
    uint64_t open, dead;
    uint32_t top;    // LDS address of the queue's first free key
    uint32_t top_off; // kOff: of its first free offset
};
constexpr uint32_t kFnvLo = 0x84222325u, kFnvHi = 0xCBF29CE4u;

typedef __attribute__((address_space(3))) uint32_t lds_u32;
__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(lds_u32 *)(void *)p;
}

// Four stores, each of the lanes in its mask, all lanes active before and
// after; without a branch around each store.
__device__ __forceinline__ void lds_store4(const uint64_t *mask, const uint32_t *at,
                                           const uint32_t *lo, const uint32_t *hi)
{
    __asm__ volatile("s_mov_b64 exec, %0\n\t"
                     "ds_write2_b32 %4, %8, %12 offset1:1\n\t"
                     "s_mov_b64 exec, %1\n\t"
                     "ds_write2_b32 %5, %9, %13 offset1:1\n\t"
                     "s_mov_b64 exec, %2\n\t"
                     "ds_write2_b32 %6, %10, %14 offset1:1\n\t"
                     "s_mov_b64 exec, %3\n\t"
                     "ds_write2_b32 %7, %11, %15 offset1:1\n\t"
                     "s_mov_b64 exec, -1"
                     : : "s"(mask[0]), "s"(mask[1]), "s"(mask[2]), "s"(mask[3]), "v"(at[0]),
                         "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(lo[0]), "v"(lo[1]), "v"(lo[2]),
                         "v"(lo[3]), "v"(hi[0]), "v"(hi[1]), "v"(hi[2]), "v"(hi[3])
                     : "memory");
}
__device__ __forceinline__ void lds_store4_u16(const uint64_t *mask, const uint32_t *at,
                                               const uint32_t *v)
{
    __asm__ volatile("s_mov_b64 exec, %0\n\t"
                     "ds_write_b16 %4, %8\n\t"
                     "s_mov_b64 exec, %1\n\t"
                     "ds_write_b16 %5, %9\n\t"
                     "s_mov_b64 exec, %2\n\t"
                     "ds_write_b16 %6, %10\n\t"
                     "s_mov_b64 exec, %3\n\t"
                     "ds_write_b16 %7, %11\n\t"
                     "s_mov_b64 exec, -1"
                     : : "s"(mask[0]), "s"(mask[1]), "s"(mask[2]), "s"(mask[3]), "v"(at[0]),
                         "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(v[0]), "v"(v[1]), "v"(v[2]),
                         "v"(v[3])
                     : "memory");
}

// Takes byte K of w into the hash, (h ^ b) * (2^40 + 435) mod 2^64, or starts
// over in the lanes of `sep`.
template <int K>
__device__ __forceinline__ void fnv_step(uint32_t &lo, uint32_t &hi, uint32_t w, uint64_t sep)
{
    const uint32_t x = xor_byte<K>(lo, w);
    const uint64_t p = (uint64_t)x * 435u;
    lo = lanes_select(sep, kFnvLo, (uint32_t)p);
    hi = lanes_select(sep, kFnvHi, hi * 435u + (x << 8) + (uint32_t)(p >> 32));
}

// Eight steps, the bytes of w0 and w1 in every lane: lanes that read whitespace
// with a word open queue the word's key; every hash takes the byte in or starts
// over after whitespace.  kPast: past the spans, where only open words go on.
// The masks of all steps come first, then the queue positions, then the
// hashes, then the stores: step by step, each step's vector -> scalar ->
// vector chain was waited for.
template <bool kOff, bool kPast>
__device__ __forceinline__ void wc_steps(WcWalk<kOff> &s, uint32_t w0, uint32_t w1, uint32_t zero,
                                         uint32_t at)
{
    const uint32_t s0 = wc_space_tops(w0), s1 = wc_space_tops(w1);
    uint64_t sep[8] = {byte_mask<0>(s0, zero), byte_mask<1>(s0, zero),
                       byte_mask<2>(s0, zero), byte_mask<3>(s0, zero),
                       byte_mask<0>(s1, zero), byte_mask<1>(s1, zero),
                       byte_mask<2>(s1, zero), byte_mask<3>(s1, zero)};
    masks_ready(sep);
    uint64_t ends[8];
    uint32_t pos[8], start[8], off[8], lo[8], hi[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        ends[k] = sep[k] & s.open;
        if constexpr (kOff)
            start[k] = s.start; // of the word that ends here
        if constexpr (kPast) {
            s.open &= ~sep[k];
        } else {
            const uint64_t was = s.open;
            s.dead &= ~sep[k];
            s.open = ~(sep[k] | s.dead);
            if constexpr (kOff)
                s.start = lanes_select(s.open & ~was, at + k, s.start);
        }
        const uint32_t before = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(ends[k] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ends[k], 0u));
        const uint32_t count = (uint32_t)__popcll(ends[k]);
        pos[k] = s.top + 8 * before;
        s.top += 8 * count;
        __asm__("" : "+s"(s.top)); // keeps the address one shift-add
        if constexpr (kOff) {
            off[k] = s.top_off + 2 * before;
            s.top_off += 2 * count;
            __asm__("" : "+s"(s.top_off));
        }
    }
#define SPARKCL_WC_HASH(k, W)                                                  \
    lo[k] = s.lo;                                                              \
    hi[k] = s.hi;                                                              \
    fnv_step<(k) & 3>(s.lo, s.hi, W, sep[k]);
    SPARKCL_WC_HASH(0, w0)
    SPARKCL_WC_HASH(1, w0)
    SPARKCL_WC_HASH(2, w0)
    SPARKCL_WC_HASH(3, w0)
    SPARKCL_WC_HASH(4, w1)
    SPARKCL_WC_HASH(5, w1)
    SPARKCL_WC_HASH(6, w1)
    SPARKCL_WC_HASH(7, w1)
#undef SPARKCL_WC_HASH
    lds_store4(ends, pos, lo, hi);
    lds_store4(ends + 4, pos + 4, lo + 4, hi + 4);
    if constexpr (kOff) {
        lds_store4_u16(ends, off, start);
        lds_store4_u16(ends + 4, off + 4, start + 4);
    }
}

// The scan front end shared by counting and locating.  The waves of the grid
// take chunks of 64 spans of `span` bytes (a multiple of 16, at most
// kWcMaxSpan) in turn, a wave's chunks in ascending order, neighbours on
// different CUs; word(h, off) is called with the keys of up to 64 words at a
// time and, for kOff, the byte offsets of their first bytes.  The words for
// which it returns true, a minority, are queued once more and handed to
// missed(count, h, off), again 64 at a time (count: of the lanes, from the
// first on; all are active): what it costs is then paid by full waves.
// Returns the number of words this wave saw.
//
// Bound by vector-instruction issue: about 13 instructions per step and 64
// bytes of text (71% of the SIMDs' cycles in the walk alone), and 16 more steps
// per span for the words that cross its end.  The walk touches no LDS but the
// queue; chunks of long spans keep those steps and the chunks' starts rare
// (512 MiB as one span of 2 KiB per lane, 340 us; as eight of 256 bytes, 366).
template <bool kOff, class Word, class Missed>
__device__ __forceinline__ uint64_t wc_scan(const uint8_t *text, uint64_t n, uint32_t span,
                                            Word word, Missed missed)
{
    __shared__ uint32_t queue[kWcWaves][2 * kWcQueue]; // keys, low words first
    __shared__ uint16_t queue_off[kOff ? kWcWaves : 1][kOff ? kWcQueue : 1];
    __shared__ uint64_t miss_queue[kWcWaves][kWcMissed];
    __shared__ uint16_t miss_off[kOff ? kWcWaves : 1][kOff ? kWcMissed : 1];
    const uint32_t lane = threadIdx.x & 63u, wave = uni(threadIdx.x >> 6);
    const uint32_t *q = queue[wave];
    const uint16_t *qo = kOff ? queue_off[wave] : nullptr;
    const uint32_t q0 = uni(lds_address(q)), qo0 = kOff ? uni(lds_address(qo)) : 0;
    auto key = [&](uint32_t i) -> uint64_t { return (uint64_t)q[2 * i + 1] << 32 | q[2 * i]; };
    uint64_t *mq = miss_queue[wave];
    uint16_t *mo = kOff ? miss_off[wave] : nullptr;
    uint32_t nmiss = 0;
    auto words64 = [&](bool valid, uint64_t h, uint32_t off, uint64_t c0) {
        const bool miss = valid && word(h, c0 + off);
        const uint64_t m = __ballot(miss);
        if (miss) {
            const uint32_t at = nmiss + __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            mq[at] = h;
            if (kOff)
                mo[at] = (uint16_t)off;
        }
        nmiss += (uint32_t)__popcll(m);
        if (nmiss >= 64) {
            nmiss -= 64;
            missed(64u, mq[nmiss + lane], kOff ? c0 + mo[nmiss + lane] : 0ull);
        }
    };
    const uint64_t bytes = 64ull * span;
    const uint64_t nchunks = (n + bytes - 1) / bytes;
    const uint32_t steps = span / 16;
    uint32_t zero = 0;
    __asm__ volatile("v_mov_b32 %0, 0" : "=v"(zero)); // a register, not a constant
    uint64_t words = 0;
    WcWalk<kOff> s;
    s.top = q0;
    s.top_off = qo0;
    s.start = 0;
    // 64 bytes per lane at a time, the next 64 loaded ahead, also those of the
    // next chunk; what lies past the end is read at the end and put right later
    const uint64_t last = n - 16;
    auto load = [&](uint64_t at, wc_u4 (&v)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[u] = wc_span(text, min(at + 16 * u, last));
    };
    auto byte_before = [&](uint64_t at) -> uint32_t {
        return at > 0 && at <= n ? *(wc_gu1 *)(text + at - 1) : 0x20u;
    };
    const uint64_t c_step = (uint64_t)gridDim.x * kWcWaves;
    uint64_t c = (uint64_t)wave * gridDim.x + blockIdx.x;
    wc_u4 cur[4], nx[4], first[4];
    uint32_t before_next = 0x20u;
    if (c < nchunks) {
        load(c * bytes + (uint64_t)lane * span, first);
        before_next = byte_before(c * bytes + (uint64_t)lane * span);
    }
    for (; c < nchunks; c += c_step) {
        const uint64_t c0 = c * bytes;
        const uint64_t at = c0 + (uint64_t)lane * span;
        const uint32_t before = before_next;
        wc_take(nx, first);
        if (c + c_step < nchunks) {
            load(at + c_step * bytes, first);
            before_next = byte_before(at + c_step * bytes);
        }
        s.dead = ~__ballot(wc_space(before));
        s.open = 0;
        s.lo = kFnvLo;
        s.hi = kFnvHi;
        const uint32_t from = s.top;
        // 16 bytes per lane and round; rounds past the span go on while a
        // word is open
        for (uint32_t r = 0; r < steps || s.open != 0;) {
            wc_take(cur, nx);
            load(at + 16ull * r + 64, nx);
#pragma unroll 1
            for (int u = 0; u < 4 && (r < steps || s.open != 0); ++u, ++r) {
                if (c0 + 63ull * span + 16ull * r + 16 > n)
                    cur[0] = wc_span_end(cur[0], n, at + 16ull * r);
                uint32_t w0 = cur[0].x, w1 = cur[0].y;
                uint32_t rel = kOff ? lane * span + 16 * r : 0;
#pragma unroll 1
                for (int half = 0; half < 2; ++half) {
                    if (r < steps)
                        wc_steps<kOff, false>(s, w0, w1, zero, rel);
                    else
                        wc_steps<kOff, true>(s, w0, w1, zero, rel);
                    while (s.top >= q0 + 64 * 8) { // the queue's last 64 words
                        s.top -= 64 * 8;
                        s.top_off -= 64 * 2;
                        words += 64;
                        const uint32_t i = (s.top - q0) / 8 + lane;
                        words64(true, key(i), kOff ? qo[i] : 0u, kOff ? c0 : 0ull);
                    }
                    w0 = cur[0].z;
                    w1 = cur[0].w;
                    rel += 8;
                }
#pragma unroll
                for (int v = 0; v < 3; ++v)
                    cur[v] = cur[v + 1];
            }
        }
        words += (int64_t)((int32_t)(s.top - from) / 8);
        if (kOff) { // queued offsets are the chunk's own
            const bool valid = lane < (s.top - q0) / 8;
            words64(valid, key(lane), qo[lane], c0);
            missed(nmiss, mq[lane], c0 + mo[lane]);
            s.top = q0;
            s.top_off = qo0;
            nmiss = 0;
        }
    }
    if (!kOff) {
        words64(lane < (s.top - q0) / 8, key(lane), 0u, 0ull);
        missed(nmiss, mq[lane], 0ull);
    }
    return words;
}

__global__ __launch_bounds__(kWcScanBlock, 4) void k_wordcount(WcArgs a)
{
    __shared__ __attribute__((aligned(16))) uint64_t sk[kWcSlots];
    // 32 bits each: a block counts at most one word per two bytes of the text it
    // scans, and it scans either a few KiB or about 1/512 of the text (a grid of
    // two blocks per CU), which is limited to 2^40 bytes
    __shared__ uint32_t sc[kWcSlots];
    __shared__ uint32_t scnt[1u << kWcPartBits];    // spill appends per partition
    const uint32_t tid = threadIdx.x;
    for (uint32_t i = tid; i < kWcSlots; i += kWcScanBlock) {
        sk[i] = 0;
        sc[i] = 0;
    }
    for (uint32_t i = tid; i < (1u << kWcPartBits); i += kWcScanBlock)
        scnt[i] = 0;
    __syncthreads();
    const uint64_t words = wc_scan<false>(
        a.text, a.n, a.span,
        [&](uint64_t h, uint64_t) -> bool {
            const uint32_t at = h != 0 ? wc_place(sk, (uint32_t)h & (kWcSets - 1), h) : kNoSlot;
            if (at != kNoSlot)
                atomicAdd(&sc[at], 1u);
            return at == kNoSlot;
        },
        [&](uint32_t count, uint64_t h, uint64_t) {
            if ((tid & 63u) < count)
                wc_spill(scnt, a, h);
        });
    __syncthreads();
    if (a.spill_cap != 0) {
        // the table as it stands, for the merge: a set's slots hold the same
        // partition's keys in every block
        const uint64_t row = (uint64_t)blockIdx.x * kWcSlots;
        for (uint32_t i = tid; i < kWcSlots; i += kWcScanBlock) {
            a.table_keys[row + i] = sk[i];
            a.table_counts[row + i] = sc[i];
        }
        for (uint32_t p = tid; p < (1u << kWcPartBits); p += kWcScanBlock)
            a.spill_cnt[((uint64_t)blockIdx.x << kWcPartBits) | p] = min(scnt[p], a.spill_cap);
    } else {
        for (uint32_t i = tid; i < kWcSlots; i += kWcScanBlock)
            if (sk[i])
                wc_global_add(a, sk[i], sc[i]);
    }
    if ((tid & 63u) == 0 && words)
        atomicAdd((unsigned long long *)&a.ctl[0], (unsigned long long)words);
}

// A text shorter than the 16 bytes that the scan loads at a time, between
// spaces: n of the 32 bytes at `out`.
__global__ void k_wc_pad(const uint8_t *text, uint64_t n, uint8_t *out)
{
    out[threadIdx.x] = threadIdx.x < n ? text[threadIdx.x] : (uint8_t)0x20;
}

// ---- WordCount's words: the first occurrence of each key --------------------
// A lookup table of the wanted keys and the lowest offset seen of each (open
// addressing, key 0 = empty; the key 0 itself has index + 1 in ctl[0] and its
// offset in ctl[2]), then one pass of the scan front end in which every word
// whose key is in the table lowers that key's offset to its own with an atomic
// minimum, unless the offset that it reads beside the key is already lower.
// Most words don't come that far: the block keeps the keys it has met in LDS,
// each with (a 256th of) the lowest offset that one of its words took to the
// table, and a word past that offset is done.  The others wait until there are
// 64 of them, so that a wave reads the table for all its lanes: random reads
// of L2, which bound the pass without the LDS keys (one in three words comes
// to the table), and are one per word with key and offset side by side.  256 MiB
// of Zipf text, 10^5 keys: 762 us with three reads for every word, 499 us now.
// (the table's size is no power of two; Knuth's multiplicative hash of the key)
__device__ __forceinline__ uint64_t wl_slot(uint64_t h, uint64_t slots)
{
    return __umul64hi(h * 0x9E3779B97F4A7C15ull, slots);
}

__global__ __launch_bounds__(kBlock) void k_wl_build(WlArgs l)
{
    const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= l.nkeys)
        return;
    const uint64_t h = l.keys[i];
    if (h == 0) {
        if (atomicCAS((unsigned long long *)&l.ctl[0], 0ull, (unsigned long long)(i + 1)) != 0)
            atomicOr((unsigned long long *)&l.ctl[1], 1ull); // the key 0 twice
        l.ctl[2] = ~0ull;
        return;
    }
    uint64_t s = wl_slot(h, l.slots);
    for (uint64_t probe = 0; probe < l.slots; ++probe) {
        // (a read first: a swap is a round trip to the memory side)
        uint64_t old = l.table[s].key;
        if (old == 0)
            old = atomicCAS((unsigned long long *)&l.table[s].key, 0ull, (unsigned long long)h);
        if (old == 0) {
            l.table[s].off = ~0ull;
            l.offsets[i] = s; // until k_wl_result
            return;
        }
        if (old == h) {
            atomicOr((unsigned long long *)&l.ctl[1], 1ull); // a key twice
            l.offsets[i] = s;
            return;
        }
        s = s + 1 == l.slots ? 0 : s + 1;
    }
}

// The result of key i, after every word: its slot's offset in place of the slot.
__device__ __forceinline__ void wl_result(const WlArgs &l, uint64_t i)
{
    l.offsets[i] = ld_agent(l.keys[i] == 0 ? &l.ctl[2] : &l.table[l.offsets[i]].off);
}

__global__ __launch_bounds__(kBlock) void k_wl_result(WlArgs l)
{
    const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < l.nkeys)
        wl_result(l, i);
}

// The table's part of a word.
__device__ __forceinline__ void wl_lookup(const WlArgs &l, uint64_t h, uint64_t off)
{
    if (h == 0) {
        if (l.ctl[0] && l.ctl[2] > off)
            atomicMin((unsigned long long *)&l.ctl[2], (unsigned long long)off);
        return;
    }
    // a third of the slots at least is empty, so a probe run ends
    uint64_t s = wl_slot(h, l.slots);
    for (uint64_t probe = 0; probe < l.slots; ++probe) {
        const ulonglong2 e = *reinterpret_cast<const ulonglong2 *>(l.table + s);
        if (e.x == h) {
            if (e.y > off)
                atomicMin((unsigned long long *)&l.table[s].off, (unsigned long long)off);
            return;
        }
        if (e.x == 0)
            return;
        s = s + 1 == l.slots ? 0 : s + 1;
    }
}

// FEW: at most kWlFew keys are wanted, and most words are none of them.  A bit
// for each of 4096 values of a word's hash then drops those first, which
// otherwise pass through the block's table, the second queue and the global
// table, and the block that ends last writes the results, which saves a launch.
// Ten keys in 128 MiB of 8-letter words that hardly repeat: 191 us without the
// bits, 146 so; in 256 MiB of Zipf text 308 and 244, in 4 KiB 32 and 31 a call.
// (Where every word is wanted the bits only cost: 1000 keys in 128 MiB of just
// these words 190 us without them, 198 with.)
constexpr uint32_t kWlBits = 8 * kWlFew;
__device__ __forceinline__ uint32_t wl_bit(uint64_t h)
{
    return (uint32_t)(h >> 32) & (kWlBits - 1);
}

template <bool FEW>
__global__ __launch_bounds__(kWcScanBlock, 4) void k_wl_scan(WlArgs l)
{
    __shared__ __attribute__((aligned(16))) uint64_t sk[2 * kWlSets];
    __shared__ uint32_t sv[2 * kWlSets]; // lowest offset / 256 taken to the table (n <= 2^40)
    __shared__ uint32_t wanted[FEW ? kWlBits / 32 : 1];
    __shared__ uint32_t last;
    for (uint32_t i = threadIdx.x; i < 2 * kWlSets; i += kWcScanBlock) {
        sk[i] = 0;
        sv[i] = ~0u;
    }
    if constexpr (FEW) {
        for (uint32_t i = threadIdx.x; i < kWlBits / 32; i += kWcScanBlock)
            wanted[i] = 0;
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < (uint32_t)l.nkeys; i += kWcScanBlock) {
            const uint32_t b = wl_bit(l.keys[i]);
            atomicOr(&wanted[b / 32], 1u << (b % 32));
        }
    }
    __syncthreads();
    (void)wc_scan<true>(
        l.text, l.n, l.span,
        [&](uint64_t h, uint64_t off) -> bool {
            if constexpr (FEW) {
                const uint32_t b = wl_bit(h);
                if ((wanted[b / 32] >> (b % 32) & 1u) == 0)
                    return false;
            }
            const uint32_t at =
                h != 0 ? wc_place(sk, __umulhi((uint32_t)h, kWlSets), h) : kNoSlot;
            if (at != kNoSlot) {
                const uint32_t mine = (uint32_t)(off >> 8);
                // (the second test drops most of the same word's others among
                // these 64 words)
                if (sv[at] < mine || atomicMin(&sv[at], mine) < mine)
                    return false; // a word before this one goes to the table
            }
            return true;
        },
        [&](uint32_t count, uint64_t h, uint64_t off) {
            if ((threadIdx.x & 63u) < count)
                wl_lookup(l, h, off);
        });
    if constexpr (FEW) {
        own_stores_complete(); // and the atomics
        __syncthreads();
        if (threadIdx.x == 0)
            last = atomicAdd((unsigned long long *)&l.ctl[3], 1ull) == gridDim.x - 1;
        __syncthreads();
        if (last)
            for (uint32_t i = threadIdx.x; i < (uint32_t)l.nkeys; i += kWcScanBlock)
                wl_result(l, i);
    }
}

// Merge: block p counts partition p's words, from the scan blocks' spill regions
// and from its sets of their tables, in an LDS table, and adds each distinct
// key to the global table once.  Keys that find no LDS slot go there directly.
// One block per partition, so that a key costs one global atomic: eight blocks
// of each, and the scan blocks adding their own tables (two million keys),
// spent most of 200 us on them.
//
// A wave takes one scan block's region at a time, K keys per lane, with the
// next region's keys in flight.  72 KiB of LDS: a block of 96 KiB does not
// start on a CU that holds two blocks of the serving executor, small as their
// own LDS is.
constexpr uint32_t kWcMergeSlots = 6144;
constexpr uint32_t kWcMergeProbes = 8;

// The slot of key h (not 0) in the merge's table, or kNoSlot.
__device__ __forceinline__ uint32_t wc_merge_place(uint64_t *mk, uint64_t h)
{
    // (other bits of the key make the partition)
    uint32_t s = __umulhi((uint32_t)(h >> 32), kWcMergeSlots);
    for (uint32_t q = 0; q < kWcMergeProbes; ++q) {
        uint64_t key = mk[s];
        if (key == 0) {
            key = atomicCAS((unsigned long long *)&mk[s], 0ull, (unsigned long long)h);
            key = key == 0 ? h : key;
        }
        if (key == h)
            return s;
        s = s + 1 == kWcMergeSlots ? 0 : s + 1;
    }
    return kNoSlot;
}

// add(h) for partition p's spilled keys.
template <int K, class Add>
__device__ __forceinline__ void wc_merge_regions(const WcArgs &a, uint32_t scan_grid, Add add)
{
    const uint32_t p = blockIdx.x;
    const uint32_t lane = threadIdx.x & 63u, wave = uni(threadIdx.x >> 6);
    uint64_t h[K], next[K];
    uint32_t left = 0; // keys of the region in flight past those loaded
    uint64_t from = 0; // where they start
    auto load = [&](uint64_t at, uint32_t cnt) {
#pragma unroll
        for (int u = 0; u < K; ++u)
            next[u] = lane + 64 * u < cnt ? a.spill[at + lane + 64 * u] : 0;
        left = cnt > 64 * K ? cnt - 64 * K : 0;
        from = at + 64 * K;
    };
    // 64 regions' counts at a time
    for (uint32_t b0 = wave; b0 < scan_grid; b0 += 64 * kWcBlockWaves) {
        const uint32_t mine = b0 + lane * kWcBlockWaves;
        const uint32_t counts =
            mine < scan_grid ? a.spill_cnt[((uint64_t)mine << kWcPartBits) | p] : 0;
        const uint32_t regions = min(64u, (scan_grid - b0 + kWcBlockWaves - 1) / kWcBlockWaves);
        auto region = [&](uint32_t at) -> uint64_t {
            return (((uint64_t)(b0 + at * kWcBlockWaves) << kWcPartBits) | p) * a.spill_cap;
        };
        uint32_t j = 0;
        load(region(0), __builtin_amdgcn_readlane(counts, 0));
        while (j < regions) {
#pragma unroll
            for (int u = 0; u < K; ++u) {
                h[u] = next[u];
                __asm__ volatile("" : "+v"(h[u]) : : "memory"); // before the loads, as wc_take
            }
            if (left) // a region of more than 64 K keys
                load(from, left);
            else if (++j < regions)
                load(region(j), __builtin_amdgcn_readlane(counts, j));
            // one copy of the insert, the keys rotated through h[0]
#pragma unroll 1
            for (int u = 0; u < K; ++u) {
                if (h[0]) // spilled keys are never 0
                    add(h[0]);
#pragma unroll
                for (int w = 0; w + 1 < K; ++w)
                    h[w] = h[w + 1];
            }
        }
    }
}

__global__ __launch_bounds__(kWcBlock) void k_wc_merge(WcArgs a, uint32_t scan_grid)
{
    __shared__ uint64_t mk[kWcMergeSlots];
    __shared__ uint32_t mc[kWcMergeSlots];
    for (uint32_t i = threadIdx.x; i < kWcMergeSlots; i += kWcBlock) {
        mk[i] = 0;
        mc[i] = 0;
    }
    __syncthreads();
    auto add = [&](uint64_t h, uint32_t c) {
        const uint32_t s = wc_merge_place(mk, h);
        if (s == kNoSlot) {
            wc_global_add(a, h, c);
            return;
        }
        // 32 bits hold a block's words (k_wordcount); a partition's, of all blocks,
        // may pass them: what carries goes to the table
        const uint32_t old = atomicAdd(&mc[s], c);
        if (old + c < old)
            wc_global_add(a, h, 1ull << 32);
    };
    // the partition's slots of the scan blocks' tables, two blocks per wave
    constexpr uint32_t kShare = 2 * kWcPartSets;
    for (uint32_t i = threadIdx.x; i < scan_grid * kShare; i += kWcBlock) {
        const uint64_t at = (uint64_t)(i / kShare) * kWcSlots + blockIdx.x * kShare + i % kShare;
        const uint64_t h = a.table_keys[at];
        if (h)
            add(h, a.table_counts[at]);
    }
    wc_merge_regions<6>(a, scan_grid, [&](uint64_t h) { add(h, 1u); });
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kWcMergeSlots; i += kWcBlock)
        if (mk[i])
            wc_global_add(a, mk[i], mc[i]);
}

// Compaction of the global table into the caller's key/count arrays
// (unordered); ctl[3] counts the distinct keys, also those past `cap`.  Each
// block holds its slots' keys in registers, counts them, reserves room with
// one atomic add (a counter bumped once per key would serialise on that one
// address) and writes them there.  Blocks are large for the same reason: 1024
// blocks' adds of a table of 2^20 slots took most of 20 us, 256 take 9.
__global__ __launch_bounds__(kWcBlock) void k_wc_compact(WcArgs a, uint64_t *out_keys,
                                                         uint64_t *out_counts, uint64_t cap)
{
    __shared__ uint32_t sh_wave[kWcBlockWaves];
    __shared__ uint64_t sh_base;
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint64_t first = (uint64_t)blockIdx.x * kWcCompact + threadIdx.x;
    uint64_t k[kWcCompact / kWcBlock];
    uint32_t mine = 0; // the wave's keys
#pragma unroll
    for (uint32_t u = 0; u < kWcCompact / kWcBlock; ++u) {
        const uint64_t s = first + u * kWcBlock;
        k[u] = s <= a.mask ? a.keys[s] : 0;
    }
#pragma unroll
    for (uint32_t u = 0; u < kWcCompact / kWcBlock; ++u)
        mine += (uint32_t)__popcll(__ballot(k[u] != 0));
    if (lane == 0)
        sh_wave[wave] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t total = 0;
        for (uint32_t w = 0; w < kWcBlockWaves; ++w) {
            const uint32_t n = sh_wave[w];
            sh_wave[w] = total;
            total += n;
        }
        sh_base = total ? atomicAdd((unsigned long long *)&a.ctl[3], (unsigned long long)total)
                        : 0;
    }
    __syncthreads();
    uint64_t base = sh_base + sh_wave[wave];
#pragma unroll
    for (uint32_t u = 0; u < kWcCompact / kWcBlock; ++u) {
        const uint64_t set = __ballot(k[u] != 0);
        if (k[u] != 0) {
            const uint64_t pos = base + __popcll(set & ((1ull << lane) - 1));
            if (pos < cap) {
                out_keys[pos] = k[u];
                out_counts[pos] = a.counts[first + u * kWcBlock];
            }
        }
        base += __popcll(set);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && a.ctl[1]) {
        const uint64_t pos = atomicAdd((unsigned long long *)&a.ctl[3], 1ull);
        if (pos < cap) {
            out_keys[pos] = 0;
            out_counts[pos] = a.ctl[1];
        }
    }
}

// Synthetic data for the autotuner: a cheap hash pattern in [-1, 1).
__global__ __launch_bounds__(kBlock) void k_fill_pattern(float *p, uint64_t n,
                                                         uint32_t salt)
{
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
        uint32_t h = (uint32_t)i * 0x9E3779B1u ^ salt;
        h ^= h >> 15;
        h *= 0x85EBCA6Bu;
        h ^= h >> 13;
        p[i] = (float)((int32_t)(h >> 8) - (1 << 23)) * (1.0f / 8388608.0f);
    }
}

// ---- resident serving executor -------------------------------------------
// Block 0 is the dispatcher: it polls the host ring's tail word (system
// scope), copies each new descriptor into the device table, writes the task's
// tiles into the tile map and publishes the new tile count.  Every other block
// is a worker.  A worker takes one tile ticket at a time with an atomic add
// (one round trip, no retries), then polls the published-tile word with
// exponential backoff until its ticket is published, and runs the tile
// exactly as the batch executor does; a task's last tile writes its result to
// host memory and then its completion word.  Every wait is bounded: the
// dispatcher leaves on the host's stop word, or after idle_ticks without new
// work, setting the stop bit of the published-tile word (and the abort bit
// when the host asked to abort).  A worker leaves only on the abort bit, or
// when the stop bit is set and its ticket is unpublished: a claimed ticket is
// never given up while the dispatcher lives, however long the wait for its
// tile (under a light load the highest claims wait for hundreds of tasks).
// The stop bit is or-ed into the final published count, so a worker that sees
// it also sees every tile that will ever be published in this launch.
// Tickets are issued in order and a worker never leaves holding a published
// ticket, so every published tile runs before the grid drains.  A ticket left
// unpublished at exit is discarded by the next launch's prologue, which
// restarts the tickets at the published count.  A dispatcher that stops
// polling would leave the workers waiting; the host's watchdog covers that
// case (it aborts the launch).

static_assert(offsetof(TaskDev, ntiles) == 96, "word 24 of a descriptor");
static_assert(offsetof(TaskDev, tile_first) == 120, "words 30-31 of a descriptor");

// Descriptors copied per round of the dispatcher: one per 32-thread group, so
// a burst of arrivals costs one host-memory round trip per 8 tasks.
constexpr uint32_t kServeBatch = kBlock / 32;

__device__ __forceinline__ void serve_dispatch(const ServeArgs &a)
{
    __shared__ uint64_t sh_tail, sh_stop;
    __shared__ uint32_t sh_nt[kServeBatch], sh_first_lo[kServeBatch], sh_first_hi[kServeBatch];
    uint64_t taken = uni64(ld_agent(&a.dev->taken));
    uint64_t last = wall_clock64();
    for (;;) {
        if (threadIdx.x == 0) {
            sh_tail = __hip_atomic_load(&a.host->tail, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_SYSTEM);
            sh_stop = __hip_atomic_load(&a.host->stop, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_SYSTEM);
        }
        __syncthreads();
        const uint64_t tail = uni64(sh_tail);
        const uint32_t stop = uni((uint32_t)sh_stop);
        __syncthreads();
        if (stop) {
            if (threadIdx.x == 0 && stop >= 2)
                __hip_atomic_fetch_or(&a.dev->tiles_pub, kServeAbortBit, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
        if (tail > taken) {
            uint64_t pub = 0;
            // Descriptors taken .. tail-1, kServeBatch at a time: group g of
            // 32 threads copies descriptor s0 + g (one 32-bit word per
            // thread) from the host ring to the device table and writes its
            // tile-map entries.  The tile ranges of different descriptors are
            // disjoint (the host assigned them), so the groups work apart.
            const uint32_t g = threadIdx.x >> 5, l = threadIdx.x & 31u;
            for (uint64_t s0 = taken; s0 < tail; s0 += kServeBatch) {
                const uint64_t s = s0 + g;
                const uint32_t slot = (uint32_t)(s & (a.cap - 1));
                uint32_t nt = 0;
                uint64_t first = 0;
                if (s < tail) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
                    uint32_t *src = reinterpret_cast<uint32_t *>(
                                        const_cast<TaskDev *>(a.ring + slot)) + l;
                    uint32_t *dst = reinterpret_cast<uint32_t *>(a.table + slot) + l;
                    const uint32_t w = __hip_atomic_load(src, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_SYSTEM);
                    __hip_atomic_store(dst, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (l == 24)
                        sh_nt[g] = w;
                    if (l == 30)
                        sh_first_lo[g] = w;
                    if (l == 31)
                        sh_first_hi[g] = w;
                }
                __syncthreads();
                if (s < tail) {
                    nt = sh_nt[g];
                    first = ((uint64_t)sh_first_hi[g] << 32) | sh_first_lo[g];
                    for (uint32_t k = l; k < nt; k += 32)
                        __hip_atomic_store(a.tilemap + ((first + k) & (a.tile_cap - 1)), slot,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                // the last descriptor of the round ends the published range
                const uint32_t last = (uint32_t)min((uint64_t)kServeBatch, tail - s0) - 1;
                pub = (((uint64_t)uni(sh_first_hi[last]) << 32) | uni(sh_first_lo[last])) +
                      uni(sh_nt[last]);
                __syncthreads();
            }
            // table and tile-map entries were written with agent-scope atomic
            // stores; once they are complete the new tile count is published
            own_stores_complete();
            __syncthreads();
            if (threadIdx.x == 0) {
                st_agent(&a.dev->taken, tail);
                own_stores_complete();
                st_agent(&a.dev->tiles_pub, pub);
            }
            taken = tail;
            last = wall_clock64();
            continue;
        }
        if (wall_clock64() - last > a.idle_ticks)
            break;
        __builtin_amdgcn_s_sleep(16);
    }
    if (threadIdx.x == 0)
        __hip_atomic_fetch_or(&a.dev->tiles_pub, kServeStopBit, __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void serve_work(const ServeArgs &a)
{
    __shared__ uint64_t sh_tile;
    __shared__ TaskDev sh_task;
    constexpr uint64_t kNone = ~0ull;
    for (;;) {
        if (threadIdx.x == 0) {
            const uint64_t c = __hip_atomic_fetch_add(&a.dev->claim, 1ull, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
            uint64_t got = kNone;
            uint32_t backoff = 1;
            for (;;) {
                const uint64_t w = ld_agent(&a.dev->tiles_pub);
                if (w & kServeAbortBit)
                    break;
                if (c < (w & kServeCountMask)) {
                    got = c;
                    break;
                }
                if (w & kServeStopBit)
                    break;
                // s_sleep takes an immediate: a few fixed steps of backoff
                if (backoff == 1)
                    __builtin_amdgcn_s_sleep(1);
                else if (backoff == 2)
                    __builtin_amdgcn_s_sleep(4);
                else
                    __builtin_amdgcn_s_sleep(16);
                backoff = backoff < 3 ? backoff + 1 : 3;
            }
            sh_tile = got;
        }
        __syncthreads();
        const uint64_t t = uni64(sh_tile);
        if (t == kNone)
            break;
        // Acquire before touching the task: the descriptor, and the task's
        // inputs, which the caller may have rewritten since this resident
        // kernel last read that memory (its L2 is not invalidated between
        // tasks the way it is between kernel launches).
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (threadIdx.x < 32) {
            const uint32_t slot = __hip_atomic_load(a.tilemap + (t & (a.tile_cap - 1)),
                                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            uint32_t *src = reinterpret_cast<uint32_t *>(a.table + slot) + threadIdx.x;
            reinterpret_cast<uint32_t *>(&sh_task)[threadIdx.x] =
                __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        const uint32_t j = uni((uint32_t)(t - sh_task.tile_first));
        run_tile(&sh_task, j, a.out);
        __syncthreads();
    }
}

__global__ __launch_bounds__(kBlock) void k_serve(ServeArgs a)
{
    if (blockIdx.x == 0)
        serve_dispatch(a);
    else
        serve_work(a);
}

// Launch prologue: clear the stop bit and restart the tickets at the
// published count (no worker of the previous launch is alive to hold one).
__global__ void k_serve_prologue(ServeDev *d)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const uint64_t pub = d->tiles_pub & kServeCountMask;
        d->tiles_pub = pub;
        d->claim = pub;
    }
}

int hip_status(hipError_t e)
{
    return e == hipSuccess ? SPARKCL_OK : SPARKCL_EHIP;
}

} // namespace

int launch_task(const TaskDev *dtask, uint32_t ntiles, uint32_t grid,
                const LaunchOut &out, void *stream, uint32_t block)
{
    if (block != 256 && block != 512 && block != 1024)
        return SPARKCL_EINVAL;
    if (ntiles == 0 || grid == 0)
        return SPARKCL_EINVAL;
    grid = grid < ntiles ? grid : ntiles;
    hipLaunchKernelGGL(k_task, dim3(grid), dim3(block), 0, (hipStream_t)stream,
                       dtask, out);
    return hip_status(hipGetLastError());
}

int launch_chain(const TaskDev *dtasks, const TileRef *tiles, uint32_t ntiles,
                 const ChainDev *chain, uint32_t grid, const LaunchOut &out, uint32_t unroll,
                 void *stream)
{
    if (ntiles == 0 || grid == 0 || !chain || (unroll != 4 && unroll != 8))
        return SPARKCL_EINVAL;
    if (unroll == 8)
        hipLaunchKernelGGL(k_chain<8>, dim3(grid), dim3(kBlock), 0, (hipStream_t)stream,
                           dtasks, tiles, ntiles, chain, out);
    else
        hipLaunchKernelGGL(k_chain<4>, dim3(grid), dim3(kBlock), 0, (hipStream_t)stream,
                           dtasks, tiles, ntiles, chain, out);
    return hip_status(hipGetLastError());
}

int launch_batch(const TaskDev *dtasks, const TileRef *tiles, uint32_t ntiles,
                 uint32_t grid, const LaunchOut &out, void *stream, uint32_t block,
                 bool mc_only)
{
    if (ntiles == 0 || grid == 0 || (block != 256 && block != 512 && block != 1024))
        return SPARKCL_EINVAL;
    if (mc_only)
        hipLaunchKernelGGL(k_batch_mc, dim3(grid), dim3(block), 0, (hipStream_t)stream,
                           dtasks, tiles, ntiles, out);
    else
        hipLaunchKernelGGL(k_batch, dim3(grid), dim3(block), 0, (hipStream_t)stream,
                           dtasks, tiles, ntiles, out);
    return hip_status(hipGetLastError());
}

int launch_map(const TaskDev *dtasks, uint32_t ntasks, uint64_t tile0, uint64_t ntiles,
               void *stream)
{
    if (ntasks == 0 || ntiles == 0)
        return SPARKCL_EINVAL;
    return in_launches(ntiles, kBlock, [&](uint64_t at, uint32_t grid) {
        hipLaunchKernelGGL(k_map, dim3(grid), dim3(kBlock), 0, (hipStream_t)stream, dtasks,
                           ntasks, tile0 + at);
        return hip_status(hipGetLastError());
    });
}

int launch_wc_pad(const uint8_t *text, uint64_t n, uint8_t *out, void *stream)
{
    if (n > kWcPad)
        return SPARKCL_EINVAL;
    hipLaunchKernelGGL(k_wc_pad, dim3(1), dim3(kWcPad), 0, (hipStream_t)stream, text, n, out);
    return hip_status(hipGetLastError());
}

int launch_wordcount(const WcArgs &a, uint32_t grid, void *stream)
{
    if (grid == 0 || a.n < 16 || !a.keys || !a.counts || !a.ctl || ((a.mask + 1) & a.mask) ||
        (a.spill_cap != 0 &&
         (!a.spill || !a.spill_cnt || !a.table_keys || !a.table_counts)) ||
        a.span == 0 || a.span % 16 != 0 ||
        a.span > kWcMaxSpan)
        return SPARKCL_EINVAL;
    hipLaunchKernelGGL(k_wordcount, dim3(grid), dim3(kWcScanBlock), 0, (hipStream_t)stream, a);
    return hip_status(hipGetLastError());
}

int launch_wc_merge(const WcArgs &a, uint32_t scan_grid, void *stream)
{
    if (a.spill_cap == 0 || scan_grid == 0 || !a.table_keys || !a.table_counts)
        return SPARKCL_EINVAL;
    hipLaunchKernelGGL(k_wc_merge, dim3(1u << kWcPartBits), dim3(kWcBlock), 0,
                       (hipStream_t)stream, a, scan_grid);
    return hip_status(hipGetLastError());
}

int launch_wc_compact(const WcArgs &a, uint64_t *keys, uint64_t *counts, uint64_t cap,
                      void *stream)
{
    const uint64_t grid = (a.mask + kWcCompact) / kWcCompact;
    if (grid > 0x7fffffffull)
        return SPARKCL_EINVAL;
    hipLaunchKernelGGL(k_wc_compact, dim3((uint32_t)grid), dim3(kWcBlock), 0,
                       (hipStream_t)stream, a, keys, counts, cap);
    return hip_status(hipGetLastError());
}

int launch_wordcount_locate(const WlArgs &l, uint32_t scan_grid, void *stream)
{
    if (scan_grid == 0 || !l.offsets || !l.table || !l.ctl || l.nkeys == 0 || !l.keys ||
        l.nkeys > 0xFFFFFFFFull || 3 * l.nkeys > 2 * l.slots ||
        l.span == 0 || l.span % 16 != 0 || l.span > kWlMaxSpan || (l.n != 0 && l.n < 16))
        return SPARKCL_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const dim3 keys((uint32_t)((l.nkeys + kBlock - 1) / kBlock));
    hipLaunchKernelGGL(k_wl_build, keys, dim3(kBlock), 0, s, l);
    int rc = hip_status(hipGetLastError());
    const bool few = l.nkeys <= kWlFew;
    if (rc == SPARKCL_OK && l.n != 0) {
        if (few)
            hipLaunchKernelGGL((k_wl_scan<true>), dim3(scan_grid), dim3(kWcScanBlock), 0, s, l);
        else
            hipLaunchKernelGGL((k_wl_scan<false>), dim3(scan_grid), dim3(kWcScanBlock), 0, s, l);
        rc = hip_status(hipGetLastError());
    }
    if (rc == SPARKCL_OK && (l.n == 0 || !few)) {
        hipLaunchKernelGGL(k_wl_result, keys, dim3(kBlock), 0, s, l);
        rc = hip_status(hipGetLastError());
    }
    return rc;
}

int launch_tree(const TreeArgs &a, uint32_t combiner, void *stream)
{
    if (a.len == 0 || a.count == 0 || a.chunk == 0 ||
        (combiner != SPARKCL_VADD && combiner != SPARKCL_VMAX))
        return SPARKCL_EINVAL;
    const uint32_t nchunks = (uint32_t)(((uint64_t)a.count + a.chunk - 1) / a.chunk);
    if (nchunks > 1 && (a.chunk & (a.chunk - 1)))
        return SPARKCL_EINVAL;
    const bool add = combiner == SPARKCL_VADD;
    hipStream_t s = (hipStream_t)stream;
    if (a.groups != 0) {
        const uint64_t ncol = a.len < 4 ? a.len : (a.len + 3) / 4;
        const uint64_t tiles = a.cols ? (ncol + a.cols - 1) / a.cols : 0;
        if (tiles == 0 || tiles > 65535 || (a.groups & (a.groups - 1)) || a.chunk % a.groups ||
            ((a.chunk / a.groups) & (a.chunk / a.groups - 1)) ||
            a.chunk / a.groups > kTreeFlatPer ||
            (uint64_t)a.cols * a.groups > a.threads || a.threads > kTreeFlatThreads || a.threads % 64)
            return SPARKCL_EINVAL;
        const dim3 grid(nchunks, (uint32_t)tiles), block(a.threads);
        const bool nt = a.len >= 4 && a.len * a.count * 4 > kTreeCached;
#define SPARKCL_FLAT_AS(V, COMB, NT)                                           \
    do {                                                                       \
        if (a.ptrs)                                                            \
            hipLaunchKernelGGL((k_tree_flat<V, COMB, NT, true>), grid, block, 0, s, a); \
        else                                                                   \
            hipLaunchKernelGGL((k_tree_flat<V, COMB, NT, false>), grid, block, 0, s, a); \
    } while (0)
#define SPARKCL_FLAT(V, NT)                                                    \
    do {                                                                       \
        if (add)                                                               \
            SPARKCL_FLAT_AS(V, SPARKCL_VADD, NT);                              \
        else                                                                   \
            SPARKCL_FLAT_AS(V, SPARKCL_VMAX, NT);                              \
    } while (0)
        if (a.len < 4)
            SPARKCL_FLAT(1, false);
        else if (nt)
            SPARKCL_FLAT(4, true);
        else
            SPARKCL_FLAT(4, false);
#undef SPARKCL_FLAT
#undef SPARKCL_FLAT_AS
        return hip_status(hipGetLastError());
    }
    if (a.len < 4 || a.chunk > (1u << (kTreeSlots - 1)) || nchunks > 65535)
        return SPARKCL_EINVAL;
    if (a.cpt != 1) {
        if ((a.cpt != 2 && a.cpt != 4) || a.chunk > kTreeWideChunk ||
            (a.threads != (uint32_t)kBlock && !(a.threads == kTreeWideBig && a.cpt == 4)))
            return SPARKCL_EINVAL;
        const uint64_t per_block = (uint64_t)a.threads * a.cpt;
        const uint64_t cb = ((a.len + 3) / 4 + per_block - 1) / per_block;
        if (cb > 0x7fffffffull)
            return SPARKCL_EINVAL;
        const dim3 grid((uint32_t)cb, nchunks);
        const dim3 block(a.threads);
        if (add) {
            if (a.threads == kTreeWideBig)
                hipLaunchKernelGGL((k_tree_wide<SPARKCL_VADD, 4, kTreeWideBig>), grid, block, 0, s, a);
            else if (a.cpt == 4)
                hipLaunchKernelGGL((k_tree_wide<SPARKCL_VADD, 4, kBlock>), grid, block, 0, s, a);
            else
                hipLaunchKernelGGL((k_tree_wide<SPARKCL_VADD, 2, kBlock>), grid, block, 0, s, a);
        } else {
            if (a.threads == kTreeWideBig)
                hipLaunchKernelGGL((k_tree_wide<SPARKCL_VMAX, 4, kTreeWideBig>), grid, block, 0, s, a);
            else if (a.cpt == 4)
                hipLaunchKernelGGL((k_tree_wide<SPARKCL_VMAX, 4, kBlock>), grid, block, 0, s, a);
            else
                hipLaunchKernelGGL((k_tree_wide<SPARKCL_VMAX, 2, kBlock>), grid, block, 0, s, a);
        }
        return hip_status(hipGetLastError());
    }
    const uint64_t colblocks = ((a.len + 3) / 4 + kBlock - 1) / kBlock;
    if (colblocks > 0x7fffffffull)
        return SPARKCL_EINVAL;
    const dim3 grid((uint32_t)colblocks, nchunks);
    if (add)
        hipLaunchKernelGGL((k_tree<SPARKCL_VADD>), grid, dim3(kBlock), 0, s, a);
    else
        hipLaunchKernelGGL((k_tree<SPARKCL_VMAX>), grid, dim3(kBlock), 0, s, a);
    return hip_status(hipGetLastError());
}

int launch_zero(void *p, uint64_t bytes, void *stream)
{
    if (bytes % 4 != 0 || ((uintptr_t)p & 3u))
        return SPARKCL_EINVAL;
    const uint64_t words = bytes / 4;
    if (words == 0)
        return SPARKCL_OK;
    uint64_t grid = (words / 4 + kBlock) / kBlock;
    if (grid > 4096)
        grid = 4096;
    hipLaunchKernelGGL(k_zero, dim3((uint32_t)grid), dim3(kBlock), 0,
                       (hipStream_t)stream, (uint32_t *)p, words);
    return hip_status(hipGetLastError());
}

int launch_fill_pattern(float *p, uint64_t n, uint32_t salt, void *stream)
{
    if (n == 0)
        return SPARKCL_OK;
    uint64_t grid = (n + kBlock - 1) / kBlock;
    if (grid > 8192)
        grid = 8192;
    hipLaunchKernelGGL(k_fill_pattern, dim3((uint32_t)grid), dim3(kBlock), 0,
                       (hipStream_t)stream, p, n, salt);
    return hip_status(hipGetLastError());
}

int launch_serve(const ServeArgs &a, uint32_t workers, void *stream)
{
    if (workers == 0 || a.cap == 0 || (a.cap & (a.cap - 1)) || a.tile_cap == 0 ||
        (a.tile_cap & (a.tile_cap - 1)))
        return SPARKCL_EINVAL;
    hipLaunchKernelGGL(k_serve_prologue, dim3(1), dim3(64), 0, (hipStream_t)stream, a.dev);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return hip_status(e);
    hipLaunchKernelGGL(k_serve, dim3(workers + 1), dim3(kBlock), 0, (hipStream_t)stream, a);
    return hip_status(hipGetLastError());
}

int batch_blocks_per_cu(int *out)
{
    return hip_status(hipOccupancyMaxActiveBlocksPerMultiprocessor(
        out, reinterpret_cast<const void *>(k_batch), kBlock, 0));
}

int batch_mc_blocks_per_cu(int *out)
{
    return hip_status(hipOccupancyMaxActiveBlocksPerMultiprocessor(
        out, reinterpret_cast<const void *>(k_batch_mc), kBlock, 0));
}

int chain_blocks_per_cu(int *out)
{
    return hip_status(hipOccupancyMaxActiveBlocksPerMultiprocessor(
        out, reinterpret_cast<const void *>(k_chain<4>), kBlock, 0));
}

} // namespace sparkcl
