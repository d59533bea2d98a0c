// corey_entropy_hist: fixed-bin histogram entropy (Eq. 1) and r = H / log K on gfx950.
//
// Three sweeps, as the paper's estimation protocol states them (a min/max pass, a bin-count pass, an
// O(K) reduction):
//   k_entropy_init      clears the partial counts and the range keys (a kernel, not a memset, so a caller may
//                       capture it); only the general path needs it
//   k_entropy_range     lo/hi per histogram: 16-byte loads, wave + workgroup reduction, one pair of integer
//                       atomics per workgroup on order-preserving keys
//   k_entropy_count     bin index per value in binary32 (subtract, multiply, truncate: the ABI's definition),
//                       counts privatised in LDS (several copies per workgroup) and merged with integer atomics, so the
//                       result is exact and independent of scheduling
//                       (merged into kParts partial histograms in the workspace, so that the merging atomics
//                       of many workgroups do not all queue on the same few cache lines)
//   k_entropy_finalise  sums the partial histograms into counts, then p_k, H = -sum p log(p + eps) and r in
//                       double, one workgroup per histogram
// Few values take one launch, k_entropy_small: range, counts and reduction of a histogram in one workgroup.
// The common calls (one histogram over the whole tensor, aligned, every value or every stride-th block of a
// power-of-two number of 16-byte words; a histogram per sequence, rows starting at words) take the *_flat kernels: the range sweep leaves one partial range per
// workgroup (no atomics, so nothing has to be cleared first; it also clears the partial counts), the count sweep
// starts by reducing those partials, and only the sampled 16-byte words are fetched at all.  When the producer of the
// tensor hands over its partial ranges (and, beside them, partial histograms it cleared) the statistic is ONE launch,
// the count sweep, plus the reduction; the reduction leaves those partial histograms cleared for the next call.  The
// reduction itself (corey_finalise.h) can also be left to a routed scan (corey_route_device_deferred).
// All of it is bandwidth work: no matrix instructions.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <mutex>

#include "corey_finalise.h"
#include "corey_internal.h"
#include "corey_range.h"

namespace {

using corey::bf16_to_f32;

using corey_range::kThreads;
using corey_range::key_value;
using corey_range::order_key;
using corey_range::Handoff;
using corey_range::RangePart;
using corey_range::RangeSlot;
using corey_range::RangeFold;
using corey_range::usable_range;
using corey_range::word4;
using corey_range::reduce_range_keys;
constexpr int kVecBytes = 16;
using corey_range::kParts;     // partial histograms per histogram in the workspace
constexpr int kMaxBlocks = COREY_RANGE_PARTS;  // most workgroups per sweep (four per compute unit) and partial ranges kept
// Most histograms of the per-sequence flat sweeps: 16 workgroups of the 1024 for each.  64 histograms of 49152 to 3 million values take 27 to
// 96 % of the general kernels' time; so would 65 to 128 (21 to 96 %; bf16, 96 of 512 x 1024: 172 us there, 42 in sweeps), beyond which a
// histogram would have fewer than the eight workgroups the general kernels give it.
constexpr int kMostRowHistograms = 64;
constexpr int kFlatBlocks = 512;               // workgroups of a flat sweep: two per compute unit measured 4 % (exact) to
                                               // 11 % (sampled) faster than four (fewer LDS clears, merges and range folds)

template <typename T> struct Elem;
template <> struct Elem<float> {
    static constexpr int kVec = 4;
    static __device__ __forceinline__ float widen(float v) { return v; }
};
template <> struct Elem<uint16_t> {                       // bfloat16 bit patterns
    static constexpr int kVec = 8;
    static __device__ __forceinline__ float widen(uint16_t v) { return bf16_to_f32(v); }
    static __device__ __forceinline__ void widen2(uint32_t w, float& a, float& b)
    {
        a = __uint_as_float(w << 16);
        b = __uint_as_float(w & 0xffff0000u);
    }
};
template <> struct Elem<_Float16> {                       // IEEE binary16
    static constexpr int kVec = 8;
    static __device__ __forceinline__ float widen(_Float16 v) { return (float)v; }
    static __device__ __forceinline__ void widen2(uint32_t w, float& a, float& b)
    {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        h2 h;
        __builtin_memcpy(&h, &w, 4);
        a = (float)h.x;
        b = (float)h.y;
    }
};

// Geometry of one histogram: `rows` rows of `len` valid values, `row_stride` apart, starting at `base`.
struct Geometry {
    int64_t base, rows, len, row_stride;
};

__device__ __forceinline__ Geometry geometry(int h, int64_t B, int64_t D, int64_t L, const int32_t* seqlens)
{
    Geometry g;
    if (seqlens) {
        int64_t len = seqlens[h];
        len = len < 0 ? 0 : (len > L ? L : len);
        g.base = (int64_t)h * D * L;
        g.rows = D;
        g.len = len;
    } else {
        g.base = 0;
        g.rows = B * D;
        g.len = L;
    }
    g.row_stride = L;
    return g;
}

constexpr int kUnroll = 4;   // 16-byte loads a thread keeps in flight

// Which of the values numbered idx, idx + 1, ... (memory order within one histogram) are sampled: every stride-th
// block of `block` consecutive values.
struct SamplePhase {
    int64_t pos, bph, block, stride;
    __device__ __forceinline__ SamplePhase(int64_t idx, int64_t block_, int64_t stride_) : block(block_), stride(stride_)
    {
        if (((block & (block - 1)) | (stride & (stride - 1))) == 0) {   // powers of two (uniform): no division
            const int lb = 63 - __clzll((long long)block);
            pos = idx & (block - 1);
            bph = (idx >> lb) & (stride - 1);
        } else {
            const int64_t blk = idx / block;
            pos = idx - blk * block;
            bph = blk % stride;
        }
    }
    __device__ __forceinline__ bool take_and_advance()
    {
        const bool take = bph == 0;
        if (++pos == block) {
            pos = 0;
            if (++bph == stride) bph = 0;
        }
        return take;
    }
};

// Visit every sampled value of histogram `h` once: f(value).  A row is cut into slabs of kThreads 16-byte vectors
// (one vector per thread); a workgroup takes kUnroll consecutive slabs at a time, grid-stride, whichever rows they
// fall in (short rows: several rows per turn), and loads all of them before any is consumed so that enough bytes
// are in flight to cover HBM latency.  The (row, slab) cursor is stepped, never divided, inside the loop.
// `vector_ok` says rows are 16-byte aligned (pointer and L); otherwise, and in the ragged last slab of a row,
// values are fetched one by one where no whole vector fits.
// Apply a per-value function to the values of one 16-byte vector.
template <typename T, typename F>
__device__ __forceinline__ void each_of_vector(const uint32_t __attribute__((ext_vector_type(4)))& raw, F&& f)
{
    T v[Elem<T>::kVec];
    __builtin_memcpy(v, &raw, kVecBytes);
#pragma unroll
    for (int e = 0; e < Elem<T>::kVec; ++e) f(Elem<T>::widen(v[e]));
}

// The grid is sized on the host from L; the valid lengths are only known here.  active_groups says how many of the
// launched workgroups a histogram keeps busy (about kTurns turns each): the others leave at once instead of paying a
// workgroup's fixed costs (clearing and merging the LDS counters) for a sliver of data.
constexpr int kTurns = 2;
template <typename T>
__device__ __forceinline__ int64_t active_groups(const Geometry& g)
{
    constexpr int64_t kSlab = (int64_t)kThreads * Elem<T>::kVec;
    const int64_t nslab = g.rows * ((g.len + kSlab - 1) / kSlab);
    const int64_t n = (nslab + kUnroll * kTurns - 1) / (kUnroll * kTurns);
    return n < 1 ? 1 : (n > (int64_t)gridDim.x ? (int64_t)gridDim.x : n);
}

// `fv` takes a whole 16-byte vector of values that are all used (stride 1); `f` one value.
template <typename T, typename F, typename FV>
__device__ __forceinline__ void for_each_value(const T* x, const Geometry& g, int64_t stride, int64_t block, bool vector_ok,
                                               int64_t nwg, F&& f, FV&& fv)
{
    constexpr int V = Elem<T>::kVec;
    constexpr int64_t kSlab = (int64_t)kThreads * V;
    typedef uint32_t vec4 __attribute__((ext_vector_type(4)));
    if (g.len == 0) return;
    const bool all = stride == 1;
    const int64_t spr = (g.len + kSlab - 1) / kSlab;           // slabs per row
    const int64_t nslab = g.rows * spr;
    const int64_t step = nwg * kUnroll;                         // nwg workgroups (blockIdx.x < nwg) share the histogram
    const int64_t step_r = step / spr, step_o = step - step_r * spr;
    int64_t s = (int64_t)blockIdx.x * kUnroll;
    int64_t r = s / spr, o = s - r * spr;                       // row and slab within the row of slab s
    const int64_t tid_off = (int64_t)threadIdx.x * V;
    // sampling in power-of-two blocks of whole vectors, every power-of-two-th block, rows of whole vectors
    const bool vec_blocks = !all && ((block & (block - 1)) | (stride & (stride - 1))) == 0 && block % V == 0 && g.len % V == 0;
    const int block_log2 = 63 - __clzll((long long)block);
    for (; s < nslab; s += step) {                              // everything about the cursor is uniform
        int64_t row_k[kUnroll], t0_k[kUnroll];
        int nk = 0;
        bool fast = vector_ok;
        {
            int64_t rk = r, ok = o;
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) {
                row_k[k] = rk;
                t0_k[k] = ok * kSlab;
                if (s + k < nslab) {
                    ++nk;
                    fast = fast && (t0_k[k] + kSlab <= g.len);
                }
                if (++ok == spr) {
                    ok = 0;
                    ++rk;
                }
            }
        }
        if (fast && nk == kUnroll && vec_blocks) {              // whole slabs, sampled in blocks of whole vectors:
            vec4 raw[kUnroll];                                  // a vector is used or skipped (not even fetched) as one
            bool take[kUnroll];
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) {
                const int64_t idx = row_k[k] * g.len + t0_k[k] + tid_off;
                take[k] = ((idx >> block_log2) & (stride - 1)) == 0;
                if (take[k]) raw[k] = *reinterpret_cast<const vec4*>(x + g.base + row_k[k] * g.row_stride + t0_k[k] + tid_off);
            }
#pragma unroll
            for (int k = 0; k < kUnroll; ++k)
                if (take[k]) fv(raw[k]);
        } else if (fast && nk == kUnroll) {                     // kUnroll whole slabs
            vec4 raw[kUnroll];
#pragma unroll
            for (int k = 0; k < kUnroll; ++k)
                raw[k] = *reinterpret_cast<const vec4*>(x + g.base + row_k[k] * g.row_stride + t0_k[k] + tid_off);
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) {
                if (all) {
                    fv(raw[k]);
                    continue;
                }
                T v[V];
                __builtin_memcpy(v, &raw[k], kVecBytes);
                {
                    SamplePhase ph(row_k[k] * g.len + t0_k[k] + tid_off, block, stride);   // index of v[0] in memory order
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        if (ph.take_and_advance()) f(Elem<T>::widen(v[e]));
                }
            }
        } else if (vector_ok) {                                 // a ragged slab among them, or the last turn: every thread
            vec4 raw[kUnroll];                                  // still fetches its whole vectors before it uses any
            int nvalid[kUnroll];
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) {
                const int64_t left = g.len - (t0_k[k] + tid_off);
                nvalid[k] = (k < nk && left > 0) ? (left < V ? (int)left : V) : 0;
                if (nvalid[k] == V)
                    raw[k] = *reinterpret_cast<const vec4*>(x + g.base + row_k[k] * g.row_stride + t0_k[k] + tid_off);
            }
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) {
                if (nvalid[k] == 0) continue;
                const int64_t t0 = t0_k[k] + tid_off;
                const T* row = x + g.base + row_k[k] * g.row_stride;
                if (nvalid[k] == V) {
                    if (all) {
                        fv(raw[k]);
                    } else {
                        T v[V];
                        __builtin_memcpy(v, &raw[k], kVecBytes);
                        SamplePhase ph(row_k[k] * g.len + t0, block, stride);
#pragma unroll
                        for (int e = 0; e < V; ++e)
                            if (ph.take_and_advance()) f(Elem<T>::widen(v[e]));
                    }
                } else if (all) {                              // the thread that straddles the end of the row
                    for (int e = 0; e < nvalid[k]; ++e) f(Elem<T>::widen(row[t0 + e]));
                } else {
                    SamplePhase ph(row_k[k] * g.len + t0, block, stride);
                    for (int e = 0; e < nvalid[k]; ++e)
                        if (ph.take_and_advance()) f(Elem<T>::widen(row[t0 + e]));
                }
            }
        } else {                                                // unaligned rows: value by value
            for (int k = 0; k < nk; ++k) {
                const T* row = x + g.base + row_k[k] * g.row_stride;
                const int64_t t0 = t0_k[k] + tid_off;
                if (t0 >= g.len) continue;
                const int nv = (g.len - t0 < V) ? (int)(g.len - t0) : V;
                if (all) {
                    for (int e = 0; e < nv; ++e) f(Elem<T>::widen(row[t0 + e]));
                } else {
                    SamplePhase ph(row_k[k] * g.len + t0, block, stride);
                    for (int e = 0; e < nv; ++e)
                        if (ph.take_and_advance()) f(Elem<T>::widen(row[t0 + e]));
                }
            }
        }
        r += step_r;
        o += step_o;
        if (o >= spr) {
            o -= spr;
            ++r;
        }
    }
}

// Range slots of the general sweeps: every histogram has kSubSlots of them and a workgroup publishes into slot
// blockIdx.x % kSubSlots (a thousand workgroups that finish together would otherwise queue their atomics on one
// address: that queue, not the data, set the time of the range sweep); the count sweep folds them.
constexpr int kSubSlots = 32;

__global__ __launch_bounds__(kThreads) void k_entropy_init(uint32_t* parts, int64_t nparts, RangeSlot* slots, int nh, RangeSlot* subs)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const RangeSlot empty = {0xffffffffu, 0u, 0u, 0u};
    if (i < nparts) parts[i] = 0u;
    if (i < nh) slots[i] = empty;
    if (i < (int64_t)nh * kSubSlots) subs[i] = empty;
}

// ... and the integer atomics that publish it.  The slot is read first and an atomic is issued only if it
// would change it: extremes only move one way, so a stale read can cost a redundant atomic but never lose an
// update, and almost all workgroups skip the contended atomics.
__device__ __forceinline__ void publish_range(float lo, float hi, bool nan, RangeSlot* slot)
{
    uint32_t klo = (lo <= hi) ? order_key(lo) : 0xffffffffu;
    uint32_t khi = (lo <= hi) ? order_key(hi) : 0u;
    uint32_t knan = nan ? 1u : 0u;
    reduce_range_keys(klo, khi, knan);
    if (threadIdx.x == 0) {
        if (klo < __atomic_load_n(&slot->lo_key, __ATOMIC_RELAXED)) atomicMin(&slot->lo_key, klo);
        if (khi > __atomic_load_n(&slot->hi_key, __ATOMIC_RELAXED)) atomicMax(&slot->hi_key, khi);
        if (knan) atomicOr(&slot->saw_nan, 1u);
    }
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_entropy_range(const T* __restrict__ x, int64_t B, int64_t D, int64_t L,
                                                            const int32_t* __restrict__ seqlens, int64_t stride, int64_t block,
                                                            int vector_ok, RangeSlot* subs)
{
    const int h = blockIdx.y;
    const Geometry g = geometry(h, B, D, L, seqlens);
    const int64_t nwg = active_groups<T>(g);
    if ((int64_t)blockIdx.x >= nwg) return;                     // uniform
    float lo = INFINITY, hi = -INFINITY;
    uint32_t mag = 0u;                                          // whole vectors: NaN is read off the largest magnitude pattern
    bool nan = false;
    for_each_value(
        x, g, stride, block, vector_ok != 0, nwg,
        [&](float v) {
            nan |= (v != v);
            lo = fminf(lo, v);       // fminf/fmaxf drop a NaN operand; NaNs are flagged separately
            hi = fmaxf(hi, v);
        },
        [&](const word4& q) { RangeFold<T>::fold(q, lo, hi, mag); });
    nan |= RangeFold<T>::saw_nan(mag);
    publish_range(lo, hi, nan, &subs[h * kSubSlots + blockIdx.x % kSubSlots]);
}

// ---------------------------------------------------------------------------------------------------------
// The common calls: the values are a flat array of 16-byte words; a workgroup walks it grid-stride with kUnroll loads in
// flight per lane and little but straight-line code in between.

// The 16-byte words of a flat sweep, numbered consecutively.  kAll: the tensor's words.  kSampled: the tensor is cut into blocks of
// 2^bw_log2 words and every stride-th block is used.  kRows: histogram h is the valid part of sequence h, D rows of seqlens[h]
// values; rows start at words, and the last word of a row may hold values beyond the valid ones (`rem` of it are valid, 0: all).
enum Mode { kAll, kSampled, kRows };
struct Words {
    int64_t nwords, stride;     // kAll, kSampled
    const int32_t* seqlens;     // kRows
    int64_t D, L;
    int bw_log2;
};
template <typename T, int MODE> struct WordMap {
    static constexpr int V = Elem<T>::kVec;
    int64_t nwords, stride, base;
    int bw_log2, rem;
    uint32_t wpr, row_words, magic;
    __device__ __forceinline__ WordMap(const Words& w, int h) : nwords(w.nwords), stride(w.stride), base(0), bw_log2(w.bw_log2), rem(0)
    {
        if constexpr (MODE == kRows) {
            int64_t len = w.seqlens[h];
            len = len < 0 ? 0 : (len > w.L ? w.L : len);
            rem = (int)(len % V);
            wpr = (uint32_t)((len + V - 1) / V);
            row_words = (uint32_t)(w.L / V);
            nwords = w.D * (int64_t)wpr;
            base = (int64_t)h * w.D * row_words;
            magic = wpr > 1 ? (uint32_t)(0xffffffffu / wpr) + 1u : 0u;       // ceil(2^32 / wpr) or one more
        }
    }
    // (kRows: the host keeps the words of a histogram below 2^31; the quotient by the rounded-up reciprocal is then right or one
    // too large)
    __device__ __forceinline__ int64_t operator()(int64_t i) const
    {
        if constexpr (MODE == kSampled) {
            const int64_t sb = i >> bw_log2;
            return ((sb * stride) << bw_log2) + (i - (sb << bw_log2));
        } else if constexpr (MODE == kRows) {
            const uint32_t n = (uint32_t)i;
            uint32_t r = wpr > 1 ? __umulhi(n, magic) : n;
            r -= r * wpr > n ? 1u : 0u;
            return base + (int64_t)r * row_words + (n - r * wpr);
        } else {
            return i;
        }
    }
    // valid values of word i
    __device__ __forceinline__ int valid(int64_t i) const
    {
        if constexpr (MODE != kRows) return V;
        if (rem == 0) return V;                                // uniform
        const uint32_t n = (uint32_t)i + 1u;
        uint32_t r = wpr > 1 ? __umulhi(n, magic) : n;
        r -= r * wpr > n ? 1u : 0u;
        return r * wpr == n ? rem : V;                          // the next word starts a row
    }
};

// The first `valid` values of a word, the others replaced by the first one (for a range).
template <typename T> __device__ __forceinline__ word4 only_valid(word4 q, int valid)
{
    const uint32_t first = sizeof(T) == 2 ? (q.x & 0xffffu) * 0x10001u : q.x;
    constexpr int PER = sizeof(T) == 2 ? 2 : 1;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t keep = valid >= PER * (k + 1) ? 0xffffffffu : (valid <= PER * k ? 0u : 0xffffu);
        q[k] = (q[k] & keep) | (first & ~keep);
    }
    return q;
}

// Bound by memory.  Histogram blockIdx.y, one partial range per workgroup, no atomics.  A padded batch of two (8192 and 2048 of 8192
// steps, 4096 channels, bf16, 84 MB valid) by the general kernels (a row cursor, ranges published by atomics, a launch that clears
// their slots): 31.7 us and 4.8 for the clearing, the counts 23.0; as rows of words 21.1 and 18.5 (4.0 and 4.5 TB/s), the step with
// its scan 226.5 -> 208.6.
template <typename T, int MODE>
__global__ __launch_bounds__(kThreads) void k_entropy_range_flat(const word4* __restrict__ x, const Words words,
                                                                 RangePart* __restrict__ rparts, uint32_t* __restrict__ parts,
                                                                 int64_t nparts)
{
    // the partial counts the next sweep adds into
    for (int64_t i = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kThreads + threadIdx.x; i < nparts;
         i += (int64_t)gridDim.y * gridDim.x * kThreads)
        parts[i] = 0u;
    const WordMap<T, MODE> map(words, blockIdx.y);
    const int64_t nwords = map.nwords;
    float lo = INFINITY, hi = -INFINITY;
    uint32_t mag = 0u;
    const int64_t step = (int64_t)gridDim.x * kThreads * kUnroll;
    int64_t base = (int64_t)blockIdx.x * kThreads * kUnroll;
    auto fold = [&](const word4& q, int64_t i) {
        if (MODE == kRows && map.rem != 0) RangeFold<T>::fold(only_valid<T>(q, map.valid(i)), lo, hi, mag);
        else RangeFold<T>::fold(q, lo, hi, mag);
    };
    for (; base + kThreads * kUnroll <= nwords; base += step) {
        word4 q[kUnroll];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) q[k] = x[map(base + k * kThreads + threadIdx.x)];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) fold(q[k], base + k * kThreads + threadIdx.x);
    }
    if (base < nwords) {                                      // ragged end: at most one workgroup, one trip to memory
        word4 q[kUnroll];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            const int64_t i = base + k * kThreads + threadIdx.x;
            if (i < nwords) q[k] = x[map(i)];
        }
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            const int64_t i = base + k * kThreads + threadIdx.x;
            if (i < nwords) fold(q[k], i);
        }
    }
    uint32_t klo = (lo <= hi) ? order_key(lo) : 0xffffffffu;
    uint32_t khi = (lo <= hi) ? order_key(hi) : 0u;
    uint32_t knan = RangeFold<T>::saw_nan(mag) ? 1u : 0u;
    reduce_range_keys(klo, khi, knan);
    if (threadIdx.x == 0) {
        RangePart rp;
        rp.lo_key = klo; rp.hi_key = khi; rp.saw_nan = knan; rp.pad = 0u;
        rparts[blockIdx.y * gridDim.x + blockIdx.x] = rp;
    }
}

constexpr int kMaxLdsBins = 8192;   // uint32 counters in LDS (32 KiB)

// Private copies of the K counters a workgroup keeps in LDS: a power of two below what fits, 32 at most.  The copies of one bin
// are neighbours (word bin * copies + copy, a lane's copy being its number modulo the copies): with 32 of them a lane's
// counters all sit in a bank of the lane's own, so the adds of a wave never queue on a bank whatever the bins; with fewer,
// lanes of different copies still never meet.  (Copies K + 1 words apart met by chance: 33.5 million values at K = 1024 34.3 us
// against 33.1; at K = 256, where the sweep is bound by memory, 31.3 against 31.1.)  Where only two fit, one: clearing and adding up
// the second costs what its fewer meetings give back (K = 4096, two and one: 64 x 256 values 27.2 and 25.8 us for the statistic,
// 33.5 million 44.8 and 44.6; K = 2500, where three fit, 33.5 million: two 40.0, one 40.6).
template <int NT = kThreads> struct LdsBins {
    uint32_t* s;
    int log2;                                                   // copies = 1 << log2
    uint32_t lane_byte, shift;
    __device__ __forceinline__ LdsBins(uint32_t* s_bins, int K) : s(s_bins)
    {
        const int fit = kMaxLdsBins / K;
        log2 = fit < 3 ? 0 : min(5, 31 - __clz(fit));
        lane_byte = (threadIdx.x & ((1u << log2) - 1u)) * 4u;
        shift = (uint32_t)log2 + 2u;
    }
    __device__ __forceinline__ void clear(int K) const
    {
        for (int i = threadIdx.x; i < ((K << log2) + 3) / 4; i += NT) reinterpret_cast<word4*>(s)[i] = word4{0u, 0u, 0u, 0u};
    }
    __device__ __forceinline__ void add(uint32_t k, uint32_t n = 1u) const
    {
        atomicAdd(reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(s) + ((k << shift) + lane_byte)), n);
    }
    // the copies of bin k; neighbouring lanes start at different words, so that their reads spread over the banks
    __device__ __forceinline__ uint32_t total(int k) const
    {
        uint32_t c = 0;
        if (log2 >= 2) {
            const int quads = 1 << (log2 - 2);
            const word4* q = reinterpret_cast<const word4*>(s) + k * quads;
            for (int w = 0; w < quads; ++w) {
                const word4 v = q[(w + k) & (quads - 1)];
                c += (v.x + v.y) + (v.z + v.w);
            }
        } else {
            for (int w = 0; w < (1 << log2); ++w) c += s[(k << log2) + w];
        }
        return c;
    }
};

template <typename T>
__global__ __launch_bounds__(kThreads) void k_entropy_count(const T* __restrict__ x, int64_t B, int64_t D, int64_t L,
                                                            const int32_t* __restrict__ seqlens, int64_t stride, int64_t block,
                                                            int vector_ok, int K, const RangeSlot* __restrict__ subs,
                                                            RangeSlot* __restrict__ slots, uint32_t* parts)
{
    __shared__ __align__(16) uint32_t s_bins[kMaxLdsBins];
    __shared__ RangeSlot s_slot;
    const int h = blockIdx.y;
    const Geometry g = geometry(h, B, D, L, seqlens);
    const int64_t nwg = active_groups<T>(g);
    if ((int64_t)blockIdx.x >= nwg) return;                     // uniform; workgroup 0 always stays
    {   // the range: every workgroup folds the histogram's sub-slots (half a KB from L2)
        uint32_t klo = 0xffffffffu, khi = 0u, knan = 0u;
        if (threadIdx.x < kSubSlots) {
            const RangeSlot rs = subs[h * kSubSlots + threadIdx.x];
            klo = rs.lo_key;
            khi = rs.hi_key;
            knan = rs.saw_nan;
        }
        reduce_range_keys(klo, khi, knan);
        if (threadIdx.x == 0) {
            s_slot.lo_key = klo; s_slot.hi_key = khi; s_slot.saw_nan = knan; s_slot.pad = 0u;
            if (blockIdx.x == 0) slots[h] = s_slot;           // for the reduction kernel
        }
        __syncthreads();
    }
    float lo, hi;
    if (!usable_range(s_slot, &lo, &hi)) return;              // counts stay zero, H and r become NaN
    const LdsBins<> bins(s_bins, K);
    bins.clear(K);
    __syncthreads();

    if (hi == lo) {
        uint32_t n = 0;
        for_each_value(x, g, stride, block, vector_ok != 0, nwg, [&](float) { ++n; },
                       [&](const word4&) { n += Elem<T>::kVec; });
        if (n) bins.add(0u, n);
    } else {
        const float scale = (float)((double)K / ((double)hi - (double)lo));
        const int top = K - 1;
        auto bin = [&](float v) {
            const float q = __fmul_rn(__fsub_rn(v, lo), scale);   // two separate binary32 roundings
            int k = (int)q;                                        // truncation; q >= 0
            k = k > top ? top : (k < 0 ? 0 : k);
            bins.add((uint32_t)k);
        };
        for_each_value(x, g, stride, block, vector_ok != 0, nwg, bin, [&](const word4& q) { each_of_vector<T>(q, bin); });
    }
    __syncthreads();
    uint32_t* out = parts + ((int64_t)h * kParts + blockIdx.x % kParts) * K;
    for (int k = threadIdx.x; k < K; k += kThreads) {
        const uint32_t c = bins.total(k);
        if (c) atomicAdd(&out[k], c);
    }
}

// Adds values to a workgroup's counters: the bin index as the interface defines it.
template <typename T, int NT> struct Binner {
    LdsBins<NT> bins;
    float lo, scale;
    uint32_t top;
    __device__ __forceinline__ Binner(uint32_t* s_bins, int K, float lo_, float hi) : bins(s_bins, K), lo(lo_), top((uint32_t)K - 1u)
    {
        scale = hi == lo ? 0.f : (float)((double)K / ((double)hi - (double)lo));     // degenerate range: everything in bin 0
    }
    __device__ __forceinline__ void bin(float v) const
    {
        const float q = __fmul_rn(__fsub_rn(v, lo), scale);    // two separate binary32 roundings
        // truncation; q >= 0 (a degenerate range has scale 0: bin 0).  The conversion to unsigned saturates, so a value
        // outside a stale range still lands inside the counters.
        bins.add(min(__float2uint_rz(q), top));
    }
    template <bool SOME> __device__ __forceinline__ void fold(const word4& q, int valid) const      // SOME: the first `valid` values
    {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if constexpr (sizeof(T) == 2) {
                float a, b;
                Elem<T>::widen2(w[k], a, b);
                if (!SOME || 2 * k < valid) bin(a);
                if (!SOME || 2 * k + 1 < valid) bin(b);
            } else {
                if (!SOME || k < valid) bin(__uint_as_float(w[k]));
            }
        }
    }
};

template <typename T, int MODE>
__global__ __launch_bounds__(kThreads) void k_entropy_count_flat(const word4* __restrict__ x, const Words words, int K,
                                                                 const RangePart* __restrict__ rparts, int nrparts,
                                                                 RangeSlot* __restrict__ slots, uint32_t* parts)
{
    __shared__ __align__(16) uint32_t s_bins[kMaxLdsBins];
    __shared__ RangeSlot s_slot;
    const int h = blockIdx.y;
    const WordMap<T, MODE> map(words, h);
    const int64_t nwords = map.nwords;
    // A small or sampled sweep is one or two turns long: its time is trips to memory one after another.  The partial ranges (of the sweep
    // before, or of the tensor's producer: a few KB from L2) are requested in one go, the first words behind them, and the counters
    // are cleared while both are on their way; a partial turn is one trip, too.
    // (One layer, convolution to scan, bf16: 1536 channels of 2048 steps, every 8th block sampled, 39.9 -> 38.7 us; 2048 of 977, every value,
    // 35.4 -> 34.5; the larger sweeps gain 0 to 0.7 %.  The partial turn as one more form of the loop's own fetch and count, which fetched
    // it a turn ahead there too, cost the sweeps of many turns 0.4 to 0.9 %.)
    const int64_t step = (int64_t)gridDim.x * kThreads * kUnroll;
    int64_t base = (int64_t)blockIdx.x * kThreads * kUnroll;
    if (MODE == kRows && base >= nwords && blockIdx.x > 0) return;      // uniform: a sequence too short for this workgroup
    constexpr int kPartTurns = COREY_RANGE_PARTS / kThreads;
    static_assert(kPartTurns * kThreads == COREY_RANGE_PARTS && kMaxBlocks <= COREY_RANGE_PARTS, "every partial range is read");
    RangePart rp[kPartTurns];
#pragma unroll
    for (int k = 0; k < kPartTurns; ++k) rp[k] = rparts[h * nrparts + min((int)threadIdx.x + k * kThreads, nrparts - 1)];
    word4 q[kUnroll], qn[kUnroll];
    auto fetch_rest = [&] {                                   // the words of a partial turn
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            const int64_t i = base + k * kThreads + threadIdx.x;
            if (i < nwords) q[k] = x[map(i)];
        }
    };
    bool have = base + kThreads * kUnroll <= nwords;
    const bool only_rest = !have;
    if (have) {
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) q[k] = x[map(base + k * kThreads + threadIdx.x)];
    } else {
        fetch_rest();
    }
    const LdsBins<kThreads> bins(s_bins, K);
    bins.clear(K);
    uint32_t klo = 0xffffffffu, khi = 0u, knan = 0u;
#pragma unroll
    for (int k = 0; k < kPartTurns; ++k) {
        klo = min(klo, rp[k].lo_key);
        khi = max(khi, rp[k].hi_key);
        knan |= rp[k].saw_nan;
    }
    reduce_range_keys(klo, khi, knan);
    if (threadIdx.x == 0) {
        s_slot.lo_key = klo; s_slot.hi_key = khi; s_slot.saw_nan = knan; s_slot.pad = 0u;
        if (blockIdx.x == 0) slots[h] = s_slot;               // for the reduction
    }
    __syncthreads();                                          // the range; the counters are cleared
    float lo, hi;
    if (!usable_range(s_slot, &lo, &hi)) return;              // counts stay zero, H and r become NaN
    const Binner<T, kThreads> b(s_bins, K, lo, hi);
    auto fold = [&](const word4& w, int64_t i) {
        if (MODE == kRows && map.rem != 0) b.template fold<true>(w, map.valid(i));
        else b.template fold<false>(w, 0);
    };
    while (have) {                                            // the next turn's words are requested before this turn's are counted;
        int64_t at = base + threadIdx.x;
        base += step;                                         // two turns per iteration, so the two sets of registers swap roles
        have = base + kThreads * kUnroll <= nwords;           // without being copied
        if (have) {
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) qn[k] = x[map(base + k * kThreads + threadIdx.x)];
        }
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) fold(q[k], at + k * kThreads);
        if (!have) break;
        at = base + threadIdx.x;
        base += step;
        have = base + kThreads * kUnroll <= nwords;
        if (have) {
#pragma unroll
            for (int k = 0; k < kUnroll; ++k) q[k] = x[map(base + k * kThreads + threadIdx.x)];
        }
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) fold(qn[k], at + k * kThreads);
    }
    if (base < nwords) {                                      // ragged end: at most one workgroup
        if (!only_rest) fetch_rest();
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            const int64_t i = base + k * kThreads + threadIdx.x;
            if (i < nwords) fold(q[k], i);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += kThreads) {
        const uint32_t c = b.bins.total(k);
        if (c) atomicAdd(&parts[((size_t)h * kParts + blockIdx.x % kParts) * K + k], c);
    }
}

// A histogram of few words, start to end in one workgroup: its words stay in registers between the range and the counts, and
// the counts in LDS until they are reduced.  Bound by latency: one trip to memory instead of a chain of launches and their trips.
// Range, counts, reduction and rule of 64 x 256 binary32 values at K = 16: 8.8 us in three launches, 7.2 in one (with the scan 16.4 and
// 14.3 a step).  The one compute unit's counts are what grows: the line lies at 40960 values (us, three launches and one: K = 16,
// binary32, 32768 values 9.4 and 8.4, 49152 9.2 and 9.7; bf16, 32768 9.5 and 8.2, 49152 9.6 and 9.4, 65536 9.6 and 10.5; K = 256 the
// same within 0.4; K = 4096 24 and 14 at 32768, 23 and 17 at 65536).  Several histograms are counted side by side: bf16, 80 x 512 values
// each, 8 sequences 12.3 us in sweeps and 11.3 in one launch, 64 13.7 and 11.6; of 250 forms with 1 to 64 sequences the sweeps
// are faster in five, by 3 to 9 % (40960 values of binary32); from 65, where they end, the one launch takes 0.1 to 0.4 of the time.
constexpr int kSmallThreads = 1024;
constexpr int64_t kSmallValues = 40960;
template <typename T, int MODE>
__global__ __launch_bounds__(kSmallThreads) void k_entropy_small(const word4* __restrict__ x, const Words words, const corey_finalise::Args a)
{
    __shared__ __align__(16) uint32_t s_bins[kMaxLdsBins];
    __shared__ RangeSlot s_slot;
    const int h = blockIdx.x;
    const WordMap<T, MODE> map(words, h);
    const int nwords = (int)map.nwords;
    constexpr int kSmallWords = (int)(kSmallValues / Elem<T>::kVec / kSmallThreads);      // words a lane keeps at most
    static_assert((int64_t)kSmallWords * Elem<T>::kVec * kSmallThreads == kSmallValues, "whole turns of the workgroup");
    word4 q[kSmallWords];
#pragma unroll
    for (int k = 0; k < kSmallWords; ++k) {
        if (k * kSmallThreads >= nwords) break;                // uniform
        const int i = (int)threadIdx.x + k * kSmallThreads;
        if (i < nwords) q[k] = x[map(i)];
    }
    corey_finalise::Context cx(a, h, RangeSlot{});
    cx.take_log(a.K);
    const LdsBins<kSmallThreads> bins(s_bins, a.K);
    bins.clear(a.K);
    float lo = INFINITY, hi = -INFINITY;
    uint32_t mag = 0u;
#pragma unroll
    for (int k = 0; k < kSmallWords; ++k) {
        if (k * kSmallThreads >= nwords) break;
        const int i = (int)threadIdx.x + k * kSmallThreads;
        if (i >= nwords) continue;
        if (MODE == kRows && map.rem != 0) RangeFold<T>::fold(only_valid<T>(q[k], map.valid(i)), lo, hi, mag);
        else RangeFold<T>::fold(q[k], lo, hi, mag);
    }
    uint32_t klo = (lo <= hi) ? order_key(lo) : 0xffffffffu;
    uint32_t khi = (lo <= hi) ? order_key(hi) : 0u;
    uint32_t knan = RangeFold<T>::saw_nan(mag) ? 1u : 0u;
    reduce_range_keys<kSmallThreads>(klo, khi, knan);
    if (threadIdx.x == 0) {
        s_slot.lo_key = klo; s_slot.hi_key = khi; s_slot.saw_nan = knan; s_slot.pad = 0u;
    }
    __syncthreads();                                            // the range; the counters are cleared
    cx.slot = s_slot;
    const bool ok = usable_range(s_slot, &lo, &hi);             // uniform; else the counts stay zero, H and r become NaN
    if (ok) {
        const Binner<T, kSmallThreads> b(s_bins, a.K, lo, hi);
#pragma unroll
        for (int k = 0; k < kSmallWords; ++k) {
            if (k * kSmallThreads >= nwords) break;
            const int i = (int)threadIdx.x + k * kSmallThreads;
            if (i >= nwords) continue;
            if (MODE == kRows && map.rem != 0) b.template fold<true>(q[k], map.valid(i));
            else b.template fold<false>(q[k], 0);
        }
    }
    __syncthreads();
    uint32_t c[corey_finalise::kPer] = {};
#pragma unroll
    for (int i = 0; i < corey_finalise::kPer; ++i) {
        if (i * kThreads >= a.K) break;
        const int k = (int)threadIdx.x + i * kThreads;
        if (threadIdx.x < kThreads && k < a.K) c[i] = bins.total(k);
    }
    corey_finalise::reduce_counts<kSmallThreads>(a, h, true, cx, c);
}

// The O(K) reduction and the chunk rule (corey_finalise.h), one workgroup per histogram.
__global__ __launch_bounds__(kThreads) void k_entropy_finalise(const corey_finalise::Args a)
{
    corey_finalise::finalise(a, (int)blockIdx.x, true);
}

// One thread per histogram.
__global__ void k_select_chunk(const double* __restrict__ r, const int32_t* __restrict__ seqlens, int64_t L_all, int nh,
                               corey_policy p, int32_t* __restrict__ chunks)
{
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= nh) return;
    chunks[h] = corey_finalise::chunk_rule(r[h], seqlens ? (int64_t)seqlens[h] : L_all, p);
}

size_t slots_bytes(int64_t nh)
{
    const size_t raw = (size_t)nh * sizeof(RangeSlot);
    return (raw + 255) / 256 * 256;
}

size_t parts_bytes(int64_t nh, int32_t K) { return ((size_t)nh * kParts * K * sizeof(uint32_t) + 255) / 256 * 256; }

size_t workspace_bytes(int64_t nh, int32_t K)
{
    return slots_bytes(nh) + parts_bytes(nh, K) + (size_t)kMaxBlocks * sizeof(RangePart) + slots_bytes(nh * kSubSlots);
}

// Fold given partial ranges into the first sub-slot of the (single) histogram (the others stay empty).
__global__ __launch_bounds__(kThreads) void k_entropy_fold_parts(const RangePart* __restrict__ rparts, int nrparts, RangeSlot* slots)
{
    uint32_t klo = 0xffffffffu, khi = 0u, knan = 0u;
    for (int i = threadIdx.x; i < nrparts; i += kThreads) {
        const RangePart rp = rparts[i];
        klo = min(klo, rp.lo_key);
        khi = max(khi, rp.hi_key);
        knan |= rp.saw_nan;
    }
    reduce_range_keys(klo, khi, knan);
    if (threadIdx.x == 0) {
        slots[0].lo_key = klo; slots[0].hi_key = khi; slots[0].saw_nan = knan; slots[0].pad = 0u;
    }
}

// Workgroups of a flat sweep over `nwords` words.
int64_t flat_blocks(int64_t nwords, int64_t most)
{
    const int64_t blocks = (nwords + (int64_t)kThreads * kUnroll - 1) / ((int64_t)kThreads * kUnroll);
    return blocks < 1 ? 1 : (blocks > most ? most : blocks);
}

// Both sweeps of nh histograms; the largest has `most_words` words.
template <typename T, int MODE>
void launch_flat(const void* x, const Words& words, int64_t most_words, int nh, int32_t K, RangeSlot* slots, uint32_t* parts,
                 RangePart* rparts, hipStream_t stream)
{
    int64_t most = kMaxBlocks / nh;                            // partial ranges there is room for
    most = most > kFlatBlocks ? kFlatBlocks : most;
    const int64_t blocks = flat_blocks(most_words, most);
    const dim3 grid((unsigned)blocks, (unsigned)nh);
    const word4* xw = static_cast<const word4*>(x);
    k_entropy_range_flat<T, MODE><<<grid, dim3(kThreads), 0, stream>>>(xw, words, rparts, parts, (int64_t)nh * kParts * K);
    k_entropy_count_flat<T, MODE><<<grid, dim3(kThreads), 0, stream>>>(xw, words, K, rparts, (int)blocks, slots, parts);
}

// The sampled words of a tensor of `nwords` words: every stride-th block of bw of them.
Words sampled_words(int64_t nwords, int64_t bw, int64_t stride)
{
    Words w = {};
    const int64_t nb = (nwords + bw - 1) / bw;                  // blocks in the tensor (the last may be short)
    const int64_t ns = (nb + stride - 1) / stride;              // sampled blocks
    const int64_t last_first = (ns - 1) * stride * bw;          // first word of the last sampled block
    const int64_t last_words = nwords - last_first < bw ? nwords - last_first : bw;
    while (((int64_t)1 << w.bw_log2) < bw) ++w.bw_log2;
    w.nwords = (ns - 1) * bw + last_words;
    w.stride = stride;
    return w;
}

// What the caller wants done with the partial histograms once the sweeps are enqueued.
struct Tail {
    const corey_policy* pol;            // NULL: statistic only
    int32_t* chunks_out;
    double ema_lambda;
    double* ema_state;
    uint32_t* chunk_calls;
    corey_finalise::Args* defer;        // not NULL: do not launch the reduction, describe it here instead
};

template <typename T>
int launch(const void* x, int64_t B, int64_t D, int64_t L, const int32_t* seqlens, int32_t K, double eps, int64_t stride,
           int64_t block, uint32_t* counts, double* H_out, double* r_out, float* range_out, RangeSlot* slots, hipStream_t stream,
           const Tail& tail, Handoff* handoff)
{
    const int nh = seqlens ? (int)B : 1;
    uint32_t* parts = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(slots) + slots_bytes(B));
    RangePart* rparts = reinterpret_cast<RangePart*>(reinterpret_cast<char*>(parts) + parts_bytes(B, K));
    RangeSlot* subs = reinterpret_cast<RangeSlot*>(rparts + kMaxBlocks);
    const int64_t nparts = (int64_t)nh * kParts * K;
    uint32_t* final_parts = parts;                              // where the reduction finds the partial histograms
    bool rezero = false;

    constexpr int V = Elem<T>::kVec;
    const int64_t E = B * D * L;
    const bool flat_ok = !seqlens && reinterpret_cast<uintptr_t>(x) % kVecBytes == 0 && E % V == 0;
    const int64_t bw = block / V;                              // 16-byte words per sampling block
    const bool blocks_ok = flat_ok && block % V == 0 && corey::is_pow2(bw);      // sampled runs are whole 16-byte words
    // per sequence: rows of whole words, and a partial range for every workgroup
    const bool row_words = seqlens && stride == 1 && reinterpret_cast<uintptr_t>(x) % kVecBytes == 0 && L % V == 0;
    const bool rows_ok = row_words && D * (L / V) < ((int64_t)1 << 31) && nh <= kMostRowHistograms;
    Words all = {};
    all.nwords = E / V;
    corey_finalise::Args fa = {};
    fa.slots = slots; fa.counts = counts; fa.H_out = H_out; fa.r_out = r_out; fa.range_out = range_out;
    fa.chunks_out = tail.pol ? tail.chunks_out : nullptr; fa.seqlens = seqlens; fa.ema_state = tail.ema_state;
    fa.chunk_calls = tail.chunk_calls; fa.L_all = L; fa.eps = eps; fa.ema_lambda = tail.ema_lambda;
    if (tail.pol) fa.pol = *tail.pol;
    fa.K = K; fa.nh = nh;
    if (!handoff && !tail.defer && stride == 1 && (seqlens ? row_words && D * L <= kSmallValues : flat_ok && E <= kSmallValues)) {
        all.seqlens = seqlens; all.D = D; all.L = L;
        auto go = [&](auto kernel) { kernel<<<dim3((unsigned)nh), dim3(kSmallThreads), 0, stream>>>(static_cast<const word4*>(x), all, fa); };
        if (seqlens) go(k_entropy_small<T, kRows>);
        else go(k_entropy_small<T, kAll>);
        const hipError_t e = hipGetLastError();
        return e != hipSuccess ? corey::hip_fail(e, "corey_entropy_hist launch") : COREY_OK;
    }
    if (handoff && flat_ok && (stride == 1 || blocks_ok)) {
        // the producer of x left its partial ranges and cleared partial histograms beside them: one launch, the count sweep
        // (over every word, or over the words of every stride-th block), whose workgroups fold the partial ranges themselves
        const Words w = stride > 1 ? sampled_words(E / V, bw, stride) : all;
        const dim3 grid((unsigned)flat_blocks(w.nwords, kFlatBlocks));
        if (stride == 1)
            k_entropy_count_flat<T, kAll><<<grid, dim3(kThreads), 0, stream>>>(static_cast<const word4*>(x), w, K, handoff->parts,
                                                                             COREY_RANGE_PARTS, slots, handoff->counts);
        else
            k_entropy_count_flat<T, kSampled><<<grid, dim3(kThreads), 0, stream>>>(static_cast<const word4*>(x), w, K, handoff->parts,
                                                                                 COREY_RANGE_PARTS, slots, handoff->counts);
        final_parts = handoff->counts;
        rezero = true;                                          // left cleared for the next statistic on this buffer
    } else if (handoff) {
        // unaligned tensor: one workgroup folds the partial ranges into the slot, then the general count sweep
        k_entropy_init<<<dim3((unsigned)((nparts + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream>>>(parts, nparts, slots, nh, subs);
        k_entropy_fold_parts<<<dim3(1), dim3(kThreads), 0, stream>>>(handoff->parts, COREY_RANGE_PARTS, subs);
        const bool vector_ok = (reinterpret_cast<uintptr_t>(x) % kVecBytes == 0) && (L % V == 0);
        const int64_t seg = (int64_t)kThreads * V * kUnroll;
        int64_t blocks = B * D * ((L + seg - 1) / seg);
        blocks = blocks < 1 ? 1 : (blocks > kMaxBlocks ? kMaxBlocks : blocks);
        k_entropy_count<T><<<dim3((unsigned)blocks, 1), dim3(kThreads), 0, stream>>>(static_cast<const T*>(x), B, D, L, nullptr, stride,
                                                                                   block, vector_ok ? 1 : 0, K, subs, slots, parts);
    } else if (flat_ok && stride == 1) {
        launch_flat<T, kAll>(x, all, all.nwords, 1, K, slots, parts, rparts, stream);
    } else if (blocks_ok) {
        const Words w = sampled_words(E / V, bw, stride);
        launch_flat<T, kSampled>(x, w, w.nwords, 1, K, slots, parts, rparts, stream);
    } else if (rows_ok) {
        Words w = {};
        w.seqlens = seqlens; w.D = D; w.L = L;
        launch_flat<T, kRows>(x, w, D * (L / V), nh, K, slots, parts, rparts, stream);
    } else {
        k_entropy_init<<<dim3((unsigned)((nparts + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream>>>(parts, nparts, slots, nh, subs);
        const bool vector_ok = (reinterpret_cast<uintptr_t>(x) % kVecBytes == 0) && (L % V == 0);
        const int64_t rows = seqlens ? D : B * D;
        const int64_t seg = (int64_t)kThreads * V * kUnroll;
        const int64_t units = rows * ((L + seg - 1) / seg);
        // about kMaxBlocks workgroups over all histograms (each pays for clearing and merging its LDS counters), at
        // least 8 per histogram
        const int64_t cap = kMaxBlocks / nh > 8 ? kMaxBlocks / nh : 8;
        int64_t blocks = units < 1 ? 1 : units;
        if (blocks > cap) blocks = cap;
        const dim3 grid((unsigned)blocks, (unsigned)nh);
        k_entropy_range<T><<<grid, dim3(kThreads), 0, stream>>>(static_cast<const T*>(x), B, D, L, seqlens, stride, block,
                                                               vector_ok ? 1 : 0, subs);
        k_entropy_count<T><<<grid, dim3(kThreads), 0, stream>>>(static_cast<const T*>(x), B, D, L, seqlens, stride, block,
                                                               vector_ok ? 1 : 0, K, subs, slots, parts);
    }
    fa.parts = final_parts; fa.rezero = rezero ? 1 : 0;
    if (tail.defer) *tail.defer = fa;                           // the scan's call will do it
    else k_entropy_finalise<<<dim3((unsigned)nh), dim3(kThreads), 0, stream>>>(fa);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return corey::hip_fail(e, "corey_entropy_hist launch");
    return COREY_OK;
}

}  // namespace

namespace corey {

// The policy as the GPU rule will apply it: the host rule's checks (r = 0.5 is a placeholder that no mode rejects), and
// no chunk the scan cannot run (the rule's result goes straight into selective_scan_fwd's chunks_dev and into the
// chunk-distribution counters, which have a slot per power of two up to COREY_MAX_CHUNK).
int check_device_policy(const char* who, const corey_policy* p, int64_t L)
{
    using corey::fail;
    int32_t probe = 0;
    const int st = corey_select_chunk(0.5, L < 1 ? 1 : L, p, &probe);
    if (st != COREY_OK) return st;
    if (p->mode == 1 && !corey::is_pow2(p->short_chunk)) return fail(COREY_EINVAL, "%s: short_chunk = %d", who, p->short_chunk);
    const bool entropy = p->mode == 0 || p->mode == 1 || p->mode == 4;
    const bool table = p->mode == 1 || p->mode == 2;
    if ((entropy && p->c_max > COREY_MAX_CHUNK) || (table && p->short_chunk > COREY_MAX_CHUNK) ||
        (p->mode == 2 && p->long_chunk > COREY_MAX_CHUNK) || (p->mode == 3 && p->static_chunk > COREY_MAX_CHUNK) ||
        (p->mode == 4 && p->safe_chunk > COREY_MAX_CHUNK))
        return fail(COREY_EINVAL, "%s: the policy can select a chunk above %d", who, COREY_MAX_CHUNK);
    return COREY_OK;
}

int launch_finalise(const corey_finalise::Args& a, hipStream_t stream)
{
    k_entropy_finalise<<<dim3((unsigned)a.nh), dim3(kThreads), 0, stream>>>(a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "entropy reduction launch");
    return COREY_OK;
}

int launch_entropy_finalise(const uint32_t* parts, uint32_t* counts, int32_t K, double eps, const void* slot, double* H_out,
                            double* r_out, float* range_out, const corey_policy* pol, int32_t* chunks_out, int64_t L,
                            hipStream_t stream)
{
    corey_finalise::Args fa = {};
    fa.parts = const_cast<uint32_t*>(parts); fa.slots = static_cast<const RangeSlot*>(slot); fa.counts = counts; fa.H_out = H_out;
    fa.r_out = r_out; fa.range_out = range_out; fa.chunks_out = pol ? chunks_out : nullptr; fa.L_all = L; fa.eps = eps;
    if (pol) fa.pol = *pol;
    fa.K = K; fa.nh = 1;
    fa.rezero = 1;                                              // the next statistic from the same table adds into them again
    return launch_finalise(fa, stream);
}

}  // namespace corey

using corey::check_device_policy;

extern "C" int corey_select_chunk_device(const double* r_dev, const int32_t* seqlens, int64_t L, int32_t nh,
                                         const corey_policy* p, int32_t* chunks_out, void* hip_stream)
{
    using corey::fail;
    if (!r_dev || !p || !chunks_out) return fail(COREY_ENULL, "corey_select_chunk_device: r_dev, p and chunks_out are required");
    if (nh < 1) return fail(COREY_EINVAL, "corey_select_chunk_device: nh = %d < 1", nh);
    if (!seqlens && L < 1) return fail(COREY_EINVAL, "corey_select_chunk_device: L = %lld < 1", (long long)L);
    const int st = check_device_policy("corey_select_chunk_device", p, L);
    if (st != COREY_OK) return st;
    k_select_chunk<<<dim3((unsigned)((nh + 63) / 64)), dim3(64), 0, static_cast<hipStream_t>(hip_stream)>>>(r_dev, seqlens, L, nh, *p, chunks_out);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return corey::hip_fail(e, "corey_select_chunk_device launch");
    return COREY_OK;
}

extern "C" size_t corey_entropy_hist_workspace(int64_t B, int32_t K)
{
    if (B < 1 || K < 2 || K > COREY_MAX_BINS) return 0;
    return workspace_bytes(B, K);
}

namespace {

int entropy_hist_impl(const char* who, const void* x, corey_dtype dt, int64_t B, int64_t D, int64_t L, const int32_t* seqlens, int32_t K,
                      double eps, int64_t stride, int64_t block, uint32_t* counts_out, double* H_out, double* r_out, float* range_out,
                      void* workspace, size_t workspace_bytes_given, void* hip_stream, const Tail& tail, void* range_parts)
{
    using corey::fail;
    if (!x || !counts_out || !H_out || !r_out) return fail(COREY_ENULL, "%s: x, counts_out, H_out and r_out are required", who);
    if (dt != COREY_F32 && dt != COREY_BF16 && dt != COREY_F16) return fail(COREY_EINVAL, "%s: unknown dtype %d", who, (int)dt);
    if (B < 1 || D < 1 || L < 1) return fail(COREY_ESHAPE, "%s: B, D, L must be >= 1", who);
    if (B > 65535) return fail(COREY_ESHAPE, "%s: B = %lld exceeds 65535", who, (long long)B);
    if ((double)B * (double)D * (double)L >= 9.0e18) return fail(COREY_ESHAPE, "%s: B*D*L overflows", who);
    if ((double)B * (double)D * (double)L >= 4294967296.0 && stride == 1)
        return fail(COREY_ESHAPE, "%s: more than 2^32-1 samples would overflow the 32-bit counts", who);
    if (K < 2 || K > COREY_MAX_BINS) return fail(COREY_EINVAL, "%s: K = %d outside [2, %d]", who, K, COREY_MAX_BINS);
    if (!(eps >= 0.0)) return fail(COREY_EINVAL, "%s: eps must be >= 0", who);
    if (stride < 1 || block < 1) return fail(COREY_EINVAL, "%s: stride and block must be >= 1", who);
    if (range_parts && seqlens)
        return fail(COREY_EINVAL, "%s: range_parts needs the whole-tensor statistic (seqlens NULL)", who);
    if (range_parts && reinterpret_cast<uintptr_t>(range_parts) % 16 != 0) return fail(COREY_EINVAL, "%s: range_parts must be 16-byte aligned", who);
    const size_t need = workspace_bytes(B, K);
    if (!workspace || workspace_bytes_given < need) return fail(COREY_EWORKSPACE, "%s: workspace of %zu bytes required", who, need);
    if (reinterpret_cast<uintptr_t>(workspace) % 16 != 0) return fail(COREY_EWORKSPACE, "%s: workspace must be 16-byte aligned", who);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    RangeSlot* slots = static_cast<RangeSlot*>(workspace);
    Handoff* handoff = static_cast<Handoff*>(range_parts);
    if (dt == COREY_F32)
        return launch<float>(x, B, D, L, seqlens, K, eps, stride, block, counts_out, H_out, r_out, range_out, slots, stream, tail, handoff);
    if (dt == COREY_F16)
        return launch<_Float16>(x, B, D, L, seqlens, K, eps, stride, block, counts_out, H_out, r_out, range_out, slots, stream, tail, handoff);
    return launch<uint16_t>(x, B, D, L, seqlens, K, eps, stride, block, counts_out, H_out, r_out, range_out, slots, stream, tail, handoff);
}

}  // namespace

extern "C" int corey_entropy_hist(const void* x, corey_dtype dt, int64_t B, int64_t D, int64_t L, const int32_t* seqlens,
                                  int32_t K, double eps, int64_t stride, int64_t block, uint32_t* counts_out, double* H_out,
                                  double* r_out, float* range_out, void* range_parts, void* workspace,
                                  size_t workspace_bytes_given, void* hip_stream)
{
    return entropy_hist_impl("corey_entropy_hist", x, dt, B, D, L, seqlens, K, eps, stride, block, counts_out, H_out, r_out, range_out,
                             workspace, workspace_bytes_given, hip_stream, Tail{}, range_parts);
}

// ---------------------------------------------------------------------------------------------------------
// corey_entropy_hist_static: the same statistic for callers that cannot allocate (HIP graph capture, serving loops
// that may not call hipMalloc).  The workspace of corey_entropy_hist lives in an array in the GPU's global memory that is
// part of the library's code object: every GPU the library runs on holds its own copy at its own address until the
// process ends.  On the host the array's name is only a handle: the address kernels can use is asked for once per
// device (hipGetSymbolAddress, with that device current) and kept.
static __device__ __align__(256) unsigned char scratch[COREY_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};      // address of `scratch` on each device, filled on first use

// The current device's copy of `scratch` (NULL after recording the error).
void* static_scratch(const char* who)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        corey::hip_fail(e, who);
        return nullptr;
    }
    if (dev < 0 || dev >= kMaxDevices) {
        corey::fail(COREY_EUNSUPPORTED, "%s: device index %d beyond the %d this entry point keeps an address for", who, dev, kMaxDevices);
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            corey::hip_fail(e, "hipGetSymbolAddress(scratch)");
            return nullptr;
        }
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}

}  // namespace

extern "C" int corey_entropy_hist_static(const void* x, corey_dtype dt, int64_t B, int64_t D, int64_t L, const int32_t* seqlens,
                                         int32_t K, double eps, int64_t stride, int64_t block, uint32_t* counts_out, double* H_out,
                                         double* r_out, float* range_out, void* range_parts, void* hip_stream)
{
    const size_t need = corey_entropy_hist_workspace(B, K);     // 0 for invalid B or K: the common checks below name those
    if (need > COREY_STATIC_SCRATCH_BYTES)
        return corey::fail(COREY_EWORKSPACE, "corey_entropy_hist_static: B = %lld with K = %d needs %zu bytes of scratch, the built-in "
                           "buffer holds %d (use corey_entropy_hist with a workspace of your own)", (long long)B, K, need,
                           COREY_STATIC_SCRATCH_BYTES);
    void* ws = static_scratch("corey_entropy_hist_static");
    if (!ws) return COREY_EHIP;
    return entropy_hist_impl("corey_entropy_hist_static", x, dt, B, D, L, seqlens, K, eps, stride, block, counts_out, H_out, r_out,
                             range_out, ws, COREY_STATIC_SCRATCH_BYTES, hip_stream, Tail{}, range_parts);
}

extern "C" int corey_route_device(const void* x, corey_dtype dt, int64_t B, int64_t D, int64_t L, const int32_t* seqlens,
                                  int32_t K, double eps, int64_t stride, int64_t block, const corey_policy* p,
                                  double ema_lambda, double* ema_state, uint32_t* chunk_calls,
                                  uint32_t* counts_out, double* H_out, double* r_out, float* range_out, void* range_parts,
                                  int32_t* chunks_out, void* workspace, size_t workspace_bytes_given, void* hip_stream)
{
    using corey::fail;
    if (!p || !chunks_out) return fail(COREY_ENULL, "corey_route_device: p and chunks_out are required");
    if (ema_state && !(ema_lambda >= 0.0 && ema_lambda < 1.0))
        return fail(COREY_EINVAL, "corey_route_device: ema_lambda = %g outside [0, 1)", ema_lambda);
    const int st = check_device_policy("corey_route_device", p, L);
    if (st != COREY_OK) return st;
    Tail tail = {};
    tail.pol = p; tail.chunks_out = chunks_out; tail.ema_lambda = ema_lambda; tail.ema_state = ema_state; tail.chunk_calls = chunk_calls;
    return entropy_hist_impl("corey_route_device", x, dt, B, D, L, seqlens, K, eps, stride, block, counts_out, H_out, r_out, range_out,
                             workspace, workspace_bytes_given, hip_stream, tail, range_parts);
}

static_assert(sizeof(corey_finalise::Args) <= sizeof(corey_deferred_route), "the opaque ticket holds the reduction's arguments");

extern "C" int corey_route_device_deferred(const void* x, corey_dtype dt, int64_t B, int64_t D, int64_t L, const int32_t* seqlens,
                                           int32_t K, double eps, int64_t stride, int64_t block, const corey_policy* p,
                                           uint32_t* chunk_calls, uint32_t* counts_out, double* H_out, double* r_out,
                                           float* range_out, void* range_parts, int32_t* chunks_out, void* workspace,
                                           size_t workspace_bytes_given, corey_deferred_route* route, void* hip_stream)
{
    using corey::fail;
    if (!p || !chunks_out || !route) return fail(COREY_ENULL, "corey_route_device_deferred: p, chunks_out and route are required");
    const int st = check_device_policy("corey_route_device_deferred", p, L);
    if (st != COREY_OK) return st;
    corey_finalise::Args fa = {};
    Tail tail = {};
    tail.pol = p; tail.chunks_out = chunks_out; tail.chunk_calls = chunk_calls; tail.defer = &fa;
    const int rc = entropy_hist_impl("corey_route_device_deferred", x, dt, B, D, L, seqlens, K, eps, stride, block, counts_out, H_out, r_out,
                                     range_out, workspace, workspace_bytes_given, hip_stream, tail, range_parts);
    if (rc != COREY_OK) return rc;
    memset(route, 0, sizeof(*route));
    memcpy(route, &fa, sizeof(fa));
    return COREY_OK;
}
