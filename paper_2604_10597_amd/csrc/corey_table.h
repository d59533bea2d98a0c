// Bit-pattern table of a 16-bit tensor: how often each of the 65536 storage bit patterns occurs.
//
// The fixed-bin histogram of Eq. 1 needs the tensor's range before a value can be binned, which is why the paper's
// estimator makes two passes (a min/max pass, then a bin-count pass).  For 16-bit storage there is a range-free
// intermediate: count the bit patterns in ONE pass, then take range and bin counts from the table (the bin of a value
// depends on the value and the range only, so binning 65536 patterns with their multiplicities gives exactly the counts
// of binning every element).  Whoever produces or reads the tensor anyway can fill the table on the way.
//
// A workgroup of kLanes lanes keeps the whole table in LDS: 32768 words, each holding two 16-bit counters (the pattern
// of magnitude m with sign 0 in the low half, with sign 1 in the high half).  A counter uses 15 bits; bit 15 is a
// guard.  An element adds 1 to its half with a returning LDS atomic; the lane that sees its counter go from 0x7fff to
// 0x8000 takes 0x8000 off again and records the pattern in the workgroup's overflow list (one entry = 32768
// occurrences).  The workgroup meets at a barrier at least every kRoundAdds = 32768 elements: a counter starts a round
// below 0x8000 and gains at most 32768, so its half never carries into its neighbour's, sees at most one guard crossing
// per round, and is below 0x8000 again at the barrier whatever the interleaving of the lanes.  All arithmetic is integer
// and every element is counted exactly once: the table is exact and independent of scheduling.
// The pattern 0x0000 (+0.0: most of a sparse activation tensor) is counted in a word of the lane's own instead (32 bits,
// no guard needed), which keeps a wave full of zeros from queueing on one LDS address.  A lane issues the adds of a whole
// 16-byte word (8 elements) before it looks at what they returned, and it looks first at the OR of the returned words:
// a guard crossing needs bit 14 of a counter set beforehand, so when neither half of any returned word has it (the usual
// case: a workgroup sees a few dozen occurrences of a pattern) no element needs the exact test.
// At the end the workgroup writes the parts of its table that hold counts (two bytes per pattern) plus a small tail (zeros,
// overflow list) to its own slab of the caller's workspace: no global atomics, nothing to clear beforehand.
#ifndef COREY_TABLE_H
#define COREY_TABLE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "corey_range.h"

namespace corey_table {

constexpr int kLanes = 1024;            // lanes per workgroup of a kernel that fills a table (16 waves: one workgroup per compute unit)
constexpr int kWords = 32768;           // LDS words of the table
constexpr int kRoundAdds = 32768;       // most elements a workgroup may add between two barriers
constexpr int kMaxSlabs = 256;          // most workgroups that fill tables in one launch (one per compute unit)
constexpr int kMaxOver = 1024;          // overflow entries a workgroup can record: 32768 elements each, 2^25 elements per workgroup
constexpr int kParts = corey_range::kParts;

constexpr int kUnitWords = 256;         // words of a slab that are written and read, or left out, together: a wave's 16-byte words
constexpr int kUnits = kWords / kUnitWords;

struct Head {                           // per workgroup: what its slab does not hold
    uint32_t n_over;                    // entries of the workgroup's overflow list in use
    uint32_t zeros;                     // occurrences of pattern 0x0000
    uint32_t units[kUnits / 32];        // the units of its slab that were written; the others hold no counts
};
struct Tail {                           // per workgroup: the overflow list
    uint16_t over[kMaxOver];            // patterns that crossed the guard bit (each entry stands for 32768 occurrences)
};

struct Shared {                         // LDS bookkeeping beside the table
    uint32_t n_over;
    uint16_t over[kMaxOver];
    uint32_t zeros[kLanes];             // per lane: occurrences of pattern 0x0000
    uint32_t units[kUnits / 32];
};

// Values of the storage bit patterns.  kDense: a tensor's values are spread over most of the table (binary16: a dozen of its 32
// exponents, 1024 patterns each), so that a look at every occurring pattern for the range costs more than the way round it below:
// 1 million N(0,1) values, binary16 10.1 -> 9.1 us, wide ones 14.4 -> 10.1; bfloat16, whose values fill a tenth of the table, 8.1 -> 8.4.
template <typename T> struct Pattern;
template <> struct Pattern<uint16_t> {  // bfloat16
    static constexpr uint32_t kInf = 0x7f80u;
    static constexpr bool kDense = false;
    static __device__ __forceinline__ float value(uint32_t p) { return __uint_as_float(p << 16); }
};
template <> struct Pattern<_Float16> {
    static constexpr uint32_t kInf = 0x7c00u;
    static constexpr bool kDense = true;
    static __device__ __forceinline__ float value(uint32_t p)
    {
        const uint16_t b = (uint16_t)p;
        _Float16 h;
        __builtin_memcpy(&h, &b, 2);
        return (float)h;
    }
};

// Layout of the caller's workspace (corey_pattern_table_workspace() bytes, 256-byte aligned).
struct Workspace {
    corey_range::RangeSlot* slots;      // [1]   range of the histogram, for the reduction kernel
    uint32_t* parts;                    // [kParts][COREY_MAX_BINS] partial histograms the binning kernel adds into
    corey_range::RangePart* rparts;     // [kMaxSlabs] partial ranges of the kernel that filled the tables
    uint32_t* nslabs;                   // [1]   slabs that kernel wrote
    Head* heads;                        // [kMaxSlabs]
    Tail* tails;                        // [kMaxSlabs]
    uint32_t* slabs;                    // [kMaxSlabs][kWords]
};

constexpr size_t kSlotsBytes = 256;
constexpr size_t kPartsBytes = (size_t)kParts * COREY_MAX_BINS * sizeof(uint32_t);
constexpr size_t kRpartsBytes = (size_t)kMaxSlabs * sizeof(corey_range::RangePart);
constexpr size_t kCountBytes = 256;
constexpr size_t kHeadsBytes = (size_t)kMaxSlabs * sizeof(Head);      // (whole 256 bytes)
constexpr size_t kTailsBytes = ((size_t)kMaxSlabs * sizeof(Tail) + 255) / 256 * 256;
constexpr size_t kSlabsBytes = (size_t)kMaxSlabs * kWords * sizeof(uint32_t);
constexpr size_t kWorkspaceBytes = kSlotsBytes + kPartsBytes + kRpartsBytes + kCountBytes + kHeadsBytes + kTailsBytes + kSlabsBytes;

inline __host__ __device__ Workspace carve(void* base)
{
    char* p = static_cast<char*>(base);
    Workspace w;
    w.slots = reinterpret_cast<corey_range::RangeSlot*>(p);
    p += kSlotsBytes;
    w.parts = reinterpret_cast<uint32_t*>(p);
    p += kPartsBytes;
    w.rparts = reinterpret_cast<corey_range::RangePart*>(p);
    p += kRpartsBytes;
    w.nslabs = reinterpret_cast<uint32_t*>(p);
    p += kCountBytes;
    w.heads = reinterpret_cast<Head*>(p);
    p += kHeadsBytes;
    w.tails = reinterpret_cast<Tail*>(p);
    p += kTailsBytes;
    w.slabs = reinterpret_cast<uint32_t*>(p);
    return w;
}

// Clear the workgroup's table and bookkeeping; also this workgroup's share of the partial histograms (the binning kernel,
// which runs after every table is written, adds into them).  Ends with a barrier.
__device__ __forceinline__ void begin(uint32_t* s_tab, Shared& sh, const Workspace& ws)
{
    typedef uint32_t word4 __attribute__((ext_vector_type(4)));
    const word4 zero = {0u, 0u, 0u, 0u};
    for (int i = threadIdx.x; i < kWords / 4; i += kLanes) reinterpret_cast<word4*>(s_tab)[i] = zero;
    if (threadIdx.x == 0) sh.n_over = 0u;
    if (threadIdx.x < kUnits / 32) sh.units[threadIdx.x] = 0u;
    sh.zeros[threadIdx.x] = 0u;
    for (int i = blockIdx.x * kLanes + threadIdx.x; i < kParts * COREY_MAX_BINS; i += gridDim.x * kLanes) ws.parts[i] = 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) *ws.nslabs = gridDim.x;
    __syncthreads();
}

// The exact test after an add returned `old`: did this add take the element's counter from 0x7fff to 0x8000?  Then take
// 32768 off again and record them.
__device__ __forceinline__ void settle(uint32_t* s_tab, Shared& sh, uint32_t p, uint32_t old)
{
    if (p == 0u) return;                                      // the lane's own 32-bit zero counter has no guard
    const uint32_t hi = p >> 15;
    const uint32_t cnt = (hi ? old >> 16 : old) & 0xffffu;
    if (cnt == 0x7fffu) {
        atomicAdd(&s_tab[p & 0x7fffu], 0u - ((hi ? 0x10000u : 1u) << 15));
        const uint32_t slot = atomicAdd(&sh.n_over, 1u);
        if (slot < (uint32_t)kMaxOver) sh.over[slot] = (uint16_t)p;
    }
}

// Issue the add for one element with storage bits p (0 ... 65535); returns what the counter's word held before.
__device__ __forceinline__ uint32_t add_issue(uint32_t* s_tab, Shared& sh, uint32_t p)
{
    const uint32_t inc = (p >> 15) ? 0x10000u : 1u;           // the sign bit picks the half
    uint32_t* word = (p == 0u) ? &sh.zeros[threadIdx.x] : &s_tab[p & 0x7fffu];
    return atomicAdd(word, inc);                              // returning LDS atomic
}

// Count one element.
__device__ __forceinline__ void add(uint32_t* s_tab, Shared& sh, uint32_t p)
{
    settle(s_tab, sh, p, add_issue(s_tab, sh, p));
}

// The eight elements of one 16-byte word: all adds first, then one look at the OR of what they returned.  Words without a zero
// pattern need no look at each of their elements for one: an element is then its place (two instructions), its half (two) and
// its add.  The wave takes either form as a whole: with the choice left to the lanes a few zeros made it issue both, sixteen adds
// for eight values (84 million bf16 values, one in a hundred zero: 45.4 us, as it is 36.4).
__device__ __forceinline__ void add_word4(uint32_t* s_tab, Shared& sh, const uint32_t (&w)[4])
{
    typedef uint16_t half2 __attribute__((ext_vector_type(2)));
    half2 h[4];
    __builtin_memcpy(h, w, 16);
    const half2 least = __builtin_elementwise_min(__builtin_elementwise_min(h[0], h[1]), __builtin_elementwise_min(h[2], h[3]));
    uint32_t old[8], any = 0u;
    if (!__any(least.x == 0 || least.y == 0)) {                // over the lanes that have a word
        char* tab = reinterpret_cast<char*>(s_tab);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            old[2 * k] = atomicAdd(reinterpret_cast<uint32_t*>(tab + ((w[k] << 2) & 0x1fffcu)), __umul24((w[k] >> 15) & 1u, 0xffffu) + 1u);
            old[2 * k + 1] = atomicAdd(reinterpret_cast<uint32_t*>(tab + ((w[k] >> 14) & 0x1fffcu)), __umul24(w[k] >> 31, 0xffffu) + 1u);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            old[2 * k] = add_issue(s_tab, sh, w[k] & 0xffffu);
            old[2 * k + 1] = add_issue(s_tab, sh, w[k] >> 16);
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) any |= old[e];
    if (any & 0x40004000u) {                                  // some counter (or a zero counter) was at 16384 or more
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            settle(s_tab, sh, w[k] & 0xffffu, old[2 * k]);
            settle(s_tab, sh, w[k] >> 16, old[2 * k + 1]);
        }
    }
}

// Fold a pattern that occurs into a range.
template <typename T> __device__ __forceinline__ void fold_pattern(uint32_t p, uint32_t& klo, uint32_t& khi, uint32_t& knan)
{
    if ((p & 0x7fffu) > Pattern<T>::kInf) {
        knan = 1u;
        return;
    }
    const uint32_t key = corey_range::order_key(Pattern<T>::value(p));
    klo = min(klo, key);
    khi = max(khi, key);
}

// Write the workgroup's table, tail and partial range to its slab.  FROM_TABLE: the range is read off the table (three instructions
// a value less in the loop that fills it); otherwise the lanes hand in what they saw.  Reduced over the workgroup either way (valid
// in thread 0 afterwards).  Only the units of the table that hold counts are written: a tensor's values lie in a dozen
// of bfloat16's 128 pairs of exponents, and 128 KiB per workgroup, mostly zeros, went to memory and back.
template <typename T, bool FROM_TABLE>
__device__ __forceinline__ void end(uint32_t* s_tab, Shared& sh, const Workspace& ws, uint32_t& klo, uint32_t& khi, uint32_t& knan)
{
    typedef uint32_t word4 __attribute__((ext_vector_type(4)));
    __syncthreads();                                          // every add has landed
    uint32_t zeros = sh.zeros[threadIdx.x];
    const uint32_t n_over = sh.n_over < (uint32_t)kMaxOver ? sh.n_over : (uint32_t)kMaxOver;
    if constexpr (FROM_TABLE) {
        klo = 0xffffffffu; khi = 0u; knan = 0u;
        if (zeros) fold_pattern<T>(0u, klo, khi, knan);
        for (uint32_t i = threadIdx.x; i < n_over; i += kLanes) fold_pattern<T>(sh.over[i], klo, khi, knan);
    }
    for (int off = 32; off > 0; off >>= 1) zeros += (uint32_t)__shfl_xor((int)zeros, off);
    // kDense: a lane meets its 16-byte words in the order of their patterns' magnitudes, so it notes the first and the last of either
    // sign and looks at the counts in two of them once they are known.
    constexpr int kInfWord = (int)(Pattern<T>::kInf / 4);      // (infinity is a word's first pattern)
    int pos_first = -1, pos_last = -1, neg_first = -1, neg_last = -1;
    auto fold_words = [&](int i, const word4& v, bool pos, bool neg) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (pos && (v[e] & 0xffffu)) fold_pattern<T>(4 * i + e, klo, khi, knan);
            if (neg && (v[e] >> 16)) fold_pattern<T>((4 * i + e) | 0x8000u, klo, khi, knan);
        }
    };
    word4* slab = reinterpret_cast<word4*>(ws.slabs + (size_t)blockIdx.x * kWords);
    for (int i = threadIdx.x; i < kWords / 4; i += kLanes) {
        const word4 v = reinterpret_cast<const word4*>(s_tab)[i];
        if (__ballot((v.x | v.y | v.z | v.w) != 0u) == 0ull) continue;       // uniform over the wave
        slab[i] = v;
        const int unit = i / (kUnitWords / 4);
        if ((threadIdx.x & 63) == 0) atomicOr(&sh.units[unit >> 5], 1u << (unit & 31));
        if constexpr (FROM_TABLE) {
            if (!Pattern<T>::kDense || i >= kInfWord) {        // (beyond: infinity and NaN)
                fold_words(i, v, true, true);
            } else {
                const uint32_t any = v.x | v.y | v.z | v.w;
                if (any & 0xffffu) {
                    pos_first = pos_first < 0 ? i : pos_first;
                    pos_last = i;
                }
                if (any >> 16) {
                    neg_first = neg_first < 0 ? i : neg_first;
                    neg_last = i;
                }
            }
        }
    }
    if constexpr (FROM_TABLE && Pattern<T>::kDense) {
        const int lowest = neg_last >= 0 ? neg_last : pos_first, highest = pos_last >= 0 ? pos_last : neg_first;
        if (lowest >= 0) fold_words(lowest, reinterpret_cast<const word4*>(s_tab)[lowest], neg_last < 0, neg_last >= 0);
        if (highest >= 0) fold_words(highest, reinterpret_cast<const word4*>(s_tab)[highest], pos_last >= 0, pos_last < 0);
    }
    corey_range::reduce_range_keys<kLanes>(klo, khi, knan);   // holds a barrier: the units are known, all zero counts have been read
    if ((threadIdx.x & 63) == 0) sh.zeros[threadIdx.x >> 6] = zeros;         // the waves' totals
    __syncthreads();
    Tail* tail = ws.tails + blockIdx.x;
    for (uint32_t i = threadIdx.x; i < n_over; i += kLanes) tail->over[i] = sh.over[i];
    if (threadIdx.x == 0) {
        uint32_t z = 0u;
        for (int w = 0; w < kLanes / 64; ++w) z += sh.zeros[w];
        Head h;
        h.n_over = n_over;
        h.zeros = z;
#pragma unroll
        for (int k = 0; k < kUnits / 32; ++k) h.units[k] = sh.units[k];
        ws.heads[blockIdx.x] = h;
        corey_range::RangePart rp;
        rp.lo_key = klo; rp.hi_key = khi; rp.saw_nan = knan; rp.pad = 0u;
        ws.rparts[blockIdx.x] = rp;
    }
}

}  // namespace corey_table
#endif
