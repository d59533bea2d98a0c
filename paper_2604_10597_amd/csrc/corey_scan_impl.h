// Kernels of selective_scan_fwd (Mamba-1 selective-scan forward with a run-time chunk) for gfx950, as templates
// over the storage type.  Each storage type is instantiated in translation units of its own (corey_scan_f32.hip,
// corey_scan_bf16.hip, corey_scan_f16.hip, and corey_scan_any_*.hip for the kernels that read the chunk from device memory) so
// that they compile in parallel; corey_scan.hip holds the host entry.
//
// One kernel per call for launches of few rows (see kDirectRows), two for the others.
//
// k_relayout_bc   (launches of many rows) converts B and C ([B, N, L]) once to fp32 in the caller's workspace, tile by tile, in exactly
//                 the order the scan's lanes read them.  B and C are shared by every channel of a sequence, so
//                 doing this once per call removes all conversion work from the scan (a few MB of traffic against
//                 the scan's hundreds).
//
// k_scan          A workgroup of 256 lanes owns ROWS channels of one sequence and walks the time axis in tiles of
//                 CHUNK steps.  The tile geometry is a compile-time constant (one instantiation per chunk, chosen at
//                 launch from the run-time chunk), so every LDS address in the inner loop is an immediate offset.
//                 Inside a tile a row is spread over LPR = CHUNK / K consecutive lanes, each lane owning K (16, 8 or
//                 4) consecutive time steps: loads of u / delta / z and the store of y are one vector per lane (16 bytes
//                 or more; 8 for four 16-bit values), contiguous along L.  The fp32 B / C values of a few states at a time are copied from the
//                 workspace straight into LDS (global_load_lds, no registers), double buffered; in a launch of few rows a
//                 lane loads those of its own steps as stored.  A chunk longer than a wave's lanes take is walked in parts
//                 (tile_of).  For every state index n a lane
//   1. discretises its K steps (a_i = exp2(dl_i A log2e), b_i = dl_i B_i u_i) and folds them, from a zero state,
//      into the pair (P, h) of the affine map  x -> P x + h  of its sub-block (P is one exp2 of the summed dl);
//      the first lane of the row also applies its map to the state carried from the previous tile;
//   2. takes part in an inclusive scan of the pairs across the lanes of the row (the pair operator is associative),
//      written as single DPP instructions; h then is the true state at the end of the lane's sub-block.  No row is
//      wider than a wave;
//   3. receives the state entering its sub-block from the lane to its left, replays its K steps from it and
//      accumulates y_i += C_i h_i.
// The fp32 state carried from tile to tile lives in LDS; the last lane of a row refreshes it.
// The work is a recurrence plus elementwise maths: no matrix instructions.
#ifndef COREY_SCAN_IMPL_H
#define COREY_SCAN_IMPL_H

#include <hip/hip_runtime.h>

#include <type_traits>

#include "corey_finalise.h"
#include "corey_internal.h"

namespace corey_scan {

using corey::bf16_to_f32;
using corey::f32_to_bf16;

constexpr int kBlock = 256;   // lanes per workgroup: four waves, one per SIMD of a compute unit
constexpr int kWaves = kBlock / 64;
constexpr int kStageFloats = 2048;    // fp32 values of B (and of C) per LDS staging buffer (two buffers)
constexpr int kMaxGroup = 4;          // most states staged (and unrolled) per group
constexpr int kPad = COREY_MAX_CHUNK; // the relaid-out time axis is padded to whole tiles
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// The tile a launch walks at a time: the chunk, or parts of a long one.  64 lanes of 16 steps are one wave; a row over two
// waves would hand every state's sub-block products from wave to wave through LDS and a barrier (chunk 2048 on 8192 rows of
// 4096 steps: 195 us with rows over two waves, 139 us in parts of 1024).  With more rows than the GPU holds waves the parts
// are 512 steps: two rows share a wave's lane scan and its reads of B and C (the same layer: 135 us; 5120 rows of 16384 steps
// 357 us in parts of 1024, 323 us in parts of 512 with the two kinds of rows below).
constexpr int kMaxTile = 1024;
constexpr int64_t kManyRows = 4096;   // four waves on each of the 1024 SIMDs
__host__ __device__ inline int tile_of(int chunk, int64_t rows)
{
    const int most = rows > kManyRows ? 512 : kMaxTile;
    return chunk < most ? chunk : most;
}

// Geometry of one (K, CHUNK) instantiation; CHUNK is the tile walked at a time.
template <int K, int CHUNK> struct Geo {
    static_assert(CHUNK >= K && CHUNK / K <= 64, "a tile row must fit one wave");
    static constexpr int LPR = CHUNK / K;                       // lanes per row
    static constexpr int SEG = LPR;                             // lanes a scan runs over
    static constexpr int ROWS = kBlock / LPR;                   // rows per workgroup
    static constexpr int G = kStageFloats / CHUNK < 1 ? 1 : (kStageFloats / CHUNK > kMaxGroup ? kMaxGroup : kStageFloats / CHUNK);
    static_assert(kMaxGroup % G == 0, "the padded state count must be whole groups");
    static constexpr int STAGE = G * CHUNK;                     // floats per operand per staging buffer
};

// Time steps per lane, chosen per channel range.  16 steps halve the lane-scan work per value and stage B / C once for
// twice as many rows of a workgroup; 8 steps double the waves per row and need fewer registers.  Measured on channel
// counts 1024 ... 16384 at chunks 128 ... 512: while every row can have a wave of its own with all of them resident
// (four waves per SIMD: 4096 waves), 8 steps win.  Beyond that the fastest launch gives the channels below d16 sixteen
// steps, in whole layers of one workgroup per compute unit, and the remaining channels (less than one such layer)
// eight: the two kinds of workgroups then fill the SIMDs evenly (e.g. 5120 rows at chunk 512: 4096 rows as two
// 16-step waves per SIMD plus 1024 rows as one 8-step wave, 10 % faster than either geometry alone).
// plan_d16 returns d16: channels [0, d16) of every sequence take 16 steps per lane, [d16, D) take 8; 0 and D are the
// pure launches.  It runs on the host, for every tile that a chunk read from device memory may ask for (Plans).
inline int64_t plan_d16(int64_t B, int64_t D, int chunk, int rows_cap)
{
    chunk = tile_of(chunk, B * D);
    if (chunk > 512) return D;                                   // a row of 8-step lanes would no longer fit one wave
    if (chunk < 128)                                             // 16-step rows would leave workgroup lanes idle here
        return (B * D * (chunk / 16) < 172032) ? 0 : D;
    const int64_t waves8 = B * D * (chunk / 8) / 64;
    if (waves8 <= 4096) return 0;
    int rows16 = kBlock * 16 / chunk;                            // rows of a 16-step workgroup
    rows16 = rows16 < rows_cap ? rows16 : rows_cap;
    const int64_t layer = (int64_t)256 * rows16 / B / 32 * 32;   // channels per sequence in one workgroup per compute unit
    if (layer < 32) return D;
    return D / layer * layer;
}

// Steps per lane of the channels that do not take 16 (all of them when d16 = 0): 8, or 4 when even 8-step rows leave
// most SIMDs without a wave (short tiles or few channels: a row is only chunk / 8 lanes wide).  Halving the steps doubles
// the lanes at the price of a longer lane scan per value.  Measured on 1024 ... 8192 channels at chunks 16 ... 512:
// 4 steps win by 10 ... 35 % while the 8-step launch has at most about 1500 waves (1.5 per SIMD) and a 4-step row still
// fits one wave (chunk <= 256); with 2 steps the lane scan costs more than the extra waves bring at chunks of 64 and up.
constexpr int64_t kFewWaves = 1536;
inline int plan_klo(int64_t B, int64_t D, int chunk, int64_t d16)
{
    if (d16 != 0 || chunk > 256) return 8;
    return B * D * (chunk / 8) / 64 <= kFewWaves ? 4 : 8;
}

// A launch of one kind of row that still leaves the SIMDs short of waves (small layers, short tiles) gives every channel
// TWO rows in the same workgroup, each with half of the states: twice the waves, each with half the per-state work and
// all of the per-token work, and one exchange of partial y per tile through LDS.  The staging group must hold at least
// one state of each half (every tile does), and only the geometries such a launch can have are built.  What counts is the tile
// walked: chunk 2048 takes the launch of 1024 (bf16, 64 rows of 4096 steps: one row per channel 37.1 us, two 23.5; 256 of 32768 264
// and 159; binary32 284 and 175).
constexpr int64_t kSplitWaves = 1536;
inline int plan_split(int64_t B, int64_t D, int N, int chunk, int64_t d16, int klo, int allow)
{
    if (!allow || N < 4 || (d16 > 0 && d16 < D)) return 0;    // (fewer than four states: the second row would hold padding only)
    chunk = tile_of(chunk, B * D);
    const int K = d16 >= D ? 16 : klo;
    if (!((K == 16 && chunk == 1024) || (K == 8 && chunk == 512) || (K == 4 && chunk <= 256))) return 0;
    const int lpr = chunk / K < 1 ? 1 : chunk / K;
    return B * D * lpr / 64 <= kSplitWaves ? 1 : 0;
}

// ------------------------------------------------------------------------------------------- storage types
// A lane keeps its K consecutive stored values as raw 16-byte words (Raw) and widens them when needed.
template <typename T> struct Io;
template <> struct Io<float> {
    static constexpr int kVec = 4;     // elements per 16-byte word
    static __device__ __forceinline__ float ld(const float* p) { return *p; }
    static __device__ __forceinline__ void st(float* p, float v) { *p = v; }
    static __device__ __forceinline__ void unpack(const uint4v& q, float* out)
    {
        out[0] = __uint_as_float(q.x); out[1] = __uint_as_float(q.y);
        out[2] = __uint_as_float(q.z); out[3] = __uint_as_float(q.w);
    }
    static __device__ __forceinline__ uint4v pack(const float* v)
    {
        uint4v q;
        q.x = __float_as_uint(v[0]); q.y = __float_as_uint(v[1]); q.z = __float_as_uint(v[2]); q.w = __float_as_uint(v[3]);
        return q;
    }
};
template <> struct Io<uint16_t> {                         // bfloat16 storage
    static constexpr int kVec = 8;
    static __device__ __forceinline__ float ld(const uint16_t* p) { return bf16_to_f32(*p); }
    static __device__ __forceinline__ void st(uint16_t* p, float v) { *p = f32_to_bf16(v); }
    static __device__ __forceinline__ void unpack(const uint4v& q, float* out)
    {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            out[2 * k] = __uint_as_float(w[k] << 16);
            out[2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
        }
    }
    // round to nearest even in hardware (v_cvt_pk_bf16_f32)
    static __device__ __forceinline__ uint32_t pack2(float lo, float hi)
    {
        float2v f;
        f.x = lo; f.y = hi;
        const bf16x2 h = __builtin_convertvector(f, bf16x2);
        uint32_t r;
        __builtin_memcpy(&r, &h, 4);
        return r;
    }
    static __device__ __forceinline__ uint4v pack(const float* v)
    {
        uint4v q;
        q.x = pack2(v[0], v[1]); q.y = pack2(v[2], v[3]); q.z = pack2(v[4], v[5]); q.w = pack2(v[6], v[7]);
        return q;
    }
};
template <> struct Io<_Float16> {                         // IEEE binary16 storage
    static constexpr int kVec = 8;
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    static __device__ __forceinline__ float ld(const _Float16* p) { return (float)*p; }
    static __device__ __forceinline__ void st(_Float16* p, float v) { *p = (_Float16)v; }
    static __device__ __forceinline__ void unpack(const uint4v& q, float* out)
    {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            h2 h;
            __builtin_memcpy(&h, &w[k], 4);
            out[2 * k] = (float)h.x;
            out[2 * k + 1] = (float)h.y;
        }
    }
    static __device__ __forceinline__ uint32_t pack2(float lo, float hi)    // round to nearest even
    {
        float2v f;
        f.x = lo; f.y = hi;
        const h2 h = __builtin_convertvector(f, h2);
        uint32_t r;
        __builtin_memcpy(&r, &h, 4);
        return r;
    }
    static __device__ __forceinline__ uint4v pack(const float* v)
    {
        uint4v q;
        q.x = pack2(v[0], v[1]); q.y = pack2(v[2], v[3]); q.z = pack2(v[4], v[5]); q.w = pack2(v[6], v[7]);
        return q;
    }
};

template <typename T, int K> struct Raw {
    static constexpr int kBytes = K * (int)sizeof(T);           // 4 or 8 (short runs: one load), else whole 16-byte words
    static constexpr int kWords = kBytes / 16 > 0 ? kBytes / 16 : 1;
    uint4v w[kWords];                                          // a short run uses the first kBytes of w[0]
};

// Rows of [.., L] tensors start at any multiple of the element size (L may be odd): vector accesses are written as copies of
// unaligned memory, which gfx950 does with the same 16-byte instructions.
template <typename T, int K> __device__ __forceinline__ Raw<T, K> load_full(const T* p)
{
    Raw<T, K> r;
    r.w[0] = uint4v{0u, 0u, 0u, 0u};                           // (a short run fills the first kBytes only)
    __builtin_memcpy(&r, p, Raw<T, K>::kBytes);
    return r;
}

// Drop the first `s` values (uniform, 0 < s < K) and fill with zero bits from behind.
template <typename T, int K> __device__ __forceinline__ void drop_first(Raw<T, K>& r, int s)
{
    constexpr int NW = (Raw<T, K>::kBytes + 3) / 4;
    uint32_t w[NW + 1];
#pragma unroll
    for (int k = 0; k < NW; ++k) w[k] = r.w[k / 4][k % 4];
    w[NW] = 0u;
    int words = s;
    if constexpr (sizeof(T) == 2) {
        words = s >> 1;
        if (s & 1) {
#pragma unroll
            for (int k = 0; k < NW; ++k) w[k] = __builtin_amdgcn_alignbit(w[k + 1], w[k], 16);
        }
    }
#pragma unroll
    for (int step = 1; step < NW; step *= 2) {
        if (words & step) {
#pragma unroll
            for (int k = 0; k < NW; ++k) w[k] = k + step < NW ? w[k + step] : 0u;
        }
    }
#pragma unroll
    for (int k = 0; k < NW; ++k) r.w[k / 4][k % 4] = w[k];
}

// The end of the rows.  In a sequence's last, partial tile a lane's vector may reach beyond its row into the next one: those
// values become zero bits where they are used (keep).  In the last row of a tensor it would reach beyond the tensor: there the
// lane takes the K values that end the row instead, and they are shifted down to their places (shift).  Reading the straddling
// lane's values one by one would be K loads.
template <typename T, int K> struct Tail {
    static constexpr int NW = (Raw<T, K>::kBytes + 3) / 4;
    int shift;                 // uniform: K - L % K, what the lane at the end of the last row has to shift by (0: L is a multiple of K)
    bool at_end;               // this lane's steps reach beyond L
    uint32_t keep[NW];         // bits of the values before nvalid
    __device__ __forceinline__ void init(int64_t L, int64_t t0, int nvalid)
    {
        shift = (int)(L % K) == 0 ? 0 : K - (int)(L % K);
        at_end = t0 + K > L;
        constexpr int PER = sizeof(T) == 2 ? 2 : 1;
#pragma unroll
        for (int w = 0; w < NW; ++w)
            keep[w] = nvalid >= PER * (w + 1) ? 0xffffffffu : (nvalid <= PER * w ? 0u : 0xffffu);
    }
    // (a lane wholly beyond the row holds nothing of use before or after)
    __device__ __forceinline__ void place(Raw<T, K>& r) const
    {
        if (shift != 0 && at_end) drop_first<T, K>(r, shift);
    }
    __device__ __forceinline__ void mask(Raw<T, K>& r) const
    {
#pragma unroll
        for (int w = 0; w < NW; ++w) r.w[w / 4][w % 4] &= keep[w];
    }
};

// The same for rows shorter than one lane's run, value by value.
template <typename T, int K> __device__ __forceinline__ Raw<T, K> load_few(const T* p, int nvalid)
{
    T tmp[K];
#pragma unroll
    for (int i = 0; i < K; ++i) tmp[i] = T(0);
#pragma unroll
    for (int i = 0; i < K; ++i)
        if (i < nvalid) tmp[i] = p[i];
    Raw<T, K> r;
    r.w[0] = uint4v{0u, 0u, 0u, 0u};
    __builtin_memcpy(&r, tmp, Raw<T, K>::kBytes);
    return r;
}

template <typename T, int K>
__device__ __forceinline__ void widen(const Raw<T, K>& r, float (&out)[K])
{
    if constexpr (Raw<T, K>::kBytes < 16) {
        float all[Io<T>::kVec];
        Io<T>::unpack(r.w[0], all);
#pragma unroll
        for (int i = 0; i < K; ++i) out[i] = all[i];
    } else {
#pragma unroll
        for (int v = 0; v < Raw<T, K>::kWords; ++v) Io<T>::unpack(r.w[v], &out[v * Io<T>::kVec]);
    }
}

template <typename T, int K>
__device__ __forceinline__ void store_items(T* p, int nstore, const float (&v)[K])
{
    constexpr int V = Io<T>::kVec;
    if (nstore == K) {
        Raw<T, K> r;
        if constexpr (Raw<T, K>::kBytes < 16) {
            float all[V];
#pragma unroll
            for (int i = 0; i < V; ++i) all[i] = i < K ? v[i < K ? i : 0] : 0.f;
            r.w[0] = Io<T>::pack(all);
        } else {
#pragma unroll
            for (int k = 0; k < K / V; ++k) r.w[k] = Io<T>::pack(&v[k * V]);
        }
        __builtin_memcpy(p, &r, Raw<T, K>::kBytes);
    } else {
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (i < nstore) Io<T>::st(p + i, v[i]);
    }
}

// ------------------------------------------------------------------------------------------- elementwise maths
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// log(1 + e^x) = max(x, 0) + log1p(e^{-|x|}).  log1p(e) is taken as log(w), w = fl(1 + e), plus the repair
// e - (w - 1) of the rounding in w (its 1/w factor lies in [1/2, 1] and the repair is below one ulp of w, so
// dropping the factor costs < 3e-8 absolute): the small tail e << 1 stays accurate to binary32 relative precision.
__device__ __forceinline__ float softplus(float x)
{
    const float e = fast_exp2(-fabsf(x) * kLog2e);
    const float w = 1.f + e;
    const float fix = e - (w - 1.f);
    float pos;                                             // max(x, 0) in one instruction: fmaxf would first quiet a signalling
    asm("v_max_f32_e32 %0, 0, %1" : "=v"(pos) : "v"(x));   // NaN with a second one, which x (a sum) cannot be
    return pos + fmaf(__builtin_amdgcn_logf(w), kLn2, fix);
}

// z * sigmoid(z)
__device__ __forceinline__ float silu(float z)
{
    return z * __builtin_amdgcn_rcpf(1.f + fast_exp2(-z * kLog2e));
}

// ------------------------------------------------------------------------------------------- bursts
// How a SIMD of gfx950 issues vector instructions decides the shape of this kernel.  Measured with register-only loops: a
// plain fp32 instruction of a wave takes 2 cycles as long as ANOTHER wave of the SIMD has a plain instruction to issue beside
// it (4.3 cycles for a wave on its own); an exponential takes 8 and a DPP instruction 4, and nothing issues beside them.  When
// every wave mixes the kinds, some wave is nearly always at an exponential and the plain instructions of the others run at the
// unpaired rate: a loop of the scan's own mix (83 plain, 12 DPP, 17 exponentials per state of a 16-step lane) takes 490
// cycles per wave.  Gathered into bursts, and the bursts issued at raised wave priority so that a wave gets through
// its burst before the others go on and the waves' plain stretches fall together, the same instructions take 355, against
// 83 * 2 + 12 * 4.2 + 17 * 8.2 = 356 by the single rates.  Hence: transcendentals and DPP chains below are written as asm blocks
// that raise the priority, run the burst and lower it again.
#define COREY_BURST(body) "s_setprio 1\n\t" body "s_setprio 0"
#define COREY_T(op, n) op " %" #n ", %" #n "\n\t"
#define COREY_T4(op, a, b, c, d) COREY_T(op, a) COREY_T(op, b) COREY_T(op, c) COREY_T(op, d)
#define COREY_T16(op) COREY_T4(op, 0, 1, 2, 3) COREY_T4(op, 4, 5, 6, 7) COREY_T4(op, 8, 9, 10, 11) COREY_T4(op, 12, 13, 14, 15)
#define COREY_V4(v, i) "+v"(v[i]), "+v"(v[i + 1]), "+v"(v[i + 2]), "+v"(v[i + 3])
#define COREY_V16(v) COREY_V4(v, 0), COREY_V4(v, 4), COREY_V4(v, 8), COREY_V4(v, 12)
// (a result of the last transcendental may be read one wait state later: the s_setprio 0 is that wait state)
#define COREY_BURST_FN(name, op)                                                                                             \
    template <int K> __device__ __forceinline__ void name(float (&v)[K])                                                     \
    {                                                                                                                        \
        if constexpr (K == 16) asm volatile(COREY_BURST(COREY_T16(op)) : COREY_V16(v));                                      \
        else if constexpr (K == 8)                                                                                           \
            asm volatile(COREY_BURST(COREY_T4(op, 0, 1, 2, 3) COREY_T4(op, 4, 5, 6, 7)) : COREY_V4(v, 0), COREY_V4(v, 4));   \
        else asm volatile(COREY_BURST(COREY_T4(op, 0, 1, 2, 3)) : COREY_V4(v, 0));                                           \
        static_assert(K == 4 || K == 8 || K == 16, "steps per lane");                                                        \
    }
COREY_BURST_FN(exp2_burst, "v_exp_f32_e32")
COREY_BURST_FN(log2_burst, "v_log_f32_e32")
COREY_BURST_FN(rcp_burst, "v_rcp_f32_e32")
// ... of K decays and the one over the lane's whole sub-block.  FIRST raises the priority and LAST lowers it (several states'
// bursts one after another).
template <int K, bool FIRST, bool LAST> __device__ __forceinline__ void decay_burst(float (&v)[K], float& p)
{
    static_assert(K == 4 || K == 8 || K == 16, "steps per lane");
#define COREY_DECAYS(body, ...)                                                                              \
    do {                                                                                                     \
        if constexpr (FIRST && LAST) asm volatile("s_setprio 1\n\t" body "s_setprio 0" : __VA_ARGS__);       \
        else if constexpr (FIRST) asm volatile("s_setprio 1\n\t" body "s_nop 0" : __VA_ARGS__);              \
        else if constexpr (LAST) asm volatile(body "s_setprio 0" : __VA_ARGS__);                             \
        else asm volatile(body "s_nop 0" : __VA_ARGS__);                                                     \
    } while (0)
    if constexpr (K == 16) COREY_DECAYS(COREY_T16("v_exp_f32_e32") COREY_T("v_exp_f32_e32", 16), COREY_V16(v), "+v"(p));
    else if constexpr (K == 8)
        COREY_DECAYS(COREY_T4("v_exp_f32_e32", 0, 1, 2, 3) COREY_T4("v_exp_f32_e32", 4, 5, 6, 7) COREY_T("v_exp_f32_e32", 8),
                     COREY_V4(v, 0), COREY_V4(v, 4), "+v"(p));
    else COREY_DECAYS(COREY_T4("v_exp_f32_e32", 0, 1, 2, 3) COREY_T("v_exp_f32_e32", 4), COREY_V4(v, 0), "+v"(p));
#undef COREY_DECAYS
}

// softplus() and y *= silu(z) of a lane's K steps, stage by stage so that the transcendentals form bursts.
template <int K> __device__ __forceinline__ void softplus_all(float (&x)[K])
{
    float w[K], fix[K];
#pragma unroll
    for (int i = 0; i < K; ++i) w[i] = -fabsf(x[i]) * kLog2e;
    exp2_burst<K>(w);
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const float e = w[i];
        w[i] = 1.f + e;
        fix[i] = e - (w[i] - 1.f);
        asm("v_max_f32_e32 %0, 0, %1" : "=v"(x[i]) : "v"(x[i]));
    }
    log2_burst<K>(w);
#pragma unroll
    for (int i = 0; i < K; ++i) x[i] += fmaf(w[i], kLn2, fix[i]);
}

template <typename T, int K> __device__ __forceinline__ void gate_all(const Raw<T, K>& z_raw, float (&y)[K])
{
    float z[K], s[K];
    widen<T, K>(z_raw, z);
#pragma unroll
    for (int i = 0; i < K; ++i) s[i] = -z[i] * kLog2e;
    exp2_burst<K>(s);
#pragma unroll
    for (int i = 0; i < K; ++i) s[i] = 1.f + s[i];
    rcp_burst<K>(s);
#pragma unroll
    for (int i = 0; i < K; ++i) y[i] *= z[i] * s[i];
}

// ------------------------------------------------------------------------------------------- lane scan (DPP)
// Inclusive scan, over the SEG consecutive lanes of a row inside one wave, of the per-lane affine maps
// x -> P x + h (oldest lane first), and the fetch of the left neighbour's result: a Hillis-Steele scan whose steps are
// single DPP instructions,
//     h += h[lane - s] * P ;  P *= P[lane - s] ;
// lanes without a source (DPP bound control off) keep their value, which is composing with the identity.  The last step
// leaves P stale (only h is wanted afterwards).  `left` holds the state entering the row's first lane and leaves as the
// state entering this lane's sub-block: the neighbour's h, unchanged in the first lane.
// The instructions are written out because the hazard rules matter: a DPP source register needs two wait
// states after the VALU write that produced it (inside a step pair: the other instruction plus s_nop 0), and
// five after a VALU write of EXEC (s_setprio and s_nop 3 up front).
#define COREY_DPP_H(ctrl) "v_fmac_f32_dpp %0, %0, %1 " ctrl " bank_mask:0xf\n\t"
#define COREY_DPP_P(ctrl) "v_mul_f32_dpp %1, %1, %1 " ctrl " bank_mask:0xf\n\t"
#define COREY_DPP_STEP(ctrl) COREY_DPP_H(ctrl) COREY_DPP_P(ctrl) "s_nop 0\n\t"
#define COREY_ROW_STEPS3                                                                   \
    COREY_DPP_STEP("row_shr:1 row_mask:0xf") COREY_DPP_STEP("row_shr:2 row_mask:0xf")      \
    COREY_DPP_STEP("row_shr:4 row_mask:0xf")

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}

// ... two of them at a time: each fills the other's wait states
#define COREY_DPP2_H(ctrl) COREY_DPP_H(ctrl) "v_fmac_f32_dpp %3, %3, %4 " ctrl " bank_mask:0xf\n\t"
#define COREY_DPP2_STEP(ctrl)                                                               \
    COREY_DPP2_H(ctrl) COREY_DPP_P(ctrl) "v_mul_f32_dpp %4, %4, %4 " ctrl " bank_mask:0xf\n\t"
#define COREY_ROW2_STEPS3                                                                   \
    COREY_DPP2_STEP("row_shr:1 row_mask:0xf") COREY_DPP2_STEP("row_shr:2 row_mask:0xf")     \
    COREY_DPP2_STEP("row_shr:4 row_mask:0xf")
#define COREY_DPP2_LEFT(ctrl)                                                               \
    "v_mov_b32_dpp %2, %0 " ctrl "\n\tv_mov_b32_dpp %5, %3 " ctrl "\n\t"

template <int SEG>
__device__ __forceinline__ void scan_segment(int jseg, float& P, float& h, float& left)
{
    if constexpr (SEG == 64) {
        asm volatile(COREY_BURST("s_nop 3\n\t" COREY_ROW_STEPS3 COREY_DPP_STEP("row_shr:8 row_mask:0xf")
                                 COREY_DPP_STEP("row_bcast:15 row_mask:0xa") COREY_DPP_H("row_bcast:31 row_mask:0xc") "s_nop 1\n\t"
                                 "v_mov_b32_dpp %2, %0 wave_shr:1 row_mask:0xf bank_mask:0xf\n\t")
                     : "+v"(h), "+v"(P), "+v"(left));
    } else if constexpr (SEG == 32) {
        // DPP rows are 16 lanes: a shift by one inside every row leaves the rows' first lanes alone; the odd rows' first lanes
        // (16, 48) take the last lane of the row before them first (row_bcast:15 on rows 1 and 3, limited by the bank mask to
        // lanes 0..3 of the row, of which 1..3 are overwritten by the shift that follows)
        asm volatile(COREY_BURST("s_nop 3\n\t" COREY_ROW_STEPS3 COREY_DPP_STEP("row_shr:8 row_mask:0xf")
                                 COREY_DPP_H("row_bcast:15 row_mask:0xa") "s_nop 1\n\t"
                                 "v_mov_b32_dpp %2, %0 row_bcast:15 row_mask:0xa bank_mask:0x1\n\t"
                                 "v_mov_b32_dpp %2, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\t")
                     : "+v"(h), "+v"(P), "+v"(left));
    } else if constexpr (SEG == 16) {
        asm volatile(COREY_BURST("s_nop 3\n\t" COREY_ROW_STEPS3 COREY_DPP_H("row_shr:8 row_mask:0xf") "s_nop 1\n\t"
                                 "v_mov_b32_dpp %2, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\t")
                     : "+v"(h), "+v"(P), "+v"(left));
    } else if constexpr (SEG > 1) {
        // segments shorter than a DPP row: the shifted-in partner must come from the same segment
        {
            const float ho = dpp_move<0x111>(h), Po = dpp_move<0x111>(P);        // row_shr:1
            const bool take = jseg >= 1;
            h = take ? fmaf(P, ho, h) : h;
            P = take ? P * Po : P;
        }
        if constexpr (SEG > 2) {
            const float ho = dpp_move<0x112>(h), Po = dpp_move<0x112>(P);        // row_shr:2
            const bool take = jseg >= 2;
            h = take ? fmaf(P, ho, h) : h;
            P = take ? P * Po : P;
        }
        if constexpr (SEG > 4) {
            const float ho = dpp_move<0x114>(h), Po = dpp_move<0x114>(P);        // row_shr:4
            const bool take = jseg >= 4;
            h = take ? fmaf(P, ho, h) : h;
            P = take ? P * Po : P;
        }
        const float ho = dpp_move<0x111>(h);
        left = jseg == 0 ? left : ho;
    }
}

template <int SEG, int Q>
__device__ __forceinline__ void scan_segments(int jseg, float (&P)[Q], float (&h)[Q], float (&left)[Q])
{
    if constexpr (Q == 1 || SEG < 16) {
#pragma unroll
        for (int q = 0; q < Q; ++q) scan_segment<SEG>(jseg, P[q], h[q], left[q]);
    } else {
        static_assert(Q % 2 == 0, "states at a time");
#pragma unroll
        for (int q = 0; q < Q; q += 2) {
            if constexpr (SEG == 64)
                asm volatile(COREY_BURST("s_nop 3\n\t" COREY_ROW2_STEPS3 COREY_DPP2_STEP("row_shr:8 row_mask:0xf")
                                         COREY_DPP2_STEP("row_bcast:15 row_mask:0xa") COREY_DPP2_H("row_bcast:31 row_mask:0xc") "s_nop 0\n\t"
                                         COREY_DPP2_LEFT("wave_shr:1 row_mask:0xf bank_mask:0xf"))
                             : "+v"(h[q]), "+v"(P[q]), "+v"(left[q]), "+v"(h[q + 1]), "+v"(P[q + 1]), "+v"(left[q + 1]));
            else if constexpr (SEG == 32)
                asm volatile(COREY_BURST("s_nop 3\n\t" COREY_ROW2_STEPS3 COREY_DPP2_STEP("row_shr:8 row_mask:0xf")
                                         COREY_DPP2_H("row_bcast:15 row_mask:0xa") "s_nop 0\n\t"
                                         COREY_DPP2_LEFT("row_bcast:15 row_mask:0xa bank_mask:0x1")
                                         COREY_DPP2_LEFT("row_shr:1 row_mask:0xf bank_mask:0xf"))
                             : "+v"(h[q]), "+v"(P[q]), "+v"(left[q]), "+v"(h[q + 1]), "+v"(P[q + 1]), "+v"(left[q + 1]));
            else
                asm volatile(COREY_BURST("s_nop 3\n\t" COREY_ROW2_STEPS3 COREY_DPP2_H("row_shr:8 row_mask:0xf") "s_nop 0\n\t"
                                         COREY_DPP2_LEFT("row_shr:1 row_mask:0xf bank_mask:0xf"))
                             : "+v"(h[q]), "+v"(P[q]), "+v"(left[q]), "+v"(h[q + 1]), "+v"(P[q + 1]), "+v"(left[q + 1]));
        }
    }
}

// The state goes from a row's last lane to its first through LDS, between two tiles or, in a row of a single group of states, two
// statements.  A row lies inside one wave, whose LDS accesses are done in order: no wait and no barrier, only the compiler has
// to leave them in that order.
__device__ __forceinline__ void carry_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); }

// ------------------------------------------------------------------------------------------- kernel arguments
// How a launch takes one tile.
struct RowPlan {
    int32_t d16;            // channels below d16 take 16 steps per lane, the others klo (see plan_d16)
    int32_t g16;            // workgroups of the launch that take those
    int32_t klo;            // 8 or 4 (see plan_klo)
    int32_t split;          // the states of a channel are shared by two rows (see plan_split)
};
inline RowPlan row_plan(int64_t B, int64_t D, int64_t N, int chunk, int rows_cap, int allow_split)
{
    const int64_t d16 = plan_d16(B, D, chunk, rows_cap);
    const int klo = plan_klo(B, D, chunk, d16);
    return RowPlan{(int32_t)d16, 0, klo, plan_split(B, D, (int)N, chunk, d16, klo, allow_split)};
}

// ... and every tile, for a chunk read from device memory (chunks walked in the same tiles are taken the same way).  Worked out on the
// host: on the GPU its divisions were 800 scalar instructions between the chunk and the first request for data.  Direct launches read the
// flags only: what a kernel has to know is in the way of its first request, too.
constexpr int kPlans = 7;
static_assert(COREY_MIN_CHUNK == 16 && kMaxTile == 16 << (kPlans - 1), "a plan for every tile");
__host__ __device__ constexpr int plan_index(int tile) { return 27 - __builtin_clz((unsigned)tile); }
struct Plans {
    uint32_t split, four;   // bit plan_index(tile): split; klo is 4
    int32_t d16[kPlans], g16[kPlans];
    void set(int tile, const RowPlan& r)
    {
        const int i = plan_index(tile);
        split = (split & ~(1u << i)) | (uint32_t)(r.split != 0) << i;
        four = (four & ~(1u << i)) | (uint32_t)(r.klo == 4) << i;
        d16[i] = r.d16;
        g16[i] = r.g16;
    }
    __host__ __device__ RowPlan get(int tile) const
    {
        const int i = plan_index(tile);
        return RowPlan{d16[i], g16[i], four >> i & 1u ? 4 : 8, (int32_t)(split >> i & 1u)};
    }
};

struct ScanArgs {
    const void* u;
    const void* delta;
    const float* A;
    const void* Bm;
    const void* Cm;
    const float* Dv;
    const void* z;
    const float* dbias;
    const float* h0;
    const int32_t* seqlens;
    const int32_t* chunks_dev;
    void* y;
    float* last_state;
    float* ws_B;            // relaid-out fp32 B, [B][N * Lpad]
    float* ws_C;
    float* ws_B8;           // the same operands in the order of the 8- or 4-step rows of this launch (ws_B / ws_C: the 16-step ones)
    float* ws_C8;
    RowPlan host;           // of the host chunk
    Plans plans;            // of every tile if the chunk is read from device memory, else of the host chunk's (for the relayout)
    int32_t direct;         // B and C are read as stored (see kDirectRows); the workspace is not used
    int64_t L, Lpad;
    int64_t rows_total;     // B * D (input of the items-per-lane rule)
    int32_t D, N;
    int32_t Np;             // N rounded up to whole staging groups (a multiple of 4); states N..Np-1 are zero padding
    int32_t chunk;          // host chunk (also the fallback for invalid device entries)
    int32_t rows_cap;       // most rows a workgroup may hold (LDS budget for the carried state)
    int32_t softplus;
    int32_t allow_structured;   // take the power-chain path when A[d, n] = (n + 1) A[d, 0] (16-bit storage only)
    int32_t one_chunk;      // chunks_dev holds a single entry that applies to every sequence
    corey_finalise::Args route;   // route.parts != NULL: the statistic's reduction and the chunk rule run at the start of this call
};

__device__ __forceinline__ int resolve_chunk(const ScanArgs& a, int b)
{
    int chunk = a.chunk;
    if (a.chunks_dev) {
        const int c = a.chunks_dev[a.one_chunk ? 0 : b];
        if (c >= COREY_MIN_CHUNK && c <= COREY_MAX_CHUNK && (c & (c - 1)) == 0) chunk = c;
    }
    return chunk;
}

// Workspace layout of one operand for sequence b, chunk c (lpr = c / K lanes per row): value (n, t) of tile
// tau = t / c lives at   b*N*Lpad + tau*N*c + ((n*(K/4) + q) * lpr + j) * 4 + e,   t - tau*c = j*K + q*4 + e.
// For a fixed quarter q of a lane's K steps consecutive lanes j read consecutive 16-byte words, the values
// of one state are c consecutive floats and a group of states of one tile is one contiguous block, so a
// workgroup stages it with straight 16-byte copies.  Steps at or beyond the sequence length are written as 0, and so
// are the padding states N..Np-1 (N here is the padded count Np): with B = C = 0 they contribute nothing.
template <typename T>
__global__ __launch_bounds__(256) void k_relayout_bc(const T* __restrict__ Bm, const T* __restrict__ Cm, float* __restrict__ ws_B,
                                                     float* __restrict__ ws_C, float* __restrict__ ws_B8, float* __restrict__ ws_C8,
                                                     const int32_t* __restrict__ seqlens, const int32_t* __restrict__ chunks_dev,
                                                     int one_chunk, int chunk_host, const Plans plans, int64_t Bn, int64_t D,
                                                     int Nreal, int N, int64_t L, int64_t Lpad, corey_finalise::Args route)
{
    const int b = blockIdx.y;
    int chunk = chunk_host;
    if (route.parts) {
        // the end of the entropy statistic, left to this kernel: every workgroup reduces the partial histograms of its
        // sequence's statistic and applies the chunk rule (all arrive at the same chunk); the first one publishes counts, H,
        // r and the chunk, which is where the scan kernel that follows reads it.  The partial histograms are read by all
        // workgroups here, so clearing them for the next call is left to that scan kernel.
        route.rezero = 0;
        const bool first = blockIdx.x == 0 && (route.nh > 1 || b == 0);
        const int c = corey_finalise::finalise(route, route.nh > 1 ? b : 0, first);
        if (c >= COREY_MIN_CHUNK && c <= COREY_MAX_CHUNK && (c & (c - 1)) == 0) chunk = c;
    } else if (chunks_dev) {
        const int c = chunks_dev[one_chunk ? 0 : b];
        if (c >= COREY_MIN_CHUNK && c <= COREY_MAX_CHUNK && (c & (c - 1)) == 0) chunk = c;
    }
    chunk = tile_of(chunk, Bn * D);                              // the layout is by the tiles the scan walks
    const int klo = plans.four >> plan_index(chunk) & 1u ? 4 : 8;
    int d16 = 0;
#pragma unroll
    for (int i = 0; i < kPlans; ++i) {                           // (an index into the argument would have it copied to scratch memory)
        int di = plans.d16[i];
        asm("" : "+s"(di));
        if (plan_index(chunk) == i) d16 = di;
    }
    int64_t len = L;
    if (seqlens) {
        const int64_t sl = seqlens[b];
        len = sl < 0 ? 0 : (sl > L ? L : sl);
    }
    const int slots_log2 = __ffs(chunk / 4) - 1;                 // 16-byte slots per (tile, state)
    const int64_t ntiles = (len + chunk - 1) / chunk;            // tiles the scan will actually visit
    const int64_t total = (ntiles * N) << slots_log2;
    const T* Bs = Bm + (int64_t)b * Nreal * L;
    const T* Cs = Cm + (int64_t)b * Nreal * L;
    struct Quad { T v[4]; };
    for (int pass = 0; pass < 2; ++pass) {                       // the order of the 16-step rows, then that of the others
        const int K = pass == 0 ? 16 : (klo == 8 ? 8 : 4);       // 4 or fewer steps per lane read B / C in time order
        if (pass == 0 ? d16 <= 0 : d16 >= D) continue;           // no channel of this sequence uses it
        if (chunk < K) continue;
        const int lpr = chunk / K;
        const int lpr_log2 = __ffs(lpr) - 1;
        float4v* oB = reinterpret_cast<float4v*>((pass == 0 ? ws_B : ws_B8) + (int64_t)b * N * Lpad);
        float4v* oC = reinterpret_cast<float4v*>((pass == 0 ? ws_C : ws_C8) + (int64_t)b * N * Lpad);
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
            const int slot = (int)(i & ((1 << slots_log2) - 1));
            const int64_t tn = i >> slots_log2;                  // tau * N + n
            const int64_t tau = tn / N;
            const int n = (int)(tn - tau * N);
            const int j = slot & (lpr - 1);
            const int q = slot >> lpr_log2;
            const int64_t t = n < Nreal ? tau * chunk + (int64_t)j * K + q * 4 : len;     // padding states read nothing
            const T* pb = Bs + (int64_t)n * L + t;
            const T* pc = Cs + (int64_t)n * L + t;
            float4v vb, vc;
            if (t + 4 <= len) {                      // four values of each operand in one load
                Quad qb, qc;
                __builtin_memcpy(&qb, pb, sizeof(Quad));
                __builtin_memcpy(&qc, pc, sizeof(Quad));
                vb.x = Io<T>::ld(&qb.v[0]); vb.y = Io<T>::ld(&qb.v[1]); vb.z = Io<T>::ld(&qb.v[2]); vb.w = Io<T>::ld(&qb.v[3]);
                vc.x = Io<T>::ld(&qc.v[0]); vc.y = Io<T>::ld(&qc.v[1]); vc.z = Io<T>::ld(&qc.v[2]); vc.w = Io<T>::ld(&qc.v[3]);
            } else {
                vb.x = (t + 0 < len) ? Io<T>::ld(pb + 0) : 0.f; vb.y = (t + 1 < len) ? Io<T>::ld(pb + 1) : 0.f;
                vb.z = (t + 2 < len) ? Io<T>::ld(pb + 2) : 0.f; vb.w = (t + 3 < len) ? Io<T>::ld(pb + 3) : 0.f;
                vc.x = (t + 0 < len) ? Io<T>::ld(pc + 0) : 0.f; vc.y = (t + 1 < len) ? Io<T>::ld(pc + 1) : 0.f;
                vc.z = (t + 2 < len) ? Io<T>::ld(pc + 2) : 0.f; vc.w = (t + 3 < len) ? Io<T>::ld(pc + 3) : 0.f;
            }
            oB[i] = vb;
            oC[i] = vc;
        }
    }
}

// Start the copy of NFLOAT consecutive floats (a multiple of 4) of each operand from the workspace into an LDS
// staging buffer.  Every wave copies 64 sixteen-byte words per instruction; the words go from global memory to
// LDS without passing through registers and are complete when the wave's vmcnt reaches zero.
template <int NFLOAT, bool SCALAR_BASE>
__device__ __forceinline__ void stage_async(const float* __restrict__ srcB, const float* __restrict__ srcC, float* dstB,
                                            float* dstC, int wave, int lane)
{
    constexpr int SLOTS = NFLOAT / 4;
#pragma unroll
    for (int s0 = 0; s0 < SLOTS; s0 += kBlock) {
        const int s = s0 + wave * 64;
        if (SLOTS % kBlock == 0 || s + lane < SLOTS) {
            // uniform base + 32-bit lane offset in bytes
            uint32_t voff = (uint32_t)(s + lane) * 16u;
            // SCALAR_BASE: the empty asm keeps the offset from being widened to 64 bits outside the tile loop, so that the
            // copy uses its scalar-base addressing mode; otherwise the compiler adds base and offset with one vector
            // instruction per copy.  Tiles of 1024 stage few states per group and gain from it (-7 %, measured
            // on 5120 channels while those walked such tiles); at 512 and below the other schedule measured 1 % faster.
            if constexpr (SCALAR_BASE) asm volatile("" : "+v"(voff));
            __builtin_amdgcn_global_load_lds(reinterpret_cast<const char*>(srcB) + voff, dstB + (size_t)s * 4, 16, 0, 0);
            __builtin_amdgcn_global_load_lds(reinterpret_cast<const char*>(srcC) + voff, dstC + (size_t)s * 4, 16, 0, 0);
        }
    }
}

// Whether every lane of the workgroup holds a nonzero value; a barrier.  (Another barrier has to pass before the next call.)
__device__ __forceinline__ bool all_lanes(int v)
{
    __shared__ int s_all[kWaves];
    const bool wave_all = __all(v);
    if ((threadIdx.x & 63) == 0) s_all[threadIdx.x >> 6] = wave_all;
    __syncthreads();
    int all = 1;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) all &= s_all[w];
    return __builtin_amdgcn_readfirstlane(all) != 0;
}

// Floats of dynamic LDS one workgroup of the (K, CHUNK) geometry needs for `rows` rows of N states.
template <int K, int CHUNK>
__host__ __device__ constexpr int lds_floats(int rows, int N, bool split, bool direct)
{
    // N: padded state count; a split launch adds the partial y of the rows that hold the second half of the states
    return (direct ? 0 : 4 * Geo<K, CHUNK>::STAGE) + 2 * rows * N + N + kMaxGroup * kBlock + N + (split ? (direct ? 2 : 1) * (kBlock / 2) * K : 0);
}

// ------------------------------------------------------------------------------------------- the scan
// What a lane has before the walk begins: its parameters, and in direct launches of lanes of up to 8 steps its first tile as stored.
template <typename T, int K> struct FirstTile {
    Raw<T, K> u, delta;
    float bias, Dd;
};

// The start of a group of rows is trips to memory with nothing beside them, so they are made together: the first tile, the rows'
// parameters, A with what decides its structure, and the carried state.  Returns whether every row has the structured A; the LDS
// arrays are there.  (Lane numbers are worked out here and again in the walk: kept for it, they would fill its registers.)
// With the plan of a routed tile from the host instead of the device, against structure, arrays and first tile one after another: scan
// of 1024 fp16 rows of 4096 steps at chunk 512 29.7 -> 28.6 us; routed layers, bf16, 1536 rows of 2048 steps 39.5 -> 37.4, 2048 of 977
// 34.9 -> 33.6, steps of 8192 rows of 4096 170.5 -> 167.1, two padded sequences of 4096 rows 207.1 -> 204.3.  Staged launches and lanes
// of 16 steps (the first two of these layers) ask for their first tile in the walk: 16 registers kept until then spill there (41.4 us
// and 34.6).
template <typename T, int K, int CHUNK, bool SPLIT, bool DIRECT>
__device__ __forceinline__ bool start_group(const ScanArgs& a, float* s_mem, const int rows, const int d0, FirstTile<T, K>& first)
{
    constexpr int LPR = Geo<K, CHUNK>::LPR;
    constexpr int STAGE = DIRECT ? 0 : Geo<K, CHUNK>::STAGE;
    const int b = blockIdx.y;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int row_local = tid / LPR, j = tid % LPR;
    const int ch_local = SPLIT ? row_local >> 1 : row_local;
    const int half = SPLIT ? row_local & 1 : 0;
    const bool active = ch_local < rows && d0 + ch_local < a.D;
    const int rl = active ? ch_local : 0;
    const int N = a.Np, Nreal = a.N;
    const int64_t L = a.L;
    if constexpr (DIRECT && K < 16) {
        // (in a sequence of less than a tile the lanes beyond the row and the one at the end of the tensor read further to the left)
        int64_t at = (int64_t)j * K;
        if (at + K > L && (at >= L || (b == (int)gridDim.y - 1 && d0 + rl == a.D - 1))) at = L - K;
        const int64_t row = ((int64_t)b * a.D + d0 + rl) * L + at;
        first.u = load_full<T, K>(static_cast<const T*>(a.u) + row);
        first.delta = load_full<T, K>(static_cast<const T*>(a.delta) + row);
    }
    first.bias = (a.dbias && active) ? a.dbias[d0 + ch_local] : 0.f;
    first.Dd = (a.Dv && active && half == 0) ? a.Dv[d0 + ch_local] : 0.f;      // the skip term enters once per channel
    float* s_carry = s_mem + 4 * STAGE;
    float* s_A2 = s_carry + rows * N;
    float* s_zero = s_A2 + rows * N;
    int chain = sizeof(T) == 2 && a.allow_structured ? 1 : 0;   // fp32 storage keeps the one-exponential-per-state path
    const float inv_N = 1.f / (float)N;
    for (int i = tid; i < rows * N; i += kBlock) {
        const int r = (int)(((float)i + 0.5f) * inv_N), n = i - r * N;      // (exact: fewer than 2^14 values)
        const int64_t dd = d0 + r;
        float Av = 0.f, h = 0.f;
        if (dd < a.D && n < Nreal) {
            Av = a.A[dd * Nreal + n];
            if (a.h0) h = a.h0[((int64_t)b * a.D + dd) * Nreal + n];
            if (chain) chain = Av == (float)(n + 1) * a.A[dd * Nreal];
        }
        s_carry[i] = h;
        s_A2[i] = Av * kLog2e;
    }
    for (int i = tid; i < N; i += kBlock) s_zero[i] = 0.f;
    // binary32 has no such path, and no flags in LDS: 16 bytes of them ahead of the staged copies, which then do not begin at LDS address
    // 0, took routed scans of 1536 rows at chunk 16, 2048 steps, from 281 to 291 us
    if constexpr (sizeof(T) == 2) return all_lanes(chain);
    __syncthreads();
    return false;
}

// The rows d0 .. d0 + rows - 1 of sequence blockIdx.y, start to end.
//
// STRUCT: every row of the group has A[d, n] = (n + 1) A[d, 0] (the S4D-real initialisation Mamba starts from, and
// the benchmark's A = -(n + 1)).  Then exp(dl A[d, n]) = exp(dl A[d, 0])^(n + 1): one exponential per time step
// instead of one per (time step, state), the decay of state n following from that of state n - 1 by one multiply
// (likewise the sub-block product P).  The chain adds at most n roundings (about (n + 1) 2^-24 relative) to a decay.
//
// SPLIT: a channel has two rows of the workgroup (neighbours), the first with states [0, N/2), the second with
// [N/2, N); `rows` counts channels.  Both do the per-token work; the second hands its partial y to the first through
// LDS at the end of every tile, and the first adds the skip term, gates and stores.
// DIRECT: B and C are read where they are, as stored: every lane loads the K values of its steps (one or two 16-byte words per
// operand and state, a set of states ahead) and widens them, two instructions per value more than from the fp32 copy.  In
// return there is no staging, no barrier in the loop, and no launch before this one.  Which launches: see kDirectRows.
template <typename T, int K, int CHUNK, bool STRUCT, bool SPLIT, int W, bool DIRECT>
__device__ __forceinline__ void scan_group(const ScanArgs& a, float* s_mem, const int rows, const int d0, const FirstTile<T, K>& first)
{
    using Gm = Geo<K, CHUNK>;
    constexpr int NS = SPLIT ? 2 : 1;                       // rows per channel
    constexpr int LPR = Gm::LPR, SEG = Gm::SEG, G = DIRECT ? (K == 16 ? NS : kMaxGroup) : Gm::G, STAGE = DIRECT ? 0 : Gm::STAGE;
    constexpr int GH = G / NS;                              // states of one row per staging group
    static_assert(!SPLIT || (G >= 2 && Gm::ROWS >= 2), "a split row needs a state of its own in every staging group");
    constexpr int E = K < 4 ? K : 4;                        // staged B / C values a lane reads per LDS instruction
    constexpr int KQ = K / E;
    // States worked on at a time: with two, each fills the other's wait states.  Rows of 8 steps have one where the registers are
    // 128 and two states spill: in binary32, whose stored values take twice the room, inside the loop (4096 rows of 4096 steps at
    // chunk 512: 107.8 us, with one 97.2; at chunk 256 115.4 and 106.7); in 16 bits at tiles of 512, where the spills are at a tile's
    // ends (176 bytes a lane; 4096 rows of 1000 steps 31.4 and 28.3, of 4096 80.5 and 78.7; 2560 rows of 7 steps 20.4 and 17.5), while at 256
    // two states are worth theirs (68 to 72 bytes; 4096 rows of 4096 steps 85.3 and 87.6, of 1000 32.8 and 30.0).
    constexpr bool kTight = K == 8 && W == 4 && !DIRECT && (sizeof(T) == 4 || CHUNK == 512);
    constexpr int Q = K < 16 && GH > 1 && !kTight ? 2 : 1;
    static_assert(GH % Q == 0, "whole sets of states");
    constexpr bool kEarlyC = K < 16 || W < 4;               // C is requested ahead of the folds where there are registers for it
    typedef float BCv __attribute__((ext_vector_type(E)));
    typedef float GHv __attribute__((ext_vector_type(GH)));

    const int b = blockIdx.y;
    // opaque: a kernel holds several of these bodies, and lane numbers computed for all of them in advance would fill the
    // registers of each
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int row_local = tid / LPR;
    const int j = tid % LPR;                                // sub-block of this lane inside the tile
    const int ch_local = SPLIT ? row_local >> 1 : row_local; // channel of this lane inside the group
    const int half = SPLIT ? row_local & 1 : 0;             // which half of the states its row holds
    const int d = d0 + ch_local;
    const bool active = ch_local < rows && d < a.D;
    const int rl = active ? ch_local : 0;                   // safe LDS row for idle lanes
    int N = a.Np;                                           // padded state count: whole staging groups, no tail group
    // The 4-step binary32 kernels: opaque, so that what follows from N and L for the walk is worked out here.  Worked out ahead of the loop
    // over the groups of rows, it filled the scalar registers before the start's first request: sequences of one tile, against the start in
    // several trips, took 1.05 times as long at chunk 64 and 1.04 at 128, with this 1.02 and 1.01; of several tiles 0.94 and 0.96, with
    // this 0.93 and 0.94.
    constexpr bool kOpaque = sizeof(T) == 4 && DIRECT && K == 4 && W == 3;
    if constexpr (kOpaque) asm volatile("" : "+s"(N));
    const int NH = N / NS;                                  // states per row (N is a multiple of 4: whole half-groups)
    const int n_first = half * NH;                          // first state of this lane's row
    const int Nreal = a.N;
    int64_t L = a.L;
    if constexpr (kOpaque) asm volatile("" : "+s"(L));
    int64_t len = L;
    if (a.seqlens) {
        const int64_t s = a.seqlens[b];
        len = s < 0 ? 0 : (s > L ? L : s);
    }

    float* s_stage = s_mem;                                 // [2 buffers][B, C][STAGE] staged fp32 operands
    float* s_carry = s_stage + 4 * STAGE;                   // [rows][N] state carried tile to tile
    float* s_A2 = s_carry + rows * N;                       // [rows][N] A * log2(e)
    float* s_zero = s_A2 + rows * N;                        // [N] zeros: the "carried state" of lanes that are not first in their row
    float* s_sink = s_zero + N;                             // [kMaxGroup * kBlock + N] where lanes that are not last in their row "store" the state
    float* s_ypart = s_sink + kMaxGroup * kBlock + N;       // SPLIT: [K][kBlock / 2] partial y of the second rows
    // u, delta, z and y are addressed as a base that is uniform over the workgroup (the group's first row; it lives in
    // scalar registers and advances by a tile per iteration) plus ONE 32-bit byte offset per lane that never changes
    // (the lane's row inside the group and its sub-block inside a tile): four 64-bit pointers per lane would not fit the
    // register budget of the 16-step geometries.  The host limits the rows of a group so that the offset fits 32 bits.
    const int64_t row0 = ((int64_t)b * a.D + d0) * L;
    const T* u_grp = static_cast<const T*>(a.u) + row0;
    const T* dl_grp = static_cast<const T*>(a.delta) + row0;
    const T* z_grp = a.z ? static_cast<const T*>(a.z) + row0 : nullptr;
    T* y_grp = static_cast<T*>(a.y) + row0;
    const uint32_t lane_off = (uint32_t)(((int64_t)rl * L + (int64_t)j * K) * (int64_t)sizeof(T));
    auto at = [lane_off](const T* uniform_base) __attribute__((always_inline)) {
        return reinterpret_cast<const T*>(reinterpret_cast<const char*>(uniform_base) + lane_off);
    };
    const bool z_on = z_grp != nullptr;
    const float* wsB = (K < 16 ? a.ws_B8 : a.ws_B) + (int64_t)b * N * a.Lpad;    // each kind of row has its own order of B / C
    const float* wsC = (K < 16 ? a.ws_C8 : a.ws_C) + (int64_t)b * N * a.Lpad;
    const float bias = first.bias, Dd = first.Dd;
    const bool sp = a.softplus != 0;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);    // uniform: addresses built from it stay in scalar registers
    const int jseg = lane & (SEG - 1);
    // per-state arrays are indexed with the state's number inside the row: the row's first state is folded into the bases
    const float* A2_row = s_A2 + rl * N + n_first;
    const float* carry_rd = ((active && j == 0) ? s_carry + rl * N : s_zero) + n_first;
    // every lane stores its end-of-sub-block states of a group (a store under a mask in this loop sends the compiler's
    // register allocation to scratch): the row's last lane into the carried state, all others into scratch of their own
    float* carry_wr = (active && j == LPR - 1) ? s_carry + rl * N + n_first : s_sink + tid * kMaxGroup;
    // DIRECT: the set of states after the one being worked on, as stored.  A lane's place inside a row of B / C is a 32-bit
    // offset from a uniform base: its steps of a full tile, or of the row's last part (see Tail)
    const T* Bseq = static_cast<const T*>(a.Bm) + (int64_t)b * N * L;
    const T* Cseq = static_cast<const T*>(a.Cm) + (int64_t)b * N * L;
    const uint32_t half_off = (uint32_t)((int64_t)n_first * L * (int64_t)sizeof(T));
    uint32_t bc_off = 0, bc_off_last = 0;                   // (the latter: in the tensor's last row, see Tail)
    const int n_last = b == (int)gridDim.y - 1 ? NH - 1 : -1;   // the state (of the second half, if there are two) whose row that is
    Raw<T, K> b_nx[Q], c_nx[Q];
    auto fetch = [&](auto full_c, const int n, const int64_t from) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < Q; ++s) {
            const int64_t row = (int64_t)(n + s) * L + from;
            uint32_t off = bc_off;
            if constexpr (!decltype(full_c)::value) off = n + s == n_last ? bc_off_last : bc_off;
            b_nx[s] = load_full<T, K>(reinterpret_cast<const T*>(reinterpret_cast<const char*>(Bseq + row) + off));
            c_nx[s] = load_full<T, K>(reinterpret_cast<const T*>(reinterpret_cast<const char*>(Cseq + row) + off));
        }
    };
    // staging: one block of GH states per row kind and operand, [half][GH][CHUNK]
    auto stage_group = [&](const int64_t tau_s, const int n_s, float* dst) __attribute__((always_inline)) {
        constexpr bool kScalarBase = CHUNK >= 1024;
#pragma unroll
        for (int hs = 0; hs < NS; ++hs) {
            const int64_t off = (tau_s * N + hs * NH + n_s) * CHUNK;
            stage_async<GH * CHUNK, kScalarBase>(wsB + off, wsC + off, dst + hs * GH * CHUNK, dst + STAGE + hs * GH * CHUNK, wave, lane);
        }
    };

    int buf = 0;                                            // staging buffer holding the group about to be used
    const int64_t ntiles = (len + CHUNK - 1) / CHUNK;
    const int64_t nfull = len / CHUNK;                      // tiles that lie inside the sequence: no masks anywhere
    if constexpr (!DIRECT) {
        if (len > 0) stage_group(0, 0, s_stage);
    }

    // Geometries with at most 8 steps per lane have the registers to fetch the next tile's u and delta while the last
    // group of states of the current tile is computed, which takes the HBM latency out of every tile's start.
    constexpr bool kTileAhead = K <= 8;
    // The gate of a partial tile comes with the tile where registers allow: a short sequence is that tile alone, and a request in its
    // last group of states is a trip to memory with little beside it (binary32, 64 rows of 1 step at chunk 16: 10.0 -> 9.3 us).
    constexpr bool kGateFirst = !DIRECT && K < 16;
    Raw<T, K> u_nx, d_nx;
    if constexpr (DIRECT && kTileAhead) {                   // the first tile's; in the walk always those of the next
        u_nx = first.u;
        d_nx = first.delta;
    }
    bool have_nx = false;                                   // staged launches: they hold the next tile's; uniform over the workgroup
    GHv cin_nx, A2_nx;
    if constexpr (DIRECT) {
        cin_nx = *reinterpret_cast<const GHv*>(carry_rd);
        if constexpr (!STRUCT) A2_nx = *reinterpret_cast<const GHv*>(A2_row);
    }
    auto walk_tile = [&](auto full_c, const int64_t tau) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full_c)::value;
        const int64_t tile = tau * CHUNK;
        const int64_t t0 = tile + (int64_t)j * K;
        // the sequence's last, partial tile: valid steps of this lane (within the sequence) and steps that get a y written (within L)
        int nvalid = K, nstore = K;
        Tail<T, K> tail;
        if constexpr (!FULL) {
            nvalid = nstore = 0;
            if (active) {
                nvalid = (t0 >= len) ? 0 : (len - t0 < K ? (int)(len - t0) : K);
                nstore = (t0 >= L) ? 0 : (L - t0 < K ? (int)(L - t0) : K);
            }
            tail.init(L, t0, nvalid);
        }
        // Where this lane's vectors start: its steps; in the partial tile no lane reads beyond the tensor (L < K: value by value)
        const int64_t t0_last = FULL || t0 + K <= L ? t0 : L - K;                   // in the tensor's last row
        const bool in_last = !FULL && b == (int)gridDim.y - 1 && d0 + rl == a.D - 1;    // ... which is this lane's row of u, delta and z
        const int64_t t0_row = FULL || in_last || t0 >= L ? t0_last : t0;
        auto load_row = [&](const T* base) __attribute__((always_inline)) {
            if constexpr (FULL) return load_full<T, K>(at(base + tile));
            if (DIRECT || L >= K) {
                Raw<T, K> r = load_full<T, K>(at(base + tile) + (t0_row - t0));
                if (in_last) tail.place(r);
                return r;
            }
            return load_few<T, K>(at(base + tile), nvalid);
        };
        if constexpr (DIRECT) {
            bc_off = half_off + (uint32_t)((FULL ? (int64_t)j * K : (t0 >= L ? t0_last : t0)) * (int64_t)sizeof(T));
            bc_off_last = half_off + (uint32_t)(t0_last * (int64_t)sizeof(T));
            if (!FULL || tau == 0) fetch(full_c, 0, FULL ? tile : 0);
        }
        float dl[K], du[K], yv[K];
        Raw<T, K> z_raw;                                    // the gate is fetched with the tile and used after the last state
        if (kTileAhead && (DIRECT || (FULL && have_nx))) {  // fetched one tile ago
            if constexpr (!FULL) {
                if (in_last) {
                    tail.place(u_nx);
                    tail.place(d_nx);
                }
                tail.mask(u_nx);
            }
            widen<T, K>(d_nx, dl);
            widen<T, K>(u_nx, du);
        } else {
            Raw<T, K> u_raw = load_row(u_grp), d_raw = load_row(dl_grp);
            if constexpr (kGateFirst && !FULL)
                if (z_on) z_raw = load_row(z_grp);
            if constexpr (!FULL) {
                tail.mask(u_raw);
            }
            widen<T, K>(d_raw, dl);
            widen<T, K>(u_raw, du);
        }
        have_nx = false;
        float S = 0.f;
#pragma unroll
        for (int i = 0; i < K; ++i) dl[i] = dl[i] + bias;
        if (sp) softplus_all<K>(dl);
        if constexpr (!FULL) {
#pragma unroll
            for (int i = 0; i < K; ++i) dl[i] = (i < nvalid) ? dl[i] : 0.f;   // padded steps: dl = 0 -> a = 1, b = 0 (identity)
        }
#pragma unroll
        for (int i = 0; i < K; ++i) {
            yv[i] = Dd * du[i];                             // the skip term D u opens the sum over states
            du[i] = dl[i] * du[i];
            S += dl[i];
        }
        float av_chain[K], P_chain = 1.f, P_base = 1.f;      // STRUCT: decay of the current state, built up state by state
        if constexpr (STRUCT) {
            const float A20 = s_A2[rl * N];
#pragma unroll
            for (int i = 0; i < K; ++i) {
                // a row that starts at state n_first starts its chain at the decay of state 0 to the power n_first
                dl[i] *= A20;
                av_chain[i] = SPLIT ? dl[i] * (float)n_first : 1.f;
            }
            P_base = S * A20;
            if constexpr (SPLIT) {
                P_chain = P_base * (float)n_first;
                decay_burst<K, true, true>(av_chain, P_chain);
            }
            decay_burst<K, true, true>(dl, P_base);                      // from here on dl holds the decay of state 0
        }

        // DIRECT, but for long tiles of binary32: the gate and the next tile of a full one are requested a group before the last, behind that
        // group's request for the next states.  Loads return in order, so requested ahead of those, or in the last group, their trip to
        // memory stood between a wave and its next states or its gate.  Scans of 64 to 3072 rows of 33 to 4096 steps at chunks 16 and 64:
        // 16 bits 0.96 to 0.97 of the time, binary32 0.92 to 0.96; at 256 and 512 the same (binary32 up to 1.06 there: not done); routed to
        // 1024, where a lane of 16 steps asks for the gate alone, 0.98 (layer of 1536 bf16 rows of 2048 steps 37.2 -> 36.0 us).
        // Unconditional, so that the wait for the states can leave them out: without a gate or a next tile they repeat what is there.
        auto request_tile = [&] __attribute__((always_inline)) {
            z_raw = load_full<T, K>(at((z_on ? z_grp : u_grp) + tile));
            if constexpr (kTileAhead) {
                const int64_t next = tau + 1 < nfull ? tile + CHUNK : tile;
                u_nx = load_full<T, K>(at(u_grp + next));
                d_nx = load_full<T, K>(at(dl_grp + next));
            }
        };
        constexpr bool kAhead = DIRECT && FULL && (sizeof(T) == 2 || CHUNK <= 128);    // (takes the last two groups out of their loop)
        if constexpr (DIRECT) {
            auto groups = [&](auto ask_c, const int n_from, const int n_to) __attribute__((always_inline)) {
                for (int n0 = n_from; n0 < n_to; n0 += GH) {
#include "corey_scan_group.h"
                }
            };
            if constexpr (kAhead) {
                if (NH > GH) {
                    groups(std::false_type{}, 0, NH - 2 * GH);
                    groups(std::true_type{}, NH - 2 * GH, NH - GH);
                } else {
                    request_tile();
                }
                groups(std::false_type{}, NH - GH, NH);
            } else {
                groups(std::false_type{}, 0, NH);
            }
        } else {
            const std::false_type ask_c;
            for (int n0 = 0; n0 < NH; n0 += GH) {
#include "corey_scan_group.h"
            }
        }

        if constexpr (SPLIT) {                              // the second row of a channel hands over its part of the sum over states
            // (DIRECT: two buffers in turn, because nothing else separates these reads from the next tile's writes)
            float* yp = s_ypart + (DIRECT ? (int)(tau & 1) * (K * (kBlock / 2)) : 0) + ch_local * LPR + j;
            if (half == 1 && active) {
#pragma unroll
                for (int i = 0; i < K; ++i) yp[i * (kBlock / 2)] = yv[i];
            }
            __syncthreads();                                // (staged: the next tile's barriers separate these reads from its writes)
            if (half == 0 && active) {
#pragma unroll
                for (int i = 0; i < K; ++i) yv[i] += yp[i * (kBlock / 2)];
            }
        }
        const bool writer = active && half == 0;            // the row that gates and stores y

        T* y_lane = const_cast<T*>(at(y_grp + tile));
        if constexpr (FULL) {
            if (!SPLIT || writer) {
                if (z_on) gate_all<T, K>(z_raw, yv);
                if (active) store_items<T, K>(y_lane, K, yv);
            }
        } else if (nstore > 0 && (!SPLIT || writer)) {
            if (nvalid > 0 && z_on) gate_all<T, K>(z_raw, yv);
#pragma unroll
            for (int i = 0; i < K; ++i)
                if (i >= nvalid) yv[i] = 0.f;                // padded positions are written as zero
            store_items<T, K>(y_lane, nstore, yv);
        }
    };
    for (int64_t tau = 0; tau < nfull; ++tau) walk_tile(std::true_type{}, tau);
    if (nfull < ntiles) {
        if constexpr (DIRECT && kTileAhead) {
            if (nfull > 0) {
                const int64_t t0 = nfull * CHUNK + (int64_t)j * K;
                const int64_t back = t0 + K > L && (t0 >= L || (b == (int)gridDim.y - 1 && d0 + rl == a.D - 1)) ? L - K - t0 : 0;
                u_nx = load_full<T, K>(at(u_grp + nfull * CHUNK) + back);
                d_nx = load_full<T, K>(at(dl_grp + nfull * CHUNK) + back);
            }
        }
        walk_tile(std::false_type{}, nfull);
    }

    // tiles wholly beyond the sequence: y is written as zero
    if (active && half == 0) {
        float zero[K];
#pragma unroll
        for (int i = 0; i < K; ++i) zero[i] = 0.f;
        for (int64_t tile = ntiles * CHUNK; tile < L; tile += CHUNK) {
            const int64_t t0 = tile + (int64_t)j * K;
            const int nstore = (t0 >= L) ? 0 : (L - t0 < K ? (int)(L - t0) : K);
            if (nstore > 0) store_items<T, K>(const_cast<T*>(at(y_grp + tile)), nstore, zero);
        }
    }
    __syncthreads();                                         // last writes of the carried state are visible

    for (int i = tid; i < rows * N; i += kBlock) {
        const int r = i / N, n = i - r * N;
        const int dd = d0 + r;
        if (dd < a.D && n < Nreal) a.last_state[((int64_t)b * a.D + dd) * Nreal + n] = s_carry[i];
    }
}

// A workgroup takes groups of `rows` rows of its sequence, grid-stride.  A launch whose grid was sized from the
// run-time chunk gives every workgroup exactly one group; a launch that reads the chunk from device memory sizes
// its grid from the host's hint and is correct for any chunk (more groups than workgroups: some take several in
// turn; fewer: the surplus leaves at once).
template <typename T, int K, int CHUNK, bool SPLIT, int W, bool DIRECT>
__device__ __forceinline__ void scan_rows(const ScanArgs& a, float* s_mem, const int64_t d_first, const int64_t d_end,
                                          const int64_t wg, const int64_t nwg)
{
    constexpr int kChannels = Geo<K, CHUNK>::ROWS / (SPLIT ? 2 : 1);                  // channels of a full group
    const int rows_full = kChannels < a.rows_cap ? kChannels : a.rows_cap;
    for (int64_t d0 = d_first + wg * rows_full; d0 < d_end; d0 += nwg * rows_full) {   // uniform over the workgroup
        const int rows = d_end - d0 < rows_full ? (int)(d_end - d0) : rows_full;     // the range's last group may be short
        FirstTile<T, K> first;
        const bool structured = start_group<T, K, CHUNK, SPLIT, DIRECT>(a, s_mem, rows, (int)d0, first);
        if (sizeof(T) == 2 && structured) scan_group<T, K, CHUNK, true, SPLIT, W, DIRECT>(a, s_mem, rows, (int)d0, first);
        else scan_group<T, K, CHUNK, false, SPLIT, W, DIRECT>(a, s_mem, rows, (int)d0, first);
        __syncthreads();                                     // the LDS arrays are set up afresh for the next group
    }
}

// Launches of at most this many rows read B and C directly (three waves of one row per SIMD): with few waves to fill in, what
// staging costs (a launch before the scan, a barrier per group of states, the copies' share of every wave's issue slots) is
// more than the widening.  Measured in bf16, staged scan plus relayout against direct: 1024 rows of 4096 steps 38 and 32 us, 1536 of
// 2048 28 and 22, 2048 of 4096 50 and 47; 8192 rows of 4096 141 and 147.
// In binary32 a lane of 8 or 16 steps has twice the bytes in flight: two waves per SIMD fit, and the words of a 16-step lane are 64
// bytes apart.  Beyond 1024 rows those launches read directly only where they know that all of their waves fit (4096 steps,
// staged and direct, us: chunk 512, 1536 rows in pairs of rows 50.4 and 58.4, 2048 rows one each 62.3 and 55.0, 2560 rows 67.3 and
// 81.4; chunk 1024, 1536 rows 46.1 and 64.8, 2048 53.6 and 74.9, 3072 66.1 and 110; chunk 256, lanes of 4 steps, a wave a row and three
// waves per SIMD (waves_target), 1536 rows 57.2 and 49.0, 3072 77.6 and 73.8, of 1000 steps 27.9 and 25.1); with the chunk in device
// memory they are staged (chunk 256 76.5 and 100 at 3072 rows, 1024 60 and 77 at 2048; 512 62.6 and 56 there).
constexpr int64_t kDirectRows = 3072, kDirectRowsF32 = 1024, kDirectWavesF32 = 2048;
inline bool direct_launch(int64_t B, int64_t D, int64_t N, int64_t L, bool f32, bool routed, int64_t d16, int klo, int split)
{
    const int64_t rows = B * D;
    if (rows > kDirectRows || N % kMaxGroup != 0 || L < 16) return false;
    if (!f32 || rows <= kDirectRowsF32) return true;
    if (routed || d16 > 0) return false;
    return klo == 4 || rows * (split ? 2 : 1) <= kDirectWavesF32;      // (a row of 8-step lanes is a wave: only tiles of 512 have them here)
}
// The geometries of direct launches (below) are those that the plan gives so few rows.
static_assert(kDirectRows * (256 / 8) / 64 <= kFewWaves, "tiles up to 256 take 4 steps per lane");
static_assert(kDirectRows * (512 / 8) / 64 <= 4096 && kDirectRows * (64 / 16) < 172032, "no 16-step lanes below tiles of 1024");
static_assert(kDirectRows <= kManyRows, "tiles of 1024 are not divided");

// Which geometries the plan can give a launch of either kind.
template <int K, int CHUNK, bool DIRECT> constexpr bool geometry_exists()
{
    if (DIRECT) return (K == 16 && CHUNK == 1024) || (K == 8 && CHUNK == 512) || (K == 4 && CHUNK >= 4 && CHUNK <= 256);
    return CHUNK >= K && (K == 16 || (K == 8 && CHUNK <= 512) || (K == 4 && CHUNK <= 256));
}
template <int K, int CHUNK> constexpr bool split_exists()
{
    return (K == 16 && CHUNK == 1024) || (K == 8 && CHUNK == 512) || (K == 4 && CHUNK >= 4 && CHUNK <= 256);
}

// Waves per SIMD the registers of a kernel leave room for.  512 registers serve 4 waves with 128 each, 3 with 168, 2 with 256.
// Plain instructions of two waves pair only across the two halves a SIMD's waves are dealt to, so 4 waves (2 + 2) use the issue
// slots better than 3, but with 128 registers a 16-step lane cannot hold C ahead of its use.  Measured: 4096 + 1024 rows of
// 16384 steps at chunk 512 (a mixed launch: 3 waves per SIMD whatever the budget) 329 us with 168 registers, 347 with 128; 8192
// rows of 4096 (4 waves per SIMD) 143 and 135.  Direct launches have at most 3 waves per SIMD (binary32 runs of 8 and 16 steps need
// 256 registers, and the dispatch sends them only launches of 2).
template <typename T, int K, int CHUNK, bool DIRECT> constexpr int waves_target()
{
    if (DIRECT) return sizeof(T) == 4 && K != 4 ? 2 : 3;
    return K == 16 && CHUNK > 512 ? 3 : 4;
}

// One geometry, chosen on the host from the run-time chunk.
template <typename T, int K, int CHUNK, bool DIRECT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(waves_target<T, K, CHUNK, DIRECT>()))) void k_scan(const ScanArgs a)
{
    extern __shared__ __align__(16) float s_mem[];
    constexpr int W = waves_target<T, K, CHUNK, DIRECT>();
    if constexpr (split_exists<K, CHUNK>()) {
        if (a.host.split) {
            scan_rows<T, K, CHUNK, true, W, DIRECT>(a, s_mem, 0, a.D, blockIdx.x, gridDim.x);
            return;
        }
    }
    scan_rows<T, K, CHUNK, false, W, DIRECT>(a, s_mem, 0, a.D, blockIdx.x, gridDim.x);
}

template <int CHUNK> __host__ __device__ inline int rows_of(int K, int rows_cap, int split = 0)
{
    const int lpr = CHUNK / K < 1 ? 1 : CHUNK / K;
    const int rows = kBlock / lpr / (split ? 2 : 1);        // channels of a workgroup
    return rows < rows_cap ? rows : rows_cap;
}

// A workgroup takes its share of one sequence's channels: the first g16 those below d16 with 16 steps per lane, the others the
// rest with 8 or 4.  With a grid sized for exactly these two kinds every workgroup has one row group;
// any other grid is still correct (row groups are taken grid-stride within each kind).  Direct launches have one kind of row, a
// geometry for each tile.
template <typename T, int CHUNK, int W, bool DIRECT>
__device__ __forceinline__ void scan_by_kind(const ScanArgs& a, float* s_mem, const RowPlan& plan)
{
    if constexpr (DIRECT) {
        constexpr int K = CHUNK == 1024 ? 16 : (CHUNK == 512 ? 8 : 4);
        static_assert(geometry_exists<K, CHUNK, true>() && split_exists<K, CHUNK>(), "the geometry of direct launches");
        if (plan.split) scan_rows<T, K, CHUNK, true, W, true>(a, s_mem, 0, a.D, blockIdx.x, gridDim.x);
        else scan_rows<T, K, CHUNK, false, W, true>(a, s_mem, 0, a.D, blockIdx.x, gridDim.x);
    } else if (plan.split) {                                     // one kind of row, two rows per channel
        if (plan.d16 >= a.D) {
            if constexpr (split_exists<16, CHUNK>()) scan_rows<T, 16, CHUNK, true, W, false>(a, s_mem, 0, a.D, blockIdx.x, gridDim.x);
        } else if (plan.klo == 8) {
            if constexpr (split_exists<8, CHUNK>()) scan_rows<T, 8, CHUNK, true, W, false>(a, s_mem, 0, a.D, blockIdx.x, gridDim.x);
        } else {
            if constexpr (split_exists<4, CHUNK>()) scan_rows<T, 4, CHUNK, true, W, false>(a, s_mem, 0, a.D, blockIdx.x, gridDim.x);
        }
    } else {
        const int64_t nwg = gridDim.x, g16 = plan.g16;
        const int64_t wg = (int64_t)blockIdx.x - g16;
        if ((int64_t)blockIdx.x < g16) {
            if constexpr (geometry_exists<16, CHUNK, false>()) scan_rows<T, 16, CHUNK, false, W, false>(a, s_mem, 0, plan.d16, blockIdx.x, g16);
        } else if (plan.klo == 8) {
            if constexpr (geometry_exists<8, CHUNK, false>()) scan_rows<T, 8, CHUNK, false, W, false>(a, s_mem, plan.d16, a.D, wg, nwg - g16);
        } else {
            if constexpr (geometry_exists<4, CHUNK, false>()) scan_rows<T, 4, CHUNK, false, W, false>(a, s_mem, plan.d16, a.D, wg, nwg - g16);
        }
    }
}

// Both kinds of workgroups in one launch (host chunk, 0 < d16 < D).
template <typename T, int CHUNK>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3))) void k_scan_mix(const ScanArgs a)
{
    extern __shared__ __align__(16) float s_mem[];
    RowPlan plan = a.host;
    plan.split = 0;                                              // (two kinds of rows)
    scan_by_kind<T, CHUNK, 3, false>(a, s_mem, plan);
}

// Per-sequence chunk read from device memory: every geometry of the launch's kind in one kernel, selected per workgroup.
template <typename T, int W, bool DIRECT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(W))) void k_scan_any(const ScanArgs a)
{
    extern __shared__ __align__(16) float s_mem[];
    const int chunk = resolve_chunk(a, blockIdx.y);
    if (a.route.parts && a.route.rezero && blockIdx.x == 0 && blockIdx.y == 0) {
        // the statistic's partial histograms live in the buffer its producer handed over and have been reduced by the kernel
        // before this one: leave them cleared for the next count sweep, which adds into them without a clearing launch
        const int n = a.route.nh * corey_range::kParts * a.route.K;
        for (int i = threadIdx.x; i < n; i += kBlock) a.route.parts[i] = 0u;
    }
#define COREY_CASE(C)                                                                       \
    case C:                                                                                 \
        scan_by_kind<T, C, W, DIRECT>(a, s_mem, a.plans.get(C));                           \
        break;
    switch (tile_of(chunk, a.rows_total)) {
        COREY_CASE(16) COREY_CASE(32) COREY_CASE(64) COREY_CASE(128) COREY_CASE(256) COREY_CASE(512) COREY_CASE(1024)
    default: break;
    }
#undef COREY_CASE
}

// The two large kernels of a storage type have a translation unit of their own (they take as long to compile as the rest).
#define COREY_SCAN_ANY(how, T, W) how template __global__ void k_scan_any<T, W, false>(const ScanArgs);
#ifndef COREY_SCAN_ANY_HERE
COREY_SCAN_ANY(extern, float, 3) COREY_SCAN_ANY(extern, float, 4)
COREY_SCAN_ANY(extern, uint16_t, 3) COREY_SCAN_ANY(extern, uint16_t, 4)
COREY_SCAN_ANY(extern, _Float16, 3) COREY_SCAN_ANY(extern, _Float16, 4)
#endif

// ------------------------------------------------------------------------------------------- launch
struct LaunchPlan {
    int chunk;              // host chunk
    bool routed;            // per-sequence device chunks
    int64_t B, D, N;
    hipStream_t stream;
};

inline int a_np(int64_t N) { return (int)((N + kMaxGroup - 1) / kMaxGroup * kMaxGroup); }

template <int K, int CHUNK, bool DIRECT>
inline void geometry(int64_t nrows, int64_t N, int rows_cap, int split, int64_t& gx, size_t& lds)
{
    gx = 0;
    lds = 0;
    if constexpr (geometry_exists<K, CHUNK, DIRECT>()) {
        const int full = Geo<K, CHUNK>::ROWS / (split ? 2 : 1);
        int rows = full < rows_cap ? full : rows_cap;
        gx = (nrows + rows - 1) / rows;
        lds = (size_t)lds_floats<K, CHUNK>(rows, a_np(N), split != 0, DIRECT) * sizeof(float);
    }
}

// Grid and LDS of a launch whose channels below d16 take 16 steps per lane and the others klo.
template <int CHUNK, bool DIRECT>
inline void launch_geometry(const LaunchPlan& p, int rows_cap, const RowPlan& r, int64_t& gx, size_t& lds)
{
    gx = 0;
    lds = 0;
    int64_t g = 0;
    size_t l = 0;
    if (r.d16 > 0) {
        geometry<16, CHUNK, DIRECT>(r.d16, p.N, rows_cap, r.split, g, l);
        gx += g;
        lds = l > lds ? l : lds;
    }
    if (r.d16 < p.D) {
        if (r.klo == 8) geometry<8, CHUNK, DIRECT>(p.D - r.d16, p.N, rows_cap, r.split, g, l);
        else geometry<4, CHUNK, DIRECT>(p.D - r.d16, p.N, rows_cap, r.split, g, l);
        gx += g;
        lds = l > lds ? l : lds;
    }
}

// Workgroups, of nwg, that take the channels below d16.
template <int CHUNK> inline int32_t share16(const LaunchPlan& p, int rows_cap, const RowPlan& r, int64_t nwg)
{
    const int rows16 = rows_of<CHUNK>(16, rows_cap), rows8 = rows_of<CHUNK>(r.klo, rows_cap);
    const int64_t n16 = (r.d16 + rows16 - 1) / rows16, n8 = (p.D - r.d16 + rows8 - 1) / rows8;
    int64_t g16 = n16;
    if (n16 + n8 != nwg) {                                       // a grid sized for another chunk: share it in proportion
        g16 = n8 == 0 ? nwg : (n16 == 0 ? 0 : (nwg * n16 + (n16 + n8) / 2) / (n16 + n8));
        if (n16 > 0 && g16 < 1) g16 = 1;
        if (n8 > 0 && g16 > nwg - 1) g16 = nwg - 1;
    }
    return (int32_t)g16;
}

template <typename T, bool DIRECT>
inline void launch_kernels(ScanArgs& a, const LaunchPlan& p)
{
    int64_t gx = 0, g;
    size_t lds = 0, l;
#define COREY_TILES(p, c)                                                                   \
    switch (tile_of(c, (p).B * (p).D)) {                                                    \
        COREY_CASE(16) COREY_CASE(32) COREY_CASE(64) COREY_CASE(128) COREY_CASE(256) COREY_CASE(512) COREY_CASE(1024)   \
    default: break;                                                                         \
    }
    if (p.routed) {
        // grid from the host's chunk (the caller's hint: workgroups take row groups grid-stride, so any grid is correct),
        // LDS for the largest need of any geometry the plans hold
        for (int c = COREY_MIN_CHUNK; c <= COREY_MAX_CHUNK; c *= 2) {
            g = 0;
            l = 0;
#define COREY_CASE(C)                                                                       \
    case C:                                                                                 \
        launch_geometry<C, DIRECT>(p, a.rows_cap, a.plans.get(C), g, l);          \
        break;
            COREY_TILES(p, c)
#undef COREY_CASE
            lds = l > lds ? l : lds;
            if (c == p.chunk) gx = g;
        }
        if (gx < 2) gx = 2;     // two kinds of rows chosen by the chunk in memory need a workgroup for each kind (a surplus one leaves at once)
        if constexpr (!DIRECT) {
#define COREY_CASE(C) a.plans.g16[plan_index(C)] = share16<C>(p, a.rows_cap, a.plans.get(C), gx);
            COREY_CASE(16) COREY_CASE(32) COREY_CASE(64) COREY_CASE(128) COREY_CASE(256) COREY_CASE(512) COREY_CASE(1024)
#undef COREY_CASE
        }
        const dim3 grid((unsigned)gx, (unsigned)p.B), block(kBlock);
        if constexpr (DIRECT) {
            k_scan_any<T, waves_target<T, 16, 1024, true>(), true><<<grid, block, lds, p.stream>>>(a);
        } else {
            // registers for the long tiles: three waves per SIMD if those give two kinds of rows, or if the sequences' lengths
            // differ (the longest one's waves, a part of the launch, decide: 233 us against 254 for the padded pair); else four
            const int64_t d16_512 = a.plans.get(512).d16;
            if ((d16_512 > 0 && d16_512 < p.D) || a.seqlens) k_scan_any<T, 3, false><<<grid, block, lds, p.stream>>>(a);
            else k_scan_any<T, 4, false><<<grid, block, lds, p.stream>>>(a);
        }
        return;
    }
    const dim3 block(kBlock);
#define COREY_LAUNCH(K, C)                                                                  \
    if constexpr (geometry_exists<K, C, DIRECT>()) k_scan<T, K, C, DIRECT><<<dim3((unsigned)gx, (unsigned)p.B), block, lds, p.stream>>>(a)
    RowPlan& r = a.host;
#define COREY_CASE(C)                                                                       \
    case C:                                                                                 \
        launch_geometry<C, DIRECT>(p, a.rows_cap, r, gx, lds);                               \
        r.g16 = share16<C>(p, a.rows_cap, r, gx);                                            \
        if (r.d16 >= p.D) { COREY_LAUNCH(16, C); }                                          \
        else if (r.d16 > 0) {                                                               \
            if constexpr (!DIRECT && C <= 512) k_scan_mix<T, C><<<dim3((unsigned)gx, (unsigned)p.B), block, lds, p.stream>>>(a);   \
        }                                                                                   \
        else if (r.klo == 8) { COREY_LAUNCH(8, C); }                                        \
        else { COREY_LAUNCH(4, C); }                                                        \
        break;
    COREY_TILES(p, p.chunk)
#undef COREY_CASE
#undef COREY_LAUNCH
#undef COREY_TILES
}

template <typename T>
inline void launch_scan(ScanArgs& a, const LaunchPlan& p)
{
    if (a.direct) {
        launch_kernels<T, true>(a, p);
        return;
    }
    // relayout of B and C: one 16-byte word per lane, enough workgroups to cover the operand a few times over
    int64_t rb = (a.Np * a.Lpad / 4 + 255) / 256;
    rb = rb < 1 ? 1 : (rb > 2048 ? 2048 : rb);
    k_relayout_bc<T><<<dim3((unsigned)rb, (unsigned)p.B), dim3(256), 0, p.stream>>>(
        static_cast<const T*>(a.Bm), static_cast<const T*>(a.Cm), a.ws_B, a.ws_C, a.ws_B8, a.ws_C8, a.seqlens, a.chunks_dev,
        a.one_chunk, p.chunk, a.plans, p.B, p.D, (int)p.N, a.Np, a.L, a.Lpad, a.route);
    launch_kernels<T, false>(a, p);
}

}  // namespace corey_scan
#endif
