// selective_state_update: one generated token, i.e. the scan's recurrence taken for a single step from the carried
// state (the state selective_scan_fwd leaves in last_state), updated in place.
//
// A (sequence, channel) row owns N consecutive binary32 states.  A row is spread over LPR = 2^k lanes, each lane
// taking 16-byte groups of four states (LPR = ceil(N / 4) rounded up to a power of two, at most 64), so a wave reads
// and writes whole contiguous stretches of the state tensor; the row's readout sum_n C[n] h'[n] is folded across
// its lanes with butterfly shuffles and its first lane applies the skip term and the gate.  The arithmetic is the
// scan kernel's: softplus, exp2(dl * (A * log2 e)), one fused multiply-add per state.
// Work bound by the state traffic (8 bytes per state); nothing here is a contraction.
#include <hip/hip_runtime.h>

#include "corey_internal.h"
#include "corey_scan_impl.h"

namespace {

using corey_scan::fast_exp2;
using corey_scan::Io;
using corey_scan::kLog2e;
using corey_scan::silu;
using corey_scan::softplus;

constexpr int kThreads = 256;
typedef float float4v __attribute__((ext_vector_type(4)));

// Sets of 256 lanes a workgroup takes.  Up to a line every set is a workgroup of its own, above it pairs.  One by one and in pairs,
// states from HBM, us: binary32, 5120 channels of 16 states, 26 sequences (2080 sets) 6.4 and 7.2, 40 8.6 and 9.4, 64 (5120 sets) 11.9
// and 12.7, 80 14.3 and 15.3, 96 (7680 sets) 17.7 and 17.8; bf16 26 7.1 and 7.3, 40 9.4 and 9.6, 52 (4160 sets) 11.1 and 11.4, 64
// 12.9 and 12.9 (14.4 and 14.2 with the convolution's step in front), 64 of 1024 channels of 64 states (4096 sets) 11.1 and 10.8.
// More sets than two: 512 sequences (40960 sets, bf16) 72.8 us one by one, 70.9 in pairs, 74.4 in fours, 89.6 in eights.
constexpr int kSets = 2;
template <typename T> constexpr uint64_t many_sets() { return sizeof(T) == 4 ? 6400 : 4000; }

// States in whole, aligned groups of four: U sets of rows per workgroup, every load of theirs issued before any use, B and C by
// words of four values (value by value they are eight loads of two bytes in a lane, and the trips to memory queue behind them).
// Bound by memory: 512 sequences of 5120 channels with 16 states, fresh from HBM, 88.6 -> 70.9 us, 4.1 -> 5.1 TB/s (a copy reaches
// 5.4); 64 sequences 15.0 -> 12.7 us.  Same operations in the same order as below.
template <typename T, int U>
__global__ __launch_bounds__(kThreads) void k_state_update(float* __restrict__ state, const T* __restrict__ x,
                                                           const T* __restrict__ delta, const float* __restrict__ A,
                                                           const T* __restrict__ Bt, const T* __restrict__ Ct,
                                                           const float* __restrict__ Dv, const T* __restrict__ z,
                                                           const float* __restrict__ dbias, T* __restrict__ y, uint32_t rows,
                                                           uint32_t D, int N, int lpr_log2, int use_softplus)
{
    const int LPR = 1 << lpr_log2;                          // 4 LPR >= N: a lane has one group at most
    const int j = (int)threadIdx.x & (LPR - 1);
    const bool on = 4 * j < N;
    const int n = on ? 4 * j : 0;                           // lanes without a group load the row's first and store nothing
    uint32_t row[U];
    bool active[U];
    float4v h[U], a[U];
    T bv[U][4], cv[U][4], xr[U], dr[U], zr[U];
    float bias[U], skip[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const uint32_t r = (uint32_t)((((uint64_t)blockIdx.x * U + k) * kThreads + threadIdx.x) >> lpr_log2);
        active[k] = r < rows;                               // whole rows are active or not: LPR divides the wave
        row[k] = active[k] ? r : rows - 1;
        const uint32_t b = row[k] / D, d = row[k] - b * D;
        h[k] = *reinterpret_cast<const float4v*>(state + (size_t)row[k] * N + n);
        a[k] = *reinterpret_cast<const float4v*>(A + (size_t)d * N + n);
        __builtin_memcpy(bv[k], Bt + (size_t)b * N + n, sizeof(bv[k]));
        __builtin_memcpy(cv[k], Ct + (size_t)b * N + n, sizeof(cv[k]));
        xr[k] = x[row[k]];
        dr[k] = delta[row[k]];
        zr[k] = z ? z[row[k]] : T(0);
        bias[k] = dbias ? dbias[d] : 0.f;
        skip[k] = Dv ? Dv[d] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const float xv = Io<T>::ld(&xr[k]);
        float dl = Io<T>::ld(&dr[k]) + bias[k];
        if (use_softplus) dl = softplus(dl);
        const float dx = dl * xv;
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float hn = fmaf(fast_exp2(dl * (a[k][i] * kLog2e)), h[k][i], dx * Io<T>::ld(&bv[k][i]));
            h[k][i] = hn;
            acc = fmaf(Io<T>::ld(&cv[k][i]), hn, acc);
        }
        if (!on) acc = 0.f;
        if (active[k] && on) *reinterpret_cast<float4v*>(state + (size_t)row[k] * N + n) = h[k];
        for (int m = LPR >> 1; m >= 1; m >>= 1) acc += __shfl_xor(acc, m);
        if (active[k] && j == 0) {
            float yv = acc + (Dv ? skip[k] * xv : 0.f);
            if (z) yv *= silu(Io<T>::ld(&zr[k]));
            Io<T>::st(y + row[k], yv);
        }
    }
}

// Any N and any alignment of the states and of A: value by value.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_state_update_any(float* __restrict__ state, const T* __restrict__ x,
                                                               const T* __restrict__ delta, const float* __restrict__ A,
                                                               const T* __restrict__ Bt, const T* __restrict__ Ct,
                                                               const float* __restrict__ Dv, const T* __restrict__ z,
                                                               const float* __restrict__ dbias, T* __restrict__ y, uint32_t rows,
                                                               uint32_t D, int N, int lpr_log2, int use_softplus)
{
    const uint64_t gid = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
    const uint32_t row = (uint32_t)(gid >> lpr_log2);
    const int LPR = 1 << lpr_log2;
    const int j = (int)(gid & (uint64_t)(LPR - 1));
    const bool active = row < rows;                         // whole rows are active or not: LPR divides the wave
    float acc = 0.f, xv = 0.f;
    uint32_t d = 0;
    if (active) {
        const uint32_t b = row / D;
        d = row - b * D;
        xv = Io<T>::ld(x + row);
        float dl = Io<T>::ld(delta + row) + (dbias ? dbias[d] : 0.f);
        if (use_softplus) dl = softplus(dl);
        const float dx = dl * xv;
        float* hrow = state + (size_t)row * N;
        const float* arow = A + (size_t)d * N;
        const T* brow = Bt + (size_t)b * N;
        const T* crow = Ct + (size_t)b * N;
        for (int i = 4 * j; i < N && i < 4 * j + 4; ++i) {
            const float hn = fmaf(fast_exp2(dl * (arow[i] * kLog2e)), hrow[i], dx * Io<T>::ld(brow + i));
            hrow[i] = hn;
            acc = fmaf(Io<T>::ld(crow + i), hn, acc);
        }
    }
    for (int m = LPR >> 1; m >= 1; m >>= 1) acc += __shfl_xor(acc, m);
    if (active && j == 0) {
        float yv = acc + (Dv ? Dv[d] * xv : 0.f);
        if (z) yv *= silu(Io<T>::ld(z + row));
        Io<T>::st(y + row, yv);
    }
}

template <typename T>
void launch(void* state, const void* x, const void* delta, const float* A, const void* Bt, const void* Ct, const float* Dv,
            const void* z, const float* dbias, void* y, int64_t B, int64_t D, int64_t N, int softplus_on, hipStream_t stream)
{
    static_assert(COREY_MAX_STATE <= 4 * 64, "a lane has one group of four states at most");
    int lpr_log2 = 0;
    while ((1 << lpr_log2) < (N + 3) / 4 && lpr_log2 < 6) ++lpr_log2;
    const bool vector_ok = (N % 4) == 0 && reinterpret_cast<uintptr_t>(state) % 16 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0;
    const uint64_t lanes = (uint64_t)(B * D) << lpr_log2;
    const uint64_t sets = (lanes + kThreads - 1) / kThreads;
    auto go = [&](auto kernel, uint64_t blocks) {
        kernel<<<dim3((unsigned)blocks), dim3(kThreads), 0, stream>>>(
            static_cast<float*>(state), static_cast<const T*>(x), static_cast<const T*>(delta), A, static_cast<const T*>(Bt),
            static_cast<const T*>(Ct), Dv, static_cast<const T*>(z), dbias, static_cast<T*>(y), (uint32_t)(B * D), (uint32_t)D, (int)N,
            lpr_log2, softplus_on);
    };
    if (!vector_ok) go(k_state_update_any<T>, sets);
    else if (sets > many_sets<T>()) go(k_state_update<T, kSets>, (sets + kSets - 1) / kSets);
    else go(k_state_update<T, 1>, sets);
}

}  // namespace

extern "C" int selective_state_update(void* state, const void* x, const void* delta, const float* A, const void* Bt,
                                      const void* Ct, const float* Dv, const void* z, const float* delta_bias,
                                      int32_t delta_softplus, void* y, corey_dtype dt, int64_t B, int64_t D, int64_t N,
                                      void* hip_stream)
{
    using corey::fail;
    if (!state || !x || !delta || !A || !Bt || !Ct || !y)
        return fail(COREY_ENULL, "selective_state_update: state, x, delta, A, Bt, Ct and y are required");
    if (dt != COREY_F32 && dt != COREY_BF16 && dt != COREY_F16) return fail(COREY_EINVAL, "selective_state_update: unknown dtype %d", (int)dt);
    if (B < 1 || D < 1 || N < 1 || N > COREY_MAX_STATE)
        return fail(COREY_ESHAPE, "selective_state_update: B, D >= 1 and 1 <= N <= %d required", COREY_MAX_STATE);
    if ((double)B * (double)D >= 33554432.0)                // 2^25 rows: every index below stays far inside 32 / 64 bits
        return fail(COREY_ESHAPE, "selective_state_update: B*D must stay below 2^25");
    if (reinterpret_cast<uintptr_t>(state) % 4 != 0) return fail(COREY_EINVAL, "selective_state_update: state must be 4-byte aligned");
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const int sp = delta_softplus ? 1 : 0;
    if (dt == COREY_F32) launch<float>(state, x, delta, A, Bt, Ct, Dv, z, delta_bias, y, B, D, N, sp, stream);
    else if (dt == COREY_F16) launch<_Float16>(state, x, delta, A, Bt, Ct, Dv, z, delta_bias, y, B, D, N, sp, stream);
    else launch<uint16_t>(state, x, delta, A, Bt, Ct, Dv, z, delta_bias, y, B, D, N, sp, stream);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return corey::hip_fail(e, "selective_state_update launch");
    return COREY_OK;
}
