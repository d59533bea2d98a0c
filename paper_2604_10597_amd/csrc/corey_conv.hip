// causal_conv1d_silu_fwd: the causal depthwise convolution and SiLU that produce the scan input u, with the range of
// u (what the histogram's first sweep would compute) taken in the same pass.
//
// Three kernels, one launch each:
//   k_conv1d_silu        rows of at least two vectors.  A lane takes 16-byte vectors of consecutive time steps, whichever rows
//                        they fall in, two at a time so that their loads are in flight together.
//   k_conv1d_silu_step   one step (generation): a lane takes the 4 bytes of x that one (fp32) or two rows make up, and the
//                        window of earlier inputs beside them.
//   k_conv1d_silu_short  what is left, a lane per row.
// The taps are accumulated oldest first with fused multiply-adds in binary32, v * sigmoid(v) is rounded once to the storage
// type.  The minimum and maximum are taken over the values as stored (the histogram will see those bits), kept per lane and
// reduced once per workgroup into a partial range; corey_entropy_hist reduces the COREY_RANGE_PARTS partials.
// Bandwidth work (x in, u out): no matrix instructions.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "corey_internal.h"
#include "corey_range.h"
#include "corey_table.h"

namespace {

using corey::bf16_to_f32;
using corey_range::kThreads;
using corey_range::order_key;
using corey_range::Handoff;
using corey_range::RangePart;
using corey_range::reduce_range_keys;

constexpr float kLog2e = 1.4426950408889634f;
typedef uint32_t word4 __attribute__((ext_vector_type(4)));
typedef uint32_t word4e __attribute__((ext_vector_type(4), aligned(2)));     // at any element
typedef float float2v __attribute__((ext_vector_type(2)));

// Storage type: widen one element, round a vector of values (to nearest even), elements per 16-byte vector.
template <typename T> struct St;
template <> struct St<float> {
    static constexpr int kVec = 4;
    static __device__ __forceinline__ float widen(float v) { return v; }
    static __device__ __forceinline__ void narrow(const float (&v)[4], float (&out)[4])
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = v[e];
    }
};
template <> struct St<uint16_t> {                       // bfloat16 bit patterns
    static constexpr int kVec = 8;
    static __device__ __forceinline__ float widen(uint16_t v) { return bf16_to_f32(v); }
    static __device__ __forceinline__ void narrow(const float (&v)[8], uint16_t (&out)[8])
    {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            float2v f;
            f.x = v[e]; f.y = v[e + 1];
            const bf16x2 h = __builtin_convertvector(f, bf16x2);    // v_cvt_pk_bf16_f32
            __builtin_memcpy(&out[e], &h, 4);
        }
    }
};
template <> struct St<_Float16> {
    static constexpr int kVec = 8;
    static __device__ __forceinline__ float widen(_Float16 v) { return (float)v; }
    static __device__ __forceinline__ void narrow(const float (&v)[8], _Float16 (&out)[8])
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float f = v[e];
            asm("" : "+v"(f));      // the binary32 value, which the range follows too, is what is rounded: seen together with the
            out[e] = (_Float16)f;   // product it comes from, the compiler may round that to binary16 in one step (v_fma_mixlo)
        }
    }
};

// min / max that return the other operand when one is NaN (the hardware's IEEE-mode behaviour), without the
// canonicalising extra instruction the generic fminf / fmaxf lowering adds per call
__device__ __forceinline__ float vmin(float a, float b)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float vmax(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

constexpr int H = COREY_MAX_CONV - 1;                     // most earlier inputs a tap reaches back to

// The inputs one lane needs for one vector of outputs, one by one: xs[H + e] = x[t0 + e] and the H inputs before them
// (xs[H - k] = x[t0 - k]), from state_in before the row starts, or zero.
template <typename T>
__device__ __forceinline__ void load_inputs(const T* __restrict__ xr, const T* __restrict__ state_row, int64_t t0, int nvalid,
                                            int W, float (&xs)[H + St<T>::kVec])
{
    constexpr int V = St<T>::kVec;
#pragma unroll
    for (int e = 0; e < V; ++e) xs[H + e] = (e < nvalid) ? St<T>::widen(xr[t0 + e]) : 0.f;
#pragma unroll
    for (int k = 1; k <= H; ++k) {
        const int64_t t = t0 - k;
        float v = 0.f;
        if (t >= 0) v = St<T>::widen(xr[t]);
        else if (state_row && t + (W - 1) >= 0) v = St<T>::widen(state_row[t + (W - 1)]);
        xs[H - k] = v;
    }
}

// One vector of outputs from its inputs: taps oldest first with fused multiply-adds, v * sigmoid(v), one rounding to
// the storage type.  Rounding to nearest is monotonic, so the range of the stored values is the rounded range of the
// unrounded ones: lo / hi follow the binary32 results and are rounded once at the end of the kernel.
template <typename T, int W, bool FULL>
__device__ __forceinline__ void conv_vector(const float (&xs)[H + St<T>::kVec], const float (&w)[W], float bs, int nvalid,
                                            T (&out)[St<T>::kVec], float& lo, float& hi, bool& nan)
{
    constexpr int V = St<T>::kVec;
    float val[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        float acc = bs;
#pragma unroll
        for (int k = 0; k < W; ++k) acc = fmaf(w[k], xs[H + e - (W - 1) + k], acc);
        val[e] = acc * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-acc * kLog2e));
        if (FULL || e < nvalid) {
            nan |= (val[e] != val[e]);
            lo = vmin(lo, val[e]);
            hi = vmax(hi, val[e]);
        }
    }
    St<T>::narrow(val, out);
}

// A lane's position: vector v of row `row`, whose channel is d.  A lane visits every step-th vector (step: the lanes of the
// launch), numbered row * nvec + v; the host divides that stride once (q rows, rem vectors, qd channels), the lane only adds.
struct Cursor {
    int64_t row, v, d;
};
struct Walk {
    int64_t rows, D, L;
    int64_t nvec;            // vectors of a row: ceil(L / V)
    int64_t turns;           // vectors of a lane
    int64_t q, rem, qd;
};
__device__ __forceinline__ Cursor advance(Cursor c, const Walk& s)
{
    c.v += s.rem;
    const int64_t carry = (c.v >= s.nvec) ? 1 : 0;
    c.v -= carry ? s.nvec : 0;
    c.row += s.q + carry;
    c.d += s.qd + carry;
    c.d -= (c.d >= s.D) ? s.D : 0;
    return c;
}
// How a launch of single steps is walked: `groups` groups of channels in each of B sequences; lane l takes group l mod groups of the
// sequences l / groups, l / groups + across, ..., `units` of them at a time.
struct StepWalk {
    int64_t B, groups, lanes;
    uint32_t across;
    int units;
};
// n / d of a lane or workgroup number: 32 bits whatever the tensor (a divisor beyond them gives 0 either way)
__device__ __forceinline__ uint32_t quotient(uint32_t n, int64_t d) { return n / (uint32_t)min(d, (int64_t)0x7fffffff); }

// Count the values of one vector, without its first `skip`, in the workgroup's bit-pattern table (16-bit storage).
template <typename T>
__device__ __forceinline__ void table_add_vector(uint32_t* s_tab, corey_table::Shared& sh, const T (&out)[St<T>::kVec], int skip, int nvalid)
{
    if constexpr (sizeof(T) == 2) {
        if (skip == 0 && nvalid == St<T>::kVec) {
            uint32_t w[4];
            __builtin_memcpy(w, out, 16);
            corey_table::add_word4(s_tab, sh, w);
        } else {
#pragma unroll
            for (int e = 0; e < St<T>::kVec; ++e) {
                if (e >= skip && e < nvalid) {
                    uint16_t bits;
                    __builtin_memcpy(&bits, &out[e], 2);
                    corey_table::add(s_tab, sh, bits);
                }
            }
        }
    }
}

// What a workgroup leaves for the statistic: the extremes rounded once to the storage type, the workgroup's partial range
// (entries no workgroup owns say "nothing seen").
template <typename T> __device__ __forceinline__ void round_extremes(float& lo, float& hi)
{
    if (lo <= hi) {
        float pad[St<T>::kVec];
        T st[St<T>::kVec];
#pragma unroll
        for (int e = 0; e < St<T>::kVec; ++e) pad[e] = (e == 0) ? lo : hi;
        St<T>::narrow(pad, st);
        lo = St<T>::widen(st[0]);
        hi = St<T>::widen(st[1]);
    }
}
template <int NT> __device__ __forceinline__ void write_parts(RangePart* rparts, uint32_t klo, uint32_t khi, uint32_t knan)
{
    if (threadIdx.x == 0) {
        RangePart rp;
        rp.lo_key = klo; rp.hi_key = khi; rp.saw_nan = knan; rp.pad = 0u;
        rparts[blockIdx.x] = rp;
    }
    if (blockIdx.x == 0)
        for (int i = gridDim.x + threadIdx.x; i < COREY_RANGE_PARTS; i += NT) {
            RangePart rp;
            rp.lo_key = 0xffffffffu; rp.hi_key = 0u; rp.saw_nan = 0u; rp.pad = 0u;
            rparts[i] = rp;
        }
}

// NT lanes per workgroup.  A row's last vector is moved back to end with the row, so that every vector is whole: the values it
// shares with the one before are computed and stored twice, with the same bits (and their range is the same).  That needs
// L >= 2 V (the H inputs before a vector that does not start its row are then in the row, too).  Lanes beyond the last vector
// redo it.  No row needs to be aligned: gfx950 takes 16-byte accesses at any element's address.
// TABLE: the workgroup also counts the bit patterns of the values it stores (corey_table.h: NT = corey_table::kLanes, at most
// corey_table::kMaxSlabs workgroups, 16-bit storage; each value once: the shared ones by the vector before); a turn of the
// loop adds at most U * NT * 8 = 16384 values and ends at a barrier, inside the table's bound of 32768 per round.  Rows of
// fewer than two vectors come here with TABLE only, and are read value by value.
template <typename T, int W, int NT, bool TABLE, bool WAVES>
__global__ __launch_bounds__(NT) void k_conv1d_silu(const T* __restrict__ x, const float* __restrict__ weight,
                                                    const float* __restrict__ bias, const T* __restrict__ state_in,
                                                    T* __restrict__ u, T* __restrict__ state_out, Handoff* __restrict__ handoff,
                                                    void* table_ws, const Walk wk)
{
    if (handoff) corey_range::clear_handoff_counts(handoff);   // the statistic's count sweep adds into them
    constexpr int V = St<T>::kVec;
    constexpr int U = 2;                                      // vectors in flight per lane
    constexpr int P = H + 1;                                  // values fetched before a vector: 8 or 16 bytes
    static_assert(!TABLE || (NT == corey_table::kLanes && U * NT * 8 <= corey_table::kRoundAdds && sizeof(T) == 2),
                  "a turn must stay inside the table's round");
    __shared__ uint32_t s_tab[TABLE ? corey_table::kWords : 1];
    __shared__ corey_table::Shared sh;
    corey_table::Workspace tws = {};
    if constexpr (TABLE) {
        tws = corey_table::carve(table_ws);
        corey_table::begin(s_tab, sh, tws);
    }
    const int64_t L = wk.L;
    // WAVES: the position of the wave's first lane, uniform
    const uint32_t tid = WAVES ? __builtin_amdgcn_readfirstlane(threadIdx.x) : threadIdx.x;
    const int64_t sub = WAVES ? threadIdx.x & 63 : 0;
    const uint32_t lane = blockIdx.x * NT + tid;
    Cursor cur;
    cur.row = quotient(lane, wk.nvec);
    cur.v = lane - cur.row * wk.nvec;
    cur.d = cur.row - quotient((uint32_t)cur.row, wk.D) * wk.D;
    float lo = INFINITY, hi = -INFINITY;
    bool nan = false;

    auto vectors = [&](auto nu) {
        constexpr int NU = decltype(nu)::value;
        Cursor c[NU];
        int64_t t0[NU], off[NU];
        bool past[NU];
        T curv[NU][V], prev[NU][P];
        float w[NU][W], bs[NU];
#pragma unroll
        for (int j = 0; j < NU; ++j) {                        // every load of these vectors before any use
            past[j] = cur.row >= wk.rows;
            c[j] = cur;
            if (past[j]) c[j] = Cursor{wk.rows - 1, wk.nvec - (WAVES ? 64 : 1), wk.D - 1};
            cur = advance(cur, wk);
            t0[j] = WAVES ? (c[j].v + sub) * V : min(c[j].v * V, L - V);
            off[j] = c[j].row * L + t0[j];
            __builtin_memcpy(curv[j], x + off[j], 16);
            __builtin_memcpy(prev[j], x + (t0[j] > 0 ? off[j] - P : off[j]), sizeof(T) * P);
            __builtin_memcpy(w[j], weight + c[j].d * W, sizeof(float) * W);
            bs[j] = bias ? bias[c[j].d] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < NU; ++j) {
            float xs[H + V];
#pragma unroll
            for (int e = 0; e < V; ++e) xs[H + e] = St<T>::widen(curv[j][e]);
#pragma unroll
            for (int k = 1; k <= H; ++k) xs[H - k] = St<T>::widen(prev[j][P - k]);
            if ((!WAVES || c[j].v == 0) && t0[j] == 0) {                                 // the row starts here: its past is in state_in, or zero
#pragma unroll
                for (int k = 1; k <= H; ++k)
                    xs[H - k] = (state_in && k <= W - 1) ? St<T>::widen(state_in[c[j].row * (W - 1) + (W - 1 - k)]) : 0.f;
            }
            T out[V];
            conv_vector<T, W, true>(xs, w[j], bs[j], V, out, lo, hi, nan);
            word4 q;
            __builtin_memcpy(&q, out, 16);
            __builtin_nontemporal_store(q, reinterpret_cast<word4e*>(u + off[j]));
            if constexpr (TABLE)
                if (!past[j]) table_add_vector<T>(s_tab, sh, out, (int)(c[j].v * V - t0[j]), V);
        }
    };
    auto values = [&]() {                                     // one vector of a row of fewer than two
        const Cursor c = cur;
        cur = advance(cur, wk);
        if (c.row >= wk.rows) return;
        const T* xr = x + c.row * L;
        const T* sr = state_in ? state_in + c.row * (W - 1) : nullptr;
        const int64_t t0 = c.v * V;
        const int nvalid = (L - t0 < V) ? (int)(L - t0) : V;
        float xs[H + V], w[W];
        load_inputs<T>(xr, sr, t0, nvalid, W, xs);
#pragma unroll
        for (int k = 0; k < W; ++k) w[k] = weight[c.d * W + k];
        T out[V];
        conv_vector<T, W, false>(xs, w, bias ? bias[c.d] : 0.f, nvalid, out, lo, hi, nan);
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (e < nvalid) u[c.row * L + t0 + e] = out[e];
        table_add_vector<T>(s_tab, sh, out, 0, nvalid);
    };

    int64_t left = wk.turns;                                  // uniform
    if (TABLE && L < 2 * V) {
        for (; left > 0; --left) {
            values();
            __syncthreads();                                  // end of the table's round
        }
    } else {
        for (; left >= U; left -= U) {
            vectors(std::integral_constant<int, U>{});
            if constexpr (TABLE) __syncthreads();
        }
        if (left > 0) {
            vectors(std::integral_constant<int, 1>{});
            if constexpr (TABLE) __syncthreads();
        }
    }

    if (W > 1 && state_out) {                                 // the last W - 1 inputs of every row, oldest first: side by side
        const int64_t n = wk.rows * (W - 1);                  // over the lanes (written with the rows' last vectors, a few bytes
        for (int64_t i = blockIdx.x * NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) {     // of a line from each XCD, they cost 5 % of the kernel)
            const int64_t r = i / (W - 1 > 0 ? W - 1 : 1);
            const int64_t t = L - (W - 1) + (i - r * (W - 1));
            T v = T(0);
            if (t >= 0) v = x[r * L + t];
            else if (state_in) v = state_in[r * (W - 1) + (t + (W - 1))];
            state_out[i] = v;
        }
    }

    if (handoff || TABLE) {
        round_extremes<T>(lo, hi);
        uint32_t klo = (lo <= hi) ? order_key(lo) : 0xffffffffu;
        uint32_t khi = (lo <= hi) ? order_key(hi) : 0u;
        uint32_t knan = nan ? 1u : 0u;
        if constexpr (TABLE) corey_table::end<T, false>(s_tab, sh, tws, klo, khi, knan);     // also reduces the keys into thread 0
        else reduce_range_keys<NT>(klo, khi, knan);
        if (handoff) write_parts<NT>(handoff->parts, klo, khi, knan);
    }
}

// One step with the carried state (generation): bound by the window it moves (W - 1 values in, W - 1 out beside one of x and u).
// A lane takes R channels, as many as 4 bytes of x hold: the windows of R rows are then whole words (12 bytes at four taps), side by
// side over the wave.  It keeps its channels and walks the sequences, so that taps and bias, more bytes than the step itself, are
// loaded once per lane, and has up to kStepUnits sequences in flight.  512 sequences of 5120 channels, bf16: 16.9 us (2.5 TB/s) with lanes
// that walked rows of any channel and loaded the taps with each, 13.6 (3.1 TB/s) now; with non-temporal stores of the window 13.2, but
// 64 sequences, whose window the next step finds in a cache, lose 0.3; three in flight 14.3.
// UNITS: 1 where every lane has one sequence, else kStepUnits.  A small batch is one trip to memory and the code's own way into the
// compute units: five absent bodies, jumped over twice, were 0.4 of its 3.4 us (bf16, 5120 channels, state and inputs in a cache: 1 sequence
// 3.44 -> 3.04 us, 64 4.20 -> 3.83; 128 and more, which take kStepUnits, unchanged).
// R = 2 needs an even D and rows that start at words (the caller checks); other 16-bit tensors take the kernel below.
constexpr int kStepUnits = 6;

template <typename T, int W, int UNITS>
__global__ __launch_bounds__(kThreads) void k_conv1d_silu_step(const T* __restrict__ x, const float* __restrict__ weight,
                                                               const float* __restrict__ bias, const T* __restrict__ state_in,
                                                               T* __restrict__ u, T* __restrict__ state_out,
                                                               Handoff* __restrict__ handoff, const StepWalk wk)
{
    if (handoff) corey_range::clear_handoff_counts(handoff);
    constexpr int R = 4 / (int)sizeof(T);
    constexpr int NS = R * (W - 1);                           // values of R windows
    float lo = INFINITY, hi = -INFINITY;
    bool nan = false;
    const uint32_t lane = blockIdx.x * kThreads + threadIdx.x;
    const uint32_t s0 = quotient(lane, wk.groups);            // the first sequence of this lane (0 where the lanes are fewer than the groups)
    const int units = UNITS == 1 ? 1 : wk.units;
    if (s0 < wk.across) {
        for (int64_t v = (int64_t)lane - (int64_t)s0 * wk.groups; v < wk.groups; v += wk.lanes) {      // (one turn but for very many channels)
            float w[R * W], bs[R];
            __builtin_memcpy(w, weight + v * R * W, sizeof(w));
#pragma unroll
            for (int i = 0; i < R; ++i) bs[i] = bias ? bias[v * R + i] : 0.f;
            for (int64_t s = s0; s < wk.B; s += (int64_t)units * wk.across) {
                int64_t r[UNITS];                             // first row of the group
                T xv[UNITS][R], win[UNITS][NS > 0 ? NS : 1];
#pragma unroll
                for (int j = 0; j < UNITS; ++j) {
                    if (j < units) {                          // uniform
                        const int64_t sj = s + (int64_t)j * wk.across;
                        r[j] = ((sj < wk.B ? sj : s) * wk.groups + v) * R;      // beyond the last sequence the lane's first is done again
                        __builtin_memcpy(xv[j], __builtin_assume_aligned(x + r[j], 4), 4);
                        if (W > 1) {
                            if (state_in) {
                                __builtin_memcpy(win[j], __builtin_assume_aligned(state_in + r[j] * (W - 1), 4), sizeof(T) * NS);
                            } else {
#pragma unroll
                                for (int k = 0; k < NS; ++k) win[j][k] = T(0);
                            }
                        }
                    }
                }
#pragma unroll
                for (int j = 0; j < UNITS; ++j) {
                    if (j < units) {
                        T out[R], moved[NS > 0 ? NS : 1];
#pragma unroll
                        for (int i = 0; i < R; ++i) {
                            float acc = bs[i];
#pragma unroll
                            for (int k = 0; k < W - 1; ++k) acc = fmaf(w[i * W + k], St<T>::widen(win[j][i * (W - 1) + k]), acc);
                            acc = fmaf(w[i * W + W - 1], St<T>::widen(xv[j][i]), acc);
                            const float val = acc * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-acc * kLog2e));
                            nan |= (val != val);
                            lo = vmin(lo, val);
                            hi = vmax(hi, val);
                            float one[St<T>::kVec];
                            T st[St<T>::kVec];
#pragma unroll
                            for (int e = 0; e < St<T>::kVec; ++e) one[e] = val;
                            St<T>::narrow(one, st);
                            out[i] = st[0];
#pragma unroll
                            for (int k = 0; k < W - 1; ++k) moved[i * (W - 1) + k] = (k + 1 < W - 1) ? win[j][i * (W - 1) + k + 1] : xv[j][i];
                        }
                        __builtin_memcpy(__builtin_assume_aligned(u + r[j], 4), out, 4);
                        if (W > 1 && state_out) __builtin_memcpy(__builtin_assume_aligned(state_out + r[j] * (W - 1), 4), moved, sizeof(T) * NS);
                    }
                }
                if (UNITS == 1) break;
            }
        }
    }
    if (handoff) {
        round_extremes<T>(lo, hi);
        uint32_t klo = (lo <= hi) ? order_key(lo) : 0xffffffffu;
        uint32_t khi = (lo <= hi) ? order_key(hi) : 0u;
        uint32_t knan = nan ? 1u : 0u;
        reduce_range_keys(klo, khi, knan);
        write_parts<kThreads>(handoff->parts, klo, khi, knan);
    }
}

// Rows of fewer than two vectors (a few steps with the carried state): one lane per row.  A lane keeps the row's window of
// W - 1 earlier inputs in registers and walks its L steps.
template <typename T, int W>
__global__ __launch_bounds__(kThreads) void k_conv1d_silu_short(const T* __restrict__ x, const float* __restrict__ weight,
                                                                const float* __restrict__ bias, const T* __restrict__ state_in,
                                                                T* __restrict__ u, T* __restrict__ state_out,
                                                                Handoff* __restrict__ handoff, int64_t rows, int64_t D, int L)
{
    if (handoff) corey_range::clear_handoff_counts(handoff);
    float lo = INFINITY, hi = -INFINITY;
    bool nan = false;
    for (int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x; r < rows; r += (int64_t)gridDim.x * kThreads) {
        const int64_t d = ((uint64_t)r >> 32 || (uint64_t)D >> 32) ? r % D : (int64_t)((uint32_t)r % (uint32_t)D);
        float w[W], win[W];                                   // win[k]: the input the tap w[k] multiplies at the current step
#pragma unroll
        for (int k = 0; k < W; ++k) w[k] = weight[d * W + k];
#pragma unroll
        for (int k = 0; k < W - 1; ++k) win[k + 1] = state_in ? St<T>::widen(state_in[r * (W - 1) + k]) : 0.f;
        const float bs = bias ? bias[d] : 0.f;
        T raw[W > 1 ? W - 1 : 1];                             // the stored form of the window, for state_out
#pragma unroll
        for (int k = 0; k < W - 1; ++k) raw[k] = state_in ? state_in[r * (W - 1) + k] : T(0);
        for (int t = 0; t < L; ++t) {
#pragma unroll
            for (int k = 0; k < W - 1; ++k) win[k] = win[k + 1];
#pragma unroll
            for (int k = 0; k + 1 < W - 1; ++k) raw[k] = raw[k + 1];
            const T xt = x[r * L + t];
            win[W - 1] = St<T>::widen(xt);
            if constexpr (W > 1) raw[W - 2] = xt;
            float acc = bs;
#pragma unroll
            for (int k = 0; k < W; ++k) acc = fmaf(w[k], win[k], acc);
            const float val = acc * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-acc * kLog2e));
            nan |= (val != val);
            lo = vmin(lo, val);
            hi = vmax(hi, val);
            float one[St<T>::kVec];
            T st[St<T>::kVec];
#pragma unroll
            for (int e = 0; e < St<T>::kVec; ++e) one[e] = val;
            St<T>::narrow(one, st);
            u[r * L + t] = st[0];
        }
        if (state_out)
#pragma unroll
            for (int k = 0; k < W - 1; ++k) state_out[r * (W - 1) + k] = raw[k];
    }
    if (handoff) {
        round_extremes<T>(lo, hi);
        uint32_t klo = (lo <= hi) ? order_key(lo) : 0xffffffffu;
        uint32_t khi = (lo <= hi) ? order_key(hi) : 0u;
        uint32_t knan = nan ? 1u : 0u;
        reduce_range_keys(klo, khi, knan);
        write_parts<kThreads>(handoff->parts, klo, khi, knan);
    }
}

// Fewest workgroups of a launch that also clears the hand-over's 256 KiB of counters: one 16-byte store per lane.  (Left to the
// one workgroup that 64 rows of 16 steps fill, the clearing was 1.5 of 5.3 us.)
constexpr int64_t kClearBlocks = corey_range::kParts * COREY_MAX_BINS / 4 / kThreads;

// How `rows` rows of `nvec` vectors are walked by `least` to `most` workgroups of `threads` lanes, each lane the same number of
// vectors.
Walk plan_walk(int64_t rows, int64_t D, int64_t L, int64_t nvec, int threads, int64_t least, int64_t most, int64_t* blocks)
{
    Walk w = {};
    w.rows = rows; w.D = D; w.L = L; w.nvec = nvec;
    const int64_t total = rows * nvec;
    w.turns = (total + threads * most - 1) / (threads * most);
    *blocks = (total + threads * w.turns - 1) / (threads * w.turns);
    if (*blocks < least) *blocks = least;
    const int64_t step = *blocks * threads;
    w.q = step / nvec;
    w.rem = step - w.q * nvec;
    w.qd = w.q % D;
    return w;
}

template <typename T>
void launch(const void* x_, const float* weight, const float* bias, const void* state_in_, void* u_, void* state_out_, void* rparts,
            void* table_ws, int64_t B, int64_t D, int64_t L, int W, hipStream_t stream)
{
    constexpr int V = St<T>::kVec;
    const T *x = static_cast<const T*>(x_), *state_in = static_cast<const T*>(state_in_);
    T *u = static_cast<T*>(u_), *state_out = static_cast<T*>(state_out_);
    Handoff* handoff = static_cast<Handoff*>(rparts);
    const int64_t rows = B * D;
    int64_t blocks = 0;
    if constexpr (sizeof(T) == 2) {
        if (table_ws) {                                       // one workgroup of 1024 lanes per compute unit, each with a table
            constexpr int NT = corey_table::kLanes;
            const Walk wk = plan_walk(rows, D, L, (L + V - 1) / V, NT, 1, corey_table::kMaxSlabs, &blocks);
            auto go_table = [&](auto kernel) {
                kernel<<<dim3((unsigned)blocks), dim3(NT), 0, stream>>>(x, weight, bias, state_in, u, state_out, handoff, table_ws, wk);
            };
            switch (W) {
            case 1: go_table(k_conv1d_silu<T, 1, NT, true, false>); break;
            case 2: go_table(k_conv1d_silu<T, 2, NT, true, false>); break;
            case 3: go_table(k_conv1d_silu<T, 3, NT, true, false>); break;
            default: go_table(k_conv1d_silu<T, 4, NT, true, false>); break;
            }
            return;
        }
    }
    constexpr int R = 4 / (int)sizeof(T);
    bool words = D % R == 0;
    for (const void* p : {x_, (const void*)u_, state_in_, (const void*)state_out_})
        if (reinterpret_cast<uintptr_t>(p) % 4 != 0) words = false;
    if (L == 1 && words) {
        StepWalk wk = {};
        wk.B = B;
        wk.groups = D / R;
        const int64_t most = (int64_t)COREY_RANGE_PARTS * kThreads / wk.groups;     // sequences side by side, at most
        const int64_t turns = most < 1 ? B : (B + most - 1) / most;
        wk.across = (uint32_t)(most < 1 ? 1 : (B + turns - 1) / turns);
        const int64_t passes = (turns + kStepUnits - 1) / kStepUnits;
        wk.units = (int)((turns + passes - 1) / passes);
        blocks = most < 1 ? COREY_RANGE_PARTS : (wk.across * wk.groups + kThreads - 1) / kThreads;
        const int64_t least = handoff ? kClearBlocks : 1;
        blocks = blocks < least ? least : blocks;
        wk.lanes = blocks * kThreads;
        auto go_step = [&](auto kernel) {
            kernel<<<dim3((unsigned)blocks), dim3(kThreads), 0, stream>>>(x, weight, bias, state_in, u, state_out, handoff, wk);
        };
        auto taps = [&](auto units) {
            constexpr int UNITS = decltype(units)::value;
            switch (W) {
            case 1: go_step(k_conv1d_silu_step<T, 1, UNITS>); break;
            case 2: go_step(k_conv1d_silu_step<T, 2, UNITS>); break;
            case 3: go_step(k_conv1d_silu_step<T, 3, UNITS>); break;
            default: go_step(k_conv1d_silu_step<T, 4, UNITS>); break;
            }
        };
        if (turns == 1) taps(std::integral_constant<int, 1>{});
        else taps(std::integral_constant<int, kStepUnits>{});
        return;
    }
    if (L < 2 * V) {
        blocks = (rows + kThreads - 1) / kThreads;
        blocks = blocks > COREY_RANGE_PARTS ? COREY_RANGE_PARTS : (handoff && blocks < kClearBlocks ? kClearBlocks : blocks);
        auto go_short = [&](auto kernel) {
            kernel<<<dim3((unsigned)blocks), dim3(kThreads), 0, stream>>>(x, weight, bias, state_in, u, state_out, handoff, rows, D, (int)L);
        };
        switch (W) {
        case 1: go_short(k_conv1d_silu_short<T, 1>); break;
        case 2: go_short(k_conv1d_silu_short<T, 2>); break;
        case 3: go_short(k_conv1d_silu_short<T, 3>); break;
        default: go_short(k_conv1d_silu_short<T, 4>); break;
        }
        return;
    }
    const Walk wk = plan_walk(rows, D, L, (L + V - 1) / V, kThreads, handoff ? kClearBlocks : 1, COREY_RANGE_PARTS, &blocks);
    auto go = [&](auto kernel) {
        kernel<<<dim3((unsigned)blocks), dim3(kThreads), 0, stream>>>(x, weight, bias, state_in, u, state_out, handoff, nullptr, wk);
    };
    auto taps = [&](auto waves) {                             // the tap count is a compile-time constant of the kernel
        constexpr bool WV = decltype(waves)::value;
        switch (W) {
        case 1: go(k_conv1d_silu<T, 1, kThreads, false, WV>); break;
        case 2: go(k_conv1d_silu<T, 2, kThreads, false, WV>); break;
        case 3: go(k_conv1d_silu<T, 3, kThreads, false, WV>); break;
        default: go(k_conv1d_silu<T, 4, kThreads, false, WV>); break;
        }
    };
    if (L % (64 * V) == 0) taps(std::true_type{});            // 64 vectors in a row: whole waves stay in one row
    else taps(std::false_type{});
}

}  // namespace

extern "C" int causal_conv1d_silu_fwd(const void* x, const float* weight, const float* bias, const void* state_in, void* u,
                                      void* state_out, void* range_parts, void* pattern_table, size_t pattern_table_bytes,
                                      corey_dtype dt, int64_t B, int64_t D, int64_t L, int32_t W, void* hip_stream)
{
    using corey::fail;
    if (!x || !weight || !u) return fail(COREY_ENULL, "causal_conv1d_silu_fwd: x, weight and u are required");
    if (dt != COREY_F32 && dt != COREY_BF16 && dt != COREY_F16) return fail(COREY_EINVAL, "causal_conv1d_silu_fwd: unknown dtype %d", (int)dt);
    if (W < 1 || W > COREY_MAX_CONV) return fail(COREY_EINVAL, "causal_conv1d_silu_fwd: W = %d outside [1, %d]", W, COREY_MAX_CONV);
    if (B < 1 || D < 1 || L < 1) return fail(COREY_ESHAPE, "causal_conv1d_silu_fwd: B, D, L must be >= 1");
    if ((double)B * (double)D * (double)L >= 4.0e18) return fail(COREY_ESHAPE, "causal_conv1d_silu_fwd: B*D*L overflows");
    if (x == u) return fail(COREY_EINVAL, "causal_conv1d_silu_fwd: u may not alias x");
    if (range_parts && reinterpret_cast<uintptr_t>(range_parts) % 16 != 0)
        return fail(COREY_EINVAL, "causal_conv1d_silu_fwd: range_parts must be 16-byte aligned");
    if (pattern_table) {
        if (dt == COREY_F32) return fail(COREY_EUNSUPPORTED, "causal_conv1d_silu_fwd: the bit-pattern table exists for 16-bit storage only");
        if (pattern_table_bytes < corey_table::kWorkspaceBytes || reinterpret_cast<uintptr_t>(pattern_table) % 256 != 0)
            return fail(COREY_EWORKSPACE, "causal_conv1d_silu_fwd: pattern_table needs %zu bytes, 256-byte aligned", corey_table::kWorkspaceBytes);
        if ((double)B * (double)D * (double)L >= 4294967296.0)
            return fail(COREY_ESHAPE, "causal_conv1d_silu_fwd: more than 2^32-1 values would overflow the table's 32-bit totals");
    }
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (dt == COREY_F32) launch<float>(x, weight, bias, state_in, u, state_out, range_parts, nullptr, B, D, L, W, stream);
    else if (dt == COREY_F16) launch<_Float16>(x, weight, bias, state_in, u, state_out, range_parts, pattern_table, B, D, L, W, stream);
    else launch<uint16_t>(x, weight, bias, state_in, u, state_out, range_parts, pattern_table, B, D, L, W, stream);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return corey::hip_fail(e, "causal_conv1d_silu_fwd launch");
    return COREY_OK;
}
