// One group of states of a tile: the body of the two loops over the groups in scan_group (corey_scan_impl.h), whose names it uses.
// n0 is the number, inside the row, of the group's first state; ask_c says whether the gate and the next tile are requested in it.
//
// A text included twice (so without a guard), not a function: direct launches need it in three loops, and the staged ones run slower
// with any form of function around it.  Inlined, that gave their two ways to start a copy (the next group, the next tile) one tail
// behind selects, ahead of the copies.  Staged scans as plain loop and as function, us: chunk 16, 4096 bf16 rows of 2048 steps 282 and
// 294, of 977 144 and 151, binary32 277 and 290, routed binary32, 1536 rows of 2048, 278 and 289; chunk 64, 4096 bf16 rows of 2048
// 85.6 and 89.5.  And the loops of direct launches as one unrolled loop over three ranges are slower than as a function: binary32,
// chunk 16, 3 to 6 %.
const float* s_B = s_stage + buf * 2 * STAGE;
const float* s_C = s_B + STAGE;
// A and the carried state of the group's states (the latter was written a tile ago by this wave's own lanes).  Staged:
// requested here, they arrive while the wave waits below.  DIRECT: requested during the last replays of the group before.
GHv cin_g, A2_g, h_g;
if constexpr (DIRECT) {
    cin_g = cin_nx;
    A2_g = A2_nx;
} else {
    cin_g = *reinterpret_cast<const GHv*>(carry_rd + n0);
    if constexpr (!STRUCT) A2_g = *reinterpret_cast<const GHv*>(A2_row + n0);
}
if constexpr (!DIRECT) {
    // this group's copy (started one group earlier) has landed; every wave is past the previous group
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}
const bool last_group = n0 + GH >= NH;
if constexpr (!DIRECT) {                        // start the copy of the next group: same tile, or the first group of the next
    if (!last_group) stage_group(tau, n0 + GH, s_stage + (buf ^ 1) * 2 * STAGE);
    else if (tau + 1 < ntiles) stage_group(tau + 1, 0, s_stage + (buf ^ 1) * 2 * STAGE);
}
if (!kAhead && last_group) {                    // the gate, and the next tile if it is a full one, arrive while it is computed
    if constexpr (!kGateFirst || FULL)
        if (z_on) z_raw = load_row(z_grp);
    if constexpr (kTileAhead) {
        if (FULL && tau + 1 < nfull) {
            u_nx = load_full<T, K>(at(u_grp + tile + CHUNK));
            d_nx = load_full<T, K>(at(dl_grp + tile + CHUNK));
            if constexpr (!DIRECT) have_nx = true;
        }
    }
}
buf ^= 1;
const BCv* bq0 = reinterpret_cast<const BCv*>(s_B + half * GH * CHUNK) + j;
const BCv* cq0 = reinterpret_cast<const BCv*>(s_C + half * GH * CHUNK) + j;
// Q states at a time.  Order of the work: request B (and A, the carried state) from LDS; the products dl A; the
// exponentials as one burst, which covers that trip; the folds; request C; the lane scans, which cover part of that
// one; the replays.
auto states = [&](const int nl) __attribute__((always_inline)) {
    const BCv* bq = bq0 + nl * KQ * LPR;
    const BCv* cq = cq0 + nl * KQ * LPR;
    float P[Q], h[Q];
    float av[Q][K], bv[Q][K];
    BCv b4[Q][KQ], c4[Q][KQ];
    Raw<T, K> b_raw[Q], c_raw[Q];
    if constexpr (DIRECT) {
#pragma unroll
        for (int s = 0; s < Q; ++s) {
            b_raw[s] = b_nx[s];
            c_raw[s] = c_nx[s];
        }
        // (after the row's last full tile this reads a set nobody uses: cheaper than a branch among the states)
        const bool more = n0 + nl + Q < NH;
        fetch(full_c, more ? n0 + nl + Q : 0, FULL ? (more || tau + 1 >= nfull ? tile : tile + CHUNK) : 0);
        if (decltype(ask_c)::value && nl == 0) {
            __builtin_amdgcn_sched_barrier(0);
            request_tile();
        }
    } else {
#pragma unroll
        for (int s = 0; s < Q; ++s)
#pragma unroll
            for (int q = 0; q < KQ; ++q) b4[s][q] = bq[(s * KQ + q) * LPR];
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (STRUCT) {
#pragma unroll
        for (int s = 0; s < Q; ++s) {
#pragma unroll
            for (int i = 0; i < K; ++i) {
                av_chain[i] *= dl[i];           // decay of state n from that of state n - 1
                av[s][i] = av_chain[i];
            }
            P_chain *= P_base;
            P[s] = P_chain;
        }
    } else {
#pragma unroll
        for (int s = 0; s < Q; ++s) {
#pragma unroll
            for (int i = 0; i < K; ++i) av[s][i] = dl[i] * A2_g[nl + s];
            P[s] = S * A2_g[nl + s];
        }
        if constexpr (Q == 1) {
            decay_burst<K, true, true>(av[0], P[0]);
        } else {
            decay_burst<K, true, false>(av[0], P[0]);
#pragma unroll
            for (int s = 1; s + 1 < Q; ++s) decay_burst<K, false, false>(av[s], P[s]);
            decay_burst<K, false, true>(av[Q - 1], P[Q - 1]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);          // (nothing of the folds before the burst is through)
    float bw[Q][K], cw[Q][K];                   // DIRECT
    if constexpr (DIRECT) {
#pragma unroll
        for (int s = 0; s < Q; ++s) {
            if constexpr (!FULL) {
                if (n0 + nl + s == n_last) tail.place(b_raw[s]);
                tail.mask(b_raw[s]);
            }
            widen<T, K>(b_raw[s], bw[s]);
        }
    }
    if constexpr (kEarlyC && !DIRECT) {
#pragma unroll
        for (int s = 0; s < Q; ++s)
#pragma unroll
            for (int q = 0; q < KQ; ++q) c4[s][q] = cq[(s * KQ + q) * LPR];
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < K; ++i)
#pragma unroll
        for (int s = 0; s < Q; ++s) {
            bv[s][i] = du[i] * (DIRECT ? bw[s][i] : b4[s][i / E][i % E]);
            h[s] = i == 0 ? bv[s][i] : fmaf(av[s][i], h[s], bv[s][i]);      // the fold starts from a zero state
        }
    float hh[Q];                                // true state entering this lane's sub-block
#pragma unroll
    for (int s = 0; s < Q; ++s) {
        hh[s] = cin_g[nl + s];                  // the row's first lane starts from the carried state (0 elsewhere)
        h[s] = fmaf(P[s], hh[s], h[s]);
    }
    scan_segments<SEG, Q>(jseg, P, h, hh);      // h: state at the end of this lane's sub-block
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < Q; ++s) h_g[nl + s] = h[s];
    if (DIRECT && nl + Q == GH) {
        *reinterpret_cast<GHv*>(carry_wr + n0) = h_g;
        carry_fence();
        const int nn = last_group ? 0 : n0 + GH;
        cin_nx = *reinterpret_cast<const GHv*>(carry_rd + nn);
        if constexpr (!STRUCT) A2_nx = *reinterpret_cast<const GHv*>(A2_row + nn);
    }
#pragma unroll
    for (int s = 0; s < Q; ++s)
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
            if constexpr (DIRECT) {
                if (q == 0) {
                    if constexpr (!FULL)
                        if (n0 + nl + s == n_last) tail.place(c_raw[s]);
                    widen<T, K>(c_raw[s], cw[s]);
                }
            } else if constexpr (!kEarlyC) {
                c4[s][q] = cq[(s * KQ + q) * LPR];
            }
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int i = E * q + e;
                hh[s] = fmaf(av[s][i], hh[s], bv[s][i]);
                yv[i] = fmaf(DIRECT ? cw[s][i] : c4[s][q][e], hh[s], yv[i]);
            }
        }
};
#pragma unroll
for (int nl = 0; nl < GH; nl += Q) states(nl);      // straight-line code for the whole group
if constexpr (!DIRECT) {
    *reinterpret_cast<GHv*>(carry_wr + n0) = h_g;
    carry_fence();
}
