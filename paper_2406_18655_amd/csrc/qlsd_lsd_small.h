// Per-shot LSD device code for small codes (one wavefront per shot): n <= 192 faults, m <= 128 checks, H in
// LDS, columns of any weight (lsd_small_shape).  The same function of a shot as decode_shot, with the clusters
// held by the lanes instead of union-find arrays in LDS:
//   * the shot's faults are ranked by key once, and sets of faults are bit sets over ranks (3 words);
//   * lane c holds cluster c: its checks (a bit set), its candidates (the ranks of every fault that meets
//     its checks and is not taken) and its number of faults; which lanes are alive, invalid or frozen are
//     wave-uniform masks.  A cluster's pick is its lowest candidate bit;
//   * a picked fault's checks and the union of its checks' fault sets (one table entry per rank, built
//     once per shot) are read by the picking lane, all clusters at once; then the picked faults are taken
//     in ascending key order: the clusters whose checks meet the fault's are found by one ballot and united
//     in the lowest of them, which gives the partition of simultaneous claims and unions (Def. 4.4: two
//     clusters merge iff they are linked by faults picked this round), and the column goes to the basis,
//     whose rows are the checks themselves;
//   * a cluster is invalid iff its checks meet the rows the reduced syndrome leaves unsolved.
// Bound by latency: a round waits for two dependent LDS reads, where decode_shot's selection, claim, union
// and validity phases through LDS arrays wait for about 25.  What remains is the ranking of the faults
// (n LDS reads, 3n compares), the tables and the serial loads of each shot.  Measured on the [[144,12,12]]
// code: 12.9k shots that 10 rounds of BP leave, kernel alone 329 -> 260 us; decode with BP of 30 rounds
// in the same kernel, 1% physical error rate, 234 -> 147 us.  Shots with more than 64 flipped checks
// (clusters at the start) are left to decode_shot.
#pragma once
#include "qlsd_lsd_dev.h"

namespace qlsd {

namespace {

struct SmallLds {
    uint64_t *tab;     // n x (W + kSmallWords) by rank: the fault's checks; the ranks of every fault that meets them
                       // (its first n words hold the keys while they are ranked)
    uint64_t *adj;     // m x kSmallWords: ranks of the check's faults
    uint32_t *cbit;    // kSmallFaults / 32: the correction
    uint8_t *rank_of;  // n: rank of each fault
    uint8_t *at_rank;  // n: fault of each rank
    uint8_t *seed;     // 64: check of each cluster at the start
};

template <int W>
__device__ __forceinline__ SmallLds carve_small(unsigned char *base, int m, int n) {
    SmallLds L;
    L.tab = (uint64_t *)base;
    L.adj = L.tab + (size_t)n * (W + kSmallWords);
    L.cbit = (uint32_t *)(L.adj + (size_t)m * kSmallWords);
    L.rank_of = (uint8_t *)(L.cbit + kSmallFaults / 32);
    L.at_rank = L.rank_of + kSmallFaults;
    L.seed = L.at_rank + kSmallFaults;
    return L;
}

// Returns false (nothing written) if the shot is left to decode_shot.
template <int W>
__device__ __forceinline__ bool decode_small(const LsdArgs &A, unsigned char *base, const GView<true> &g, int shot,
                                             int lane) {
    constexpr int NW = kSmallWords;
    const int m = A.g.m, n = A.g.n;
    const float *llr = A.llr + (size_t)shot * n;
    const uint8_t *syn = A.syn + (size_t)shot * m;
    uint8_t *corr = A.corr + (size_t)shot * n;
    // every load of the shot is issued before the first is used
    uint8_t sy[W];
    float v[NW];
#pragma unroll
    for (int s = 0; s < W; s++) sy[s] = s * 64 + lane < m ? syn[s * 64 + lane] : 0;
#pragma unroll
    for (int q = 0; q < NW; q++) {
        const int j = q * 64 + lane;
        v[q] = 0.f;
        if (j < n) v[q] = A.coherent_llr ? __int_as_float(atomicCAS((int *)llr + j, 0, 0)) : llr[j];
    }
    uint64_t clustered[W];
    int nseed = 0;
#pragma unroll
    for (int s = 0; s < W; s++) {
        clustered[s] = ballot(sy[s] & 1);
        nseed += __popcll(clustered[s]);
    }
    if (nseed > 64) return false;

    const SmallLds L = carve_small<W>(base, m, n);
    constexpr int TW = W + NW;  // words of a table entry
    uint8_t status = QLSD_ST_LSD_RUN;
    int rounds = 0;
    auto finish = [&](uint8_t st, int ncl, int maxc) {
        wave_sync();
        if ((n & 15) == 0 && (((uintptr_t)corr) & 15) == 0) {
            for (int c = lane; c < (n >> 4); c += 64) {
                const uint32_t bits = (L.cbit[c >> 1] >> ((c & 1) * 16)) & 0xffffu;
                uint32_t o[4];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t nb = bits >> (4 * k);
                    o[k] = (nb & 1u) | ((nb & 2u) << 7) | ((nb & 4u) << 14) | ((nb & 8u) << 21);
                }
                ((uint4 *)corr)[c] = make_uint4(o[0], o[1], o[2], o[3]);
            }
        } else {
            for (int j = lane; j < n; j += 64) corr[j] = (uint8_t)((L.cbit[j >> 5] >> (j & 31)) & 1u);
        }
        if (A.info && lane == 0) {
            qlsd_shot_info inf;
            inf.status = st;
            inf.reserved = 0;
            inf.bp_iters = (int16_t)A.bp_iters;
            inf.n_clusters = (int16_t)ncl;
            inf.rounds = (int16_t)rounds;
            inf.max_cluster_cols = maxc;
            A.info[shot] = inf;
        }
    };
    bool nan = false;
    uint64_t key[NW];
#pragma unroll
    for (int q = 0; q < NW; q++) {
        const int j = q * 64 + lane;
        nan |= v[q] != v[q];
        key[q] = j < n ? ((uint64_t)ordered_key(v[q]) << 32) | (uint32_t)j : ~0ull;
        if (j < n) L.tab[j] = key[q];
    }
    if (lane < kSmallFaults / 32) L.cbit[lane] = 0u;
    // cluster c starts at the c-th flipped check
#pragma unroll
    for (int s = 0, before = 0; s < W; s++) {
        if ((clustered[s] >> lane) & 1ull) L.seed[before + __popcll(clustered[s] & ((1ull << lane) - 1ull))] = (uint8_t)(s * 64 + lane);
        before += __popcll(clustered[s]);
    }
    if (ballot(nan) || nseed == 0) {
        if (A.cstats && lane == 0) A.cstats[shot] = qlsd_cluster_stats{0, 0, 0, 0};
        finish(ballot(nan) ? QLSD_ST_LSD_RUN | QLSD_ST_BAD_LLR : QLSD_ST_LSD_RUN, 0, 0);
        return true;
    }
    wave_sync();
    // ranks: each lane counts the keys below its own (keys are distinct)
    int rank[NW];
#pragma unroll
    for (int q = 0; q < NW; q++) rank[q] = 0;
#pragma unroll 8
    for (int j = 0; j < n; j++) {
        const uint64_t k = L.tab[j];
#pragma unroll
        for (int q = 0; q < NW; q++) rank[q] += k < key[q] ? 1 : 0;
    }
#pragma unroll
    for (int q = 0; q < NW; q++) {
        const int j = q * 64 + lane;
        if (j < n) {
            L.rank_of[j] = (uint8_t)rank[q];
            L.at_rank[rank[q]] = (uint8_t)j;
        }
    }
    wave_sync();
#pragma unroll
    for (int s = 0; s < W; s++) {
        const int i = s * 64 + lane;
        if (i < m) {
            uint64_t a[NW];
#pragma unroll
            for (int w = 0; w < NW; w++) a[w] = 0;
            const int e1 = g.row_ptr(i + 1);
            for (int e = g.row_ptr(i); e < e1; e++) {
                const int r = L.rank_of[g.col_idx(e)];
#pragma unroll
                for (int w = 0; w < NW; w++) a[w] |= (r >> 6) == w ? 1ull << (r & 63) : 0ull;
            }
#pragma unroll
            for (int w = 0; w < NW; w++) L.adj[i * NW + w] = a[w];
        }
    }
    wave_sync();
    // (the keys were last read before the barrier above)
#pragma unroll
    for (int q = 0; q < NW; q++) {
        const int j = q * 64 + lane;
        if (j < n) {
            uint64_t e[TW];
#pragma unroll
            for (int w = 0; w < TW; w++) e[w] = 0;
            const int c1 = g.col_ptr(j + 1);
            for (int c = g.col_ptr(j); c < c1; c++) {
                const int i = g.row_idx(c);
#pragma unroll
                for (int s = 0; s < W; s++) e[s] |= (i >> 6) == s ? 1ull << (i & 63) : 0ull;
#pragma unroll
                for (int w = 0; w < NW; w++) e[W + w] |= L.adj[i * NW + w];
            }
#pragma unroll
            for (int w = 0; w < TW; w++) L.tab[rank[q] * TW + w] = e[w];
        }
    }
    wave_sync();

    ColBasis<W> B;
    B.init(lane);
#pragma unroll
    for (int s = 0; s < W; s++) B.sp[s] = clustered[s];
    uint64_t ck[W], cand[NW];  // this lane's cluster: checks, candidate ranks
    int cnt = 0;               // its faults
    int col_at[W];             // pivot row 64 s + lane: the fault of its column
    {
        const int i = lane < nseed ? L.seed[lane] : 0;
#pragma unroll
        for (int s = 0; s < W; s++) {
            ck[s] = lane < nseed && (i >> 6) == s ? 1ull << (i & 63) : 0ull;
            col_at[s] = 0;
        }
#pragma unroll
        for (int w = 0; w < NW; w++) cand[w] = lane < nseed ? L.adj[i * NW + w] : 0ull;
    }
    uint64_t alive = nseed == 64 ? ~0ull : (1ull << nseed) - 1ull, invalid = alive, frozen = 0;
    uint64_t taken[NW];
#pragma unroll
    for (int w = 0; w < NW; w++) taken[w] = 0;

    while (invalid) {
        // picks: the lowest candidate of every invalid cluster; one without any is frozen (UNSAT)
        uint64_t any = 0;
#pragma unroll
        for (int w = 0; w < NW; w++) any |= cand[w];
        const uint64_t has = ballot(any != 0), sel = invalid & has;
        if (invalid & ~has) {
            frozen |= invalid & ~has;
            status |= QLSD_ST_UNSAT;
        }
        if (!sel) break;
        int rk = 0;
#pragma unroll
        for (int w = NW - 1; w >= 0; w--)
            if (cand[w]) rk = 64 * w + __builtin_ctzll(cand[w]);
        const bool pick = (sel >> lane) & 1ull;
        uint64_t ent[TW];  // the picked fault's checks; every fault that meets them
        {
            const uint64_t *e = L.tab + (pick ? rk : 0) * TW;
#pragma unroll
            for (int w = 0; w < TW; w++) ent[w] = e[w];
        }
        const int fl = L.at_rank[pick ? rk : 0];
        // the picked ranks, each once, and in ascending order the lane that picked each
        uint64_t todo[NW];
#pragma unroll
        for (int w = 0; w < NW; w++) todo[w] = 0;
        bool more = (sel & (sel - 1)) != 0;
        if (more) {
            for (uint64_t t = sel; t; t &= t - 1) {
                const int r = __builtin_amdgcn_readlane(rk, __builtin_ctzll(t));
#pragma unroll
                for (int w = 0; w < NW; w++) todo[w] |= (r >> 6) == w ? 1ull << (r & 63) : 0ull;
            }
        }
        int l = __builtin_ctzll(sel);
#pragma unroll 1
        do {
            int r = __builtin_amdgcn_readlane(rk, l);
            if (more) {
#pragma unroll
                for (int w = NW - 1; w >= 0; w--)
                    if (todo[w]) r = 64 * w + __builtin_ctzll(todo[w]);
                l = __builtin_ctzll(ballot(pick && rk == r));
                uint64_t left = 0;
#pragma unroll
                for (int w = 0; w < NW; w++) {
                    if ((r >> 6) == w) todo[w] &= todo[w] - 1;
                    left |= todo[w];
                }
                more = left != 0;
            }
#pragma unroll
            for (int w = 0; w < NW; w++) taken[w] |= (r >> 6) == w ? 1ull << (r & 63) : 0ull;
            uint64_t add_ck[W], add_cand[NW], rows[W];
#pragma unroll
            for (int s = 0; s < W; s++) rows[s] = add_ck[s] = readlane64(ent[s], l);
#pragma unroll
            for (int w = 0; w < NW; w++) add_cand[w] = readlane64(ent[W + w], l);
            const int fault = __builtin_amdgcn_readlane(fl, l);
            // the clusters it touches (dead lanes hold no checks)
            uint64_t meet = 0;
#pragma unroll
            for (int s = 0; s < W; s++) meet |= ck[s] & add_ck[s];
            uint64_t ov = ballot(meet != 0);
            const int root = __builtin_ctzll(ov);
            ov &= ov - 1;
            alive &= ~ov;
            int add_cnt = 1;
            for (; ov; ov &= ov - 1) {
                const int c = __builtin_ctzll(ov);
#pragma unroll
                for (int s = 0; s < W; s++) add_ck[s] |= readlane64(ck[s], c);
#pragma unroll
                for (int w = 0; w < NW; w++) add_cand[w] |= readlane64(cand[w], c);
                add_cnt += __builtin_amdgcn_readlane(cnt, c);
                if (lane == c) {
#pragma unroll
                    for (int s = 0; s < W; s++) ck[s] = 0;
                }
            }
            if (lane == root) {
#pragma unroll
                for (int s = 0; s < W; s++) ck[s] |= add_ck[s];
#pragma unroll
                for (int w = 0; w < NW; w++) cand[w] = (cand[w] | add_cand[w]) & ~taken[w];
                cnt += add_cnt;
            }
#pragma unroll
            for (int s = 0; s < W; s++) clustered[s] |= add_ck[s];
            // the column, on the rows of its checks
            B.ns = W == 2 && clustered[W - 1] ? 2 : 1;
            const int row = B.tier([&](auto N) {
                constexpr int NS = decltype(N)::value;
                uint64_t t[W];
#pragma unroll
                for (int w = 0; w < W; w++) t[w] = 0;
#pragma unroll
                for (int s = 0; s < NS; s++)
                    for (uint64_t k = rows[s]; k; k &= k - 1) B.template fold_slice<NS>(s, __builtin_ctzll(k), t);
                return B.template add<NS>(t);
            });
#pragma unroll
            for (int s = 0; s < W; s++) col_at[s] = row == s * 64 + lane ? fault : col_at[s];
        } while (more);
        uint64_t bad = 0;
#pragma unroll
        for (int s = 0; s < W; s++) bad |= ck[s] & B.unsolved(s);
        invalid = ballot(bad != 0) & alive & ~frozen;
        rounds++;
    }

    // the solution on the pivot rows of every cluster not frozen
    uint64_t x[W];
#pragma unroll
    for (int s = 0; s < W; s++) x[s] = B.sp[s] & B.piv[s];
    for (uint64_t f = frozen; f; f &= f - 1) {
#pragma unroll
        for (int s = 0; s < W; s++) x[s] &= ~readlane64(ck[s], __builtin_ctzll(f));
    }
#pragma unroll
    for (int s = 0; s < W; s++)
        if ((x[s] >> lane) & 1ull) atomicOr(&L.cbit[col_at[s] >> 5], 1u << (col_at[s] & 31));
    const int ncl = __popcll(alive);
    int mx = 0;
    if (A.info || A.cstats) {
        uint32_t c = (alive >> lane) & 1ull ? (uint32_t)cnt : 0u, big = c, tot = c, sq = c * c;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const uint32_t o = (uint32_t)__shfl_xor((int)big, off, 64);
            big = o > big ? o : big;
            if (A.cstats) {
                tot += (uint32_t)__shfl_xor((int)tot, off, 64);
                sq += (uint32_t)__shfl_xor((int)sq, off, 64);
            }
        }
        mx = (int)big;
        if (A.cstats && lane == 0) A.cstats[shot] = qlsd_cluster_stats{ncl, mx, (int)tot, (int)sq};
    }
    finish(status, ncl, mx);
    return true;
}

}  // namespace

}  // namespace qlsd
