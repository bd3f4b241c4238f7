// The last rounds of a product sumcheck in one block (k_sc_tail in k_sumcheck.hip), and what the kernel with helper blocks
// (k_schelp.hip) shares with it.
#pragma once
#include "spec_rounds.cuh"

struct RoundArgs {
    FrTab src8[3];     // packed source tables (first round, first fused round)
    F9Tab work[3];     // lazy 29-bit-limb work tables (written by every fused round)
    uint64_t m;        // half length of the tables this round sums over
    const Fr* chal;    // challenge of the previous round (fused rounds)
    Fr* part;          // partial sums: block b, evaluation x at part[b * (K+1) + x]
};

// where the tables of the first round come from
enum ScTailSource {
    SC_SRC_PACKED = 0,     // ra.src8, 2 m packed entries: nothing is bound
    SC_SRC_PACKED_FOLD,    // ra.src8, 4 m packed entries: one challenge is bound
    SC_SRC_WORK,           // ra.work, 4 m lazy entries: one challenge is bound
    SC_SRC_PACKED_W4,      // ra.src8, 8 m packed entries (below 2 r): two challenges are bound, sum_i w4[i] T[b + 2 i m]
};

struct ScTailArgs {
    RoundArgs ra;          // ra.m = pairs of the first round handled here
    int rounds;            // rounds handled here (the last ones of the sumcheck), at least one
    int first_chal;        // challenge index of the round before the first one handled here
    DevState* st;
    uint32_t rounds_off;   // proof offset of g of the first round handled here
    uint32_t finals_off;
    int scal_base;
    int source;            // ScTailSource
    const Fr* w4;
    int first;                 // the first round here is the sumcheck's first: claim_0 = g(0) + g(1) is written, and
    uint32_t claim_off;        // absorbed (1) or not (2: the transcript already fixes it)
    uint32_t claim_copy_off;   // != 0: a second place in the proof for claim_0
};

constexpr int SC_TAIL_PAIRS = 512;
constexpr int SC_TAIL_LOG = 10;   // rounds handled in one block at most
constexpr int SC_TAIL_THREADS = 1024;
static_assert(SC_TAIL_THREADS >= SPEC_MIN_THREADS, "the waves beside the hashes");
constexpr int SC_TAIL_Q = 4;      // waves per evaluation point
static_assert(1 << SC_TAIL_LOG == 2 * SC_TAIL_PAIRS, "the tables of the first round fit");

template <int K>
struct ScTailLds {
    uint32_t el[K][9][2 * SC_TAIL_PAIRS];

    __device__ __forceinline__ F9 ld(int k, uint32_t i) const {
        F9 x;
#pragma unroll
        for (int l = 0; l < 9; ++l) x.v[l] = el[k][l][i];
        return x;
    }
    __device__ __forceinline__ void st(int k, uint32_t i, const F9& x) {
#pragma unroll
        for (int l = 0; l < 9; ++l) el[k][l][i] = x.v[l];
    }
};

template <int K>
struct ScTailShared {
    static constexpr int NPTS = K + 1, DEG = K < 2 ? 2 : K;     // K = 1 takes no round the short way
    ScTailLds<K> T;
    F9 qsum[NPTS][SC_TAIL_Q];
    uint32_t g[NPTS][8];                      // the round's evaluations, canonical
    F9 g9[NPTS];
    TsShared S;
    SpecShared<DEG> X;
    Fr f[4];
};

// entry i of table k of the first round (m pairs); v: the challenge that is bound, if one is
__device__ __forceinline__ F9 sc_tail_entry(const ScTailArgs& a, int k, uint32_t i, uint32_t m, const F9& v) {
    if (a.source == SC_SRC_PACKED) return fr_unpack(tab_ld(a.ra.src8[k], i));
    if (a.source == SC_SRC_PACKED_W4) {
        uint64_t cols[17];
#pragma unroll
        for (int c = 0; c < 17; ++c) cols[c] = 0;
#pragma unroll 1
        for (int q = 0; q < 4; ++q)
            f9_cols_mac(cols, fr_unpack(a.w4[q]), fr_unpack(tab_ld(a.ra.src8[k], i + 2ull * q * m)));
        f9_cols_norm<17>(cols);
        return f9_redc(cols);       // below 1.2 r
    }
    F9 t0, t1;
    if (a.source == SC_SRC_PACKED_FOLD) {
        t0 = fr_unpack(tab_ld(a.ra.src8[k], i));
        t1 = fr_unpack(tab_ld(a.ra.src8[k], i + 2ull * m));
    } else {
        t0 = f9tab_ld(a.ra.work[k], i);
        t1 = f9tab_ld(a.ra.work[k], i + 2ull * m);
    }
    return f9_norm_reduce(f9_add(t0, f9_mul(f9_sub(t1, t0), v)));
}

// prod_k of the lines of pair (b, b + m) at x = 0 .. 3: normal times normal at most
template <int K, class Tables>
__device__ __forceinline__ F9 sc_pair_value(const Tables& T, int x, uint32_t b, uint32_t m) {
    F9 prod = f9_zero();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        F9 e = T.ld(k, x == 0 ? b : b + m);
        if (x >= 2) {   // hi + (x - 1)(hi - lo); limbs below 2^30.6
            const F9 dn = f9_norm(f9_sub(e, T.ld(k, b)));
            e = f9_add(e, dn);
            if (x == 3) e = f9_add(e, dn);
            if (k == 0) e = f9_norm(e);   // the running product needs one normal factor
        }
        prod = k == 0 ? e : f9_mul(prod, e);
    }
    return prod;
}

// The final fold of the length-2 tables at v, finals into the proof and the transcript; keep_idx >= 0: v goes to that challenge
template <int K>
__device__ __forceinline__ void sc_tail_finals(const ScTailArgs& a, ScTailShared<K>& L, const F9& v, int keep_idx) {
    DevState* st = a.st;
    const int tid = threadIdx.x;
    if (tid < K) {
        const F9 lo = L.T.ld(tid, 0);
        const Fr x = f9_to_fr(f9_add(lo, f9_mul(f9_sub(L.T.ld(tid, 1), lo), v)));
        L.f[tid] = x;
        st->scal[a.scal_base + tid] = x;
    } else if (tid == 320 && keep_idx >= 0) {
        store_challenge(st, keep_idx, v);
    }
    __syncthreads();
    block_absorb_frs(L.S, 'f', L.f, K, (uint32_t*)(st->proof + a.finals_off));
    block_ts_store(L.S, st);
}

// The round's evaluations g9[x] (normal, below 4.4 r; one lane each) stand in L.g9 / L.g behind a barrier: claim_0 if it is due here.
template <int K>
__device__ __forceinline__ void sc_tail_claim(const ScTailArgs& a, ScTailShared<K>& L) {
    DevState* st = a.st;
    if (threadIdx.x == 0)
        round_claim_out(L.S, f9_norm(f9_add(L.g9[0], L.g9[1])), (uint32_t*)(st->proof + a.claim_off),
                        a.claim_copy_off ? (uint32_t*)(st->proof + a.claim_copy_off) : nullptr);
    __syncthreads();
}

// One round the long way: entries folded (read(k, i), in place or not) into W, the sums, the challenge.  shorter: the next round is taken the short way
// and its coefficients beside this one's hashes.
template <int K, class Tables, class Entry>
__device__ __forceinline__ F9 sc_tail_round(const ScTailArgs& a, ScTailShared<K>& L, Tables& W, int t, uint32_t m, bool shorter,
                                            const F9& v, Entry entry) {
    constexpr int NPTS = K + 1;
    DevState* st = a.st;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, beside = spec_beside_index(wave);
    const int lg = 32 - __clz((int)m);      // log2(2 m)
    for (uint32_t id = tid; id < ((uint32_t)K << lg); id += SC_TAIL_THREADS) {
        const int k = (int)(id >> lg);
        const uint32_t i = id & (2 * m - 1);
        W.st(k, i, entry(k, i));
    }
    __syncthreads();
    // evaluation point x: a wave goes to the SIMD of its index modulo four, so the waves of one quarter of the
    // pairs take neighbouring indices (all on one SIMD: 7.6 thousand cycles more)
    const int nq = m <= 64 ? 1 : m <= 128 ? 2 : SC_TAIL_Q;
    const int x = wave & 3, quarter = wave >> 2;
    if (x < NPTS && quarter < nq) {
        F9 acc = f9_zero();
        for (uint32_t b = 64 * quarter + lane; b < m; b += 64 * SC_TAIL_Q)
            acc = f9_norm_reduce(f9_add(acc, sc_pair_value<K>(W, x, b, m)));
        const F9 s = wave_sum_lazy(acc, m < 64 ? (int)m : 64);
        if (lane == 0) L.qsum[x][quarter] = s;
    }
    if (nq > 1) __syncthreads();
    else __builtin_amdgcn_wave_barrier();            // the wave's own sum
    if (x < NPTS && quarter == 0 && lane == 0) {
        F9 s = L.qsum[x][0];
        for (int q = 1; q < nq; ++q) s = f9_add(s, L.qsum[x][q]);
        s = f9_norm(s);                              // below 4.4 r
        if (t == 0 && a.first) L.g9[x] = s;
        const Fr plain = f9_canonical(s);
#pragma unroll
        for (int l = 0; l < 8; ++l) L.g[x][l] = plain.v[l];
    }
    __syncthreads();
    if (t == 0 && a.first) sc_tail_claim<K>(a, L);
    if (wave < 2) {
        // the transcript takes g(0), g(2), ..
        wave_frame_draw1_open(L.S, 'g', K, [&](uint32_t i) -> uint32_t { return L.g[i < 8 ? 0 : (i >> 3) + 1][i & 7]; },
                              t == 0 && a.first == 1);
    } else if (shorter && beside < NPTS) {
        if constexpr (K >= 2) spec_product_coefficients<K>(W, L.X, beside, 0, m >> 1);
    } else if (wave == 5) {
        // beside the hashes: this round's evaluations and the challenge before them
        uint32_t* dst = (uint32_t*)(st->proof + a.rounds_off) + 8 * NPTS * t;
        if (lane < 8 * NPTS) dst[lane] = L.g[lane >> 3][lane & 7];
        if (lane == 32 && t > 0) store_challenge(st, a.first_chal + t, v);
    }
    __syncthreads();
    return L.S.v9;
}

// The last rounds of a product sumcheck in one block, all of them up to 2^10 entries: once a round has at most a few
// pairs per thread, a kernel launch per round costs more than the round.  The folded tables live in LDS
// (2 SC_TAIL_PAIRS entries each, folded in place: entry i takes entry i + 2m, read by no other thread; `big` in front of them, while
// they are longer).  A round of
// more than SPEC_MAX_PAIRS pairs is two phases: a thread per (table, entry) folds, then wave (point, quarter) multiplies
// and sums its pairs; while waves 0 and 1 hash, wave 3 writes the proof.  g(1) is summed like the others (the waves of
// its SIMD would be idle), so that no claim is carried along.  Shorter rounds leave only the hashes in the
// chain (spec_rounds.cuh): 2^10 entries took 191 us with two tables when every round went through the phases and the
// first two through launches of their own.
template <int K, class Big>
__device__ __forceinline__ void sc_tail_block(const ScTailArgs& a, ScTailShared<K>& L, Big& big) {
    constexpr int NPTS = K + 1;
    DevState* st = a.st;
    const int tid = threadIdx.x, wave = tid >> 6, beside = spec_beside_index(wave);
    uint32_t m = (uint32_t)a.ra.m;
    F9 v = f9_zero();                                    // the challenge bound next
    if (a.source == SC_SRC_PACKED_FOLD || a.source == SC_SRC_WORK) v = fr_unpack(st->chal[a.first_chal]);
    auto fold = [&](auto& T, int k, uint32_t i, uint32_t half) {
        const F9 t0 = T.ld(k, i);
        return f9_norm_reduce(f9_add(t0, f9_mul(f9_sub(T.ld(k, i + half), t0), v)));
    };
    int t = 0;
    if constexpr (Big::LONG) {
        for (; m > SC_TAIL_PAIRS; ++t, m >>= 1)
            v = sc_tail_round<K>(a, L, big, t, m, false, v, [&](int k, uint32_t i) {
                return t == 0 ? sc_tail_entry(a, k, i, m, v) : fold(big, k, i, 2 * m);
            });
    }
    const int in_lds = t;
    while (t < a.rounds) {
        const bool shorter = K >= 2 && m <= 2 * SPEC_MAX_PAIRS && t + 1 < a.rounds;      // the next round
        v = sc_tail_round<K>(a, L, L.T, t, m, shorter, v, [&](int k, uint32_t i) {
            if (t == 0) return sc_tail_entry(a, k, i, m, v);
            if constexpr (Big::LONG)
                if (t == in_lds) return fold(big, k, i, 2 * m);
            return fold(L.T, k, i, 2 * m);
        });
        ++t;
        m >>= 1;
        if (shorter) break;
    }
    const int left = a.rounds - t;
    if (left > 0) {
        if constexpr (K >= 2) {
            if (wave == 0) spec_chain<K>(L.S, L.X, v, left);
            else if (wave == 1)
                spec_second<K>(L.S, L.X, st, left, a.rounds_off + (uint32_t)t * NPTS * 32, a.first_chal + 1 + t, v, true);
            else if (beside < NPTS)
                spec_beside<K>(L.T, K, L.X, beside, v, left, m,
                               [&](int round, uint32_t q) { spec_product_coefficients<K>(L.T, L.X, beside, round, q); }, [](const F9&) {});
        }
        __syncthreads();
        v = L.X.v9[(left - 1) & 1];
    }
    sc_tail_finals<K>(a, L, v, left == 0 ? a.first_chal + t : -1);
}
struct ScNoBig {
    static constexpr bool LONG = false;
};
