// The short rounds of a sumcheck inside one block, with the sums of a round taken before its challenge is known.
//
// A round's evaluations g_t(x) are polynomials in the challenge v_{t-1} that has not been drawn yet:
//   g_t(x) = sum_i P_t[x][i] v_{t-1}^i,  i <= the degree.
// While wave 0 hashes round t-1, other waves take the coefficients P_t from the tables with v_{t-2} bound, so that
// once v_{t-1} is drawn wave 0 needs two products in a row for all g_t(x) and hashes on: what a round adds to the
// chain of challenges is its two compressions, three products and no barrier.  With fold, sums and barriers in that
// chain a round of few pairs took 26 thousand cycles (two tables; 30 thousand for three), of which the hashes were 12 with
// a lane per compression and are 9 with two.
// The waves of the block meet through counters in LDS: the operations of one wave on LDS complete in order, every
// counter only grows, and whoever waits waits for work that does not depend on the waiting wave's own later steps.
#pragma once
#include "dev_common.cuh"

// rounds of at most this many pairs are taken this way: above it the sums take longer than the hashes they run next to
constexpr uint32_t SPEC_MAX_PAIRS = 32;
// waves 0 and 1 hash, waves 2, 3, 6, 7 take the coefficients (and with them wave 5 may write the proof of the round before)
constexpr int SPEC_MIN_THREADS = 512;

template <int DEG>
struct SpecShared {
    F9 P[2][DEG + 1][4];              // [round & 1]: coefficients, plain form (not Montgomery), normal, below 1.1 r
    uint32_t out[2][DEG + 1][8];      // evaluations, canonical
    F9 v9[2];                         // challenges, normal, below 2.1 r
    uint32_t v_done;                  // challenges drawn here
    uint32_t w_done;                  // rounds whose message words stand in LDS
    uint32_t p_done[DEG + 1];         // rounds whose coefficients stand in P
    uint32_t folded;                  // folds done, counted by wave
    uint32_t dump[4];                 // where lanes without a word to write put it
};

typedef volatile __attribute__((address_space(3))) uint32_t* spec_vptr;
typedef volatile __attribute__((address_space(3))) uint16_t* spec_vptr16;
__device__ __forceinline__ spec_vptr spec_ptr(uint32_t* p) { return (spec_vptr)(__attribute__((address_space(3))) uint32_t*)p; }
// waves 2, 3, 6, 7, on the SIMDs that the hashes of waves 0 and 1 leave free: 0 .. 3; the others: 4
__device__ __forceinline__ int spec_beside_index(int wave) { return (wave & 2) && wave < 8 ? ((wave >> 2) << 1) | (wave & 1) : 4; }
// an entry pair bound at v
__device__ __forceinline__ F9 spec_bind(const F9& lo, const F9& hi, const F9& v) {
    return f9_norm_reduce(f9_add(lo, f9_mul(f9_sub(hi, lo), v)));
}
__device__ __forceinline__ void spec_order() { asm volatile("" ::: "memory"); }   // keeps the compiler from moving LDS accesses
template <int SLEEP = 1>
__device__ __forceinline__ void spec_wait(uint32_t* counter, uint32_t at_least) {
    while (__builtin_amdgcn_readfirstlane(*spec_ptr(counter)) < at_least) __builtin_amdgcn_s_sleep(SLEEP);
    spec_order();
}
__device__ __forceinline__ void spec_post(uint32_t* counter, uint32_t value) {
    spec_order();
    if ((threadIdx.x & 63) == 0) *spec_ptr(counter) = value;
    spec_order();
}

// one thread, before a barrier
template <int DEG>
__device__ __forceinline__ void spec_init(SpecShared<DEG>& X) {
    X.v_done = X.w_done = X.folded = 0;
    for (int x = 0; x <= DEG; ++x) X.p_done[x] = 0;
}

// Bytes of the 'g' frame of DEG evaluations behind a block boundary.  Its block rows: the whole block, then the draw's
// three, which begin with the frame's other REM bytes.
template <int DEG>
struct SpecFrame {
    static constexpr uint32_t DATA = 32u * DEG, REM = (10u + DATA) % 64;
    static_assert((10u + DATA) / 64 == 1 && REM <= 50, "one whole block, one closing block per hash");
};

// Wave 0: `rounds` rounds.  The stream is block-aligned; v_prev (normal, below 2.1 r) is the challenge before the
// first of them.
template <int DEG>
__device__ __forceinline__ void spec_chain(TsShared& S, SpecShared<DEG>& X, F9 v, int rounds) {
    using FR = SpecFrame<DEG>;
    const uint32_t lane = threadIdx.x & 63, x = (lane >> 2) & 3, i = lane & 3;
    // what does not change in the block rows: the frame's head, tags (byte REM), 0x80 behind the index; the length is
    // written in every round
    {
        const uint32_t row = lane >> 4, w = lane & 15;
        uint32_t word = 0;
        if (lane == 0) word = (1u << 24) | ((uint32_t)'g' << 16) | ((FR::DATA & 0xffu) << 8);
        if (row >= 1) {
            if (w == FR::REM >> 2) word |= (0xF0u + row - 1) << (24 - 8 * (FR::REM & 3));
            if (row < 3 && w == (FR::REM + 5) >> 2) word |= 0x80u << (24 - 8 * ((FR::REM + 5) & 3));
        }
        S.msg[lane] = word;
    }
    spec_order();
    uint64_t nblk = S.nblk;
    // evaluation x >= 2 stands in slot x - 1 of the frame (the transcript does not take x = 1); lane 4 x + i writes its
    // words of block row i
    const uint32_t slot = x == 0 ? 0 : x - 1;
    const bool writes = lane < 16 && x != 1 && x <= DEG;
    for (int t = 0; t < rounds; ++t) {
        for (int y = 0; y <= DEG; ++y) spec_wait(&X.p_done[y], (uint32_t)t + 1);
        F9 p = f9_zero();
        if (x <= DEG && i <= DEG) p = X.P[t & 1][x][i];
        // level 1: P1 v (i = 1), v v (i = 2), P3 v (i = 3); level 2 (i = 2): (P2 + P3 v) v^2
        const F9 q1 = f9_mul(i == 2 ? v : p, v);
        F9 s = p;
        if (DEG == 3) {
#pragma unroll
            for (int l = 0; l < 9; ++l) s.v[l] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)q1.v[l], 0xB1, 0xf, 0xf, true);
        }
        const F9 q2 = f9_mul(s, q1);
        F9 g = i == 0 ? p : i == 1 ? q1 : i == 2 ? q2 : f9_zero();
        f9_add_dpp<0xB1>(g);
        f9_add_dpp<0x4E>(g);                       // all four lanes: below 3.4 r, limbs below 3 * 2^29
        const Fr plain = fr_pack(f9_cond_sub(f9_norm_reduce_sum(g)));
        if (lane < 16 && i == 0 && x <= DEG) {
#pragma unroll
            for (int l = 0; l < 8; ++l) X.out[t & 1][x][l] = plain.v[l];
        }
        {
            // limb l stands in the lower half of word 2 + 8 slot + l and the upper half of the next
            uint32_t b[8];
#pragma unroll
            for (int l = 0; l < 8; ++l) b[l] = sha::bswap32(plain.v[l]);
#pragma unroll
            for (int j = 0; j <= 8; ++j) {
                const uint32_t k = 2 + 8 * slot + j;
                const bool mine = writes && (i == 0) == (k < 16);
                const spec_vptr at = spec_ptr(mine ? S.msg + 16 * i + (k & 15) : X.dump);
                if (j == 0) *(spec_vptr16)at = (uint16_t)(b[0] >> 16);
                else if (j == 8) *((spec_vptr16)at + 1) = (uint16_t)b[7];
                else *at = __builtin_amdgcn_alignbit(b[j - 1], b[j], 16);
            }
        }
        if (lane >= 16 && lane < 18) {             // the length of the hashed stream, in bits
            const uint64_t bits = ((nblk + 1) * 64u + FR::REM + 5u) * 8u;
            S.msg[16 * (lane - 15) + 14] = (uint32_t)(bits >> 32);
            S.msg[16 * (lane - 15) + 15] = (uint32_t)bits;
        }
        spec_post(&X.w_done, (uint32_t)t + 1);
        const F9 m = ts_frame_passes(S, 1, 4u * (uint32_t)t);
        nblk += 2;
#pragma unroll
        for (int l = 0; l < 9; ++l) v.v[l] = __builtin_amdgcn_readfirstlane(m.v[l]);
        if (lane == 0) X.v9[t & 1] = v;
        spec_post(&X.v_done, (uint32_t)t + 1);
    }
    if (lane == 0) {
        S.nblk = nblk;
        S.fill = 0;
        S.seq = 0;
    }
}

// Wave 1: the schedules; evaluations to the proof at rounds_off, challenges to chal_idx, .. (the one before the first
// round, `before`, to chal_idx - 1 if keep_before)
template <int DEG>
__device__ __forceinline__ void spec_second(TsShared& S, SpecShared<DEG>& X, DevState* st, int rounds, uint32_t rounds_off,
                                            int chal_idx, const F9& before, bool keep_before) {
    const uint32_t lane = threadIdx.x & 63;
    for (int t = 0; t < rounds; ++t) {
        spec_wait(&X.w_done, (uint32_t)t + 1);
        ts_schedules(S, 4, 4u * (uint32_t)t);
        uint32_t* dst = (uint32_t*)(st->proof + rounds_off) + 8 * (DEG + 1) * t;
        if (lane < 8 * (DEG + 1)) dst[lane] = X.out[t & 1][lane >> 3][lane & 7];
        if (lane == 32 && (t > 0 || keep_before)) store_challenge(st, chal_idx + t - 1, t > 0 ? X.v9[(t - 1) & 1] : before);
    }
    spec_wait(&X.v_done, (uint32_t)rounds);
    if (lane == 32 && rounds > 0) store_challenge(st, chal_idx + rounds - 1, X.v9[(rounds - 1) & 1]);
}

// Small-integer combination c0 a0 + .. + c3 a3 of normal values below 2.42 r, reduced: normal, below 1.1 r.  The sum of the |c| is at
// most 15 or so: 40 r is added, so that the value is between 2 r and 80 r and the estimate of its quotient never too large.
__device__ __forceinline__ F9 f9_combine4(const int (&c)[4], const F9& a0, const F9& a1, const F9& a2, const F9& a3) {
    int64_t acc[9];
#pragma unroll
    for (int l = 0; l < 9; ++l) {
        int64_t s = 40ll * (int64_t)frc::MOD9[l];
        s += (int64_t)c[0] * (int32_t)a0.v[l];
        s += (int64_t)c[1] * (int32_t)a1.v[l];
        s += (int64_t)c[2] * (int32_t)a2.v[l];
        s += (int64_t)c[3] * (int32_t)a3.v[l];
        acc[l] = s;
    }
    const int64_t q = (int64_t)(((uint64_t)(uint32_t)acc[8] * 565u) >> 32);
    F9 o;
    int64_t carry = 0;
#pragma unroll
    for (int l = 0; l < 8; ++l) {
        const int64_t y = acc[l] - q * (int64_t)frc::MOD9[l] + carry;
        o.v[l] = (uint32_t)y & frc::M29;
        carry = y >> 29;
    }
    o.v[8] = (uint32_t)(acc[8] - q * (int64_t)frc::MOD9[8] + carry);
    return o;
}

// Row of 16 lanes: the value y of the challenge before (0, 1, (DEG = 3: -1,) infinity) at which it takes the polynomial.
// c: the combination of T(b), T(b + q), T(b + 2 q), T(b + 3 q) that a table's line through x and y is
template <int DEG>
__device__ __forceinline__ void spec_line(int row, int x, int (&c)[4]) {
    const int y0 = row == 0 ? 1 : row == 1 ? 0 : (DEG == 3 && row == 2) ? 2 : -1;    // the line in y: y0 T_0 + y1 T_1
    const int y1 = row == 0 ? 0 : row == 1 ? 1 : (DEG == 3 && row == 2) ? -1 : 1;
    c[0] = y0 * (1 - x);
    c[1] = y0 * x;
    c[2] = y1 * (1 - x);
    c[3] = y1 * x;
}

// The coefficients in y of a polynomial of degree DEG from its values at y = 0, 1, (DEG = 3: -1,) infinity, one value per
// row of 16 lanes (the same in all its lanes, normal, below 1.1 r, Montgomery), to P in plain form.  One wave.
template <int DEG>
__device__ __forceinline__ void spec_coefficients(SpecShared<DEG>& X, int x, int round, const F9& value) {
    const int lane = threadIdx.x & 63, i = lane & 3;
    F9 y[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int l = 0; l < 9; ++l) y[q].v[l] = q <= DEG ? (uint32_t)__builtin_amdgcn_readlane((int)value.v[l], 16 * q) : 0u;
    // DEG 2: c0 = s0, c1 = s1 - s0 - s2, c2 = s2.  DEG 3 (values s0, s1, s-1, s_inf): c0 = s0, c3 = s_inf and, doubled,
    // c1 = s1 - s-1 - 2 s_inf, c2 = s1 + s-1 - 2 s0
    int c[4] = {0, 0, 0, 0};
    if (i == 0) c[0] = 1;
    else if (DEG == 2 && i == 1) { c[0] = -1; c[1] = 1; c[2] = -1; }
    else if (DEG == 2 && i == 2) c[2] = 1;
    else if (DEG == 3 && i == 1) { c[1] = 1; c[2] = -1; c[3] = -2; }
    else if (DEG == 3 && i == 2) { c[0] = -2; c[1] = 1; c[2] = 1; }
    else if (DEG == 3 && i == 3) c[3] = 1;
    const F9 s = f9_combine4(c, y[0], y[1], y[2], y[3]);
    // times the plain integers 1 and 1/2 = (r + 1) / 2: out of the Montgomery form
    constexpr uint32_t HALF[8] = {0x80000001u, 0x7fffffffu, 0x7fff2dffu, 0xa9ded201u,
                                  0x04d0ec02u, 0x199cec04u, 0x94cebea4u, 0x39f6d3a9u};
    Fr one = fr_zero();
    one.v[0] = 1;
    const F9 k = fr_unpack(DEG == 3 && (i == 1 || i == 2) ? fr_const(HALF) : one);
    const F9 o = f9_mul(s, k);           // below 1.02 r
    if (lane <= DEG) X.P[round & 1][x][lane] = o;
    spec_post(&X.p_done[x], (uint32_t)round + 1);
}

// One wave: the coefficients in the challenge of the round before of g(x), a sum of products of K tables, for a round of q pairs,
// from tables of 4 q entries.  Rows of 16 lanes take the values y = 0, 1, (K = 3: -1,) infinity of that challenge, the
// lanes of a row the pairs.
template <int K, class Tables>
__device__ __forceinline__ void spec_product_coefficients(Tables& T, SpecShared<K>& X, int x, int round, uint32_t q) {
    const int lane = threadIdx.x & 63, row = lane >> 4;
    int c[4];
    spec_line<K>(row, x, c);
    F9 acc = f9_zero();
    // Lanes without a pair compute too: with few lanes of a wave at work in such a loop everything on the compute unit ran up to
    // twice as long every other time (hashes of 10.3 thousand cycles a round took 14 to 19).
    for (uint32_t b0 = 0; b0 < q; b0 += 16) {       // at most SPEC_MAX_PAIRS / 16 sums of normal values
        const uint32_t mine = b0 + (lane & 15), b = mine < q ? mine : 0;
        F9 prod = f9_zero();
#pragma unroll 1
        for (int k = 0; k < K; ++k) {
            const F9 e = f9_combine4(c, T.ld(k, b), T.ld(k, b + q), T.ld(k, b + 2 * q), T.ld(k, b + 3 * q));
            prod = k == 0 ? e : f9_mul(prod, e);
        }
        if (mine >= q) prod = f9_zero();
        acc = f9_add(acc, prod);
    }
    spec_coefficients<K>(X, x, round, wave_sum_lazy(f9_norm(acc), 16));
}

// Waves 2, 3, 6, 7 (on the two SIMDs that the hashes leave free): point x = 0 .. DEG beside the hashes of `rounds`
// rounds of `ntab` tables.  Before round t: tables of 4 q entries that round's coefficients are taken from already, q pairs
// in round 0.  coef(t, q): the coefficients of round t; each(v): what else is done with the challenge before round t.
// first > 0: rounds 0 .. first - 1 are over, each wave has counted once in X.folded, and q belongs to round `first`.
template <int DEG, class Tables, class Coef, class Each>
__device__ __forceinline__ void spec_beside(Tables& T, int ntab, SpecShared<DEG>& X, int x, F9 v, int rounds, uint32_t q, Coef coef,
                                            Each each, int first = 0) {
    const uint32_t lane = threadIdx.x & 63, counted = first ? 1u : 0u;
    for (int t = first; t < rounds; ++t, q >>= 1) {
        // the tables may be folded once every point has its coefficients of round t from them
        if (t > 0) spec_wait<8>(&X.v_done, (uint32_t)t);
        for (int y = 0; y <= DEG; ++y) spec_wait(&X.p_done[y], (uint32_t)t + 1);
        if (t > 0) v = X.v9[(t - 1) & 1];
        const uint32_t lg = 32 - __clz((int)q);          // log2(2 q)
        for (uint32_t id = 64 * x + lane; id < ((uint32_t)ntab << lg); id += 64 * (DEG + 1)) {
            const int k = (int)(id >> lg);
            const uint32_t i = id & (2 * q - 1);
            const F9 t0 = T.ld(k, i);
            T.st(k, i, f9_norm_reduce(f9_add(t0, f9_mul(f9_sub(T.ld(k, i + 2 * q), t0), v))));
        }
        spec_order();
        if (lane == 0) __hip_atomic_fetch_add(&X.folded, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        spec_wait(&X.folded, (uint32_t)(DEG + 1) * ((uint32_t)(t - first) + 1 + counted));
        if (t + 1 < rounds) coef(t + 1, q >> 1);
        each(v);
    }
}
