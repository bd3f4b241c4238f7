// The last i-rounds of zkReLU, from 2^9 rows of tables on, in one launch with helper blocks (help.cuh).
//
// With a launch for the sums and one for the hashes a round takes 30 us however few rows it has, and in one block (k_zk_short) 16 to 26 us
// a round of at most 8 pairs.  Here the columns of the bits are dealt out, two to a helper, with a copy of beta_I each, and the four linear
// equations to four helpers each, one for each point x; every table stays in its helper's LDS to the last pair of rows.  What they
// send is the sums of a round ahead of its challenge, as polynomials in the one before it, so that a round in the leader is its
// hashes (6 us) and the part of the helpers' work that is longer than they are.
//
// Bound by a helper's latency: a turn from one challenge to the message after it is 17 to 18 thousand cycles at few rows (tables and sums
// bound 7, squares 3.5, sums 6 to 7, the message 1), 27 with 512 rows, and 6 to 12 on the way through memory, next to 14 for the leader's
// hashes: a round takes 27 to 34.  Whole zkrelu_prove calls (us,
// launches per round and one block for the last / like this): two slices of 48 columns 2^9 rows 514 / 492, 2^12 622 / 559, 2^14 692 / 599,
// 2^19 989 / 919; two of 7 2^12 588 / 449, 2^14 773 / 521, 2^19 1156 / 885.
//
// The binarity part of a round over pairs of rows is beta_I(x) B(x), B(x) = sum_j w_j (e_j^2 - e_j) a quadratic in x.  With P[i] the
// sum at row i and D[b] = sum_j w_j (e_hi - e_lo)^2 of a pair, binding y in P and D needs no columns:
//   P(y) = P_lo + y (P_hi - P_lo) + y (y - 1) D,    D(y) = Q_0 + y (Q_1 - Q_0) + y (y - 1) Q_inf,
// Q_0, Q_1, Q_inf the sums of (e_hi - e_lo)^2 at y = 0, 1 and of its leading coefficient: three squares per column and four rows are
// all that a round takes from the columns, and B(x) at any y follows from nine sums.
#include "help.cuh"
#include "spec_rounds.cuh"

namespace {

constexpr int ZH_THREADS = 1024, ZH_ROWS = 2 * ZK_ZHELP_PAIRS, ZH_PARTS = 8;
constexpr int ZH_COLUMNS = (2 * 64 + 1) / 2, ZH_EQS = 4;    // helpers with columns (two slices of at most 64, in pairs), linear equations, at most
static_assert(ZH_COLUMNS + ZH_EQS <= ZK_HELP_SLOTS, "a place for the message of every pair of columns and of every equation");
static_assert(ZH_COLUMNS + 4 * ZH_EQS <= ZK_HELP_SLOTS, "zk_helpers_fit counts that many helpers");
constexpr int LIN = 10;                   // tables: (1 - sign) | beta_Z Z | beta_A Z' | beta_GA G_A | beta_GZ G_A' | beta_I

template <int N>
using Plane9 = uint32_t[9][N];
template <int N>
__device__ __forceinline__ F9 ld9(const Plane9<N>& t, uint32_t i) {
    F9 x;
#pragma unroll
    for (int l = 0; l < 9; ++l) x.v[l] = t[l][i];
    return x;
}
template <int N>
__device__ __forceinline__ void st9(Plane9<N>& t, uint32_t i, const F9& x) {
#pragma unroll
    for (int l = 0; l < 9; ++l) t[l][i] = x.v[l];
}

struct ZhMessage {
    F9 sum[ZH_PARTS][4][4];       // [part][x][row]
    F9 v;
    uint32_t stop;
};
struct ZhColumns {
    ZhMessage M;
    Plane9<ZH_ROWS> col[2], beta, P;
    Plane9<ZH_ROWS / 2> D[2];     // by the round's lowest bit
    Plane9<ZH_ROWS / 4> Q[3];
    F9 w[2];                      // beta_J, times r' in the second slice
};
struct ZhLinear {
    ZhMessage M;
    Plane9<ZH_ROWS> tab[3];
};
struct ZhLeader {
    TsShared S;
    SpecShared<3> X;
    uint32_t g[4][8];
    F9 weight[2][64];             // of a leader that goes on alone: beta_J, r' beta_J
    F9 part[3][ZK_ZHELP_PAIRS];   // its sums over the columns
    F9 sum[4][4];
    uint32_t alone;
};

__device__ __forceinline__ F9 col_weight(const ZkShortJob& a, int k, int j) {
    return fr_unpack(k == 0 ? a.bJ[j] : fr_mul_ni(*a.rp, a.bJ[j]));
}
__device__ __forceinline__ F9Tab col_table(const ZkShortJob& a, int k, int j) {
    F9Tab t;
    t.p = a.aux + (uint64_t)(k * a.nbits + j) * 9 * a.ps;
    t.ps = a.ps;
    return t;
}
// tables of the linear equation e: tab[which], which < 2 (+ 1 where 1 - sign is a factor)
__device__ __forceinline__ int lin_table(int e, int which) { return which == 2 ? 0 : 1 + 2 * e + which; }

// A quadratic's values from (value at 0, value at 1, leading coefficient) as a combination of them: normal, below 1.1 r.  row: the place in
// y of a row of lanes (0, 1, -1, infinity)
__device__ __forceinline__ F9 combine3(int c0, int c1, int c2, const F9& a0, const F9& a1, const F9& a2) {
    const int c[4] = {c0, c1, c2, 0};
    return f9_combine4(c, a0, a1, a2, a2);
}
__device__ __forceinline__ F9 quad_y(int row, const F9& a0, const F9& a1, const F9& lead) {
    return combine3(row == 0 ? 1 : row == 2 ? 2 : 0, row == 1 ? 1 : row == 2 ? -1 : 0, row == 2 ? 2 : row == 3 ? 1 : 0, a0, a1, lead);
}
__device__ __forceinline__ F9 quad_x(int x, const F9& a0, const F9& a1, const F9& lead) {
    return combine3(x == 0 ? 1 : x == 1 ? 0 : 1 - x, x, x * (x - 1), a0, a1, lead);
}
// the line through (lo, hi) at x = 0 .. 3, limbs below 2^30.6
__device__ __forceinline__ F9 line_at(int x, const F9& lo, const F9& hi) {
    if (x == 0) return lo;
    if (x == 1) return hi;
    const F9 d = f9_norm(f9_sub(hi, lo));
    F9 e = f9_add(hi, d);
    if (x == 3) e = f9_add(e, d);
    return e;
}

// the message of round t, from the parts' sums: points x0 .. x1 - 1, slot `slot` (all threads call)
__device__ __forceinline__ void zh_send(ZhMessage& M, ZkHelpMail* mail, int slot, int t, int x0, int x1, int parts) {
    const int tid = threadIdx.x, x = tid >> 2, row = tid & 3;
    __syncthreads();
    if (tid < 16 && x >= x0 && x < x1 && (t > 0 || row == 0) && !M.stop) {
        F9 s = M.sum[0][x][row];
        for (int p = 1; p < parts; ++p) s = f9_add(s, M.sum[p][x][row]);     // at most 8 normal values below 2.41 r
        help_write(mail->coef[t & 1][tid][slot], help_tag(t), f9_norm_reduce_sum(s));
    }
}

// every challenge but the last one of the call; false: none comes any more
__device__ __forceinline__ bool zh_challenge(ZhMessage& M, const ZkHelpLaunch& help, int t) {
    if (threadIdx.x < 64 && !help_challenge(help, t, M.v) && threadIdx.x == 0) M.stop = 1;
    __syncthreads();
    return M.stop == 0;
}

__device__ __forceinline__ void zh_columns(const ZkShortJob& a, DevState* st, const ZkHelpLaunch& help, ZhColumns& H, int h) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, x = wave & 3, row = lane >> 4;
    const int slices = a.has_ga ? 2 : 1, total = slices * a.nbits;
    const F9 one9 = fr_unpack(fr_one());
    F9 v = fr_unpack(st->chal[a.chal - 1]);
    uint32_t n = 2 * (uint32_t)a.pairs;
    if (tid < 2) {
        const int id = 2 * h + tid, k = id / a.nbits;
        H.w[tid] = id < total ? col_weight(a, k, id - k * a.nbits) : f9_zero();
    }
    for (uint32_t id = tid; id < 3 * n; id += ZH_THREADS) {
        const int c = (int)(id / n), at = 2 * h + c, k = at / a.nbits;
        const uint32_t i = id & (n - 1);
        F9 e = f9_zero();
        if (c == 2 || at < total) {
            const F9Tab t = c == 2 ? a.tab[9] : col_table(a, k, at - k * a.nbits);
            e = spec_bind(f9tab_ld(t, i), f9tab_ld(t, i + n), v);
        }
        if (c == 2) st9(H.beta, i, e);
        else st9(H.col[c], i, e);
    }
    __syncthreads();
    for (uint32_t id = tid; id < n + n / 2; id += ZH_THREADS) {
        F9 s = f9_zero();
        const uint32_t i = id < n ? id : id - n;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const F9 e = ld9(H.col[c], i);
            F9 z;
            if (id < n) z = f9_mul(e, f9_sub(e, one9));
            else z = f9_sqr(f9_norm(f9_sub(ld9(H.col[c], i + n / 2), e)));
            s = f9_add(s, f9_mul(H.w[c], z));
        }
        s = f9_norm_reduce(s);
        if (id < n) st9(H.P, i, s);
        else st9(H.D[0], i, s);
    }
    __syncthreads();
    {
        const uint32_t q = n >> 1;
        const int part = wave >> 2, parts = q <= 64 ? 1 : q <= 128 ? 2 : 4;
        if (part < parts) {
            F9 acc = f9_zero();
            for (uint32_t b0 = 64 * part; b0 < q; b0 += 256) {
                const uint32_t mine = b0 + lane, b = mine < q ? mine : 0;
                const F9 B = quad_x(x, ld9(H.P, b), ld9(H.P, b + q), ld9(H.D[0], b));
                F9 s = f9_mul(B, line_at(x, ld9(H.beta, b), ld9(H.beta, b + q)));
                if (mine >= q) s = f9_zero();
                acc = f9_norm_reduce(f9_add(acc, s));
            }
            const F9 s = wave_sum_lazy(acc);
            if (lane == 0) H.M.sum[part][x][0] = s;
        }
        if (wave == 0 && !help_may_go(help) && lane == 0) H.M.stop = 1;
        zh_send(H.M, help.mail, h, 0, 0, 4, parts);
        if (H.M.stop) return;
    }
    for (int t = 1;; ++t) {
        const uint32_t q = n >> 2;
        Plane9<ZH_ROWS / 2>& D = H.D[(t - 1) & 1];
        // Q: a thread per square, the two columns in neighbouring lanes
        for (uint32_t id0 = 64 * wave; id0 < 6 * q; id0 += ZH_THREADS) {
            const uint32_t mine = id0 + lane, id = mine < 6 * q ? mine : lane & 1;
            const int which = (int)(id / (2 * q)), c = lane & 1;
            const uint32_t b = (id % (2 * q)) >> 1;
            const int k[4] = {which == 1 ? 0 : which == 0 ? -1 : 1, which == 1 ? 0 : which == 0 ? 1 : -1, which == 0 ? 0 : -1, which == 0 ? 0 : 1};
            const F9 z = f9_combine4(k, ld9(H.col[c], b), ld9(H.col[c], b + q), ld9(H.col[c], b + 2 * q), ld9(H.col[c], b + 3 * q));
            F9 s = f9_mul(H.w[c], f9_sqr(z));
            f9_add_dpp<0xB1>(s);
            s = f9_norm_reduce(s);
            if (mine < 6 * q && c == 0) st9(H.Q[which], b, s);
        }
        __syncthreads();
        const int part = wave >> 2, parts = q <= 16 ? 1 : q <= 32 ? 2 : 4;
        if (part < parts) {
            int c[4];
            spec_line<3>(row, x, c);
            F9 acc = f9_zero();
            for (uint32_t b0 = 16 * part; b0 < q; b0 += 64) {
                const uint32_t mine = b0 + (lane & 15), b = mine < q ? mine : 0;
                F9 B;
                if (x == 0) {
                    B = quad_y(row, ld9(H.P, b), ld9(H.P, b + 2 * q), ld9(D, b));
                } else if (x == 1) {
                    B = quad_y(row, ld9(H.P, b + q), ld9(H.P, b + 3 * q), ld9(D, b + q));
                } else {
                    const F9 B0 = quad_y(row, ld9(H.P, b), ld9(H.P, b + 2 * q), ld9(D, b));
                    const F9 B1 = quad_y(row, ld9(H.P, b + q), ld9(H.P, b + 3 * q), ld9(D, b + q));
                    B = quad_x(x, B0, B1, quad_y(row, ld9(H.Q[0], b), ld9(H.Q[1], b), ld9(H.Q[2], b)));
                }
                const F9 e = f9_combine4(c, ld9(H.beta, b), ld9(H.beta, b + q), ld9(H.beta, b + 2 * q), ld9(H.beta, b + 3 * q));
                F9 s = f9_mul(B, e);
                if (mine >= q) s = f9_zero();
                acc = f9_norm_reduce(f9_add(acc, s));
            }
            const F9 s = wave_sum_lazy(acc, 16);
            if ((lane & 15) == 0) H.M.sum[part][x][row] = s;
        }
        zh_send(H.M, help.mail, h, t, 0, 4, parts);
        if (!zh_challenge(H.M, help, t - 1)) return;
        v = H.M.v;
        const uint32_t half = n >> 1;
        // all lanes of a wave compute, also those without an entry (see spec_product_coefficients)
        if (wave < 8) {                    // tables
            for (uint32_t id0 = 64 * wave; id0 < 3 * half; id0 += 512) {
                const uint32_t mine = id0 + lane, id = mine < 3 * half ? mine : 0, i = id & (half - 1);
                const int c = (int)(id / half);
                Plane9<ZH_ROWS>& T = c == 2 ? H.beta : H.col[c];
                const F9 e = spec_bind(ld9(T, i), ld9(T, i + half), v);
                if (mine < 3 * half) st9(T, i, e);
            }
        } else {                           // sums: P on waves 10, 11, 8, 9, D on 15, 12, 13, 14: short ones on a SIMD that has nothing else
            const bool second = wave >= 12;
            const uint32_t count = second ? q : half;
            for (uint32_t i0 = 64 * ((wave + (second ? 1 : 2)) & 3); i0 < count; i0 += 256) {
                const uint32_t mine = i0 + lane, i = mine < count ? mine : 0;
                F9 lo, hi, lead;
                if (second) {
                    lo = ld9(H.Q[0], i);
                    hi = ld9(H.Q[1], i);
                    lead = ld9(H.Q[2], i);
                } else {
                    lo = ld9(H.P, i);
                    hi = ld9(H.P, i + half);
                    lead = ld9(D, i);
                }
                // lo + v (hi - lo + (v - 1) lead)
                const F9 slope = f9_norm(f9_add(f9_sub(hi, lo), f9_mul(lead, f9_sub(v, one9))));
                const F9 s = f9_norm_reduce(f9_add(lo, f9_mul(slope, v)));
                if (mine < count) {
                    if (second) st9(H.D[t & 1], i, s);
                    else st9(H.P, i, s);
                }
            }
        }
        n = half;
        __syncthreads();
        if (n == 2) break;
    }
    if (tid == 0) help_report(help);      // the last challenge is read
    // the last pair, not bound
    if (tid < 6) {
        const int c = tid >> 1, at = 2 * h + c, k = at / a.nbits;
        const uint32_t i = tid & 1;
        if (c == 2) {
            if (h == 0) f9tab_st(a.beta_out, i, ld9(H.beta, i));
        } else if (at < total) {
            f9tab_st(col_table(a, k, at - k * a.nbits), i, ld9(H.col[c], i));
        }
    }
}

// equation e at point x
__device__ __forceinline__ void zh_linear(const ZkShortJob& a, DevState* st, const ZkHelpLaunch& help, ZhLinear& H, int e, int x, int slot) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, row = lane >> 4, nt = (e & 1) ? 3 : 2;
    F9 v = fr_unpack(st->chal[a.chal - 1]);
    uint32_t n = 2 * (uint32_t)a.pairs;
    for (uint32_t id = tid; id < nt * n; id += ZH_THREADS) {
        const int k = (int)(id / n);
        const uint32_t i = id & (n - 1);
        const F9Tab t = a.tab[lin_table(e, k)];
        st9(H.tab[k], i, spec_bind(f9tab_ld(t, i), f9tab_ld(t, i + n), v));
    }
    __syncthreads();
    {
        const uint32_t q = n >> 1;
        const int parts = q <= 64 ? 1 : q <= 128 ? 2 : 4;
        if (wave < parts) {
            const uint32_t mine = 64 * wave + lane, b = mine < q ? mine : 0;
            F9 s = f9_norm(line_at(x, ld9(H.tab[0], b), ld9(H.tab[0], b + q)));
            for (int k = 1; k < nt; ++k) s = f9_mul(s, line_at(x, ld9(H.tab[k], b), ld9(H.tab[k], b + q)));
            s = f9_norm_reduce(s);
            if (mine >= q) s = f9_zero();
            s = wave_sum_lazy(s);
            if (lane == 0) H.M.sum[wave][x][0] = s;
        }
        if (wave == 0 && !help_may_go(help) && lane == 0) H.M.stop = 1;
        zh_send(H.M, help.mail, slot, 0, x, x + 1, parts);
        if (H.M.stop) return;
    }
    int c[4];
    spec_line<3>(row, x, c);
    for (int t = 1;; ++t) {
        __syncthreads();
        const uint32_t q = n >> 2;
        const int parts = (int)((q + 15) >> 4);
        if (wave < parts) {
            const uint32_t mine = 16 * wave + (lane & 15), b = mine < q ? mine : 0;
            F9 s = f9_zero();
#pragma unroll 1
            for (int k = 0; k < nt; ++k) {
                const F9 y = f9_combine4(c, ld9(H.tab[k], b), ld9(H.tab[k], b + q), ld9(H.tab[k], b + 2 * q), ld9(H.tab[k], b + 3 * q));
                s = k == 0 ? y : f9_mul(s, y);
            }
            if (mine >= q || (row == 3 && nt == 2)) s = f9_zero();       // two factors have no third power of y
            s = wave_sum_lazy(s, 16);
            if ((lane & 15) == 0) H.M.sum[wave][x][row] = s;
        }
        zh_send(H.M, help.mail, slot, t, x, x + 1, parts);
        if (!zh_challenge(H.M, help, t - 1)) return;
        v = H.M.v;
        const uint32_t half = n >> 1;
        for (uint32_t id0 = 64 * wave; id0 < nt * half; id0 += ZH_THREADS) {
            const uint32_t mine = id0 + lane, id = mine < nt * half ? mine : 0, i = id & (half - 1);
            Plane9<ZH_ROWS>& T = H.tab[id / half];
            const F9 y = spec_bind(ld9(T, i), ld9(T, i + half), v);
            if (mine < nt * half) st9(T, i, y);
        }
        n = half;
        if (n == 2) break;
    }
    __syncthreads();
    if (tid == 0) help_report(help);      // the last challenge is read
    if (x == 0 && tid < 2 * nt && !(e == 3 && tid >= 4)) {       // 1 - sign by the second equation
        const int k = tid >> 1;
        f9tab_st(a.tab[lin_table(e, k)], tid & 1, ld9(H.tab[k], tid & 1));
    }
}

// one wave: the sums over `count` slots of the values 4 x + row of round t
__device__ __forceinline__ F9 zh_collect(const ZkHelpMail* mail, int t, int x, int count, HelpWait& w) {
    constexpr int N = ZK_HELP_SLOTS / 16;
    const int lane = threadIdx.x & 63, row = lane >> 4, first = lane & 15;
    const bool mine = t > 0 || row == 0;
    F9 s;
    for (;;) {
        uint32_t bad = 0;
        s = f9_zero();
#pragma unroll
        for (int q = 0; q < N; ++q) {
            if (16 * q >= count) break;
            const bool read = mine && first + 16 * q < count;
            const uint64_t* at = (const uint64_t*)mail->coef[t & 1][4 * x + row][first + 16 * q];
            uint64_t e[HELP_WORDS / 2];
#pragma unroll
            for (int l = 0; l < HELP_WORDS / 2; ++l) e[l] = __hip_atomic_load(at + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int l = 0; l < 9; ++l) {
                const uint32_t word = (uint32_t)(e[l >> 1] >> (32 * (l & 1)));
                bad |= read ? (word ^ help_tag(t)) >> 29 : 0u;
                s.v[l] += read ? word & frc::M29 : 0u;
            }
        }
        if (__ballot(bad != 0) == 0 || w.late || !w.again()) break;
    }
    return wave_sum_lazy(f9_norm(s), 16);       // at most 80 values below 1.1 r
}

// The leader without helpers: every round on the tables in device memory, folded in place
__device__ __forceinline__ void zh_alone(const ZkShortJob& a, DevState* st, ZhLeader& L) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int slices = a.has_ga ? 2 : 1, total = slices * a.nbits, x = wave & 3;
    if (tid < 128) {
        const int k = tid >> 6;
        L.weight[k][lane] = lane < a.nbits && k < slices ? col_weight(a, k, lane) : f9_zero();
    }
    F9 v = fr_unpack(st->chal[a.chal - 1]);
    const F9 one9 = fr_unpack(fr_one());
    uint32_t m = (uint32_t)a.pairs;
    auto present = [&](int t) { return a.has_ga || t < 5 || t == 9; };
    for (int t = 0; t < a.rounds; ++t, m >>= 1) {
        __syncthreads();
        for (uint32_t id = tid; id < (uint32_t)(total + LIN) * 2 * m; id += ZH_THREADS) {
            const int c = (int)(id / (2 * m));
            const uint32_t i = id & (2 * m - 1);
            if (c >= total && !present(c - total)) continue;
            const F9Tab tab = c >= total ? a.tab[c - total] : col_table(a, c / a.nbits, c % a.nbits);
            f9tab_st(tab, i, spec_bind(f9tab_ld(tab, i), f9tab_ld(tab, i + 2 * m), v));
        }
        __syncthreads();
        for (uint32_t b = wave; b < m; b += ZH_THREADS / 64) {      // lanes: columns
            F9 s[3] = {f9_zero(), f9_zero(), f9_zero()};
            for (int k = 0; k < slices; ++k) {
                if (lane >= a.nbits) continue;
                const F9Tab tab = col_table(a, k, lane);
                const F9 lo = f9tab_ld(tab, b), hi = f9tab_ld(tab, b + m), w = L.weight[k][lane];
                s[0] = f9_norm_reduce(f9_add(s[0], f9_mul(w, f9_mul(lo, f9_sub(lo, one9)))));
                s[1] = f9_norm_reduce(f9_add(s[1], f9_mul(w, f9_mul(hi, f9_sub(hi, one9)))));
                s[2] = f9_norm_reduce(f9_add(s[2], f9_mul(w, f9_sqr(f9_norm(f9_sub(hi, lo))))));
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const F9 y = wave_sum_lazy(s[q]);
                if (lane == 0) L.part[q][b] = y;
            }
        }
        __syncthreads();
        F9 acc = f9_zero();
        for (uint32_t b = 64 * (wave >> 2) + lane; b < m; b += 256) {
            auto line = [&](int tab) { return line_at(x, f9tab_ld(a.tab[tab], b), f9tab_ld(a.tab[tab], b + m)); };
            for (int e = 0; e < 2 * slices; ++e) {
                F9 p = f9_mul(f9_norm(line(1 + 2 * e)), line(2 + 2 * e));
                if (e & 1) p = f9_mul(p, line(0));
                acc = f9_norm_reduce(f9_add(acc, p));
            }
            acc = f9_norm_reduce(f9_add(acc, f9_mul(quad_x(x, L.part[0][b], L.part[1][b], L.part[2][b]), line(9))));
        }
        acc = wave_sum_lazy(acc);
        if (lane == 0) L.sum[wave >> 2][x] = acc;
        __syncthreads();
        if (tid < 4) {
            const Fr plain = f9_canonical(f9_norm_reduce_sum(f9_add(f9_add(L.sum[0][tid], L.sum[1][tid]), f9_add(L.sum[2][tid], L.sum[3][tid]))));
#pragma unroll
            for (int l = 0; l < 8; ++l) L.g[tid][l] = plain.v[l];
        }
        __syncthreads();
        if (wave < 2) wave_frame_draw1_open(L.S, 'g', 3, [&](uint32_t i) -> uint32_t { return L.g[i < 8 ? 0 : (i >> 3) + 1][i & 7]; });
        else if (wave == 5 && lane < 32) ((uint32_t*)(st->proof + a.rounds_off + 128u * (uint32_t)t))[lane] = L.g[lane >> 3][lane & 7];
        __syncthreads();
        v = L.S.v9;
        if (tid == 320) store_challenge(st, a.chal + t, v);
    }
    __syncthreads();
    if (tid < 2 && a.beta_out.p != a.tab[9].p) f9tab_st(a.beta_out, tid, f9tab_ld(a.tab[9], tid));
}

__device__ __forceinline__ void zh_leader(const ZkShortJob& a, DevState* st, const ZkHelpLaunch& help, ZhLeader& L, uint32_t helpers, int slots) {
    ZkHelpMail* mail = help.mail;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int beside = spec_beside_index(wave);
    if (tid == 0) spec_init(L.X);
    block_ts_load(L.S, st, true);
    if (wave == 0) help_gather(help, helpers, &L.alone);
    __syncthreads();
    if (L.alone) {
        zh_alone(a, st, L);
        block_ts_store(L.S, st);
        return;
    }
    HelpWait w;
    w.begin(help.wait);
    if (beside < 4) {
        const F9 s = zh_collect(mail, 0, beside, slots, w);
        if (lane == 0) {
            const Fr plain = f9_canonical(s);
#pragma unroll
            for (int l = 0; l < 8; ++l) L.g[beside][l] = plain.v[l];
        }
    }
    __syncthreads();
    if (wave < 2) wave_frame_draw1_open(L.S, 'g', 3, [&](uint32_t i) -> uint32_t { return L.g[i < 8 ? 0 : (i >> 3) + 1][i & 7]; });
    else if (beside < 4) spec_coefficients<3>(L.X, beside, 0, zh_collect(mail, 1, beside, slots, w));
    else if (wave == 5 && lane < 32) ((uint32_t*)(st->proof + a.rounds_off))[lane] = L.g[lane >> 3][lane & 7];
    __syncthreads();
    F9 v = L.S.v9;
    const int left = a.rounds - 1;
    if (wave == 0) {
        spec_chain<3>(L.S, L.X, v, left);
    } else if (wave == 1) {
        spec_second<3>(L.S, L.X, st, left, a.rounds_off + 128, a.chal + 1, v, true);
    } else if (beside < 4) {
        for (int s = 0; s < left; ++s) {          // v_s is there; rounds s + 2 and later follow from it
            if (s > 0) {
                spec_wait(&L.X.v_done, (uint32_t)s);
                v = L.X.v9[(s - 1) & 1];
            }
            if (beside == 0) help_publish(mail, s, v);
            if (s + 1 < left) spec_coefficients<3>(L.X, beside, s + 1, zh_collect(mail, s + 2, beside, slots, w));
        }
        // beside the last round's hashes: that every helper has read its last challenge
        if (beside == 0)
            while (help_ld(&mail->started[help.epoch & 1]) != 2 * helpers && w.again()) __builtin_amdgcn_s_sleep(4);
    }
    help_end(mail, st, w.late, &L.alone, ZH_THREADS);
    block_ts_store(L.S, st);
}

union ZhLds {
    ZhLeader leader;
    ZhColumns columns;
    ZhLinear linear;
};
__global__ __launch_bounds__(ZH_THREADS) void k_zk_helped(ZkShortJob a, DevState* st, ZkHelpLaunch help, int columns) {
    __shared__ __align__(16) unsigned char lds[sizeof(ZhLds)];
    const int b = (int)blockIdx.x, eqs = a.has_ga ? 4 : 2;
    if (b == 0) {
        zh_leader(a, st, help, *(ZhLeader*)lds, (uint32_t)(columns + 4 * eqs), columns + eqs);
        return;
    }
    if (threadIdx.x == 0) {
        help_report(help);
        ((ZhMessage*)lds)->stop = 0;
    }
    const int e = b - 1 - columns;
    if (e < 0) zh_columns(a, st, help, *(ZhColumns*)lds, b - 1);
    else zh_linear(a, st, help, *(ZhLinear*)lds, e >> 2, e & 3, columns + (e >> 2));
}

}  // namespace

int zk_short_pairs(const zkdl_ctx* ctx) { return zk_help_mode(ctx) == ZKDL_HELPERS_OFF ? ZK_SHORT_PAIRS : ZK_ZHELP_PAIRS; }

// rounds from which on helpers take part (three: 472 us of a call, 485 without)
constexpr int ZHELP_MIN_ROUNDS = 3;
static_assert(1 << (ZHELP_MIN_ROUNDS - 2) <= ZK_SHORT_PAIRS && ZHELP_MIN_ROUNDS >= 2, "fewer rounds fit k_zk_short");

bool zk_helped_rounds(zkdl_ctx* ctx, const ZkShortJob& job) {
    if (zk_help_mode(ctx) == ZKDL_HELPERS_OFF || job.rounds < ZHELP_MIN_ROUNDS) return false;
    const int slices = job.has_ga ? 2 : 1, columns = (slices * job.nbits + 1) / 2, helpers = columns + 8 * slices;
    hipLaunchKernelGGL(k_zk_helped, dim3(1 + helpers), dim3(ZH_THREADS), 0, ctx->stream, job,
                       ctx->dev, zk_help_launch(ctx, 2ull * job.pairs * (slices * job.nbits + LIN)), columns);
    return true;
}
