// The last i-rounds of zkReLU, of at most ZK_SHORT_PAIRS pairs of rows, in one block with every table in LDS.
//
// With helper blocks (k_zkhelp.hip) only calls with one or two i-rounds left come here; without them the last four.
// Round by round they are two launches each, nearly all of it latency: 19 us for the round's kernel, which takes one column
// per block to have anything to run side by side, and 13 for the one that adds its partial sums up, hashes and draws.
// Here a round is a fold, two barriers and the hashes.  The columns of Z and G_A take 72 KB of LDS in 16 rows, which
// sets the line at 8 pairs: with 32 rows they would fill it.
// Four rounds of 48 columns in a kernel trace: 62 us with one slice (a 256 x 256 layer), 79 to 94 with two (a step of 8 x 1024);
// the rounds before them, of the same work as two launches each, take 30 us apiece there.
#include "spec_rounds.cuh"

namespace {

constexpr int SHORT_THREADS = 1024, ROWS = 2 * ZK_SHORT_PAIRS;
constexpr int ROW_WORDS = 9 * 64 + 8;     // limb-major over 64 columns; rows begin eight banks apart (see the fill)
constexpr int LIN = 10;                   // tables: (1 - sign) | beta_Z Z | beta_A Z' | beta_GA G_A | beta_GZ G_A' | beta_I

struct ShortLds {
    uint32_t col[2][ROWS][ROW_WORDS];
    uint32_t lin[LIN][9][ROWS];
    F9 weight[2][64];                     // beta_J, r' beta_J
    F9 part[3][2][ZK_SHORT_PAIRS];        // column sums per slice: of p(lo), p(hi), (hi - lo)^2, p(e) = e^2 - e
    F9 sum[2][3][ZK_SHORT_PAIRS];         // [round & 1]: both slices

    __device__ __forceinline__ F9 column(int k, int row, int j) const {
        F9 x;
#pragma unroll
        for (int l = 0; l < 9; ++l) x.v[l] = col[k][row][64 * l + j];
        return x;
    }
    __device__ __forceinline__ void set_column(int k, int row, int j, const F9& x) {
#pragma unroll
        for (int l = 0; l < 9; ++l) col[k][row][64 * l + j] = x.v[l];
    }
    __device__ __forceinline__ F9 table(int t, int row) const {
        F9 x;
#pragma unroll
        for (int l = 0; l < 9; ++l) x.v[l] = lin[t][l][row];
        return x;
    }
    __device__ __forceinline__ void set_table(int t, int row, const F9& x) {
#pragma unroll
        for (int l = 0; l < 9; ++l) lin[t][l][row] = x.v[l];
    }
};

// small-integer combination of the column sums of one pair: normal, below 1.1 r (values below 2.42 r, |c| at most 11
// together: 30 r is added, so that the value lies between 2 r and 57 r)
__device__ __forceinline__ F9 combine3(int c0, int c1, int c2, const F9& a0, const F9& a1, const F9& a2) {
    int64_t acc[9];
#pragma unroll
    for (int l = 0; l < 9; ++l)
        acc[l] = 30ll * (int64_t)frc::MOD9[l] + (int64_t)c0 * (int32_t)a0.v[l] + (int64_t)c1 * (int32_t)a1.v[l] +
                 (int64_t)c2 * (int32_t)a2.v[l];
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

__global__ __launch_bounds__(SHORT_THREADS) void k_zk_short(ZkShortJob a, DevState* st) {
    __shared__ ShortLds S;
    __shared__ TsShared TS;
    __shared__ RoundShared R;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    block_ts_load(TS, st);
    round_begin(R, st, 4);
    const int slices = a.has_ga ? 2 : 1;
    const F9 one9 = fr_unpack(fr_one());
    F9 v = fr_unpack(st->chal[a.chal - 1]);
    int m = a.pairs;
    // Fill: both rows of every pair with the previous challenge bound.  Eight columns by eight pairs a wave: the pairs are
    // neighbours in memory, and the columns' rows lie eight banks apart in LDS
    {
        const int c = 8 * wave + (lane >> 3), k = c >> 6, j = c & 63, b = lane & 7;
        if (k < slices && j < a.nbits && b < m) {
            F9Tab t;
            t.p = a.aux + (uint64_t)(k * a.nbits + j) * 9 * a.ps;
            t.ps = a.ps;
            const F9 t0 = f9tab_ld(t, b), t1 = f9tab_ld(t, b + m), t2 = f9tab_ld(t, b + 2 * m), t3 = f9tab_ld(t, b + 3 * m);
            S.set_column(k, b, j, spec_bind(t0, t2, v));
            S.set_column(k, b + m, j, spec_bind(t1, t3, v));
        }
    }
    const int ti = tid >> 3, tb = tid & 7;                 // tables of the linear equations: threads 0 .. 79
    const bool present = ti < LIN && (a.has_ga || ti < 5 || ti == 9);
    if (present && tb < m) {
        const F9Tab t = a.tab[ti];
        const F9 t0 = f9tab_ld(t, tb), t1 = f9tab_ld(t, tb + m), t2 = f9tab_ld(t, tb + 2 * m), t3 = f9tab_ld(t, tb + 3 * m);
        S.set_table(ti, tb, spec_bind(t0, t2, v));
        S.set_table(ti, tb + m, spec_bind(t1, t3, v));
    } else if (tid >= 128 && tid < 256) {
        const int j = tid & 63, k = (tid >> 6) & 1;
        F9 x = f9_zero();
        if (j < a.nbits) x = fr_unpack(k == 0 ? a.bJ[j] : fr_mul(*a.rp, a.bJ[j]));
        S.weight[k][j] = x;
    }
    __syncthreads();
    for (int t = 0; t < a.rounds; ++t, m >>= 1) {
        // column sums: a wave has a pair and a slice, its lanes the columns
        for (int task = wave; task < slices * m; task += SHORT_THREADS / 64) {
            const int k = task >= m ? 1 : 0, b = task - k * m;
            F9 w = f9_zero(), sq = f9_zero(), lo = f9_zero(), hi = f9_zero();
            const bool live = lane < a.nbits;
            if (live) {
                w = S.weight[k][lane];
                if (t == 0) {
                    lo = S.column(k, b, lane);
                    hi = S.column(k, b + m, lane);
                } else {
                    lo = spec_bind(S.column(k, b, lane), S.column(k, b + 2 * m, lane), v);
                    hi = spec_bind(S.column(k, b + m, lane), S.column(k, b + 3 * m, lane), v);
                    S.set_column(k, b, lane, lo);
                    S.set_column(k, b + m, lane, hi);
                }
                sq = f9_mul(w, f9_sqr(f9_norm(f9_sub(hi, lo))));
            }
            const F9 sd = wave_sum_lazy(sq);
            if (lane == 0) S.part[2][k][b] = sd;
            if (t == 0) {      // later rounds bind these sums
                F9 x = f9_zero(), y = f9_zero();
                if (live) {
                    x = f9_mul(w, f9_mul(lo, f9_sub(lo, one9)));
                    y = f9_mul(w, f9_mul(hi, f9_sub(hi, one9)));
                }
                x = wave_sum_lazy(x);
                y = wave_sum_lazy(y);
                if (lane == 0) {
                    S.part[0][k][b] = x;
                    S.part[1][k][b] = y;
                }
            }
        }
        if (t > 0) {
            // the other tables, on waves that have no columns after the first round
            const int id = tid - (SHORT_THREADS - 128), i = id >> 3, b = id & 7;
            if (id >= 0 && i < LIN && (a.has_ga || i < 5 || i == 9) && b < m) {
                const F9 lo = spec_bind(S.table(i, b), S.table(i, b + 2 * m), v), hi = spec_bind(S.table(i, b + m), S.table(i, b + 3 * m), v);
                S.set_table(i, b, lo);
                S.set_table(i, b + m, hi);
            }
            // (1 - v) SA + v SC - v (1 - v) SD of the 2 m pairs of the round before
            const int p = tid - (SHORT_THREADS - 192);
            if (p >= 0 && p < 2 * m) {
                const F9 (&in)[3][ZK_SHORT_PAIRS] = S.sum[(t - 1) & 1];
                const F9 vv = f9_mul(v, f9_sub(v, one9));       // v normal, below 2.1 r
                S.sum[t & 1][p >= m ? 1 : 0][p & (m - 1)] =
                    f9_norm_reduce(f9_add(f9_add(in[0][p], f9_mul(f9_sub(in[1][p], in[0][p]), v)), f9_mul(in[2][p], vv)));
            }
        }
        __syncthreads();
        uint32_t* proof_dst = (uint32_t*)(st->proof + a.rounds_off + 128u * (uint32_t)t);
        if (wave < 4) {
            // wave: point x; lanes: pair, and the four equations and the binarity term
            const int term = lane >> 3, b = lane & 7, x = wave;
            auto line = [&](int tab) {      // limbs below 2^30.6
                const F9 lo = S.table(tab, b), hi = S.table(tab, b + m);
                if (x == 0) return lo;
                if (x == 1) return hi;
                const F9 d = f9_norm(f9_sub(hi, lo));
                F9 e = f9_add(hi, d);
                if (x == 3) e = f9_add(e, d);
                return e;
            };
            F9 prod = f9_zero();
            if (b < m && term < (a.has_ga ? 4 : 2)) {
                prod = f9_norm(line(1 + 2 * term));
                if (term & 1) prod = f9_mul(prod, line(0));
                prod = f9_norm_reduce(f9_mul(prod, line(2 + 2 * term)));
            } else if (b < m && term == 4) {
                F9 s[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    if (q < 2 && t > 0) {
                        s[q] = S.sum[t & 1][q][b];
                    } else {
                        s[q] = S.part[q][0][b];
                        if (slices == 2) s[q] = f9_norm(f9_add(s[q], S.part[q][1][b]));     // below 2.2 r
                        if (x == 0) S.sum[t & 1][q][b] = s[q];
                    }
                }
                // SA, SC, -SA + 2 SC + 2 SD, -2 SA + 3 SC + 6 SD
                const F9 g = combine3(x == 0 ? 1 : x == 1 ? 0 : 1 - x, x, x * (x - 1), s[0], s[1], s[2]);
                prod = f9_norm_reduce(f9_mul(g, line(9)));
            }
            const F9 s = wave_sum_lazy(prod);
            if (lane == 0) round_eval_out(TS, R, proof_dst, x, s, true);
        }
        v = block_close_round(TS, R, st, 4, false, a.rounds_off + 128u * (uint32_t)t, a.chal + t);
    }
    round_end(R, st, 4, a.chal + a.rounds - 1);
    // the last pair of everything, not yet bound
    {
        const int k = wave & 1, row = (wave >> 1) & 1;
        if (wave < 4 && k < slices && lane < a.nbits) {
            F9Tab t;
            t.p = a.aux + (uint64_t)(k * a.nbits + lane) * 9 * a.ps;
            t.ps = a.ps;
            f9tab_st(t, row, S.column(k, row, lane));
        }
        const int id = tid - 256, i = id >> 1;
        if (id >= 0 && i < LIN && (a.has_ga || i < 5 || i == 9)) f9tab_st(i == 9 ? a.beta_out : a.tab[i], id & 1, S.table(i, id & 1));
    }
    block_ts_store(TS, st);
}

}  // namespace

int zk_short_rounds(zkdl_ctx* ctx, const ZkShortJob& job) {
    if (zk_helped_rounds(ctx, job)) return ZKDL_OK;
    hipLaunchKernelGGL(k_zk_short, dim3(1), dim3(SHORT_THREADS), 0, ctx->stream, job, ctx->dev);
    return ZKDL_OK;
}
