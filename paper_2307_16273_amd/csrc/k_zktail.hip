// The end of zkReLU's combined sumcheck in one block: the tables over i at the full i-point, the log2 J rounds over j, the
// finals, and the merge of the three claims on aux.
//
// With every i bound, the summand over j is
//   a0 [L0 + B0 (a0 - 1)] + a1 [L1 + B1 (a1 - 1)],
//   L0 = r^2 beta_Z(v) s + r beta_A(v)(1-sign(v)) s',   B0 = beta_I(v) beta_J,
//   L1, B1 the same for slice 1 (with r'), a_k = aux~(k, v, j):
// six tables of J entries.  Bound by the hashes of 2 log2 J + 1 rounds one after the other.  The first round of either
// sumcheck is taken at once, point x = 0, 1, .. by wave x; the others have their coefficients in the challenge before
// them taken beside the hashes (spec_rounds.cuh), and so has the product of beta~(wbar, .) for the merge.  J = 64, kernel
// traces of the benchmark: 211 us on average (172 at least) with fold, sums and barriers between the hashes, 154 (131) like this.
#include "dev_common.cuh"
#include "spec_rounds.cuh"

namespace {

constexpr int TAIL_THREADS = 512, LIN_TABLES = 10;
static_assert(TAIL_THREADS >= SPEC_MIN_THREADS, "the waves beside the hashes");
enum { T_NS = 0, T_BZ, T_Z, T_BA, T_ZP, T_BGA, T_GA, T_BGZ, T_GAP, T_BI };

template <int N, int ENTRIES>
struct LdsTables {
    uint32_t el[N][9][ENTRIES];

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
    // value at x = 0 .. 3 of the line through entries i, i + half: normal, below 15.3 r
    __device__ __forceinline__ F9 line(int k, uint32_t i, uint32_t half, int x) const {
        const F9 hi = ld(k, x == 0 ? i : i + half);
        if (x < 2) return hi;
        const F9 d = f9_norm(f9_sub(hi, ld(k, i)));
        F9 e = f9_add(hi, d);
        if (x == 3) e = f9_add(e, d);
        return f9_norm(e);
    }
};
typedef LdsTables<6, 64> JTables;         // a0, a1, L0, L1, B0, B1 over j
typedef LdsTables<2, 128> MergeTables;    // aux, weights over (slice, j)

// The coefficients of point x of a j-round of q pairs.  A row's lanes take (pair, slice); the polynomial's value at infinity in the
// challenge is its cubic term, a a B.
__device__ __forceinline__ void j_coefficients(JTables& T, SpecShared<3>& X, int x, int round, uint32_t q) {
    const int lane = threadIdx.x & 63, row = lane >> 4;
    int c[4];
    spec_line<3>(row, x, c);
    const F9 one9 = fr_unpack(fr_one());
    F9 acc = f9_zero();
    for (uint32_t i = lane & 15; i < 2 * q; i += 16) {        // at most two sums of values below 1.3 r
        const uint32_t b = i >> 1;
        const int k = i & 1;
        F9 e[3];
#pragma unroll 1
        for (int w = 0; w < 3; ++w) {
            const int t = 2 * w + k;
            e[w] = f9_combine4(c, T.ld(t, b), T.ld(t, b + q), T.ld(t, b + 2 * q), T.ld(t, b + 3 * q));
        }
        F9 am = f9_sub(e[0], one9), l = e[1];
        if (row == 3) {
            am = e[0];
            l = f9_zero();
        }
        acc = f9_add(acc, f9_mul(e[0], f9_add(l, f9_mul(e[2], am))));
    }
    spec_coefficients<3>(X, x, round, wave_sum_lazy(f9_norm(acc), 16));
}

__global__ __launch_bounds__(TAIL_THREADS) void k_zk_tail(ZkTailJob a, DevState* st) {
    __shared__ TsShared TS;
    __shared__ SpecShared<3> X;
    __shared__ SpecShared<2> XM;
    __shared__ JTables T;
    __shared__ MergeTables M;
    __shared__ Fr S[64], SP[64];
    __shared__ F9 E[64];                                   // beta~(wbar, .) over j
    __shared__ Fr sc[LIN_TABLES];
    __shared__ Fr fin[3];
    __shared__ Fr rho[3];
    __shared__ uint32_t g[4][8];                           // a round's evaluations, canonical
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int beside = wave & 2 ? ((wave >> 2) << 1) | (wave & 1) : 4;    // waves 2, 3, 6, 7: 0 .. 3
    if (tid == 0) {
        spec_init<3>(X);
        spec_init<2>(XM);
    }
    block_ts_load(TS, st);
    const int J = 1 << a.lj, nbits = a.q_bits + a.r_bits;
    const Fr one = fr_one();
    Fr vlast = fr_zero();
    if (a.li >= 1) vlast = st->chal[a.chal_v + a.li - 1];

    // scalars: the tables over i at the full i-point
    if (tid < LIN_TABLES) {
        bool present = a.has_ga || !(tid == T_BGA || tid == T_GA || tid == T_BGZ || tid == T_GAP);
        Fr lo = fr_zero();
        if (present) {
            lo = f9_to_fr(f9tab_ld(a.tab[tid], 0));
            if (a.li >= 1) {
                Fr hi = f9_to_fr(f9tab_ld(a.tab[tid], 1));
                lo = fr_add(lo, fr_mul_ni(vlast, fr_sub(hi, lo)));
            }
        }
        sc[tid] = lo;
    } else if (tid >= 64 && tid < 192) {
        // aux~(k, v, j) for k = wave - 1
        const int j = lane, k = wave - 1;
        Fr val = fr_zero();
        if (j < nbits && (k == 0 || a.has_ga)) {
            const int64_t* src = k == 0 ? a.z : a.ga;
            if (a.li <= 1) {
                // the bits of one integer, or with one challenge the line through those of two
                if (((uint64_t)src[0] >> j) & 1) val = fr_sub(one, vlast);
                if (a.li == 1 && (((uint64_t)src[1] >> j) & 1)) val = fr_add(val, vlast);
            } else {
                // the columns were written with mat_bound challenges bound; later rounds
                // folded them down to two rows
                F9Tab col;
                col.p = a.aux + (uint64_t)(k * nbits + j) * 9 * a.ps;
                col.ps = a.ps;
                val = f9_to_fr(f9tab_ld(col, 0));
                if (a.li > a.mat_bound) {
                    Fr hi = f9_to_fr(f9tab_ld(col, 1));
                    val = fr_add(val, fr_mul_ni(vlast, fr_sub(hi, val)));
                }
            }
        }
        const F9 val9 = fr_unpack(val);
        T.st(k, j, val9);
        if (j < J) M.st(0, J * k + j, val9);
    } else if (tid >= 192 && tid < 256) {
        // s_{Q+R}(j) and s'(j) (Sec. 3.1, App. A)
        const int j = lane;
        Fr s = fr_zero(), sp = fr_zero();
        if (j < nbits) {
            if (j < nbits - 1) s = fr_from_i64((int64_t)1 << j);
            else s = fr_from_i64(j == 63 ? INT64_MIN : -((int64_t)1 << j));
            if (j == a.r_bits - 1) sp = one;
            else if (j >= a.r_bits && j < nbits - 1) sp = fr_from_i64((int64_t)1 << (j - a.r_bits));
            else if (j == nbits - 1) sp = fr_from_i64(-((int64_t)1 << (a.q_bits - 1)));
        }
        S[j] = s;
        SP[j] = sp;
    }
    __syncthreads();
    if (wave < 4) {
        // L0, L1, B0, B1: one table per wave
        const int j = lane;
        const Fr ns = sc[T_NS];
        Fr val = fr_zero();
        if (j < J) {
            if (wave == 0) val = fr_add(fr_mul_ni(sc[T_BZ], S[j]), fr_mul_ni(fr_mul_ni(sc[T_BA], ns), SP[j]));
            else if (wave == 1) val = fr_add(fr_mul_ni(sc[T_BGA], S[j]), fr_mul_ni(fr_mul_ni(sc[T_BGZ], ns), SP[j]));
            else if (wave == 2) val = fr_mul_ni(sc[T_BI], a.bJ[j]);
            else val = fr_mul_ni(fr_mul_ni(st->weights[4], sc[T_BI]), a.bJ[j]);
        }
        T.st(2 + wave, j, fr_unpack(val));
    }
    __syncthreads();
    const F9 one9 = fr_unpack(one);

    // ---- rounds over j ----
    F9 v, e = one9;
    // e: lane's entry of beta~(wbar, .), a factor with every challenge (by one wave)
    auto bind_weight = [&](const F9& u, int var) {
        e = f9_mul(e, (lane >> (a.lj - 1 - var)) & 1 ? u : f9_norm_reduce(f9_sub(one9, u)));
    };
    {
        const int half = J >> 1, left = a.lj - 1;
        const uint32_t proof_off = a.rounds_off + (uint32_t)a.li * 128;
        if (wave < 4) {
            // wave: point x = 0 .. 3; lane = 2 j + slice, j < half <= 32: the first 2 half lanes are busy
            const int k = lane & 1, j = lane >> 1;
            F9 f = f9_zero();
            if (j < half) {
                const F9 av = T.line(k, j, half, wave), lv = T.line(2 + k, j, half, wave), bv = T.line(4 + k, j, half, wave);
                // (a - 1 + 4r) below 20 r, times b: below 5.4 r; plus l: below 21 r, times a: below 5.6 r
                f = f9_norm_reduce(f9_mul(av, f9_add(lv, f9_mul(bv, f9_sub(av, one9)))));
            }
            const F9 s = wave_sum_lazy(f, 2 * half);
            if (lane == 0) {
                const Fr plain = f9_canonical(s);
#pragma unroll
                for (int l = 0; l < 8; ++l) g[wave][l] = plain.v[l];
            }
        }
        __syncthreads();
        // the transcript takes g(0), g(2), g(3)
        if (wave < 2) wave_frame_draw1_open(TS, 'g', 3, [&](uint32_t i) -> uint32_t { return g[i < 8 ? 0 : (i >> 3) + 1][i & 7]; });
        else if (beside < 4 && left > 0) j_coefficients(T, X, beside, 0, half >> 1);
        else if (wave == 5 && lane < 32) ((uint32_t*)(st->proof + proof_off))[lane] = g[lane >> 3][lane & 7];
        __syncthreads();
        v = TS.v9;
        if (left > 0) {
            if (wave == 0) {
                spec_chain<3>(TS, X, v, left);
            } else if (wave == 1) {
                spec_second<3>(TS, X, st, left, proof_off + 128, a.chal_v + a.li + 1, v, true);
            } else if (beside < 4) {
                int var = 0;
                spec_beside<3>(T, 6, X, beside, v, left, (uint32_t)half >> 1,
                               [&](int round, uint32_t q) { j_coefficients(T, X, beside, round, q); },
                               [&](const F9& u) {
                                   if (beside == 3) bind_weight(u, var++);
                               });
            }
            __syncthreads();
            v = X.v9[(left - 1) & 1];
        } else if (tid == 320) {
            store_challenge(st, a.chal_v + a.li, v);
        }
    }
    if (beside == 3) {
        bind_weight(v, a.lj - 1);
        E[lane] = e;                 // normal, below 1.1 r
    }
    // finals: aux~(0, v, wbar), aux~(1, v, wbar), aux~(0, v, Q+R-1) = 1 - (1 - sign)(v)
    if (tid < 3) {
        Fr x = fr_sub(one, sc[T_NS]);
        if (tid < 2) {
            const F9 lo = T.ld(tid, 0);
            x = f9_to_fr(f9_add(lo, f9_mul(f9_sub(T.ld(tid, 1), lo), v)));
        }
        fin[tid] = x;
        st->scal[4 + tid] = x;
    }
    __syncthreads();
    block_absorb_frs(TS, 'f', fin, 3, (uint32_t*)(st->proof + a.finals_off));
    block_challenges(TS, st, a.chal_rho, 3);   // rho0..2: one vector draw
    if (tid < 3) rho[tid] = st->chal[a.chal_rho + tid];
    __syncthreads();
    if (tid >= 256 && tid < 320) {             // the claim, its three products side by side
        F9 x = f9_zero();
        if (lane < 3) x = f9_mul(fr_unpack(rho[lane]), fr_unpack(fin[lane]));
        const F9 s = wave_sum_lazy(x, 4);
        if (lane == 0) {
            const Fr mc = f9_to_fr(s);
            st->claim = mc;
            const Fr plain = fr_from_mont_ni(mc);
            uint32_t* dst = (uint32_t*)(st->proof + a.merge_claim_off);
            for (int l = 0; l < 8; ++l) dst[l] = plain.v[l];
        }
    }
    // E(0, j) = rho0 beta(wbar, j) + rho2 [j == Q+R-1],  E(1, j) = rho1 beta(wbar, j): tables over (k, j) of
    // 2 J entries
    if (tid < 2 * J) {
        const int k = tid >= J, j = tid - k * J;
        F9 w = f9_mul(fr_unpack(rho[k]), E[j]);
        if (k == 0 && j == nbits - 1) w = f9_norm(f9_add(w, fr_unpack(rho[2])));
        M.st(1, tid, w);                       // below 2.1 r
    }
    __syncthreads();

    // ---- merge sumcheck over (k, j): k first, then the variables of j ----
    {
        const int half = J, left = a.lj;
        if (wave < 3) {
            // wave: point x; lane = index below half (half <= 64)
            F9 f = f9_zero();
            if (lane < half) f = f9_norm_reduce(f9_mul(M.line(0, lane, half, wave), M.line(1, lane, half, wave)));
            const F9 s = wave_sum_lazy(f, half);
            if (lane == 0) {
                const Fr plain = f9_canonical(s);
#pragma unroll
                for (int l = 0; l < 8; ++l) g[wave][l] = plain.v[l];
            }
        }
        __syncthreads();
        // the transcript takes g(0), g(2)
        if (wave < 2) wave_frame_draw1_open(TS, 'g', 2, [&](uint32_t i) -> uint32_t { return g[i < 8 ? 0 : 2][i & 7]; });
        else if (beside < 3) spec_product_coefficients<2>(M, XM, beside, 0, (uint32_t)half >> 1);
        else if (wave == 5 && lane < 24) ((uint32_t*)(st->proof + a.merge_rounds_off))[lane] = g[lane >> 3][lane & 7];
        __syncthreads();
        v = TS.v9;
        if (wave == 0)
            spec_chain<2>(TS, XM, v, left);
        else if (wave == 1)
            spec_second<2>(TS, XM, st, left, a.merge_rounds_off + 96, a.chal_rho + 4, v, true);
        else if (beside < 3)
            spec_beside<2>(M, 2, XM, beside, v, left, (uint32_t)half >> 1,
                           [&](int round, uint32_t q) { spec_product_coefficients<2>(M, XM, beside, round, q); }, [](const F9&) {});
        __syncthreads();
        v = XM.v9[(left - 1) & 1];
    }
    if (tid < 2) {
        const F9 lo = M.ld(tid, 0);
        const Fr x = f9_to_fr(f9_add(lo, f9_mul(f9_sub(M.ld(tid, 1), lo), v)));
        fin[tid] = x;
        st->scal[7 + tid] = x;
    }
    __syncthreads();
    block_absorb_frs(TS, 'f', fin, 2, (uint32_t*)(st->proof + a.merge_finals_off));
    block_ts_store(TS, st);
}

}  // namespace

void zk_tail(zkdl_ctx* ctx, const ZkTailJob& job) {
    hipLaunchKernelGGL(k_zk_tail, dim3(1), dim3(TAIL_THREADS), 0, ctx->stream, job, ctx->dev);
}
