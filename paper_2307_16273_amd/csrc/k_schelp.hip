// The last rounds of a product sumcheck in one launch: a block that closes the rounds and helper blocks that hold the tables.
//
// Up to 2^15 entries a table is too long for one block's arithmetic and too short for a launch per round: two dependent launches
// take 25 to 35 us whatever they do, while the transcript step of a round takes 6.  Here 16 to 64 helper blocks keep a
// slice of every table each in their LDS, from the first round to the one at which 2^7 entries are left, and what they send is
// the sums of a round AHEAD of its challenge: the coefficients of g_t(x) as polynomials in v_{t-1} (spec_rounds.cuh).  The
// block that hashes therefore waits only for what a trip to the helpers and back takes longer than a round of its own; a trip, the fold and the next
// sums run beside the hashes of a round.  The last seven rounds' tables move to the hashing block.  Bound by the hashes there: 15 thousand
// cycles a round, of which the two compressions are 11 and the products before them 4; a trip to the helpers and back, with its fold and
// sums, takes 12 with tables of 2^12 entries, 17 with two and 25 with three of 2^15 (through memory and back 4 to 10 of it), so that such a
// round takes 15 to 18, 16 to 20 and 21 to 27.
// Whole sumcheck_product calls (us, launches per round and one block for the last ten / like this): two tables 2^9 112 / 109,
// 2^10 130 / 116, 2^12 181 / 130, 2^14 214 / 154, 2^15 234 / 165, three 2^9 124 / 116, 2^10 147 / 124, 2^12 206 / 142, 2^14 261 / 169,
// 2^15 288 / 190.
//
// Messages and progress: help.cuh.
#include "help.cuh"
#include "sc_tail.cuh"

constexpr int HELP_LEFT_LOG = 7;                  // entries (log2) at which the tables move to the leader
constexpr int HELP_MIN_LOG_W = 4, HELP_MAX_LOG_W = 6;     // helpers (log2)
static_assert(ZK_HELP_BLOCKS == 1 << HELP_MAX_LOG_W && HELP_MAX_LOG_W < HELP_LEFT_LOG, "owners by bits that no helper binds");
static_assert(ZK_HELP_MAX_LOG - HELP_MAX_LOG_W <= SC_TAIL_LOG, "a slice fits the LDS tables");
static_assert(2u << HELP_LEFT_LOG <= 4 * 2 * SPEC_MAX_PAIRS, "after them the leader's rounds are short ones");

// Entry j of helper h among 2^lw: the owner stands in the bits below 2^6 (no round before the tables move binds or pairs by them) and
// as high as that allows, so that the words of a plane that a helper reads come in runs of 2^(6 - lw).
__device__ __forceinline__ uint32_t help_global(uint32_t h, uint32_t j, int lw) {
    const int s = HELP_LEFT_LOG - 1 - lw;
    return ((j >> s) << (HELP_LEFT_LOG - 1)) | (h << s) | (j & ((1u << s) - 1));
}

template <int K>
struct HelpShared {
    ScTailLds<K> T;
    F9 sum[4][4][4];       // [part][x][row]
    F9 v;
    uint32_t stop;
};

// sums of the parts -> the message of round t (values 4 x + row)
template <int K>
__device__ __forceinline__ void help_send(HelpShared<K>& H, ZkHelpMail* mail, int h, int t, int parts) {
    const int tid = threadIdx.x;
    __syncthreads();
    if (tid < 16 && !H.stop) {
        const int x = tid >> 2, row = tid & 3;
        F9 s = H.sum[0][x][row];
        for (int p = 1; p < parts; ++p) s = f9_add(s, H.sum[p][x][row]);
        s = f9_norm_reduce(s);                           // below 2.41 r
        if (x <= K && (t == 0 ? row == 0 : row <= K)) help_write(mail->coef[t & 1][tid][h], help_tag(t), s);
    }
}

template <int K>
__device__ __forceinline__ void help_block(const ScTailArgs& a, const ZkHelpLaunch& help, HelpShared<K>& H, int h, int lw) {
    ZkHelpMail* mail = help.mail;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, x = wave & 3, part = wave >> 2;
    if (tid == 0) {
        help_report(help);
        H.stop = 0;
    }
    const uint32_t m = (uint32_t)a.ra.m;
    const uint32_t keep = 1u << (HELP_LEFT_LOG - lw);    // entries of a table that go to the leader in the end
    uint32_t n = (2 * m) >> lw;                          // entries of a table here
    F9 v = f9_zero();
    if (a.source == SC_SRC_PACKED_FOLD || a.source == SC_SRC_WORK) v = fr_unpack(a.st->chal[a.first_chal]);
    for (uint32_t id = tid; id < K * n; id += SC_TAIL_THREADS) {
        const int k = (int)(id / n);
        const uint32_t j = id & (n - 1);
        H.T.st(k, j, sc_tail_entry(a, k, help_global((uint32_t)h, j, lw), m, v));
    }
    __syncthreads();
    // round 0: plain evaluations
    {
        const uint32_t q = n >> 1;
        const int parts = q <= 64 ? 1 : q <= 128 ? 2 : 4;
        if (x <= K && part < parts) {
            F9 acc = f9_zero();
            for (uint32_t b = 64 * part + lane; b < q; b += 256) acc = f9_norm_reduce(f9_add(acc, sc_pair_value<K>(H.T, x, b, q)));
            const F9 s = wave_sum_lazy(acc, q < 64 ? (int)q : 64);
            if (lane == 0) H.sum[part][x][0] = s;
        }
        // all helpers, or none
        if (wave == 0 && !help_may_go(help) && lane == 0) H.stop = 1;
        help_send<K>(H, mail, h, 0, parts);              // (writes behind its barrier, if at all)
        if (H.stop) return;
    }
    for (int t = 1;; ++t) {
        // coefficients in v_{t-1} of round t, from the tables with v_{t-2} bound
        __syncthreads();
        const uint32_t q = n >> 2;
        const int parts = q <= 16 ? 1 : q <= 32 ? 2 : 4;
        if (x <= K && part < parts) {
            int c[4];
            spec_line<K>(lane >> 4, x, c);
            F9 acc = f9_zero();
            for (uint32_t b0 = 16 * part; b0 < q; b0 += 64) {
                const uint32_t mine = b0 + (lane & 15), b = mine < q ? mine : 0;
                F9 prod = f9_zero();
#pragma unroll 1
                for (int k = 0; k < K; ++k) {
                    const F9 e = f9_combine4(c, H.T.ld(k, b), H.T.ld(k, b + q), H.T.ld(k, b + 2 * q), H.T.ld(k, b + 3 * q));
                    prod = k == 0 ? e : f9_mul(prod, e);
                }
                if (mine >= q) prod = f9_zero();
                acc = f9_norm_reduce(f9_add(acc, prod));
            }
            const F9 s = wave_sum_lazy(acc, 16);         // per row
            if ((lane & 15) == 0) H.sum[part][x][lane >> 4] = s;
        }
        help_send<K>(H, mail, h, t, parts);
        // v_{t-1}
        if (wave == 0 && !help_challenge(help, t - 1, H.v) && lane == 0) H.stop = 1;
        __syncthreads();
        if (H.stop) return;
        v = H.v;
        for (uint32_t id = tid; id < K * (n >> 1); id += SC_TAIL_THREADS) {
            const int k = (int)(id / (n >> 1));
            const uint32_t j = id & ((n >> 1) - 1);
            const F9 t0 = H.T.ld(k, j);
            H.T.st(k, j, f9_norm_reduce(f9_add(t0, f9_mul(f9_sub(H.T.ld(k, j + (n >> 1)), t0), v))));
        }
        n >>= 1;
        if (n == keep) break;
    }
    // The last entries go to the leader.  (Written by the fold, under a condition on n, they cost more: the compiler makes
    // the loop's last turn a copy of its own, which runs from a cold instruction cache.)
    __syncthreads();
    if (tid < (int)(K * keep)) {
        const int k = tid >> (HELP_LEFT_LOG - lw);
        const uint32_t j = (uint32_t)tid & (keep - 1);
        help_write(mail->tab[k][help_global((uint32_t)h, j, lw)], help_tag(0), H.T.ld(k, j));
    }
}

// one wave: the sums over the helpers of the values 4 x + row of round t, in every lane of row `row`: below 1.1 r
template <int N>
__device__ __forceinline__ F9 help_collect_n(const uint32_t* p, int t, bool mine, HelpWait& w) {
    F9 e[N];
    help_read<N>(p, 16 * HELP_WORDS, help_tag(t), mine, e, w);
    F9 s = e[0];
#pragma unroll
    for (int q = 1; q < N; ++q) s = f9_add(s, e[q]);
    return s;
}
__device__ __forceinline__ F9 help_collect(const ZkHelpMail* mail, int t, int x, int deg, int lw, HelpWait& w) {
    const int lane = threadIdx.x & 63, row = lane >> 4;
    const bool mine = t == 0 ? row == 0 : row <= deg;
    const uint32_t* p = mail->coef[t & 1][4 * x + row][lane & 15];
    F9 s = lw == 4 ? help_collect_n<1>(p, t, mine, w) : lw == 5 ? help_collect_n<2>(p, t, mine, w) : help_collect_n<4>(p, t, mine, w);
    if (!mine) s = f9_zero();
    return wave_sum_lazy(f9_norm(s), 16);
}
static_assert(ZK_HELP_BLOCKS <= 64, "sums of 64 values below 2.41 r are below 160 r");

// long tables in device memory, for a leader that goes on alone
struct ScBig {
    static constexpr bool LONG = true;
    uint32_t* p;
    __device__ __forceinline__ F9 ld(int k, uint32_t i) const {
        F9 x;
#pragma unroll
        for (int l = 0; l < 9; ++l) x.v[l] = p[(((size_t)k * 9 + l) << ZK_HELP_MAX_LOG) + i];
        return x;
    }
    __device__ __forceinline__ void st(int k, uint32_t i, const F9& x) {
#pragma unroll
        for (int l = 0; l < 9; ++l) p[(((size_t)k * 9 + l) << ZK_HELP_MAX_LOG) + i] = x.v[l];
    }
};

template <int K>
__device__ __forceinline__ void help_leader(const ScTailArgs& a, const ZkHelpLaunch& help, ScTailShared<K>& L, uint32_t* alone, int lw) {
    constexpr int NPTS = K + 1;
    DevState* st = a.st;
    ZkHelpMail* mail = help.mail;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, beside = spec_beside_index(wave);
    if (tid == 0) spec_init(L.X);
    block_ts_load(L.S, st, true);
    if (wave == 0) help_gather(help, 1u << lw, alone);
    __syncthreads();
    if (*alone) {
        ScBig big = {mail->scratch};
        sc_tail_block<K>(a, L, big);
        return;
    }
    HelpWait w;
    w.begin(help.wait);
    // round 0
    if (beside < NPTS) {
        const F9 s = help_collect(mail, 0, beside, K, lw, w);
        if (lane == 0) {
            L.g9[beside] = s;
            const Fr plain = f9_canonical(s);
#pragma unroll
            for (int l = 0; l < 8; ++l) L.g[beside][l] = plain.v[l];
        }
    }
    __syncthreads();
    if (a.first) sc_tail_claim<K>(a, L);
    if (wave < 2) {
        wave_frame_draw1_open(L.S, 'g', K, [&](uint32_t i) -> uint32_t { return L.g[i < 8 ? 0 : (i >> 3) + 1][i & 7]; }, a.first == 1);
    } else if (beside < NPTS) {
        spec_coefficients<K>(L.X, beside, 0, help_collect(mail, 1, beside, K, lw, w));
    } else if (wave == 5) {
        uint32_t* dst = (uint32_t*)(st->proof + a.rounds_off);
        if (lane < 8 * NPTS) dst[lane] = L.g[lane >> 3][lane & 7];
    }
    __syncthreads();
    F9 v = L.S.v9;
    const int left = a.rounds - 1, moved = a.rounds - HELP_LEFT_LOG;     // the tables with `moved` challenges bound come here
    if (wave == 0) {
        spec_chain<K>(L.S, L.X, v, left);
    } else if (wave == 1) {
        spec_second<K>(L.S, L.X, st, left, a.rounds_off + (uint32_t)NPTS * 32, a.first_chal + 2, v, true);
    } else if (beside < NPTS) {
        // s: v_s is there; what follows from it
        for (int s = 0; s < moved; ++s) {
            if (s > 0) {
                spec_wait(&L.X.v_done, (uint32_t)s);
                v = L.X.v9[(s - 1) & 1];
            }
            if (beside == 0) help_publish(mail, s, v);
            if (s + 1 < moved) {
                spec_coefficients<K>(L.X, beside, s + 1, help_collect(mail, s + 2, beside, K, lw, w));
            } else {
                constexpr uint32_t left_n = 1u << HELP_LEFT_LOG;
                for (uint32_t id = 64 * beside + lane; id < K * left_n; id += 64 * NPTS) {
                    F9 e[1];
                    help_read<1>(mail->tab[id >> HELP_LEFT_LOG][id & (left_n - 1)], 0, help_tag(0), true, e, w);
                    L.T.st((int)(id >> HELP_LEFT_LOG), id & (left_n - 1), e[0]);
                }
                spec_order();
                if (lane == 0) __hip_atomic_fetch_add(&L.X.folded, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                spec_wait(&L.X.folded, (uint32_t)NPTS);
                spec_product_coefficients<K>(L.T, L.X, beside, s + 1, left_n >> 2);
            }
        }
        spec_beside<K>(L.T, K, L.X, beside, v, left, 1u << (HELP_LEFT_LOG - 2),
                       [&](int round, uint32_t q) { spec_product_coefficients<K>(L.T, L.X, beside, round, q); }, [](const F9&) {}, moved);
    }
    help_end(mail, st, w.late, alone, SC_TAIL_THREADS);
    v = L.X.v9[(left - 1) & 1];
    sc_tail_finals<K>(a, L, v, -1);
}

template <int K>
union HelpLds {
    ScTailShared<K> leader;
    HelpShared<K> helper;
};
template <int K>
__global__ __launch_bounds__(SC_TAIL_THREADS) void k_sc_helped(ScTailArgs a, ZkHelpLaunch help, int lw) {
    __shared__ __align__(16) unsigned char lds[sizeof(HelpLds<K>)];
    __shared__ uint32_t alone;
    if (blockIdx.x == 0) help_leader<K>(a, help, *(ScTailShared<K>*)lds, &alone, lw);
    else help_block<K>(a, help, *(HelpShared<K>*)lds, (int)blockIdx.x - 1, lw);
}

// Helpers by the number of rounds: more of them share the arithmetic of the longest tables and make the leader's sums longer.  Whole calls (us, 16 / 32 /
// 64 helpers), three tables: 2^11 131 / 133 / 137, 2^13 158 / 156 / 156, 2^14 197 / 175 / 169, 2^15 - / 217 / 190; two: 2^12 129 / 131 / 135,
// 2^14 162 / 154 / 153, 2^15 187 / 179 / 166.
constexpr int HELP_64_ROUNDS = 14, HELP_32_ROUNDS = 13;

int zk_tail_log(const zkdl_ctx* ctx) { return zk_help_mode(ctx) == ZKDL_HELPERS_OFF ? SC_TAIL_LOG : ZK_HELP_MAX_LOG; }

ZkHelpLaunch zk_help_launch(zkdl_ctx* ctx, uint64_t entries) {
    // 31 bits; one launch after the other, neighbours differ in the lowest one
    ctx->help_epoch = ctx->help_epoch >= 0x7fffffffu ? 2 : ctx->help_epoch + 1;
    ctx->help_unread = true;
    ZkHelpLaunch help;
    help.mail = ctx->help;
    help.epoch = ctx->help_epoch;
    help.wait = ctx->help_wait;
    help.report = zk_help_report_ticks(entries);
    help.quiet = ctx->help_mode == ZKDL_HELPERS_ABSENT;
    return help;
}

void zk_launch_helped(zkdl_ctx* ctx, int K, const ScTailArgs& a) {
    const ZkHelpLaunch help = zk_help_launch(ctx, (uint64_t)K << a.rounds);
    const int lw = a.rounds >= HELP_64_ROUNDS ? 6 : a.rounds >= HELP_32_ROUNDS ? 5 : 4;
    const dim3 grid(1 + (1 << lw)), block(SC_TAIL_THREADS);
    if (K == 2) hipLaunchKernelGGL(k_sc_helped<2>, grid, block, 0, ctx->stream, a, help, lw);
    else hipLaunchKernelGGL(k_sc_helped<3>, grid, block, 0, ctx->stream, a, help, lw);
}
