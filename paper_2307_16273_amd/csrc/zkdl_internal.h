// Internal declarations shared by the translation units of the library.
#pragma once
#include <stdint.h>
#include <stddef.h>
#include <map>
#include <vector>
#include <hip/hip_runtime.h>

#include "fr.cuh"
#include "sha256.cuh"
#include "../../include/zkdl.h"

constexpr int ZK_MAX_CHAL = 1024;          // challenges one call may draw
constexpr int ZK_PROOF_CAP = 1 << 17;      // proof bytes one call may write
constexpr int ZK_MAX_PART_BLOCKS = 1024;   // partial-sum slots of a round kernel
// Two-round passes of a product sumcheck (k_scpair.hip): the digit sums of a block are exact in 32 bits for
// 2^16 values, so the largest tables take 2^(ZK_PAIR_MAX_LOG - 2 - 16) blocks, 36 sums each; behind them the
// four fold coefficients and 4 KB of their digits.
constexpr int ZK_PAIR_MAX_LOG = 30, ZK_PAIR_BATCH = 256;
constexpr uint64_t ZK_PAIR_BLOCK_VALUES = 1 << 16;
constexpr int ZK_PAIR_SUMS = 36 << (ZK_PAIR_MAX_LOG - 2 - 16), ZK_PAIR_FOLD = 4 + 128;
static_assert(ZK_PAIR_BLOCK_VALUES * 128 * 128 <= 1u << 30, "digit sums with a bit to spare");
constexpr int ZK_PARTIALS = ZK_PAIR_SUMS + ZK_PAIR_FOLD;    // partial sums of one kernel (field elements)
constexpr int ZK_MAX_EVALS = 4;            // evaluations per round polynomial (degree <= 3)
constexpr int ZK_BLOCK = 256;
// Helper blocks of the last rounds (help.cuh): how many a product sumcheck has at most (k_schelp.hip; zkReLU has up to 80, k_zkhelp.hip), the
// places for messages of a round, the longest tables (log2) of a product that go to them, and the time (ticks of 10 ns) after which a
// wait for a running block is given up.
constexpr int ZK_HELP_BLOCKS = 64, ZK_HELP_SLOTS = 80, ZK_HELP_MAX_LOG = 15;
constexpr uint64_t ZK_HELP_WAIT_TICKS = 400000000;
constexpr uint32_t ZK_ERR_RANGE = 1u, ZK_ERR_HELPERS = 2u;     // DevState::err
constexpr int ZK_PEND_CAP = 448;         // bytes of host-known transcript frames waiting for the next transcript kernel
constexpr int ZK_STATE_HEAD = 128;       // bytes at the start of DevState that a call sets from the host

// Device-resident state of the call in flight.
struct DevState {
    uint32_t ts_state[8];   // transcript: SHA-256 chaining value after the last block of the stream
    uint32_t err;           // ZK_ERR_RANGE: zkReLU input out of range; ZK_ERR_HELPERS: a helper block has stopped answering
    uint32_t ts_nblk[2];    // transcript: number of 64-byte blocks in the stream (low, high word)
    uint32_t lag_npts;      // != 0: claim is owed, claim = g(chal[lag_chal]) with the coefficients lag[]
    uint32_t lag_chal;
    uint32_t ts_fill;       // transcript: bytes of the unfinished block
    uint32_t pad0[2];
    uint32_t ts_buf[16];    // transcript: the unfinished block, big-endian words, zero beyond ts_fill
    Fr claim;               // claim of the running sumcheck (Montgomery); current if lag_npts == 0
    Fr lag[4];              // Lagrange coefficients of the last round polynomial
    Fr inv2, inv6;          // constants of the Lagrange formulas
    Fr weights[8];          // zkReLU: r^2, r, r'r^2, r'r, r'
    Fr scal[64];            // scalars handed between kernels (claims, finals)
    Fr chal[ZK_MAX_CHAL];   // challenges, Montgomery form
    uint8_t chal_le[ZK_MAX_CHAL * 32];
    uint8_t proof[ZK_PROOF_CAP];
};

// Where the leader and the helper blocks of a launch write to one another: field elements as limbs with a tag in the upper
// three bits of each word, ten words an element.  Zero between launches but for `go` and `started`.
struct ZkHelpMail {
    uint32_t go;                                   // of the launch: 2 epoch (all helpers run), 2 epoch + 1 (the leader goes on alone)
    uint32_t started[2];                           // helpers that run, by the epoch's lowest bit (k_zk_helped: and those that have read all)
    alignas(64) uint32_t v[2][16];                 // challenges, by the round's lowest bit
    alignas(64) uint32_t coef[2][16][ZK_HELP_SLOTS][10];   // sums of a round, by the round's lowest bit
    alignas(64) uint32_t tab[3][128][10];          // the tables when they go over to the leader
    alignas(64) uint32_t scratch[3 * 9 << ZK_HELP_MAX_LOG];  // long tables of a leader that goes on alone
};

enum TensorKind { TK_FR = 0, TK_I32 = 1, TK_I64 = 2 };

struct zkdl_tensor {
    int kind;
    int ndim;
    uint64_t shape[ZKDL_MAX_DIMS];
    uint64_t numel;
    void* data;      // TK_FR: uint32_t planes (8 * numel words); else the integers
    bool owned;
};

struct zkdl_transcript {
    ts::State s;
};

constexpr int ZK_MAX_PATCHES = 64;       // proof-header records of one call
struct HeaderPatch {
    size_t off;
    uint32_t words[8];
    int n;
};

struct zkdl_ctx {
    int device;
    hipStream_t stream;
    int last_hip;
    DevState* dev;            // device
    uint8_t* host_stage;      // pinned host staging (sizeof(DevState))
    Fr* partials;             // device: ZK_PARTIALS partial sums
    void* static_scratch;     // device address, on this context's device, of the library's static work memory
    std::multimap<size_t, void*> free_blocks;
    std::map<void*, size_t> live_blocks;
    // per-call bookkeeping (host mirrors of device cursors)
    int n_chal;
    size_t proof_len;
    HeaderPatch patches[ZK_MAX_PATCHES];
    int n_patches;
    bool patch_overflow;
    // transcript frames known on the host (protocol headers) that the next transcript
    // kernel absorbs before anything else
    uint8_t pend[ZK_PEND_CAP];
    uint32_t pend_len;
    // zkReLU: the columns of a round are cut into chunks until this many threads are busy
    uint64_t zk_fill_threads;
    // zkReLU: claims and first rounds from one contraction where the stack's size allows it
    bool zk_contraction;
    // helper blocks of the last rounds: their memory, launches so far, ZKDL_HELPERS_*
    ZkHelpMail* help;
    uint32_t help_epoch;
    int help_mode;            // (zk_help_mode: with a look at the device)
    int compute_units;        // of the device
    uint64_t help_wait;       // ticks after which a wait for a running block is given up
    bool help_unread;         // helpers were launched, and no call has seen yet that all their messages were read
    // commitment keys: narrow (8) or wide (12) windows of a tensor entry's tables, 0: chosen by table size
    int commit_wbits;
    // optional per-kernel-class timing with HIP events on the context's stream
    bool prof_on;
    struct ProfSpan {
        hipEvent_t e0, e1;
        int cls;
    };
    std::vector<ProfSpan> prof_spans;   // pool; the first prof_used are pending
    size_t prof_used;
    double prof_ms[ZKDL_PROF_CLASSES];
    double prof_bytes[ZKDL_PROF_CLASSES];
    uint64_t prof_launches[ZKDL_PROF_CLASSES];
};

// Brackets one kernel launch when profiling is on; `bytes` = algorithmic bytes it moves.
void zk_prof_begin(zkdl_ctx* ctx, int cls, double bytes);
void zk_prof_end(zkdl_ctx* ctx);

#define ZK_HIP(ctx, call)                       \
    do {                                        \
        hipError_t e__ = (call);                \
        if (e__ != hipSuccess) {                \
            (ctx)->last_hip = (int)e__;         \
            return ZKDL_EHIP;                   \
        }                                       \
    } while (0)

// scratch allocator of the context (caches freed blocks)
void* zk_alloc(zkdl_ctx* ctx, size_t bytes);
void zk_free(zkdl_ctx* ctx, void* p);

static inline FrTab make_tab(void* p, uint64_t ps) {
    FrTab t;
    t.p = (uint32_t*)p;
    t.ps = ps;
    return t;
}
static inline FrTab tab_offset(const FrTab& t, uint64_t elems) {
    FrTab o = t;
    o.p += elems;
    return o;
}

// ---- k_basic.hip -------------------------------------------------------------
void zk_launch_convert(zkdl_ctx* ctx, const void* src, int kind_or_le, uint64_t n, FrTab out);
void zk_launch_download(zkdl_ctx* ctx, FrTab in, uint64_t n, uint8_t* out_le_dev);
void zk_launch_points_to_mont(zkdl_ctx* ctx, const uint8_t* le_dev, int n, Fr* out);
// chal[dst .. dst + n) = given coordinates: canonical little-endian bytes on the device, or
// (le_dev == nullptr) copies of chal[idx->v[i]]; n <= ZK_CHAL_SET_MAX
constexpr int ZK_CHAL_SET_MAX = 128;
struct ChalIdx {
    int16_t v[ZK_CHAL_SET_MAX];
};
void zk_launch_chal_set(zkdl_ctx* ctx, int dst, int n, const uint8_t* le_dev, const ChalIdx* idx);
// beta~(point, .) for the m challenges point[0..m) (device, Montgomery, AoS)
int zk_build_beta(zkdl_ctx* ctx, const Fr* point, int m, FrTab out);
// beta~(point, .) of m <= ZK_BETA_DIRECT_MAX canonical little-endian coordinates in host memory (any 256-bit values,
// taken mod r); nothing is copied from the host after the call returns.  Whole mle_partial_eval calls on one row of 2^m
// field elements (us, the point copied and the table made of two half tables / like this): m = 2 28 / 23, 6 30 / 24,
// 10 39 / 30, 12 44 / 32, 13 55 / 40, 14 61 / 50, 15 84 / 71, 16 117 / 109; with 64 entries behind each, m = 12 99 / 89,
// 16 309 / 297.  The line is not where the two cross: it is the longest point the launch's arguments are sized for.
constexpr int ZK_BETA_DIRECT_MAX = 16;
void zk_launch_beta_direct(zkdl_ctx* ctx, const uint8_t* le_host, int m, FrTab out);
// several tables with two launches in all (tables of more than 2^22 entries are built one by one)
struct BetaJob {
    const Fr* point;   // device, Montgomery form, m coordinates
    int m;
    FrTab out;         // 2^m entries
};
int zk_build_beta_many(zkdl_ctx* ctx, const BetaJob* jobs, int n);
// I = 1: whether the contraction gives every row of A entries a lane (else a wave)
bool zk_pe_lane_per_row(int kind, uint64_t O, uint64_t A);
// out[o, i] = sum_a beta[a] * src[o, a, i]; src kind TK_*; out has O * I elements
int zk_partial_eval(zkdl_ctx* ctx, int kind, const void* src, uint64_t O, uint64_t A, uint64_t I,
                    FrTab beta, FrTab out);
void zk_launch_broadcast_rows(zkdl_ctx* ctx, FrTab src, uint64_t rows, uint64_t inner, FrTab out);
void zk_launch_soa_to_aos(zkdl_ctx* ctx, FrTab in, int n, Fr* out);
void zk_launch_shift_rows(zkdl_ctx* ctx, FrTab src, uint64_t rows, uint64_t inner, uint32_t period,
                          FrTab out);

// ---- k_sumcheck.hip ------------------------------------------------------------
// Runs all rounds of a degree-K product sumcheck on K packed tables of length 2^d.
// The sources are read only; work_mem (zk_sumcheck_work_bytes(K, d) bytes) receives the
// folded tables.  Writes one SC block at ctx->proof_len, draws d challenges.
size_t zk_sumcheck_work_bytes(int K, int d);
int zk_sumcheck_product(zkdl_ctx* ctx, int K, const FrTab* src, void* work_mem, int d,
                        int finals_scal_base);
// The product sumcheck on (beta~(p, .), X0, X1) for 2^d entries, d >= ZK_HD_MIN_LOG and d >= zk_tail_log + 2 (so from 2^17 entries on, and
// from 2^14 without helper blocks), with two folded tables: the same proof bytes and transcript as zk_sumcheck_product on the three tables.  x: X0, X1
// packed; wsuf[t], t < d - zk_tail_log: beta~(p_[t+1:], .), 2^(d-t-1) entries; eq_tail: 2^(zk_tail_log + 1) work-table
// entries of scratch; work_mem: zk_sumcheck_work_bytes(2, d); p_idx: challenge index of p_0.
constexpr int ZK_HD_MIN_LOG = 14;
// wsuf[t_last] built; fills wsuf[t_last - 1] .. wsuf[t_first], each from the one after it
void zk_hadamard_suffix_tables(zkdl_ctx* ctx, const FrTab* wsuf, int t_last, int t_first, int d, int p_idx);
// xi != nullptr: X0, X1 are int32 arrays on the device; the first two rounds read them, x and wsuf[0] are
// unused and the first round's weights are split[0][b >> split_lb] * split[1][b & (2^split_lb - 1)]
// (beta~ of the leading d - 1 - split_lb and of the last split_lb coordinates of p_[1:]).
int zk_hadamard_eq(zkdl_ctx* ctx, const FrTab* x, const int32_t* const* xi, const FrTab* wsuf, const FrTab* split,
                   int split_lb, void* work_mem, F9Tab eq_tail, int d, int p_idx, int finals_scal_base);
// Queues the frame of a protocol header (label, n <= 8 little-endian u32 words); it is absorbed
// by the next zk_launch_draw / zk_flush_frames, in stream order before everything that follows.
void zk_absorb_words(zkdl_ctx* ctx, const char* label, const uint32_t* words, int n);
// absorbs the queued frames, then draws `count` challenges into chal[chal_base ..)
void zk_launch_draw(zkdl_ctx* ctx, int chal_base, int count);
static inline void zk_flush_frames(zkdl_ctx* ctx) { zk_launch_draw(ctx, 0, 0); }

// ---- k_schelp.hip ----------------------------------------------------------------
// the longest tables (log2) that one launch takes to their end
int zk_tail_log(const zkdl_ctx* ctx);
struct ScTailArgs;
// Helpers run all at once or not at all, each in a compute unit of its own (LDS tables, 1024 threads), next to the leader.  A device
// that has no room for the largest launch, as a partition of 64 compute units or fewer, would wait for them in vain each time: there every
// round has its launches.
static inline bool zk_helpers_fit(int compute_units) { return compute_units > ZK_HELP_SLOTS; }
static inline int zk_help_mode(const zkdl_ctx* ctx) { return zk_helpers_fit(ctx->compute_units) ? ctx->help_mode : ZKDL_HELPERS_OFF; }
// of one launch with helpers
struct ZkHelpLaunch {
    ZkHelpMail* mail;
    uint32_t epoch;
    uint64_t wait, report;    // ticks: for a running block; for the helpers to report
    bool quiet;               // helpers do not report, as if they started too late (ZKDL_HELPERS_ABSENT)
};
// How long the leader waits for its helpers to report before it goes on alone.  On a quiet device all have reported within a few us;
// next to kernels that fill the device with short blocks they wait for a whole compute unit each, up to the end of the kernel that
// holds it.  A leader alone takes 10 to 20 ns an entry of its tables longer than launches per round (us, quiet device: product of three tables of
// 2^15 entries 1279 against 288, of two 906 / 245, of three of 2^12 305 / 207; zkReLU's last rounds on 512 rows of 106 tables 1826 / 762), so it
// waits about that long: 20 ns an entry, at least 40 us.  Whole calls beside additions over 1 GB (us, launches per round / 40 us
// whatever the size / this rule): product of three tables 2^15 577 / 2059 / 380, of two 2^13 381 / 707 / 369, zkReLU of 2^17 rows 1751 / 4052 / 1532;
// beside copies of as much: 459 / 1127 / 464, 456 / 458 / 458, 1631 / 1380 / 1381.  Waiting for 1 ms at every size gains no more.
static inline uint64_t zk_help_report_ticks(uint64_t entries) { return 2 * entries < 4000 ? 4000 : 2 * entries; }
ZkHelpLaunch zk_help_launch(zkdl_ctx* ctx, uint64_t entries);      // entries: of all its tables
void zk_launch_helped(zkdl_ctx* ctx, int K, const ScTailArgs& a);

// ---- k_scpair.hip ------------------------------------------------------------------
// The first J pairs of rounds of a product of K = 2 or 3 packed tables of 2^d entries, two rounds per pass.  Up to 2^15 entries the
// whole sumcheck is one launch with helper blocks; above that whole sumchecks took (us, one round per launch in front of it /
// two rounds per pass): K = 2: 2^16 209 / 206, 2^20 - / 306; K = 3: 2^17 281 / 272, 2^18 323 / 306, 2^19 374 / 346.
constexpr int ZK_PAIR_MIN_LOG = 16;
// blocks of the pass over m values of b (a power of two, at least one batch): one per compute unit (its digits fill the
// LDS), and as many as the exact sums ask for
static inline uint64_t zk_pair_blocks(uint64_t m) {
    const uint64_t fill = m / ZK_PAIR_BATCH < 256 ? m / ZK_PAIR_BATCH : 256, exact = m / ZK_PAIR_BLOCK_VALUES;
    return fill > exact ? fill : exact;
}
int zk_product_pairs(zkdl_ctx* ctx, int K, const FrTab* src, void* work_mem, int d, int J, uint32_t rounds_off, uint32_t claim_off,
                     FrTab* tab, const Fr** w_out);

// ---- k_reindex.hip ---------------------------------------------------------------
struct ReindexJob {
    int K;
    const int32_t* map[ZKDL_REINDEX_MAX_K];   // device: stack index of the j-th tensor of sub-stack k, -1 = zero
    uint64_t len[ZKDL_REINDEX_MAX_K];
    FrTab beta[ZKDL_REINDEX_MAX_K];           // beta~(u_k, .)
    const uint32_t* row_off;                  // device: inverse maps by stack index, 2^ln + 1 offsets into ent
    const uint32_t* ent;                      // device: k in the top 3 bits, j in the other 29
};
// claims of the sub-stacks -> scal[8 ..), absorbed and written to the proof; K coefficients drawn;
// P built into p; product sumcheck on (p, t) over ln variables, finals at scal[0], scal[1]
int zk_reindex(zkdl_ctx* ctx, const ReindexJob& job, FrTab t, FrTab p, int ln, void* work_mem);
// maps of a chained window built on the device: maps [K N], row_off [N + 1], ent [K N], K = 1 + with_ident
void zk_launch_layer_maps(zkdl_ctx* ctx, uint32_t N, uint32_t L, int with_ident, int32_t* maps, uint32_t* row_off,
                          uint32_t* ent);

// claims st->scal[scal_base .. + K) absorbed under "c" and written to the proof at proof_off, then n_draw challenges
// drawn into chal[chal_base ..)
void zk_launch_absorb_claims(zkdl_ctx* ctx, int scal_base, int K, uint32_t proof_off, int chal_base, int n_draw);

// K claims X~(p_k) on the table x (2^d entries) -> one: the claims -> scal[8 ..), absorbed and written
// to the proof; K coefficients drawn; P = sum_k r_k beta[k] built into p; product sumcheck on (p, x),
// finals at scal[0], scal[1]
int zk_merge(zkdl_ctx* ctx, int K, const FrTab* beta, FrTab x, FrTab p, int d, void* work_mem);

// The same for a stack X [N, rows * cols] on tables of the inner size: claim k at the ln + ld
// challenges from point[k] on (stack coordinates first).  Claims -> scal[8 ..) and the proof; K
// coefficients drawn; two product sumchecks (inner over (k, x), then over the stack index), the last
// finals at scal[0], scal[1].  The work memory is appended to `keep` (free it once the stream has
// drained).
struct StackMergeJob {
    int K;
    const Fr* point[ZKDL_REINDEX_MAX_K];   // device, Montgomery form
    int kind;                              // TK_*
    const void* X;                         // TK_FR: const FrTab*; else the integers (device)
    uint64_t N, rows, cols;
};
int zk_stack_merge(zkdl_ctx* ctx, const StackMergeJob& job, std::vector<void*>& keep);

// ---- k_zkrelu.hip ----------------------------------------------------------------
// optimized aggregated matrix-product protocol: stack rounds with f_t, then the single-product sumcheck
int zk_matmul_ft(zkdl_ctx* ctx, const FrTab* src, void* work_mem, int ln, int l2, const FrTab* wsuf, int w_idx,
                 int finals_scal_base);
// given_points != 0: u_Z, u_A, u_GA, u_GZ already stand in chal[n_chal .. n_chal + 4 log2 D); only u_bin is drawn
int zk_zkrelu(zkdl_ctx* ctx, const int64_t* z_dev, const int64_t* ga_dev, uint64_t D, int Q, int R,
              int given_points);

// ---- k_zkprefix.hip ---------------------------------------------------------------
// The input claims, r, r' and the first ZK_PREFIX_VARS i-rounds of zkReLU from one contraction over the rows on the
// matrix cores; then the tables of the linear equations and beta_I with those variables bound (D / 32 entries
// each).  At least one step of 32 rows per value of the leading variables; above 2^26 rows the digit sums leave the
// range of the reduction.  In between it is nowhere slower; whole zkrelu_prove calls (us, round by round / contraction),
// one slice and two:
//   Q + R = 2    2^10 580 / 516, 634 / 548   2^14 759 / 725, 832 / 761   2^18 1001 / 899, 1122 / 957    2^21 1525 / 1102, 1899 / 1209
//   Q + R = 7    2^10 689 / 601, 785 / 644   2^14 921 / 858, 1122 / 973  2^18 1212 / 1072, 1448 / 1237  2^21 1749 / 1302, 2285 / 1549
//   Q + R = 48   2^10 670 / 634, 695 / 648   2^14 834 / 817, 883 / 823   2^18 1137 / 952, 1257 / 1026   2^21 1893 / 1408, 2525 / 1671
//   Q + R = 63   2^10 672 / 641, 709 / 666   2^14 831 / 830, 877 / 852   2^18 1186 / 989, 1313 / 1031   2^21 2463 / 1477, 3470 / 1783
constexpr int ZK_PREFIX_VARS = 5, ZK_PREFIX_MIN_LOG = 10, ZK_PREFIX_MAX_LOG = 26;
struct ZkPrefixJob {
    const int64_t* z;
    const int64_t* ga;       // nullptr: G_A = 0
    uint64_t D;
    int q_bits, r_bits;
    FrTab H[5], L[5];        // beta~ of the coordinates after the leading five of u_Z, u_A, u_GA, u_GZ, u_bin, in two factors
    int lb;                  // coordinates in L
    const Fr* bJ;
    int chal_u[5], chal_r, chal_v;
    uint32_t claims_off, claim0_off, rounds_off;
    F9Tab val[5];            // out: Z, Z', 1 - sign, G_A, G_A'
    F9Tab eq[5];             // out: beta_Z, beta_A, beta_GA, beta_GZ with their weights, beta_I
};
int zk_prefix_rounds(zkdl_ctx* ctx, const ZkPrefixJob& job);

// ---- k_zkshort.hip ----------------------------------------------------------------
// The last i-rounds of zkReLU, from one of at most zk_short_pairs pairs of rows on, in one launch.  The tables hold
// 4 pairs entries, the previous challenge still to be bound; afterwards the two entries of the last pair.
constexpr int ZK_SHORT_PAIRS = 8, ZK_ZHELP_PAIRS = 256;     // in one block; with helper blocks (then one block has the last two rounds at most)
int zk_short_pairs(const zkdl_ctx* ctx);
struct ZkShortJob {
    int pairs, rounds;       // of the first round (a power of two), 1 + log2(pairs)
    F9Tab tab[10];           // 1 - sign | beta_Z, Z | beta_A, Z' | beta_GA, G_A | beta_GZ, G_A' | beta_I
    F9Tab beta_out;          // where beta_I goes
    uint32_t* aux;           // columns: entry (k, j, i), limb l at ((k * nbits + j) * 9 + l) * ps + i
    uint64_t ps;
    int nbits, has_ga;
    const Fr* bJ;
    const Fr* rp;
    int chal;                // index of the first round's challenge; the one before it stands there already
    uint32_t rounds_off;
};
int zk_short_rounds(zkdl_ctx* ctx, const ZkShortJob& job);
// ---- k_zkhelp.hip: the same with helper blocks; false if these rounds are not taken that way
bool zk_helped_rounds(zkdl_ctx* ctx, const ZkShortJob& job);
// What follows the i-rounds: the last fold, the j-rounds, finals and the merge of the three aux claims
struct ZkTailJob {
    F9Tab tab[10];           // as in ZkShortJob, two entries each (one without i-rounds), the last challenge to be bound
    uint32_t* aux;           // columns, rows as left by the last i-round
    uint64_t ps;
    const int64_t* z;        // read when there are no columns (at most one i-round)
    const int64_t* ga;
    const Fr* bJ;
    int has_ga;
    int li, lj, q_bits, r_bits;
    int mat_bound;           // i-challenges bound when the columns were written
    int chal_v;              // index of the first round challenge (i-rounds, then j-rounds)
    int chal_rho;            // rho0..2, then the merge challenges
    uint32_t rounds_off;     // g's of the combined sumcheck (all rounds)
    uint32_t finals_off, merge_claim_off, merge_rounds_off, merge_finals_off;
};
void zk_tail(zkdl_ctx* ctx, const ZkTailJob& job);

// ---- k_general.hip -----------------------------------------------------------------
// the batched matrix product in the general aggregated form: header frame, draw of (w, u), the "ZKGA"
// block; finals Y~, X0~, X1~ -> scal[scal_base ..), scal[scal_base + 3] is used as well
int zk_matmul_general(zkdl_ctx* ctx, const zkdl_tensor* X0, const zkdl_tensor* X1, const zkdl_tensor* Y, int ln,
                      int l1, int l2, int l3, int scal_base);

// ---- api.hip -----------------------------------------------------------------------
size_t zk_claims_unlinked(zkdl_claim* claims_out, const uint8_t* proof, uint32_t L, uint32_t B, uint32_t width, uint32_t T,
                          uint32_t Q, uint32_t R, int cf, size_t pf, int ca, size_t pa, int cw, size_t pw, int cz, size_t pz,
                          size_t pend);
void zk_write_proof_words(zkdl_ctx* ctx, const uint32_t* words, int n);   // appends a header
void zk_host_absorb_u32(zkdl_transcript* t, const char* label, const uint32_t* words, int n);
