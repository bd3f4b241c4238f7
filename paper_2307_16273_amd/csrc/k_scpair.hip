// Product sumchecks of two or three tables, two rounds per pass over the tables (Sec. 2.2).
//
// Write an index as (x0, x1, b), x0 and x1 the variables of two consecutive rounds.  The round polynomials of both
// are sums over b of the bivariate G(X, Y) = sum_b A(X, Y, b) B(X, Y, b) [C(X, Y, b)], so one pass that takes G's
// coefficients serves both rounds and both of their transcript steps, and the next pass binds both challenges on the
// way: the tables are read once and written at a quarter of their length per two rounds, instead of being read twice
// and written at a half and a quarter.
//   K = 3: the products P_uv = A_uv B_uv at u, v in {0, 1, inf} (A_inf = A_1 - A_0: nine products per four entries)
//     and the 36 sums over b of P_uv C_q, q = (x0, x1);
//   K = 2: the 16 sums of A_p B_q.
// Those sums are inner products of field elements over b: with elements as 32 signed digits of 8 bits, the 32 x 32
// matrix of digit products summed over b is a matrix product in integers (v_mfma_i32_32x32x32_i8, exact: |sum| <=
// 2^30 for 2^16 products per block), one reduction per block and sum at the end.  So a pass multiplies 9 (or no) field
// elements per four entries of each table where the two fused rounds multiplied 18 (6) and folded twice, 12 (8).
// The folds are constant matrices: sum_i w_i T_i = sum over the 128 bytes of four sources times (w_i 2^(8 k) mod r), whose
// digits the step that draws the challenges prepares; no multiplications, 110 instructions per folded entry for the carries.
// Three tables of 2^24: first pass 753 us (3.8 k instructions per SIMD and 256 values of b, at 57% of the issue rate; 2.1 TB/s),
// second 467 us (4.3 TB/s, the rate of a copy), third 129 us: the whole sumcheck 2439 -> 1889 us.  One thread per value of b, at
// one wave per SIMD: 1.61 ms for the first pass; products kept in registers over a barrier instead of the LDS filled to the
// last byte: spills, whose reloads wait for the loads of the next batch (1.11 ms too).
// A digit operand wants one digit of 16 values of b per lane while a thread makes 32 digits of one b: a thread writes
// its elements to LDS as rows of 32 bytes and the transposing LDS read (ds_read_b64_tr_b8: eight bytes of
// eight rows) hands them over.
#include <string.h>
#include "dev_common.cuh"
#include "spec_rounds.cuh"

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) v2i* lds_v2i_ptr;
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

constexpr int SP_B = ZK_PAIR_BATCH;      // values of b per batch
constexpr int SP_THREADS = 2 * SP_B;     // two threads per value of b: two waves per SIMD
constexpr int SP_AREA = SP_B * 32;       // bytes of one element per value of b

struct SpArgs {
    FrTab src[3];      // MODE 0: 4 m entries; MODE 1: 16 m entries, folded on the way into dst (4 m; may be src itself)
    FrTab dst[3];
    uint64_t m;        // values of b; a multiple of SP_B
    const v4i* wdig;   // MODE 1: digits of the fold coefficients' multiples (SpFinArgs)
    Fr* part;          // [value][block]
};

// 0x8080..80 - r: the bytes of x + this, each less 128, are signed digits of x - r, for x < 2 r
constexpr uint32_t SP_BIAS[8] = {0x8080807fu, 0x80808081u, 0x80822481u, 0x2cc2dc7du, 0x76dea87bu, 0x4d46a878u, 0x56e30338u, 0x0c92d92du};

__device__ __forceinline__ void put_digits(uint8_t* row, const Fr& x) {
    uint32_t y[8];
    uint64_t c = 0;
#pragma unroll
    for (int l = 0; l < 8; ++l) {
        c += (uint64_t)x.v[l] + SP_BIAS[l];
        y[l] = (uint32_t)c ^ 0x80808080u;
        c >>= 32;
    }
    u4* p = (u4*)row;
    p[0] = u4{y[0], y[1], y[2], y[3]};
    p[1] = u4{y[4], y[5], y[6], y[7]};
}

// operand of 32 rows (elements) from `rows`: lane = digit % 32, half = 16 of the rows.  In a group of 16 lanes every lane
// points at eight bytes of a row; the group's lanes 0..7 (8..15) receive one byte each of the eight rows that its even
// (odd) lanes point at.
__device__ __forceinline__ v4i get_operand(const uint8_t* rows) {
    const int lane = threadIdx.x & 63;
    const uint8_t* p = rows + (16 * (lane >> 5) + ((lane >> 1) & 7)) * 32 + 16 * ((lane >> 4) & 1) + 8 * (lane & 1);
    const v2i a = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)p);
    const v2i b = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(p + 8 * 32));
    return v4i{a[0], a[1], b[0], b[1]};
}

// A block's digit matrices (36 or 16, 32 x 32 each, |entry| <= 2^30) to field elements,
//   sum_kl Y[k][l] 2^(8 (k + l)) / 2^261
// (two Montgomery forms multiplied: the Montgomery form of the product), value x to part[x * nblk].  words: per matrix
// four rows of 64 sums of four digits, row q and lane 32 h + l: word 2 q + h of column l.  Eight threads per matrix
// take four columns each: a wave per matrix with a column per lane did eight times the multiplications, 2.6 us per matrix.
template <int NV>
__device__ __forceinline__ void write_sums(const int64_t* words, Fr* part, uint32_t nblk) {
    const int x = threadIdx.x >> 3, g = threadIdx.x & 7;
    if (x >= NV) return;
    const int64_t* wp = words + 256 * x + 4 * g;
    uint32_t o[10];
    int64_t cy = 0, up = 0;
#pragma unroll
    for (int k = 0; k < 10; ++k) {
        // r * 2^50 keeps the value positive (|sum| < 2^(31 + 25 + 248))
        cy += up + (int64_t)(uint32_t)((k >= 1 && k <= 8 ? frc::MOD[k - 1] << 18 : 0u) | (k >= 2 && k <= 9 ? frc::MOD[k - 2] >> 14 : 0u));
        up = 0;
        if (k < 8) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t w = wp[64 * (k >> 1) + 32 * (k & 1) + j];          // below 2^55
                cy += (int64_t)((uint64_t)(uint32_t)w << (8 * j));
                up += (w >> 32) * (1 << (8 * j));
            }
        }
        o[k] = (uint32_t)cy;
        cy >>= 32;
    }
    F9 lo, hi = f9_zero();
#pragma unroll
    for (int l = 0; l < 9; ++l) {
        const int bit = 29 * l, k = bit >> 5, sh = bit & 31;
        lo.v[l] = (uint32_t)((((uint64_t)o[k + 1] << 32) | o[k]) >> sh) & frc::M29;
    }
    const uint64_t top = (((uint64_t)o[9] << 32) | o[8]) >> 5;                   // bits from 261 on
    hi.v[0] = (uint32_t)top & frc::M29;
    hi.v[1] = (uint32_t)(top >> 29);
    const F9 v = f9_norm_reduce_sum(f9_add(lo, f9_mul(hi, fr_unpack(fr_const(frc::R2)))));
    Fr sc = fr_zero();                   // 2^(32 g)
#pragma unroll
    for (int k = 0; k < 8; ++k) sc.v[k] = g == k ? 1u : 0u;
    F9 s = f9_norm_reduce(f9_mul(v, fr_unpack(sc)));
    f9_add_dpp<0xB1>(s);                 // the eight neighbours: limbs below 2^32
    f9_add_dpp<0x4E>(s);
    f9_add_dpp<0x141>(s);
    if (g == 0) part[(uint64_t)x * nblk] = f9_to_fr(f9_norm_reduce_sum(s));
}

// Two tiles of digit columns (tile 0: values 0..31 of the wave's 64, tile 1: 32..63; lane = value % 32, register i =
// digit 8 (i / 4) + 4 (lane / 32) + i % 4, below 2^22 each) to the words of the lane's own value: word k is
// lo[k] + 2^16 hi[k]
__device__ __forceinline__ void column_words(const v16i& d0, const v16i& d1, int (&lo)[8], int (&hi)[8]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        // the lower half of a wave has even words, the upper half odd ones: exchange the halves of the two tiles
        const auto a = __builtin_amdgcn_permlane32_swap(d0[4 * q] + d0[4 * q + 1] * 256, d1[4 * q] + d1[4 * q + 1] * 256, false, false);
        const auto b = __builtin_amdgcn_permlane32_swap(d0[4 * q + 2] + d0[4 * q + 3] * 256, d1[4 * q + 2] + d1[4 * q + 3] * 256, false, false);
        lo[2 * q] = (int)a[0];
        lo[2 * q + 1] = (int)a[1];
        hi[2 * q] = (int)b[0];
        hi[2 * q + 1] = (int)b[1];
    }
}

// what the columns and base (nine words) add up to, non-negative and below 2^15 r: mod r and below 1.14 r
__device__ __forceinline__ Fr columns_value(const v16i& d0, const v16i& d1, const uint32_t (&base)[9]) {
    int lo[8], hi[8];
    column_words(d0, d1, lo, hi);
    uint32_t o[8];
    int64_t cy = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        cy += (int64_t)lo[k] + (int64_t)hi[k] * 65536 + (int64_t)base[k];
        o[k] = (uint32_t)cy;
        cy >>= 32;
    }
    cy += base[8];
    // value / 2^224 = cy : o[7] (the value is below 2^15 r); 0x23550 = floor(2^48 / (floor(r / 2^224) + 1)): the quotient is
    // short by at most one, and that only for a rest below 0.14 r
    const uint64_t top = ((uint64_t)cy << 32) | o[7];
    const uint32_t q = (uint32_t)(((top >> 16) * 0x23550u) >> 32);
    Fr x;
    int64_t c = 0;
    uint64_t bq = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        bq += (uint64_t)q * frc::MOD[k];
        c += (int64_t)o[k] - (int64_t)(uint32_t)bq;
        x.v[k] = (uint32_t)c;
        c >>= 32;
        bq >>= 32;
    }
    return x;
}

template <int K, int MODE>
__global__ __launch_bounds__(SP_THREADS, 1) void k_sp_pass(SpArgs a) {
    // K = 3: the packed entries of the first two tables (eight words per value of b and entry, by word), then eight of
    // the nine products and the four entries of the third table; the ninth product follows into the first entry's place
    // once all have been read.  K = 2: four left entries and four right ones.
    constexpr int LEFT = K == 3 ? 9 : 4, NT = (LEFT + 1) / 2;    // operands on the left; tiles per wave
    constexpr int NE = 2 * K;                                    // entries loaded per thread
    constexpr int NV = 4 * LEFT;
    constexpr int PARK = K == 3 ? 8 : 0, RIGHT = K == 3 ? 16 : 4, AREAS = RIGHT + 4;
    __shared__ alignas(16) uint8_t smem[AREAS * SP_AREA];
    static_assert(AREAS * SP_AREA <= 160 * 1024 && NV * 256 * 8 <= AREAS * SP_AREA && NV * 8 <= SP_THREADS, "the sums' words reuse the digits' room");
    const int tid = threadIdx.x, bl = tid & (SP_B - 1), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = wave >> 2;
    // entry of which table the j-th entry of this half is: the first (second) table's four and two of the third's
    auto slot = [&](int j) { return j < 4 ? 4 * half + j : 4 + 2 * half + j; };
    auto put_entry = [&](int g, const Fr& x) {
        if (K == 3 && g < 8) {
            uint32_t* park = (uint32_t*)smem + 8 * g * SP_B + bl;
#pragma unroll
            for (int l = 0; l < 8; ++l) park[l * SP_B] = x.v[l];
        } else {
            put_digits(smem + (K == 3 ? RIGHT + g - 8 : g) * SP_AREA + bl * 32, x);
        }
    };
    const uint64_t m = a.m, step = (uint64_t)gridDim.x * SP_B;
    const FrTab own = a.src[half];
    v16i acc[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[i][j] = 0;
    // MODE 0: the next batch's entries; MODE 1: the sources of the next entry
    Fr raw[MODE == 0 ? NE : 1];
    v4i t[2][4];
    auto load = [&](uint64_t b) {
#pragma unroll
        for (int j = 0; j < NE; ++j) raw[MODE == 0 ? j : 0] = tab_ld(j < 4 ? own : a.src[2], b + (uint64_t)(slot(j) & 3) * m);
    };
    auto fetch = [&](int j, uint64_t b0) {
        // 64 values of b per wave as two tiles of 32; lane / 32 = half of the words
        const FrTab& s = j < 4 ? own : a.src[2];
        const uint32_t* p = s.p + (uint64_t)(4 * (lane >> 5)) * s.ps + b0 + 64 * (wave & 3) + (lane & 31) + (uint64_t)(slot(j) & 3) * m;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int l = 0; l < 4; ++l) t[h][i][l] = (int)p[l * s.ps + (uint64_t)(4 * i) * m + 32 * h];
    };
    uint64_t b0 = blockIdx.x * (uint64_t)SP_B;
    if (MODE == 0) load(b0 + bl);
    else fetch(0, b0);
    v4i wm[4];
    uint32_t base[9];
    if (MODE == 1) {
        // the bytes of a source less 128 are what is multiplied: 128 times the sum of a column's digits is what is missing
        v16i bias;
#pragma unroll
        for (int j = 0; j < 16; ++j) bias[j] = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            wm[i] = a.wdig[64 * i + lane];
            bias = __builtin_amdgcn_mfma_i32_32x32x32_i8(wm[i], v4i{(int)0x80808080, (int)0x80808080, (int)0x80808080, (int)0x80808080}, bias, 0, 0, 0);
        }
        int lo[8], hi[8];
        column_words(bias, bias, lo, hi);        // the same in every lane
        int64_t cy = 0;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            if (k < 8) cy -= (int64_t)lo[k] + (int64_t)hi[k] * 65536;
            base[k] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)cy);
            cy >>= 32;
        }
    }
    for (; b0 < m; b0 += step) {
        const uint64_t nb = b0 + step < m ? b0 + step : b0;      // the last batch asks for its own again
        if (MODE == 0) {
#pragma unroll
            for (int j = 0; j < NE; ++j) put_entry(slot(j), raw[MODE == 0 ? j : 0]);
            load(nb + bl);
        } else {
            // sum_i w_i T[b + (q + 4 i) m]
#pragma unroll 1
            for (int j = 0; j < NE; ++j) {
                v16i d0, d1;
#pragma unroll
                for (int i = 0; i < 16; ++i) d0[i] = d1[i] = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    d0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(wm[i], t[0][i] ^ (int)0x80808080, d0, 0, 0, 0);
                    d1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(wm[i], t[1][i] ^ (int)0x80808080, d1, 0, 0, 0);
                }
                if (j + 1 < NE) fetch(j + 1, b0);
                else fetch(0, nb);
                const Fr x = columns_value(d0, d1, base);
                tab_st(j < 4 ? a.dst[half] : a.dst[2], b0 + bl + (uint64_t)(slot(j) & 3) * m, x);
                put_entry(slot(j), x);
            }
        }
        __syncthreads();
        if (K == 3) {
            auto entry = [&](int g) {
                const uint32_t* park = (const uint32_t*)smem + 8 * g * SP_B + bl;
                Fr y;
#pragma unroll
                for (int l = 0; l < 8; ++l) y.v[l] = park[l * SP_B];
                return fr_unpack(y);
            };
            // products at (u, v), 2 = inf.  Sources are below 2 r, differences below 6 r; the double differences, below
            // 12 r, are reduced in one factor: every product is below 2 r
            // the order on the left: 00, 01, 10, 11, 0 inf, 1 inf, inf 0, inf 1, inf inf
            uint8_t* row = smem + (PARK + 4 * half) * SP_AREA + bl * 32;
            if (half == 0) {
                F9 d = f9_zero(), e = f9_zero();
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const F9 x = entry(q), y = entry(4 + q);
                    d = q == 0 || q == 3 ? f9_add(d, x) : f9_sub(d, x);
                    e = q == 0 || q == 3 ? f9_add(e, y) : f9_sub(e, y);
                    put_digits(row + q * SP_AREA, fr_pack(f9_mul(x, y)));
                }
                const Fr ninth = fr_pack(f9_mul(f9_norm_reduce(d), f9_norm(e)));
                __syncthreads();         // the parked entries have been read
                put_digits(smem + bl * 32, ninth);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    // (0, inf), (1, inf), (inf, 0), (inf, 1)
                    const int p = q == 0 ? 0 : q == 1 ? 2 : q == 2 ? 0 : 1, n = q == 0 ? 1 : q == 1 ? 3 : q == 2 ? 2 : 3;
                    put_digits(row + q * SP_AREA, fr_pack(f9_mul(f9_norm(f9_sub(entry(n), entry(p))), f9_norm(f9_sub(entry(4 + n), entry(4 + p))))));
                }
                __syncthreads();
            }
            __syncthreads();
        }
        // wave: its half of the left operands against entry (wave % 4) of the last table
        const uint8_t* right = smem + (RIGHT + (wave & 3)) * SP_AREA;
        const uint8_t* left = smem + (K == 3 ? PARK + 4 * half : 2 * half) * SP_AREA;
#pragma unroll 2
        for (int ks = 0; ks < SP_B / 32; ++ks) {
            const v4i r = get_operand(right + ks * 1024);
#pragma unroll
            for (int i = 0; i < LEFT / 2; ++i)
                acc[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(get_operand(left + i * SP_AREA + ks * 1024), r, acc[i], 0, 0, 0);
            if (K == 3 && half == 0)
                acc[NT - 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(get_operand(smem + ks * 1024), r, acc[NT - 1], 0, 0, 0);
        }
        __syncthreads();
    }
    int64_t* words = (int64_t*)smem;
#pragma unroll
    for (int i = 0; i < NT; ++i)
        if (i < LEFT / 2 || half == 0) {
            // left operands 0..3, 4..7 (K = 2: 0, 1 and 2, 3), then the ninth
            const int u = i == LEFT / 2 ? LEFT - 1 : LEFT / 2 * half + i;
            int64_t* w = words + (LEFT * (wave & 3) + u) * 256 + lane;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                w[64 * q] = (int64_t)acc[i][4 * q] + (int64_t)acc[i][4 * q + 1] * 256 + (int64_t)acc[i][4 * q + 2] * 65536 +
                            (int64_t)acc[i][4 * q + 3] * 16777216;
        }
    __syncthreads();
    write_sums<NV>(words, a.part + blockIdx.x, gridDim.x);
}

// ---- the two transcript steps --------------------------------------------------------------------
struct SpFinArgs {
    const Fr* part;        // [q][left][block]
    int nblk;
    DevState* st;
    int chal_idx;          // of the first of the two rounds
    uint32_t proof_off;    // where its g(0..K) go; the second round's follow
    int first;             // claim_0 = g(0) + g(1) is written and absorbed first
    uint32_t claim_off;
    Fr* w;                 // out: the four fold coefficients of the two challenges
    v4i* wdig;             // out: the signed digits of w_i 2^(8 k) mod r, i < 4, k < 32, as the pass's operands: digit l at
                           // byte 16 (64 i + 32 (k / 16) + l) + k % 16
};

constexpr int SP_FIN_THREADS = 1024;
static_assert(SP_FIN_THREADS >= SPEC_MIN_THREADS, "the waves beside the hashes");

// With left basis phi (K = 3: 1 - x, x, x^2 - x; K = 2: 1 - x, x) and right basis psi (1 - x, x),
//   G(X, Y) = sum phi_u(X) psi_x(X) phi_v(Y) psi_y(Y) G[(u, v)][(x, y)]:
// the first round sums over y = v in {0, 1}, the second has X bound.  Bound by its chain of hashes: the second round's
// polynomial is worked out in the first challenge while that is being drawn (spec_rounds.cuh).  With the basis products, the
// sums and their barriers between the two hashes the eight finalisers of a product of 2^24 entries took 254 us, not 215.
template <int K>
__global__ __launch_bounds__(SP_FIN_THREADS) void k_sp_finalise(SpFinArgs a) {
    constexpr int U = K == 3 ? 3 : 2, LEFT = U * U, NV = 4 * LEFT, NTERM = 2 * U, NPTS = K + 1;
    __shared__ F9 G[NV], H[NTERM], co[NPTS][NTERM];
    __shared__ TsShared S;
    __shared__ RoundShared R;            // the first round's values
    __shared__ SpecShared<K> X;
    __shared__ F9 wl[4];
    __shared__ alignas(16) uint8_t dig[4096];
    DevState* st = a.st;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    auto phi = [](int u, int x) { return u == 0 ? 1 - x : u == 1 ? x : x * x - x; };
    // the place of (u, v) on the left
    auto at = [](int u, int v) { return K == 2 ? 2 * u + v : u < 2 ? (v < 2 ? 2 * u + v : 4 + u) : v < 2 ? 6 + v : 8; };
    // a row of 16 lanes per value: all values' partial sums are on their way at once
    const int row = tid >> 4;
    if (row < NV) {
        const Fr* part = a.part + (uint64_t)row * a.nblk;
        F9 s = f9_zero();
        for (int c = tid & 15; c < a.nblk; c += 128) {
            Fr p[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) p[q] = c + 16 * q < a.nblk ? part[c + 16 * q] : fr_zero();
#pragma unroll
            for (int q = 0; q < 8; ++q) s = f9_add(q == 7 ? f9_norm(s) : s, fr_unpack(p[q]));   // limbs below 2^32
            s = f9_norm_reduce(s);       // below 2.41 r + 8 r before
        }
        f9_add_dpp<0xB1>(s);
        f9_add_dpp<0x4E>(s);
        f9_add_dpp<0x141>(s);
        s = f9_norm(s);
        f9_add_dpp<0x140>(s);            // the row's total, below 39 r
        s = f9_norm_reduce_sum(s);
        if ((tid & 15) == 0) G[row] = s;
    }
    if (tid == 0) spec_init<K>(X);
    block_ts_load(S, st);
    // phi_u(x) psi_y(x) at the evaluation points (small integers)
    if (tid >= 256 && tid < 256 + NPTS * NTERM) {
        const int x = (tid - 256) / NTERM, u = (tid - 256) % NTERM >> 1, y = tid & 1;
        co[x][2 * u + y] = fr_unpack(fr_from_i64(phi(u, x) * (y ? x : 1 - x)));
    }
    if (tid < NTERM) {                   // y = v in {0, 1} summed out
        const int u = tid >> 1, x = tid & 1;
        H[tid] = f9_norm_reduce(f9_add(G[(2 * x) * LEFT + at(u, 0)], G[(2 * x + 1) * LEFT + at(u, 1)]));
    }
    __syncthreads();
    // g(x) of the first round: wave x, lane = term
    if (wave < NPTS) {
        F9 s = f9_zero();
        if (lane < NTERM) s = f9_norm_reduce(f9_mul(co[wave][lane], H[lane]));
        s = wave_sum_lazy(s, 8);
        if (lane == 0) round_eval_out(S, R, (uint32_t*)(st->proof + a.proof_off), wave, s, true);
    }
    __syncthreads();
    if (a.first) {
        if (tid == 0) round_claim_out(S, f9_norm(f9_add(R.g9[0], R.g9[1])), (uint32_t*)(st->proof + a.claim_off), nullptr);
        __syncthreads();
    }
    const int beside = (wave & 2) && wave < 8 ? ((wave >> 2) << 1) | (wave & 1) : NPTS;    // waves 2, 3, 6, 7: 0 .. 3
    if (wave < 2) {
        wave_frame_draw1_open(S, 'g', K, [&](uint32_t i) -> uint32_t { return S.canon[i >> 3][i & 7]; }, a.first != 0);
    } else if (beside < NPTS) {
        // g(x) of the second round as a polynomial in the first challenge v: its values at v = 0, 1, (K = 3: -1,) infinity,
        // a row of 16 lanes each, are small-integer combinations of the sums:
        //   sum over (u, x'), (v', y') of phi_u(v) psi_x'(v) phi_v'(x) psi_y'(x) G[(u, v')][(x', y')]
        const int x = beside, y = K == 3 ? (lane >> 4 == 2 ? -1 : lane >> 4) : lane >> 4;
        const bool inf = lane >> 4 == K;                       // the coefficient of v^K
        int64_t acc[9];
#pragma unroll
        for (int l = 0; l < 9; ++l) acc[l] = 300ll * (int64_t)frc::MOD9[l];     // the terms are below 240 r together
        for (int term = lane & 15; term < NTERM * NTERM; term += 16) {
            const int o = term / NTERM, i = term % NTERM, vv = o >> 1, yy = o & 1, u = i >> 1, xx = i & 1;
            int c = phi(vv, x) * (yy ? x : 1 - x);
            if (inf) c *= (K == 3 ? (u == 2 ? 1 : 0) : (u ? 1 : -1)) * (xx ? 1 : -1);
            else c *= phi(u, y) * (xx ? y : 1 - y);
            const F9& g = G[(2 * xx + yy) * LEFT + at(u, vv)];
#pragma unroll
            for (int l = 0; l < 9; ++l) acc[l] += (int64_t)c * (int32_t)g.v[l];
        }
        const int64_t q = (int64_t)(((uint64_t)(uint32_t)acc[8] * 565u) >> 32);
        F9 val;
        int64_t carry = 0;
#pragma unroll
        for (int l = 0; l < 8; ++l) {
            const int64_t z = acc[l] - q * (int64_t)frc::MOD9[l] + carry;
            val.v[l] = (uint32_t)z & frc::M29;
            carry = z >> 29;
        }
        val.v[8] = (uint32_t)(acc[8] - q * (int64_t)frc::MOD9[8] + carry);     // below 2.1 r
        if (K == 2 && lane >= 48) val = f9_zero();
        spec_coefficients<K>(X, x, 0, wave_sum_lazy(val, 16));
    }
    __syncthreads();
    const F9 v0 = S.v9;
    if (wave == 0) spec_chain<K>(S, X, v0, 1);
    else if (wave == 1) spec_second<K>(S, X, st, 1, a.proof_off + NPTS * 32, a.chal_idx + 1, v0, true);
    __syncthreads();
    if (tid < 4) {                       // (1 - v0)(1 - v1), (1 - v0) v1, v0 (1 - v1), v0 v1
        const F9 one9 = fr_unpack(fr_one()), v1 = X.v9[0];
        const F9 w = f9_cond_sub(f9_mul(tid & 2 ? v0 : f9_norm(f9_sub(one9, v0)), tid & 1 ? v1 : f9_sub(one9, v1)));
        a.w[tid] = fr_pack(w);
        wl[tid] = w;
    }
    __syncthreads();
    if (tid < 128) {
        const int i = tid >> 5, k = tid & 31;
        Fr s = fr_zero();
#pragma unroll
        for (int l = 0; l < 8; ++l) s.v[l] = (k >> 2) == l ? 1u << (8 * (k & 3)) : 0u;
        const Fr y = fr_pack(f9_cond_sub(f9_mul(wl[i], fr_unpack(s))));   // plain w_i 2^(8 k), below r
        uint32_t c = 0;
#pragma unroll
        for (int l = 0; l < 8; ++l) {
            // balanced digits: bytes of y + 0x80..80, each less 128
            const uint64_t t = (uint64_t)y.v[l] + 0x80808080u + c;
            c = (uint32_t)(t >> 32);
            const uint32_t word = (uint32_t)t ^ 0x80808080u;
#pragma unroll
            for (int j = 0; j < 4; ++j) dig[16 * (64 * i + 32 * (k >> 4) + 4 * l + j) + (k & 15)] = (uint8_t)(word >> (8 * j));
        }
    }
    __syncthreads();
    if (tid < 256) a.wdig[tid] = ((const v4i*)dig)[tid];
    block_ts_store(S, st);
}

}  // namespace

// passes of two rounds each over tables of 2^d entries, ZK_PAIR_MIN_LOG <= d <= ZK_PAIR_MAX_LOG, K = 2 or 3: the first J pairs of rounds (the caller has
// written the block's header and takes over with *tab, 2^(d - 2 (J - 1)) entries, and the coefficients *w that bind
// the last pair's challenges).  work_mem: K 2^(d - 2) packed entries.
int zk_product_pairs(zkdl_ctx* ctx, int K, const FrTab* src, void* work_mem, int d, int J, uint32_t rounds_off, uint32_t claim_off,
                     FrTab* tab, const Fr** w_out) {
    const uint64_t quarter = (uint64_t)1 << (d - 2);
    FrTab work[3];
    for (int k = 0; k < K; ++k) work[k] = make_tab((uint32_t*)work_mem + (size_t)k * 8 * quarter, quarter);
    Fr* w = ctx->partials + ZK_PAIR_SUMS;                      // behind the partial sums
    v4i* wdig = (v4i*)(w + 4);
    const int npts = K + 1;
    for (int j = 0; j < J; ++j) {
        SpArgs sa;
        for (int k = 0; k < 3; ++k) {
            sa.src[k] = j <= 1 ? src[k < K ? k : 0] : work[k < K ? k : 0];
            sa.dst[k] = work[k < K ? k : 0];
        }
        sa.m = (uint64_t)1 << (d - 2 * j - 2);
        sa.wdig = wdig;
        sa.part = ctx->partials;
        const uint64_t grid = zk_pair_blocks(sa.m);
        // algorithmic bytes: the tables once; later passes four source entries per entry written as well
        zk_prof_begin(ctx, j ? ZKDL_PROF_SC_ROUND_FUSED : ZKDL_PROF_SC_ROUND_FIRST, (double)K * (j ? 640.0 : 128.0) * (double)sa.m);
        if (K == 3) {
            if (j) hipLaunchKernelGGL((k_sp_pass<3, 1>), dim3((unsigned)grid), dim3(SP_THREADS), 0, ctx->stream, sa);
            else hipLaunchKernelGGL((k_sp_pass<3, 0>), dim3((unsigned)grid), dim3(SP_THREADS), 0, ctx->stream, sa);
        } else {
            if (j) hipLaunchKernelGGL((k_sp_pass<2, 1>), dim3((unsigned)grid), dim3(SP_THREADS), 0, ctx->stream, sa);
            else hipLaunchKernelGGL((k_sp_pass<2, 0>), dim3((unsigned)grid), dim3(SP_THREADS), 0, ctx->stream, sa);
        }
        zk_prof_end(ctx);
        SpFinArgs fa;
        fa.part = ctx->partials;
        fa.nblk = (int)grid;
        fa.st = ctx->dev;
        fa.chal_idx = ctx->n_chal;
        ctx->n_chal += 2;
        fa.proof_off = rounds_off + (uint32_t)(2 * j) * npts * 32;
        fa.first = j == 0;
        fa.claim_off = claim_off;
        fa.w = w;
        fa.wdig = wdig;
        zk_prof_begin(ctx, ZKDL_PROF_FINALISE, 64.0 * npts);
        if (K == 3) hipLaunchKernelGGL(k_sp_finalise<3>, dim3(1), dim3(SP_FIN_THREADS), 0, ctx->stream, fa);
        else hipLaunchKernelGGL(k_sp_finalise<2>, dim3(1), dim3(SP_FIN_THREADS), 0, ctx->stream, fa);
        zk_prof_end(ctx);
    }
    for (int k = 0; k < 3; ++k) tab[k] = J == 1 ? src[k < K ? k : 0] : work[k < K ? k : 0];
    *w_out = w;
    return ZKDL_OK;
}
