// zkReLU (Sec. 3.1, App. A): the input claims and the first five i-rounds from one pass over the integers.
//
// Write a row as i = (s, rho), s the five leading variables, rho the others, and X for the five challenges.
// Every equality factor splits, beta~(u, (X, rho)) = beta~(u_hi, X) beta~(u_lo, rho), and the bits and integers
// of a row with X bound are sum_s chi_s(X) (value of row (s, rho)), so the combined sum is
//   sum_e w_e beta~(u^e_hi, X) Q_e(X),
//   Z, G_A:            Q = sum_s chi_s V[s],            V[s]    = sum_rho beta~(u_lo, rho) value(s, rho),
//   A, G_Z:            Q = sum_{s,s'} chi_s chi_s' M[s][s'], M  = sum_rho beta~(u_lo, rho) (1 - sign)(s, rho) value(s', rho),
//   both binarities:   Q = - sum_{s<s'} chi_s chi_s' N[s][s'],  N = sum_{rho,k,j} beta~(u_lo, rho) c_k beta_J(j)
//                      [bit_(k,j)(s, rho) != bit_(k,j)(s', rho)]     (sum_s chi_s = 1, bits are idempotent),
// polynomials of a few thousand coefficients: the claims are their values at u_hi, and the five rounds and their
// transcript steps run on them in one block (k_zk_prefix).  The rows are read once, when the coefficients are
// taken, and once more when the five challenges are bound.
//
// The coefficients are exact contractions over rho of bits or of 8-bit digits with the field elements
// beta~(u_lo, rho), which enter as 32 signed digits of 8 bits: matrix products in integers, on the matrix cores
// (v_mfma_i32_32x32x32_i8: 32 digits x 32 columns, 32 values of rho per instruction; |sum| < 2^31 for 2^17 values).
//   * N: the columns of a tile are 32 of the bit columns (k, j) of one pair (s, s').  A lane holds one bit column as a
//     word of 32 values of rho, so the operand is (W_s ^ W_s') & 0x01010101 << t, one v_bitop3 per register: byte p of
//     register t is the bit of rho = 8 p + t with the weight 2^t (-128 for t = 7), and the digits of that rho are those
//     of 2^-t beta~ (-2^-7 beta~).
//   * M, V: the columns are the 32 rows s' of one digit of the value, masked by the sign bytes of s.
// The cost is 496 pairs x (Q+R) columns per slice and rho, 15.5 bit products per bit of the input.  A round each on
// the integers (look-up tables of beta_J, split equality tables, column sums handed on) took 4.1 ms, claims included,
// for the 2^23 rows of two slices of sixteen steps of the 8 x 1024 network and 4.9 ms for 2^24 rows of one; here
// the operands take 0.23 ms, the pairs 0.33 ms, the values 0.21 ms and claims and rounds 0.16 ms (0.28, 0.42, 0.14,
// 0.15 ms for the 2^24 rows).
#include <string.h>
#include "dev_common.cuh"

namespace {

constexpr int PV = 5;                    // variables bound together
constexpr int PS = 1 << PV;              // values of s
constexpr int PAIR_TILES = 512;          // 28 blocks of 4 x 4 pairs, 4 tiles of two diagonal blocks (12 pairs each, 4 unused)

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

struct PrefixArgs {
    const int64_t* z;
    const int64_t* ga;       // nullptr: one slice
    uint64_t P;              // values of rho, a multiple of 32
    uint32_t NB;             // P / 32
    int nbits, r_bits, q_bits;
    int ns;                  // slices
    int G;                   // groups of 32 bit columns
    int nbZ, nbP;            // digits of Z / G_A and of their rescaled values
    uint32_t* bits;          // [block of 32 rho][s][32 G]: bit columns, bit rho % 32
    int8_t* dig;             // [value][digit][s][rho]; values Z, Z', G_A, G_A'
    uint8_t* nsign;          // [s][rho]: 0xff where the sign bit of Z is 0
    v4i* wd;                 // [e][block of 32 rho][64 lanes]: digit operands of the five points; block NB is zero
    int* part;               // pairs: [chunk][tile][4][64][4]
    int chunks;
    uint32_t blocks_per_chunk;
    int* part_v;             // matrices and vectors: the same
    int n_tiles_v, chunks_v;
    uint32_t blocks_per_chunk_v;
    FrTab H[5], L[5];        // beta~(u_lo, rho) = H[rho >> lb] L[rho % 2^lb], packed: Z, A, G_A, G_Z, I
    int lb;
    const Fr* bJ;
    uint32_t* N9;            // [slice][group][PAIR_TILES] lazy limbs (nine words each)
    uint32_t* M9;            // [eq][digit][s][s']
    uint32_t* V9;            // [eq][digit][s]
    DevState* st;
};

__device__ __forceinline__ int64_t rescale_half_up(int64_t x, int r_bits) {
    return (x >> r_bits) + ((x >> (r_bits - 1)) & 1);
}

__device__ __forceinline__ bool in_range(int64_t x, int nbits) {
    if (nbits >= 64) return true;
    const int64_t top = x >> (nbits - 1);
    return top == 0 || top == -1;
}

// in-place transpose of a 32 x 32 bit matrix: afterwards bit p of a[j] is what bit j of a[p] was
__device__ __forceinline__ void transpose32(uint32_t a[32]) {
#pragma unroll
    for (int s = 0; s < 5; ++s) {
        const int j = 16 >> s;
        const uint32_t m = s == 0 ? 0x0000FFFFu : s == 1 ? 0x00FF00FFu : s == 2 ? 0x0F0F0F0Fu : s == 3 ? 0x33333333u : 0x55555555u;
#pragma unroll
        for (int k = 0; k < 32; ++k) {
            if (k & j) continue;
            const uint32_t t = ((a[k] >> j) ^ a[k + j]) & m;
            a[k] ^= t << j;
            a[k + j] ^= t;
        }
    }
}

// ---- the integers as bit columns, digits and sign bytes ------------------------------------------
constexpr int PL_ROWS = 1024;            // values of rho per block

// Bound by its stores (the digits, the sign and the bits are 20 bytes per integer of 56 bits): a thread has four
// neighbouring integers and stores their digits as one word (a byte per lane and store, and every transposed word to a line of its own: 247 us for 2^23
// integers, 97 like this), and the transposed
// words go out through LDS, neighbouring columns by neighbouring lanes.
__global__ __launch_bounds__(256) void k_zk_planes(PrefixArgs a) {
    __shared__ uint64_t zz[2][PL_ROWS + PL_ROWS / 32];   // a padding word every 32 rows: the transposing lanes read with
                                                         // a stride of 33 entries, not 32
    const int tid = threadIdx.x, s = blockIdx.y;
    const uint64_t r0 = (uint64_t)blockIdx.x * PL_ROWS;
    const uint32_t n = a.P - r0 < PL_ROWS ? (uint32_t)(a.P - r0) : PL_ROWS;   // a multiple of 32
    bool bad = false;
    static_assert(PL_ROWS == 4 * 256, "four rows per thread");
    const uint32_t i = 4 * tid;
    if (i < n) {
        const uint64_t row = (uint64_t)s * a.P + r0 + i;
        for (int k = 0; k < a.ns; ++k) {
            const int64_t* src = (k ? a.ga : a.z) + row;
            int64_t x[4], y[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = src[q];
            uint32_t ns = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bad |= !in_range(x[q], a.nbits);
                zz[k][i + (i >> 5) + q] = (uint64_t)x[q];
                ns |= ((x[q] >> (a.nbits - 1)) & 1) ? 0u : 0xffu << (8 * q);
                y[q] = rescale_half_up(x[q], a.r_bits);
            }
            if (k == 0) *(uint32_t*)(a.nsign + row) = ns;
            // signed digits: x = d + 256 x', d in [-128, 127], x' = (x >> 8) + bit 7
            int8_t* out = a.dig + (uint64_t)k * (a.nbZ + a.nbP) * PS * a.P + row;
            auto digits = [&](int64_t (&z)[4], int count) {
                for (int e = 0; e < count; ++e) {
                    uint32_t w = 0;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        w |= ((uint32_t)z[q] & 0xffu) << (8 * q);
                        z[q] = (z[q] >> 8) + ((z[q] >> 7) & 1);
                    }
                    *(uint32_t*)out = w;
                    out += (uint64_t)PS * a.P;
                }
            };
            digits(x, a.nbZ);
            digits(y, a.nbP);
        }
    }
    if (bad) atomicOr(&a.st->err, ZK_ERR_RANGE);
    __syncthreads();
    // thread = (block of 32 rows, slice, half word): 32 words in, 32 bit columns out
    constexpr uint32_t STRIDE = 129;                     // words of a block of rows: up to 2 x 64 columns, and one
    static_assert(sizeof zz >= PL_ROWS / 32 * STRIDE * 4, "the columns take the integers' place");
    uint32_t* words = (uint32_t*)&zz[0][0];
    const uint32_t nblk = n >> 5, halves = a.nbits > 32 ? 2 : 1, columns = a.ns * a.nbits;
    const uint32_t b = tid % nblk, kw = tid / nblk, k = kw / halves, w = kw % halves;
    uint32_t m[32];
    if (k < (uint32_t)a.ns) {
#pragma unroll
        for (int r = 0; r < 32; ++r) m[r] = ((const uint32_t*)zz[k])[2 * (33 * b + r) + w];
        transpose32(m);
    }
    __syncthreads();
    if (k < (uint32_t)a.ns) {
        const int cnt = a.nbits - 32 * (int)w;
#pragma unroll
        for (int r = 0; r < 32; ++r)
            if (r < cnt) words[b * STRIDE + k * a.nbits + 32 * w + r] = m[r];
    }
    __syncthreads();
    uint32_t* out = a.bits + ((r0 >> 5) * PS + s) * (32 * a.G);
    const uint32_t wave = tid >> 6, lane = tid & 63;
    for (uint32_t r = wave; r < nblk; r += 4)
        for (uint32_t c = lane; c < columns; c += 64) out[(uint64_t)r * PS * 32 * a.G + c] = words[r * STRIDE + c];
}

// ---- the weights beta~(u_lo, rho) as digit operands ----------------------------------------------
__global__ __launch_bounds__(256) void k_zk_weight_digits(PrefixArgs a) {
    __shared__ uint8_t stage[8 * 1024];
    __shared__ F9 scale[8];              // 2^-t, the last one negated
    const int tid = threadIdx.x, e = blockIdx.y;
    if (a.ns == 1 && (e == 2 || e == 3)) return;
    if (tid < 8) {
        Fr c = fr_one();
        for (int t = 0; t < tid; ++t) {          // halved: r is odd, c + r below 2^256
            const uint32_t odd = 0u - (c.v[0] & 1u);
            uint64_t cy = 0;
#pragma unroll
            for (int l = 0; l < 8; ++l) {
                cy += (uint64_t)c.v[l] + (frc::MOD[l] & odd);
                c.v[l] = (uint32_t)cy;
                cy >>= 32;
            }
#pragma unroll
            for (int l = 0; l < 8; ++l) c.v[l] = (c.v[l] >> 1) | (l < 7 ? c.v[l < 7 ? l + 1 : 7] << 31 : 0u);
        }
        scale[tid] = fr_unpack(tid == 7 ? fr_neg(c) : c);
    }
    __syncthreads();
    const uint64_t rho = (uint64_t)blockIdx.x * 256 + tid;
    if (rho < a.P) {
        F9 w = f9_mul(fr_unpack(tab_ld(a.H[e], rho >> a.lb)), fr_unpack(tab_ld(a.L[e], rho & (((uint64_t)1 << a.lb) - 1))));
        // place of rho among the 32 of its block: lane half h, byte b of the 16
        const uint32_t q = (uint32_t)rho & 31;
        uint32_t h, b;
        if (e == 4) {                    // rho = 8 p + t: register t % 4 of half t / 4, byte p
            const uint32_t t = q & 7, p = q >> 3;
            h = t >> 2;
            b = (t & 3) * 4 + p;
            w = f9_mul(w, scale[t]);
        } else {
            h = q >> 4;
            b = q & 15;
        }
        const Fr c = fr_pack(f9_cond_sub(w));
        // balanced digits: the bytes of c + 0x8080..80, each less 128
        uint64_t cy = 0;
        uint8_t* dst = stage + (tid >> 5) * 1024 + h * 512 + b;
#pragma unroll
        for (int l = 0; l < 8; ++l) {
            cy += (uint64_t)c.v[l] + 0x80808080u;
            const uint32_t x = (uint32_t)cy ^ 0x80808080u;
            cy >>= 32;
#pragma unroll
            for (int i = 0; i < 4; ++i) dst[(4 * l + i) * 16] = (uint8_t)(x >> (8 * i));
        }
    }
    __syncthreads();
    const uint64_t blk0 = (uint64_t)blockIdx.x * 8;
    for (int i = tid; i < 512; i += 256)
        if (blk0 + (i >> 6) < a.NB) a.wd[((uint64_t)e * (a.NB + 1) + blk0) * 64 + i] = ((const v4i*)stage)[i];
    if (blockIdx.x == 0 && tid < 64) a.wd[((uint64_t)e * (a.NB + 1) + a.NB) * 64 + tid] = v4i{0, 0, 0, 0};
}

// ---- the contractions on the matrix cores --------------------------------------------------------
// A block takes four tasks of a chunk of rho, one per wave, and brings the operands of a batch of steps (32 values of rho
// each) to LDS while the batch before it is multiplied:
//   k_zk_gram_pairs: task (group g, block pb) = the sixteen pairs (s, s') of one 4 x 4 block of the triangle, or the
//     twelve of two diagonal blocks: eight words and one digit operand are read for sixteen products of 32 cycles;
//   k_zk_gram_values: matrix tasks (eq, digits, s) = up to four digits against four values of s, vector tasks
//     (eq, digit) as matrix tasks with the mask left out.
// One wave per SIMD holds 256 accumulators.  The pairs are bound by the matrix cores (busy 55 % of the time) and the operands'
// v_bitop3, which one wave issues between the products and not beside them (VALU 37 %); the values by the latency of a
// batch's loads (matrix cores 28 %, 2.5 TB/s, LDS 16 %).  With the operands prefetched into registers the compiler waited for all of them once
// per turn of the pipeline: 2.0 ms for the 2^23 rows of two slices.
constexpr int GP_BATCH = 8, GV_BATCH = 4;

__device__ __forceinline__ void store_tile(int* part, int n_tiles, int chunk, int tile, const v16i& acc) {
    const int lane = threadIdx.x & 63;
    v4i* out = (v4i*)part + ((uint64_t)chunk * n_tiles + tile) * 256 + lane;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v4i o = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        out[64 * q] = o;
    }
}

struct PairShared {
    v4i w[2][GP_BATCH][PS][8];           // words: [buffer][step][s][four columns]
    v4i d[2][GP_BATCH][64];              // digit operands
};

template <bool DIAG>
__device__ __forceinline__ void gram_pairs(const PrefixArgs& a, PairShared& S, int chunk, int g, int pb, uint32_t b0, uint32_t b1) {
    const int tid = threadIdx.x, lane = tid & 63;
    int I, J;                            // the two blocks of four values of s
    if (DIAG) {
        I = 2 * (pb - 28);
        J = I + 1;
    } else {
        int k = pb;
        for (I = 0; k >= 7 - I; ++I) k -= 7 - I;
        J = I + 1 + k;
    }
    uint32_t mask[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) mask[t] = 0x01010101u << (t + 4 * (lane >> 5));
    constexpr int NP = DIAG ? 12 : 16;
    v16i acc[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[i][j] = 0;
    // steps beyond the chunk's end: its last block with the zero weights
    const v4i* wd = a.wd + (uint64_t)4 * (a.NB + 1) * 64;
    const uint32_t rowq = 8u * a.G;      // quads per (block, s)
    const v4i* bits = (const v4i*)a.bits + (tid >> 3) * rowq + 8 * g + (tid & 7);
    v4i rw[GP_BATCH], rd[GP_BATCH / 4];
    auto fetch = [&](uint32_t b) {
#pragma unroll
        for (int u = 0; u < GP_BATCH; ++u) rw[u] = bits[(uint64_t)(b + u < b1 ? b + u : b1 - 1) * PS * rowq];
#pragma unroll
        for (int q = 0; q < GP_BATCH / 4; ++q) {
            const uint32_t c = b + 4 * q + (tid >> 6);
            rd[q] = wd[(uint64_t)(c < b1 ? c : a.NB) * 64 + lane];
        }
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int u = 0; u < GP_BATCH; ++u) (&S.w[buf][u][0][0])[tid] = rw[u];
#pragma unroll
        for (int q = 0; q < GP_BATCH / 4; ++q) (&S.d[buf][4 * q][0])[tid] = rd[q];
    };
    fetch(b0);
    put(0);
    __syncthreads();
    int buf = 0;
    for (uint32_t b = b0; b < b1; b += GP_BATCH, buf ^= 1) {
        const bool more = b + GP_BATCH < b1;
        if (more) fetch(b + GP_BATCH);
        const uint32_t* words = (const uint32_t*)&S.w[buf][0][0][0] + (lane & 31);
#pragma unroll 2
        for (int u = 0; u < GP_BATCH; ++u) {
            uint32_t w[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = words[(u * PS + (i < 4 ? 4 * I + i : 4 * J + i - 4)) * 32];
            const v4i d = S.d[buf][u][lane];
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                int x, y;
                if (DIAG) {
                    constexpr int PX[6] = {0, 0, 0, 1, 1, 2}, PY[6] = {1, 2, 3, 2, 3, 3};
                    x = PX[i % 6] + 4 * (i / 6);
                    y = PY[i % 6] + 4 * (i / 6);
                } else {
                    x = i >> 2;
                    y = 4 + (i & 3);
                }
                v4i v;
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t] = (int)__builtin_amdgcn_bitop3_b32(w[x], w[y], mask[t], 0x28);   // (x ^ y) & mask
                acc[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(d, v, acc[i], 0, 0, 0);
            }
        }
        if (more) put(buf ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < NP; ++i) store_tile(a.part, a.G * PAIR_TILES, chunk, (g * 32 + pb) * 16 + i, acc[i]);
}

// neighbouring blocks of the grid go to different XCDs: with a chunk per XCD (8 or 16 of them) its tasks share one L2
__global__ __launch_bounds__(256, 1) void k_zk_gram_pairs(PrefixArgs a) {
    __shared__ PairShared S;
    const int chunk = blockIdx.x % a.chunks, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t b0 = (uint32_t)chunk * a.blocks_per_chunk;
    const uint32_t b1 = b0 + a.blocks_per_chunk < a.NB ? b0 + a.blocks_per_chunk : a.NB;
    const int task = blockIdx.x / a.chunks * 4 + wave, g = task >> 5, pb = task & 31;
    // the last four blocks of pairs are the diagonal ones: all waves of a block take the same branch
    if (pb < 28) gram_pairs<false>(a, S, chunk, g, pb, b0, b1);
    else gram_pairs<true>(a, S, chunk, g, pb, b0, b1);
}

constexpr int MAT_E = 4;                 // digits of a matrix task

// A block of k_zk_gram_values: (eq, group of four digits), four of the eight sets of four values of s (half 0, 1), or
// (half 2) the vector of eq for digits 16 w .. of Z: the four waves share the rows' digits.
struct ValueShared {
    v4i v[2][GV_BATCH][MAT_E][64];       // digits: [buffer][step][digit][2 s' + lane half]
    v4i m[2][GV_BATCH][64];              // sign bytes: [2 s + lane half]
    v4i d[2][GV_BATCH][64];
};

template <bool VEC>
__device__ __forceinline__ void gram_values(const PrefixArgs& a, ValueShared& S, int chunk, int eq, int e0, int half, uint32_t b0,
                                            uint32_t b1) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nd = VEC ? a.nbZ : a.nbP;
    const uint64_t plane = (uint64_t)PS * a.P;
    // thread = (digit of the group, row and half): a digit beyond the last repeats it and is not stored
    const int ed = e0 + wave < nd ? e0 + wave : nd - 1;
    const v4i* val = (const v4i*)(a.dig + ((uint64_t)eq * (a.nbZ + a.nbP) + (VEC ? 0 : a.nbZ) + ed) * plane + (uint64_t)(lane >> 1) * a.P) + (lane & 1);
    const v4i* msk = (const v4i*)(a.nsign + (uint64_t)(lane >> 1) * a.P) + (lane & 1);
    const v4i* wd = a.wd + (uint64_t)(VEC ? 2 * eq : 2 * eq + 1) * (a.NB + 1) * 64 + lane;   // Z, G_A; A, G_Z
    constexpr int NE = VEC ? 1 : MAT_E, NS = VEC ? 1 : 4;
    v16i acc[NE][NS];
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[e][i][j] = 0;
    v4i rv[GV_BATCH], rm, rd;
    auto fetch = [&](uint32_t b) {       // wave w brings digit w of every step, sign bytes and weights of step w
#pragma unroll
        for (int u = 0; u < GV_BATCH; ++u) rv[u] = val[2 * (uint64_t)(b + u < b1 ? b + u : b1 - 1)];
        const uint32_t c = b + wave;
        rm = msk[2 * (uint64_t)(c < b1 ? c : b1 - 1)];
        rd = wd[(uint64_t)(c < b1 ? c : a.NB) * 64];
    };
    static_assert(GV_BATCH == 4 && MAT_E == 4, "a wave per step and per digit");
    auto put = [&](int buf) {
#pragma unroll
        for (int u = 0; u < GV_BATCH; ++u) S.v[buf][u][wave][lane] = rv[u];
        S.m[buf][wave][lane] = rm;
        S.d[buf][wave][lane] = rd;
    };
    fetch(b0);
    put(0);
    __syncthreads();
    const int at = 2 * (lane & 31) + (lane >> 5), h = lane >> 5;
    int buf = 0;
    for (uint32_t b = b0; b < b1; b += GV_BATCH, buf ^= 1) {
        const bool more = b + GV_BATCH < b1;
        if (more) fetch(b + GV_BATCH);
#pragma unroll
        for (int u = 0; u < GV_BATCH; ++u) {
            const v4i d = S.d[buf][u][lane];
            if (VEC) {
                acc[0][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(d, S.v[buf][u][wave][at], acc[0][0], 0, 0, 0);
            } else {
                v4i v[NE], m[NS];
#pragma unroll
                for (int e = 0; e < NE; ++e) v[e] = S.v[buf][u][e][at];
#pragma unroll
                for (int i = 0; i < NS; ++i) m[i] = S.m[buf][u][2 * (16 * half + 4 * wave + i) + h];
#pragma unroll
                for (int e = 0; e < NE; ++e)
#pragma unroll
                    for (int i = 0; i < NS; ++i)
                        acc[e][i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(d, v[e] & m[i], acc[e][i], 0, 0, 0);
            }
        }
        if (more) put(buf ^ 1);
        __syncthreads();
    }
    if (VEC) {
        if (e0 + wave < nd) store_tile(a.part_v, a.n_tiles_v, chunk, a.ns * a.nbP * PS + eq * nd + e0 + wave, acc[0][0]);
    } else {
#pragma unroll
        for (int e = 0; e < NE; ++e)
            if (e0 + e < nd) {
#pragma unroll
                for (int i = 0; i < NS; ++i)
                    store_tile(a.part_v, a.n_tiles_v, chunk, (eq * nd + e0 + e) * PS + 16 * half + 4 * wave + i, acc[e][i]);
            }
    }
}

__global__ __launch_bounds__(256, 1) void k_zk_gram_values(PrefixArgs a) {
    __shared__ ValueShared S;
    const int chunk = blockIdx.x % a.chunks_v;
    const uint32_t b0 = (uint32_t)chunk * a.blocks_per_chunk_v;
    const uint32_t b1 = b0 + a.blocks_per_chunk_v < a.NB ? b0 + a.blocks_per_chunk_v : a.NB;
    int task = blockIdx.x / a.chunks_v;
    const int ng = (a.nbP + MAT_E - 1) / MAT_E;
    if (task < a.ns * ng * 2) {
        gram_values<false>(a, S, chunk, task / (2 * ng), task / 2 % ng * MAT_E, task & 1, b0, b1);
        return;
    }
    task -= a.ns * ng * 2;
    const int nv = (a.nbZ + MAT_E - 1) / MAT_E;
    gram_values<true>(a, S, chunk, task / nv, task % nv * MAT_E, 0, b0, b1);
}

// ---- from digit sums to field elements -----------------------------------------------------------
// r * 2^30: more than any |sum| (|digit sums| < 2^35, so |sum| < 2^284)
struct Words10 {
    uint32_t w[10];
};
__device__ __forceinline__ Words10 offset_words() {
    Words10 o;
#pragma unroll
    for (int i = 0; i < 10; ++i) o.w[i] = (i < 8 ? frc::MOD[i] << 30 : 0u) | (i >= 1 && i <= 8 ? frc::MOD[i - 1] >> 2 : 0u);
    return o;
}

// the column of this lane (lane % 32) of a tile, summed over the chunks: lanes l and l + 32 hold the digits
// 8 q + 4 (lane / 32) + i in register 4 q + i; both return the value, normal and below 1.2 r
__device__ __forceinline__ F9 tile_value(const int* part, int n_tiles, int chunks, int tile) {
    const int lane = threadIdx.x & 63, h = lane >> 5;
    int64_t y[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) y[i] = 0;
    const v4i* p = (const v4i*)part + (uint64_t)tile * 256 + lane;
    for (int c = 0; c < chunks; c += 4) {          // four chunks' loads in flight
        v4i x[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) x[u][q] = p[(uint64_t)(c + u < chunks ? c + u : c) * n_tiles * 256 + 64 * q];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (c + u < chunks) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) y[4 * q + i] += x[u][q][i];
            }
    }
    int64_t w[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t own = y[4 * q] + y[4 * q + 1] * 256 + y[4 * q + 2] * 65536 + y[4 * q + 3] * 16777216;
        const int64_t oth = (int64_t)(((uint64_t)(uint32_t)__shfl_xor((int)(own >> 32), 32, 64) << 32) |
                                      (uint32_t)__shfl_xor((int)own, 32, 64));
        w[2 * q] = h ? oth : own;
        w[2 * q + 1] = h ? own : oth;
    }
    const Words10 off = offset_words();
    uint32_t o[10];
    int64_t cy = 0;
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        cy += (i < 8 ? w[i] : 0) + (int64_t)off.w[i];
        o[i] = (uint32_t)cy;
        cy >>= 32;
    }
    F9 lo, hi = f9_zero();
#pragma unroll
    for (int l = 0; l < 9; ++l) {
        const int bit = 29 * l, k = bit >> 5, sh = bit & 31;
        lo.v[l] = (uint32_t)((((uint64_t)o[k + 1] << 32) | o[k]) >> sh) & frc::M29;
    }
    hi.v[0] = (uint32_t)((((uint64_t)o[9] << 32) | o[8]) >> 5);    // bits 261 .. 287
    // 2^261 is the Montgomery radix: hi * 2^261 = montgomery(hi, R^2)
    return f9_norm_reduce_sum(f9_add(lo, f9_mul(hi, fr_unpack(fr_const(frc::R2)))));
}

__device__ __forceinline__ void st9(uint32_t* p, const F9& x) {
#pragma unroll
    for (int l = 0; l < 9; ++l) p[l] = x.v[l];
}
__device__ __forceinline__ F9 ld9(const uint32_t* p) {
    F9 x;
#pragma unroll
    for (int l = 0; l < 9; ++l) x.v[l] = p[l];
    return x;
}

__global__ __launch_bounds__(256) void k_zk_gram_reduce(PrefixArgs a) {
    const int lane = threadIdx.x & 63;
    int job = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (job < a.G * PAIR_TILES) {
        const int g = job / PAIR_TILES, t = job % PAIR_TILES;
        if (t >= 28 * 16 && (t & 15) >= 12) return;      // unused tile of a diagonal block
        const F9 v = tile_value(a.part, a.G * PAIR_TILES, a.chunks, job);
        const int col = 32 * g + (lane & 31);
        const bool in = lane < 32 && col < a.ns * a.nbits;
        const int k = col >= a.nbits ? 1 : 0;
        F9 x = f9_zero();
        if (in) x = f9_mul(v, fr_unpack(a.bJ[col - k * a.nbits]));
        for (int q = 0; q < a.ns; ++q) {
            F9 y = x;
            if (k != q) y = f9_zero();
            const F9 s = wave_sum_lazy(y, 32);
            if (lane == 0) st9(a.N9 + ((uint64_t)(q * a.G + g) * PAIR_TILES + t) * 9, s);
        }
        return;
    }
    // a digit of the matrices or vectors: times 256^e; the next kernel adds the digits up
    job -= a.G * PAIR_TILES;
    const bool mat = job < a.ns * a.nbP * PS;
    if (!mat) job -= a.ns * a.nbP * PS;
    if (!mat && job >= a.ns * a.nbZ) return;
    const int nd = mat ? a.nbP : a.nbZ, s = job % PS, e = mat ? job / PS % nd : job % nd, eq = mat ? job / (PS * nd) : job / nd;
    Fr c = fr_zero();                    // 256^e, e <= 8
    if (e < 8) c.v[e >> 2] = 1u << (8 * (e & 3));
    else c.v[2] = 1;
    F9 v = tile_value(a.part_v, a.n_tiles_v, a.chunks_v, mat ? job : a.ns * a.nbP * PS + job);
    v = f9_mul(v, fr_unpack(fr_to_mont(c)));
    if (lane < 32)
        st9(mat ? a.M9 + ((uint64_t)((eq * nd + e) * PS + s) * PS + lane) * 9 : a.V9 + (uint64_t)((eq * nd + e) * PS + lane) * 9, v);
}

// ---- claims and the five rounds ------------------------------------------------------------------
struct PrefixRounds {
    DevState* st;
    const uint32_t* N9;
    const uint32_t* M9;
    const uint32_t* V9;
    int ns, G, nbP, nbZ;
    int chal_u[5];           // first challenge of the five points (their leading PV coordinates are u_hi)
    int chal_r, chal_v;
    uint32_t claims_off, claim0_off, rounds_off;
    Fr* chi;                 // out: PS coefficients at the five challenges
    Fr* pre;                 // out: w_e beta~(u^e_hi, v), e = Z, A, G_A, G_Z; beta~(u^I_hi, v)
};

constexpr int PR_THREADS = 1024;

__global__ __launch_bounds__(PR_THREADS) void k_zk_prefix(PrefixRounds a) {
    __shared__ uint32_t M[3][9][PS * PS];        // A, G_Z, binarity (strictly upper triangle, negated)
    __shared__ uint32_t V[2][9][PS];             // Z, G_A
    __shared__ uint32_t E[5][9][PS];             // beta~(u_hi, s), later beta~(u_[t+1:], b)
    __shared__ F9 pe[5], fac[5][4];
    __shared__ F9 part[4][5];
    __shared__ Fr c4[4];
    __shared__ TsShared S;
    __shared__ RoundShared R;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    DevState* st = a.st;
    block_ts_load(S, st);
    round_begin(R, st, 4);
    auto ld = [](const uint32_t* t, int stride, int i) {
        F9 x;
#pragma unroll
        for (int l = 0; l < 9; ++l) x.v[l] = t[l * stride + i];
        return x;
    };
    auto sto = [](uint32_t* t, int stride, int i, const F9& x) {
#pragma unroll
        for (int l = 0; l < 9; ++l) t[l * stride + i] = x.v[l];
    };
    const Fr one = fr_one();
    // tables of the two matrices and vectors (zero without the backward slice), beta~(u_hi, .)
    for (int i = tid; i < 2 * PS * PS; i += PR_THREADS) {
        const int q = i / (PS * PS), k = i % (PS * PS);
        F9 x = f9_zero();
        if (q < a.ns)
            for (int e = 0; e < a.nbP; ++e) x = f9_norm_reduce(f9_add(x, ld9(a.M9 + (uint64_t)((q * a.nbP + e) * PS * PS + k) * 9)));
        sto(&M[q][0][0], PS * PS, k, x);
    }
    if (tid < 2 * PS) {
        const int q = tid / PS, k = tid % PS;
        F9 x = f9_zero();
        if (q < a.ns)
            for (int e = 0; e < a.nbZ; ++e) x = f9_norm_reduce(f9_add(x, ld9(a.V9 + (uint64_t)((q * a.nbZ + e) * PS + k) * 9)));
        sto(&V[q][0][0], PS, k, x);
    } else if (tid >= 128 && tid < 128 + 5 * PS) {
        const int e = (tid - 128) / PS, s = (tid - 128) % PS;
        F9 x = fr_unpack(one);
        if (e == 4 || a.ns == 2 || e < 2)
            for (int q = 0; q < PV; ++q) {
                const Fr u = st->chal[a.chal_u[e] + q];
                x = f9_mul(x, fr_unpack(((s >> (PV - 1 - q)) & 1) ? u : fr_sub(one, u)));
            }
        sto(&E[e][0][0], PS, s, x);      // normal, below 2 r
    }
    __syncthreads();
    // the input claims: values of the polynomials at u_hi (only the diagonals of the matrices: one row each)
    if (wave < 4) {
        F9 x = f9_zero();
        if (lane < PS) {
            const F9 v = (wave & 1) ? ld(&M[wave >> 1][0][0], PS * PS, lane * (PS + 1)) : ld(&V[wave >> 1][0][0], PS, lane);
            x = f9_norm_reduce(f9_mul(ld(&E[wave][0][0], PS, lane), v));
        }
        const F9 s = wave_sum_lazy(x, PS);
        if (lane == 0) c4[wave] = f9_to_fr(s);
    }
    __syncthreads();
    if (tid < 4) st->scal[tid] = c4[tid];
    block_absorb_frs(S, 'c', c4, 4, (uint32_t*)(st->proof + a.claims_off));
    block_challenges(S, st, a.chal_r, 2);   // r, r': one draw
    __syncthreads();
    if (wave == 15) {                        // weights r^2, r, r' r^2, r' r and the claim, a product per lane
        const F9 r = fr_unpack(st->chal[a.chal_r]), rp = fr_unpack(st->chal[a.chal_r + 1]);
        F9 w = f9_mul(r, lane & 1 ? fr_unpack(one) : r);
        if (lane & 2) w = f9_mul(w, rp);
        w = f9_cond_sub(w);
        F9 x = f9_zero();
        if (lane < 4) {
            st->weights[lane] = fr_pack(w);
            pe[lane] = w;
            x = f9_mul(w, fr_unpack(c4[lane]));
        } else if (lane == 4) {
            st->weights[4] = fr_pack(rp);
            pe[4] = fr_unpack(one);
        }
        const F9 s = wave_sum_lazy(x, 4);
        if (lane == 0) {
            const Fr plain = f9_canonical(s);
            uint32_t* dst = (uint32_t*)(st->proof + a.claim0_off);
            for (int l = 0; l < 8; ++l) dst[l] = plain.v[l];
        }
    }
    // binarity: -(N_0 + r' N_1) above the diagonal
    for (int i = tid; i < PS * PS; i += PR_THREADS) {
        const int s = i / PS, s2 = i % PS;
        F9 x = f9_zero();
        if (s < s2) {
            const int I = s >> 2, J = s2 >> 2;
            int t;                           // tile of the pair
            if (I == J) {
                const int x4 = s & 3, y4 = s2 & 3, k = x4 == 0 ? y4 - 1 : x4 == 1 ? y4 + 1 : 5;
                t = (28 + (I >> 1)) * 16 + (I & 1) * 6 + k;
            } else {
                t = (I * 7 - I * (I - 1) / 2 + (J - I - 1)) * 16 + (s & 3) * 4 + (s2 & 3);
            }
            F9 n[2];
            for (int q = 0; q < 2; ++q) {
                n[q] = f9_zero();
                if (q < a.ns)
                    for (int g = 0; g < a.G; ++g)
                        n[q] = f9_norm_reduce(f9_add(n[q], ld9(a.N9 + ((uint64_t)(q * a.G + g) * PAIR_TILES + t) * 9)));
            }
            if (a.ns == 2) n[0] = f9_norm_reduce(f9_add(n[0], f9_mul(n[1], fr_unpack(st->chal[a.chal_r + 1]))));
            x = f9_norm_reduce(f9_sub(f9_zero(), n[0]));
        }
        sto(&M[2][0][0], PS * PS, i, x);
    }
    // beta~(u_[1:], b): the leading variable summed out
    if (tid >= 512 && tid < 512 + 5 * PS / 2) {
        const int e = (tid - 512) / (PS / 2), b = (tid - 512) % (PS / 2);
        sto(&E[e][0][0], PS, b, f9_norm_reduce(f9_add(ld(&E[e][0][0], PS, b), ld(&E[e][0][0], PS, b + PS / 2))));
    }
    __syncthreads();

    F9 v = f9_zero(), pe9 = f9_zero(), chi9 = fr_unpack(one);
    int n = PS;                              // values of the variables that are still open
    for (int t = 0; t < PV; ++t) {
        if (t > 0) {
            // bind v_{t-1}: rows and columns in one pass in place (an entry comes from four that no other one comes
            // from); vectors, weights and factors beside them
            const int h = n >> 1;
            for (int i = tid; i < 3 * h * h; i += PR_THREADS) {
                const int q = i / (h * h), k = i % (h * h), c0 = (k / h) * PS + k % h;
                const uint32_t* m = &M[q][0][0];
                const F9 m0 = ld(m, PS * PS, c0), m1 = ld(m, PS * PS, c0 + h), m2 = ld(m, PS * PS, c0 + h * PS), m3 = ld(m, PS * PS, c0 + h * PS + h);
                const F9 lo = f9_norm_reduce(f9_add(m0, f9_mul(f9_sub(m2, m0), v))), hi = f9_norm_reduce(f9_add(m1, f9_mul(f9_sub(m3, m1), v)));
                sto(&M[q][0][0], PS * PS, c0, f9_norm_reduce(f9_add(lo, f9_mul(f9_sub(hi, lo), v))));
            }
            if (wave == 13 && lane < 2 * h) {
                const int q = lane / h, b = lane % h;
                const F9 lo = ld(&V[q][0][0], PS, b), hi = ld(&V[q][0][0], PS, b + h);
                sto(&V[q][0][0], PS, b, f9_norm_reduce(f9_add(lo, f9_mul(f9_sub(hi, lo), v))));
            }
            if (wave == 14) {                // n / 4 weights remain of the n / 2 used in the round before
                const int q4 = n >> 2;
                for (int i = lane; i < 5 * q4; i += 64) {
                    const int e = i / q4, b = i % q4;
                    sto(&E[e][0][0], PS, b, f9_norm_reduce(f9_add(ld(&E[e][0][0], PS, b), ld(&E[e][0][0], PS, b + q4))));
                }
            }
            n = h;
        }
        // p_e, the bound factors of beta~(u_hi, X), times the line (1 - u)(1 - x) + u x at x = 0 .. 3: 1 - u, u, 3 u - 1,
        // 5 u - 2
        if (wave == 15 && lane < 20) {
            const int e = lane >> 2, x = lane & 3;
            const Fr u = st->chal[a.chal_u[e] + t], u2 = fr_add(u, u);
            const Fr l = x == 0 ? fr_sub(one, u) : x == 1 ? u : x == 2 ? fr_sub(fr_add(u2, u), one)
                                                                      : fr_sub(fr_add(fr_add(u2, u2), u), fr_add(one, one));
            if (t > 0) {                     // (1 - u) + v (2 u - 1) of the variable before
                const Fr w = st->chal[a.chal_u[e] + t - 1], l0 = fr_sub(one, w);
                pe9 = f9_mul(pe9, f9_norm(f9_add(fr_unpack(l0), f9_mul(fr_unpack(fr_sub(w, l0)), v))));
            } else {
                pe9 = pe[e];
            }
            fac[e][x] = f9_mul(pe9, fr_unpack(l));
            if (x == 0) pe[e] = pe9;
        }
        // coefficients of the rows at the challenges so far
        if (wave == 12 && lane < PS && t > 0) chi9 = f9_mul(chi9, (lane >> (PV - t)) & 1 ? v : f9_norm_reduce(f9_sub(fr_unpack(one), v)));
        __syncthreads();
        const int h = n >> 1;
        uint32_t* proof_dst = (uint32_t*)(st->proof + a.rounds_off + 128u * (uint32_t)t);
        // row of 16 lanes = (equation, point): sum over the boolean rest b < h <= 16
        if (wave < 5) {
            const int combo = tid >> 4, e = combo >> 2, xi = combo & 3, b = tid & 15;
            F9 x = f9_zero();
            if (b < h) {
                F9 y;
                if (e == 0 || e == 2) {
                    const F9 lo = ld(&V[e >> 1][0][0], PS, b), hi = ld(&V[e >> 1][0][0], PS, b + h);
                    y = xi == 0 ? lo : hi;
                    if (xi >= 2) {           // hi + (x - 1)(hi - lo)
                        const F9 d = f9_norm(f9_sub(hi, lo));
                        y = f9_add(hi, d);
                        if (xi == 3) y = f9_add(y, d);
                        y = f9_norm_reduce(y);
                    }
                } else {
                    const uint32_t* m = &M[e == 4 ? 2 : e >> 1][0][0];
                    const F9 m00 = ld(m, PS * PS, b * PS + b);
                    y = m00;
                    if (xi == 1) {
                        y = ld(m, PS * PS, (b + h) * PS + b + h);
                    } else if (xi) {
                        const F9 m11 = ld(m, PS * PS, (b + h) * PS + b + h);
                        const F9 cr = f9_add(ld(m, PS * PS, b * PS + b + h), ld(m, PS * PS, (b + h) * PS + b));
                        const F9 c2 = f9_norm_reduce(f9_add(cr, cr)), d4 = f9_norm_reduce(f9_add(f9_add(m11, m11), f9_add(m11, m11)));
                        if (xi == 2) {       // M00 - 2 cr + 4 M11
                            y = f9_norm_reduce(f9_add(m00, f9_sub(d4, c2)));
                        } else {             // 4 M00 - 6 cr + 9 M11
                            const F9 a4 = f9_norm_reduce(f9_add(f9_add(m00, m00), f9_add(m00, m00)));
                            const F9 c6 = f9_norm_reduce(f9_add(f9_add(c2, c2), c2));
                            y = f9_norm_reduce(f9_add(f9_add(a4, d4), f9_add(d4, f9_sub(m11, c6))));   // below 13.7 r before
                        }
                    }
                }
                x = f9_norm_reduce(f9_mul(y, ld(&E[e][0][0], PS, b)));
            }
            const F9 s = wave_sum_lazy(x, 16);   // DPP within each row of 16: every row its own sum
            if (b == 0) part[xi][e] = f9_mul(s, fac[e][xi]);
        }
        __syncthreads();
        if (wave < 4 && lane == 0) {
            F9 s = part[wave][0];
#pragma unroll
            for (int e = 1; e < 5; ++e) s = f9_add(s, part[wave][e]);
            round_eval_out(S, R, proof_dst, wave, f9_norm_reduce(s), true);
        }
        v = block_close_round(S, R, st, 4, false, a.rounds_off + 128u * (uint32_t)t, a.chal_v + t);
    }
    round_end(R, st, 4, a.chal_v + PV - 1);
    // coefficients of the 32 rows and factors of the equality tables at the five challenges
    if (wave == 12 && lane < PS) {
        chi9 = f9_mul(chi9, lane & 1 ? v : f9_norm_reduce(f9_sub(fr_unpack(one), v)));
        a.chi[lane] = fr_pack(f9_cond_sub(chi9));
    } else if (wave == 13 && lane < 5) {
        const Fr u = st->chal[a.chal_u[lane] + PV - 1], l0 = fr_sub(one, u);
        a.pre[lane] = f9_to_fr(f9_mul(pe[lane], f9_norm(f9_add(fr_unpack(l0), f9_mul(fr_unpack(fr_sub(u, l0)), v)))));
    }
    block_ts_store(S, st);
}

// ---- the five challenges bound -------------------------------------------------------------------
// Tables of the linear equations and beta_I, P entries each.  Values: sum_s chi_s x_s with x_s shifted to be
// non-negative, x_s + 2^(bits - 1): sum_s chi_s = 1, so the shift is subtracted once.
struct BindArgs {
    PrefixArgs p;
    const Fr* chi;
    const Fr* pre;
    F9Tab val[5];            // Z, Z', 1 - sign, G_A, G_A'
    F9Tab eq[5];             // Z, A, G_A, G_Z, I
};

__device__ __forceinline__ void mac3(uint64_t* cols, const F9& c, uint64_t x, bool wide) {
    const uint32_t m0 = (uint32_t)x & frc::M29, m1 = (uint32_t)(x >> 29) & frc::M29, m2 = (uint32_t)(x >> 58);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        cols[i] += (uint64_t)c.v[i] * m0;
        cols[i + 1] += (uint64_t)c.v[i] * m1;
        if (wide) cols[i + 2] += (uint64_t)c.v[i] * m2;
    }
}

// carried 11-column sum (columns 0..9 below 2^29) less 2^k, normal and below 2.41 r
__device__ __forceinline__ F9 bound_value(uint64_t* cols, int k) {
    cols11_carry(cols);
    Fr sh = fr_zero();
    sh.v[k >> 5] = 1u << (k & 31);
    const F9 s = f9_mul(fr_unpack(sh), fr_unpack(fr_const(frc::R2)));    // Montgomery form of 2^k
    return f9_norm_reduce(f9_sub(cols11_value(cols), f9_cond_sub(s)));
}

constexpr int BIND_ROWS = 128;           // threads per block: small ones, so that 2^14 entries reach every compute unit
template <bool WIDE>
__global__ __launch_bounds__(BIND_ROWS) void k_zk_bind(BindArgs a) {
    __shared__ F9 chi[PS], pre[5];
    const int tid = threadIdx.x;
    if (tid < PS) chi[tid] = fr_unpack(a.chi[tid]);
    else if (tid >= 64 && tid < 69) pre[tid - 64] = fr_unpack(a.pre[tid - 64]);
    __syncthreads();
    const PrefixArgs& p = a.p;
    const uint64_t rho = (uint64_t)blockIdx.x * BIND_ROWS + tid;
    if (rho >= p.P) return;
    const int role = blockIdx.y;         // an equality table, or the values of a slice
    if (role < 5) {
        const int e = role;
        if (p.ns == 1 && (e == 2 || e == 3)) return;
        const uint64_t hi = rho >> p.lb, lo = rho & (((uint64_t)1 << p.lb) - 1);
        const F9 w = f9_mul(f9_mul(fr_unpack(tab_ld(p.H[e], hi)), fr_unpack(tab_ld(p.L[e], lo))), pre[e]);
        f9tab_st(a.eq[e], rho, w);
        return;
    }
    const int k = role - 5;
    {
        const int64_t* src = k ? p.ga : p.z;
        uint64_t c0[12], c1[12], cs[9];
#pragma unroll
        for (int i = 0; i < 12; ++i) c0[i] = c1[i] = 0;
#pragma unroll
        for (int i = 0; i < 9; ++i) cs[i] = 0;
        const uint64_t offz = (uint64_t)1 << (p.nbits - 1), offq = (uint64_t)1 << (p.q_bits - 1);
        int64_t x = src[rho];
#pragma unroll 1
        for (int s = 0; s < PS; ++s) {
            const int64_t nx = src[(uint64_t)(s + 1 < PS ? s + 1 : s) * p.P + rho];
            const F9 c = chi[s];
            mac3(c0, c, (uint64_t)x + offz, WIDE);
            mac3(c1, c, (uint64_t)rescale_half_up(x, p.r_bits) + offq, WIDE);
            const uint64_t keep = ((x >> (p.nbits - 1)) & 1) ? 0 : ~(uint64_t)0;
#pragma unroll
            for (int i = 0; i < 9; ++i) cs[i] += c.v[i] & keep;
            if ((s & 3) == 3) {          // four products of 2^58 and less per column and limb of x
#pragma unroll
                for (int i = 0; i + 1 < 12; ++i) {
                    c0[i + 1] += c0[i] >> 29;
                    c0[i] &= frc::M29;
                    c1[i + 1] += c1[i] >> 29;
                    c1[i] &= frc::M29;
                }
            }
            x = nx;
        }
        // column 11 is empty without the third limb, and below 2^11 with it: the sums are below 2^(255 + 5 + 64)
        c0[10] += c0[11] << 29;
        c1[10] += c1[11] << 29;
        f9tab_st(a.val[k ? 3 : 0], rho, bound_value(c0, p.nbits - 1));
        f9tab_st(a.val[k ? 4 : 1], rho, bound_value(c1, p.q_bits - 1));
        if (k == 0) {
            F9 ns;
            uint64_t cy = 0;
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                cy += cs[i];
                ns.v[i] = i < 8 ? (uint32_t)cy & frc::M29 : (uint32_t)cy;
                cy >>= 29;
            }
            f9tab_st(a.val[2], rho, f9_norm_reduce_sum(ns));   // at most 32 values below r
        }
    }
}

}  // namespace

// Lays out and launches the pass; see the declaration in zkdl_internal.h
int zk_prefix_rounds(zkdl_ctx* ctx, const ZkPrefixJob& j) {
    PrefixArgs a = {};
    a.z = j.z;
    a.ga = j.ga;
    a.P = j.D >> PV;
    a.NB = (uint32_t)(a.P >> 5);
    a.nbits = j.q_bits + j.r_bits;
    a.r_bits = j.r_bits;
    a.q_bits = j.q_bits;
    a.ns = j.ga ? 2 : 1;
    a.G = (a.ns * a.nbits + 31) / 32;
    a.nbZ = a.nbits / 8 + 1;             // signed digits of a nbits-bit value
    a.nbP = (j.q_bits + 1) / 8 + 1;      // |Z'| <= 2^(Q-1), the bound included
    // A block per compute unit.  A chunk of at most 4095 blocks of rho keeps the sums below 2^31 (32 products of at
    // most 2^14 per block).
    auto cut = [&](unsigned blocks, int* chunks, uint32_t* per) {
        uint32_t c = 256u / blocks;
        if (c < (a.NB + 4094) / 4095) c = (a.NB + 4094) / 4095;
        if (c < 1) c = 1;
        if (c > a.NB) c = a.NB;
        *per = (a.NB + c - 1) / c;
        *chunks = (int)((a.NB + *per - 1) / *per);
    };
    const int ng = (a.nbP + MAT_E - 1) / MAT_E, nv = (a.nbZ + MAT_E - 1) / MAT_E;
    const unsigned pair_blocks = (unsigned)a.G * 8, value_blocks = (unsigned)(a.ns * (2 * ng + nv));
    cut(pair_blocks, &a.chunks, &a.blocks_per_chunk);
    cut(value_blocks, &a.chunks_v, &a.blocks_per_chunk_v);
    a.n_tiles_v = a.ns * (a.nbP * PS + a.nbZ);
    const size_t b_bits = (size_t)PS * a.NB * 32 * a.G * 4, b_dig = (size_t)a.ns * (a.nbZ + a.nbP) * j.D, b_ns = j.D;
    const size_t b_wd = (size_t)5 * (a.NB + 1) * 1024, b_part = (size_t)a.chunks * a.G * PAIR_TILES * 4096,
                 b_part_v = (size_t)a.chunks_v * a.n_tiles_v * 4096;
    const size_t b_n9 = (size_t)a.ns * a.G * PAIR_TILES * 36, b_m9 = (size_t)a.ns * a.nbP * PS * PS * 36, b_v9 = (size_t)a.ns * a.nbZ * PS * 36;
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    uint8_t* mem = (uint8_t*)zk_alloc(ctx, up(b_bits) + up(b_dig) + up(b_ns) + up(b_wd) + up(b_part) + up(b_part_v) + up(b_n9) + up(b_m9) + up(b_v9) + 64 * 32);
    if (!mem) return ZKDL_ENOMEM;
    uint8_t* q = mem;
    a.bits = (uint32_t*)q;
    q += up(b_bits);
    a.dig = (int8_t*)q;
    q += up(b_dig);
    a.nsign = q;
    q += up(b_ns);
    a.wd = (v4i*)q;
    q += up(b_wd);
    a.part = (int*)q;
    q += up(b_part);
    a.part_v = (int*)q;
    q += up(b_part_v);
    a.N9 = (uint32_t*)q;
    q += up(b_n9);
    a.M9 = (uint32_t*)q;
    q += up(b_m9);
    a.V9 = (uint32_t*)q;
    q += up(b_v9);
    Fr* chi = (Fr*)q;
    for (int e = 0; e < 5; ++e) {
        a.H[e] = j.H[e];
        a.L[e] = j.L[e];
    }
    a.lb = j.lb;
    a.bJ = j.bJ;
    a.st = ctx->dev;
    hipLaunchKernelGGL(k_zk_planes, dim3((unsigned)((a.P + PL_ROWS - 1) / PL_ROWS), PS), dim3(256), 0, ctx->stream, a);
    hipLaunchKernelGGL(k_zk_weight_digits, dim3((unsigned)((a.P + 255) / 256), 5), dim3(256), 0, ctx->stream, a);
    zk_prof_begin(ctx, ZKDL_PROF_ZK_BIN, 8.0 * a.ns * (double)j.D);   // the integers, read once
    hipLaunchKernelGGL(k_zk_gram_pairs, dim3(pair_blocks * (unsigned)a.chunks), dim3(256), 0, ctx->stream, a);
    zk_prof_end(ctx);
    hipLaunchKernelGGL(k_zk_gram_values, dim3(value_blocks * (unsigned)a.chunks_v), dim3(256), 0, ctx->stream, a);
    const unsigned jobs = (unsigned)(a.G * PAIR_TILES + a.ns * a.nbP * PS + a.ns * a.nbZ);
    hipLaunchKernelGGL(k_zk_gram_reduce, dim3((jobs + 3) / 4), dim3(256), 0, ctx->stream, a);
    PrefixRounds pr = {};
    pr.st = ctx->dev;
    pr.N9 = a.N9;
    pr.M9 = a.M9;
    pr.V9 = a.V9;
    pr.ns = a.ns;
    pr.G = a.G;
    pr.nbP = a.nbP;
    pr.nbZ = a.nbZ;
    for (int e = 0; e < 5; ++e) pr.chal_u[e] = j.chal_u[e];
    pr.chal_r = j.chal_r;
    pr.chal_v = j.chal_v;
    pr.claims_off = j.claims_off;
    pr.claim0_off = j.claim0_off;
    pr.rounds_off = j.rounds_off;
    pr.chi = chi;
    pr.pre = chi + PS;
    hipLaunchKernelGGL(k_zk_prefix, dim3(1), dim3(PR_THREADS), 0, ctx->stream, pr);
    BindArgs b = {};
    b.p = a;
    b.chi = chi;
    b.pre = chi + PS;
    for (int e = 0; e < 5; ++e) {
        b.val[e] = j.val[e];
        b.eq[e] = j.eq[e];
    }
    zk_prof_begin(ctx, ZKDL_PROF_ZK_LIN, 8.0 * a.ns * (double)j.D + (a.ns == 2 ? 10.0 : 6.0) * 32.0 * (double)a.P);
    const dim3 bind_grid((unsigned)((a.P + BIND_ROWS - 1) / BIND_ROWS), 5 + a.ns);
    // the third limb of a shifted value exists above 58 bits
    if (a.nbits > 58) hipLaunchKernelGGL(k_zk_bind<true>, bind_grid, dim3(BIND_ROWS), 0, ctx->stream, b);
    else hipLaunchKernelGGL(k_zk_bind<false>, bind_grid, dim3(BIND_ROWS), 0, ctx->stream, b);
    zk_prof_end(ctx);
    zk_free(ctx, mem);       // the block is handed out again in stream order
    return ZKDL_OK;
}
