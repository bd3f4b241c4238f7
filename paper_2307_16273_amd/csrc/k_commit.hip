// Pedersen commitments on G1 of BLS12-381 and the row-wise commitment of a tensor (Sec. 2.3; Sec. 1.1;
// Protocol zkdl, the commit and proof-of-evaluation lines).
//
//   Commit(S; rho) = rho H + sum_i S_i G_i                                   (Sec. 2.3, additive notation)
//
// A tensor of 2^m quantised integers is laid out as R = 2^ceil(m/2) rows of C = 2^floor(m/2) columns and
// every row is committed with the same C generators and its own blinding scalar: the commitment has
// R = O(sqrt(size)) group elements (Sec. 1.1).  Generators are derived from a label by hashing to the
// curve (try-and-increment on SHA-256, cofactor cleared), so nobody knows a relation between them.
//
// Scalars are small: tensors are 32-bit (activations, weights, gradients) or 64-bit (pre-activations)
// signed integers, a negative entry x being the field element r - |x|, i.e. -|x| G.  The sum therefore
// runs over fixed-base window tables: |x| is written in signed digits, for every generator and window the multiples d 2^shift G,
// d = 1 .. half the window's range, are built once with the key, in affine form (112 bytes an entry), and a commitment is a plain
// sum of one table entry or its negative per non-zero digit - no doublings and no buckets.  The windows are unequal (CkWindows): a wide one
// for the bits that every weight has, narrow ones for those that few have; keys that are too wide for that take narrow windows throughout.
// The blinding term rho H (rho a full field element) uses the same kind of table with 32 windows.  All sums use the complete projective formulas of fq.cuh: a row's sum may be
// taken in any order.
#include <string.h>
#include <new>
#include <vector>

#include "dev_common.cuh"
#include "fq.cuh"

namespace {

constexpr int CK_WBITS = 8;                      // bits per window of the blinding scalar's table
constexpr int CK_DIGITS = (1 << CK_WBITS) - 1;   // its entries per window: d = 1..255
constexpr int CK_H_WINDOWS = 256 / CK_WBITS;     // windows of a 255-bit blinding scalar
constexpr uint64_t CK_WIDE_MAX_BYTES = (uint64_t)12 << 30;   // wide windows up to 8192 columns of 32-bit entries (8.5 GB)
constexpr int CK_MAX_LABEL = 16;

// Windows of a tensor entry, from the lowest bits up: bits each, summing to the entry's width.  A digit of a window of w bits is
// between -2^(w-1) and 2^(w-1), the top one (what is left with its carry) between 0 and 2^(w-1): |x| is at most 2^(width - 1).
// With n windows |x| up to 2^(bits - 1) has n digits or fewer.  Wide: a table of 9280 entries a column of 32-bit entries, 19460 of 64-bit.
// The lowest window decides what a weight costs: of 2^23 normal values with sigma 2900 each has 1.00 digits, with unsigned digits of
// 12 bits 1.16 (from tables of 12285 and 24570 entries).  The other windows are such that no |x| has more digits than it has unsigned
// ones of 12 bits (ck_no_longer).  64-bit windows of 14, 14, 10, 11, 11 and 4 bits did not keep to that above 2^59, and their tables lay
// closer to 2 MB apart; commitments of 2^20 entries, us, unsigned digits / those windows / these: sigma 2^25 719 / 620 / 604, 2^42
// 943 / 955 / 906, 2^58 1109 / 1135 / 1064, 2^60 1169 / 1239 / 1123.
// Narrow: likewise for unsigned digits of 8 bits (576 and 1088 entries instead of 1020 and 2040).
template <int BITS, bool WIDE>
struct CkWindows;
template <>
struct CkWindows<32, true> {
    static constexpr int N = 3, W[N] = {14, 11, 7};
};
template <>
struct CkWindows<64, true> {
    static constexpr int N = 6, W[N] = {14, 14, 11, 11, 11, 3};
};
template <>
struct CkWindows<32, false> {
    static constexpr int N = 4, W[N] = {9, 8, 8, 7};
};
template <>
struct CkWindows<64, false> {
    static constexpr int N = 8, W[N] = {9, 8, 8, 8, 8, 8, 8, 7};
};
template <class C>
constexpr int ck_entries(int k = C::N) {      // table entries of the windows below k
    int n = 0;
    for (int i = 0; i < k; ++i) n += 1 << (C::W[i] - 1);
    return n;
}
template <class C>
constexpr int ck_shift(int k) {
    int n = 0;
    for (int i = 0; i < k; ++i) n += C::W[i];
    return n;
}
static_assert(ck_entries<CkWindows<64, true>>() <= 1 << 15 && ck_entries<CkWindows<32, true>>() <= 1 << 15, "a queued digit has 15 bits");
static_assert(ck_shift<CkWindows<32, true>>(3) == 32 && ck_shift<CkWindows<64, true>>(6) == 64 &&
              ck_shift<CkWindows<32, false>>(4) == 32 && ck_shift<CkWindows<64, false>>(8) == 64, "windows cover the entry");

// what fits n unsigned digits of `bits` bits fits n windows
template <class C>
constexpr bool ck_no_longer(int bits) {
    for (int n = 1; n < C::N; ++n)
        if (ck_shift<C>(n) - 1 < bits * n) return false;
    return true;
}
static_assert(ck_no_longer<CkWindows<32, true>>(12) && ck_no_longer<CkWindows<64, true>>(12) && ck_no_longer<CkWindows<32, false>>(8) &&
              ck_no_longer<CkWindows<64, false>>(8), "no entry takes more additions than with unsigned digits");

// the windows of a table as the kernel that builds it takes them
struct CkLayout {
    int windows;
    int shift[CK_H_WINDOWS];
    uint32_t first[CK_H_WINDOWS + 1];       // entries of the windows below, all of them at the end
    uint32_t chunks[CK_H_WINDOWS + 1];      // the same of their chunks of CK_CHUNK entries
};

struct LabelArg {
    uint8_t bytes[15 + CK_MAX_LABEL];   // "zkdl-mi355x/g1/" followed by the label
    uint32_t len;
};

// 2^384 * 2^812 mod q: brings the top 128 bits of a 512-bit hash into Montgomery form
// (fq_mul(hi, R2X) = hi 2^384 R mod q); checked against repeated doubling in zk_commit_selfcheck
__device__ __host__ inline Fq r2x_const() {
    Fq c = fq_const(fqc::R2);
    for (int i = 0; i < 384; ++i) c = fq_add(c, c);
    return c;
}

__device__ inline void sha_one_block(const uint8_t* msg, uint32_t len, uint32_t out[8]) {   // len <= 55
    uint32_t w[16];
    for (int i = 0; i < 16; ++i) w[i] = 0;
    for (uint32_t i = 0; i < len; ++i) w[i >> 2] |= (uint32_t)msg[i] << (24 - 8 * (i & 3));
    w[len >> 2] |= 0x80u << (24 - 8 * (len & 3));
    w[15] = len * 8;
    uint32_t h[8] = {0x6a09e667u, 0xbb67ae85u, 0x3c6ef372u, 0xa54ff53au, 0x510e527fu, 0x9b05688cu, 0x1f83d9abu, 0x5be0cd19u};
    sha::compress(h, w);
    for (int i = 0; i < 8; ++i) out[i] = h[i];
}

// plain a < plain b ?  (both below q, plain limbs)
__device__ inline bool limbs_less(const Fq& a, const Fq& b) {
    for (int i = fqc::L - 1; i >= 0; --i) {
        if (a.v[i] != b.v[i]) return a.v[i] < b.v[i];
    }
    return false;
}

// Generator `index` of the label: for ctr = 0, 1, .. the candidate x = int_be(SHA256(tag || u32be(index) ||
// u32be(ctr) || 0) || SHA256(.. || 1)) mod q; the first x for which x^3 + 4 is a square gives (x, y) with the
// smaller root y; cleared of the cofactor; a candidate that becomes the identity is skipped.
__global__ __launch_bounds__(64) void k_ck_generators(LabelArg label, uint64_t ncols, G1* gens, Fq r2x) {
    const uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (i > ncols) return;
    const uint32_t index = i < ncols ? (uint32_t)i : 0xFFFFFFFFu;   // the last one is the blinding generator H
    uint8_t msg[56];
    for (uint32_t b = 0; b < label.len; ++b) msg[b] = label.bytes[b];
    uint32_t at = label.len;
    for (int b = 0; b < 4; ++b) msg[at + b] = (uint8_t)(index >> (24 - 8 * b));
    at += 8;
    Fq four = fq_add(fq_one(), fq_one());
    four = fq_add(four, four);
    for (uint32_t ctr = 0;; ++ctr) {
        for (int b = 0; b < 4; ++b) msg[at - 4 + b] = (uint8_t)(ctr >> (24 - 8 * b));
        uint32_t dg[16];
        msg[at] = 0;
        sha_one_block(msg, at + 1, dg);
        msg[at] = 1;
        sha_one_block(msg, at + 1, dg + 8);
        // the 64 digest bytes as a big-endian integer: little-endian byte k is byte 63 - k of the digests
        uint8_t le[64];
        for (int k = 0; k < 64; ++k) {
            const int pos = 63 - k;
            le[k] = (uint8_t)(dg[pos >> 2] >> (24 - 8 * (pos & 3)));
        }
        uint8_t hi48[48];
        for (int k = 0; k < 48; ++k) hi48[k] = k < 16 ? le[48 + k] : 0;
        const Fq x = fq_add(fq_reduce_to_mont(fq_limbs_from_bytes(le)), fq_mul(fq_limbs_from_bytes(hi48), r2x));
        const Fq rhs = fq_add(fq_mul(fq_sqr(x), x), four);
        Fq y = fq_pow(rhs, fqc::EXP_SQRT);
        if (!fq_eq(fq_sqr(y), rhs)) continue;
        const Fq yn = fq_neg(y);
        if (limbs_less(fq_from_mont(yn), fq_from_mont(y))) y = yn;
        G1 p;
        p.X = x;
        p.Y = y;
        p.Z = fq_one();
        p = g1_mul_words(p, fqc::COFACTOR);
        if (fq_is_zero(p.Z)) continue;
        gens[i] = p;
        return;
    }
}

// One copy of the 406-multiply-add field product for the kernels that add points in a loop.  Its operands go in and
// out as vectors: of two structs of fourteen words the calling convention puts the second one in scratch memory, whose
// stores and loads every product then waited for.
typedef uint32_t FqV __attribute__((ext_vector_type(16)));
__device__ __forceinline__ FqV fqv_from(const Fq& a) {
    FqV o;
#pragma unroll
    for (int i = 0; i < fqc::L; ++i) o[i] = a.v[i];
    o[14] = o[15] = 0;
    return o;
}
__device__ __forceinline__ Fq fqv_to(const FqV& a) {
    Fq o;
#pragma unroll
    for (int i = 0; i < fqc::L; ++i) o.v[i] = a[i];
    return o;
}
__device__ __noinline__ FqV fq_mul_v(FqV a, FqV b) { return fqv_from(fq_mul(fqv_to(a), fqv_to(b))); }
__device__ __forceinline__ Fq fq_mul_ni(const Fq& a, const Fq& b) { return fqv_to(fq_mul_v(fqv_from(a), fqv_from(b))); }
struct FqMulOutOfLine {
    __device__ Fq operator()(const Fq& a, const Fq& b) const { return fq_mul_ni(a, b); }
};

struct G1A {   // affine, never the identity
    Fq x, y;
};
constexpr int CK_CHUNK = 16;   // table entries per thread of k_ck_tables

static void ck_layout_add(CkLayout* l, int shift, uint32_t entries) {
    const int k = l->windows++;
    l->shift[k] = shift;
    l->first[k + 1] = l->first[k] + entries;
    l->chunks[k + 1] = l->chunks[k] + (entries + CK_CHUNK - 1) / CK_CHUNK;
}
template <class C>
static CkLayout ck_layout() {
    CkLayout l = {};
    for (int k = 0; k < C::N; ++k) ck_layout_add(&l, ck_shift<C>(k), 1u << (C::W[k] - 1));
    return l;
}

// table[g * l.first[l.windows] + l.first[k] + d - 1] = d 2^shift_k gens[g], affine.  One thread per
// (g, k, 16 digits): the window's base by doublings, the first digit times the base by double-and-add, then one addition and one
// inversion per entry.
__global__ __launch_bounds__(64) void k_ck_tables(const G1* gens, uint64_t ngens, CkLayout l, G1A* table) {
    const uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    const uint32_t per = l.chunks[l.windows];
    const uint64_t g = t / per;
    const uint32_t chunk = (uint32_t)(t % per);
    if (g >= ngens) return;
    int k = 0;
    while (chunk >= l.chunks[k + 1]) ++k;
    const FqMulOutOfLine mul;
    G1 base = gens[g];
#pragma unroll 1
    for (int s = 0; s < l.shift[k]; ++s) base = g1_dbl_with(base, mul);
    const uint32_t first = CK_CHUNK * (chunk - l.chunks[k]) + 1, entries = l.first[k + 1] - l.first[k];
    G1 acc = g1_identity();
#pragma unroll 1
    for (int bit = 31 - __clz((int)first); bit >= 0; --bit) {
        acc = g1_dbl_with(acc, mul);
        if ((first >> bit) & 1) acc = g1_add_with(acc, base, mul);
    }
    G1A* out = table + g * (uint64_t)l.first[l.windows] + l.first[k];
#pragma unroll 1
    for (uint32_t d = first; d < first + CK_CHUNK && d <= entries; ++d) {   // acc = d base
        const Fq zi = fq_inv_steps(acc.Z);
        G1A e;
        e.x = fq_mul_ni(acc.X, zi);
        e.y = fq_mul_ni(acc.Y, zi);
        out[d - 1] = e;
        acc = g1_add_with(acc, base, mul);
    }
}

// the product without its conditional subtraction, for the additions without reductions (coordinates below 6q)
__device__ __noinline__ FqV fq_mul_lazy_v(FqV a, FqV b) { return fqv_from(fq_mul_t<false>(fqv_to(a), fqv_to(b))); }
__device__ __forceinline__ Fq fq_mul_lazy_ni(const Fq& a, const Fq& b) {
    return fqv_to(fq_mul_lazy_v(fqv_from(a), fqv_from(b)));
}
struct FqMulLazyOutOfLine {
    __device__ Fq operator()(const Fq& a, const Fq& b) const { return fq_mul_lazy_ni(a, b); }
};
__device__ inline G1 g1_add_lazy_ni(const G1& p, const G1& q) { return g1_add_lazy_with(p, q, FqMulLazyOutOfLine()); }
__device__ inline G1 g1_add_mixed_lazy(const G1& p, const Fq& x2, const Fq& y2) {
    return g1_add_mixed_lazy_with(p, x2, y2, FqMulLazyInline());   // 40 KB of code in the loop: calls cost 4 %
}

__device__ inline G1 g1_shfl_down(const G1& p, int off) {
    G1 q;
#pragma unroll
    for (int i = 0; i < fqc::L; ++i) {
        q.X.v[i] = __shfl_down(p.X.v[i], off, 64);
        q.Y.v[i] = __shfl_down(p.Y.v[i], off, 64);
        q.Z.v[i] = __shfl_down(p.Z.v[i], off, 64);
    }
    return q;
}

constexpr uint32_t CK_QUEUE = 1024;   // ring of digits waiting for a lane: at most 63 left over + 64 x 8 new ones

// One wave per row: sums[row] = rho_row H + sum_c x[row, c] G_c (projective).  The wave reads 64 entries at a time and
// puts their non-zero digits (table entry, sign, column: one word) on a ring in LDS, window by window with
// a ballot and a prefix count; whenever 64 digits wait, every lane takes one and adds its table entry.  Lanes
// therefore never wait for each other's zero digits or shorter entries: a row of n digits costs ceil(n / 64)
// additions per lane.  Lane k < 32 also starts from window k of the blinding scalar.  The 64 partial sums are added
// by a shuffle tree.  The additions skip every reduction: the running sum's coordinates stay below 6q; the table
// entries are affine and below q, so an addition in the loop has eleven products, six of them in three sums that are
// reduced once (fq_mul2_lazy).  Bound by the multiply-adds: a commitment to 2^23 32-bit integers in rows of 2048 took
// 2.98 ms with the products' operands through scratch memory, 2.35 in registers and with the shared reductions, 2.25 with
// the products in line, 2.11 since the rows' inversions are division steps (0.14 ms of them before), and 1.9 with the
// signed digits of unequal windows (1.16 additions an entry before).
template <typename INT, class C>
__global__ __launch_bounds__(64) void k_commit_rows(const INT* x, uint64_t cols, const G1A* table,
                                                    const uint32_t* rho_le, const G1A* h_table, G1* sums) {
    static_assert(CK_H_WINDOWS <= 64 && CK_WBITS == 8, "one lane per window (byte) of the blinding scalar");
    constexpr uint32_t ENTRIES = (uint32_t)ck_entries<C>();   // of a column
    __shared__ uint32_t queue[CK_QUEUE];
    const uint64_t row = blockIdx.x;
    const int lane = threadIdx.x;
    G1 acc = g1_identity();
    if (rho_le) {
        const uint32_t d = lane < CK_H_WINDOWS ? (rho_le[row * 8 + (lane >> 2)] >> (8 * (lane & 3))) & 255u : 0u;
        if (d) {
            const G1A e = h_table[lane * CK_DIGITS + d - 1];
            acc.X = e.x;
            acc.Y = e.y;
            acc.Z = fq_one();
        }
    }
    const INT* xr = x + row * cols;
    const uint64_t below = ((uint64_t)1 << lane) - 1;   // the lanes before this one
    uint32_t head = 0, tail = 0;                        // the same in every lane
    G1A ahead;                                          // the table entry that the lane adds next
    bool waits = false, negative = false;               // it has one; with which sign
    for (uint64_t c0 = 0;; c0 += 64) {
        const bool last = c0 >= cols;                   // nothing new: what is left
        const uint64_t c = c0 + (uint64_t)lane;         // below 2^15
        uint64_t mag = 0;
        uint32_t sign = 0;
        if (c < cols) {
            const INT s = xr[c];
            sign = s < 0 ? 1u : 0u;
            mag = sign ? (uint64_t)0 - (uint64_t)(int64_t)s : (uint64_t)s;
        }
#pragma unroll
        for (int k = 0; k < C::N; ++k) {
            if (__ballot(mag != 0) == 0) break;
            // the digit d of window k; above half the window's range it is d - 2^w, with a carry (never in the top window)
            uint32_t d = (uint32_t)mag & ((1u << C::W[k]) - 1), flip = 0;
            mag >>= C::W[k];
            if (k + 1 < C::N && d > 1u << (C::W[k] - 1)) {
                d = (1u << C::W[k]) - d;
                flip = 1;
                mag += 1;
            }
            const uint64_t has = __ballot(d != 0);
            if (d) queue[(tail + (uint32_t)__popcll(has & below)) % CK_QUEUE] =
                       (d - 1 + (uint32_t)ck_entries<C>(k)) | ((sign ^ flip) << 15) | ((uint32_t)c << 16);
            tail += (uint32_t)__popcll(has);
        }
        __syncthreads();   // one wave: orders the ring's writes before its reads
        for (;;) {
            const uint32_t n = tail - head;
            if (n < 64 && !(last && (n || __ballot(waits)))) break;
            const bool take = (uint32_t)lane < n;
            G1A next = ahead;
            uint32_t item = 0;
            if (take) {
                item = queue[(head + (uint32_t)lane) % CK_QUEUE];
                next = table[(uint64_t)(item >> 16) * ENTRIES + (item & 0x7fffu)];
            }
            if (waits) {
                const Fq yn = fq_sub2_lazy<2, 1>(fq_zero(), ahead.y, fq_zero());   // 2q - y: x = r - |x| as a field element is -|x| G
                Fq y2;
#pragma unroll
                for (int i = 0; i < fqc::L; ++i) y2.v[i] = negative ? yn.v[i] : ahead.y.v[i];
                acc = g1_add_mixed_lazy(acc, ahead.x, y2);
            }
            ahead = next;
            waits = take;
            negative = (item >> 15) & 1u;
            head += n < 64 ? n : 64;
        }
        if (last) break;
    }
#pragma unroll 1
    for (int off = 32; off >= 1; off >>= 1) acc = g1_add_lazy_ni(acc, g1_shfl_down(acc, off));
    if (lane == 0) sums[row] = acc;   // coordinates below 6q
}

// affine bytes of the row sums: one inversion per row, one lane per row
__global__ __launch_bounds__(64) void k_commit_affine(const G1* sums, uint64_t rows, uint8_t* out) {
    const uint64_t row = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (row >= rows) return;
    g1_to_bytes(g1_reduce(sums[row]), out + row * 96);
}

// ---- the verifier's side of an opening: two sums of scalar multiples with full field elements as scalars ----
// 96 affine bytes -> Montgomery projective; *ok = false unless both coordinates are below q and the point is on
// the curve (or the bytes are all zero: the identity)
__device__ inline G1 g1_from_bytes(const uint8_t* b, bool* ok) {
    bool all_zero = true;
    for (int i = 0; i < 96; ++i) all_zero = all_zero && b[i] == 0;
    if (all_zero) return g1_identity();
    const Fq xp = fq_limbs_from_bytes(b), yp = fq_limbs_from_bytes(b + 48);
    const Fq q = fq_const(fqc::Q);
    if (!limbs_less(xp, q) || !limbs_less(yp, q)) *ok = false;
    G1 p;
    p.X = fq_to_mont(xp);
    p.Y = fq_to_mont(yp);
    p.Z = fq_one();
    Fq four = fq_add(fq_one(), fq_one());
    four = fq_add(four, four);
    const Fq rhs = fq_add(fq_mul_ni(fq_mul_ni(p.X, p.X), p.X), four);
    if (!fq_eq(fq_mul_ni(p.Y, p.Y), rhs)) *ok = false;
    return p;
}

// ---- a point operation shared by eight lanes -----------------------------------------------------------------
// The complete addition is two levels of six independent field products with linear steps between them (it doubles as
// well).  Lane j < 6 of a group of eight takes the j-th product of each level.  A point is kept as the six products of
// the second level that gave it, T_0 .. T_5, in LDS - X = T_1 - T_0, Y = T_2 + T_3, Z = T_4 + T_5 - so that the next
// operation's lanes read just the rows that their own operands are sums of: no lane forms coordinates that it does not
// multiply, and nothing goes round by shuffles.  (With every lane gathering all products of a level by shuffles and
// forming whole points, an operation took 5.4 us; like this 3.8.)  Every value stays non-negative by a multiple
// of q and is carried, not reduced: the Montgomery product takes normal operands up to 2^12 q and leaves less than
// 1.0001 q for the operands that occur here (below 40 q and 30 q).
constexpr int COOP = 8;           // lanes per point operation
constexpr int CROW = 20;          // words per row of 14 limbs: 16-byte aligned, rows begin on different banks
struct CoopPoint {
    alignas(16) uint32_t t[7][CROW];     // T_0 .. T_5, and a row of zeros
};
typedef __attribute__((address_space(3))) CoopPoint* CoopLds;
typedef const __attribute__((address_space(3))) sha::u32x4* lds_row4;

// rows of the operands of lane j.  Level 1, of a point: minus row n, plus rows p0 .. p3 (row 6: zeros); 2q more where
// X is among them:  X, Y, Z, X + Y, Y + Z, X + Z
__device__ const uint8_t COOP_ROWS1[COOP][5] = {{0, 1, 6, 6, 6}, {6, 2, 3, 6, 6}, {6, 4, 5, 6, 6}, {0, 1, 2, 3, 6},
                                                {6, 2, 3, 4, 5}, {0, 1, 4, 5, 6}, {6, 6, 6, 6, 6}, {6, 6, 6, 6, 6}};
// Level 2, of the level-1 products t0, t1, t2, p3, p4, p5: {row, coefficient} three times, then multiples of q.
//   t3 = p3 - t0 - t1, t4 = p4 - t1 - t2, y3 = 12 (p5 - t0 - t2), t1' = t1 - 12 t2, z3 = t1 + 12 t2, x3 = 3 t0;
//   products t4 y3, t3 t1', y3 x3, t1' z3, x3 t3, z3 t4
__device__ const int8_t COOP_ROWS2[COOP][2][7] = {
    {{1, -1, 2, -1, 4, 1, 3}, {0, -12, 2, -12, 5, 12, 25}},
    {{0, -1, 1, -1, 3, 1, 3}, {1, 1, 2, -12, 6, 0, 13}},
    {{0, -12, 2, -12, 5, 12, 25}, {0, 3, 6, 0, 6, 0, 0}},
    {{1, 1, 2, -12, 6, 0, 13}, {1, 1, 2, 12, 6, 0, 0}},
    {{0, 3, 6, 0, 6, 0, 0}, {0, -1, 1, -1, 3, 1, 3}},
    {{1, 1, 2, 12, 6, 0, 0}, {1, -1, 2, -1, 4, 1, 3}},
    {{6, 0, 6, 0, 6, 0, 0}, {6, 0, 6, 0, 6, 0, 0}},
    {{6, 0, 6, 0, 6, 0, 0}, {6, 0, 6, 0, 6, 0, 0}}};

struct CoopLane {
    int j;
    int rows1[5];             // row numbers
    uint32_t k1[fqc::L];      // what the carry pass of level 1 adds to a limb, see there
    int lin[2][7];
};
__device__ inline CoopLane coop_lane(int j) {
    CoopLane L;
    L.j = j;
#pragma unroll
    for (int k = 0; k < 5; ++k) L.rows1[k] = COOP_ROWS1[j][k];
    const uint32_t x = L.rows1[0] == 0 ? 2u : 0u;        // multiples of q
#pragma unroll
    for (int i = 0; i < fqc::L; ++i) L.k1[i] = x * fqc::Q[i] + (i < fqc::L - 1 ? 1u << 30 : 0u) - (i ? 2u : 0u);
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int k = 0; k < 7; ++k) L.lin[o][k] = COOP_ROWS2[j][o][k];
    return L;
}
__device__ __forceinline__ Fq coop_row(CoopLds p, int row) {
    Fq o;
    const lds_row4 r = (lds_row4)p->t[row];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const sha::u32x4 w = r[q];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (4 * q + k < fqc::L) o.v[4 * q + k] = w[k];
    }
    return o;
}
__device__ __forceinline__ void coop_row_store(CoopLds p, int row, const Fq& x) {
    typedef __attribute__((address_space(3))) sha::u32x4* row4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        sha::u32x4 w = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (4 * q + k < fqc::L) w[k] = x.v[4 * q + k];
        ((row4)p->t[row])[q] = w;
    }
}
__device__ __forceinline__ void coop_order() { asm volatile("" ::: "memory"); }   // one wave's LDS accesses run in order

__device__ __forceinline__ Fq coop_operand1(const CoopLane& L, CoopLds p) {
    const Fq n = coop_row(p, L.rows1[0]), a = coop_row(p, L.rows1[1]), b = coop_row(p, L.rows1[2]), c = coop_row(p, L.rows1[3]),
             d = coop_row(p, L.rows1[4]);
    // Every limb below the top one is lent 2^30, taken back as 2 from the limb above: between 2^29 and 2^32, no signs
    Fq o;
    uint32_t u = 0;
#pragma unroll
    for (int i = 0; i < fqc::L; ++i) {
        u = a.v[i] + b.v[i] + c.v[i] + d.v[i] - n.v[i] + L.k1[i] + (u >> 29);
        o.v[i] = i < fqc::L - 1 ? (u & fqc::M29) : u;
    }
    return o;
}
__device__ __forceinline__ Fq coop_operand2(const int (&c)[7], CoopLds p) {
    const Fq x = coop_row(p, c[0]), y = coop_row(p, c[2]), z = coop_row(p, c[4]);
    Fq o;
    int64_t acc = 0;
#pragma unroll
    for (int i = 0; i < fqc::L; ++i) {
        acc += (int64_t)c[6] * (int64_t)fqc::Q[i] + (int64_t)c[1] * (int32_t)x.v[i] + (int64_t)c[3] * (int32_t)y.v[i] +
               (int64_t)c[5] * (int32_t)z.v[i];
        o.v[i] = i < fqc::L - 1 ? ((uint32_t)acc & fqc::M29) : (uint32_t)acc;
        acc >>= 29;
    }
    return o;
}
// *p += *q for every group of eight lanes of the calling wave that writes (q may be p: a doubling, or a point that another group
// of the same wave writes in the same call: it is read first); tmp: the group's own rows
__device__ __forceinline__ void coop_add(const CoopLane& L, CoopLds p, CoopLds q, CoopLds tmp, bool write) {
    const Fq t = fq_mul_lazy_ni(coop_operand1(L, p), coop_operand1(L, q));
    if (L.j < 6) coop_row_store(tmp, L.j, t);
    coop_order();
    const Fq r = fq_mul_lazy_ni(coop_operand2(L.lin[0], tmp), coop_operand2(L.lin[1], tmp));
    coop_order();
    if (write && L.j < 6) coop_row_store(p, L.j, r);
    coop_order();
}
// one lane: coordinates (normal limbs, below 2 q) to the rows of a point, its row of zeros included
__device__ __forceinline__ void coop_set(CoopLds p, const G1& x) {
    coop_row_store(p, 0, fq_zero());
    coop_row_store(p, 1, x.X);
    coop_row_store(p, 2, x.Y);
    coop_row_store(p, 3, fq_zero());
    coop_row_store(p, 4, x.Z);
    coop_row_store(p, 5, fq_zero());
    coop_row_store(p, 6, fq_zero());
}
// one lane: the coordinates, below q
__device__ __forceinline__ G1 coop_get(CoopLds p) {
    auto combine = [&](int minus, int plus0, int plus1, int k) {
        const Fq n = coop_row(p, minus), a = coop_row(p, plus0), b = coop_row(p, plus1);
        Fq o;
        int64_t acc = 0;
#pragma unroll
        for (int i = 0; i < fqc::L; ++i) {
            acc += (int64_t)a.v[i] + b.v[i] - n.v[i] + (int64_t)k * fqc::Q[i];
            o.v[i] = i < fqc::L - 1 ? ((uint32_t)acc & fqc::M29) : (uint32_t)acc;
            acc >>= 29;
        }
        return fq_mul_ni(o, fq_one());
    };
    G1 g;
    g.X = combine(0, 1, 6, 2);
    g.Y = combine(6, 2, 3, 0);
    g.Z = combine(6, 4, 5, 0);
    return g;
}

constexpr int MSM_TERMS = 8;                      // terms per block
constexpr int MSM_GROUPS = 4;                     // groups of lanes per term: the doublings, two sums, the check's sum
constexpr int MSM_THREADS = MSM_TERMS * MSM_GROUPS * COOP;

// |z| for the curve's parameter z = -0xd201000000010000: r = z^4 - z^2 + 1 = (-z^2)^2 + (-z^2) + 1, so -z^2 is a
// cube root of unity modulo r.  The map phi(x, y) = (beta x, y), beta a cube root of unity in F_q, is an
// endomorphism of the curve; on the subgroup of order r it is multiplication by a cube root of unity modulo r, and
// beta is chosen (on the host, by trying both roots on a subgroup point: endo_beta) so that phi(P) = -z^2 P there.
constexpr uint64_t CK_Z_ABS = 0xd201000000010000ull;
constexpr uint32_t CK_ZZ[4] = {0x00000000u, 0x00000001u, 0x0001a402u, 0xac45a401u};          // z^2
constexpr uint32_t CK_ZZ_RECIP[6] = {0x034eb4b9u, 0xf6cfee2eu, 0x63f6e522u, 0xe01faaddu, 0x7c6becf1u, 0x1u};   // floor(2^288 / z^2)

// k = a + b z^2 with a < z^2: out[0..3] = a, out[4..7] = b (32-bit words, least significant first) for k < 2^128 z^2
// (every k < r < z^4).  b = floor(k / z^2) from the reciprocal: floor(floor(k / 2^96) M / 2^192) with
// M = floor(2^288 / z^2) is at most 2 too small.
__host__ __device__ inline void scalar_split(const uint32_t k[8], uint32_t out[8]) {
    uint32_t prod[11];
    for (int i = 0; i < 11; ++i) prod[i] = 0;
    for (int i = 0; i < 5; ++i) {
        uint64_t c = 0;
        for (int l = 0; l < 6; ++l) {
            c += (uint64_t)k[3 + i] * CK_ZZ_RECIP[l] + prod[i + l];
            prod[i + l] = (uint32_t)c;
            c >>= 32;
        }
        prod[i + 6] = (uint32_t)c;
    }
    uint32_t b[4], a[5], bz[5];
    for (int i = 0; i < 4; ++i) b[i] = prod[6 + i];
    for (int i = 0; i < 5; ++i) bz[i] = 0;
    for (int i = 0; i < 4; ++i) {          // b z^2 modulo 2^160
        uint64_t c = 0;
        for (int l = 0; l < 4 && i + l < 5; ++l) {
            c += (uint64_t)b[i] * CK_ZZ[l] + bz[i + l];
            bz[i + l] = (uint32_t)c;
            c >>= 32;
        }
        if (i == 0) bz[4] = (uint32_t)c;
    }
    int64_t bor = 0;
    for (int i = 0; i < 5; ++i) {
        const int64_t d = (int64_t)k[i] - (int64_t)bz[i] + bor;
        a[i] = (uint32_t)d;
        bor = d >> 32;
    }
    for (int it = 0; it < 3; ++it) {
        uint32_t d[5];
        int64_t w = 0;
        for (int i = 0; i < 5; ++i) {
            w += (int64_t)a[i] - (int64_t)(i < 4 ? CK_ZZ[i] : 0u);
            d[i] = (uint32_t)w;
            w >>= 32;
        }
        if (w < 0) break;                  // a < z^2
        uint64_t c = 1;
        for (int i = 0; i < 5; ++i) a[i] = d[i];
        for (int i = 0; i < 4; ++i) {
            c += b[i];
            b[i] = (uint32_t)c;
            c >>= 32;
        }
    }
    for (int i = 0; i < 4; ++i) {
        out[i] = a[i];
        out[4 + i] = b[i];
    }
}

// The split scalars of the two sums: the weights beta~(v_row, .) of the rows, then T (plain, below r), then rho* (zero
// without one)
__global__ __launch_bounds__(ZK_BLOCK) void k_msm_scalars(FrTab b_row, uint64_t nrows, const Fr* t_le, uint64_t cols, uint32_t* scal) {
    const uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (t >= nrows + cols + 1) return;
    const Fr k = t < nrows ? fr_from_mont(tab_ld(b_row, t)) : t_le[t - nrows];
    uint32_t out[8];
    scalar_split(k.v, out);
#pragma unroll
    for (int w = 0; w < 8; ++w) scal[8 * t + w] = out[w];
}

// One block: flags[1] = 1 unless sum_c beta~(v_col, c) T_c = y (T, y plain)
__global__ __launch_bounds__(ZK_BLOCK) void k_msm_value(FrTab b_col, const Fr* t_le, uint64_t cols, Fr y, uint32_t* flags) {
    __shared__ uint32_t red[64];
    Fr acc = fr_zero();
    for (uint64_t c = threadIdx.x; c < cols; c += blockDim.x) acc = fr_add(acc, fr_mul(tab_ld(b_col, c), t_le[c]));   // plain
    acc = block_sum(acc, red);
    if (threadIdx.x == 0) flags[1] = fr_eq(acc, y) ? 0u : 1u;
}

// Four groups of eight lanes per term of two sums in one launch: the blocks below nb_bytes take the points given as
// affine bytes (term t = 8 block + .. < n_bytes, scalar scal[t]), the others the key's generators (term t' < n_g1, scalar
// scal[n_bytes + t']).  A scalar k < r comes split as k = a + b z^2 with a, b < 2^128, so that k P = a P + b (-phi(P))
// for P in the subgroup: half as many doublings.  Group 0 doubles 2^i P; beside it group 1 adds it to a's sum where
// bit i of a is set (else the identity: the formulas are complete, and the wave stays in step), group 2 to b's sum, and
// group 3 to z^2 P for the check below: 128 operations long, however many bits are set (206 with the additions of a
// windowed method in the same chain).  Then sum a + (-phi)(sum b), and the block's terms in three more: part[block].
// The points given as bytes are checked to be elements of the subgroup, for which the split holds and in which Sec. 2.3
// works: phi(P) = -z^2 P exactly when r P = O (if phi(P) = -z^2 P then (z^4 - z^2 + 1) P = (phi^2 + phi + 1) P = O;
// conversely phi acts on the subgroup as the root -z^2 by the choice of beta).
// bad[0] is set if a point given as bytes is malformed or outside the subgroup.
// Bound by the chain: 0.55 ms for 512 + 513 terms, 1.18 as windows of four bits in one group of lanes.
__global__ __launch_bounds__(MSM_THREADS) void k_msm_terms(const uint8_t* pts_bytes, uint64_t n_bytes, unsigned nb_bytes,
                                                           const G1* pts_g1, const G1* pt_h, uint64_t n_g1, const uint32_t* scal,
                                                           G1* part, uint32_t* bad, Fq beta) {
    __shared__ CoopPoint pt[MSM_TERMS][MSM_GROUPS], tmp[MSM_TERMS][MSM_GROUPS], ident;
    const int tid = threadIdx.x, tt = tid / (MSM_GROUPS * COOP), g = tid / COOP % MSM_GROUPS;
    const CoopLane L = coop_lane(tid % COOP);
    const bool from_bytes = blockIdx.x < nb_bytes;
    const uint64_t t = (from_bytes ? blockIdx.x : blockIdx.x - nb_bytes) * (uint64_t)MSM_TERMS + tt;
    const bool live = t < (from_bytes ? n_bytes : n_g1);
    bool ok = true;
    G1 base = g1_identity();
    if (live) base = from_bytes ? g1_from_bytes(pts_bytes + 96 * t, &ok) : t + 1 < n_g1 ? pts_g1[t] : *pt_h;
    uint32_t k[4] = {0, 0, 0, 0};
    if (live && (g == 1 || g == 2)) {
        const uint32_t* sp = scal + 8 * (from_bytes ? t : n_bytes + t) + (g == 2 ? 4 : 0);
#pragma unroll
        for (int w = 0; w < 4; ++w) k[w] = sp[w];
    } else if (from_bytes && g == 3) {
#pragma unroll
        for (int w = 0; w < 4; ++w) k[w] = CK_ZZ[w];
    }
    const CoopLds own = (CoopLds)&pt[tt][g], mine = (CoopLds)&tmp[tt][g], dbl = (CoopLds)&pt[tt][0], zero = (CoopLds)&ident;
    if (L.j == 0) {
        coop_set(own, g == 0 ? base : g1_identity());
        coop_set(mine, g1_identity());
    }
    if (tid == 1) coop_set(zero, g1_identity());
    __syncthreads();
#pragma unroll 1
    for (int w = 0; w < 4; ++w) {
        const uint32_t word = w == 0 ? k[0] : w == 1 ? k[1] : w == 2 ? k[2] : k[3];
#pragma unroll 1
        for (int bit = 0; bit < 32; ++bit) coop_add(L, own, g == 0 || ((word >> bit) & 1u) ? dbl : zero, mine, true);
    }
    if (L.j == 0) {
        if (g == 2) {                          // -phi of the second sum
            G1 s = coop_get(own);
            s.X = fq_mul_ni(s.X, beta);
            s.Y = fq_neg(s.Y);
            coop_set(own, s);
        } else if (g == 3 && from_bytes && live && !fq_is_zero(base.Z)) {      // P affine: beta x Z' = X' and y Z' = -Y'
            const G1 zz = coop_get(own);
            ok = ok && fq_eq(fq_mul_ni(fq_mul_ni(beta, base.X), zz.Z), zz.X);
            ok = ok && fq_is_zero(fq_add(fq_mul_ni(base.Y, zz.Z), zz.Y));
        }
        if (live && !ok) bad[0] = 1;
    }
    coop_order();
    coop_add(L, own, g == 1 ? (CoopLds)&pt[tt][2] : zero, mine, g == 1);
#pragma unroll 1
    for (int off = MSM_TERMS / 2; off >= 1; off >>= 1) {
        __syncthreads();
        const bool adds = g == 1 && tt < off;
        coop_add(L, own, adds ? (CoopLds)&pt[tt + off][1] : zero, mine, adds);
    }
    if (tt == 0 && g == 1 && L.j == 0) part[blockIdx.x] = coop_get(own);
}

// Block b: the sum of its n0 / n1 points of part: 64 groups of lanes adding every 64th, six more additions; projective at
// proj[b], coordinates below q (the caller compares two sums by cross-multiplication and needs no inversion for that).
constexpr int MSM_FIN_THREADS = 512, MSM_FIN_GROUPS = MSM_FIN_THREADS / COOP;
__global__ __launch_bounds__(MSM_FIN_THREADS) void k_msm_finish(const G1* part, uint64_t n0, uint64_t n1, G1* proj) {
    __shared__ CoopPoint pt[MSM_FIN_GROUPS], tmp[MSM_FIN_GROUPS], next[MSM_FIN_GROUPS];
    const int grp = threadIdx.x / COOP;
    const CoopLane L = coop_lane(threadIdx.x % COOP);
    const G1* src = blockIdx.x ? part + n0 : part;
    const uint64_t n = blockIdx.x ? n1 : n0;
    const CoopLds own = (CoopLds)&pt[grp], mine = (CoopLds)&tmp[grp], nx = (CoopLds)&next[grp];
    if (L.j == 0) {
        coop_set(own, (uint64_t)grp < n ? src[grp] : g1_identity());
        coop_set(mine, g1_identity());
    }
    coop_order();
#pragma unroll 1
    for (uint64_t i = MSM_FIN_GROUPS; i < n; i += MSM_FIN_GROUPS) {   // every group runs the same number of trips
        if (L.j == 0) coop_set(nx, i + grp < n ? src[i + grp] : g1_identity());
        coop_order();
        coop_add(L, own, nx, mine, true);
    }
#pragma unroll 1
    for (int off = MSM_FIN_GROUPS / 2; off >= 1; off >>= 1) {
        __syncthreads();
        coop_add(L, own, grp < off ? (CoopLds)&pt[grp + off] : own, mine, grp < off);
    }
    if (threadIdx.x == 0) proj[blockIdx.x] = coop_get(own);
}

__global__ __launch_bounds__(64) void k_ck_export(const G1* gens, uint64_t first, uint64_t count, uint8_t* out) {
    const uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (i >= count) return;
    g1_to_bytes(gens[first + i], out + i * 96);
}

}  // namespace

struct zkdl_commit_key {
    uint64_t ncols;
    int max_bits;     // widest tensor entry served: 32 or 64
    bool wide;        // CkWindows<max_bits, wide>
    G1* gens;         // device: ncols generators, then H
    G1A* table;       // device: [ncols][ck_entries], affine
    G1A* h_table;     // device: [32][255]
};

// ---- host: the endomorphism's constant and the split of a scalar -------------------------------------------------
// a point of the curve found by trying x = 1, 2, .. (Montgomery form, Z = 1)
static bool host_curve_point(G1* out) {
    Fq xs = fq_zero();
    const Fq four = fq_add(fq_add(fq_one(), fq_one()), fq_add(fq_one(), fq_one()));
    for (int t = 0; t < 64; ++t) {
        xs = fq_add(xs, fq_one());
        const Fq rhs = fq_add(fq_mul(fq_sqr(xs), xs), four);
        const Fq y = fq_pow(rhs, fqc::EXP_SQRT);
        if (fq_eq(fq_sqr(y), rhs) && !fq_is_zero(y)) {
            out->X = xs;
            out->Y = y;
            out->Z = fq_one();
            return true;
        }
    }
    return false;
}

// beta with phi(P) = (beta x, y) = -z^2 P on the subgroup: beta = (-1 +- sqrt(-3)) / 2, the sign found by trying both
// on a point that the cofactor has taken into the subgroup.  false if neither fits (a broken constant).
static bool make_endo_beta(Fq* beta) {
    const Fq one = fq_one(), two = fq_add(one, one), m3 = fq_neg(fq_add(two, one));
    const Fq s = fq_pow(m3, fqc::EXP_SQRT);
    if (!fq_eq(fq_sqr(s), m3)) return false;
    const Fq half = fq_inv_steps(two);
    const Fq cand[2] = {fq_mul(fq_sub(s, one), half), fq_mul(fq_sub(fq_neg(s), one), half)};
    G1 p0;
    if (!host_curve_point(&p0)) return false;
    const G1 p = g1_mul_words(p0, fqc::COFACTOR);
    if (fq_is_zero(p.Z)) return false;
    const uint32_t zw[2] = {(uint32_t)CK_Z_ABS, (uint32_t)(CK_Z_ABS >> 32)};
    const G1 q = g1_mul_words(g1_mul_words(p, zw), zw);   // z^2 P
    for (int c = 0; c < 2; ++c) {
        const bool x_fits = fq_eq(fq_mul(fq_mul(cand[c], p.X), q.Z), fq_mul(q.X, p.Z));
        const bool y_fits = fq_is_zero(fq_add(fq_mul(p.Y, q.Z), fq_mul(q.Y, p.Z)));
        if (x_fits && y_fits && !fq_eq(cand[c], one) && fq_eq(fq_mul(fq_sqr(cand[c]), cand[c]), one)) {
            *beta = cand[c];
            return true;
        }
    }
    return false;
}

static bool endo_beta(Fq* beta) {
    static Fq value;
    static const bool ok = make_endo_beta(&value);
    *beta = value;
    return ok;
}

// k = a + b z^2 with a < z^2: out[0..3] = a, out[4..7] = b (32-bit words, least significant first); false unless
// b < 2^128 (true for every k < r < z^4).  Long division in base 2^32 (Knuth, Algorithm D; the divisor's top bit
// is set, so nothing is shifted), and the result is multiplied out again before it is trusted.  What scalar_split, which
// the kernels run, is held to, and the check of its range.
static bool glv_split(const uint32_t k[8], uint32_t out[8]) {
    const unsigned __int128 zz = (unsigned __int128)CK_Z_ABS * CK_Z_ABS;
    uint32_t v[4], un[9], q[5];
    for (int i = 0; i < 4; ++i) v[i] = (uint32_t)(zz >> (32 * i));
    for (int i = 0; i < 8; ++i) un[i] = k[i];
    un[8] = 0;
    for (int jj = 4; jj >= 0; --jj) {
        const uint64_t num = ((uint64_t)un[jj + 4] << 32) | un[jj + 3];
        uint64_t qhat = num / v[3], rhat = num % v[3];
        while (qhat >> 32 || qhat * v[2] > ((rhat << 32) | un[jj + 2])) {
            --qhat;
            rhat += v[3];
            if (rhat >> 32) break;
        }
        uint64_t carry = 0;
        int64_t borrow = 0;
        for (int i = 0; i < 4; ++i) {
            const uint64_t prod = qhat * v[i] + carry;
            carry = prod >> 32;
            const int64_t d = (int64_t)un[jj + i] - (int64_t)(uint32_t)prod - borrow;
            un[jj + i] = (uint32_t)d;
            borrow = d < 0 ? 1 : 0;
        }
        const int64_t d = (int64_t)un[jj + 4] - (int64_t)carry - borrow;
        un[jj + 4] = (uint32_t)d;
        if (d < 0) {   // the estimate was one too large: add the divisor back
            --qhat;
            uint64_t c = 0;
            for (int i = 0; i < 4; ++i) {
                c += (uint64_t)un[jj + i] + v[i];
                un[jj + i] = (uint32_t)c;
                c >>= 32;
            }
            un[jj + 4] += (uint32_t)c;
        }
        q[jj] = (uint32_t)qhat;
    }
    if (q[4] != 0) return false;
    unsigned __int128 a = 0, b = 0;
    for (int i = 3; i >= 0; --i) {
        a = (a << 32) | un[i];
        b = (b << 32) | q[i];
        out[i] = un[i];
        out[4 + i] = q[i];
    }
    if (a >= zz || un[4] || un[5] || un[6] || un[7]) return false;
    // a + b z^2 = k, multiplied out in 32-bit words
    uint32_t back[9] = {0};
    for (int i = 0; i < 4; ++i) {
        uint64_t c = 0;
        for (int l = 0; l < 4; ++l) {
            c += (uint64_t)q[i] * v[l] + back[i + l];
            back[i + l] = (uint32_t)c;
            c >>= 32;
        }
        back[i + 4] += (uint32_t)c;
    }
    uint64_t c = 0;
    for (int i = 0; i < 8; ++i) {
        c += (uint64_t)back[i] + (i < 4 ? un[i] : 0u);
        if ((uint32_t)c != k[i]) return false;
        c >>= 32;
    }
    return c == 0;
}

extern "C" int zkdl_host_scalar_split(const zkdl_fr* k, uint8_t out[32]) {
    if (!k || !out) return ZKDL_EINVAL;
    uint32_t kw[8], ab[8];
    memcpy(kw, k->le, 32);
    if (!glv_split(kw, ab)) return ZKDL_EINVAL;   // out of range
    scalar_split(kw, ab);
    memcpy(out, ab, 32);
    return ZKDL_OK;
}

// host-side check of the constants of fq.cuh (no GPU needed): Montgomery one and R^2 by repeated doubling,
// the Montgomery factor, the square-root and inversion exponents
static int commit_selfcheck_run() {
    Fq x = fq_zero();
    x.v[0] = 1;
    for (int i = 0; i < 406; ++i) x = fq_add(x, x);
    if (!fq_eq(x, fq_const(fqc::ONE))) return ZKDL_EINVAL;
    for (int i = 0; i < 406; ++i) x = fq_add(x, x);
    if (!fq_eq(x, fq_const(fqc::R2))) return ZKDL_EINVAL;
    if (((fqc::Q[0] * fqc::NINV) & fqc::M29) != fqc::M29) return ZKDL_EINVAL;   // q * (-q^{-1}) = -1 mod 2^29
    // 3^(q-2) * 3 = 1 and (3^2)^((q+1)/4) = +-3
    Fq three = fq_add(fq_one(), fq_add(fq_one(), fq_one()));
    if (!fq_eq(fq_mul(fq_inv(three), three), fq_one())) return ZKDL_EINVAL;
    Fq root = fq_pow(fq_sqr(three), fqc::EXP_SQRT);
    if (!fq_eq(root, three) && !fq_eq(root, fq_neg(three))) return ZKDL_EINVAL;
    // the inversion by division steps against a^(q-2): limb values 1, 2, q - 1, 2^380, then a chain of products
    Fq probe[16];
    probe[0] = fq_zero();
    probe[0].v[0] = 1;
    probe[1] = fq_add(probe[0], probe[0]);
    probe[2] = fq_sub(fq_zero(), probe[0]);
    probe[3] = fq_zero();
    probe[3].v[13] = 1u << 3;
    probe[4] = fq_one();
    probe[5] = fq_neg(fq_one());
    for (int i = 6; i < 16; ++i) probe[i] = fq_add(fq_mul(probe[i - 1], fq_add(three, probe[i - 3])), probe[i - 2]);
    for (int i = 0; i < 16; ++i)
        if (!fq_eq(fq_inv_steps(probe[i]), fq_inv(probe[i]))) return ZKDL_EINVAL;
    if (!fq_is_zero(fq_inv_steps(fq_zero()))) return ZKDL_EINVAL;
    // the additions without reductions against the reduced one, on multiples of a point found by trying x = 1, 2, ..:
    // a running sum that only ever goes through the lazy forms (so its coordinates take the bounds the kernel's do),
    // the sum from the identity, a point added to itself and to its negative
    G1 base;
    if (!host_curve_point(&base)) return ZKDL_EINVAL;
    auto same = [](const G1& a, const G1& b) {   // equal as projective points, coordinates reduced
        return fq_eq(fq_mul(a.X, b.Z), fq_mul(b.X, a.Z)) && fq_eq(fq_mul(a.Y, b.Z), fq_mul(b.Y, a.Z)) &&
               fq_is_zero(a.Z) == fq_is_zero(b.Z);
    };
    auto affine = [](const G1& p, Fq* x, Fq* y) {
        const Fq zi = fq_inv_steps(p.Z);
        *x = fq_mul(p.X, zi);
        *y = fq_mul(p.Y, zi);
    };
    const FqMulLazyInline lazy;
    G1 term = base, sum = g1_identity(), lsum = g1_identity(), msum = g1_identity();
    for (int i = 0; i < 40; ++i) {
        Fq tx, ty;
        affine(term, &tx, &ty);
        Fq y2 = ty;
        if (i % 3 == 1) {   // every third term negated the way the kernel negates (2q - y)
            term = g1_neg(term);
            y2 = fq_sub2_lazy<2, 1>(fq_zero(), ty, fq_zero());
        }
        sum = g1_add(sum, term);
        lsum = g1_add_lazy_with(lsum, term, lazy);
        msum = g1_add_mixed_lazy_with(msum, tx, y2, lazy);
        if (!same(g1_reduce(lsum), sum) || !same(g1_reduce(msum), sum)) return ZKDL_EINVAL;
        if (!same(g1_reduce(g1_add_lazy_with(lsum, msum, lazy)), g1_dbl(sum))) return ZKDL_EINVAL;   // two lazy operands
        term = g1_add(g1_dbl(term), base);
    }
    {
        Fq bx, by;
        affine(base, &bx, &by);
        const Fq byn = fq_sub2_lazy<2, 1>(fq_zero(), by, fq_zero());
        if (!same(g1_reduce(g1_add_mixed_lazy_with(base, bx, by, lazy)), g1_dbl(base))) return ZKDL_EINVAL;
        const G1 o = g1_reduce(g1_add_mixed_lazy_with(base, bx, byn, lazy));
        if (!fq_is_zero(o.Z) || !fq_is_zero(o.X)) return ZKDL_EINVAL;
        const G1 o2 = g1_reduce(g1_add_lazy_with(base, g1_neg(base), lazy));
        if (!fq_is_zero(o2.Z) || !fq_is_zero(o2.X)) return ZKDL_EINVAL;
    }
    // the endomorphism: its constant, and the split of a scalar on edge values (0, 1, z^2 - 1, z^2, z^2 + 1, r - 1,
    // 2^256 - 1 is refused) and on a chain of mixed words; with the split, k P = a P + b (-phi(P)) on a subgroup point
    Fq beta;
    if (!endo_beta(&beta)) return ZKDL_EINVAL;
    {
        const unsigned __int128 zz = (unsigned __int128)CK_Z_ABS * CK_Z_ABS;
        uint32_t ks[8][8] = {};
        ks[1][0] = 1;
        for (int i = 0; i < 4; ++i) {
            ks[2][i] = (uint32_t)((zz - 1) >> (32 * i));
            ks[3][i] = (uint32_t)(zz >> (32 * i));
            ks[4][i] = (uint32_t)((zz + 1) >> (32 * i));
        }
        for (int i = 0; i < 8; ++i) ks[5][i] = frc::MOD[i];
        ks[5][0] -= 1;
        uint32_t w = 0x9e3779b9u;
        for (int i = 0; i < 8; ++i) {
            w = w * 1664525u + 1013904223u;
            ks[6][i] = i == 7 ? (w & 0x3fffffffu) : w;
            ks[7][i] = i == 7 ? 0x73eda752u : ~w;
        }
        const G1 p = g1_mul_words(base, fqc::COFACTOR);   // in the subgroup
        G1 nphi = p;                                      // -phi(P) = (beta X, -Y, Z)
        nphi.X = fq_mul(p.X, beta);
        nphi.Y = fq_neg(p.Y);
        for (int t = 0; t < 8; ++t) {
            uint32_t ab[8];
            if (!glv_split(ks[t], ab)) return ZKDL_EINVAL;
            uint32_t fast[8];
            scalar_split(ks[t], fast);
            if (memcmp(fast, ab, sizeof ab) != 0) return ZKDL_EINVAL;
            const uint32_t a4[4] = {ab[0], ab[1], ab[2], ab[3]}, b4[4] = {ab[4], ab[5], ab[6], ab[7]};
            if (t >= 5 && !same(g1_mul_words(p, ks[t]), g1_add(g1_mul_words(p, a4), g1_mul_words(nphi, b4))))
                return ZKDL_EINVAL;
        }
        uint32_t all_ones[8], ab[8];
        for (int i = 0; i < 8; ++i) all_ones[i] = 0xffffffffu;
        if (glv_split(all_ones, ab)) return ZKDL_EINVAL;   // the quotient does not fit 128 bits
        // a point outside the subgroup does not pass the membership test phi(P) = -z^2 P
        const uint32_t zw[2] = {(uint32_t)CK_Z_ABS, (uint32_t)(CK_Z_ABS >> 32)};
        const G1 q = g1_mul_words(g1_mul_words(base, zw), zw);
        const bool base_in = fq_is_zero(g1_mul_words(base, frc::MOD).Z);
        const bool passes = fq_eq(fq_mul(fq_mul(beta, base.X), q.Z), fq_mul(q.X, base.Z)) &&
                            fq_is_zero(fq_add(fq_mul(base.Y, q.Z), fq_mul(q.Y, base.Z)));
        if (base_in != passes) return ZKDL_EINVAL;
    }
    return ZKDL_OK;
}

// the checks run once per process: they take some milliseconds of host arithmetic
extern "C" int zkdl_commit_selfcheck(void) {
    static const int rc = commit_selfcheck_run();
    return rc;
}

extern "C" int zkdl_commit_key_destroy(zkdl_ctx* ctx, zkdl_commit_key* key) {
    if (!ctx || !key) return ZKDL_EINVAL;
    (void)hipStreamSynchronize(ctx->stream);
    zk_free(ctx, key->gens);
    zk_free(ctx, key->table);
    zk_free(ctx, key->h_table);
    delete key;
    return ZKDL_OK;
}

extern "C" int zkdl_commit_key_create(zkdl_ctx* ctx, const char* label, uint64_t ncols, int max_bits,
                                      zkdl_commit_key** out) {
    if (!ctx || !label || !out || (max_bits != 32 && max_bits != 64)) return ZKDL_EINVAL;
    const size_t ll = strlen(label);
    if (ll > (size_t)CK_MAX_LABEL || ncols == 0 || (ncols & (ncols - 1)) || ncols > ((uint64_t)1 << 15)) return ZKDL_EINVAL;
    if (zkdl_commit_selfcheck() != ZKDL_OK) return ZKDL_EINVAL;
    ZK_HIP(ctx, hipSetDevice(ctx->device));
    zkdl_commit_key* key = new (std::nothrow) zkdl_commit_key();
    if (!key) return ZKDL_ENOMEM;
    key->ncols = ncols;
    key->max_bits = max_bits;
    // wide windows save additions (a 32-bit entry has three digits at most instead of four, one of 14 bits a single
    // digit) and cost 16 times the entries: taken while the tables stay a small part of the memory
    const CkLayout wide = max_bits == 32 ? ck_layout<CkWindows<32, true>>() : ck_layout<CkWindows<64, true>>();
    const CkLayout narrow = max_bits == 32 ? ck_layout<CkWindows<32, false>>() : ck_layout<CkWindows<64, false>>();
    key->wide = ctx->commit_wbits ? ctx->commit_wbits > 8 : sizeof(G1A) * ncols * (uint64_t)wide.first[wide.windows] <= CK_WIDE_MAX_BYTES;
    const CkLayout& lay = key->wide ? wide : narrow;
    CkLayout lay_h = {};
    for (int k = 0; k < CK_H_WINDOWS; ++k) ck_layout_add(&lay_h, CK_WBITS * k, CK_DIGITS);
    key->gens = (G1*)zk_alloc(ctx, sizeof(G1) * (ncols + 1));
    key->table = (G1A*)zk_alloc(ctx, sizeof(G1A) * ncols * lay.first[lay.windows]);
    key->h_table = (G1A*)zk_alloc(ctx, sizeof(G1A) * CK_H_WINDOWS * CK_DIGITS);
    if (!key->gens || !key->table || !key->h_table) {
        zkdl_commit_key_destroy(ctx, key);
        return ZKDL_ENOMEM;
    }
    LabelArg la;
    memcpy(la.bytes, "zkdl-mi355x/g1/", 15);
    memcpy(la.bytes + 15, label, ll);
    la.len = (uint32_t)(15 + ll);
    const Fq r2x = r2x_const();
    hipLaunchKernelGGL(k_ck_generators, dim3((unsigned)((ncols + 1 + 63) / 64)), dim3(64), 0, ctx->stream, la, ncols,
                       key->gens, r2x);
    // threads per (generator, window): a 16th of the entries
    const uint64_t nt = ncols * lay.chunks[lay.windows], nh = lay_h.chunks[CK_H_WINDOWS];
    hipLaunchKernelGGL(k_ck_tables, dim3((unsigned)((nt + 63) / 64)), dim3(64), 0, ctx->stream, key->gens, ncols, lay, key->table);
    hipLaunchKernelGGL(k_ck_tables, dim3((unsigned)((nh + 63) / 64)), dim3(64), 0, ctx->stream, key->gens + ncols, (uint64_t)1, lay_h,
                       key->h_table);
    hipError_t e = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) {
        ctx->last_hip = (int)e;
        zkdl_commit_key_destroy(ctx, key);
        return ZKDL_EHIP;
    }
    *out = key;
    return ZKDL_OK;
}

extern "C" int zkdl_commit_key_generators(zkdl_ctx* ctx, const zkdl_commit_key* key, uint64_t first, uint64_t count,
                                          uint8_t* host_out) {
    if (!ctx || !key || !host_out || first + count > key->ncols + 1 || count == 0) return ZKDL_EINVAL;
    uint8_t* dev = (uint8_t*)zk_alloc(ctx, count * 96);
    if (!dev) return ZKDL_ENOMEM;
    hipLaunchKernelGGL(k_ck_export, dim3((unsigned)((count + 63) / 64)), dim3(64), 0, ctx->stream, key->gens, first, count, dev);
    hipError_t e = hipMemcpyAsync(host_out, dev, count * 96, hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    zk_free(ctx, dev);
    ZK_HIP(ctx, e);
    return ZKDL_OK;
}

template <typename INT, int BITS>
static void launch_commit_rows(zkdl_ctx* ctx, const zkdl_commit_key* key, const INT* x, uint64_t rows, uint64_t cols, const uint32_t* rho,
                               G1* part) {
    const dim3 grid((unsigned)rows), block(64);
    if (key->wide)
        hipLaunchKernelGGL((k_commit_rows<INT, CkWindows<BITS, true>>), grid, block, 0, ctx->stream, x, cols, key->table, rho, key->h_table, part);
    else
        hipLaunchKernelGGL((k_commit_rows<INT, CkWindows<BITS, false>>), grid, block, 0, ctx->stream, x, cols, key->table, rho, key->h_table, part);
}

extern "C" int hyrax_commit(zkdl_ctx* ctx, const zkdl_commit_key* key, const zkdl_tensor* X, const zkdl_fr* blind,
                            uint8_t* commitments_out, size_t* ncommit) {
    if (!ctx || !key || !X || !commitments_out || !ncommit) return ZKDL_EINVAL;
    if (X->kind != TK_I32 && X->kind != TK_I64) return ZKDL_EINVAL;
    if (X->kind == TK_I64 && key->max_bits < 64) return ZKDL_EINVAL;
    int m = 0;
    while (((uint64_t)1 << m) < X->numel) ++m;
    if (((uint64_t)1 << m) != X->numel) return ZKDL_EINVAL;
    const uint64_t cols = (uint64_t)1 << (m / 2), rows = (uint64_t)1 << (m - m / 2);
    if (cols > key->ncols) return ZKDL_EINVAL;
    if (*ncommit < rows) {
        *ncommit = rows;
        return ZKDL_ESMALL;
    }
    for (uint64_t j = 0; blind && j < rows; ++j) {   // blinding scalars are field elements: below r
        bool below = false;
        for (int i = 31; i >= 0 && !below; --i) {
            const uint8_t rb = (uint8_t)(frc::MOD[i >> 2] >> (8 * (i & 3)));
            if (blind[j].le[i] > rb) return ZKDL_EINVAL;
            below = blind[j].le[i] < rb;
        }
        if (!below) return ZKDL_EINVAL;
    }
    ZK_HIP(ctx, hipSetDevice(ctx->device));
    G1* part = (G1*)zk_alloc(ctx, sizeof(G1) * rows);
    uint8_t* out_dev = (uint8_t*)zk_alloc(ctx, rows * 96);
    uint32_t* rho_dev = blind ? (uint32_t*)zk_alloc(ctx, rows * 32) : nullptr;
    int rc = (part && out_dev && (!blind || rho_dev)) ? ZKDL_OK : ZKDL_ENOMEM;
    hipError_t e = hipSuccess;
    if (rc == ZKDL_OK && blind) e = hipMemcpyAsync(rho_dev, blind, rows * 32, hipMemcpyHostToDevice, ctx->stream);
    if (rc == ZKDL_OK && e == hipSuccess) {
        // the windows are the key's, whatever the tensor's width
        if (X->kind == TK_I32 && key->max_bits == 32)
            launch_commit_rows<int32_t, 32>(ctx, key, (const int32_t*)X->data, rows, cols, rho_dev, part);
        else if (X->kind == TK_I32)
            launch_commit_rows<int32_t, 64>(ctx, key, (const int32_t*)X->data, rows, cols, rho_dev, part);
        else
            launch_commit_rows<int64_t, 64>(ctx, key, (const int64_t*)X->data, rows, cols, rho_dev, part);
        hipLaunchKernelGGL(k_commit_affine, dim3((unsigned)((rows + 63) / 64)), dim3(64), 0, ctx->stream, part, rows, out_dev);
        e = hipMemcpyAsync(commitments_out, out_dev, rows * 96, hipMemcpyDeviceToHost, ctx->stream);
    }
    hipError_t e2 = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess) e = e2;
    if (e == hipSuccess) e = hipGetLastError();
    zk_free(ctx, part);
    zk_free(ctx, out_dev);
    zk_free(ctx, rho_dev);
    if (rc != ZKDL_OK) return rc;
    ZK_HIP(ctx, e);
    *ncommit = rows;
    return ZKDL_OK;
}

static bool canonical_bytes(const zkdl_fr& a) {     // below r
    uint32_t w[8];
    memcpy(w, a.le, 32);
    for (int l = 7; l >= 0; --l)
        if (w[l] != frc::MOD[l]) return w[l] < frc::MOD[l];
    return false;
}

extern "C" int hyrax_verify(zkdl_ctx* ctx, const zkdl_commit_key* key, const uint8_t* commitments, size_t nrows,
                            const zkdl_fr* point, size_t npoint, const zkdl_fr* T, const zkdl_fr* rho, const zkdl_fr* y,
                            int* verdict, uint8_t* combined_out) {
    if (!ctx || !key || !commitments || !T || !y || !verdict || (npoint && !point)) return ZKDL_EINVAL;
    if (nrows == 0 || (nrows & (nrows - 1)) || nrows > ((size_t)1 << 16)) return ZKDL_EINVAL;
    int lr = 0;
    while (((size_t)1 << lr) < nrows) ++lr;
    if ((int)npoint < lr || (int)npoint - lr > 15) return ZKDL_EINVAL;
    const int lc = (int)npoint - lr;
    const uint64_t cols = (uint64_t)1 << lc;
    if (cols > key->ncols) return ZKDL_EINVAL;
    *verdict = 1;
    for (size_t i = 0; i < npoint; ++i)
        if (!canonical_bytes(point[i])) return ZKDL_OK;
    for (uint64_t c = 0; c < cols; ++c)
        if (!canonical_bytes(T[c])) return ZKDL_OK;
    if (!canonical_bytes(*y) || (rho && !canonical_bytes(*rho))) return ZKDL_OK;
    Fq beta;
    if (!endo_beta(&beta)) return ZKDL_EINVAL;
    ZK_HIP(ctx, hipSetDevice(ctx->device));
    // sum 1: the row commitments with the weights beta~(v_row, .); sum 2: Commit(T; rho*) on the key's generators
    const uint64_t n2 = cols + 1;
    const unsigned g1 = (unsigned)((nrows + MSM_TERMS - 1) / MSM_TERMS), g2 = (unsigned)((n2 + MSM_TERMS - 1) / MSM_TERMS);
    // T, rho* (zero without one), the kernels' two flags and the commitments go in front of the kernels, in one copy from the
    // context's pinned memory where it holds them: from the caller's pages, between the kernels, the GPU waited 0.07 ms for 64 KB.
    // Longer ones (2048 rows and more) come from the caller's pages all the same, with nothing allocated here that could fail.
    const size_t head_bytes = 32 * n2 + 64, in_bytes = head_bytes + nrows * 96;
    const bool staged = in_bytes <= sizeof(DevState);
    uint8_t* rest = ctx->host_stage + (staged ? 32 * cols : 0);      // rho*, the flags
    memset(rest, 0, 32 + 64);
    if (rho) memcpy(rest, rho->le, 32);
    if (staged) {
        memcpy(ctx->host_stage, T, 32 * cols);
        memcpy(ctx->host_stage + head_bytes, commitments, nrows * 96);
    }
    uint32_t* d_head = (uint32_t*)zk_alloc(ctx, in_bytes);
    const uint8_t* d_comm = (const uint8_t*)d_head + head_bytes;
    uint32_t* d_scal = (uint32_t*)zk_alloc(ctx, 32 * (nrows + n2));
    void* d_beta = zk_alloc(ctx, 32 * (nrows + cols));
    G1* d_part = (G1*)zk_alloc(ctx, sizeof(G1) * (g1 + g2));
    G1* d_proj = (G1*)zk_alloc(ctx, 2 * sizeof(G1));
    int rc = (d_head && d_scal && d_beta && d_part && d_proj) ? ZKDL_OK : ZKDL_ENOMEM;
    uint32_t h_flags[2] = {0, 0};
    G1 h_proj[2];
    hipError_t e = hipSuccess;
    if (rc == ZKDL_OK) {
        uint32_t* d_flags = d_head + 8 * n2;
        const FrTab b_row = make_tab(d_beta, nrows), b_col = make_tab((uint32_t*)d_beta + 8 * nrows, cols);
        Fr yp;
        memcpy(yp.v, y->le, 32);
        if (staged) {
            e = hipMemcpyAsync(d_head, ctx->host_stage, in_bytes, hipMemcpyHostToDevice, ctx->stream);
        } else {
            e = hipMemcpyAsync(d_head, T, 32 * cols, hipMemcpyHostToDevice, ctx->stream);
            if (e == hipSuccess) e = hipMemcpyAsync(d_head + 8 * cols, rest, 32 + 64, hipMemcpyHostToDevice, ctx->stream);
            if (e == hipSuccess) e = hipMemcpyAsync(d_head + head_bytes / 4, commitments, nrows * 96, hipMemcpyHostToDevice, ctx->stream);
        }
        if (e == hipSuccess) {
            zk_launch_beta_direct(ctx, (const uint8_t*)point, lr, b_row);
            zk_launch_beta_direct(ctx, (const uint8_t*)(point + lr), lc, b_col);
            hipLaunchKernelGGL(k_msm_scalars, dim3((unsigned)((nrows + n2 + ZK_BLOCK - 1) / ZK_BLOCK)), dim3(ZK_BLOCK), 0, ctx->stream,
                               b_row, (uint64_t)nrows, (const Fr*)d_head, cols, d_scal);
            hipLaunchKernelGGL(k_msm_value, dim3(1), dim3(ZK_BLOCK), 0, ctx->stream, b_col, (const Fr*)d_head, cols, yp, d_flags);
            hipLaunchKernelGGL(k_msm_terms, dim3(g1 + g2), dim3(MSM_THREADS), 0, ctx->stream, d_comm, (uint64_t)nrows, g1, key->gens,
                               key->gens + key->ncols, n2, d_scal, d_part, d_flags, beta);
            hipLaunchKernelGGL(k_msm_finish, dim3(2), dim3(MSM_FIN_THREADS), 0, ctx->stream, d_part, (uint64_t)g1, (uint64_t)g2, d_proj);
            e = hipMemcpyAsync(h_proj, d_proj, 2 * sizeof(G1), hipMemcpyDeviceToHost, ctx->stream);
            if (e == hipSuccess) e = hipMemcpyAsync(h_flags, d_flags, 8, hipMemcpyDeviceToHost, ctx->stream);
        }
    }
    hipError_t e2 = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess) e = e2;
    if (e == hipSuccess) e = hipGetLastError();
    zk_free(ctx, d_head);
    zk_free(ctx, d_scal);
    zk_free(ctx, d_beta);
    zk_free(ctx, d_part);
    zk_free(ctx, d_proj);
    if (rc != ZKDL_OK) return rc;
    ZK_HIP(ctx, e);
    if (h_flags[0]) return ZKDL_OK;                // verdict 1: a commitment is not an element of the group
    // C* as bytes: the inversion, one chain of steps, takes a lane of the GPU 0.07 ms and this thread 0.01
    if (combined_out) g1_to_bytes(h_proj[0], combined_out);
    // X1 Z2 = X2 Z1 and Y1 Z2 = Y2 Z1 (the identity is (0, 1, 0): it equals only itself)
    const G1 &a = h_proj[0], &b = h_proj[1];
    const bool same = fq_eq(fq_mul(a.X, b.Z), fq_mul(b.X, a.Z)) && fq_eq(fq_mul(a.Y, b.Z), fq_mul(b.Y, a.Z)) &&
                      fq_is_zero(a.Z) == fq_is_zero(b.Z);
    if (!same) {
        *verdict = 2;                              // Commit(T; rho*) is not the combined commitment
        return ZKDL_OK;
    }
    *verdict = h_flags[1] ? 3 : 0;                 // 3: <T, beta~(v_col, .)> != y
    return ZKDL_OK;
}
