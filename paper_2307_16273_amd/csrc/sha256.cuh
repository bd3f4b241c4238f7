// SHA-256 (FIPS 180-4) and the Fiat-Shamir transcript built on it, usable from
// host code and from a single GPU thread.
//
// The paper's verifier sends a uniform field element after each round
// polynomial (App. B); the transcript replaces that message by a hash.  The
// transcript is one byte stream:
//   stream_0         = "zkdl-mi355x/v3" zero-padded to 56 bytes || u64le(seed)
//   absorb(label, m) : stream <- stream || u8(|label|) || label || u64le(|m|) || m
//   challenges(n)    : for i < n: d0 = SHA256(stream || 0xF0 || u32le(i)),
//                      d1 = SHA256(stream || 0xF1 || u32le(i)), c_i = int_le(d0 || d1) mod r;
//                      then stream <- stream || 0xF2 || zero bytes up to the next multiple of 64.
//                      challenge() = challenges(1)[0].
//   digest()         = SHA256(stream)
// The state is the SHA-256 chaining value after the last whole block, the block count and the
// bytes of the unfinished block.  After a draw the stream is block-aligned, so a sumcheck round
// (a 106-byte frame, then one challenge) is one compression for the frame's first 64 bytes and
// then three independent ones from that chaining value: the two hashes of the draw (last block:
// the other 42 bytes, tag, index, padding, bit length) and the block that extends the stream.
// No message schedule depends on a chaining value, so they are all computed beforehand, in
// other lanes than the one that runs the rounds.
#pragma once
#include <stdint.h>
#include <hip/hip_runtime.h>
#include "fr.cuh"

#define SHA_HD __host__ __device__ inline

namespace sha {

SHA_HD uint32_t rotr(uint32_t x, int n) { return (x >> n) | (x << (32 - n)); }

SHA_HD uint32_t kconst(int i) {
    constexpr uint32_t K[64] = {
        0x428a2f98, 0x71374491, 0xb5c0fbcf, 0xe9b5dba5, 0x3956c25b, 0x59f111f1, 0x923f82a4, 0xab1c5ed5,
        0xd807aa98, 0x12835b01, 0x243185be, 0x550c7dc3, 0x72be5d74, 0x80deb1fe, 0x9bdc06a7, 0xc19bf174,
        0xe49b69c1, 0xefbe4786, 0x0fc19dc6, 0x240ca1cc, 0x2de92c6f, 0x4a7484aa, 0x5cb0a9dc, 0x76f988da,
        0x983e5152, 0xa831c66d, 0xb00327c8, 0xbf597fc7, 0xc6e00bf3, 0xd5a79147, 0x06ca6351, 0x14292967,
        0x27b70a85, 0x2e1b2138, 0x4d2c6dfc, 0x53380d13, 0x650a7354, 0x766a0abb, 0x81c2c92e, 0x92722c85,
        0xa2bfe8a1, 0xa81a664b, 0xc24b8b70, 0xc76c51a3, 0xd192e819, 0xd6990624, 0xf40e3585, 0x106aa070,
        0x19a4c116, 0x1e376c08, 0x2748774c, 0x34b0bcb5, 0x391c0cb3, 0x4ed8aa4a, 0x5b9cca4f, 0x682e6ff3,
        0x748f82ee, 0x78a5636f, 0x84c87814, 0x8cc70208, 0x90befffa, 0xa4506ceb, 0xbef9a3f7, 0xc67178f2};
    return K[i];
}

// Message schedule with the round constants folded in: wk[t] = W[t] + K[t].  It does not
// depend on the chaining value, so on the GPU it runs in other lanes than the rounds.
SHA_HD void schedule_wk(const uint32_t w_in[16], uint32_t wk[64]) {
    uint32_t w[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = w_in[i];
#pragma unroll
    for (int i = 0; i < 64; ++i) {
        if (i >= 16) {
            uint32_t w15 = w[(i + 1) & 15], w2 = w[(i + 14) & 15];
            uint32_t s0 = rotr(w15, 7) ^ rotr(w15, 18) ^ (w15 >> 3);
            uint32_t s1 = rotr(w2, 17) ^ rotr(w2, 19) ^ (w2 >> 10);
            w[i & 15] = w[i & 15] + s0 + w[(i + 9) & 15] + s1;
        }
        wk[i] = w[i & 15] + kconst(i);
    }
}

// the 64 rounds on a prepared schedule
SHA_HD void rounds(uint32_t h[8], const uint32_t wk[64]) {
    uint32_t a = h[0], b = h[1], c = h[2], d = h[3], e = h[4], f = h[5], g = h[6], hh = h[7];
#pragma unroll
    for (int i = 0; i < 64; ++i) {
        uint32_t S1 = rotr(e, 6) ^ rotr(e, 11) ^ rotr(e, 25);
        uint32_t ch = (e & f) | (~e & g);              // bit select: v_bfi_b32
        uint32_t t1 = hh + S1 + ch + wk[i];
        uint32_t S0 = rotr(a, 2) ^ rotr(a, 13) ^ rotr(a, 22);
        uint32_t ab = a ^ b;
        uint32_t mj = (ab & c) | (~ab & b);            // majority as a bit select
        hh = g; g = f; f = e; e = d + t1; d = c; c = b; b = a; a = t1 + S0 + mj;
    }
    h[0] += a; h[1] += b; h[2] += c; h[3] += d; h[4] += e; h[5] += f; h[6] += g; h[7] += hh;
}

// one compression of a 64-byte block given as 16 big-endian words
SHA_HD void compress(uint32_t h[8], uint32_t w[16]) {
    uint32_t wk[64];
    schedule_wk(w, wk);
    rounds(h, wk);
}

#if defined(__HIPCC__)
// Compact device versions for the single-wave transcript steps.  Those steps execute
// every instruction once per launch, from a cold instruction cache, so code bytes cost as
// much as instructions: the bodies below are loops of 16 rounds and are not inlined.
struct Words8 {
    uint32_t v[8];
};
struct Words16 {
    uint32_t v[16];
};

static __device__ const uint32_t K_TABLE[64] = {
    0x428a2f98, 0x71374491, 0xb5c0fbcf, 0xe9b5dba5, 0x3956c25b, 0x59f111f1, 0x923f82a4, 0xab1c5ed5,
    0xd807aa98, 0x12835b01, 0x243185be, 0x550c7dc3, 0x72be5d74, 0x80deb1fe, 0x9bdc06a7, 0xc19bf174,
    0xe49b69c1, 0xefbe4786, 0x0fc19dc6, 0x240ca1cc, 0x2de92c6f, 0x4a7484aa, 0x5cb0a9dc, 0x76f988da,
    0x983e5152, 0xa831c66d, 0xb00327c8, 0xbf597fc7, 0xc6e00bf3, 0xd5a79147, 0x06ca6351, 0x14292967,
    0x27b70a85, 0x2e1b2138, 0x4d2c6dfc, 0x53380d13, 0x650a7354, 0x766a0abb, 0x81c2c92e, 0x92722c85,
    0xa2bfe8a1, 0xa81a664b, 0xc24b8b70, 0xc76c51a3, 0xd192e819, 0xd6990624, 0xf40e3585, 0x106aa070,
    0x19a4c116, 0x1e376c08, 0x2748774c, 0x34b0bcb5, 0x391c0cb3, 0x4ed8aa4a, 0x5b9cca4f, 0x682e6ff3,
    0x748f82ee, 0x78a5636f, 0x84c87814, 0x8cc70208, 0x90befffa, 0xa4506ceb, 0xbef9a3f7, 0xc67178f2};

// three-input bit operations in one instruction (truth table in the immediate)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint32_t choose(uint32_t e, uint32_t f, uint32_t g) {   // e ? f : g
    return __builtin_amdgcn_bitop3_b32(e, f, g, 0xCA);
}
__device__ __forceinline__ uint32_t majority(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}
__device__ __forceinline__ uint32_t big_sigma1(uint32_t e) { return xor3(rotr(e, 6), rotr(e, 11), rotr(e, 25)); }
__device__ __forceinline__ uint32_t big_sigma0(uint32_t a) { return xor3(rotr(a, 2), rotr(a, 13), rotr(a, 22)); }
__device__ __forceinline__ uint32_t small_sigma0(uint32_t w) { return xor3(rotr(w, 7), rotr(w, 18), w >> 3); }
__device__ __forceinline__ uint32_t small_sigma1(uint32_t w) { return xor3(rotr(w, 17), rotr(w, 19), w >> 10); }

typedef __attribute__((address_space(3))) uint32_t* lds_u32_ptr;
typedef const __attribute__((address_space(3))) uint32_t* lds_u32_cptr;

static __device__ __noinline__ Words8 compress_ni(Words8 hin, Words16 win) {
    uint32_t w[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = win.v[i];
    uint32_t a = hin.v[0], b = hin.v[1], c = hin.v[2], d = hin.v[3], e = hin.v[4], f = hin.v[5],
             g = hin.v[6], hh = hin.v[7];
#pragma unroll 1
    for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (r > 0) w[i] = w[i] + small_sigma0(w[(i + 1) & 15]) + w[(i + 9) & 15] + small_sigma1(w[(i + 14) & 15]);
            uint32_t t1 = hh + big_sigma1(e) + choose(e, f, g) + K_TABLE[16 * r + i] + w[i];
            uint32_t t2 = big_sigma0(a) + majority(a, b, c);
            hh = g; g = f; f = e; e = d + t1; d = c; c = b; b = a; a = t1 + t2;
        }
    }
    Words8 o;
    o.v[0] = hin.v[0] + a; o.v[1] = hin.v[1] + b; o.v[2] = hin.v[2] + c; o.v[3] = hin.v[3] + d;
    o.v[4] = hin.v[4] + e; o.v[5] = hin.v[5] + f; o.v[6] = hin.v[6] + g; o.v[7] = hin.v[7] + hh;
    return o;
}

__device__ inline Words8 iv_words() {
    Words8 h = {{0x6a09e667, 0xbb67ae85, 0x3c6ef372, 0xa54ff53a, 0x510e527f, 0x9b05688c, 0x1f83d9ab,
                 0x5be0cd19}};
    return h;
}

// ---- one compression: the rounds in one wave, its schedule in another, both split over two lanes ------------
// A compression is a chain, and one wave issues an instruction every 5.4 cycles whatever its lanes do, so a chain
// gets shorter only by fewer instructions in a row.  Both halves of a round have the same shape - three rotations of
// a state word, a bit selection, sums - so two lanes do them side by side: the "low" lane holds a, b, c, d, the "high"
// lane e, f, g, h; the majority of a, b, c is the selection of b or c by the bits in which a and b agree, and the two
// sums change places by DPP operands (low and high lanes mirror each other inside groups of eight, and are told
// apart by the bank masks).  A round is ten instructions instead of fourteen; a pass over one block 4.3 thousand cycles
// instead of 5.9 (one wave alone, schedule at hand).  The schedule splits into even and odd words in the same way:
// seven instructions a word instead of eleven, so that it stays ahead of the faster rounds.
//   lane 8 g + j, j < 4, and lane 8 g + 7 - j: low and high lane of block row 4 g + j.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef volatile const __attribute__((address_space(3))) u32x4* lds_u32x4_vcptr;
typedef volatile __attribute__((address_space(3))) uint32_t* lds_u32_vptr;

struct Half {
    uint32_t v[4];
};

__device__ __forceinline__ bool half_is_high() { return (threadIdx.x & 4) != 0; }
__device__ __forceinline__ uint32_t half_row() {
    const uint32_t l = threadIdx.x & 63;
    return ((l >> 3) << 2) | ((l & 4) ? 7 - (l & 7) : (l & 3));
}

// Words 16 .. 63 of the schedules, round constants included.  The lane pair of a row: msg = its sixteen message words
// (LDS); wk = its schedule row (16-byte aligned; words 0 .. 15 are not written), k64 = the round constants.  After each
// sixteen words *seq = base + the groups that stand in LDS (the operations of one wave on LDS complete in order).
static __device__ __noinline__ void schedule_ahead(lds_u32_cptr msg, lds_u32_ptr wk, lds_u32_cptr k64, lds_u32_vptr seq,
                                                   uint32_t base) {
    // the low lane holds the even words, the high lane the odd ones
    const uint32_t p = half_is_high() ? 1 : 0;
    uint32_t w[8], s[8], k[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = msg[2 * i + p];
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = small_sigma0(w[i]);
#pragma unroll 1
    for (uint32_t r = 1; r < 4; ++r) {
#pragma unroll
        for (int i = 0; i < 8; ++i) k[i] = k64[16 * r + 2 * i + p];
        uint32_t t0, t1, t2;
        // word n+16 = word n + sigma0(word n+1) + word n+9 + sigma1(word n+14): for the even words of step i the other
        // lane's i and i+4, for the odd ones the other lane's i+1 and i+5.  Every DPP source is at least two
        // instructions old (the s_nop covers the first).  Instructions of eight bytes that straddle an eight-byte
        // boundary issue a sixth slower (a pass over a block: 3.8 thousand cycles aligned, 4.5 not).
#define ZK_SHA_SCHED(W, S, S1, W4, W5, W7)                                                     \
    "v_add_u32_dpp " W ", " S ", " W " row_half_mirror row_mask:0xf bank_mask:0x5\n\t"         \
    "v_alignbit_b32 %[t0], " W7 ", " W7 ", 17\n\t"                                             \
    "v_add_u32_dpp " W ", " S1 ", " W " row_half_mirror row_mask:0xf bank_mask:0xa\n\t"        \
    "v_alignbit_b32 %[t1], " W7 ", " W7 ", 19\n\t"                                             \
    "v_add_u32_dpp " W ", " W4 ", " W " row_half_mirror row_mask:0xf bank_mask:0x5\n\t"        \
    "v_lshrrev_b32 %[t2], 10, " W7 "\n\t"                                                      \
    "v_add_u32_dpp " W ", " W5 ", " W " row_half_mirror row_mask:0xf bank_mask:0xa\n\t"        \
    "v_bitop3_b32 %[t0], %[t0], %[t1], %[t2] bitop3:0x96\n\t"                                  \
    "v_add_u32 " W ", " W ", %[t0]\n\t"                                                        \
    "v_alignbit_b32 %[t0], " W ", " W ", 7\n\t"                                                \
    "v_alignbit_b32 %[t1], " W ", " W ", 18\n\t"                                               \
    "v_lshrrev_b32 %[t2], 3, " W "\n\t"                                                        \
    "v_bitop3_b32 " S ", %[t0], %[t1], %[t2] bitop3:0x96\n\t"
        asm volatile("s_nop 1\n\t.p2align 3\n\t"
            ZK_SHA_SCHED("%[w0]", "%[s0]", "%[s1]", "%[w4]", "%[w5]", "%[w7]")
            ZK_SHA_SCHED("%[w1]", "%[s1]", "%[s2]", "%[w5]", "%[w6]", "%[w0]")
            ZK_SHA_SCHED("%[w2]", "%[s2]", "%[s3]", "%[w6]", "%[w7]", "%[w1]")
            ZK_SHA_SCHED("%[w3]", "%[s3]", "%[s4]", "%[w7]", "%[w0]", "%[w2]")
            ZK_SHA_SCHED("%[w4]", "%[s4]", "%[s5]", "%[w0]", "%[w1]", "%[w3]")
            ZK_SHA_SCHED("%[w5]", "%[s5]", "%[s6]", "%[w1]", "%[w2]", "%[w4]")
            ZK_SHA_SCHED("%[w6]", "%[s6]", "%[s7]", "%[w2]", "%[w3]", "%[w5]")
            ZK_SHA_SCHED("%[w7]", "%[s7]", "%[s0]", "%[w3]", "%[w4]", "%[w6]")
            : [w0] "+v"(w[0]), [w1] "+v"(w[1]), [w2] "+v"(w[2]), [w3] "+v"(w[3]), [w4] "+v"(w[4]), [w5] "+v"(w[5]),
              [w6] "+v"(w[6]), [w7] "+v"(w[7]), [s0] "+v"(s[0]), [s1] "+v"(s[1]), [s2] "+v"(s[2]), [s3] "+v"(s[3]),
              [s4] "+v"(s[4]), [s5] "+v"(s[5]), [s6] "+v"(s[6]), [s7] "+v"(s[7]), [t0] "=&v"(t0), [t1] "=&v"(t1),
              [t2] "=&v"(t2));
#undef ZK_SHA_SCHED
#pragma unroll
        for (int i = 0; i < 8; ++i) wk[16 * r + 2 * i + p] = w[i] + k[i];
        asm volatile("" ::: "memory");
        if ((threadIdx.x & 63) == 0) *seq = base + r;
        asm volatile("" ::: "memory");
    }
}

// The 64 rounds of one block for every lane pair; hin and the result are the lane's half of the chaining value.  msg, k,
// wk (16-byte aligned): message words, round constants and schedule row for the high lane; the low lane is given
// sixteen zero words for all three (it adds nothing) and step 0 instead of 16.  Group r of the schedule is read half a
// group ahead, together with *seq, and again until *seq >= base + r (the other wave gets there).
static __device__ __noinline__ Half rounds_behind(Half hin, lds_u32_cptr msg, lds_u32_cptr k, lds_u32_cptr wk, uint32_t step,
                                                  lds_u32_vptr seq, uint32_t base) {
    uint32_t s0 = hin.v[0], s1 = hin.v[1], s2 = hin.v[2], s3 = hin.v[3];
    const bool high = half_is_high();
    const uint32_t r0 = high ? 6 : 2, r1 = high ? 11 : 13, r2 = high ? 25 : 22, m = high ? 0u : ~0u;
    u32x4 y[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) y[q] = ((lds_u32x4_vcptr)msg)[q];
#pragma unroll
    for (int q = 0; q < 4; ++q) y[q] += ((lds_u32x4_vcptr)k)[q];
    // T: h + W + K in the high lane, zero in the low one; NEXT makes the next round's in the place of its W + K.
    // bitop3 0xd2: m ? ~(S0 ^ S1) : S0.  The two instructions between the sum rb and its DPP use are the two wait
    // states that a DPP source needs.
#define ZK_SHA_ROUND(S0, S1, S2, S3, T, NEXT)                                                              \
    "v_alignbit_b32 %[ra], " S0 ", " S0 ", %[r0]\n\t"                                                      \
    "v_bitop3_b32 %[x], " S0 ", " S1 ", %[m] bitop3:0xd2\n\t"                                              \
    "v_alignbit_b32 %[rb], " S0 ", " S0 ", %[r1]\n\t"                                                      \
    "v_alignbit_b32 %[rc], " S0 ", " S0 ", %[r2]\n\t"                                                      \
    "v_bitop3_b32 %[x], %[x], " S1 ", " S2 " bitop3:0xca\n\t"                                              \
    "v_bitop3_b32 %[ra], %[ra], %[rb], %[rc] bitop3:0x96\n\t"                                              \
    "v_add3_u32 %[rb], %[ra], %[x], " T "\n\t"                                                             \
    "v_add_u32_dpp " S3 ", " S3 ", %[rb] row_half_mirror row_mask:0xf bank_mask:0xa\n\t"                   \
    NEXT                                                                                                   \
    "v_add_u32_dpp " S3 ", %[rb], %[rb] row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
#define ZK_SHA_NEXT(S2, T) "v_add_u32_dpp " T ", " S2 ", " T " quad_perm:[0,1,2,3] row_mask:0xf bank_mask:0xa\n\t"
#define ZK_SHA_QUAD(A, B, C, D, E)                                                                         \
    ZK_SHA_ROUND("%[a]", "%[b]", "%[c]", "%[d]", A, ZK_SHA_NEXT("%[c]", B))                                \
    ZK_SHA_ROUND("%[d]", "%[a]", "%[b]", "%[c]", B, ZK_SHA_NEXT("%[b]", C))                                \
    ZK_SHA_ROUND("%[c]", "%[d]", "%[a]", "%[b]", C, ZK_SHA_NEXT("%[a]", D))                                \
    ZK_SHA_ROUND("%[b]", "%[c]", "%[d]", "%[a]", D, E)
#define ZK_SHA_EIGHT(X0, X1)                                                                               \
    asm volatile("s_nop 1\n\t.p2align 3\n\t" ZK_SHA_NEXT("%[d]", "%[w0]")                                  \
        ZK_SHA_QUAD("%[w0]", "%[w1]", "%[w2]", "%[w3]", ZK_SHA_NEXT("%[d]", "%[w4]"))                      \
        ZK_SHA_QUAD("%[w4]", "%[w5]", "%[w6]", "%[w7]", "s_nop 0\n\t")                                     \
        : [a] "+v"(s0), [b] "+v"(s1), [c] "+v"(s2), [d] "+v"(s3), [ra] "=&v"(ra), [rb] "=&v"(rb), [rc] "=&v"(rc),   \
          [x] "=&v"(xx), [w0] "+v"(X0[0]), [w1] "+v"(X0[1]), [w2] "+v"(X0[2]), [w3] "+v"(X0[3]), [w4] "+v"(X1[0]),   \
          [w5] "+v"(X1[1]), [w6] "+v"(X1[2]), [w7] "+v"(X1[3])                                             \
        : [r0] "v"(r0), [r1] "v"(r1), [r2] "v"(r2), [m] "v"(m))
#pragma unroll 1
    for (uint32_t r = 1;; ++r) {
        uint32_t ra, rb, rc, xx, seen = 0;
        ZK_SHA_EIGHT(y[0], y[1]);
        wk += step;
        u32x4 z[4] = {y[0], y[0], y[0], y[0]};
        if (r < 4) {                 // half a group before its first use: later, and it would be waited for
            seen = *seq;
#pragma unroll
            for (int q = 0; q < 4; ++q) z[q] = ((lds_u32x4_vcptr)wk)[q];
        }
        ZK_SHA_EIGHT(y[2], y[3]);
        if (r == 4) break;
        while (__builtin_amdgcn_readfirstlane(seen) < base + r) {
            seen = *seq;
#pragma unroll
            for (int q = 0; q < 4; ++q) z[q] = ((lds_u32x4_vcptr)wk)[q];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) y[q] = z[q];
    }
#undef ZK_SHA_EIGHT
#undef ZK_SHA_QUAD
#undef ZK_SHA_NEXT
#undef ZK_SHA_ROUND
    Half o;
    o.v[0] = hin.v[0] + s0; o.v[1] = hin.v[1] + s1; o.v[2] = hin.v[2] + s2; o.v[3] = hin.v[3] + s3;
    return o;
}

#endif

SHA_HD uint32_t bswap32(uint32_t x) {
    return (x >> 24) | ((x >> 8) & 0xff00u) | ((x << 8) & 0xff0000u) | (x << 24);
}

SHA_HD void bytes_to_words(const uint8_t b[32], uint32_t w[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
        w[i] = ((uint32_t)b[4 * i] << 24) | ((uint32_t)b[4 * i + 1] << 16) | ((uint32_t)b[4 * i + 2] << 8) | b[4 * i + 3];
}

SHA_HD void words_to_bytes(const uint32_t w[8], uint8_t b[32]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        b[4 * i] = (uint8_t)(w[i] >> 24);
        b[4 * i + 1] = (uint8_t)(w[i] >> 16);
        b[4 * i + 2] = (uint8_t)(w[i] >> 8);
        b[4 * i + 3] = (uint8_t)w[i];
    }
}

}  // namespace sha

namespace ts {

constexpr uint32_t MAX_LABEL = 32;

// chaining value after the last whole block of the stream, the number of whole blocks, and
// the bytes of the unfinished block
struct State {
    uint32_t h[8];
    uint64_t nblk;
    uint8_t buf[64];
    uint32_t fill;
};

SHA_HD void compress_bytes(uint32_t h[8], const uint8_t blk[64]) {
    uint32_t w[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const uint8_t* p = blk + 4 * i;
        w[i] = ((uint32_t)p[0] << 24) | ((uint32_t)p[1] << 16) | ((uint32_t)p[2] << 8) | p[3];
    }
    sha::compress(h, w);
}

SHA_HD void push_byte(State& s, uint8_t b) {
    s.buf[s.fill++] = b;
    if (s.fill == 64) {
        compress_bytes(s.h, s.buf);
        s.nblk += 1;
        s.fill = 0;
    }
}

SHA_HD void init(State& s, uint64_t seed) {
    const uint32_t iv[8] = {0x6a09e667, 0xbb67ae85, 0x3c6ef372, 0xa54ff53a,
                            0x510e527f, 0x9b05688c, 0x1f83d9ab, 0x5be0cd19};
    for (int i = 0; i < 8; ++i) s.h[i] = iv[i];
    s.nblk = 0;
    s.fill = 0;
    const char dom[] = "zkdl-mi355x/v3";
    for (int i = 0; i < 56; ++i) push_byte(s, i < (int)sizeof(dom) - 1 ? (uint8_t)dom[i] : 0);
    for (int i = 0; i < 8; ++i) push_byte(s, (uint8_t)(seed >> (8 * i)));
}

// stream <- stream || u8(label_len) || label || u64le(n) || data
SHA_HD void absorb(State& s, const char* label, uint32_t label_len, const uint8_t* data, uint64_t n) {
    push_byte(s, (uint8_t)label_len);
    for (uint32_t i = 0; i < label_len; ++i) push_byte(s, (uint8_t)label[i]);
    for (int i = 0; i < 8; ++i) push_byte(s, (uint8_t)(n >> (8 * i)));
    for (uint64_t i = 0; i < n; ++i) push_byte(s, data[i]);
}

// SHA256(stream || tail), tail of at most 8 bytes, as big-endian words
SHA_HD void tail_digest_w(const State& s, const uint8_t* tail, uint32_t tail_len, uint32_t out[8]) {
    State f = s;
    const uint64_t bits = (s.nblk * 64 + s.fill + tail_len) * 8;
    for (uint32_t i = 0; i < tail_len; ++i) push_byte(f, tail[i]);
    push_byte(f, 0x80);
    while (f.fill != 56) push_byte(f, 0);
    for (int i = 7; i >= 0; --i) push_byte(f, (uint8_t)(bits >> (8 * i)));
    for (int i = 0; i < 8; ++i) out[i] = f.h[i];
}

// element idx of a draw (Montgomery form)
SHA_HD Fr challenge_elem(const State& s, uint32_t idx) {
    uint32_t d[2][8];
    for (uint32_t j = 0; j < 2; ++j) {
        const uint8_t tail[5] = {(uint8_t)(0xF0 + j), (uint8_t)idx, (uint8_t)(idx >> 8), (uint8_t)(idx >> 16),
                                 (uint8_t)(idx >> 24)};
        tail_digest_w(s, tail, 5, d[j]);
    }
    Fr lo, hi;
#pragma unroll
    for (int l = 0; l < 8; ++l) {
        lo.v[l] = sha::bswap32(d[0][l]);   // little-endian limbs of the digest bytes
        hi.v[l] = sha::bswap32(d[1][l]);
    }
    return fr_from_wide(lo, hi);
}

// the stream extension that follows a draw: 0xF2, then zeros up to the block boundary
SHA_HD void ratchet(State& s) {
    push_byte(s, 0xF2);
    while (s.fill != 0) push_byte(s, 0);
}

// canonical little-endian bytes of a Montgomery-form element
SHA_HD void fr_to_le(const Fr& mont, uint8_t out[32]) {
    Fr plain = fr_from_mont(mont);
#pragma unroll
    for (int l = 0; l < 8; ++l) {
        out[4 * l] = (uint8_t)plain.v[l];
        out[4 * l + 1] = (uint8_t)(plain.v[l] >> 8);
        out[4 * l + 2] = (uint8_t)(plain.v[l] >> 16);
        out[4 * l + 3] = (uint8_t)(plain.v[l] >> 24);
    }
}

// draw one challenge; returns it in Montgomery form and, if le_out != nullptr,
// as 32 canonical little-endian bytes
SHA_HD Fr challenge(State& s, uint8_t* le_out) {
    Fr c = challenge_elem(s, 0);
    ratchet(s);
    if (le_out) fr_to_le(c, le_out);
    return c;
}

SHA_HD void digest(const State& s, uint8_t out[32]) {
    uint32_t w[8];
    tail_digest_w(s, nullptr, 0, w);
    sha::words_to_bytes(w, out);
}

}  // namespace ts
