// Device helpers shared by the sumcheck kernels: block reduction of field
// elements, the block-cooperative transcript steps, Lagrange evaluation.
//
// Transcript steps are latency-bound (SHA-256 compressions are sequential), so
// whatever is independent is spread over lanes: the canonical forms of the
// elements to absorb, the message assembly, the three hashes of a challenge
// draw, the terms of the Lagrange sum.  All block_* functions must be called by
// every thread of the block (they contain barriers); blockDim.x >= 64.
#pragma once
#include "zkdl_internal.h"

// Sum of one Fr per thread over the block; result valid in thread 0.
// red: 64 words of LDS.
__device__ __forceinline__ Fr block_sum(Fr x, uint32_t* red) {
    const int tid = threadIdx.x;
    // first inside each wave with cross-lane shuffles, then across the waves via LDS
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        Fr y;
#pragma unroll
        for (int l = 0; l < 8; ++l) y.v[l] = __shfl_down(x.v[l], off, 64);
        x = fr_add(x, y);
    }
    const int wave = tid >> 6, lane = tid & 63;
    const int n_waves = (blockDim.x + 63) >> 6;
    __syncthreads();   // red may still be read from a previous call
    if (lane == 0) {
#pragma unroll
        for (int l = 0; l < 8; ++l) red[l * 8 + wave] = x.v[l];
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < n_waves; ++w) {
            Fr y;
#pragma unroll
            for (int l = 0; l < 8; ++l) y.v[l] = red[l * 8 + w];
            x = fr_add(x, y);
        }
    }
    return x;
}

// Sums N lazy values per thread (normal limbs, each below 2.41 r) over a block of at most
// 8 waves; thread j < N returns the fully reduced sum of value j, other threads zero.
// Limbs are added without carries: three shuffle levels take them from below 2^29 to below
// 2^32, a carry pass follows, three more levels, then a reducing pass (the wave's sum is
// below 64 * 2.41 r < 2^263); at most 8 such wave sums are added before the final reduction.
// red: BLOCK_SUM_LAZY_WORDS words of LDS.
constexpr int BLOCK_SUM_LAZY_WORDS = 8 * ZK_MAX_EVALS * 9;

// x plus the lane that the DPP control selects inside rows of 16 lanes (every lane of the row is a sum afterwards)
template <int CTRL>
__device__ __forceinline__ void f9_add_dpp(F9& s) {
#pragma unroll
    for (int l = 0; l < 9; ++l)
        s.v[l] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s.v[l], CTRL, 0xf, 0xf, true);
}

// Sum over the first `width` lanes of a wave (a power of two, the same in all lanes; the other lanes hold
// zero) of a lazy value (normal limbs, below 2.41 r); every lane must call; lane 0 returns the total, normal
// and below 1.1 r.  The levels inside a row of 16 lanes are DPP operands of the additions (one instruction
// per limb, no trip through the LDS crossbar): neighbours, pairs, halves of a row mirrored.
__device__ __forceinline__ F9 wave_sum_lazy(F9 s, int width = 64) {
    if (width > 1) {
        f9_add_dpp<0xB1>(s);        // quad_perm 1,0,3,2
        f9_add_dpp<0x4E>(s);        // quad_perm 2,3,0,1
        if (width > 4) {
            f9_add_dpp<0x141>(s);   // row_half_mirror
            s = f9_norm(s);
            f9_add_dpp<0x140>(s);   // row_mirror
        }
        if (width > 16) {
#pragma unroll
            for (int off = 16; off <= 32; off <<= 1)
#pragma unroll
                for (int l = 0; l < 9; ++l) s.v[l] += __shfl_down(s.v[l], off, 64);
        }
    }
    return f9_norm_reduce_sum(s);
}

template <int N>
__device__ __forceinline__ Fr block_sum_lazy(const F9 (&x)[N], uint32_t* red) {
    static_assert(N <= ZK_MAX_EVALS, "red is sized for ZK_MAX_EVALS values");
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int n_waves = (blockDim.x + 63) >> 6;
    F9 s[N];
#pragma unroll
    for (int j = 0; j < N; ++j) s[j] = wave_sum_lazy(x[j]);
    __syncthreads();   // red may still be read from a previous call
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int l = 0; l < 9; ++l) red[(wave * N + j) * 9 + l] = s[j].v[l];
    }
    __syncthreads();
    Fr out = fr_zero();
    if (tid < N) {
        F9 t = f9_zero();
        for (int w = 0; w < n_waves; ++w)
#pragma unroll
            for (int l = 0; l < 9; ++l) t.v[l] += red[(w * N + tid) * 9 + l];
        out = f9_to_fr(t);
    }
    return out;
}

constexpr int TS_MAX_ABSORB = 8;     // field elements per device-side absorb
constexpr int TS_MAX_DRAW = 64;      // challenges per block_challenges chunk
constexpr int TS_MAX_BLOCKS = 8;     // whole blocks one append may complete (ZK_PEND_CAP + 63 bytes)

constexpr int TS_WK_STRIDE = 68;     // words per schedule row: 64, and 4 so that rows begin on different banks

// LDS working set of the transcript steps
struct TsShared {
    uint32_t state[8];                       // chaining value after the last whole block of the stream
    uint64_t nblk;                           // whole blocks in the stream
    uint32_t fill;                           // bytes of the unfinished block
    uint32_t bufsel;                         // which of buf[] holds them
    uint32_t buf[2][16];                     // unfinished block, big-endian words, zero beyond fill
    uint32_t msg[16 * (TS_MAX_BLOCKS + 3)];  // blocks being absorbed, then a draw's three blocks
    alignas(16) uint32_t wk[TS_MAX_BLOCKS + 3][TS_WK_STRIDE];   // their schedules
    uint32_t seq;                            // groups of schedule words published (0 between steps)
    uint32_t k16[16];                        // the first sixteen round constants
    uint32_t canon[TS_MAX_ABSORB][8];        // canonical little-endian limbs being absorbed
    uint32_t dig[2 * TS_MAX_DRAW + 1][8];    // digests of a challenge draw
    Fr tmp[TS_MAX_ABSORB];
    Fr v;
};

__device__ __forceinline__ void block_ts_load(TsShared& S, const DevState* st) {
    if (threadIdx.x < 8) S.state[threadIdx.x] = st->ts_state[threadIdx.x];
    if (threadIdx.x >= 16 && threadIdx.x < 32) S.buf[0][threadIdx.x - 16] = st->ts_buf[threadIdx.x - 16];
    if (threadIdx.x >= 32 && threadIdx.x < 48) S.k16[threadIdx.x - 32] = sha::K_TABLE[threadIdx.x - 32];
    if (threadIdx.x == 8) {
        S.nblk = ((uint64_t)st->ts_nblk[1] << 32) | st->ts_nblk[0];
        S.fill = st->ts_fill;
        S.bufsel = 0;
        S.seq = 0;
    }
    __syncthreads();
}

__device__ __forceinline__ void block_ts_store(const TsShared& S, DevState* st) {
    __syncthreads();
    if (threadIdx.x < 8) st->ts_state[threadIdx.x] = S.state[threadIdx.x];
    if (threadIdx.x >= 16 && threadIdx.x < 32) st->ts_buf[threadIdx.x - 16] = S.buf[S.bufsel][threadIdx.x - 16];
    if (threadIdx.x == 8) {
        st->ts_nblk[0] = (uint32_t)S.nblk;
        st->ts_nblk[1] = (uint32_t)(S.nblk >> 32);
        st->ts_fill = S.fill;
    }
}

// Appends `len` bytes, given by frame(q), to the stream.  Lane j of wave 0 prepares the
// schedule of whole block j, then lane 0 runs the rounds block after block.  frame(q) may read
// S.canon; a barrier is taken first.
template <class FrameByte>
__device__ __forceinline__ void block_append(TsShared& S, uint32_t len, FrameByte frame) {
    __syncthreads();
    const uint32_t fill = S.fill, sel = S.bufsel;
    const uint32_t total = fill + len;
    const uint32_t nb = total / 64, rem = total % 64;
    const uint64_t nblk_after = S.nblk + nb;
    auto stream_byte = [&](uint32_t p) -> uint32_t {   // byte p counted from the start of the unfinished block
        if (p < fill) return (S.buf[sel][p >> 2] >> (24 - 8 * (p & 3))) & 0xffu;
        return frame(p - fill) & 0xffu;
    };
    // every thread builds whole words, byte by byte: the whole blocks, the new unfinished block
    for (uint32_t j = threadIdx.x; j < 16 * nb + 16; j += blockDim.x) {
        uint32_t word = 0;
        if (j < 16 * nb) {
#pragma unroll
            for (int b = 0; b < 4; ++b) word = (word << 8) | stream_byte(4 * j + b);
            S.msg[j] = word;
        } else {
            const uint32_t q0 = 4 * (j - 16 * nb);
#pragma unroll
            for (int b = 0; b < 4; ++b) word = (word << 8) | (q0 + b < rem ? stream_byte(64 * nb + q0 + b) : 0u);
            S.buf[sel ^ 1][j - 16 * nb] = word;
        }
    }
    __syncthreads();
    if (threadIdx.x < nb) {
        sha::Words16 w;
#pragma unroll
        for (int i = 0; i < 16; ++i) w.v[i] = S.msg[16 * threadIdx.x + i];
        sha::schedule_wk_lds(w, (sha::lds_u32_ptr)S.wk[threadIdx.x]);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (nb > 0) {
            sha::Words8 h;
#pragma unroll
            for (int i = 0; i < 8; ++i) h.v[i] = S.state[i];
            for (uint32_t blk = 0; blk < nb; ++blk) h = sha::rounds_lds(h, (sha::lds_u32_cptr)S.wk[blk]);
#pragma unroll
            for (int i = 0; i < 8; ++i) S.state[i] = h.v[i];
        }
        S.nblk = nblk_after;
        S.fill = rem;
        S.bufsel = sel ^ 1;
    }
    __syncthreads();
}

// stream <- stream || 0x01 || label || u64le(32 count) || canon[0..count) for a one-character
// label; canon must be complete (a barrier is taken first).
template <class Limb>
__device__ __forceinline__ uint32_t ts_frame1_byte(Limb limb, char label, uint32_t data_len, uint32_t q) {
    if (q == 0) return 1u;
    if (q == 1) return (uint32_t)(uint8_t)label;
    if (q < 10) return q - 2 < 4 ? (data_len >> (8 * (q - 2))) & 0xffu : 0u;
    const uint32_t d = q - 10;
    return d < data_len ? (limb(d >> 2) >> (8 * (d & 3))) & 0xffu : 0u;
}

__device__ inline void block_absorb1(TsShared& S, char label, int count) {
    const uint32_t data_len = 32u * (uint32_t)count;
    auto limb = [&](uint32_t i) -> uint32_t { return S.canon[i >> 3][i & 7]; };
    block_append(S, 10u + data_len, [&](uint32_t q) -> uint32_t { return ts_frame1_byte(limb, label, data_len, q); });
}

// canonical forms of vals[0..count) (Montgomery, LDS or global) -> proof words (if
// proof_dst) and into the transcript under a one-character label
__device__ inline void block_absorb_frs(TsShared& S, char label, const Fr* vals, int count,
                                        uint32_t* proof_dst) {
    if (threadIdx.x < (unsigned)count) {
        Fr plain = fr_from_mont_ni(vals[threadIdx.x]);
#pragma unroll
        for (int l = 0; l < 8; ++l) {
            S.canon[threadIdx.x][l] = plain.v[l];
            if (proof_dst) proof_dst[8 * threadIdx.x + l] = plain.v[l];
        }
    }
    block_absorb1(S, label, count);
}

// draws `count` challenges into st->chal[base..), st->chal_le; one stream extension.
// The first one is also left in S.v.  Works for any unfinished block (the closing blocks of
// a hash are two when it holds more than 50 bytes).  The blocks of all hashes differ in the tag and the index
// alone: the rest is put together once, word by word, and every lane adds its own bytes (each lane building its
// blocks byte by byte took longer than the compression).
__device__ inline void block_challenges(TsShared& S, DevState* st, int base, int count) {
    if (count <= 0) return;
    __syncthreads();
    const uint32_t rem = S.fill, sel = S.bufsel;
    const uint32_t last = rem + 14 > 64 ? 1u : 0u;
    const uint64_t bits = (S.nblk * 64u + rem + 5u) * 8u;
    // words 0..31: the closing blocks without tag and index (0x80 at byte rem + 5, the length at the end)
    if (threadIdx.x < 32) {
        const uint32_t i = threadIdx.x, p80 = rem + 5;
        uint32_t word = i < 16 && 4 * i < rem ? S.buf[sel][i] : 0u;
        if (i < 16 && 4 * i < rem && rem - 4 * i < 4) word &= ~(0xffffffffu >> (8 * (rem - 4 * i)));
        S.msg[48 + i] = word;                                   // the stream's own bytes (for the extension as well)
        if (i == p80 >> 2) word |= 0x80u << (24 - 8 * (p80 & 3));
        if (i == 16 * last + 14) word = (uint32_t)(bits >> 32);
        if (i == 16 * last + 15) word = (uint32_t)bits;
        S.msg[i] = word;
    }
    __syncthreads();
    for (int c0 = 0; c0 < count; c0 += TS_MAX_DRAW) {
        const int n = count - c0 < TS_MAX_DRAW ? count - c0 : TS_MAX_DRAW;
        const bool lastchunk = c0 + n >= count;
        const int jobs = 2 * n + (lastchunk ? 1 : 0);
        for (int t = threadIdx.x; t < jobs; t += blockDim.x) {
            sha::Words8 h;
#pragma unroll
            for (int i = 0; i < 8; ++i) h.v[i] = S.state[i];
            const bool elem = t < 2 * n;
            const uint32_t tag = elem ? 0xF0u + (uint32_t)(t & 1) : 0xF2u;
            const uint32_t idx = elem ? (uint32_t)(c0 + (t >> 1)) : 0u;
            const uint32_t nbk = elem ? last + 1 : 1u;
            // tag at byte rem, the index (below 2^16) little-endian behind it
            const uint64_t own = ((uint64_t)tag << 56) | ((uint64_t)(idx & 0xffu) << 48) | ((uint64_t)(idx >> 8) << 40);
            const uint32_t w0 = rem >> 2, sh = 8 * (rem & 3);
            const uint32_t o0 = (uint32_t)(own >> (32 + sh)), o1 = (uint32_t)((own >> sh) & 0xffffffffu);
            for (uint32_t blk = 0; blk < nbk; ++blk) {
                sha::Words16 w;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const uint32_t k = 16 * blk + i;
                    w.v[i] = S.msg[(elem ? 0u : 48u) + k] | (k == w0 ? o0 : 0u) | (k == w0 + 1 ? o1 : 0u);
                }
                h = sha::compress_ni(h, w);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) S.dig[t][i] = h.v[i];
        }
        __syncthreads();
        // wide reduction: one lane per half, then one lane per element
        for (int t = threadIdx.x; t < 2 * n; t += blockDim.x) {
            Fr x;
#pragma unroll
            for (int l = 0; l < 8; ++l) x.v[l] = sha::bswap32(S.dig[t][l]);
            Fr m = fr_mul_ni(fr_const((t & 1) ? frc::W3 : frc::R2), x);
#pragma unroll
            for (int l = 0; l < 8; ++l) S.dig[t][l] = m.v[l];
        }
        __syncthreads();
        for (int t = threadIdx.x; t < n; t += blockDim.x) {
            Fr lo, hi;
#pragma unroll
            for (int l = 0; l < 8; ++l) {
                lo.v[l] = S.dig[2 * t][l];
                hi.v[l] = S.dig[2 * t + 1][l];
            }
            Fr c = fr_add(lo, hi);
            st->chal[base + c0 + t] = c;
            if (c0 + t == 0) S.v = c;
            Fr plain = fr_from_mont_ni(c);
            uint32_t* le = (uint32_t*)(st->chal_le + 32 * (size_t)(base + c0 + t));
#pragma unroll
            for (int l = 0; l < 8; ++l) le[l] = plain.v[l];
        }
        __syncthreads();
        if (lastchunk) {
            if (threadIdx.x < 8) S.state[threadIdx.x] = S.dig[2 * n][threadIdx.x];
            if (threadIdx.x == 8) {
                S.nblk += 1;
                S.fill = 0;
            }
        }
        __syncthreads();
    }
}

// g(v) from the prepared Lagrange coefficients c[k] = g(k) / prod_{j != k} (k - j), npts = 2..4,
// by one wave (all 64 lanes call, no barrier inside); lane 0 returns the value.
//   npts = 4: g(v) = (v-2)(v-3) [c0 (v-1) + c1 v] + v (v-1) [c2 (v-3) + c3 (v-2)]
//   npts = 3: g(v) = (v-2) [c0 (v-1) + c1 v] + c2 v (v-1)
//   npts = 2: g(v) = c0 (v-1) + c1 v
// The operands of each level are selected per lane and multiplied by one call: lanes that
// branch to separate calls would run them one after the other.
__device__ inline Fr wave_lagrange(const Fr* c, int npts, const Fr& v) {
    const int lane = threadIdx.x & 63;
    const Fr one = fr_one();
    const Fr v1 = fr_sub(v, one), v2 = fr_sub(v1, one), v3 = fr_sub(v2, one);
    // level 1, lanes 0..5: c0 (v-1), c1 v, c2 (v-3) | c2 v, c3 (v-2), (v-2)(v-3), v (v-1)
    Fr A = lane == 4 ? v2 : v;
    if (lane < npts) A = c[lane];
    Fr B = lane == 1 ? v : v1;
    if (npts == 4) {
        if (lane == 2 || lane == 4) B = v3;
        else if (lane == 3) B = v2;
    } else if (lane == 2) {
        B = v;
    }
    const Fr p = fr_mul_ni(A, B);
    // level 2, lanes 0, 1
    Fr qa, qb, qc;   // products of lanes 2 lane, 2 lane + 1, 4 + lane
#pragma unroll
    for (int l = 0; l < 8; ++l) {
        qa.v[l] = __shfl(p.v[l], (2 * lane) & 63, 64);
        qb.v[l] = __shfl(p.v[l], (2 * lane + 1) & 63, 64);
        qc.v[l] = __shfl(p.v[l], (4 + lane) & 63, 64);
    }
    Fr r;
    if (npts == 2) {
        r = fr_add(qa, qb);   // lane 0: q0 + q1
    } else {
        Fr A2, B2;
        if (npts == 4) {
            A2 = qc;                   // lane 0: (v-2)(v-3), lane 1: v (v-1)
            B2 = fr_add(qa, qb);       // lane 0: q0 + q1, lane 1: q2 + q3
        } else {
            A2 = lane == 0 ? v2 : qa;  // lane 1: q2 = c2 v
            B2 = lane == 0 ? fr_add(qa, qb) : v1;
        }
        r = fr_mul_ni(A2, B2);
        Fr r1;
#pragma unroll
        for (int l = 0; l < 8; ++l) r1.v[l] = __shfl(r.v[l], 1, 64);
        r = fr_add(r, r1);
    }
    return r;
}

// The claim of the last finished round may still be owed: a round kernel needs only the
// challenge, so the evaluation g_t(v_t) is left to whoever needs the claim next, who does it
// in a spare wave next to other work.  One wave calls this; afterwards st->claim is current.
__device__ inline void wave_resolve_claim(DevState* st) {
    const uint32_t npts = st->lag_npts;   // wave-uniform
    if (npts) {
        const Fr c = wave_lagrange(st->lag, (int)npts, st->chal[st->lag_chal]);
        if ((threadIdx.x & 63) == 0) {
            st->claim = c;
            st->lag_npts = 0;
        }
    }
}

// A frame of `count` <= 3 elements and a draw of one challenge, for an unfinished block after the frame of at
// most 50 bytes (one closing block per hash): the step of every round.  Wave 0 runs the rounds (lane 0 the `nb`
// whole blocks that the frame completes - one after a draw, when the stream is block-aligned - then lanes 0..2
// the draw's three), wave 1 the schedules of all blocks side by side, sixteen words ahead; the other waves only
// meet the closing barrier.  Bound by the two dependent compressions: 64 rounds of 14 instructions at 5.4 cycles, what
// one wave issues, are 4.8 thousand cycles; in the verifier they take 5.8 to 8.1 and, the draw's with the first product
// of the reduction, 7.4 to 10.8, next to 1.3 for building the blocks and 1.3 for the rest.  With the steps one after the other in block-wide phases (six barriers) the 2^10-entry
// sumcheck of two tables took 231 us, like this and with the work beside it in wave 2, 191 us.  Leaves v in S.v
// and the new chaining value in S.state.
// limb(i): limb i % 8 of the i / 8-th element (canonical).
template <class Limb>
__device__ __forceinline__ void wave_frame_draw1(TsShared& S, char label, int count, Limb limb) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t data_len = 32u * (uint32_t)count, fill = S.fill, total = fill + 10u + data_len;
    const uint32_t nb = total >> 6, rem = total & 63;
    if (wave < 2) {
        const uint64_t bits = ((S.nblk + nb) * 64u + rem + 5u) * 8u;
        const uint32_t nlimb = 8u * (uint32_t)count, sel = S.bufsel, wr = rem >> 2;
        // blocks in rows: the whole ones, then the draw's three (the two closing blocks, the extension)
        for (uint32_t j = lane; j < 16 * (nb + 3); j += 64) {
            const uint32_t row = j >> 4, i = j & 15;
            const bool draw = row >= nb;
            const uint32_t k = draw ? 16 * nb + i : j, t = row - nb;   // word k of the stream from the unfinished block on
            uint32_t word = 0;
            if (fill == 0) {
                // data start at byte 10: a word is the upper half of one limb and the lower half of the next
                const uint32_t ip = k - 3, in = k - 2;
                const uint32_t lp = (k >= 3 && ip < nlimb) ? limb(ip) : 0u;
                const uint32_t ln = (k >= 2 && in < nlimb) ? limb(in) : 0u;
                word = (((lp >> 16) & 0xffu) << 24) | ((lp >> 24) << 16) | ((ln & 0xffu) << 8) | ((ln >> 8) & 0xffu);
                if (k == 0) word = (1u << 24) | ((uint32_t)(uint8_t)label << 16) | ((data_len & 0xffu) << 8);
            } else {
#pragma unroll
                for (uint32_t b = 0; b < 4; ++b) {
                    const uint32_t p = 4 * k + b;
                    const uint32_t x = p < fill ? (S.buf[sel][p >> 2] >> (24 - 8 * (p & 3))) & 0xffu
                                       : p < total ? ts_frame1_byte(limb, label, data_len, p - fill) : 0u;
                    word = (word << 8) | x;
                }
            }
            if (draw) {
                // tag at byte rem, four zero index bytes, then 0x80 in the hashes (not in the extension)
                const uint32_t sh = 24 - 8 * (rem & 3);
                if (i == wr) word |= (0xF0u + t) << sh;
                if (t < 2) {
                    if (i == (rem + 5) >> 2) word |= 0x80u << (24 - 8 * ((rem + 5) & 3));
                    if (i == 14) word = (uint32_t)(bits >> 32);
                    if (i == 15) word = (uint32_t)bits;
                }
            }
            if (wave == 0) S.wk[row][i] = word + S.k16[i];
            else S.msg[j] = word;     // the schedule wave's own copy: its lane r reads row r back
        }
        __builtin_amdgcn_wave_barrier();   // LDS operations of a wave complete in order: no wait needed
        if (wave == 0) {
            sha::Words8 h;
#pragma unroll
            for (int q = 0; q < 8; ++q) h.v[q] = S.state[q];
            for (uint32_t blk = 0; blk < nb; ++blk) {
                if (lane == 0) h = sha::rounds_behind(h, (sha::lds_u32_cptr)S.wk[blk], (sha::lds_u32_ptr)&S.seq);
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) h.v[q] = __builtin_amdgcn_readfirstlane(h.v[q]);
            Fr m = fr_zero();
            if (lane < 3) {
                const sha::Words8 ow =
                    sha::rounds_behind(h, (sha::lds_u32_cptr)S.wk[nb + lane], (sha::lds_u32_ptr)&S.seq);
                if (lane == 2) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) S.state[q] = ow.v[q];
                } else {
                    Fr x;
#pragma unroll
                    for (int l = 0; l < 8; ++l) x.v[l] = sha::bswap32(ow.v[l]);
                    m = fr_mul_ni(fr_const(lane ? frc::W3 : frc::R2), x);
                }
            }
            Fr lo, hi;
#pragma unroll
            for (int l = 0; l < 8; ++l) {
                lo.v[l] = __builtin_amdgcn_readlane(m.v[l], 0);
                hi.v[l] = __builtin_amdgcn_readlane(m.v[l], 1);
            }
            const Fr v = fr_add(lo, hi);
            if (lane == 0) {
                S.v = v;
                S.nblk += nb + 1;
                S.fill = 0;
                S.seq = 0;      // the schedule wave has published its last group: it was waited for
            }
        } else if (lane < (int)nb + 3) {
            sha::Words16 w;
#pragma unroll
            for (int q = 0; q < 16; ++q) w.v[q] = S.msg[16 * lane + q];
            sha::schedule_ahead(w, (sha::lds_u32_ptr)S.wk[lane], (sha::lds_u32_ptr)&S.seq);
        }
    }
    __syncthreads();
}

__device__ __forceinline__ bool frame_draw1_fits(const TsShared& S, int count) {
    return count <= 3 && ((S.fill + 10u + 32u * (uint32_t)count) & 63) <= 50;
}

// S.canon[0..count) go into the transcript under a one-character label, then one challenge is drawn: it is
// returned to every thread and stored in st->chal[chal_idx] (Montgomery form) and st->chal_le (canonical).
// side() is run by wave 2 while the hashes run (no barrier inside).  Needs blockDim.x >= 192.
template <class Side>
__device__ inline Fr block_absorb_draw1_side(TsShared& S, DevState* st, char label, int count, int chal_idx, Side side) {
    const int tid = threadIdx.x;
    __syncthreads();
    Fr v;
    if (frame_draw1_fits(S, count)) {
        if ((tid >> 6) == 2) side();
        wave_frame_draw1(S, label, count, [&](uint32_t i) -> uint32_t { return S.canon[i >> 3][i & 7]; });
        v = S.v;
        if (tid == (int)blockDim.x - 64) {   // a lane of the last wave
            const Fr plain = fr_from_mont_ni(v);
            uint32_t* le = (uint32_t*)(st->chal_le + 32 * (size_t)chal_idx);
#pragma unroll
            for (int l = 0; l < 8; ++l) le[l] = plain.v[l];
        }
    } else {
        // the unfinished block leaves no room for single closing blocks: the general steps
        if ((tid >> 6) == 2) side();
        block_absorb1(S, label, count);
        block_challenges(S, st, chal_idx, 1);
        v = S.v;
    }
    if (tid == 0) st->chal[chal_idx] = v;
    return v;
}

__device__ inline Fr block_absorb_draw1(TsShared& S, DevState* st, char label, int count, int chal_idx) {
    return block_absorb_draw1_side(S, st, label, count, chal_idx, [] {});
}

// First part of closing a round: g_t(0..npts-1) (LDS, Montgomery, npts = 2..4) go to the proof
// and into the transcript, the round's challenge v_t is drawn and returned to every thread.
// The Lagrange coefficients of g_t are left in S.tmp[0..npts) for the claim g_t(v_t).
// Needs blockDim.x >= 192: while wave 0 hashes, wave 1 prepares the coefficients and wave 2
// later writes the canonical form of the challenge.
__device__ inline Fr block_round_challenge(TsShared& S, DevState* st, const Fr* g, int npts,
                                           uint32_t proof_off, int chal_idx, char label = 'g',
                                           bool skip1 = true) {
    const int tid = threadIdx.x;
    uint32_t* proof_dst = (uint32_t*)(st->proof + proof_off);
    __syncthreads();
    // canonical forms (wave 0) | Lagrange coefficients (wave 1).  The transcript takes
    // g(0), g(2), .., g(npts-1): g(1) is fixed by the claim the transcript already determines.
    // (skip1 = false, the f_t of the optimized matrix-product protocol: all evaluations.)
    if (tid < npts) {
        Fr plain = fr_from_mont_ni(g[tid]);
        const int slot = (!skip1 || tid == 0) ? tid : tid - 1;
#pragma unroll
        for (int l = 0; l < 8; ++l) {
            if (!skip1 || tid != 1) S.canon[slot][l] = plain.v[l];
            proof_dst[8 * tid + l] = plain.v[l];
        }
    } else if (tid >= 64 && tid < 64 + npts) {
        const int k = tid - 64;
        Fr c = g[k];
        if (npts == 3) {            // 1/2, -1, 1/2
            c = (k == 1) ? fr_neg(c) : fr_mul_ni(c, st->inv2);
        } else if (npts == 4) {     // -1/6, 1/2, -1/2, 1/6
            c = fr_mul_ni(c, (k == 0 || k == 3) ? st->inv6 : st->inv2);
            if (k == 0 || k == 2) c = fr_neg(c);
        } else if (k == 0) {        // -1, 1
            c = fr_neg(c);
        }
        S.tmp[k] = c;
    }
    return block_absorb_draw1(S, st, label, skip1 ? npts - 1 : npts, chal_idx);
}

// ---- closing a round without waiting for what the transcript does not need ----------------------
// The transcript takes g(0), g(2), ..: the evaluation g(1) = claim - g(0), the coefficients of g and the claim
// itself are needed by the proof bytes and by the round after next at the earliest, so wave 2 works them out
// while waves 0 and 1 hash (two passes of 6 to 11 thousand cycles each), and the canonical form of a sum is taken
// by the lane that has just finished the sum.
struct RoundShared {
    F9 g9[ZK_MAX_EVALS];      // the evaluations summed in this round, lazy
    F9 coef[ZK_MAX_EVALS];    // 1 / prod_{j != k} (k - j) for the number of points in use
    Fr lag[ZK_MAX_EVALS];     // Lagrange coefficients of the last closed round
    Fr claim;                 // current if owed == 0, else claim = g(v_prev) with the coefficients lag[]
    Fr v_prev;
    uint32_t owed;            // number of coefficients
};

// once per kernel, between two barriers of the caller; npts = 2..4
__device__ inline void round_begin(RoundShared& R, const DevState* st, int npts) {
    const int tid = threadIdx.x;
    if (tid >= 128 && tid < 128 + npts) {
        const int k = tid - 128;
        Fr c;
        if (npts == 4) c = (k == 0 || k == 3) ? st->inv6 : st->inv2;         // -1/6, 1/2, -1/2, 1/6
        else c = (npts == 3 && k != 1) ? st->inv2 : fr_one();                // 1/2, -1, 1/2; -1, 1
        const bool neg = npts == 4 ? (k == 0 || k == 2) : npts == 3 ? k == 1 : k == 0;
        R.coef[k] = fr_unpack(neg ? fr_neg(c) : c);
    } else if (tid == 64) {
        R.claim = st->claim;
        R.owed = st->lag_npts;
        R.v_prev = st->chal[st->lag_npts ? st->lag_chal : 0];
    } else if (tid > 64 && tid <= 64 + ZK_MAX_EVALS) {
        R.lag[tid - 65] = st->lag[tid - 65];
    }
}

// one thread: evaluation x of the round, a lazy sum (normal, below 2.41 r), to the proof and to the transcript's
// inputs (skip1: the transcript does not take x = 1)
__device__ __forceinline__ void round_eval_out(TsShared& S, RoundShared& R, uint32_t* proof_dst, int x, const F9& s,
                                               bool skip1) {
    R.g9[x] = s;
    const Fr plain = f9_canonical(s);
    const int slot = (!skip1 || x == 0) ? x : x - 1;
    if (!skip1 || x != 1) {
#pragma unroll
        for (int l = 0; l < 8; ++l) S.canon[slot][l] = plain.v[l];
    }
#pragma unroll
    for (int l = 0; l < 8; ++l) proof_dst[8 * x + l] = plain.v[l];
}

// wave 2, next to the hashes: the claim if it is owed, g(1) if it is derived, the coefficients of g
__device__ inline void wave_round_side(RoundShared& R, int npts, bool derive1, uint32_t* proof_dst) {
    const int lane = threadIdx.x & 63;
    if (derive1 && R.owed) {
        const Fr c = wave_lagrange(R.lag, (int)R.owed, R.v_prev);
        if (lane == 0) R.claim = c;
    }
    __builtin_amdgcn_wave_barrier();
    if (lane < npts) {
        F9 g = R.g9[lane];
        if (derive1 && lane == 1) {
            g = f9_norm(f9_sub(fr_unpack(R.claim), R.g9[0]));
            const Fr plain = f9_canonical(g);
#pragma unroll
            for (int l = 0; l < 8; ++l) proof_dst[8 + l] = plain.v[l];
        }
        R.lag[lane] = fr_pack(f9_cond_sub(f9_mul(g, R.coef[lane])));
    }
    if (lane == 0) R.owed = (uint32_t)npts;
}

// Closes a round whose sums have gone through round_eval_out: the challenge, to every thread.  The claim
// g(v) stays owed in R (to the next round, or to the next kernel after round_end).
__device__ inline Fr block_close_round(TsShared& S, RoundShared& R, DevState* st, int npts, bool derive1, uint32_t proof_off,
                                       int chal_idx, char label = 'g', bool skip1 = true) {
    uint32_t* proof_dst = (uint32_t*)(st->proof + proof_off);
    const Fr v = block_absorb_draw1_side(S, st, label, skip1 ? npts - 1 : npts, chal_idx,
                                         [&] { wave_round_side(R, npts, derive1, proof_dst); });
    if (threadIdx.x == 0) R.v_prev = v;   // read by wave 2 after the next barrier
    return v;
}

// leaves the owed claim to the next kernel (after the last block_close_round)
__device__ inline void round_end(const RoundShared& R, DevState* st, int npts, int chal_idx) {
    const int tid = threadIdx.x;
    if (tid >= 64 && tid < 64 + npts) st->lag[tid - 64] = R.lag[tid - 64];
    if (tid == 64) {
        st->lag_npts = (uint32_t)npts;
        st->lag_chal = (uint32_t)chal_idx;
    }
}

// Closes a round completely: challenge, then the next claim g_t(v_t) in st->claim.
__device__ inline Fr block_finalise_round(TsShared& S, DevState* st, const Fr* g, int npts,
                                          uint32_t proof_off, int chal_idx) {
    const Fr v = block_round_challenge(S, st, g, npts, proof_off, chal_idx);
    if ((threadIdx.x >> 6) == 1) {
        const Fr c = wave_lagrange(S.tmp, npts, v);
        if ((threadIdx.x & 63) == 0) st->claim = c;
    }
    __syncthreads();
    return v;
}

// Lazy sum of the partial sums part[b * npts + x], b < nblk (reduced values), by one wave; lane 0 returns it
__device__ __forceinline__ F9 wave_reduce_partials(const Fr* part, int nblk, int npts, int x) {
    const int lane = threadIdx.x & 63;
    F9 s = f9_zero();
    // up to eight rows of 64 partials at a time, their loads issued together: the loop is
    // bound by memory latency
    for (int base = 0; base < nblk; base += 512) {
        const int rows = (nblk - base + 63) / 64 < 8 ? (nblk - base + 63) / 64 : 8;   // wave-uniform
        Fr p[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (q < rows) {
                const int b = base + 64 * q + lane;
                p[q] = b < nblk ? part[(uint64_t)b * npts + x] : fr_zero();
            }
        }
        // limbs: at most 2^29 + 7 * 2^29 between two reductions
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (q < rows) s = q == 7 ? f9_add(f9_norm(s), fr_unpack(p[q])) : f9_add(s, fr_unpack(p[q]));
        s = f9_norm_reduce(s);
    }
    return wave_sum_lazy(s, nblk >= 64 ? 64 : nblk > 32 ? 64 : nblk > 16 ? 32 : nblk > 4 ? 16 : nblk > 1 ? 4 : 1);
}

// Sums per-block partial sums part[b * npts + x], b < nblk, into g[x] (LDS): wave x
// handles evaluation x on its own.  Needs blockDim.x >= 64 * npts.
__device__ inline void block_reduce_partials(const Fr* part, int nblk, int npts, Fr* g) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (wave < npts) {
        Fr s = fr_zero();
        // up to eight rows of 64 partials at a time, their loads issued together: the loop is
        // bound by memory latency
        for (int base = 0; base < nblk; base += 512) {
            const int rows = (nblk - base + 63) / 64 < 8 ? (nblk - base + 63) / 64 : 8;   // wave-uniform
            Fr p[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (q < rows) {
                    const int b = base + 64 * q + lane;
                    p[q] = b < nblk ? part[(uint64_t)b * npts + wave] : fr_zero();
                }
            }
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (q < rows) s = fr_add(s, p[q]);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            Fr y;
#pragma unroll
            for (int l = 0; l < 8; ++l) y.v[l] = __shfl_down(s.v[l], off, 64);
            s = fr_add(s, y);
        }
        if (lane == 0) g[wave] = s;
    }
    __syncthreads();
}

// ---- Montgomery form times plain integer --------------------------------------------------------
// A value in Montgomery form times a plain integer is the Montgomery form of the product: such
// products are accumulated as 64-bit columns of 29-bit limb products with no reduction, and reduced
// once per thread or per output.
// cols += c * mag for a normal or negated-normal c (limbs below 2^30.6) and mag < 2^58
__device__ __forceinline__ void cols11_mac(uint64_t* cols, const F9& c, uint64_t mag) {
    const uint32_t m0 = (uint32_t)mag & frc::M29, m1 = (uint32_t)(mag >> 29);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        cols[i] += (uint64_t)c.v[i] * m0;
        cols[i + 1] += (uint64_t)c.v[i] * m1;
    }
}

// cols += p * c for a signed c, |c| < 2^58, and a normal p below 2.6 r: a negative c turns p
// into 4r - p
__device__ __forceinline__ void cols11_mac_signed(uint64_t* cols, const F9& p, int64_t c) {
    const bool neg = c < 0;
    const uint64_t mag = neg ? (uint64_t)0 - (uint64_t)c : (uint64_t)c;
    F9 q;
#pragma unroll
    for (int i = 0; i < 9; ++i) q.v[i] = neg ? frc::C4R[i] - p.v[i] : p.v[i];
    cols11_mac(cols, q, mag);
}

// carries of an 11-column accumulator: columns 0..9 below 2^29 afterwards
__device__ __forceinline__ void cols11_carry(uint64_t* cols) {
#pragma unroll
    for (int k = 0; k + 1 < 11; ++k) {
        cols[k + 1] += cols[k] >> 29;
        cols[k] &= frc::M29;
    }
}

// carried 11-column sum V -> lazy value congruent to it, normal and below 2.41 r:
// V = low nine limbs + 2^261 * high part, and 2^261 is the Montgomery radix, so the high part
// times R^2 as a Montgomery product is congruent to 2^261 * high part
__device__ __forceinline__ F9 cols11_value(const uint64_t* cols) {
    F9 vlo, vhi = f9_zero();
#pragma unroll
    for (int i = 0; i < 9; ++i) vlo.v[i] = (uint32_t)cols[i];
    vhi.v[0] = (uint32_t)cols[9];
    vhi.v[1] = (uint32_t)cols[10] & frc::M29;
    vhi.v[2] = (uint32_t)(cols[10] >> 29) & frc::M29;
    vhi.v[3] = (uint32_t)(cols[10] >> 58);
    return f9_norm_reduce(f9_add(vlo, f9_mul(vhi, fr_unpack(fr_const(frc::R2)))));
}

// a0 + v0 (a2 - a0) in Montgomery form from the integers; k = (R^2, -R^2, v0 R^2, -v0 R^2),
// canonical.  Four products below 2^58 per column; the result is normal and below 2 r.
__device__ __forceinline__ F9 fold_ints(const F9* k, int64_t a0, int64_t a2) {
    const int64_t d = a2 - a0;
    const bool n0 = a0 < 0, nd = d < 0;
    uint64_t cols[17];
#pragma unroll
    for (int c = 0; c < 17; ++c) cols[c] = 0;
    F9 c0, cd;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        c0.v[i] = n0 ? k[1].v[i] : k[0].v[i];
        cd.v[i] = nd ? k[3].v[i] : k[2].v[i];
    }
    cols11_mac(cols, c0, n0 ? (uint64_t)0 - (uint64_t)a0 : (uint64_t)a0);
    cols11_mac(cols, cd, nd ? (uint64_t)0 - (uint64_t)d : (uint64_t)d);
    return f9_redc(cols);
}

// ---- launchers defined in k_sumcheck.hip ----
void zk_launch_finalise(zkdl_ctx* ctx, int nblk, int npts, int chal_idx, uint32_t proof_off, int first,
                        uint32_t claim_off, int derive1);
