// Device helpers shared by the sumcheck kernels: block reduction of field
// elements, the block-cooperative transcript steps, Lagrange evaluation.
//
// Transcript steps are latency-bound (SHA-256 compressions are sequential), so
// whatever is independent is spread over lanes: the canonical forms of the
// elements to absorb, the message assembly, the three hashes of a challenge
// draw, the terms of the Lagrange sum.  All block_* functions must be called by
// every thread of the block (they contain barriers).  Sums take any whole number of waves; a
// transcript step takes two at least, for wave 1 fills part of the working set and runs the
// schedules that wave 0 waits for; closing a round takes the wave of its side work besides.
#pragma once
#include "zkdl_internal.h"

constexpr int TS_MIN_THREADS = 128;       // block_ts_load, block_append, absorbs and draws
constexpr int ROUND_SIDE_WAVE = 2;        // block_close_round's side work, unless told another wave
static_assert(ZK_BLOCK >= TS_MIN_THREADS && ZK_BLOCK >= 64 * (ROUND_SIDE_WAVE + 1), "blocks that close rounds");

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
    alignas(16) uint32_t msg[16 * (TS_MAX_BLOCKS + 3)];   // blocks being absorbed, then a draw's three blocks
    alignas(16) uint32_t wk[TS_MAX_BLOCKS + 3][TS_WK_STRIDE];   // their schedules from word 16 on
    uint32_t seq;                            // groups of schedule words published (0 between steps)
    alignas(16) uint32_t k64[64];            // the round constants
    alignas(16) uint32_t zero16[16];         // what the low lanes of a compression read for their schedule
    uint32_t canon[TS_MAX_ABSORB][8];        // canonical little-endian limbs being absorbed
    uint32_t claim[8];                       // the same of a claim absorbed in front of them
    uint32_t dig[2 * TS_MAX_DRAW + 1][8];    // digests of a challenge draw
    Fr tmp[TS_MAX_ABSORB];
    F9 v9;                                   // wave_frame_draw1's challenge: normal, below 2.1 r
    Fr v;
};

// the parts of the working set that never change (blockDim.x >= TS_MIN_THREADS)
__device__ __forceinline__ void block_ts_constants(TsShared& S) {
    if (threadIdx.x >= 64 && threadIdx.x < 128) S.k64[threadIdx.x - 64] = sha::K_TABLE[threadIdx.x - 64];
    if (threadIdx.x >= 48 && threadIdx.x < 64) S.zero16[threadIdx.x - 48] = 0;
}

// open: no barrier behind it (the caller's next one will do)
__device__ __forceinline__ void block_ts_load(TsShared& S, const DevState* st, bool open = false) {
    if (threadIdx.x < 8) S.state[threadIdx.x] = st->ts_state[threadIdx.x];
    if (threadIdx.x >= 16 && threadIdx.x < 32) S.buf[0][threadIdx.x - 16] = st->ts_buf[threadIdx.x - 16];
    block_ts_constants(S);
    if (threadIdx.x == 8) {
        S.nblk = ((uint64_t)st->ts_nblk[1] << 32) | st->ts_nblk[0];
        S.fill = st->ts_fill;
        S.bufsel = 0;
        S.seq = 0;
    }
    if (!open) __syncthreads();
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

// chaining value halves of a wave's lanes, from and to S.state
__device__ __forceinline__ sha::Half ts_state_half(const TsShared& S) {
    sha::Half h;
    const int o = sha::half_is_high() ? 4 : 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) h.v[q] = S.state[o + q];
    return h;
}
__device__ __forceinline__ void ts_state_store(TsShared& S, const sha::Half& h) {
    const int o = sha::half_is_high() ? 4 : 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) S.state[o + q] = h.v[q];
}
// the compression of block row `row` for the calling lane (wave 0; wave 1 runs the schedules)
__device__ __forceinline__ sha::Half ts_rounds(TsShared& S, const sha::Half& h, uint32_t row, uint32_t base = 0) {
    const bool high = sha::half_is_high();
    const sha::lds_u32_cptr zero = (sha::lds_u32_cptr)S.zero16;
    return sha::rounds_behind(h, high ? (sha::lds_u32_cptr)(S.msg + 16 * row) : zero, high ? (sha::lds_u32_cptr)S.k64 : zero,
                              high ? (sha::lds_u32_cptr)S.wk[row] : zero, high ? 16u : 0u, (sha::lds_u32_vptr)&S.seq, base);
}
// wave 1: the schedules of rows 0 .. n-1 from S.msg
__device__ __forceinline__ void ts_schedules(TsShared& S, uint32_t n, uint32_t base = 0) {
    uint32_t row = sha::half_row();
    if (row >= n) row = 0;         // lanes without a row of their own do the first one's again, see spec_product_coefficients
    if (n > 0)
        sha::schedule_ahead((sha::lds_u32_cptr)(S.msg + 16 * row), (sha::lds_u32_ptr)S.wk[row], (sha::lds_u32_cptr)S.k64,
                            (sha::lds_u32_vptr)&S.seq, base);
}

// Appends `len` bytes, given by frame(q), to the stream.  A lane pair of wave 1 per whole block prepares the
// schedules, sixteen words ahead of wave 0, which runs the rounds block after block.  frame(q) may read S.canon; a
// barrier is taken first.  Needs blockDim.x >= TS_MIN_THREADS.
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
    if (threadIdx.x < 64) {
        if (threadIdx.x < 8 && nb > 0) {
            sha::Half h = ts_state_half(S);
            for (uint32_t blk = 0; blk < nb; ++blk) h = ts_rounds(S, h, blk);
            if ((threadIdx.x & 3) == (sha::half_is_high() ? 3 : 0)) ts_state_store(S, h);    // lanes 0 and 7
        }
        if (threadIdx.x == 0) {
            S.nblk = nblk_after;
            S.fill = rem;
            S.bufsel = sel ^ 1;
            S.seq = 0;      // the schedule wave has published its last group: it was waited for
        }
    } else if (threadIdx.x < 128) {
        ts_schedules(S, nb);
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

// The general steps are out of line, one copy per kernel each; they are given the working set as an LDS pointer (a
// generic one would make every access to it a flat instruction).
typedef __attribute__((address_space(3))) TsShared* TsLds;

static __device__ __noinline__ void block_absorb1_ni(TsLds s, char label, int count) {
    TsShared& S = *(TsShared*)s;
    const uint32_t data_len = 32u * (uint32_t)count;
    auto limb = [&](uint32_t i) -> uint32_t { return S.canon[i >> 3][i & 7]; };
    block_append(S, 10u + data_len, [&](uint32_t q) -> uint32_t { return ts_frame1_byte(limb, label, data_len, q); });
}
__device__ __forceinline__ void block_absorb1(TsShared& S, char label, int count) {
    block_absorb1_ni((TsLds)&S, label, count);
}

// canonical forms of vals[0..count) (Montgomery, LDS or global) -> proof words (if
// proof_dst) and into the transcript under a one-character label
__device__ __forceinline__ void block_absorb_frs(TsShared& S, char label, const Fr* vals, int count,
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
static __device__ __noinline__ void block_challenges_ni(TsLds s, DevState* st, int base, int count) {
    TsShared& S = *(TsShared*)s;
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

__device__ __forceinline__ void block_challenges(TsShared& S, DevState* st, int base, int count) {
    block_challenges_ni((TsLds)&S, st, base, count);
}

// g(v) from the prepared Lagrange coefficients c[k] = g(k) / prod_{j != k} (k - j), npts = 2..4,
// by one wave (all 64 lanes call, no barrier inside); lane k < npts holds c[k]; lane 0 returns the value.
//   npts = 4: g(v) = (v-2)(v-3) [c0 (v-1) + c1 v] + v (v-1) [c2 (v-3) + c3 (v-2)]
//   npts = 3: g(v) = (v-2) [c0 (v-1) + c1 v] + c2 v (v-1)
//   npts = 2: g(v) = c0 (v-1) + c1 v
// The operands of each level are selected per lane and multiplied by one call: lanes that
// branch to separate calls would run them one after the other.
static __device__ __noinline__ Fr wave_lagrange_ni(Fr ck, int npts, Fr v) {
    const int lane = threadIdx.x & 63;
    const Fr one = fr_one();
    const Fr v1 = fr_sub(v, one), v2 = fr_sub(v1, one), v3 = fr_sub(v2, one);
    // level 1, lanes 0..5: c0 (v-1), c1 v, c2 (v-3) | c2 v, c3 (v-2), (v-2)(v-3), v (v-1)
    Fr A = lane == 4 ? v2 : v;
    if (lane < npts) A = ck;
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

__device__ __forceinline__ Fr wave_lagrange(const Fr* c, int npts, const Fr& v) {
    return wave_lagrange_ni(c[(threadIdx.x & 63) < (unsigned)npts ? threadIdx.x & 63 : 0], npts, v);
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

// Wave 0 (lanes 0 .. 7, and every further eight the same): the `nb` whole blocks in rows 0 .. nb - 1, then the draw's three in the rows behind them
// (`two`: a hash has a second closing block, rows nb + 3 and nb + 4); the new chaining value goes to S.state, lane 0
// returns the challenge (normal, below 2.1 r).  The lane pairs all take the whole blocks, so that the next three start
// from the result: pairs 0 and 1 with the closing blocks of the draw, pairs 2 and 3 with the extension of the stream.
__device__ __forceinline__ F9 ts_frame_passes(TsShared& S, uint32_t nb, uint32_t base, bool two = false) {
    sha::Half h = ts_state_half(S);
    const uint32_t pair = sha::half_row() & 3, t = pair < 2 ? pair : 2;
    for (uint32_t blk = 0; blk <= nb; ++blk) h = ts_rounds(S, h, blk < nb ? blk : nb + t, base);
    if (pair == 2) ts_state_store(S, h);
    if (two) h = ts_rounds(S, h, nb + 3 + (t & 1), base);
    // 2^256 hi + lo as two products: low half and high half of a digest meet in the low lane
    Fr x;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        x.v[q] = sha::bswap32(h.v[q]);
        x.v[4 + q] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x.v[q], 0x141, 0xf, 0xf, true);
    }
    F9 m = f9_mul(fr_unpack(fr_const(pair ? frc::W3 : frc::R2)), fr_unpack(x));   // below 1.04 r
#pragma unroll
    for (int l = 0; l < 9; ++l)
        m.v[l] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m.v[l], 0xB1, 0xf, 0xf, true);   // pairs 0 and 1
    return f9_norm(m);
}

// A frame of `count` <= 3 elements - with_claim: the frame of S.claim, label 'c', in front of it - and a draw of one
// challenge: the step of every round.  Wave 0 runs the rounds of the whole blocks that the frames complete (one after a
// draw, when the stream is block-aligned), then those of the draw; wave 1 the schedules of all blocks side by side,
// sixteen words ahead; the other waves do nothing here.  Bound by the two dependent compressions of 4.3 thousand cycles
// (64 rounds of ten instructions) and three products' worth of arithmetic around them.  One lane per compression and the
// claim's frame as a step of its own: 5.9 thousand per compression, 22 us for a sumcheck's first round.  Leaves v in
// S.v9 and the new chaining value in S.state.
// limb(i): limb i % 8 of the i / 8-th element (canonical).
template <class Limb>
__device__ __forceinline__ void wave_frame_draw1_open(TsShared& S, char label, int count, Limb limb, bool with_claim = false) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (wave >= 2) return;
    const uint32_t data_len = 32u * (uint32_t)count, fill = S.fill, pre = with_claim ? 42u : 0u;
    const uint32_t total = fill + pre + 10u + data_len, nb = total >> 6, rem = total & 63;
    const uint32_t two = rem > 50 ? 1 : 0;      // tag, index, 0x80 and length do not fit behind the frame
    const uint64_t bits = ((S.nblk + nb) * 64u + rem + 5u) * 8u;
    const uint32_t nlimb = 8u * (uint32_t)count, sel = S.bufsel;
    // blocks in rows: the whole ones, then the draw's three (the two closing blocks, the extension), then the second
    // closing blocks
    for (uint32_t j = lane; j < 16 * (nb + 3 + 2 * two); j += 64) {
        const uint32_t row = j >> 4, i = j & 15;
        const bool draw = row >= nb, second = row >= nb + 3;
        const uint32_t t = row - nb - (second ? 3 : 0);
        const uint32_t k = draw ? 16 * nb + (second ? 16 : 0) + i : j;   // word k of the stream from the unfinished block on
        uint32_t word = 0;
        if (fill + pre == 0) {
            // data start at byte 10: a word is the upper half of one limb and the lower half of the next
            const uint32_t ip = k - 3, in = k - 2;
            const uint32_t lp = (k >= 3 && ip < nlimb) ? limb(ip) : 0u;
            const uint32_t ln = (k >= 2 && in < nlimb) ? limb(in) : 0u;
            word = (((lp >> 16) & 0xffu) << 24) | ((lp >> 24) << 16) | ((ln & 0xffu) << 8) | ((ln >> 8) & 0xffu);
            if (k == 0) word = (1u << 24) | ((uint32_t)(uint8_t)label << 16) | ((data_len & 0xffu) << 8);
        } else {
#pragma unroll 1
            for (uint32_t b = 0; b < 4; ++b) {
                const uint32_t p = 4 * k + b, q = p - fill;
                uint32_t x = 0;
                if (p < fill) x = S.buf[sel][p >> 2] >> (24 - 8 * (p & 3));
                else if (q < pre) x = ts_frame1_byte([&](uint32_t l) -> uint32_t { return S.claim[l]; }, 'c', 32u, q);
                else if (p < total) x = ts_frame1_byte(limb, label, data_len, q - pre);
                word = (word << 8) | (x & 0xffu);
            }
        }
        if (draw) {
            // tag at byte rem, four zero index bytes, then 0x80 in the hashes (not in the extension)
            const uint32_t w = k - 16 * nb;
            if (w == rem >> 2) word |= (0xF0u + t) << (24 - 8 * (rem & 3));
            if (t < 2) {
                if (w == (rem + 5) >> 2) word |= 0x80u << (24 - 8 * ((rem + 5) & 3));
                if (w == 16 * two + 14) word = (uint32_t)(bits >> 32);
                if (w == 16 * two + 15) word = (uint32_t)bits;
            }
        }
        S.msg[j] = word;     // by both waves, the same: neither waits for the other
    }
    __builtin_amdgcn_wave_barrier();   // LDS operations of a wave complete in order: no wait needed
    if (wave == 0) {
        const F9 m = ts_frame_passes(S, nb, 0, two);
        if (lane == 0) S.v9 = m;
        if (lane == 0) {
            S.nblk += nb + 1;
            S.fill = 0;
            S.seq = 0;      // the schedule wave has published its last group: it was waited for
        }
    } else {
        ts_schedules(S, nb + 3 + 2 * two);
    }
}
// the same with the closing barrier
template <class Limb>
__device__ __forceinline__ void wave_frame_draw1(TsShared& S, char label, int count, Limb limb, bool with_claim = false) {
    wave_frame_draw1_open(S, label, count, limb, with_claim);
    __syncthreads();
}

// the challenge of wave_frame_draw1, reduced
__device__ __forceinline__ Fr ts_challenge(const TsShared& S) { return fr_pack(f9_cond_sub(f9_cond_sub(S.v9))); }

// challenge v (normal, below 2.1 r) to its places; one lane
__device__ __forceinline__ void store_challenge(DevState* st, int idx, const F9& v) {
    const Fr x = fr_pack(f9_cond_sub(f9_cond_sub(v)));
    st->chal[idx] = x;
    const Fr plain = fr_from_mont_ni(x);
    uint32_t* le = (uint32_t*)(st->chal_le + 32 * (size_t)idx);
#pragma unroll
    for (int l = 0; l < 8; ++l) le[l] = plain.v[l];
}

// S.canon[0..count), count <= 3, go into the transcript under a one-character label (with_claim: behind the frame of
// S.claim), then one challenge is drawn: it is returned to every thread, lazy (normal, below 2.1 r), and stored in
// st->chal[chal_idx] (Montgomery form) and st->chal_le (canonical) by a lane of the last wave; nobody waits for that
// lane before the next barrier.  side() is run by wave `side_wave` >= 2 while the hashes run (no barrier inside).
template <class Side>
__device__ __forceinline__ F9 block_absorb_draw1_side(TsShared& S, DevState* st, char label, int count, int chal_idx, bool with_claim,
                                                      int side_wave, Side side) {
    const int tid = threadIdx.x;
    __syncthreads();
    if ((tid >> 6) == side_wave) side();
    wave_frame_draw1(S, label, count, [&](uint32_t i) -> uint32_t { return S.canon[i >> 3][i & 7]; }, with_claim);
    if (tid == (int)blockDim.x - 64) store_challenge(st, chal_idx, S.v9);   // a lane of the last wave
    return S.v9;
}

__device__ inline Fr block_absorb_draw1(TsShared& S, DevState* st, char label, int count, int chal_idx) {
    block_absorb_draw1_side(S, st, label, count, chal_idx, false, ROUND_SIDE_WAVE, [] {});
    return ts_challenge(S);
}

// First part of closing a round: g_t(0..npts-1) (LDS, Montgomery, npts = 2..4) go to the proof
// and into the transcript, the round's challenge v_t is drawn and returned to every thread.
// The Lagrange coefficients of g_t are left in S.tmp[0..npts) for the claim g_t(v_t).
// Needs blockDim.x >= TS_MIN_THREADS: wave 1 prepares the coefficients beside wave 0's canonical forms.
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
// itself are needed by the proof bytes and by the round after next at the earliest, so another wave works them out
// while waves 0 and 1 hash, and the canonical form of a sum is taken by the lane that has just finished the sum.
struct RoundShared {
    F9 g9[ZK_MAX_EVALS];      // the evaluations summed in this round, lazy
    F9 coef[ZK_MAX_EVALS];    // 1 / prod_{j != k} (k - j) for the number of points in use
    Fr lag[ZK_MAX_EVALS];     // Lagrange coefficients of the last closed round
    Fr claim;                 // of the round, where g(1) is derived from it
};

// R.coef[k], k < npts = 2..4
__device__ __forceinline__ void round_coefficient(RoundShared& R, const DevState* st, int npts, int k) {
    Fr c;
    if (npts == 4) c = (k == 0 || k == 3) ? st->inv6 : st->inv2;         // -1/6, 1/2, -1/2, 1/6
    else c = (npts == 3 && k != 1) ? st->inv2 : fr_one();                // 1/2, -1, 1/2; -1, 1
    const bool neg = npts == 4 ? (k == 0 || k == 2) : npts == 3 ? k == 1 : k == 0;
    R.coef[k] = fr_unpack(neg ? fr_neg(c) : c);
}

// once per kernel that derives no g(1), between two barriers of the caller
__device__ __forceinline__ void round_begin(RoundShared& R, const DevState* st, int npts) {
    const int k = (int)threadIdx.x - 64 * ROUND_SIDE_WAVE;
    if (k >= 0 && k < npts) round_coefficient(R, st, npts, k);
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

// one wave, next to the hashes: g(1) if it is derived, the coefficients of g
__device__ __forceinline__ void wave_round_side(RoundShared& R, int npts, bool derive1, uint32_t* proof_dst) {
    const int lane = threadIdx.x & 63;
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
}

// A wave that has no sums to take, before they are there: what round_begin does, and the claim, which the round before
// may have left owed - two products and their operands, 8 thousand cycles, which behind the sums would outlast the hashes.
__device__ __forceinline__ void wave_round_begin(RoundShared& R, const DevState* st, int npts, bool derive1) {
    const int lane = threadIdx.x & 63;
    const uint32_t owed = st->lag_npts;
    Fr claim = st->claim;
    if (derive1 && owed) claim = wave_lagrange_ni(st->lag[lane & 3], (int)owed, st->chal[st->lag_chal]);
    if (lane < npts) round_coefficient(R, st, npts, lane);
    if (lane == 0) R.claim = claim;
}

// Closes a round whose sums have gone through round_eval_out: the challenge, to every thread (lazy: normal, below
// 2.1 r).  Nothing here evaluates the claim g(v): its coefficients are in R.lag, for round_end.
__device__ __forceinline__ F9 block_close_round(TsShared& S, RoundShared& R, DevState* st, int npts, bool derive1, uint32_t proof_off,
                                                int chal_idx, char label = 'g', bool skip1 = true, bool with_claim = false,
                                                int side_wave = ROUND_SIDE_WAVE) {
    uint32_t* proof_dst = (uint32_t*)(st->proof + proof_off);
    return block_absorb_draw1_side(S, st, label, skip1 ? npts - 1 : npts, chal_idx, with_claim, side_wave,
                                   [&] { wave_round_side(R, npts, derive1, proof_dst); });
}

// claim_0 of a sumcheck, which its first round absorbs in front of the evaluations (with_claim), a lazy sum (normal,
// below 4.9 r), to the transcript's inputs and the proof; one thread, before block_close_round
__device__ __forceinline__ void round_claim_out(TsShared& S, const F9& c, uint32_t* dst, uint32_t* copy_dst) {
    const Fr plain = f9_canonical(c);
#pragma unroll
    for (int l = 0; l < 8; ++l) {
        S.claim[l] = plain.v[l];
        dst[l] = plain.v[l];
        if (copy_dst) copy_dst[l] = plain.v[l];
    }
}

// leaves the owed claim to the next kernel (after the last block_close_round)
__device__ __forceinline__ void round_end(const RoundShared& R, DevState* st, int npts, int chal_idx) {
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
