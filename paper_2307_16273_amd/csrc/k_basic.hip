// Conversion into Fr, equality-polynomial tables, and MLE partial evaluation
// (Eq. multilinear-extension, Sec. 2.2) for gfx950.
#include <string.h>
#include "zkdl_internal.h"

// ---------------------------------------------------------------------------
// integer / byte sources -> Fr (Montgomery, SoA)
// ---------------------------------------------------------------------------
template <int KIND>
__device__ __forceinline__ Fr load_src(const void* src, uint64_t i) {
    if (KIND == TK_I32) return fr_from_i64((int64_t)((const int32_t*)src)[i]);
    if (KIND == TK_I64) return fr_from_i64(((const int64_t*)src)[i]);
    if (KIND == TK_FR) {
        // never reached: Fr sources are read through FrTab
        return fr_zero();
    }
    // raw 32-byte little-endian values
    const uint32_t* p = (const uint32_t*)src + 8 * i;
    Fr x;
#pragma unroll
    for (int l = 0; l < 8; ++l) x.v[l] = p[l];
    return fr_to_mont(x);
}

constexpr int KIND_LE = 3;

template <int KIND>
__global__ __launch_bounds__(ZK_BLOCK) void k_convert(const void* src, uint64_t n, FrTab out) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        tab_st(out, i, load_src<KIND>(src, i));
}

static unsigned grid_for(uint64_t n, unsigned cap = 65536) {
    uint64_t b = (n + ZK_BLOCK - 1) / ZK_BLOCK;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

// the column sums of the lazy partial-evaluation kernels stay in range for this many elements per thread
constexpr uint64_t PE_LAZY_MAX_CHUNK = 4096;

void zk_launch_convert(zkdl_ctx* ctx, const void* src, int kind, uint64_t n, FrTab out) {
    unsigned g = grid_for(n);
    if (kind == TK_I32)
        hipLaunchKernelGGL(k_convert<TK_I32>, dim3(g), dim3(ZK_BLOCK), 0, ctx->stream, src, n, out);
    else if (kind == TK_I64)
        hipLaunchKernelGGL(k_convert<TK_I64>, dim3(g), dim3(ZK_BLOCK), 0, ctx->stream, src, n, out);
    else
        hipLaunchKernelGGL(k_convert<KIND_LE>, dim3(g), dim3(ZK_BLOCK), 0, ctx->stream, src, n, out);
}

__global__ __launch_bounds__(ZK_BLOCK) void k_download(FrTab in, uint64_t n, uint32_t* out) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x) {
        Fr x = fr_from_mont(tab_ld(in, i));
#pragma unroll
        for (int l = 0; l < 8; ++l) out[8 * i + l] = x.v[l];
    }
}

void zk_launch_download(zkdl_ctx* ctx, FrTab in, uint64_t n, uint8_t* out_le_dev) {
    hipLaunchKernelGGL(k_download, dim3(grid_for(n)), dim3(ZK_BLOCK), 0, ctx->stream, in, n,
                       (uint32_t*)out_le_dev);
}

__global__ void k_points_to_mont(const uint32_t* le, int n, Fr* out) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        Fr x;
#pragma unroll
        for (int l = 0; l < 8; ++l) x.v[l] = le[8 * i + l];
        out[i] = fr_to_mont(x);
    }
}

void zk_launch_points_to_mont(zkdl_ctx* ctx, const uint8_t* le_dev, int n, Fr* out) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_points_to_mont, dim3((n + 63) / 64), dim3(64), 0, ctx->stream,
                       (const uint32_t*)le_dev, n, out);
}

// chal[dst + i] (and its little-endian copy) = the i-th given coordinate: taken from canonical
// little-endian bytes, or, with le == nullptr, a copy of chal[idx.v[i]]
__global__ void k_chal_set(DevState* st, int dst, int n, const uint32_t* le, ChalIdx idx) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    Fr x, xm;
    if (le) {
#pragma unroll
        for (int l = 0; l < 8; ++l) x.v[l] = le[8 * i + l];
        xm = fr_to_mont(x);
    } else {
        xm = st->chal[idx.v[i]];
        x = fr_from_mont(xm);
    }
    st->chal[dst + i] = xm;
    uint32_t* out = (uint32_t*)(st->chal_le + 32 * (size_t)(dst + i));
#pragma unroll
    for (int l = 0; l < 8; ++l) out[l] = x.v[l];
}

void zk_launch_chal_set(zkdl_ctx* ctx, int dst, int n, const uint8_t* le_dev, const ChalIdx* idx) {
    if (n <= 0) return;
    ChalIdx none = {};
    hipLaunchKernelGGL(k_chal_set, dim3((n + 63) / 64), dim3(64), 0, ctx->stream, ctx->dev, dst, n,
                       (const uint32_t*)le_dev, idx ? *idx : none);
}

// ---------------------------------------------------------------------------
// beta~(u, .): the multilinear extension of the equality indicator (Sec. 2.2),
// beta~(u, b) = prod_k (u_k b_k + (1 - u_k)(1 - b_k)), u_0 <-> most significant bit.
// Up to 2^BETA_SMALL_MAX entries: every block doubles the two half tables in LDS, side by side and from the last
// coordinate of each upwards (T[b + size] = T[b] u_k; T[b] -= T[b + size]), and takes its entries as products of the two:
// m / 2 + 1 products in a row and nothing through memory between them.  Doubling the whole table in place in memory by
// one block took 15 us for m = 10, this way 9.
// ---------------------------------------------------------------------------
constexpr int BETA_SMALL_MAX = 12;
constexpr int BETA_MAX_SMALL = 16;
constexpr int BETA_MAX_OUTER = 8;

struct BetaSmallBatch {
    const Fr* point[BETA_MAX_SMALL];
    int m[BETA_MAX_SMALL];
    FrTab out[BETA_MAX_SMALL];
};

__global__ __launch_bounds__(ZK_BLOCK) void k_beta_small_batch(BetaSmallBatch bb) {
    constexpr int HALF = BETA_SMALL_MAX / 2;
    __shared__ F9 T[2][1 << HALF];       // the halves of the point: leading, trailing coordinates
    __shared__ F9 u[BETA_SMALL_MAX];
    const int m = bb.m[blockIdx.x], hb = m / 2, lb = m - hb, tid = threadIdx.x;
    const FrTab out = bb.out[blockIdx.x];
    if ((uint64_t)blockIdx.y * blockDim.x >= (uint64_t)1 << m) return;
    if (tid < m) u[tid] = fr_unpack(bb.point[blockIdx.x][tid]);
    else if (tid >= 64 && tid < 66) T[tid - 64][0] = fr_unpack(fr_one());
    __syncthreads();
    const int half = tid >> 6, i = tid & 63;
    for (int k = 0; k < lb; ++k) {
        const int bits = half ? lb : hb;
        if (half < 2 && k < bits && i < 1 << k) {
            const F9 e = T[half][i], hi = f9_mul(e, u[(half ? m : hb) - 1 - k]);   // normal, below 1.1 r
            T[half][i + (1 << k)] = hi;
            T[half][i] = f9_norm_reduce(f9_sub(e, hi));
        }
        __syncthreads();
    }
    const uint32_t b = blockIdx.y * blockDim.x + tid;
    if (b < 1u << m) tab_st(out, b, fr_pack(f9_cond_sub(f9_mul(T[0][b >> lb], T[1][b & ((1u << lb) - 1)]))));
}

static void launch_beta_small(zkdl_ctx* ctx, const BetaSmallBatch& sb, int n) {
    int top = 0;
    for (int i = 0; i < n; ++i) top = sb.m[i] > top ? sb.m[i] : top;
    const unsigned per = top > 8 ? 1u << (top - 8) : 1u;
    static_assert(ZK_BLOCK == 1 << 8, "entries per block");
    hipLaunchKernelGGL(k_beta_small_batch, dim3((unsigned)n, per), dim3(ZK_BLOCK), 0, ctx->stream, sb);
}

// out[(h << lo_bits) | l] = hi[h] * lo[l]
__global__ __launch_bounds__(ZK_BLOCK) void k_beta_outer(FrTab hi, FrTab lo, int lo_bits, uint64_t n,
                                                         FrTab out) {
    uint64_t mask = ((uint64_t)1 << lo_bits) - 1;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x) {
        Fr a = tab_ld(hi, i >> lo_bits);
        Fr b = tab_ld(lo, i & mask);
        tab_st(out, i, fr_mul(a, b));
    }
}

int zk_build_beta(zkdl_ctx* ctx, const Fr* point, int m, FrTab out) {
    if (m <= BETA_SMALL_MAX) {
        BetaSmallBatch sb;
        sb.point[0] = point;
        sb.m[0] = m;
        sb.out[0] = out;
        launch_beta_small(ctx, sb, 1);
        return ZKDL_OK;
    }
    int hb = m / 2, lb = m - hb;
    uint64_t hn = (uint64_t)1 << hb, ln = (uint64_t)1 << lb;
    void* tmp = zk_alloc(ctx, (hn + ln) * 32);
    if (!tmp) return ZKDL_ENOMEM;
    FrTab th = make_tab(tmp, hn);
    FrTab tl = make_tab((uint32_t*)tmp + 8 * hn, ln);
    int rc = zk_build_beta(ctx, point, hb, th);
    if (rc == ZKDL_OK) rc = zk_build_beta(ctx, point + hb, lb, tl);
    if (rc == ZKDL_OK) {
        uint64_t n = (uint64_t)1 << m;
        hipLaunchKernelGGL(k_beta_outer, dim3(grid_for(n)), dim3(ZK_BLOCK), 0, ctx->stream, th, tl,
                           lb, n, out);
    }
    zk_free(ctx, tmp);   // stream-ordered reuse: later kernels on the same stream run after this one
    return rc;
}

// The table of a point in host memory, 2^m entries, m <= ZK_BETA_DIRECT_MAX, in one launch: the coordinates are
// kernel arguments.  A block has the products of all pairs of coordinates, then of all fours in LDS, and an entry is a product of
// at most four of those: bound by five products one after the other (6.6 us for m = 12, 11.2 with the factors
// of an entry one by one; a copy, a conversion, two doubling tables and their outer product were five dependent steps: 21 us of kernels
// and as much between them).
struct BetaDirectArgs {
    Fr le[ZK_BETA_DIRECT_MAX];
    int m;
    FrTab out;
};

__global__ __launch_bounds__(64) void k_beta_direct(BetaDirectArgs a) {
    static_assert(ZK_BETA_DIRECT_MAX == 16, "sixteen coordinates, eight pairs, four fours");
    __shared__ F9 f[16][2], pair[8][4], four[4][16];   // by bits of the entry from the lowest; 1 above the point's coordinates
    const int tid = threadIdx.x;
    if (tid < 16) {
        Fr u0 = fr_one(), u1 = fr_one();
        if (tid < a.m) {
            Fr x;
#pragma unroll
            for (int l = 0; l < 8; ++l) x.v[l] = a.le[a.m - 1 - tid].v[l];
            u1 = fr_to_mont(x);
            u0 = fr_sub(fr_one(), u1);
        }
        f[tid][0] = fr_unpack(u0);
        f[tid][1] = fr_unpack(u1);
    }
    __syncthreads();
    if (tid < 32) pair[tid >> 2][tid & 3] = f9_mul(f[(tid >> 2) * 2][tid & 1], f[(tid >> 2) * 2 + 1][(tid >> 1) & 1]);
    __syncthreads();
    four[tid >> 4][tid & 15] = f9_mul(pair[(tid >> 4) * 2][tid & 3], pair[(tid >> 4) * 2 + 1][(tid >> 2) & 3]);
    __syncthreads();
    const uint32_t b = blockIdx.x * 64u + (uint32_t)tid;
    if (b >= (1u << a.m)) return;
    F9 x = four[0][b & 15];
    for (int k = 1; 4 * k < a.m; ++k) x = f9_mul(x, four[k][(b >> (4 * k)) & 15]);   // normal, below 2 r
    tab_st(a.out, b, fr_pack(f9_cond_sub(x)));
}

void zk_launch_beta_direct(zkdl_ctx* ctx, const uint8_t* le_host, int m, FrTab out) {
    BetaDirectArgs a;
    memset(&a, 0, sizeof a);
    memcpy(a.le, le_host, 32 * (size_t)m);
    a.m = m;
    a.out = out;
    hipLaunchKernelGGL(k_beta_direct, dim3(((1u << m) + 63) / 64), dim3(64), 0, ctx->stream, a);
}

// ---- several tables at once: one launch for all small tables, one for all outer products ----
struct BetaOuterBatch {
    FrTab hi[BETA_MAX_OUTER], lo[BETA_MAX_OUTER], out[BETA_MAX_OUTER];
    int lo_bits[BETA_MAX_OUTER];
    uint64_t n[BETA_MAX_OUTER];
};

__global__ __launch_bounds__(ZK_BLOCK) void k_beta_outer_batch(BetaOuterBatch ob) {
    const int q = blockIdx.y;
    const FrTab hi = ob.hi[q], lo = ob.lo[q], out = ob.out[q];
    const int lo_bits = ob.lo_bits[q];
    const uint64_t n = ob.n[q], mask = ((uint64_t)1 << lo_bits) - 1;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        tab_st(out, i, fr_mul(tab_ld(hi, i >> lo_bits), tab_ld(lo, i & mask)));
}

int zk_build_beta_many(zkdl_ctx* ctx, const BetaJob* jobs, int n) {
    BetaSmallBatch sb;
    BetaOuterBatch ob;
    int ns = 0, no = 0;
    uint64_t tmp_elems = 0, max_n = 0;
    for (int i = 0; i < n; ++i) {
        const int m = jobs[i].m;
        if (m > BETA_SMALL_MAX && m <= 2 * BETA_SMALL_MAX) tmp_elems += ((uint64_t)1 << (m / 2)) + ((uint64_t)1 << (m - m / 2));
    }
    void* tmp = tmp_elems ? zk_alloc(ctx, tmp_elems * 32) : nullptr;
    if (tmp_elems && !tmp) return ZKDL_ENOMEM;
    uint32_t* tp = (uint32_t*)tmp;
    int rc = ZKDL_OK;
    for (int i = 0; i < n && rc == ZKDL_OK; ++i) {
        const int m = jobs[i].m;
        const bool split = m > BETA_SMALL_MAX && m <= 2 * BETA_SMALL_MAX;
        if (m > 2 * BETA_SMALL_MAX || ns + (split ? 2 : 1) > BETA_MAX_SMALL || (split && no + 1 > BETA_MAX_OUTER)) {
            rc = zk_build_beta(ctx, jobs[i].point, m, jobs[i].out);   // large or surplus tables: one by one
            continue;
        }
        if (!split) {
            sb.point[ns] = jobs[i].point;
            sb.m[ns] = m;
            sb.out[ns] = jobs[i].out;
            ++ns;
            continue;
        }
        const int hb = m / 2, lb = m - hb;
        const uint64_t hn = (uint64_t)1 << hb, ln = (uint64_t)1 << lb;
        const FrTab th = make_tab(tp, hn);
        tp += 8 * hn;
        const FrTab tl = make_tab(tp, ln);
        tp += 8 * ln;
        sb.point[ns] = jobs[i].point;
        sb.m[ns] = hb;
        sb.out[ns] = th;
        ++ns;
        sb.point[ns] = jobs[i].point + hb;
        sb.m[ns] = lb;
        sb.out[ns] = tl;
        ++ns;
        ob.hi[no] = th;
        ob.lo[no] = tl;
        ob.out[no] = jobs[i].out;
        ob.lo_bits[no] = lb;
        ob.n[no] = (uint64_t)1 << m;
        if (ob.n[no] > max_n) max_n = ob.n[no];
        ++no;
    }
    if (rc == ZKDL_OK && ns > 0)
        launch_beta_small(ctx, sb, ns);
    if (rc == ZKDL_OK && no > 0)
        hipLaunchKernelGGL(k_beta_outer_batch, dim3(grid_for(max_n, 4096), no), dim3(ZK_BLOCK), 0, ctx->stream, ob);
    zk_free(ctx, tmp);   // stream-ordered reuse
    return rc;
}

// ---------------------------------------------------------------------------
// partial evaluation: out[o, i] = sum_a beta[a] * T[o, a, i]
// ---------------------------------------------------------------------------
template <int KIND>
__device__ __forceinline__ Fr pe_load(const void* src, uint64_t idx) {
    if (KIND == TK_FR) {
        const FrTab* t = (const FrTab*)src;
        return tab_ld(*t, idx);
    }
    return load_src<KIND>(src, idx);
}

struct PeArgs {
    const void* src;   // integers, or unused for Fr
    FrTab fr_src;      // Fr source
    FrTab beta;
    FrTab out;         // chunk c of output element e at index c * (O*I) + e
    uint64_t O, A, I;
    uint64_t a_chunk;  // contracted-axis entries per chunk
};

template <int KIND>
__device__ __forceinline__ Fr pe_elem(const PeArgs& p, uint64_t idx) {
    if (KIND == TK_FR) return tab_ld(p.fr_src, idx);
    return load_src<KIND>(p.src, idx);
}

// one thread per output element (o, i): coalesced when I is large
template <int KIND>
__global__ __launch_bounds__(ZK_BLOCK) void k_pe_mid(PeArgs p) {
    uint64_t n_out = p.O * p.I;
    uint64_t a0 = (uint64_t)blockIdx.y * p.a_chunk;
    uint64_t a1 = a0 + p.a_chunk;
    if (a1 > p.A) a1 = p.A;
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < n_out;
         e += (uint64_t)gridDim.x * blockDim.x) {
        uint64_t o = e / p.I, i = e - o * p.I;
        Fr acc = fr_zero();
        for (uint64_t a = a0; a < a1; ++a) {
            Fr x = pe_elem<KIND>(p, (o * p.A + a) * p.I + i);
            acc = fr_add(acc, fr_mul(tab_ld(p.beta, a), x));
        }
        tab_st(p.out, (uint64_t)blockIdx.y * n_out + e, acc);
    }
}

__device__ __forceinline__ Fr wave_sum(Fr x) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        Fr y;
#pragma unroll
        for (int l = 0; l < 8; ++l) y.v[l] = __shfl_down(x.v[l], off, 64);
        x = fr_add(x, y);
    }
    return x;   // lane 0 holds the sum
}

// innermost axis contracted (I == 1): one wave per (output row, chunk), lanes stride over a
template <int KIND>
__global__ __launch_bounds__(ZK_BLOCK) void k_pe_inner(PeArgs p) {
    const int lane = threadIdx.x & 63;
    uint64_t wave = (blockIdx.x * (uint64_t)blockDim.x + threadIdx.x) >> 6;
    uint64_t n_waves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
    uint64_t chunks = (p.A + p.a_chunk - 1) / p.a_chunk;
    uint64_t n_items = p.O * chunks;
    for (uint64_t it = wave; it < n_items; it += n_waves) {
        uint64_t c = it / p.O, o = it - c * p.O;
        uint64_t a0 = c * p.a_chunk, a1 = a0 + p.a_chunk;
        if (a1 > p.A) a1 = p.A;
        Fr acc = fr_zero();
        for (uint64_t a = a0 + lane; a < a1; a += 64) {
            Fr x = pe_elem<KIND>(p, o * p.A + a);
            acc = fr_add(acc, fr_mul(tab_ld(p.beta, a), x));
        }
        acc = wave_sum(acc);
        if (lane == 0) tab_st(p.out, c * p.O + o, acc);
    }
}

// Lazy variants: the products of one output are summed as 64-bit columns of 29-bit limb
// products and reduced once (f9_cols_*, f9_redc), instead of one Montgomery product and one
// modular addition per source element.  Thread per output element (o, i), block = 256 consecutive
// outputs; blockIdx.y selects the chunk of the contracted axis; beta_a is the same for every thread
// of an iteration and is unpacked once per block into LDS.
//
// Fr source: sum_a beta_a T_a, 81 multiply-adds per element, both in Montgomery form, so the
// reduced sum is the Montgomery form of the result.
// (integer sources: k_pe_mid_int and k_pe_inner_int below.)
constexpr int PE_FR_TILE = 256;   // entries of beta unpacked into LDS at a time
template <int KIND>
__global__ __launch_bounds__(ZK_BLOCK) void k_pe_mid_lazy(PeArgs p) {
    static_assert(KIND == TK_FR, "Fr sources only");
    __shared__ uint32_t sb[9][PE_FR_TILE];
    const uint64_t n_out = p.O * p.I;
    const uint64_t a0 = (uint64_t)blockIdx.y * p.a_chunk;
    uint64_t a1 = a0 + p.a_chunk;
    if (a1 > p.A) a1 = p.A;
    const uint64_t nblk = (n_out + ZK_BLOCK - 1) / ZK_BLOCK;
    for (uint64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
        const uint64_t e = blk * ZK_BLOCK + threadIdx.x;
        const bool live = e < n_out;
        const uint64_t o = live ? e / p.I : 0, i = live ? e - o * p.I : 0;
        uint64_t c[17];
#pragma unroll
        for (int k = 0; k < 17; ++k) c[k] = 0;
        int pending = 0;
        for (uint64_t at = a0; at < a1; at += PE_FR_TILE) {
            const int na = (int)(a1 - at < PE_FR_TILE ? a1 - at : PE_FR_TILE);
            __syncthreads();   // the previous tile is no longer read
            if ((int)threadIdx.x < na) {   // beta of the tile, unpacked once per block (every thread reads the same entry)
                const F9 b9 = fr_unpack(tab_ld(p.beta, at + threadIdx.x));
#pragma unroll
                for (int l = 0; l < 9; ++l) sb[l][threadIdx.x] = b9.v[l];
            }
            __syncthreads();
            if (live) {
#pragma unroll 2
                for (int k = 0; k < na; ++k) {
                    F9 b9;
#pragma unroll
                    for (int l = 0; l < 9; ++l) b9.v[l] = sb[l][k];
                    const F9 x9 = fr_unpack(tab_ld(p.fr_src, (o * p.A + at + k) * p.I + i));
                    f9_cols_mac(c, b9, x9);
                    if (++pending == 4) {
                        pending = 0;
                        f9_cols_norm<17>(c);
                    }
                }
            }
        }
        if (live) {
            f9_cols_norm<17>(c);
            tab_st(p.out, (uint64_t)blockIdx.y * n_out + e, f9_to_fr(f9_norm_reduce(f9_redc(c))));
        }
    }
}

// ---- integers times beta as signed columns ----
// beta_a x_a in 29-bit limbs of beta: an int32 is one factor of nine signed multiply-adds, an int64 three limbs of 29, 29
// and 6 (signed) bits, 27 multiply-adds.  The products go into signed 64-bit columns, carried every fourth element.  The
// sum is "beta times integer", a Montgomery form already: an offset of a power of two makes it non-negative, it is
// reduced (divide by 2^261), multiplied back by 2^522 mod r, and the offset's residue is taken off again.
template <int KIND>
struct PeInt;
template <>
struct PeInt<TK_I32> {
    typedef int32_t T;
    static constexpr int COLS = 10, OFF_COL = 9, OFF_BIT = 56;   // |sum| < 2^286: chunks of at most 2^27 entries
};
template <>
struct PeInt<TK_I64> {
    typedef int64_t T;
    static constexpr int COLS = 12, OFF_COL = 11, OFF_BIT = 30;  // |sum| < 2^345
};

template <int KIND>
__device__ __forceinline__ void pe_int_mac(int64_t (&c)[PeInt<KIND>::COLS], const F9& b, typename PeInt<KIND>::T x) {
    if constexpr (KIND == TK_I32) {
#pragma unroll
        for (int l = 0; l < 9; ++l) c[l] += (int64_t)(int32_t)b.v[l] * (int64_t)x;
    } else {
        const int32_t x0 = (int32_t)((uint32_t)x & frc::M29), x1 = (int32_t)((uint32_t)(x >> 29) & frc::M29),
                      x2 = (int32_t)(x >> 58);
#pragma unroll
        for (int l = 0; l < 9; ++l) {
            c[l] += (int64_t)(int32_t)b.v[l] * (int64_t)x0;
            c[l + 1] += (int64_t)(int32_t)b.v[l] * (int64_t)x1;
            c[l + 2] += (int64_t)(int32_t)b.v[l] * (int64_t)x2;
        }
    }
}
// four products below 2^60 in magnitude per column (int64: two of them and a small one, 2^58.1 each)
template <int KIND>
__device__ __forceinline__ void pe_int_carry(int64_t (&c)[PeInt<KIND>::COLS]) {
#pragma unroll
    for (int l = 0; l + 1 < PeInt<KIND>::COLS; ++l) {
        c[l + 1] += c[l] >> 29;
        c[l] &= (int64_t)frc::M29;
    }
}
template <int KIND>
__device__ __forceinline__ Fr pe_int_value(const int64_t (&c)[PeInt<KIND>::COLS]) {
    constexpr int SH = 29 * PeInt<KIND>::OFF_COL + PeInt<KIND>::OFF_BIT - 261;   // the offset over 2^261
    uint64_t cols[17];
#pragma unroll
    for (int k = 0; k < 17; ++k) cols[k] = k < PeInt<KIND>::COLS ? (uint64_t)c[k] : 0;
    cols[PeInt<KIND>::OFF_COL] += (uint64_t)1 << PeInt<KIND>::OFF_BIT;            // the top column: positive now
    const F9 r2 = fr_unpack(fr_const(frc::R2));
    F9 off = f9_zero();
    off.v[SH / 29] = 1u << (SH % 29);
    const F9 koff = f9_mul(off, r2);                      // 2^SH 2^261 mod r (up to a multiple of r), below 2r
    const F9 val = f9_mul(f9_redc(cols), r2);             // normal, below 2r
    return f9_to_fr(f9_sub(val, koff));
}

// Middle axis contracted, integer source: thread = output (o, i), block = 256 consecutive outputs.
// beta of the chunk is unpacked once per block into LDS (every thread reads the same entry of an
// iteration); the integers of eight rows are requested together before they are used.
constexpr int PE_MID_TILE = 256;
template <int KIND>
__global__ __launch_bounds__(ZK_BLOCK) void k_pe_mid_int(PeArgs p) {
    typedef typename PeInt<KIND>::T T;
    __shared__ uint32_t sb[9][PE_MID_TILE];
    const uint64_t n_out = p.O * p.I;
    const uint64_t a0 = (uint64_t)blockIdx.y * p.a_chunk;
    uint64_t a1 = a0 + p.a_chunk;
    if (a1 > p.A) a1 = p.A;
    const T* src = (const T*)p.src;
    const uint64_t nblk = (n_out + ZK_BLOCK - 1) / ZK_BLOCK;
    for (uint64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
        const uint64_t e = blk * ZK_BLOCK + threadIdx.x;
        const bool live = e < n_out;
        const uint64_t o = live ? e / p.I : 0, i = live ? e - o * p.I : 0;
        const T* col = src + (o * p.A) * p.I + i;
        int64_t c[PeInt<KIND>::COLS];
#pragma unroll
        for (int k = 0; k < PeInt<KIND>::COLS; ++k) c[k] = 0;
        for (uint64_t at = a0; at < a1; at += PE_MID_TILE) {
            const int na = (int)(a1 - at < PE_MID_TILE ? a1 - at : PE_MID_TILE);
            __syncthreads();   // the previous tile is no longer read
            if ((int)threadIdx.x < na) {
                const F9 b9 = fr_unpack(tab_ld(p.beta, at + threadIdx.x));
#pragma unroll
                for (int l = 0; l < 9; ++l) sb[l][threadIdx.x] = b9.v[l];
            }
            __syncthreads();
            if (live) {
                for (int k0 = 0; k0 < na; k0 += 8) {
                    T x[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) x[u] = k0 + u < na ? col[(at + k0 + u) * p.I] : 0;
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int k = k0 + u < na ? k0 + u : 0;
                        F9 b9;
#pragma unroll
                        for (int l = 0; l < 9; ++l) b9.v[l] = sb[l][k];
                        pe_int_mac<KIND>(c, b9, x[u]);
                        if ((u & 3) == 3) pe_int_carry<KIND>(c);
                    }
                }
            }
        }
        if (live) tab_st(p.out, (uint64_t)blockIdx.y * n_out + e, pe_int_value<KIND>(c));
    }
}

// Innermost axis contracted, integer source: one wave per tile of 64 output rows and one chunk
// of the axis.  The tile of integers is read row by row (each row segment is contiguous, so
// the loads coalesce; 16 KB of them are requested before the first is used) and transposed through LDS; then
// lane = row, and beta_a is the same for all lanes of an iteration.
template <int KIND>
__global__ __launch_bounds__(64) void k_pe_inner_int(PeArgs p) {
    typedef typename PeInt<KIND>::T T;
    constexpr int ROWS = 256 / sizeof(T);        // requested together
    __shared__ T tile[64][65];
    __shared__ F9 sb[64];
    const int lane = threadIdx.x;
    const uint64_t row0 = (uint64_t)blockIdx.x * 64;
    const uint64_t a0 = (uint64_t)blockIdx.y * p.a_chunk;
    uint64_t a1 = a0 + p.a_chunk;
    if (a1 > p.A) a1 = p.A;
    const T* src = (const T*)p.src;
    int64_t c[PeInt<KIND>::COLS];
#pragma unroll
    for (int k = 0; k < PeInt<KIND>::COLS; ++k) c[k] = 0;
    const int rows_here = (int)(p.O - row0 < 64 ? p.O - row0 : 64);
    for (uint64_t at = a0; at < a1; at += 64) {
        const int na = (int)(a1 - at < 64 ? a1 - at : 64);
        if (lane < na) sb[lane] = fr_unpack(tab_ld(p.beta, at + lane));
        const T* seg = src + row0 * p.A + at + lane;
        for (int r0 = 0; r0 < rows_here; r0 += ROWS) {
            T x[ROWS];
#pragma unroll
            for (int u = 0; u < ROWS; ++u)
                x[u] = (lane < na && r0 + u < rows_here) ? seg[(uint64_t)(r0 + u) * p.A] : 0;
#pragma unroll
            for (int u = 0; u < ROWS; ++u) tile[r0 + u][lane] = x[u];
        }
        __syncthreads();
        if (lane < rows_here) {
            for (int k0 = 0; k0 < na; k0 += 4) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k = k0 + u < na ? k0 + u : 0;
                    pe_int_mac<KIND>(c, sb[k], k0 + u < na ? tile[lane][k] : (T)0);
                }
                pe_int_carry<KIND>(c);
            }
        }
        __syncthreads();
    }
    if (lane < rows_here) tab_st(p.out, (uint64_t)blockIdx.y * p.O + row0 + lane, pe_int_value<KIND>(c));
}

// out[e] = sum_c part[c * n + e].  A block takes OUTS outputs and shares each one's chunks among 256 / OUTS lanes, with four
// chunks' loads in flight per lane.  Bound by the chain of trips to memory: with 64 outputs a block, 512 outputs in 256 chunks are
// eight blocks of sixteen such trips each.  Figures at the rule below.
template <int OUTS>
__global__ __launch_bounds__(ZK_BLOCK) void k_sum_chunks(FrTab part, uint64_t n, uint64_t chunks,
                                                         FrTab out) {
    constexpr int WAYS = ZK_BLOCK / OUTS;
    static_assert(WAYS == 4 || WAYS == 16 || WAYS == 64, "summed four to one");
    __shared__ uint32_t w9[9][ZK_BLOCK];
    const int way = threadIdx.x / OUTS, lane = threadIdx.x % OUTS;
    for (uint64_t e0 = blockIdx.x * (uint64_t)OUTS; e0 < n; e0 += gridDim.x * (uint64_t)OUTS) {
        const uint64_t e = e0 + lane;
        F9 acc = f9_zero();
        if (e < n) {
            for (uint64_t c = way; c < chunks; c += 4 * WAYS) {
                Fr x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (c + WAYS * q < chunks) x[q] = tab_ld(part, (c + WAYS * q) * n + e);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (c + WAYS * q < chunks) acc = f9_add(acc, fr_unpack(x[q]));   // limbs below 5 * 2^29
                acc = f9_norm_reduce(acc);
            }
        }
        // four to one until one is left
#pragma unroll
        for (int w = WAYS; w > 1; w /= 4) {
            if (way < w)
#pragma unroll
                for (int l = 0; l < 9; ++l) w9[l][threadIdx.x] = acc.v[l];
            __syncthreads();
            if (way < w / 4) {
#pragma unroll
                for (int q = 1; q < 4; ++q)
#pragma unroll
                    for (int l = 0; l < 9; ++l) acc.v[l] += w9[l][threadIdx.x + q * (w / 4) * OUTS];   // below 10 r
                if (w > 4) acc = f9_norm_reduce(acc);
            }
            __syncthreads();
        }
        if (way == 0 && e < n) tab_st(out, e, f9_to_fr(acc));
    }
}

// Outputs a block by the number of chunks: a lane makes at most four trips up to 256 chunks; beyond, fewer outputs a block cost
// shorter runs of each plane (16 bytes) and still win.  64 / 16 / 4 outputs a block (us): 16384 outputs in 16 chunks 4.2 / 6.6 / 18,
// 8192 in 32 4.5 / 5.7 / 13, 4096 in 64 6.2 / 5.6 / 13, 2048 in 128 10 / 6.2 / 13, 1024 in 256 18 / 8.9 / 13, 512 in 256
// 18 / 8.1 / 9.0, one in 1024 72 / 28 / 6.9, 8 in 1024 106 / 17 / 6.8, 64 in 4096 234 / 70 / 44, 8 in 4096 353 / 60 / 18.
constexpr uint64_t SUM_64_CHUNKS = 32, SUM_16_CHUNKS = 256;
static void launch_sum_chunks(zkdl_ctx* ctx, FrTab part, uint64_t n, uint64_t chunks, FrTab out) {
    if (chunks <= SUM_64_CHUNKS)
        hipLaunchKernelGGL(k_sum_chunks<64>, dim3(grid_for(4 * n)), dim3(ZK_BLOCK), 0, ctx->stream, part, n, chunks, out);
    else if (chunks <= SUM_16_CHUNKS)
        hipLaunchKernelGGL(k_sum_chunks<16>, dim3(grid_for(16 * n)), dim3(ZK_BLOCK), 0, ctx->stream, part, n, chunks, out);
    else
        hipLaunchKernelGGL(k_sum_chunks<4>, dim3(grid_for(64 * n)), dim3(ZK_BLOCK), 0, ctx->stream, part, n, chunks, out);
}

static void launch_pe(zkdl_ctx* ctx, int kind, bool inner, const PeArgs& p, dim3 grid) {
    const dim3 block(ZK_BLOCK);
    if (kind == TK_I32) {
        if (inner) hipLaunchKernelGGL(k_pe_inner<TK_I32>, grid, block, 0, ctx->stream, p);
        else hipLaunchKernelGGL(k_pe_mid_int<TK_I32>, grid, block, 0, ctx->stream, p);
    } else if (kind == TK_I64) {
        if (inner) hipLaunchKernelGGL(k_pe_inner<TK_I64>, grid, block, 0, ctx->stream, p);
        else hipLaunchKernelGGL(k_pe_mid_int<TK_I64>, grid, block, 0, ctx->stream, p);
    } else {
        if (inner) hipLaunchKernelGGL(k_pe_inner<TK_FR>, grid, block, 0, ctx->stream, p);
        else if (p.a_chunk <= PE_LAZY_MAX_CHUNK) hipLaunchKernelGGL(k_pe_mid_lazy<TK_FR>, grid, block, 0, ctx->stream, p);
        else hipLaunchKernelGGL(k_pe_mid<TK_FR>, grid, block, 0, ctx->stream, p);
    }
}

// The innermost axis (I = 1) of an integer source of O rows of A entries: a lane per row (k_pe_inner_int) or a wave along
// each row (k_pe_inner).
// An int32 costs a lane nine multiply-adds, so that 64 rows side by side win from one wave's width on.  An int64 costs it
// 27, and lanes without a row idle: few rows leave most of a wave unused, and short inputs are bound by the tile's serial
// chain.  Whole mle_partial_eval calls on int64 (us, wave along the row / lane per row):
//   rows x 2^k: 1 x 2^13 44 / 52, 1 x 2^20 163 / 390, 1 x 2^23 512 / 1755, 8 x 2^20 314 / 393, 16 x 2^17 114 / 140,
//   16 x 2^18 176 / 164, 32 x 2^13 40 / 49, 32 x 2^14 64 / 56, 32 x 2^18 284 / 167, 64 x 2^12 38 / 43, 64 x 2^13 46 / 47,
//   64 x 2^14 77 / 55, 1024 x 2^8 31 / 38, 1024 x 2^9 39 / 40, 1024 x 2^10 53 / 41, 4096 x 2^6 30 / 35, 4096 x 2^7 36 / 38,
//   4096 x 2^11 177 / 61.
bool zk_pe_lane_per_row(int kind, uint64_t O, uint64_t A) {
    if (kind == TK_FR || A < 64) return false;
    if (kind == TK_I32) return true;
    if (O < 16) return false;
    const uint64_t from = (uint64_t)1 << (O >= 32 ? 19 : 22);   // entries in all
    return A >= (from + O - 1) / O;
}

int zk_partial_eval(zkdl_ctx* ctx, int kind, const void* src, uint64_t O, uint64_t A, uint64_t I,
                    FrTab beta, FrTab out) {
    PeArgs p;
    p.src = src;
    if (kind == TK_FR) p.fr_src = *(const FrTab*)src;
    else p.fr_src = make_tab(nullptr, 0);
    p.beta = beta;
    p.O = O;
    p.A = A;
    p.I = I;
    uint64_t n_out = O * I;
    const bool inner = (I == 1);
    if (inner && zk_pe_lane_per_row(kind, O, A)) {
        // row tiles of 64 outputs x chunks of the axis, about a thousand single-wave blocks
        const uint64_t tiles = (O + 63) / 64;
        uint64_t chunks = 1;
        while (tiles * chunks < 1024 && A / (chunks * 2) >= 64) chunks *= 2;
        while (A / chunks > PE_LAZY_MAX_CHUNK) chunks *= 2;
        if (tiles <= 0x7fffffffu && chunks <= 65535) {
            p.a_chunk = (A + chunks - 1) / chunks;
            void* tmp = nullptr;
            if (chunks > 1) {
                tmp = zk_alloc(ctx, chunks * n_out * 32);
                if (!tmp) return ZKDL_ENOMEM;
                p.out = make_tab(tmp, chunks * n_out);
            } else {
                p.out = out;
            }
            zk_prof_begin(ctx, ZKDL_PROF_PARTIAL_EVAL,
                          (kind == TK_I32 ? 4.0 : 8.0) * (double)O * (double)A + 32.0 * (double)A + 32.0 * (double)n_out);
            const dim3 grid((unsigned)tiles, (unsigned)chunks);
            if (kind == TK_I32) hipLaunchKernelGGL(k_pe_inner_int<TK_I32>, grid, dim3(64), 0, ctx->stream, p);
            else hipLaunchKernelGGL(k_pe_inner_int<TK_I64>, grid, dim3(64), 0, ctx->stream, p);
            zk_prof_end(ctx);
            if (chunks > 1) {
                launch_sum_chunks(ctx, p.out, n_out, chunks, out);
                zk_free(ctx, tmp);
            }
            return ZKDL_OK;
        }
    }
    // split the contracted axis until there is enough parallel work: the thread-per-output
    // kernels hide their load latency only with several waves per SIMD (~256k threads)
    uint64_t units = inner ? n_out * 64 : n_out;
    uint64_t chunks = 1;
    const uint64_t want_units = inner ? 65536 : 262144;
    while (units * chunks < want_units && chunks * 2 <= A && (A / (chunks * 2)) >= (inner ? 64u : 4u)) chunks *= 2;
    while (!inner && A / chunks > PE_LAZY_MAX_CHUNK && chunks < 32768) chunks *= 2;
    p.a_chunk = (A + chunks - 1) / chunks;
    void* tmp = nullptr;
    if (chunks > 1) {
        tmp = zk_alloc(ctx, chunks * n_out * 32);
        if (!tmp) return ZKDL_ENOMEM;
        p.out = make_tab(tmp, chunks * n_out);
    } else {
        p.out = out;
    }
    dim3 grid;
    if (inner) {
        uint64_t waves = n_out * chunks;
        grid = dim3(grid_for(waves * 64, 16384));
    } else {
        grid = dim3(grid_for(n_out, 16384), (unsigned)chunks);
    }
    // algorithmic bytes: the source once, beta once per (outer, inner) tile is cached: count it once, the output
    const double esz = kind == TK_FR ? 32.0 : kind == TK_I32 ? 4.0 : 8.0;
    zk_prof_begin(ctx, ZKDL_PROF_PARTIAL_EVAL, esz * (double)O * (double)A * (double)I + 32.0 * (double)A + 32.0 * (double)n_out);
    launch_pe(ctx, kind, inner, p, grid);
    zk_prof_end(ctx);
    if (chunks > 1) {
        launch_sum_chunks(ctx, p.out, n_out, chunks, out);
        zk_free(ctx, tmp);
    }
    return ZKDL_OK;
}

// out[r * inner + i] = src[r] : the stack-axis table beta~(w, n) seen over (n, i)
__global__ __launch_bounds__(ZK_BLOCK) void k_broadcast_rows(FrTab src, uint64_t rows, uint64_t inner,
                                                             FrTab out) {
    uint64_t n = rows * inner;
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < n;
         e += (uint64_t)gridDim.x * blockDim.x)
        tab_st(out, e, tab_ld(src, e / inner));
}

void zk_launch_broadcast_rows(zkdl_ctx* ctx, FrTab src, uint64_t rows, uint64_t inner, FrTab out) {
    hipLaunchKernelGGL(k_broadcast_rows, dim3(grid_for(rows * inner)), dim3(ZK_BLOCK), 0, ctx->stream,
                       src, rows, inner, out);
}

// out[r] = src[r + 1] unless r is the last slot of its period, where out[r] = 0:
// the stack re-indexing "layer l <- layer l+1" of the gradA family
__global__ __launch_bounds__(ZK_BLOCK) void k_shift_rows(FrTab src, uint64_t rows, uint64_t inner,
                                                         uint32_t period, FrTab out) {
    uint64_t n = rows * inner;
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < n;
         e += (uint64_t)gridDim.x * blockDim.x) {
        uint64_t r = e / inner;
        bool last = (r % period) == period - 1;
        tab_st(out, e, last ? fr_zero() : tab_ld(src, e + inner));
    }
}

void zk_launch_shift_rows(zkdl_ctx* ctx, FrTab src, uint64_t rows, uint64_t inner, uint32_t period,
                          FrTab out) {
    hipLaunchKernelGGL(k_shift_rows, dim3(grid_for(rows * inner)), dim3(ZK_BLOCK), 0, ctx->stream, src,
                       rows, inner, period, out);
}

// small SoA table -> array of structures (tables that single-block kernels index directly)
__global__ void k_soa_to_aos(FrTab in, int n, Fr* out) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = tab_ld(in, i);
}

void zk_launch_soa_to_aos(zkdl_ctx* ctx, FrTab in, int n, Fr* out) {
    hipLaunchKernelGGL(k_soa_to_aos, dim3((n + 63) / 64), dim3(64), 0, ctx->stream, in, n, out);
}
