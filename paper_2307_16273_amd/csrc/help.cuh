// Helper blocks: blocks of one launch that work for a block that hashes (the leader, block 0), and how they talk to each other.
//
// Messages go through device memory by 32-bit words that carry their own validity: limbs have 29 bits, the upper three
// hold a number that follows from the round (never 0), and whoever waits re-reads until every word has it.  No flag, no fence, one trip.  The
// accesses are agent-scope atomics, which the L2s of the eight XCDs do not hold back.  A slot is written again two rounds later, after its reader has shown by
// another message that it has read it; the leader clears all slots before it ends.
//
// Progress.  Helpers report when they start.  If not all of them have in time (ZkHelpLaunch::report; other streams fill the GPU), the leader
// goes on alone, with the tables in device memory; so no block ever waits for one that is not running.  A helper that starts later reads its
// tables and makes its first sums like any other (k_zk_helped's leader folds the same tables in place meanwhile: what it has then is of no
// use to anyone), looks at `go`, and leaves without a message.  Waits for running blocks end all the same (ZkHelpLaunch::wait; after 0 ticks: at the first look), with an error for the caller.
#pragma once
#include "dev_common.cuh"

constexpr int HELP_WORDS = 10;                    // words of a message's field element: nine limbs, read in pairs

__device__ __forceinline__ uint32_t help_tag(int t) { return (uint32_t)(1 + t % 7) << 29; }
__device__ __forceinline__ void help_st(uint32_t* p, uint32_t x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint32_t help_ld(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

struct HelpWait {
    uint64_t until;
    uint32_t n;
    bool late;       // the same in every lane of a wave
    __device__ __forceinline__ void begin(uint64_t ticks) {
        until = wall_clock64() + ticks;
        n = 0;
        late = ticks == 0;
    }
    // another look at the message? (a clock read every 16 looks)
    __device__ __forceinline__ bool again() {
        if ((++n & 15) == 0 && wall_clock64() > until) late = true;
        return !late;
    }
};

// N field elements of the calling lane from messages p[0], p[stride], ..; the whole wave waits until all its lanes have theirs
template <int N>
__device__ __forceinline__ bool help_read(const uint32_t* p, uint32_t stride, uint32_t tag, bool mine, F9 (&out)[N], HelpWait& w) {
    for (;;) {
        uint32_t bad = 0;
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const uint64_t* at = (const uint64_t*)(p + (size_t)q * stride);
            uint64_t x[HELP_WORDS / 2];
#pragma unroll
            for (int l = 0; l < HELP_WORDS / 2; ++l) x[l] = __hip_atomic_load(at + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int l = 0; l < 9; ++l) {
                const uint32_t word = (uint32_t)(x[l >> 1] >> (32 * (l & 1)));
                bad |= (word ^ tag) >> 29;
                out[q].v[l] = word & frc::M29;
            }
        }
        if (__ballot(mine && bad != 0) == 0) return true;
        if (w.late || !w.again()) return false;
    }
}
// a normal field element, limb by limb
__device__ __forceinline__ void help_write(uint32_t* p, uint32_t tag, const F9& x) {
#pragma unroll
    for (int l = 0; l < 9; ++l) help_st(p + l, tag | x.v[l]);
}


// ---- helpers ----
__device__ __forceinline__ void help_report(const ZkHelpLaunch& a) {     // one thread, first of all
    if (!a.quiet) __hip_atomic_fetch_add(&a.mail->started[a.epoch & 1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// one wave, before the first message: whether all helpers run
__device__ __forceinline__ bool help_may_go(const ZkHelpLaunch& a) {
    HelpWait w;
    w.begin(a.wait);
    uint32_t go = help_ld(&a.mail->go);
    while ((go >> 1) != a.epoch && w.again()) {
        __builtin_amdgcn_s_sleep(2);
        go = help_ld(&a.mail->go);
    }
    return go == 2 * a.epoch;
}
// one wave: challenge v_t to LDS; false if it does not come
__device__ __forceinline__ bool help_challenge(const ZkHelpLaunch& a, int t, F9& v) {
    const int lane = threadIdx.x & 63;
    HelpWait w;
    w.begin(a.wait);
    const uint32_t tag = help_tag(t);
    uint32_t word = 0;
    for (;;) {
        word = lane < 9 ? help_ld(&a.mail->v[t & 1][lane]) : tag;
        if (__ballot(((word ^ tag) >> 29) != 0) == 0) break;
        if (!w.again()) break;
    }
    if (lane < 9) v.v[lane] = word & frc::M29;
    return !w.late;
}

// ---- the leader ----
// one wave: all `count` helpers, or none of them (*alone = 1)
__device__ __forceinline__ void help_gather(const ZkHelpLaunch& a, uint32_t count, uint32_t* alone) {
    ZkHelpMail* mail = a.mail;
    const uint32_t epoch = a.epoch;
    HelpWait w;
    w.begin(a.report);
    bool all = help_ld(&mail->started[epoch & 1]) == count;
    while (!all && w.again()) all = help_ld(&mail->started[epoch & 1]) == count;
    if ((threadIdx.x & 63) == 0) {
        help_st(&mail->go, 2 * epoch + (all ? 0 : 1));
        help_st(&mail->started[(epoch + 1) & 1], 0);     // nobody counts there until the next launch
        *alone = all ? 0 : 1;
    }
}
// one wave: v_t to the helpers
__device__ __forceinline__ void help_publish(ZkHelpMail* mail, int t, const F9& v) {
    const int lane = threadIdx.x & 63;
    if (lane < 9) {
        uint32_t word = v.v[0];
#pragma unroll
        for (int l = 1; l < 9; ++l) word = lane == l ? v.v[l] : word;
        help_st(&mail->v[t & 1][lane], help_tag(t) | word);
    }
}
// The end (all threads call).  Every message has been read: empty slots for the next launch.  After a wait that was given up a helper may
// still write; then the mail stays as it is, and the host, which sees the error, clears it before the next call.
__device__ __forceinline__ void help_end(ZkHelpMail* mail, DevState* st, bool late, uint32_t* flag, int threads) {
    if (late && (threadIdx.x & 63) == 0) {
        atomicOr(&st->err, ZK_ERR_HELPERS);
        *flag = 1;
    }
    __syncthreads();
    if (*flag) return;
    for (uint32_t i = threadIdx.x; i < sizeof(mail->coef) / 4; i += threads) help_st((uint32_t*)mail->coef + i, 0);
    for (uint32_t i = threadIdx.x; i < sizeof(mail->tab) / 4; i += threads) help_st((uint32_t*)mail->tab + i, 0);
    if (threadIdx.x < sizeof(mail->v) / 4) help_st((uint32_t*)mail->v + threadIdx.x, 0);
}
