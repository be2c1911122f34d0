// gfx950 kernels of the Elastic Shadow Pricing hot path (paper Sec. 3.2), as
// templates; esp_kernels.hip dispatches on R at run time and the
// esp_inst_*.hip files instantiate the fused kernels (split by R so that
// they compile in parallel).
//
// One price iteration = one launch of a fused kernel:
//   score   s_jk = u_jk - sum_r lambda_r d_jkr          (Sec. 3.2.2, bracket of Eq. 6)
//   select  c_j  = argmax_k s_jk, lowest k on ties     (Sec. 3.2.2 per-job subproblem)
//   demand  U_r  = sum_j d_{j,c_j,r}, exact             (Sec. 3.2.3, under Eq. 8)
//   update  lambda_r <- max(0, lambda_r + eta_t (U_r - C_r))  (Eq. 8)
//
// With several workgroups per cluster, such a launch ends once every workgroup
// has published its exact demand sums; every workgroup of the cluster then
// computes U and the update itself at the start of the next launch (integer
// sums: all obtain the same bits), so no workgroup waits for a last one to
// finish the update.  With one workgroup per cluster the workgroup updates at
// the end of its own iteration.  Launches of several iterations exchange the
// sums among the workgroups at the end of each (resident_complete).
//
// Table layout (built by the packer): per cluster, one fp32 column for the
// utility and one per resource, each a sequence of 256-entry tiles.  A
// wavefront scores one tile per step with one 128-bit load per lane per
// column (lane l holds entries 4l .. 4l+3 of the tile).
//
// Arithmetic contract: binary64, no contraction (`fp contract(off)` below and
// -ffp-contract=off on the command line), rent summed left to right over r.
// The demand sum is exact: each fp32 demand is turned into a 128-bit integer
// multiple of 2^shift (the column's lowest set bit, fixed by the packer),
// integers are added in any order, and the total is rounded once to binary64
// (round-to-nearest-even).  No floating-point atomics are used.
#pragma once

#include <algorithm>
#include <type_traits>

#include "esp_device.hpp"

#pragma clang fp contract(off)

namespace esp {

// ---------------------------------------------------------------------------
// Cluster completion: per-workgroup sums -> last workgroup -> U, Eq. 8 update
// ---------------------------------------------------------------------------

// eta_t of Eq. 8 for the launch's step index t: eta0 or eta0 / sqrt(t), one
// IEEE division and one correctly rounded square root in binary64 (no fast
// math), so the value equals the host's.
__device__ __forceinline__ double step_size(const KArgs &a, int cl, int t) {
    const double e0 = a.eta0[cl];
    return a.rule == 1 ? e0 / sqrt(static_cast<double>(t)) : e0;
}

// U_r from the cluster's exact total, the Eq. 8 update and the stop test for
// resource r (one thread per resource of the cluster's last workgroup).
// lam_cur (LDS) holds the prices the iteration selected at.  Gather: the
// launch is esp_reduce_demand's, whose workgroups flag invalid choices
// (flag 4) during the launch; no other launch sets that flag.  An update
// (lam_out set) happens only with one workgroup per cluster (deferred
// completion otherwise), so the prices, the trace rows and the iteration
// count each have one writer in a launch; the next launch reads them after
// the launch boundary: plain stores.
template <int R, bool Gather>
__device__ __forceinline__ void complete_resource(const KArgs &a, int cl, int r, u128 tot, const double *lam_cur,
                                                  int *s_ok, double *s_newlam) {
    const bool bad =
        Gather && a.flags && (__hip_atomic_load(&a.flags[cl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 4);
    const double U = bad ? __builtin_nan("") : fx_to_double(tot, a.shift[cl * R + r]);
    if (a.demand_out) a.demand_out[cl * R + r] = U;
    if (a.tr_U) a.tr_U[cl * R + r] = U;
    int ok = 1;
    if (a.lam_out) {
        const double lo = lam_cur[r];
        const double g = U - a.cap[cl * R + r];
        const double x = lo + step_size(a, cl, a.t) * g;
        const double ln = (x > 0.0) ? x : 0.0;
        a.lam_out[cl * R + r] = ln;
        if (a.tr_lam) a.tr_lam[cl * R + r] = ln;
        s_newlam[r] = ln;
        const double diff = fabs(ln - lo);
        const double scale = lo > 1.0 ? lo : 1.0;
        ok = diff <= a.tol * scale;
    }
    s_ok[r] = ok;
}

// Per-cluster bookkeeping after the update (thread 0 of the last workgroup).
// Returns whether the cluster stops (tol reached).
template <int R, bool Gather>
__device__ __forceinline__ int complete_cluster(const KArgs &a, int cl, const int *s_ok) {
    int stop = 0;
    if (Gather && a.flags && (a.flags[cl] & 4)) atomicAnd(&a.flags[cl], ~4);
    if (a.lam_out) {
        if (a.iters_done) a.iters_done[cl] = a.iter_no;
        int all = 1;
        for (int r = 0; r < R; ++r) all &= s_ok[r];
        if (a.tol > 0.0 && all && a.flags) {
            atomicOr(&a.flags[cl], kFlagStopped);
            stop = 1;
        }
    }
    return stop;
}

// The demand sums of one iteration: U, the Eq. 8 update and the per-cluster
// bookkeeping in the last workgroup.  s_newlam / s_stop (LDS) receive the new
// prices and the stop decision there.
template <int R, bool Gather>
__device__ bool finish_cluster(const KArgs &a, int cl, int blk, const u128 *bsum, const double *lam_cur,
                               double *s_newlam, int *s_stop) {
    __shared__ int s_ok[R];
    const bool last = cluster_sums<R>(a, cl, blk, bsum, [&](int r, u128 tot) {
        complete_resource<R, Gather>(a, cl, r, tot, lam_cur, s_ok, s_newlam);
    });
    if (!last) return false;
    if (threadIdx.x == 0) *s_stop = complete_cluster<R, Gather>(a, cl, s_ok);
    __syncthreads();
    return true;
}

// ---------------------------------------------------------------------------
// Deferred completion (several workgroups per cluster)
// ---------------------------------------------------------------------------

// Complete iteration m of cluster cl (step index t_m) from the sums it
// published into buffer m & 1, whose first loads (partial_loads) are in v:
// U_m, lambda_{m+1} of Eq. 8 and the stop test.  lam_m (LDS) holds the
// prices iteration m selected at; lam_next (LDS) receives lambda_{m+1};
// s_red is LDS scratch.  All threads take part and get whether the tolerance
// is met.  The writer (workgroup 0 of the cluster) also stores
// lambda_{m+1} into the caller's prices and lam_ws, the trace rows of
// iteration m, the iteration count, and m as the stop iteration.
template <int R, typename A>
__device__ bool complete_iteration(const KArgs &a, int cl, int m, int t_m, bool writer, const double *lam_m,
                                   double *lam_next, u128 *s_red, const A (&v)[kSumLoads]) {
    __shared__ int s_ok[R];
    partial_totals<R, A, false>(a, m & 1, cl, v, s_red);
    const int t = threadIdx.x;
    if (t < R) {
        const size_t i = static_cast<size_t>(cl) * R + t;
        const double U = fx_to_double(s_red[t], a.shift[i]);
        const double lo = lam_m[t];
        const double g = U - a.cap[i];
        const double x = lo + step_size(a, cl, t_m) * g;
        const double ln = (x > 0.0) ? x : 0.0;
        lam_next[t] = ln;
        const double diff = fabs(ln - lo);
        const double scale = lo > 1.0 ? lo : 1.0;
        s_ok[t] = diff <= a.tol * scale;
        if (writer) {
            const size_t BR = static_cast<size_t>(a.B) * R;
            a.lam_dst[i] = ln;
            a.lam_ws[static_cast<size_t>((m + 1) & 1) * BR + i] = ln;
            if (a.trace_U) a.trace_U[static_cast<size_t>(m - 1) * BR + i] = U;
            if (a.trace_lam) a.trace_lam[static_cast<size_t>(m - 1) * BR + i] = ln;
        }
    }
    __syncthreads();
    int all = 1;
#pragma unroll
    for (int r = 0; r < R; ++r) all &= s_ok[r];
    const bool stop = a.tol > 0.0 && all;
    if (writer && t == 0) {
        if (a.iters_done) a.iters_done[cl] = m;
        if (stop) __hip_atomic_store(&a.conv_at[cl], m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return stop;
}

// The loads of a launch's pending completion (pend_m > 0).  They are issued
// before the first tiles' loads, so they return first and the completion
// runs while the tiles are still in flight; they are issued whether or not
// the completion turns out to be needed.
template <int R, typename A>
struct Pending {
    A v[kSumLoads];      // this thread's first published sums of iteration pend_m
    double lam_m = 0.0;  // thread t < R: lambda_{pend_m}[t]
    int conv = 0;        // conv_at[cl]
};

// conv: conv_at[cl], read by the caller at the start of the launch together
// with the cluster's flags.  Within a launch conv_at changes only from 0 to
// pend_m (workgroup 0 completing pend_m itself), and both values lead to the
// same path, so a value read before that store is as good as one read after.
// The loads are issued whether or not a completion is pending, from valid
// addresses and without branches, so that the compiler waits for exactly
// these loads (and not for the tile loads issued after them) where they are
// used.
template <int R, typename A>
__device__ __forceinline__ void pending_loads(const KArgs &a, int cl, int conv, Pending<R, A> &p) {
    const int k = a.pend_m & 1;
    p.conv = conv;
    p.lam_m = a.lam_ws[static_cast<size_t>(k) * a.B * R + static_cast<size_t>(cl) * R + threadIdx.x % R];
    partial_loads<R, A, false>(a, k, cl, p.v);
}

// Prices of the launch's first iteration, into s_lam (LDS).  A launch with a
// pending completion first completes iteration pend_m, unless the cluster
// met the tolerance at an earlier iteration (conv_at 0 or pend_m: complete
// it here; every workgroup then reaches the same decision).  Returns false
// when the cluster has nothing left to do in this launch (it has converged
// and the launch runs solve iterations).
template <int R, typename A>
__device__ bool launch_prices(const KArgs &a, int cl, int blk, const Pending<R, A> &p, double *s_lam,
                              double *s_tmp, u128 *s_red) {
    const int t = threadIdx.x;
    if (a.pend_m > 0) {
        if (p.conv == 0 || p.conv >= a.pend_m) {
            if (t < R) s_tmp[t] = p.lam_m;
            __syncthreads();
            const bool stop =
                complete_iteration<R, A>(a, cl, a.pend_m, a.pend_t, blk == 0, s_tmp, s_lam, s_red, p.v);
            return !(stop && a.defer);
        }
        if (a.defer) return false;
        // met the tolerance earlier: the caller's prices are final and are not
        // written in this launch
    }
    if (t < R) s_lam[t] = a.lam_in[cl * R + t];
    __syncthreads();
    return true;
}

// End of iteration m in a deferred launch: publish the workgroup's sums
// (bsum, LDS) into buffer m & 1.  Plain stores: the next launch reads the sums
// after the launch boundary.
template <int R>
__device__ __forceinline__ void publish_iteration(const KArgs &a, int cl, int blk, int m, const u128 *bsum) {
    const int t = threadIdx.x;
    if (t < R) {
        uint64_t *p = partials_of<R>(a, m & 1, cl) + (static_cast<size_t>(blk) * R + t) * 2;
        const u128 v = bsum[t];
        p[0] = static_cast<uint64_t>(v);
        p[1] = static_cast<uint64_t>(v >> 64);
    }
}

// ---------------------------------------------------------------------------
// Multi-iteration launches: every iteration is completed inside the launch;
// with several workgroups per cluster their exact sums meet in counted words.
// ---------------------------------------------------------------------------
//
// Streaming launches use it too: a barrier of the grid and every workgroup
// reading every other's sums took 3 to 4 us more of each iteration (262,144
// ragged jobs x 6 21.0 -> 18.6 us, 1,048,576 64.8 -> 62.0, 262,144 x 12 x 8 23.2 ->
// 20.5), which also puts them ahead of one launch per iteration (21.6, 63.7, 22.9).

// A workgroup's sum for resource r is split into a.limbs limbs (one when the
// cluster's total fits kCountShift bits, else kLimbBits each): words of a
// 64-bit value below kCountShift and a count above.  The limbs of iteration m
// take three steps, each with agent-scope atomics only:
//  1. every workgroup adds its words, each with a count of one, to one of
//     `copies` copies of them (copy blk mod copies) with a returning atomic
//     add; the add that completes a copy's count returns the copy's sum;
//  2. that lane adds the copy's sum to the root words the same way, and the
//     add that completes the root has the cluster's total;
//  3. that lane stores the total, tagged with m, to `replicas` release words;
//     every workgroup polls its replica for the tag.
// So adds to one address stay few (each takes the memory side about 11 ns),
// and polls never touch a line that is still being added to: polling the
// copies themselves cost 0.4 to 1.5 us more at 128 to 256 workgroups.  An
// exchange alone takes 1.67 us for 64 to 256 workgroups; one in which each
// workgroup reads every other's words 2.4 and 4.2 us for 128 and 256.
//
// Copies and root have two sets, by the parity of m.  The lane that completes
// a word's count clears it at once (no other add to it comes before m + 2):
// it waits for the clear to have been performed before its own next add, in
// m + 1, and nobody adds to m + 2 before m + 1 is complete.  Release words
// alternate too; the tag tells m from m - 2.  The solve's prologue clears the
// words.
constexpr uint64_t kLimbMask = (1ull << kLimbBits) - 1;
constexpr int kSlotWords = kSyncStride / 2;    // 64-bit words of a 256-byte slot of the exchange words
constexpr int kReplicas = 4;

// Where this lane's word (lane = limb * R + resource) is added and released;
// fixed per launch.  Copies lie in slots of their own; with at most 8 words
// both sets fill a slot's first 128-byte line, and a release line its second.
struct Exchange {
    uint64_t *copy, *root, *release;           // set 0 of each
    int set_words, release_words;              // words from set 0 to set 1
    int replica_words;                         // words between replicas
    int words;                                 // R * limbs (lanes that take part)
    int in_copy;                               // workgroups that add to this copy
    int copies, replicas, first_replica;
};
template <int R>
__device__ __forceinline__ Exchange exchange_of(const KArgs &a, int cl, int blk, int lane) {
    uint64_t *const base = reinterpret_cast<uint64_t *>(a.sync + static_cast<size_t>(cl) * kSyncSlots * kSyncStride);
    Exchange x;
    x.words = R * a.limbs;
    const int q = lane < x.words ? lane : 0;
    const int line = (x.words + 7) / 8 * 8;                // 8, 16 or 24 words
    const int span = (2 * line + kSlotWords - 1) / kSlotWords * kSlotWords;   // both sets of a copy
    x.copies = min(a.nblk, exchange_copies(x.words));
    x.replicas = min(a.nblk, kReplicas);
    const int mine = blk % x.copies;
    x.in_copy = a.nblk / x.copies + (mine < a.nblk % x.copies ? 1 : 0);
    x.set_words = line;
    x.copy = base + mine * span + q;
    const int top = exchange_copies(x.words);
    x.root = base + top * span + q;
    // 17 slots: 16 copies and the root with release lines in the second halves, or 8 (4) copies, the
    // root and 8 release lines of 16 (24) words
    static_assert(kSyncSlots * kSlotWords >= 5 * 64 + 2 * kReplicas * 24, "4 copies of 24 words fit");
    static_assert(kSyncSlots >= 17, "16 copies and the root fit");
    x.release_words = line == 8 ? kSlotWords : line;
    x.replica_words = 2 * x.release_words;
    x.first_replica = blk % x.replicas;
    x.release = base + (line == 8 ? kSlotWords / 2 : (top + 1) * span) + q;
    return x;
}

// Sum of v over the lanes with the same index modulo RP (a power of two up to
// 8), in every lane: rotations inside the 16-lane rows, then row swaps.
template <typename A>
struct Words {                                 // a value as 32-bit words
    uint32_t w[sizeof(A) / 4];
};
template <typename A, typename Move>
__device__ __forceinline__ A moved(A v, Move &&move) {
    Words<A> x = __builtin_bit_cast(Words<A>, v);
#pragma unroll
    for (uint32_t &w : x.w) w = static_cast<uint32_t>(move(static_cast<int>(w)));
    return __builtin_bit_cast(A, x);
}
template <int RP, typename A>
__device__ __forceinline__ A lane_sum(A v) {
    constexpr int kRor1 = 0x121, kRor2 = 0x122, kRor4 = 0x124, kRor8 = 0x128;
    if constexpr (RP <= 1) v += moved(v, [](int x) { return dpp_i<kRor1>(x); });
    if constexpr (RP <= 2) v += moved(v, [](int x) { return dpp_i<kRor2>(x); });
    if constexpr (RP <= 4) v += moved(v, [](int x) { return dpp_i<kRor4>(x); });
    v += moved(v, [](int x) { return dpp_i<kRor8>(x); });
    // both halves of a swap of x with itself: the other row in every lane of one of them
    Words<A> lo = __builtin_bit_cast(Words<A>, v), hi = lo;
#pragma unroll
    for (size_t i = 0; i < sizeof(A) / 4; ++i) {
        const auto p = __builtin_amdgcn_permlane16_swap(lo.w[i], hi.w[i], false, false);
        lo.w[i] = p[0];
        hi.w[i] = p[1];
    }
    v = __builtin_bit_cast(A, lo) + __builtin_bit_cast(A, hi);
    lo = hi = __builtin_bit_cast(Words<A>, v);
#pragma unroll
    for (size_t i = 0; i < sizeof(A) / 4; ++i) {
        const auto p = __builtin_amdgcn_permlane32_swap(lo.w[i], hi.w[i], false, false);
        lo.w[i] = p[0];
        hi.w[i] = p[1];
    }
    return __builtin_bit_cast(A, lo) + __builtin_bit_cast(A, hi);
}

// The smallest power of two not below R: in resident launches lane l
// accumulates resource l mod RP (the lanes with l mod RP >= R nothing).
template <int R>
constexpr int kResidentStep = R <= 1 ? 1 : R <= 2 ? 2 : R <= 4 ? 4 : 8;

// Step sizes eta_t of all iterations of a resident launch, computed once at
// its start by the whole workgroup (the same IEEE operations as step_size, so
// the same bits), so that no division or square root lies on an iteration's
// path.  The caller synchronizes the workgroup before the first read.
__device__ __forceinline__ const double *resident_etas(const KArgs &a, int cl) {
    __shared__ double s_eta[kLaunchChunk];
    for (int i = threadIdx.x; i < a.n_iters; i += blockDim.x) s_eta[i] = step_size(a, cl, a.t + i);
    return s_eta;
}

// What does not change between the iterations, or is carried over, in lanes
// r < R of wavefront 0.
struct ResidentCtx {
    double lo;            // the iteration's price of resource r
    double cap;           // its capacity and fixed-point window
    int shift;
    int done;             // iterations completed in this launch
    bool stop;            // the last one met the tolerance
};

// prices: the launch's starting prices of the cluster, [R]
template <int R>
__device__ __forceinline__ ResidentCtx resident_ctx(const KArgs &a, int cl, int lane, const double *prices) {
    const int r = lane < R ? lane : R - 1;
    ResidentCtx c;
    c.lo = prices[r];
    c.cap = a.cap[static_cast<size_t>(cl) * R + r];
    c.shift = a.shift[static_cast<size_t>(cl) * R + r];
    c.done = 0;
    c.stop = false;
    // loaded before the loop: a load still counted as pending there would make
    // every iteration wait for all of its own stores
    asm volatile("" : "+v"(c.lo), "+v"(c.cap), "+v"(c.shift));
    return c;
}

// The exchange of iteration m: this lane's word `v` (lanes below xch.words)
// becomes the cluster's total.  Returns false after about 2 s (resident_outputs
// records it).  Nothing else ends a wait: the status word is shared by all
// clusters and may hold an error of another cluster or of an earlier call.  A
// workgroup gives up once, so the others of its cluster do after at most 2 s more.
__device__ __forceinline__ bool exchange_total(const Exchange &xch, int m, int lane, uint64_t &v) {
    constexpr uint64_t kOne = 1ull << kCountShift, kLow = kOne - 1;
    const int par = m & 1;
    const uint64_t tag = static_cast<uint64_t>(m % 255 + 1) << kCountShift;
    uint64_t *const release = xch.release + par * xch.release_words;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the clears of iteration m - 1 have been performed
    if (lane < xch.words) {
        uint64_t *const copy = xch.copy + par * xch.set_words;
        const uint64_t c = __hip_atomic_fetch_add(copy, kOne + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (static_cast<int>(c >> kCountShift) == xch.in_copy - 1) {
            v += c & kLow;
            uint64_t *const root = xch.root + par * xch.set_words;
            const uint64_t t = __hip_atomic_fetch_add(root, kOne + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(copy, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (static_cast<int>(t >> kCountShift) == xch.copies - 1) {
                v += t & kLow;
                for (int k = 0; k < xch.replicas; ++k)
                    __hip_atomic_store(release + k * xch.replica_words, tag | v, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(root, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    const uint64_t *const from = release + xch.first_replica * xch.replica_words;
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    // (conditions of the whole wavefront only: a branch per lane in here lengthens every poll, 4,096
    // jobs x 32 x 4 2.51 -> 2.44 us an iteration without it)
    for (int tries = 1;; ++tries) {
        const uint64_t x = __hip_atomic_load(from, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v = x & kLow;
        if (__ballot((x & ~kLow) != tag) == 0) return true;   // (lanes without a word read word 0)
        if ((tries & 63) == 0 && __builtin_amdgcn_s_memrealtime() - t0 > 200000000ull) return false;
    }
}

// End of iteration `it` (0-based) of a resident launch.  `acc` is this lane's
// exact partial sum for resource lane mod kResidentStep<R> (0 in lanes without
// one); lam receives lambda_{m+1}.  An iteration is one dependent chain, so
// only its latency counts:
//  1. each wavefront totals its lanes in registers and posts R sums in LDS;
//  2. after the barrier wavefront 0 adds the wavefronts' sums, and with
//     several workgroups exchanges them;
//  3. its lanes r < R compute U_r (exact total rounded once), lambda_r of Eq. 8
//     and the stop test, in the same bits in every workgroup, and post the new
//     prices for a second barrier (in workgroup 0 they also write the trace
//     rows; the prices and counts are written once, by resident_outputs).
// Returns false when the cluster stops here or a wait timed out.
// Group > 0: `acc` is the wavefront's total already, of resource lane / Group.
// between() runs in every wavefront before the second barrier: a streaming
// launch issues its next tile loads there, wavefront 0 after its exchange
// (memory returns in order: loads issued before would hold the exchange up).
struct Nothing {
    __device__ __forceinline__ void operator()() const {}
};
// The wavefronts' sums of an iteration (LDS).  A launch of fewer than Waves
// wavefronts sets them to 0 first: those of the missing ones stay so.
template <int R, int Waves, typename A>
__device__ __forceinline__ A (&wave_sums())[Waves][R] {
    __shared__ A s_wave[Waves][R];
    return s_wave;
}
template <int R, int Waves, int Group, typename A, typename Between = Nothing>
__device__ __forceinline__ bool resident_complete(const KArgs &a, int it, int cl, int blk, int wave, int lane, A acc,
                                                  double eta, double (&lam)[R], ResidentCtx &ctx, const Exchange &xch,
                                                  Between &&between = {}) {
    A(&s_wave)[Waves][R] = wave_sums<R, Waves, A>();
    __shared__ double s_price[R];
    __shared__ int s_go;
    if constexpr (Group > 0) {
        if (lane % Group == 0 && lane / Group < R) s_wave[wave][lane / Group] = acc;
    } else {
        const A ws = lane_sum<kResidentStep<R>>(acc);
        if (lane < R) s_wave[wave][lane] = ws;
    }
    __syncthreads();
    if (wave == 0) {
        // (every partial sum fits the accumulator type A: the packer sized A for
        // the whole column's total)
        A tot = 0;
        if constexpr (std::is_floating_point_v<A> || Waves <= kBlockWaves) {
#pragma unroll
            for (int w = 0; w < Waves; ++w) tot += s_wave[w][lane % R];
        } else {
            // (integer sums: with the upper wavefronts' behind a branch, 3,000 jobs x 16 x 5 of 54-bit
            // sums 3.61 -> 3.50 us an iteration, 9,000 x 64 x 8 of 96-bit ones 5.26 -> 5.13; binary64 ones
            // lose as much by it)
            A x[Waves];
#pragma unroll
            for (int w = 0; w < Waves; ++w) x[w] = s_wave[w][lane % R];
#pragma unroll
            for (int w = 0; w < kBlockWaves; ++w) tot += x[w];
            if (a.res_waves > kBlockWaves) {
#pragma unroll
                for (int w = kBlockWaves; w < Waves; ++w) tot += x[w];
            }
        }
        bool go = true;
        if (a.nblk > 1) {
            // lane l R + r exchanges limb l of resource r
            uint64_t v = fx_words(tot, ctx.shift);
            if constexpr (!std::is_floating_point_v<A>) if (xch.words > R)
                v = static_cast<uint64_t>(static_cast<u128>(tot) >> (kLimbBits * (lane < xch.words ? lane / R : 0))) & kLimbMask;
            go = exchange_total(xch, a.iter_no + it, lane, v);
            if constexpr (std::is_floating_point_v<A>) {
                tot = fx_to_double(v, ctx.shift);
            } else if (xch.words == R) {
                tot = static_cast<A>(v);
            } else {
                u128 t = 0;
                for (int l = 0; l < a.limbs; ++l)
                    t += static_cast<u128>(static_cast<uint64_t>(
                             __shfl(static_cast<unsigned long long>(v), l * R + lane % R))) << (kLimbBits * l);
                tot = static_cast<A>(t);         // the exact total, which fits A
            }
        }
        // U, Eq. 8 and the stop test in lanes r < R
        const double lo = ctx.lo;
        const double U = fx_to_double(tot, ctx.shift);
        const double gd = U - ctx.cap;
        const double next = lo + eta * gd;
        const double ln = (next > 0.0) ? next : 0.0;
        const double scale = lo > 1.0 ? lo : 1.0;
        const bool ok = (lane >= R) | (fabs(ln - lo) <= a.tol * scale);
        const bool stop = (a.tol > 0.0) & (__ballot(!ok) == 0);
        if (lane < R) s_price[lane] = ln;
        if (lane == 0) s_go = go & !stop;
        if (go) {
            ctx.lo = ln;
            ctx.done = it + 1;
            ctx.stop = stop;
            if ((blk == 0) & (lane < R)) {
                const size_t row = (static_cast<size_t>(it) * a.B + cl) * R + lane;
                if (a.tr_lam) a.tr_lam[row] = ln;
                if (a.tr_U) a.tr_U[row] = U;
            }
        }
    }
    between();
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) lam[r] = s_price[r];
    return s_go != 0;
}

// End of a resident launch: the prices, the update count and the stop flag of
// its last completed iteration; and a wait that ran out of time, in the status
// and in the cluster's flags, so that later launches of the solve skip its
// iterations (here and not where it is found: its constants would take
// registers of the whole loop).
template <int R>
__device__ __forceinline__ void resident_outputs(const KArgs &a, int cl, int blk, int wave, int lane,
                                                 const ResidentCtx &ctx) {
    if (wave != 0) return;
    if ((lane == 0) & !ctx.stop & (ctx.done < a.n_iters)) {
        atomicOr(&a.flags[cl], kFlagAborted);
        atomicCAS(a.status, 0, kStatusTimeout);
    }
    if ((blk != 0) | (ctx.done == 0)) return;
    if (lane < R) a.lam_out[static_cast<size_t>(cl) * R + lane] = ctx.lo;
    if (lane == 0) {
        if (a.iters_done) a.iters_done[cl] = a.iter_no + ctx.done - 1;
        if (ctx.stop) atomicOr(&a.flags[cl], kFlagStopped);
    }
}

// Per-iteration view of the arguments of a persistent launch.
template <int R>
__device__ __forceinline__ KArgs iteration_args(const KArgs &a, int it) {
    KArgs ai = a;
    const size_t i = static_cast<size_t>(it);
    ai.t = a.t + it;
    if (a.tr_lam) ai.tr_lam = a.tr_lam + i * a.B * R;
    if (a.tr_U) ai.tr_U = a.tr_U + i * a.B * R;
    if (a.choice) ai.choice = a.choice + i * a.B * a.N;
    ai.iter_no = a.iter_no + it;
    ai.reverse = a.reverse ^ (a.sweep_alt & it & 1);
    return ai;
}

// ---------------------------------------------------------------------------
// Dense families: K = 4 * LPJ configurations per job, LPJ lanes per job
// ---------------------------------------------------------------------------

// A valid price (Eq. 8): finite and not negative.
__device__ __forceinline__ bool price_ok(double x) {
    return x >= 0.0 && x <= 0x1p400;            // false for NaN and +-Inf
}

// Whether a launch has nothing to do for cluster cl.  A launch that checks its
// prices itself (a.check: a selection at the caller's prices, which then needs
// no launch of k_prepare before it, 2 us and the gap to the next launch) skips
// a cluster with a bad price; its first workgroup records what k_prepare would.
template <int R>
__device__ __forceinline__ bool skip_cluster(const KArgs &a, int cl, int blk) {
    if (!a.check) return a.flags && (a.flags[cl] & a.skip_mask);
    bool ok = true;
#pragma unroll
    for (int r = 0; r < R; ++r) ok = ok && price_ok(a.lam_in[cl * R + r]);
    if (blk == 0 && threadIdx.x == 0) {
        a.flags[cl] = (a.flags[cl] & kFlagFrozen) | (ok ? 0 : kFlagError);
        if (!ok) atomicCAS(a.status, 0, kStatusNonfinite);
    }
    return !ok;
}

// Launch modes of the fused kernels, one instance each, so that the
// one-iteration instance does without the code (and the registers) of the
// multi-iteration ones.  Multi-iteration launches complete every iteration
// themselves (resident_complete).
constexpr int kOnePass = 0;          // one iteration or one selection per launch
constexpr int kPersist = 1;          // several iterations, the table streamed in each
// CSR tables: several iterations over tiles held in registers for the whole
// launch (each wavefront has at most two: no table loads inside the loop).
// (Dense tables have k_resident.)
constexpr int kResident = 2;

template <int R, int LPJ, typename A, int Mode>
__global__ __launch_bounds__(kBlockThreads) void k_dense(KArgs a) {
    constexpr int JPT = kWaveSize / LPJ;       // jobs per tile
    constexpr int RS = Mode == kPersist ? kResidentStep<R> : R;   // lane l accumulates resource l mod RS
    constexpr int Q = kWaveSize / RS;          // accumulating lanes per resource
    __shared__ float s_stage[kBlockWaves][JPT][R];
    __shared__ u128 s_acc[kBlockThreads];
    __shared__ u128 s_wsum[kBlockWaves][R];
    __shared__ u128 s_bsum[R];
    __shared__ double s_lam[R];
    __shared__ double s_newlam[R];
    __shared__ int s_stop;

    const int cl = blockIdx.x / a.nblk;
    const int blk = blockIdx.x - cl * a.nblk;
    const int conv = a.conv_at[cl];            // with the flags: one wait for both
    if (Mode == kOnePass ? skip_cluster<R>(a, cl, blk) : (a.flags && (a.flags[cl] & a.skip_mask))) return;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x == 0) s_stop = 0;

    double lam[R];                             // prices of the current iteration

    const float *col = a.table + cl * a.cluster_stride;
    const bool acc_lane = Mode == kPersist ? lane % RS < R : lane < Q * R;
    const int my_r = acc_lane ? lane % RS : 0;
    const int my_q = lane / RS;
    const int my_shift = a.shift[cl * R + my_r];
    const int gl = lane % LPJ;                 // lane within its job group
    const int jt = lane / LPJ;                 // job within the tile
    A acc = 0;

    const int stride = a.nblk * kBlockWaves;
    const size_t lane_off = static_cast<size_t>(lane) * 4;
    // Tiles are swept front to back, or back to front when `rev` is set; the
    // exact demand sum does not depend on the order.
    const int last = a.tiles - 1;
    const double sw = a.has_pen ? a.switch_cost[cl] : 0.0;
    auto load_tile = [&](int t, int rev, f4 &u, f4 (&d)[R], f4 &pn) {
        const int tl = rev ? last - t : t;
        const float *p = col + static_cast<size_t>(tl) * kTileEntries + lane_off;
        u = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p));
#pragma unroll
        for (int r = 0; r < R; ++r)
            d[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p + (r + 1) * a.col_len));
        if (a.has_pen) pn = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p + (R + 1) * a.col_len));
    };
    // Score, select and stage one tile held in registers.
    auto process = [&](const KArgs &ai, int t, const f4 &u, const f4 (&d)[R], const f4 &pn) {
        const int tl = ai.reverse ? last - t : t;
        double best = 0.0;
        int bi = 0;
        // The lane's best of its 4 entries (lowest index on ties); the
        // penalty test is taken once per tile (a uniform branch), not per entry.
        auto lane_best = [&](auto pen) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                double rent = static_cast<double>(d[0][i]) * lam[0];
#pragma unroll
                for (int r = 1; r < R; ++r) rent = rent + static_cast<double>(d[r][i]) * lam[r];
                double sc = static_cast<double>(u[i]) - rent;
                if constexpr (decltype(pen)::value) sc = penalize(sc, pn[i], sw);
                if (i == 0 || sc > best) { best = sc; bi = i; }
            }
        };
        if (a.has_pen) lane_best(std::true_type{});
        else lane_best(std::false_type{});
        int k = gl * 4 + bi;
        group_argmax<LPJ>(best, k);
        const int j = tl * JPT + jt;
        const bool owner = ((k >> 2) == gl) & (j < ai.N);   // this lane holds the winning entry
        if (ai.choice && owner) ai.choice[static_cast<size_t>(cl) * ai.N + j] = k;
        if (ai.reduce) {
            const int w = k & 3;
            float v[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float lo = (w & 1) ? d[r][1] : d[r][0];
                const float hi = (w & 1) ? d[r][3] : d[r][2];
                v[r] = (w & 2) ? hi : lo;
            }
            if ((j >= ai.N) & (gl == 0)) {
#pragma unroll
                for (int r = 0; r < R; ++r) s_stage[wave][jt][r] = 0.0f;   // jobs past N add nothing
            }
            if (owner) {
#pragma unroll
                for (int r = 0; r < R; ++r) s_stage[wave][jt][r] = v[r];
            }
            wave_sync();
            if (acc_lane) {
#pragma unroll 1
                for (int q = my_q; q < JPT; q += Q) acc += fx_of<A>(s_stage[wave][q][my_r], my_shift);
            }
            wave_sync();
        }
    };
    // Three register buffers, rotated by unrolling: while one tile is scored
    // the loads of the next two are in flight (18 KB per wavefront at R = 8).
    // In a persistent launch the first two loads of the next iteration are
    // issued before its prices are there.
    f4 ua, ub, uc, pa = {}, pb = {}, pc = {};
    f4 da[R], db[R], dc[R];
    const int tile0 = blk * kBlockWaves + wave;
    // Loads of tiles past the end are clamped to the last tile (never
    // processed): no branches, so that the compiler's waits for earlier loads
    // do not wait for these.
    auto prefetch_two = [&](int rev) {
        load_tile(min(tile0, last), rev, ua, da, pa);
        load_tile(min(tile0 + stride, last), rev, ub, db, pb);
    };
    Pending<R, A> pend;
    if constexpr (Mode == kOnePass) pending_loads<R, A>(a, cl, conv, pend);    // issued first: they return first
    prefetch_two(a.reverse);                   // in flight during a pending completion
    const double *etas = nullptr;
    ResidentCtx rctx = {};
    Exchange xch = {};
    if constexpr (Mode == kOnePass) {
        if (!launch_prices<R, A>(a, cl, blk, pend, s_lam, s_newlam, s_acc)) return;
#pragma unroll
        for (int r = 0; r < R; ++r) lam[r] = s_lam[r];
    } else {
        etas = resident_etas(a, cl);
#pragma unroll
        for (int r = 0; r < R; ++r) lam[r] = a.lam_in[cl * R + r];
        rctx = resident_ctx<R>(a, cl, lane, a.lam_in + static_cast<size_t>(cl) * R);
        xch = exchange_of<R>(a, cl, blk, lane);
        __syncthreads();
    }
    for (int it = 0; it < a.n_iters; ++it) {
        const KArgs ai = iteration_args<R>(a, it);
        const int rev = ai.reverse;
        // Loads past the end are clamped to the last tile (never
        // processed): without branches around them the compiler waits
        // for each tile's own loads only.
        for (int tile = tile0; tile < a.tiles; tile += 3 * stride) {
            const int t1 = tile + stride, t2 = tile + 2 * stride;
            load_tile(min(t2, last), rev, uc, dc, pc);
            process(ai, tile, ua, da, pa);
            load_tile(min(t2 + stride, last), rev, ua, da, pa);
            if (t1 < a.tiles) process(ai, t1, ub, db, pb);
            load_tile(min(t2 + 2 * stride, last), rev, ub, db, pb);
            if (t2 < a.tiles) process(ai, t2, uc, dc, pc);
        }
        if (!ai.reduce) return;
        if constexpr (Mode == kPersist) {
            // (the last iteration's loads go unused)
            const bool go = resident_complete<R, kBlockWaves, 0, A>(a, it, cl, blk, wave, lane, acc, etas[it], lam, rctx, xch,
                                                                    [&]() { prefetch_two(rev ^ a.sweep_alt); });
            acc = 0;
            if (go && it + 1 < a.n_iters) continue;
            resident_outputs<R>(a, cl, blk, wave, lane, rctx);
            break;
        }

        // Workgroup sum per resource (integer adds: any order gives the same value).
        s_acc[threadIdx.x] = acc_lane ? static_cast<u128>(acc) : static_cast<u128>(0);
        acc = 0;
        __syncthreads();
        if (threadIdx.x < kBlockWaves * R) {
            const int w = threadIdx.x / R, r = threadIdx.x % R;
            u128 v = 0;
#pragma unroll   // independent LDS loads, all in flight
            for (int q = 0; q < Q; ++q) v += s_acc[w * kWaveSize + q * R + r];
            s_wsum[w][r] = v;
        }
        __syncthreads();
        if (threadIdx.x < R) {
            u128 v = 0;
#pragma unroll
            for (int w = 0; w < kBlockWaves; ++w) v += s_wsum[w][threadIdx.x];
            s_bsum[threadIdx.x] = v;
        }
        __syncthreads();
        if (a.defer) publish_iteration<R>(ai, cl, blk, ai.iter_no, s_bsum);   // the next launch completes it
        else finish_cluster<R, false>(ai, cl, blk, s_bsum, s_lam, s_newlam, &s_stop);
        break;                                 // (one iteration per launch)
    }
}

// ---------------------------------------------------------------------------
// Dense families, resident: several iterations over tiles kept on chip
// ---------------------------------------------------------------------------

// A wavefront keeps its first two tiles in registers and the others (a.lds_tiles
// at most, none in ESP_MODE_RESIDENT) in LDS, loaded once per launch: at R = 8
// a workgroup holds 32 tiles, 256 of them 75 MB.  Iterations follow each other
// with no table loads, so their cost is the latency of scoring the wavefronts'
// tiles (two wavefronts per SIMD overlap), the workgroup's sums and, with
// several workgroups, one exchange through memory (resident_complete).
// Streaming the same table costs a pass at memory bandwidth and a barrier of
// the grid per iteration.  Measured per iteration, 64 configurations x 8
// resources, against the streaming persistent driver: 9,000 jobs (20.7 MB)
// 8.5 -> 3.6 us, 12,000 (27.6 MB) 9.9 -> 3.6, 24,000 (55 MB) 13.1 -> 5.5;
// against four wavefronts per workgroup with every workgroup reading every
// other's sums: 4,096 jobs x 32 x 4 4.1 -> 2.4, 64 x 8 x 4 1.25 -> 0.85.
// A kernel of its own: the registers and branches of the streaming loops cost
// every iteration here.  A = double when the whole sum fits 53 bits (a.sum_f64):
// every partial sum is exact in binary64, so the conversions to and from fixed
// point leave the chain (64 jobs x 8 x 4 1.04 -> 0.95 us an iteration, 4,096 x 32 x
// 4 2.76 -> 2.55, 700 x 4 x 8 2.06 -> 1.76).
template <int R, int LPJ, typename A>
__global__ __launch_bounds__(kResidentThreads) void k_resident(KArgs a) {
    constexpr int JPT = kWaveSize / LPJ;       // jobs per tile
    constexpr int RS = kResidentStep<R>;       // lane l accumulates resource l mod RS
    constexpr int Q = kWaveSize / RS;          // accumulating lanes per resource
    constexpr int kPer = (JPT + Q - 1) / Q;    // jobs of a tile per accumulating lane
    extern __shared__ f4 s_tiles[];            // [kResidentWaves][a.lds_tiles][columns][64 lanes]
    __shared__ float s_stage[kResidentWaves][JPT][R];
    const int cl = blockIdx.x / a.nblk;
    const int blk = blockIdx.x - cl * a.nblk;
    if (a.flags[cl] & a.skip_mask) return;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float *col = a.table + cl * a.cluster_stride;
    const bool acc_lane = lane % RS < R;
    const int my_r = acc_lane ? lane % RS : 0;
    const int my_q = lane / RS;
    const int my_shift = a.shift[cl * R + my_r];
    const int gl = lane % LPJ;                 // lane within its job group
    const int jt = lane / LPJ;                 // job within the tile
    // tile s of wavefront w: every workgroup's wavefront w before any's w + 1, so that the wavefronts
    // that share a SIMD (w and w + 4) both have tiles only when there are more than 4 per workgroup
    const int stride = a.nblk * a.res_waves;
    const int tile0 = wave * a.nblk + blk;
    const int last = a.tiles - 1;
    const double sw = a.has_pen ? a.switch_cost[cl] : 0.0;
    auto load_tile = [&](int t, f4 &u, f4 (&d)[R], f4 &pn) {
        const float *p = col + static_cast<size_t>(t) * kTileEntries + static_cast<size_t>(lane) * 4;
        u = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p));
#pragma unroll
        for (int r = 0; r < R; ++r)
            d[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p + (r + 1) * a.col_len));
        if (a.has_pen) pn = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p + (R + 1) * a.col_len));
    };
    // tile s of this wavefront's LDS tiles (its tile tile0 + (2 + s) stride)
    const int cols = R + 1 + (a.has_pen ? 1 : 0);
    f4 *const mine = s_tiles + static_cast<size_t>(wave) * a.lds_tiles * cols * kWaveSize + lane;
    auto lds_tile = [&](int s, f4 &u, f4 (&d)[R], f4 &pn) {
        const f4 *p = mine + static_cast<size_t>(s) * cols * kWaveSize;
        u = p[0];
#pragma unroll
        for (int r = 0; r < R; ++r) d[r] = p[(r + 1) * kWaveSize];
        if (a.has_pen) pn = p[(R + 1) * kWaveSize];
    };
    double lam[R];                             // prices of the current iteration
    A acc = 0;
    int32_t *choice = nullptr;                 // the iteration's trace of choices
    auto process = [&](int tl, const f4 &u, const f4 (&d)[R], const f4 &pn) {
        double best = 0.0;
        int bi = 0;
        auto lane_best = [&](auto pen) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                double rent = static_cast<double>(d[0][i]) * lam[0];
#pragma unroll
                for (int r = 1; r < R; ++r) rent = rent + static_cast<double>(d[r][i]) * lam[r];
                double sc = static_cast<double>(u[i]) - rent;
                if constexpr (decltype(pen)::value) sc = penalize(sc, pn[i], sw);
                if (i == 0 || sc > best) { best = sc; bi = i; }
            }
        };
        if (a.has_pen) lane_best(std::true_type{});
        else lane_best(std::false_type{});
        int k = gl * 4 + bi;
        group_argmax<LPJ>(best, k);
        const int j = tl * JPT + jt;
        const bool owner = ((k >> 2) == gl) & (j < a.N);   // this lane holds the winning entry
        if (choice && owner) choice[static_cast<size_t>(cl) * a.N + j] = k;
        const int w = k & 3;
        float v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float lo = (w & 1) ? d[r][1] : d[r][0];
            const float hi = (w & 1) ? d[r][3] : d[r][2];
            v[r] = (w & 2) ? hi : lo;
            v[r] = j < a.N ? v[r] : 0.0f;                  // jobs past N add nothing
        }
        if ((k >> 2) == gl) {
#pragma unroll
            for (int r = 0; r < R; ++r) s_stage[wave][jt][r] = v[r];
        }
        wave_sync();
        float x[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int q = my_q + i * Q;
            x[i] = s_stage[wave][q < JPT ? q : JPT - 1][my_r];
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            acc += fx_of<A>((acc_lane & (my_q + i * Q < JPT)) ? x[i] : 0.0f, my_shift);
        wave_sync();
    };
    f4 ua, ub, up, pa = {}, pb = {}, pp = {};
    f4 da[R], db[R], dp[R];
    load_tile(min(tile0, last), ua, da, pa);               // clamped: no branch
    load_tile(min(tile0 + stride, last), ub, db, pb);
    const int n_lds = max(0, min(a.lds_tiles, (a.tiles - tile0 - 2 * stride + stride - 1) / stride));
#pragma unroll 1
    for (int s = 0; s < n_lds; ++s) {
        load_tile(tile0 + (2 + s) * stride, up, dp, pp);
        f4 *p = mine + static_cast<size_t>(s) * cols * kWaveSize;
        p[0] = up;
#pragma unroll
        for (int r = 0; r < R; ++r) p[(r + 1) * kWaveSize] = dp[r];
        if (a.has_pen) p[(R + 1) * kWaveSize] = pp;
    }
    wave_sync();
    if (threadIdx.x < kResidentWaves * R) wave_sums<R, kResidentWaves, A>()[threadIdx.x / R][threadIdx.x % R] = 0;
    const double *etas = resident_etas(a, cl);
#pragma unroll
    for (int r = 0; r < R; ++r) lam[r] = a.lam_in[cl * R + r];
    const Exchange xch = exchange_of<R>(a, cl, blk, lane);
    ResidentCtx ctx = resident_ctx<R>(a, cl, lane, a.lam_in + static_cast<size_t>(cl) * R);
    __syncthreads();
    for (int it = 0; it < a.n_iters; ++it) {
        if (a.choice) choice = a.choice + static_cast<size_t>(it) * a.B * a.N;
        acc = 0;
        if (tile0 < a.tiles) process(tile0, ua, da, pa);
        if (tile0 + stride < a.tiles) process(tile0 + stride, ub, db, pb);
#pragma unroll 1   // (the SIMD's other wavefront fills the wait for LDS)
        for (int s = 0; s < n_lds; ++s) {
            lds_tile(s, up, dp, pp);
            process(tile0 + (2 + s) * stride, up, dp, pp);
        }
        if (!resident_complete<R, kResidentWaves, 0, A>(a, it, cl, blk, wave, lane, acc, etas[it], lam, ctx, xch)) break;
    }
    resident_outputs<R>(a, cl, blk, wave, lane, ctx);
}

// ---------------------------------------------------------------------------
// CSR families (ragged sizes 1..256): whole families packed into tiles
// ---------------------------------------------------------------------------

// s = max(s, o) in the lanes of m (no NaN among the scores): one instruction
// under EXEC, which is saved and restored.  The last two instructions are the
// wait states a DPP read of s needs (not seen by the compiler behind assembly).
__device__ __forceinline__ void max_in_lanes(double &s, double o, uint64_t m) {
    uint64_t ex;
    asm volatile("s_mov_b64 %[ex], exec\n\t"
                 "s_mov_b64 exec, %[m]\n\t"
                 "v_max_f64 %[s], %[s], %[o]\n\t"
                 "s_mov_b64 exec, %[ex]\n\t"
                 "s_nop 1"
                 : [s] "+v"(s), [ex] "=&s"(ex)
                 : [o] "v"(o), [m] "s"(m));
}

// One step of an inclusive segmented max-scan over lanes: the lanes of m have
// no segment start between the lane the value comes from (exclusive) and
// themselves.
template <int CTRL>
__device__ __forceinline__ void seg_scan_step(double &s, uint64_t m) {
    max_in_lanes(s, dpp_any_d<CTRL>(s), m);
}

// Segmented inclusive max-scan of s over the lanes.
__device__ __forceinline__ void seg_scan(double &s, const ScanLanes &l) {
    seg_scan_step<kDppRowShr1>(s, l.row1);
    seg_scan_step<kDppRowShr2>(s, l.row2);
    seg_scan_step<kDppRowShr4>(s, l.row4);
    seg_scan_step<kDppRowShr8>(s, l.row8);
    seg_scan_step<kDppRowBcast15>(s, l.rows);
    seg_scan_step<kDppRowBcast31>(s, l.halves);
}

// The lanes of m whose next higher lane of m is in `next` (a subset of m).
// Mirrored, the next lane of m above each lane of `next`: a bit added just
// above it carries through the zeros of m.
__device__ __forceinline__ uint64_t lanes_before(uint64_t m, uint64_t next) {
    const uint64_t rm = __builtin_bitreverse64(m), rn = __builtin_bitreverse64(next);
    return __builtin_bitreverse64((~rm + (rn << 1)) & rm);
}

// Two wavefronts per SIMD (at most 256 registers): two workgroups of 4 wavefronts
// per CU, all of them resident in a cooperative launch, or one of 8 where the
// tiles stay in registers (an iteration there costs an exchange, cheaper among
// half as many workgroups, and the latency of a wavefront's one or two tiles:
// 100 ragged jobs x 8 3.3 -> 2.1 us, 60,000 x 4 4.1 -> 3.9, 200,000 x 5 x 3 4.6 -> 4.2).
constexpr int csr_waves(int mode) { return mode == kResident ? kResidentWaves : kBlockWaves; }

// The scoring is 76 of a tile's VALU instructions (R = 6); who wins is worked
// out on lane masks in scalar registers, which leaves about 190 of the 351 that
// per-lane flags, indices and staged winners took.  A pass over a small table
// is bound by its tiles' latency, over a large one by memory.
//
// Direct: each lane adds the demands of its own winners in binary64, exactly:
// the packer takes this form when a lane's sum of a pass fits 53 bits of the
// column's fixed-point window (a.lane_f64).  Otherwise the winners' demands are
// staged in LDS and added as fixed-point integers, resource by lane (more
// instructions, and the LDS round trips of a tile's winners on its chain).
// Measured with one launch per pass, 6 resources: 1,048,576 jobs (388 MB) 64.7 ->
// 63.0 us, three register sets instead of two 62.6 but 24.1 against 23.0 on
// 262,144 jobs x 12 x 8.
template <int R, typename A, int Mode, bool Direct>
__global__ __launch_bounds__(csr_waves(Mode) * kWaveSize, 2) void k_csr(KArgs a) {
    constexpr int Waves = csr_waves(Mode);
    constexpr int RS = Mode != kOnePass ? kResidentStep<R> : R;   // lane l accumulates resource l mod RS
    constexpr int Q = kWaveSize / RS;          // accumulating lanes per resource
    __shared__ float s_stage[Direct ? 1 : Waves][Direct ? 1 : kTileEntries][R];
    __shared__ u128 s_acc[Mode == kOnePass ? kBlockThreads : 1];
    __shared__ u128 s_wsum[Waves][R];
    __shared__ u128 s_bsum[R];
    __shared__ double s_lam[R];
    __shared__ double s_newlam[R];
    __shared__ int s_stop;

    const int cl = blockIdx.x / a.nblk;
    const int blk = blockIdx.x - cl * a.nblk;
    const int conv = a.conv_at[cl];            // with the flags: one wait for both
    if (Mode == kOnePass ? skip_cluster<R>(a, cl, blk) : (a.flags && (a.flags[cl] & a.skip_mask))) return;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x == 0) s_stop = 0;

    double lam[R];                             // prices of the current iteration
    const bool acc_lane = Mode != kOnePass ? lane % RS < R : lane < Q * R;
    const int my_r = acc_lane ? lane % RS : 0;
    const int my_q = lane / RS;
    const int my_shift = a.shift[cl * R + my_r];
    A acc = 0;
    double sum[R];                             // this lane's demand sums of the pass (Direct)
#pragma unroll
    for (int r = 0; r < R; ++r) sum[r] = 0.0;

    const float *col = a.table + cl * a.cluster_stride;
    const size_t lane_off = static_cast<size_t>(lane) * 4;
    struct Heads { uint64_t m[4]; };           // m[i]: the lanes whose entry i starts a job
    // Direct: the wavefront's totals, of resource l / 8 in lane l; the lanes' sums start again
    auto take_totals = [&]() {
        uint64_t x[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            x[r] = static_cast<uint64_t>(ldexp(sum[r], -a.shift[cl * R + r]));
            sum[r] = 0.0;
        }
        return wave_totals<R>(x);
    };
    const double sw = a.has_pen ? a.switch_cost[cl] : 0.0;
    const int stride = a.nblk * (Mode == kResident ? a.res_waves : Waves);
    const int last = a.tiles - 1;
    auto load_tile = [&](int t, int rev, f4 &u, f4 (&d)[R], f4 &pn, Heads &h) {
        const int tl = rev ? last - t : t;
        const float *p = col + static_cast<size_t>(tl) * kTileEntries + lane_off;
        u = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p));
#pragma unroll
        for (int r = 0; r < R; ++r)
            d[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p + (r + 1) * a.col_len));
        if (a.has_pen) pn = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p + (R + 1) * a.col_len));
#pragma unroll
        for (int i = 0; i < 4; ++i) h.m[i] = scalar_word(a.meta + tl, i);
    };
    // Score one tile, find every family's winner and add up (or stage) the
    // winners' demands, or write the choices.  Everything about where families
    // start and who wins is a mask over the lanes in scalar registers.
    auto process = [&](const KArgs &ai, int t, const f4 &u, const f4 (&d)[R], const f4 &pn, const Heads &h) {
        const int tl = ai.reverse ? last - t : t;
        double sc[4];
        // the penalty test is taken once per tile (a uniform branch)
        auto scores = [&](auto pen) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                double rent = static_cast<double>(d[0][i]) * lam[0];
#pragma unroll
                for (int r = 1; r < R; ++r) rent = rent + static_cast<double>(d[r][i]) * lam[r];
                sc[i] = static_cast<double>(u[i]) - rent;
                if constexpr (decltype(pen)::value) sc[i] = penalize(sc[i], pn[i], sw);
            }
        };
        if (a.has_pen) scores(std::true_type{});
        else scores(std::false_type{});
        // Lane-local pass: one running best (lowest entry on ties, at[q]: the
        // lanes where it is entry q) that restarts at every head.  At a head
        // the run so far is either a segment that began at an earlier head of
        // this lane (complete: its winner is marked, win[q]) or, before the
        // lane's first head, this lane's part of a segment from lower lanes
        // (pre, entry q in the lanes pre_at[q]).  At the end the run is the
        // segment left open at the lane's end.
        double run = sc[0], pre = sc[0];
        uint64_t at[4] = {~0ull, 0, 0, 0}, win[4] = {0, 0, 0, 0}, pre_at[3] = {0, 0, 0};
        uint64_t open = h.m[0];
#pragma unroll
        for (int i = 1; i < 4; ++i) {
            const uint64_t done = h.m[i] & open, first = h.m[i] & ~open;
            const uint64_t take = h.m[i] | mask_of(sc[i] > run);
            pre = in_mask(first) ? run : pre;
            run = in_mask(take) ? sc[i] : run;
#pragma unroll
            for (int q = 0; q < i; ++q) {
                win[q] |= done & at[q];
                pre_at[q] |= first & at[q];
                at[q] &= ~take;
            }
            at[i] = take;
            open |= h.m[i];
        }
        const uint64_t heads = open;           // lanes with a head
        // Segment maxima across lanes: after the scan, top is the largest score
        // of the segment open at this lane's end, over its slots up to here.
        double top = run;
        seg_scan(top, scan_lanes(heads));
        const double prev = dpp_any_d<kDppWaveShr1>(top);    // at the previous lane (a tile starts with a head)
        // The winner of a segment is its first slot with the segment's largest
        // score: in the lane where the running maximum last rose (a head, or a
        // run strictly above everything before it), its run's best, unless the
        // part of the next head lane before its first head (slots above all of
        // the segment's others) beats it strictly (pre_wins there).
        const uint64_t rise = heads | mask_of(top > prev);
        const uint64_t pre_wins = heads & ~h.m[0] & mask_of(pre > prev);
        const uint64_t run_wins = rise & ~lanes_before(rise, rise & ~(heads & ~pre_wins));
#pragma unroll
        for (int q = 0; q < 4; ++q) win[q] |= (run_wins & at[q]) | (q < 3 ? pre_wins & pre_at[q < 3 ? q : 0] : 0ull);
        if (ai.choice) {
            // job = first_job + (heads at or before the slot) - 1;
            // config = slot - (the last head at or before it)
            int j = static_cast<int>(static_cast<uint32_t>(scalar_word(a.meta + tl, 4))) - 1 +
                    static_cast<int>(below_lane(h.m[3], below_lane(h.m[2], below_lane(h.m[1], below_lane(h.m[0], 0u)))));
            const int mine = lane * 4 + (in_mask(h.m[3]) ? 3 : in_mask(h.m[2]) ? 2 : in_mask(h.m[1]) ? 1 : 0);
            const uint64_t lower = heads & ((1ull << lane) - 1ull);
            int start = __shfl(mine, lower ? 63 - __clzll(lower) : 0);
            int32_t *const out = ai.choice + static_cast<size_t>(cl) * a.N;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool head = in_mask(h.m[i]);
                start = head ? lane * 4 + i : start;
                j += head ? 1 : 0;
                if (in_mask(win[i])) out[j] = lane * 4 + i - start;
            }
        }
        if (!ai.reduce) return;
        if constexpr (Direct) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (!in_mask(win[i])) continue;
#pragma unroll
                for (int r = 0; r < R; ++r) sum[r] += static_cast<double>(d[r][i]);
            }
        } else {
            // Rank of this lane's first winner among the tile's winners (slot
            // order: lane, then entry); n_win is the same for every lane.
            int rank = static_cast<int>(below_lane(win[3], below_lane(win[2], below_lane(win[1], below_lane(win[0], 0u)))));
            const int n_win = __popcll(win[0]) + __popcll(win[1]) + __popcll(win[2]) + __popcll(win[3]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (!in_mask(win[i])) continue;
#pragma unroll
                for (int r = 0; r < R; ++r) s_stage[wave][rank][r] = d[r][i];
                ++rank;
            }
            wave_sync();
            if (acc_lane) {
#pragma unroll 1
                for (int q = my_q; q < n_win; q += Q) acc += fx_of<A>(s_stage[wave][q][my_r], my_shift);
            }
            wave_sync();
        }
    };
    // One tile of prefetch: the next tile's loads are in flight while the
    // current one is scored (a deeper prefetch measured no faster).  Two
    // register sets take turns (the loop body appears twice), so the
    // prefetched tile is scored where it landed, without copies.
    f4 nu, npn = {}, bu, bpn = {};
    f4 nd[R], bd[R];
    Heads nhw = {}, bhw = {};
    // (resident: the wavefronts that share a SIMD both have a tile only with more than 4 per workgroup)
    const int tile0 = Mode == kResident ? wave * a.nblk + blk : blk * Waves + wave;
    Pending<R, A> pend;
    if constexpr (Mode == kOnePass) pending_loads<R, A>(a, cl, conv, pend);   // issued first: they return first
    load_tile(min(tile0, last), a.reverse, nu, nd, npn, nhw);   // in flight during a pending completion (clamped: no branch)
    if constexpr (Mode == kResident)
        load_tile(min(tile0 + stride, last), a.reverse, bu, bd, bpn, bhw);   // the launch's second tile
    const double *etas = nullptr;
    ResidentCtx rctx = {};
    Exchange xch = {};
    if constexpr (Mode == kOnePass) {
        if (!launch_prices<R, A>(a, cl, blk, pend, s_lam, s_newlam, s_acc)) return;
#pragma unroll
        for (int r = 0; r < R; ++r) lam[r] = s_lam[r];
    } else {
        if (Mode == kResident && threadIdx.x < Waves * R) wave_sums<R, Waves, A>()[threadIdx.x / R][threadIdx.x % R] = 0;
        etas = resident_etas(a, cl);
#pragma unroll
        for (int r = 0; r < R; ++r) lam[r] = a.lam_in[cl * R + r];
        rctx = resident_ctx<R>(a, cl, lane, a.lam_in + static_cast<size_t>(cl) * R);
        xch = exchange_of<R>(a, cl, blk, lane);
        __syncthreads();
    }
    for (int it = 0; it < a.n_iters; ++it) {
        const KArgs ai = iteration_args<R>(a, it);
        const int rev = ai.reverse;
        if constexpr (Mode == kResident) {
            // the wavefront's tiles stay in the two register sets (loaded front to back)
            if (tile0 < a.tiles) process(ai, tile0, nu, nd, npn, nhw);
            if (tile0 + stride < a.tiles) process(ai, tile0 + stride, bu, bd, bpn, bhw);
        } else {
            for (int tile = tile0; tile < a.tiles; tile += 2 * stride) {
                load_tile(min(tile + stride, last), rev, bu, bd, bpn, bhw);   // clamped: no branch
                process(ai, tile, nu, nd, npn, nhw);
                if (tile + stride >= a.tiles) break;
                load_tile(min(tile + 2 * stride, last), rev, nu, nd, npn, nhw);
                process(ai, tile + stride, bu, bd, bpn, bhw);
            }
        }
        if (!ai.reduce) return;
        if constexpr (Mode != kOnePass) {
            if constexpr (Direct) acc = take_totals();
            const bool go = resident_complete<R, Waves, Direct ? 8 : 0, A>(
                a, it, cl, blk, wave, lane, acc, etas[it], lam, rctx, xch, [&]() {
                    // (the last iteration's loads go unused)
                    if constexpr (Mode == kPersist) load_tile(min(tile0, last), rev ^ a.sweep_alt, nu, nd, npn, nhw);
                });
            acc = 0;
            if (go && it + 1 < a.n_iters) continue;
            resident_outputs<R>(a, cl, blk, wave, lane, rctx);
            break;
        }

        if constexpr (Direct) {
            const uint64_t tot = take_totals();
            if ((lane & 7) == 0 && lane / 8 < R) s_wsum[wave][lane / 8] = tot;
        } else {
            s_acc[threadIdx.x] = acc_lane ? static_cast<u128>(acc) : static_cast<u128>(0);
            acc = 0;
            __syncthreads();
        }
        if (!Direct && threadIdx.x < kBlockWaves * R) {
            const int w = threadIdx.x / R, r = threadIdx.x % R;
            u128 v = 0;
#pragma unroll   // independent LDS loads, all in flight
            for (int q = 0; q < Q; ++q) v += s_acc[w * kWaveSize + q * R + r];
            s_wsum[w][r] = v;
        }
        __syncthreads();
        if (threadIdx.x < R) {
            u128 v = 0;
#pragma unroll
            for (int w = 0; w < kBlockWaves; ++w) v += s_wsum[w][threadIdx.x];
            s_bsum[threadIdx.x] = v;
        }
        __syncthreads();
        if (a.defer) publish_iteration<R>(ai, cl, blk, ai.iter_no, s_bsum);   // the next launch completes it
        else finish_cluster<R, false>(ai, cl, blk, s_bsum, s_lam, s_newlam, &s_stop);
        break;                                 // (one iteration per launch)
    }
}

// ---------------------------------------------------------------------------
// Gather: U from caller-supplied choices (granular esp_reduce_demand)
// ---------------------------------------------------------------------------

// Each job's R demands lie in R columns at an arbitrary slot: a chain of two
// (CSR: three) dependent loads per job, bound by their latency, so the kernel
// keeps up to kGatherJobs jobs per thread in flight.  Totals over a wavefront's
// lanes stay in registers.  Workgroups are small (4 wavefronts), so that many
// clusters' workgroups, or a plan's 512, are on the device at once; 16
// wavefronts pay only where a workgroup of the plan has thousands of jobs with
// few loads each (gather_wide).  us a call, one job at a time in 4 wavefronts ->
// 16 wavefronts -> 4: 16 clusters of 8,192 jobs x 32 x 6 24.9 -> 21.3 -> 20.2 (near the
// 100 MB of lines that it touches), 262,144 x 16 x 8 31.4 -> 26.5 -> 24.9, 64 of 2,000 x
// 12 x 6 15.6 -> 28.5 -> 10.8, 600 of 200 x 12 x 8 18.5 -> 30.2 -> 13.7; 1,000,000 x 4 x 3
// 24.6 -> 16.8 -> 19.2.
constexpr int kGatherJobs = 4;
// 16 wavefronts -> 4, jobs per workgroup, us: 3 resources 2,083 11.3 -> 10.4, 3,125 12.3 -> 12.5,
// 10,400 24.0 -> 31.2; 4 resources 2,500 10.3 -> 10.7, 8,000 23.6 -> 25.6; 6 resources 5,208 24.0 ->
// 23.2; 8 resources 3,906 26.8 -> 27.0.
inline bool gather_wide(int R, int N, int nblk) { return R <= 4 && N / nblk >= 2500; }

template <int R, typename A, int Threads>
__global__ __launch_bounds__(Threads) void k_gather(KArgs a) {
    constexpr int Waves = Threads / kWaveSize;
    __shared__ A s_wave[Waves][R];
    __shared__ u128 s_bsum[R];
    __shared__ int s_bad;
    const int cl = blockIdx.x / a.nblk;
    const int blk = blockIdx.x - cl * a.nblk;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x / kWaveSize;
    const float *col = a.table + cl * a.cluster_stride;
    const int32_t *choice = a.choice_in + static_cast<size_t>(cl) * a.N;
    A acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0;
    int sh[R];
#pragma unroll
    for (int r = 0; r < R; ++r) sh[r] = a.shift[cl * R + r];
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    bool bad = false;
    const int64_t step = static_cast<int64_t>(a.nblk) * Threads;
    const int64_t first = static_cast<int64_t>(blk) * Threads;      // the workgroup's first job of a step
    for (int64_t w0 = first; w0 < a.N; w0 += kGatherJobs * step) {
        // The loads of up to kGatherJobs steps in flight together; a step past the end is
        // skipped by the whole workgroup, jobs past the end in the last step are clamped
        // (loaded, not added).
        int c[kGatherJobs] = {};
        uint32_t slot[kGatherJobs] = {}, size[kGatherJobs] = {};
#pragma unroll
        for (int u = 0; u < kGatherJobs; ++u) {
            if (w0 + u * step >= a.N) continue;
            const int64_t j = w0 + u * step + threadIdx.x;
            const int jc = static_cast<int>(j < a.N ? j : a.N - 1);
            c[u] = choice[jc];
            if (a.K > 0) {
                slot[u] = static_cast<uint32_t>(jc) * static_cast<uint32_t>(a.K);
                size[u] = static_cast<uint32_t>(a.K);
            } else {
                const JobSlot js = a.jobs[jc];
                slot[u] = js.slot;
                size[u] = js.size;
            }
        }
        float v[kGatherJobs][R] = {};
#pragma unroll
        for (int u = 0; u < kGatherJobs; ++u) {
            if (w0 + u * step >= a.N) continue;
            const bool in = (c[u] >= 0) & (static_cast<uint32_t>(c[u]) < size[u]);
            bad |= !in;
            if (in & (w0 + u * step + threadIdx.x < a.N)) {
                const size_t e = static_cast<size_t>(slot[u]) + static_cast<uint32_t>(c[u]);
#pragma unroll
                for (int r = 0; r < R; ++r) v[u][r] = col[(r + 1) * a.col_len + e];
            }
        }
#pragma unroll
        for (int u = 0; u < kGatherJobs; ++u) {
            if (w0 + u * step >= a.N) continue;
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] += fx_of<A>(v[u][r], sh[r]);
        }
    }
    if (bad) s_bad = 1;
    // lane r of each wavefront: its total for resource r
    A mine = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const A t = lane_sum<1>(acc[r]);
        mine = lane == r ? t : mine;
    }
    if (lane < R) s_wave[wave][lane] = mine;
    __syncthreads();
    if (threadIdx.x < R) {
        u128 v = 0;
#pragma unroll
        for (int w = 0; w < Waves; ++w) v += static_cast<u128>(s_wave[w][threadIdx.x]);
        s_bsum[threadIdx.x] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_bad) {
        atomicOr(&a.flags[cl], 4);
        atomicCAS(a.status, 0, kStatusInvalid);
    }
    __shared__ double s_newlam[R];
    __shared__ int s_stop;
    finish_cluster<R, true>(a, cl, blk, s_bsum, nullptr, s_newlam, &s_stop);
}

// ---------------------------------------------------------------------------
// Granular price update (esp_update_prices) and price validation
// ---------------------------------------------------------------------------

template <int R>
__global__ void k_update(KArgs a, const double *demand_in, int B) {
    const int cl = blockIdx.x * blockDim.x + threadIdx.x;
    if (cl >= B) return;
    bool ok = true;
    for (int r = 0; r < R; ++r) {
        const double U = demand_in[cl * R + r];
        ok = ok && price_ok(a.lam_in[cl * R + r]) && (U >= -0x1p200 && U <= 0x1p200);
    }
    if (!ok) {
        atomicCAS(a.status, 0, kStatusNonfinite);
        return;
    }
    for (int r = 0; r < R; ++r) {
        const double lo = a.lam_in[cl * R + r];
        const double g = demand_in[cl * R + r] - a.cap[cl * R + r];
        const double x = lo + step_size(a, cl, a.t) * g;
        a.lam_out[cl * R + r] = (x > 0.0) ? x : 0.0;
    }
}

// Validate prices before a solve or a selection; mark bad clusters.  A valid
// price -0.0 is stored back as +0.0 when `canon` is set (the solve's in/out
// prices; never -0.0 afterwards, as after the projection of Eq. 8).  For a
// solve (iters_done set) also reset the per-solve counters and store the
// starting prices as lambda_1 (lam_ws[1]) for the first deferred completion.
template <int R>
__global__ void k_prepare(KArgs a, const double *lam, double *canon, int B) {
    const int cl = blockIdx.x * blockDim.x + threadIdx.x;
    // the resident exchange words start at 0 (a.xch_clear words, or none)
    for (size_t i = cl; i < a.xch_clear; i += static_cast<size_t>(gridDim.x) * blockDim.x)
        reinterpret_cast<uint64_t *>(a.sync)[i] = 0ull;
    if (cl >= B) return;
    bool ok = true;
    for (int r = 0; r < R; ++r) ok = ok && price_ok(lam[cl * R + r]);
    a.flags[cl] = (a.flags[cl] & kFlagFrozen) | (ok ? 0 : kFlagError);
    if (ok && canon) {
        for (int r = 0; r < R; ++r)
            if (__double_as_longlong(lam[cl * R + r]) == static_cast<long long>(0x8000000000000000ull))
                canon[cl * R + r] = 0.0;
    }
    if (a.iters_done) {
        a.iters_done[cl] = 0;
        a.tickets[cl] = 0u;          // 0 between launches; cleared for scratch shared between solves
        a.conv_at[cl] = 0;
        for (int r = 0; r < R; ++r) {
            const double v = lam[cl * R + r];
            a.lam_ws[static_cast<size_t>(B) * R + static_cast<size_t>(cl) * R + r] = (v == 0.0) ? 0.0 : v;
        }
    }
    if (!ok) atomicCAS(a.status, 0, kStatusNonfinite);
}

// Closing launch of a deferred solve without a final selection: one
// workgroup per cluster completes the solve's last iteration (pend_m).
template <int R>
__global__ __launch_bounds__(kBlockThreads) void k_finish(KArgs a) {
    __shared__ u128 s_red[kBlockThreads];
    __shared__ double s_tmp[R];
    __shared__ double s_lam[R];
    const int cl = blockIdx.x;
    if (a.flags && (a.flags[cl] & a.skip_mask)) return;
    Pending<R, u128> pend;
    pending_loads<R, u128>(a, cl, a.conv_at[cl], pend);
    (void)launch_prices<R, u128>(a, cl, 0, pend, s_lam, s_tmp, s_red);
}

// ---------------------------------------------------------------------------
// Launchers (runtime R / LPJ -> template instance)
// ---------------------------------------------------------------------------

template <int R, typename A>
hipError_t launch_dense_ra(int lpj, const KArgs &a, int B, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>(B) * a.nblk), block(kBlockThreads);
    switch (lpj) {
        case 1: hipLaunchKernelGGL((k_dense<R, 1, A, kOnePass>), grid, block, 0, s, a); break;
        case 2: hipLaunchKernelGGL((k_dense<R, 2, A, kOnePass>), grid, block, 0, s, a); break;
        case 4: hipLaunchKernelGGL((k_dense<R, 4, A, kOnePass>), grid, block, 0, s, a); break;
        case 8: hipLaunchKernelGGL((k_dense<R, 8, A, kOnePass>), grid, block, 0, s, a); break;
        case 16: hipLaunchKernelGGL((k_dense<R, 16, A, kOnePass>), grid, block, 0, s, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int R>
hipError_t launch_dense_r(int lpj, const KArgs &a, int B, hipStream_t s) {
    return a.acc128 ? launch_dense_ra<R, u128>(lpj, a, B, s) : launch_dense_ra<R, uint64_t>(lpj, a, B, s);
}

// A cooperative launch of `blocks` workgroups of kernel f: refused on the host
// when the device cannot hold them all at once (nothing is enqueued then).
inline hipError_t launch_cooperative(const void *f, unsigned blocks, const KArgs &a, int threads, size_t lds,
                                     hipStream_t s) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, threads, lds) != hipSuccess)
        return hipErrorInvalidValue;
    if (static_cast<int64_t>(blocks) > static_cast<int64_t>(per_cu) * cus) return hipErrorCooperativeLaunchTooLarge;
    KArgs copy = a;
    void *args[] = {&copy};
    return hipLaunchCooperativeKernel(f, dim3(blocks), dim3(threads), args, static_cast<unsigned>(lds), s);
}

// A multi-iteration launch of kernel f with `lds` bytes of dynamic LDS, at most
// lds_max.  With one workgroup per cluster no workgroup waits for another: an
// ordinary launch.  Otherwise a cooperative one, so that the workgroups of a
// cluster are co-resident.  The kernel's limit of dynamic LDS belongs to the
// process: every launch sets the same value, so that another thread's launch of
// the kernel, with fewer tiles, cannot lower it in between.
inline hipError_t launch_multi(const void *f, unsigned blocks, const KArgs &a, int words, hipStream_t s,
                               int threads = kBlockThreads, size_t lds = 0, size_t lds_max = 0) {
    // a copy's count field (the registers let no more workgroups be co-resident anyway)
    if (a.nblk > 255 * exchange_copies(words)) return hipErrorCooperativeLaunchTooLarge;
    if (lds > 0) {
        const hipError_t e =
            hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_max));
        if (e != hipSuccess) return e;
    }
    if (a.nblk == 1) {
        KArgs copy = a;
        void *args[] = {&copy};
        return hipLaunchKernel(f, dim3(blocks), dim3(threads), args, lds, s);
    }
    return launch_cooperative(f, blocks, a, threads, lds, s);
}

template <int R, int LPJ, typename A>
const void *dense_multi_kernel(const KArgs &a, bool resident) {
    if constexpr (sizeof(A) == 8)
        if (resident && a.sum_f64) return reinterpret_cast<const void *>(&k_resident<R, LPJ, double>);
    if (resident) return reinterpret_cast<const void *>(&k_resident<R, LPJ, A>);
    return reinterpret_cast<const void *>(&k_dense<R, LPJ, A, kPersist>);
}

template <int R, typename A>
hipError_t launch_dense_coop_ra(int lpj, const KArgs &a, int B, bool resident, hipStream_t s) {
    const void *f = nullptr;
    switch (lpj) {
        case 1: f = dense_multi_kernel<R, 1, A>(a, resident); break;
        case 2: f = dense_multi_kernel<R, 2, A>(a, resident); break;
        case 4: f = dense_multi_kernel<R, 4, A>(a, resident); break;
        case 8: f = dense_multi_kernel<R, 8, A>(a, resident); break;
        case 16: f = dense_multi_kernel<R, 16, A>(a, resident); break;
        default: return hipErrorInvalidValue;
    }
    const size_t lds = resident ? resident_lds(R + 1 + (a.has_pen ? 1 : 0), a.lds_tiles) : 0;
    return launch_multi(f, static_cast<unsigned>(B) * a.nblk, a, R * a.limbs, s,
                        resident ? a.res_waves * kWaveSize : kBlockThreads, lds,
                        resident_lds_limit(R, lpj));
}

template <int R>
hipError_t launch_dense_coop_r(int lpj, const KArgs &a, int B, bool resident, hipStream_t s) {
    if (a.defer) return hipErrorInvalidValue;              // these launches complete their iterations
    return a.acc128 ? launch_dense_coop_ra<R, u128>(lpj, a, B, resident, s)
                    : launch_dense_coop_ra<R, uint64_t>(lpj, a, B, resident, s);
}

template <int R, int Threads>
hipError_t launch_gather_rt(const KArgs &a, int B, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>(B) * a.nblk), block(Threads);
    if (a.acc128)
        hipLaunchKernelGGL((k_gather<R, u128, Threads>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((k_gather<R, uint64_t, Threads>), grid, block, 0, s, a);
    return hipGetLastError();
}

template <int R>
hipError_t launch_gather_r(const KArgs &a, int B, hipStream_t s) {
    if constexpr (R <= 4)
        if (gather_wide(R, a.N, a.nblk)) return launch_gather_rt<R, 1024>(a, B, s);
    return launch_gather_rt<R, kBlockThreads>(a, B, s);
}

template <int R>
hipError_t launch_update_r(const KArgs &a, const double *demand_in, int B, hipStream_t s) {
    hipLaunchKernelGGL((k_update<R>), dim3((B + 255) / 256), dim3(256), 0, s, a, demand_in, B);
    return hipGetLastError();
}

template <int R>
hipError_t launch_prepare_r(const KArgs &a, const double *lam, double *canon, int B, hipStream_t s) {
    const size_t blocks = std::max<size_t>((static_cast<size_t>(B) + 255) / 256,
                                           std::min<size_t>((a.xch_clear + 255) / 256, 256));
    hipLaunchKernelGGL((k_prepare<R>), dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, a, lam, canon, B);
    return hipGetLastError();
}

template <int R>
hipError_t launch_finish_r(const KArgs &a, int B, hipStream_t s) {
    hipLaunchKernelGGL((k_finish<R>), dim3(static_cast<unsigned>(B)), dim3(kBlockThreads), 0, s, a);
    return hipGetLastError();
}

template <int R>
hipError_t launch_csr_r(const KArgs &a, int B, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>(B) * a.nblk), block(kBlockThreads);
    if (a.acc128)
        hipLaunchKernelGGL((k_csr<R, u128, kOnePass, false>), grid, block, 0, s, a);
    else if (a.lane_f64)
        hipLaunchKernelGGL((k_csr<R, uint64_t, kOnePass, true>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((k_csr<R, uint64_t, kOnePass, false>), grid, block, 0, s, a);
    return hipGetLastError();
}

template <int R, typename A, bool Direct>
const void *csr_multi_kernel(bool resident) {
    if (resident) return reinterpret_cast<const void *>(&k_csr<R, A, kResident, Direct>);
    return reinterpret_cast<const void *>(&k_csr<R, A, kPersist, Direct>);
}

template <int R>
hipError_t launch_csr_coop_r(const KArgs &a, int B, bool resident, hipStream_t s) {
    if (a.defer) return hipErrorInvalidValue;              // these launches complete their iterations
    const void *f = a.acc128 ? csr_multi_kernel<R, u128, false>(resident)
                    : a.lane_f64 ? csr_multi_kernel<R, uint64_t, true>(resident)
                                 : csr_multi_kernel<R, uint64_t, false>(resident);
    return launch_multi(f, static_cast<unsigned>(B) * a.nblk, a, R * a.limbs, s,
                        resident ? a.res_waves * kWaveSize : kBlockThreads);
}


// Instances compiled in the esp_inst_*.hip files.
#define ESP_FUSED_LAUNCHERS(X) \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8)
#define ESP_DENSE_DECL(RR, EXT)                                                                      \
    EXT template hipError_t launch_dense_r<RR>(int, const KArgs &, int, hipStream_t);                  \
    EXT template hipError_t launch_dense_coop_r<RR>(int, const KArgs &, int, bool, hipStream_t);
#define ESP_CSR_DECL(RR, EXT)                                                                        \
    EXT template hipError_t launch_csr_r<RR>(const KArgs &, int, hipStream_t);                         \
    EXT template hipError_t launch_csr_coop_r<RR>(const KArgs &, int, bool, hipStream_t);

}  // namespace esp
