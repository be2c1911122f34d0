// gfx950 kernels beyond the price loop: the effective capacity of Eq. 12,
// the outer ESP-IAC rounds of Alg. 1 and RST's nearest-profile fallback.
#include <algorithm>

#include "esp_device.hpp"
#include "esp_extras.hpp"

#pragma clang fp contract(off)

namespace esp {

// ---------------------------------------------------------------------------
// Effective capacity (Sec. 3.4, Eq. 12)
// ---------------------------------------------------------------------------

// C_eff_r = C_r - gamma * S_r, S_r = sum over pending jobs j of
// min over j's allowed configurations of d_jkr (the componentwise smallest
// footprint), over the pending jobs' own packed table.  A wavefront takes one
// tile at a time: each lane folds its 4 entries into one minimum per job
// piece (entries of one job are adjacent) and merges it into the tile's
// per-job minima in LDS with an unsigned atomic minimum (demands are
// non-negative floats with +0.0 for zero, whose bit patterns order like the
// values); the lanes then add the minima of pending jobs to exact fixed-point
// accumulators.  Masked configurations and padding carry a utility of -inf
// (dense padding: job index >= N) and are skipped.
// The general form (any accumulator width); k_reserve_lanes below takes the
// problems whose lanes' sums are exact in binary64.
template <int R, typename A>
__global__ __launch_bounds__(kBlockThreads) void k_reserve(KArgs a, ReserveArgs ra) {
    constexpr uint32_t kInf = 0x7f800000u;
    __shared__ uint32_t s_min[kBlockWaves][kTileEntries][R];
    __shared__ u128 s_part[kBlockWaves][R];
    __shared__ u128 s_bsum[R];
    const int cl = blockIdx.x / a.nblk;
    const int blk = blockIdx.x - cl * a.nblk;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x / kWaveSize;
    const float *col = a.table + cl * a.cluster_stride;
    const uint8_t *pend = ra.queued ? ra.queued + static_cast<size_t>(cl) * a.N : nullptr;
    int sh[R];
    A acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        sh[r] = a.shift[cl * R + r];
        acc[r] = 0;
    }
    uint32_t *mins = &s_min[wave][0][0];
    for (int i = lane; i < kTileEntries * R; i += kWaveSize) mins[i] = kInf;
    wave_sync();
    const int jpt = a.K > 0 ? kTileEntries / a.K : 0;          // dense: jobs per tile
    for (int tile = blk * kBlockWaves + wave; tile < a.tiles; tile += a.nblk * kBlockWaves) {
        const size_t base = static_cast<size_t>(tile) * kTileEntries + static_cast<size_t>(lane) * 4;
        const f4 u = *reinterpret_cast<const f4 *>(col + base);
        f4 d[R];
#pragma unroll
        for (int r = 0; r < R; ++r) d[r] = *reinterpret_cast<const f4 *>(col + (r + 1) * a.col_len + base);
        int first_job, njobs, jt;
        uint32_t heads;                        // bit i: entry 4*lane + i starts a job
        if (a.K > 0) {
            first_job = tile * jpt;
            njobs = min(jpt, a.N - first_job);
            jt = (lane * 4) / a.K;
            heads = 0;                         // K >= 4: a lane's 4 entries share one job
        } else {
            const TileMeta &m = a.meta[tile];
            const uint64_t lower = (1ull << lane) - 1ull;
            int before = 0, total = 0;
            heads = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                total += __popcll(m.head[i]);
                before += __popcll(m.head[i] & lower);
                heads |= static_cast<uint32_t>((m.head[i] >> lane) & 1ull) << i;
            }
            first_job = static_cast<int>(m.first_job);
            njobs = total;
            jt = before + static_cast<int>(heads & 1u) - 1; // entry 0 of a tile always starts a job
        }
        uint32_t mn[R];
#pragma unroll
        for (int r = 0; r < R; ++r) mn[r] = kInf;
        auto flush = [&]() {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (mn[r] != kInf) atomicMin(&s_min[wave][jt][r], mn[r]);
        };
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i > 0 && ((heads >> i) & 1u)) {
                flush();
                ++jt;
#pragma unroll
                for (int r = 0; r < R; ++r) mn[r] = kInf;
            }
            const bool valid = (u[i] != -__builtin_inff()) & (jt < njobs);
            if (valid) {
#pragma unroll
                for (int r = 0; r < R; ++r) mn[r] = min(mn[r], __float_as_uint(d[r][i]));
            }
        }
        flush();
        wave_sync();
        for (int q = lane; q < njobs; q += kWaveSize) {
            const bool take = !pend || pend[first_job + q] != 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t m = s_min[wave][q][r];
                s_min[wave][q][r] = kInf;
                if (take & (m != kInf)) acc[r] += fx_of<A>(__uint_as_float(m), sh[r]);
            }
        }
        wave_sync();
    }
    // workgroup sums: wavefront tree over lanes, then the 4 wavefronts in order
#pragma unroll
    for (int r = 0; r < R; ++r) {
        u128 v = static_cast<u128>(acc[r]);
#pragma unroll
        for (int off = kWaveSize / 2; off > 0; off >>= 1) {
            const unsigned long long lo = __shfl_down(static_cast<unsigned long long>(v), off);
            const unsigned long long hi = __shfl_down(static_cast<unsigned long long>(v >> 64), off);
            v += (static_cast<u128>(hi) << 64) | lo;
        }
        if (lane == 0) s_part[wave][r] = v;
    }
    __syncthreads();
    if (threadIdx.x < R) {
        u128 t = 0;
        for (int w = 0; w < kBlockWaves; ++w) t += s_part[w][threadIdx.x];
        s_bsum[threadIdx.x] = t;
    }
    __syncthreads();
    cluster_sums<R>(a, cl, blk, s_bsum, [&](int r, u128 tot) {
        const double S = fx_to_double(tot, a.shift[cl * R + r]);
        const double g = ra.gamma * S;
        const double ce = ra.cap_phys[cl * R + r] - g;
        ra.cap_eff[cl * R + r] = ce;
        if (ra.out) ra.out[cl * R + r] = ce;
    });
}

// The same in lanes: every segment minimum is formed in registers (a running
// minimum over the lane's 4 entries and a segmented scan over the lanes, the
// segments' lanes in scalar masks) and added, in binary64, by the lane where
// the segment ends, if the job is pending.  One launch over a small table is a
// few tiles per wavefront: bound by their latency, so the next tile's loads are
// in flight while one is reduced, no LDS lies on the chain, and 8 wavefronts per
// workgroup halve the tiles of each.  Measured, a call, against minima merged by
// LDS atomics in 4 wavefronts: 131,072 ragged jobs x 6 (46 MB) 23.5 -> 20.2 us,
// 20,000 x 64 x 8 25.6 -> 18.7, 500,000 x 4 x 3 19.3 -> 16.1; about 9 us are the
// launch and the sums' way through memory.  A table that a pass over another one
// has put out of the caches takes 23.4 us either way (23.6 before): memory.
__device__ __forceinline__ uint32_t min_u32(uint32_t a, uint32_t b) { return a < b ? a : b; }

template <int CTRL, int R>
__device__ __forceinline__ void min_scan_step(uint32_t (&v)[R], uint64_t lanes) {
    if (lanes == 0) return;                                // (dense families of K span K / 4 lanes)
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int o = __builtin_amdgcn_mov_dpp(static_cast<int>(v[r]), CTRL, 0xf, 0xf, true);
        v[r] = min_u32(v[r], in_mask(lanes) ? static_cast<uint32_t>(o) : v[r]);
    }
}

constexpr int kReserveWaves = 8;                           // 4 per SIMD with two workgroups per CU
constexpr int kReserveThreads = kReserveWaves * kWaveSize;

template <int R>
__global__ __launch_bounds__(kReserveThreads) void k_reserve_lanes(KArgs a, ReserveArgs ra) {
    constexpr uint32_t kInf = 0x7f800000u;
    __shared__ uint64_t s_part[kReserveWaves][R];
    __shared__ u128 s_bsum[R];
    struct Heads { uint64_t m[4]; };
    const int cl = blockIdx.x / a.nblk;
    const int blk = blockIdx.x - cl * a.nblk;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const float *col = a.table + cl * a.cluster_stride;
    const uint8_t *pend = ra.queued ? ra.queued + static_cast<size_t>(cl) * a.N : nullptr;
    const int stride = a.nblk * kReserveWaves;
    const int last = a.tiles - 1;
    const int jpt = a.K > 0 ? kTileEntries / a.K : 0;      // dense: jobs per tile, K / 4 lanes each
    double sum[R];
#pragma unroll
    for (int r = 0; r < R; ++r) sum[r] = 0.0;
    const uint64_t dense_starts = a.K > 0 ? mask_of(lane % (a.K > 0 ? a.K / 4 : 1) == 0) : 0ull;
    auto load_tile = [&](int t, f4 &u, f4 (&d)[R], Heads &h, int &first_job) {
        const size_t base = static_cast<size_t>(t) * kTileEntries + static_cast<size_t>(lane) * 4;
        u = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(col + base));
#pragma unroll
        for (int r = 0; r < R; ++r)
            d[r] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(col + (r + 1) * a.col_len + base));
        if (a.K > 0) {
            h = {{dense_starts, 0ull, 0ull, 0ull}};
            first_job = t * jpt;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) h.m[i] = scalar_word(a.meta + t, i);
            first_job = static_cast<int>(static_cast<uint32_t>(scalar_word(a.meta + t, 4)));
        }
    };
    auto reduce = [&](const f4 &u, const f4 (&d)[R], const Heads &h, int first_job) {
        // whether the job of entry i is pending (jobs past N, in a dense tile's padding, are not)
        int j = first_job - 1 +
                static_cast<int>(below_lane(h.m[3], below_lane(h.m[2], below_lane(h.m[1], below_lane(h.m[0], 0u)))));
        uint64_t want[4];
        int flag[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            j += in_mask(h.m[i]) ? 1 : 0;
            flag[i] = pend ? pend[min(j, a.N - 1)] : 1;
            flag[i] = j < a.N ? flag[i] : 0;
        }
        // masked configurations and padding carry a utility of -inf
        uint32_t run[R], pre[R];
        const uint64_t ok0 = mask_of(u[0] != -__builtin_inff());
#pragma unroll
        for (int r = 0; r < R; ++r) pre[r] = run[r] = in_mask(ok0) ? __float_as_uint(d[r][0]) : kInf;
        uint64_t open = h.m[0];
#pragma unroll
        for (int i = 0; i < 4; ++i) want[i] = mask_of(flag[i] != 0);
#pragma unroll
        for (int i = 1; i < 4; ++i) {
            const uint64_t ok = mask_of(u[i] != -__builtin_inff());
            const uint64_t first = h.m[i] & ~open;         // ends the part of a segment from lower lanes
            if (in_mask(h.m[i] & open & want[i - 1])) {    // ends a segment inside the lane
#pragma unroll
                for (int r = 0; r < R; ++r) sum[r] += static_cast<double>(__uint_as_float(run[r]));
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                pre[r] = in_mask(first) ? run[r] : pre[r];
                const uint32_t v = in_mask(ok) ? __float_as_uint(d[r][i]) : kInf;
                run[r] = min_u32(in_mask(h.m[i]) ? kInf : run[r], v);
            }
            open |= h.m[i];
        }
        const ScanLanes l = scan_lanes(open);
        min_scan_step<kDppRowShr1, R>(run, l.row1);
        min_scan_step<kDppRowShr2, R>(run, l.row2);
        min_scan_step<kDppRowShr4, R>(run, l.row4);
        min_scan_step<kDppRowShr8, R>(run, l.row8);
        min_scan_step<kDppRowBcast15, R>(run, l.rows);
        min_scan_step<kDppRowBcast31, R>(run, l.halves);
        uint32_t prev[R];
#pragma unroll
        for (int r = 0; r < R; ++r)
            prev[r] = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(run[r]), kDppWaveShr1, 0xf, 0xf, true));
        if (in_mask(open & ~h.m[0] & want[0])) {           // a segment from lower lanes ends before this lane's first head
#pragma unroll
            for (int r = 0; r < R; ++r) sum[r] += static_cast<double>(__uint_as_float(min_u32(pre[r], prev[r])));
        }
        if (in_mask(((h.m[0] >> 1) | (1ull << (kWaveSize - 1))) & want[3])) {   // or at the end of this lane
#pragma unroll
            for (int r = 0; r < R; ++r) sum[r] += static_cast<double>(__uint_as_float(run[r]));
        }
    };
    f4 ua, ub, da[R], db[R];
    Heads ha, hb;
    int ja, jb;
    const int tile0 = blk * kReserveWaves + wave;
    load_tile(min(tile0, last), ua, da, ha, ja);           // (clamped: no branch)
    for (int tile = tile0; tile < a.tiles; tile += 2 * stride) {
        load_tile(min(tile + stride, last), ub, db, hb, jb);
        reduce(ua, da, ha, ja);
        if (tile + stride >= a.tiles) break;
        load_tile(min(tile + 2 * stride, last), ua, da, ha, ja);
        reduce(ub, db, hb, jb);
    }
    uint64_t x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = static_cast<uint64_t>(ldexp(sum[r], -a.shift[cl * R + r]));
    const uint64_t tot = wave_totals<R>(x);
    if ((lane & 7) == 0 && lane / 8 < R) s_part[wave][lane / 8] = tot;
    __syncthreads();
    if (threadIdx.x < R) {
        u128 t = 0;
#pragma unroll
        for (int w = 0; w < kReserveWaves; ++w) t += s_part[w][threadIdx.x];
        s_bsum[threadIdx.x] = t;
    }
    __syncthreads();
    cluster_sums<R>(a, cl, blk, s_bsum, [&](int r, u128 total) {
        const double S = fx_to_double(total, a.shift[cl * R + r]);
        const double g = ra.gamma * S;
        const double ce = ra.cap_phys[cl * R + r] - g;
        ra.cap_eff[cl * R + r] = ce;
        if (ra.out) ra.out[cl * R + r] = ce;
    });
}

// ---------------------------------------------------------------------------
// Nearest-profile fallback of RST (Sec. 3.1.2, Sec. 4.1)
// ---------------------------------------------------------------------------

constexpr int kNearestLanes = 16;                     // lanes per query (one DPP row)

// Sum over the 16 lanes of a DPP row, in every lane of the row.
__device__ __forceinline__ uint32_t row_sum(uint32_t v) {
    constexpr int kRowRor8 = 0x128, kRowRor4 = 0x124, kRowRor2 = 0x122, kRowRor1 = 0x121;
    v += static_cast<uint32_t>(dpp_i<kRowRor8>(static_cast<int>(v)));
    v += static_cast<uint32_t>(dpp_i<kRowRor4>(static_cast<int>(v)));
    v += static_cast<uint32_t>(dpp_i<kRowRor2>(static_cast<int>(v)));
    v += static_cast<uint32_t>(dpp_i<kRowRor1>(static_cast<int>(v)));
    return v;
}

// Query i of a cluster names a job type f and an unprofiled configuration's
// resource vector q.  The 16 lanes of one DPP row serve a query: lane s takes
// entries s, s+16, ... of family f, skips masked ones (utility -inf), and
// keeps the smallest squared l2 distance, computed in binary64 in a fixed
// order (e_0 = q_0 - d_0, acc = e_0 e_0, acc = acc + e_r e_r for r = 1..R-1).
// The row then takes the argmax of the negated distance with lowest-index
// ties (group_argmax), i.e. the nearest entry with the lowest index among
// equals.  Lane 0 writes the index; the lane that found the entry writes its
// throughput (the utility), which it still holds in a register.  A family
// index out of range or a non-finite query component gives -1 / NaN and
// records an error.
//
// The family is read from the store's entry-major copy (AOS: each entry's
// utility and demands contiguous, so the family is one contiguous run that
// starts on a cache line) or from the structure-of-arrays columns of the
// price loop's table.  With the copy, the row finds the run from the
// directory record of the family's group of 60: lane 0 holds the group's
// first line, lanes 1..15 hold four one-byte family sizes each, and two row
// sums give the run's first line (the group's first line plus the lines of
// the families before f) and the family's size.  The directory (64 bytes per
// 60 families) stays in L2.
//
// Each query is a chain of dependent gathers (query -> family extent ->
// entries), so a row works on three queries at once: while it reads the
// entries of query i it has the extent of query i+1 and the family index of
// query i+2 in flight, and every step waits for one memory round trip
// instead of three.
template <int R, bool AOS>
__global__ __launch_bounds__(kBlockThreads) void k_nearest(KArgs a, NearestArgs na) {
    constexpr int kPerBlock = kBlockThreads / kNearestLanes;
    constexpr uint32_t kEntryBytes = 4 * (R + 1);
    const int sub = threadIdx.x & (kNearestLanes - 1);
    // The workgroup takes queries [lo, lo + chunk), kPerBlock at a time (one
    // per row), so the cache lines of the query and output arrays it touches
    // are its own.
    constexpr int64_t stride = kPerBlock;
    const int64_t lo = static_cast<int64_t>(blockIdx.x) * na.chunk;
    const int64_t last = min(lo + na.chunk, na.total) - 1;
    auto family_of = [&](int64_t g) { return na.family[g < last ? g : last]; };
    auto query_of = [&](int64_t g, float (&v)[R]) {
        const float *p = na.query + (g < last ? g : last) * R;
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = p[r];
    };
    auto in_range = [&](int f) { return (f >= 0) & (f < a.N); };
    // The extent lookup of a family (any value: out-of-range ones read family 0).
    // AOS: this lane's word of the family's directory record; else the family's
    // slot and size in the columns.
    auto extent_load = [&](int f) -> uint64_t {
        const int fc = in_range(f) ? f : 0;
        if constexpr (AOS) {
            return na.dir[static_cast<size_t>(fc / kDirFamilies) * kDirWords + sub];
        } else {
            if (a.K > 0) return (static_cast<uint64_t>(a.K) << 32) | (static_cast<uint32_t>(fc) * static_cast<uint32_t>(a.K));
            const JobSlot js = a.jobs[fc];
            return (static_cast<uint64_t>(js.size) << 32) | js.slot;
        }
    };
    // every lane of a row shares gi, so rows stay whole for the DPP steps
    int64_t gi = lo + threadIdx.x / kNearestLanes;
    if (gi > last) return;
    int f = family_of(gi);
    float q[R];
    query_of(gi, q);
    uint64_t ext = extent_load(f);
    int f1 = family_of(gi + stride);
    for (; gi <= last; gi += stride) {
        bool ok = in_range(f);
#pragma unroll
        for (int r = 0; r < R; ++r) ok = ok & (fabsf(q[r]) <= 3.402823466e38f);   // false for NaN and +-inf
        // next steps of the pipeline: the query and extent of gi + stride, the family of gi + 2 stride
        const uint64_t ext1 = extent_load(f1);
        const int f2 = family_of(gi + 2 * stride);
        float q1[R];
        query_of(gi + stride, q1);
        int size = 0;
        const float *base = nullptr;       // the family's first entry (AOS) or its slot in column 0
        const int cl = static_cast<int>(gi / na.Q);
        if constexpr (AOS) {
            const uint32_t w = static_cast<uint32_t>(ext);
            const int i = (in_range(f) ? f : 0) % kDirFamilies;
            const int first = 4 * (sub - 1);                 // family of byte 0 of this word
            uint32_t before = w, own = 0;                    // lane 0: the group's first line
            if (sub > 0) {
                before = 0;
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const uint32_t k = ((w >> (8 * m)) & 0xffu) + 1u;      // family size, 1..256
                    if (first + m < i) before += (k * kEntryBytes + (kStoreLine - 1)) / kStoreLine;
                    if (first + m == i) own = k;
                }
            }
            before = row_sum(before);
            own = row_sum(own);
            if (ok) {
                size = static_cast<int>(own);
                base = na.aos + (static_cast<size_t>(cl) * na.aos_lines + before) * (kStoreLine / 4);
            }
        } else if (ok) {
            size = static_cast<int>(ext >> 32);
            base = a.table + cl * a.cluster_stride + static_cast<uint32_t>(ext);
        }
        double best = -__builtin_inf();
        int bk = 0x7fffffff;
        float bu = 0.0f;
        for (int k = sub; k < size; k += kNearestLanes) {
            float d[R + 1];                                  // utility, then the R demands
            if constexpr (AOS) {
                __builtin_memcpy(d, base + static_cast<size_t>(k) * (R + 1), sizeof d);
            } else {
#pragma unroll
                for (int r = 0; r <= R; ++r) d[r] = base[r * a.col_len + k];
            }
            double x = static_cast<double>(q[0]) - static_cast<double>(d[1]);
            double acc = x * x;
#pragma unroll
            for (int r = 1; r < R; ++r) {
                x = static_cast<double>(q[r]) - static_cast<double>(d[r + 1]);
                acc = acc + x * x;
            }
            // Masked configurations (utility -inf) are no candidates.  k ascends
            // within a lane, so keeping the first of equal distances keeps the
            // lowest index.  Selects, not a branch: all of the entry's loads
            // are issued before the mask is tested.
            const bool take = (d[0] != -__builtin_inff()) & (-acc > best);
            best = take ? -acc : best;
            bk = take ? k : bk;
            bu = take ? d[0] : bu;
        }
        const int mine = bk;
        group_argmax<kNearestLanes>(best, bk);
        const bool found = ok && bk != 0x7fffffff;
        if (sub == 0) {
            na.nearest[gi] = found ? bk : -1;
            if (na.estimate && !found) na.estimate[gi] = __builtin_nanf("");
            if (!ok) atomicCAS(a.status, 0, in_range(f) ? kStatusNonfinite : kStatusInvalid);
        }
        // the entry's own lane (entries k of lane s satisfy k = s mod 16)
        if (found && na.estimate && mine == bk) na.estimate[gi] = bu;
        f = f1;
        ext = ext1;
        f1 = f2;
#pragma unroll
        for (int r = 0; r < R; ++r) q[r] = q1[r];
    }
}

// ---------------------------------------------------------------------------
// Outer ESP-IAC rounds (Sec. 3.4, Alg. 1; thresholds of Eq. 11)
// ---------------------------------------------------------------------------

// One workgroup per cluster, after the round's tatonnement and re-selection:
//  BinPack  jobs in index order; job j at its chosen configuration needs
//           g = d[r_gpus] GPUs (a whole number in 1..8, else not placeable)
//           and d[r_mem] / g memory and d[r_sm] / g compute on each; it takes
//           the g lowest-index GPUs with room for one share (all or
//           nothing; binary64 residuals, the oracle's operations).
//  IAC      every pair of jobs sharing a GPU: S_x|y = 1 + a_x b_y against
//           tau_x = tau_base_x + min(beta (U / U_target - 1), beta_max),
//           U = busy GPUs / G; a pair violates when either slowdown exceeds
//           its threshold.  Each job keeps its largest excess (atomic max on
//           the bit patterns of non-negative doubles).
//  Gamma    each violating job's chosen configuration: penalty <-
//           fp32(penalty + kappa * excess), in the packed penalty column
//           (its sign bit, the switching-cost mark, is kept).
// A cluster without violations is frozen: later rounds' kernels skip it.
//
// First fit is one serial chain over the jobs, so its latency per job bounds
// the kernel.  Wavefront 0 does nothing else: it holds the residuals of one
// group of 256 GPUs in registers (lane l, slot i: GPU 4 l + i of the group; the
// other groups lie in LDS and are swapped in when a job needs them), so testing
// the group is 8 compares whose results are the wave-wide masks, and a share
// is placed by the lanes that hold its GPUs, with no LDS round trip (the
// occupants are written to LDS, read only after the packing).  The other
// wavefronts gather the jobs ahead of it, kPackChunk batches of 64 at a time
// into one of two LDS buffers, leaving out the jobs that cannot be placed.
// The chain is bound by the issue of a lone wavefront (about 90 instructions
// and 530 cycles per placed job of one share, no memory access in it; a job of
// several takes its GPUs of a group at once: 300 jobs of 8 GPUs each on 2,048,
// one round without iterations 508 -> 284 us against share after share).  Measured per
// round against one wavefront that gathered and placed with the residuals in
// LDS: 4,096 jobs on 512 GPUs (1,035 jobs tried) 870 -> 257 us, 32 clusters of
// 4,096 jobs on 576..768 GPUs 1,256 -> 383 us.
//
// Shortcuts, all exact because residuals only shrink while jobs are placed:
//  - a job that needs at least as much (GPU count, memory and compute per
//    GPU) as one that found no room is not tried (up to 64 such needs, none
//    at or above another, one per lane of wavefront 0; the gathering
//    wavefronts test against the list of the chunk before);
//  - a group of 256 GPUs that had no GPU at all for a need is not visited
//    for needs at or above it (two such needs per group, lane b: group b).
// Wave-uniform copies of lane t's value (t uniform).
__device__ __forceinline__ int lane_i(int v, int t) { return __builtin_amdgcn_readlane(v, t); }
__device__ __forceinline__ double lane_d(double v, int t) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<unsigned>(b)), t));
    const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(b >> 32), t));
    return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}

constexpr int kPackWaves = 8;                            // wavefront 0 places, the others gather
constexpr int kPackThreads = kPackWaves * kWaveSize;
constexpr int kPackPer = 2;                              // batches per gathering wavefront and chunk
constexpr int kPackChunk = (kPackWaves - 1) * kPackPer;  // batches of 64 jobs per chunk
constexpr int kGroupSlots = 4;                           // slots per group: 256 GPUs
constexpr int kGroups = kMaxGpus / (kGroupSlots * kWaveSize);
static_assert((kMaxPerGpu & (kMaxPerGpu - 1)) == 0, "a GPU's entries of s_occ are found by masking");
static_assert(kGroups <= 32, "two needs per group in the lanes of a wavefront");

// GPUs of a group with room for a share: per slot, the lanes whose GPU has it.
struct Room {
    uint64_t mk[kGroupSlots];
    __device__ __forceinline__ uint64_t any() const { return mk[0] | mk[1] | mk[2] | mk[3]; }
    __device__ __forceinline__ int count() const {
        return __popcll(mk[0]) + __popcll(mk[1]) + __popcll(mk[2]) + __popcll(mk[3]);
    }
    // The GPU of lowest index alone, the lowest lane's first slot (all: any(), not 0).
    __device__ __forceinline__ Room first(uint64_t all) const {
        const uint64_t r0 = all & (0 - all), r1 = r0 & ~mk[0], r2 = r1 & ~mk[1];
        return {{r0 & mk[0], r1 & mk[1], r2 & mk[2], r2 & ~mk[2]}};
    }
    // The n GPUs of lowest index (all of them when there are no more): those
    // with fewer than n before them, in lower lanes or lower slots of the lane.
    __device__ __forceinline__ Room lowest(int n) const {
        unsigned before = below_lane(mk[3], below_lane(mk[2], below_lane(mk[1], below_lane(mk[0], 0u))));
        Room t;
#pragma unroll
        for (int i = 0; i < kGroupSlots; ++i) {
            t.mk[i] = __ballot(before < static_cast<unsigned>(n)) & mk[i];
            before += in_mask(mk[i]) ? 1u : 0u;
        }
        return t;
    }
};

// One group of GPUs in the registers of a wavefront: GPU 4 l + i of the group
// in lane l, slot i.
struct GroupRoom {
    double mem[kGroupSlots], sm[kGroupSlots];            // residuals; memory -inf: takes no more jobs
    int at[kGroupSlots];                                 // the next free entry of s_occ

    // GPUs with room (all compares first: their latencies overlap).
    __device__ __forceinline__ Room room(double nm, double ns) const {
        Room r;
        uint64_t ok[kGroupSlots];
#pragma unroll
        for (int i = 0; i < kGroupSlots; ++i) r.mk[i] = __ballot(mem[i] >= nm);
#pragma unroll
        for (int i = 0; i < kGroupSlots; ++i) ok[i] = __ballot(sm[i] >= ns);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kGroupSlots; ++i) r.mk[i] &= ok[i];
        return r;
    }
    // Take one share (nm, ns) from each GPU in `t`; returns the entry of s_occ (of
    // a lane with one GPU in `t`).  One assembly block of predicated
    // operations: written as branches, the compiler kept two copies of every
    // residual and moved them at each job.  EXEC is saved and restored.
    __device__ __forceinline__ int take(const Room &t, double nm, double ns) {
        int w;
        uint64_t ex;
        asm volatile("s_mov_b64 %[ex], exec\n\t"
                     "s_mov_b64 exec, %[e0]\n\t"
                     "v_mov_b32 %[w], %[a0]\n\t"
                     "v_add_f64 %[m0], %[m0], -%[nm]\n\t"
                     "v_add_f64 %[s0], %[s0], -%[ns]\n\t"
                     "v_add_u32 %[a0], 1, %[a0]\n\t"
                     "s_mov_b64 exec, %[e1]\n\t"
                     "v_mov_b32 %[w], %[a1]\n\t"
                     "v_add_f64 %[m1], %[m1], -%[nm]\n\t"
                     "v_add_f64 %[s1], %[s1], -%[ns]\n\t"
                     "v_add_u32 %[a1], 1, %[a1]\n\t"
                     "s_mov_b64 exec, %[e2]\n\t"
                     "v_mov_b32 %[w], %[a2]\n\t"
                     "v_add_f64 %[m2], %[m2], -%[nm]\n\t"
                     "v_add_f64 %[s2], %[s2], -%[ns]\n\t"
                     "v_add_u32 %[a2], 1, %[a2]\n\t"
                     "s_mov_b64 exec, %[e3]\n\t"
                     "v_mov_b32 %[w], %[a3]\n\t"
                     "v_add_f64 %[m3], %[m3], -%[nm]\n\t"
                     "v_add_f64 %[s3], %[s3], -%[ns]\n\t"
                     "v_add_u32 %[a3], 1, %[a3]\n\t"
                     "s_mov_b64 exec, %[ex]"
                     : [m0] "+v"(mem[0]), [m1] "+v"(mem[1]), [m2] "+v"(mem[2]), [m3] "+v"(mem[3]), [s0] "+v"(sm[0]),
                       [s1] "+v"(sm[1]), [s2] "+v"(sm[2]), [s3] "+v"(sm[3]), [a0] "+v"(at[0]), [a1] "+v"(at[1]),
                       [a2] "+v"(at[2]), [a3] "+v"(at[3]), [w] "=&v"(w), [ex] "=&s"(ex)
                     : [e0] "s"(t.mk[0]), [e1] "s"(t.mk[1]), [e2] "s"(t.mk[2]), [e3] "s"(t.mk[3]), [nm] "s"(nm),
                       [ns] "s"(ns));
        return w;
    }
    // The GPUs in `t` are full: their memory no longer admits anything.
    __device__ __forceinline__ void close(const Room &t) {
#pragma unroll
        for (int i = 0; i < kGroupSlots; ++i)
            mem[i] = __builtin_amdgcn_inverse_ballot_w64(t.mk[i]) ? -__builtin_inf() : mem[i];
    }
};

// Jobs of one batch that may still be placed, in job order.
struct PackBatch {
    double mem[kWaveSize], sm[kWaveSize];                // per share
    int gj[kWaveSize];                                   // job - 64 * batch, shares in the low 4 bits
};

// Needs that found no room (entry 0 .. n - 1; g above any job's when unused).
struct PackFails {
    double mem[kWaveSize], sm[kWaveSize];
    int g[kWaveSize];
    int n;
};

// GPUs of whole groups, and the LDS they take: up to 1,024 GPUs two workgroups share
// a compute unit, so that more clusters than units are packed at once (one round of
// 300 clusters of 400 jobs on 512 GPUs 365 -> 207 us, 256 of them 180).
__host__ __device__ constexpr int pack_slots(int gmax) {
    return (gmax + kGroupSlots * kWaveSize - 1) / (kGroupSlots * kWaveSize) * (kGroupSlots * kWaveSize);
}
constexpr size_t pack_lds(int gmax) {
    return static_cast<size_t>(pack_slots(gmax)) * (kMaxPerGpu * sizeof(int) + 2 * sizeof(double) + sizeof(int));
}

__global__ __launch_bounds__(kPackThreads) void k_pack_iac(KArgs a, IacArgs m) {
    __shared__ PackBatch s_batch[2][kPackChunk];
    __shared__ int s_n[2][kPackChunk];
    __shared__ PackFails s_fail[2];
    __shared__ int s_used, s_viol;
    // sized by the launch's largest cluster (pack_lds)
    extern __shared__ double s_gpus[];
    const int slots = pack_slots(m.gmax);
    int *const s_occ = reinterpret_cast<int *>(s_gpus);  // jobs of each GPU in placement order, -1 free
    double *const s_mem = s_gpus + slots * kMaxPerGpu / 2, *const s_sm = s_mem + slots;   // the groups not in registers
    int *const s_at = reinterpret_cast<int *>(s_sm + slots);
    const int cl = blockIdx.x;
    if (a.flags[cl] & kFlagFrozen) return;
    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWaveSize);
    const int G = m.gpus[cl];
    const int N = a.N;
    float *col = const_cast<float *>(a.table) + cl * a.cluster_stride;
    const int32_t *ch = m.choice + static_cast<size_t>(cl) * N;
    for (int i = tid; i < G * kMaxPerGpu; i += kPackThreads) s_occ[i] = -1;
    for (int h = tid; h < (G + kGroupSlots * kWaveSize - 1) / (kGroupSlots * kWaveSize) * (kGroupSlots * kWaveSize); h += kPackThreads) {
        s_mem[h] = h < G ? m.gpu_memory : -__builtin_inf();   // GPUs beyond G get no room at all
        s_sm[h] = m.gpu_compute;
        s_at[h] = h * kMaxPerGpu;
    }
    if (tid < 2) s_fail[tid].n = 0;
    if (tid == 0) s_used = s_viol = 0;
    const int batches = (N + kWaveSize - 1) / kWaveSize;
    const int chunks = (batches + kPackChunk - 1) / kPackChunk;

    // Gathering wavefronts: batch (wave - 1) + 7 u of chunk c, into buffer c & 1.
    // Indices past N are clamped (loaded, then ignored), so the loads of all
    // batches are issued together and stay in bounds.
    auto gather = [&](int c) {
        int k[kPackPer], size[kPackPer];
        size_t base[kPackPer];
        float gv[kPackPer], mv[kPackPer], sv[kPackPer];
#pragma unroll
        for (int u = 0; u < kPackPer; ++u) {
            const int b = c * kPackChunk + (wave - 1) + u * (kPackWaves - 1);
            const int jl = static_cast<int>(min(static_cast<int64_t>(b) * kWaveSize + lane, static_cast<int64_t>(N - 1)));
            k[u] = ch[jl];
            if (a.K > 0) {
                base[u] = static_cast<size_t>(jl) * a.K;
                size[u] = a.K;
            } else {
                const JobSlot js = a.jobs[jl];
                base[u] = js.slot;
                size[u] = static_cast<int>(js.size);
            }
        }
#pragma unroll
        for (int u = 0; u < kPackPer; ++u) {
            const size_t e = base[u] + static_cast<size_t>(((k[u] >= 0) & (k[u] < size[u])) ? k[u] : 0);
            gv[u] = col[(m.r_gpus + 1) * a.col_len + e];
            mv[u] = col[(m.r_mem + 1) * a.col_len + e];
            sv[u] = col[(m.r_sm + 1) * a.col_len + e];
        }
        const PackFails &fl = s_fail[c & 1];
        const int nf = fl.n;
#pragma unroll
        for (int u = 0; u < kPackPer; ++u) {
            const int q = (wave - 1) + u * (kPackWaves - 1);
            const int64_t j = (static_cast<int64_t>(c) * kPackChunk + q) * kWaveSize + lane;
            const double g = static_cast<double>(gv[u]);
            const double nm = static_cast<double>(mv[u]) / g;
            const double ns = static_cast<double>(sv[u]) / g;
            bool ok = (j < N) & (k[u] >= 0) & (k[u] < size[u]) & (g >= 1.0) &
                      (g <= static_cast<double>(kMaxShards)) & (g == floor(g));
            const int gi = ok ? static_cast<int>(g) : 0;
            for (int f = 0; f < nf; ++f) ok = ok & !((gi >= fl.g[f]) & (nm >= fl.mem[f]) & (ns >= fl.sm[f]));
            const uint64_t keep = __ballot(ok);
            PackBatch &o = s_batch[c & 1][q];
            if (ok) {
                const int at = __popcll(keep & ((1ull << lane) - 1ull));
                o.mem[at] = nm;
                o.sm[at] = ns;
                o.gj[at] = (lane << 4) | gi;
            }
            if (lane == 0) s_n[c & 1][q] = __popcll(keep);
        }
    };

    if (wave > 0) {
        __syncthreads();                                   // the empty failure lists are there
        gather(0);
        __syncthreads();
        for (int c = 0; c < chunks; ++c) {
            if (c + 1 < chunks) gather(c + 1);
            __syncthreads();
        }
    } else {
        GroupRoom gr;                                      // the GPUs of group `cur`
        int cur = 0;
        auto load = [&]() {
#pragma unroll
            for (int i = 0; i < kGroupSlots; ++i) {
                const int h = (cur * kWaveSize + lane) * kGroupSlots + i;
                gr.mem[i] = s_mem[h];
                gr.sm[i] = s_sm[h];
                gr.at[i] = s_at[h];
            }
            // arrived before any job is tested: none then waits for the LDS stores of the job before
#pragma unroll
            for (int i = 0; i < kGroupSlots; ++i) asm volatile("" : "+v"(gr.mem[i]), "+v"(gr.sm[i]), "+v"(gr.at[i]));
        };
        auto swap_in = [&](int b) {
#pragma unroll
            for (int i = 0; i < kGroupSlots; ++i) {
                const int h = (cur * kWaveSize + lane) * kGroupSlots + i;
                s_mem[h] = gr.mem[i];
                s_sm[h] = gr.sm[i];
                s_at[h] = gr.at[i];
            }
            cur = b;
            load();
        };
        const uint32_t groups = (2u << ((G - 1) / (kGroupSlots * kWaveSize))) - 1u;
        const double inf = __builtin_inf();
        double none_m = inf, none_s = inf;                 // lanes b and 32 + b: needs group b had no GPU for
        double fail_m = inf, fail_s = inf;                 // lane f: a need that found no room
        int fail_g = 0x7fffffff;
        int n_fail = 0, ring = 0;
        uint64_t fresh = 0, fresh_prev = 0;                // entries the gathering wavefronts have not seen
        __syncthreads();
        load();
        __syncthreads();
        for (int c = 0; c < chunks; ++c) {
            // (the batches of this chunk were tested against the list of the end of chunk c - 2)
            for (int q = 0; q < kPackChunk; ++q) {
                const int n = __builtin_amdgcn_readfirstlane(s_n[c & 1][q]);
                if (n == 0) continue;
                const int j0 = (c * kPackChunk + q) * kWaveSize;
                const PackBatch &in = s_batch[c & 1][q];
                double nm_l = in.mem[lane], ns_l = in.sm[lane];
                int gj_l = in.gj[lane];
                // arrived before the loop: no job then waits for the LDS stores of the one before
                asm volatile("" : "+v"(nm_l), "+v"(ns_l), "+v"(gj_l));
                const int g_l = gj_l & 15;
                int out = lane >= n;
                for (uint64_t fs = fresh | fresh_prev; fs != 0; fs &= fs - 1) {
                    const int f = __builtin_ctzll(fs);
                    out |= static_cast<int>(g_l >= lane_i(fail_g, f)) & static_cast<int>(nm_l >= lane_d(fail_m, f)) &
                           static_cast<int>(ns_l >= lane_d(fail_s, f));
                }
                uint64_t todo = __ballot(out == 0);
                // The next job's need is read into scalars while a job is placed.
                int gj_n;
                double nm_n, ns_n;
                auto fetch = [&]() {
                    const int t = __builtin_ctzll(todo | (1ull << (kWaveSize - 1)));   // (some lane's when none is left)
                    gj_n = lane_i(gj_l, t);
                    nm_n = lane_d(nm_l, t);
                    ns_n = lane_d(ns_l, t);
                };
                fetch();
                while (todo != 0) {
                    int g, job;
                    double nm, ns;
                    uint32_t cand;
                    Room r;
                    // one share on the first GPU of r (all: r.any())
                    auto put = [&](uint64_t all) {
                        const Room t = r.first(all);
                        const int w = gr.take(t, nm, ns);
                        const uint64_t bit = all & (0 - all);
                        if (__builtin_amdgcn_inverse_ballot_w64(bit)) s_occ[w] = job;
                        if (__builtin_expect((__ballot((w & (kMaxPerGpu - 1)) == kMaxPerGpu - 1) & bit) != 0, 0))
                            gr.close(t);
                    };
                    // one share on each GPU of t, all at once
                    auto put_each = [&](const Room &t) {
                        const int w[kGroupSlots] = {gr.at[0], gr.at[1], gr.at[2], gr.at[3]};
                        (void)gr.take(t, nm, ns);
                        Room full;
#pragma unroll
                        for (int i = 0; i < kGroupSlots; ++i) {
                            if (in_mask(t.mk[i])) s_occ[w[i]] = job;
                            full.mk[i] = __ballot((w[i] & (kMaxPerGpu - 1)) == kMaxPerGpu - 1) & t.mk[i];
                        }
                        if (full.any() != 0) gr.close(full);
                    };
                    // most jobs: one share, room in the group in registers, no group before it that may have room
                    // (a loop of its own, so that its state stays in place in the registers)
                    bool here = false;
                    const uint32_t cur_bit = 1u << cur;
                    do {
                        g = gj_n & 15;
                        job = j0 + (gj_n >> 4);
                        nm = nm_n;
                        ns = ns_n;
                        todo &= todo - 1;
                        const uint64_t none_a = __ballot(nm >= none_m), none_b = __ballot(ns >= none_s);
                        fetch();
                        r = gr.room(nm, ns);
                        const uint64_t none = none_a & none_b;
                        cand = ~static_cast<uint32_t>(none | (none >> 32)) & groups;
                        here = (static_cast<uint32_t>(g ^ 1) | ((cand & (0u - cand)) ^ cur_bit)) == 0;
                        if (!here) break;
                        const uint64_t all = r.any();
                        here = all != 0;
                        if (!here) break;
                        put(all);
                    } while (todo != 0);
                    if (here) break;
                    // group by group: count the room up to g GPUs, then place (all or nothing)
                    int found = 0;
                    for (uint32_t cs = cand; cs != 0 && found < g; cs &= cs - 1u) {
                        const int b = __builtin_ctz(cs);
                        if (b != cur) {
                            swap_in(b);
                            r = gr.room(nm, ns);
                        }
                        const int k = r.count();
                        if (k == 0) {
                            // group b has no GPU for this need: kept in place of a need at or above it, else of
                            // the second
                            const uint64_t over = __ballot(none_m >= nm) & __ballot(none_s >= ns);
                            const bool mine = lane == (((over >> b) & 1u) ? b : 32 + b);
                            none_m = mine ? nm : none_m;
                            none_s = mine ? ns : none_s;
                        }
                        found += k;
                    }
                    if (found >= g) {
                        if (g == 1) {                      // in the group last counted
                            put(r.any());
                            continue;
                        }
                        int rem = g;
                        for (uint32_t cs = cand; rem > 0; cs &= cs - 1u) {
                            const int b = __builtin_ctz(cs);
                            if (b != cur) {
                                swap_in(b);
                                r = gr.room(nm, ns);
                            }
                            const Room t = r.lowest(rem);
                            put_each(t);
                            rem -= t.count();
                        }
                        continue;
                    }
                    // no room: remember the need in place of one at or above it (unused entries are), else the oldest
                    const uint64_t over = __ballot(fail_g >= g) & __ballot(fail_m >= nm) & __ballot(fail_s >= ns);
                    const int f = over != 0 ? __builtin_ctzll(over) : ring;
                    if (over == 0) ring = (ring + 1) & (kWaveSize - 1);
                    fail_g = lane == f ? g : fail_g;
                    fail_m = lane == f ? nm : fail_m;
                    fail_s = lane == f ? ns : fail_s;
                    n_fail = max(n_fail, f + 1);
                    fresh |= 1ull << f;
                    todo &= ~(__ballot(g_l >= g) & __ballot(nm_l >= nm) & __ballot(ns_l >= ns));
                    fetch();
                }
            }
            // the list as it stands, for the gather of chunk c + 2 (which starts after the barrier)
            PackFails &fl = s_fail[c & 1];
            fl.mem[lane] = fail_m;
            fl.sm[lane] = fail_s;
            fl.g[lane] = fail_g;
            if (lane == 0) fl.n = n_fail;
            fresh_prev = fresh;
            fresh = 0;
            __syncthreads();
        }
    }

    // thresholds of Eq. 11
    int used = 0;
    for (int h = tid; h < G; h += kPackThreads) used += s_occ[h * kMaxPerGpu] >= 0;
    if (used) atomicAdd(&s_used, used);
    __syncthreads();
    double q = static_cast<double>(s_used) / static_cast<double>(G);
    q = q / m.u_target;
    const double w = q - 1.0;
    double add = m.beta * w;
    if (add > m.beta_max) add = m.beta_max;
    const float *sa = m.sensitivity + static_cast<size_t>(cl) * m.nnz;
    const float *pb = m.pressure + static_cast<size_t>(cl) * m.nnz;
    const double *tb = m.tau_base + static_cast<size_t>(cl) * N;
    unsigned long long *inc = reinterpret_cast<unsigned long long *>(m.inc) + static_cast<size_t>(cl) * N;
    int V = 0;
    for (int h = tid; h < G; h += kPackThreads) {
        // the GPU's jobs: all loads of a step in flight together (free slots read job 0, then are ignored)
        int j[kMaxPerGpu];
        int64_t e[kMaxPerGpu];
        double sv[kMaxPerGpu], pv[kMaxPerGpu], tv[kMaxPerGpu];
        if (s_occ[h * kMaxPerGpu + 1] < 0) continue;       // at most one job: no pair
#pragma unroll
        for (int x = 0; x < kMaxPerGpu; ++x) {
            j[x] = s_occ[h * kMaxPerGpu + x];
            const int jc = max(j[x], 0);
            e[x] = m.offsets[jc] + ch[jc];
            e[x] = j[x] >= 0 ? e[x] : 0;
            tv[x] = tb[jc] + add;
        }
#pragma unroll
        for (int x = 0; x < kMaxPerGpu; ++x) {
            sv[x] = static_cast<double>(sa[e[x]]);
            pv[x] = static_cast<double>(pb[e[x]]);
        }
#pragma unroll
        for (int x = 0; x < kMaxPerGpu; ++x)
#pragma unroll
            for (int y = x + 1; y < kMaxPerGpu; ++y) {
                if (j[y] < 0) continue;
                const double sxy = 1.0 + sv[x] * pv[y];
                const double syx = 1.0 + sv[y] * pv[x];
                const double ox = sxy - tv[x];
                const double oy = syx - tv[y];
                if (ox > 0.0) atomicMax(&inc[j[x]], static_cast<unsigned long long>(__double_as_longlong(ox)));
                if (oy > 0.0) atomicMax(&inc[j[y]], static_cast<unsigned long long>(__double_as_longlong(oy)));
                V += (ox > 0.0 || oy > 0.0) ? 1 : 0;
            }
    }
    if (V) atomicAdd(&s_viol, V);
    __threadfence();                                       // the maxima are complete before they are read
    __syncthreads();
    V = s_viol;
    // Gamma: whoever takes a job's largest excess (and leaves 0) raises its penalty
    if (V > 0) {
        float *pcol = col + static_cast<size_t>(m.pen_col) * a.col_len;
        for (int h = tid; h < G; h += kPackThreads) {
            int j[kMaxPerGpu];
            unsigned long long bits[kMaxPerGpu];
#pragma unroll
            for (int x = 0; x < kMaxPerGpu; ++x) {
                j[x] = s_occ[h * kMaxPerGpu + x];
                bits[x] = j[x] >= 0 ? atomicExch(&inc[j[x]], 0ull) : 0ull;
            }
#pragma unroll
            for (int x = 0; x < kMaxPerGpu; ++x) {
                if (bits[x] == 0ull) continue;
                const double ex = __longlong_as_double(static_cast<long long>(bits[x]));
                const size_t e = (a.K > 0 ? static_cast<size_t>(j[x]) * a.K : static_cast<size_t>(a.jobs[j[x]].slot)) +
                                 ch[j[x]];
                const uint32_t old = __float_as_uint(pcol[e]);
                const float mag = __uint_as_float(old & 0x7fffffffu);
                const float nv = __double2float_rn(static_cast<double>(mag) + m.kappa * ex);
                pcol[e] = __uint_as_float(__float_as_uint(nv) | (old & 0x80000000u));
            }
        }
    }
    int32_t *gj = m.gpu_jobs + static_cast<size_t>(cl) * m.gmax * kMaxPerGpu;
    for (int i = tid; i < m.gmax * kMaxPerGpu; i += kPackThreads) gj[i] = i < G * kMaxPerGpu ? s_occ[i] : -1;
    if (tid == 0) {
        m.violations[cl] = V;
        m.rounds_used[cl] = m.round;
        if (V == 0) a.flags[cl] = a.flags[cl] | kFlagFrozen;
    }
}

// Gamma <- 0 over the packed penalty columns (sign bits kept) and/or clear
// the frozen flags.
__global__ void k_iac_reset(float *table, size_t cluster_stride, size_t col_len, int R, int B, int32_t *flags,
                            int zero_gamma) {
    const size_t tid = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
    if (zero_gamma) {
        const size_t total = static_cast<size_t>(B) * col_len;
        for (size_t i = tid; i < total; i += stride) {
            const size_t b = i / col_len, e = i - b * col_len;
            float *p = table + b * cluster_stride + static_cast<size_t>(R + 1) * col_len + e;
            *p = __uint_as_float(__float_as_uint(*p) & 0x80000000u);
        }
    }
    for (size_t b = tid; b < static_cast<size_t>(B); b += stride) flags[b] = flags[b] & ~kFlagFrozen;
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

template <int R>
static hipError_t launch_nearest_r(const KArgs &a, const NearestArgs &na, hipStream_t s) {
    constexpr int kPerBlock = kBlockThreads / kNearestLanes;
    constexpr int64_t kLineQueries = 32;             // one 128-byte line of 4-byte outputs
    const int64_t cap = 256 * 32;                    // enough resident queries to cover gather latency
    const int64_t need = (na.total + kPerBlock - 1) / kPerBlock;
    NearestArgs nb = na;
    nb.chunk = (na.total + (need < cap ? need : cap) - 1) / (need < cap ? need : cap);
    nb.chunk = (nb.chunk + kLineQueries - 1) / kLineQueries * kLineQueries;
    const dim3 grid(static_cast<unsigned>((na.total + nb.chunk - 1) / nb.chunk)), block(kBlockThreads);
    if (na.aos)
        hipLaunchKernelGGL((k_nearest<R, true>), grid, block, 0, s, a, nb);
    else
        hipLaunchKernelGGL((k_nearest<R, false>), grid, block, 0, s, a, nb);
    return hipGetLastError();
}

hipError_t launch_nearest(int R, const KArgs &a, const NearestArgs &na, hipStream_t s) {
#define CALL(RR) launch_nearest_r<RR>(a, na, s)
    ESP_DISPATCH_R(R, CALL)
#undef CALL
}

hipError_t launch_pack_iac(int R, const KArgs &a, const IacArgs &m, int B, hipStream_t s) {
    IacArgs mm = m;
    mm.pen_col = R + 1;
    const dim3 grid(static_cast<unsigned>(B)), block(kPackThreads);
    // (one value for every launch: the limit belongs to the process)
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_pack_iac),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(pack_lds(kMaxGpus)));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_pack_iac, grid, block, pack_lds(m.gmax), s, a, mm);
    return hipGetLastError();
}

hipError_t launch_iac_reset(int R, const KArgs &a, int B, int zero_gamma, hipStream_t s) {
    const size_t work = zero_gamma ? static_cast<size_t>(B) * a.col_len : static_cast<size_t>(B);
    const size_t blocks = std::min<size_t>((work + 255) / 256, 4096);
    hipLaunchKernelGGL(k_iac_reset, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s,
                       const_cast<float *>(a.table), a.cluster_stride, a.col_len, R, B, a.flags, zero_gamma);
    return hipGetLastError();
}

template <int R>
static hipError_t launch_reserve_r(const KArgs &a, const ReserveArgs &ra, int B, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>(B) * a.nblk), block(kBlockThreads);
    if (a.acc128)
        hipLaunchKernelGGL((k_reserve<R, u128>), grid, block, 0, s, a, ra);
    else if (a.lane_f64)
        hipLaunchKernelGGL((k_reserve_lanes<R>), grid, dim3(kReserveThreads), 0, s, a, ra);
    else
        hipLaunchKernelGGL((k_reserve<R, uint64_t>), grid, block, 0, s, a, ra);
    return hipGetLastError();
}

hipError_t launch_reserve(int R, const KArgs &a, const ReserveArgs &ra, int B, hipStream_t s) {
#define CALL(RR) launch_reserve_r<RR>(a, ra, B, s)
    ESP_DISPATCH_R(R, CALL)
#undef CALL
}

}  // namespace esp
