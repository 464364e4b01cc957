// Top-B retention decision and hole-fill compaction plan (Sec. 3 eviction rule; ties keep the lower position).
//
// One 1024-thread workgroup per sequence.  Cases:
//  * n <= B: keep everything, nothing moves.
//  * n == B + 1 (every steady decode step): evict the single minimum under (u ascending, position
//    descending) -- one pass and a workgroup argmin.
//  * otherwise: MSB-first radix select (4 passes of 8 bits) over order-preserving utility keys finds the
//    B-th largest key tau; if more tokens tie at tau than are needed, a second radix select over positions
//    finds the largest kept position among the ties.
// The plan then pairs, in ascending order, the dropped slots below k = min(B, n) ("holes") with the kept
// slots at or above k ("tails"): per-segment counts from wave ballots, a scan over the segments, and ballot
// prefixes inside them; it records the pair count per sequence.  Measured on first-step-shaped utilities
// against one sweep of 1024-slot blocks with two barriers each: 76 -> 68 us at batch 8 x 32,769 tokens,
// 284 -> 235 us at batch 2 x 131,073, 23 -> 29 us at batch 32 x 8,193.
#include "kernels.h"
#include "kv_common.h"

namespace ikv {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;

constexpr int kMaxSegs = 2048;  // plan segments (a multiple of 64)
#ifndef IKV_SEL_BATCH
#define IKV_SEL_BATCH 8
#endif
constexpr int kBatch = IKV_SEL_BATCH;  // loads issued together by the histogram sweeps
constexpr int kPlanBatch = 16;  // 64-slot groups whose decisions a wave loads together in the plan sweeps

struct SelShared {
    unsigned hist[256];
    unsigned bcast[4];
    unsigned seg[kMaxSegs][2];  // per plan segment: holes, tails (then their offsets)
    uint32_t best_key[kWaves];
    int best_pos[kWaves];
    int best_idx[kWaves];
};

// Digit selection after a histogram pass: wave 0 scans the 256 bins in the requested order and publishes the
// digit whose bin holds the krem-th element, the count before it and the bin count.
__device__ void find_digit(SelShared& sh, unsigned krem, bool descending) {
    const int lane = threadIdx.x % kWave;
    if (threadIdx.x >= kWave) return;
    unsigned c[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int bin = descending ? 255 - (lane * 4 + j) : lane * 4 + j;
        c[j] = sh.hist[bin];
        sum += c[j];
    }
    unsigned incl = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const unsigned t = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += t;
    }
    unsigned before = incl - sum;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (before < krem && krem <= before + c[j]) {
            sh.bcast[0] = descending ? 255 - (lane * 4 + j) : lane * 4 + j;
            sh.bcast[1] = before;
            sh.bcast[2] = c[j];
        }
        before += c[j];
    }
}

// Histogram increments of one thread, aggregated over runs of equal digits: the utilities of a step cluster
// in a few exponents, so most keys of the leading passes fall in one or two bins, where one LDS atomic per key
// would serialise the whole workgroup on a single address.
struct RunCounter {
    unsigned bin = 0xffffffffu, count = 0;
    __device__ void add(unsigned* hist, unsigned d) {
        if (d != bin) {
            if (count) atomicAdd(&hist[bin], count);
            bin = d;
            count = 0;
        }
        ++count;
    }
    __device__ void flush(unsigned* hist) {
        if (count) atomicAdd(&hist[bin], count);
    }
};

__global__ __launch_bounds__(kThreads) void select_kernel(SelectArgs a) {
    __shared__ SelShared sh;
    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const float* ub = a.u + (size_t)b * a.cap;
    const int32_t* pb = a.pos + (size_t)b * a.cap;
    const int n = a.n, B = a.budget;
    const int k = min(B, n);

    // decision: mode 0 keep all, 1 evict `winner`, 2 threshold (tau, pi)
    int mode;
    int winner = -1;
    uint32_t tau = 0;
    int pi = 0x7fffffff;
    if (n <= B) {
        mode = 0;
    } else if (n == B + 1) {
        mode = 1;
        uint32_t bk = 0xffffffffu;
        int bp = -1, bi = -1;
        for (int i = tid; i < n; i += kThreads) {
            const uint32_t key = float_key(ub[i]);
            const int ps = pb[i];
            if (bi < 0 || key < bk || (key == bk && ps > bp)) {
                bk = key;
                bp = ps;
                bi = i;
            }
        }
#pragma unroll
        for (int o = kWave / 2; o >= 1; o >>= 1) {
            const uint32_t ok = __shfl_xor(bk, o, kWave);
            const int op = __shfl_xor(bp, o, kWave);
            const int oi = __shfl_xor(bi, o, kWave);
            if (oi >= 0 && (bi < 0 || ok < bk || (ok == bk && op > bp))) {
                bk = ok;
                bp = op;
                bi = oi;
            }
        }
        if (lane == 0) {
            sh.best_key[wave] = bk;
            sh.best_pos[wave] = bp;
            sh.best_idx[wave] = bi;
        }
        __syncthreads();
        bk = sh.best_key[0];
        bp = sh.best_pos[0];
        bi = sh.best_idx[0];
        for (int w = 1; w < kWaves; ++w) {
            const int oi = sh.best_idx[w];
            if (oi >= 0 && (bi < 0 || sh.best_key[w] < bk || (sh.best_key[w] == bk && sh.best_pos[w] > bp))) {
                bk = sh.best_key[w];
                bp = sh.best_pos[w];
                bi = oi;
            }
        }
        winner = bi;
    } else {
        mode = 2;
        uint32_t prefix = 0, pmask = 0;
        unsigned krem = (unsigned)B;
        unsigned ties = 0;
        for (int shift = 24; shift >= 0; shift -= 8) {
            if (tid < 256) sh.hist[tid] = 0;
            __syncthreads();
            RunCounter rc;
            for (int i0 = tid; i0 < n; i0 += kThreads * kBatch) {
                uint32_t key[kBatch];
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    const int i = i0 + j * kThreads;
                    key[j] = i < n ? float_key(ub[i]) : 0u;
                }
#pragma unroll
                for (int j = 0; j < kBatch; ++j)
                    if (i0 + j * kThreads < n && (key[j] & pmask) == prefix) rc.add(sh.hist, (key[j] >> shift) & 255u);
            }
            rc.flush(sh.hist);
            __syncthreads();
            find_digit(sh, krem, true);
            __syncthreads();
            prefix |= sh.bcast[0] << shift;
            pmask |= 255u << shift;
            krem -= sh.bcast[1];
            ties = sh.bcast[2];
            __syncthreads();
        }
        tau = prefix;
        if (krem < ties) {
            // keep the krem lowest positions among the ties: krem-th smallest position
            uint32_t pp = 0, pm = 0;
            for (int shift = 24; shift >= 0; shift -= 8) {
                if (tid < 256) sh.hist[tid] = 0;
                __syncthreads();
                RunCounter rc;
                for (int i = tid; i < n; i += kThreads) {
                    if (float_key(ub[i]) != tau) continue;
                    const uint32_t ps = (uint32_t)pb[i];
                    if ((ps & pm) == pp) rc.add(sh.hist, (ps >> shift) & 255u);
                }
                rc.flush(sh.hist);
                __syncthreads();
                find_digit(sh, krem, false);
                __syncthreads();
                pp |= sh.bcast[0] << shift;
                pm |= 255u << shift;
                krem -= sh.bcast[1];
                __syncthreads();
            }
            pi = (int)pp;
        }
    }

    auto keep_of = [&](int i) -> bool {
        switch (mode) {
            case 0: return true;
            case 1: return i != winner;
            default: {
                const uint32_t key = float_key(ub[i]);
                return key > tau || (key == tau && pb[i] <= pi);
            }
        }
    };

    if (a.keep_out) {
        uint8_t* ko = a.keep_out + (size_t)b * a.cap;
        for (int i0 = tid; i0 < n; i0 += kThreads * kBatch) {
            bool kp[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) kp[j] = i0 + j * kThreads < n && keep_of(i0 + j * kThreads);
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                if (i0 + j * kThreads < n) ko[i0 + j * kThreads] = kp[j] ? 1 : 0;
        }
    }

    if (!a.pair_dst) return;  // the decision alone is wanted
    int32_t* pdst = a.pair_dst + (size_t)b * a.max_pairs;
    int32_t* psrc = a.pair_src + (size_t)b * a.max_pairs;
    if (mode == 0) {
        if (tid == 0) a.npairs[b] = 0;
        return;
    }
    if (mode == 1) {
        if (tid == 0) {
            // k = n - 1: the only slot >= k is n - 1
            int np = 0;
            if (winner != n - 1 && a.max_pairs > 0) {
                pdst[0] = winner;
                psrc[0] = n - 1;
                np = 1;
            }
            a.npairs[b] = np;
        }
        return;
    }

    // Plan: the ascending holes (dropped slots < k) pair with the ascending tails (kept slots >= k).  The slots
    // are cut into segments of kSegGroups x 64; wave w takes segments w, w + kWaves, ...  A first sweep counts
    // each segment's holes and tails, a scan over the segments gives their offsets, and a second sweep writes
    // every hole and tail at its rank (segment offset + earlier groups of the segment + ballot prefix).  The
    // sweeps have no barrier inside, so the loads of u and pos stay in flight.
    const int groups = (n + kWave - 1) / kWave;
    // 64-slot groups per segment: at least one batch of loads, and at most kMaxSegs segments
    const int seg_groups = max(kPlanBatch, (groups + kMaxSegs - 1) / kMaxSegs);
    const int nseg = (groups + seg_groups - 1) / seg_groups;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    // keep decisions of kBatch consecutive 64-slot groups from g0 (loads issued together)
    auto keep_batch = [&](int g0, int g1, bool (&kp)[kPlanBatch]) {
#pragma unroll
        for (int j = 0; j < kPlanBatch; ++j) {
            const int i = (g0 + j) * kWave + lane;
            kp[j] = g0 + j < g1 && i < n && keep_of(i);
        }
    };
    for (int sg = wave; sg < nseg; sg += kWaves) {
        unsigned ch = 0, ct = 0;
        const int g1 = min(groups, (sg + 1) * seg_groups);
        for (int g0 = sg * seg_groups; g0 < g1; g0 += kPlanBatch) {
            bool kp[kPlanBatch];
            keep_batch(g0, g1, kp);
#pragma unroll
            for (int j = 0; j < kPlanBatch; ++j) {
                const int i = (g0 + j) * kWave + lane;
                const bool in = g0 + j < g1 && i < n;
                ch += __popcll(__ballot(in && i < k && !kp[j]));
                ct += __popcll(__ballot(in && i >= k && kp[j]));
            }
        }
        if (lane == 0) {
            sh.seg[sg][0] = ch;
            sh.seg[sg][1] = ct;
        }
    }
    __syncthreads();
    // exclusive scan of the segment counts (wave 0; kMaxSegs / 64 entries per lane)
    if (wave == 0) {
        constexpr int kPer = kMaxSegs / kWave;
        unsigned h[kPer], t[kPer], sh_ = 0, st = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int sg = lane * kPer + j;
            h[j] = sg < nseg ? sh.seg[sg][0] : 0u;
            t[j] = sg < nseg ? sh.seg[sg][1] : 0u;
            sh_ += h[j];
            st += t[j];
        }
        unsigned ih = sh_, it = st;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const unsigned xh = __shfl_up(ih, o, kWave), xt = __shfl_up(it, o, kWave);
            if (lane >= o) {
                ih += xh;
                it += xt;
            }
        }
        unsigned oh = ih - sh_, ot = it - st;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int sg = lane * kPer + j;
            if (sg < nseg) {
                sh.seg[sg][0] = oh;
                sh.seg[sg][1] = ot;
            }
            oh += h[j];
            ot += t[j];
        }
        if (lane == kWave - 1) {
            sh.bcast[0] = ih;  // totals
            sh.bcast[1] = it;
        }
    }
    __syncthreads();
    for (int sg = wave; sg < nseg; sg += kWaves) {
        unsigned oh = sh.seg[sg][0], ot = sh.seg[sg][1];
        const int g1 = min(groups, (sg + 1) * seg_groups);
        for (int g0 = sg * seg_groups; g0 < g1; g0 += kPlanBatch) {
            bool kp[kPlanBatch];
            keep_batch(g0, g1, kp);
#pragma unroll
            for (int j = 0; j < kPlanBatch; ++j) {
                const int i = (g0 + j) * kWave + lane;
                const bool in = g0 + j < g1 && i < n;
                const bool hole = in && i < k && !kp[j];
                const bool tail = in && i >= k && kp[j];
                const uint64_t mh = __ballot(hole), mt = __ballot(tail);
                if (hole) {
                    const unsigned r = oh + __popcll(mh & below);
                    if (r < (unsigned)a.max_pairs) pdst[r] = i;
                }
                if (tail) {
                    const unsigned r = ot + __popcll(mt & below);
                    if (r < (unsigned)a.max_pairs) psrc[r] = i;
                }
                oh += __popcll(mh);
                ot += __popcll(mt);
            }
        }
    }
    if (tid == 0) {
        const unsigned np = min(sh.bcast[0], sh.bcast[1]);
        a.npairs[b] = (int)min(np, (unsigned)a.max_pairs);
    }
}

// ---- Plan of a given decision ---------------------------------------------------------------------------
// The pairs of a retention mask (kv_compact): the ascending holes (dropped slots < k) and the ascending tails (kept
// slots >= k), each at its rank.  Slots [0, k) and [k, n) are cut into slices of kPlanSlice, one workgroup each; a
// workgroup counts what its region holds before its slice itself (the mask's bytes, four to a load, at most 128 KB
// for a 131,073-token sequence), so one launch without any exchange does.  Workgroup 0 of a sequence counts both
// regions for the pair count.  One workgroup per sequence that swept the mask twice, byte by byte, left kv_compact of
// small rows at 30 us for 8 sequences of 32,769 slots and 85 for 2 of 131,073; now 12.7 and 14.6.
constexpr int kPlanSlice = 4096;

// Nonzero bytes of m[s, e), s <= e, over the workgroup (every thread gets the count; two barriers).
__device__ unsigned count_kept(const uint8_t* m, int s, int e, unsigned* red) {
    const int tid = threadIdx.x;
    const uintptr_t at = reinterpret_cast<uintptr_t>(m + s);
    const int head = min(e - s, (int)((4 - at % 4) % 4));  // bytes before the first whole word
    const int words = (e - s - head) / 4;
    const uint32_t* w = reinterpret_cast<const uint32_t*>(m + s + head);
    unsigned c = 0;
    auto kept = [](uint32_t x) { return (unsigned)__popc((((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) & 0x80808080u); };
    for (int i0 = tid; i0 < words; i0 += kThreads * kBatch) {
        uint32_t x[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) x[j] = i0 + j * kThreads < words ? w[i0 + j * kThreads] : 0u;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) c += kept(x[j]);
    }
    const int rest = e - s - head - words * 4;  // bytes after the last whole word
    if (tid < head) c += m[s + tid] != 0;
    if (tid < rest) c += m[e - 1 - tid] != 0;
#pragma unroll
    for (int o = kWave / 2; o >= 1; o >>= 1) c += __shfl_xor(c, o, kWave);
    if (tid % kWave == 0) red[tid / kWave] = c;
    __syncthreads();
    unsigned t = 0;
#pragma unroll
    for (int j = 0; j < kWaves; ++j) t += red[j];
    __syncthreads();
    return t;
}

__global__ __launch_bounds__(kThreads) void plan_kernel(SelectArgs a, int hole_slices) {
    __shared__ unsigned red[kWaves];
    constexpr int kGroups = kPlanSlice / kThreads;  // 64-slot groups per wave
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int n = a.n, k = min(a.budget, n);
    const uint8_t* m = a.keep_in + (size_t)b * a.cap;
    const bool tails = (int)blockIdx.x >= hole_slices;
    const int first = tails ? k : 0, end = tails ? n : k;
    const int lo = first + ((int)blockIdx.x - (tails ? hole_slices : 0)) * kPlanSlice, hi = min(end, lo + kPlanSlice);
    // this wave's slots, loaded before the counts
    const int base = lo + wave * kGroups * kWave;
    bool mine[kGroups];  // a hole, or a tail
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        const int i = base + g * kWave + lane;
        mine[g] = i < hi && (m[i] != 0) == tails;
    }
    unsigned before = count_kept(m, first, lo, red);
    if (!tails) before = (unsigned)(lo - first) - before;
    uint64_t mask[kGroups];
    unsigned c = 0;
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        mask[g] = __ballot(mine[g]);
        c += __popcll(mask[g]);
    }
    if (lane == 0) red[wave] = c;
    __syncthreads();
    for (int w = 0; w < wave; ++w) before += red[w];
    int32_t* out = (tails ? a.pair_src : a.pair_dst) + (size_t)b * a.max_pairs;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        const unsigned r = before + __popcll(mask[g] & below);
        if (mine[g] && r < (unsigned)a.max_pairs) out[r] = base + g * kWave + lane;
        before += __popcll(mask[g]);
    }
    if (blockIdx.x != 0) return;
    __syncthreads();
    const unsigned holes = (unsigned)k - count_kept(m, 0, k, red);
    const unsigned kept = count_kept(m, k, n, red);
    if (tid == 0) a.npairs[b] = (int)min(min(holes, kept), (unsigned)a.max_pairs);
}

// ---- Multi-workgroup selection: long sequences in a small batch ------------------------------------------
// One workgroup per sequence leaves most of the chip idle when the batch is small and the sequences long (the
// selection of a 128k-token first step at batch 2 took ~0.3 ms).  In the threshold case (n > B + 1) the same
// radix select then runs as a short sequence of launches over P slices of every sequence:
//   4 x per-slice 256-bin histograms of the digit under the prefix found so far.  Each workgroup first takes the
//   previous digit itself, from the bins that the previous launch left for every slice (two sets of bins, written
//   in turn): a launch of its own for that, one workgroup per sequence, took as long as the histograms;
//   one launch for the last digit and for ties at tau (the position select of the single-workgroup kernel; it is
//   skipped unless more tokens tie at tau than are kept),
//   per-slice hole and tail counts and the decision, when asked for, then (when the pairs are wanted) the pairs:
//   every slice writes its holes and tails at the ranks that follow the slices before it.
// kv_topk_select, which wants no pairs, back to back: 8 sequences of 32,769 tokens 35 -> 22 us, 2 of 131,073 51 -> 30.
// The decisions and pairs are those of the single-workgroup kernel.  Scratch: P x 256 bins twice (the second set in
// the first pair list, which is written last: n >= 1,024 P slots) and P x 2 counts per sequence, and a few state
// words.
__device__ __forceinline__ unsigned wave_sum_u(unsigned x) {
#pragma unroll
    for (int o = kWave / 2; o >= 1; o >>= 1) x += __shfl_xor(x, o, kWave);
    return x;
}

constexpr int kWideThreads = 512;
constexpr int kWideMaxParts = 128;
constexpr int kWideMinRows = 16384;  // shorter sequences keep the single-workgroup kernel
constexpr int kWideSlice = 1024;     // fewest slots per slice
constexpr int kStateWords = 8;

int wide_parts_max(int batch) {
    const int p = 512 / batch;
    return p < 4 ? 0 : (p > kWideMaxParts ? kWideMaxParts : p);
}

int wide_parts(int batch, int n) {
    if (n < kWideMinRows) return 0;
    int p = wide_parts_max(batch);
    if (p > n / kWideSlice) p = n / kWideSlice;
    return p < 4 ? 0 : p;
}

// Selection state of a sequence before a digit is taken: the digits found so far, the rank wanted among the keys
// that have them, and how many keys have them.  Word 6 of the state: the position bound among ties.
struct WideState {
    uint32_t prefix;
    unsigned krem, ties;
};

struct Wide {
    unsigned* hist[2];  // [batch][P][256] each; hist[1] in rows of hist1_stride words per sequence
    size_t hist1_stride;
    unsigned* cnt;      // [batch][P][2]
    unsigned* st;       // [batch][kStateWords]: two WideStates in turn, the position bound
    int P, slice;
    __device__ int lo(int p) const { return p * slice; }
    __device__ unsigned* bins(int pass, int b) const {
        return pass % 2 ? hist[1] + (size_t)b * hist1_stride : hist[0] + (size_t)b * P * 256;
    }
    __device__ WideState* state(int pass, int b) const {  // before digit `pass` (0: the leading one) is taken
        return reinterpret_cast<WideState*>(st + (size_t)b * kStateWords) + pass % 2;
    }
};

Wide wide_of(const SelectArgs& a, int P) {
    Wide w;
    const size_t pm = (size_t)wide_parts_max(a.batch);
    w.hist[0] = a.wide;
    w.hist[1] = a.wide_bins;
    w.hist1_stride = (size_t)a.max_pairs;
    w.cnt = a.wide + (size_t)a.batch * pm * 256;
    w.st = w.cnt + (size_t)a.batch * pm * 2;
    w.P = P;
    w.slice = ((a.n + P - 1) / P + kWave - 1) / kWave * kWave;
    return w;
}

// The state after digit `pass` from the bins every slice left for it (every thread gets it; all kN threads call).
template <int kN>
__device__ WideState wide_digit(SelShared& sh, const SelectArgs& a, const Wide& w, int b, int pass) {
    const int tid = threadIdx.x, bin = tid % 256;
    constexpr int kParts = kN / 256, kAhead = 16;
    const WideState old = pass == 0 ? WideState{0u, (unsigned)a.budget, 0u} : *w.state(pass, b);
    const unsigned* hb = w.bins(pass, b) + bin;
    unsigned c = 0;
    for (int p0 = tid / 256; p0 < w.P; p0 += kParts * kAhead) {
        unsigned x[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) x[j] = p0 + j * kParts < w.P ? hb[(size_t)(p0 + j * kParts) * 256] : 0u;
#pragma unroll
        for (int j = 0; j < kAhead; ++j) c += x[j];
    }
    if (tid < 256) sh.hist[tid] = 0;
    __syncthreads();
    atomicAdd(&sh.hist[bin], c);
    __syncthreads();
    find_digit(sh, old.krem, true);
    __syncthreads();
    return WideState{old.prefix | (sh.bcast[0] << (24 - 8 * pass)), old.krem - sh.bcast[1], sh.bcast[2]};
}

__global__ __launch_bounds__(kWideThreads) void wide_hist_kernel(SelectArgs a, Wide w, int pass) {
    __shared__ SelShared sh;
    __shared__ unsigned hist[256];
    const int p = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int shift = 24 - 8 * pass;
    const float* ub = a.u + (size_t)b * a.cap;
    const int lo = w.lo(p), hi = min(a.n, lo + w.slice);
    if (tid < 256) hist[tid] = 0;
    uint32_t prefix = 0;
    if (pass > 0) {
        const WideState st = wide_digit<kWideThreads>(sh, a, w, b, pass - 1);
        prefix = st.prefix;
        if (p == 0 && tid == 0) *w.state(pass, b) = st;  // (the slices read state(pass - 1))
    }
    const uint32_t pmask = pass == 0 ? 0u : 0xffffffffu << (shift + 8);
    __syncthreads();
    RunCounter rc;
    for (int i0 = lo + tid; i0 < hi; i0 += kWideThreads * kBatch) {
        uint32_t key[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int i = i0 + j * kWideThreads;
            key[j] = i < hi ? float_key(ub[i]) : 0u;
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            if (i0 + j * kWideThreads < hi && (key[j] & pmask) == prefix) rc.add(hist, (key[j] >> shift) & 255u);
    }
    rc.flush(hist);
    __syncthreads();
    if (tid < 256) w.bins(pass, b)[(size_t)p * 256 + tid] = hist[tid];
}

// The last digit, and ties at tau: the krem lowest positions among them are kept (position radix select, one
// workgroup).
__global__ __launch_bounds__(kThreads) void wide_ties_kernel(SelectArgs a, Wide w) {
    __shared__ SelShared sh;
    const int b = blockIdx.x, tid = threadIdx.x;
    unsigned* st = w.st + (size_t)b * kStateWords;
    const WideState last = wide_digit<kThreads>(sh, a, w, b, 3);
    const uint32_t tau = last.prefix;
    unsigned krem = last.krem;
    if (tid == 0) *w.state(4, b) = last;
    if (krem >= last.ties) {
        if (tid == 0) st[6] = 0x7fffffffu;
        return;
    }
    __syncthreads();
    const float* ub = a.u + (size_t)b * a.cap;
    const int32_t* pb = a.pos + (size_t)b * a.cap;
    uint32_t pp = 0, pm = 0;
    for (int shift = 24; shift >= 0; shift -= 8) {
        if (tid < 256) sh.hist[tid] = 0;
        __syncthreads();
        RunCounter rc;
        for (int i = tid; i < a.n; i += kThreads) {
            if (float_key(ub[i]) != tau) continue;
            const uint32_t ps = (uint32_t)pb[i];
            if ((ps & pm) == pp) rc.add(sh.hist, (ps >> shift) & 255u);
        }
        rc.flush(sh.hist);
        __syncthreads();
        find_digit(sh, krem, false);
        __syncthreads();
        pp |= sh.bcast[0] << shift;
        pm |= 255u << shift;
        krem -= sh.bcast[1];
        __syncthreads();
    }
    if (tid == 0) st[6] = pp;
}

__device__ __forceinline__ bool wide_keep(const SelectArgs& a, const Wide& w, int b, int i) {
    const uint32_t tau = w.state(4, b)->prefix;
    const int bound = (int)w.st[(size_t)b * kStateWords + 6];
    const uint32_t key = float_key(a.u[(size_t)b * a.cap + i]);
    return key > tau || (key == tau && a.pos[(size_t)b * a.cap + i] <= bound);
}

// Per slice: holes (dropped slots < k) and tails (kept slots >= k), and the decision when asked for.
__global__ __launch_bounds__(kWideThreads) void wide_count_kernel(SelectArgs a, Wide w) {
    __shared__ unsigned part[kWideThreads / kWave][2];
    const int p = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int k = min(a.budget, a.n);
    const int lo = w.lo(p), hi = min(a.n, lo + w.slice);
    unsigned ch = 0, ct = 0;
    for (int i = lo + tid; i < hi; i += kWideThreads) {
        const bool kp = wide_keep(a, w, b, i);
        if (a.keep_out) a.keep_out[(size_t)b * a.cap + i] = kp ? 1 : 0;
        ch += i < k && !kp;
        ct += i >= k && kp;
    }
    ch = wave_sum_u(ch);
    ct = wave_sum_u(ct);
    if (tid % kWave == 0) {
        part[tid / kWave][0] = ch;
        part[tid / kWave][1] = ct;
    }
    __syncthreads();
    if (tid == 0) {
        unsigned h = 0, t = 0;
        for (int j = 0; j < kWideThreads / kWave; ++j) {
            h += part[j][0];
            t += part[j][1];
        }
        w.cnt[((size_t)b * w.P + p) * 2] = h;
        w.cnt[((size_t)b * w.P + p) * 2 + 1] = t;
    }
}

// Pairs: wave j of a slice takes its j-th eighth (whole 64-slot groups) and writes its holes and tails at the
// ranks after the earlier slices and eighths; the last slice records the pair count.
__global__ __launch_bounds__(kWideThreads) void wide_plan_kernel(SelectArgs a, Wide w) {
    constexpr int kW = kWideThreads / kWave;
    __shared__ unsigned base[2], wc[kW][2];
    const int p = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int k = min(a.budget, a.n);
    const int lo = w.lo(p), hi = min(a.n, lo + w.slice);
    if (wave == 0) {  // holes and tails of the slices before this one (P <= 128: two per lane)
        unsigned h = 0, t = 0;
        for (int q = lane; q < p; q += kWave) {
            h += w.cnt[((size_t)b * w.P + q) * 2];
            t += w.cnt[((size_t)b * w.P + q) * 2 + 1];
        }
        h = wave_sum_u(h);
        t = wave_sum_u(t);
        if (lane == 0) {
            base[0] = h;
            base[1] = t;
        }
    }
    const int groups = hi > lo ? (hi - lo + kWave - 1) / kWave : 0;
    const int per = (groups + kW - 1) / kW;
    const int g0 = wave * per, g1 = min(groups, g0 + per);
    unsigned ch = 0, ct = 0;
    for (int g = g0; g < g1; ++g) {
        const int i = lo + g * kWave + lane;
        const bool in = i < hi;
        const bool kp = in && wide_keep(a, w, b, i);
        ch += __popcll(__ballot(in && i < k && !kp));
        ct += __popcll(__ballot(in && i >= k && kp));
    }
    if (lane == 0) {
        wc[wave][0] = ch;
        wc[wave][1] = ct;
    }
    __syncthreads();
    unsigned oh = base[0], ot = base[1];
    for (int j = 0; j < wave; ++j) {
        oh += wc[j][0];
        ot += wc[j][1];
    }
    int32_t* pdst = a.pair_dst + (size_t)b * a.max_pairs;
    int32_t* psrc = a.pair_src + (size_t)b * a.max_pairs;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    for (int g = g0; g < g1; ++g) {
        const int i = lo + g * kWave + lane;
        const bool in = i < hi;
        const bool kp = in && wide_keep(a, w, b, i);
        const bool hole = in && i < k && !kp;
        const bool tail = in && i >= k && kp;
        const uint64_t mh = __ballot(hole), mt = __ballot(tail);
        if (hole) {
            const unsigned r = oh + __popcll(mh & below);
            if (r < (unsigned)a.max_pairs) pdst[r] = i;
        }
        if (tail) {
            const unsigned r = ot + __popcll(mt & below);
            if (r < (unsigned)a.max_pairs) psrc[r] = i;
        }
        oh += __popcll(mh);
        ot += __popcll(mt);
    }
    if (p == w.P - 1 && tid == 0) {
        unsigned h = base[0], t = base[1];
        for (int j = 0; j < kW; ++j) {
            h += wc[j][0];
            t += wc[j][1];
        }
        a.npairs[b] = (int)min(min(h, t), (unsigned)a.max_pairs);
    }
}

}  // namespace

size_t select_wide_words(int batch) {
    const size_t pm = (size_t)wide_parts_max(batch);
    return pm ? (size_t)batch * (pm * 258 + kStateWords) : 0;
}

hipError_t launch_plan(const SelectArgs& a, hipStream_t s) {
    const int k = a.budget < a.n ? a.budget : a.n;
    const int hole_slices = (k + kPlanSlice - 1) / kPlanSlice, tail_slices = (a.n - k + kPlanSlice - 1) / kPlanSlice;
    if (a.batch > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(plan_kernel, dim3(hole_slices + tail_slices, a.batch), dim3(kThreads), 0, s, a, hole_slices);
    return hipGetLastError();
}

hipError_t launch_select(const SelectArgs& a, hipStream_t s) {
    const int P = a.wide ? wide_parts(a.batch, a.n) : 0;
    if (a.n <= a.budget + 1 || P == 0) {
        hipLaunchKernelGGL(select_kernel, dim3(a.batch), dim3(kThreads), 0, s, a);
        return hipGetLastError();
    }
    const Wide w = wide_of(a, P);
    const dim3 sliced(P, a.batch);
    for (int pass = 0; pass < 4; ++pass)
        hipLaunchKernelGGL(wide_hist_kernel, sliced, dim3(kWideThreads), 0, s, a, w, pass);
    hipLaunchKernelGGL(wide_ties_kernel, dim3(a.batch), dim3(kThreads), 0, s, a, w);
    hipLaunchKernelGGL(wide_count_kernel, sliced, dim3(kWideThreads), 0, s, a, w);
    if (a.pair_dst) hipLaunchKernelGGL(wide_plan_kernel, sliced, dim3(kWideThreads), 0, s, a, w);
    return hipGetLastError();
}

}  // namespace ikv
