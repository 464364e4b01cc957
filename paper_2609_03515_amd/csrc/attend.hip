// Decode attention fused with the eviction score (Eq. 1) for gfx950.
//
// At every layer a decoder attends its last query over the cached rows; the method's per-step score is the
// same softmax, mean-pooled over query heads.  Computing both in one kernel lets a single pass over K serve
// the attention output and the score (the separate score pass is the dominant per-step cost of the method in
// the paper's profiling), and V is read once for the output.
//
// One workgroup per (layer, sequence, KV head, row chunk):
//   1. K pass: logits of the chunk's rows for the group's heads into LDS (the scorer's lane machinery and
//      dynamic unit claiming), running per-head max;
//   2. e = exp(z - max) in place with per-head sums (with the score: a pass of its own; without: by the wave
//      that claims a block in the V pass), then the V pass: on the matrix cores for bf16 rows of d = 128 and padded
//      groups of 4 to 16 (VUnit); else every lane accumulates e_h(row) * v(row) for the GP heads over its 16-byte
//      V chunks, the probabilities of a row being GP consecutive LDS words;
//   3. cross-lane (vector form) and cross-wave reduction in a fixed order, then either the normalised output (one
//      chunk per slab) or the chunk's unnormalised partial output with its per-head (max, sum);
//   4. when the score is wanted: the group probability sums r of the rows (one chunk), or the chunk's
//      exponentials (several chunks), which a combine kernel turns into outputs and scores.
// Chunks exist so that one layer's slabs (batch x KV heads, e.g. 64) still occupy all 256 CUs.
#include "stream_lane.h"

namespace ikv {
namespace {

#ifndef IKV_ATTN_TARGET
#define IKV_ATTN_TARGET 256
#endif
#ifndef IKV_ATTN_NBUF
#define IKV_ATTN_NBUF 0
#endif
#ifndef IKV_ATTN_MIN_ROWS
#define IKV_ATTN_MIN_ROWS 256
#endif
// workgroups per launch wanted: one per CU.  Measured for one decoder layer at batch 8 (64 slabs): 256 chunks
// beat 512 by 8%; counts that are not a multiple of the CU count (320, 384) leave CUs unevenly loaded.
constexpr int kAttnTargetWgs = IKV_ATTN_TARGET;
constexpr int kAttnMinRows = IKV_ATTN_MIN_ROWS;   // smallest chunk: below it a chunk's fixed costs dominate

template <int GP>
__device__ __forceinline__ void read_probs(const float* src, float (&e)[GP]) {
    if constexpr (GP >= 4) {
#pragma unroll
        for (int i = 0; i < GP; i += 4) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(src + i);
            e[i] = v.x;
            e[i + 1] = v.y;
            e[i + 2] = v.z;
            e[i + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < GP; ++i) e[i] = src[i];
    }
}

// Several chunks per slab: a combine kernel after the chunks' launch, as many workgroups.  With
//   f_h(c) = exp(m_c - M_h) / S_h,  M_h = max_c m_c,  S_h = sum_c exp(m_c - M_h) S_c
// the slab's first workgroup adds the outputs, o_h = sum_c f_h(c) o_c (upper half of its threads), and, when emitting,
// every workgroup takes the scores of its chunk's rows (lower half), r(row) = sum_{h in group} f_h(c) e_h(row), from
// the exponentials e_h = exp(z_h - m_c) that the chunk wrote.
// The kernel moves little and is bound by its chain of memory latencies, so every thread issues all of its loads
// (partial outputs of up to kAhead chunks, or the GP exponentials of its four rows) before the statistics are
// taken, and those are one load per (head, chunk) and a reduction over the lanes of a row.  It had taken the chunks'
// pairs, then the outputs and the heads' rows in turn, one latency each.  The workgroups are numbered like the
// chunks', so that a chunk's exponentials are read by the XCD whose L2 wrote them:
// 28 layer calls of 32 sequences x 4 KV heads x 2,049 rows (7 heads each, 2 chunks) 884 -> 818 us, 32 of 8 x 8 x 3,278
// (4 heads, 4 chunks) 793 -> 782, against rows in parts of 2,048 and a workgroup of their own for the outputs
// (short chunks in parts of 1,024 rows: one sequence of the latter shape, 13 chunks, 427 against 413).
// Electing the last chunk of a slab inside the attention kernel instead was measured twice at the 8B shape:
// with a device-scope release/acquire fence in every chunk (a full L2 write-back and invalidate) 5x slower per
// layer; with the partials written and read back by device-scope (write-through) accesses and a completion
// wait before the arrival count, no faster without the score (the chunk's store, count and reload round trips
// cost what the kernel boundary does) and 9% slower with it (one workgroup per slab takes the score's rows).
constexpr int kCombineThreads = 512;
constexpr int kCombineHalf = kCombineThreads / 2;
// workgroups per slab: one per chunk, or one without scores
__host__ __device__ constexpr int combine_parts(int nchunk, bool emit) { return emit ? nchunk : 1; }

// Slab and chunk of workgroup `block` of `slabs` x `chunks`: the chunks of a slab are eight workgroups apart, so that
// the XCDs, which take workgroups in turn, each hold whole slabs (a last group of fewer than eight slabs: in order).
struct SlabChunk {
    int s, c;
};
__device__ __forceinline__ SlabChunk slab_chunk(int block, int slabs, int chunks) {
    constexpr int kXcds = 8;
    const int full = slabs / kXcds * kXcds * chunks;
    if (block >= full) return {block / chunks, block % chunks};
    const int r = block % (kXcds * chunks);
    return {block / (kXcds * chunks) * kXcds + r % kXcds, r / kXcds};
}

template <typename T, int D, int GP, int kAhead>
__global__ __launch_bounds__(kCombineThreads) void attend_combine_kernel(ScoreArgs a) {
    __shared__ float fs[GP * kWave];
    __shared__ float cm[GP], ci[GP];  // more chunks than are staged: M_h and 1 / S_h
    const int tid = threadIdx.x, nchunk = a.nchunk, group = a.group;
    const SlabChunk sc = slab_chunk(blockIdx.x, a.layers * a.batch * a.hkv, combine_parts(nchunk, a.emit));
    const int s = sc.s, chunk = sc.c;  // slab: (l * batch + b) * hkv + g, l relative to the call
    const size_t head0 = (size_t)(s / a.hkv) * a.hq + (size_t)(s % a.hkv) * group;
    const float2* pp = a.part + head0 * nchunk;  // [head][chunk]
    const bool staged = nchunk <= kWave;

    // this thread's loads: four rows of every head, or four outputs of one head over the first chunks
    const bool outputs = tid >= kCombineHalf;
    const int row_end = min(a.n, (chunk + 1) * a.chunk_rows);  // (rows up to the padded stride are scratch)
    int row = chunk * a.chunk_rows + (outputs ? 0 : tid) * 4;
    constexpr int kQuads = D / 4;
    int quad = tid - kCombineHalf;
    const int quad_end = chunk == 0 ? group * kQuads : 0;
    auto out_of = [&](int q, int c) __attribute__((always_inline)) {
        return *reinterpret_cast<const f32x4*>(a.opart + ((head0 + q / kQuads) * nchunk + c) * D + q % kQuads * 4);
    };
    f32x4 x[GP > kAhead ? GP : kAhead];
    auto load_outputs = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < kAhead; ++c)
            if (c0 + c < nchunk) x[c] = out_of(quad, c0 + c);
    };
    auto load_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < GP; ++h)
            if (h < group) x[h] = *reinterpret_cast<const f32x4*>(a.z + (head0 + h) * a.n_stride + row);
    };
    if (outputs) {
        if (quad < quad_end) load_outputs(0);
    } else if (a.emit && row < row_end) {
        load_rows();
    }

    // one (head, chunk) pair per lane: a row of 16 lanes per head, or a wave; more chunks than that are taken from
    // memory again where needed.  (A chunk with an infinite logit has no factor: w is NaN, and stays it.)
    if (nchunk <= 16) {
        const int h = tid / 16, c = tid % 16;
        if (h < group) {
            const float2 p = c < nchunk ? pp[h * nchunk + c] : make_float2(-INFINITY, 0.0f);
            const float w = __expf(p.x - row_allmax(p.x));
            const float tot = group_allsum<16>(w * p.y);
            if (c < nchunk) fs[h * nchunk + c] = tot > 0.0f ? w / tot : w * 0.0f;
        }
    } else if (staged) {
        const int c = tid % kWave;
        for (int h = tid / kWave; h < group; h += kCombineThreads / kWave) {
            const float2 p = c < nchunk ? pp[h * nchunk + c] : make_float2(-INFINITY, 0.0f);
            const float w = __expf(p.x - wave_max(p.x));
            const float tot = wave_sum(w * p.y);
            if (c < nchunk) fs[h * nchunk + c] = tot > 0.0f ? w / tot : w * 0.0f;
        }
    } else if (tid < group) {
        const float2* ph = pp + (size_t)tid * nchunk;
        float mx = -INFINITY, tot = 0.0f;
        for (int c = 0; c < nchunk; ++c) mx = fmaxf(mx, ph[c].x);
        for (int c = 0; c < nchunk; ++c) tot = fmaf(__expf(ph[c].x - mx), ph[c].y, tot);
        cm[tid] = mx;
        ci[tid] = tot > 0.0f ? 1.0f / tot : 0.0f;
    }
    __syncthreads();
    auto factor = [&](int h, int c) __attribute__((always_inline)) {
        return staged ? fs[h * nchunk + c] : __expf(pp[(size_t)h * nchunk + c].x - cm[h]) * ci[h];
    };

    if (!outputs) {
        if (!a.emit) return;
        float f[GP];
#pragma unroll
        for (int h = 0; h < GP; ++h) f[h] = h < group ? factor(h, chunk) : 0.0f;
        for (bool first = true; row < row_end; row += kCombineHalf * 4, first = false) {
            if (!first) load_rows();
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int h = 0; h < GP; ++h)
                if (h < group) acc += x[h] * f[h];
            *reinterpret_cast<f32x4*>(a.r + (size_t)s * a.n_stride + row) = acc;
        }
        return;
    }
    if (a.emit_norms && chunk == 0 && tid / kWave == kCombineThreads / kWave - 1) {
        float tot = 0.0f;
        for (int c = tid % kWave; c < nchunk; c += kWave) tot += a.npart[(size_t)s * nchunk + c];
        tot = wave_sum(tot);
        if (tid % kWave == 0) a.vinv[s] = tot > 0.0f ? (float)a.n / tot : 0.0f;
    }
    T* ob = static_cast<T*>(a.o) + head0 * D;
    for (bool first = true; quad < quad_end; quad += kCombineHalf, first = false) {
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int c0 = 0; c0 < nchunk; c0 += kAhead) {
            if (!first || c0 != 0) load_outputs(c0);
#pragma unroll
            for (int c = 0; c < kAhead; ++c)
                if (c0 + c < nchunk) acc += x[c] * factor(quad / kQuads, c0 + c);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) Elem<T>::store(ob + quad * 4 + j, acc[j]);
    }
}

// Matrix-core V pass, for bf16 rows of d = 128 and padded groups of 4 to 16: the product of the group's
// probabilities with the rows' values, 16 rows at a time, as v_mfma_f32_16x16x16_bf16 with the rows as the
// contracted index.
//  * V: load j of a unit gives lane 16 g + p the 16 bytes p (columns 8 p .. 8 p + 7) of row 4 j + g, so one load
//    instruction reads 1 KiB of consecutive rows.  Element j of the contraction's slice g is taken to be row 4 j + g;
//    a column of the lane's four rows then needs only byte permutes of the lane's own registers, and MFMA x covers
//    the columns 8 p + x (p < 16), eight of them the whole row.
//  * probabilities: lane 16 g + h holds those of head h for the same rows.  They stay 32-bit numbers: each is the
//    sum of three bf16 parts (its upper 8 significant bits, the next 8, the last 8: exact), and each part takes an
//    MFMA of its own, whose products are exact and accumulated in fp32.
//  * the result of MFMA x in lane 16 g + p is heads 4 g .. 4 g + 3 of column 8 p + x: nothing is left to be added
//    across lanes.
// On the vector ALUs each lane held GP x 16 accumulators (8 heads), which a wave then added across its lanes with
// LDS-crossbar shuffles and the workgroup wave by wave: 64 us for one layer of 32 sequences x 4 KV heads x 2,049 rows
// (7 heads per KV head), 25 us so; with 4 heads (8 sequences x 8 KV heads x 3,278 rows) 0.3 us of 25 per layer
// call.  Units of 32 rows (16x16x32 MFMAs, two units in flight) left the waves further apart at the end of the
// pass: 882 against 871 us for 28 layer calls of the former shape; three or four units of 16 rows in flight 877 and
// 901.  Groups of 1 and 2 keep the vector form: its accumulators are few and most of an MFMA would be padding.
typedef short __attribute__((ext_vector_type(4))) s16x4;
typedef uint32_t __attribute__((ext_vector_type(2))) u32x2;

template <typename T, int D, int GP>
constexpr bool use_mfma_v() {
    return std::is_same<T, bf16_t>::value && D == 128 && GP >= 4;
}

struct VUnit {
    static constexpr int kRows = 16;
    static constexpr int kN = kRows / 4;  // rows per lane
    static constexpr int kRowBytes = 256;
    typedef u32x4 buf_t[kN];
    int g, p;
    __device__ VUnit() {
        const int lane = threadIdx.x & (kWave - 1);
        g = lane / 16;
        p = lane % 16;
    }
    __device__ int row(int u, int j) const { return u * kRows + 4 * j + g; }
    // LDS word of (row 4 j + g of the unit, head 0) from the unit's first: see KUnit for the layout of the blocks
    template <int GP>
    __device__ static int word(int g, int j) {
        return GP >= 8 ? (4 * j + g) * GP : j / 4 * kWave + g * 16 + j % 4 * 4;
    }
    __device__ void load(__amdgpu_buffer_rsrc_t vrs, int u, buf_t& dst) const {
        const int off = (u * kRows + g) * kRowBytes + p * 16;
#pragma unroll
        for (int j = 0; j < kN; ++j)
            dst[j] = __builtin_amdgcn_raw_buffer_load_b128(vrs, off + j * 4 * kRowBytes, 0,
                                                           IKV_NT_LOADS ? kNonTemporal : 0);
    }
    // halves of two registers as one: the low ones (even columns) or the high ones (odd columns, or the upper 16
    // bits of two floats)
    __device__ static uint32_t low2(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
    __device__ static uint32_t high2(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
    __device__ static f32x4 mfma(u32x2 a, u32x2 b, f32x4 acc) {
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b),
                                                         acc, 0, 0, 0);
    }
    // acc[x] += probabilities e (rows row(u, 0 .. kN - 1) of head p; zero for heads and rows that are none) times V
    __device__ static void add(const buf_t& v, float (&e)[kN], f32x4 (&acc)[8]) {
        u32x2 part[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
#pragma unroll
            for (int i = 0; i < kN / 2; ++i) part[k][i] = high2(__float_as_uint(e[2 * i]), __float_as_uint(e[2 * i + 1]));
            if (k < 2)
#pragma unroll
                for (int j = 0; j < kN; ++j) e[j] -= __uint_as_float(__float_as_uint(e[j]) & 0xffff0000u);
        }
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            u32x2 c;
#pragma unroll
            for (int i = 0; i < kN / 2; ++i)
                c[i] = x % 2 ? high2(v[2 * i][x / 2], v[2 * i + 1][x / 2]) : low2(v[2 * i][x / 2], v[2 * i + 1][x / 2]);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                acc[x] = mfma(part[k], c, acc[x]);
            }
        }
    }
};

// One lane's output t = sum e(row) v(row)[col0 + lane] over the rows [0, nrows) of bf16 values `vrs` (128 columns), where
// some t of the wave is not finite although no probability e(row) >= 0 is NaN: from the infinities and NaN among its
// values, with e v = NaN for e = 0.  Where there are none, the sum itself left the range and stays.  The wave reads its 64
// columns of every row, 8 rows to a load and kAhead loads in flight, and no probability but those it needs.  A layer call of
// 8 x 8 slabs of 3,278 rows (finite: 20.5 us) with a NaN query, NaN values or infinities in every value column of one
// sequence: 45, 45 and 43 us where each thread summed its output again row by row, now 20.3 (no sum is taken), 20.6 and 32.
template <class ProbF>
__device__ float nonfinite_column(__amdgpu_buffer_rsrc_t vrs, int col0, int nrows, float t, ProbF prob) {
    constexpr int kAhead = 8, kRowBytes = 256;
    const int lane = threadIdx.x & (kWave - 1);
    const int r = lane / 8, c = lane % 8;  // row of the load, chunk of eight columns
    uint32_t up = 0, down = 0, none = 0;   // columns of the chunk with a product +inf, -inf, or NaN
    for (int r0 = r; r0 - r < nrows && !__all(none == 0xffu); r0 += 8 * kAhead) {
        u32x4 x[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j)  // (rows past the last one read zeros)
            x[j] = __builtin_amdgcn_raw_buffer_load_b128(vrs, (r0 + 8 * j) * kRowBytes + col0 * 2 + c * 16, 0, 0);
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            // bit i: column i is not finite (the exponent of its half word is all ones) nor already known to give NaN
            uint32_t odd = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t m = ((x[j][i] & 0x7f807f80u) + 0x00800080u) & 0x80008000u;
                odd |= (m >> 15 | m >> 30) << 2 * i;
            }
            odd = odd & 0xffu & ~none;
            if (!odd) continue;
            const bool zero = prob(r0 + 8 * j) == 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t v = x[j][i / 2] >> (i % 2 * 16) & 0xffffu, bit = odd & 1u << i;
                if (zero || (v & 0x7fu))
                    none |= bit;
                else if (v & 0x8000u)
                    down |= bit;
                else
                    up |= bit;
            }
        }
    }
    uint32_t all = none | up << 8 | down << 16;
#pragma unroll
    for (int o = 8; o < kWave; o <<= 1) all |= __shfl_xor(all, o, kWave);
    all = __shfl(all, lane / 8, kWave) >> lane % 8;
    if ((all & 1u) || ((all & 0x100u) && (all & 0x10000u))) return NAN;
    return all & 0x100u ? INFINITY : all & 0x10000u ? -INFINITY : t;
}

// Waves per SIMD the compiler must leave room for: bf16 rows of d = 128 with groups of 4 (the 8B shape) are held
// to 128 registers, i.e. two workgroups per CU, which the all-layer call (2,048 workgroups) uses (99 are taken; a
// form that took 129 was 1% slower in that call).  Other instances keep what they need.
template <typename T, int D, int GP, bool kV>
constexpr int attend_waves_per_eu() {
    return (kV && GP == 4 && D == 128 && std::is_same<T, bf16_t>::value) ? 4 : 1;
}

// kV = false: score only (no V pass, no output), for scoring long slabs in chunks: the chunks write their
// logits and per-head (max, sum) for the scorer's finish kernel.
template <typename T, int D, int GP, bool kV>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(attend_waves_per_eu<T, D, GP, kV>())))
void attend_kernel(ScoreArgs a) {
    using L = Lane<T, D, GP>;
    using E = Elem<T>;
    using chunk_t = typename L::chunk_t;
    constexpr int RPG = L::RPG, CPL = L::CPL, RPW = L::RPW, LPR = L::LPR, EPC = L::EPC;
    // K/V loads of two units in flight, one when a lane's share of a unit is already large (a single head
    // per KV head: 16 rows per lane), which would otherwise spill
    constexpr int kNbuf = IKV_ATTN_NBUF > 0 ? IKV_ATTN_NBUF : (RPG * CPL > 8 ? 1 : 2);
    using KP = KUnit<T, D, GP>;
    constexpr int kNbufK = use_mfma<T, D, GP>() ? 2 : kNbuf;  // K units in flight (16 rows each on MFMA)

    // the waves' partial outputs are added in one step when every wave's slice fits 16 KiB of LDS (GP * D <= 512
    // floats: groups up to 4 at d = 128), else wave by wave (one barrier each); the sums are the same
    constexpr bool kMV = kV && use_mfma_v<T, D, GP>();
    constexpr bool kFirstV = kV && (kMV || kNbuf == 2);
    constexpr bool kWaveSlices = kWaves * GP * D <= 4096 && !kMV;
    // matrix-core form: at most 32 KiB of slices.  Beside more than 47 KiB of logits they leave a CU one workgroup, which
    // is enough: one call over 28 layers x 32 sequences x 4 KV heads (7 heads) streams K and V at 6.9 TB/s with 2,049 rows
    // (64 KiB of logits, one workgroup: 546 us, 587 with the score) and at 6.7 with 1,100 (35 KiB, two: 302 and 321).  The
    // vector form (190 registers, one workgroup) took 1,022, 1,045, 782 and 804.
    constexpr int kMVSlices = GP > 8 ? kWaves / 2 : kWaves;
    extern __shared__ float zs[];
    __shared__ float red_m[kWaves][GP], red_s[kWaves][GP], red_n[kWaves];
    __shared__ float obuf[kV ? (kMV ? kMVSlices : kWaveSlices ? kWaves : 1) * GP * D : 1];
    __shared__ int next_unit[2];

    const L ln;
    const KP kp;
    const SlabChunk sc = slab_chunk(blockIdx.x, a.layers * a.batch * a.hkv, a.nchunk);
    const int chunk = sc.c, s = sc.s;  // slab: (l * batch + b) * hkv + g, l relative to the call
    const int g = s % a.hkv;
    const int lb = s / a.hkv;
    const int b = lb % a.batch;
    const int row0 = chunk * a.chunk_rows;
    const int nrows = min(a.n - row0, a.chunk_rows);  // >= 1: the plan leaves no empty chunk
    const int nunits = (nrows + RPW - 1) / RPW;          // LDS blocks of logits (and V units)
    const int nku = (nrows + KP::kRows - 1) / KP::kRows;  // claimed units of the K pass
    const size_t base = ((size_t)s * a.cap + row0) * D;
    const __amdgpu_buffer_rsrc_t krs = raw_rsrc(static_cast<const T*>(a.k) + base, nrows * L::kRowBytes);
    const __amdgpu_buffer_rsrc_t vrs = raw_rsrc(static_cast<const T*>(a.v) + base, nrows * L::kRowBytes);
    const __amdgpu_buffer_rsrc_t prs = raw_rsrc(a.pos + (size_t)b * a.cap + row0, nrows * 4);

    // the first unit of a wave is its own index, in both passes: its loads wait for no claim and no barrier (the same
    // decode steps 812, 758 and 398 us with every unit claimed, 801, 744 and 387 so).  Without the V pass the form of
    // 8 f32 heads then takes 132 registers, one workgroup per CU: so 474 us for 8 slabs of 131,073 rows and 927 for 16,
    // with every unit claimed and both counters set by one thread (128 registers, two workgroups) 482 and 946.
    constexpr bool kFirstK = kNbufK == 2;
    typename KP::max_t mk = kp.max_init();
    typename KP::buf_t kbuf[kNbufK];
    int pbuf[kNbufK];
    if (kFirstK && ln.wave < nku) kp.load(krs, prs, ln.wave, kbuf[0], pbuf[0]);
    if (threadIdx.x < 2) next_unit[threadIdx.x] = threadIdx.x == 0 ? (kFirstK ? kWaves : 0) : (kFirstV ? kWaves : 0);
    typename KP::q_t qv;
    kp.load_q(a, (size_t)lb, g, qv);
    __syncthreads();
    auto claim = [&](int which) -> int {
        int u = 0;
        if (ln.lane == 0) u = atomicAdd(&next_unit[which], 1);
        return __builtin_amdgcn_readfirstlane(u);
    };

    // 1. K pass
    claimed_units<kNbufK>(
        nku, kFirstK ? ln.wave : -1, [&]() __attribute__((always_inline)) { return claim(0); },
        [&](auto slot, int u) __attribute__((always_inline)) { kp.load(krs, prs, u, kbuf[slot], pbuf[slot]); },
        [&](auto slot, int u) __attribute__((always_inline)) { kp.logits(a, kbuf[slot], qv, pbuf[slot], u, nrows, zs, mk); });

    // the V stream's first loads are issued now, so their latency overlaps the K pass's epilogue (barriers
    // wait for LDS only, not for these loads)
    chunk_t vbuf[kMV ? 1 : kNbuf][RPG][CPL];
    int vfirst = -1;
    const VUnit vu;
    constexpr int kNbufV = 2;
    int vnext[kNbufV];
    typename VUnit::buf_t vbufm[kMV ? kNbufV : 1];
    const int nvu = kMV ? (nrows + VUnit::kRows - 1) / VUnit::kRows : nunits;
    if constexpr (kMV) {
#pragma unroll
        for (int j = 0; j < kNbufV - 1; ++j) {
            vnext[j] = j == 0 ? ln.wave : claim(1);
            vu.load(vrs, vnext[j], vbufm[j]);
        }
    } else if constexpr (kV && kNbuf == 2) {
        vfirst = ln.wave;
        ln.load_rows(vrs, vfirst, vbuf[0]);
    }

    // per-head max, then the exponentials in place with their per-head sums: in a pass of their own when a score
    // is produced (several chunks: the logits go to HBM on the way, for the finish or combine kernel), else
    // inside the V pass (below)
    kp.publish_max(mk, red_m[ln.wave]);
    __syncthreads();
    float m = red_m[0][ln.hh];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m = fmaxf(m, red_m[w][ln.hh]);

    float* zl = zs + ln.wave * kWave + ln.lane;
    constexpr int kStep = kWaves * kWave;
    const int mine = nunits > ln.wave ? (nunits - ln.wave + kWaves - 1) / kWaves : 0;
    const bool write_z = !kV && a.emit && a.nchunk > 1;  // (with V, a chunk's exponentials are stored later)
    // this lane's head's logit row (lanes of one wave hold different heads: stored by address)
    float* zrow = a.z + ((size_t)lb * a.hq + (size_t)g * a.group + ln.hh) * a.n_stride + row0;
    float ssum = 0.0f;
    auto expo = [&](float z, int unit) {
        // -inf: padded head or row past the end
        if (write_z && z != -INFINITY) store_stream_at(zrow + ln.unit_row(unit), z);
        return z == -INFINITY ? 0.0f : __expf(z - m);
    };
    // Measured for one decoder layer per call (8B shape): exponentials inside the V pass save the pass and its
    // barrier (32 calls 790 -> 769 us without the score).  With the score, a slab cut in chunks then stores its
    // exponentials after the streams (stored during the V pass, with the logits, they had cost 842 -> 867 us);
    // one chunk per slab keeps the pass, whose sums are the scorer's bit for bit.
    const bool exp_apart = !kV || (a.emit && a.nchunk == 1);
    if (exp_apart) {
        int i = 0;
        for (; i + kEpi <= mine; i += kEpi) {
            float e[kEpi];
#pragma unroll
            for (int v = 0; v < kEpi; ++v) e[v] = zl[(i + v) * kStep];
#pragma unroll
            for (int v = 0; v < kEpi; ++v) {
                e[v] = expo(e[v], ln.wave + (i + v) * kWaves);
                ssum += e[v];
                if (kV) zl[(i + v) * kStep] = e[v];
            }
        }
        for (; i < mine; ++i) {
            const float e = expo(zl[i * kStep], ln.wave + i * kWaves);
            ssum += e;
            if (kV) zl[i * kStep] = e;
        }
#pragma unroll
        for (int o = GP; o < kWave; o <<= 1) ssum += __shfl_xor(ssum, o, kWave);
        if (ln.lane < GP) red_s[ln.wave][ln.lane] = ssum;
        __syncthreads();  // also publishes every exponential to the V pass
    }
    if constexpr (!kV) {
        if (threadIdx.x < a.group) {
            const size_t h = (size_t)lb * a.hq + (size_t)g * a.group + threadIdx.x;
            float mx = red_m[0][threadIdx.x], tot = red_s[0][threadIdx.x];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) {
                mx = fmaxf(mx, red_m[w][threadIdx.x]);
                tot += red_s[w][threadIdx.x];
            }
            a.part[h * a.nchunk + chunk] = make_float2(mx, tot);
        }
        return;
    } else {

    // 2. V pass: acc[h][c][x] = sum over this lane's rows of e_h(row) * v(row)[(p + c LPR) EPC + x]; with
    //    emit_norms also the rows' value norms (VNorm), written out and summed.  Without the score the wave
    //    that claims a block first turns its logits into exponentials in place (each lane the word it owns) and
    //    adds them to its sums; the block's probabilities are then read by the wave's own lanes, so no
    //    workgroup barrier separates the exponentials from the V stream.
    const __amdgpu_buffer_rsrc_t vns =
        raw_rsrc(a.vn + (size_t)s * a.n_stride + row0, a.emit_norms ? nrows * 4 : 0);
    float nsum = 0.0f;
    f32x4 accm[kMV ? 8 : 1];
    float acc[kMV ? 1 : GP][kMV ? 1 : CPL][EPC];
    if constexpr (kMV) {
#pragma unroll
        for (int x = 0; x < 8; ++x) accm[x] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        const int h = vu.p;  // the head whose probabilities this lane supplies (none past GP)
        float mh = 0.0f;
        if (h < GP) {
            mh = red_m[0][h];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) mh = fmaxf(mh, red_m[w][h]);
        }
        auto& ubuf = vnext;
        bool more = true;
        while (more) {
#pragma unroll
            for (int j = 0; j < kNbufV; ++j) {
                const int slot = (j + kNbufV - 1) % kNbufV;
                ubuf[slot] = claim(1);
                vu.load(vrs, ubuf[slot], vbufm[slot]);
                if (more && ubuf[j] < nvu) {
                    // all of the lane's words are read before any is used; rows past the chunk and padded lanes
                    // read word 0 and count as zero
                    float e[VUnit::kN];
                    int word[VUnit::kN];
                    bool in[VUnit::kN];
#pragma unroll
                    for (int r = 0; r < VUnit::kN; ++r) {
                        in[r] = h < GP && vu.row(ubuf[j], r) < nrows;
                        word[r] = in[r] ? ubuf[j] * VUnit::kRows * GP + VUnit::word<GP>(vu.g, r) + h : 0;
                        e[r] = zs[word[r]];
                    }
                    if (!exp_apart) {
#pragma unroll
                        for (int r = 0; r < VUnit::kN; ++r) {
                            e[r] = in[r] ? __expf(e[r] - mh) : 0.0f;
                            ssum += e[r];
                        }
                        if (a.emit)
#pragma unroll
                            for (int r = 0; r < VUnit::kN; ++r)
                                if (in[r]) zs[word[r]] = e[r];
                    } else {
#pragma unroll
                        for (int r = 0; r < VUnit::kN; ++r) e[r] = in[r] ? e[r] : 0.0f;
                    }
                    if (a.emit_norms) {  // VNorm: the rows' l2 norms, summed over the 16 lanes of a row
#pragma unroll
                        for (int r = 0; r < VUnit::kN; ++r) {
                            const chunk_t c[1] = {vbufm[j][r]};
                            const float nrm = row_norm_lanes<T, 16, 1>(c);
                            const int row = vu.row(ubuf[j], r);
                            if (vu.p == 0 && row < nrows) {
                                store_stream(vns, row * 4, nrm);
                                nsum += nrm;
                            }
                        }
                    }
                    VUnit::add(vbufm[j], e, accm);
                } else {
                    more = false;
                }
            }
        }
    } else {
#pragma unroll
        for (int h = 0; h < GP; ++h)
#pragma unroll
            for (int c = 0; c < CPL; ++c)
#pragma unroll
                for (int x = 0; x < EPC; ++x) acc[h][c][x] = 0.0f;
        int ubuf[kNbuf];
        if constexpr (kNbuf == 2) ubuf[0] = vfirst;
        bool more = true;
        while (more) {
#pragma unroll
            for (int j = 0; j < kNbuf; ++j) {
                const int slot = (j + kNbuf - 1) % kNbuf;
                ubuf[slot] = claim(1);
                ln.load_rows(vrs, ubuf[slot], vbuf[slot]);
                if (more && ubuf[j] < nunits) {
                    float* eb = zs + ubuf[j] * kWave;
                    if (!exp_apart) {
                        const float e = expo(eb[ln.lane], ubuf[j]);
                        ssum += e;
                        eb[ln.lane] = e;
                        __builtin_amdgcn_wave_barrier();  // (the reads below are of words other lanes just wrote)
                    }
                    // row k * NG + grp of the unit: its GP probabilities are words grp * LPR + k * GP + [0, GP)
                    const float* eu = eb + ln.grp * LPR;
#pragma unroll
                    for (int k = 0; k < RPG; ++k) {
                        float e[GP];
                        read_probs<GP>(eu + k * GP, e);
                        float ss = 0.0f;
#pragma unroll
                        for (int c = 0; c < CPL; ++c) {
                            float f[EPC];
                            E::unpack(vbuf[j][k][c], f);
#pragma unroll
                            for (int h = 0; h < GP; ++h)
#pragma unroll
                                for (int x = 0; x < EPC; ++x) acc[h][c][x] = fmaf(e[h], f[x], acc[h][c][x]);
#pragma unroll
                            for (int x = 0; x < EPC; ++x) ss = fmaf(f[x], f[x], ss);
                        }
                        if (a.emit_norms) {  // VNorm: the row's l2 norm, summed over its lane group
                            ss = group_allsum<LPR>(ss);
                            const int row = ubuf[j] * RPW + k * L::NG + ln.grp;
                            if (ln.p == 0 && row < nrows) {
                                const float nrm = sqrtf(ss);
                                store_stream(vns, row * 4, nrm);
                                nsum += nrm;
                            }
                        }
                    }
                } else {
                    more = false;
                }
            }
        }
    }

    if (a.emit_norms) {
#pragma unroll
        for (int o = kWave / 2; o >= 1; o >>= 1) nsum += __shfl_xor(nsum, o, kWave);
        if (ln.lane == 0) red_n[ln.wave] = nsum;  // read after the barriers below
    }
    if (!exp_apart) {  // the sums the waves took over the blocks they claimed
        if constexpr (!kMV)
#pragma unroll
            for (int o = GP; o < 16; o <<= 1) ssum += __shfl_xor(ssum, o, kWave);
        ssum = rows_allsum(ssum);
        if (ln.lane < GP) red_s[ln.wave][ln.lane] = ssum;  // read after the barriers below
    }

    // 3. vector form: lanes holding the same chunk of different rows (stride LPR), then the waves in order.  With 16
    //    lanes per row the four rows hold the same chunks: four accumulators at a time are reduced over the rows with
    //    row swaps, leaving accumulator 4i + r in row r (in the butterfly's order, so the sums are unchanged),
    //    and every lane stores its share of the wave's slice (64 cross-row shuffles of a butterfly had kept the LDS
    //    crossbar busy for ~1 us after the V pass).
    constexpr int kAcc = GP * CPL * EPC;
    constexpr bool kRowSwaps = kWaveSlices && LPR == 16 && kAcc % 4 == 0;
    if constexpr (!kRowSwaps && !kMV) {
#pragma unroll
        for (int o = LPR; o < kWave; o <<= 1)
#pragma unroll
            for (int h = 0; h < GP; ++h)
#pragma unroll
                for (int c = 0; c < CPL; ++c)
#pragma unroll
                    for (int x = 0; x < EPC; ++x) acc[h][c][x] += __shfl_xor(acc[h][c][x], o, kWave);
    }
    if constexpr (kMV) {
        // nothing to add across lanes: each wave's (or, for 16 heads, each pair of waves') partial in a slice of its
        // own, then the slices in order by the thread that later stores the output
        auto slice_of = [&](int i, int half) __attribute__((always_inline)) {
            return reinterpret_cast<f32x4*>(obuf + ln.wave % kMVSlices * GP * D + (4 * vu.g + i) * D + 8 * vu.p) + half;
        };
        if (ln.wave < kMVSlices && 4 * vu.g < GP)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int half = 0; half < 2; ++half)
                    *slice_of(i, half) = f32x4{accm[4 * half][i], accm[4 * half + 1][i], accm[4 * half + 2][i],
                                               accm[4 * half + 3][i]};
        __syncthreads();
        if constexpr (kMVSlices < kWaves) {
            if (ln.wave >= kMVSlices && 4 * vu.g < GP)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int half = 0; half < 2; ++half)
                        *slice_of(i, half) += f32x4{accm[4 * half][i], accm[4 * half + 1][i], accm[4 * half + 2][i],
                                                    accm[4 * half + 3][i]};
            __syncthreads();
        }
        for (int idx = threadIdx.x; idx < a.group * D; idx += kThreads) {
            float t = obuf[idx];
#pragma unroll
            for (int w = 1; w < kMVSlices; ++w) t += obuf[w * GP * D + idx];
            // A value row with an infinity or NaN: the zero parts of a probability turn it into NaN here, where the
            // product e v itself may be an infinity.  Taken again by the wave, whose lanes hold 64 columns of one head.
            if (__builtin_amdgcn_ballot_w64(!(fabsf(t) < INFINITY))) {
                const int h = idx / D;
                float sum = red_s[0][h], mh = red_m[0][h];
#pragma unroll
                for (int w = 1; w < kWaves; ++w) {
                    sum += red_s[w][h];
                    mh = fmaxf(mh, red_m[w][h]);
                }
                const bool logits = !exp_apart && !a.emit;
                if (sum == sum)
                    t = nonfinite_column(vrs, idx % D - ln.lane, nrows, t, [&](int row) __attribute__((always_inline)) {
                        const int rib = row % RPW;
                        const float z = zs[row / RPW * kWave + rib % L::NG * LPR + rib / L::NG * GP + h];
                        return logits ? __expf(z - mh) : z;
                    });
                else
                    t = sum;  // (a NaN query or key: every product of the head is in doubt)
            }
            obuf[idx] = t;
        }
    } else if constexpr (kWaveSlices) {
        // each wave's partial in its own slice; then output idx = ((w0 + w1) + w2) + ... by the thread that later
        // stores it (the same thread-to-output mapping as the stores below, so no barrier between)
        float* slice = obuf + ln.wave * GP * D;
        if constexpr (kRowSwaps) {
            const float* flat = &acc[0][0][0];  // index (h CPL + c) EPC + x
            const int r = ln.lane / 16;
#pragma unroll
            for (int i = 0; i < kAcc / 4; ++i) {
                const float t = rows_sum4(flat[4 * i], flat[4 * i + 1], flat[4 * i + 2], flat[4 * i + 3]);
                const int ai = 4 * i + r;
                const int h = ai / (CPL * EPC), c = ai / EPC % CPL, x = ai % EPC;
                slice[h * D + (ln.p + c * LPR) * EPC + x] = t;
            }
        } else if (ln.lane < LPR) {
#pragma unroll
            for (int h = 0; h < GP; ++h)
#pragma unroll
                for (int c = 0; c < CPL; ++c)
#pragma unroll
                    for (int x = 0; x < EPC; ++x) slice[h * D + (ln.p + c * LPR) * EPC + x] = acc[h][c][x];
        }
        __syncthreads();
        for (int idx = threadIdx.x; idx < a.group * D; idx += kThreads) {
            float t = obuf[idx];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) t += obuf[w * GP * D + idx];
            obuf[idx] = t;
        }
    } else {
        for (int w = 0; w < kWaves; ++w) {
            if (ln.wave == w && ln.lane < LPR) {
#pragma unroll
                for (int h = 0; h < GP; ++h)
#pragma unroll
                    for (int c = 0; c < CPL; ++c)
#pragma unroll
                        for (int x = 0; x < EPC; ++x) {
                            const int idx = h * D + (ln.p + c * LPR) * EPC + x;
                            obuf[idx] = w == 0 ? acc[h][c][x] : obuf[idx] + acc[h][c][x];
                        }
            }
            __syncthreads();
        }
    }
    if (a.emit && a.nchunk > 1) {
        // the chunk's exponentials e_h(row) = exp(z - m_h) (m_h: this chunk's maximum), every block's already in
        // LDS (the barriers above follow the V pass), to the logit rows for the combine: 4 rows of one head per
        // thread and 16-byte store; rows past the chunk give 0 (rows are padded to a multiple of 64)
        float* zc = a.z + ((size_t)lb * a.hq + (size_t)g * a.group) * a.n_stride + row0;
        const int quads = (nrows + 3) / 4;
        for (int t = threadIdx.x; t < GP * quads; t += kThreads) {
            // heads vary fastest: a wave's LDS reads then spread over the banks (rows fastest, the 8-head layout's
            // stride of 32 words between a wave's threads put them all on two)
            const int h = t % GP, r0 = t / GP * 4;
            if (h >= a.group) continue;
            f32x4 e;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = r0 + j, rib = row % RPW;
                e[j] = row < nrows ? zs[row / RPW * kWave + rib % L::NG * LPR + rib / L::NG * GP + h] : 0.0f;
            }
            *reinterpret_cast<f32x4*>(zc + (size_t)h * a.n_stride + r0) = e;
        }
    }
    auto head_sum = [&](int h) {
        float t = red_s[0][h];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) t += red_s[w][h];
        return t;
    };
    auto head_max = [&](int h) {
        float t = red_m[0][h];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) t = fmaxf(t, red_m[w][h]);
        return t;
    };
    const size_t head0 = (size_t)lb * a.hq + (size_t)g * a.group;
    if (a.emit_norms && threadIdx.x == 0) {
        float tot = 0.0f;
        for (int w = 0; w < kWaves; ++w) tot += red_n[w];
        if (a.nchunk == 1)
            a.vinv[s] = tot > 0.0f ? (float)a.n / tot : 0.0f;
        else
            a.npart[(size_t)s * a.nchunk + chunk] = tot;
    }
    if (a.nchunk == 1) {
        T* ob = static_cast<T*>(a.o) + head0 * D;
        for (int idx = threadIdx.x; idx < a.group * D; idx += kThreads) {
            const float tot = head_sum(idx / D);
            E::store(ob + idx, tot > 0.0f ? obuf[idx] / tot : 0.0f);
        }
    } else {
        for (int idx = threadIdx.x; idx < a.group * D; idx += kThreads) {
            const int h = idx / D;
            a.opart[((head0 + h) * a.nchunk + chunk) * D + idx % D] = obuf[idx];
        }
        if (threadIdx.x < a.group)
            a.part[(head0 + threadIdx.x) * a.nchunk + chunk] =
                make_float2(head_max(threadIdx.x), head_sum(threadIdx.x));
        return;
    }

    // 4. one chunk: the score's group probability sums, staged in each unit's first RPW words (the V pass is over, so
    //    only this wave reads its units, but for the non-finite outputs above, whose threads read every row's words)
    //    and written with 16-byte stores
    if (a.emit && a.nchunk == 1) {
        if constexpr (kMV) __syncthreads();
        static_assert(RPW % 4 == 0, "the coalesced store moves 4 rows at a time");
        const float tot = head_sum(ln.hh);
        const float inv = tot > 0.0f ? 1.0f / tot : 0.0f;
        const int row_in = ln.kk * L::NG + ln.grp;  // this lane's row inside a unit
        int i = 0;
        for (; i + kEpi <= mine; i += kEpi) {  // kEpi units' reads in flight at a time
            float e[kEpi];
#pragma unroll
            for (int v = 0; v < kEpi; ++v) e[v] = zl[(i + v) * kStep];
#pragma unroll
            for (int v = 0; v < kEpi; ++v) e[v] = group_allsum<GP>(e[v] * inv);
            if (ln.hh == 0)
#pragma unroll
                for (int v = 0; v < kEpi; ++v) zs[(ln.wave + (i + v) * kWaves) * kWave + row_in] = e[v];
        }
        for (; i < mine; ++i) {
            const float sum = group_allsum<GP>(zl[i * kStep] * inv);
            if (ln.hh == 0) zs[(ln.wave + i * kWaves) * kWave + row_in] = sum;
        }
        __syncthreads();
        const __amdgpu_buffer_rsrc_t rrs = raw_rsrc(a.r + (size_t)s * a.n_stride, a.n_stride * 4);
        for (int j = threadIdx.x; j * 4 < nrows; j += kThreads) {
            const int row = j * 4;
            store_stream(rrs, row * 4, *reinterpret_cast<const f32x4*>(&zs[(row / RPW) * kWave + row % RPW]));
        }
    }
    }  // kV
}

template <typename T, int D, int GP>
hipError_t launch_attend_gp(const ScorePlan& plan, const ScoreArgs& a, hipStream_t s) {
    if constexpr (Geometry<T, D, 1>::kChunks < GP) {
        return hipErrorInvalidValue;
    } else {
        auto kern = attend_kernel<T, D, GP, true>;
        if (plan.lds_bytes > 64 * 1024) {
            static std::atomic<bool> raised[kMaxDevices];
            const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), raised);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, dim3(plan.grid), dim3(kThreads), plan.lds_bytes, s, a);
        if (plan.split) {
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            // more than eight chunks' partial outputs in flight only where there are more (one sequence of 8 KV heads x
            // 3,278 rows, 13 chunks: 424 -> 416 us for 32 layer calls; with 4 chunks the registers cost 0.2%)
            auto combine = plan.nchunk > 8 ? attend_combine_kernel<T, D, GP, 16> : attend_combine_kernel<T, D, GP, 8>;
            hipLaunchKernelGGL(combine, dim3(plan.grid / plan.nchunk * combine_parts(plan.nchunk, a.emit)),
                               dim3(kCombineThreads), 0, s, a);
        }
        return hipGetLastError();
    }
}

template <typename T, int D, int GP>
hipError_t launch_chunks_gp(const ScorePlan& plan, const ScoreArgs& a, hipStream_t s) {
    if constexpr (Geometry<T, D, 1>::kChunks < GP) {
        return hipErrorInvalidValue;
    } else {
        auto kern = attend_kernel<T, D, GP, false>;
        if (plan.lds_bytes > 64 * 1024) {
            static std::atomic<bool> raised[kMaxDevices];
            const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), raised);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, dim3(plan.grid), dim3(kThreads), plan.lds_bytes, s, a);
        return hipGetLastError();
    }
}

template <typename T, int D>
hipError_t launch_chunks_d(const ScorePlan& plan, const ScoreArgs& a, hipStream_t s) {
    switch (plan.group_pad) {
        case 1: return launch_chunks_gp<T, D, 1>(plan, a, s);
        case 2: return launch_chunks_gp<T, D, 2>(plan, a, s);
        case 4: return launch_chunks_gp<T, D, 4>(plan, a, s);
        case 8: return launch_chunks_gp<T, D, 8>(plan, a, s);
        case 16: return launch_chunks_gp<T, D, 16>(plan, a, s);
        default: return hipErrorInvalidValue;
    }
}

template <typename T, int D>
hipError_t launch_attend_d(const ScorePlan& plan, const ScoreArgs& a, hipStream_t s) {
    switch (plan.group_pad) {
        case 1: return launch_attend_gp<T, D, 1>(plan, a, s);
        case 2: return launch_attend_gp<T, D, 2>(plan, a, s);
        case 4: return launch_attend_gp<T, D, 4>(plan, a, s);
        case 8: return launch_attend_gp<T, D, 8>(plan, a, s);
        case 16: return launch_attend_gp<T, D, 16>(plan, a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool attend_plan(int dtype, int head_dim, int group, int n, int slabs, ScorePlan* plan, size_t max_lds) {
    if (slabs < 1 || !score_plan(dtype, head_dim, group, 1, plan)) return false;
    const int rpw = kWave / plan->group_pad;  // rows per unit
    if (max_lds == 0 || max_lds > kFastLdsMax) max_lds = kFastLdsMax;
    const int lds_rows = (int)(max_lds / (kWave * sizeof(float))) * rpw;
    const int want = (kAttnTargetWgs + slabs - 1) / slabs;
    const int by_rows = (n + kAttnMinRows - 1) / kAttnMinRows;
    int nchunk = (n + lds_rows - 1) / lds_rows;
    nchunk = max(nchunk, min(want, by_rows));
    int rows = (n + nchunk - 1) / nchunk;
    rows = (rows + rpw - 1) / rpw * rpw;  // <= lds_rows, a multiple of rpw
    plan->chunk_rows = rows;
    plan->nchunk = (n + rows - 1) / rows;
    plan->split = plan->nchunk > 1;
    plan->lds_bytes = (size_t)(rows / rpw) * kWave * sizeof(float);
    plan->grid = slabs * plan->nchunk;
    return true;
}

AttendBound attend_bound(int dtype, int head_dim, int group, int n, int slabs_per_layer, int layers) {
    AttendBound r{0, false};
    ScorePlan p;
    if (slabs_per_layer < 1 || layers < 1 || !score_plan(dtype, head_dim, group, 1, &p)) return r;
    const int rpw = kWave / p.group_pad;
    const long lds_rows = (long)(kFastLdsMax / (kWave * sizeof(float))) * rpw;
    const long c0 = (n + lds_rows - 1) / lds_rows;
    const long by_rows = (n + kAttnMinRows - 1) / kAttnMinRows;
    const long want1 = (kAttnTargetWgs + slabs_per_layer - 1) / slabs_per_layer;
    // a call over lc layers makes lc * nchunk(lc) chunks per slab column, nchunk = max(c0, min(want, by_rows))
    // with want = ceil(target / (lc * slabs_per_layer)); lc * want <= target / slabs_per_layer + lc
    const long by_target = layers * c0 > want1 + layers ? layers * c0 : want1 + layers;
    const long by_size = layers * (c0 > by_rows ? c0 : by_rows);
    r.chunk_layers = by_target < by_size ? by_target : by_size;
    r.may_split = c0 > 1 || (by_rows > 1 && want1 > 1);
    return r;
}

hipError_t launch_score_chunks(int dtype, int head_dim, const ScorePlan& plan, const ScoreArgs& a, hipStream_t s) {
    if (dtype == 0) {
        if (head_dim == 64) return launch_chunks_d<float, 64>(plan, a, s);
        if (head_dim == 128) return launch_chunks_d<float, 128>(plan, a, s);
    } else {
        if (head_dim == 64) return launch_chunks_d<bf16_t, 64>(plan, a, s);
        if (head_dim == 128) return launch_chunks_d<bf16_t, 128>(plan, a, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_attend(int dtype, int head_dim, const ScorePlan& plan, const ScoreArgs& a, hipStream_t s) {
    if (dtype == 0) {
        if (head_dim == 64) return launch_attend_d<float, 64>(plan, a, s);
        if (head_dim == 128) return launch_attend_d<float, 128>(plan, a, s);
    } else {
        if (head_dim == 64) return launch_attend_d<bf16_t, 64>(plan, a, s);
        if (head_dim == 128) return launch_attend_d<bf16_t, 128>(plan, a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace ikv
