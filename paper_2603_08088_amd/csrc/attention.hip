// tree_verify_attention: tree-masked attention of the draft-tree query rows against the committed
// prefix cache plus the tree's own K/V (Section 3.3, "Execution view" and "Tree attention mask").
//
// Five kernels compute the per-split partial (m, l, O):
//   * attn_mfma_kernel   bf16: K/V tiles staged through LDS, QK^T and PV on
//                        v_mfma_f32_32x32x16_bf16, online softmax in registers, the ancestor mask applied
//                        as a per-row bitmask only on the tree tile.
//   * attn_wide_kernel   bf16, d = 128, many rows over long splits: the same work unit with 64 rows a wavefront, the tile loop
//                        in assembly (attn_wide_loop.py), v_mfma_f32_16x16x32_bf16.
//   * attn_blocks_kernel bf16, launches that are short of work: the same products, every wavefront with 32-key blocks of
//                        its own instead of a tile shared by the workgroup.
//   * attn_f32_kernel    fp32: both products on v_mfma_f32_16x16x4_f32, no barrier in the tile loop.
//   * attn_generic_kernel  any supported dtype / head dim, fp32 VALU arithmetic, one wavefront per query
//                        row; bf16 with a negative scale, and where ETV_ATTN_FLAG_GENERIC asks for it, as an independent check.
// and attn_combine_kernel merges the splits by log-sum-exp.  With a single split the partial kernels write
// the final output themselves.
//
// Scores are kept in "scaled log2 units" t = (q.k) * scale * log2(e) so that exp is a bare v_exp_f32
// (bf16 kernels; fp32 keeps results below the normal range).
#include "etv_common.h"
#include "attn_wide_loop.h"
#include <atomic>
#include <type_traits>

namespace etv {

struct AttnParams {
    const void *q, *k_cache, *v_cache, *kt, *vt;
    const int32_t *block_table, *prefix_len, *n_nodes;
    const uint64_t *bitmask;
    void *out;
    float *lse;
    float *part_o, *part_m, *part_l;
    int B, T_max, Hq, Hkv, G, d, block_size, max_blocks, P_cap, P_max, words;
    int chunk;   // prefix keys per split, multiple of 64
    int nsplit;  // splits the launch provides; sequence b uses max(1, ceil(P_b / chunk)) of them
    // partial results, split-major so that one workgroup writes one contiguous region:
    //   part_o [B][nsplit][Hq][T_max][d], part_m / part_l [B][nsplit][Hq][T_max]
    int pairs;   // mfma kernels: 32-row chunks of the packed query rows of a KV head
    int wgp;     // mfma kernels: workgroups per (b, kv head, split)
    float scale_log2;
    // mfma kernel, batches of 2 .. 64 sequences with splits: the B * nsplit split slots are shared out among the
    // sequences by their lengths (on the device, where the lengths are), slot-major partials
    //   part_o [B * nsplit][Hq][T_max][d]; split_tab[b] = (first slot, splits in use) for the combine kernel
    int stagger;  // fp32 kernel: chunks of a KV head if the second workgroup of a compute unit starts late, else 0
    int balanced;
    int2 *split_tab;
    uint32_t inv_g, inv_hkv, inv_nsplit, inv_chunk;  // floor(2^32 / G) and so on, for fast_div
};

constexpr float kLn2 = 0.6931471805599453f;
typedef __attribute__((ext_vector_type(2))) float f32x2;
// memory that no kernel writes while it is read: uniform addresses go through scalar loads
typedef __attribute__((address_space(4))) const int32_t *const_i32_ptr;

__device__ __forceinline__ int seq_prefix_len(const AttnParams &p, int b) { return clampi(p.prefix_len[b], 0, p.P_max); }
__device__ __forceinline__ int seq_nsplit(const AttnParams &p, int P) { return max(1, (P + p.chunk - 1) / p.chunk); }
// partial row of split slot `slot` (= b * nsplit + s where every sequence owns nsplit slots)
__device__ __forceinline__ size_t part_row(const AttnParams &p, int slot, int h, int k) {
    return ((size_t)slot * p.Hq + h) * p.T_max + k;
}

// element offset of prefix row `key` of KV head kvh (contiguous or paged cache)
__device__ __forceinline__ size_t prefix_row_offset(const AttnParams &p, int b, int kvh, int key) {
    if (p.block_size > 0) {
        int blk = p.block_table[(size_t)b * p.max_blocks + key / p.block_size];
        return (((size_t)blk * p.Hkv + kvh) * p.block_size + (key % p.block_size)) * (size_t)p.d;
    }
    return (((size_t)b * p.P_cap + key) * p.Hkv + kvh) * (size_t)p.d;
}
__device__ __forceinline__ size_t tree_row_offset(const AttnParams &p, int b, int kvh, int j) {
    return (((size_t)b * p.T_max + j) * p.Hkv + kvh) * (size_t)p.d;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Balanced splits.  With one split size for the whole batch a ragged batch leaves the split slots of its short
// sequences empty while the workgroups of its longest sequence decide the launch time.  Here the launch's
// S = B * nsplit slots are shared out by length: L = the smallest tile count with sum_b max(1, ceil(tiles_b / L))
// <= S (tiles_b: 64-key tiles of the prefix and of the tree), sequence b gets ceil(tiles_b / L) consecutive slots
// and cuts its prefix evenly over them; its last split in use also takes the tree.  Every wavefront works this
// out for itself, lane i holding sequence i (B <= 64): integer arithmetic only, so all of them agree.
struct SplitShare {
    int b, j, nvalid, start, tps, P_raw, n_raw;  // sequence, split within it, splits in use, first slot, tiles per split
    bool live;
};
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uni64(uint64_t v) {
    return (uint64_t)(uint32_t)uni((int)(uint32_t)v) | (uint64_t)(uint32_t)uni((int)(uint32_t)(v >> 32)) << 32;
}
// It stands before a workgroup's first load, so it is written for latency: lane moves of the vector unit instead of shuffles through
// LDS, uniform divisions only, and the owner's shares alone are worked out.  fp32, B = 2, T = 33, P = 771 / 1003 18.4 -> 17.0 us; bf16
// calls whose splits follow the lengths 0.3 ... 0.8 us (B = 3, T = 4, P = 2816: 15.0 -> 14.4).
__device__ inline SplitShare balanced_share(const AttnParams &p, const int32_t *prefix_len, const int32_t *n_nodes, int B, int x, int lane) {
    const int at = min(lane, B - 1);
    const bool has = lane < B;
    const int P_raw = prefix_len[at], n_raw = n_nodes[at];
    const int P = clampi(P_raw, 0, p.P_max), n = clampi(n_raw, 0, p.T_max);
    const int pt = has ? (P + 63) >> 6 : 0;
    const int tt = pt + (has ? (n + 63) >> 6 : 0);
    const int S = B * p.nsplit;
    const auto last = [](int v) { return __builtin_amdgcn_readlane(v, 63); };
    const int total = last(wave_scan_sum(tt));
    int hi = max(1, last(wave_scan_max(tt)));                                              // one slot per sequence always fits
    if (S > B) hi = min(hi, max(1, (int)((uint32_t)(total + (S - B) - 1) / (uint32_t)(S - B))));  // sum (tiles_b / L + 1) <= S
    int lo = min(hi, max(1, (int)((uint32_t)(total + S - 1) / (uint32_t)S)));
    const auto slots_of = [&](int L) {  // of the lane's sequence, L tiles to a slot
        uint32_t rem;
        const uint32_t q = fast_div((uint32_t)(tt + L - 1), (uint32_t)L, 0xffffffffu / (uint32_t)L, rem);
        return has ? max(1, (int)q) : 0;
    };
    while (lo < hi) {  // sum_b max(1, ceil(tiles_b / L)) falls as L grows
        const int mid = (lo + hi) >> 1;
        if (last(wave_scan_sum(slots_of(mid))) <= S) hi = mid;
        else lo = mid + 1;
    }
    const int ns = slots_of(lo);
    const int start = wave_scan_sum(ns) - ns;  // strictly increasing over the sequences
    const int owner = uni(__popcll(__ballot(has && start <= x)) - 1);
    const auto of_owner = [&](int v) { return __builtin_amdgcn_readlane(v, owner & 63); };
    SplitShare r;
    r.b = owner;
    r.start = of_owner(start);
    r.j = x - r.start;
    const uint32_t o_ns = (uint32_t)max(of_owner(ns), 1);
    r.tps = max(1, (int)(((uint32_t)of_owner(tt) + o_ns - 1) / o_ns));
    r.nvalid = max(1, (int)(((uint32_t)of_owner(pt) + (uint32_t)r.tps - 1) / (uint32_t)r.tps));  // in use: those that hold prefix keys
    r.P_raw = of_owner(P_raw);
    r.n_raw = of_owner(n_raw);
    r.live = owner >= 0 && r.j < r.nvalid;
    return r;
}
__device__ __forceinline__ SplitShare balanced_share(const AttnParams &p, int x, int lane) {
    return balanced_share(p, p.prefix_len, p.n_nodes, p.B, x, lane);
}

template <typename T>
__device__ __forceinline__ float load_elem(const T *p, size_t i);
template <>
__device__ __forceinline__ float load_elem<float>(const float *p, size_t i) { return p[i]; }
template <>
__device__ __forceinline__ float load_elem<uint16_t>(const uint16_t *p, size_t i) { return bf16_bits_to_float(p[i]); }

template <typename T>
__device__ __forceinline__ void store_elem(T *p, size_t i, float v);
template <>
__device__ __forceinline__ void store_elem<float>(float *p, size_t i, float v) { p[i] = v; }
template <>
__device__ __forceinline__ void store_elem<uint16_t>(uint16_t *p, size_t i, float v) { p[i] = float_to_bf16_bits(v); }

template <typename T, int D>
__device__ __forceinline__ float dot_row(const float *sq, const T *row) {
    float acc = 0.f;
    if constexpr (sizeof(T) == 4) {
        const float4 *r4 = reinterpret_cast<const float4 *>(row);
#pragma unroll 4
        for (int c = 0; c < D / 4; c++) {
            float4 x = r4[c];
            acc = fmaf(sq[4 * c], x.x, acc);
            acc = fmaf(sq[4 * c + 1], x.y, acc);
            acc = fmaf(sq[4 * c + 2], x.z, acc);
            acc = fmaf(sq[4 * c + 3], x.w, acc);
        }
    } else {
        const uint4 *r8 = reinterpret_cast<const uint4 *>(row);
#pragma unroll 4
        for (int c = 0; c < D / 8; c++) {
            uint4 x = r8[c];
            uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int e = 0; e < 4; e++) {
                acc = fmaf(sq[8 * c + 2 * e], __uint_as_float(w[e] << 16), acc);
                acc = fmaf(sq[8 * c + 2 * e + 1], __uint_as_float(w[e] & 0xffff0000u), acc);
            }
        }
    }
    return acc;
}

// Values that are not finite, on the matrix-core kernels of fp32 and of heads of 64.  A key that a row does not see must not
// reach it whatever its value, but 0 * inf and 0 * NaN in a product are NaN.  So where a tile with masked keys holds such a
// value (rare, found with a few integer instructions per tile), the product runs with zeros in its place, and after the last
// tile the wavefront goes through its masked keys once more for the columns that each of its rows has to add +inf, -inf or,
// for NaN, both to.  (In a tile without masked keys every row sees every key.)
// One group of keys base .. base + count - 1 of the tree or the prefix; `vis`: those that the lane's row sees.
template <typename T, int D>
__device__ __forceinline__ void find_nonfinite(const AttnParams &p, int b, int kvh, int P, bool tree, int base, int count, uint64_t vis,
                                               uint64_t (&up)[D / 64], uint64_t (&down)[D / 64]) {
    const int lane = threadIdx.x & 63;
#pragma unroll 1
    for (int j = 0; j < count; j++) {
        const T *row = tree && p.vt ? static_cast<const T *>(p.vt) + tree_row_offset(p, b, kvh, base + j)
                                    : static_cast<const T *>(p.v_cache) + prefix_row_offset(p, b, kvh, (tree ? P : 0) + base + j);
#pragma unroll
        for (int c = 0; c < D / 64; c++) {
            const float x = load_elem<T>(row, lane + 64 * c);
            const bool bad = !(fabsf(x) < INFINITY);
            const uint64_t u = __ballot(bad && x != -INFINITY), d = __ballot(bad && x != INFINITY);
            if ((vis >> j) & 1ull) { up[c] |= u; down[c] |= d; }
        }
    }
}

// ----------------------------------------------------------------------------------------------
// Generic kernel: grid (T_max, Hq, B * nsplit), one wavefront per (query row, head, split).
// QK: lane = key (row dot product against q held in LDS); PV: lane = head-dim column, the weight of
// key j broadcast by a lane read.
// ----------------------------------------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(64) attn_generic_kernel(AttnParams p) {
    constexpr int DPL = D / 64;
    const int k = blockIdx.x, h = blockIdx.y;
    const int b = blockIdx.z / p.nsplit, s = blockIdx.z % p.nsplit;
    const int lane = threadIdx.x;
    const int n = clampi(p.n_nodes[b], 0, p.T_max);
    const int P = seq_prefix_len(p, b);
    const int nvalid = seq_nsplit(p, P);
    if (s >= nvalid) return;
    const bool direct = (p.nsplit == 1);
    T *out = static_cast<T *>(p.out);
    const size_t orow = (((size_t)b * p.T_max + k) * p.Hq + h) * D;
    if (k >= n) {
        if (direct) {
#pragma unroll
            for (int i = 0; i < DPL; i++) store_elem<T>(out, orow + lane + 64 * i, 0.f);
            if (p.lse && lane == 0) p.lse[((size_t)b * p.Hq + h) * p.T_max + k] = -INFINITY;
        }
        return;
    }
    __shared__ float sq[D];
    const T *q = static_cast<const T *>(p.q);
#pragma unroll
    for (int i = 0; i < DPL; i++) sq[lane + 64 * i] = load_elem<T>(q, orow + lane + 64 * i);
    __syncthreads();
    const int kvh = h / p.G;
    const T *kc = static_cast<const T *>(p.k_cache), *vc = static_cast<const T *>(p.v_cache);
    const T *kt = static_cast<const T *>(p.kt), *vt = static_cast<const T *>(p.vt);
    float m = -INFINITY, l = 0.f;
    float o[DPL];
#pragma unroll
    for (int i = 0; i < DPL; i++) o[i] = 0.f;

    auto tile = [&](float sc, bool valid, int count, auto v_row_of) {
        float tmax = wave_max(valid ? sc : -INFINITY);
        float m_new = fmaxf(m, tmax);
        if (m_new == -INFINITY) return;  // nothing visible yet
        float alpha = exp2f(m - m_new);
        float pv = valid ? exp2f(sc - m_new) : 0.f;
        l = l * alpha + wave_sum(pv);
#pragma unroll
        for (int i = 0; i < DPL; i++) o[i] *= alpha;
        m = m_new;
        for (int j = 0; j < count; j++) {
            float pj = __shfl(pv, j);
            if (pj == 0.f) continue;  // wave-uniform
            const T *vr = v_row_of(j);
#pragma unroll
            for (int i = 0; i < DPL; i++) o[i] = fmaf(pj, load_elem<T>(vr, lane + 64 * i), o[i]);
        }
    };

    const int k0 = s * p.chunk, k1 = min(P, k0 + p.chunk);
    for (int t0 = k0; t0 < k1; t0 += 64) {
        const int key = t0 + lane;
        const bool valid = key < k1;
        float sc = 0.f;
        if (valid) sc = dot_row<T, D>(sq, kc + prefix_row_offset(p, b, kvh, key)) * p.scale_log2;
        tile(sc, valid, min(64, k1 - t0), [&](int j) { return vc + prefix_row_offset(p, b, kvh, t0 + j); });
    }
    if (s == nvalid - 1) {
        const uint64_t *mrow = p.bitmask + ((size_t)b * p.T_max + k) * p.words;
        for (int t0 = 0; t0 < n; t0 += 64) {
            const int j = t0 + lane;
            const bool valid = (j < n) && ((mrow[t0 >> 6] >> lane) & 1ull);
            float sc = 0.f;
            // tree rows: the step's own buffer, or (kt null) the cache tail, node j at position P + j
            if (valid)
                sc = (kt ? dot_row<T, D>(sq, kt + tree_row_offset(p, b, kvh, j))
                         : dot_row<T, D>(sq, kc + prefix_row_offset(p, b, kvh, P + j))) * p.scale_log2;
            tile(sc, valid, min(64, n - t0), [&](int jj) {
                return kt ? vt + tree_row_offset(p, b, kvh, t0 + jj) : vc + prefix_row_offset(p, b, kvh, P + t0 + jj);
            });
        }
    }
    if (direct) {
        const float inv = 1.f / l;
#pragma unroll
        for (int i = 0; i < DPL; i++) store_elem<T>(out, orow + lane + 64 * i, o[i] * inv);
        if (p.lse && lane == 0) p.lse[((size_t)b * p.Hq + h) * p.T_max + k] = (m + log2f(l)) * kLn2;
    } else {
        const size_t pr = part_row(p, b * p.nsplit + s, h, k);
#pragma unroll
        for (int i = 0; i < DPL; i++) p.part_o[pr * D + lane + 64 * i] = o[i];
        if (lane == 0) {
            p.part_m[pr] = m;
            p.part_l[pr] = l;
        }
    }
}

// ----------------------------------------------------------------------------------------------
// Combine: grid (row groups of a sequence, B).  out = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s.
// ----------------------------------------------------------------------------------------------
// WPR wavefronts per query row (b, k, h), 4 / WPR rows per workgroup; a lane owns D / (64 * WPR) consecutive output
// elements (two wavefronts per row for small launches, where the latency of a row's chain is what counts).  U splits are a
// batch, whose loads are in flight together; further batches, for launches with more splits than that, update a
// running (M, L, acc) that is rescaled when a later batch raises the maximum.  Lane i of every sixteen works out the weight of
// split i % U, so a batch costs one exponential and a few lane moves instead of U exponentials in every lane.
// What bounds it is latency: what the first addresses need are leading scalar arguments, as in the key-block kernel.  Before, the
// arguments, two 64-bit divisions, the sizes and the partials came one after the other: 32 layers of B = 1, T = 60, P = 2048 with four
// splits 470.7 -> 433.0 us, 63 drawn calls with splits 6 % shorter on average, one sequence with 108 splits 16.6 -> 14.3.
// AHEAD: so many splits of the first batch are asked for together with the sizes (every sequence owns the same slots, which exist
// whatever the lengths are; what an absent one or a padded row's holds is not used), the others of the batch behind them.  That
// hides a trip, and reads partials that nobody wrote where P_max is a bound well above the prefixes or rows are padded.  Up to kCombineAhead
// bytes the whole batch is worth it, beyond that two splits of kCombineAheadTwo, and none where even these are more.  B = 1, 32/8 heads,
// whole call, whole batch / nothing / by this rule: T = 128, P_max = 32768 (15 splits), P = 32768 68.5 / 69.7 / 68.8 us, P = 2048 59.1 / 57.3 /
// 57.3, with 16 nodes 42.5 / 39.4 / 39.5; P_max = P = 6000 (6 splits) 29.4 / 30.1 / 29.5; T = 256, P_max = 6000 (3 splits), 32 nodes, P = 375
// 19.0 / 17.7 / 17.6; B = 66, T = 16, 4/1 heads (6 splits), P_max = 4096, P = 512 19.2 / 18.4 / 18.1.
// SHARED: the four wavefronts of a workgroup take every fourth split of one row and merge through LDS, for launches whose
// splits would otherwise be several batches in series.  32 rows, 43 splits: 9.0 -> 4.7 us; 16 rows, 107 splits: 18.2 -> 7.4;
// with many rows the batches of different rows overlap anyway (1920 rows, 32 splits: 9.0, shared 11.2), and up to 16 splits
// one wavefront's single batch is as fast or faster: a row whose sequence has no more is left to the first wavefront (whole
// call, B = 2, T = 16, 32/8 heads, 24 equal splits launched and some 12 used 18.0 us, shared 20.1; one sequence with 24 10.7, 12.1).
template <typename T, int D, int WPR, int U, bool SHARED, bool BALANCED, int AHEAD>
__global__ void __launch_bounds__(256)
attn_combine_kernel(const int32_t *sizes, const int32_t *n_nodes, const float *part_o, const float *part_m, const float *part_l, int Hq,
                    uint32_t inv_hq, int T_max, int nsplit, AttnParams p) {
    constexpr int E = D / (64 * WPR);
    static_assert(E >= 1 && (!SHARED || WPR == 1), "at least one element per lane");
    static_assert(AHEAD == 0 || (!SHARED && !BALANCED && (AHEAD == 2 || AHEAD == U)), "slots that are known without the sizes");
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = SHARED ? (int)blockIdx.x : (int)blockIdx.x * (4 / WPR) + wv / WPR;  // of the sequence
    const int lane = (wv % WPR) * 64 + (threadIdx.x & 63);  // position within the row, in units of E elements
    if (row >= Hq * T_max) return;
    uint32_t h_;
    const int k = (int)fast_div(row, Hq, inv_hq, h_), h = (int)h_, b = blockIdx.y;
    const uint32_t sstride = (uint32_t)Hq * T_max;  // rows between consecutive splits
    T *out = static_cast<T *>(p.out);
    const size_t orow = (((size_t)b * T_max + k) * Hq + h) * D + (size_t)lane * E;
    const size_t lrow = ((size_t)b * Hq + h) * T_max + k;
    // A batch: splits first, first + step, ... of `count`.  Lane i of every sixteen holds the statistics of split i % U of the batch (one
    // load each, one exponential for all), and every lane its elements of all of them.
    typedef std::conditional_t<E == 2, f32x2, float> elems;
    const int u_own = threadIdx.x & (U - 1);
    float m_own, l_own;
    elems os[U];
    auto fetch_part = [&](auto from, auto to, size_t pr0, int first, int step, int count) {  // elements of the batch's splits from ... to - 1
#pragma unroll
        for (int u = decltype(from)::value; u < decltype(to)::value; u++) {
            const int x = first + u * step;
            os[u] = *reinterpret_cast<const elems *>(part_o + (pr0 + (size_t)(uint32_t)(x < count ? x : 0) * sstride) * D + (size_t)lane * E);
        }
    };
    auto fetch_own = [&](size_t pr0, int first, int step, int count) {
        const int own = first + u_own * step;
        const size_t r_own = pr0 + (size_t)(uint32_t)(own < count ? own : 0) * sstride;
        m_own = part_m[r_own];
        l_own = part_l[r_own];
    };
    constexpr std::integral_constant<int, 0> none;
    constexpr std::integral_constant<int, AHEAD> ahead;
    constexpr std::integral_constant<int, U> all;
    auto fetch = [&](size_t pr0, int first, int step, int count) {
        fetch_own(pr0, first, step, count);
        fetch_part(none, all, pr0, first, step, count);
    };
    const size_t pr_fixed = ((size_t)((uint32_t)b * nsplit) * Hq + h) * T_max + k;
    const int n_raw = ((const_i32_ptr)(uintptr_t)n_nodes)[b];
    int first_slot = 0, nvalid, P_raw = 0;
    if constexpr (BALANCED) {
        first_slot = ((const_i32_ptr)(uintptr_t)sizes)[2 * b];
        nvalid = ((const_i32_ptr)(uintptr_t)sizes)[2 * b + 1];
    } else {
        P_raw = ((const_i32_ptr)(uintptr_t)sizes)[b];
        if constexpr (AHEAD == U) {
            fetch(pr_fixed, 0, 1, nsplit);
            // all of them here and now, with the arguments: one trip
            if constexpr (U == 8)
                asm volatile("" ::"s"(n_raw), "s"(P_raw), "s"(p.P_max), "s"(p.chunk), "s"(p.inv_chunk), "s"(p.out), "s"(p.lse), "v"(m_own), "v"(l_own),
                             "v"(os[0]), "v"(os[1]), "v"(os[2]), "v"(os[3]), "v"(os[4]), "v"(os[5]), "v"(os[6]), "v"(os[7]));
            else
                asm volatile("" ::"s"(n_raw), "s"(P_raw), "s"(p.P_max), "s"(p.chunk), "s"(p.inv_chunk), "s"(p.out), "s"(p.lse), "v"(m_own), "v"(l_own),
                             "v"(os[0]), "v"(os[1]), "v"(os[2]), "v"(os[3]), "v"(os[4]), "v"(os[5]), "v"(os[6]), "v"(os[7]), "v"(os[U - 8]),
                             "v"(os[U - 7]), "v"(os[U - 6]), "v"(os[U - 5]), "v"(os[U - 4]), "v"(os[U - 3]), "v"(os[U - 2]), "v"(os[U - 1]));
        } else if constexpr (AHEAD > 0) {
            fetch_own(pr_fixed, 0, 1, nsplit);
            fetch_part(none, ahead, pr_fixed, 0, 1, nsplit);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" ::"s"(n_raw), "s"(P_raw), "s"(p.P_max), "s"(p.chunk), "s"(p.inv_chunk), "s"(p.out), "s"(p.lse));
        }
        uint32_t rem;
        nvalid = max(1, (int)fast_div(clampi(P_raw, 0, p.P_max) + p.chunk - 1, p.chunk, p.inv_chunk, rem));
    }
    if (k >= clampi(n_raw, 0, T_max)) {
        if (SHARED && wv > 0) return;  // uniform over the workgroup: no barrier is left behind
#pragma unroll
        for (int e = 0; e < E; e++) store_elem<T>(out, orow + e, 0.f);
        if (p.lse && lane == 0) p.lse[lrow] = -INFINITY;
        return;
    }
    const size_t pr0 = BALANCED ? ((size_t)(uint32_t)first_slot * Hq + h) * T_max + k : pr_fixed;
    if constexpr (AHEAD > 0 && AHEAD < U) fetch_part(ahead, all, pr0, 0, 1, nvalid);
    // (splits shared out by length: a sequence may have far fewer than nsplit)
    const bool many = SHARED && nvalid > U;
    if (SHARED && !many && wv > 0) return;  // uniform over the workgroup, as below
    float M = -INFINITY, L = 0.f, acc[E];
#pragma unroll
    for (int e = 0; e < E; e++) acc[e] = 0.f;
    auto over = [](float v, auto f) {  // over the U lanes of a batch, in every lane
        const auto turn = [](float x, auto ctrl) {
            return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), decltype(ctrl)::value, 0xf, 0xf, false));
        };
        if (U == 16) v = f(v, turn(v, std::integral_constant<int, 0x128>{}));  // 8, 4, 2, 1 lanes round the sixteen
        v = f(v, turn(v, std::integral_constant<int, 0x124>{}));
        v = f(v, turn(v, std::integral_constant<int, 0x122>{}));
        return f(v, turn(v, std::integral_constant<int, 0x121>{}));
    };
    auto take = [&](auto every, int first) {  // splits first, first + every, ...
        constexpr int step = decltype(every)::value;
        for (int s0 = first; s0 < nvalid; s0 += U * step) {
            if (AHEAD == 0 || s0 > 0) fetch(pr0, s0, step, nvalid);
            if (s0 + u_own * step >= nvalid) m_own = -INFINITY;
            const float Mb = fmaxf(M, over(m_own, [](float x, float y) { return fmaxf(x, y); }));
            if (Mb == -INFINITY) continue;  // nothing visible in this batch or before
            const float keep = exp2f(M - Mb);  // 0 while M is still -inf
            M = Mb;
            const bool there = m_own != -INFINITY;  // absent or empty split: its l and O may be uninitialised memory
            const float w = there ? exp2f(m_own - M) : 0.f;
            const uint32_t present = (uint32_t)__ballot(there);
            L = fmaf(L, keep, over(there ? w * l_own : 0.f, [](float x, float y) { return x + y; }));
#pragma unroll
            for (int e = 0; e < E; e++) acc[e] *= keep;
#pragma unroll
            for (int u = 0; u < U; u++) {
                const float wu = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), u));
                const uint32_t mask = 0u - ((present >> u) & 1u);
                if constexpr (E == 2) {
                    acc[0] = fmaf(wu, __uint_as_float(__float_as_uint(os[u][0]) & mask), acc[0]);
                    acc[1] = fmaf(wu, __uint_as_float(__float_as_uint(os[u][1]) & mask), acc[1]);
                } else {
                    acc[0] = fmaf(wu, __uint_as_float(__float_as_uint(os[u]) & mask), acc[0]);
                }
            }
        }
    };
    if (many) take(std::integral_constant<int, 4>{}, wv);
    else take(std::integral_constant<int, 1>{}, 0);
    if (many) {
        __shared__ float s_m[4], s_l[4], s_acc[4][D];
        if (lane == 0) { s_m[wv] = M; s_l[wv] = L; }
#pragma unroll
        for (int e = 0; e < E; e++) s_acc[wv][lane * E + e] = acc[e];
        __syncthreads();
        if (wv > 0) return;
        M = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
        L = 0.f;
#pragma unroll
        for (int e = 0; e < E; e++) acc[e] = 0.f;
#pragma unroll
        for (int x = 0; x < 4; x++) {
            const float w = s_m[x] == -INFINITY ? 0.f : exp2f(s_m[x] - M);
            L = fmaf(w, s_l[x], L);
#pragma unroll
            for (int e = 0; e < E; e++) acc[e] = fmaf(w, s_acc[x][lane * E + e], acc[e]);
        }
    }
    if constexpr (E == 2 && sizeof(T) == 2) {
        *reinterpret_cast<uint32_t *>(out + orow) = (uint32_t)float_to_bf16_bits(acc[0] / L) | (uint32_t)float_to_bf16_bits(acc[1] / L) << 16;
    } else {
#pragma unroll
        for (int e = 0; e < E; e++) store_elem<T>(out, orow + e, acc[e] / L);
    }
    if (p.lse && lane == 0) p.lse[lrow] = (M + log2f(L)) * kLn2;
}

// ----------------------------------------------------------------------------------------------
// MFMA kernel (bf16, d = 128 or 64; sizes below for d = 128).
//
// Work unit: (split, KV head x row group, sequence).  A workgroup has NW wavefronts (8, or 4 for small
// trees); wavefront w owns one 32-row chunk of the KV head's packed query rows and all of them share the K/V tiles of
// their KV head through LDS, so each prefix K/V byte is fetched from HBM once per G*T query rows.  Two
// wavefronts are resident per SIMD: while one runs the softmax on the vector ALU the other feeds the
// matrix cores.
//
// K/V tiles (64 keys x 256 B each) travel HBM -> LDS with asynchronous direct-to-LDS loads
// (global_load_lds_dwordx4: no registers, completion tracked by vmcnt) into a ring of NS stages, so
// NS-1 tiles (32 KiB each) are in flight per workgroup while one is being consumed; one workgroup
// barrier per tile.  A direct-to-LDS load writes lane i's 16 bytes at (base + 16 i), so rows cannot be
// padded; instead the 16-byte chunk c of key row r is stored at chunk position c ^ (r & 15) in the K tile
// and c ^ (((r & 3) << 1) | ((r >> 2) & 1)) in the V tile, which spreads the 16-byte K reads (consecutive rows,
// same chunk) and the 8-byte transpose reads of V (4 consecutive rows x 32 B) over the LDS banks.
//
// The two wavefronts of a SIMD (w and w+4) run one phase apart: wavefronts 0..3 do QK(t), softmax(t),
// PV(t) inside ring step t, wavefronts 4..7 do PV(t-1), QK(t), softmax(t).  The tile barrier would otherwise
// keep them in lockstep, both wanting the matrix core, then both the vector ALU; shifted, one wavefront's
// softmax overlaps the other's products.  A V tile therefore lives one ring step longer than a K tile, and
// the ring refills the stage of tile t-2 (two tiles in flight) rather than that of tile t-1.
//
// Per 64-key tile and wavefront (32x32x16 MFMA, 64-lane layouts: A/B operand lane = (row|col l%32,
// 8 contraction values at 8*(l/32)); accumulator lane = (col l%32, rows 8*(i/4) + 4*(l/32) + i%4)):
//   S^T[key, q] = K[key, :] . Q[q, :]      A = K rows from LDS (16-byte reads), B = Q held in registers
//   online softmax down each accumulator column (a query row lives in lanes l and l^32)
//   O^T[d, q]  += V^T[d, key] P^T[key, q]  A = V^T via the LDS transpose read (ds_read_b64_tr_b16),
//                                          B = P^T taken straight from the S^T accumulator registers
// Both products keep the query index on the accumulator column, so the softmax statistics and the
// rescale of O never cross lanes.
//
// d = 64 runs the same loop on tiles of half the bytes, with three bf16 parts per probability (Geo::NP): twice the
// products per score, and a softmax that splits its weights, so the vector ALU bounds it from T = 32 up.  32/8 heads, B = 32,
// P = 4096: T = 32 90 us, T = 128 276 us (two parts, 16 bits of the weights: 76 and 230); B = 1, P = 32768, T = 128 80 us (68).
// ----------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int KT = 64;  // keys per tile

// Sizes that follow from the head dimension (128 or 64).
template <int D>
struct Geo {
    static constexpr int ROW_BYTES = 2 * D;               // one K or V row of a KV head, bf16
    static constexpr int TILE_BYTES = KT * ROW_BYTES;     // 16 KiB at d = 128
    static constexpr int STAGE_BYTES = 2 * TILE_BYTES;    // K tile then V tile
    static constexpr int RPU = 1024 / ROW_BYTES;          // key rows of a 1 KiB load unit (64 lanes x 16 B): 4 or 8
    static constexpr int CPR = ROW_BYTES / 16;            // 16-byte chunks of a row: 16 or 8
    static constexpr int KK = D / 16;                     // 16-wide contraction steps of Q . K
    static constexpr int DB = D / 32;                     // 32-wide output column blocks
    // bf16 parts of a probability in the PV product.  At d = 64 a probability enters it with all its 24 bits: three
    // parts of eight, whose products with a bf16 V are exact in fp32.
    static constexpr int NP = D == 64 ? 3 : 1;
};

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    f32x2 v = {a, b};
    bf16x2 r = __builtin_convertvector(v, bf16x2);
    return __builtin_bit_cast(uint32_t, r);
}

// Two fp32 values as bf16 pairs hi + mid + lo, exactly: the upper half of the value, of the remainder, and the rest, which
// has at most the last eight of the 24 bits.
__device__ __forceinline__ void split_bf16x3(float a, float b, uint32_t &hi, uint32_t &mid, uint32_t &lo) {
    const auto upper = [](float x) { return __uint_as_float(__float_as_uint(x) & 0xffff0000u); };
    const auto halves = [](float x, float y) { return __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u); };
    hi = halves(a, b);
    a -= upper(a); b -= upper(b);
    mid = halves(a, b);
    lo = halves(a - upper(a), b - upper(b));
}

// acc + the two bf16 values of a packed pair, in fp32: one instruction for two probabilities.  The row sum is
// taken over the probabilities as rounded to bf16, i.e. over exactly the weights the PV product uses.
__device__ __forceinline__ float pair_sum(uint32_t packed, float acc) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, packed), __builtin_bit_cast(bf16x2, 0x3f803f80u),
                                           acc, false);
}

// 16 bytes per lane from global memory straight into LDS at (lds_addr + 16 * lane); asynchronous.
__device__ __forceinline__ void async_load16(const void *gptr, uint32_t lds_addr) {
    // lds_addr is the same in every lane; readfirstlane says so to the compiler whatever it concluded about the loop
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off\n" ::"v"(gptr),
                 "s"(__builtin_amdgcn_readfirstlane(lds_addr)) : "memory");
}
// wait until at most N of this wavefront's vector-memory loads are outstanding (N < 64)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}
// every LDS access this wavefront has issued is done (the buffer it read may be filled again)
__device__ __forceinline__ void wait_lds_reads() {
    __builtin_amdgcn_s_waitcnt(0xc07f);
    asm volatile("" ::: "memory");
}
// max / sum of a value with its partner in the other half of the wavefront (lane ^ 32) without touching
// LDS: v_permlane32_swap exchanges the upper 32 lanes of one register with the lower 32 of another.  (A
// ds_bpermute shuffle here would make the wavefront wait for its pending V-fragment LDS reads as well.)
__device__ __forceinline__ float half_swap_max(float v) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// Three-input max as one instruction (v_maximum3_f32).  fmaxf would first canonicalise each MFMA result with an extra
// v_max; an asm statement hides from the compiler that the instruction reads a matrix result, and it then issues before
// that result is written (the maximum of a row came out stale now and then).
__device__ __forceinline__ float max3(float a, float b, float c) {
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}
__device__ __forceinline__ float half_swap_sum(float v) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// sum with the partner in the other half of its 32 lanes (lane ^ 16)
__device__ __forceinline__ float quarter_swap_sum(float v) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// chunk-position swizzles (measured on gfx950: 16-byte reads reach the full 256 B/clk only with a 4-bit
// row term; the 8-byte transpose reads are fastest with the 3-bit term below).  Rows of 128 B (d = 64) lie two to a
// 256-byte line of the banks: the K term uses the row pair, and the V term moves rows 2, 3 of four to the other half.
template <int D>
__device__ __forceinline__ int kswz_of_row(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
template <int D>
__device__ __forceinline__ int vswz_of_row(int r) { return D == 128 ? (((r & 3) << 1) | ((r >> 2) & 1)) : ((r & 2) << 1); }

extern __shared__ __attribute__((aligned(1024))) uint8_t attn_smem[];

// Asynchronous loads of one 64-key K/V tile into ring stage (ti % NS).  A tile is 16 (d = 64: 8) chunk pairs of
// 1 KiB (4 (8) key rows of K, the same rows of V).  Issuing wavefront w takes pairs w, w+4, ...; in a chunk
// lane i fetches key row 4j + i/16 (8j + i/8) and the 16-byte piece that belongs at chunk position i%16 (i%8) of
// that row.  Pair w + 4u holds rows 16u + 4w .. +3 (32u + 8w .. +7): the lane's place within those 16 rows (and with
// it both swizzles) does not depend on u, so a load is a scalar base per u plus one per-lane 32-bit offset, and the
// address arithmetic of a tile is scalar (a wavefront's instruction issue rate is what bounds a tile step).
template <int D, int NW>
struct TileLoader {
    // wavefronts that issue loads: all 4 of a small workgroup; of 8, only wavefronts 0..3, which otherwise
    // idle at the tile barrier while wavefronts 4..7 (one phase behind) finish their longer chain
    static constexpr int NI = 4;
    static constexpr int U = Geo<D>::TILE_BYTES / 1024 / NI;  // chunk pairs per issuing wavefront and tile: 4 or 2
    // 16-key block of the tile in which pair w + 4u lies
    static __device__ __forceinline__ int block_of(int w, int u) { return (Geo<D>::RPU * (w + NI * u)) >> 4; }
    const uint8_t *kc, *vc, *kt, *vt;
    const uint8_t *kf, *vf;  // full tiles: kc / vc advanced by head_off (paged) or seq_off (contiguous)
    const int32_t *bt;
    size_t row_stride, seq_off, blk_stride, head_off;  // strides are below 2^32
    uint32_t smem_addr;
    int wave, l_row, l_pos, k0, k1, npt, n;
    int P;      // prefix length of the sequence
    bool tail;  // the tree rows live in the cache itself, node j at position P + j (no separate tree buffer)
    uint32_t kcol, vcol;  // per-lane source column (bytes) for the K tile / the V tile swizzle
    uint32_t koff, voff;  // per-lane byte offset from the scalar base of a chunk pair (full tiles)
};

// 16 bytes per lane from (uniform base + per-lane 32-bit offset) into LDS at (lds_addr + 16 * lane)
// NT: streaming (nontemporal) load.  Plain loads sustain 6.0-6.4 TB/s on this machine, streaming ones 7.1 TB/s, but
// a streamed line does not stay in L2 for another workgroup: used only when one workgroup reads each K/V byte.
template <bool NT>
__device__ __forceinline__ void async_load16_s(const void *sbase, uint32_t voff, uint32_t lds_addr) {
    if (NT)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt\n" ::"v"(voff), "s"(sbase), "s"(lds_addr) : "memory");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n" ::"v"(voff), "s"(sbase), "s"(lds_addr) : "memory");
}

// full prefix tile (all 64 keys exist): straight-line address arithmetic.  For a paged cache the physical
// block ids are fetched with scalar loads by fetch_blocks() ahead of the wait and barrier of the ring step,
// so their latency is hidden; the block table is read-only for the kernel (constant address space).
template <int D, int NW>
__device__ __forceinline__ void fetch_blocks(const TileLoader<D, NW> &ld, int ti, int (&blk)[TileLoader<D, NW>::U]) {
    const int lb0 = (ld.k0 + ti * KT) >> 4;
#pragma unroll
    for (int u = 0; u < TileLoader<D, NW>::U; u++)
        blk[u] = ((const_i32_ptr)(uintptr_t)ld.bt)[lb0 + TileLoader<D, NW>::block_of(ld.wave, u)];
}

template <int D, int NW, int NS, bool PAGED, bool NT>
__device__ __forceinline__ void issue_full_tile(const TileLoader<D, NW> &ld, int ti, const int (&blk)[TileLoader<D, NW>::U]) {
    constexpr int U = TileLoader<D, NW>::U, NI = TileLoader<D, NW>::NI;
    constexpr int TILE_BYTES = Geo<D>::TILE_BYTES;
    const uint32_t dst = ld.smem_addr + (uint32_t)(ti % NS) * Geo<D>::STAGE_BYTES + (uint32_t)ld.wave * 1024;
#pragma unroll
    for (int u = 0; u < U; u++) {
        // kf / vf: the cache pointers advanced to this KV head's part of block 0 (paged) or of row 0 of the sequence
        const size_t off = PAGED ? (size_t)(uint32_t)blk[u] * (size_t)(uint32_t)ld.blk_stride
                                 : (size_t)(uint32_t)(ld.k0 + ti * KT + Geo<D>::RPU * NI * u) * (size_t)(uint32_t)ld.row_stride;
        async_load16_s<NT>(ld.kf + off, ld.koff, dst + u * (NI * 1024));
        async_load16_s<NT>(ld.vf + off, ld.voff, dst + TILE_BYTES + u * (NI * 1024));
    }
}

// ragged last prefix tile or tree tile: rows past the end re-read the last valid row (masked later)
template <int D, int NW>
__device__ __forceinline__ void issue_edge_tile(const TileLoader<D, NW> &ld, int ti, int place) {
    constexpr int U = TileLoader<D, NW>::U, NI = TileLoader<D, NW>::NI;
    constexpr int ROW_BYTES = Geo<D>::ROW_BYTES, RPU = Geo<D>::RPU;
    const bool tree = ti >= ld.npt;
    const int base = tree ? (ti - ld.npt) * KT : ld.k0 + ti * KT;
    const int last = (tree ? ld.n : ld.k1) - 1;
    const uint32_t stage = ld.smem_addr + (uint32_t)place * Geo<D>::STAGE_BYTES;
    const bool own = tree && !ld.tail;  // rows of the step's own tree buffer
    const uint8_t *ksrc = own ? ld.kt : ld.kc;
    const uint8_t *vsrc = own ? ld.vt : ld.vc;
    size_t offs[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const int j = ld.wave + NI * u;
        const int r_in = RPU * j + ld.l_row;
        const int key = min(base + r_in, last);
        size_t off;
        if (own) {
            off = (size_t)key * ld.row_stride;
        } else if (tree) {
            // in-place branch cache: node `key` sits at cache position P + key.  P is arbitrary, so the rows
            // of a chunk may lie in two blocks: the block id is looked up per lane.
            const int pos = ld.P + key;
            if (ld.bt) off = (size_t)ld.bt[pos >> 4] * ld.blk_stride + ld.head_off + (size_t)(pos & 15) * ROW_BYTES;
            else off = ld.seq_off + (size_t)pos * ld.row_stride;
        } else if (ld.bt) {
            // the logical block is the same for the whole chunk (its rows are clamped into one block)
            const int lb = __builtin_amdgcn_readfirstlane(min(base + RPU * j, last) >> 4);
            const int blk = ((const_i32_ptr)(uintptr_t)ld.bt)[lb];
            off = (size_t)blk * ld.blk_stride + ld.head_off + (size_t)(key & 15) * ROW_BYTES;
        } else {
            off = ld.seq_off + (size_t)key * ld.row_stride;
        }
        offs[u] = off;
    }
    // all of K, then all of V (attn_wide_kernel counts on the order)
#pragma unroll
    for (int u = 0; u < U; u++) async_load16(ksrc + offs[u] + ld.kcol, stage + (ld.wave + NI * u) * 1024);
#pragma unroll
    for (int u = 0; u < U; u++) async_load16(vsrc + offs[u] + ld.vcol, stage + Geo<D>::TILE_BYTES + (ld.wave + NI * u) * 1024);
}

// LDS view of one staged tile plus the per-lane fragment offsets (bytes) that do not depend on the tile.
struct TileView {
    int krow;          // K fragment row offset: row (lane%32) of key block 0; block 1 is 32 rows further
    int ksw;           // swizzle term of that row (the same for row + 32)
    int vrow, vsw, vchunk, vsub;  // V transpose-read row within a 16-key step, its swizzle, chunk, sub-offset
    int hh;            // lane / 32
};

// How far the running reference of a row may lag behind its true maximum (log2 units) before the
// accumulators are rescaled: exp2 arguments stay <= kLazy, so P <= 256 and nothing overflows, and the
// rescale of the O registers (which live in accumulator registers and cost three instructions each to
// touch) becomes rare after the first tiles.
constexpr float kLazy = 8.0f;

// Can a row reach the exponentials of a tile without a finite score so far?  Where keys are masked, and at d = 64 also where
// products overflow to -inf (such keys weigh nothing).
template <int D, bool MASKED>
constexpr bool kMayBeEmpty = MASKED || D == 64;

// V^T fragments of 32 keys (key block kb) of the V tile at lv.
template <int D>
__device__ __forceinline__ void load_v_frags(const TileView &tv, const uint8_t *lv, int kb, bf16x8 (&vf)[2][Geo<D>::DB]) {
    constexpr int ROW_BYTES = Geo<D>::ROW_BYTES;
#pragma unroll
    for (int st = 0; st < 2; st++) {
        const uint8_t *vr = lv + (32 * kb + 16 * st + tv.vrow) * ROW_BYTES + tv.vsub;
#pragma unroll
        for (int db = 0; db < Geo<D>::DB; db++) {
            const int cpos = ((4 * db + tv.vchunk) ^ tv.vsw) << 4;
            const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(vr + cpos));
            const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(vr + 8 * ROW_BYTES + cpos));
            const bf16x4 a0 = __builtin_bit_cast(bf16x4, v0), a1 = __builtin_bit_cast(bf16x4, v1);
            vf[st][db] = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    }
}

// Heads of 64, masked keys: values that are not finite out of the fragments of 32 keys; true if there were any.
__device__ __forceinline__ bool take_out_nonfinite(bf16x8 (&vf)[2][2]) {
    const auto ill = [](uint32_t w) { return (w & 0x7f807f80u) + 0x00800080u; };  // bit 15 of a half: all ones in the exponent
    uint32_t any = 0;
#pragma unroll
    for (int x = 0; x < 4; x++) {
        const uint4 w = __builtin_bit_cast(uint4, vf[x >> 1][x & 1]);
        any |= (ill(w.x) | ill(w.y)) | (ill(w.z) | ill(w.w));
    }
    if (__builtin_expect(!__any((any & 0x80008000u) != 0), 1)) return false;
    const auto keep = [&](uint32_t w) { return w & ~(((ill(w) >> 15) & 0x00010001u) * 0xffffu); };
#pragma unroll
    for (int x = 0; x < 4; x++) {
        uint4 w = __builtin_bit_cast(uint4, vf[x >> 1][x & 1]);
        w = uint4{keep(w.x), keep(w.y), keep(w.z), keep(w.w)};
        vf[x >> 1][x & 1] = __builtin_bit_cast(bf16x8, w);
    }
    return true;
}

// What find_nonfinite found for the lane's row, added to its outputs (columns 32 db + 8 (i / 4) + 4 hh + i % 4).
__device__ __forceinline__ void add_nonfinite(f32x16 (&oacc)[2], uint64_t up, uint64_t down, int hh) {
    up >>= 4 * hh; down >>= 4 * hh;
#pragma unroll
    for (int db = 0; db < 2; db++)
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int bit = 32 * db + 8 * (i >> 2) + (i & 3);
            oacc[db][i] += ((up >> bit) & 1ull ? INFINITY : 0.f) + ((down >> bit) & 1ull ? -INFINITY : 0.f);
        }
}

// The B operands of a PV product over 32 keys from the packed probabilities of a lane.
__device__ __forceinline__ void pack_frags(const uint32_t (&pk)[8], bf16x8 (&pf)[2]) {
    const uint4 l = {pk[0], pk[1], pk[2], pk[3]}, h = {pk[4], pk[5], pk[6], pk[7]};
    pf[0] = __builtin_bit_cast(bf16x8, l);
    pf[1] = __builtin_bit_cast(bf16x8, h);
}

// First half of a 64-key tile for one wavefront (32 query rows): S^T = K Q^T, mask, running reference,
// P^T = exp2(S^T * scale - m) packed to bf16 in pf[key block][16-key step].  MASKED: key kin of the tile is
// visible to the lane's row iff bit kin of `vis`.
template <int D, bool MASKED>
__device__ __forceinline__ void qk_softmax(const TileView &tv, const uint8_t *lk, const bf16x8 (&qreg)[Geo<D>::KK],
                                           f32x16 (&oacc)[Geo<D>::DB], float &m_run, float &l_run, float scale_log2,
                                           uint64_t vis, bf16x8 (&pf)[Geo<D>::NP][2][2]) {
    constexpr int ROW_BYTES = Geo<D>::ROW_BYTES, KK = Geo<D>::KK;
    // two independent accumulator chains (keys 0..31 and 32..63)
    f32x16 s0, s1;
#pragma unroll
    for (int i = 0; i < 16; i++) { s0[i] = 0.f; s1[i] = 0.f; }
    {
        bf16x8 ka[KK], kb[KK];
#pragma unroll
        for (int kk = 0; kk < KK; kk++) {
            const int col = (((2 * kk + tv.hh) ^ tv.ksw) << 4);
            ka[kk] = *reinterpret_cast<const bf16x8 *>(lk + tv.krow + col);
            kb[kk] = *reinterpret_cast<const bf16x8 *>(lk + tv.krow + 32 * ROW_BYTES + col);
        }
#pragma unroll
        for (int kk = 0; kk < KK; kk++) {
            s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[kk], qreg[kk], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kb[kk], qreg[kk], s1, 0, 0, 0);
        }
    }
    if (MASKED) {
        const uint32_t lo = (uint32_t)(vis >> (4 * tv.hh)), hi = (uint32_t)(vis >> (32 + 4 * tv.hh));
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int bit = 8 * (i >> 2) + (i & 3);
            s0[i] = ((lo >> bit) & 1u) ? s0[i] : -INFINITY;
            s1[i] = ((hi >> bit) & 1u) ? s1[i] : -INFINITY;
        }
    }
    float rmax = max3(s0[0], s1[0], s0[1]);
    rmax = max3(rmax, s1[1], s0[2]);
    rmax = max3(rmax, s1[2], s0[3]);
    rmax = max3(rmax, s1[3], s1[15]);
#pragma unroll
    for (int i = 4; i < 15; i += 1) rmax = max3(rmax, s0[i], s1[i]);
    rmax = fmaxf(rmax, s0[15]);
    rmax = half_swap_max(rmax);
    const float tmax = rmax * scale_log2;  // scale_log2 > 0
    const bool lift = tmax > m_run + kLazy;  // also true for the first visible keys (reference -inf)
    if (__any(lift)) {
        // only the rows that need it move their reference; the others multiply by exactly 1, so a row's
        // arithmetic never depends on what the other rows of the wavefront see
        const float m_new = lift ? tmax : m_run;
        const float alpha = lift ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.f;
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < Geo<D>::DB; db++)
#pragma unroll
            for (int i = 0; i < 16; i++) oacc[db][i] *= alpha;
    }
    const float neg_m = (kMayBeEmpty<D, MASKED> && m_run == -INFINITY) ? 0.f : -m_run;
    float psum = 0.f, psum2 = 0.f;  // two chains
    uint32_t pk[Geo<D>::NP][2][8];
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
        const float a0 = __builtin_amdgcn_exp2f(fmaf(s0[i], scale_log2, neg_m));
        const float a1 = __builtin_amdgcn_exp2f(fmaf(s0[i + 1], scale_log2, neg_m));
        const float b0 = __builtin_amdgcn_exp2f(fmaf(s1[i], scale_log2, neg_m));
        const float b1 = __builtin_amdgcn_exp2f(fmaf(s1[i + 1], scale_log2, neg_m));
        if constexpr (Geo<D>::NP == 3) {
            split_bf16x3(a0, a1, pk[0][0][i >> 1], pk[1][0][i >> 1], pk[2][0][i >> 1]);
            split_bf16x3(b0, b1, pk[0][1][i >> 1], pk[1][1][i >> 1], pk[2][1][i >> 1]);
            psum += a0 + a1;
            psum2 += b0 + b1;
        } else {
            pk[0][0][i >> 1] = pack_bf16x2(a0, a1);
            pk[0][1][i >> 1] = pack_bf16x2(b0, b1);
            psum = pair_sum(pk[0][0][i >> 1], psum);
            psum2 = pair_sum(pk[0][1][i >> 1], psum2);
        }
    }
#pragma unroll
    for (int x = 0; x < Geo<D>::NP; x++)
#pragma unroll
        for (int kb = 0; kb < 2; kb++) pack_frags(pk[x][kb], pf[x][kb]);
    l_run += psum + psum2;
}

// Second half: O^T += V^T P^T over the 64 keys of the V tile at lv; D / 32 independent accumulator chains.  `ill` is set
// where a tile with masked keys holds values that are not finite.
template <int D>
__device__ __forceinline__ void pv_accumulate(const TileView &tv, const uint8_t *lv, const bf16x8 (&pf)[Geo<D>::NP][2][2],
                                              f32x16 (&oacc)[Geo<D>::DB], bool masked, bool &ill) {
    constexpr int DB = Geo<D>::DB;
    bf16x8 vf[2][DB];
    load_v_frags<D>(tv, lv, 0, vf);
#pragma unroll
    for (int kb = 0; kb < 2; kb++) {
        bf16x8 va[2][DB];
#pragma unroll
        for (int st = 0; st < 2; st++)
#pragma unroll
            for (int db = 0; db < DB; db++) va[st][db] = vf[st][db];
        if (kb == 0) load_v_frags<D>(tv, lv, 1, vf);  // the second half's fragments fly during the first half's products
        if constexpr (D == 64)
            if (masked && take_out_nonfinite(va)) ill = true;
#pragma unroll
        for (int st = 0; st < 2; st++)
#pragma unroll
            for (int db = 0; db < DB; db++)
#pragma unroll
                for (int x = 0; x < Geo<D>::NP; x++)
                    oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[st][db], pf[x][kb][st], oacc[db], 0, 0, 0);
    }
}

// Key-halves variants: a wavefront takes 32 of the 64 keys of a tile (key block kb); two wavefronts share a
// 32-row chunk and keep independent running (m, l, O), merged once after the last tile.  Halves the
// per-tile dependency chain of a wavefront, which is what bounds the rate when a workgroup has fewer chunks
// than wavefronts.  vis32: visibility bits of the wavefront's 32 keys; apply: a uniform switch for callers that keep one
// copy of the code for masked and unmasked blocks.
struct Nothing {
    __device__ void operator()() const {}
};
// between(): runs once K is in registers, beside the score products
template <int D, bool MASKED, class F = Nothing>
__device__ __forceinline__ void qk_softmax_half(const TileView &tv, const uint8_t *lk, int kb, const bf16x8 (&qreg)[Geo<D>::KK],
                                                f32x16 (&oacc)[Geo<D>::DB], float &m_run, float &l_run, float scale_log2,
                                                uint32_t vis32, bf16x8 (&pf)[Geo<D>::NP][2], bool apply = true, F &&between = F{}) {
    constexpr int ROW_BYTES = Geo<D>::ROW_BYTES, KK = Geo<D>::KK;
    // two accumulator chains over the even / odd 16-wide d steps, summed afterwards
    f32x16 s0, s1;
#pragma unroll
    for (int i = 0; i < 16; i++) { s0[i] = 0.f; s1[i] = 0.f; }
    {
        bf16x8 ka[KK];
        const uint8_t *kr = lk + tv.krow + kb * (32 * ROW_BYTES);
#pragma unroll
        for (int kk = 0; kk < KK; kk++)
            ka[kk] = *reinterpret_cast<const bf16x8 *>(kr + (((2 * kk + tv.hh) ^ tv.ksw) << 4));
        if constexpr (D == 128 && !std::is_same_v<F, Nothing>)  // all in flight: with two registers in turn every product waits for a read
            asm volatile("" ::"v"(ka[0]), "v"(ka[1]), "v"(ka[2]), "v"(ka[3]), "v"(ka[4]), "v"(ka[5]), "v"(ka[6]), "v"(ka[7]));
#pragma unroll
        for (int kk = 0; kk < KK; kk += 2) {
            s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[kk], qreg[kk], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[kk + 1], qreg[kk + 1], s1, 0, 0, 0);
        }
    }
    between();
#pragma unroll
    for (int i = 0; i < 16; i++) s0[i] += s1[i];
    if (MASKED && apply) {
        const uint32_t lo = vis32 >> (4 * tv.hh);
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int bit = 8 * (i >> 2) + (i & 3);
            s0[i] = ((lo >> bit) & 1u) ? s0[i] : -INFINITY;
        }
    }
    float rmax = max3(s0[0], s0[1], s0[2]);
#pragma unroll
    for (int i = 3; i < 15; i += 2) rmax = max3(rmax, s0[i], s0[i + 1]);
    rmax = fmaxf(rmax, s0[15]);
    rmax = half_swap_max(rmax);
    const float tmax = rmax * scale_log2;
    const bool lift = tmax > m_run + kLazy;
    if (__any(lift)) {
        const float m_new = lift ? tmax : m_run;
        const float alpha = lift ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.f;
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < Geo<D>::DB; db++)
#pragma unroll
            for (int i = 0; i < 16; i++) oacc[db][i] *= alpha;
    }
    const float neg_m = (kMayBeEmpty<D, MASKED> && m_run == -INFINITY) ? 0.f : -m_run;
    float psum = 0.f;
    uint32_t pk[Geo<D>::NP][8];
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
        const float a0 = __builtin_amdgcn_exp2f(fmaf(s0[i], scale_log2, neg_m));
        const float a1 = __builtin_amdgcn_exp2f(fmaf(s0[i + 1], scale_log2, neg_m));
        if constexpr (Geo<D>::NP == 3) {
            split_bf16x3(a0, a1, pk[0][i >> 1], pk[1][i >> 1], pk[2][i >> 1]);
            psum += a0 + a1;
        } else {
            pk[0][i >> 1] = pack_bf16x2(a0, a1);
            psum = pair_sum(pk[0][i >> 1], psum);
        }
    }
#pragma unroll
    for (int x = 0; x < Geo<D>::NP; x++) pack_frags(pk[x], pf[x]);
    l_run += psum;
}

template <int D, bool AT_ONCE = false>
__device__ __forceinline__ void pv_accumulate_half(const TileView &tv, const uint8_t *lv, int kb, const bf16x8 (&pf)[Geo<D>::NP][2],
                                                   f32x16 (&oacc)[Geo<D>::DB], bool masked, bool &ill) {
    bf16x8 vf[2][Geo<D>::DB];
    load_v_frags<D>(tv, lv, kb, vf);
    if constexpr (D == 128 && AT_ONCE)
        asm volatile("" ::"v"(vf[0][0]), "v"(vf[0][1]), "v"(vf[0][2]), "v"(vf[0][3]), "v"(vf[1][0]), "v"(vf[1][1]), "v"(vf[1][2]), "v"(vf[1][3]));
    if constexpr (D == 64)
        if (masked && take_out_nonfinite(vf)) ill = true;
#pragma unroll
    for (int st = 0; st < 2; st++)
#pragma unroll
        for (int db = 0; db < Geo<D>::DB; db++)
#pragma unroll
            for (int x = 0; x < Geo<D>::NP; x++)
                oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[st][db], pf[x][st], oacc[db], 0, 0, 0);
}

template <int D, int NW, int NS, bool PAGED, bool KH>
__global__ void __launch_bounds__(NW * 64, 2) attn_mfma_kernel(AttnParams p) {
    using Loader = TileLoader<D, NW>;
    constexpr int ROW_BYTES = Geo<D>::ROW_BYTES, TILE_BYTES = Geo<D>::TILE_BYTES, STAGE_BYTES = Geo<D>::STAGE_BYTES;
    constexpr int KK = Geo<D>::KK, DB = Geo<D>::DB;
    constexpr int LPW = 2 * Loader::U;  // direct-to-LDS loads an issuing wavefront issues per tile
    uint8_t *const smem = attn_smem;
    const uint32_t smem_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)attn_smem;

    // Row groups (wg) of one KV head read the same K/V.  Workgroups go to the 8 XCDs round-robin by linear id;
    // with wg as the slow index the ids of one (split, KV head) differ by multiples of nsplit * Hkv, i.e. (for
    // Hkv a multiple of 8) they share an XCD and the second reader of a K/V line finds it in that XCD's L2.
    const int wg = blockIdx.y / p.Hkv, kvh = blockIdx.y % p.Hkv;
    const int tid = threadIdx.x, lane = tid & 63;
    SplitShare share{};
    if (p.balanced) {  // grid (B * nsplit slots, Hkv * row groups): which sequence and split is this slot?
        share = balanced_share(p, (int)blockIdx.x, lane);
        if (!share.live) return;  // uniform over the workgroup
        if (share.j == 0 && blockIdx.y == 0 && tid == 0) p.split_tab[share.b] = make_int2(share.start, share.nvalid);
    }
    const int b = p.balanced ? share.b : (int)blockIdx.z;
    // The split index is rotated by the sequence index.  Unrotated, split s of every sequence lands on XCD s
    // (mod 8 with the head): in a ragged batch the first splits are all full and the last ones short or absent,
    // so some XCDs carry all the long workgroups and finish half as late again as the others.  (Not rotated by
    // the KV head: in a contiguous cache the heads of a key row are neighbours in memory, and the XCD that
    // reads one of them should read all of them at about the same time.)
    const int s = p.balanced ? share.j : (int)((blockIdx.x + blockIdx.z) % p.nsplit);
    const int chunk = p.balanced ? share.tps * KT : p.chunk;  // prefix keys per split of this sequence
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c32 = lane & 31, hh = lane >> 5;

    // Start-up.  The caches are cold when a kernel starts and every dependent trip to memory costs the better
    // part of a microsecond, so the trips before the first tile load are made as few as possible: one for the
    // kernel arguments (all of them, not a few at a time as they come up), one for the sequence's sizes
    // together with the physical block ids of the first tiles.  Those ids are read before it is known how long
    // the prefix is: the index is clamped into the table row, and an id is used only if its tile turns out to
    // be a full prefix tile.
    constexpr bool kShifted = (NW == 8);
    constexpr int PD = kShifted ? NS - 2 : NS - 1;  // tiles in flight behind the one being consumed
    static_assert(PD >= 1 && PD <= 3, "ring depth");
    asm volatile("" ::"s"(p.q), "s"(p.k_cache), "s"(p.v_cache), "s"(p.kt), "s"(p.vt), "s"(p.block_table),
                 "s"(p.prefix_len), "s"(p.n_nodes), "s"(p.bitmask), "s"(p.T_max), "s"(p.Hq), "s"(p.G),
                 "s"(p.max_blocks), "s"(p.P_cap), "s"(p.P_max), "s"(p.words), "s"(p.chunk), "s"(p.pairs));
    int n_raw, P_raw;
    if (p.balanced) {
        n_raw = share.n_raw; P_raw = share.P_raw;
    } else {
        n_raw = ((const_i32_ptr)(uintptr_t)p.n_nodes)[b]; P_raw = ((const_i32_ptr)(uintptr_t)p.prefix_len)[b];
    }
    // (the four blocks of a tile are consecutive table entries; an issuing wavefront needs U of them)
    int blk_pro[PD][Loader::U];
    const int lb_first = (s * p.chunk) >> 4;
    const bool spec = PAGED && !p.balanced && lb_first + 4 * PD <= p.max_blocks;  // the whole range lies inside the table row
    if (spec) {
        const const_i32_ptr bt_row = (const_i32_ptr)(uintptr_t)(p.block_table + (size_t)b * p.max_blocks + lb_first);
#pragma unroll
        for (int t = 0; t < PD; t++)
#pragma unroll
            for (int u = 0; u < Loader::U; u++) blk_pro[t][u] = bt_row[4 * t + Loader::block_of(wave & 3, u)];
    } else {
#pragma unroll
        for (int t = 0; t < PD; t++)
#pragma unroll
            for (int u = 0; u < Loader::U; u++) blk_pro[t][u] = 0;
    }
    // one wait for all of them
    if constexpr (PD == 3 && Loader::U == 4)
        asm volatile("" ::"s"(n_raw), "s"(P_raw),
                     "s"(blk_pro[0][0]), "s"(blk_pro[0][1]), "s"(blk_pro[0][2]), "s"(blk_pro[0][3]),
                     "s"(blk_pro[1][0]), "s"(blk_pro[1][1]), "s"(blk_pro[1][2]), "s"(blk_pro[1][3]),
                     "s"(blk_pro[2][0]), "s"(blk_pro[2][1]), "s"(blk_pro[2][2]), "s"(blk_pro[2][3]));
    else if constexpr (PD == 2 && Loader::U == 4)
        asm volatile("" ::"s"(n_raw), "s"(P_raw),
                     "s"(blk_pro[0][0]), "s"(blk_pro[0][1]), "s"(blk_pro[0][2]), "s"(blk_pro[0][3]),
                     "s"(blk_pro[1][0]), "s"(blk_pro[1][1]), "s"(blk_pro[1][2]), "s"(blk_pro[1][3]));
    else if constexpr (PD == 1 && Loader::U == 4)
        asm volatile("" ::"s"(n_raw), "s"(P_raw),
                     "s"(blk_pro[0][0]), "s"(blk_pro[0][1]), "s"(blk_pro[0][2]), "s"(blk_pro[0][3]));
    else if constexpr (PD == 3 && Loader::U == 2)
        asm volatile("" ::"s"(n_raw), "s"(P_raw),
                     "s"(blk_pro[0][0]), "s"(blk_pro[0][1]),
                     "s"(blk_pro[1][0]), "s"(blk_pro[1][1]),
                     "s"(blk_pro[2][0]), "s"(blk_pro[2][1]));
    else if constexpr (PD == 2 && Loader::U == 2)
        asm volatile("" ::"s"(n_raw), "s"(P_raw),
                     "s"(blk_pro[0][0]), "s"(blk_pro[0][1]),
                     "s"(blk_pro[1][0]), "s"(blk_pro[1][1]));
    else
        asm volatile("" ::"s"(n_raw), "s"(P_raw),
                     "s"(blk_pro[0][0]), "s"(blk_pro[0][1]));

    const int n = clampi(n_raw, 0, p.T_max);
    const int P = clampi(P_raw, 0, p.P_max);
    const int nvalid = p.balanced ? share.nvalid : seq_nsplit(p, P);
    if (s >= nvalid) return;  // uniform over the workgroup
    const bool direct = (p.nsplit == 1);

    // The G * T_max query rows of a KV head are numbered r = k * G + g (node k, head-in-group g) and cut into
    // chunks of 32: a small tree fills whole MFMA tiles with rows of several heads instead of padding every
    // head to 32 rows.  Wavefront `wave` of row group `wg` owns chunk `pair`; with key halves (KH) a chunk
    // belongs to two wavefronts, wave and wave + NW/2, which take key block kb = 0 / 1 of every tile.
    constexpr int CW = KH ? NW / 2 : NW;  // chunks per workgroup
    const int kb = KH ? wave / CW : 0;
    const int pair = wg * CW + (KH ? wave % CW : wave);
    const bool active = pair < p.pairs;
    const int r = (active ? pair : 0) * 32 + c32;
    const int kq = r / p.G;              // the lane's node
    const int h = kvh * p.G + (r - kq * p.G);  // and query head
    // wavefront-uniform: does the chunk hold any valid row?  If not the wavefront only takes part in loads and barriers
    const bool wactive = active && pair * 32 < n * p.G;

    const int k0 = s * chunk, k1 = min(P, k0 + chunk);
    const int nfull = (k1 > k0) ? (k1 - k0) / KT : 0;               // full prefix tiles
    const int npt = (k1 > k0) ? (k1 - k0 + KT - 1) / KT : 0;        // prefix tiles incl. a ragged last one
    const int ntt = (s == nvalid - 1) ? (n + KT - 1) / KT : 0;      // tree tiles
    const int nt = npt + ntt;

    Loader ld;
    ld.kc = static_cast<const uint8_t *>(p.k_cache); ld.vc = static_cast<const uint8_t *>(p.v_cache);
    ld.kt = static_cast<const uint8_t *>(p.kt) + ((size_t)b * p.T_max * p.Hkv + kvh) * ROW_BYTES;
    ld.vt = static_cast<const uint8_t *>(p.vt) + ((size_t)b * p.T_max * p.Hkv + kvh) * ROW_BYTES;
    ld.bt = PAGED ? p.block_table + (size_t)b * p.max_blocks : nullptr;
    ld.row_stride = (size_t)p.Hkv * ROW_BYTES;
    ld.seq_off = ((size_t)b * p.P_cap * p.Hkv + kvh) * ROW_BYTES;   // contiguous cache: row 0 of (b, kvh)
    ld.blk_stride = (size_t)p.Hkv * 16 * ROW_BYTES;                  // paged cache: one block, all heads
    ld.head_off = (size_t)kvh * 16 * ROW_BYTES;
    ld.kf = ld.kc + (PAGED ? ld.head_off : ld.seq_off); ld.vf = ld.vc + (PAGED ? ld.head_off : ld.seq_off);
    ld.smem_addr = smem_addr; ld.wave = wave; ld.l_row = lane / Geo<D>::CPR; ld.l_pos = lane % Geo<D>::CPR;
    ld.k0 = k0; ld.k1 = k1; ld.npt = npt; ld.n = n; ld.P = P; ld.tail = (p.kt == nullptr);
    {
        // the lane's row within the 16 rows that pair `wave` + 4u covers, the same for every u
        const int r_in = Geo<D>::RPU * wave + ld.l_row;
        ld.kcol = (uint32_t)((ld.l_pos ^ kswz_of_row<D>(r_in)) * 16);
        ld.vcol = (uint32_t)((ld.l_pos ^ vswz_of_row<D>(r_in)) * 16);
        const uint32_t rowpart = PAGED ? (uint32_t)((r_in & 15) * ROW_BYTES) : (uint32_t)r_in * (uint32_t)ld.row_stride;
        ld.koff = rowpart + ld.kcol;
        ld.voff = rowpart + ld.vcol;
    }
    const bool issuer = wave < Loader::NI;
    // one workgroup per (split, KV head): nobody else reads these K/V bytes, so they are streamed past L2
    const bool stream_kv = p.wgp == 1;
    // prologue: fill the ring, then fetch Q and the mask row while those loads fly
#pragma unroll
    for (int t = 0; t < PD; t++) {
        if (t >= nt || !issuer) continue;
        if (t < nfull) {
            if (PAGED && !spec) fetch_blocks<D, NW>(ld, t, blk_pro[t]);
            if (stream_kv) issue_full_tile<D, NW, NS, PAGED, true>(ld, t, blk_pro[t]);
            else issue_full_tile<D, NW, NS, PAGED, false>(ld, t, blk_pro[t]);
        } else {
            issue_edge_tile<D, NW>(ld, t, t % NS);
        }
    }

    const uint16_t *qp = static_cast<const uint16_t *>(p.q);
    // Q as B operand: lane holds query row kq, d values 16*kk + 8*hh .. +7
    bf16x8 qreg[KK];
    uint64_t mbits0 = 0, mbits1 = 0, mbits2 = 0, mbits3 = 0;  // the row's ancestor bits, one word per tree tile
    const bool rv = active && kq < n;
    if (rv) {
        const uint64_t *mrow = p.bitmask + ((size_t)b * p.T_max + kq) * p.words;
        mbits0 = mrow[0];
        if (p.words > 1) mbits1 = mrow[1];
        if (p.words > 2) mbits2 = mrow[2];
        if (p.words > 3) mbits3 = mrow[3];
    }
#pragma unroll
    for (int kk = 0; kk < KK; kk++) {
        uint4 v = {0, 0, 0, 0};
        if (rv) v = *reinterpret_cast<const uint4 *>(qp + (((size_t)b * p.T_max + kq) * p.Hq + h) * D + 16 * kk + 8 * hh);
        qreg[kk] = __builtin_bit_cast(bf16x8, v);
    }

    f32x16 oacc[DB];
    float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int db = 0; db < DB; db++)
#pragma unroll
        for (int i = 0; i < 16; i++) oacc[db][i] = 0.f;

    // Q and the mask row must have arrived before the loop: a wait the compiler can see here keeps it from
    // placing a vmcnt(0) inside the loop, which would also drain the asynchronous tile loads every iteration
    wait_vmcnt<0>();

    // per-lane LDS offsets (bytes within a tile) that do not depend on the tile
    const int g16 = lane >> 4, i16 = lane & 15;
    const int vrow = 4 * hh + (i16 >> 2);  // V row within a 16-key step (second read: +8)
    TileView tv{c32 * ROW_BYTES, kswz_of_row<D>(c32), vrow, vswz_of_row<D>(vrow),
                2 * (g16 & 1) + ((i16 & 3) >> 1), 8 * (i16 & 1), hh};

    // Ring step: wait for tile ti, barrier, refill.  PD = tiles in flight behind the one being consumed.
    // With 8 wavefronts the V tile of step ti-1 is still being read by wavefronts 4..7 during step ti, so
    // the stage that is refilled is the one of tile ti-2.
    auto ring_step = [&](int ti) {
        const int tn = ti + PD;  // tile to issue in this step
        int blk[Loader::U];
        const bool full_next = issuer && tn < nfull;
        if (PAGED && full_next) fetch_blocks<D, NW>(ld, tn, blk);  // scalar loads fly during the wait below
        const int ahead = min(PD - 1, nt - 1 - ti);  // younger tiles whose loads may still be outstanding
        if (PD >= 3 && ahead >= 2) wait_vmcnt<2 * LPW>();
        else if (PD >= 2 && ahead == 1) wait_vmcnt<LPW>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();  // everyone's part of tile ti is in LDS; the refilled stage is no longer read
        asm volatile("" ::: "memory");
        if (full_next) {
            if (stream_kv) issue_full_tile<D, NW, NS, PAGED, true>(ld, tn, blk);
            else issue_full_tile<D, NW, NS, PAGED, false>(ld, tn, blk);
        }
        else if (issuer && tn < nt) issue_edge_tile<D, NW>(ld, tn, tn % NS);
    };
    auto tile_vis = [&](int ti) -> uint64_t {
        if (ti < npt) return (1ull << (k1 - k0 - nfull * KT)) - 1ull;  // ragged last prefix tile: 1..63 keys
        const int w = ti - npt;                                         // tree tile: the row's ancestor bits
        const uint64_t lo = (w & 1) ? mbits1 : mbits0, hi = (w & 1) ? mbits3 : mbits2;
        return (w & 2) ? hi : lo;
    };
    bf16x8 pf[Geo<D>::NP][2][2];        // whole tiles: [part][key block][16-key step]
    bf16x8 pfh[Geo<D>::NP][2];          // key halves: [part][16-key step]
    // one tile for one wavefront, in two parts (the parts run in different ring steps for late wavefronts)
    auto part_qk = [&](int t, bool masked) {
        const uint8_t *lk = smem + (t % NS) * STAGE_BYTES;
        if (KH) {
            const uint32_t v32 = masked ? (uint32_t)(tile_vis(t) >> (32 * kb)) : ~0u;
            if (masked) qk_softmax_half<D, true>(tv, lk, kb, qreg, oacc, m_run, l_run, p.scale_log2, v32, pfh);
            else qk_softmax_half<D, false>(tv, lk, kb, qreg, oacc, m_run, l_run, p.scale_log2, v32, pfh);
        } else {
            if (masked) qk_softmax<D, true>(tv, lk, qreg, oacc, m_run, l_run, p.scale_log2, tile_vis(t), pf);
            else qk_softmax<D, false>(tv, lk, qreg, oacc, m_run, l_run, p.scale_log2, ~0ull, pf);
        }
    };
    bool ill = false;
    auto part_pv = [&](int t, bool masked) {
        const uint8_t *lv = smem + (t % NS) * STAGE_BYTES + TILE_BYTES;
        if (KH) pv_accumulate_half<D>(tv, lv, kb, pfh, oacc, masked, ill);
        else pv_accumulate<D>(tv, lv, pf, oacc, masked, ill);
    };
    int ti = 0;
    if (!kShifted || wave < 4) {
        // QK(t), softmax(t), PV(t) within ring step t
        for (; ti < nfull; ti++) {  // full prefix tiles: no masking code at all
            ring_step(ti);
            if (!wactive) continue;
            part_qk(ti, false);
            part_pv(ti, false);
        }
        for (; ti < nt; ti++) {     // ragged last prefix tile and tree tiles
            ring_step(ti);
            if (!wactive) continue;
            part_qk(ti, true);
            part_pv(ti, true);
        }
    } else {
        // one phase behind: PV(t-1), QK(t), softmax(t) within ring step t; the last PV after the loop
        for (; ti < nfull; ti++) {
            ring_step(ti);
            if (!wactive) continue;
            if (ti > 0) part_pv(ti - 1, false);
            part_qk(ti, false);
        }
        for (; ti < nt; ti++) {
            ring_step(ti);
            if (!wactive) continue;
            if (ti > 0) part_pv(ti - 1, ti > nfull);
            part_qk(ti, true);
        }
        if (nt > 0 && wactive) part_pv(nt - 1, nt > nfull);
    }
    if constexpr (D == 64) {
        if (ill) {
            uint64_t up[1] = {0}, down[1] = {0};
            for (int t = nfull; t < nt; t++) {
                const bool tree = t >= npt;
                const int base = tree ? (t - npt) * KT : k0 + t * KT, count = min(KT, (tree ? n : k1) - base);
                const uint64_t own = KH ? 0xffffffffull << (32 * kb) : ~0ull;  // the keys that this wavefront takes
                find_nonfinite<uint16_t, D>(p, b, kvh, P, tree, base, count, rv ? tile_vis(t) & own : 0, up, down);
            }
            add_nonfinite(oacc, up[0], down[0], hh);
        }
    }

    if (KH) {
        // Merge the two key halves of a chunk through LDS (the ring is no longer needed): the kb = 1
        // wavefront hands its (m, l, O) to its kb = 0 partner, which rescales both to the larger reference.
        __builtin_amdgcn_s_barrier();  // every wavefront has finished reading tiles; no tile load is outstanding
        asm volatile("" ::: "memory");
        float4 *mx = reinterpret_cast<float4 *>(smem) + (size_t)(wave % CW) * ((4 * DB + 1) * 64);
        if (kb == 1 && wactive) {
#pragma unroll
            for (int db = 0; db < DB; db++)
#pragma unroll
                for (int ig = 0; ig < 4; ig++)
                    mx[(4 * db + ig) * 64 + lane] = float4{oacc[db][4 * ig], oacc[db][4 * ig + 1], oacc[db][4 * ig + 2], oacc[db][4 * ig + 3]};
            mx[4 * DB * 64 + lane] = float4{m_run, l_run, 0.f, 0.f};
        }
        __syncthreads();
        if (kb == 1) return;
        if (wactive) {
            const float4 ml = mx[4 * DB * 64 + lane];
            const float m_new = fmaxf(m_run, ml.x);
            const float fa = (m_run == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
            const float fb = (ml.x == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(ml.x - m_new);
            m_run = m_new;
            l_run = l_run * fa + ml.y * fb;
#pragma unroll
            for (int db = 0; db < DB; db++)
#pragma unroll
                for (int ig = 0; ig < 4; ig++) {
                    const float4 o = mx[(4 * db + ig) * 64 + lane];
                    oacc[db][4 * ig] = oacc[db][4 * ig] * fa + o.x * fb;
                    oacc[db][4 * ig + 1] = oacc[db][4 * ig + 1] * fa + o.y * fb;
                    oacc[db][4 * ig + 2] = oacc[db][4 * ig + 2] * fa + o.z * fb;
                    oacc[db][4 * ig + 3] = oacc[db][4 * ig + 3] * fa + o.w * fb;
                }
        }
    }

    // ---- epilogue
    if (!active || kq >= p.T_max) return;
    uint16_t *out = static_cast<uint16_t *>(p.out);
    const float l_tot = half_swap_sum(l_run);
    const size_t lrow = ((size_t)b * p.Hq + h) * p.T_max + kq;
    if (direct) {
        const size_t orow = (((size_t)b * p.T_max + kq) * p.Hq + h) * D;
        const float inv = rv ? 1.f / l_tot : 0.f;
#pragma unroll
        for (int db = 0; db < DB; db++)
#pragma unroll
            for (int ig = 0; ig < 4; ig++) {
                const int dcol = 32 * db + 8 * ig + 4 * hh;
                uint2 w;
                w.x = rv ? pack_bf16x2(oacc[db][4 * ig] * inv, oacc[db][4 * ig + 1] * inv) : 0u;
                w.y = rv ? pack_bf16x2(oacc[db][4 * ig + 2] * inv, oacc[db][4 * ig + 3] * inv) : 0u;
                *reinterpret_cast<uint2 *>(out + orow + dcol) = w;
            }
        if (p.lse && hh == 0) p.lse[lrow] = rv ? (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2 : -INFINITY;
    } else if (rv) {
        const size_t pr = part_row(p, p.balanced ? (int)blockIdx.x : b * p.nsplit + s, h, kq);
#pragma unroll
        for (int db = 0; db < DB; db++)
#pragma unroll
            for (int ig = 0; ig < 4; ig++) {
                const int dcol = 32 * db + 8 * ig + 4 * hh;
                float4 w = {oacc[db][4 * ig], oacc[db][4 * ig + 1], oacc[db][4 * ig + 2], oacc[db][4 * ig + 3]};
                *reinterpret_cast<float4 *>(p.part_o + pr * D + dcol) = w;
            }
        if (hh == 0) {
            p.part_m[pr] = m_run;
            p.part_l[pr] = l_tot;
        }
    }
}

// ----------------------------------------------------------------------------------------------
// Wide kernel (bf16, d = 128): trees of many rows over long splits.
//
// Work unit: (split, KV head x group of 256 rows, sequence), one workgroup of four wavefronts, one per SIMD; wavefront w owns the
// 32-row chunks w and w + 4, so that a fragment of K or V is read from LDS once for 64 rows, and one chunk's softmax runs between
// the matrix instructions of the other.  Swizzles and register layouts are those of attn_mfma_kernel, four ring places of 32 KiB
// and three tiles in flight.  The loop over the tiles is written by attn_wide_loop.py.
//
// What bounds a tile is the power.  With 32x32x16 matrix instructions it took 2574 cycles, 2176 of them matrix instructions, and the
// clock was 1.48 GHz with everything in the loop, 1.67 without the tile loads, 1.78 with the matrix instructions alone: 1.73, 1.55
// and 1.23 us.  The 16x16x32 instructions that it has now cost the same cycles and less power, but leave fewer issue slots beside
// them (2 against 3 for the same product), so the streams are paced by slots.  B = 32, P = 4096, 32/8 heads: T = 128 288-295 us on the
// tile kernel, 255 here with 32x32x16, 249 with 16x16x32, 242-256 paced (two rounds of workgroups; of a round's 122 us about 13 are
// start-up, the first references and the output); T = 32, one chunk a wavefront, 100.6-103.2 -> 91.4-95.5.  B = 1, T = 128, P = 32768 with
// its combine: 83.5-84.7 -> 74.0-78.1.  Against the eight wavefronts of attn_mfma_kernel a round costs 4 us more and a tile a quarter less.
// Peaked scores: every row that moves its reference stops the matrix cores (`lift` in attn_wide_loop.py has the figures).
// ----------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(32))) float f32x32;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;

struct WideGeo {
    static constexpr int NW = 4, CW = 8, NS = 4, AHEAD = 3;  // wavefronts, chunks, ring places, tiles asked for before the loop
    static constexpr int MASKED = 3;                         // tiles with masked keys that the loop takes (its asm names three masks)
    static constexpr int RING = NS * Geo<128>::STAGE_BYTES;
    static constexpr int Q_AT = 3 * Geo<128>::STAGE_BYTES;   // Q until the loop has read it: 16 KiB a wavefront
    static constexpr int OUT_AT = RING;                      // outputs on their way to memory: 8 KiB a wavefront
    static constexpr int LDS = RING + NW * 8192;             // all 160 KiB of a compute unit
};

// form: nodes of a tree (16 bits), splits shared out by length (1), a single split (1), sequences if shared out (8)
static uint32_t wide_form(const AttnParams &p) {
    return (uint32_t)p.T_max | (p.balanced ? 1u : 0u) << 16 | (p.nsplit == 1 ? 1u : 0u) << 17 | (p.balanced ? (uint32_t)p.B : 0u) << 18;
}

template <bool PAGED, bool NT, bool MANY>
__global__ void __launch_bounds__(256, 1)
attn_wide_kernel(const int32_t *prefix_len, const int32_t *n_nodes, const uint64_t *bitmask, const int32_t *block_table, uint32_t Hkv,
                 uint32_t inv_hkv, uint32_t G, uint32_t inv_g, int max_blocks, uint32_t form, AttnParams p) {
    constexpr int D = 128, AHEAD = WideGeo::AHEAD, MASKED = WideGeo::MASKED;
    constexpr int ROW_BYTES = Geo<D>::ROW_BYTES, TILE_BYTES = Geo<D>::TILE_BYTES, STAGE_BYTES = Geo<D>::STAGE_BYTES;
    uint8_t *const smem = attn_smem;
    const uint32_t smem_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)attn_smem;

    // grid, shares of a ragged batch and the rotation of the split index: as in attn_mfma_kernel
    const int T_max = (int)(form & 0xffffu);
    const bool balanced = (form >> 16 & 1u) != 0, single = (form >> 17 & 1u) != 0;
    uint32_t rem;
    const int wg = (int)fast_div(blockIdx.y, Hkv, inv_hkv, rem), kvh = (int)rem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    SplitShare share{};
    int s_ = 0, chunk_ = 0;
    if (balanced) {
        share = balanced_share(p, prefix_len, n_nodes, (int)(form >> 18), (int)blockIdx.x, lane);
        if (!share.live) return;  // uniform over the workgroup
        if (share.j == 0 && blockIdx.y == 0 && tid == 0) p.split_tab[share.b] = make_int2(share.start, share.nvalid);
        s_ = share.j;
        chunk_ = share.tps * KT;
    } else if (!single) {
        asm volatile("" ::"s"(p.nsplit), "s"(p.inv_nsplit), "s"(p.chunk));  // nobody else waits for these
        fast_div(blockIdx.x + blockIdx.z, (uint32_t)p.nsplit, p.inv_nsplit, rem);
        s_ = (int)rem;
        chunk_ = p.chunk;
    }
    const int b = uni(balanced ? share.b : (int)blockIdx.z), s = uni(s_);
    const int k0 = uni(s * chunk_);
    const const_i32_ptr bt = (const_i32_ptr)(uintptr_t)(PAGED ? block_table + (size_t)b * max_blocks : nullptr);
    // One trip for the other arguments, the sizes, the wavefront's blocks of the first full tiles (read before it is known whether the
    // prefix reaches that far, used only if it does) and the ancestor bits of the lane's four rows.
    const int lb0 = (k0 >> 4) + wave;
    const bool spec = PAGED && (k0 >> 4) + 4 * AHEAD <= max_blocks;
    int blk0 = 0, blk1 = 0, blk2 = 0;
    if (spec) {
        blk0 = bt[lb0];
        blk1 = bt[lb0 + 4];
        blk2 = bt[lb0 + 8];
    }
    const int n_raw = balanced ? share.n_raw : ((const_i32_ptr)(uintptr_t)n_nodes)[b];
    const int P_raw = balanced ? share.P_raw : ((const_i32_ptr)(uintptr_t)prefix_len)[b];
    // The 64 packed rows r = k * G + g (node k, head g of the group) of the wavefront's two chunks, lane i working out row i.
    struct Row { int kq; uint32_t at; bool in_launch; };  // at: byte offset of the row in its sequence's part of Q and of the output (below
                                                          // 2^32: at most 256 nodes of 65536 heads)
    const int pairs = (int)((G * (uint32_t)T_max + 31) >> 5);  // 32-row chunks of a KV head
    auto own_row = [&](int l) -> Row {
        const int pair = wg * WideGeo::CW + wave + WideGeo::NW * (l >> 5);
        uint32_t g;
        const int kq = (int)fast_div((uint32_t)(pair * 32 + (l & 31)), G, inv_g, g);
        return {kq, ((uint32_t)kq * Hkv * G + (uint32_t)kvh * G + g) * ROW_BYTES, pair < pairs && kq < T_max};
    };
    // The lane's own four rows: of chunk x the rows lane % 16 (y = 0) and 16 + lane % 16 (y = 1).
    auto own_four = [&](int l, uint32_t v, uint32_t (&of)[2][2]) {
#pragma unroll
        for (int x = 0; x < 2; x++)
#pragma unroll
            for (int y = 0; y < 2; y++) of[x][y] = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (32 * x + 16 * y + (l & 15)), (int)v);
    };
    const Row row = own_row(lane);
    uint32_t kq_of[2][2];
    own_four(lane, row.in_launch ? (uint32_t)row.kq : 0xffffffffu, kq_of);  // no row there: no node
    // ancestor bits of these rows, the first two words (with MANY: read where they are needed); of rows that are not there node 0's
    uint64_t bits0[2][2] = {{0, 0}, {0, 0}}, bits1[2][2] = {{0, 0}, {0, 0}};
    const uint32_t words = (uint32_t)(T_max + 63) >> 6;
    if constexpr (!MANY) {
        const uint64_t *const mask = bitmask + (size_t)b * T_max * words;
        const uint32_t second = words > 1 ? 1 : 0;
#pragma unroll
        for (int x = 0; x < 2; x++)
#pragma unroll
            for (int y = 0; y < 2; y++) {
                const uint32_t at = (kq_of[x][y] == 0xffffffffu ? 0u : kq_of[x][y]) * words;
                bits0[x][y] = mask[at];
                bits1[x][y] = mask[at + second];
            }
    }
    asm volatile("" ::"s"(n_raw), "s"(P_raw), "s"(blk0), "s"(blk1), "s"(blk2), "s"(p.q), "s"(p.k_cache), "s"(p.v_cache), "s"(p.kt), "s"(p.vt),
                 "s"(p.P_cap), "s"(p.P_max), "s"(p.chunk), "s"(p.inv_chunk), "s"(p.scale_log2));
    asm volatile("" ::"v"(bits0[0][0]), "v"(bits0[0][1]), "v"(bits0[1][0]), "v"(bits0[1][1]), "v"(bits1[0][0]), "v"(bits1[0][1]),
                 "v"(bits1[1][0]), "v"(bits1[1][1]));
    const int n = uni(clampi(n_raw, 0, T_max)), P = uni(clampi(P_raw, 0, p.P_max));
    const int chunk = uni(single ? p.chunk : chunk_);
    const int nvalid = uni(balanced ? share.nvalid : single ? 1 : max(1, (int)fast_div((uint32_t)(P + chunk - 1), (uint32_t)chunk, p.inv_chunk, rem)));
    if (s >= nvalid) return;  // uniform over the workgroup
    const bool direct = single;

    const int k1 = min(P, k0 + chunk);
    const int nfull = (k1 > k0) ? (k1 - k0) / KT : 0;
    const int npt = (k1 > k0) ? (k1 - k0 + KT - 1) / KT : 0;
    const int ntt = (s == nvalid - 1) ? (n + KT - 1) / KT : 0;
    const int edges = npt - nfull + ntt;  // tiles with masked keys: edge e is tile nfull + e of the split

    const bool tail = (p.kt == nullptr);
    const size_t row_stride = (size_t)Hkv * ROW_BYTES, blk_stride = row_stride * 16;  // both below 2^32
    const size_t head_at = PAGED ? (size_t)kvh * 16 * ROW_BYTES : ((size_t)b * p.P_cap * Hkv + kvh) * ROW_BYTES;
    const uint8_t *const kf = static_cast<const uint8_t *>(p.k_cache) + head_at, *const vf = static_cast<const uint8_t *>(p.v_cache) + head_at;
    const size_t tree_at = ((size_t)b * T_max * Hkv + kvh) * ROW_BYTES;
    // the lane, anew: what is worked out from it for use ahead of and behind the loop is not kept in registers during it
    auto again = [&]() -> int {
        int l = lane;
        asm volatile("" : "+v"(l));
        return l;
    };
    // A wavefront brings rows 16 w .. 16 w + 15 of a tile (of a full one: one cache block), four rows a load.  The lane's source
    // columns under the swizzles: load j holds rows 4 j + lane / 16 of the 16.
    struct Columns { uint32_t k[4], v[2]; };
    auto columns = [&](int l) -> Columns {
        Columns c;
#pragma unroll
        for (int j = 0; j < 4; j++) c.k[j] = (uint32_t)(((l & 15) ^ kswz_of_row<D>(4 * j + (l >> 4))) * 16);
#pragma unroll
        for (int j = 0; j < 2; j++) c.v[j] = (uint32_t)(((l & 15) ^ vswz_of_row<D>(4 * j + (l >> 4))) * 16);
        return c;
    };
    u32x4 koff, voff;  // full tiles: the lane's pieces relative to the block
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const Columns c = columns(lane);
        const uint32_t at = (uint32_t)(4 * j + (lane >> 4)) * (PAGED ? (uint32_t)ROW_BYTES : (uint32_t)row_stride);
        koff[j] = at + c.k[j];
        voff[j] = at + c.v[j & 1];
    }
    const uint32_t lds_wave = smem_addr + (uint32_t)wave * 4096;
    auto full_offset = [&](int t, int id) -> size_t {
        return PAGED ? (size_t)(uint32_t)uni(id) * (size_t)(uint32_t)blk_stride
                     : (size_t)(uint32_t)(k0 + t * KT + 16 * wave) * (size_t)(uint32_t)row_stride;
    };
    // The loads of a tile: all of K, then all of V (the loop counts on the order).
    auto issue_full = [&](size_t off, int place) {
        const uint32_t dst = lds_wave + (uint32_t)place * STAGE_BYTES;
#pragma unroll
        for (int j = 0; j < 4; j++) async_load16_s<NT>(kf + off, koff[j], dst + j * 1024);
#pragma unroll
        for (int j = 0; j < 4; j++) async_load16_s<NT>(vf + off, voff[j], dst + TILE_BYTES + j * 1024);
    };
    // Edge e: rows past the end repeat the last one.
    auto issue_edge = [&](int e, int place) {
        const uint32_t dst = lds_wave + (uint32_t)place * STAGE_BYTES;
        const int w = nfull + e - npt;  // tree tile, or -1: the ragged end of the prefix
        const int l = again(), r0 = 16 * wave + (l >> 4);
        const Columns col = columns(l);
        uint32_t at[4];
        if (w >= 0 && !tail) {  // the step's own tree buffer
            const uint8_t *const kt = static_cast<const uint8_t *>(p.kt) + tree_at, *const vt = static_cast<const uint8_t *>(p.vt) + tree_at;
#pragma unroll
            for (int j = 0; j < 4; j++) at[j] = (uint32_t)min(w * KT + r0 + 4 * j, n - 1) * (uint32_t)row_stride;
#pragma unroll
            for (int j = 0; j < 4; j++) async_load16_s<false>(kt, at[j] + col.k[j], dst + j * 1024);
#pragma unroll
            for (int j = 0; j < 4; j++) async_load16_s<false>(vt, at[j] + col.v[j & 1], dst + TILE_BYTES + j * 1024);
            return;
        }
        // cache positions pos0 .. last; an in-place branch cache has node j at position P + j
        const int pos0 = w >= 0 ? P + w * KT : k0 + nfull * KT, last = w >= 0 ? P + n - 1 : k1 - 1;
        if (!PAGED) {
            const size_t off = (size_t)(uint32_t)pos0 * (size_t)(uint32_t)row_stride;
#pragma unroll
            for (int j = 0; j < 4; j++) at[j] = (uint32_t)min(r0 + 4 * j, last - pos0) * (uint32_t)row_stride;
#pragma unroll
            for (int j = 0; j < 4; j++) async_load16_s<false>(kf + off, at[j] + col.k[j], dst + j * 1024);
#pragma unroll
            for (int j = 0; j < 4; j++) async_load16_s<false>(vf + off, at[j] + col.v[j & 1], dst + TILE_BYTES + j * 1024);
            return;
        }
        // 16 positions in a row lie in two blocks at most
        const int i0 = uni(min(pos0 + 16 * wave, last) >> 4), i1 = uni(min(i0 + 1, last >> 4));
        const int id0 = bt[i0], id1 = bt[i1];
        const size_t b0 = (size_t)(uint32_t)uni(id0) * blk_stride, b1 = (size_t)(uint32_t)uni(id1) * blk_stride;
        size_t off[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int pos = min(pos0 + r0 + 4 * j, last);
            off[j] = ((pos >> 4) == i0 ? b0 : b1) + (uint32_t)(pos & 15) * ROW_BYTES;
        }
#pragma unroll
        for (int j = 0; j < 4; j++) async_load16(kf + off[j] + col.k[j], dst + j * 1024);
#pragma unroll
        for (int j = 0; j < 4; j++) async_load16(vf + off[j] + col.v[j & 1], dst + TILE_BYTES + j * 1024);
    };
    // keys of edge e that a row of the lane sees, those of its part of the wavefront: bit 4 kb + i for key 16 kb + 4 (lane / 16) + i;
    // a row that is not there sees all, so that its sums stay finite
    auto edge_vis = [&](int x, int y, int e, int l) -> uint32_t {
        const int w = nfull + e - npt;
        uint64_t vis = (1ull << (k1 - k0 - nfull * KT)) - 1ull;
        if (w >= 0) {
            if constexpr (MANY) {
                vis = 0;
                if (kq_of[x][y] != 0xffffffffu) vis = bitmask[((size_t)b * T_max + kq_of[x][y]) * words + w];
            } else {
                vis = (w & 1) ? bits1[x][y] : bits0[x][y];
            }
        }
        if (kq_of[x][y] >= (uint32_t)n) return 0xffffu;
        const uint32_t lo = (uint32_t)vis >> (4 * (l >> 4)), hi = (uint32_t)(vis >> 32) >> (4 * (l >> 4));
        return (lo & 15u) | ((lo >> 12) & 0xf0u) | ((hi & 15u) << 8) | ((hi >> 4) & 0xf000u);
    };

    // Q, 1 KiB a load, laid out like K rows, to the ring's last place and the space behind it; rows that are not there repeat
    // node 0's.  A sequence without keys reads none: it has no pass of the loop, whose barriers keep a wavefront's Q apart from the
    // outputs that others stage in the same LDS.
    if (edges + nfull > 0) {
        const uint8_t *const qseq = reinterpret_cast<const uint8_t *>(uni64((uint64_t)(uintptr_t)p.q + (size_t)b * T_max * (int)(Hkv * G) * ROW_BYTES));
        const uint32_t from = row.in_launch && row.kq < n ? row.at : (uint32_t)(kvh * (int)G) * ROW_BYTES;
        const Columns c = columns(lane);
        uint32_t at[16];
#pragma unroll
        for (int u = 0; u < 16; u++) at[u] = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (4 * u + (lane >> 4)), (int)from);
#pragma unroll
        for (int u = 0; u < 16; u++)
            async_load16_s<false>(qseq, at[u] + c.k[u & 3], smem_addr + WideGeo::Q_AT + (uint32_t)wave * 16384 + u * 1024);
    }

    f32x32 oa0, oa1, ob0, ob1;  // zeroed by the first pass of the loop, beside its first products
    f32x4 nm = {INFINITY, INFINITY, INFINITY, INFINITY}, sum = {0.f, 0.f, 0.f, 0.f};  // minus the references (-inf so far), sums
    // The order of work: a full tile, whose maximum is the rows' first reference (over the few nodes that a row sees of the tree
    // it would be farther from the largest score, and the largest probability is exact only where it is 1), the tiles with masked
    // keys, the other full tiles.  The loop wants masked tiles among its first three: with a ragged end of the prefix ahead of two
    // tree tiles that one leads, and trees of more than 128 nodes take a pass for the first three tiles (it does not touch Q's place).
    const bool lead_full = nfull > 0 && !(edges == MASKED && npt > nfull);
    // (MANY: trees of more than 128 nodes.  Without a second pass the outputs stay in accumulation registers on the way.)
    int e_done = 0, f_done = 0;
    bool again_pass = edges + nfull > 0;
#pragma unroll 1
    while (again_pass) {
        const uint32_t done = uni(e_done + f_done);
        // chunk `wave` of the group and chunk `wave` + 4 (a small group is spread over the SIMDs): how many of them hold rows?
        const uint32_t chunks = uni((int)((wg * WideGeo::CW + wave) * 32 < n * (int)G) + (int)((wg * WideGeo::CW + wave + WideGeo::NW) * 32 < n * (int)G));
        const int lead = lead_full && f_done == 0 ? 1 : 0, e_left = edges - e_done;
        const bool more = MANY && e_left > MASKED - lead;  // not the last pass
        const int ne = more ? (lead ? MASKED - 1 : e_left - MASKED) : e_left, masked = lead + ne, nt = masked + (more ? 0 : nfull - f_done - lead);
        const int l = again();
        u32x2 vis[MASKED];  // visible keys of the first tiles for chunk A and chunk B, two rows of 16 bits each
#pragma unroll
        for (int e = 0; e < MASKED; e++)
#pragma unroll
            for (int x = 0; x < 2; x++) {
                vis[e][x] = 0xffffffffu;
                if (e >= lead && e < masked) vis[e][x] = edge_vis(x, 0, e_done + e - lead, l) | edge_vis(x, 1, e_done + e - lead, l) << 16;
            }
#pragma unroll 1
        for (int c = 0; c < AHEAD; c++) {
            if (c >= lead && c < masked) {
                issue_edge(e_done + c - lead, c);
            } else if (c < nt) {
                const int t = f_done + (c < lead ? 0 : c - ne);  // 0, 1, 2
                int id = t == 0 ? blk0 : (t == 1 ? blk1 : blk2);
                if (PAGED && !spec) id = bt[lb0 + 4 * t];
                issue_full(full_offset(t, id), c);
            }
        }
        const int l16 = l & 15, g = l >> 4, vrow = 4 * g + (l16 >> 2);
        u32x4 kaddr, vaddr;
#pragma unroll
        for (int ds = 0; ds < 4; ds++) kaddr[ds] = smem_addr + l16 * ROW_BYTES + (((4 * ds + g) ^ kswz_of_row<D>(l16)) << 4);
#pragma unroll
        for (int db = 0; db < 4; db++)
            vaddr[db] = smem_addr + vrow * ROW_BYTES + 8 * (l16 & 1) + (((2 * db + ((l16 & 3) >> 1)) ^ vswz_of_row<D>(vrow)) << 4);
        uint32_t left = uni(nt), n_masked = uni(masked), idx = uni(f_done + AHEAD - ne);  // idx: the loop's fourth tile among the full ones
        uint64_t off = PAGED ? 0 : uni64(full_offset((int)idx, 0));
        const uint32_t last_full = uni(nfull - 1);
        const uint64_t ids = uni64((uint64_t)(uintptr_t)bt + (PAGED ? 4 * (uint64_t)lb0 : 0));
        const uint64_t kbase = uni64((uint64_t)(uintptr_t)kf), vbase = uni64((uint64_t)(uintptr_t)vf);
        const uint32_t stride = uni(PAGED ? (int)blk_stride : (int)(KT * row_stride));
        const uint32_t lds_wave_s = uni(lds_wave), q_off = uni(WideGeo::Q_AT + wave * 16384);
#define ETV_WIDE(LOOP) \
        asm volatile(LOOP : "+{a[0:31]}"(oa0), "+{a[32:63]}"(oa1), "+{a[64:95]}"(ob0), "+{a[96:127]}"(ob1), \
                     "+{v[208:211]}"(kaddr), "+{v[212:215]}"(vaddr), "+{v[224:227]}"(nm), "+{v[228:231]}"(sum), \
                     "+{v[240:241]}"(vis[0]), "+{v[242:243]}"(vis[1]), "+{v[244:245]}"(vis[2]), "+{s40}"(left), "+{s68}"(n_masked), \
                     "+{s[48:49]}"(off), "+{s59}"(idx) \
                     : "{v[216:219]}"(koff), "{v[220:223]}"(voff), "{s53}"(last_full), "{s69}"(done), "{s70}"(chunks), "{s[54:55]}"(ids), "{s[60:61]}"(kbase), "{s[62:63]}"(vbase), \
                       "{s64}"(stride), "{s65}"(lds_wave_s), "{s66}"(p.scale_log2), "{s67}"(q_off) \
                     : ETV_WIDE_CLOBBERS)
        if constexpr (PAGED && NT) ETV_WIDE(ETV_WIDE_LOOP_PAGED_NT);
        else if constexpr (PAGED) ETV_WIDE(ETV_WIDE_LOOP_PAGED);
        else if constexpr (NT) ETV_WIDE(ETV_WIDE_LOOP_FLAT_NT);
        else ETV_WIDE(ETV_WIDE_LOOP_FLAT);
#undef ETV_WIDE
        e_done += ne;
        f_done += nt - ne;
        again_pass = more;
        if (more) __builtin_amdgcn_s_barrier();  // nobody reads the places any more
    }

    wait_vmcnt<0>();  // nothing on its way to LDS is left behind
    // ---- outputs, through the wavefront's own 8 KiB of LDS so that whole rows (of a group: neighbours) go out together:
    // 32 rows of 16 pieces of 16 bytes, piece c of row r at c ^ (r % 16)
    uint8_t *const oseq = static_cast<uint8_t *>(p.out) + (size_t)b * T_max * (int)(Hkv * G) * ROW_BYTES;
    uint8_t *const stage = smem + WideGeo::OUT_AT + wave * 8192;
    const int l2 = again(), piece = l2 & 15, sub = l2 >> 4;
    const Row row2 = own_row(l2);
    uint32_t kq2[2][2], at2[2][2];
    own_four(l2, row2.in_launch ? (uint32_t)row2.kq : 0xffffffffu, kq2);
    own_four(l2, row2.at, at2);
    // piece c of the lane's row y (rows lane % 16 and 16 + lane % 16: the same swizzle)
    const uint32_t own = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)stage + piece * 256 + (piece << 4);
    auto put = [&](int y, int c) -> uint8_t * {
        return (uint8_t *)(__attribute__((address_space(3))) uint8_t *)(uintptr_t)((own ^ (c << 4)) + y * 4096);
    };
    auto send = [&](int x, uint32_t from, auto &&dst) {  // dst(v): where the 16 pieces of a row go whose lane has v = from
        wait_lds_reads();  // the pieces are in LDS
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const int r_in = 4 * i + sub;
            const uint32_t at = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (32 * x + r_in), (int)from);
            const uint4 v = *reinterpret_cast<const uint4 *>(stage + r_in * 256 + ((piece ^ (r_in & 15)) << 4));
            if (at != 0xffffffffu) *reinterpret_cast<uint4 *>(dst(at) + piece * 16) = v;
        }
        wait_lds_reads();  // the place may be written again
    };
#pragma unroll
    for (int x = 0; x < 2; x++) {
        if (wg * WideGeo::CW + wave + WideGeo::NW * x >= pairs) break;  // uniform over the wavefront
        const f32x32 &o0 = x ? ob0 : oa0, &o1 = x ? ob1 : oa1;
        auto o = [&](int i) { return i < 32 ? o0[i & 31] : o1[i & 31]; };  // 4 (2 db + y) + i: column 16 db + 4 (lane / 16) + i of row y
        float l_tot[2];
        bool valid[2];
#pragma unroll
        for (int y = 0; y < 2; y++) {
            valid[y] = kq2[x][y] < (uint32_t)n;
            l_tot[y] = quarter_swap_sum(half_swap_sum(sum[2 * x + y]));
        }
        auto head = [&](int y) { return at2[x][y] / ROW_BYTES - kq2[x][y] * (int)(Hkv * G); };
        if (direct) {
            const bool whole = __all(valid[0] && valid[1]);  // else padded rows: zeros
#pragma unroll
            for (int y = 0; y < 2; y++) {
                const float inv = 1.f / l_tot[y];
#pragma unroll
                for (int db = 0; db < 8; db++) {
                    const int at = 4 * (2 * db + y);
                    uint2 w = {pack_bf16x2(o(at) * inv, o(at + 1) * inv), pack_bf16x2(o(at + 2) * inv, o(at + 3) * inv)};
                    if (!whole) w = valid[y] ? w : uint2{0u, 0u};
                    *reinterpret_cast<uint2 *>(put(y, 2 * db + (sub >> 1)) + 8 * (sub & 1)) = w;
                }
            }
            send(x, row2.in_launch ? row2.at : 0xffffffffu, [&](uint32_t at) { return oseq + at; });
            if (p.lse && sub == 0)
#pragma unroll
                for (int y = 0; y < 2; y++)
                    if (kq2[x][y] != 0xffffffffu)
                        p.lse[((size_t)b * (int)(Hkv * G) + head(y)) * T_max + kq2[x][y]] =
                            valid[y] ? (-nm[2 * x + y] + __builtin_amdgcn_logf(l_tot[y])) * kLn2 : -INFINITY;
        } else {
            // rows of the slot's partials: head, then node
            const size_t slot_row = part_row(p, balanced ? (int)blockIdx.x : b * p.nsplit + s, 0, 0);
            float *const part = p.part_o + slot_row * D;
            const uint32_t prow = (row2.at / ROW_BYTES - row2.kq * (int)(Hkv * G)) * T_max + row2.kq;
#pragma unroll
            for (int hf = 0; hf < 2; hf++) {  // half a row of fp32 each time
#pragma unroll
                for (int y = 0; y < 2; y++)
#pragma unroll
                    for (int d4 = 0; d4 < 4; d4++) {
                        const int at = 4 * (2 * (4 * hf + d4) + y);
                        *reinterpret_cast<float4 *>(put(y, 4 * d4 + sub)) = float4{o(at), o(at + 1), o(at + 2), o(at + 3)};
                    }
                send(x, row2.in_launch && row2.kq < n ? prow : 0xffffffffu,
                     [&](uint32_t at) { return reinterpret_cast<uint8_t *>(part + (size_t)at * D + 64 * hf); });
            }
            if (sub == 0)
#pragma unroll
                for (int y = 0; y < 2; y++)
                    if (valid[y]) {
                        const size_t pr = slot_row + head(y) * T_max + kq2[x][y];
                        p.part_m[pr] = -nm[2 * x + y];
                        p.part_l[pr] = l_tot[y];
                    }
        }
    }
}

// ----------------------------------------------------------------------------------------------
// Key-block kernel (bf16, d = 128 or 64): launches that are short of work.
//
// Work unit: (split, KV head, sequence) x 32-row chunk of the KV head's packed query rows, one workgroup of eight
// wavefronts.  attn_mfma_kernel shares a tile among the chunks of a workgroup and walks through a split tile by tile, a
// barrier and a whole chain (fragment reads, products, softmax, products) per 64 keys; where a split is a handful of
// tiles that chain and the extra splits that keep the chip busy are all there is to its time.  Here every wavefront takes
// 32-key blocks of its own (block t goes to wavefront t % 8), so a workgroup has 256 keys in flight at once, there is no
// barrier in the loop, and the eight (m, l, O) merge once through LDS: the same keys need an eighth of the steps, and
// fewer splits.  The price is that K/V are fetched once per chunk instead of once per workgroup of chunks; the chunks of
// one (split, KV head, sequence) get ids that differ by 8, so they run side by side on one XCD and all but the first
// reader find the bytes in its L2.
//
// A wavefront owns a K and a V buffer of one block each (8 KiB + 8 KiB at d = 128), filled by direct-to-LDS loads: K of
// the next block is requested when the score products have read this one's, V when the value products have.  Q (one
// copy for the workgroup) and the rows' ancestor bits come the same way, so that nothing the compiler tracks is
// outstanding and no wait of its own drains the block loads.
//
// Start-up is a third of a short launch, so it is one trip to memory: what the first addresses need are leading scalar arguments,
// which are in registers when the kernel starts (the -amdgpu-kernarg-preload-count of the build), and the sequence's sizes, the
// first block ids and the other arguments are asked for together.  K of the first block goes out first, then Q, then V.  The
// loads of a block with masked keys know their block ids beforehand too (a look-up per lane and load kept these wavefronts from the
// first barrier for 2.3 us).  Whether K/V bytes have one reader and whether the split slots follow the lengths are template
// arguments: a branch per load, and a wait for the arguments before the sizes are asked for, otherwise.
// What bounds a step is the LDS pipe (K and V written, read once for 32 rows: 256 KiB per compute unit and step) and, with one chunk, the
// latency of the next block.  Behind the start-up a launch of two or three steps is a chain of instructions, one every 3.5 ns: the
// fragments of a product are all read before the first of its instructions (the compiler takes them two by two and waits each time), zeros
// and LDS addresses are ready before the sizes arrive, K of the next block is asked for beside the products of this one, and the merge reads all
// eight outputs without a branch (wavefronts without a block leave zeros), also where there are one or two blocks.
//
// Against the tile kernel: B = 1, 32/8 heads of 128, T = 60, P = 2048 16.1 -> 12.0 us (4 splits instead of 8); B = 32, T = 8,
// P = 4096 87.4 -> 82 (128 KiB in flight per compute unit: 6.6 TB/s).  The start-up and the chain, against three trips and
// fragments two by two: 32 layers of B = 1, T = 60, P = 2048 510 -> 421 us (with the combine launches); heads of 64, B = 4, T = 48,
// P = 900 ... 1500 13.3 -> 11.25; B = 1, T = 4 ... 60, P = 0 ... 40 5.4 ... 6.0 -> 5.1 ... 5.5, P = 200 7.7 ... 9.5 -> 6.5 ... 7.4.
// ----------------------------------------------------------------------------------------------
constexpr int KB_NW = 8;     // wavefronts of a workgroup
constexpr int KB_KEYS = 32;  // keys of a block

template <int D>
struct KbGeo {
    static constexpr int BLOCK = KB_KEYS * Geo<D>::ROW_BYTES;  // K (or V) bytes of a block: 8 or 4 KiB
    static constexpr int U = BLOCK / 1024;                     // 1 KiB loads of a block: 8 or 4
    static constexpr int Q_AT = KB_NW * 2 * BLOCK;             // LDS: wavefront buffers, Q, ancestor bits, (m, l)
    static constexpr int BITS_AT = Q_AT + BLOCK;               // 4 words x 32 rows x 8 B
    static constexpr int ML_AT = BITS_AT + 4 * 256;
    static constexpr int LDS = ML_AT + KB_NW * 32 * 8;         // 139 KiB (one workgroup per compute unit) or 71 KiB (two)
};

// 4 bytes per lane from global memory straight into LDS at (lds_addr + 4 * lane); asynchronous.
__device__ __forceinline__ void async_load4(const void *gptr, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off\n" ::"v"(gptr),
                 "s"(__builtin_amdgcn_readfirstlane(lds_addr)) : "memory");
}

template <int D, bool PAGED, bool BALANCED, bool NT>
__global__ void __launch_bounds__(KB_NW * 64, D == 64 ? 4 : 2)
attn_blocks_kernel(const int32_t *prefix_len, const int32_t *n_nodes, const int32_t *block_table, int Hkv, uint32_t inv_hkv, int slots, int nsplit,
                   uint32_t inv_nsplit, int max_blocks, int chunk_, uint32_t inv_chunk, AttnParams p) {
    using G_ = KbGeo<D>;
    constexpr int ROW_BYTES = Geo<D>::ROW_BYTES, KK = Geo<D>::KK, DB = Geo<D>::DB, RPU = Geo<D>::RPU, CPR = Geo<D>::CPR;
    constexpr int BLOCK = G_::BLOCK, U = G_::U, UH = U / 2;  // UH loads cover 16 rows
    constexpr int VP = D == 128 ? 2 : 1;                     // the V swizzle of a load repeats with this period
    uint8_t *const smem = attn_smem;
    const uint32_t smem_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)attn_smem;
    const int tid = threadIdx.x, lane = tid & 63, c32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // grid (8, chunks, units / 8): the linear id is ((unit / 8) * chunks + chunk) * 8 + unit % 8, unit = slot * Hkv + KV head
    const int rg = blockIdx.y;
    uint32_t rem;
    const int slot = (int)fast_div(blockIdx.z * 8 + blockIdx.x, Hkv, inv_hkv, rem);
    const int kvh = (int)rem;
    if (slot >= slots) return;  // uniform over the workgroup
    SplitShare share{};
    if constexpr (BALANCED) {
        share = balanced_share(p, slot, lane);
        if (!share.live) return;  // uniform over the workgroup
    }
    const int slot_b = (int)fast_div(slot, nsplit, inv_nsplit, rem);
    const int b = uni(BALANCED ? share.b : slot_b), s = BALANCED ? share.j : (int)rem, chunk = BALANCED ? share.tps * KT : chunk_;
    const int k0 = s * chunk;
    const const_i32_ptr bt = (const_i32_ptr)(uintptr_t)(PAGED ? block_table + (size_t)b * max_blocks : nullptr);
    // One trip for the sizes, the other arguments and the two cache blocks of the wavefront's first key block; those ids are
    // read before it is known whether the prefix reaches that far (inside the table in any case), and used only if it does.
    const int lb0 = (k0 >> 4) + 2 * wave;
    int blk0 = 0, blk1 = 0;
    if (PAGED) {
        blk0 = bt[min(lb0, max_blocks - 1)];
        blk1 = bt[min(lb0 + 1, max_blocks - 1)];
    }
    const int n_raw = BALANCED ? share.n_raw : ((const_i32_ptr)(uintptr_t)n_nodes)[b];
    const int P_raw = BALANCED ? share.P_raw : ((const_i32_ptr)(uintptr_t)prefix_len)[b];
    // Ready before the sizes are: the views of the wavefront's buffers, as in the tile kernel, and zeros.
    const int g16 = lane >> 4, i16 = lane & 15;
    const int vrow = 4 * hh + (i16 >> 2);
    const TileView tv{c32 * ROW_BYTES, kswz_of_row<D>(c32), vrow, vswz_of_row<D>(vrow),
                      2 * (g16 & 1) + ((i16 & 3) >> 1), 8 * (i16 & 1), hh};
    const uint8_t *const lk = smem + wave * (2 * BLOCK), *const lv = lk + BLOCK;
    f32x16 oacc[DB];
    float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int db = 0; db < DB; db++)
#pragma unroll
        for (int i = 0; i < 16; i++) oacc[db][i] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; db++) asm volatile("" : "+v"(oacc[db]));
    asm volatile("" ::"s"(n_raw), "s"(P_raw), "s"(blk0), "s"(blk1), "s"(p.q), "s"(p.k_cache), "s"(p.v_cache), "s"(p.kt), "s"(p.vt),
                 "s"(p.bitmask), "s"(p.T_max), "s"(p.Hq), "s"(p.G), "s"(p.inv_g), "s"(p.P_cap), "s"(p.P_max), "s"(p.words), "s"(p.scale_log2));
    const int n = clampi(n_raw, 0, p.T_max), P = clampi(P_raw, 0, p.P_max);
    const int nvalid = BALANCED ? share.nvalid : max(1, (int)fast_div(P + chunk - 1, chunk, inv_chunk, rem));
    if (s >= nvalid) return;  // uniform over the workgroup
    const bool direct = (nsplit == 1);
    const bool active = rg * 32 < n * p.G;  // does the chunk hold a valid row?
    const int k1 = min(P, k0 + chunk);
    const int nfull = (active && k1 > k0) ? (k1 - k0) >> 5 : 0;     // full prefix blocks
    const int npb = (active && k1 > k0) ? (k1 - k0 + 31) >> 5 : 0;  // prefix blocks incl. a ragged last one
    const bool with_tree = active && s == nvalid - 1;
    const int nt = npb + (with_tree ? (n + 31) >> 5 : 0);

    const uint8_t *const kc = static_cast<const uint8_t *>(p.k_cache), *const vc = static_cast<const uint8_t *>(p.v_cache);
    const auto mul = [](uint32_t x, uint32_t y) { return (uint64_t)x * y; };
    const uint32_t hstride = (uint32_t)Hkv * ROW_BYTES;  // between the rows of a head (contiguous cache, tree buffer)
    const uint32_t blk_stride = 16 * hstride;
    const uint64_t head_at = PAGED ? (uint64_t)((uint32_t)kvh * 16 * ROW_BYTES) : mul(b, p.P_cap) * hstride + (uint32_t)kvh * ROW_BYTES;
    const uint32_t rstride = PAGED ? (uint32_t)ROW_BYTES : hstride;
    const uint32_t kbuf = smem_addr + (uint32_t)wave * (2 * BLOCK), vbuf = kbuf + BLOCK;
    const int l_row = lane / CPR, l_pos = lane % CPR;
    // chunk-position swizzles as in the tile kernel: load u covers rows RPU * u + l_row of the block
    uint32_t koff[UH], voff[VP];
#pragma unroll
    for (int x = 0; x < UH; x++) koff[x] = l_row * rstride + (l_pos ^ kswz_of_row<D>(RPU * x + l_row)) * 16;
#pragma unroll
    for (int x = 0; x < VP; x++) voff[x] = l_row * rstride + (l_pos ^ vswz_of_row<D>(RPU * x + l_row)) * 16;
    // The cache blocks that key block x lies in: two, or three where the tree rows begin anywhere (in-place branch cache).
    auto block_ids = [&](int x, int &i0, int &i1, int &i2) {
        if (PAGED && !(x >= npb && p.kt)) {
            const int first = (x >= npb ? P + (x - npb) * KB_KEYS : k0 + x * KB_KEYS) >> 4, last = (x >= npb ? P + n - 1 : k1 - 1) >> 4;
            i0 = bt[first];
            i1 = bt[min(first + 1, last)];
            i2 = bt[min(first + 2, last)];
        }
    };
    auto issue_full = [&](int x, int i0, int i1, int i2, const uint8_t *cache, uint32_t dst, bool is_v) {
        const uint8_t *b0 = cache + head_at + (PAGED ? mul(uni(i0), blk_stride) : mul(k0 + x * KB_KEYS, hstride));
        const uint8_t *b1 = PAGED ? cache + head_at + mul(uni(i1), blk_stride) : b0 + blk_stride;
#pragma unroll
        for (int u = 0; u < U; u++)
            async_load16_s<NT>((u < UH ? b0 : b1) + (uint32_t)((u % UH) * RPU) * rstride, is_v ? voff[u % VP] : koff[u % UH], dst + u * 1024);
    };
    // Ragged last prefix block and tree blocks: rows past the end repeat the last valid one (masked later).  The block ids are
    // there already, so that no load of the loop waits for another.
    auto issue_edge = [&](int x, int i0, int i1, int i2, const uint8_t *cache, const void *own_rows, uint32_t dst, bool is_v) {
        const bool tree = x >= npb;
        const int base = tree ? (x - npb) * KB_KEYS : k0 + x * KB_KEYS;
        const int last = (tree ? n : k1) - 1 - base;
        const bool own = tree && own_rows;
        const int pos = tree ? P + base : base;  // in-place branch cache: node j at position P + j
        if (!PAGED || own) {
            const uint8_t *src = own ? static_cast<const uint8_t *>(own_rows) + mul(b * p.T_max + base, hstride) + (uint32_t)kvh * ROW_BYTES
                                     : cache + head_at + mul(pos, hstride);
#pragma unroll 1
            for (int u = 0; u < U; u++) {
                const int r = RPU * u + l_row;
                async_load16_s<false>(src, min(r, last) * hstride + (l_pos ^ (is_v ? vswz_of_row<D>(r) : kswz_of_row<D>(r))) * 16,
                                      dst + u * 1024);
            }
        } else {
            const uint8_t *src = cache + head_at;
#pragma unroll 1
            for (int u = 0; u < U; u++) {
                const int r = RPU * u + l_row, at = (pos & 15) + min(r, last);
                const int blk = at < 16 ? i0 : (at < 32 ? i1 : i2);
                async_load16(src + mul(blk, blk_stride) + ((at & 15) * ROW_BYTES + (l_pos ^ (is_v ? vswz_of_row<D>(r) : kswz_of_row<D>(r))) * 16),
                             dst + u * 1024);
            }
        }
    };
    auto issue = [&](int x, int i0, int i1, int i2, bool is_v) {
        if (x < nfull) issue_full(x, i0, i1, i2, is_v ? vc : kc, is_v ? vbuf : kbuf, is_v);
        else issue_edge(x, i0, i1, i2, is_v ? vc : kc, is_v ? p.vt : p.kt, is_v ? vbuf : kbuf, is_v);
    };

    // K of the first block, then Q and the ancestor bits, then V: the first products wait for all but V.
    int t = wave;
    if (active) {
        int i0 = blk0, i1 = blk1, i2 = 0;
        if (t < nt) {
            if (t >= npb) block_ids(t, i0, i1, i2);
            issue(t, i0, i1, i2, false);
        }
        // Q, 1 KiB per wavefront, laid out like a K block; padded rows repeat node 0's (their results are dropped)
        if (wave < U) {
            const int row = RPU * wave + l_row;
            int kq = (int)fast_div(rg * 32 + row, p.G, p.inv_g, rem), h = kvh * p.G + (int)rem;
            if (kq >= n) { kq = 0; h = kvh * p.G; }
            async_load16(static_cast<const uint8_t *>(p.q) + (((size_t)b * p.T_max + kq) * p.Hq + h) * ROW_BYTES +
                             (l_pos ^ kswz_of_row<D>(row)) * 16, smem_addr + G_::Q_AT + wave * 1024);
        }
        if (with_tree && wave < p.words) {  // word `wave` of the ancestor bits of the 32 rows
            int kq = (int)fast_div(rg * 32 + (lane >> 1), p.G, p.inv_g, rem);
            if (kq >= n) kq = 0;
            async_load4(reinterpret_cast<const uint32_t *>(p.bitmask + ((size_t)b * p.T_max + kq) * p.words + wave) + (lane & 1),
                        smem_addr + G_::BITS_AT + wave * 256);
        }
        if (t < nt) {
            issue(t, i0, i1, i2, true);
            wait_vmcnt<U>();
        } else {
            wait_vmcnt<0>();
        }
    }
    __builtin_amdgcn_s_barrier();  // Q and the ancestor bits are in LDS
    asm volatile("" ::: "memory");

    auto block_vis = [&](int x) {  // keys of block x that the lane's row sees
        uint32_t vis = ~0u;
        if (x >= npb) vis = *reinterpret_cast<const uint32_t *>(smem + G_::BITS_AT + ((x - npb) >> 1) * 256 + c32 * 8 + ((x - npb) & 1) * 4);
        else if (x >= nfull) vis = (1u << (k1 - k0 - x * KB_KEYS)) - 1u;  // ragged last prefix block: 1..31 keys
        return vis;
    };
    bool ill = false;
    if (t < nt) {
        bf16x8 qreg[KK];
        const uint8_t *lq = smem + G_::Q_AT + c32 * ROW_BYTES;
#pragma unroll
        for (int kk = 0; kk < KK; kk++) qreg[kk] = *reinterpret_cast<const bf16x8 *>(lq + (((2 * kk + hh) ^ tv.ksw) << 4));
        for (; t < nt; t += KB_NW) {
            const int tn = t + KB_NW;
            int i0 = 0, i1 = 0, i2 = 0;
            if (tn < nt) block_ids(tn, i0, i1, i2);  // they fly during this block's products
            wait_vmcnt<U>();  // K of block t (V may still be on its way)
            asm volatile("" ::: "memory");
            bf16x8 pf[Geo<D>::NP][2];
            // one copy of the code for masked and unmasked blocks: a launch this short pays for every instruction it fetches
            const uint32_t vis = block_vis(t);
            qk_softmax_half<D, true>(tv, lk, 0, qreg, oacc, m_run, l_run, p.scale_log2, vis, pf, t >= nfull, [&] {
                wait_lds_reads();
                if (tn < nt) issue(tn, i0, i1, i2, false);
            });
            if (tn < nt) wait_vmcnt<U>();  // V of block t (K of the next one may still be on its way)
            else wait_vmcnt<0>();
            asm volatile("" ::: "memory");
            pv_accumulate_half<D, true>(tv, lv, 0, pf, oacc, t >= nfull, ill);
            wait_lds_reads();
            if (tn < nt) issue(tn, i0, i1, i2, true);
        }
    }

    if constexpr (D == 64) {
        if (ill) {
            uint64_t up[1] = {0}, down[1] = {0};
            for (int x = nfull + ((wave - nfull) & (KB_NW - 1)); x < nt; x += KB_NW) {  // the masked ones of the wavefront's blocks
                const bool tree = x >= npb;
                const int base = tree ? (x - npb) * KB_KEYS : k0 + x * KB_KEYS, count = min(KB_KEYS, (tree ? n : k1) - base);
                find_nonfinite<uint16_t, D>(p, b, kvh, P, tree, base, count, block_vis(x), up, down);
            }
            add_nonfinite(oacc, up[0], down[0], hh);
        }
    }

    // ---- merge the wavefronts: each leaves O in its own K/V buffers (same size), 16-byte piece c of row r at c ^ r
    constexpr int CH = D / 4;  // 16-byte pieces of an fp32 output row
    float2 *const ml = reinterpret_cast<float2 *>(smem + G_::ML_AT);
    {
        const float l_tot = half_swap_sum(l_run);
        float4 *dst = reinterpret_cast<float4 *>(smem + wave * (2 * BLOCK)) + c32 * CH;
#pragma unroll
        for (int db = 0; db < DB; db++)
#pragma unroll
            for (int ig = 0; ig < 4; ig++)
                dst[(8 * db + 2 * ig + hh) ^ (c32 & (CH - 1))] =
                    float4{oacc[db][4 * ig], oacc[db][4 * ig + 1], oacc[db][4 * ig + 2], oacc[db][4 * ig + 3]};
        if (hh == 0) ml[wave * 32 + c32] = float2{m_run, l_tot};
    }
    __syncthreads();
    if (BALANCED && share.j == 0 && kvh == 0 && rg == 0 && tid == 0) p.split_tab[b] = make_int2(share.start, share.nvalid);
    const int row = tid >> 4, piece = tid & 15;  // a row's 16 threads own pieces `piece` and (d = 128) piece + 16
    const int kq2 = (int)fast_div(rg * 32 + row, p.G, p.inv_g, rem), h2 = kvh * p.G + (int)rem;
    if (kq2 >= p.T_max) return;
    const bool rv = kq2 < n;
    if (!rv && !direct) return;
    // all reads of the statistics in one trip, then all reads of the outputs, without a branch: a wavefront without a block left zeros
    float2 e[KB_NW];
    float M = -INFINITY, L = 0.f;
#pragma unroll
    for (int x = 0; x < KB_NW; x++) e[x] = ml[x * 32 + row];
#pragma unroll
    for (int x = 0; x < KB_NW; x++) {
        M = fmaxf(M, e[x].x);
    }
    float4 acc[D / 64];
#pragma unroll
    for (int v = 0; v < D / 64; v++) acc[v] = float4{0.f, 0.f, 0.f, 0.f};
    const auto add = [&](int x, const float4 (&o)[D / 64]) {
        const float w = e[x].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(e[x].x - M);
        L = fmaf(w, e[x].y, L);
#pragma unroll
        for (int v = 0; v < D / 64; v++) {
            acc[v].x = fmaf(w, o[v].x, acc[v].x); acc[v].y = fmaf(w, o[v].y, acc[v].y);
            acc[v].z = fmaf(w, o[v].z, acc[v].z); acc[v].w = fmaf(w, o[v].w, acc[v].w);
        }
    };
#pragma unroll
    for (int x = 0; x < KB_NW; x++) {
        float4 o[D / 64];
#pragma unroll
        for (int v = 0; v < D / 64; v++) o[v] = reinterpret_cast<const float4 *>(smem + x * (2 * BLOCK))[row * CH + ((piece + 16 * v) ^ (row & (CH - 1)))];
        add(x, o);
    }
    if (direct) {
        uint16_t *orow = static_cast<uint16_t *>(p.out) + (((size_t)b * p.T_max + kq2) * p.Hq + h2) * D;
        const float inv = rv ? 1.f / L : 0.f;
#pragma unroll
        for (int v = 0; v < D / 64; v++) {
            uint2 w = {0u, 0u};
            if (rv) {
                w.x = pack_bf16x2(acc[v].x * inv, acc[v].y * inv);
                w.y = pack_bf16x2(acc[v].z * inv, acc[v].w * inv);
            }
            *reinterpret_cast<uint2 *>(orow + 4 * (piece + 16 * v)) = w;
        }
        if (p.lse && piece == 0) p.lse[((size_t)b * p.Hq + h2) * p.T_max + kq2] = rv ? (M + __builtin_amdgcn_logf(L)) * kLn2 : -INFINITY;
    } else {
        const size_t pr = part_row(p, slot, h2, kq2);
#pragma unroll
        for (int v = 0; v < D / 64; v++) *reinterpret_cast<float4 *>(p.part_o + pr * D + 4 * (piece + 16 * v)) = acc[v];
        if (piece == 0) {
            p.part_m[pr] = M;
            p.part_l[pr] = L;
        }
    }
}

// ----------------------------------------------------------------------------------------------
// fp32 kernel (d = 128 or 64): both products on v_mfma_f32_16x16x4_f32, which multiplies and adds in fp32.
//
// Work unit: (split, KV head, sequence) x 16-row chunk of the KV head's packed query rows, one workgroup of four
// wavefronts that take the 16-key tiles of the split in turn and merge their (m, l, O) through LDS at the end.  No tile
// is shared inside a workgroup, so the loop has no barrier.  A wavefront owns a K and a V buffer of one tile each, filled by
// direct-to-LDS loads: K of the next tile is requested when the score products' operand is in registers, V when the value products'
// is, so that each has most of a tile to arrive.  (The K operand wants a different row in each of 16 neighbouring lanes, which the
// vector memory path serves at a quarter of its rate; Q, the same way, is fetched once for the workgroup.)  As on the key-block
// kernel the start-up is one trip to memory for the sizes, the first block ids and the arguments, and nothing in the loop waits for
// a look-up.
// The chunks of one (split, KV head, sequence) re-read its K/V; their ids differ by 8, so they run side by side
// on one XCD and find it in that XCD's L2.  Where there is one chunk, the loads stream past L2.
// What bounds it: a tile is 64 matrix instructions, 0.86 us at d = 128 (0.43 at 64); two wavefronts of a SIMD take 1.0 us a tile
// each, a lone one 1.3, so the plan fills two workgroups per compute unit.  The wavefronts of a SIMD only gain from each other while one
// multiplies and the other does not: without a priority of the products some of the kernel's forms ran them in step, others not
// (B = 4, T = 120, 8/2 heads of 128, P = 9397, two equal splits: paged 174 us, contiguous 189, paged with shares by length 191; now 170 ...
// 171), and with V read behind the softmax a lone wavefront took 1.47 us (B = 2, T = 100, 8/8 heads, P = 12000 292 us, now 276 ... 279).  The
// same loads spread between the matrix
// instructions left V and K half the time to arrive (1.77 us a tile of a lone wavefront); eight wavefronts a workgroup in place of
// two workgroups were 2 ... 4 % faster in launches that leave the chip idle and 7 % slower in large ones.
//
// 64-lane layouts of the 16x16x4 instruction: A / B operand lane = (row | col l % 16, contraction index l / 16),
// accumulator lane = (col l % 16, rows 4 * (l / 16) + i).  With c = l % 16, g = l / 16:
//   S^T[key, q]: A = K[c][16 j + 4 g + e], B = Q[c][16 j + 4 g + e], e = 0..3 from one 16-byte load
//   O^T[d, q]:   B = p[i] of key 4 g + i straight from the S^T accumulator, A = V[4 g + i][64 v + 4 c + e], e = 0..3 from
//                one 16-byte load: accumulator (v, e) holds columns d = 64 v + 4 * row + e
// so a query row is a lane column in both, and only the row maximum crosses lanes (c, g) -> (c, g').
//
// Against V straight to registers, K one tile ahead in LDS, and three trips to memory before the first load: B = 2, T = 33, 16/4
// heads of 128, P = 771 / 1003 18.8 -> 16.6 us (graph of calls); B = 1, T = 8, 8/8 heads, P = 300 10.2 -> 7.7; T = 1, 8/2 heads, P =
// 16384 17.9 -> 15.4; B = 12, T = 20, 32/32 heads of 64, P = 150 14.4 -> 12.7; B = 2, T = 200, 16/4 heads, P = 300 31.7 -> 27.8;
// B = 16, T = 128, P = 2048, 32/8 heads of 128 657 -> 627, 113 TFLOP/s (the library's fp32 matrix product reaches 144 ... 154 on
// this machine).
// ----------------------------------------------------------------------------------------------

__device__ __forceinline__ float quad_max(float v) {  // over the lanes c, c + 16, c + 32, c + 48
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

constexpr int F32_NW = 4;    // wavefronts of a workgroup
constexpr int F32_GRID_Y = 32768;  // units / 8 of the grid's second dimension; the third has the rest
constexpr int F32_ROWS = 16; // query rows of a chunk = keys of a tile

template <int D>
struct F32Geo {
    static constexpr int NW = F32_NW;
    static constexpr int ROWB = 4 * D, TILE = F32_ROWS * ROWB;  // bytes of a K (V, Q, output) row and of 16 of them: 8 or 4 KiB
    static constexpr int CPR = ROWB / 16, RPL = 64 / CPR;       // 16-byte pieces of a row, rows of a 1 KiB load
    static constexpr int LOADS = TILE / 1024;                   // 1 KiB loads of a tile: 8 or 4
    static constexpr int Q_AT = NW * 2 * TILE;                  // LDS: wavefront buffers, Q, ancestor bits, (m, l)
    static constexpr int BITS_AT = Q_AT + TILE;                 // 4 words x 32 x 8 B (16 rows, twice)
    static constexpr int ML_AT = BITS_AT + 4 * 256;
    static constexpr int LDS = ML_AT + NW * F32_ROWS * 8;
};

template <int D, bool PAGED, bool BALANCED, bool NT>
__global__ void __launch_bounds__(F32_NW * 64, 2)
attn_f32_kernel(const int32_t *prefix_len, const int32_t *n_nodes, const int32_t *block_table, int Hkv, uint32_t inv_hkv, int slots, int nsplit,
                uint32_t inv_nsplit, int max_blocks, int chunk_, uint32_t inv_chunk, AttnParams p) {
    using G_ = F32Geo<D>;
    constexpr int NW = F32_NW, KJ = D / 16, VB = D / 64, ROWB = G_::ROWB, TILE = G_::TILE, CPR = G_::CPR, RPL = G_::RPL, LOADS = G_::LOADS;
    uint8_t *const smem = attn_smem;
    const uint32_t smem_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)attn_smem;
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // grid (8 * chunks, units / 8, its rest): the linear id is ((unit / 8) * chunks + chunk) * 8 + unit % 8, unit = slot * Hkv + KV head
    const int rg = blockIdx.x >> 3;
    uint32_t rem;
    const int slot = (int)fast_div((blockIdx.z * F32_GRID_Y + blockIdx.y) * 8 + (blockIdx.x & 7), Hkv, inv_hkv, rem);
    const int kvh = (int)rem;
    if ((uint32_t)slot >= (uint32_t)slots) return;  // uniform over the workgroup
    SplitShare share{};
    if constexpr (BALANCED) {
        share = balanced_share(p, slot, lane);
        if (!share.live) return;  // uniform over the workgroup
    }
    const int slot_b = (int)fast_div(slot, nsplit, inv_nsplit, rem);
    const int b = uni(BALANCED ? share.b : slot_b), s = BALANCED ? share.j : (int)rem, chunk = BALANCED ? share.tps * KT : chunk_;
    const int k0 = s * chunk;
    const const_i32_ptr bt = (const_i32_ptr)(uintptr_t)(PAGED ? block_table + (size_t)b * max_blocks : nullptr);
    // One trip for the sizes, the other arguments and the cache block of the wavefront's first tile, which is read before it is known
    // whether the prefix reaches that far (inside the table in any case), and used only if it does.
    int blk0 = 0;
    if (PAGED) blk0 = bt[min((k0 >> 4) + wave, max_blocks - 1)];
    const int n_raw = BALANCED ? share.n_raw : ((const_i32_ptr)(uintptr_t)n_nodes)[b];
    const int P_raw = BALANCED ? share.P_raw : ((const_i32_ptr)(uintptr_t)prefix_len)[b];
    asm volatile("" ::"s"(n_raw), "s"(P_raw), "s"(blk0), "s"(p.q), "s"(p.k_cache), "s"(p.v_cache), "s"(p.kt), "s"(p.vt), "s"(p.bitmask),
                 "s"(p.T_max), "s"(p.Hq), "s"(p.G), "s"(p.inv_g), "s"(p.P_cap), "s"(p.P_max), "s"(p.words), "s"(p.scale_log2), "s"(p.stagger));
    // The two workgroups of a compute unit share its matrix cores evenly and end together, and where a third follows, some compute units
    // then take two of these while as many take none (3, 4 and 2 workgroups on 228, 14 and 14).  With the second 32 of an XCD 3 us
    // late the ends lie apart.
    if (p.stagger && ((int)blockIdx.y * p.stagger + rg) >> 5 == 1) __builtin_amdgcn_s_sleep(127);
    const int n = clampi(n_raw, 0, p.T_max), P = clampi(P_raw, 0, p.P_max);
    const int nvalid = BALANCED ? share.nvalid : max(1, (int)fast_div(P + chunk - 1, chunk, inv_chunk, rem));
    if (s >= nvalid) return;  // uniform over the workgroup
    const bool direct = (nsplit == 1);
    const bool active = rg * F32_ROWS < n * p.G;  // does the chunk hold a valid row?
    const int k1 = min(P, k0 + chunk);
    const int nfull = (active && k1 > k0) ? (k1 - k0) >> 4 : 0;     // full prefix tiles
    const int npt = (active && k1 > k0) ? (k1 - k0 + 15) >> 4 : 0;  // prefix tiles incl. a ragged last one
    const bool with_tree = active && s == nvalid - 1;
    const int nt = npt + (with_tree ? (n + 15) >> 4 : 0);

    const uint8_t *const kc = static_cast<const uint8_t *>(p.k_cache), *const vc = static_cast<const uint8_t *>(p.v_cache);
    const auto mul = [](uint32_t x, uint32_t y) { return (uint64_t)x * y; };
    const uint32_t hstride = (uint32_t)Hkv * ROWB;  // between the rows of a head (contiguous cache, tree buffer)
    const uint32_t blk_stride = 16 * hstride;
    const uint64_t head_at = PAGED ? (uint64_t)((uint32_t)kvh * 16 * ROWB) : mul(b, p.P_cap) * hstride + (uint32_t)kvh * ROWB;
    const uint32_t rstride = PAGED ? (uint32_t)ROWB : hstride;
    // A 1 KiB load covers RPL rows, 64 / RPL lanes each.  16-byte piece x of row r of K (and of Q) is kept at position x ^ r, which
    // spreads the reads of 16 rows at one piece over all banks; V is read in whole rows and lies as it comes.
    const uint32_t kbuf = smem_addr + (uint32_t)wave * (2 * TILE), vbuf = kbuf + TILE;
    const int l_row = lane / CPR, l_pos = lane % CPR;
    uint32_t koff[LOADS];
#pragma unroll
    for (int u = 0; u < LOADS; u++) koff[u] = l_row * rstride + (l_pos ^ (RPL * u + l_row)) * 16;
    const uint32_t voff = l_row * rstride + l_pos * 16;
    // The cache blocks that tile x lies in: one, or two where the tree rows begin anywhere (in-place branch cache).
    auto block_ids = [&](int x, int &i0, int &i1) {
        if (PAGED) {
            const int first = x >= npt ? (P + (x - npt) * F32_ROWS) >> 4 : (k0 >> 4) + x;
            i0 = bt[min(first, max_blocks - 1)];
            i1 = bt[min(first + 1, max_blocks - 1)];
        }
    };
    auto issue_full = [&](int x, int i0, const uint8_t *cache, uint32_t dst, bool is_v) {
        const uint8_t *src = cache + head_at + (PAGED ? mul(uni(i0), blk_stride) : mul(k0 + x * F32_ROWS, hstride));
#pragma unroll
        for (int u = 0; u < LOADS; u++) async_load16_s<NT>(src + (uint32_t)(RPL * u) * rstride, is_v ? voff : koff[u], dst + u * 1024);
    };
    // Ragged last prefix tile and tree tiles: rows past the end repeat the last valid one (masked later).
    auto issue_edge = [&](int x, int i0, int i1, const uint8_t *cache, const void *own_rows, uint32_t dst, bool is_v) {
        const bool tree = x >= npt;
        const int base = tree ? (x - npt) * F32_ROWS : k0 + x * F32_ROWS;
        const int last = (tree ? n : k1) - 1 - base;
        const bool own = tree && own_rows;
        const int pos = tree ? P + base : base;  // in-place branch cache: node j at position P + j
        if (!PAGED || own) {
            const uint8_t *src = own ? static_cast<const uint8_t *>(own_rows) + mul(b * p.T_max + base, hstride) + (uint32_t)kvh * ROWB
                                     : cache + head_at + mul(pos, hstride);
#pragma unroll
            for (int u = 0; u < LOADS; u++) {
                const int r = RPL * u + l_row;
                async_load16_s<false>(src, min(r, last) * hstride + (is_v ? l_pos : l_pos ^ r) * 16, dst + u * 1024);
            }
        } else {
            const uint8_t *src = cache + head_at;
#pragma unroll
            for (int u = 0; u < LOADS; u++) {
                const int r = RPL * u + l_row, at = (pos & 15) + min(r, last);
                async_load16(src + mul(at < 16 ? i0 : i1, blk_stride) + ((at & 15) * ROWB + (is_v ? l_pos : l_pos ^ r) * 16), dst + u * 1024);
            }
        }
    };
    auto issue = [&](int x, int i0, int i1, bool is_v) {
        if (x < nfull) issue_full(x, i0, is_v ? vc : kc, is_v ? vbuf : kbuf, is_v);
        else issue_edge(x, i0, i1, is_v ? vc : kc, is_v ? p.vt : p.kt, is_v ? vbuf : kbuf, is_v);
    };

    // K of the first tile, then Q and the ancestor bits, then V: the first products wait for all but V.
    int t = wave, i0 = blk0, i1 = 0;
    if (active) {
        if (t < nt) {
            if (t >= npt) block_ids(t, i0, i1);
            issue(t, i0, i1, false);
        }
        // Q, laid out like a K tile; padded rows repeat node 0's (their results are dropped)
#pragma unroll
        for (int u = wave; u < LOADS; u += NW) {
            const int row = RPL * u + l_row;
            int kq = (int)fast_div(rg * F32_ROWS + row, p.G, p.inv_g, rem), h = kvh * p.G + (int)rem;
            if (kq >= n) { kq = 0; h = kvh * p.G; }
            async_load16(static_cast<const uint8_t *>(p.q) + (((size_t)b * p.T_max + kq) * p.Hq + h) * ROWB + (l_pos ^ row) * 16,
                         smem_addr + G_::Q_AT + u * 1024);
        }
        if (with_tree && wave < p.words) {  // word `wave` of the ancestor bits of the 16 rows
            int kq = (int)fast_div(rg * F32_ROWS + ((lane >> 1) & 15), p.G, p.inv_g, rem);
            if (kq >= n) kq = 0;
            async_load4(reinterpret_cast<const uint32_t *>(p.bitmask + ((size_t)b * p.T_max + kq) * p.words + wave) + (lane & 1),
                        smem_addr + G_::BITS_AT + wave * 256);
        }
        if (t < nt) {
            issue(t, i0, i1, true);
            if (t + NW < nt) block_ids(t + NW, i0, i1);
            wait_vmcnt<LOADS>();
        } else {
            wait_vmcnt<0>();
        }
    }
    __builtin_amdgcn_s_barrier();  // Q and the ancestor bits are in LDS
    asm volatile("" ::: "memory");

    const uint8_t *const lk = smem + wave * (2 * TILE), *const lv = lk + TILE;
    f32x4 qf[KJ], o[VB][4];
    float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
    for (int v = 0; v < VB; v++)
#pragma unroll
        for (int e = 0; e < 4; e++) o[v][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto tile_vis = [&](int x) -> uint32_t {  // keys of tile x that the lane's row sees
        if (x < nfull) return 0xffffu;
        if (x < npt) return (1u << (k1 - k0 - x * F32_ROWS)) - 1u;  // ragged last prefix tile: 1..15 keys
        const int w = x - npt;
        return *reinterpret_cast<const uint16_t *>(smem + G_::BITS_AT + (w >> 2) * 256 + c * 8 + (w & 3) * 2);
    };
    bool ill = false;
    if (t < nt) {
        const uint8_t *const lq = smem + G_::Q_AT + c * ROWB;
#pragma unroll
        for (int j = 0; j < KJ; j++) qf[j] = *reinterpret_cast<const f32x4 *>(lq + (((4 * j + g) ^ c) * 16));
        const uint8_t *const krow = lk + c * ROWB;
        const uint8_t *const vrow = lv + 4 * g * ROWB + c * 16;
#pragma unroll 1
        for (; t < nt; t += NW) {
            const int tn = t + NW;
            const bool masked = t >= nfull;
            wait_vmcnt<LOADS>();  // K of tile t (V may still be on its way)
            asm volatile("" ::: "memory");
            f32x4 kf[KJ], s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;  // two chains
#pragma unroll
            for (int j = 0; j < KJ; j++) kf[j] = *reinterpret_cast<const f32x4 *>(krow + (((4 * j + g) ^ c) * 16));
            const uint32_t vis = tile_vis(t);
            wait_lds_reads();
            if (tn < nt) issue(tn, i0, i1, false);
            __builtin_amdgcn_s_setprio(1);  // products ahead of the other wavefront's softmax
#pragma unroll
            for (int j = 0; j < KJ; j += 2)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][e], qf[j][e], s0, 0, 0, 0);
                    s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j + 1][e], qf[j + 1][e], s1, 0, 0, 0);
                }
            __builtin_amdgcn_s_setprio(0);
            if (tn < nt) wait_vmcnt<LOADS>();  // V of tile t (K of the next one may still be on its way)
            else wait_vmcnt<0>();
            asm volatile("" ::: "memory");
            f32x4 vf[4][VB];
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int v = 0; v < VB; v++) vf[i][v] = *reinterpret_cast<const f32x4 *>(vrow + i * ROWB + 256 * v);
            __builtin_amdgcn_sched_barrier(0);  // these reads fly during the softmax, which ends at the next one
            float sc[4];
#pragma unroll
            for (int i = 0; i < 4; i++) sc[i] = ((vis >> (4 * g + i)) & 1u) ? (s0[i] + s1[i]) * p.scale_log2 : -INFINITY;
            const float tmax = quad_max(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])));
            const bool lift = tmax > m_run + kLazy;
            if (__any(lift)) {
                const float m_new = lift ? tmax : m_run;
                const float alpha = lift ? exp2f(m_run - m_new) : 1.f;
                m_run = m_new;
                l_run *= alpha;
#pragma unroll
                for (int v = 0; v < VB; v++)
#pragma unroll
                    for (int e = 0; e < 4; e++) o[v][e] *= alpha;
            }
            const float ref = m_run == -INFINITY ? 0.f : m_run;  // no finite score so far: masked keys, or products that overflow
            float pr[4];  // exp2f, here and below: weights below the normal range stay (the bare instruction makes them zero)
#pragma unroll
            for (int i = 0; i < 4; i++) pr[i] = exp2f(sc[i] - ref);
            l_run += (pr[0] + pr[1]) + (pr[2] + pr[3]);
            __builtin_amdgcn_sched_barrier(0);
            wait_lds_reads();
            if (tn < nt) {
                issue(tn, i0, i1, true);
                if (tn + NW < nt) block_ids(tn + NW, i0, i1);  // they fly during a whole tile
            }
            if (masked) {
                uint32_t top = 0;
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int v = 0; v < VB; v++)
#pragma unroll
                        for (int e = 0; e < 4; e++) top = max(top, __float_as_uint(vf[i][v][e]) & 0x7fffffffu);
                if (__builtin_expect(__any(top >= 0x7f800000u), 0)) {
                    ill = true;
#pragma unroll
                    for (int i = 0; i < 4; i++)
#pragma unroll
                        for (int v = 0; v < VB; v++)
#pragma unroll
                            for (int e = 0; e < 4; e++) vf[i][v][e] = fabsf(vf[i][v][e]) < INFINITY ? vf[i][v][e] : 0.f;
                }
            }
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int v = 0; v < VB; v++)
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        o[v][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i][v][e], pr[i], o[v][e], 0, 0, 0);
            __builtin_amdgcn_s_setprio(0);
        }
    }
    if (ill) {
        uint64_t up[VB] = {}, down[VB] = {};
        for (int x = nfull + ((wave - nfull) & (NW - 1)); x < nt; x += NW) {  // the masked ones of the wavefront's tiles
            const bool tree = x >= npt;
            const int base = tree ? (x - npt) * F32_ROWS : k0 + x * F32_ROWS, count = min(F32_ROWS, (tree ? n : k1) - base);
            find_nonfinite<float, D>(p, b, kvh, P, tree, base, count, tile_vis(x), up, down);
        }
#pragma unroll
        for (int v = 0; v < VB; v++)
#pragma unroll
            for (int e = 0; e < 4; e++)
#pragma unroll
                for (int i = 0; i < 4; i++) {  // column 64 v + 16 g + 4 i + e
                    const int bit = 16 * g + 4 * i + e;
                    o[v][e][i] += ((up[v] >> bit) & 1ull ? INFINITY : 0.f) + ((down[v] >> bit) & 1ull ? -INFINITY : 0.f);
                }
    }

    // ---- merge the wavefronts: each leaves O in its own K buffer (same size and swizzle)
    float2 *const ml = reinterpret_cast<float2 *>(smem + G_::ML_AT);
    const int live = min(NW, nt);
    if (wave < live) {
        const float l_tot = quarter_swap_sum(half_swap_sum(l_run));
        uint8_t *const dst = smem + wave * (2 * TILE) + c * ROWB;
#pragma unroll
        for (int v = 0; v < VB; v++)
#pragma unroll
            for (int i = 0; i < 4; i++)
                *reinterpret_cast<f32x4 *>(dst + (((16 * v + 4 * g + i) ^ c) * 16)) = f32x4{o[v][0][i], o[v][1][i], o[v][2][i], o[v][3][i]};
        if (g == 0) ml[wave * F32_ROWS + c] = float2{m_run, l_tot};
    }
    __syncthreads();
    if (BALANCED && share.j == 0 && kvh == 0 && rg == 0 && tid == 0) p.split_tab[b] = make_int2(share.start, share.nvalid);
    constexpr int TPR = NW * 64 / F32_ROWS < CPR ? NW * 64 / F32_ROWS : CPR;  // threads of a row: pieces `piece`, `piece` + TPR, ...
    const int row = tid / TPR, piece = tid % TPR;
    if (row >= F32_ROWS) return;
    const int kq2 = (int)fast_div(rg * F32_ROWS + row, p.G, p.inv_g, rem), h2 = kvh * p.G + (int)rem;
    if (kq2 >= p.T_max) return;
    const bool rv = kq2 < n;
    if (!rv && !direct) return;
    // all reads of the statistics in one trip, then all reads of the outputs (those of absent wavefronts are skipped)
    float2 st[NW];
    float M = -INFINITY, L = 0.f;
#pragma unroll
    for (int x = 0; x < NW; x++) st[x] = ml[x * F32_ROWS + row];
#pragma unroll
    for (int x = 0; x < NW; x++) {
        if (x >= live) st[x] = float2{-INFINITY, 0.f};
        M = fmaxf(M, st[x].x);
    }
    f32x4 acc[CPR / TPR];
#pragma unroll
    for (int v = 0; v < CPR / TPR; v++) acc[v] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < NW; x++) {
        if (x >= live) break;  // uniform
        const float w = st[x].x == -INFINITY ? 0.f : exp2f(st[x].x - M);
        L = fmaf(w, st[x].y, L);
        const uint8_t *src = smem + x * (2 * TILE) + row * ROWB;
#pragma unroll
        for (int v = 0; v < CPR / TPR; v++) {
            const f32x4 ox = *reinterpret_cast<const f32x4 *>(src + (((piece + TPR * v) ^ row) * 16));
#pragma unroll
            for (int e = 0; e < 4; e++) acc[v][e] = fmaf(w, ox[e], acc[v][e]);
        }
    }
    const size_t pr = part_row(p, slot, h2, kq2);
    float *dst = direct ? static_cast<float *>(p.out) + (((size_t)b * p.T_max + kq2) * p.Hq + h2) * D : p.part_o + pr * D;
    const float inv = direct ? 1.f / L : 1.f;
#pragma unroll
    for (int v = 0; v < CPR / TPR; v++) {
#pragma unroll
        for (int e = 0; e < 4; e++) acc[v][e] = rv ? acc[v][e] * inv : 0.f;
        *reinterpret_cast<f32x4 *>(dst + 4 * (piece + TPR * v)) = acc[v];
    }
    if (piece == 0) {
        if (direct) {
            if (p.lse) p.lse[((size_t)b * p.Hq + h2) * p.T_max + kq2] = rv ? (M + log2f(L)) * kLn2 : -INFINITY;
        } else {
            p.part_m[pr] = M;
            p.part_l[pr] = L;
        }
    }
}

// ----------------------------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------------------------
struct Plan {
    bool mfma, kh;  // mfma: the bf16 kernels on matrix instructions
    bool f32;       // attn_f32_kernel
    bool blocks;    // attn_blocks_kernel
    bool wide;      // attn_wide_kernel (nw is 8: the chunks that its four wavefronts can take)
    int nw, ns, pairs, wgp, chunk, nsplit;
    bool balanced;  // split slots shared out among the sequences by their lengths, on the device
};

static bool supported(const etv_attn_desc *h) {
    if (h->B < 0 || h->T_max < 1 || h->Hq < 1 || h->Hkv < 1 || h->d < 1) return false;
    if (h->Hq > 65536) return false;  // keeps the byte strides of a cache row and of a block below 2^32
    return true;
}

// Launch shape at d = 64, and at d = 128 the price of the tile kernel in the choice against key blocks (what then runs there is
// pick_tile_shape's).  Cost model in microseconds, fitted on MI355X: workgroups run in rounds of the slots the chip
// offers; a round costs its tiles plus tree tiles and ramp-up; every extra split writes and re-reads one
// (m, l, O) set per query row and needs the combine launch.  A tile costs about 2.8 us for an 8-wavefront
// workgroup (two wavefronts per SIMD), the same for two 4-wavefront workgroups sharing a compute unit, and
// about 1.7 us for a 4-wavefront workgroup that has a compute unit to itself (1.5 us when at most two of its
// wavefronts hold valid rows).
constexpr double kTileKhAlone = 1.1, kTileKhShared = 2.2, kTileKh8 = 1.65;
// whole tiles: one 8-wavefront workgroup per compute unit (its two wavefronts per SIMD run one phase apart and it
// fetches each tile once) is 4-7 % faster in sustained runs than two 4-wavefront workgroups, which cost 2.8 together
constexpr double kTileWhole8 = 2.65;
// At d = 64 a tile costs about 0.6 of that in every shape (the softmax does not shrink), and what the constants pick is
// the best forced shape or within 5 % of it (seven workloads, B = 1 ... 32, T = 8 ... 128), so they serve both.
static long f32_blocks(const etv_attn_desc *h, const Plan &pl) {
    return ((long)h->B * pl.nsplit * h->Hkv + 7) / 8 * 8 * pl.pairs;
}
// fp32 kernel: workgroups of the fullest compute unit (the chunks of a (split, KV head, sequence) stay on one XCD, which takes every
// eighth of these), and tiles of a wavefront that takes the tree's too
static long f32_fullest(const etv_attn_desc *h, int chunks, int ns) { return (((long)max(1, h->B) * h->Hkv * ns + 7) / 8 * chunks + 31) / 32; }
static int f32_tiles(const etv_attn_desc *h, int tps) { return (tps * (KT / F32_ROWS) + (h->T_max + F32_ROWS - 1) / F32_ROWS + F32_NW - 1) / F32_NW; }

// bytes of the partial results of ns splits (and of the split table)
static size_t split_workspace(const etv_attn_desc *h, int ns) {
    return (size_t)h->B * h->Hq * h->T_max * ns * ((size_t)h->d + 2) * sizeof(float) + 1024;
}

// Splits that this file chooses by itself stay within the array of etv_tree_verify_attention_static, whose callers cannot
// bring a workspace, on every matrix-core kernel and at any size.
static bool beyond_array(const etv_attn_desc *h, int ns) { return ns > 1 && split_workspace(h, ns) > ETV_ATTN_STATIC_WORKSPACE_BYTES; }

// The next split count worth a look: with tps tiles per split now, the smallest count whose splits are shorter (the counts
// between differ only in empty splits).  Some 2 * sqrt(tiles) candidates instead of all of them, on every call.
static int next_split_count(int tiles, int tps) { return tps > 1 ? (tiles + tps - 2) / (tps - 1) : tiles + 1; }

// Launch shape of a bf16 call with heads of 128 on the tile and wide kernels.  Microseconds: a round of workgroups costs its tiles and a
// start-up; a tile costs the more, the more of the chip's wavefronts have rows (the clock follows the power); K/V bytes on top, and splits
// as before.  On 500 drawn workloads with every shape at up to five split counts (profiles/attention_tile_shapes.csv) the pick is 1.5 % behind
// the best measured shape on average and 8 % at the 95th percentile, and no other constants pick better.  The wide kernel passes the
// eight wavefronts of the tile kernel from about 14 tiles a split on: 1-2 tiles 1.12, 9-11 tiles 1.02, 16-39 tiles 0.96, 64 and more 0.88 of its
// time.  With three or four chunks each of its wavefronts has one; it gains over long splits (B = 32, T = 32, P = 4096: 93.6 us, the tile
// kernel 105.6; B = 8, T = 113, 32/32 heads, P = 8735: 176 and 201), loses over short ones (B = 16, T = 76, 32/32 heads, P = 124: 24.8 and 20.0),
// and with two chunks, half of its wavefronts idle, it is rarely ahead (B = 25, T = 35, 32/32 heads, P = 1653: 142 and 123), so it starts
// at three.
struct TileShape {
    int nw, kh, wide, chunks;                // wavefronts; key halves; wide; chunks of a workgroup (wide: 4 if it needs no more)
    double alone, least, full, start;        // a tile alone on a compute unit (nw = 4), with few, with all wavefronts busy; a round
};
constexpr TileShape kTileShapes[] = {{8, 0, 1, 8, 0.0, 1.05, 1.15, 7.72}, {8, 0, 1, 4, 0.0, 0.71, 0.75, 4.71}, {8, 0, 0, 8, 0.0, 1.26, 1.68, 3.81},
                                     {8, 1, 0, 4, 0.0, 0.78, 1.00, 4.06}, {4, 0, 0, 4, 1.15, 1.66, 1.86, 2.62}, {4, 1, 0, 2, 0.63, 0.92, 1.24, 3.45}};

// Trees of more than 128 nodes: the wide kernel's pass for the first masked tiles, a round.  Without it the model took the wide kernel for
// short prefixes (B = 23, T = 199, 32/32 heads, P = 377: 99 us, tile kernel 81): of 300 draws with T = 129 ... 256 35 were more
// than 3 % slower than before there was a wide kernel (by up to 15 %) and 66 faster, now 16 and 67.
constexpr double kWideSecondPass = 5.0;

static bool shape_allowed(const etv_attn_desc *h, int pairs, int nw, int kh) {
    if (kh && (h->flags & ETV_ATTN_FLAG_WHOLE_TILE)) return false;
    if (!kh && (h->flags & ETV_ATTN_FLAG_KEY_HALVES)) return false;
    // larger workgroups only for more chunks than the smaller ones hold
    if (nw == 8 && (pairs <= (kh ? 2 : 4) || (h->flags & ETV_ATTN_FLAG_SMALL_WG))) return false;
    if (nw == 4 && (h->flags & ETV_ATTN_FLAG_LARGE_WG) && pairs > (kh ? 2 : 4)) return false;
    return true;
}

// Flags that ask for a shape of the tile kernel leave the wide one out, unless its own flag is there too.
static bool tile_shape_allowed(const etv_attn_desc *h, int pairs, const TileShape &sh) {
    if (h->flags & ETV_ATTN_FLAG_WIDE) return sh.wide && (pairs <= 4) == (sh.chunks == 4);
    if (!sh.wide) return shape_allowed(h, pairs, sh.nw, sh.kh);
    return pairs > 2 && (pairs <= 4) == (sh.chunks == 4) &&
           !(h->flags & (ETV_ATTN_FLAG_SMALL_WG | ETV_ATTN_FLAG_LARGE_WG | ETV_ATTN_FLAG_WHOLE_TILE | ETV_ATTN_FLAG_KEY_HALVES));
}

// false: the flags leave no shape
static bool pick_tile_shape(const etv_attn_desc *h, Plan &pl) {
    const int tiles = max(1, (h->P_max + KT - 1) / KT), B = max(1, h->B);
    const int forced_tps = h->kv_split > 0 ? min(tiles, (h->kv_split + KT - 1) / KT) : 0;
    const double part_us = 2.0 * B * h->Hq * h->T_max * (h->d + 2.0) * 4.0 / 3.0e6;
    const double fixed = 4.66 + 4.0 * B * h->P_max * (double)h->Hkv * h->d / 25.0e6;
    const int tree_tiles = (h->T_max + KT - 1) / KT;
    double best = 1e30;
    for (const TileShape &sh : kTileShapes) {
        if (!tile_shape_allowed(h, pl.pairs, sh)) continue;
        const int cw = sh.chunks, wgp = (pl.pairs + cw - 1) / cw;
        const long units = (long)B * h->Hkv * wgp;
        const double held = (double)pl.pairs / (wgp * cw);  // part of a workgroup's chunks that have rows
        for (int ns = forced_tps ? (tiles + forced_tps - 1) / forced_tps : 1, tps; ns <= tiles; ns = forced_tps ? tiles + 1 : next_split_count(tiles, tps)) {
            tps = forced_tps ? forced_tps : (tiles + ns - 1) / ns;
            if (!forced_tps && beyond_array(h, ns)) break;
            const long wgs = units * ns;
            const bool alone = sh.nw == 4 && wgs <= 256;
            const double slots = sh.nw == 4 && !alone ? 512.0 : 256.0;
            const double busy = sh.full * held * (wgs < slots ? wgs / slots : 1.0);
            const double tile = alone ? sh.alone : (busy > sh.least ? busy : sh.least);
            const double start = sh.start + (sh.wide && h->T_max > 128 ? kWideSecondPass : 0.0);
            const double est = ceil(wgs / slots) * ((tps + tree_tiles * (ns > 1 ? 0.6 : 1.0)) * tile + start) + fixed +
                               (ns > 1 ? 2.25 + ns * part_us * 0.6 : 0.0);
            if (est < best) {
                best = est;
                pl.nw = sh.nw; pl.kh = sh.kh; pl.wide = sh.wide; pl.wgp = wgp; pl.chunk = tps * KT; pl.nsplit = ns;
                pl.ns = sh.nw == 8 || alone ? 4 : 2;  // ring places
            }
        }
    }
    return best < 1e30;
}

static Plan make_plan(const etv_attn_desc *h) {
    Plan pl{};
    const int tiles = max(1, (h->P_max + KT - 1) / KT);
    const int B = max(1, h->B);
    // d is 64 or 128.  The row groups of all KV heads share a grid dimension of at most 65535; thousands of heads with the
    // largest trees that go beyond it stay on the kernel with a workgroup per row.
    const long rows = (long)(h->Hq / h->Hkv) * h->T_max;
    // The bf16 kernels take a row's maximum before they scale it, which a negative scale turns into its minimum; such calls go to
    // the kernel that scales first.  (Turning the signs of Q round in them instead costs every short launch: B = 22, T = 7,
    // 32/32 heads, P = 95 16.7 -> 17.6 us.)
    const bool generic = (h->flags & ETV_ATTN_FLAG_GENERIC) != 0 || (h->dtype == ETV_BF16 && h->scale < 0.f);
    pl.mfma = h->dtype == ETV_BF16 && !generic && (h->d == 128 || h->Hkv * ((rows + 63) / 64) <= 65535);
    pl.f32 = h->dtype == ETV_F32 && !generic;
    if (pl.f32) {
        // A workgroup puts one wavefront on each SIMD of a compute unit and the matrix cores bound the launch: its time is
        // the tiles of a wavefront times the workgroups of the fullest compute unit, which run in twos (fours at d = 64) with an odd one by
        // itself at the end, and a start for each such round; every split adds partials and a combine step, the first one the combine launch.
        // Measured per tile: 1.0 us at d = 128 (0.6 at d = 64) for each of an even number of workgroups, 1.38 us (0.7) for the odd one, 1.3
        // (0.95) in a launch of lone ones; 0.86 (0.43) are matrix instructions.  The rest is fitted to 324 calls at up to twelve split counts
        // (profiles/attention_f32_plan_picks.csv): the choice is 1.7 % behind the best count on average, with workgroups counted over
        // all 256 compute units and an odd one priced like any other it was 3.2 %, and up to 52 %.
        pl.pairs = (int)((rows + F32_ROWS - 1) / F32_ROWS);
        const bool d128 = h->d == 128;
        const double busy = d128 ? 1.0 : 0.6, odd = d128 ? 1.38 : 0.7, lone = d128 ? 1.3 : 0.95;
        const int together = d128 ? 2 : 4;
        const double part_us = 0.4 * 2.0 * B * h->Hq * h->T_max * (h->d + 2.0) * 4.0 / 3.0e6;
        const int forced_tps = h->kv_split > 0 ? min(tiles, (h->kv_split + KT - 1) / KT) : 0;
        double best = 1e30;
        for (int ns = forced_tps ? (tiles + forced_tps - 1) / forced_tps : 1, tps; ns <= tiles; ns = forced_tps ? tiles + 1 : next_split_count(tiles, tps)) {
            tps = forced_tps ? forced_tps : (tiles + ns - 1) / ns;
            if (!forced_tps && beyond_array(h, ns)) break;
            const double per_wave = ceil((tps * 4.0 + (h->T_max + 15) / 16) / F32_NW);
            const long full = (((long)B * h->Hkv * ns + 7) / 8 * pl.pairs + 31) / 32;
            const double tile = full == 1 ? lone : ((full & 1) ? (full - 1) * busy + odd : full * busy);
            const double est = per_wave * tile + (full + together - 1) / together * 3.0 + (ns > 1 ? 3.0 + ns * (part_us + 0.15) : 0.0);
            if (est < best) {
                best = est;
                pl.chunk = tps * KT; pl.nsplit = ns;
            }
        }
        pl.balanced = pl.nsplit > 1 && B >= 2 && B <= 64 && !(h->flags & ETV_ATTN_FLAG_UNIFORM_SPLITS);
        return pl;
    }
    if (!pl.mfma) {
        const long units = ((long)B * h->Hq * h->T_max + 7) / 8;  // 8 resident wavefronts ~ one workgroup slot
        int tps;
        if (h->kv_split > 0) {
            tps = (h->kv_split + KT - 1) / KT;
        } else {
            long want = (256 + units - 1) / units;
            want = want < 1 ? 1 : (want > tiles ? tiles : want);
            tps = (int)((tiles + want - 1) / want);
        }
        pl.chunk = tps * KT;
        pl.nsplit = (tiles + tps - 1) / tps;
        return pl;
    }
    pl.pairs = ((h->Hq / h->Hkv) * h->T_max + 31) / 32;  // 32-row chunks of the G * T_max packed rows of a KV head
    const double part_us = 2.0 * B * h->Hq * h->T_max * (h->d + 2.0) * 4.0 / 3.0e6;
    double best = 1e30, best_lat = 0.0;
    // a batch with splits: the slots go to the sequences by length (lane i of a wavefront plans sequence i)
    const bool shared_out = B >= 2 && B <= 64 && !(h->flags & ETV_ATTN_FLAG_UNIFORM_SPLITS);
    const bool blocks_only = (h->flags & ETV_ATTN_FLAG_KEY_BLOCKS) != 0;
    const int shape_flags = ETV_ATTN_FLAG_SMALL_WG | ETV_ATTN_FLAG_LARGE_WG | ETV_ATTN_FLAG_WHOLE_TILE | ETV_ATTN_FLAG_KEY_HALVES |
                            (h->d == 128 ? ETV_ATTN_FLAG_WIDE : 0);
    const long block_slots = h->d == 64 ? 512 : 256;  // workgroups of the key-block kernel that run at once
    const bool maybe_blocks = blocks_only || (!(h->flags & shape_flags) && ((long)B * h->Hkv + 7) / 8 * pl.pairs <= block_slots / 8);
    // The tile kernel's shape at d = 64.  At d = 128 pick_tile_shape has the last word; there this is only the price against which the
    // key-block kernel is weighed, and is left out where that one is no candidate.
    for (int nw = 4; nw <= 8 && !blocks_only && (h->d == 64 || maybe_blocks); nw += 4) {
        for (int kh = 0; kh <= 1; kh++) {
            const int cw = kh ? nw / 2 : nw;  // chunks per workgroup
            if (!shape_allowed(h, pl.pairs, nw, kh)) continue;
            const int wgp = (pl.pairs + cw - 1) / cw;
            const long units = (long)B * h->Hkv * wgp;
            // candidates: every distinct number of splits, or the one split size the caller asks for
            const int forced_tps = h->kv_split > 0 ? min(tiles, (h->kv_split + KT - 1) / KT) : 0;
            for (int ns = forced_tps ? (tiles + forced_tps - 1) / forced_tps : 1, tps; ns <= tiles; ns = forced_tps ? tiles + 1 : next_split_count(tiles, tps)) {
                tps = forced_tps ? forced_tps : (tiles + ns - 1) / ns;
                if (!forced_tps && h->d == 64 && beyond_array(h, ns)) break;
                const long wgs = units * ns;
                const bool alone = (nw == 4 && wgs <= 256);
                const double slots = nw == 8 ? 256.0 : 512.0;
                double t_tile;
                if (kh) t_tile = alone ? kTileKhAlone : (nw == 8 ? kTileKh8 : kTileKhShared);
                else t_tile = alone ? (pl.pairs <= 2 ? 1.5 : 1.7) : (nw == 8 ? kTileWhole8 : 2.8);
                const double rounds = ceil((double)wgs / slots);
                const double est = rounds * (tps + 1.5) * t_tile + 4.0 + (ns > 1 ? 4.6 + ns * part_us : 0.0);
                if (est < best) {
                    best = est;
                    best_lat = rounds * (tps + 1.0) * t_tile;
                    pl.nw = nw; pl.kh = kh; pl.wgp = wgp; pl.chunk = tps * KT; pl.nsplit = ns;
                    pl.ns = nw == 8 ? 4 : (alone ? 4 : 2);  // ring stages: a lone small workgroup can afford four
                }
            }
        }
    }
    if (maybe_blocks) {
        // Key-block kernel against the pick so far, for launches that fit the chip at once (one workgroup per compute unit, two
        // at d = 64): a further round pays start-up and merge again, and the other kernel is then always ahead.  Microseconds,
        // fitted to 488 workloads (B = 1 ... 32, T = 1 ... 256, P = 64 ... 30000, both head sizes) by what the choice costs against the
        // best measured shape, and twice over against the tile kernel's own pick; with the wide kernel beside the tile kernel it costs
        // 1.15 % against the better of the two (1682 drawn calls).  A
        // wavefront's block is 2.0 (2.33 where a single chunk waits for HBM and not for its neighbours' lines in L2; d = 64 1.4,
        // and 2.3 times that with two workgroups on a compute unit); the memory side is the K/V bytes once at 6.9 TB/s and once
        // more per further chunk at 46 TB/s.  The pick so far counts as 3 % faster than its estimate: what a wrong one costs.
        const bool d64 = h->d == 64;
        const double kv_bytes = 4.0 * B * h->P_max * (double)h->Hkv * h->d, part2_us = part_us * 0.67;
        if (best < 1e30) {
            const double lat = 0.78 * best_lat * (d64 ? 0.68 : 1.0) + 6.6, mem = 7.15 + kv_bytes / 5.7e6;
            best = 0.97 * ((lat > mem ? lat : mem) + (pl.nsplit > 1 ? 3.3 + pl.nsplit * part2_us : 0.0));
        }
        const long units = (long)B * h->Hkv * pl.pairs;
        const double mem = 4.75 + kv_bytes / 6.9e6 + (pl.pairs - 1) * kv_bytes / 46.0e6, mem25 = mem * mem * sqrt(mem);
        const int tree_blocks = (h->T_max + KB_KEYS - 1) / KB_KEYS;
        const int forced_tps = h->kv_split > 0 ? min(tiles, (h->kv_split + KT - 1) / KT) : 0;
        for (int ns = forced_tps ? (tiles + forced_tps - 1) / forced_tps : 1, tps; ns <= tiles; ns = forced_tps ? tiles + 1 : next_split_count(tiles, tps)) {
            tps = forced_tps ? forced_tps : (tiles + ns - 1) / ns;
            const long wgs = units * ns;
            // the chunks of a (split, KV head, sequence) stay on one XCD: the fullest of the eight has to hold all of its own at once
            const long fullest = ((long)B * ns * h->Hkv + 7) / 8 * pl.pairs;
            if (fullest > block_slots / 8 && !(blocks_only && (ns == 1 || forced_tps))) break;
            if (((long)B * ns * h->Hkv + 7) / 8 > 65535 || pl.pairs > 65535) break;  // grid dimensions
            if (!forced_tps && beyond_array(h, ns)) break;
            const int most = (2 * tps + tree_blocks + KB_NW - 1) / KB_NW, usual = (2 * tps + KB_NW - 1) / KB_NW;
            const double steps = ns > 1 ? 0.5 * (most + usual) : most;  // only the last split takes the tree
            const double t_step = d64 ? (wgs > 256 ? 3.2 : 1.4) : (pl.pairs == 1 ? 2.33 : 2.0);
            const double lat = steps * t_step + (d64 ? 2.4 : 3.3);
            const double est = pow(lat * lat * sqrt(lat) + mem25, 0.4) + (ns > 1 ? 3.05 + ns * part2_us + (shared_out ? 1.2 : 0.0) : 0.0);
            if (est < best) {
                best = est;
                pl.blocks = true; pl.nw = KB_NW; pl.kh = false; pl.wgp = pl.pairs; pl.chunk = tps * KT; pl.nsplit = ns; pl.ns = 0;
            }
        }
    }
    bool picked = best < 1e30;
    if (h->d == 128 && !pl.blocks) picked = pick_tile_shape(h, pl) && !blocks_only;
    pl.balanced = pl.nsplit > 1 && shared_out;
    if (!picked) {  // flags that leave no shape (whole tiles and key halves, a launch too large for key blocks): a single split
        pl.nw = (pl.pairs > 4 && !(h->flags & ETV_ATTN_FLAG_SMALL_WG)) ? 8 : 4;
        pl.kh = false; pl.wide = false;
        pl.wgp = (pl.pairs + pl.nw - 1) / pl.nw;
        pl.chunk = tiles * KT; pl.nsplit = 1; pl.ns = pl.nw == 8 ? 4 : 2;
    }
    return pl;
}

template <int D, int NW, int NS, bool PAGED, bool KH>
static int32_t launch_mfma(const AttnParams &p, dim3 grid, hipStream_t st) {
    constexpr size_t lds = (size_t)NS * Geo<D>::STAGE_BYTES;
    static const bool lds_ok = [] {  // opt in to more than 64 KiB of dynamic LDS, once per process
        return hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_mfma_kernel<D, NW, NS, PAGED, KH>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess;
    }();
    if (!lds_ok) return ETV_ERR_HIP;
    hipLaunchKernelGGL((attn_mfma_kernel<D, NW, NS, PAGED, KH>), grid, dim3(NW * 64), lds, st, p);
    return check_launch();
}

template <bool PAGED, bool NT, bool MANY>
static int32_t launch_wide(const AttnParams &p, dim3 grid, hipStream_t st) {
    constexpr size_t lds = WideGeo::LDS;
    static const bool lds_ok = [] {
        return hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_wide_kernel<PAGED, NT, MANY>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess;
    }();
    if (!lds_ok) return ETV_ERR_HIP;
    hipLaunchKernelGGL((attn_wide_kernel<PAGED, NT, MANY>), grid, dim3(256), lds, st, p.prefix_len, p.n_nodes, p.bitmask, p.block_table,
                       (uint32_t)p.Hkv, p.inv_hkv, (uint32_t)p.G, p.inv_g, p.max_blocks, wide_form(p), p);
    return check_launch();
}

template <int D, bool PAGED, bool BALANCED, bool NT>
static int32_t launch_blocks(const AttnParams &p, dim3 grid, hipStream_t st) {
    static const bool lds_ok = [] {
        return hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_blocks_kernel<D, PAGED, BALANCED, NT>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, KbGeo<D>::LDS) == hipSuccess;
    }();
    if (!lds_ok) return ETV_ERR_HIP;
    hipLaunchKernelGGL((attn_blocks_kernel<D, PAGED, BALANCED, NT>), grid, dim3(KB_NW * 64), KbGeo<D>::LDS, st, p.prefix_len, p.n_nodes,
                       p.block_table, p.Hkv, p.inv_hkv, p.B * p.nsplit, p.nsplit, p.inv_nsplit, p.max_blocks, p.chunk, p.inv_chunk, p);
    return check_launch();
}
template <int D>
static int32_t launch_blocks_form(bool paged, const AttnParams &p, dim3 grid, hipStream_t st) {
    // a single reader of its K/V bytes streams them past L2
    switch ((paged ? 4 : 0) + (p.balanced ? 2 : 0) + (p.pairs == 1 ? 1 : 0)) {
    case 0: return launch_blocks<D, false, false, false>(p, grid, st);
    case 1: return launch_blocks<D, false, false, true>(p, grid, st);
    case 2: return launch_blocks<D, false, true, false>(p, grid, st);
    case 3: return launch_blocks<D, false, true, true>(p, grid, st);
    case 4: return launch_blocks<D, true, false, false>(p, grid, st);
    case 5: return launch_blocks<D, true, false, true>(p, grid, st);
    case 6: return launch_blocks<D, true, true, false>(p, grid, st);
    default: return launch_blocks<D, true, true, true>(p, grid, st);
    }
}

template <int D, bool PAGED, bool BALANCED, bool NT>
static int32_t launch_f32(const AttnParams &p, dim3 grid, hipStream_t st) {
    static const bool lds_ok = [] {
        return hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_f32_kernel<D, PAGED, BALANCED, NT>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, F32Geo<D>::LDS) == hipSuccess;
    }();
    if (!lds_ok) return ETV_ERR_HIP;
    hipLaunchKernelGGL((attn_f32_kernel<D, PAGED, BALANCED, NT>), grid, dim3(F32_NW * 64), F32Geo<D>::LDS, st, p.prefix_len, p.n_nodes,
                       p.block_table, p.Hkv, p.inv_hkv, p.B * p.nsplit, p.nsplit, p.inv_nsplit, p.max_blocks, p.chunk, p.inv_chunk, p);
    return check_launch();
}
template <int D>
static int32_t launch_f32_form(bool paged, const AttnParams &p, dim3 grid, hipStream_t st) {
    // a single reader of its K/V bytes streams them past L2
    switch ((paged ? 4 : 0) + (p.balanced ? 2 : 0) + (p.pairs == 1 ? 1 : 0)) {
    case 0: return launch_f32<D, false, false, false>(p, grid, st);
    case 1: return launch_f32<D, false, false, true>(p, grid, st);
    case 2: return launch_f32<D, false, true, false>(p, grid, st);
    case 3: return launch_f32<D, false, true, true>(p, grid, st);
    case 4: return launch_f32<D, true, false, false>(p, grid, st);
    case 5: return launch_f32<D, true, false, true>(p, grid, st);
    case 6: return launch_f32<D, true, true, false>(p, grid, st);
    default: return launch_f32<D, true, true, true>(p, grid, st);
    }
}

constexpr size_t kCombineAhead = 8u << 20, kCombineAheadTwo = 5u << 20;  // see AHEAD

template <typename T, int D, int WPR, int U, bool SHARED>
static void launch_combine_form(const AttnParams &p, dim3 grid, hipStream_t st) {
    const size_t split_bytes = (size_t)p.B * p.Hq * p.T_max * D * sizeof(float);
    const bool fixed = !SHARED && !p.balanced;
    const auto kernel = p.balanced ? attn_combine_kernel<T, D, WPR, U, SHARED, true, 0>
                        : fixed && min(p.nsplit, U) * split_bytes <= kCombineAhead ? attn_combine_kernel<T, D, WPR, U, SHARED, false, SHARED ? 0 : U>
                        : fixed && 2 * split_bytes <= kCombineAheadTwo ? attn_combine_kernel<T, D, WPR, U, SHARED, false, SHARED ? 0 : 2>
                                                                       : attn_combine_kernel<T, D, WPR, U, SHARED, false, 0>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, p.balanced ? reinterpret_cast<const int32_t *>(p.split_tab) : p.prefix_len, p.n_nodes,
                       p.part_o, p.part_m, p.part_l, p.Hq, fast_div_inv(p.Hq), p.T_max, p.nsplit, p);
}
template <typename T, int D, int WPR>
static void launch_combine(const AttnParams &p, bool shared, hipStream_t st) {
    const unsigned rows = (unsigned)p.T_max * p.Hq, per_wg = shared ? 1 : 4 / WPR;
    const dim3 grid((rows + per_wg - 1) / per_wg, p.B);
    if (shared) launch_combine_form<T, D, 1, 16, true>(p, grid, st);
    else if (p.nsplit > 8) launch_combine_form<T, D, WPR, 16, false>(p, grid, st);  // many splits: sixteen per batch of loads
    else launch_combine_form<T, D, WPR, 8, false>(p, grid, st);
}

// 8 wavefronts: one workgroup per compute unit with a 4-stage ring (128 KiB of LDS at d = 128);
// 4 wavefronts: two workgroups per compute unit with 2 stages each, or 4 stages when the grid is small
template <int D>
static int32_t launch_mfma_shape(const Plan &pl, bool paged, const AttnParams &p, dim3 grid, hipStream_t st) {
    if constexpr (D == 128)
        if (pl.wide) {
            switch ((paged ? 4 : 0) + (p.wgp == 1 ? 2 : 0) + (p.T_max > 128 ? 1 : 0)) {
            case 0: return launch_wide<false, false, false>(p, grid, st);
            case 1: return launch_wide<false, false, true>(p, grid, st);
            case 2: return launch_wide<false, true, false>(p, grid, st);
            case 3: return launch_wide<false, true, true>(p, grid, st);
            case 4: return launch_wide<true, false, false>(p, grid, st);
            case 5: return launch_wide<true, false, true>(p, grid, st);
            case 6: return launch_wide<true, true, false>(p, grid, st);
            default: return launch_wide<true, true, true>(p, grid, st);
            }
        }
    const int shape = (pl.nw == 8 ? 0 : (pl.ns == 4 ? 1 : 2)) * 4 + (paged ? 2 : 0) + (pl.kh ? 1 : 0);
    switch (shape) {
    case 0: return launch_mfma<D, 8, 4, false, false>(p, grid, st);
    case 1: return launch_mfma<D, 8, 4, false, true>(p, grid, st);
    case 2: return launch_mfma<D, 8, 4, true, false>(p, grid, st);
    case 3: return launch_mfma<D, 8, 4, true, true>(p, grid, st);
    case 4: return launch_mfma<D, 4, 4, false, false>(p, grid, st);
    case 5: return launch_mfma<D, 4, 4, false, true>(p, grid, st);
    case 6: return launch_mfma<D, 4, 4, true, false>(p, grid, st);
    case 7: return launch_mfma<D, 4, 4, true, true>(p, grid, st);
    case 8: return launch_mfma<D, 4, 2, false, false>(p, grid, st);
    case 9: return launch_mfma<D, 4, 2, false, true>(p, grid, st);
    case 10: return launch_mfma<D, 4, 2, true, false>(p, grid, st);
    default: return launch_mfma<D, 4, 2, true, true>(p, grid, st);
    }
}

}  // namespace etv

extern "C" int32_t etv_tree_verify_attention_plan(const etv_attn_desc *h, etv_attn_plan *out) {
    if (!h || !out || !etv::supported(h) || h->Hq % h->Hkv != 0) return ETV_ERR_INVALID_ARG;
    const etv::Plan pl = etv::make_plan(h);
    out->mfma = pl.mfma ? 1 : 0;
    out->wavefronts = pl.mfma ? pl.nw : (pl.f32 ? etv::F32_NW : 1);
    out->key_halves = pl.mfma && pl.kh ? 1 : 0;
    out->ring_stages = pl.mfma ? pl.ns : 0;
    out->row_groups = pl.mfma ? pl.wgp : (pl.f32 ? pl.pairs : 0);
    out->kv_split = pl.chunk;
    out->n_splits = pl.nsplit;
    out->balanced_splits = pl.balanced ? 1 : 0;
    out->workgroups = pl.mfma || pl.f32 ? (int64_t)pl.nsplit * h->Hkv * out->row_groups * (h->B > 0 ? h->B : 0)
                                        : (int64_t)h->T_max * h->Hq * (h->B > 0 ? h->B : 0) * pl.nsplit;
    return ETV_OK;
}

extern "C" int32_t etv_tree_verify_attention_kernel(const etv_attn_desc *h) {
    if (!h || !etv::supported(h) || h->Hq % h->Hkv != 0) return ETV_ERR_INVALID_ARG;
    const etv::Plan pl = etv::make_plan(h);
    if (!pl.mfma) return pl.f32 ? ETV_ATTN_KERNEL_F32 : ETV_ATTN_KERNEL_GENERIC;
    return pl.blocks ? ETV_ATTN_KERNEL_KEY_BLOCKS : (pl.wide ? ETV_ATTN_KERNEL_WIDE : ETV_ATTN_KERNEL_TILE);
}

extern "C" size_t etv_tree_verify_attention_workspace_bytes(const etv_attn_desc *h) {
    if (!h || !etv::supported(h) || h->B == 0) return 0;
    etv::Plan pl = etv::make_plan(h);
    if (pl.nsplit <= 1) return 256;
    return etv::split_workspace(h, pl.nsplit);  // partials, then 64 (first slot, splits) pairs
}

namespace etv {
// argument checks and launches shared by the two entry points (caller's workspace / the library's static one)
static int32_t attention_run(const etv_attn_desc *h, const void *q, const void *k_cache, const void *v_cache,
                             const int32_t *block_table, const int32_t *prefix_len, const void *kt, const void *vt,
                             const uint64_t *bitmask, const int32_t *n_nodes, void *out, float *lse, void *workspace,
                             size_t workspace_bytes, void *stream) {
    if (!h || !q || !prefix_len || !bitmask || !n_nodes || !out) return ETV_ERR_INVALID_ARG;
    if ((kt == nullptr) != (vt == nullptr)) return ETV_ERR_INVALID_ARG;
    const bool tail = (kt == nullptr);  // in-place branch cache: the tree rows are in the cache behind the prefix
    if (!supported(h)) return ETV_ERR_INVALID_ARG;
    if (h->Hq % h->Hkv != 0) return ETV_ERR_INVALID_ARG;
    if (h->dtype != ETV_F32 && h->dtype != ETV_BF16) return ETV_ERR_UNSUPPORTED;
    if (h->d != 64 && h->d != 128) return ETV_ERR_UNSUPPORTED;
    if (h->T_max > ETV_ATTN_MAX_TREE) return ETV_ERR_UNSUPPORTED;
    if (h->P_max < 0) return ETV_ERR_INVALID_ARG;
    if (h->block_size != 0 && h->block_size != 16) return ETV_ERR_UNSUPPORTED;
    if (h->block_size > 0 && (!block_table || h->max_blocks < 1)) return ETV_ERR_INVALID_ARG;
    const long reach = (long)h->P_max + (tail ? h->T_max : 0);  // cache positions the kernel may read
    if (h->block_size > 0 && reach > (long)h->max_blocks * h->block_size) return ETV_ERR_INVALID_ARG;
    if (h->block_size == 0 && reach > h->P_cap) return ETV_ERR_INVALID_ARG;
    if (reach > 0 && (!k_cache || !v_cache)) return ETV_ERR_INVALID_ARG;
    if (h->kv_split < 0) return ETV_ERR_INVALID_ARG;
    const uintptr_t align = (uintptr_t)q | (uintptr_t)k_cache | (uintptr_t)v_cache | (uintptr_t)kt | (uintptr_t)vt |
                            (uintptr_t)out | (uintptr_t)workspace;
    if (align & 15) return ETV_ERR_INVALID_ARG;
    if (h->B == 0) return ETV_OK;
    if (h->B > 65535) return ETV_ERR_UNSUPPORTED;

    Plan pl = make_plan(h);
    if ((long)h->B * pl.nsplit > 65535 && !pl.mfma && !pl.f32) return ETV_ERR_UNSUPPORTED;
    if (pl.f32 && f32_blocks(h, pl) > 0x7fffffffL) return ETV_ERR_UNSUPPORTED;
    if (pl.nsplit > 1) {
        if (!workspace || workspace_bytes < split_workspace(h, pl.nsplit))
            return ETV_ERR_WORKSPACE_TOO_SMALL;
    }
    AttnParams p{};
    p.q = q; p.k_cache = k_cache; p.v_cache = v_cache; p.kt = kt; p.vt = vt;
    p.block_table = block_table; p.prefix_len = prefix_len; p.n_nodes = n_nodes; p.bitmask = bitmask;
    p.out = out; p.lse = lse;
    p.B = h->B; p.T_max = h->T_max; p.Hq = h->Hq; p.Hkv = h->Hkv; p.G = h->Hq / h->Hkv; p.d = h->d;
    p.block_size = h->block_size; p.max_blocks = h->max_blocks; p.P_cap = h->P_cap; p.P_max = h->P_max;
    p.words = (h->T_max + 63) / 64;
    p.chunk = pl.chunk; p.nsplit = pl.nsplit; p.pairs = pl.pairs; p.wgp = pl.wgp;
    p.inv_g = fast_div_inv(p.G); p.inv_hkv = fast_div_inv(p.Hkv); p.inv_nsplit = fast_div_inv(p.nsplit); p.inv_chunk = fast_div_inv(p.chunk);
    const float scale = (h->scale == 0.f) ? 1.0f / sqrtf((float)h->d) : h->scale;
    p.scale_log2 = scale * 1.4426950408889634f;
    if (pl.nsplit > 1) {
        size_t rows = (size_t)h->B * h->Hq * h->T_max * pl.nsplit;
        p.part_o = static_cast<float *>(workspace);
        p.part_m = p.part_o + rows * h->d;
        p.part_l = p.part_m + rows;
        p.split_tab = reinterpret_cast<int2 *>(p.part_l + rows);  // 8-byte aligned: rows * (d + 2) floats in
        p.balanced = pl.balanced;
    }
    hipStream_t st = as_stream(stream);
    int32_t rc;
    if (pl.blocks) {
        const dim3 grid(8, pl.pairs, ((unsigned)h->B * pl.nsplit * h->Hkv + 7) / 8);
        rc = h->d == 128 ? launch_blocks_form<128>(h->block_size > 0, p, grid, st) : launch_blocks_form<64>(h->block_size > 0, p, grid, st);
    } else if (pl.mfma) {
        const dim3 grid = pl.balanced ? dim3(pl.nsplit * h->B, h->Hkv * pl.wgp, 1) : dim3(pl.nsplit, h->Hkv * pl.wgp, h->B);
        rc = h->d == 128 ? launch_mfma_shape<128>(pl, h->block_size > 0, p, grid, st)
                         : launch_mfma_shape<64>(pl, h->block_size > 0, p, grid, st);
    } else if (pl.f32) {
        const unsigned units8 = (unsigned)(((long)h->B * pl.nsplit * h->Hkv + 7) / 8);
        // Three or five workgroups on the fullest compute unit, two at a time, of 24 tiles and more: shorter ones gain nothing, with seven
        // and more it is lost in the rest, and at d = 64 four run at a time.
        // B = 6, T = 64, 32/8 heads, P = 2000 148.7 -> 125.8 us, P = 1500 117.5 -> 99.2, B = 13, T = 48 170.0 -> 153.2.
        const long full = f32_fullest(h, pl.pairs, pl.nsplit);
        p.stagger = h->d == 128 && (full == 3 || full == 5) && f32_tiles(h, pl.chunk / KT) >= 24 ? pl.pairs : 0;
        const dim3 grid(8 * (unsigned)pl.pairs, min(units8, (unsigned)F32_GRID_Y), (units8 + F32_GRID_Y - 1) / F32_GRID_Y);
        rc = h->d == 128 ? launch_f32_form<128>(h->block_size > 0, p, grid, st) : launch_f32_form<64>(h->block_size > 0, p, grid, st);
    } else {
        dim3 grid(h->T_max, h->Hq, h->B * pl.nsplit);
        if (h->dtype == ETV_F32 && h->d == 64)
            hipLaunchKernelGGL((attn_generic_kernel<float, 64>), grid, dim3(64), 0, st, p);
        else if (h->dtype == ETV_F32)
            hipLaunchKernelGGL((attn_generic_kernel<float, 128>), grid, dim3(64), 0, st, p);
        else if (h->d == 64)
            hipLaunchKernelGGL((attn_generic_kernel<uint16_t, 64>), grid, dim3(64), 0, st, p);
        else
            hipLaunchKernelGGL((attn_generic_kernel<uint16_t, 128>), grid, dim3(64), 0, st, p);
        rc = check_launch();
    }
    if (rc != ETV_OK || pl.nsplit == 1) return rc;
    const long crows = (long)h->B * h->T_max * h->Hq;
    const bool shared = pl.nsplit > 16 && crows <= 1024;      // more splits than one batch of a wavefront
    const bool two = !shared && h->d == 128 && crows <= 512;  // very few rows: two wavefronts per row
    if (h->dtype == ETV_F32 && h->d == 64) launch_combine<float, 64, 1>(p, shared, st);
    else if (h->dtype == ETV_F32 && two) launch_combine<float, 128, 2>(p, shared, st);
    else if (h->dtype == ETV_F32) launch_combine<float, 128, 1>(p, shared, st);
    else if (h->d == 64) launch_combine<uint16_t, 64, 1>(p, shared, st);
    else if (two) launch_combine<uint16_t, 128, 2>(p, shared, st);
    else launch_combine<uint16_t, 128, 1>(p, shared, st);
    return check_launch();
}
}  // namespace etv

extern "C" int32_t etv_tree_verify_attention(const etv_attn_desc *h, const void *q, const void *k_cache,
                                             const void *v_cache, const int32_t *block_table,
                                             const int32_t *prefix_len, const void *kt, const void *vt,
                                             const uint64_t *bitmask, const int32_t *n_nodes, void *out, float *lse,
                                             void *workspace, size_t workspace_bytes, void *stream) {
    return etv::attention_run(h, q, k_cache, v_cache, block_table, prefix_len, kt, vt, bitmask, n_nodes, out, lse,
                              workspace, workspace_bytes, stream);
}

// ----------------------------------------------------------------------------------------------
// The same call for callers that cannot allocate or carry a workspace (code under graph capture, serving loops):
// the split partials go to a fixed array in device memory that the library owns.  Each GPU holds its own copy
// of the array at its own address; the address is asked for once per device and only that pointer is ever
// handed to a kernel (the array's name is a host-side stand-in in host code, not a device address).
// ----------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[ETV_ATTN_STATIC_WORKSPACE_BYTES];

namespace etv {
constexpr int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices];           // per device, filled on the first call on that device
static std::atomic<int> g_scratch_state[kMaxDevices];  // 0 unset, 1 being set, 2 set

static int32_t static_scratch(void **ptr) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return ETV_ERR_HIP;
    if (g_scratch_state[dev].load(std::memory_order_acquire) != 2) {
        int expect = 0;
        if (g_scratch_state[dev].compare_exchange_strong(expect, 1, std::memory_order_acq_rel)) {
            void *d = nullptr;
            const hipError_t e = hipGetSymbolAddress(&d, HIP_SYMBOL(scratch));  // device `dev` is current
            if (e != hipSuccess || d == nullptr) {
                g_last_hip_error = (int32_t)e;
                g_scratch_state[dev].store(0, std::memory_order_release);
                return ETV_ERR_HIP;
            }
            g_scratch_ptr[dev] = d;
            g_scratch_state[dev].store(2, std::memory_order_release);
        } else {
            while (g_scratch_state[dev].load(std::memory_order_acquire) == 1) { /* another thread is asking */ }
            if (g_scratch_state[dev].load(std::memory_order_acquire) != 2) return ETV_ERR_HIP;
        }
    }
    *ptr = g_scratch_ptr[dev];
    return ETV_OK;
}
}  // namespace etv

extern "C" int32_t etv_tree_verify_attention_static(const etv_attn_desc *h, const void *q, const void *k_cache,
                                                    const void *v_cache, const int32_t *block_table,
                                                    const int32_t *prefix_len, const void *kt, const void *vt,
                                                    const uint64_t *bitmask, const int32_t *n_nodes, void *out,
                                                    float *lse, void *stream) {
    if (!h) return ETV_ERR_INVALID_ARG;
    // sizes beyond the array are refused before anything is launched
    if (etv_tree_verify_attention_workspace_bytes(h) > (size_t)ETV_ATTN_STATIC_WORKSPACE_BYTES)
        return ETV_ERR_WORKSPACE_TOO_SMALL;
    void *ws = nullptr;
    const int32_t rc = etv::static_scratch(&ws);
    if (rc != ETV_OK) return rc;
    // Nothing in the array has to start at zero: a launch writes every (m, l, O) partial it later merges, and
    // never reads one it has not written (absent splits and padded rows are skipped), so the last call's
    // contents are harmless.
    return etv::attention_run(h, q, k_cache, v_cache, block_table, prefix_len, kt, vt, bitmask, n_nodes, out, lse, ws,
                              (size_t)ETV_ATTN_STATIC_WORKSPACE_BYTES, stream);
}
