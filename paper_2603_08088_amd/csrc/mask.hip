// build_tree_mask: ancestor bitmask, dense 4D mask, depths and structural-invariant status.
// Section 3.2 ("Ancestor tables", "Structural invariants") and Section 3.3 ("Tree attention
// mask", "Implementation note": compact ancestor encoding produced on the device).
// tensorize_tree: the same launch also writes position ids (Section 3.3 "Execution view": prefix
// length + depth) and the table of root-to-leaf paths that the gather and the acceptance step
// consume, so nothing about the tree is computed on the host.
#include <algorithm>

#include "etv_common.h"

namespace etv {

constexpr int kMaskWords = ETV_MAX_TREE / 64;

// One workgroup per sequence, one thread per node row.  Instead of materialising the
// (D_max+1) x T ancestor table, each thread follows its own parent chain (bounded by the
// node count) and ORs the visited rows into registers: the same relation, no table.
//
// Paths (PATHS): a leaf is a valid node that no valid node names as its parent; leaves are
// ranked in ascending row order with one ballot per wavefront; the thread of the leaf ranked r writes row r from
// the last sixteen nodes of its chain, kept in registers as they were visited (deeper leaves walk once more, back to
// front), then pads the row with -1; rows beyond the last leaf are filled by all threads together.
//
// One workgroup and no bandwidth: what bounds it are the trips to memory and LDS in series.  Sizes, parents and the prefix length
// come in one trip (the parent of a row behind the last node is read and dropped), the chain is walked once, and beyond 32 nodes
// 256 threads share the dense mask and the padding whatever the node count is.  The dense mask of a large tree is spread over
// several workgroups (blockIdx.y, in batches that leave room for them), each of which works out the few KiB of rows for itself; the first writes everything else.  With paths, in graphs: B = 1,
// T = 60 4.7 -> 3.8 us; B = 32, T = 128 6.9 -> 4.8; B = 4, T = 250 30.5 -> 5.0 (16.2 without the further workgroups).
// Without paths nothing of a chain is kept but its bits (PATHS): bit mask of B = 4096, T = 128 6.5 -> 5.9 us, of B = 32, T = 60 3.03 -> 2.88.
template <bool PATHS>
__global__ void __launch_bounds__(ETV_MAX_TREE) build_tree_mask_kernel(
    const int32_t *__restrict__ parent, const int32_t *__restrict__ n_nodes, int T_max, int words,
    const int32_t *__restrict__ prefix_len, uint64_t *__restrict__ bitmask, uint8_t *__restrict__ dense, int32_t *__restrict__ depth,
    int32_t *__restrict__ status, int32_t *__restrict__ position_ids,
    int32_t *__restrict__ retrieve, int32_t *__restrict__ n_paths, int L_max, int W) {
    __shared__ int32_t s_ep[ETV_MAX_TREE];                 // effective parent after range/closure repair
    __shared__ uint64_t s_bits[ETV_MAX_TREE][kMaskWords];  // rows, for the cooperative dense write
    __shared__ int32_t s_status;
    __shared__ uint8_t s_child[ETV_MAX_TREE];
    __shared__ int32_t s_wave_leaves[ETV_MAX_TREE / 64];
    const int b = blockIdx.x, part = blockIdx.y, parts = gridDim.y;
    const int k = threadIdx.x;
    const int32_t p = parent[(size_t)b * T_max + min(k, T_max - 1)];
    const int n_raw = n_nodes[b];
    const int P_raw = prefix_len ? prefix_len[b] : 0;
    if (k == 0) s_status = 0;
    if constexpr (PATHS) s_child[k] = 0;
    const int n = clampi(n_raw, 0, T_max);
    int32_t st = 0, ep = 0;
    if (k < n) {
        if (k == 0) {
            if (p != 0) st |= ETV_TREE_RANGE;
        } else if (p < 0 || p >= T_max) {
            st |= ETV_TREE_RANGE;
        } else if (p >= n) {
            st |= ETV_TREE_CLOSURE;
        } else {
            ep = p;
        }
        s_ep[k] = ep;
    }
    __syncthreads();
    uint64_t bits[kMaskWords];
#pragma unroll
    for (int w = 0; w < kMaskWords; w++) bits[w] = 0;
    uint64_t chain = 0, chain_hi = 0;  // the last sixteen nodes visited, a byte each, the latest lowest
    int dep = 0;
    if (k < n) {
        int cur = k, steps = 0;
        while (cur != 0 && steps < n) {
#pragma unroll
            for (int w = 0; w < kMaskWords; w++)
                if ((cur >> 6) == w) bits[w] |= 1ull << (cur & 63);
            if constexpr (PATHS) {
                chain_hi = chain_hi << 8 | chain >> 56;
                chain = chain << 8 | (uint32_t)cur;
            }
            cur = s_ep[cur];
            steps++;
        }
        if (cur == 0) {
            bits[0] |= 1ull;
            dep = steps;
        } else {  // the chain never reaches the root: a cycle.  Re-attach k to the root.
            st |= ETV_TREE_CYCLE;
#pragma unroll
            for (int w = 0; w < kMaskWords; w++) bits[w] = ((k >> 6) == w) ? (1ull << (k & 63)) : 0ull;
            bits[0] |= 1ull;
            dep = 1;
            chain = (uint32_t)k;
            ep = 0;  // s_ep keeps the cycle: no chain that reaches the root passes it
        }
    }
    if constexpr (PATHS)
        if (k >= 1 && k < n) s_child[ep] = 1;
    if (st) atomicOr(&s_status, st);
    if (k < T_max) {
#pragma unroll
        for (int w = 0; w < kMaskWords; w++) {
            s_bits[k][w] = bits[w];
            if (w < words && part == 0) bitmask[((size_t)b * T_max + k) * words + w] = bits[w];
        }
        if (depth && part == 0) depth[(size_t)b * T_max + k] = dep;
        if (position_ids && part == 0) position_ids[(size_t)b * T_max + k] = max(P_raw, 0) + dep;
    }
    __syncthreads();
    if (PATHS && part == 0) {
        const bool leaf = k < n && !s_child[k];
        const unsigned long long lb = __ballot(leaf);
        const int wv = k >> 6;
        int rank = __popcll(lb & ((1ull << (k & 63)) - 1ull));
        int total = __popcll(lb);
        if (blockDim.x > 64) {
            if ((k & 63) == 0) s_wave_leaves[wv] = total;
            __syncthreads();
            total = 0;
            for (int w = 0; w < (int)(blockDim.x >> 6); w++) {
                if (w < wv) rank += s_wave_leaves[w];
                total += s_wave_leaves[w];
            }
        }
        int32_t *rows = retrieve + (size_t)b * L_max * W;
        st = 0;
        if (leaf && rank < L_max) {
            int32_t *row = rows + (size_t)rank * W;
            if (dep + 1 > W) st |= ETV_TREE_DEPTH;
            if (dep <= 16) {
                row[0] = 0;
                for (int i = 1; i <= min(dep, W - 1); i++) {
                    row[i] = (int32_t)(chain & 255);
                    chain = chain >> 8 | chain_hi << 56;
                    chain_hi >>= 8;
                }
            } else {
                int cur = k;
                for (int i = dep; i >= 0; i--) {  // dep <= n - 1: the walk above reached the root in dep steps
                    if (i < W) row[i] = cur;
                    cur = s_ep[cur];
                }
            }
            for (int i = dep + 1; i < W; i++) row[i] = -1;
        }
        if (total > L_max) st |= ETV_TREE_PATHS;
        const int kept = min(total, L_max);
        for (int e = kept * W + k; e < L_max * W; e += blockDim.x) rows[e] = -1;
        if (n_paths && k == 0) n_paths[b] = kept;
        if (st) atomicOr(&s_status, st);
        __syncthreads();
    }
    if (k == 0 && part == 0) status[b] = s_status;
    if (dense) {
        uint8_t *out = dense + (size_t)b * T_max * T_max;
        if ((T_max & 3) == 0 && (((uintptr_t)dense) & 3) == 0) {
            // four mask bytes per store: thread k keeps one 4-byte group of a row and walks down the rows
            // (groups = T_max / 4 <= 64 <= blockDim: one division per thread, none per element)
            const int groups = T_max >> 2;
            // exact: every quotient is 0.5 / 64 or more from a whole number
            const auto by_groups = [&](int x) { return (int)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)groups)); };
            const int row0 = by_groups(k), g = k - row0 * groups, rstep = by_groups((int)blockDim.x);
            uint32_t *out4 = reinterpret_cast<uint32_t *>(out);
#pragma unroll 4
            for (int row = row0 + part * rstep; row < T_max && row0 < rstep; row += parts * rstep) {
                const uint32_t nib = (uint32_t)(s_bits[row][g >> 4] >> ((g & 15) * 4)) & 15u;
                out4[row * groups + g] = (nib * 0x00204081u) & 0x01010101u;  // bit i of the nibble -> byte i
            }
        } else {
            // rows begin anywhere: the aligned words of the whole matrix, which may span rows, and bytes at its two ends
            const int total = T_max * T_max, ahead = (int)((uintptr_t)out & 3);
            const float inv = __builtin_amdgcn_rcpf((float)T_max);
            const auto byte_of = [&](int e) {
                const int row = (int)(((float)e + 0.5f) * inv), col = e - row * T_max;  // exact: 0.5 / 256 or more from a whole number
                return (uint32_t)(s_bits[row][col >> 6] >> (col & 63)) & 1u;
            };
#pragma unroll 2
            for (int e = 4 * (part * (int)blockDim.x + k) - ahead; e < total; e += 4 * parts * (int)blockDim.x) {
                if (e >= 0 && e + 4 <= total) {
                    *reinterpret_cast<uint32_t *>(out + e) = byte_of(e) | byte_of(e + 1) << 8 | byte_of(e + 2) << 16 | byte_of(e + 3) << 24;
                } else {
                    for (int i = max(e, 0); i < min(e + 4, total); i++) out[i] = (uint8_t)byte_of(i);
                }
            }
        }
    }
}

// Work beside the nodes' own (the dense mask, the padding of the paths) is shared by 256 threads from 33 nodes on, and a dense mask of more
// than 64 nodes by several workgroups, four words a thread: 4 at 128 nodes, 16 at 256.  Both only while the launch leaves compute
// units idle, up to two workgroups of 256 threads for each or four with the parts: beyond that further ones repeat the chains for
// nothing.  Dense masks, B = 2048, T = 128 10.2 us with a workgroup a tree, 16.7 with four, 9.3 by this rule; B = 256, T = 256 9.1, 11.8
// (sixteen) and 6.8; neither mask nor paths, B = 4096, T = 40 4.4 us with 64 threads, 6.0 with 256.
static int mask_threads(int B, int T_max, bool more_work) { return more_work && T_max > 32 && B <= 512 ? ETV_MAX_TREE : (T_max + 63) / 64 * 64; }
static int mask_parts(int B, int T_max, const void *dense) { return dense ? std::max(1, std::min((T_max * T_max + 4095) / 4096, 1024 / B)) : 1; }

}  // namespace etv

extern "C" int32_t etv_build_tree_mask(const int32_t *parent, const int32_t *n_nodes, int32_t B, int32_t T_max,
                                       uint64_t *bitmask, uint8_t *dense, int32_t *depth, int32_t *status,
                                       void *stream) {
    if (!parent || !n_nodes || !bitmask || !status || B < 0) return ETV_ERR_INVALID_ARG;
    if (T_max < 1) return ETV_ERR_INVALID_ARG;
    if (T_max > ETV_MAX_TREE) return ETV_ERR_UNSUPPORTED;
    if (B == 0) return ETV_OK;
    int threads = etv::mask_threads(B, T_max, dense != nullptr);
    int words = (T_max + 63) / 64;
    hipLaunchKernelGGL(etv::build_tree_mask_kernel<false>, dim3(B, etv::mask_parts(B, T_max, dense)), dim3(threads), 0, etv::as_stream(stream), parent,
                       n_nodes, (int)T_max, words, (const int32_t *)nullptr, bitmask, dense, depth, status,
                       (int32_t *)nullptr, (int32_t *)nullptr, (int32_t *)nullptr, 0, 0);
    return etv::check_launch();
}

extern "C" int32_t etv_tensorize_tree(const int32_t *parent, const int32_t *n_nodes, const int32_t *prefix_len,
                                      int32_t B, int32_t T_max, int32_t L_max, int32_t W, uint64_t *bitmask,
                                      uint8_t *dense, int32_t *depth, int32_t *position_ids, int32_t *retrieve,
                                      int32_t *n_paths, int32_t *status, void *stream) {
    if (!parent || !n_nodes || !bitmask || !retrieve || !status || B < 0) return ETV_ERR_INVALID_ARG;
    if (T_max < 1 || L_max < 1 || W < 1) return ETV_ERR_INVALID_ARG;
    if (position_ids && !prefix_len) return ETV_ERR_INVALID_ARG;
    if (T_max > ETV_MAX_TREE) return ETV_ERR_UNSUPPORTED;
    if ((long)L_max * W > (1l << 24)) return ETV_ERR_UNSUPPORTED;
    if (B == 0) return ETV_OK;
    int threads = etv::mask_threads(B, T_max, true);
    int words = (T_max + 63) / 64;
    hipLaunchKernelGGL(etv::build_tree_mask_kernel<true>, dim3(B, etv::mask_parts(B, T_max, dense)), dim3(threads), 0, etv::as_stream(stream), parent,
                       n_nodes, (int)T_max, words, prefix_len, bitmask, dense, depth, status, position_ids, retrieve,
                       n_paths, (int)L_max, (int)W);
    return etv::check_launch();
}
