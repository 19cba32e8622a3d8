// Greedy acceptance, bonus token and KV roll-back (paper Algorithm 1: the walk
// for the longest accepted prefix, the bonus token from the target's own
// prediction, and the roll-back of the KV cache along the accepted path).  All
// integer work; results are exact.
#include "common.hpp"

namespace {

// The tree's arrays and, for every node, its ancestor-or-self set as a 128-bit mask (bit a of anc[i] set when a is
// on the path root..i): the tree attention mask in compact form.  One workgroup, parent[] in LDS.  Bound by one
// launch: as two kernels (upload, then masks from the uploaded parents) every new tree paid a second one, 1.2 us of the
// 26.5 us that a tree and its attention over 4096 rows take.
__global__ __launch_bounds__(CATS_MAX_TREE) void cats_tree_upload(TreeUploadArgs a, int n, int32_t* token,
                                                                  int32_t* parent, int32_t* depth, u32x4* anc) {
    __shared__ int32_t s_parent[CATS_MAX_TREE];
    const int i = threadIdx.x;
    if (i < n) {
        token[i] = a.token[i];
        parent[i] = s_parent[i] = a.parent[i];
        depth[i] = a.depth[i];
    }
    __syncthreads();
    if (i >= n) return;
    u32x4 mask = u32x4{0u, 0u, 0u, 0u};
    int node = i;
    for (int step = 0; step <= CATS_MAX_DEPTH && node >= 0; ++step) {
        const uint32_t bit = 1u << (node & 31);
        const int w = node >> 5;
        mask |= u32x4{w == 0 ? bit : 0u, w == 1 ? bit : 0u, w == 2 ? bit : 0u, w == 3 ? bit : 0u};
        node = s_parent[node];
    }
    anc[i] = mask;
}

// A node is accepted when every node on its path (root excluded) carries the
// token the target predicts at that node's parent.  The committed path ends at
// the deepest accepted node, lowest index first among equals.
// edge_ok (optional): per node, 1 when the node's token passes the acceptance criterion at its
// parent; absent = greedy, the token must equal the parent's argmax.
struct WalkShared {
    int32_t tok[CATS_MAX_TREE], par[CATS_MAX_TREE], dep[CATS_MAX_TREE], amax[CATS_MAX_TREE];
    int key[CATS_MAX_TREE / 64];
    int n, bonus;                        // accepted nodes below the root, bonus token
    int32_t path[CATS_MAX_DEPTH + 1];    // nodes 0 .. n of the committed path
};
// The whole workgroup (64 or 128 threads); the result is in s for all of them.
__device__ __forceinline__ void accept_walk(const AcceptArgs& a, WalkShared& s) {
    const int tid = threadIdx.x, nt = blockDim.x;
    for (int i = tid; i < a.T; i += nt) {
        s.tok[i] = a.token[i];
        s.par[i] = a.parent[i];
        s.dep[i] = a.depth[i];
        s.amax[i] = a.amax[i];
    }
    __syncthreads();
    int key = -1;  // depth * MAX_TREE + (MAX_TREE-1 - index): larger = deeper, then lower index
    for (int i = tid; i < a.T; i += nt) {
        bool ok = true;
        int node = i;
        for (int step = 0; step < CATS_MAX_DEPTH && node > 0; ++step) {
            const int p = s.par[node];
            ok = ok && (a.edge_ok ? a.edge_ok[node] != 0 : s.tok[node] == s.amax[p]);
            node = p;
        }
        if (ok) key = max(key, s.dep[i] * CATS_MAX_TREE + (CATS_MAX_TREE - 1 - i));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) key = max(key, __shfl_xor(key, o));
    if ((tid & 63) == 0) s.key[tid >> 6] = key;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < nt / 64; ++w) key = max(key, s.key[w]);
        const int best = CATS_MAX_TREE - 1 - (key % CATS_MAX_TREE);
        s.n = s.dep[best];
        s.bonus = s.amax[best];
        int node = best;
        for (int k = s.n; k >= 0; --k) {
            s.path[k] = node;
            node = s.par[node];
        }
    }
    __syncthreads();
}
__device__ __forceinline__ void write_result(const AcceptArgs& a, const WalkShared& s) {
    const int k = threadIdx.x;
    if (k <= CATS_MAX_DEPTH) {
        a.out->path[k] = k > s.n ? -1 : s.path[k];
        a.out->tokens[k] = k > s.n ? -1 : s.tok[s.path[k]];
    }
    if (k == 0) {
        a.out->n_accepted = s.n;
        a.out->bonus_token = s.bonus;
        a.out->new_ctx_len = a.ctx_len + s.n + 1;
    }
}

__global__ __launch_bounds__(CATS_MAX_TREE) void cats_accept(AcceptArgs a) {
    __shared__ WalkShared s;
    accept_walk(a, s);
    write_result(a, s);
}

// Typical acceptance (the criterion the paper cites for Acc = typical): node j passes when the
// probability of its token under its parent's distribution p = softmax(logits / temperature)
// exceeds min(epsilon, delta * exp(-H(p))).  The parent's log-sum-exp and entropy come from the
// LM-head epilogue; the one logit needed per node is added up from the GEMM's partial tiles.
__global__ __launch_bounds__(CATS_MAX_TREE) void cats_typical_edges(TypicalArgs a) {
    const int j = threadIdx.x;
    if (j >= a.T) return;
    if (j == 0) {
        a.edge_ok[0] = 1;
        a.prob[0] = 1.f;
        a.thr[0] = 0.f;
        return;
    }
    const int p = a.parent[j];
    const float logit = row_scale(a.ns, p) * sum_pieces(a.part, a.plan, a.T, a.ld, p, a.token[j]);
    const float prob = expf(logit * a.inv_temp - a.lse[p]);
    const float thr = fminf(a.epsilon, a.delta * expf(-a.entropy[p]));
    a.prob[j] = prob;
    a.thr[j] = thr;
    a.edge_ok[j] = prob > thr ? 1 : 0;
}

// Row ctx_len + path[k] -> row ctx_len + k for k = 0..n-1, one workgroup per (layer, head, keys or
// values): keys are [row][dim], values [dim][row]; thread dd owns one head dimension, reads all its source
// elements first and only then writes, so overlapping source/destination rows cannot clobber each other.
// Rows that stay where they are (the root's always) are not read: bound by the 128-byte line that every (layer, head,
// dimension) of the values costs, 26 MB for 40 layers of 40 heads.  cats_accept_compact, reading every row of the path ->
// this, us: that shape with nothing accepted 11.0 -> 5.1, 32 layers of 32 heads with four nodes accepted 12.3 -> 10.9.
__device__ __forceinline__ void compact_rows(const CompactArgs& a, int n, const int32_t* committed) {
    const int l = blockIdx.x, h = blockIdx.y, which = blockIdx.z, dd = threadIdx.x;
    int path[CATS_MAX_DEPTH + 1];
    bf16_t val[CATS_MAX_DEPTH + 1];
#pragma unroll
    for (int k = 0; k <= CATS_MAX_DEPTH; ++k) path[k] = k < n ? committed[k] : k;
    if (which == 0) {
        bf16_t* base = a.k[l] + (static_cast<size_t>(h) * a.max_ctx + a.ctx_len) * a.d + dd;
#pragma unroll
        for (int k = 0; k <= CATS_MAX_DEPTH; ++k)
            if (path[k] != k) val[k] = base[static_cast<size_t>(path[k]) * a.d];
#pragma unroll
        for (int k = 0; k <= CATS_MAX_DEPTH; ++k)
            if (path[k] != k) base[static_cast<size_t>(k) * a.d] = val[k];
    } else {
        bf16_t* base = a.v[l] + (static_cast<size_t>(h) * a.d + dd) * a.max_ctx + a.ctx_len;
#pragma unroll
        for (int k = 0; k <= CATS_MAX_DEPTH; ++k)
            if (path[k] != k) val[k] = base[path[k]];
#pragma unroll
        for (int k = 0; k <= CATS_MAX_DEPTH; ++k)
            if (path[k] != k) base[k] = val[k];
    }
}

// The roll-back alone, along the path of an earlier walk.
__global__ void cats_kv_compact(CompactArgs a, const cats_accept_result* res) {
    compact_rows(a, res->n_accepted + 1, res->path);
}

// The walk and the roll-back behind it in one launch: every workgroup walks the tree for itself, the first one writes the
// result.  The walk is a few hundred bytes of L2 hits and dependent LDS reads: up to CATS_MAX_DEPTH parents for a node (for two,
// one after the other, where the 64 threads of head size 64 have more than 64 nodes) and the committed path's again.  Bound by
// that latency where there is little to move, else by the values' lines (compact_rows).  What is saved is a dependent launch:
// with the tree upload, the rotation table beside the first rows and the final rows written in place, a two-layer step of 15
// nodes takes 81.9 instead of 88.8 us; alone, 2 layers of 64 heads of 64, 128 nodes, a path of 16 accepted 8.7 -> 7.6.
__global__ __launch_bounds__(128) void cats_accept_compact(AcceptArgs w, CompactArgs a) {
    __shared__ WalkShared s;
    accept_walk(w, s);
    if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0) write_result(w, s);
    compact_rows(a, s.n + 1, s.path);
}

}  // namespace

void launch_tree_upload(const TreeUploadArgs& a, int n, int32_t* token, int32_t* parent,
                        int32_t* depth, u32x4* anc, hipStream_t st) {
    hipLaunchKernelGGL(cats_tree_upload, dim3(1), dim3(CATS_MAX_TREE), 0, st, a, n, token, parent, depth, anc);
}

void launch_accept(const AcceptArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(cats_accept, dim3(1), dim3(CATS_MAX_TREE), 0, st, a);
}

void launch_accept_compact(const AcceptArgs& w, const CompactArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(cats_accept_compact, dim3(a.n_layers, a.nh, 2), dim3(a.d), 0, st, w, a);
}

void launch_typical_edges(const TypicalArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(cats_typical_edges, dim3(1), dim3(CATS_MAX_TREE), 0, st, a);
}

void launch_compact(const CompactArgs& a, const cats_accept_result* res, hipStream_t st) {
    hipLaunchKernelGGL(cats_kv_compact, dim3(a.n_layers, a.nh, 2), dim3(a.d), 0, st, a, res);
}
