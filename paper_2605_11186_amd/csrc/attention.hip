// Tree-masked attention over the KV cache plus the tree nodes (paper Fig. 4,
// right-lower: the tree attention mask; Sec. 3.2 "Target verification pass").
//
// Node i attends to cache rows [0, ctx_len) and to rows ctx_len + a for every a
// on its root-to-node path.  The ancestor sets are 128-bit masks, built from parent[] in
// LDS by cats_tree_upload when the tree is set and read here one mask per query.
//
// Work split: one workgroup of W waves per (head, chunk of key blocks, group of
// 16 or 32 queries, see attn_split); wave w takes the chunk's blocks w, w + W, ... and the waves'
// partial results are merged through LDS.  With more than one chunk the workgroup then
// publishes its chunk's result, and the last workgroup of a (head, query group) to arrive adds
// up all chunks in chunk order with the usual log-sum-exp rescaling and writes the output:
// one kernel, no separate merge launch.
// What bounds it: at short contexts a chain of memory round trips (queries and first block, values with
// low parts, hand-over between chunks), at long ones the waves' arithmetic and the 128-byte lines a compute
// unit can have in flight.  One register set: the next block's keys and values are requested into the registers that
// this block's products have just freed.  Four or eight waves, see attn_waves.  With eight waves, head_dim 128
// and 32 queries the 256 registers of a wave do not quite do: 16 spill around the run of blocks with low parts (at most one or two
// blocks of a wave), none in the context loop.  Four waves of 64 queries (half the key and value traffic) were slower than
// eight waves of 32 at every size: 33.3 against 25.8 us at 64 nodes / 4096 rows, 26.2 against 18.3 at 63 / 1024.
// Scores are computed transposed, S^T = K Q^T, with the 16x16x32 bf16 MFMA, so a
// lane owns ONE query column and 8 keys of every 32-key block: the running
// max / sum of the online softmax are per-lane scalars shared by four lanes and
// reduced with two wave shuffles, and the probabilities are already laid out as
// the B operand of the second product O^T = V^T P^T.  Queries and probabilities are
// fed as high + low bf16 parts.  V is cached transposed ([head][dim][row]) so that its A
// operand is a plain 128-bit load as well; no LDS round trip for K, V or P.
// The key blocks that hold rows appended by the running call (the tree's own rows) also take
// those rows' low parts from the window beside the cache (see AttnArgs): one more product per
// fragment there, so that tree nodes see each other at about 16 mantissa bits while context
// rows are what the bf16 cache holds.
#include <type_traits>

#include "common.hpp"

namespace {

// which 16-bit elements of an 8-key vector belong to keys key0 + e in [lo, hi): all ones there, zero elsewhere
__device__ __forceinline__ u32x4 keys_kept(int key0, int lo, int hi) {
    u32x4 m;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int ka = key0 + 2 * e, kb = ka + 1;
        m[e] = (ka >= lo && ka < hi ? 0x0000FFFFu : 0u) | (kb >= lo && kb < hi ? 0xFFFF0000u : 0u);
    }
    return m;
}

// 16-byte device-coherent store: it goes past the XCD's L2
__device__ __forceinline__ void store_coherent16(float* p, f32x4 v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1" ::"v"(p), "v"(v) : "memory");
}

// 16-byte device-coherent load (sc1: it bypasses the per-XCD caches) at a byte offset from a base that is
// the same for the whole wave; a builtin, so that the compiler knows when the value has arrived.
constexpr int AUX_SC1 = 16;
__device__ __forceinline__ f32x4 load_coherent16(const float* base, uint32_t bytes, uint32_t offset) {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, bytes, 0x00027000);
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, offset, 0, AUX_SC1));
}

// MFMA 16x16x32 bf16 (wave64): lane l supplies, for A, row l%16 and
// k = 8*(l/16)..+7; for B, column l%16 and the same k; its 4 results are
// D[4*(l/16) + r][l%16].
// QB: 16-query groups per wave (a workgroup covers QN = 16 * QB queries); W: waves per workgroup.
template <int D, int QB, int W>
__global__ __launch_bounds__(64 * W) void cats_tree_attention_kernel(AttnArgs a) {
    constexpr int QN = 16 * QB;
    constexpr int KS = D / 32;  // k-steps of the score product
    constexpr int DB = D / 16;  // 16-row blocks of O^T
    __shared__ float s_o[W][QN][D + 4];
    __shared__ float s_ml[W][QN][2];
    __shared__ int s_last;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, q4 = lane >> 4;
    const int chunk = blockIdx.x, h = blockIdx.y, qbase = blockIdx.z * QN;
    const int S = a.ctx_len, T = a.T, Tq = a.Tq;   // T tree nodes are keys; Tq of them (from q0) are queries
    const int n_keys = S + T;

    // ancestor-or-self masks of this lane's queries
    u32x4 anc[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int t = qbase + 16 * qb + m;
        anc[qb] = t < Tq ? a.anc[a.q0 + t] : u32x4{0u, 0u, 0u, 0u};
    }

    // Q^T fragments (B operand of the score product): column = query, k = dim; queries come
    // as high + low bf16 parts (the low part may be absent)
    bf16x8 qf[QB][KS], qfl[QB][KS];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int t = qbase + 16 * qb + m;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            u32x4 v = u32x4{0u, 0u, 0u, 0u}, vl = u32x4{0u, 0u, 0u, 0u};
            const size_t off = static_cast<size_t>(min(t, Tq - 1)) * a.H + h * D + 32 * s + 8 * q4;
            if (t < Tq) {
                v = *reinterpret_cast<const u32x4*>(a.q + off);
                if (a.q_lo) vl = *reinterpret_cast<const u32x4*>(a.q_lo + off);
            }
            qf[qb][s] = as_bf16x8(v);
            qfl[qb][s] = as_bf16x8(vl);
        }
    }

    f32x4 o[QB][DB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int db = 0; db < DB; ++db) o[qb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mrun[QB], lrun[QB];   // running maximum (base 2), this lane's share of the row sum
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        mrun[qb] = -1e30f;
        lrun[qb] = 0.f;
    }
    bool fresh = true;           // nothing accumulated yet (wave-uniform)

    const float scale = rsqrtf(static_cast<float>(D)) * 1.44269504088896340736f;   // 1/sqrt(d) * log2(e)
    const bf16_t* kbase = a.kc + static_cast<size_t>(h) * a.max_ctx * D;
    const bf16_t* vbase = a.vt + static_cast<size_t>(h) * D * a.max_ctx;

    const int n_blocks = (n_keys + ATTN_KB - 1) / ATTN_KB;
    // Chunks are contiguous runs of key blocks (neighbouring blocks share cache lines of the
    // transposed values) of equal cost: a block that holds tree rows counts twice (masks, low
    // parts, no prefetch), so the chunk that ends with them gets fewer blocks.  Cost units: block b
    // starts at unit b below the first tree block tb, at tb + 2 (b - tb) from there on; chunk c
    // owns the blocks whose first unit lies in [c U / n, (c + 1) U / n).
    const int tree_blk = min(n_blocks, S / ATTN_KB);
    const int units = tree_blk + 2 * (n_blocks - tree_blk);
    auto first_block_at = [&](int u) {   // first block whose first unit is >= u
        return u <= tree_blk ? u : tree_blk + (u - tree_blk + 1) / 2;
    };
    const int blk_begin = first_block_at((chunk * units + a.n_chunks - 1) / a.n_chunks);
    const int blk_end = chunk + 1 == a.n_chunks ? n_blocks
                                                : first_block_at(((chunk + 1) * units + a.n_chunks - 1) / a.n_chunks);
    constexpr int blk_stride = W;

    // The K / V fragments of one 32-key block.  Score-block rows are permuted so that a lane
    // ends up with 8 consecutive keys: sub-block b, MFMA row mm <-> key j0 + 8*(mm/4) + 4*b + mm%4.
    // V^T fragments: row = dim, k = 8 consecutive keys starting at j0 + 8*q4.
    // Element numbers inside a head take 64 bits (2^25 keys of 128 are 2^32): a block's place is added to the head's
    // base as a scalar, a lane's place inside a key block takes 32.  A lane's row of values is formed anew at every
    // load where registers are short (head_dim 128; the empty asm keeps it there) and kept as a pointer where they
    // are not.  Launches inside a layer against 32-bit numbers (which are wrong there), us: 32 heads of 128, 16 nodes, 512
    // rows 13.9 -> 13.6, 1024 rows 14.6 -> 14.3, 4096 rows 21.8 -> 21.2; with the values' row kept 14.5, 15.6, 22.7.
    // Heads of 64: the same within 1 % either way over 36 sizes.
    auto load_k = [&](bf16x8 (&kf)[2][KS], int blk) {
        const bf16_t* kb = kbase + static_cast<size_t>(__builtin_amdgcn_readfirstlane(blk)) * (ATTN_KB * D);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const uint32_t off = static_cast<uint32_t>(8 * (m >> 2) + 4 * b + (m & 3)) * D + 8 * q4;
#pragma unroll
            for (int s = 0; s < KS; ++s) kf[b][s] = as_bf16x8(*reinterpret_cast<const u32x4*>(kb + off + 32 * s));
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    const bf16_t* v_row = vbase + static_cast<size_t>(m) * a.max_ctx + 8 * q4;
    auto load_v = [&](bf16x8 (&vf)[DB], int blk) {
        const bf16_t* vb = v_row + static_cast<uint32_t>(blk * ATTN_KB);
        if constexpr (D == 128) {
            int m_here = m;
            asm volatile("" : "+v"(m_here));
            const size_t v_lane = static_cast<size_t>(m_here) * a.max_ctx + 8 * q4;
            vb = vbase + __builtin_amdgcn_readfirstlane(blk * ATTN_KB) + v_lane;
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
            vf[db] = as_bf16x8(*reinterpret_cast<const u32x4*>(vb + static_cast<size_t>(16 * db) * a.max_ctx));
        __builtin_amdgcn_sched_barrier(0);
    };
    // The low parts of the same fragments from the window; rows outside [lo_begin, lo_end) are
    // stale there and come out as zeros.  Addresses are clamped into the window (what a clamp
    // moves is masked anyway: the window covers every row of the range).
    const int win_base = S & ~(ATTN_KB - 1);
    // (one mask of eight keys for all of a block's dims; formed at each vector, and with the ancestor bits looked up key by
    // key, masks were more than half of the instructions, at about 2 ns each, of a block with low parts.  Launches in a
    // layer, us: 32 heads of 128, 63 nodes / 1024 rows 14.3 -> 13.7, 128 / 512 15.9 -> 14.8, 16 / 512 8.6 as before)
    auto keep = [](bf16x8 (&v)[DB], u32x4 m) {
#pragma unroll
        for (int db = 0; db < DB; ++db) v[db] = as_bf16x8(__builtin_bit_cast(u32x4, v[db]) & m);
    };
    auto mask_v = [&](bf16x8 (&v)[DB], int blk) {   // rows past the tree may hold anything
        if ((blk + 1) * ATTN_KB > n_keys) keep(v, keys_kept(blk * ATTN_KB + 8 * q4, 0, n_keys));
    };
    auto request_k_lo = [&](bf16x8 (&kf)[2][KS], int blk) {
        const bf16_t* kl = a.k_lo + static_cast<size_t>(h) * TREE_WIN * D;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int key = blk * ATTN_KB + 8 * (m >> 2) + 4 * b + (m & 3);
            const int w = min(key - win_base, TREE_WIN - 1);
#pragma unroll
            for (int s = 0; s < KS; ++s)
                kf[b][s] = as_bf16x8(*reinterpret_cast<const u32x4*>(kl + static_cast<size_t>(w) * D + 32 * s + 8 * q4));
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto keep_k_lo = [&](bf16x8 (&kf)[2][KS], int blk) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int key = blk * ATTN_KB + 8 * (m >> 2) + 4 * b + (m & 3);
            const bool ok = key >= a.lo_begin && key < a.lo_end;
#pragma unroll
            for (int s = 0; s < KS; ++s)
                kf[b][s] = as_bf16x8(ok ? __builtin_bit_cast(u32x4, kf[b][s]) : u32x4{0u, 0u, 0u, 0u});
        }
    };
    auto request_v_lo = [&](bf16x8 (&vf)[DB], int blk) {
        // (the window of a head is small: 32-bit offsets where registers are short)
        const bf16_t* vl = a.vt_lo + static_cast<size_t>(h) * D * TREE_WIN;
        const int key0 = blk * ATTN_KB + 8 * q4;
        const int w0 = min(key0 - win_base, TREE_WIN - 8);
#pragma unroll
        for (int db = 0; db < DB; ++db)
            vf[db] = as_bf16x8(*reinterpret_cast<const u32x4*>(
                D == 128 ? vl + static_cast<uint32_t>((16 * db + m) * TREE_WIN + w0)
                         : vl + static_cast<size_t>(16 * db + m) * TREE_WIN + w0));
        __builtin_amdgcn_sched_barrier(0);
    };
    auto keep_v_lo = [&](bf16x8 (&vf)[DB], int blk) { keep(vf, keys_kept(blk * ATTN_KB + 8 * q4, a.lo_begin, a.lo_end)); };

    // MODE 0: every key of the block is a context row (no mask, no tail: straight-line code);
    // MODE 1: the block may hold tree rows and rows past the tree; MODE 2: as 1, and the block
    // also has low parts of keys and values.  Scores and running maxima are kept in
    // the base-2 domain (the scale carries log2 e), so that every exponential is one v_exp_f32.
    bf16x8 kf[2][KS], vf[DB];
    f32x4 st[QB][2];
    auto scores = [&](const bf16x8 (&k)[2][KS], const bf16x8 (&kl)[2][KS], auto lo_tag) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                st[qb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    st[qb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[b][s], qf[qb][s], st[qb][b], 0, 0, 0);
                    st[qb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[b][s], qfl[qb][s], st[qb][b], 0, 0, 0);
                    if constexpr (decltype(lo_tag)::value)
                        st[qb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kl[b][s], qf[qb][s], st[qb][b], 0, 0, 0);
                }
            }
    };
    // the block's probabilities and their product with its values
    auto weigh = [&](const bf16x8 (&v)[DB], const bf16x8 (&vl)[DB], int blk, auto mode_tag) {
        constexpr int MODE = decltype(mode_tag)::value;
        constexpr bool LO = MODE == 2;
        const int key0 = blk * ATTN_KB + 8 * q4;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            // this lane: query column m of group qb, keys key0 .. + 7.  Bit i of vis: key0 + i may be seen (context rows all
            // may, tree rows by the ancestor mask, rows past the tree not: their bits are zero)
            uint32_t vis = 0xffu;
            if constexpr (MODE != 0) {
                const int rel = key0 - S, w = rel >> 5;   // eight bits from bit rel of (ones below bit 0 | mask | zeros)
                const u32x4 am = anc[qb];
                auto word = [&](int i) { return i < 0 ? ~0u : (i == 0 ? am[0] : (i == 1 ? am[1] : (i == 2 ? am[2] : (i == 3 ? am[3] : 0u)))); };
                vis = __builtin_amdgcn_alignbit(word(w + 1), word(w), rel & 31);
            }
            float sc[8];
            float bmax = -1e30f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                sc[i] = MODE == 0 || ((vis >> i) & 1u) ? st[qb][i >> 2][i & 3] * scale : -1e30f;
                bmax = fmaxf(bmax, sc[i]);
            }
            bmax = fmaxf(bmax, __shfl_xor(bmax, 16));
            bmax = fmaxf(bmax, __shfl_xor(bmax, 32));
            // The running maximum may lag behind the true one by up to 8 (base 2): the
            // probabilities then reach 2^8 at most, and the accumulated output is rescaled only
            // when some lane of the wave needs it (wave-uniform branch; rare after the first
            // block), which saves the pass over the accumulators in the common case.
            if (__builtin_amdgcn_ballot_w64(bmax > mrun[qb] + 8.f) != 0) {
                const float mnew = fmaxf(mrun[qb], bmax);
                const float alpha = __builtin_amdgcn_exp2f(mrun[qb] - mnew);
                mrun[qb] = mnew;
                lrun[qb] *= alpha;
                if (!fresh) {
#pragma unroll
                    for (int db = 0; db < DB; ++db) o[qb][db] *= alpha;
                }
            }
            const float mref = mrun[qb];
            float p[8];
            float psum = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float e = __builtin_amdgcn_exp2f(sc[i] - mref);
                p[i] = MODE == 0 || ((vis >> i) & 1u) ? e : 0.f;
                psum += p[i];
            }
            lrun[qb] += psum;
            // probabilities as high + low bf16 parts: the second product sees them to ~16 bits
            u32x4 pv, pvl;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t hi, lo;
                split_bf2(p[2 * e], p[2 * e + 1], hi, lo);
                pv[e] = hi;
                pvl[e] = lo;
            }
            const bf16x8 pf = as_bf16x8(pv), pfl = as_bf16x8(pvl);
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                o[qb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[db], pf, o[qb][db], 0, 0, 0);
                o[qb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[db], pfl, o[qb][db], 0, 0, 0);
                if constexpr (LO)
                    o[qb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vl[db], pf, o[qb][db], 0, 0, 0);
            }
            if constexpr (MODE != 0) __builtin_amdgcn_sched_barrier(0);   // one group's masks at a time: registers
        }
        fresh = false;
    };

    // This wave's blocks come in three runs: the blocks with low parts, the blocks that hold tree
    // rows without low parts (rows an earlier call appended, or a caller's own rows), at most five
    // per head together, then the context-only blocks.  Those need no second set of registers for
    // the loads in flight: the next block's keys are requested as soon as this block's scores
    // have used up theirs, its values once the products have, and the other wave of the SIMD
    // works meanwhile.
    const bool have_lo = a.k_lo != nullptr && a.lo_end > a.lo_begin;
    const int lo_blk = have_lo ? min(blk_end, a.lo_begin / ATTN_KB) : blk_end;   // first block with low parts
    const int ctx_end = min(lo_blk, tree_blk);                                // blocks below hold context rows only
    const int my_begin = blk_begin + wave;
    // this wave's first block at or after `from`
    auto my_first = [&](int from) {
        return my_begin + (max(from - my_begin, 0) + blk_stride - 1) / blk_stride * blk_stride;
    };
    // the costlier blocks first: their loads go out with the kernel's first requests
    if (have_lo) {
        for (int blk = my_first(lo_blk); blk < blk_end; blk += blk_stride) {
            bf16x8 vl[DB];
            {
                bf16x8 kl[2][KS];
                load_k(kf, blk);
                request_k_lo(kl, blk);
                if constexpr (QB == 1) {   // registers for all of the block: one memory round trip instead of two
                    load_v(vf, blk);
                    request_v_lo(vl, blk);
                }
                keep_k_lo(kl, blk);
                scores(kf, kl, std::true_type{});
            }
            if constexpr (QB > 1) {
                load_v(vf, blk);
                request_v_lo(vl, blk);
            }
            keep_v_lo(vl, blk);
            mask_v(vf, blk);
            weigh(vf, vl, blk, std::integral_constant<int, 2>{});
        }
    }
    for (int blk = my_first(ctx_end); blk < lo_blk; blk += blk_stride) {
        load_k(kf, blk);
        load_v(vf, blk);
        scores(kf, kf, std::false_type{});
        mask_v(vf, blk);
        weigh(vf, vf, blk, std::integral_constant<int, 1>{});
    }
    if (my_begin < ctx_end) {
        int blk = my_begin;
        load_k(kf, blk);
        load_v(vf, blk);
        for (; blk + blk_stride < ctx_end; blk += blk_stride) {
            scores(kf, kf, std::false_type{});
            load_k(kf, blk + blk_stride);
            weigh(vf, vf, blk, std::integral_constant<int, 0>{});
            load_v(vf, blk + blk_stride);
        }
        scores(kf, kf, std::false_type{});
        weigh(vf, vf, blk, std::integral_constant<int, 0>{});
    }

    // every wave parks its running max, row sum and unnormalised output in LDS ...
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        float l = lrun[qb];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        const int ql = 16 * qb + m;
#pragma unroll
        for (int db = 0; db < DB; ++db)
            *reinterpret_cast<f32x4*>(&s_o[wave][ql][16 * db + 4 * q4]) = o[qb][db];
        if (q4 == 0) {
            s_ml[wave][ql][0] = mrun[qb];
            s_ml[wave][ql][1] = l;
        }
    }
    __syncthreads();
    // ... and the workgroup merges them (fixed wave order) into the chunk's result.
    // thread -> (query ql, dims 4 (i TPQ + c) .. + 3 for i < NI): the TPQ threads of a query cover
    // 4 TPQ consecutive dims per i, so every 16-byte access of a wave falls into whole 128-byte lines
    constexpr int TPQ = 64 * W / QN < D / 4 ? 64 * W / QN : D / 4;   // threads per query (any others are done)
    constexpr int NI = D / (4 * TPQ);
    static_assert(NI >= 1 && NI * 4 * TPQ == D, "merge mapping");
    const int ql = threadIdx.x / TPQ, c4 = 4 * (threadIdx.x % TPQ);
    const bool mine = ql < QN && qbase + ql < Tq;   // rows that hold no query are left out
    float M = -1e30f, l = 0.f;
    f32x4 acc[NI];
    if (mine) {
#pragma unroll
        for (int w = 0; w < W; ++w) M = fmaxf(M, s_ml[w][ql][0]);
        float wgt[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            wgt[w] = __builtin_amdgcn_exp2f(s_ml[w][ql][0] - M);
            l += wgt[w] * s_ml[w][ql][1];
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < W; ++w) acc[i] += wgt[w] * *reinterpret_cast<const f32x4*>(&s_o[w][ql][4 * TPQ * i + c4]);
        }
    }

    // out[t][h*D + dims] = num / den as high (+ low) bf16 parts
    auto write_out = [&](const f32x4 (&num)[NI], float den) {
        const float inv = 1.0f / den;
        const size_t o_off = static_cast<size_t>(qbase + ql) * a.H + h * D + c4;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            uint2 hi, lo;
            split_bf2(num[i][0] * inv, num[i][1] * inv, hi.x, lo.x);
            split_bf2(num[i][2] * inv, num[i][3] * inv, hi.y, lo.y);
            *reinterpret_cast<uint2*>(a.out + o_off + 4 * TPQ * i) = hi;
            if (a.out_lo) *reinterpret_cast<uint2*>(a.out_lo + o_off + 4 * TPQ * i) = lo;
        }
    };
    if (a.n_chunks == 1) {
        if (mine) write_out(acc, l);
        return;
    }

    // Publish this chunk.  The values move with device-coherent stores and loads (sc1: they
    // bypass the per-XCD caches) in whole 128-byte lines; waiting for the stores' acknowledgement
    // before the arrival count is raised orders them without a cache write-back / invalidate.
    if (mine) {
        const size_t slot = (static_cast<size_t>(h) * a.n_chunks + chunk) * a.t_pad + qbase + ql;
        float* po = a.po + slot * D + c4;
#pragma unroll
        for (int i = 0; i < NI; ++i) store_coherent16(po + 4 * TPQ * i, acc[i]);
        if (threadIdx.x % TPQ == 0) {
            __hip_atomic_store(a.pml + slot * 2, M, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(a.pml + slot * 2 + 1, l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();   // every thread's stores have been acknowledged
    int* counter = a.arrivals + h * gridDim.z + blockIdx.z;
    if (threadIdx.x == 0)
        s_last = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.n_chunks - 1;
    __syncthreads();
    if (!s_last) return;
    if (threadIdx.x == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
    if (!mine) return;
    // last workgroup of this (head, query group): out = sum_c exp2(m_c - M) O_c / sum_c exp2(m_c - M) l_c,
    // chunks in index order, eight chunks' loads in flight at a time (one memory round trip for
    // up to eight chunks), rescaled to the running maximum between groups.  (Sharing this among the chunks'
    // workgroups, each waiting for the others' arrivals, was slower: 16.7 against 12.6 us at 32 heads of 128, 32 nodes,
    // 1024 rows.)
    constexpr int MG = 8;
    const float* po_head = a.po + static_cast<size_t>(h) * a.n_chunks * a.t_pad * D;
    const uint32_t po_bytes = static_cast<uint32_t>(a.n_chunks * a.t_pad) * D * 4;
    float Mg = -1e30f;
    f32x4 num[NI];
    float den = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) num[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < a.n_chunks; c0 += MG) {
        f32x4 v[MG][NI];
        float mc[MG], lc[MG];
#pragma unroll
        for (int j = 0; j < MG; ++j) {
            const int c = min(c0 + j, a.n_chunks - 1);
            const size_t sl = (static_cast<size_t>(h) * a.n_chunks + c) * a.t_pad + qbase + ql;
            mc[j] = __hip_atomic_load(a.pml + sl * 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            lc[j] = __hip_atomic_load(a.pml + sl * 2 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t off = static_cast<uint32_t>(c * a.t_pad + qbase + ql) * D + c4;
#pragma unroll
            for (int i = 0; i < NI; ++i) v[j][i] = load_coherent16(po_head, po_bytes, 4 * (off + 4 * TPQ * i));
        }
        float Mn = Mg;
#pragma unroll
        for (int j = 0; j < MG; ++j) Mn = fmaxf(Mn, mc[j]);   // clamped repeats do not change the maximum
        const float resc = __builtin_amdgcn_exp2f(Mg - Mn);
        den *= resc;
#pragma unroll
        for (int i = 0; i < NI; ++i) num[i] *= resc;
        Mg = Mn;
#pragma unroll
        for (int j = 0; j < MG; ++j) {
            if (c0 + j < a.n_chunks) {
                const float wc = __builtin_amdgcn_exp2f(mc[j] - Mg);
                den += wc * lc[j];
#pragma unroll
                for (int i = 0; i < NI; ++i) num[i] += wc * v[j][i];
            }
        }
    }
    write_out(num, den);
}

// ---------------------------------------------------------------- single query
// One query node against rows [0, ctx_len) and its own path (see DecodeAttnArgs).  grid (chunks,
// heads), 256 threads; a workgroup takes its chunk in passes of DEC_TILE keys (normally one).
// Nothing here is a matrix product worth a matrix core: a pass is 64 KB of keys and values, and
// the launch is one memory round trip (partial sums, keys and values are all requested before the
// first of them is used), a few hundred fused multiply-adds per thread, and the store of the
// chunk's result (see DecodeAttnArgs: the following product merges the chunks).
//   scores: a key row is D/8 16-byte pieces, one per lane, summed over those lanes;
//   values: the cache is transposed, a dim's 128 keys are 16 16-byte pieces, one per lane.
// Rows that must stay invisible (later siblings, rows past the tree, the node's own row, which is
// being written meanwhile) are excluded by selects, never by a multiplication with zero, and so are rows whose weight has
// underflowed to zero, whatever their values hold; a tile of context rows with no zero weight goes without.
// What bounds it: an empty launch takes 2.2 us, the memory round trip 3 and a wave's instructions 2 ns each, 7 of 10 us
// with no key, value or partial sum loaded.  So: as few instructions as possible (no selects in full tiles, sums over 16
// lanes on the vector ALU instead of shuffles through LDS) and not more workgroups than compute units where avoidable (the
// node's own row is nobody's chunk: behind 1024 rows 32 heads have 256 workgroups, not 288).  32 heads of 128, launches in
// a layer, us: 1024 rows 9.9 -> 6.7, 1024 + 1 to 5 nodes 9.6 -> 7.5; the output projection behind it 9.8 -> 9.0 where it merges
// eight chunks instead of nine, 9.9 -> 9.4 with nine.
__device__ __forceinline__ bool mask_bit(const u32x4& m, int i) {
    const uint32_t w = i < 64 ? (i < 32 ? m[0] : m[1]) : (i < 96 ? m[2] : m[3]);
    return (w >> (i & 31)) & 1u;
}

template <int D>
__global__ __launch_bounds__(256) void cats_decode_attention(DecodeAttnArgs a) {
    constexpr int LPK = D / 8;           // lanes per key row
    constexpr int KPP = 256 / LPK;       // keys per score pass
    constexpr int KP = DEC_TILE / KPP;   // score passes per tile
    constexpr int VP = D / 16;           // value passes per tile (16 dims each)
    constexpr int HALF = D / 2;
    constexpr int PB = 8;                // partial sums requested at once per column
    __shared__ float s_q[D], s_kn[D], s_vn[D];
    __shared__ float s_sc[DEC_TILE];
    __shared__ __align__(16) float s_o[D];
    __shared__ float s_new;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int chunk = blockIdx.x, h = blockIdx.y;
    const int S = a.ctx_len, node = a.node;
    const int own = S + node;   // the node's own row: the last chunk's, beside its keys
    const bool owner = chunk == a.n_chunks - 1;
    const int key_begin = chunk * a.span, key_end = owner ? own : key_begin + a.span;
    const u32x4 anc = a.anc[node];
    bf16_t* kbase = a.kc + static_cast<size_t>(h) * a.max_ctx * D;
    bf16_t* vbase = a.vt + static_cast<size_t>(h) * D * a.max_ctx;
    const float scale = rsqrtf(static_cast<float>(D)) * 1.44269504088896340736f;   // 1/sqrt(d) * log2(e)
    auto visible = [&](int j) { return j < key_end && (j < S || mask_bit(anc, j - S)); };

    // requests: this wave's two columns of q, k or v (waves 0..2; k and v only where the node's
    // own row lives), then the first tile's keys and values
    const int role = wave;
    const bool builds = lane < HALF && (role == 0 || (owner && role <= 2));
    const int N = 3 * a.H;
    const int col = min(role, 2) * a.H + h * D + min(lane, HALF - 1);
    const int pieces = plan_pieces(a.plan, plan_col_tile(a.plan, col));   // both columns lie in the same tile
    float pa[PB], pb[PB];
    RowSquares sq;
    float2 cs = make_float2(1.f, 0.f);
    if (builds) {
        sq = row_squares_load(a.ns, 0);
        if (role < 2) cs = a.cs[lane];
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const float* p = a.part + static_cast<size_t>(min(i, pieces - 1)) * N + col;
            pa[i] = p[0];
            pb[i] = p[HALF];
        }
    }
    u32x4 kf[KP], vf[VP];
    auto load_tile = [&](int t0) {
#pragma unroll
        for (int p = 0; p < KP; ++p) {
            const int key = min(t0 + KPP * p + tid / LPK, a.max_ctx - 1);
            kf[p] = *reinterpret_cast<const u32x4*>(kbase + static_cast<size_t>(key) * D + 8 * (tid % LPK));
        }
#pragma unroll
        for (int p = 0; p < VP; ++p) {
            const int j0 = min(t0 + 8 * (tid % 16), a.max_ctx - 8);
            vf[p] = *reinterpret_cast<const u32x4*>(vbase + static_cast<size_t>(16 * p + tid / 16) * a.max_ctx + j0);
        }
    };
    load_tile(key_begin);

    // q (every workgroup), k and v of the node's own row (its owner): sum, scale, rotate
    if (builds) {
        float va = 0.f, vb = 0.f;
#pragma unroll
        for (int i = 0; i < PB; ++i)
            if (i < pieces) {
                va += pa[i];
                vb += pb[i];
            }
        for (int i = PB; i < pieces; ++i) {
            const float* p = a.part + static_cast<size_t>(i) * N + col;
            va += p[0];
            vb += p[HALF];
        }
        const float rs = row_scale(a.ns, sq);
        va *= rs;
        vb *= rs;
        const float r0 = role < 2 ? va * cs.x - vb * cs.y : va;
        const float r1 = role < 2 ? va * cs.y + vb * cs.x : vb;
        if (role == 0) {
            s_q[lane] = r0;
            s_q[lane + HALF] = r1;
        } else {
            const bf16_t h0 = f2bf(r0), h1 = f2bf(r1);
            float* dst = role == 1 ? s_kn : s_vn;
            dst[lane] = bf2f(h0) + bf2f(f2bf(r0 - bf2f(h0)));   // the row as later products of this call see it:
            dst[lane + HALF] = bf2f(h1) + bf2f(f2bf(r1 - bf2f(h1)));   // high + low part
            if (role == 1) {
                kbase[static_cast<size_t>(own) * D + lane] = h0;
                kbase[static_cast<size_t>(own) * D + lane + HALF] = h1;
            } else {
                vbase[static_cast<size_t>(lane) * a.max_ctx + own] = h0;
                vbase[static_cast<size_t>(lane + HALF) * a.max_ctx + own] = h1;
            }
        }
    }
    __syncthreads();
    float qs[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) qs[e] = s_q[8 * (tid % LPK) + e];
    if (wave == 3 && owner) {   // the node's own key
        float acc = 0.f;
        for (int d = lane; d < D; d += 64) acc += s_q[d] * s_kn[d];
        acc = wave_sum64(acc);
        if (lane == 0) s_new = acc * scale;
    }

    float m_run = -1e30f, l_run = 0.f, o_run[VP];
#pragma unroll
    for (int p = 0; p < VP; ++p) o_run[p] = 0.f;
    for (int t0 = key_begin;;) {
        const bool full = t0 + DEC_TILE <= min(key_end, S);   // context rows alone (the same for the whole workgroup)
        // scores of the tile's keys
        float sc[KP];
#pragma unroll
        for (int p = 0; p < KP; ++p) {
            float dot = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dot = fmaf(__uint_as_float(kf[p][e] << 16), qs[2 * e], dot);
                dot = fmaf(__uint_as_float(kf[p][e] & 0xFFFF0000u), qs[2 * e + 1], dot);
            }
            sc[p] = sum_lanes<LPK>(dot) * scale;
        }
        if (!full)
#pragma unroll
            for (int p = 0; p < KP; ++p)
                if (!visible(t0 + KPP * p + tid / LPK)) sc[p] = -INFINITY;
        if (tid % LPK == 0)
#pragma unroll
            for (int p = 0; p < KP; ++p) s_sc[KPP * p + tid / LPK] = sc[p];
        __syncthreads();
        const bool own_here = owner && t0 + DEC_TILE >= key_end;   // with the last tile
        // tile maximum (every wave works it out for itself), this thread's 8 keys' weights, tile sum
        float m_t = fmaxf(s_sc[lane], s_sc[lane + 64]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m_t = fmaxf(m_t, __shfl_xor(m_t, o));
        if (own_here) m_t = fmaxf(m_t, s_new);
        m_t = fmaxf(m_t, -1e30f);
        float pw[8], l_t = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            pw[e] = __builtin_amdgcn_exp2f(s_sc[8 * (tid % 16) + e] - m_t);
            l_t += pw[e];
        }
        l_t = sum_lanes<16>(l_t);
        const float p_new = own_here ? __builtin_amdgcn_exp2f(s_new - m_t) : 0.f;
        l_t += p_new;
        // weighted values: 16 dims per pass, a dim's keys over 16 lanes
        const float m_new = fmaxf(m_run, m_t);
        const float c_run = __builtin_amdgcn_exp2f(m_run - m_new), c_t = __builtin_amdgcn_exp2f(m_t - m_new);
        float acc[VP];
        // (every wave holds all of the tile's weights; a zero one, hidden or underflowed, must not meet an infinite value)
        float least = pw[0];
#pragma unroll
        for (int e = 1; e < 8; ++e) least = fminf(least, pw[e]);
        if (full && __builtin_amdgcn_ballot_w64(least == 0.f) == 0) {
#pragma unroll
            for (int p = 0; p < VP; ++p) {
                acc[p] = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[p] += pw[2 * e] * __uint_as_float(vf[p][e] << 16);
                    acc[p] += pw[2 * e + 1] * __uint_as_float(vf[p][e] & 0xFFFF0000u);
                }
            }
        } else {
#pragma unroll
            for (int p = 0; p < VP; ++p) {
                acc[p] = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float v0 = __uint_as_float(vf[p][e] << 16), v1 = __uint_as_float(vf[p][e] & 0xFFFF0000u);
                    acc[p] += pw[2 * e] != 0.f ? pw[2 * e] * v0 : 0.f;
                    acc[p] += pw[2 * e + 1] != 0.f ? pw[2 * e + 1] * v1 : 0.f;
                }
            }
        }
#pragma unroll
        for (int p = 0; p < VP; ++p) {
            acc[p] = sum_lanes<16>(acc[p]);
            if (own_here) acc[p] += p_new * s_vn[16 * p + tid / 16];
            o_run[p] = o_run[p] * c_run + acc[p] * c_t;
        }
        l_run = l_run * c_run + l_t * c_t;
        m_run = m_new;
        t0 += DEC_TILE;
        if (t0 >= key_end) break;
        __syncthreads();   // the scores are overwritten by the next tile
        load_tile(t0);
    }
    if (tid % 16 == 0) {
#pragma unroll
        for (int p = 0; p < VP; ++p) s_o[16 * p + tid / 16] = o_run[p];
    }
    __syncthreads();

    // The chunk's result: unnormalised sums, running maximum and row sum.  The output projection
    // merges a head's chunks while it builds its input columns, so nothing is handed over between
    // workgroups here and the launch ends with these stores.
    const size_t slot = static_cast<size_t>(h) * a.n_chunks + chunk;
    if (tid < D / 4)
        *reinterpret_cast<f32x4*>(a.po + slot * D + 4 * tid) = *reinterpret_cast<const f32x4*>(&s_o[4 * tid]);
    if (tid == 0) {
        a.pml[slot * 2] = m_run;
        a.pml[slot * 2 + 1] = l_run;
    }
}

__global__ void cats_zero_i32(int* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

}  // namespace

void launch_zero_i32(int* p, int n, hipStream_t st) {
    hipLaunchKernelGGL(cats_zero_i32, dim3((n + 255) / 256), dim3(256), 0, st, p, n);
}

void launch_decode_attention(const DecodeAttnArgs& a, hipStream_t st) {
    const dim3 grid(a.n_chunks, a.nh);
    if (a.d == 128)
        hipLaunchKernelGGL((cats_decode_attention<128>), grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((cats_decode_attention<64>), grid, dim3(256), 0, st, a);
}

void launch_attention(const AttnArgs& a, hipStream_t st) {
    const dim3 grid(a.n_chunks, a.nh, (a.Tq + a.queries - 1) / a.queries);
#define CATS_ATTN(DV, QBV, WV) hipLaunchKernelGGL((cats_tree_attention_kernel<DV, QBV, WV>), grid, dim3(64 * WV), 0, st, a)
    if (a.queries == 16) {
        if (a.d == 64)
            CATS_ATTN(64, 1, 8);
        else if (a.waves == 8)
            CATS_ATTN(128, 1, 8);
        else
            CATS_ATTN(128, 1, 4);
    } else {
        if (a.d == 64)
            CATS_ATTN(64, 2, 8);
        else if (a.waves == 8)
            CATS_ATTN(128, 2, 8);
        else
            CATS_ATTN(128, 2, 4);
    }
#undef CATS_ATTN
}
