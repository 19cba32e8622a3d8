// How an attention launch is cut into workgroups.  Plain C++: the host decides, and a CPU test calls the rules.
#pragma once
#include <algorithm>

constexpr int ATTN_KB = 32;   // keys per block

struct AttnSplit {
    int queries;   // of a workgroup: 16 or 32
    int chunks;    // key chunks per (head, query group)
    int waves;     // of a workgroup: 4 or 8
};

// Key chunks per (head, query group): the launch has heads * query groups * chunks workgroups,
// about one per compute unit; more chunks than that only add hand-over traffic between workgroups.
inline int attn_chunks(int rows, int n_heads, int max_chunks, int n_cus, int n_keys, int queries) {
    const int n_blocks = (n_keys + ATTN_KB - 1) / ATTN_KB;
    const int groups = (rows + queries - 1) / queries;
    const int chunks = std::max(1, n_cus / std::max(1, n_heads * groups));
    return std::min(chunks, std::min(n_blocks, max_chunks));
}
// Waves per workgroup.  Head size 64: eight (no spill, half the LDS), 2.5 to 4 % faster than four.  Head size 128: four,
// which need no spill; eight where a head has more than eight chunks, which its last workgroup then merges in more than one
// round (twice the threads halve that).  Eight -> four, us.  Up to eight chunks, alone: 32 queries, 8 heads, 97 nodes / 3500
// rows 16.7 -> 15.9; 16 queries, 32 heads, 16 / 512 7.8 -> 7.5, 64 / 1000 14.4 -> 13.8.  Beyond eight, 16 queries, whole
// attention blocks (low parts of the own rows included): 8 heads, 16 / 2000 (16 chunks) 22.9 -> 23.6, 16 / 4096 (16) 26.5 -> 27.8;
// alone the two are within 5 % either way (8 heads, 16 / 1500 9.0 -> 8.8, 16 / 4096 13.2 -> 13.8).  32 queries have more than
// eight chunks with few heads, many nodes and long contexts only; there four would be ahead with 8 heads (80 / 3500, ten chunks,
// alone 15.6 -> 14.9) and behind with 4 (80 / 3500, 21 chunks, 15.3 -> 15.9).
inline int attn_waves(int head_dim, int chunks) { return head_dim == 64 || chunks > 8 ? 8 : 4; }
// Queries of a workgroup.  With 16 a wave has half the arithmetic and half the partial results to hand over, and registers
// to request all of a block with low parts at once; beyond 16 rows every 16 of them then read all keys and values, which is
// the shorter way while a chunk has few key blocks (fewer where one chunk needs no hand-over with 16 but has all the keys).
// In a layer, 32 then 16 queries, us (32 heads of 128; in brackets blocks a chunk, chunks): 20 nodes / 300 rows 11.7 -> 7.9,
// 32 / 1024 (8, 4) 12.8 -> 10.5, 32 / 2000 (16, 4) 15.3 -> 14.0, 63 / 512 (9, 2) 12.6 -> 10.5, 33 / 1000 (17, 2) 13.5 -> 13.5,
// 64 / 2048 (33, 2) 17.5 -> 21.9, 128 / 300 (14, 1) 16.1 -> 13.5, 128 / 512 (20, 1) 16.0 -> 16.0.  Attention alone: 40 heads,
// 30 / 1500 (16, 3) 13.7 -> 14.6; 8 heads, 64 / 4096 (16, 8) 16.3 -> 14.0; 128 / 1024 (36, 1) 17.1 -> 20.1.
// Not where 16-query workgroups outnumber the compute units: some of those then take two in turn, and 32 queries fit.
// Alone, 32 then 16 queries, us: 40 heads of 128, 112 nodes / 8 rows 6.6 -> 8.8, 128 / 128 8.6 -> 11.8, 128 / 300 11.7 -> 17.2;
// 64 heads of 64, 80 / 128 6.0 -> 7.6, 96 / 300 7.4 -> 10.9; 128 heads of 64, 65 / 40 (neither fits) 8.4 -> 8.3.
// Chunks hold about four key blocks or more: the number of chunks is the blocks over four, rounded up, and the kernel deals
// them out by cost (a block with tree rows counts twice), so that 17 blocks are chunks of 4, 4, 3, 4 and 2.  Shorter ones leave
// more waves without a block and add partial results to hand over.  (Eight waves have a block each from eight blocks a chunk
// on; head size 64 stays with one chunk that far.)  In a layer, chunks down to one block -> this, us:
// 32 heads of 128, 2 nodes / 100 rows 6.6 -> 5.4, 16 / 40 7.1 -> 4.7, 16 / 512 8.6 -> 8.0; 4 heads of 64, 15 / 128 6.4 -> 4.7,
// 16 / 2000 9.6 -> 7.2, 30 / 300 7.2 -> 6.8; 32 of 128, 63 / 200 and 128 / 512 as before.
inline AttnSplit attn_split(int n_heads, int head_dim, int rows, int n_keys, int n_cus, int max_chunks) {
    const int n_blocks = (n_keys + ATTN_KB - 1) / ATTN_KB;
    max_chunks = std::min(max_chunks, head_dim == 64 && n_blocks <= 8 ? 1 : (n_blocks + 3) / 4);
    const int narrow = attn_chunks(rows, n_heads, max_chunks, n_cus, n_keys, 16);
    const bool fits = static_cast<long>(n_heads) * ((rows + 15) / 16) <= n_cus;
    const int queries = rows <= 16 || (fits && n_blocks <= (narrow == 1 ? 14 : 18 * narrow - 8)) ? 16 : 32;
    const int chunks = queries == 16 ? narrow : attn_chunks(rows, n_heads, max_chunks, n_cus, n_keys, 32);
    return {queries, chunks, attn_waves(head_dim, chunks)};
}

constexpr int DEC_TILE = 128;       // keys per pass of a workgroup
constexpr int DEC_MAX_CHUNKS = 32;  // key chunks per head at most (the context's scratch holds that many)

struct RowSplit {
    int chunks;   // per head
    int span;     // keys per chunk; the last one holds what is left
};

// Chunks of a single query: one pass each up to 4096 keys, beyond that as few blocks more as 32 chunks need.  A short last
// chunk stays a workgroup of its own also where the chip is full: handed to the chunk before it, it is that workgroup's second
// pass (its loads, scores and sums once more, one after the other), which takes longer than the workgroups saved.  In layers of
// one row (attention and its products), merged -> this, us: 32 heads of 128, 1025 to 1056 rows 38.5 -> 37.7, 1281 to 1312
// 39.3 -> 38.0; 40 heads, 2049 rows 55.0 -> 52.6; 64 heads of 64, 650 rows 36.3 -> 35.2.
inline RowSplit row_split(int n_keys) {
    const int n_blocks = std::max(1, (n_keys + ATTN_KB - 1) / ATTN_KB);
    const int per_chunk = std::max(DEC_TILE / ATTN_KB, (n_blocks + DEC_MAX_CHUNKS - 1) / DEC_MAX_CHUNKS);
    return {(n_blocks + per_chunk - 1) / per_chunk, per_chunk * ATTN_KB};
}
