// The prefill's own declarations: what its kernels and the entry point share.
#pragma once
#include "mla_internal.h"

namespace mla {

// Causal attention over materialised keys and values: a (sequence, head) pair, b * heads + h, has pages of its own and q_len
// query rows.
struct PrefillParams {
    const void* q_nope;         // [B, q_len, heads, 128] bf16
    const void* q_rope;         // [B, q_len, heads, 64]
    const void* pool;           // [pairs, max_pages] pages of 64 keys and values
    const int32_t* lens;        // [pairs]
    const void* rope;           // the keys' rope parts: of row 0 of page 0, and bytes from row to row (pages of 64 rows lie one
    int rope_pitch;             // behind the other).  16-byte aligned, both
    const int32_t* page_table;  // [B, max_pages]: their pages; an id outside [0, num_pages) leaves its 64 keys out
    int num_pages, max_pages;
    int pairs, q_len, heads;
    void* out;                  // [B, q_len, heads, 128] bf16
    float* lse;                 // [B, q_len, heads], or nullptr
    float scale;
};

bool       prefill_supported(int d_head, int d_c, int d_rope, int page_size, mla_dtype io, mla_dtype cache);
// materialise [W_UK c | W_UV c] per pair into pool2, and the pairs' lengths
hipError_t launch_prefill_materialise(const void* kv, const int32_t* page_table, const int32_t* seq_lens,
                                      const void* W_UK, const void* W_UV, void* Wcat, void* pool2, int32_t* lens2,
                                      int B, int q_len, int heads, int d_c, int num_pages, int max_pages,
                                      hipStream_t s);
// the rope parts of a cache that is not on 16 bytes: copied to dst, page by page of the sequences, [B * max_pages, 64, 64], and their
// ids there, [B, max_pages] (-1: not in the cache)
hipError_t launch_prefill_rope(const void* kv, const int32_t* page_table, const int32_t* seq_lens, void* dst, int32_t* ids,
                               int B, int d_c, int num_pages, int max_pages, hipStream_t s);
hipError_t launch_prefill_attention(const PrefillParams& p, hipStream_t s);

}  // namespace mla
