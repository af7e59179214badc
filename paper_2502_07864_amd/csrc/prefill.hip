// Prefill in the "MHA paradigm" (Sec. 3.3, first of the two attention equations): keys and values
// are materialised per head from the cached latent rows,
//     k_{j,h} = [W^{UK}_h c_j ; k^R_j],        v_{j,h} = W^{UV}_h c_j,
// and the prompt's tokens attend causally to them.  This file holds the kernels that build the materialised keys and
// values (one with a head's weights in LDS, one that streams them, and the one that lays them out for it); the attention
// itself runs on prefill_attention.hip's kernel, for which one (sequence, head) pair is a sequence of its own, and whose page
// layout (64 keys of 128 values, then the values transposed, both in the order its reads want) is described there.  The rope part of
// the keys, the same for every head, stays in the cache.
//
//   Y^T [256 x tokens] = [W^{UK}_h ; (W^{UV}_h)^T] [256 x d_c] . C^T [d_c x tokens]
//
// on v_mfma_f32_16x16x32_bf16.  A workgroup keeps the weights of one head (d_c = 512: its keys' or its values' half) in LDS for as
// long as it lives; its 16 (8) wavefronts take the head's half pages of all sequences in turn, each on its own: latent
// rows into registers as one operand, 128-bit LDS reads of the weights as the other, results rounded to bf16 and stored 16
// bytes per lane (the page layout leaves a lane eight neighbouring values of a key, or of a value dimension: the
// latter a contiguous kilobyte per wavefront).  No barrier and no weight traffic after the start.
#include "prefill_internal.h"
#include "mfma_tile.h"
#include <algorithm>
#include <type_traits>

namespace mla {
namespace {

typedef __attribute__((ext_vector_type(8))) short s16x8;

constexpr int PF_DH = 128;      // head dimension
constexpr int PF_PAGE = 64 * 2 * PF_DH;           // values per materialised page: 64 keys, then the values transposed

// Weights in LDS: row r (a dimension of the keys or of the values) of d_c values, its 16-byte piece c at position c ^ (r & 15):
// the 16 lanes that share a cycle of an operand read meet 16 different units.  The values' weights are stored k-major by the caller
// and are transposed once, at the start, by the transposing LDS read.
// Bound by the matrix pipe and the LDS reads that feed it (1 KB for two instructions of a wavefront), by the latent rows and by
// writing 512 bytes per (token, head): 26800 tokens, 28 heads, d_c = 256, mean of 100 traced launches, 152 us with 640 (the rope part copied), now 121 to
// 128 by card; weights streamed through the LDS by every workgroup, laid out by a launch of its own, took 172 + 9.  Two pages, 28 heads, d_c = 512: 11.3 (15 + 8).
// Whole pages per wavefront (eight of them): 149; a wavefront's rows requested a unit ahead: 160 to 200 (registers).
template <int D_C> constexpr int PM_WAVES = 4096 / D_C;            // wavefronts of a workgroup: 16 / 8

template <int D_C>
__global__ __launch_bounds__(PM_WAVES<D_C> * 64, PM_WAVES<D_C> / 4) void prefill_materialise_kernel(const uint16_t* kv, const int32_t* page_table,
                                                                               const int32_t* seq_lens, const uint16_t* W_UK, const uint16_t* W_UV,
                                                                               uint16_t* pool2, int32_t* lens2,
                                                                               int B, int heads, int num_pages, int max_pages, bool by_page)
{
    constexpr int ROW = D_C + 64;
    constexpr int NKS = D_C / 32;
    constexpr int WROWB = D_C * 2;                    // bytes per weight row
    constexpr int PARTS = D_C / 256;                  // kinds of workgroups: keys and values, or one of them
    constexpr int NT = 2;                             // 16-token tiles of a wavefront: half a page
    constexpr int WAVES = PM_WAVES<D_C>;
    constexpr int HALF_B = PF_DH * WROWB;             // the weights of the keys, or of the values
    constexpr int THREADS = WAVES * 64;
    constexpr int NLD = HALF_B / 16 / THREADS;        // 16-byte pieces per thread of either (4 / 16)
    constexpr int AH = D_C == 256 ? 2 : 4;            // k-steps that the LDS reads run ahead (as the registers allow)
    __shared__ __attribute__((aligned(1024))) unsigned char wbuf[2 / PARTS * HALF_B];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int kind = by_page ? blockIdx.y : blockIdx.x, share = by_page ? blockIdx.x : blockIdx.y, shares = by_page ? gridDim.x : gridDim.y;
    const int h = kind / PARTS, part = kind % PARTS;
    const bool keys = PARTS == 1 || part == 0, values = PARTS == 1 || part == 1;
    LDS_AS unsigned char* w_keys = (LDS_AS unsigned char*)wbuf;
    LDS_AS unsigned char* w_values = w_keys + (2 / PARTS - 1) * HALF_B;

    // Sequences in groups of 64, one per lane: its length, and the half pages of the group up to its end.  (One after the other
    // by scalar loads: 256 sequences of a page, one head, 50 us for the whole call, now 20.)  The first group's lengths are asked for
    // before the weights and added up while these are on their way.
    int len, upto;
    auto length_of = [&](int b) { return b < B ? seq_lens[b] : 0; };
    auto add_up = [&](int length) {
        len = max(0, min(length, max_pages * 64));
        upto = ((len + 63) >> 6) * 2;
        // running sum over the lanes: within rows of 16, then each row's total to the rows behind it
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x111, 0xf, 0xf, false);       // row_shr 1, 2, 4, 8
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x112, 0xf, 0xf, false);
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x114, 0xf, 0xf, false);
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x118, 0xf, 0xf, false);
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x142, 0xa, 0xf, false);       // row_bcast 15: rows 1 and 3
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x143, 0xc, 0xf, false);       // row_bcast 31: rows 2 and 3
    };
    const int first_length = length_of(lane);
    __builtin_amdgcn_sched_barrier(0);
    int group = 0, before = 0;                        // the group's first sequence, half pages before it

    // ---- the weights: all requested at once
    {
        u32x4 wk[NLD], wv[NLD];
        if (keys) {
#pragma unroll
            for (int i = 0; i < NLD; ++i)
                wk[i] = *reinterpret_cast<const u32x4*>(W_UK + (size_t)h * PF_DH * D_C + (i * THREADS + tid) * 8);
        }
        if (values) {
#pragma unroll
            for (int i = 0; i < NLD; ++i)
                wv[i] = *reinterpret_cast<const u32x4*>(W_UV + (size_t)h * PF_DH * D_C + (i * THREADS + tid) * 8);
        }
        __builtin_amdgcn_sched_barrier(0);
        add_up(first_length);
        if (share == 0 && keys)
            for (int b = tid; b < B; b += THREADS) lens2[(size_t)b * heads + h] = max(0, min(seq_lens[b], max_pages * 64));
        if (keys) {
#pragma unroll
            for (int i = 0; i < NLD; ++i) {           // W_UK[h] is [d_head x d_c]
                const int q = i * THREADS + tid, row = q / (D_C / 8), c = q % (D_C / 8);
                *(LDS_AS u32x4*)(w_keys + row * WROWB + ((c ^ (row & 15)) << 4)) = wk[i];
            }
        }
        if (values) {                                 // W_UV[h] is [d_c x d_head]: as it lies ...
#pragma unroll
            for (int i = 0; i < NLD; ++i) *(LDS_AS u32x4*)(w_values + (i * THREADS + tid) * 16) = wv[i];
        }
        __syncthreads();
        if (values) {                                 // ... then the wavefront's (16 dimensions x 32 k) tiles transposed
            constexpr int SHARE = PF_DH / 16 * NKS / WAVES;                    // (4 / 16)
            s16x8 t[SHARE];
#pragma unroll
            for (int i = 0; i < SHARE; ++i) {
                // the lane supplies row 32 ks + 8g + (n >> 2) (and 4 more), 8 bytes at column 16 dt + 4 (n & 3)
                const int dt = (wave * SHARE + i) / NKS, ks = (wave * SHARE + i) % NKS;
                LDS_AS unsigned char* at = w_values + (ks * 32 + g * 8 + (n >> 2)) * (PF_DH * 2) + dt * 32 + (n & 3) * 8;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)at);
                const s16x4 up = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(at + 4 * PF_DH * 2));
                t[i] = __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7);
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < SHARE; ++i) {
                const int row = (wave * SHARE + i) / NKS * 16 + n, ks = (wave * SHARE + i) % NKS;
                *(LDS_AS s16x8*)(w_values + row * WROWB + (((4 * ks + g) ^ (row & 15)) << 4)) = t[i];
            }
        }
        __syncthreads();
    }

    // A operand: weight row 16 rt + n, piece 4 ks + g
    uint32_t a_base[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) a_base[e] = (uint32_t)(n * WROWB + (((4 * e + g) ^ n) << 4));

    // ---- this wavefront's share of the half pages of all sequences laid end to end: pages are dealt to the workgroups of the
    // head first, so that few of them keep as many CUs busy as there are
    const int stride = shares * WAVES;
    for (int u = 2 * (share + shares * (wave >> 1)) + (wave & 1);; u += stride) {
        for (int all; u >= before + (all = __builtin_amdgcn_readlane(upto, 63)); add_up(length_of(group + lane))) {
            before += all;
            group += 64;
            if (group >= B) return;
        }
        const int i = __popcll(__ballot(before + upto <= u));          // the group's sequences that end before u
        const int b = group + i, L = __builtin_amdgcn_readlane(len, i);
        const int left = before + __builtin_amdgcn_readlane(upto, i) - u;                  // half pages from u to the end of sequence b
        const int pg = (((L + 63) >> 6) * 2 - left) >> 1, tok0 = (left & 1) * 32;         // page, and this wavefront's first token inside it
        const int page = ((const CONST_AS int32_t*)(page_table + (size_t)b * max_pages))[pg];
        const bool active = page >= 0 && page < num_pages;
        // the pseudo-sequence (b, h) owns pages [bh * max_pages, +max_pages) of the materialised pool; the page of an id
        // outside the cache pool, like the tokens past the sequence's end, gets zeros for values: what the weights of tokens
        // that the attention skips (zeros) are multiplied with
        const size_t page2 = ((size_t)b * heads + h) * max_pages + pg;
        const uint16_t* src = kv + (size_t)(active ? page : 0) * 64 * ROW;
        uint16_t* dst = pool2 + page2 * PF_PAGE;

        // latent rows of tokens tok0 + 16 nt + n, k = 32 ks + 8g .. + 7
        bf16x8 cb[NT][NKS];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
                cb[nt][ks] = *reinterpret_cast<const bf16x8*>(src + (tok0 + nt * 16 + n) * ROW + ks * 32 + g * 8);
        if (!active || pg * 64 + tok0 + NT * 16 > L) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const bool there = active && pg * 64 + tok0 + nt * 16 + n < L;
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks)
                    if (!there) cb[nt][ks] = __builtin_bit_cast(bf16x8, (u32x4){0u, 0u, 0u, 0u});
            }
        }

        // 32 dimensions (two row tiles of the weights) x the wavefront's tokens.  Keys: weights as the A operand (a lane ends with four
        // dimensions of a token); values: tokens as the A operand (four tokens of a dimension)
        f32x4 acc[2][NT];
        auto product = [&](auto of_keys, LDS_AS unsigned char* rows) {
            bf16x8 a[2][NKS];
            auto rd = [&](int ks) {
#pragma unroll
                for (int ml = 0; ml < 2; ++ml)
                    a[ml][ks] = *(LDS_AS bf16x8*)(rows + ml * 16 * WROWB + a_base[ks & 3] + (ks >> 2) * 256);
            };
#pragma unroll
            for (int ks = 0; ks < AH; ++ks) rd(ks);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                if (ks + AH < NKS) rd(ks + AH);
#pragma unroll
                for (int ml = 0; ml < 2; ++ml)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        const f32x4 c = ks ? acc[ml][nt] : (f32x4){0.f, 0.f, 0.f, 0.f};
                        acc[ml][nt] = decltype(of_keys)::value ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ml][ks], cb[nt][ks], c, 0, 0, 0)
                                                               : __builtin_amdgcn_mfma_f32_16x16x32_bf16(cb[nt][ks], a[ml][ks], c, 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto pack8 = [&](const f32x4& lo, const f32x4& up) {
            return (u32x4){pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]), pack_bf16x2(up[0], up[1]), pack_bf16x2(up[2], up[3])};
        };
        if (keys) {
            for (int c = 0; c < PF_DH / 32; ++c) {
                product(std::true_type{}, w_keys + c * 32 * WROWB);
                // 32 dimensions of the tokens: position 8g + 4 ml + i of the 32 is dimension 16 ml + 4g + i
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    *reinterpret_cast<u32x4*>(dst + (tok0 + nt * 16 + n) * PF_DH + c * 32 + g * 8) = pack8(acc[0][nt], acc[1][nt]);
            }
        }
        if (values) {
            for (int c = 0; c < PF_DH / 32; ++c) {
                product(std::false_type{}, w_values + c * 32 * WROWB);
                // half pages of 32 tokens, 32 dimensions: key 4 nt + i of group g is token 16 nt + 4g + i
#pragma unroll
                for (int ml = 0; ml < 2; ++ml)
#pragma unroll
                    for (int nt = 0; nt < NT; nt += 2)
                        *reinterpret_cast<u32x4*>(dst + 64 * PF_DH + (tok0 + nt * 16) * PF_DH + (c * 2 + ml) * 512 + lane * 8) =
                            pack8(acc[ml][nt], acc[ml][nt + 1]);
            }
        }
    }
}

// Wcat[h] = [W^{UK}_h ; (W^{UV}_h)^T] as 256 rows of d_c values each, for the kernel below.
// grid (d_c / 64, 4, heads): a block of 64 rows x 64 columns of Wcat[h]; rows 0 .. 127 are a copy, the others
// go through LDS (the value projection's rows are columns here: read and written 128 bytes at a time)
__global__ __launch_bounds__(256) void prefill_weights_kernel(const uint16_t* W_UK, const uint16_t* W_UV,
                                                              uint16_t* Wcat, int d_c)
{
    __shared__ uint16_t block[64][66];
    const int c0 = blockIdx.x * 64, r0 = blockIdx.y * 64, h = blockIdx.z;
    const int x = threadIdx.x & 63, y = threadIdx.x >> 6;
    uint16_t* dst = Wcat + ((size_t)h * 256 + r0) * d_c + c0;
    if (r0 < PF_DH) {
        const uint16_t* src = W_UK + ((size_t)h * PF_DH + r0) * d_c + c0;                 // W_UK[h] is [d_head x d_c]
        for (int i = y; i < 64; i += 4) dst[(size_t)i * d_c + x] = src[(size_t)i * d_c + x];
        return;
    }
    const uint16_t* src = W_UV + ((size_t)h * d_c + c0) * PF_DH + (r0 - PF_DH);          // W_UV[h] is [d_c x d_head]
    for (int i = y; i < 64; i += 4) block[i][x] = src[(size_t)i * PF_DH + x];
    __syncthreads();
    for (int i = y; i < 64; i += 4) dst[(size_t)i * d_c + x] = block[x][i];
}

// ---- many pages.  One workgroup = two pages (128 tokens) of one (sequence, head).  Wcat[h] is streamed through LDS
// in chunks of 32 rows (two row tiles, all d_c columns), double-buffered, as direct-to-LDS loads; the four
// wavefronts share every chunk.  Chunk position c ^ (row & 15) of a row holds its 16-byte piece c: the 16 lanes
// that share a cycle of an A read (rows 0 .. 7 of one piece and 8 .. 15 of its neighbour, or the reverse) then
// meet 16 different units (rows padded by 16 bytes, filled through registers, lost 3.2 of 8 cycles per read).
// A wavefront owns 32 tokens (two column tiles) and keeps their latent rows in registers.
// The first weights are asked for before anything else, page and length by scalar loads: 4 x 8192 tokens, 32 heads, d_c = 512
// 348 -> 333 us (and 11 for the weights' layout); the figures against the kernel above stand at the rule below.
template <int D_C>
__global__ __launch_bounds__(256, 2) void prefill_stream_kernel(const uint16_t* kv, const int32_t* page_table,
                                                                     const int32_t* seq_lens, const uint16_t* Wcat,
                                                                     uint16_t* pool2, int32_t* lens2,
                                                                     int heads, int num_pages, int max_pages)
{
    constexpr int ROW = D_C + 64;
    constexpr int NKS = D_C / 32;
    constexpr int WROWB = D_C * 2;                    // bytes per weight row
    constexpr int CHUNK_ROWS = 32;
    constexpr int CHUNK_B = CHUNK_ROWS * WROWB;
    constexpr int NCHUNK = 256 / CHUNK_ROWS;          // 8
    constexpr int NPL = CHUNK_B / 16 / 256;           // 16-byte pieces per thread and chunk (8 / 4)
    constexpr int AH = 4;                             // k-steps that the LDS reads run ahead
    __shared__ __attribute__((aligned(1024))) unsigned char wbuf[2 * CHUNK_B];
    LDS_AS unsigned char* lds = (LDS_AS unsigned char*)wbuf;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int bh = blockIdx.y;
    const int b = bh / heads, h = bh % heads;
    const int L = max(0, min(((const CONST_AS int32_t*)seq_lens)[b], max_pages * 64));
    // the sequence's first pages are dealt to another XCD than the one before's: tables wider than the contexts, of 16 pages for
    // instance, gave all the work to one of the eight (256 sequences of a page, 28 heads, d_c = 512, 16 pages wide: 1770 us, now 409)
    const int px = (blockIdx.x + b) % gridDim.x;
    if (px == 0 && tid == 0) lens2[bh] = L;
    if (px * 128 >= L) return;

    // this wavefront's page (waves 0, 1: the first of the pair; 2, 3: the second)
    const int pg = px * 2 + (wave >> 1);
    const bool in_seq = pg < max_pages && pg * 64 < L;
    const int page = in_seq ? ((const CONST_AS int32_t*)(page_table + (size_t)b * max_pages))[pg] : -1;
    const bool active = in_seq && page >= 0 && page < num_pages;
    // the pseudo-sequence (b, h) owns pages [bh * max_pages, +max_pages) of the materialised pool; the page of an id
    // outside the cache pool, like the tokens past the sequence's end, gets zeros for values: what the weights of tokens
    // that the attention skips (zeros) are multiplied with
    const size_t page2 = (size_t)bh * max_pages + pg;
    const uint16_t* src = kv + (size_t)(active ? page : 0) * 64 * ROW;
    uint16_t* dst = pool2 + (in_seq ? page2 : 0) * PF_PAGE;
    const int tok0 = (wave & 1) * 32;                 // this wavefront's first token inside its page

    const unsigned char* W = reinterpret_cast<const unsigned char*>(Wcat + (size_t)h * 256 * D_C);
    constexpr int RPL = 4096 / WROWB;                 // rows that one load of the workgroup covers (4 / 8)
    uint32_t woff[16 / RPL];                          // (the swizzle repeats after 16 rows)
#pragma unroll
    for (int i = 0; i < 16 / RPL; ++i) {
        const int q = i * 256 + tid, row = q / (D_C / 8), pos = q % (D_C / 8);
        woff[i] = (uint32_t)(row * WROWB + ((pos ^ (row & 15)) << 4));
    }
    const uint32_t lds_base = (uint32_t)(uintptr_t)lds;
    auto load_chunk = [&](int c) {
        const uint32_t dst = lds_base + (uint32_t)((c & 1) * CHUNK_B + wave * 1024);
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            const unsigned char* src = W + (size_t)c * CHUNK_B + (i / (16 / RPL)) * (16 * WROWB);
            const uint32_t m0v = __builtin_amdgcn_readfirstlane(dst + i * 4096);
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :: "s"(m0v), "v"(woff[i % (16 / RPL)]), "s"(src) : "memory");
        }
    };
    // A operand: weight row 16 ml + n, piece 4 ks + g
    uint32_t a_base[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) a_base[e] = (uint32_t)(n * WROWB + (((4 * e + g) ^ n) << 4));
    // Everything a workgroup reads before its first product is requested at once: a chunk of weights and the latent rows.
    load_chunk(0);
    bf16x8 cb[2][NKS];
    if (in_seq) {
        // B operands: latent rows of tokens tok0 + 16 nt + n, k = 32 ks + 8g .. + 7
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
                cb[nt][ks] = *reinterpret_cast<const bf16x8*>(src + (tok0 + nt * 16 + n) * ROW + ks * 32 + g * 8);
        if (!active || pg * 64 + tok0 + 32 > L) {
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const bool there = active && pg * 64 + tok0 + nt * 16 + n < L;
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks)
                    if (!there) cb[nt][ks] = __builtin_bit_cast(bf16x8, (u32x4){0u, 0u, 0u, 0u});
            }
        }
    }
    for (int c = 0; c < NCHUNK; ++c) {
        // my part of this chunk (requested a chunk ago) is there; the two results stored since may be on their way ...
        if (c > 0 && in_seq) wait_vmcnt<2>();
        else                 wait_vmcnt<0>();
        __syncthreads();                              // ... and everybody's, and everybody is done with the one before
        if (c + 1 < NCHUNK) load_chunk(c + 1);
        LDS_AS unsigned char* chunk = lds + (c & 1) * CHUNK_B;
        if (in_seq) {
            f32x4 acc[2][2];
#pragma unroll
            for (int ml = 0; ml < 2; ++ml)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) acc[ml][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
            // keys: weights as the A operand (a lane ends with four dimensions of a token); values: tokens as the
            // A operand (four tokens of a dimension)
            auto product = [&](auto keys) {
                bf16x8 a[2][NKS];
                auto rd = [&](int ks) {
#pragma unroll
                    for (int ml = 0; ml < 2; ++ml)
                        a[ml][ks] = *(LDS_AS bf16x8*)(chunk + ml * 16 * WROWB + a_base[ks & 3] + (ks >> 2) * 256);
                };
#pragma unroll
                for (int ks = 0; ks < AH; ++ks) rd(ks);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) {
                    if (ks + AH < NKS) rd(ks + AH);
#pragma unroll
                    for (int ml = 0; ml < 2; ++ml)
#pragma unroll
                        for (int nt = 0; nt < 2; ++nt)
                            acc[ml][nt] = decltype(keys)::value ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ml][ks], cb[nt][ks], acc[ml][nt], 0, 0, 0)
                                                                : __builtin_amdgcn_mfma_f32_16x16x32_bf16(cb[nt][ks], a[ml][ks], acc[ml][nt], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            auto pack8 = [&](const f32x4& lo, const f32x4& up) {
                return (u32x4){pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]), pack_bf16x2(up[0], up[1]), pack_bf16x2(up[2], up[3])};
            };
            if (c < NCHUNK / 2) {
                product(std::true_type{});
                // 32 dimensions of 32 tokens: position 8g + 4 ml + i of the 32 is dimension 16 ml + 4g + i
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    *reinterpret_cast<u32x4*>(dst + (tok0 + nt * 16 + n) * PF_DH + c * 32 + g * 8) = pack8(acc[0][nt], acc[1][nt]);
            } else {
                product(std::false_type{});
                // 32 tokens (this wavefront's half page) of 32 dimensions: key 4 nt + i of group g is token 16 nt + 4g + i
                uint16_t* half = dst + 64 * PF_DH + tok0 * PF_DH;
#pragma unroll
                for (int ml = 0; ml < 2; ++ml)
                    *reinterpret_cast<u32x4*>(half + ((c - NCHUNK / 2) * 2 + ml) * 512 + lane * 8) = pack8(acc[ml][0], acc[ml][1]);
            }
        }
    }
}

// a page of a sequence: 64 rows of 64 values
__global__ __launch_bounds__(256) void prefill_rope_kernel(const uint16_t* kv, const int32_t* page_table, const int32_t* seq_lens,
                                                           uint16_t* dst, int32_t* ids, int d_c, int num_pages, int max_pages)
{
    const int pg = blockIdx.x, b = blockIdx.y;
    const size_t at = (size_t)b * max_pages + pg;
    const int page = (long long)pg * 64 < seq_lens[b] ? page_table[at] : -1;
    const bool there = page >= 0 && page < num_pages;
    if (threadIdx.x == 0) ids[at] = there ? (int32_t)at : -1;
    if (!there) return;
    for (int i = threadIdx.x; i < 64 * 64; i += 256)
        dst[at * 64 * 64 + i] = kv[((size_t)page * 64 + (i >> 6)) * (d_c + 64) + d_c + (i & 63)];
}

}  // namespace

bool prefill_supported(int d_head, int d_c, int d_rope, int page_size, mla_dtype io, mla_dtype cache)
{
    return io == MLA_BF16 && cache == MLA_BF16 && d_head == PF_DH && d_rope == 64 && page_size == 64 &&
           (d_c == 256 || d_c == 512);
}

hipError_t launch_prefill_rope(const void* kv, const int32_t* page_table, const int32_t* seq_lens, void* dst, int32_t* ids,
                               int B, int d_c, int num_pages, int max_pages, hipStream_t s)
{
    prefill_rope_kernel<<<dim3(max_pages, B), 256, 0, s>>>(static_cast<const uint16_t*>(kv), page_table, seq_lens, static_cast<uint16_t*>(dst), ids,
                                                           d_c, num_pages, max_pages);
    return hipGetLastError();
}

hipError_t launch_prefill_materialise(const void* kv, const int32_t* page_table, const int32_t* seq_lens,
                                      const void* W_UK, const void* W_UV, void* Wcat, void* pool2, int32_t* lens2, int B, int q_len, int heads, int d_c, int num_pages, int max_pages,
                                      hipStream_t s)
{
    const uint16_t *rows = static_cast<const uint16_t*>(kv), *uk = static_cast<const uint16_t*>(W_UK), *uv = static_cast<const uint16_t*>(W_UV);
    uint16_t* pool = static_cast<uint16_t*>(pool2);
    // Weights in LDS (no launch of their own, no barriers) or streamed.  Whole calls, sustained, in LDS / streamed, us (pages x heads in
    // brackets; 28 heads unless said):
    // - few pages x heads, whose launches and weights count: d_c = 256, 1000 tokens (448) 45 / 51; 4 x 1000, 512 queries (1792)
    //   70 / 78; 4 x 1400, 512 (2464) 88 / 103; 8000, 512 (3500) 249 / 252; 2 x 4000, 512 (3528) 160 / 155.  d_c = 512, 1000 tokens
    //   51 / 56; 3 x 2087, 16 heads (1584) 102 / 108; 4096, 512 (1792) 153 / 150; 8 x 500, 64 (1792) 70 / 69; 4 x 1400, 512 122 / 130;
    //   4 x 2000, 512 (3584) 174 / 166.
    // - but the attention behind it is the slower for it the longer it takes itself (its reads of the pool meet other XCDs' writes;
    //   the first calls of a run are equal): d_c = 256, prompts of 2000 (896) 90 / 92, 3000 (1316) 156 / 154, 4000, 32 heads (2016)
    //   236 / 232, 5700 (2520) 402 / 366.
    // - d_c = 256, short query runs of enough (sequence, head) pairs for a workgroup of the attention on most CUs: 8 x 1000, 64
    //   queries 79 / 92, 512 136 / 143, 700 166 / 164; 8 x 2500, 64 215 / 225, 512 322 / 321; 8 x 6000, 512 722 / 756, 1024
    //   1072 / 1086, 2048 1694 / 1669; 16 x 2000, 512 490 / 505, 1024 710 / 703; 32 x 300, 128 109 / 126; 1000 x 64, 32 775 / 887.
    //   Fewer pairs: 7 x 4000, 64 295 / 304, 512 464 / 447; 4 x 5000, 64 248 / 241, 512 314 / 305; 2 x 16000, 64 574 / 590, 512
    //   618 / 597; 20000, 64 605 / 609, 512 628 / 606.  d_c = 512 reads every latent row twice: 8 x 2500, 64 288 / 282; 16 x 2000,
    //   512 612 / 605; 8 x 6000, 512 891 / 906.
    const long long pages = (long long)B * max_pages, work = pages * heads;
    const bool resident = (work <= 2560 && (d_c == 512 || q_len <= 3072)) || (d_c == 256 && q_len <= 512 && (long long)B * heads >= 224);
    if (!resident) {
        uint16_t* cat = static_cast<uint16_t*>(Wcat);
        prefill_weights_kernel<<<dim3(d_c / 64, 4, heads), 256, 0, s>>>(uk, uv, cat, d_c);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        const dim3 grid((max_pages + 1) / 2, B * heads);
        if (d_c == 512) prefill_stream_kernel<512><<<grid, 256, 0, s>>>(rows, page_table, seq_lens, cat, pool, lens2, heads, num_pages, max_pages);
        else            prefill_stream_kernel<256><<<grid, 256, 0, s>>>(rows, page_table, seq_lens, cat, pool, lens2, heads, num_pages, max_pages);
        return hipGetLastError();
    }
    // One workgroup per CU (its weights fill the LDS), the same number for every head: of one to eight rounds of them the number
    // that takes the least time, a round's weights counted as 0.3 of the page that a pair of wavefronts takes next (1000
    // tokens, 28 heads, d_c = 512: four per kind 51 us, two rounds of nine 56).  More rounds have to save an eighth (d_c = 512: a
    // twentieth) of that: 8 x 6000 tokens, 500 queries, 40 heads, three rounds counted as 0.975 of one 1004 / 972, 44 heads, two as
    // 0.95 1131 / 1091; 8 x 1000, 44 heads, three as 0.91 114 / 106; but d_c = 512, 1000 tokens, 72 heads, three as 0.91 76 / 81.
    const int kinds = heads * (d_c / 256), pairs = (d_c == 512 ? PM_WAVES<512> : PM_WAVES<256>) / 2;
    int per = 1;
    double least = 1e30;
    for (int rounds = 1; rounds <= 8; ++rounds) {
        const int n = (int)std::min<long long>(std::max(1, 256 * rounds / kinds), pages);
        const double time = (double)(((long long)kinds * n + 255) / 256) * (0.3 + (double)((pages + (long long)n * pairs - 1) / ((long long)n * pairs)));
        if (time < (d_c == 512 ? 0.95 : 0.88) * least) { least = time; per = n; }
    }
    // A multiple of eight heads, which would each stay on one XCD: the shares vary first where there are many pages, so that a page's
    // latent rows are read on one XCD only; with few, reading the weights on all of them costs more.  us by head / by page, d_c = 256,
    // 8 heads: 8 x 250 tokens (32 pages) 22.9 / 25.9, 10000 (157) 267 / 268, 28 x 800 (364) 68.7 / 58.3, 128 x 200 (512) 87 / 70; 16: 1000
    // (16) 40.5 / 43.6, 14 x 800 (182) 61.2 / 58.9, 32 x 350 (192) 62.5 / 58.2; 24: 32 x 250 (128) 66.0 / 66.3, 64 x 130 (192) 99.2 / 97.2;
    // 32: 4 x 1000 (64) 57.6 / 59.7, 64 x 130 (192) 145 / 148, 16 x 1000 (256) 193 / 190; 40: 32 x 1000 (512) 480 / 479, 8 x 6000
    // (752) 1002 / 1024.  Not multiples of eight: 28 heads by page 84 -> 91, 4000 x 4 200 -> 201.
    const bool by_page = d_c == 256 && heads % 8 == 0 && heads <= 32 && pages > std::max(160, 6 * heads);
    const dim3 grid = by_page ? dim3(per, kinds) : dim3(kinds, per);
    if (d_c == 512) prefill_materialise_kernel<512><<<grid, PM_WAVES<512> * 64, 0, s>>>(rows, page_table, seq_lens, uk, uv, pool, lens2, B, heads, num_pages, max_pages, by_page);
    else            prefill_materialise_kernel<256><<<grid, PM_WAVES<256> * 64, 0, s>>>(rows, page_table, seq_lens, uk, uv, pool, lens2, B, heads, num_pages, max_pages, by_page);
    return hipGetLastError();
}

}  // namespace mla
