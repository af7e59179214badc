// Prefill in the "MHA paradigm" (Sec. 3.3, first of the two attention equations): keys and values
// are materialised per head from the cached latent rows,
//     k_{j,h} = [W^{UK}_h c_j ; k^R_j],        v_{j,h} = W^{UV}_h c_j,
// and the prompt's tokens attend causally to them.  This file holds the two kernels that build
// the materialised keys and values; the attention itself runs on prefill_attention.hip's kernel, for which
// one (sequence, head) pair is a sequence of its own, and whose page layout (64 keys of 192 values, then
// the values transposed, both in the order its reads want) is described there.
//
//   prefill_weights_kernel      Wcat[h] = [W^{UK}_h ; W^{UV}_h] as 256 rows of d_c values each (the
//                               value projection is stored k-major by the caller and is transposed
//                               here once), so that both products read their weights row-wise.
//   prefill_materialise_kernel  one workgroup per (pair of pages, sequence, head):
//                               Y^T [256 x 128 tokens] = Wcat[h] [256 x d_c] . C^T [d_c x 128 tokens]
//                               on v_mfma_f32_16x16x32_bf16; a wavefront owns 32 tokens, keeps
//                               their latent rows in registers as the B operand and walks the 16
//                               row tiles of Wcat[h], which all four wavefronts read from LDS;
//                               results are rounded to bf16 and stored 16 bytes per lane (the page
//                               layout leaves a lane eight neighbouring values of a key, or of a
//                               value dimension: the latter a contiguous kilobyte per wavefront).
#include "mla_internal.h"
#include "mfma_tile.h"
#include <type_traits>

namespace mla {
namespace {

constexpr int PF_DH = 128;      // head dimension
constexpr int PF_KEY = 192;     // values per key: 128 + 64
constexpr int PF_PAGE = 64 * (PF_KEY + PF_DH);    // values per materialised page: 64 keys, then the values transposed

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

// One workgroup = two pages (128 tokens) of one (sequence, head).  Wcat[h] is streamed through LDS
// in chunks of 32 rows (two row tiles, all d_c columns), double-buffered, as direct-to-LDS loads; the four
// wavefronts share every chunk.  Chunk position c ^ (row & 15) of a row holds its 16-byte piece c: the 16 lanes
// that share a cycle of an A read (rows 0 .. 7 of one piece and 8 .. 15 of its neighbour, or the reverse) then
// meet 16 different units (rows padded by 16 bytes, filled through registers, lost 3.2 of 8 cycles per read).
// A wavefront owns 32 tokens (two column tiles) and keeps their latent rows in registers.
// Bound by writing 640 bytes per (token, head) beside 0.25 MFLOP of products: 4 x 8192 tokens, 32 heads, d_c = 512
// 395 -> 351 us (671 MB, 0.27 TFLOP), 26800 tokens, 28 heads, d_c = 256 190 -> 174 us (480 MB).
template <int D_C>
__global__ __launch_bounds__(256, 2) void prefill_materialise_kernel(const uint16_t* kv, const int32_t* page_table,
                                                                     const int32_t* seq_lens, const uint16_t* Wcat,
                                                                     uint16_t* pool2, int32_t* table2, int32_t* lens2,
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
    const int L = max(0, min(seq_lens[b], max_pages * 64));
    if (blockIdx.x == 0 && tid == 0) lens2[bh] = L;
    if (blockIdx.x * 128 >= L) return;

    // this wavefront's page (waves 0, 1: the first of the pair; 2, 3: the second)
    const int pg = blockIdx.x * 2 + (wave >> 1);
    const bool in_seq = pg < max_pages && pg * 64 < L;
    const int page = in_seq ? page_table[(size_t)b * max_pages + pg] : -1;
    const bool active = in_seq && page >= 0 && page < num_pages;
    // the pseudo-sequence (b, h) owns pages [bh * max_pages, +max_pages) of the materialised pool; a page id
    // outside the cache pool is passed on as "skip these tokens" (-1), and its page, like the tokens past the
    // sequence's end, gets zeros for values: what the skipped weights (zeros) are multiplied with
    const size_t page2 = (size_t)bh * max_pages + pg;
    if (in_seq && (wave & 1) == 0 && lane == 0) table2[page2] = active ? (int32_t)page2 : -1;
    const uint16_t* src = kv + (size_t)(active ? page : 0) * 64 * ROW;
    uint16_t* dst = pool2 + (in_seq ? page2 : 0) * PF_PAGE;
    const int tok0 = (wave & 1) * 32;                 // this wavefront's first token inside its page

    bf16x8 cb[2][NKS];
    if (in_seq) {
        // decoupled-rope part of the key: copied as it is (32 tokens x 8 pieces per wavefront)
        for (int i = lane; i < 32 * 8; i += 64) {
            const int tok = tok0 + (i >> 3), ch = i & 7;
            *reinterpret_cast<u32x4*>(dst + tok * PF_KEY + PF_DH + ch * 8) =
                *reinterpret_cast<const u32x4*>(src + tok * ROW + D_C + ch * 8);
        }
        // B operands: latent rows of tokens tok0 + 16 nt + n, k = 32 ks + 8g .. + 7
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const bool there = active && pg * 64 + tok0 + nt * 16 + n < L;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                u32x4 v = *reinterpret_cast<const u32x4*>(src + (tok0 + nt * 16 + n) * ROW + ks * 32 + g * 8);
                if (!there) v = (u32x4){0u, 0u, 0u, 0u};
                cb[nt][ks] = __builtin_bit_cast(bf16x8, v);
            }
        }
    }

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
    load_chunk(0);
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
                    *reinterpret_cast<u32x4*>(dst + (tok0 + nt * 16 + n) * PF_KEY + c * 32 + g * 8) = pack8(acc[0][nt], acc[1][nt]);
            } else {
                product(std::false_type{});
                // 32 tokens (this wavefront's half page) of 32 dimensions: key 4 nt + i of group g is token 16 nt + 4g + i
                uint16_t* half = dst + 64 * PF_KEY + tok0 * PF_DH;
#pragma unroll
                for (int ml = 0; ml < 2; ++ml)
                    *reinterpret_cast<u32x4*>(half + ((c - NCHUNK / 2) * 2 + ml) * 512 + lane * 8) = pack8(acc[ml][0], acc[ml][1]);
            }
        }
    }
}

}  // namespace

bool prefill_supported(int d_head, int d_c, int d_rope, int page_size, mla_dtype io, mla_dtype cache)
{
    return io == MLA_BF16 && cache == MLA_BF16 && d_head == PF_DH && d_rope == 64 && page_size == 64 &&
           (d_c == 256 || d_c == 512);
}

hipError_t launch_prefill_materialise(const void* kv, const int32_t* page_table, const int32_t* seq_lens,
                                      const void* W_UK, const void* W_UV, void* Wcat, void* pool2, int32_t* table2,
                                      int32_t* lens2, int B, int heads, int d_c, int num_pages, int max_pages,
                                      hipStream_t s)
{
    prefill_weights_kernel<<<dim3(d_c / 64, 4, heads), 256, 0, s>>>(static_cast<const uint16_t*>(W_UK),
                                                           static_cast<const uint16_t*>(W_UV),
                                                           static_cast<uint16_t*>(Wcat), d_c);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    dim3 grid((max_pages + 1) / 2, B * heads);
    if (d_c == 512)
        prefill_materialise_kernel<512><<<grid, 256, 0, s>>>(static_cast<const uint16_t*>(kv), page_table, seq_lens,
                                                             static_cast<const uint16_t*>(Wcat), static_cast<uint16_t*>(pool2),
                                                             table2, lens2, heads, num_pages, max_pages);
    else
        prefill_materialise_kernel<256><<<grid, 256, 0, s>>>(static_cast<const uint16_t*>(kv), page_table, seq_lens,
                                                             static_cast<const uint16_t*>(Wcat), static_cast<uint16_t*>(pool2),
                                                             table2, lens2, heads, num_pages, max_pages);
    return hipGetLastError();
}

}  // namespace mla
