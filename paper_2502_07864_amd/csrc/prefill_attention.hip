// Causal attention of the MHA-paradigm prefill (Sec. 3.3, first of the two attention equations) over
// the keys and values materialised per (sequence, head) by prefill.hip, one pseudo-sequence per
// (sequence, head).  Query token i of T sees the keys 0 .. L - T + i.
//
//     S^T [keys x queries]  = K [keys x 192] . Q^T [192 x queries]
//     O^T [128 x queries]  += V^T [128 x keys] . P^T [keys x queries]
//
// A page of 64 keys is 32 KB: the per-head part of the keys, W^{UK}_h c_j, as 64 rows of 128 bf16 values, then the
// values TRANSPOSED, [half page][16-dimension tile][4 groups of 8 keys][16 dimensions][8 keys].  The decoupled-rope part k^R_j, which all
// heads share, is read from the cache itself (copied to every head it was a fifth of what is written and read: 8 x 500 tokens on
// 700 .. 6000 rows, 28 heads, d_c = 256: 387 us with the copies, 376).  Both orders are made for the reads of this
// kernel (the kernel that writes them has the choice for free): inside each 32 of the 128 key
// dimensions position 8g + 4m + i holds dimension 16m + 4g + i (the queries are loaded alike), and
// key j of group g of a half page is its key 4g + j (j < 4) or 16 + 4g + j - 4, which is how the
// exponentiated scores of two 16-key blocks lie in the registers after the first contraction.  So the
// weights are, as they stand, the B operand of the second contraction, and its A operand is one plain
// 128-bit LDS read per 16 dimensions, 16 bytes per lane in lane order: no bank conflict (row-major values
// took two transposing 64-bit reads; [dimension][32 keys] puts the 16 lanes of a cycle on 8 of 16 units).
//
// Workgroup = 128 query rows of one (sequence, head) x all the keys they see; 4 wavefronts, each
// with 32 query rows of its own (two groups of 16) and a private running softmax, so the only
// workgroup barrier is the one that publishes a unit (what two tiles of 32 keys need, direct-to-LDS loads, two slots).  Every LDS read feeds two MFMAs (the two query groups).  The normaliser is a
// product too: one MFMA with an A operand of ones per tile and group sums the rounded weights.  No
// rescaling in the loop: the reference of a query is the maximum of its first tile; a later score more
// than 2^64 above it is recorded and the workgroup then redoes its keys with the exact maxima (one sweep
// that only scores, one that accumulates).
//
// What bounds it: power.  4 prompts of 8192 tokens, 32 heads (2.75 TFLOP): matrix pipes busy 57 to 60 % of 4.7 to 5.0 M cycles, at 1.77
// to 1.9 GHz; a loop of the same instructions on registers alone sustains 2.0 PFLOP/s, of 32 x 32 x 16 ones 1.8 (not taken).  With a
// barrier, five loads, ring slots modulo three and a scalar load of the page table on every tile (76 scalar instructions) the pipes
// were busy 55 % of 5.1 M cycles at a higher clock: 8 % of the cycles gave 2 to 3 % of the time.  Scored, weighed and accumulated
// one tile after the other from row-major values: 42 % of 6.7 M.  Whole call: 3036 us that way, then 2785, now 2736 in turn on one
// card; 8 x 500 new tokens on 700 .. 6000, 28 heads: 552, 396, 376; 2 x 136 on 10539, whose workgroups have a CU each: 340, 288.
#include "prefill_internal.h"
#include "mfma_tile.h"
#include <type_traits>

namespace mla {
namespace {

constexpr int PA_DK = 128;                  // values per materialised key
constexpr int PA_DR = 64;                   // and of its rope part
constexpr int PA_DV = 128;                  // dimensions of a value
constexpr int PA_ROWS = 128;                // query rows per workgroup

__global__ __launch_bounds__(MF_THREADS, 2) void prefill_attention_kernel(PrefillParams p)
{
    constexpr int ROWB = PA_DK * 2, ROPEB = PA_DR * 2;            // 256 and 128 bytes per key
    constexpr int K_B = TILE_ROWS * ROWB;       // 8192: a tile's keys
    constexpr int R_B = TILE_ROWS * ROPEB;      // 4096: their rope part
    constexpr int V_B = TILE_ROWS * PA_DV * 2;  // 8192: its values
    constexpr int PAGE_B = 2 * (K_B + V_B);     // of the pool
    constexpr int SLOT_B = PAGE_B + 2 * R_B;    // of the LDS
    constexpr int NLK = K_B / (MF_THREADS * 16), NLV = 2 * V_B / (MF_THREADS * 16);   // loads per thread: a tile's keys 2 (and rope 1), a page's values 4
    constexpr int NKS = (PA_DK + PA_DR) / 32;   // 6 k-steps of the score contraction: 4 and 2
    constexpr int NCT = PA_DV / 16;             // 8 row tiles of the value contraction

    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * SLOT_B];
    LDS_AS unsigned char* lds = (LDS_AS unsigned char*)smem;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;

    // Workgroup -> (pseudo-sequence, group of 128 query rows).  The groups of one sequence get
    // linear ids 8 apart (ids are dealt round-robin to the 8 XCDs: they run on one XCD and share the
    // sequence's rows in its L2), the groups with the most keys first, and the longest sequences first
    // (up to 64 of them: every workgroup ranks the lengths by itself): a long one started last would run
    // on alone at the end.  8 x 500 new tokens on contexts of 700 .. 6000 rows, 28 heads (the form before this one):
    // 389 us in the order of the batch, 346 longest first.
    const int Z = (p.q_len + PA_ROWS - 1) / PA_ROWS;
    const int id = blockIdx.x, rr = id >> 3;
    const int zi = Z - 1 - rr % Z;
    int b = (rr / Z) * 8 + (id & 7);
    if (b >= p.pairs) return;                       // padding of the last group of 8
    const int nseq = p.pairs / p.heads;
    if (nseq > 1 && nseq <= 64) {
        const int mine = lane < nseq ? p.lens[lane * p.heads] : -1;
        int rank = 0;
        for (int j = 0; j < nseq; ++j) {
            const int other = __builtin_amdgcn_readlane(mine, j);
            rank += other > mine || (other == mine && j < lane);
        }
        const unsigned long long hit = __ballot(lane < nseq && rank == b / p.heads);
        b = (__builtin_ffsll((long long)hit) - 1) * p.heads + b % p.heads;
    }
    b = __builtin_amdgcn_readfirstlane(b);      // (uniform, and said so: what hangs on it stays in scalar registers)
    const int hb = zi * PA_ROWS;
    const int HL = min(PA_ROWS, p.q_len - hb);      // query rows of this workgroup
    // rows of q / out: pair b is (sequence b / heads, head b % heads), its tokens heads rows apart
    const size_t io_base = (size_t)(b / p.heads) * p.q_len * p.heads + (size_t)(b % p.heads);
    auto io_row = [&](int h) -> size_t { return io_base + (size_t)h * p.heads; };

    const int32_t* const ptab = p.page_table + (size_t)(b / p.heads) * p.max_pages;      // pages of the cache
    const int L = __builtin_amdgcn_readfirstlane(max(0, min(p.lens[b], p.max_pages * 64)));

    // ---- this wave's 32 query rows -> registers (B operands of the score contraction)
    bf16x8 qreg[2][NKS];
    {
        const uint16_t* qa = static_cast<const uint16_t*>(p.q_nope);
        const uint16_t* qr = static_cast<const uint16_t*>(p.q_rope);
#pragma unroll
        for (int hi = 0; hi < 2; ++hi) {
            const int row = wave * 32 + hi * 16 + n;
            const size_t qrow = io_row(hb + min(row, HL - 1));
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                u32x4 v;
                if (ks < 4) {                   // the key dimensions' order inside each 32
                    const uint16_t* src = qa + qrow * 128 + ks * 32 + g * 4;
                    const u32x2 lo = *reinterpret_cast<const u32x2*>(src), up = *reinterpret_cast<const u32x2*>(src + 16);
                    v = (u32x4){lo[0], lo[1], up[0], up[1]};
                } else {
                    v = *reinterpret_cast<const u32x4*>(qr + qrow * 64 + (ks - 4) * 32 + g * 8);
                }
                // a negative scale changes the sign of the queries: the largest score is then the largest
                // scaled one
                const uint32_t flip = p.scale < 0.f ? 0x80008000u : 0u;
                v ^= (u32x4){flip, flip, flip, flip};
                qreg[hi][ks] = __builtin_bit_cast(bf16x8, row < HL ? v : (u32x4){0u, 0u, 0u, 0u});
            }
        }
    }

    auto visible = [&](int h) { return L - (p.q_len - 1 - h); };   // keys that query row h sees (one head: rows are tokens)
    // keys [0, row1): what the last query row of the workgroup sees (the rows are ordered by token)
    const int row1 = min(L, visible(min(hb + PA_ROWS, p.q_len) - 1));
    auto store_nothing = [&]() {                // zeros and -inf for the rows of this workgroup
        for (int i = tid; i < HL * (PA_DV / 4); i += MF_THREADS)
            *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(p.out) + io_row(hb + i / (PA_DV / 4)) * PA_DV +
                                      (i % (PA_DV / 4)) * 4) = (u32x2){0u, 0u};
        if (tid < HL && p.lse) p.lse[io_row(hb + tid)] = -INFINITY;
    };
    if (row1 <= 0) {
        store_nothing();
        return;
    }
    const int t1 = (row1 + TILE_ROWS - 1) / TILE_ROWS;            // tiles [0, t1)
    // first key that some query row of this workgroup must not see (its first row sees the least)
    const int causal_from = visible(hb);

    // Page ids, 64 at a time, a lane each (asked for beside the queries; a scalar load in every step was a wait in every step), and
    // whether all pages are there.  Of a page the cache does not have the values are zeros, and no query sees its keys.
    const int pages = (t1 + 1) / 2;
    auto ids_from = [&](int u) { return u + lane < pages ? ptab[u + lane] : 0; };
    const int32_t first_ids = ids_from(0), more_ids[3] = {ids_from(64), ids_from(128), ids_from(192)};
    auto missing = [&](int32_t id) { return (uint32_t)id >= (uint32_t)p.num_pages; };
    auto usable = [&](int32_t id) { return missing(id) ? 0 : id; };

    // ---- staging: direct-to-LDS 128-bit loads.  A step of the sweep needs the values of tile t and the keys of tile t + 1 (its
    // scores are made while tile t is accumulated).  Unit u is what the steps 2 u and 2 u + 1 need: the keys of tile 2 u + 1, the
    // values of both tiles of page u, the keys of tile 2 u + 2, which lie in this order in memory, from 8 KB behind the
    // page's start on, and the rope parts of both.  Two slots; one barrier a unit, which says that unit u is there and unit u - 1 is
    // done with.  The keys of the first tile come where they would lie in unit -1.
    const uint32_t lds_base = (uint32_t)(uintptr_t)lds;
    constexpr int K1 = 0, V0 = K_B, V1 = K_B + V_B, K2 = K_B + 2 * V_B, R1 = PAGE_B, R2 = PAGE_B + R_B;      // places in a slot
    // Chunk swizzles: 16 bytes c of key row r at position c ^ (r & 15), of its rope part at c ^ (r >> 1 & 7): the 16 lanes that share a
    // cycle of a score read meet 16 different units.
    const int P = wave * 64 + lane;
    uint32_t koff[NLK], voff[NLV];
#pragma unroll
    for (int k = 0; k < NLK; ++k) koff[k] = (uint32_t)((P >> 4) * ROWB + (((P & 15) ^ (P >> 4)) << 4) + k * 4096);     // (16 rows, alike)
#pragma unroll
    for (int k = 0; k < NLV; ++k) voff[k] = (uint32_t)(P * 16 + V0 + k * 4096);      // values: as they lie
    const uint32_t roff = (uint32_t)((P >> 3) * p.rope_pitch + (((P & 7) ^ (P >> 4 & 7)) << 4));
    const unsigned char* pool = static_cast<const unsigned char*>(p.pool) + (size_t)b * p.max_pages * PAGE_B;
    auto load16 = [&](const unsigned char* base, uint32_t off, uint32_t dst, auto at) {   // (base and dst are uniform)
        asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :: "s"(dst), "v"(off), "s"(base), "i"(decltype(at)::value) : "memory", "scc");
    };
    auto fetch_keys = [&](const unsigned char* src, uint32_t dst, auto at) {
        load16(src, koff[0], dst, at);
        load16(src, koff[1], dst, std::integral_constant<int, decltype(at)::value + 4096>{});
    };
    static_assert(NLK == 2 && NLV == 4);
    auto values_to = [&](const unsigned char* src, uint32_t dst) {
        load16(src, voff[0], dst, std::integral_constant<int, V0>{});
        load16(src, voff[1], dst, std::integral_constant<int, V0 + 4096>{});
        load16(src, voff[2], dst, std::integral_constant<int, V0 + 8192>{});
        load16(src, voff[3], dst, std::integral_constant<int, V0 + 12288>{});
    };
    const uint32_t rope_page = 64u * (uint32_t)p.rope_pitch;          // bytes from page to page
    int32_t ids;                                // ids of 64 pages
    const unsigned char* rope;                  // rope parts of the page of the unit fetched next
    auto rope_of = [&](int u) { return static_cast<const unsigned char*>(p.rope) + (uint64_t)(uint32_t)__builtin_amdgcn_readlane(ids, u & 63) * rope_page; };
    using AtK1 = std::integral_constant<int, K1>;
    using AtK2 = std::integral_constant<int, K2>;
    using AtR1 = std::integral_constant<int, R1>;
    using AtR2 = std::integral_constant<int, R2>;
    // unit u (2 u < t1): all of its page behind the first tile's keys (the second tile's, where they are not asked for, are there but
    // never used), and the next page's first keys if there is one.  Returns the number of loads this thread issued (uniform).
    auto fetch_unit = [&](int u) -> int {
        const unsigned char* src = pool + (size_t)u * PAGE_B + K_B;
        const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_base + (uint32_t)((u & 1) * SLOT_B + wave * 1024));
        fetch_keys(src, dst, AtK1{});
        values_to(src, dst);
        load16(rope + rope_page / 2, roff, dst, AtR1{});
        if (2 * u + 2 >= t1) return NLK + NLV + 1;
        fetch_keys(src + K2, dst, AtK2{});
        if (((u + 1) & 63) == 0) {
            ids = usable(ids_from(u + 1));
            asm volatile("" : "+v"(ids));       // (waited for here: behind the branch everybody would, for everything)
        }
        rope = rope_of(u + 1);
        load16(rope, roff, dst, AtR2{});
        return 2 * NLK + NLV + 2;
    };
    // the first tile's keys are there
    auto start = [&]() {
        const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_base + (uint32_t)(SLOT_B + wave * 1024));
        fetch_keys(pool, dst, AtK2{});
        rope = rope_of(0);
        load16(rope, roff, dst, AtR2{});
        if (fetch_unit(0) > NLK + NLV + 1) wait_vmcnt<2 * NLK + NLV + 2>();
        else                               wait_vmcnt<NLK + NLV + 1>();
        __syncthreads();
    };
    ids = usable(first_ids);
    start();
    bool hole = missing(first_ids) || missing(more_ids[0]) || missing(more_ids[1]) || missing(more_ids[2]);
    for (int u = 256; u < pages; u += 64) hole |= missing(ids_from(u));
    const bool all_there = !__any(hole);
    // keys of tile t that are there
    auto rows_valid = [&](int t) { return all_there || !missing(((const CONST_AS int32_t*)ptab)[t >> 1]) ? min(TILE_ROWS, row1 - t * TILE_ROWS) : 0; };
    // leading tiles that every query row of this workgroup sees whole
    const int n_full = all_there ? max(0, min(causal_from, row1)) / TILE_ROWS : 0;

    // ---- per-lane state: this lane's queries = column n of the D tiles of the two groups
    float m_ref[2] = {-INFINITY, -INFINITY};   // reference of the exponentials (log2 units)
    float top[2] = {-INFINITY, -INFINITY};     // largest score of the sweep so far, this lane's keys (unscaled)
    f32x4 lacc[2];                             // normaliser (four times the same)
    f32x4 oacc[2][NCT];
    // (never zero: a masked score is -inf and has to stay it)
    const float sc = fmaxf(fabsf(p.scale) * LOG2E, 1.17549435e-38f);
    const int my_row = wave * 32 + n;           // + 16 hi; local to the workgroup

    // score A operand: key row 16 rb + n, chunk 4 ks + g (ks 4, 5: chunk 4 (ks - 4) + g of its rope part)
    uint32_t a_base[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
        a_base[ks] = ks < 4 ? (uint32_t)(n * ROWB + (((4 * ks + g) ^ n) << 4)) : (uint32_t)(n * ROPEB + (((4 * (ks - 4) + g) ^ (n >> 1)) << 4));
    // value A operand: dimension 16 ct + n, the eight keys of lane group g
    const uint32_t v_base = (uint32_t)(lane * 16);
    const bf16x8 ones = __builtin_bit_cast(bf16x8, (u32x4){0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u});

    typedef f32x4 Scores[2][2];     // [block of 16 keys][query group]: keys 16 rb + 4g + i of query n, unscaled
    auto max3 = [](float a, float b, float c) {
        float r;                    // (a NaN loses, as in fmaxf; written out: fmaxf would quieten every operand first)
        asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
        return r;
    };
    auto raise_top = [&](const Scores& x) {
#pragma unroll
        for (int hi = 0; hi < 2; ++hi)
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) top[hi] = max3(max3(top[hi], x[rb][hi][0], x[rb][hi][1]), x[rb][hi][2], x[rb][hi][3]);
    };
    // maximum over the four lane groups (all 32 keys of the tile), on every lane
    auto over_groups = [&](float v) {
        v = fmaxf(v, __shfl_xor(v, 16));
        return fmaxf(v, __shfl_xor(v, 32));
    };
    // keys a query must not see (or that are not there) at -inf
    auto mask = [&](Scores& x, int t) {
        // (few tiles take this: what it compares with is worked out here and not kept in registers)
        const int n_valid = rows_valid(t);
        int first = 4 * g;
        asm volatile("" : "+v"(first));
#pragma unroll
        for (int hi = 0; hi < 2; ++hi) {
            const int seen = min(n_valid, visible(hb + my_row + hi * 16) - t * TILE_ROWS) - first;
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (rb * 16 + i >= seen) x[rb][hi][i] = -INFINITY;
        }
    };
    // Tokens of the last tile that come after every query of this workgroup: their values become zeros, so that
    // whatever they are (their weights are zeros, but 0 * inf is not) stays out.  Tokens past the sequence's end
    // are zeros already.
    auto drop_late_values = [&](int t) {
        const int there = row1 - t * TILE_ROWS;
        for (int u = tid; u < V_B / 16; u += MF_THREADS) {
            LDS_AS u32x4* at = (LDS_AS u32x4*)(lds + ((t >> 1) & 1) * SLOT_B + (t & 1 ? V1 : V0) + u * 16);
            const int first = 4 * ((u >> 4) & 3);        // key of the unit's first value; the fifth is 16 further on
            u32x4 v = *at;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int key = first + (d >> 1) * 16 + (d & 1) * 2;
                v[d] = key + 1 < there ? v[d] : key < there ? v[d] & 0xFFFFu : 0u;
            }
            *at = v;
        }
        __syncthreads();
    };
    const bool late_values = row1 < L && row1 % TILE_ROWS != 0;

    // ---- one step: S^T of the next tile (QK), the weights of this one from its scores x, the normaliser and the
    // values (PV).  The weights (two exponentials, a conversion and two multiply-adds per pair of scores) are
    // placed between the matrix instructions of the next tile's scores, which they do not depend on: both pipes
    // of the SIMD work on one wavefront, where a step that scored, weighed and accumulated one tile in turn left
    // each idle for the other's share (matrix pipes busy 42 %, vector pipes 45 %, LDS 20 % of the time).
    // Its first keys (k-steps 0 and 1) have been read before it, those of the page's second step by its first.  
    // PV = false: the scores alone (the first tile's).
    bf16x8 ka[2][NKS];
    auto rk = [&](uint32_t unit, bool second, int ks) {
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
            ka[rb][ks] = *(LDS_AS bf16x8*)(lds + unit + a_base[ks] + (ks < 4 ? (second ? K2 : K1) + rb * 16 * ROWB : (second ? R2 : R1) + rb * 16 * ROPEB));
    };
    auto step = [&](auto pv_tag, auto second_tag, uint32_t unit, const Scores& x, Scores& y) {
        constexpr bool PV = decltype(pv_tag)::value, SECOND = decltype(second_tag)::value;
        constexpr int V = SECOND ? V1 : V0;
        bf16x8 va[NCT];
        auto rv = [&](int ct) { va[ct] = *(LDS_AS bf16x8*)(lds + unit + v_base + V + ct * 1024); };
        float m_use[2];
        uint32_t w[2][4];
        auto weigh = [&](int j) {               // pair j of 8: query group j / 4, scores 2 (j % 4) and the one after
            const int hi = j >> 2, rb = (j >> 1) & 1, i = 2 * (j & 1);
            w[hi][2 * rb + (j & 1)] = pack_bf16x2(fast_exp2(fmaf(x[rb][hi][i], sc, -m_use[hi])),
                                                  fast_exp2(fmaf(x[rb][hi][i + 1], sc, -m_use[hi])));
        };
        if constexpr (PV) {
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) m_use[hi] = m_ref[hi] == -INFINITY ? 0.f : m_ref[hi];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            if (ks + 2 < NKS) rk(unit, SECOND, ks + 2);
            else if (PV) {
                rv(2 * (ks + 2 - NKS));
                rv(2 * (ks + 2 - NKS) + 1);
            }
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int hi = 0; hi < 2; ++hi)
                    y[rb][hi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[rb][ks], qreg[hi][ks],
                                                                        ks == 0 ? (f32x4){0.f, 0.f, 0.f, 0.f} : y[rb][hi], 0, 0, 0);
            if constexpr (PV) {
                if (ks == 0) { weigh(0); weigh(1); }
                else if (ks == 3) { weigh(4); weigh(5); }
                else weigh(ks < 3 ? ks + 1 : ks + 2);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // an LDS read
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);     // a matrix instruction
                    __builtin_amdgcn_sched_group_barrier(0x2, 3, 0);     // vector instructions in its shadow
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (PV) {
            bf16x8 pb[2];
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) pb[hi] = __builtin_bit_cast(bf16x8, (u32x4){w[hi][0], w[hi][1], w[hi][2], w[hi][3]});
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                if (ct + 4 < NCT) rv(ct + 4);
                else if (!SECOND && ct + 2 >= NCT) rk(unit, true, ct + 2 - NCT);
                if (ct == 0) {
#pragma unroll
                    for (int hi = 0; hi < 2; ++hi) lacc[hi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[hi], lacc[hi], 0, 0, 0);
                }
#pragma unroll
                for (int hi = 0; hi < 2; ++hi)
                    oacc[hi][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[ct], pb[hi], oacc[hi][ct], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // the reference of a query: the maximum of its first tile with a visible key
    bool unset = true;
    auto set_reference = [&](const Scores& x) {
        bool left = false;
#pragma unroll
        for (int hi = 0; hi < 2; ++hi) {
            float tm = max3(x[0][hi][0], x[0][hi][1], x[0][hi][2]);
            tm = max3(tm, x[0][hi][3], x[1][hi][0]);
            tm = over_groups(max3(max3(tm, x[1][hi][1], x[1][hi][2]), x[1][hi][3], tm));
            if (m_ref[hi] == -INFINITY) m_ref[hi] = tm == -INFINITY ? tm : tm * sc;
            left |= m_ref[hi] == -INFINITY;
        }
        unset = __any(left);
    };

    // ---- sweeps over the keys.  ACCUMULATE against the references (set on the way where they are not yet); if some
    // score exceeded its reference by more than FAST_GAP (rare), a sweep that only scores finds the exact maxima
    // and the accumulation is done again against them.
    enum { ACCUMULATE, MAXIMA, ACCUMULATE_AGAIN };
    for (int pass = ACCUMULATE;;) {
#pragma unroll
        for (int hi = 0; hi < 2; ++hi) {
            lacc[hi] = (f32x4){0.f, 0.f, 0.f, 0.f};
            top[hi] = -INFINITY;
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) oacc[hi][ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
        auto look_at = [&](Scores& x, int t) {   // scores of tile t, just made
            if (__builtin_expect(t >= n_full, 0)) mask(x, t);
            raise_top(x);
            if (unset) set_reference(x);
        };
        // (one form of the step for all: the last one scores what the slot holds in the place of keys, the sweep
        // for the maxima accumulates too, and neither result is used)
        using Yes = std::true_type;
        using No = std::false_type;
        Scores x, y;
        rk(SLOT_B, true, 0);
        rk(SLOT_B, true, 1);
        step(No{}, Yes{}, (uint32_t)SLOT_B, x, x);
        look_at(x, 0);
        uint32_t unit = 0;
        for (int t = 0; t < t1; t += 2) {
            wait_vmcnt<0>();
            __syncthreads();
            rk(unit, false, 0);
            rk(unit, false, 1);
            if (t + 2 < t1) fetch_unit((t >> 1) + 1);
            if (late_values && t + 2 >= t1) drop_late_values(t1 - 1);
            step(Yes{}, No{}, unit, x, y);
            if (t + 1 >= t1) break;
            look_at(y, t + 1);
            step(Yes{}, Yes{}, unit, y, x);
            if (t + 2 < t1) look_at(x, t + 2);
            unit = SLOT_B - unit;
        }
        __syncthreads();         // every wave is done with the units of this sweep
        if (pass == ACCUMULATE_AGAIN) break;
        if (pass == ACCUMULATE) {
            const bool jumped = top[0] * sc > m_ref[0] + FAST_GAP || top[1] * sc > m_ref[1] + FAST_GAP;
            // (a flag per wavefront, where start() puts nothing)
            LDS_AS int* const flags = (LDS_AS int*)(lds + SLOT_B);
            const bool mine = __any(jumped);
            if (lane == 0) flags[wave] = mine;
            __syncthreads();
            const int any = flags[0] | flags[1] | flags[2] | flags[3];
            if (__builtin_expect(!any, 1)) break;
            pass = MAXIMA;
            unset = false;
        } else {
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
                const float tm = over_groups(top[hi]);
                m_ref[hi] = tm == -INFINITY ? tm : tm * sc;
            }
            pass = ACCUMULATE_AGAIN;
        }
        if (pages > 64) ids = usable(ids_from(0));
        start();
    }
    // ---- normalise, round to bf16, transpose through LDS (a lane holds 4 consecutive columns of its
    // query per column tile) and store whole 256-byte rows
    constexpr int RSO = PA_DV * 2 + 16;         // row stride of the transposed block (padded)
    static_assert(4 * 32 * RSO <= SLOT_B, "exchange space must fit in a slot");    // (the flags lie in the other one)
    LDS_AS unsigned char* mine = lds + wave * (32 * RSO);
    float lt[2];
#pragma unroll
    for (int hi = 0; hi < 2; ++hi) {
        lt[hi] = lacc[hi][0];
        const float inv = lt[hi] > 0.f ? 1.f / lt[hi] : 0.f;
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            const f32x4 v = oacc[hi][ct] * inv;
            *(LDS_AS u32x2*)(mine + (hi * 16 + n) * RSO + (ct * 16 + g * 4) * 2) =
                (u32x2){pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        }
    }
    const int nrow = min(32, HL - wave * 32);
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += 4) {
        const int r = r0 + (lane >> 4), c = lane & 15;   // 16 lanes x 16 bytes = one row
        if (r < nrow) {
            const u32x4 v = *(LDS_AS u32x4*)(mine + r * RSO + c * 16);
            *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(p.out) + io_row(hb + wave * 32 + r) * PA_DV + c * 8) = v;
        }
    }
    if (g == 0 && p.lse) {
#pragma unroll
        for (int hi = 0; hi < 2; ++hi)
            if (my_row + hi * 16 < HL)
                p.lse[io_row(hb + my_row + hi * 16)] =
                    lt[hi] > 0.f ? (m_ref[hi] + __builtin_amdgcn_logf(lt[hi])) * LN2 : -INFINITY;
    }
}

}  // namespace

hipError_t launch_prefill_attention(const PrefillParams& p, hipStream_t s)
{
    if (!p.out || p.heads < 1) return hipErrorInvalidValue;
    const long long Z = (p.q_len + PA_ROWS - 1) / PA_ROWS;
    const long long nwg = ((long long)p.pairs + 7) / 8 * 8 * Z;
    if (nwg > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    prefill_attention_kernel<<<dim3((unsigned)nwg), dim3(MF_THREADS), 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace mla
