// Fused tail of the absorbed attention step: split-KV merge followed by the output
// up-projection (third line of the absorbed equation, Sec. 3.3, inside the brackets; App. A.2.2
// writes the same product as part of W'^O):
//     o_lat[b,h,:] = sum_s e^{lse_s - lse} o_s[b,h,:]          out[b,h,:] = o_lat[b,h,:] . W_UV[h]
// One workgroup = one head x BG batch rows, 16 wavefronts.  The whole W_UV[h] slab ([d_c x 128]
// bf16, 128 KB at d_c = 512) is requested as direct-to-LDS loads right after each wavefront's first
// partial rows; while it is in flight the wavefronts merge the partial rows (one wavefront per row
// and block of 256 columns, as in the stand-alone merge kernel: with 16 wavefronts the 16 tasks of
// 8 rows x 512 or 16 rows x 256 columns wait for memory once, side by side, where four wavefronts
// waited four times in a row), write o_lat and leave a bf16 copy in LDS as the A operand.  The
// product then runs on v_mfma_f32_16x16x32_bf16 (eight wavefronts, one tile of 16 columns each)
// with the B operand read by transposing LDS loads (W is stored k-major).  Compared with the two separate kernels this saves a launch and
// overlaps the two dependent memory latencies.  PLAN = true reads the partials where the balanced
// partition's plan puts them (a sequence's chunks one slot apart, any number of them).
#include "mla_internal.h"

namespace mla {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
#define LDS_AS __attribute__((address_space(3)))

constexpr int FT_N = 128;            // d_head
constexpr int FT_ROWB = FT_N * 2;    // bytes per W row in LDS (unpadded: filled by direct-to-LDS loads)
constexpr int FT_MAXB = 16;          // batch rows per workgroup (one MFMA M tile)
constexpr int FT_WAVES = 16;         // wavefronts per workgroup
constexpr int FT_THREADS = FT_WAVES * 64;

// 16-byte chunk swizzle of slab row r (4 bits): spreads the 16 rows x 32 bytes of one
// transposing read over the banks
__device__ __forceinline__ constexpr int ft_key(int r)
{
    return ((r & 3) << 2) | (((r >> 3) & 1) << 1) | ((r >> 4) & 1);
}

// four consecutive values of a partial row as they are stored (a batch of rows in flight costs half the
// registers it would take widened), and widened
__device__ __forceinline__ u32x2 part_bits4(const void* base, size_t elem)
{
    return *reinterpret_cast<const u32x2*>(static_cast<const uint16_t*>(base) + elem);
}
__device__ __forceinline__ f32x4 widen4(u32x2 v)
{
    return (f32x4){bf16_bits_to_f32(v[0] & 0xFFFFu), __uint_as_float(v[0] & 0xFFFF0000u),
                   bf16_bits_to_f32(v[1] & 0xFFFFu), __uint_as_float(v[1] & 0xFFFF0000u)};
}

template <int D_C, bool PLAN>
__global__ __launch_bounds__(FT_THREADS) void merge_out_proj_kernel(MergeParams p, const uint16_t* W_UV, uint16_t* out, int BG)
{
    constexpr int SLAB_B = D_C * FT_ROWB;             // 131072 / 65536
    constexpr int ARS = D_C * 2 + 16;                 // A tile row stride (padded)
    constexpr int NLOAD = SLAB_B / (FT_THREADS * 16); // 8 / 4 direct-to-LDS loads per thread
    __shared__ __attribute__((aligned(1024))) unsigned char smem[SLAB_B + FT_MAXB * ARS];
    LDS_AS unsigned char* lds = (LDS_AS unsigned char*)smem;
    LDS_AS unsigned char* atile = lds + SLAB_B;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroups of one head have linear ids that differ by a multiple of H: they land on the
    // same XCD (ids are dealt round-robin over the 8 XCDs and H is a multiple of 8 for the
    // usual shapes) and share the slab in its L2
    const int h = blockIdx.x;
    const int b0 = blockIdx.y * BG;
    const int nb = min(BG, p.B - b0);

    constexpr int CB = D_C / 256;
    constexpr int BATCH = 16;
    // balanced partition: lane l holds the plan entry of batch row b0 + l (one load for the
    // workgroup's rows, ahead of everything that depends on it)
    int plan_first = 0, plan_count = 0;
    if constexpr (PLAN) {
        if (lane < nb) {
            plan_first = p.plan[2 * (b0 + lane)];
            plan_count = p.plan[2 * (b0 + lane) + 1];
        }
    }
    // the chunks of batch row bl (wave-uniform)
    auto span_of = [&](int bl) -> ChunkSpan {
        if constexpr (PLAN) {
            const int l = __builtin_amdgcn_readfirstlane(bl);
            return planned_span(__builtin_amdgcn_readlane(plan_first, l), __builtin_amdgcn_readlane(plan_count, l), p, h);
        } else {
            return ChunkSpan{part_index(b0 + bl, h, 0, p.H, p.num_splits), 1, p.num_splits};
        }
    };
    // wave task = (batch row, block of 256 columns); partial rows [s0, s0 + BATCH) of a task
    auto task_base = [&](const ChunkSpan& c, int task) {
        return c.first * D_C + (task % CB) * 256 + lane * 4;   // element index into the partial rows
    };
    // rows past the last chunk re-read the last one (their weight is zero): no branches, the
    // kernel's code stays short and straight, which matters for a kernel this brief
    auto load_rows = [&](const ChunkSpan& c, size_t base, int s0, u32x2 (&v)[BATCH]) {
#pragma unroll
        for (int i = 0; i < BATCH; ++i)
            v[i] = part_bits4(p.o_part, base + (size_t)max(0, min(s0 + i, c.S - 1)) * (c.step * D_C));
    };

    auto weighted_rows = [&](float wt, int s0, const u32x2 (&v)[BATCH]) {
        f32x4 a = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            // the weight is 0 at and past S; rows of empty chunks were never written,
            // so what was read there is discarded, not multiplied by zero
            const float ws = lane_value(wt, s0 + i);
            const f32x4 zero = (f32x4){0.f, 0.f, 0.f, 0.f};
            a += ws * (ws != 0.f ? widen4(v[i]) : zero);
        }
        return a;
    };

    // ---- (1) the first task's chunk weights and partial rows are requested ahead of everything
    // else: they come from HBM, the slab mostly from L2 (the workgroups of a head share it).
    // Tasks past the workgroup's batch rows only clear their part of the A tile.
    const int T = nb * CB;                       // tasks with a batch row behind them
    auto request = [&](int task, u32x2 (&v)[BATCH], float& ls) {
        const ChunkSpan c = span_of(task / CB);
        ls = span_lse(p.lse_part, c, 0, lane);
        load_rows(c, task_base(c, task), 0, v);
    };
    u32x2 va[BATCH];
    float lsa = -INFINITY;
    if (wave < T) request(wave, va, lsa);
    for (int task = T + wave; task < FT_MAXB * CB; task += FT_WAVES)
        *(LDS_AS u32x2*)(atile + (task / CB) * ARS + ((task % CB) * 256 + lane * 4) * 2) = (u32x2){0u, 0u};

    // ---- (2) request W_UV[h]: LDS chunk P = row P/16, position P%16 holds chunk (P%16) ^ key(row)
    {
        const unsigned char* src = reinterpret_cast<const unsigned char*>(W_UV + (size_t)h * D_C * FT_N);
        const uint32_t lds_base = (uint32_t)(uintptr_t)lds;
        // (64 rows per load of the workgroup: the swizzle key, made of row bits below 5, is the same for all)
        const int r0 = wave * 4 + (lane >> 4);
        const unsigned char* base = src + r0 * FT_ROWB + (((lane & 15) ^ ft_key(r0)) << 4);
#pragma unroll
        for (int k = 0; k < NLOAD; ++k) {
            const unsigned char* gp = base + k * (FT_WAVES * 4 * FT_ROWB);
            const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds_base + (k * FT_WAVES + wave) * 1024);
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                         :: "s"(m0v), "v"(gp) : "memory");
        }
    }

    // ---- (3) merge (same arithmetic as the stand-alone merge kernel): this wave's tasks (one, or
    // two for 16 batch rows of 512 columns)
    auto reduce = [&](int task, u32x2 (&v)[BATCH], float ls0) {
        const int bl = task / CB, cb = task % CB, b = b0 + bl;
        const ChunkSpan c = span_of(bl);
        const size_t base = task_base(c, task);
        f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
        const ChunkWeights cw = PLAN ? span_weights(p.lse_part, c, ls0, lane) : chunk_weights(ls0);
        // (the sums of every 16 chunks are formed first and then added in order: as in the kernel for few
        // batch rows below, whose wavefronts take one such group each, and in the stand-alone merge)
        for (int blk = 0; blk < c.S; blk += 64) {      // one block unless the plan gives a sequence more than 64 chunks
            const float wt = chunk_weight(cw, blk ? span_lse(p.lse_part, c, blk, lane) : ls0);
            for (int s0 = 0; s0 < min(64, c.S - blk); s0 += BATCH) {
                if (blk + s0 > 0) load_rows(c, base, blk + s0, v);
                acc += weighted_rows(wt, s0, v);
            }
        }
        const u32x2 packed = (u32x2){f32_to_bf16_bits(acc[0]) | (f32_to_bf16_bits(acc[1]) << 16),
                                    f32_to_bf16_bits(acc[2]) | (f32_to_bf16_bits(acc[3]) << 16)};
        *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(p.o_lat) + ((size_t)b * p.H + h) * D_C + cb * 256 + lane * 4) = packed;
        *(LDS_AS u32x2*)(atile + bl * ARS + (cb * 256 + lane * 4) * 2) = packed;
        if (p.lse && cb == 0 && lane == 0) p.lse[(size_t)b * p.H + h] = cw.z > 0.f ? cw.m + logf(cw.z) : -INFINITY;
    };
    for (int task = wave; task < T; task += FT_WAVES) {
        if (task != wave) request(task, va, lsa);
        reduce(task, va, lsa);
    }

    // ---- (4) slab landed (my loads), then everybody's, and the A tile is complete
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();

    // ---- (5) out = o_lat . W_UV[h]: wavefronts 0..7 own one 16-column tile each, as two
    // interleaved chains over the even and the odd k-steps
    if (wave >= FT_N / 16) return;
    // (lane indices from a value the compiler cannot see through: the addresses of this part are worked out
    // here and not kept beside the merge's rows, for which the 128 registers of 16 wavefronts are needed)
    int lane5 = tid & 63;
    asm volatile("" : "+v"(lane5));
    const int n = lane5 & 15, g = lane5 >> 4;
    f32x4 acc[2] = {(f32x4){0.f, 0.f, 0.f, 0.f}, (f32x4){0.f, 0.f, 0.f, 0.f}};
    // transposing read: the lane supplies slab row 32ks + 8g + (n>>2) (+4), 8 bytes at column 4(n&3)
    const int cn = wave * 2 + ((n & 3) >> 1);      // 16-byte chunk of columns
    const uint32_t sub = (uint32_t)((n & 1) * 8);
#pragma unroll 4
    for (int ks = 0; ks < D_C / 32; ks += 2) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const bf16x8 a = *(LDS_AS bf16x8*)(atile + n * ARS + ((ks + j) * 32 + g * 8) * 2);
            const int r0 = (ks + j) * 32 + g * 8 + (n >> 2);
            s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (LDS_AS s16x4*)(lds + r0 * FT_ROWB + ((cn ^ ft_key(r0)) << 4) + sub));
            s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (LDS_AS s16x4*)(lds + (r0 + 4) * FT_ROWB + ((cn ^ ft_key(r0 + 4)) << 4) + sub));
            s16x8 bb = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, bb), acc[j], 0, 0, 0);
        }
    }
    // D: rows 4g..4g+3 (batch rows of this workgroup) of column n
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int bl = g * 4 + i;
        if (bl < nb)
            out[((size_t)(b0 + bl) * p.H + h) * FT_N + wave * 16 + n] = (uint16_t)f32_to_bf16_bits(acc[0][i] + acc[1][i]);
    }
}

// Few batch rows, many chunks (uniform partition): the kernel above gives fewer than one workgroup per CU,
// each pulling a whole slab and walking a row's chunks 16 at a time.  Here a workgroup is one batch row of
// one head x 128 / NS output columns (NS = 2, 4, 8 fills the chip), every group of 16 chunks is merged by a
// wavefront of its own (up to 128 chunks of 512 columns in one round of loads; their sums are added in order
// through LDS), and W's columns go to registers in one round of 128-bit loads requested beside the partial
// rows: the two waits for memory that are left run side by side.  The NS workgroups of a head repeat its merge
// (64 KB of partials at 64 chunks, from L2).  With one row the product is a matrix-vector product bound by
// reading W, on the vector pipes.  32 heads, d_c = 512, back to back in a graph: 1 row of 64 chunks 9.4 us
// above (its weights then formed chunk by chunk), 5.1 here; 4 rows 9.4 and 5.2; 2 rows of 128 chunks (merge and
// projection as two kernels) 15.0 and 7.1.
constexpr int FEW_MAXS = 256;                     // chunks: 16 groups

// MANY: 65 to FEW_MAXS chunks, weights by expf as in the stand-alone merge.
template <int D_C, int NS, bool MANY>
__global__ __launch_bounds__(FT_THREADS) void merge_out_proj_few_kernel(MergeParams p, const uint16_t* W_UV, uint16_t* out)
{
    constexpr int CB = D_C / 256;                 // blocks of 256 latent columns
    constexpr int NC = FT_N / NS;                 // output columns
    constexpr int CC = NC / 8;                    // 16-byte pieces per row of W
    constexpr int KR = FT_THREADS / CC;           // rows of W the workgroup reads at once
    constexpr int NLD = (D_C + KR - 1) / KR;      // loads per thread
    constexpr int BATCH = 16;
    __shared__ f32x4 part[CB * FEW_MAXS / BATCH][64];
    __shared__ float orow[D_C];
    __shared__ float red[FT_WAVES][NC];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = blockIdx.x, b = blockIdx.y, n0 = blockIdx.z * NC;   // a head's workgroups: ids a multiple of H apart
    const ChunkSpan c{part_index(b, h, 0, p.H, p.num_splits), 1, p.num_splits};
    const int tasks = (c.S + BATCH - 1) / BATCH * CB;   // task = (group of 16 chunks, block of columns)

    constexpr int NLS = MANY ? FEW_MAXS / 64 : 1;
    float lsb[NLS];                               // lane l: log-sum-exp of chunks l, 64 + l, ..
    u32x2 v[BATCH];
    auto load_rows = [&](int task) {              // rows past the last chunk re-read it (weight zero)
#pragma unroll
        for (int i = 0; i < BATCH; ++i)
            v[i] = part_bits4(p.o_part, (c.first + min(task / CB * BATCH + i, c.S - 1)) * D_C + task % CB * 256 + lane * 4);
    };
    if (wave < tasks) {
#pragma unroll
        for (int k = 0; k < NLS; ++k) lsb[k] = k * 64 < c.S ? span_lse(p.lse_part, c, k * 64, lane) : -INFINITY;
        load_rows(wave);
    }
    const int piece = tid % CC, k0 = tid / CC;
    const uint16_t* Wp = W_UV + (size_t)h * D_C * FT_N + n0 + piece * 8;
    u32x4 w[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int k = min(i * KR + k0, D_C - 1);
        w[i] = *reinterpret_cast<const u32x4*>(Wp + (size_t)k * FT_N);
    }

    ChunkWeights cw{};
    if (wave < tasks) {
        if constexpr (MANY) cw = chunk_weights(lsb);
        else                cw = chunk_weights(lsb[0]);
        for (int task = wave; task < tasks; task += FT_WAVES) {
            if (task != wave) load_rows(task);
            const int s0 = task / CB * BATCH;
            float ls = lsb[0];
            if constexpr (MANY) ls = s0 < 64 ? lsb[0] : s0 < 128 ? lsb[1] : s0 < 192 ? lsb[2] : lsb[3];
            const float wt = chunk_weight<MANY>(cw, ls);
            f32x4 a = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const float ws = lane_value(wt, s0 % 64 + i);              // 0 at and past S
                const f32x4 zero = (f32x4){0.f, 0.f, 0.f, 0.f};
                a += ws * (ws != 0.f ? widen4(v[i]) : zero);
            }
            part[task][lane] = a;
        }
    }
    __syncthreads();
    if (wave < CB) {
        f32x4 a = (f32x4){0.f, 0.f, 0.f, 0.f};
        const int cb = wave;
        for (int t = cb; t < tasks; t += CB) a += part[t][lane];
        const u32x2 packed = (u32x2){f32_to_bf16_bits(a[0]) | (f32_to_bf16_bits(a[1]) << 16),
                                    f32_to_bf16_bits(a[2]) | (f32_to_bf16_bits(a[3]) << 16)};
        float* o = &orow[cb * 256 + lane * 4];
        o[0] = bf16_bits_to_f32(packed[0] & 0xFFFFu); o[1] = bf16_bits_to_f32(packed[0] >> 16);
        o[2] = bf16_bits_to_f32(packed[1] & 0xFFFFu); o[3] = bf16_bits_to_f32(packed[1] >> 16);
        if (blockIdx.z == 0) {
            *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(p.o_lat) + ((size_t)b * p.H + h) * D_C + cb * 256 + lane * 4) = packed;
            if (p.lse && cb == 0 && lane == 0) p.lse[(size_t)b * p.H + h] = cw.z > 0.f ? cw.m + logf(cw.z) : -INFINITY;
        }
    }
    __syncthreads();

    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int k = i * KR + k0;
        const float x = k < D_C ? orow[min(k, D_C - 1)] : 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            acc[2 * j] = fmaf(x, bf16_bits_to_f32(w[i][j] & 0xFFFFu), acc[2 * j]);
            acc[2 * j + 1] = fmaf(x, __uint_as_float(w[i][j] & 0xFFFF0000u), acc[2 * j + 1]);
        }
    }
    // over the lanes that hold the same columns (CC apart): rotations inside rows of 16 lanes, then the rows
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (CC <= 8) acc[j] += dpp_move<0x128>(acc[j]);   // row_ror:8, 4, 2
        if (CC <= 4) acc[j] += dpp_move<0x124>(acc[j]);
        if (CC <= 2) acc[j] += dpp_move<0x122>(acc[j]);
        acc[j] = sum_rows(acc[j]);
    }
    if (lane < CC) {
#pragma unroll
        for (int j = 0; j < 8; ++j) red[wave][piece * 8 + j] = acc[j];
    }
    __syncthreads();
    if (tid < NC) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < FT_WAVES; ++i) t += red[i][tid];
        out[((size_t)b * p.H + h) * FT_N + n0 + tid] = (uint16_t)f32_to_bf16_bits(t);
    }
}

template <int D_C, bool MANY>
void launch_few(const MergeParams& p, const uint16_t* W, uint16_t* o, int ns, hipStream_t s)
{
    const dim3 grid(p.H, p.B, ns), block(FT_THREADS);
    if (ns == 8)      merge_out_proj_few_kernel<D_C, 8, MANY><<<grid, block, 0, s>>>(p, W, o);
    else if (ns == 4) merge_out_proj_few_kernel<D_C, 4, MANY><<<grid, block, 0, s>>>(p, W, o);
    else if (ns == 2) merge_out_proj_few_kernel<D_C, 2, MANY><<<grid, block, 0, s>>>(p, W, o);
    else              merge_out_proj_few_kernel<D_C, 1, MANY><<<grid, block, 0, s>>>(p, W, o);
}

}  // namespace

bool merge_out_proj_supported(const MergeParams& p, int d_head, mla_dtype io)
{
    return io == MLA_BF16 && d_head == FT_N && (p.d_c == 256 || p.d_c == 512) && p.H <= 4096 &&
           (p.plan || p.num_splits <= 64 || (p.num_splits <= FEW_MAXS && (long)p.H * p.B <= 256));
}

hipError_t launch_merge_out_proj(const MergeParams& p, const void* W_UV, void* out, hipStream_t s)
{
    // batch rows per workgroup: as few as still gives about one workgroup per CU
    int BG = 1;
    while (BG < FT_MAXB && (long)p.H * ((p.B + BG - 1) / BG) > 256) BG *= 2;
    dim3 grid(p.H, (p.B + BG - 1) / BG), block(FT_THREADS);
    const uint16_t* W = static_cast<const uint16_t*>(W_UV);
    uint16_t* o = static_cast<uint16_t*>(out);
    // At most one workgroup per CU with one batch row each, and more than the 16 chunks that the kernel above merges
    // in one round beside its slab: the kernel for few rows, the output columns cut 1 to 8 ways.  32 heads,
    // d_c = 512, back to back in a graph: 1 row of 16 chunks 4.35 above, 4.2 - 4.3 here, 32 chunks 5.2 and 4.3;
    // 8 rows of 32 chunks (columns not cut) 5.5 and 4.8, 16 rows of 16 chunks 4.8 and 8.1 (two slabs per CU);
    // d_c = 256: 1 row of 16 chunks 3.75 and 4.0, 32 chunks 4.5 and 4.1.
    int ns = 1;
    while (ns < 8 && (long)p.H * p.B * ns * 2 <= 256) ns *= 2;
    if (!p.plan && p.num_splits > 16 && (long)p.H * p.B <= 256) {
        if (p.d_c == 512 && p.num_splits > 64) launch_few<512, true>(p, W, o, ns, s);
        else if (p.d_c == 512)                 launch_few<512, false>(p, W, o, ns, s);
        else if (p.num_splits > 64)            launch_few<256, true>(p, W, o, ns, s);
        else                                   launch_few<256, false>(p, W, o, ns, s);
        return hipGetLastError();
    }
    if (p.d_c == 512 && p.plan)  merge_out_proj_kernel<512, true><<<grid, block, 0, s>>>(p, W, o, BG);
    else if (p.d_c == 512)       merge_out_proj_kernel<512, false><<<grid, block, 0, s>>>(p, W, o, BG);
    else if (p.plan)             merge_out_proj_kernel<256, true><<<grid, block, 0, s>>>(p, W, o, BG);
    else                         merge_out_proj_kernel<256, false><<<grid, block, 0, s>>>(p, W, o, BG);
    return hipGetLastError();
}

}  // namespace mla
