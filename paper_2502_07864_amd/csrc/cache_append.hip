// Cache append: the row the decode reads, produced for one new token per sequence
// (Sec. 3.3, MLA equations, left column):
//     c^{KV}_t = W^{DKV} x_t        k^R_t = RoPE(W^{KR} x_t, t)        row = [c^{KV}_t ; k^R_t]
// with RoPE as in Sec. 3.1, Eq. 1 (consecutive pairs (real, imaginary), pair i turned by
// t * base^(-2i/d^R)).  The two projections are one skinny GEMM x . [W^{DKV} ; W^{KR}]^T whose cost
// is reading the weights once: it runs on the per-head GEMM kernels with the model dimension cut
// into slices that play the part of the heads (fp32 partial rows), so that enough workgroups
// stream the weights.  One small kernel per sequence then adds the slices in a fixed order,
// rotates the rope part (angles in fp64: positions reach 10^5 radians), rounds the row to the
// cache dtype (fp8: one scale per token, absmax / 448, codes by round-to-nearest-even,
// saturating) and writes it through the page table.  bf16 io with a bf16 or fp32 cache, whose rounding needs no
// more of the row than its own column, does both in one kernel at up to 64 - 128 sequences.
#include "mla_internal.h"
#include "mfma_tile.h"

namespace mla {
namespace {

constexpr int AP_MAXN = 1024;   // longest cache row the finishing kernel holds in LDS

// fp32 -> OCP e4m3 code: nearest, ties to even, magnitudes above 448 saturate, NaN -> S.1111.111
__device__ __forceinline__ uint32_t f32_to_e4m3_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    const uint32_t sign = (u >> 24) & 0x80u;
    u &= 0x7FFFFFFFu;
    if (u > 0x7F800000u) return sign | 0x7Fu;
    const float a = __uint_as_float(u);
    if (a >= 448.f) return sign | 0x7Eu;
    if (a < 0.015625f) return sign | (uint32_t)rintf(a * 512.f);   // subnormals m * 2^-9; 8 is 2^-6
    // normal: keep 3 mantissa bits, round to nearest even (a carry moves into the exponent)
    u += 0x7FFFFu + ((u >> 20) & 1u);
    return sign | ((u >> 20) - (120u << 3));
}

// cosine and sine of the angle that rope pair i (of d_rope / 2) turns by at a position
__device__ __forceinline__ void rope_turn(const AppendParams& p, int i, int pos, double& cs, double& sn)
{
    const double theta = pow((double)p.rope_base, -2.0 * (double)i / (double)p.d_rope);
    sincos((double)pos * theta, &sn, &cs);
}

// ---- one kernel: projection, rotation, store (bf16 io; bf16 or fp32 cache; D a multiple of 32, rows of W a multiple
// of 16 columns).  A workgroup owns 16 columns for 16 sequences; its 16 wavefronts take the model dimension in pairs
// of 32 rows of W, four pairs (8 KB of W and 8 KB of x) of each on their way at once, and multiply them on
// v_mfma_f32_16x16x32_bf16; the partial sums meet in LDS.  The four workgroups that share the 128-byte lines of W
// run on one XCD, and so do those of the same columns.  What bounds it is one launch and one round trip for 262 KB
// per workgroup; as two kernels with the partial rows in memory between them, each had both.  x goes by whole lines
// and through LDS: read straight in operand order (16 rows of 8 KB by 16 neighbouring lanes) it took 2 us more.
// D = 4096, n = 576 (4.7 MB of W), us before and now: 1 sequence 8.5 -> 5.0,
// 16 9.5 -> 5.4, 64 11.6 -> 7.9.
constexpr int A1_WAVES = 16;
constexpr int A1_PAIRS = 4;               // pairs of a wavefront in flight
constexpr int A1_PAIR_B = 4096;           // a pair in LDS: 64 rows of 16 columns of W, 16 rows of 64 of x

template <int CACHE>
__global__ __launch_bounds__(A1_WAVES * 64) void append_one_kernel(AppendParams p)
{
    __shared__ __attribute__((aligned(16))) unsigned char smem[A1_WAVES * 2 * A1_PAIR_B];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int cols = p.d_c + p.d_rope;
    // column tile: groups of four tiles (64 columns, a line of W) on one XCD (ids equal mod 8)
    const int id = blockIdx.x, quad = (id >> 5) * 8 + (id & 7), tile = quad * 4 + ((id >> 3) & 3);
    if (tile * 16 >= cols) return;
    const int c0 = tile * 16, b0 = blockIdx.y * 16;
    LDS_AS unsigned char* mine = (LDS_AS unsigned char*)smem + wave * 2 * A1_PAIR_B;

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const uint16_t* W = static_cast<const uint16_t*>(p.W) + c0 + (lane & 1) * 8;
    const uint16_t* x = static_cast<const uint16_t*>(p.x) + (lane & 7) * 8;
    const int steps = p.D / 32;               // the last pair may hold one step only
    for (int q0 = wave; 2 * q0 < steps; q0 += A1_WAVES * A1_PAIRS) {
        u32x4 w[A1_PAIRS][2], a[A1_PAIRS][2];
#pragma unroll
        for (int q = 0; q < A1_PAIRS; ++q)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int st = 2 * (q0 + q * A1_WAVES) + i;
                w[q][i] = (u32x4){0u, 0u, 0u, 0u};
                if (st < steps) w[q][i] = *reinterpret_cast<const u32x4*>(W + (size_t)(st * 32 + (lane >> 1)) * cols);
            }
#pragma unroll
        for (int q = 0; q < A1_PAIRS; ++q)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                // eight rows of a pair: lane -> (row, 16 bytes of its line)
                const int pr = q0 + q * A1_WAVES, b = b0 + i * 8 + (lane >> 3);
                a[q][i] = (u32x4){0u, 0u, 0u, 0u};
                if (2 * pr + ((lane >> 2) & 1) < steps && b < p.B)
                    a[q][i] = *reinterpret_cast<const u32x4*>(x + (size_t)b * p.D + pr * 64);
            }
        // A pair at a time through the wavefront's own LDS (accesses of a wavefront complete in order).  x: 16-byte
        // unit u of row r at position u ^ (r & 7) of its 128 bytes, so that both directions are free of bank conflicts
#pragma unroll
        for (int q = 0; q < A1_PAIRS; ++q) {
            LDS_AS unsigned char* wq = mine + (q & 1) * A1_PAIR_B;
            LDS_AS unsigned char* xq = wq + 2048;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                *(LDS_AS u32x4*)(wq + i * 1024 + lane * 16) = w[q][i];
                *(LDS_AS u32x4*)(xq + i * 1024 + (lane >> 3) * 128 + ((lane & 7) ^ (lane >> 3)) * 16) = a[q][i];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                // transposing read: the lane supplies row 8g + (n>>2) (and 4 more), 8 bytes at column 4 (n&3)
                LDS_AS unsigned char* at = wq + i * 1024 + (g * 8 + (n >> 2)) * 32 + (n & 3) * 8;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)at);
                const s16x4 up = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(at + 4 * 32));
                const bf16x8 wb = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7));
                const u32x4 xa = *(LDS_AS u32x4*)(xq + n * 128 + ((i * 4 + g) ^ (n & 7)) * 16);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xa), wb, acc, 0, 0, 0);
            }
        }
    }
    // acc: lane (g, n) holds sequences 4g .. 4g+3 of column n.  The first four wavefronts finish, a thread per
    // (sequence, column); where its value goes and how it turns is looked up while the others finish
    const int b = b0 + (tid >> 4), col = c0 + (tid & 15);
    double cs = 1.0, sn = 0.0;
    long dst = -1;
    if (wave < 4 && b < p.B) {
        const int pos = p.positions[b];
        if (pos >= 0 && pos < p.max_pages * p.page_size) {                         // inside the table
            const int page = p.page_table[(size_t)b * p.max_pages + pos / p.page_size];
            if (page >= 0 && page < p.num_pages)                                   // inside the pool
                dst = ((long)page * p.page_size + pos % p.page_size) * cols + col;
            if (col >= p.d_c) rope_turn(p, (col - p.d_c) >> 1, pos, cs, sn);
        }
    }
    __syncthreads();                               // everybody is done with the weights
    float* red = reinterpret_cast<float*>(smem);   // [wave][sequence][column]
#pragma unroll
    for (int i = 0; i < 4; ++i) red[(wave * 16 + g * 4 + i) * 16 + n] = acc[i];
    __syncthreads();
    if (wave >= 4) return;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < A1_WAVES; ++w) v += red[w * 256 + tid];
    const float other = __shfl_xor(v, 1);          // the pair's other component
    if (col >= p.d_c) v = col & 1 ? (float)((double)other * sn + (double)v * cs)
                                  : (float)((double)v * cs - (double)other * sn);
    if (dst < 0) return;
    if (CACHE == MLA_F32) static_cast<float*>(p.kv)[dst] = v;
    else                  static_cast<uint16_t*>(p.kv)[dst] = (uint16_t)f32_to_bf16_bits(v);
}

template <int CACHE>   // mla_dtype of the cache
__global__ __launch_bounds__(256) void append_finish_kernel(AppendParams p)
{
    __shared__ float row[AP_MAXN];
    __shared__ float wmax[4];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int n = p.d_c + p.d_rope;
    const int pos = p.positions[b];   // requested now, needed after the sums

    // the rotation's angle, worked out while the partial rows are on their way (positions outside the table
    // are turned by nothing anybody sees)
    double sn = 0.0, cs = 1.0;
    // Slices added in index order.  The loads do not depend on the position or the page, so they
    // go out first: sixteen slices of each of this thread's columns at a time (slices past the
    // last re-read it and are not added; columns past the row likewise).
    {
        constexpr int NC = AP_MAXN / 256;
        float acc[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = 0.f;
        const float* base = p.part + (size_t)b * p.slices * n;
        for (int s0 = 0; s0 < p.slices; s0 += 16) {
            float v[NC][16];
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    v[c][i] = base[(size_t)min(s0 + i, p.slices - 1) * n + min(tid + c * 256, n - 1)];
            if (s0 == 0 && tid < p.d_rope / 2) rope_turn(p, tid, pos, cs, sn);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[c] += s0 + i < p.slices ? v[c][i] : 0.f;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (tid + c * 256 < n) row[tid + c * 256] = acc[c];
    }
    if (pos < 0 || pos >= p.max_pages * p.page_size) return;          // outside the table
    const int page = p.page_table[(size_t)b * p.max_pages + pos / p.page_size];
    if (page < 0 || page >= p.num_pages) return;                      // outside the pool
    const size_t r = (size_t)page * p.page_size + (size_t)(pos % p.page_size);
    __syncthreads();
    if (tid < p.d_rope / 2) {
        const double re = row[p.d_c + 2 * tid], im = row[p.d_c + 2 * tid + 1];
        row[p.d_c + 2 * tid]     = (float)(re * cs - im * sn);
        row[p.d_c + 2 * tid + 1] = (float)(re * sn + im * cs);
    }
    __syncthreads();

    if (CACHE == MLA_F32) {
        float* dst = static_cast<float*>(p.kv) + r * n;
        for (int j = tid; j < n; j += 256) dst[j] = row[j];
    } else if (CACHE == MLA_BF16) {
        uint16_t* dst = static_cast<uint16_t*>(p.kv) + r * n;
        for (int j = tid; j < n; j += 256) dst[j] = (uint16_t)f32_to_bf16_bits(row[j]);
    } else {
        float amax = 0.f;
        for (int j = tid; j < n; j += 256) amax = fmaxf(amax, fabsf(row[j]));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o));
        if ((tid & 63) == 0) wmax[tid >> 6] = amax;
        __syncthreads();
        amax = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
        const float scale = amax > 0.f ? amax / 448.0f : 1.0f;
        uint8_t* dst = static_cast<uint8_t*>(p.kv) + r * n;
        for (int j = tid; j < n; j += 256) dst[j] = (uint8_t)f32_to_e4m3_bits(row[j] / scale);
        if (tid == 0) p.kv_scale[r] = scale;
    }
}

}  // namespace

// Slices of the model dimension: the widest slice (fewest partial rows) that still gives the
// chip a workgroup per CU, the narrowest if none does.  Slices of a multiple of 32 up to 512
// rows suit the matrix-core GEMM; anything else runs as one slice on the scalar-FMA kernel.
int append_slices(int B, int D, int n, mla_dtype io)
{
    if (io != MLA_BF16 || D % 32 || n % 16) return (D > 512 && D % 512 == 0) ? D / 512 : 1;
    const long per_slice = (long)((n + 63) / 64) * ((B + 63) / 64);
    int best = 0;
    for (int ks = 512; ks >= 32; ks >>= 1) {
        if (D % ks) continue;
        best = D / ks;
        if ((long)best * per_slice >= 256) break;
    }
    return best > 0 ? best : 1;
}

hipError_t launch_cache_append(const AppendParams& p, mla_dtype io, mla_dtype cache, hipStream_t s)
{
    const int n = p.d_c + p.d_rope;
    // One kernel while all workgroups of an XCD run at once (four per line of W and group of 16 sequences, one per
    // CU for their LDS) and each takes its columns in two rounds at most.  us, two kernels -> one, D x n = 4096 x 576:
    // 16 sequences 9.5 -> 5.4, 64 11.6 -> 7.9, 80 (past the rule) 10.9 -> 11.7; 64 sequences, D = 8192: 13.3 -> 13.3,
    // 16 sequences, D = 16384 (past it): 11.0 -> 23.9.
    const unsigned quads = (unsigned)((n + 63) / 64), groups = (unsigned)((p.B + 15) / 16);
    if (io == MLA_BF16 && cache != MLA_FP8_E4M3 && p.D % 32 == 0 && n % 16 == 0 && p.d_c % 2 == 0 &&
        (quads + 7) / 8 * 4 * groups <= 32 && p.D <= 2 * A1_WAVES * A1_PAIRS * 64 && reinterpret_cast<uintptr_t>(p.x) % 16 == 0 &&
        reinterpret_cast<uintptr_t>(p.W) % 16 == 0) {
        const dim3 grid((quads + 7) / 8 * 32, groups), block(A1_WAVES * 64);
        if (cache == MLA_F32) append_one_kernel<MLA_F32><<<grid, block, 0, s>>>(p);
        else                  append_one_kernel<MLA_BF16><<<grid, block, 0, s>>>(p);
        return hipGetLastError();
    }
    // x [B, D] = [B, slices, D/slices] and W [D, n] = [slices, D/slices, n]: the slices are the "heads"
    hipError_t e = launch_head_gemm(p.x, p.W, p.part, p.B, p.slices, p.D / p.slices, n, io, s,
                                    /*y_f32=*/true);
    if (e != hipSuccess) return e;
    dim3 grid(p.B), block(256);
    if (cache == MLA_F32)       append_finish_kernel<MLA_F32><<<grid, block, 0, s>>>(p);
    else if (cache == MLA_BF16) append_finish_kernel<MLA_BF16><<<grid, block, 0, s>>>(p);
    else                        append_finish_kernel<MLA_FP8_E4M3><<<grid, block, 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace mla
