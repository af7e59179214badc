// Portable (scalar-FMA, fp32) kernels: paged decode for every supported dtype
// pair and shape, the split-KV merge, and the page gather test hook.
//
// The decode kernels here and in decode_tiles.hip (whichever is the faster) are the library's reference GPU
// path: the only one for fp32 caches and fp32 io and for shapes the matrix-core kernels do not
// cover.  One workgroup handles (chunk, sequence, group of HG heads); its four
// wavefronts take the chunk's rows four or eight at a time, in turn, and share nothing
// until the end: a row lives in the registers of one wavefront, lane l holding
// the four latent values 4 l .. 4 l + 3, the four from 256 further on, and (the
// first lanes) four of the rope part, so the same registers serve the score
// (second line of the absorbed attention equation, Sec. 3.3 of the paper) and the
// latent sum, and no row passes through LDS.  The sums over the lanes of all its
// scores are taken together, halving the values with every exchange of lane
// halves.  A running softmax per wavefront, joined over the four at the end.
//
// The kernel is bound by latency on a small call (one short sequence) and by the
// vector pipes on a large one (about 25 instructions per row and head for 17 useful
// ones).  The tiles stage 16 rows at a time in LDS between four workgroup
// barriers: one fp32 sequence of 1024 rows, 32 heads, d_c = 512, 16 chunks: 23.5 us on
// 64 workgroups, 10.1 here; 4 sequences of 2000 rows in 28 chunks: 53.0 and 29.4; 16 bf16 sequences of 8192
// rows in 63-row pages: 493 and 373; eight fp32 sequences of 4000 rows, every row read eight times from
// L2: 108 and 101 (back to back in a graph).
#include "mla_internal.h"
#include <type_traits>

namespace mla {
namespace {

constexpr int PR_MAX_DC = 512;    // two groups of four latent values per lane; d_rope <= 64: one on the first 16 lanes

struct bf16_tag {};
struct fp8_tag {};

// four consecutive cached values as they are stored, and widened (fp8: the codes; a token's scale is
// applied to its score and its weight)
template <typename CT> struct Raw4;
template <> struct Raw4<float> {
    float4 v;
    __device__ __forceinline__ void load(const void* base, size_t elem) { v = *reinterpret_cast<const float4*>(static_cast<const float*>(base) + elem); }
    __device__ __forceinline__ void zero() { v = make_float4(0.f, 0.f, 0.f, 0.f); }
    __device__ __forceinline__ float4 get() const { return v; }
};
template <> struct Raw4<bf16_tag> {
    uint2 v;
    __device__ __forceinline__ void load(const void* base, size_t elem) { v = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(base) + elem); }
    __device__ __forceinline__ void zero() { v = make_uint2(0u, 0u); }
    __device__ __forceinline__ float4 get() const
    {
        return make_float4(bf16_bits_to_f32(v.x & 0xFFFFu), __uint_as_float(v.x & 0xFFFF0000u),
                           bf16_bits_to_f32(v.y & 0xFFFFu), __uint_as_float(v.y & 0xFFFF0000u));
    }
};
template <> struct Raw4<fp8_tag> {
    uint32_t v;
    __device__ __forceinline__ void load(const void* base, size_t elem) { v = *reinterpret_cast<const uint32_t*>(static_cast<const uint8_t*>(base) + elem); }
    __device__ __forceinline__ void zero() { v = 0u; }
    __device__ __forceinline__ float4 get() const
    {
        const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8(v, false), hi = __builtin_amdgcn_cvt_pk_f32_fp8(v, true);
        return make_float4(lo[0], lo[1], hi[0], hi[1]);
    }
};

// a + b over the lane halves (32) or over the halves of each 32 lanes (16): lanes of the first half get the
// sum of `a`, lanes of the second the sum of `b`
__device__ __forceinline__ float fold32(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fold16(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// sum over 16 lanes, on all of them (rotations inside the row of 16)
__device__ __forceinline__ float sum16(float v)
{
    v += dpp_move<0x128>(v);   // row_ror:8, 4, 2, 1
    v += dpp_move<0x124>(v);
    v += dpp_move<0x122>(v);
    return v + dpp_move<0x121>(v);
}

__device__ __forceinline__ float dot4(float4 a, float4 b, float s)
{
    return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, fmaf(a.x, b.x, s))));
}

// ROWS: rows of a wavefront's batch (the next batch is on its way while one is used): as many as fit
// beside the queries and the sums of HG heads with two wavefronts per SIMD
// WAVES: 4, or 8 where one workgroup per CU has it to itself
template <typename QT, typename CT, int HG, int ROWS, int PR_WAVES>
__global__ __launch_bounds__(64 * PR_WAVES) void decode_portable_kernel(DecodeParams p)
{
    __shared__ __attribute__((aligned(16))) float o_s[PR_WAVES][HG][PR_MAX_DC];
    __shared__ float m_s[PR_WAVES][HG], l_s[PR_WAVES][HG];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the head groups of one chunk of rows get linear ids 8 apart: same XCD, so all but the first find
    // the rows in its L2
    const int Z = (p.H + HG - 1) / HG;
    const long id = (long)blockIdx.y * gridDim.x + blockIdx.x, rr = id >> 3;
    const long wg = (rr / Z) * 8 + (id & 7);
    if (wg >= (long)p.B * p.num_splits) return;           // padding of the last group of 8, and of the grid
    const int h0 = (int)(rr % Z) * HG, split = (int)(wg % p.num_splits), b = (int)(wg / p.num_splits);
    const int row = p.d_c + p.d_rope;
    const int nh = min(HG, p.H - h0);

    int L = p.seq_lens[b];
    L = max(0, min(L, p.max_pages * p.page_size));
    const long chunk_tok = (long)p.chunk_pages * p.page_size;
    const int j0 = (int)min((long)L, (long)split * chunk_tok);
    const int j1 = (int)min((long)L, j0 + chunk_tok);
    if (j0 >= j1) {  // empty chunk: weight zero in the merge, partial output never read
        if (tid < nh) p.lse_part[part_index(b, h0 + tid, split, p.H, p.num_splits)] = -INFINITY;
        return;
    }

    // this lane's columns: latent 4 lane and 256 + 4 lane, rope 4 lane
    const bool has[3] = {4 * lane < p.d_c, 256 + 4 * lane < p.d_c, 4 * lane < p.d_rope};
    // ---- where a batch's rows lie: lane r < ROWS looks up row r of the batch (-1: past the chunk, or on a
    // page outside the pool)
    auto locate = [&](int jb, long& at, float& scale) {
        at = -1;
        scale = 1.f;
        const int j = jb + lane;
        if (lane < ROWS && j < j1) {
            const int page = p.page_table[(size_t)b * p.max_pages + j / p.page_size];
            if (page >= 0 && page < p.num_pages) {
                at = (long)page * p.page_size + j % p.page_size;
                if constexpr (std::is_same<CT, fp8_tag>::value) scale = p.kv_scale[at];
            }
        }
    };
    struct Batch {
        Raw4<CT> v[ROWS][3];
        unsigned live;             // bit r: row r is there
        float scale;               // lane r: scale of row r (fp8)
    };
    auto fetch = [&](long at, float scale, Batch& x) {
        x.live = (unsigned)__ballot(at >= 0);
        x.scale = scale;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            // a row that is not there is read from the start of the pool and left out of the sums
            const long a = max(0L, (long)(((unsigned long)(unsigned)__builtin_amdgcn_readlane((int)(at >> 32), r) << 32) |
                                          (unsigned)__builtin_amdgcn_readlane((int)at, r)));
            const size_t base = (size_t)a * row + 4 * lane;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                x.v[r][c].zero();
                if (has[c]) x.v[r][c].load(p.kv, base + (c == 0 ? 0 : c == 1 ? 256 : p.d_c));
            }
        }
    };

    long at;
    float sc_at;
    const int jstep = PR_WAVES * ROWS;
    int jb = j0 + wave * ROWS;
    locate(jb, at, sc_at);

    // ---- query rows [q_abs | q_rope], this lane's columns
    float4 q[HG][3];
    int limit[HG];                // first row the head's query token does not see
#pragma unroll
    for (int h = 0; h < HG; ++h) {
        const int hq = h0 + min(h, nh - 1);
        const size_t bh = (size_t)b * p.H + hq;
        limit[h] = h < nh ? visible_rows(p, L, hq) : 0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            Raw4<QT> t;
            t.zero();
            if (has[c]) t.load(c < 2 ? p.q_abs : p.q_rope, c < 2 ? bh * p.d_c + c * 256 + 4 * lane : bh * p.d_rope + 4 * lane);
            q[h][c] = t.get();
        }
    }

    float4 acc[HG][2];
    float m[HG], l[HG];
#pragma unroll
    for (int h = 0; h < HG; ++h) {
        acc[h][0] = acc[h][1] = make_float4(0.f, 0.f, 0.f, 0.f);
        m[h] = -INFINITY;
        l[h] = 0.f;
    }
    const int g = lane >> 4;      // after the exchanges the 16 lanes of group g hold the scores of rows g, g + 4, ..
    constexpr int NK = ROWS / 4;
    static_assert(ROWS % 4 == 0 && ROWS <= 32, "rows of a lane group; bits of live");

    auto consume = [&](const Batch& x, int jb) {
        float s[HG][NK];
        {
            float d[HG][ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const float4 k0 = x.v[r][0].get(), k1 = x.v[r][1].get(), k2 = x.v[r][2].get();
#pragma unroll
                for (int h = 0; h < HG; ++h) d[h][r] = dot4(q[h][2], k2, dot4(q[h][1], k1, dot4(q[h][0], k0, 0.f)));
            }
#pragma unroll
            for (int h = 0; h < HG; ++h)
#pragma unroll
                for (int k = 0; k < NK; ++k)   // group g = 2 (upper half of the lanes) + (odd row of 16)
                    s[h][k] = sum16(fold16(fold32(d[h][4 * k], d[h][4 * k + 2]), fold32(d[h][4 * k + 1], d[h][4 * k + 3])));
        }
        float sck[NK];
#pragma unroll
        for (int k = 0; k < NK; ++k) sck[k] = std::is_same<CT, fp8_tag>::value ? __shfl(x.scale, g + 4 * k) : 1.f;
        float w[HG][NK];
#pragma unroll
        for (int h = 0; h < HG; ++h) {
#pragma unroll
            for (int k = 0; k < NK; ++k) {
                const bool seen = ((x.live >> (g + 4 * k)) & 1u) && jb + g + 4 * k < limit[h];
                s[h][k] = seen ? s[h][k] * sck[k] * p.scale : -INFINITY;
            }
            float tm = s[h][0];
#pragma unroll
            for (int k = 1; k < NK; ++k) tm = fmaxf(tm, s[h][k]);
            tm = fmaxf(tm, __shfl_xor(tm, 16));
            tm = fmaxf(tm, __shfl_xor(tm, 32));
            const float m_new = fmaxf(m[h], tm);
            if (__any(m_new != m[h])) {
                const float a = m_new == -INFINITY ? 1.f : expf(m[h] - m_new);   // exp(-inf) = 0 on the first batch
                l[h] *= a;
#pragma unroll
                for (int c = 0; c < 2; ++c) { acc[h][c].x *= a; acc[h][c].y *= a; acc[h][c].z *= a; acc[h][c].w *= a; }
                m[h] = m_new;
            }
#pragma unroll
            for (int k = 0; k < NK; ++k) {
                const float e = m_new == -INFINITY ? 0.f : expf(s[h][k] - m_new);
                l[h] += e;                       // this lane group's rows; joined at the end
                w[h][k] = e * sck[k];
            }
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            if ((x.live >> r) & 1u) {            // (uniform) what was read for an absent row is not even multiplied by zero
                const float4 v0 = x.v[r][0].get(), v1 = x.v[r][1].get();
#pragma unroll
                for (int h = 0; h < HG; ++h) {
                    const float wr = lane_value(w[h][r >> 2], 16 * (r & 3));
                    acc[h][0].x = fmaf(wr, v0.x, acc[h][0].x); acc[h][0].y = fmaf(wr, v0.y, acc[h][0].y);
                    acc[h][0].z = fmaf(wr, v0.z, acc[h][0].z); acc[h][0].w = fmaf(wr, v0.w, acc[h][0].w);
                    acc[h][1].x = fmaf(wr, v1.x, acc[h][1].x); acc[h][1].y = fmaf(wr, v1.y, acc[h][1].y);
                    acc[h][1].z = fmaf(wr, v1.z, acc[h][1].z); acc[h][1].w = fmaf(wr, v1.w, acc[h][1].w);
                }
            }
        }
    };

    // Whether there is a next batch is asked everywhere but in the four-wavefront form of four heads on fp8 caches, where the question
    // took 2 % more time (100 sequences of 2000 rows, 32 heads, d_c = 256: 542 us without, 554 with) and elsewhere up to 4 % less:
    // that form requests one more whose rows are all absent.
    constexpr bool NO_QUESTION = PR_WAVES == 4 && HG == 4 && std::is_same<CT, fp8_tag>::value;
    if (jb < j1) {
        Batch x0, x1;
        fetch(at, sc_at, x0);
        locate(jb + jstep, at, sc_at);
        while (true) {
            if (NO_QUESTION || jb + jstep < j1) {            // the next batch
                fetch(at, sc_at, x1);
                locate(jb + 2 * jstep, at, sc_at);
            }
            consume(x0, jb);
            jb += jstep;
            if (jb >= j1) break;
            if (NO_QUESTION || jb + jstep < j1) {
                fetch(at, sc_at, x0);
                locate(jb + 2 * jstep, at, sc_at);
            }
            consume(x1, jb);
            jb += jstep;
            if (jb >= j1) break;
        }
    }

    // ---- the wavefronts' softmax states joined: every thread finishes columns of every head
#pragma unroll
    for (int h = 0; h < HG; ++h) {
        float lt = l[h] + __shfl_xor(l[h], 16);
        lt += __shfl_xor(lt, 32);
        if (lane == 0) { m_s[wave][h] = m[h]; l_s[wave][h] = lt; }
        if (has[0]) *reinterpret_cast<float4*>(&o_s[wave][h][4 * lane]) = acc[h][0];
        if (has[1]) *reinterpret_cast<float4*>(&o_s[wave][h][256 + 4 * lane]) = acc[h][1];
    }
    __syncthreads();
    for (int h = wave; h < nh; h += PR_WAVES) {
        float mt = -INFINITY;
#pragma unroll
        for (int w = 0; w < PR_WAVES; ++w) mt = fmaxf(mt, m_s[w][h]);
        float f[PR_WAVES], lt = 0.f;
#pragma unroll
        for (int w = 0; w < PR_WAVES; ++w) {
            f[w] = mt == -INFINITY ? 0.f : expf(m_s[w][h] - mt);
            lt = fmaf(l_s[w][h], f[w], lt);
        }
        const size_t pi = part_index(b, h0 + h, split, p.H, p.num_splits);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (!has[c]) continue;
            const int col = c * 256 + 4 * lane;
            float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < PR_WAVES; ++w) {
                const float4 v = *reinterpret_cast<const float4*>(&o_s[w][h][col]);
                o[0] = fmaf(f[w], v.x, o[0]); o[1] = fmaf(f[w], v.y, o[1]);
                o[2] = fmaf(f[w], v.z, o[2]); o[3] = fmaf(f[w], v.w, o[3]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = lt > 0.f ? o[i] / lt : 0.f;
            if constexpr (std::is_same<QT, bf16_tag>::value) {
                uint2 r;
                r.x = f32_to_bf16_bits(o[0]) | (f32_to_bf16_bits(o[1]) << 16);
                r.y = f32_to_bf16_bits(o[2]) | (f32_to_bf16_bits(o[3]) << 16);
                *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.o_part) + pi * p.d_c + col) = r;
            } else {
                *reinterpret_cast<float4*>(static_cast<float*>(p.o_part) + pi * p.d_c + col) = make_float4(o[0], o[1], o[2], o[3]);
            }
        }
        if (lane == 0) p.lse_part[pi] = lt > 0.f ? mt + logf(lt) : -INFINITY;
    }
}

// ---- split-KV merge: lse = log sum_s e^{lse_s}, o = sum_s e^{lse_s - lse} o_s ----
// General kernel: any number of chunks, any d_c (multiple of 4), both partitions.  One workgroup
// per (head, sequence): the chunk weights are computed once into LDS (up to MG_MAXS chunks; more
// than that are handled MG_MAXS at a time with a running reference), then every thread streams
// its four columns with eight partial rows in flight.
constexpr int MG_MAXS = 1024;

template <bool OUT_BF16>
__global__ __launch_bounds__(128) void merge_kernel(MergeParams p)
{
    __shared__ float w_s[MG_MAXS];
    __shared__ float red_s[2];
    const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    // chunks of (b, h): uniform partition: S adjacent entries; balanced partition: the slots the
    // plan names, one every H entries ([slot, H] / [slot, H, d_c])
    const bool planned = p.plan != nullptr;
    const int S = planned ? p.plan[2 * b + 1] : p.num_splits;
    const size_t first = planned ? (size_t)p.plan[2 * b] * p.H + h : part_index(b, h, 0, p.H, p.num_splits);
    const size_t step = planned ? (size_t)p.H : 1;
    const float* lp = p.lse_part + first;

    auto block_max = [&](float v) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
        __syncthreads();
        if ((tid & 63) == 0) red_s[tid >> 6] = v;
        __syncthreads();
        return fmaxf(red_s[0], red_s[1]);
    };
    auto block_sum = [&](float v) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        __syncthreads();
        if ((tid & 63) == 0) red_s[tid >> 6] = v;
        __syncthreads();
        return red_s[0] + red_s[1];
    };

    // reference = the maximum over all chunks, normaliser = sum of e^{lse_s - max}
    float m = -INFINITY;
    for (int s = tid; s < S; s += 128) m = fmaxf(m, lp[s * step]);
    m = block_max(m);
    float z = 0.f;
    if (m != -INFINITY)
        for (int s = tid; s < S; s += 128) z += expf(lp[s * step] - m);  // exp(-inf) = 0
    z = block_sum(z);
    const float inv = z > 0.f ? 1.f / z : 0.f;

    float4 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < S; s0 += MG_MAXS) {
        const int ns = min(MG_MAXS, S - s0);
        __syncthreads();
        for (int s = tid; s < ns; s += 128) {
            const float ls = lp[(s0 + s) * step];
            w_s[s] = ls == -INFINITY ? 0.f : expf(ls - m) * inv;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {             // columns tid*4 + i*512 (d_c <= 2048 per pass)
            const int c = tid * 4 + i * 512;
            if (c >= p.d_c) break;
            const size_t src = (first + (size_t)s0 * step) * p.d_c + c;   // element index into the partial rows
            for (int s = 0; s < ns; s += 8) {
                float4 v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    v[j] = load_part4<OUT_BF16>(p.o_part, src + (size_t)min(s + j, ns - 1) * step * p.d_c);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    // weight 0 for empty chunks (their rows were never written: discarded by the
                    // select, not multiplied) and past the last chunk
                    const float w = s + j < ns ? w_s[s + j] : 0.f;
                    const bool live = w != 0.f;
                    acc[i].x = fmaf(w, live ? v[j].x : 0.f, acc[i].x); acc[i].y = fmaf(w, live ? v[j].y : 0.f, acc[i].y);
                    acc[i].z = fmaf(w, live ? v[j].z : 0.f, acc[i].z); acc[i].w = fmaf(w, live ? v[j].w : 0.f, acc[i].w);
                }
            }
        }
    }
    const size_t out_base = ((size_t)b * p.H + h) * p.d_c;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = tid * 4 + i * 512;
        if (c >= p.d_c) break;
        if (OUT_BF16) {
            uint2 o;
            o.x = f32_to_bf16_bits(acc[i].x) | (f32_to_bf16_bits(acc[i].y) << 16);
            o.y = f32_to_bf16_bits(acc[i].z) | (f32_to_bf16_bits(acc[i].w) << 16);
            *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.o_lat) + out_base + c) = o;
        } else {
            *reinterpret_cast<float4*>(static_cast<float*>(p.o_lat) + out_base + c) = acc[i];
        }
    }
    if (p.lse && tid == 0) p.lse[(size_t)b * p.H + h] = z > 0.f ? m + logf(z) : -INFINITY;
}

// Streaming variant for d_c a multiple of 256: one wavefront per (sequence, head, block of 256
// columns).  Lane s owns the log-sum-exp of chunk s; every lane streams one float4 per chunk with
// the loads of up to 16 chunks in flight.  PLAN = false: uniform partition.
// PLAN = true: the chunks the balanced partition's plan names for the sequence, any number of
// them, 64 at a time.  MANY: 65 to 256 chunks of the uniform partition, weights by expf (these calls ran on the
// general kernel, which has them so).
template <bool OUT_BF16, bool PLAN, bool MANY>
__global__ __launch_bounds__(256) void merge_wave_kernel(MergeParams p)
{
    const int lane = threadIdx.x & 63;
    const int blocks_per_row = p.d_c / 256;
    const int total = p.B * p.H * blocks_per_row;
    const int wid = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (wid >= total) return;
    const int cb = wid % blocks_per_row;
    const int bh = wid / blocks_per_row;
    const int b = bh / p.H, h = bh % p.H;
    const ChunkSpan c = PLAN ? planned_span(p.plan[2 * b], p.plan[2 * b + 1], p, h)
                             : ChunkSpan{part_index(b, h, 0, p.H, p.num_splits), 1, p.num_splits};
    const int S = c.S;

    // Start streaming the first chunks' partial rows before their weights are known.  Rows of
    // empty chunks were never written: whatever is read there is discarded by a select, not
    // multiplied by zero.
    constexpr int BATCH = 16;
    const size_t stride = c.step * (size_t)p.d_c;
    const size_t base = c.first * p.d_c + cb * 256 + lane * 4;   // element index
    const float ls0 = span_lse(p.lse_part, c, 0, lane);
    float4 v[BATCH];
    // rows past the last chunk re-read it (weight zero); a sequence without chunks reads its first slot's row
    auto row = [&](int s) { return base + (size_t)max(0, min(s, S - 1)) * stride; };
#pragma unroll
    for (int i = 0; i < BATCH; ++i) v[i] = load_part4<OUT_BF16>(p.o_part, row(i));

    const ChunkWeights cw = span_weights<MANY>(p.lse_part, c, ls0, lane);

    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int blk = 0; blk < S; blk += 64) {
        const float wt = chunk_weight<MANY>(cw, blk ? span_lse(p.lse_part, c, blk, lane) : ls0);
        for (int s0 = 0; s0 < min(64, S - blk); s0 += BATCH) {
            if (blk + s0 > 0) {
#pragma unroll
                for (int i = 0; i < BATCH; ++i) v[i] = load_part4<OUT_BF16>(p.o_part, row(blk + s0 + i));
            }
            // sums of 16 chunks, added in order (the fused merge + projection forms the same ones)
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const float ws = lane_value(wt, s0 + i);   // 0 at and past S
                const bool live = ws != 0.f;
                a.x = fmaf(ws, live ? v[i].x : 0.f, a.x); a.y = fmaf(ws, live ? v[i].y : 0.f, a.y);
                a.z = fmaf(ws, live ? v[i].z : 0.f, a.z); a.w = fmaf(ws, live ? v[i].w : 0.f, a.w);
            }
            acc.x += a.x; acc.y += a.y; acc.z += a.z; acc.w += a.w;
        }
    }
    const size_t o = (size_t)bh * p.d_c + cb * 256 + lane * 4;
    if (OUT_BF16) {
        uint2 r;
        r.x = f32_to_bf16_bits(acc.x) | (f32_to_bf16_bits(acc.y) << 16);
        r.y = f32_to_bf16_bits(acc.z) | (f32_to_bf16_bits(acc.w) << 16);
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.o_lat) + o) = r;
    } else {
        *reinterpret_cast<float4*>(static_cast<float*>(p.o_lat) + o) = acc;
    }
    if (p.lse && cb == 0 && lane == 0) p.lse[bh] = cw.z > 0.f ? cw.m + logf(cw.z) : -INFINITY;
}

// ---- page gather (byte exact) ---------------------------------------------
__global__ __launch_bounds__(256) void gather_kernel(const uint32_t* kv, const int32_t* page_table,
                                                     const int32_t* seq_lens, uint32_t* dense,
                                                     int max_len, int row_words, int page_size,
                                                     int num_pages, int max_pages)
{
    const int b = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j >= max_len) return;
    int L = min(seq_lens[b], max_pages * page_size);
    const uint32_t* src = nullptr;
    if (j < L) {
        int page = page_table[(size_t)b * max_pages + j / page_size];
        if (page >= 0 && page < num_pages)
            src = kv + ((size_t)page * page_size + (j % page_size)) * row_words;
    }
    uint32_t* dst = dense + ((size_t)b * max_len + j) * row_words;
    for (int w = lane; w < row_words; w += 64) dst[w] = src ? src[w] : 0u;
}

}  // namespace

// Which form takes a call.  Both kernels hold two workgroups per CU, so their times go in rounds of 512 workgroups,
// whatever the rest; measured on 32 .. 65536 workgroups of 200 rows each, back to back in a graph, us:
//   rows in registers, 2 heads per workgroup: up to 256 workgroups (eight wavefronts each) 15 to 23 by width, up to 512 40
//     (fp32 cache) and 28 (others); 4 heads: up to 256 22 to 28, up to 512 40, 768 63, 1024 73, 1536 107, 2048 137, 4096 268,
//     whatever the width (a row costs a whole wavefront, and is read once per 4 heads); 8 heads leave one wavefront per SIMD
//     and are slower still.  Up to 256 workgroups have a CU each, where four wavefronts left a SIMD to one: 21 to 30 and 26 to 38;
//   16-row tiles in LDS, 8 heads: fp32, d_c = 64 / 256: up to 256 32 / 44, 512 38 / 54, 1024 72 / 102, 2048 139 / 200;
//     fp8 38 / 61, 42 / 67, 83 / 131, 162 / 259: a round costs what the width does (fp32 30 us at d_c = 8, 39 at 128, 70
//     at 384), and 12 us more past 256, the second column of its threads.
// So the tiles take narrow latent rows with many heads and chunks (32 heads, 8 x 4000 fp32 rows, d_c = 64: 49 us
// against 95), and the registers wide rows (d_c = 512: 100 against 109) and whatever does not fill the chip (one
// sequence of 1024 rows, 32 heads, d_c = 64: 11.0 against 14.2).
enum Form { ROWS_2_HEADS, ROWS_4_HEADS, TILES_8_HEADS };

static Form faster_form(const DecodeParams& p, mla_dtype cache)
{
    const long long n = (long long)p.B * p.num_splits, n8 = (n + 7) / 8 * 8;
    const long long w2 = n8 * ((p.H + 1) / 2), w4 = n8 * ((p.H + 3) / 4), w8 = n * ((p.H + 7) / 8);
    const double two = w2 <= 256 ? 17.0 : w2 > 512 ? INFINITY : cache == MLA_F32 ? 40.0 : 28.0;
    const double four = w4 <= 256 ? 24.0 : 33.0 * (double)((w4 - 1) / 512) + ((w4 - 1) % 512 < 256 ? 31.0 : 40.0);
    const double round = (cache == MLA_F32 ? 28.0 + p.d_c / 10.0 : cache == MLA_BF16 ? 30.0 + p.d_c / 9.5 : 33.0 + p.d_c / 8.0) +
                         (p.d_c > 256 ? 12.0 : 0.0);
    const double tiles = w8 <= 256 ? 0.95 * round : round * (double)((w8 + 511) / 512);
    return tiles < two && tiles < four ? TILES_8_HEADS : two < four ? ROWS_2_HEADS : ROWS_4_HEADS;
}

template <typename QT, typename CT>
static hipError_t launch_portable(const DecodeParams& p, int hg, hipStream_t s)
{
    // Up to one workgroup per CU: eight wavefronts, half as many batches in a row for each (step, us, four -> eight: 1 x 1024
    // fp32 rows 20.9 -> 19.3, 3 x 520, d_c = 256, 34.0 -> 28.7, 1 x 4000, 16 heads, 33.1 -> 27.8).  Batches of four rows: of eight, they
    // spill (38 registers) and the last one is mostly rows that are not there (20.9).
    const long long n = ((long long)p.B * p.num_splits + 7) / 8 * 8;
    const long long wgs = n * ((p.H + hg - 1) / hg);
    const long long gx = wgs < (1 << 20) ? wgs : 1 << 20, gy = (wgs + gx - 1) / gx;   // a grid dimension holds 2^32 threads
    if (gy > 65535) return hipErrorInvalidValue;
    const dim3 grid((unsigned)gx, (unsigned)gy);
    const bool alone = wgs <= 256;
    if (hg == 4 && alone)  decode_portable_kernel<QT, CT, 4, 4, 8><<<grid, 512, 0, s>>>(p);
    else if (hg == 4)      decode_portable_kernel<QT, CT, 4, 4, 4><<<grid, 256, 0, s>>>(p);
    else if (alone)        decode_portable_kernel<QT, CT, 2, 4, 8><<<grid, 512, 0, s>>>(p);
    else                   decode_portable_kernel<QT, CT, 2, 8, 4><<<grid, 256, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_decode_portable(const DecodeParams& p, mla_dtype io, mla_dtype cache, hipStream_t s)
{
    const Form form = faster_form(p, cache);
    if (form == TILES_8_HEADS) return launch_decode_tiles(p, io, cache, s);
    const int hg = form == ROWS_2_HEADS ? 2 : 4;
    if (io == MLA_F32 && cache == MLA_F32) return launch_portable<float, float>(p, hg, s);
    if (io == MLA_F32 && cache == MLA_BF16) return launch_portable<float, bf16_tag>(p, hg, s);
    if (io == MLA_F32 && cache == MLA_FP8_E4M3) return launch_portable<float, fp8_tag>(p, hg, s);
    if (io == MLA_BF16 && cache == MLA_BF16) return launch_portable<bf16_tag, bf16_tag>(p, hg, s);
    if (io == MLA_BF16 && cache == MLA_FP8_E4M3) return launch_portable<bf16_tag, fp8_tag>(p, hg, s);
    return hipErrorInvalidValue;
}

hipError_t launch_merge(const MergeParams& p, mla_dtype io, hipStream_t s)
{
    // Uniform partitions of 65 to 256 chunks: the streaming kernel, but for bf16 rows that fill the chip, of which the
    // general one has more in flight (d_c = 256 / 512, us, general -> streaming: 1 x 32 rows of 80 chunks 9.5 -> 8.0 and 10.0 ->
    // 9.4, 8 x 32 of 200 18.1 -> 18.7 and 20.3 -> 22.3, 64 x 32 of 100 20.1 -> 21.0 and 34.9 -> 34.9; fp32 64 x 32 of 100 36.1
    // -> 34.9 and 79.9 -> 79.0).  Up to 256 rows it stays: the fused merge + projection forms the same bits there.
    const bool streams = p.plan || p.num_splits <= 64 || (p.num_splits <= 256 && (io == MLA_F32 || (long long)p.B * p.H <= 256));
    if (p.d_c % 256 == 0 && streams) {
        const int waves = p.B * p.H * (p.d_c / 256);
        dim3 grid((waves + 3) / 4), block(256);
        if (io == MLA_BF16) {
            if (p.plan)                 merge_wave_kernel<true, true, false><<<grid, block, 0, s>>>(p);
            else if (p.num_splits > 64) merge_wave_kernel<true, false, true><<<grid, block, 0, s>>>(p);
            else                        merge_wave_kernel<true, false, false><<<grid, block, 0, s>>>(p);
        } else {
            if (p.plan)                 merge_wave_kernel<false, true, false><<<grid, block, 0, s>>>(p);
            else if (p.num_splits > 64) merge_wave_kernel<false, false, true><<<grid, block, 0, s>>>(p);
            else                        merge_wave_kernel<false, false, false><<<grid, block, 0, s>>>(p);
        }
        return hipGetLastError();
    }
    dim3 grid(p.H, p.B), block(128);
    if (io == MLA_BF16) merge_kernel<true><<<grid, block, 0, s>>>(p);
    else                merge_kernel<false><<<grid, block, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_gather(const void* kv, const int32_t* page_table, const int32_t* seq_lens,
                         void* dense, int B, int max_len, int row_bytes, int page_size,
                         int num_pages, int max_pages, hipStream_t s)
{
    dim3 grid((max_len + 3) / 4, B), block(256);
    gather_kernel<<<grid, block, 0, s>>>(static_cast<const uint32_t*>(kv), page_table, seq_lens,
                                         static_cast<uint32_t*>(dense), max_len, row_bytes / 4,
                                         page_size, num_pages, max_pages);
    return hipGetLastError();
}

}  // namespace mla
