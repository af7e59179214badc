// Per-head batched projections of the absorbed attention equation (Sec. 3.3):
//   absorb   : q_abs[b,h,:] = q_nope[b,h,:] . W_UK[h]     (K = d_head, N = d_c)
//   out-proj : out[b,h,:]   = o_lat[b,h,:]  . W_UV[h]     (K = d_c,    N = d_head)
// Both are Y[b,h,n] = sum_k X[b,h,k] W[h,k,n]: H independent skinny GEMMs whose
// cost is reading W once.  A workgroup owns NT (64, 32 or 16) output columns of one head
// for up to 16 batch rows; its four wavefronts split k, and inside a wavefront 64 / NT lane
// groups split it further, each lane streaming one column of W (coalesced along n) against
// the batch rows held in LDS; the partial sums are reduced through LDS.  The narrower tiles
// give a small problem (one batch row, 128 output columns) a workgroup per CU.
#include "mla_internal.h"

namespace mla {
namespace {

constexpr int HG_THREADS = 256;
constexpr int HG_BT = 16;     // batch rows per workgroup
constexpr int HG_NT = 64;     // widest tile of output columns per workgroup
constexpr int HG_KC = 512;    // k staged in LDS per pass

template <bool BF16>
__device__ __forceinline__ float ld(const void* p, size_t i)
{
    if (BF16) return bf16_bits_to_f32(static_cast<const uint16_t*>(p)[i]);
    return static_cast<const float*>(p)[i];
}

template <bool BF16, bool Y_F32, int NT>
__global__ __launch_bounds__(HG_THREADS) void head_gemm_kernel(const void* X, const void* W, void* Y,
                                                                int B, int H, int K, int N)
{
    constexpr int KS = 64 / NT;          // k slices inside a wavefront
    constexpr int NSL = 4 * KS;          // k slices in all
    // batch rows of one k adjacent: a 128-bit LDS read fetches four of them (an LDS instruction
    // costs the wavefront ~17 cycles of issue whatever its width), and groups of four rows past
    // the batch are not read at all
    __shared__ __attribute__((aligned(16))) float x_t[HG_KC][HG_BT];
    __shared__ float red_s[NSL][HG_BT][NT];

    const int tid = threadIdx.x, lane = tid & 63, col = lane % NT;
    const int kg = (tid >> 6) * KS + lane / NT;      // this lane's k slice
    const int n = blockIdx.x * NT + col;
    const int h = blockIdx.y;
    const int b0 = blockIdx.z * HG_BT;
    const int nb = min(HG_BT, B - b0);
    const int nb4 = (nb + 3) / 4;      // groups of four batch rows in use

    float acc[HG_BT];
#pragma unroll
    for (int i = 0; i < HG_BT; ++i) acc[i] = 0.f;

    for (int k0 = 0; k0 < K; k0 += HG_KC) {
        const int kc = min(HG_KC, K - k0);
        __syncthreads();
        for (int idx = tid; idx < HG_BT * kc; idx += HG_THREADS) {
            int bb = idx / kc, k = idx % kc;
            x_t[k][bb] = bb < nb ? ld<BF16>(X, ((size_t)(b0 + bb) * H + h) * K + k0 + k) : 0.f;
        }
        __syncthreads();
        if (n < N) {
            const int per = (kc + NSL - 1) / NSL;
            const int kb = kg * per, ke = min(kc, kb + per);
            auto step = [&](int k, float w) {
#pragma unroll
                for (int g4 = 0; g4 < HG_BT / 4; ++g4) {
                    if (g4 < nb4) {
                        const float4 xv = *reinterpret_cast<const float4*>(&x_t[k][g4 * 4]);
                        acc[g4 * 4 + 0] = fmaf(xv.x, w, acc[g4 * 4 + 0]);
                        acc[g4 * 4 + 1] = fmaf(xv.y, w, acc[g4 * 4 + 1]);
                        acc[g4 * 4 + 2] = fmaf(xv.z, w, acc[g4 * 4 + 2]);
                        acc[g4 * 4 + 3] = fmaf(xv.w, w, acc[g4 * 4 + 3]);
                    }
                }
            };
            // eight weight loads in flight per lane: with one at a time the loop runs at the speed
            // of the memory latency (a skinny batch gives the chip few wavefronts to hide it)
            int k = kb;
            for (; k + 8 <= ke; k += 8) {
                float w[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) w[j] = ld<BF16>(W, ((size_t)h * K + k0 + k + j) * N + n);
#pragma unroll
                for (int j = 0; j < 8; ++j) step(k + j, w[j]);
            }
            for (; k < ke; ++k) step(k, ld<BF16>(W, ((size_t)h * K + k0 + k) * N + n));
        }
    }
#pragma unroll
    for (int i = 0; i < HG_BT; ++i) red_s[kg][i][col] = acc[i];
    __syncthreads();
    for (int idx = tid; idx < HG_BT * NT; idx += HG_THREADS) {
        int bb = idx / NT, nn = idx % NT;
        int oc = blockIdx.x * NT + nn;
        if (bb < nb && oc < N) {
            float v = 0.f;
#pragma unroll
            for (int sl = 0; sl < NSL; sl += 4)      // slices of one wavefront group first, as the 64-column tile always did
                v += (red_s[sl][bb][nn] + red_s[sl + 1][bb][nn]) + (red_s[sl + 2][bb][nn] + red_s[sl + 3][bb][nn]);
            size_t o = ((size_t)(b0 + bb) * H + h) * N + oc;
            if (BF16 && !Y_F32) static_cast<uint16_t*>(Y)[o] = (uint16_t)f32_to_bf16_bits(v);
            else                static_cast<float*>(Y)[o] = v;
        }
    }
}

// ---- fp32 io ------------------------------------------------------------------------------
// The same split of the work with four columns per lane: a wavefront reads 64 / (NT / 4) rows of W at once,
// each in 128-bit loads, and a workgroup's whole share of a 512-row pass (32 KB at the launcher's choice of
// NT) is requested before the batch rows are staged, so a call waits for memory once where the kernel above,
// one column and eight loads of 4 bytes per lane, waited four times.  Sums over the rows of a wavefront by
// lane exchanges, over the wavefronts through LDS.  BT: batch rows per workgroup (1, 4 or 16).  For deep products:
// where the line lies is said at the launcher's rule.
// One fp32 row of 32 heads: absorb 128 -> 512 and projection 512 -> 128 (8.4 MB of W each) 6.6 -> 4.3 and
// 8.7 -> 5.3 us.
template <int NT, int BT>
__global__ __launch_bounds__(HG_THREADS) void head_gemm_f32_kernel(const float* X, const float* W, float* Y, int B, int H, int K, int N, bool by_head)
{
    constexpr int CL = NT / 4;             // lanes per row of W
    constexpr int KR = HG_THREADS / CL;    // rows of W the workgroup reads at once
    constexpr int U = 8;                   // loads in flight per lane
    __shared__ __attribute__((aligned(16))) float x_t[HG_KC][BT];
    __shared__ __attribute__((aligned(16))) float red_s[4][BT][NT];
    const int tid = threadIdx.x, cl = tid % CL, kr = tid / CL;
    const int h = by_head ? blockIdx.x : blockIdx.y, n0 = (by_head ? blockIdx.y : blockIdx.x) * NT, b0 = blockIdx.z * BT;
    const int n = n0 + 4 * cl;
    const int nb = min(BT, B - b0);
    const bool live = n < N;               // N is a multiple of 4
    const float* Wh = W + (size_t)h * K * N + n;

    float4 acc[BT];
#pragma unroll
    for (int i = 0; i < BT; ++i) acc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k0 = 0; k0 < K; k0 += HG_KC) {
        const int kc = min(HG_KC, K - k0);
        auto load = [&](int i0, float4 (&w)[U]) {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int k = (i0 + i) * KR + kr;
                w[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (live && k < kc) w[i] = *reinterpret_cast<const float4*>(Wh + (size_t)(k0 + k) * N);
            }
        };
        auto use = [&](int i0, const float4 (&w)[U]) {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int k = min((i0 + i) * KR + kr, kc - 1);      // a row past the pass has w = 0 ...
                const bool in = (i0 + i) * KR + kr < kc;
#pragma unroll
                for (int bb = 0; bb < BT; ++bb) {
                    const float x = in ? x_t[k][bb] : 0.f;          // ... and meets a zero (not what X holds elsewhere)
                    acc[bb].x = fmaf(x, w[i].x, acc[bb].x); acc[bb].y = fmaf(x, w[i].y, acc[bb].y);
                    acc[bb].z = fmaf(x, w[i].z, acc[bb].z); acc[bb].w = fmaf(x, w[i].w, acc[bb].w);
                }
            }
        };
        float4 wa[U], wb[U];
        load(0, wa);
        if (k0) __syncthreads();           // the rows of the pass before are used up
        for (int idx = tid; idx < BT * kc; idx += HG_THREADS) {
            const int bb = idx / kc, k = idx % kc;
            x_t[k][bb] = bb < nb ? X[((size_t)(b0 + bb) * H + h) * K + k0 + k] : 0.f;
        }
        __syncthreads();
        for (int i0 = 0; i0 * KR < kc; i0 += 2 * U) {
            if ((i0 + U) * KR < kc) load(i0 + U, wb);
            use(i0, wa);
            if ((i0 + U) * KR < kc) {
                if ((i0 + 2 * U) * KR < kc) load(i0 + 2 * U, wa);
                use(i0 + U, wb);
            }
        }
    }
#pragma unroll
    for (int bb = 0; bb < BT; ++bb) {
#pragma unroll
        for (int o = CL; o < 64; o <<= 1) {
            acc[bb].x += __shfl_xor(acc[bb].x, o); acc[bb].y += __shfl_xor(acc[bb].y, o);
            acc[bb].z += __shfl_xor(acc[bb].z, o); acc[bb].w += __shfl_xor(acc[bb].w, o);
        }
        if ((tid & 63) < CL) *reinterpret_cast<float4*>(&red_s[tid >> 6][bb][4 * cl]) = acc[bb];
    }
    __syncthreads();
    for (int idx = tid; idx < nb * NT; idx += HG_THREADS) {
        const int bb = idx / NT, c = idx % NT, oc = n0 + c;
        if (oc < N) Y[((size_t)(b0 + bb) * H + h) * N + oc] = (red_s[0][bb][c] + red_s[1][bb][c]) + (red_s[2][bb][c] + red_s[3][bb][c]);
    }
}

template <int NT>
hipError_t launch_f32(const float* X, const float* W, float* Y, int B, int H, int K, int N, hipStream_t s)
{
    const int bt = B == 1 ? 1 : B <= 4 ? 4 : HG_BT;
    // Tiles of half a line of W: the heads vary first, so that those of a head are on one XCD where H is a multiple of 8 and the line
    // comes to one L2 only (1 row, 32 heads, 512 -> 128, W not in L2: 4.8 -> 3.0 us; but 28 heads 2.7 -> 3.4, whole lines 5.0 -> 5.3)
    const bool by_head = NT == 16 && H % 8 == 0;
    const unsigned tiles = (N + NT - 1) / NT, groups = (B + bt - 1) / bt;
    const dim3 grid = by_head ? dim3(H, tiles, groups) : dim3(tiles, H, groups);
    if (bt == 1)      head_gemm_f32_kernel<NT, 1><<<grid, HG_THREADS, 0, s>>>(X, W, Y, B, H, K, N, by_head);
    else if (bt == 4) head_gemm_f32_kernel<NT, 4><<<grid, HG_THREADS, 0, s>>>(X, W, Y, B, H, K, N, by_head);
    else              head_gemm_f32_kernel<NT, HG_BT><<<grid, HG_THREADS, 0, s>>>(X, W, Y, B, H, K, N, by_head);
    return hipGetLastError();
}

// ---- matrix-core variant (bf16) ---------------------------------------------------------
// One workgroup = one head x NT output columns x up to 64 batch rows, a wavefront per 16-row tile and part of the
// column tiles (PARTS: as many as fewer than 64 rows leave wavefronts for).  The whole [K x NT] slab of W[h] is staged in LDS
// once with coalesced 128-bit loads, all of them in flight at once, and shared by the four wavefronts.
// v_mfma_f32_16x16x32_bf16 wants, per lane, eight consecutive k of one column: W is stored k-major, so the B operand is read
// with the transposing LDS load (two 4-row reads per k-step); the A operand (8 consecutive k of one batch row) comes straight
// from global memory, X being tiny.  A row's k-steps are added in order by one wavefront whatever the batch, so that a
// row's bits don't depend on how many rows are beside it; sharing the k-steps of up to 16 rows out over the wavefronts as
// well gave 512 -> 128, 32 heads, 8 rows 2.8 us for 3.1.
// DEPTH: K is DEPTH or DEPTH - 32, so only the last k-step is asked about and no load repeats more than one (127 rows, 28
// heads, 320 -> 512: 12.4 us as part of a class for 257 .. 512, 9.3 now).
// Bound by one round trip to memory (warm or cold W makes no difference).  us, with a branch around each load and one wavefront
// per 16 rows whatever the batch, and now: 32 heads, 128 -> 512: 1 row 3.4, 2.1; 16 rows 3.9, 2.6; 32 rows 4.1, 2.9; 128 rows
// 5.1, 4.5; 512 -> 128: 8 rows 3.4, 3.1; 64 rows 4.6, 4.2.
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
#define LDS_AS __attribute__((address_space(3)))

constexpr int HM_LDS_BYTES = 40 * 1024;

template <int NT, bool Y_F32, int DEPTH, int PARTS>
__global__ __launch_bounds__(256) void head_gemm_mfma_kernel(const uint16_t* X, const uint16_t* W, void* Y,
                                                             int B, int H, int K, int N)
{
    constexpr int RS = NT * 2 + 16;          // LDS row stride in bytes (padded: rows shift banks)
    constexpr int CPR = NT / 8;              // 16-byte chunks per slab row
    __shared__ __attribute__((aligned(16))) unsigned char smem[DEPTH * RS];
    LDS_AS unsigned char* lds = (LDS_AS unsigned char*)smem;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    // consecutive workgroup ids go to different XCDs: keep the column tiles of one head on
    // one XCD (ids that differ by a multiple of H) so they share its L2 lines of W[h]
    const int h = blockIdx.x;
    const int n0 = blockIdx.y * NT;
    const int row0 = (blockIdx.z * 4 + wave / PARTS) * 16;                      // this wavefront's batch rows
    const int brow = row0 + n;                            // batch row of this lane's A operand

    // A operands of every k-step, requested before the slab so both are in flight, without a branch around any of them (with one
    // the compiler waits for each: 256 -> 128, 16 rows, 28 heads 2.7 -> 4.5 us): rows past the batch re-read the last
    // one and are not stored, a k-step past the last re-reads it and is not used
    const bool active = row0 < B;
    const uint16_t* xrow = X + ((size_t)min(brow, B - 1) * H + h) * K + g * 8;
    constexpr int KS = DEPTH / 32;                        // k-steps: KS or KS - 1
    u32x4 areg[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) areg[ks] = *reinterpret_cast<const u32x4*>(xrow + (ks < KS - 1 ? ks * 32 : K - 32));

    // stage W[h][0:K][n0:n0+NT] (pieces past the slab re-read its last one and are not written)
    constexpr int NLD = (DEPTH * CPR + 255) / 256;        // pieces per thread at most
    const uint16_t* Wh = W + ((size_t)h * K) * N + n0;
    u32x4 w[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int c = min(tid + i * 256, K * CPR - 1), r = c / CPR, cc = c % CPR;
        w[i] = *reinterpret_cast<const u32x4*>(Wh + (size_t)r * N + cc * 8);
    }
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int c = tid + i * 256, r = c / CPR, cc = c % CPR;
        if (c < K * CPR) *(LDS_AS u32x4*)(lds + r * RS + cc * 16) = w[i];
    }
    __syncthreads();
    if (!active) return;

    constexpr int TILES = NT / 16 / PARTS;                // column tiles of this wavefront
    const int part = (wave % PARTS) * TILES * 16;         // its first column
    f32x4 acc[TILES];
#pragma unroll
    for (int j = 0; j < TILES; ++j) acc[j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // transposing read: the lane supplies row 8g + (n>>2) (+4), 8 bytes at column 4(n&3)
    const uint32_t tr_off = (uint32_t)((g * 8 + (n >> 2)) * RS + (n & 3) * 8 + part * 2);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        if (ks < KS - 1 || K == DEPTH) {
            const bf16x8 a = __builtin_bit_cast(bf16x8, areg[ks]);
#pragma unroll
            for (int j = 0; j < TILES; ++j) {
                LDS_AS unsigned char* bp = lds + ks * 32 * RS + tr_off + j * 32;
                s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(bp));
                s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(bp + 4 * RS));
                s16x8 bb = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, bb), acc[j], 0, 0, 0);
            }
        }
    }
    // D: lane holds rows 4g..4g+3 (batch) of column n
#pragma unroll
    for (int j = 0; j < TILES; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int bb = row0 + g * 4 + i;
            if (bb < B) {
                const size_t o = ((size_t)bb * H + h) * N + n0 + part + j * 16 + n;
                if (Y_F32) static_cast<float*>(Y)[o] = acc[j][i];
                else       static_cast<uint16_t*>(Y)[o] = (uint16_t)f32_to_bf16_bits(acc[j][i]);
            }
        }
}

template <int NT, int DEPTH, int PARTS>
void launch_mfma(const uint16_t* x, const uint16_t* w, void* Y, int B, int H, int K, int N, bool y_f32, hipStream_t s)
{
    dim3 grid(H, N / NT, (B + 63) / 64), block(256);
    if (y_f32) head_gemm_mfma_kernel<NT, true, DEPTH, PARTS><<<grid, block, 0, s>>>(x, w, Y, B, H, K, N);
    else       head_gemm_mfma_kernel<NT, false, DEPTH, PARTS><<<grid, block, 0, s>>>(x, w, Y, B, H, K, N);
}

// the class of depths that K (a multiple of 32) belongs to, and the wavefronts' share of the column tiles
template <int NT, int DEPTH = 64>
void launch_depth(const uint16_t* x, const uint16_t* w, void* Y, int B, int H, int K, int N, bool y_f32, hipStream_t s)
{
    constexpr int MOST = NT / 16;                         // column tiles
    if constexpr (DEPTH <= 512 && DEPTH * (NT * 2 + 16) <= HM_LDS_BYTES) {
        if (K > DEPTH)    launch_depth<NT, DEPTH + 64>(x, w, Y, B, H, K, N, y_f32, s);
        else if (B <= 16) launch_mfma<NT, DEPTH, MOST>(x, w, Y, B, H, K, N, y_f32, s);
        else if (B <= 32) launch_mfma<NT, DEPTH, MOST < 2 ? 1 : 2>(x, w, Y, B, H, K, N, y_f32, s);
        else              launch_mfma<NT, DEPTH, 1>(x, w, Y, B, H, K, N, y_f32, s);
    }
}

template <int NT>
bool try_launch_mfma(const void* X, const void* W, void* Y, int B, int H, int K, int N, bool y_f32,
                     hipStream_t s, hipError_t* err)
{
    if (N % NT || K % 32 || K > 512 || (size_t)K * (NT * 2 + 16) > (size_t)HM_LDS_BYTES) return false;
    const uint16_t* x = static_cast<const uint16_t*>(X);
    const uint16_t* w = static_cast<const uint16_t*>(W);
    launch_depth<NT>(x, w, Y, B, H, K, N, y_f32, s);
    *err = hipGetLastError();
    return true;
}

}  // namespace

hipError_t launch_head_gemm(const void* X, const void* W, void* Y, int B, int H, int K, int N,
                            mla_dtype io, hipStream_t s, bool y_f32)
{
    if (io == MLA_BF16 && (size_t)H * (N / 16 + 1) < 60000) {
        // widest column tile that still gives the chip a workgroup per CU
        const long by = (B + 63) / 64;
        hipError_t err = hipSuccess;
        if (N % 64 == 0 && (long)H * (N / 64) * by >= 256 && try_launch_mfma<64>(X, W, Y, B, H, K, N, y_f32, s, &err)) return err;
        if (N % 32 == 0 && (long)H * (N / 32) * by >= 256 && try_launch_mfma<32>(X, W, Y, B, H, K, N, y_f32, s, &err)) return err;
        if (try_launch_mfma<16>(X, W, Y, B, H, K, N, y_f32, s, &err)) return err;
        if (try_launch_mfma<32>(X, W, Y, B, H, K, N, y_f32, s, &err)) return err;
        if (try_launch_mfma<64>(X, W, Y, B, H, K, N, y_f32, s, &err)) return err;
    }
    // widest column tile that still gives the chip a workgroup per CU
    const long per_col_tile = (long)H * ((B + HG_BT - 1) / HG_BT);
    int nt = HG_NT;
    while (nt > 16 && (long)((N + nt - 1) / nt) * per_col_tile < 256) nt /= 2;
    // fp32, rows of W on 16 bytes: four columns per load, where the sums over a workgroup's lanes (an exchange per batch
    // row and column) are paid for by a deep enough product.  us, one column per lane -> four, back to back in a graph:
    // 1 row, 32 heads, 128 -> 512: 6.1 -> 4.0, 64 -> 512: 4.5 -> 3.9, 16 -> 2048: 6.4 -> 6.7; 4 rows, 128 -> 512: 6.4 -> 5.1,
    // 64 -> 512: 4.7 -> 4.8, 4 heads 4.4 -> 4.6; 3 rows, 128 -> 576 (more than a workgroup per CU): 8 heads 4.6 -> 5.3.
    // 16-row form (its sums take the registers of more than one workgroup per CU): 64 rows, 512 -> 128: 34.4 -> 24.4,
    // 5 rows 11.7 -> 14.0, 8 rows, 1024 -> 64: 19.8 -> 21.1; 64 rows, 128 -> 512: 21.5 -> 36.3; 256 rows, 512 -> 128
    // (1024 workgroups): 74.4 -> 110.
    const bool one_round = (long long)((N + nt - 1) / nt) * per_col_tile <= 256;
    const bool wide = B == 1 ? K >= 64
                    : B <= 4 ? K >= 256 || (K >= 128 && (long long)H * N >= 8192 && one_round)
                             : B >= 12 && K >= HG_KC && (long long)K * B >= HG_KC * HG_BT && one_round;
    if (io == MLA_F32 && wide && N % 4 == 0 && reinterpret_cast<uintptr_t>(W) % 16 == 0) {
        const float *x = static_cast<const float*>(X), *w = static_cast<const float*>(W);
        float* y = static_cast<float*>(Y);
        if (nt == 64) return launch_f32<64>(x, w, y, B, H, K, N, s);
        if (nt == 32) return launch_f32<32>(x, w, y, B, H, K, N, s);
        return launch_f32<16>(x, w, y, B, H, K, N, s);
    }
    dim3 grid((N + nt - 1) / nt, H, (B + HG_BT - 1) / HG_BT), block(HG_THREADS);
#define MLA_HEAD_GEMM(NT_)                                                                                          \
    do {                                                                                                            \
        if (io == MLA_BF16 && y_f32) head_gemm_kernel<true, true, NT_><<<grid, block, 0, s>>>(X, W, Y, B, H, K, N); \
        else if (io == MLA_BF16)     head_gemm_kernel<true, false, NT_><<<grid, block, 0, s>>>(X, W, Y, B, H, K, N); \
        else                         head_gemm_kernel<false, false, NT_><<<grid, block, 0, s>>>(X, W, Y, B, H, K, N); \
    } while (0)
    if (nt == 64) MLA_HEAD_GEMM(64);
    else if (nt == 32) MLA_HEAD_GEMM(32);
    else MLA_HEAD_GEMM(16);
#undef MLA_HEAD_GEMM
    return hipGetLastError();
}

}  // namespace mla
