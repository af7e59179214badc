// fp64 matrix product on the gfx950 matrix cores, used by the offline conversion
// (activations X W^T, second moments C^T C, block power iteration S Q, the low-rank
// projections R^T W and W R of App. D.2).
//
// Workgroup tile 64 x 64, K step 16, four wavefronts in 2 x 2, each 2 x 2 tiles of v_mfma_f64_16x16x4_f64.  Lane l of a
// wavefront supplies A[l % 16][k] and B[k][l % 16], k being the same for the lanes of a group l / 16 on both sides, and
// receives D[4 r + l / 16][l % 16] in element r of the result vector.  It is bound by the matrix pipe (64 cycles an
// instruction), so everything else runs in its shadow: a K step goes from memory straight to the other LDS buffer while this
// one is multiplied, the operands of the next half step are read from LDS a half step ahead, and the one barrier of a step lies
// between its halves, when what a wavefront multiplies on both sides of it is in registers.  Three or four workgroups per CU
// (126 to 143 registers, 32 KB of LDS) fill what is left.
//
// An operand is staged as it lies in memory: k-contiguous as rows of 16 k's, else as 16 rows of consecutive m or n, in
// pieces of 16 bytes swizzled so that the operand reads meet no bank conflict.  Lane group q takes the k's 8 half + 2 q and the
// one after, which suits both.
//
// Given scratch, a product of few tiles has their K steps laid end to end and cut into equal shares, one or two per CU (three
// where the tiles are a little more than two): of a share's sums, a tile's first part lies in the result, a later one
// in the scratch, a whole one is done; a second kernel adds a tile's parts in order.  Tiles of a symmetric product are
// turned over in LDS, so that their mirror images are written in rows as well (scattered, 8 bytes at a time, 16 tokens x
// 2000 columns 16.5 us, now 13.1).
//
// TFLOP/s, the form before (128 x 128, eight wavefronts, through registers, K cut into equal slices of every tile) -> now:
// X W^T 4096^3 60 -> 67 to 69 (a library product reaches 69), 4096 x 4096 x 512 27 -> 60, 1169 x 512 x 512 7 -> 26;
// S Q 8128 x 8128 x 768 61 -> 65 to 67, 3968 x 768 57 -> 65, 1984 x 384 34 -> 49, 512 x 192 3.7 -> 6.3; C^T C of 4096 x
// 8128 (half of it counted) 55 -> 61 to 64, 4096 x 1000 7 -> 23.  Narrow ones are bound by reading S: 8128 x 32 309 -> 168 us.
// Tiles of 128 x 128 with 4 x 4 per wavefront need more than 256 registers (41).
// Registers: 124 of X W^T leave four workgroups per CU, as the 128 that its odd pitches are held to do (three more wait in scratch
// while the K loop runs; 2000 x 333 x 2000 65 -> 53 us); the others have three (C^T C held to four: 4096 x 3000 685 -> 788 us).
#include "convert_internal.h"
#include <algorithm>
#include <type_traits>

namespace mla {
namespace conv {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
#define LDS_AS __attribute__((address_space(3)))

// vmcnt(0), the other counters left alone
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

constexpr int BK = 16;
constexpr int THREADS = 256;
constexpr int BM = 64, T = 2;                 // tile, and 16 x 16 tiles of a wavefront each way

// One operand of a tile of BM rows (or columns) x 16 k's in LDS, and the thread's share of its way there: DIRECT: 16 bytes
// per lane straight to LDS (everything on 16 bytes; offsets inside a tile fit 32 bits), else through registers, element by
// element.  Layouts, in pieces of 16 bytes: k-contiguous: row mn has its 8 pieces at piece ^ (mn >> 1 & 7); else row k has its
// BM / 2 pieces at piece ^ (8 if k & 2).
template <bool K_CONTIG, bool DIRECT>
struct Operand {
    static constexpr int EPT = BM * BK / THREADS;             // elements per thread
    static constexpr int LOADS = EPT / 2;                     // direct loads per thread
    static constexpr int STAGE = BM * BK;
    using Off = std::conditional_t<DIRECT, unsigned, long>;
    Off off[DIRECT ? LOADS : EPT];                            // from the tile's corner (DIRECT: bytes, else elements)

    static __device__ __forceinline__ int at(int mn, int k)
    {
        return K_CONTIG ? mn * BK + (((k >> 1) ^ ((mn >> 1) & 7)) << 1) + (k & 1)
                        : k * BM + (((mn >> 1) ^ ((k & 2) << 2)) << 1) + (mn & 1);
    }
    static __device__ __forceinline__ int k_of(int tid, int i) { return K_CONTIG ? tid & 15 : tid / BM + (THREADS / BM) * i; }
    static __device__ __forceinline__ int mn_of(int tid, int i) { return K_CONTIG ? (tid >> 4) + (THREADS / 16) * i : tid % BM; }
    // there: rows (columns) of the tile inside the matrix; the others re-read the last one (what they give is not stored)
    __device__ __forceinline__ void place(long s_mn, long s_k, int there, int tid, int wave, int lane)
    {
        if constexpr (DIRECT) {
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                const int j = i * 4 + wave;                   // kilobyte of the stage
                if (K_CONTIG) {
                    const int row = 8 * j + (lane >> 3), piece = (lane & 7) ^ ((row >> 1) & 7);
                    off[i] = (unsigned)min(row, there - 1) * (unsigned)s_mn * 8u + piece * 16u;
                } else {
                    const int k = 2 * j + (lane >> 5), piece = (lane & (BM / 2 - 1)) ^ ((k & 2) << 2);
                    off[i] = (unsigned)k * (unsigned)s_k * 8u + (unsigned)min(piece, (there - 1) >> 1) * 16u;
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < EPT; ++i) off[i] = min(mn_of(tid, i), there - 1) * s_mn + k_of(tid, i) * s_k;
        }
    }
    // corner: element (0, first k of the step); S: where the stage lies in LDS
    __device__ __forceinline__ void load(const double* corner, double* S, int wave) const
    {
        const unsigned base = (unsigned)(uintptr_t)(LDS_AS unsigned char*)(S + wave * 128);
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const unsigned m0v = __builtin_amdgcn_readfirstlane(base + i * 4096);
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :: "s"(m0v), "v"(off[i]), "s"(corner) : "memory");
        }
    }
    // left: k's from the corner on (those past the end re-read the first, and become zero)
    __device__ __forceinline__ void fetch(const double* __restrict__ corner, long s_mn, long s_k, int there, int left, int tid, double (&v)[EPT]) const
    {
        if (!DIRECT && left >= BK) {
#pragma unroll
            for (int i = 0; i < EPT; ++i) v[i] = corner[off[i]];
            return;
        }
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int k = k_of(tid, i);
            const double x = corner[min(mn_of(tid, i), there - 1) * s_mn + (k < left ? k : 0) * s_k];
            v[i] = k < left ? x : 0.0;
        }
    }
    static __device__ __forceinline__ void stage(double* S, int tid, const double (&v)[EPT])
    {
#pragma unroll
        for (int i = 0; i < EPT; ++i) S[at(mn_of(tid, i), k_of(tid, i))] = v[i];
    }
    // the lane's k's 8 half + 2 q, + 1 of T rows (columns) 16 apart from mn0 on
    static __device__ __forceinline__ void read(const double* S, int mn0, int half, int li, int kq, double (&v)[T][2])
    {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (K_CONTIG) {
                const f64x2 x = *reinterpret_cast<const f64x2*>(S + mn0 * BK + t * 256 + li * BK + (((half * 4 + kq) ^ (li >> 1)) << 1));
                v[t][0] = x[0];
                v[t][1] = x[1];
            } else {
                const double* row = S + mn0 + (8 * half + 2 * kq) * BM + li + (((t & 1) ^ (kq & 1)) + (t & ~1)) * 16;
                v[t][0] = row[0];
                v[t][1] = row[BM];
            }
        }
    }
};

// How a product is cut: tiles_m x tiles_n tiles (symmetric: those on and above the diagonal) of BM x BM; share: K steps per
// workgroup, 0: a tile per workgroup; cols: columns of a part in the scratch.
struct Cut {
    int tiles_m, tiles_n, tiles, nk, workgroups, cols;
    long share;
};

// first tile of row tm when each row of tiles starts at the diagonal
__host__ __device__ __forceinline__ int row_start(int tm, int tiles_n) { return tm * tiles_n - tm * (tm - 1) / 2; }
// tile number -> row and column of tiles, K steps
struct Tile { int tm, tn, nk; };
__device__ __forceinline__ Tile tile_at(const GemmF64& g, const Cut& c, int tile)
{
    Tile t;
    t.nk = c.nk;
    if (g.symmetric) {
        t.tm = (int)(((2 * c.tiles_n + 1) - sqrtf((2.f * c.tiles_n + 1.f) * (2.f * c.tiles_n + 1.f) - 8.f * tile)) * 0.5f);
        while (t.tm > 0 && tile < row_start(t.tm, c.tiles_n)) --t.tm;           // (the root's rounding)
        while (tile >= row_start(t.tm + 1, c.tiles_n)) ++t.tm;
        t.tn = t.tm + tile - row_start(t.tm, c.tiles_n);
    } else if (g.lower) {                      // deepest columns first: the k's up to a column tile's last column
        t.tm = tile % c.tiles_m;
        t.tn = c.tiles_n - 1 - tile / c.tiles_m;
        t.nk = min(c.nk, ((t.tn + 1) * BM + BK - 1) / BK);
    } else {
        t.tm = tile / c.tiles_n;
        t.tn = tile % c.tiles_n;
    }
    return t;
}

__device__ __forceinline__ double scale_of(const GemmF64& g)
{
    return g.dev_mode == 1 ? g.alpha * *g.alpha_dev : g.dev_mode == 2 ? g.alpha / *g.alpha_dev : g.alpha;
}

// MIRROR: turns tiles over (C C^T has an instantiation of its own: in that of X W^T the code cost small layers 0.5 %)
template <bool A_KC, bool B_KC, bool DIRECT, bool MIRROR>
__global__ __launch_bounds__(THREADS, A_KC && B_KC ? 4 : 3) void gemm_f64_kernel(GemmF64 g, Cut c)
{
    using OpA = Operand<A_KC, DIRECT>;
    using OpB = Operand<B_KC, DIRECT>;
    extern __shared__ __attribute__((aligned(16))) double lds[];          // A, A, B, B
    double* As = lds;
    double* Bs = lds + 2 * OpA::STAGE;

    // consecutive shares (same rows of A) on one XCD: workgroup ids 8 apart run on one XCD.  Whole tiles of unequal depth: dealt out
    const int per = gridDim.x / 8;
    const int w = g.lower ? (int)blockIdx.x : (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (w >= c.workgroups) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) * (16 * T), wn = (wave & 1) * (16 * T);
    const int li = lane & 15, kq = lane >> 4;

    int tile = c.share ? (int)(w * c.share / c.nk) : w;
    long step = c.share ? w * c.share : 0;
    const long end = step + c.share;                     // (past the last tile's end the loop ends by itself)
    for (; tile < c.tiles; ++tile) {
        const Tile at = tile_at(g, c, tile);
        int kt0 = 0, kt1 = at.nk;
        if (c.share) {
            if (step >= end) break;
            const long before = (long)tile * c.nk;
            kt0 = (int)(step - before);
            kt1 = (int)min((long)c.nk, end - before);
            step = before + kt1;
        }
        const int m0 = at.tm * BM, n0 = at.tn * BM;
        OpA a;
        OpB b;
        a.place(g.sAm, g.sAk, g.M - m0, tid, wave, lane);
        b.place(g.sBn, g.sBk, g.N - n0, tid, wave, lane);
        const double* A = g.A + (long)m0 * g.sAm;
        const double* B = g.B + (long)n0 * g.sBn;
        // step kt through registers: requested, then staged
        auto fetch = [&](int kt, double (&ra)[OpA::EPT], double (&rb)[OpB::EPT]) {
            a.fetch(A + (long)kt * BK * g.sAk, g.sAm, g.sAk, g.M - m0, g.K - kt * BK, tid, ra);
            b.fetch(B + (long)kt * BK * g.sBk, g.sBn, g.sBk, g.N - n0, g.K - kt * BK, tid, rb);
        };
        auto stage = [&](int buf, const double (&ra)[OpA::EPT], const double (&rb)[OpB::EPT]) {
            OpA::stage(As + buf * OpA::STAGE, tid, ra);
            OpB::stage(Bs + buf * OpB::STAGE, tid, rb);
        };
        // step kt to a buffer straight from memory (a last step that is not full: through registers)
        auto load = [&](int kt, int buf) {
            if ((kt + 1) * BK <= g.K) {
                a.load(A + (long)kt * BK * g.sAk, As + buf * OpA::STAGE, wave);
                b.load(B + (long)kt * BK * g.sBk, Bs + buf * OpB::STAGE, wave);
            } else {
                double ra[OpA::EPT], rb[OpB::EPT];
                fetch(kt, ra, rb);
                stage(buf, ra, rb);
            }
        };
        f64x4 acc[T][T];
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j) acc[i][j] = (f64x4){0.0, 0.0, 0.0, 0.0};
        double va[2][T][2], vb[2][T][2];
        auto read = [&](int buf, auto half) {
            constexpr int h = decltype(half)::value;
            OpA::read(As + buf * OpA::STAGE, wm, h, li, kq, va[h]);
            OpB::read(Bs + buf * OpB::STAGE, wn, h, li, kq, vb[h]);
        };
        auto multiply = [&](auto half, int s) {
            constexpr int h = decltype(half)::value;
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(va[h][i][s], vb[h][j][s], acc[i][j], 0, 0, 0);
        };
        using H0 = std::integral_constant<int, 0>;
        using H1 = std::integral_constant<int, 1>;

        double ra[OpA::EPT], rb[OpB::EPT];
        if constexpr (DIRECT) {
            load(kt0, 0);
            wait_loads();
        } else {
            fetch(kt0, ra, rb);
            stage(0, ra, rb);
            if (kt0 + 1 < kt1) fetch(kt0 + 1, ra, rb);
        }
        __syncthreads();
        read(0, H0{});
        if (DIRECT && kt0 + 1 < kt1) load(kt0 + 1, 1);
        for (int kt = kt0; kt < kt1; ++kt) {
            const int buf = (kt - kt0) & 1;
            read(buf, H1{});
            __builtin_amdgcn_sched_barrier(0);
            multiply(H0{}, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (!DIRECT && kt + 1 < kt1) {               // requested a step ago
                stage(buf ^ 1, ra, rb);
                if (kt + 2 < kt1) fetch(kt + 2, ra, rb);
                __builtin_amdgcn_sched_barrier(0);
            }
            multiply(H0{}, 1);
            __builtin_amdgcn_sched_barrier(0);
            if (DIRECT) wait_loads();                    // (requested a step ago)
            __syncthreads();                             // the next step is there, and this one has been read
            if (kt + 1 < kt1) read(buf ^ 1, H0{});
            if (DIRECT && kt + 2 < kt1) load(kt + 2, buf);
            __builtin_amdgcn_sched_barrier(0);
            multiply(H1{}, 0);
            multiply(H1{}, 1);
            __builtin_amdgcn_sched_barrier(0);
        }

        // (the lane's place in a tile anew: what follows from it needs no registers during the product)
        int lx = li, ly = kq;
        asm volatile("" : "+v"(lx), "+v"(ly));
        if (kt0 > 0) {                                   // a later part of the tile's sum; gemm_f64_reduce_kernel goes on
            double* part = g.partial + (size_t)w * BM * c.cols;
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j) {
                    const int col = wn + j * 16 + lx;
                    if (col >= c.cols) continue;
#pragma unroll
                    for (int r = 0; r < 4; ++r) part[(wm + i * 16 + 4 * r + ly) * c.cols + col] = acc[i][j][r];
                }
        } else {                                         // the whole sum, or its first part in its place
            const bool whole = kt1 == at.nk, mirror = MIRROR && g.symmetric && at.tm != at.tn && whole;
            const double scale = whole ? scale_of(g) : 1.0;
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = wm + i * 16 + 4 * r + ly, col = wn + j * 16 + lx;
                        const double v = scale * acc[i][j][r];
                        if (m0 + row < g.M && n0 + col < g.N) g.C[(long)(m0 + row) * g.ldc + n0 + col] = v;
                        if (mirror) lds[col * BM + (row ^ (col & 15) << 2)] = v;       // (nobody reads the buffers any more)
                    }
            if (mirror) {                                // the mirror image in rows of its own, too
                __syncthreads();
                for (int col = wave; col < min(BM, g.N - n0); col += 4)
                    if (m0 + lane < g.M) g.C[(long)(n0 + col) * g.ldc + m0 + lane] = lds[col * BM + (lane ^ (col & 15) << 2)];
            }
        }
        if (!c.share) break;
        __syncthreads();                                 // the buffers are free for the next tile
    }
}

// C = scale * the sum of a tile's parts, in order.  grid (tiles, T * T): four 16 x 16 tiles of a wavefront per workgroup
__global__ __launch_bounds__(256) void gemm_f64_reduce_kernel(GemmF64 g, Cut c)
{
    const int tile = blockIdx.x, wave = blockIdx.y & 3, f = (blockIdx.y >> 2) * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    const Tile at = tile_at(g, c, tile);
    const long before = (long)tile * c.nk;
    const int w0 = (int)(before / c.share), w1 = (int)((before + c.nk - 1) / c.share);
    if (w0 == w1) return;                                // one workgroup had the whole tile
    const int in_row = (wave >> 1) * (16 * T) + (f / T) * 16 + (lane >> 4), in_col = (wave & 1) * (16 * T) + (f % T) * 16 + (lane & 15);
    if (in_col >= c.cols) return;
    const int row = at.tm * BM + in_row, col = at.tn * BM + in_col;
    f64x4 sum = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (row + 4 * r < g.M && col < g.N) sum[r] = g.C[(long)(row + 4 * r) * g.ldc + col];
    for (int w = w0 + 1; w <= w1; ++w) {
        const double* part = g.partial + (size_t)w * BM * c.cols + in_row * c.cols + in_col;
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[r] += part[4 * r * c.cols];
    }
    const double scale = scale_of(g);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (row + 4 * r < g.M && col < g.N) {
            g.C[(long)(row + 4 * r) * g.ldc + col] = scale * sum[r];
            if (g.symmetric && at.tm != at.tn) g.C[(long)col * g.ldc + row + 4 * r] = scale * sum[r];
        }
}

template <bool A_KC, bool B_KC, bool DIRECT, bool MIRROR = !A_KC && !B_KC>
hipError_t run(const GemmF64& g, const Cut& c, hipStream_t s)
{
    constexpr size_t lds_bytes = 2 * (Operand<A_KC, DIRECT>::STAGE + Operand<B_KC, DIRECT>::STAGE) * sizeof(double);
    static_assert(lds_bytes <= 64 * 1024, "no raised limit needed");
    gemm_f64_kernel<A_KC, B_KC, DIRECT, MIRROR><<<(c.workgroups + 7) / 8 * 8, THREADS, lds_bytes, s>>>(g, c);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !c.share) return e;
    gemm_f64_reduce_kernel<<<dim3(c.tiles, T * T), 256, 0, s>>>(g, c);
    return hipGetLastError();
}

template <bool DIRECT>
hipError_t run(const GemmF64& g, const Cut& c, hipStream_t s)
{
    const bool a_kc = g.sAk == 1, b_kc = g.sBk == 1;
    if (a_kc && b_kc) return g.symmetric ? run<true, true, DIRECT, true>(g, c, s) : run<true, true, DIRECT, false>(g, c, s);
    if (a_kc) return run<true, false, DIRECT>(g, c, s);
    if (b_kc) return run<false, true, DIRECT>(g, c, s);
    return run<false, false, DIRECT>(g, c, s);
}

}  // namespace

hipError_t launch_gemm_f64(const GemmF64& asked, hipStream_t s)
{
    GemmF64 g = asked;
    if (g.M <= 0 || g.N <= 0 || g.K <= 0) return hipErrorInvalidValue;
    if (g.symmetric && g.M != g.N) return hipErrorInvalidValue;
    if (g.lower && g.symmetric) return hipErrorInvalidValue;
    const bool a_kc = g.sAk == 1, b_kc = g.sBk == 1;
    if ((!a_kc && g.sAm != 1) || (!b_kc && g.sBn != 1)) return hipErrorInvalidValue;
    if (a_kc != b_kc) g.symmetric = 0;
    Cut c{};
    c.tiles_m = (g.M + BM - 1) / BM;
    c.tiles_n = (g.N + BM - 1) / BM;
    c.nk = (g.K + BK - 1) / BK;
    // Half the tiles of a symmetric product, and scattered stores of their mirror images, where the others would take a CU's
    // time.  The bits are the same: an entry and its image sum the same products in the same order.
    if (!g.partial && (long)c.tiles_m * c.tiles_n <= 256) g.symmetric = 0;
    c.tiles = g.symmetric ? row_start(c.tiles_m, c.tiles_n) : c.tiles_m * c.tiles_n;
    c.workgroups = c.tiles;
    c.cols = std::min(g.N, BM);
    if (g.partial && !g.lower && c.nk >= 12) {
        // Shares where whole tiles leave CUs without one, or with one less than others, and the sums are deep enough for the second
        // launch (S Q of order 90, 8 columns, 6 steps 9.2 us, without 7.0; 130 x 130, 9 steps 11.6, 8.8; 152 x 152, 10 steps 10.0, 9.5; 177 x 20,
        // 12 steps 9.6, whole tiles 12.6; 186 x 8 8.9, 10.5; but 192 x 64 9.2, 8.8): one per CU, four steps at least; two
        // from 8192 steps on, where a share is long enough to pay for its ends and the other one fills its waits; three
        // a little above two tiles per CU.  S Q, us at whole tiles, 256, 512 and 768 shares: 1000 x 65 (2016 steps) 51, 20, 26, 26;
        // 2000 x 128 (8000) 77, 29, 30, 32; 4096 x 32 (16384) 154, 45, 42, 45; 8128 x 128 (254 tiles) 376, 372, 287, 285;
        // 2304 x 512 (288) 151, -, 101, 96; 3000 x 512 (376) 196, -, 166, 157; 3000 x 600 (470) 198, -, 210, 209; 4096 x 513
        // (576) 449, -, 389, 355; 8128 x 300 (635) 750, -, 799, 798; 3968 x 768 (744) 366, -, 402, 418.  In between (384, 640) one of
        // three CUs has a share more than the others.
        const long steps = (long)c.tiles * c.nk;
        const long room = (long)(g.partial_doubles / ((size_t)BM * c.cols));
        const bool two = steps >= 8192 && c.tiles <= 400 && room >= 448, three = c.tiles > 512 && c.tiles <= 600 && room >= 768;
        const long shares = std::min({three ? 768L : two ? 512L : 256L, room, steps / 4});
        if (shares > c.tiles) {
            c.share = (steps + shares - 1) / shares;
            c.workgroups = (int)((steps + c.share - 1) / c.share);
        }
    }
    // 16 bytes per load: both operands on 16 bytes, their long strides even (and short enough for 32-bit offsets in a tile)
    auto direct_ok = [](const double* P, long s_long) { return reinterpret_cast<uintptr_t>(P) % 16 == 0 && s_long % 2 == 0 && s_long <= 1L << 22; };
    const bool direct = direct_ok(g.A, a_kc ? g.sAm : g.sAk) && direct_ok(g.B, b_kc ? g.sBn : g.sBk);
    return direct ? run<true>(g, c, s) : run<false>(g, c, s);
}

}  // namespace conv
}  // namespace mla
