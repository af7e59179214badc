// Kernels of the offline GQA -> MLA conversion other than the matrix product:
// per-group second moments (App. B, App. C), row rotation (Sec. 4.2), balancing
// (Sec. 4.3), the batched Jacobi eigensolver, and the Cholesky step of the block
// power iteration (App. D.2).  All fp64.
#include "convert_internal.h"
#include <algorithm>
#include <mutex>
#include <set>
#include <type_traits>
#include <utility>

namespace mla {
namespace conv {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------------ block reductions
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Sum over the workgroup; every thread gets the result.  red: >= 16 doubles of LDS.
__device__ __forceinline__ double block_sum(double v, double* red) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    v = wave_sum(v);
    __syncthreads();                       // red may still be read from a previous call
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < nw; ++w) t += red[w];
    return t;
}

// ------------------------------------------------------------------ App. B / App. C: second moments
// Component c of group G: pair c / g of the group (M of them), head c % g.
struct Group {
    int G, g, d, M;
    __device__ __forceinline__ int column(int c) const { return (c % g) * d + 2 * (G * M + c / g); }     // real part; imaginary: + 1
};

// grid (groups, pairs of 32-component tiles on and above the diagonal).  Sigma = sum over the tokens of x x^T + y y^T: a
// product 2 n deep on v_mfma_f64_16x16x4_f64 (lane l: component l % 16, token l / 16).  Sixteen wavefronts take four tokens
// each in turn, straight from memory, and their sums meet in LDS in order.  Bound by the loads, 16 bytes of a line per lane:
// 32 groups of 64 components, 4096 tokens: 3160 us on 32 workgroups of scalar multiply-adds, now 340.
constexpr int MW = 16;
__global__ __launch_bounds__(64 * MW) void rope_moments_kernel(const double* __restrict__ K, double* __restrict__ sigma,
                                                               int n, int g, int d, int M) {
    __shared__ double part[MW / 2][16][64];
    const int Mg = M * g, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, kq = lane >> 4;
    int ti = 0, tj = blockIdx.y;                       // row and column of tiles
    for (int row = (Mg + 31) / 32; tj >= row; --row) { tj -= row; ++ti; }
    tj += ti;
    const Group grp{(int)blockIdx.x, g, d, M};
    const long ldk = (long)g * d;
    const double *pa[2], *pb[2];
    bool in_a[2], in_b[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int ca = ti * 32 + u * 16 + li, cb = tj * 32 + u * 16 + li;
        in_a[u] = ca < Mg;
        in_b[u] = cb < Mg;
        pa[u] = K + grp.column(in_a[u] ? ca : 0);
        pb[u] = K + grp.column(in_b[u] ? cb : 0);
    }
    f64x4 acc[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = (f64x4){0.0, 0.0, 0.0, 0.0};
    constexpr int U = 4;                               // steps in flight
    for (int t0 = wave * 4; t0 < n; t0 += 4 * MW * U) {
        double a[U][2][2], b[U][2][2];                 // [step][tile][real, imaginary]
#pragma unroll
        for (int s = 0; s < U; ++s) {
            const int t = t0 + s * 4 * MW + kq;
            const long at = (long)min(t, n - 1) * ldk;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    a[s][u][i] = pa[u][at + i];
                    b[s][u][i] = pb[u][at + i];
                }
        }
#pragma unroll
        for (int s = 0; s < U; ++s) {
            const bool there = t0 + s * 4 * MW + kq < n;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < 2; ++i) {          // (what is not there is a zero on both sides, whatever was read)
                    a[s][u][i] = there && in_a[u] ? a[s][u][i] : 0.0;
                    b[s][u][i] = there && in_b[u] ? b[s][u][i] : 0.0;
                }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < 2; ++v)
                        acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s][u][i], b[s][v][i], acc[u][v], 0, 0, 0);
        }
    }
    auto slot = [&](int w, int u, int v, int r) -> double& { return part[w][(u * 2 + v) * 4 + r][lane]; };
    if (wave >= MW / 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int r = 0; r < 4; ++r) slot(wave - MW / 2, u, v, r) = acc[u][v][r];
    }
    __syncthreads();
    if (wave < MW / 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int r = 0; r < 4; ++r) slot(wave, u, v, r) += acc[u][v][r];
    }
    __syncthreads();
    // wavefront f: element f of the 16 a lane holds
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < MW / 2; ++w) sum += part[w][wave][lane];
    const int r = ti * 32 + (wave >> 3) * 16 + 4 * (wave & 3) + kq, c = tj * 32 + ((wave >> 2) & 1) * 16 + li;
    if (r < Mg && c < Mg) {
        double* out = sigma + (long)blockIdx.x * Mg * Mg;
        const double v = sum / (double)n;
        if (ti != tj || r <= c) out[(long)r * Mg + c] = v;               // (the diagonal tiles: both halves from the upper one)
        if (ti != tj || r < c) out[(long)c * Mg + r] = v;
    }
}

// ------------------------------------------------------------------ Sec. 4.2: rotation of rows, of columns, and back
// Row (column) of component r of group G, real part: the RoPE key first (r < keep at pair G * keep + r), then the NoPE key
// (pair (r - keep) * groups + G).
__device__ __forceinline__ long rotated_row(int G, int r, int keep, int groups) {
    return r < keep ? 2L * (G * keep + r) : 2L * keep * groups + 2L * ((long)(r - keep) * groups + G);
}

// grid (2 * groups, columns in tiles of 64), a wavefront per 16 columns; part 0: real rows, part 1: imaginary ones.
//   forward: out[rotated_row(r)] = sum over c of U[c][r] W[row of c]
//   BACK:    the rows of W are those of the NoPE key (rotated_row - d_rope); out[head i][row of c] = scale times the sum over
//            r >= keep of U[c][r] W[r], for each of the `per` query heads i of c's key head
// On the fp64 matrix instructions: the wavefront's part of W is read once, U from the L1.  Bound by memory; NK: 4 NK
// components at most (16, 32, 64 or 128), so that a small group has few loads, all in flight at once (those past its end
// re-read its last one and become zeros).  us, scalar multiply-adds, one form for 128 components, now: 4096 x 4096, groups of 64:
// 468, 137, 82; 1024 x 4096, groups of 8: 35, 72, 17.
template <bool BACK, int NK>
__global__ __launch_bounds__(256) void rotate_rows_kernel(const double* __restrict__ W, const double* __restrict__ U,
                                                          double* __restrict__ out, int g, int d, int M, int keep, int cols,
                                                          int per, const double* __restrict__ scale) {
    const int part = blockIdx.x & 1, Mg = M * g, groups = d / (2 * M), d_rope = 2 * keep * groups;
    const Group grp{(int)(blockIdx.x >> 1), g, d, M};
    const int lane = threadIdx.x & 63, li = lane & 15, kq = lane >> 4;
    const int col = blockIdx.y * 64 + (threadIdx.x >> 6) * 16 + li;
    const bool live = col < cols;
    const double* Ug = U + (long)grp.G * Mg * Mg;
    const int first = BACK ? keep : 0;                 // of the components that W has rows of
    double w[NK];
#pragma unroll
    for (int s = 0; s < NK; ++s) {
        const int k = 4 * s + kq, there = max(first, min(k, Mg - 1));
        const double x = W[(BACK ? rotated_row(grp.G, there, keep, groups) - d_rope : (long)grp.column(there)) * cols + (long)part * cols + min(col, cols - 1)];
        w[s] = k >= first && k < Mg ? x : 0.0;
    }
    const double f = BACK ? *scale : 1.0;
    for (int m0 = 0; m0 < Mg; m0 += 16) {
        f64x4 acc = (f64x4){0.0, 0.0, 0.0, 0.0};
        double u[NK];
        const int m = m0 + li;
#pragma unroll
        for (int s = 0; s < NK; ++s) {
            const int k = min(4 * s + kq, Mg - 1), c = min(m, Mg - 1);      // (columns past the end are not stored)
            const double x = BACK ? Ug[c * Mg + k] : Ug[k * Mg + c];
            u[s] = 4 * s + kq < Mg ? x : 0.0;
        }
#pragma unroll
        for (int s = 0; s < NK; ++s)
            if (4 * s < Mg) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(u[s], w[s], acc, 0, 0, 0);
        if (!live) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = m0 + 4 * e + kq;
            if (r >= Mg) continue;
            if (BACK) {
                const int head = r % g, row = grp.column(r) - head * d + part;
                for (int i = 0; i < per; ++i) out[((long)(head * per + i) * d + row) * cols + col] = f * acc[e];
            } else {
                out[(rotated_row(grp.G, r, keep, groups) + part) * cols + col] = acc[e];
            }
        }
    }
}

// C[t, NoPE column of (G, r, part)] = sum over c of K[t, column of c + part] U[c][r], r >= keep: the rotated key activations
// without another product with X.  grid (tokens / 16, groups / GS); 16 tokens x GS groups in LDS, a wavefront per group, both parts
// at once; results go back through LDS, so that a row is read and written in runs of 2 GS (M) values.  4096 tokens, 4096
// columns, groups of 64: 230 us, where the product X W^T with the rotated weights takes 2000.
__global__ __launch_bounds__(512) void rotate_columns_kernel(const double* __restrict__ K, const double* __restrict__ U, double* __restrict__ C,
                                                             int ldc, int n, int g, int d, int M, int keep, int GS) {
    extern __shared__ __attribute__((aligned(16))) double buf[];          // [16 tokens][component][group][part], padded
    const int Mg = M * g, groups = d / (2 * M), tid = threadIdx.x, nt = blockDim.x;
    const int t0 = blockIdx.x * 16, G0 = blockIdx.y * GS, ng = min(GS, groups - G0);
    const int pitch = Mg * GS * 2 + 2;
    const long ldk = (long)g * d;
    // component (p, j) of group G0 + q: value 2 (q M + p) + part of a run of 2 ng M values of head j
    const int run = 2 * ng * M;
    for (int idx = tid; idx < 16 * g * run; idx += nt) {
        const int x = idx % run, j = idx / run % g, t = idx / (run * g);
        const int q = x / (2 * M), p = x % (2 * M) / 2;
        buf[t * pitch + ((p * g + j) * GS + q) * 2 + (x & 1)] = t0 + t < n ? K[(t0 + t) * ldk + (long)j * d + 2 * G0 * M + x] : 0.0;
    }
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6, li = lane & 15, kq = lane >> 4;
    constexpr int NR = MOMENT_MAX_MG / 16;
    f64x4 acc[2][NR];
    const double* Ug = U + (long)(G0 + wave) * Mg * Mg;
    if (wave < ng) {
#pragma unroll
        for (int m = 0; m < NR; ++m) acc[0][m] = acc[1][m] = (f64x4){0.0, 0.0, 0.0, 0.0};
        for (int k0 = 0; k0 < Mg; k0 += 4) {
            const int k = k0 + kq;
            const double re = k < Mg ? buf[li * pitch + (k * GS + wave) * 2] : 0.0, im = k < Mg ? buf[li * pitch + (k * GS + wave) * 2 + 1] : 0.0;
#pragma unroll
            for (int m = 0; m < NR; ++m)
                if (16 * m < Mg) {
                    const double u = k < Mg && 16 * m + li < Mg ? Ug[(long)k * Mg + 16 * m + li] : 0.0;
                    acc[0][m] = __builtin_amdgcn_mfma_f64_16x16x4f64(u, re, acc[0][m], 0, 0, 0);
                    acc[1][m] = __builtin_amdgcn_mfma_f64_16x16x4f64(u, im, acc[1][m], 0, 0, 0);
                }
        }
    }
    __syncthreads();
    if (wave < ng) {
#pragma unroll
        for (int m = 0; m < NR; ++m)
            if (16 * m < Mg) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = 16 * m + 4 * e + kq;
                    if (r < Mg) {
                        buf[li * pitch + (r * GS + wave) * 2] = acc[0][m][e];
                        buf[li * pitch + (r * GS + wave) * 2 + 1] = acc[1][m][e];
                    }
                }
            }
    }
    __syncthreads();
    for (int idx = tid; idx < 16 * (Mg - keep) * 2 * ng; idx += nt) {
        const int x = idx % (2 * ng), r = idx / (2 * ng) % (Mg - keep), t = idx / (2 * ng * (Mg - keep));
        if (t0 + t < n) C[(long)(t0 + t) * ldc + 2L * ((long)r * groups + G0) + x] = buf[t * pitch + ((r + keep) * GS) * 2 + x];
    }
}

// The query side of the RoPE key: W_QR[i][a][b] = U_G[c][r] where a is (G, r, part) and b component c of the head's group, else 0
__global__ __launch_bounds__(256) void gather_w_qr_kernel(const double* __restrict__ U, double* __restrict__ W_QR, int g, int h, int d, int M, int keep) {
    const int groups = d / (2 * M), d_rope = 2 * keep * groups, per = h / g, Mg = M * g;
    const long total = (long)h * d_rope * d;
    for (long idx = (long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long)gridDim.x * 256) {
        const int b = (int)(idx % d), a = (int)(idx / d % d_rope), i = (int)(idx / ((long)d * d_rope));
        const int G = a / 2 / keep, r = a / 2 % keep, p = b / 2 - G * M;
        W_QR[idx] = (a & 1) == (b & 1) && p >= 0 && p < M ? U[((long)G * Mg + p * g + i / per) * Mg + r] : 0.0;
    }
}

// ------------------------------------------------------------------ Sec. 4.3: alpha
// One wavefront per token: Euclidean norms of its NoPE-key row and of its value row.
__global__ __launch_bounds__(256) void row_norms_kernel(const double* __restrict__ K, int ldk, int a,
                                                        const double* __restrict__ V, int ldv, int b,
                                                        double* __restrict__ norms, int n) {
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= n) return;
    double sk = 0.0, sv = 0.0;
    for (int c = lane; c < a; c += 64) { const double v = K[(long)t * ldk + c]; sk += v * v; }
    for (int c = lane; c < b; c += 64) { const double v = V[(long)t * ldv + c]; sv += v * v; }
    sk = wave_sum(sk);
    sv = wave_sum(sv);
    if (lane == 0) { norms[t] = sqrt(sk); norms[n + t] = sqrt(sv); }
}

__global__ __launch_bounds__(1024) void alpha_kernel(const double* __restrict__ norms, double* __restrict__ alpha, int n) {
    __shared__ double red[16];
    double sk = 0.0, sv = 0.0;
    for (int t = threadIdx.x; t < n; t += 1024) { sk += norms[t]; sv += norms[n + t]; }
    sk = block_sum(sk, red);
    sv = block_sum(sv, red);
    if (threadIdx.x == 0) *alpha = sk / sv;       // the 1/n of the two means cancels
}

__global__ __launch_bounds__(256) void balance_kernel(const double* K, int ldk, const double* V, int ldv,
                                                      const double* __restrict__ alpha, double* C, int n, int a, int b) {
    const double inv = 1.0 / *alpha;
    const long total = (long)n * (a + b);
    for (long idx = (long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long)gridDim.x * 256) {
        const long t = idx / (a + b);
        const int c = (int)(idx % (a + b));
        C[idx] = c < a ? K[t * ldk + c] * inv : V[t * ldv + (c - a)];
    }
}

// ------------------------------------------------------------------ Jacobi rotations of one workgroup
// A step of the round-robin schedule rotates m/2 disjoint index pairs at once: A <- J^T A J, V <- V J, J being
// the product of the step's plane rotations.  A and V have row pitch ld; an odd m has a bye (index m).  Bound by
// the step's chain: the angles of m/2 threads, a barrier, the rotations, a barrier.  Up to order 64 a thread owns the 2 x 2
// block of A where the rows of one pair meet the columns of another and two rows of V in the latter's columns: it reads them
// while the angles are worked out, and both rotations of a block are applied in registers, rows first.
struct Rotations {
    double2 cs[64];                                    // cosine, sine
};

// Pair k of a step, 0 <= step < mp - 1: (step, mp - 1) or (step + k, step - k) modulo mp - 1; the bye of an odd m is in q.
__device__ __forceinline__ void round_robin_pair(int k, int step, int mp, int& p, int& q) {
    p = step + k;
    q = step - k;
    if (p >= mp - 1) p -= mp - 1;
    if (q < 0) q += mp - 1;
    if (k == 0) q = mp - 1;
}

// 1 / sqrt(x) of a normal x: the instruction's 2^-23 or so, e = 1 - x y^2 taken out to its third power
__device__ __forceinline__ double inv_sqrt(double x) {
    const double y = __builtin_amdgcn_rsq(x), e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// The rotation (cosine, sine) that annihilates apq.  With a = (aqq - app) / 2 and h = |(a, apq)|: cos 2 phi = |a| / h, so
// c = sqrt((1 + |a| / h) / 2) and s = |apq| / (2 h c), signed like a apq: two reciprocal square roots in a chain, where
// t = 1 / (theta + sqrt(theta^2 + 1)), c = 1 / sqrt(t^2 + 1) took two divisions more.  Scaled by the largest entry's exponent,
// so that no square leaves the range.
__device__ __forceinline__ double2 rotation(double app, double aqq, double apq) {
    const int e = -__builtin_amdgcn_frexp_exp(fmax(fmax(fabs(app), fabs(aqq)), fabs(apq)));
    const double x = __builtin_amdgcn_ldexp(app, e), y = __builtin_amdgcn_ldexp(aqq, e), b = __builtin_amdgcn_ldexp(apq, e);
    const bool turns = fabs(apq) > 1e-300 && b * b > 1e-36 * fabs(x * y);
    const double a = 0.5 * (y - x);
    const double r = inv_sqrt(fma(a, a, b * b));
    const double c2 = fma(0.5 * fabs(a), r, 0.5);
    const double rc = inv_sqrt(c2);
    const double s = 0.5 * fabs(b) * r * rc;
    return make_double2(turns ? c2 * rc : 1.0, !turns ? 0.0 : a == 0.0 || (a > 0.0) == (b > 0.0) ? s : -s);
}

// a block's entries after both rotations; `pair`: its rows and columns are the same pair, whose off-diagonal entries the rotation
// was chosen to annihilate: exact zeros
__device__ __forceinline__ void rotate_block(double (&x)[4], double2 r1, double2 r2, bool pair) {
    const double pp = r1.x * x[0] - r1.y * x[2], pq = r1.x * x[1] - r1.y * x[3];      // rows
    const double qp = r1.y * x[0] + r1.x * x[2], qq = r1.y * x[1] + r1.x * x[3];
    const bool zero = pair && r1.y != 0.0;
    x[0] = r2.x * pp - r2.y * pq;                      // columns
    x[1] = zero ? 0.0 : r2.y * pp + r2.x * pq;
    x[2] = zero ? 0.0 : r2.x * qp - r2.y * qq;
    x[3] = r2.y * qp + r2.x * qq;
}

// One step, m <= 64, a thread (k1, k2) for each of the (m/2)^2 blocks (threads past them: k1 = half).  EVEN: no bye.
template <bool EVEN>
__device__ __forceinline__ void jacobi_step(double* A, double* V, int ld, int m, int step, Rotations& R, int tid, int half, int k1, int k2) {
    const int mp = 2 * half;
    const bool own = k1 < half;
    int p1, q1, p2, q2;
    round_robin_pair(own ? k1 : 0, step, mp, p1, q1);
    round_robin_pair(k2, step, mp, p2, q2);
    const bool r = EVEN || q1 < m, t = EVEN || q2 < m;               // (a bye has no second row / column)
    const int i0 = own ? 2 * k1 : 0, i1 = EVEN || i0 + 1 < m ? i0 + 1 : i0;        // rows of V
    double app = 0.0, aqq = 0.0, apq = 0.0;
    if (tid < half) {
        int p, q;
        round_robin_pair(tid, step, mp, p, q);
        if (!EVEN && q >= m) q = p;
        app = A[p * ld + p];
        aqq = A[q * ld + q];
        apq = !EVEN && q == p ? 0.0 : A[p * ld + q];
    }
    double* const a11 = A + p1 * ld + p2;
    double* const a12 = t ? A + p1 * ld + q2 : a11;
    double* const a21 = r ? A + q1 * ld + p2 : a11;
    double* const a22 = r && t ? A + q1 * ld + q2 : a11;
    double* const v = V + p2;
    double* const w = V + (t ? q2 : p2);
    double x[4] = {*a11, *a12, *a21, *a22};
    const double v0 = v[i0 * ld], w0 = w[i0 * ld], v1 = v[i1 * ld], w1 = w[i1 * ld];
    if (tid < half) R.cs[tid] = rotation(app, aqq, apq);
    __syncthreads();
    if (own) {
        const double2 r1 = R.cs[k1], r2 = R.cs[k2];
        if (!EVEN && !t) x[1] = x[3] = 0.0;
        if (!EVEN && !r) x[2] = x[3] = 0.0;
        rotate_block(x, r1, r2, k1 == k2);
        if (r && t) *a22 = x[3];
        if (r) *a21 = x[2];
        if (t) *a12 = x[1];
        *a11 = x[0];
        if (t) {
            v[i0 * ld] = r2.x * v0 - r2.y * w0;
            w[i0 * ld] = r2.y * v0 + r2.x * w0;
            if (EVEN || i1 != i0) {
                v[i1 * ld] = r2.x * v1 - r2.y * w1;
                w[i1 * ld] = r2.y * v1 + r2.x * w1;
            }
        }
    }
    __syncthreads();
}

// One step of any order: the blocks, then the pairs of V, as many to a thread as it takes.
__device__ __forceinline__ void jacobi_step_any(double* A, double* V, int ld, int m, int step, Rotations& R, int tid, int nt) {
    const int mp = m + (m & 1), half = mp / 2;
    if (tid < half) {
        int p, q;
        round_robin_pair(tid, step, mp, p, q);
        R.cs[tid] = q < m ? rotation(A[p * ld + p], A[q * ld + q], A[p * ld + q]) : make_double2(1.0, 0.0);
    }
    __syncthreads();
    for (int idx = tid; idx < half * half; idx += nt) {
        const int k1 = idx / half, k2 = idx % half;
        const double2 r1 = R.cs[k1], r2 = R.cs[k2];
        if (r1.y == 0.0 && r2.y == 0.0) continue;
        int p1, q1, p2, q2;
        round_robin_pair(k1, step, mp, p1, q1);
        round_robin_pair(k2, step, mp, p2, q2);
        const bool r = q1 < m, t = q2 < m;
        double x[4] = {A[p1 * ld + p2], t ? A[p1 * ld + q2] : 0.0, r ? A[q1 * ld + p2] : 0.0, r && t ? A[q1 * ld + q2] : 0.0};
        rotate_block(x, r1, r2, k1 == k2);
        A[p1 * ld + p2] = x[0];
        if (t) A[p1 * ld + q2] = x[1];
        if (r) A[q1 * ld + p2] = x[2];
        if (r && t) A[q1 * ld + q2] = x[3];
    }
    for (int idx = tid; idx < half * m; idx += nt) {
        const int k = idx % half, i = idx / half;
        const double2 c = R.cs[k];
        if (c.y == 0.0) continue;
        int p, q;
        round_robin_pair(k, step, mp, p, q);
        const double vp = V[i * ld + p], vq = V[i * ld + q];
        V[i * ld + p] = c.x * vp - c.y * vq;
        V[i * ld + q] = c.y * vp + c.x * vq;
    }
    __syncthreads();
}

// ------------------------------------------------------------------ batched Jacobi eigensolver, order <= 128
// One workgroup per matrix, a sweep = m - 1 (m even; else m) steps.  Small matrices live in LDS (rows padded by
// one element), larger ones in global memory (the waves of a workgroup share one vector cache, so a barrier
// orders their accesses).  At the end the eigenvalues are ranked in descending order and the columns of V are
// written over A in that order.
struct JacobiLds {
    Rotations rot;
    double diag[128];
    int rank[128];
    double red[16];
};

// SMALL: order <= 64, a thread per 2 x 2 block (EVEN order or not)
template <bool SMALL, bool EVEN>
__global__ __launch_bounds__(1024) void jacobi_kernel(double* A_all, double* evals_all, double* V_all, int* info,
                                                      int m, int max_sweeps, int in_lds) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    JacobiLds& L = *reinterpret_cast<JacobiLds*>(smem);
    double* lds_mat = reinterpret_cast<double*>(smem + ((sizeof(JacobiLds) + 15) & ~size_t(15)));
    const int tid = threadIdx.x, nt = blockDim.x;
    double* Ag = A_all + (long)blockIdx.x * m * m;
    double* Vg = V_all + (long)blockIdx.x * m * m;
    const int ld = in_lds ? m + 1 : m;
    double* A = in_lds ? lds_mat : Ag;
    double* V = in_lds ? lds_mat + (long)m * ld : Vg;

    double tot = 0.0;
    for (int idx = tid; idx < m * m; idx += nt) {
        const double v = Ag[idx];
        const int i = idx / m, j = idx % m;
        if (in_lds) A[i * ld + j] = v;
        V[i * ld + j] = i == j ? 1.0 : 0.0;
        tot += v * v;
    }
    tot = block_sum(tot, L.red);                       // squared Frobenius norm (orthogonal similarity keeps it)
    const double tol2 = 1e-26 * tot;

    const int mp = m + (m & 1), half = mp / 2, k1 = tid / half, k2 = tid % half;
    int used = -1;
    for (int sweep = 0; sweep <= max_sweeps; ++sweep) {
        double off = 0.0;
        for (int idx = tid; idx < m * m; idx += nt)
            if (idx / m != idx % m) { const double v = A[idx / m * ld + idx % m]; off += v * v; }
        off = block_sum(off, L.red);
        if (off <= tol2) { used = sweep > 0 ? sweep : 1; break; }
        if (sweep == max_sweeps) break;
        for (int step = 0; step < mp - 1; ++step) {
            if (SMALL) jacobi_step<EVEN>(A, V, ld, m, step, L.rot, tid, half, k1, k2);
            else       jacobi_step_any(A, V, ld, m, step, L.rot, tid, nt);
        }
    }

    // rank the diagonal in descending order (ties: lower index first)
    __syncthreads();
    for (int i = tid; i < m; i += nt) L.diag[i] = A[i * ld + i];
    __syncthreads();
    for (int i = tid; i < m; i += nt) {
        const double di = L.diag[i];
        int r = 0;
        for (int j = 0; j < m; ++j) { const double dj = L.diag[j]; r += (dj > di) || (dj == di && j < i); }
        L.rank[i] = r;
        evals_all[(long)blockIdx.x * m + r] = di;
    }
    __syncthreads();
    for (int idx = tid; idx < m * m; idx += nt) {
        const int i = idx / m, c = idx % m;
        Ag[(long)i * m + L.rank[c]] = V[i * ld + c];
    }
    if (tid == 0) info[blockIdx.x] = used;
}

// ------------------------------------------------------------------ Jacobi eigensolver, one large matrix
// Block Jacobi over the chip: the indices are cut into blocks of 16; a step of the round-robin schedule over the
// blocks takes disjoint pairs of blocks.  The workgroup of pair P = (I, J) rotates the 32 x 32 matrix A[P, P] in LDS,
// accumulating its rotations in a 32 x 32 orthogonal matrix Z_P: every index of I with every one of J, and in every fourth
// step those inside I and J first (they meet again in the next pairs).  Sweeps that took all 31 rotation steps every time
// converged no sooner on full and graded spectra; on low ranks and multiple eigenvalues a sweep sooner as a rule up to order 200,
// two at most (order 144 of rank 72 15 sweeps / 17, 160 with four eigenvalues 22 / 23), and as often later above (300 with three 25 / 24).
// The tiles' workgroups apply the rotations:
// A[P, Q] <- Z_P^T A[P, Q] Z_Q, V[:, Q] <- V[:, Q] Z_Q, on the fp64 matrix instructions.  Launch order on the stream is the
// only synchronisation.  A sweep of order m is m/16 - 1 such steps and annihilates every pair of indices at least once; single
// rotations spread over the chip took m - 1 launches that each rewrote A and V: order 768, 47 ms for 6 sweeps.
// What bounds it is the chain of rotation steps of a pair, so given a second matrix of scratch (the Rayleigh-Ritz matrix) a
// launch applies a step's rotations, from one matrix to the other, while the next step's pairs work out the
// block they need of its result for themselves.  Order 768, a step: 34 us as two launches with all rotation steps (23 + 11), now
// 13.0, 21.0 with the inner rotations; 16.4 where the whole matrix was read and written.  A sweep
// starts with a norm pair of launches that raises `done` once the off-diagonal part is small; later launches then return at
// once, so the host can enqueue the maximum number of sweeps without reading back.
struct WideState { double tot; int done, sweeps, at; };    // at: sweeps before `done` was raised
constexpr int JB = 16, JP = 2 * JB;                    // block, pair of blocks
constexpr int JB_INNER = 4;                            // steps between rotations inside the blocks
constexpr int JB_NORM_WGS = 64;
// Orders up to it stay with one workgroup each.  Above, given scratch, a block of p columns without iterations, ms with one workgroup /
// here: p = 65 1.68 / 1.06, 96 4.58 / 1.16, 128 11.6 / 1.47; layers whose groups have 128 components (16 of them) 12.0 / 2.1.  One of
// order 64 1.24 / 0.74, but 32 at once 1.36 / 1.27 and 48 0.58 / 0.67.
constexpr int WIDE_MIN = 64;

// (of a batch, matrix blockIdx.y, or blockIdx.x where a workgroup has one)
__global__ __launch_bounds__(256) void jw_init_kernel(double* __restrict__ V, int m, WideState* st) {
    const long total = (long)m * m;
    V += blockIdx.y * total;
    st += blockIdx.y;
    for (long idx = (long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long)gridDim.x * 256)
        V[idx] = (idx / m == idx % m) ? 1.0 : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) { st->tot = 0.0; st->done = 0; st->sweeps = -1; }
}

// Squared norms (off the diagonal, on it) from the blocks on and above the diagonal.  Up to NORM_ONE_WG one workgroup has a matrix;
// else partial ones of a share of the rows, then their sums in order.
constexpr int NORM_ONE_WG = 128;
__device__ __forceinline__ void squared_norms(const double* __restrict__ A, int m, int first, int stride, double& off, double& dia) {
    const int per = blockDim.x / 64, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;     // a row each
    for (int i = first * per + wave; i < m; i += stride * per)
        for (int j = i / JB * JB + lane; j < m; j += 64) {
            const double v = A[(long)i * m + j];
            if (i == j) dia += v * v; else off += j / JB == i / JB ? v * v : 2.0 * (v * v);
        }
}
__device__ __forceinline__ void look_at_norms(double off, double dia, int sweep, WideState* st) {
    if (sweep == 0) st->tot = off + dia;
    if (off <= 1e-26 * st->tot) { st->done = 1; st->sweeps = sweep > 0 ? sweep : 1; st->at = sweep; }
}

__global__ __launch_bounds__(1024) void jw_norm_one_kernel(const double* __restrict__ A, int m, int sweep, WideState* st) {
    __shared__ double red[16];
    st += blockIdx.x;
    if (st->done) return;
    double off = 0.0, dia = 0.0;
    squared_norms(A + (long)blockIdx.x * m * m, m, 0, 1, off, dia);
    off = block_sum(off, red);
    dia = block_sum(dia, red);
    if (threadIdx.x == 0) look_at_norms(off, dia, sweep, st);
}

__global__ __launch_bounds__(256) void jw_partial_norm_kernel(const double* __restrict__ A, int m, double* __restrict__ part, const WideState* st) {
    __shared__ double red[16];
    if (st[blockIdx.y].done) return;
    part += blockIdx.y * 2 * JB_NORM_WGS;
    double off = 0.0, dia = 0.0;
    squared_norms(A + (long)blockIdx.y * m * m, m, blockIdx.x, JB_NORM_WGS, off, dia);
    off = block_sum(off, red);
    dia = block_sum(dia, red);
    if (threadIdx.x == 0) { part[2 * blockIdx.x] = off; part[2 * blockIdx.x + 1] = dia; }
}

__global__ __launch_bounds__(64) void jw_norm_kernel(const double* __restrict__ part, int sweep, WideState* st) {
    static_assert(JB_NORM_WGS == 64, "one lane per partial norm");
    st += blockIdx.x;
    part += blockIdx.x * 2 * JB_NORM_WGS;
    if (st->done) return;
    const double off = wave_sum(part[2 * threadIdx.x]), dia = wave_sum(part[2 * threadIdx.x + 1]);
    if (threadIdx.x == 0) look_at_norms(off, dia, sweep, st);
}

// blocks I < J of pair k of a step: the rotations inside a pair take its indices in their order in the matrix (in the
// schedule's order, orders with multiple eigenvalues took up to a sweep more)
__device__ __forceinline__ void block_pair(int k, int step, int nbp, int& I, int& J) {
    int p, q;
    round_robin_pair(k, step, nbp, p, q);
    I = min(p, q);
    J = max(p, q);
}
// the pair that block b belongs to in a step
__device__ __forceinline__ int pair_of(int b, int step, int nbp) {
    const int d = b >= step ? b - step : b - step + nbp - 1;       // (b, step < nbp - 1)
    return b == nbp - 1 ? 0 : d < nbp / 2 ? d : nbp - 1 - d;
}

// index r of pair (I, J) in the matrix (>= m: not there)
__device__ __forceinline__ int pair_index(int I, int J, int r) { return (r < JB ? I : J) * JB + (r & (JB - 1)); }
// where the symmetric matrix has element (i, j): only its blocks on and above the diagonal are kept up
__device__ __forceinline__ long upper(int i, int j, int m) { return i / JB <= j / JB ? (long)i * m + j : (long)j * m + i; }

// What a step reads and writes.  A to B: the matrix (blocks on and above the diagonal) before and after the rotations; Z, D: rotations and rotated 32 x 32 matrix of
// every pair.  Without D, A is B and a pair's rotated matrix goes straight to its place.
struct WideStep {
    const double* A; double* B; double* V;
    const double* Z; const double* D;                  // of `step`, which is applied (step < 0: nothing is)
    double* Z_next; double* D_next;                    // of `next`, whose pairs are rotated (next < 0: none are)
    int m, nbp, step, next;
    const WideState* st;
};
constexpr int WLD = JP + 1;
struct WideLds { double a[2][JP * WLD], z[JP * WLD]; };

// v_mfma_f64_16x16x4: lane l supplies A[l % 16][l / 16], B[l / 16][l % 16], receives D[4 r + l / 16][l % 16]
__device__ __forceinline__ f64x4 mfma_f64(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

__host__ __device__ __forceinline__ int eights(int n) { return (n + 7) / 8 * 8; }

// element (r, c) of pair (I, J) to its place (what lies below the diagonal blocks isn't kept up)
__device__ __forceinline__ void put_pair(double* B, int m, int I, int J, int r, int c, double v) {
    const int i = pair_index(I, J, r), j = pair_index(I, J, c);
    if (i < m && j < m && (r < JB || c >= JB)) B[(long)i * m + j] = v;
}

// A thread (k1, k2) owns the 2 x 2 block of a where the rows of one rotation meet the columns of another, and two rows of z in the
// latter's columns; it writes to the other buffer of a, so that a rotation step has one barrier.  Every 16 lanes work out the
// step's 16 rotations, a lane each; those of the rows come from another lane.  Order 768 (24 pairs), a rotation step: 1.16 us as two
// phases with the angles between them, 0.74 with both rotations of a block worked out by its thread, now 0.54 (no shorter
// without the branches of rotation(): the dependent fp64 operations and the trips through LDS are what it takes).
__device__ void wide_pair(const WideStep& w, WideLds& L, int k, int tid) {
    int I, J;
    block_pair(k, w.next, w.nbp, I, J);
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lq = lane >> 4;
    double* const a0 = L.a[0];
    if (w.step < 0 || !w.D) {                          // the matrix as it lies there
        const int r = tid >> 4, c = tid & 15, i = I * JB, j = J * JB;
        auto at = [&](int row, int col) { return row < w.m && col < w.m ? w.A[(long)row * w.m + col] : 0.0; };
        const double di = at(i + r, i + c), dj = at(j + r, j + c), v = at(i + r, j + c);      // indices that are not there rotate with nothing
        a0[r * WLD + c] = di;
        a0[(JB + r) * WLD + JB + c] = dj;
        a0[r * WLD + JB + c] = v;
        a0[(JB + c) * WLD + r] = v;
    } else {
        // after the rotations of `step`: the diagonal blocks have been rotated in their pairs; [I, J] is Z_P[:, I]^T A[P, Q] Z_Q[:, J]
        const int P = pair_of(I, w.step, w.nbp), Q = pair_of(J, w.step, w.nbp);
        int PI, PJ, QI, QJ;
        block_pair(P, w.step, w.nbp, PI, PJ);
        block_pair(Q, w.step, w.nbp, QI, QJ);
        const int hp = I == PI ? 0 : JB, hq = J == QI ? 0 : JB;
        const double* const Zp = w.Z + (long)P * JP * JP + hp;
        const double* const Zq = w.Z + (long)Q * JP * JP + hq;
        // wavefront (rows 16 ra of P, columns 16 cb of Q): T = A[ra, cb] Z_Q[cb, J], then its share Z_P[ra, I]^T T of the sum
        const int ra = (wave & 1) * JB, cb = (wave >> 1) * JB;
        double x[4], zq[4], zp[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int i = pair_index(PI, PJ, ra + li), j = pair_index(QI, QJ, cb + 4 * s + lq);
            x[s] = i < w.m && j < w.m ? w.A[upper(i, j, w.m)] : 0.0;
            zq[s] = Zq[(cb + 4 * s + lq) * JP + li];
            zp[s] = Zp[(ra + 4 * s + lq) * JP + li];
        }
        const double di = w.D[(long)P * JP * JP + (hp + (tid >> 4)) * JP + hp + (tid & 15)];
        const double dj = w.D[(long)Q * JP * JP + (hq + (tid >> 4)) * JP + hq + (tid & 15)];
        f64x4 t = {0.0, 0.0, 0.0, 0.0}, sum = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s) t = mfma_f64(x[s], zq[s], t);
#pragma unroll
        for (int s = 0; s < 4; ++s) sum = mfma_f64(zp[s], t[s], sum);     // (a result tile lies in the lanes as the right operand does)
        double* const part = L.a[1];
#pragma unroll
        for (int r = 0; r < 4; ++r) part[wave * 256 + (4 * r + lq) * JB + li] = sum[r];
        __syncthreads();
        const int r = tid >> 4, c = tid & 15;
        const double v = ((part[tid] + part[256 + tid]) + part[512 + tid]) + part[768 + tid];
        a0[r * WLD + c] = di;
        a0[(JB + r) * WLD + JB + c] = dj;
        a0[r * WLD + JB + c] = v;
        a0[(JB + c) * WLD + r] = v;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int idx = tid + 256 * u;
        L.z[idx / JP * WLD + idx % JP] = idx / JP == idx % JP ? 1.0 : 0.0;
    }
    __syncthreads();
    const int k1 = tid >> 4, k2 = tid & 15;
    double* const z0 = L.z + 2 * k1 * WLD;
    double* const z1 = z0 + WLD;
    int cur = 0;
    auto rotate = [&](int p1, int q1, int p2, int q2) {
        const double* x = L.a[cur];
        double* y = L.a[cur ^ 1];
        const double dp = x[p2 * (WLD + 1)], dq = x[q2 * (WLD + 1)], o = x[p2 * WLD + q2];
        double b[4] = {x[p1 * WLD + p2], x[p1 * WLD + q2], x[q1 * WLD + p2], x[q1 * WLD + q2]};
        const double v0 = z0[p2], w0 = z0[q2], v1 = z1[p2], w1 = z1[q2];
        const double2 r2 = rotation(dp, dq, o);
        const double2 r1 = make_double2(__shfl(r2.x, k1), __shfl(r2.y, k1));
        rotate_block(b, r1, r2, k1 == k2);
        y[p1 * WLD + p2] = b[0];
        y[p1 * WLD + q2] = b[1];
        y[q1 * WLD + p2] = b[2];
        y[q1 * WLD + q2] = b[3];
        z0[p2] = r2.x * v0 - r2.y * w0;
        z0[q2] = r2.y * v0 + r2.x * w0;
        z1[p2] = r2.x * v1 - r2.y * w1;
        z1[q2] = r2.y * v1 + r2.x * w1;
        cur ^= 1;
        __syncthreads();
    };
    if (w.next % JB_INNER == 0)
        for (int s = 0; s < JB - 1; ++s) {             // both blocks: rotations 0 .. 7 and 8 .. 15
            int p1, q1, p2, q2;
            round_robin_pair(k1 & 7, s, JB, p1, q1);
            round_robin_pair(k2 & 7, s, JB, p2, q2);
            rotate(p1 + (k1 & 8) * 2, q1 + (k1 & 8) * 2, p2 + (k2 & 8) * 2, q2 + (k2 & 8) * 2);
        }
    for (int s = 0; s < JB; ++s) rotate(k1, JB + ((k1 + s) & 15), k2, JB + ((k2 + s) & 15));
    const double* x = L.a[cur];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int idx = tid + 256 * u, r = idx / JP, c = idx % JP;
        if (w.D_next) w.D_next[(long)k * JP * JP + idx] = x[r * WLD + c];
        else          put_pair(w.B, w.m, I, J, r, c, x[r * WLD + c]);
        w.Z_next[(long)k * JP * JP + idx] = L.z[r * WLD + c];
    }
}

// tile (P, Q), P <= Q, of A, or 32 rows P of V in the columns of Q; a wavefront has one 16 x 16 tile of the result
__device__ void wide_tile(const WideStep& w, WideLds& L, int P, int Q, bool on_v, int tid) {
    double* const t = L.a[0];
    double* const zq = L.a[1];
    double* const zp = L.z;
    int I, J, K, M;
    block_pair(Q, w.step, w.nbp, I, J);
    block_pair(P, w.step, w.nbp, K, M);
    if (!on_v && P == Q) {                             // rotated where the angles were found
        if (w.D)
            for (int idx = tid; idx < JP * JP; idx += 256) put_pair(w.B, w.m, I, J, idx / JP, idx % JP, w.D[(long)P * JP * JP + idx]);
        return;
    }
    double x[4], y[4], z[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int idx = tid + 256 * u;
        y[u] = w.Z[(long)Q * JP * JP + idx];
        if (on_v) {
            const int i = P * JP + idx / JP, j = pair_index(I, J, idx % JP);
            x[u] = i < w.m && j < w.m ? w.V[(long)i * w.m + j] : 0.0;
        } else {                                       // a block of 16 x 16 each, in the order it is stored in
            const int bi = u & 2 ? M : K, bj = u & 1 ? J : I, i = min(bi, bj) * JB + (tid >> 4), j = max(bi, bj) * JB + (tid & 15);
            x[u] = i < w.m && j < w.m ? w.A[(long)i * w.m + j] : 0.0;
            z[u] = w.Z[(long)P * JP * JP + idx];
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int idx = tid + 256 * u, at = idx / JP * WLD + idx % JP;
        zq[at] = y[u];
        if (on_v) t[at] = x[u];
        else {
            const bool turn = (u & 2 ? M : K) > (u & 1 ? J : I);
            const int r = turn ? tid & 15 : tid >> 4, c = turn ? tid >> 4 : tid & 15;
            t[((u & 2) * 8 + r) * WLD + (u & 1) * 16 + c] = x[u];
            zp[at] = z[u];
        }
    }
    __syncthreads();
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lq = lane >> 4;
    const int r0 = (wave >> 1) * 16, c0 = (wave & 1) * 16;
    f64x4 acc = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < JP; k += 4) acc = mfma_f64(t[(r0 + li) * WLD + k + lq], zq[(k + lq) * WLD + c0 + li], acc);
    const int bj = wave & 1 ? J : I;
    int row = P * JP + r0, col = bj * JB;
    if (!on_v) {
        __syncthreads();                               // everybody is done with t: it becomes T Z_Q
#pragma unroll
        for (int r = 0; r < 4; ++r) t[(r0 + 4 * r + lq) * WLD + c0 + li] = acc[r];
        __syncthreads();
        acc = (f64x4){0.0, 0.0, 0.0, 0.0};
        const int bi = wave >> 1 ? M : K;
        // the block, or its transpose where it is kept: the operands change places
        const double* const a = bi < bj ? zp + r0 : t + c0;
        const double* const b = bi < bj ? t + c0 : zp + r0;
#pragma unroll
        for (int k = 0; k < JP; k += 4) acc = mfma_f64(a[(k + lq) * WLD + li], b[(k + lq) * WLD + li], acc);
        row = min(bi, bj) * JB;
        col = max(bi, bj) * JB;
    }
    double* const dst = on_v ? w.V : w.B;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = row + 4 * r + lq, j = col + li;
        if (i < w.m && j < w.m) dst[(long)i * w.m + j] = acc[r];
    }
}

// grid: the pairs of `next`, if there is one, in a multiple of eight; if there is a `step`: its tiles of A on and above the diagonal in a
// multiple of eight, then those of V, rows first, in a multiple of eight: workgroup ids 8 apart run on one XCD, whose L2 has a row
// block of V from the step before.
__global__ __launch_bounds__(256) void wide_step_kernel(WideStep w) {
    __shared__ WideLds L;
    const int z = blockIdx.y, pairs = w.nbp / 2, tid = threadIdx.x;
    if (w.st[z].done) return;
    if (z > 0) {
        const long mat = (long)z * w.m * w.m, each = (long)z * pairs * JP * JP;
        w.A += mat;
        w.B += mat;
        w.V += mat;
        w.Z += each;
        w.Z_next += each;
        if (w.D) w.D += each;
        if (w.D_next) w.D_next += each;
    }
    int at = blockIdx.x;
    if (w.next >= 0) {
        if (at < pairs) wide_pair(w, L, at, tid);
        at -= eights(pairs);
        if (at < 0) return;
    }
    const int upper_tiles = pairs * (pairs + 1) / 2;
    if (at < upper_tiles) {
        int P = (int)((sqrtf(8.0f * at + 1.0f) - 1.0f) * 0.5f);         // tile (Q, P) of the lower triangle, row by row
        while (P * (P + 1) / 2 > at) --P;
        while ((P + 1) * (P + 2) / 2 <= at) ++P;
        wide_tile(w, L, at - P * (P + 1) / 2, P, false, tid);
        return;
    }
    at -= eights(upper_tiles);
    const int rows = eights((w.m + JP - 1) / JP);
    if (at >= 0 && at % rows * JP < w.m) wide_tile(w, L, at % rows, at / rows, true, tid);
}

__global__ __launch_bounds__(1024) void jw_rank_kernel(const double* __restrict__ even, const double* __restrict__ odd, int last, int m,
                                                       double* __restrict__ evals, int* __restrict__ rank, const WideState* st, int* info) {
    __shared__ double diag[EIG_MAX_M];
    st += blockIdx.x;
    evals += (long)blockIdx.x * m;
    rank += (long)blockIdx.x * m;
    info += blockIdx.x;
    const double* A = ((st->done ? st->at : last) & 1 ? odd : even) + (long)blockIdx.x * m * m;     // the matrix after that many sweeps
    for (int i = threadIdx.x; i < m; i += 1024) diag[i] = A[(long)i * m + i];
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += 1024) {
        const double di = diag[i];
        int r = 0;
        for (int j = 0; j < m; ++j) { const double dj = diag[j]; r += (dj > di) || (dj == di && j < i); }
        rank[i] = r;
        evals[r] = di;
    }
    if (threadIdx.x == 0) *info = st->done ? st->sweeps : -1;
}

__global__ __launch_bounds__(256) void jw_permute_kernel(double* __restrict__ A_out, const double* __restrict__ V,
                                                         const int* __restrict__ rank, int m) {
    const long total = (long)m * m;
    A_out += blockIdx.y * total;
    V += blockIdx.y * total;
    rank += (long)blockIdx.y * m;
    for (long idx = (long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long)gridDim.x * 256)
        A_out[(idx / m) * m + rank[idx % m]] = V[idx];
}

// ------------------------------------------------------------------ Cholesky factor and its inverse
constexpr int NB = 64;

// One launch per block column k eliminates it from both halves of [G | I]: tile (i, j) of 64 x 64 with i > k is
//     j > k:  G_ij -= L_ik L_jk^T,      L_ik = G_ik L_kk^{-T}
//     j <= k: B_ij -= L_ik X_kj,        X_kj = L_kk^{-1} B_kj      (B starts as I and lives in X)
// one workgroup each, all products on v_mfma_f64_16x16x4_f64; every workgroup multiplies the L_ik and L_jk or X_kj it
// needs itself (K = 64: 1 us each), so that nothing is written that another one reads and a column is one launch.  The
// workgroup of the next diagonal block goes on to factor and invert it: sixteen columns at a time in one wavefront's
// registers (lane = row), the rest of the block on the matrix cores.  What
// bounds it is that chain, column after column.  As separate kernels (block, panel solve, trailing product; then the
// inverse row by row with two products each) order 768 took 1330 us, then 300 (a column 27.5); with the pivots' reciprocal
// roots refined from the instruction's estimate, the rows of the small inverses side by side and one product for a square
// tile 284 (24.1); with the multipliers through LDS and the inverse beside the pivots 232 (18.8: loads 2.7, products 3, pivots
// 7.5, what is left between them 1.5, the inverse's last row 1.6).  Parts of 16 and columns past the end of the last block are left out: a call of top_eig with 5 columns
// and 5 iterations (eight of these) 345 us as separate kernels, 455 with them, 370 without.
constexpr int CP = 66;                     // row pitch of a block in LDS: 32 lanes that read 16 rows x 2 columns hit 32 units of 8 bytes

// c[t] = rows 16 wave .., columns 16 t .. of P R^T (both 64 x 64, row-major); LOWER: R is zero above its diagonal.
// Lane l holds row 4 r + l / 16, column l % 16 of a 16 x 16 tile in element r.
template <bool LOWER>
__device__ __forceinline__ void block_nt(const double* P, const double* R, int wave, int lane, f64x4 (&c)[4]) {
    const double* a = P + (16 * wave + (lane & 15)) * CP + (lane >> 4);
    const double* b = R + (lane & 15) * CP + (lane >> 4);
#pragma unroll
    for (int t = 0; t < 4; ++t) c[t] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        const double x = a[4 * ks];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (!LOWER || ks < 4 * (t + 1)) c[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, b[16 * t * CP + 4 * ks], c[t], 0, 0, 0);
    }
}

__device__ __forceinline__ void block_put(double* S, int wave, int lane, const f64x4 (&c)[4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) S[(16 * wave + 4 * r + (lane >> 4)) * CP + 16 * t + (lane & 15)] = c[t][r];
}

// 64 x 64 block at (r0, c0) of a p x p matrix; rows and columns past the end are zero
__device__ __forceinline__ void block_get(const double* __restrict__ G, long ld, int r0, int c0, int rows, int cols, int tid, double (&v)[16]) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int r = r0 + (tid >> 6) + 4 * q, c = c0 + (tid & 63);
        v[q] = r < rows && c < cols ? G[(long)r * ld + c] : 0.0;
    }
}
template <bool T>
__device__ __forceinline__ void block_stage(double* S, int tid, const double (&v)[16]) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int r = (tid >> 6) + 4 * q, c = tid & 63;
        S[T ? c * CP + r : r * CP + c] = v[q];
    }
}

__device__ __forceinline__ double read_lane(double v, int lane) {
    const long u = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readlane((int)u, lane), hi = __builtin_amdgcn_readlane((int)(u >> 32), lane);
    return __longlong_as_double((long)hi << 32 | lo);
}

// S (64 x 64, its lower half; nb rows and columns of it, identity below) = L L^T -> V = L^{-1}.  Four wavefronts; pivots not above
// floor_v are replaced by it, counted and marked in *marks (bit: column).  What stands below such a pivot is rounding: L has
// zeros there (here, and in the blocks below, whose kernel reads the marks).  Kept, it is divided by a pivot that may be
// hundreds of times smaller, and from a block that lacks some ten ranks on the factors grew past 1e308.
// Sixteen columns are one wavefront's chain, pivot after pivot (its lanes are the rows): the next column's multiplier by lane
// reads, the others' through LDS, whose products come a pivot later, beside its chain (all by lane reads: 382 cycles a pivot, three
// quarters of them for issuing reads and saving scalar registers; now 268).  Meanwhile the other wavefronts do what the caller
// has left (`beside`: from column 16 on S has to be there behind it, and V zero), then the inverse's rows above.
// WHOLE: nb = 64, known at compile time.
template <bool WHOLE, class Beside>
__device__ __forceinline__ void factor_invert(double* S, double* V, double* dinv, double* col, int nb, double floor_v, int* bad,
                                              unsigned long long* marks, int tid, Beside beside) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, kq = lane >> 4;
    unsigned long long dropped = 0;
    const int nsb = WHOLE ? 4 : (nb + 15) / 16;          // parts of 16 that hold rows: the others are left alone
    // row i of the inverse: X_ii by wavefront 1 (lane = column); X_ij = -X_ii sum_k L_ik X_kj, the sum beside it, the product behind
    // a barrier, by wavefront 2 (j = 0), 3 (1) or 0 (2)
    const int mj = wave == 0 ? 2 : wave == 1 ? 4 : wave - 2;
    f64x4 sum = {0.0, 0.0, 0.0, 0.0};
    auto inverse_row = [&](int i) {
        if (wave == 1 && lane < 16) {
            const double* L = S + 16 * i * (CP + 1);
            double x[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = r == lane ? 1.0 : 0.0;
#pragma unroll
            for (int k = 0; k < 16; ++k) {               // (a row's terms in the order of k, the rows side by side)
                x[k] *= dinv[16 * i + k];
                V[(16 * i + k) * CP + 16 * i + lane] = x[k];
#pragma unroll
                for (int r = k + 1; r < 16; ++r) x[r] -= L[r * CP + k] * x[k];
            }
        }
        if (mj < i) {
            sum = (f64x4){0.0, 0.0, 0.0, 0.0};
            for (int k = mj; k < i; ++k)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    sum = __builtin_amdgcn_mfma_f64_16x16x4f64(S[(16 * i + li) * CP + 16 * k + 4 * ks + kq], V[(16 * k + 4 * ks + kq) * CP + 16 * mj + li], sum, 0, 0, 0);
        }
    };
    auto inverse_row_products = [&](int i) {
        if (mj >= i) return;
        f64x4 c = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)                   // (a result tile lies in the lanes as the right operand does)
            c = __builtin_amdgcn_mfma_f64_16x16x4f64(-V[(16 * i + li) * CP + 16 * i + 4 * ks + kq], sum[ks], c, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) V[(16 * i + 4 * r + kq) * CP + 16 * mj + li] = c[r];
    };
    for (int sb = 0; sb < nsb; ++sb) {
        const int s0 = sb * 16;
        if (wave == 0) {
            double a[16], b[16];
#pragma unroll
            for (int c = 0; c < 16; c += 2) {
                const f64x2 v = *reinterpret_cast<const f64x2*>(S + lane * CP + s0 + c);
                a[c] = v[0];
                a[c + 1] = v[1];
            }
            double* const mine = col + lane;
            const double* const theirs = col + s0;
            auto columns = [&](auto whole) {             // (whole: all 16 rows are there, and nothing asks)
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    if (j > 0) {                         // the column before, of which only column j had its product
#pragma unroll
                        for (int k = j + 1; k < 16; ++k) a[k] -= a[j - 1] * b[k];
                    }
                    if (!decltype(whole)::value && s0 + j >= nb) {       // a row past the end
#pragma unroll
                        for (int k = j + 1; k < 16; ++k) b[k] = 0.0;
                        continue;
                    }
                    double d = read_lane(a[j], s0 + j);
                    if (__builtin_expect(!(d > floor_v), 0)) {
                        asm volatile("");                // (a branch: selects would lie in every pivot's chain)
                        d = floor_v;
                        a[j] = lane == s0 + j ? d : 0.0;
                        dropped |= 1ull << (s0 + j);
                    }
                    a[j] *= inv_sqrt(d);                 // (d is at least 1e-300)
                    if (j < 15) a[j + 1] -= a[j] * read_lane(a[j], s0 + j + 1);
                    if (j < 14) {
                        mine[64 * j] = a[j];
#pragma unroll
                        for (int k = j + 2; k < 16; ++k) b[k] = theirs[64 * j + k];
                    }
                }
            };
            if (WHOLE || s0 + 16 <= nb) columns(std::true_type{});
            else                        columns(std::false_type{});
#pragma unroll
            for (int c = 0; c < 16; c += 2)
                *reinterpret_cast<f64x2*>(S + lane * CP + s0 + c) = (f64x2){lane >= s0 + c ? a[c] : 0.0, lane > s0 + c ? a[c + 1] : 0.0};
            if (lane >= s0 && lane < s0 + 16) dinv[lane] = 1.0 / S[lane * (CP + 1)];
        } else if (sb == 0) {
            beside(wave, lane);
        } else {
            inverse_row(sb - 1);
        }
        __syncthreads();
        // what is left of the block: 16 x 16 tiles (bi, bj), bi >= bj > sb
        const int left = nsb - 1 - sb;
        for (int t = wave; t < left * (left + 1) / 2; t += 4) {
            const int u = t < 1 ? 0 : t < 3 ? 1 : 2, bi = sb + 1 + u, bj = sb + 1 + t - u * (u + 1) / 2;
            f64x4 c;
#pragma unroll
            for (int r = 0; r < 4; ++r) c[r] = S[(16 * bi + 4 * r + kq) * CP + 16 * bj + li];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                c = __builtin_amdgcn_mfma_f64_16x16x4f64(-S[(16 * bi + li) * CP + s0 + 4 * ks + kq], S[(16 * bj + li) * CP + s0 + 4 * ks + kq], c, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) S[(16 * bi + 4 * r + kq) * CP + 16 * bj + li] = c[r];
        }
        if (sb > 0 && wave > 0) inverse_row_products(sb - 1);
        if (sb + 1 < nsb) __syncthreads();
    }
    if (tid == 0) {
        *marks = dropped;
        if (dropped) atomicAdd(bad, __popcll(dropped));
    }
    // (the last row's sums read what the last products have just written)
    __syncthreads();
    inverse_row(nsb - 1);
    __syncthreads();
    inverse_row_products(nsb - 1);
    __syncthreads();
}

// Linv: p rows of 64, the inverse of diagonal block k in rows 64 k ..; marks[k]: its clamped pivots.  k = -1: only the first
// diagonal block, and the floor.
__global__ __launch_bounds__(256) void chol_step_kernel(double* G, double* X, double* Linv, unsigned long long* marks, int p, int k,
                                                        double* floor_at, int* bad) {
    __shared__ __attribute__((aligned(16))) double A[NB * CP], Z[NB * CP], D[NB * CP], dinv[NB], col[16 * NB];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k1 = k + 1, nb = min(NB, p - k1 * NB);
    int i = 0, j = 0;
    double floor_v = k < 0 ? 0.0 : *floor_at;            // (asked for here: in front of the first pivot half a microsecond)
    auto clear = [&](int w, int l) {                     // (by the wavefront that has the least beside it)
        if (w != 1) return;
#pragma unroll 6
        for (int q = 0; q < CP / 2; ++q) *reinterpret_cast<f64x2*>(D + 2 * (64 * q + l)) = (f64x2){0.0, 0.0};
    };
    auto factor = [&](double* S, auto beside) {
        if (nb == NB) factor_invert<true>(S, D, dinv, col, nb, floor_v, bad, marks + k1, tid, beside);
        else          factor_invert<false>(S, D, dinv, col, nb, floor_v, bad, marks + k1, tid, beside);
    };
    if (k < 0) {
        double v[16], mx = 0.0;
        block_get(G, p, 0, 0, p, p, tid, v);
        // floor for the pivots: 1e-13 of the largest diagonal entry (a launch of its own took 4.6 us)
        for (int d = tid; d < p; d += 256) mx = fmax(mx, G[(long)d * p + d]);
        for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
        if (lane == 0) dinv[wave] = mx;
#pragma unroll
        for (int q = 0; q < 16; ++q) {                   // (rows past the end: identity)
            const int r = (tid >> 6) + 4 * q, c = tid & 63;
            A[r * CP + c] = r < nb ? v[q] : r == c ? 1.0 : 0.0;
        }
        __syncthreads();
        floor_v = fmax(fmax(fmax(dinv[0], dinv[1]), fmax(dinv[2], dinv[3])) * 1e-13, 1e-300);
        if (tid == 0) *floor_at = floor_v;
        __syncthreads();                                 // (dinv is the factor's from here on)
        factor(A, clear);
    } else {
        // tile of the lower triangle, row by row from row k + 1
        const int t = (k + 1) * (k + 2) / 2 + (int)blockIdx.x;
        i = (int)((sqrtf(8.0f * t + 1.0f) - 1.0f) * 0.5f);
        while (i * (i + 1) / 2 > t) --i;
        while ((i + 1) * (i + 2) / 2 <= t) ++i;
        j = t - i * (i + 1) / 2;
        const bool in_G = j > k;
        double* C = in_G ? G : X;
        double vd[16], va[16], vz[16];
        const unsigned long long dropped = marks[k];  // (asked for with the blocks: behind the products 0.7 us a column)
        block_get(Linv, NB, k * NB, 0, p, NB, tid, vd);
        block_get(G, p, i * NB, k * NB, p, p, tid, va);
        const bool square = i == j;                   // L_jk is L_ik: the next diagonal block is one of these
        if (square) {
        } else if (in_G) block_get(G, p, j * NB, k * NB, p, p, tid, vz);
        else if (j < k) block_get(X, p, k * NB, j * NB, p, p, tid, vz);
        else {
#pragma unroll
            for (int q = 0; q < 16; ++q) vz[q] = (tid >> 6) + 4 * q == (tid & 63) ? 1.0 : 0.0;
        }
        f64x4 c[4], u[4];
        const int row = i * NB + 16 * wave + (lane >> 4), col0 = j * NB + (lane & 15);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                c[t][r] = j != k && row + 4 * r < p && col0 + 16 * t < p ? C[(long)(row + 4 * r) * p + col0 + 16 * t] : 0.0;
        block_stage<false>(D, tid, vd);
        block_stage<false>(A, tid, va);
        if (square) {
        } else if (in_G) block_stage<false>(Z, tid, vz);
        else block_stage<true>(Z, tid, vz);
        __syncthreads();
        f64x4 l[4];
        block_nt<true>(A, D, wave, lane, l);          // L_ik
        if (!square) block_nt<true>(Z, D, wave, lane, u);   // L_jk, or X_kj transposed
        if (dropped) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (dropped >> (16 * t + (lane & 15)) & 1) {
                    l[t] = (f64x4){0.0, 0.0, 0.0, 0.0};
                    if (!square && in_G) u[t] = (f64x4){0.0, 0.0, 0.0, 0.0};
                }
        }
        __syncthreads();
        block_put(A, wave, lane, l);
        if (!square) block_put(Z, wave, lane, u);
        __syncthreads();
        if (!(i == k1 && j == k1)) {
            block_nt<false>(A, square ? A : Z, wave, lane, u);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                c[t] -= u[t];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (row + 4 * r < p && col0 + 16 * t < p) C[(long)(row + 4 * r) * p + col0 + 16 * t] = c[t][r];
            }
            return;
        }
        // the next diagonal block goes to Z: its first 16 columns, then what is left of its lower half beside the first pivots
        auto tile = [&](int t, f64x4 have) {             // tile (wave, t)
            const double* x = A + (16 * wave + (lane & 15)) * CP + (lane >> 4);
            const double* y = A + (16 * t + (lane & 15)) * CP + (lane >> 4);
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int ks = 0; ks < 16; ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[4 * ks], y[4 * ks], acc, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int rr = 16 * wave + 4 * r + (lane >> 4), cc = 16 * t + (lane & 15);
                Z[rr * CP + cc] = rr < nb ? have[r] - acc[r] : rr == cc ? 1.0 : 0.0;
            }
        };
        tile(0, c[0]);
        __syncthreads();
        factor(Z, [&](int w, int l) {
            clear(w, l);
#pragma unroll
            for (int t = 1; t < 4; ++t)
                if (t <= w) tile(t, c[t]);
        });
    }
    for (int idx = tid; idx < nb * NB; idx += 256) Linv[(long)k1 * NB * NB + idx] = D[(idx >> 6) * CP + (idx & 63)];
}

// X = L^{-1}, its block rows scaled: X_ij = L_ii^{-1} B_ij below the diagonal, L_ii^{-1} on it, zero above
__global__ __launch_bounds__(256) void chol_finish_kernel(double* X, const double* __restrict__ Linv, int p) {
    __shared__ double Z[NB * CP], D[NB * CP];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = blockIdx.y, j = blockIdx.x;
    double v[16];
    if (i > j) {
        double z[16];
        block_get(Linv, NB, i * NB, 0, p, NB, tid, v);
        block_get(X, p, i * NB, j * NB, p, p, tid, z);
        block_stage<false>(D, tid, v);
        block_stage<true>(Z, tid, z);
        __syncthreads();
        f64x4 c[4];
        block_nt<false>(D, Z, wave, lane, c);
        const int row = i * NB + 16 * wave + (lane >> 4), col = j * NB + (lane & 15);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (row + 4 * r < p && col + 16 * t < p) X[(long)(row + 4 * r) * p + col + 16 * t] = c[t][r];
        return;
    }
    if (i == j) block_get(Linv, NB, i * NB, 0, p, NB, tid, v);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int r = i * NB + (tid >> 6) + 4 * q, c = j * NB + (tid & 63);
        if (r < p && c < p) X[(long)r * p + c] = i == j ? v[q] : 0.0;
    }
}

__global__ __launch_bounds__(256) void symmetrise_kernel(double* T, int p) {
    const long total = (long)p * p;
    for (long idx = (long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long)gridDim.x * 256) {
        const int i = (int)(idx / p), j = (int)(idx % p);
        if (i < j) {
            const double v = 0.5 * (T[idx] + T[(long)j * p + i]);
            T[idx] = v;
            T[(long)j * p + i] = v;
        }
    }
}

__global__ void fill_int_kernel(int* dst, int value, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) dst[i] = value;
}

__global__ __launch_bounds__(256) void copy_scaled_kernel(const double* __restrict__ src, long lds_, double* __restrict__ dst, long ldd,
                                                          int rows, int cols, const double* __restrict__ scale, int mode) {
    const double f = mode == 1 ? *scale : (mode == 2 ? 1.0 / *scale : 1.0);
    const long total = (long)rows * cols;
    for (long idx = (long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long)gridDim.x * 256) {
        const long r = idx / cols, c = idx % cols;
        dst[r * ldd + c] = src[r * lds_ + c] * f;
    }
}

__global__ __launch_bounds__(256) void gather_w_uv_kernel(const double* __restrict__ R, double* __restrict__ W_UV,
                                                          int g, int h, int d, int nope, int r) {
    const long total = (long)h * r * d;
    const int per = h / g;
    for (long idx = (long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long)gridDim.x * 256) {
        const int b = (int)(idx % d), rho = (int)((idx / d) % r), i = (int)(idx / ((long)d * r));
        W_UV[idx] = R[((long)nope + (long)(i / per) * d + b) * r + rho];
    }
}

inline int grid_for(long total) {
    const long b = (total + 255) / 256;
    return (int)(b < 1 ? 1 : (b > 65535 ? 65535 : b));
}

}  // namespace

hipError_t allow_dynamic_lds(const void* kernel, int bytes) {
    static std::mutex lock;
    static std::set<std::pair<const void*, int>> done;
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> hold(lock);
    if (done.count({kernel, device})) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) done.insert({kernel, device});
    return e;
}

hipError_t launch_rope_moments(const double* K, double* sigma, int n, int g, int d, int M, hipStream_t s) {
    const int tiles = (M * g + 31) / 32;
    rope_moments_kernel<<<dim3(d / (2 * M), tiles * (tiles + 1) / 2), 64 * MW, 0, s>>>(K, sigma, n, g, d, M);
    return hipGetLastError();
}

template <bool BACK>
static hipError_t rotate_rows(const double* W, const double* U, double* out, int g, int d, int M, int keep, int cols, int per,
                              const double* scale, hipStream_t s) {
    const dim3 grid(2 * (d / (2 * M)), (cols + 63) / 64);
    const auto kernel = M * g <= 16 ? &rotate_rows_kernel<BACK, 4> : M * g <= 32 ? &rotate_rows_kernel<BACK, 8>
                      : M * g <= 64 ? &rotate_rows_kernel<BACK, 16> : &rotate_rows_kernel<BACK, MOMENT_MAX_MG / 4>;
    kernel<<<grid, 256, 0, s>>>(W, U, out, g, d, M, keep, cols, per, scale);
    return hipGetLastError();
}

hipError_t launch_rotate_rows(const double* W, const double* U, double* W_out, int g, int d, int M, int keep, int cols, hipStream_t s) {
    return rotate_rows<false>(W, U, W_out, g, d, M, keep, cols, 1, nullptr, s);
}

hipError_t launch_rotate_back(const double* R, const double* U, double* W_UK, int g, int h, int d, int M, int keep, int cols,
                              const double* alpha, hipStream_t s) {
    return rotate_rows<true>(R, U, W_UK, g, d, M, keep, cols, h / g, alpha, s);
}

hipError_t launch_rotate_columns(const double* K, const double* U, double* C, int ldc, int n, int g, int d, int M, int keep, hipStream_t s) {
    const int groups = d / (2 * M), Mg = M * g;
    if (Mg == keep) return hipSuccess;                 // (nothing is left for the NoPE key)
    int GS = 8;                                        // a wavefront each; 16 tokens of them fit LDS
    while (GS > 1 && (GS / 2 >= groups || 256 * Mg * GS > 128 * 1024)) GS /= 2;
    const size_t bytes = 16 * ((size_t)Mg * GS * 2 + 2) * sizeof(double);
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&rotate_columns_kernel), 132 * 1024);
    if (e != hipSuccess) return e;
    rotate_columns_kernel<<<dim3((n + 15) / 16, (groups + GS - 1) / GS), 64 * std::max(GS, 4), bytes, s>>>(K, U, C, ldc, n, g, d, M, keep, GS);
    return hipGetLastError();
}

hipError_t launch_gather_w_qr(const double* U, double* W_QR, int g, int h, int d, int M, int keep, hipStream_t s) {
    gather_w_qr_kernel<<<grid_for((long)h * keep * (d / M) * d), 256, 0, s>>>(U, W_QR, g, h, d, M, keep);
    return hipGetLastError();
}

hipError_t launch_row_norms(const double* K, int ldk, int a, const double* V, int ldv, int b, double* norms, int n, hipStream_t s) {
    row_norms_kernel<<<(n + 3) / 4, 256, 0, s>>>(K, ldk, a, V, ldv, b, norms, n);
    return hipGetLastError();
}

hipError_t launch_alpha(const double* norms, double* alpha, int n, hipStream_t s) {
    alpha_kernel<<<1, 1024, 0, s>>>(norms, alpha, n);
    return hipGetLastError();
}

hipError_t launch_balance(const double* K, int ldk, const double* V, int ldv, const double* alpha, double* C, int n, int a, int b, hipStream_t s) {
    balance_kernel<<<grid_for((long)n * (a + b)), 256, 0, s>>>(K, ldk, V, ldv, alpha, C, n, a, b);
    return hipGetLastError();
}

// scratch behind the batch of V matrices (order > 128): the pairs' rotations, partial norms, ranks, state
static size_t jacobi_extra_bytes(int m) {
    if (m <= 128) return 256;
    const size_t pairs = ((m + JB - 1) / JB + 1) / 2;
    return pairs * JP * JP * sizeof(double) + 2 * JB_NORM_WGS * sizeof(double) + EIG_MAX_M * sizeof(int) + 256;
}
size_t jacobi_work_bytes(int batch, int m) { return (size_t)batch * m * m * sizeof(double) + jacobi_extra_bytes(m); }

// One matrix with the scratch of jacobi_extra_bytes, or, given enough of the caller's, a batch with two matrices each.
static size_t wide_spare_doubles(int batch, int m) {
    const size_t pairs = ((m + JB - 1) / JB + 1) / 2;
    return (size_t)batch * (4 * pairs * JP * JP + 2 * JB_NORM_WGS + (m + 1) / 2 + (sizeof(WideState) + 7) / 8) + 1;
}

static hipError_t launch_jacobi_wide(double* A, double* evals, double* V, void* extra, int* info, int batch, int m, int max_sweeps,
                                     const JacobiSpare& spare, hipStream_t s) {
    const int nb = (m + JB - 1) / JB, nbp = nb + (nb & 1), pairs = nbp / 2;
    const size_t each = (size_t)batch * pairs * JP * JP;
    const bool two = spare.matrix;
    double* Z = two ? spare.rest : static_cast<double*>(extra);
    double* part = Z + (two ? 4 : 1) * each;
    int* rank = reinterpret_cast<int*>(part + (size_t)batch * 2 * JB_NORM_WGS);
    WideState* st = reinterpret_cast<WideState*>(two ? part + (size_t)batch * (2 * JB_NORM_WGS + (m + 1) / 2)
                                                     : reinterpret_cast<double*>(rank + EIG_MAX_M));
    hipError_t e;
    jw_init_kernel<<<dim3(grid_for((long)m * m), batch), 256, 0, s>>>(V, m, st);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int tiles = eights(pairs * (pairs + 1) / 2) + eights((m + JP - 1) / JP) * pairs, steps = nbp - 1;
    double* const mat[2] = {A, two ? spare.matrix : A};
    double* const Zs[2] = {Z, two ? Z + each : Z};
    double* const Ds[2] = {two ? Z + 2 * each : nullptr, two ? Z + 3 * each : nullptr};
    // (a sweep has an odd number of steps: after `sweep` of them the matrix lies in mat[sweep & 1]; step n is the n-th of all)
    for (int sweep = 0; sweep <= max_sweeps; ++sweep) {
        if (m <= NORM_ONE_WG) jw_norm_one_kernel<<<batch, 1024, 0, s>>>(mat[sweep & 1], m, sweep, st);
        else {
            jw_partial_norm_kernel<<<dim3(JB_NORM_WGS, batch), 256, 0, s>>>(mat[sweep & 1], m, part, st);
            jw_norm_kernel<<<batch, 64, 0, s>>>(part, sweep, st);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (sweep == max_sweeps) break;
        for (int step = 0; step < steps; ++step) {
            const int x = (sweep + step) & 1;          // parity of n
            if (!two || (sweep == 0 && step == 0))
                wide_step_kernel<<<dim3(pairs, batch), 256, 0, s>>>(WideStep{mat[x], mat[x], V, Zs[x], nullptr, Zs[x], Ds[x], m, nbp, -1, step, st});
            const bool last = sweep + 1 == max_sweeps && step + 1 == steps;
            const int next = !two || last ? -1 : step + 1 < steps ? step + 1 : 0;
            wide_step_kernel<<<dim3(tiles + (next < 0 ? 0 : eights(pairs)), batch), 256, 0, s>>>(
                WideStep{mat[x], mat[x ^ 1], V, Zs[x], Ds[x], Zs[x ^ 1], Ds[x ^ 1], m, nbp, step, next, st});
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    jw_rank_kernel<<<batch, 1024, 0, s>>>(mat[0], mat[1], max_sweeps, m, evals, rank, st, info);
    jw_permute_kernel<<<dim3(grid_for((long)m * m), batch), 256, 0, s>>>(A, V, rank, m);
    return hipGetLastError();
}

hipError_t launch_jacobi(double* A, double* evals, double* work, int* info, int batch, int m, int max_sweeps, hipStream_t s, const JacobiSpare& spare) {
    // every sweep enqueued costs its launches even after convergence.  Single rotations over the whole
    // matrix took up to 16 where they converged; sweeps over pairs of blocks take as many or fewer on full, graded and
    // nearly diagonal spectra, but up to 7 more on low ranks and multiple eigenvalues (rank 40 or 100 of 256: 12 and 17 to 20;
    // three eigenvalues 85 times each: 24 or 25).  Orders 65 to 128: 23 at most, of either kind, with single rotations or in pairs of blocks
    const int sweeps = std::min(max_sweeps, 26);
    if (m > WIDE_MIN && spare.matrix && spare.doubles >= wide_spare_doubles(batch, m))
        return launch_jacobi_wide(A, evals, work, nullptr, info, batch, m, sweeps, spare, s);
    if (m > 128) {                                     // large matrices: the whole chip works on one at a time
        void* extra = work + (size_t)batch * m * m;
        for (int b = 0; b < batch; ++b) {
            hipError_t e = launch_jacobi_wide(A + (size_t)b * m * m, evals + (size_t)b * m, work + (size_t)b * m * m,
                                              extra, info + b, 1, m, sweeps, JacobiSpare{}, s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    const size_t head = (sizeof(JacobiLds) + 15) & ~size_t(15);
    const size_t mats = 2 * (size_t)m * (m + 1) * sizeof(double);
    const int in_lds = head + mats <= 128 * 1024;
    const size_t bytes = head + (in_lds ? mats : 0);
    const int half = (m + 1) / 2, threads = std::min(1024, std::max(64, (half * half + 63) / 64 * 64));
    const auto kernel = m > 64 ? &jacobi_kernel<false, false> : m % 2 ? &jacobi_kernel<true, false> : &jacobi_kernel<true, true>;
    hipError_t e0 = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), 128 * 1024);
    if (e0 != hipSuccess) return e0;
    kernel<<<batch, threads, bytes, s>>>(A, evals, work, info, m, max_sweeps, in_lds);
    return hipGetLastError();
}

hipError_t launch_chol_inverse(double* G, double* X, double* tmp, int p, int* bad, hipStream_t s) {
    double* floor_v = tmp;                 // one double
    auto* marks = reinterpret_cast<unsigned long long*>(tmp + 1);      // a word per block column
    double* Linv = tmp + CHOL_HEAD;        // p x 64
    hipError_t e = hipSuccess;
    const int nblk = (p + NB - 1) / NB;
    for (int k = -1; k < nblk - 1 && e == hipSuccess; ++k) {
        const int tiles = k < 0 ? 1 : nblk * (nblk + 1) / 2 - (k + 1) * (k + 2) / 2;
        chol_step_kernel<<<tiles, 256, 0, s>>>(G, X, Linv, marks, p, k, floor_v, bad);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    chol_finish_kernel<<<dim3(nblk, nblk), 256, 0, s>>>(X, Linv, p);
    return hipGetLastError();
}

hipError_t launch_symmetrise(double* T, int p, hipStream_t s) {
    symmetrise_kernel<<<grid_for((long)p * p), 256, 0, s>>>(T, p);
    return hipGetLastError();
}

hipError_t launch_fill_int(int* dst, int value, int count, hipStream_t s) {
    fill_int_kernel<<<(count + 255) / 256, 256, 0, s>>>(dst, value, count);
    return hipGetLastError();
}

hipError_t launch_copy_scaled(const double* src, long lds_, double* dst, long ldd, int rows, int cols, const double* scale, int mode, hipStream_t s) {
    copy_scaled_kernel<<<grid_for((long)rows * cols), 256, 0, s>>>(src, lds_, dst, ldd, rows, cols, scale, mode);
    return hipGetLastError();
}

hipError_t launch_gather_w_uv(const double* R, double* W_UV, int g, int h, int d, int nope, int r, hipStream_t s) {
    gather_w_uv_kernel<<<grid_for((long)h * r * d), 256, 0, s>>>(R, W_UV, g, h, d, nope, r);
    return hipGetLastError();
}

}  // namespace conv
}  // namespace mla
