// C ABI of the offline GQA -> MLA conversion (include/mla_convert_gfx950.h):
// argument checks on the host, then launches on the caller's stream.
#include "mla_convert_gfx950.h"
#include "convert_internal.h"
#include <algorithm>

using namespace mla::conv;

namespace {

constexpr int JACOBI_MAX_SWEEPS = 60;
// Rayleigh-Ritz matrix of the power iteration above order 128.  After some iterations it is nearly diagonal (4 to 8 sweeps; where
// the moment has few eigenvalues, each many times, up to 16 and beyond).  Every sweep enqueued beyond convergence costs its launches,
// which return at once: 49 at order 768, 0.08 ms.  A matrix that needs more is reported through info (-1).  Up to order 256 two more:
// rotations inside the blocks in every fourth step, not in all, shift the count of moments of two or three eigenvalues by a sweep or two
// either way (34 of 3600, orders 129 to 228, took 17 or 18 where it had been 16 or fewer; none of 1080 of orders 229 to 359).  They
// take 40 us of a layer of 192 columns, 1 %.  Without iterations the
// block is no nearer to the eigenvectors than it was given: low ranks and multiple eigenvalues take 14 to 25 sweeps (order 144 of
// rank 72 17, 256 of rank 100 19), so as many are run as for a matrix of unknown form.
constexpr int ritz_max_sweeps(int p) { return p > 256 ? 16 : 18; }

inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }
inline int st(hipError_t e) { return e == hipSuccess ? MLA_OK : MLA_ERR_HIP; }

// C = scale * op(A) op(B) helpers on row-major matrices
inline GemmF64 gemm_nt(const double* A, long lda, const double* B, long ldb, double* C, long ldc, int M, int N, int K, double alpha) {
    return GemmF64{A, lda, 1, B, 1, ldb, C, ldc, M, N, K, alpha, nullptr, 0};   // C = A B^T
}
inline GemmF64 gemm_nn(const double* A, long lda, const double* B, long ldb, double* C, long ldc, int M, int N, int K, double alpha) {
    return GemmF64{A, lda, 1, B, ldb, 1, C, ldc, M, N, K, alpha, nullptr, 0};   // C = A B
}
inline GemmF64 gemm_tn(const double* A, long lda, const double* B, long ldb, double* C, long ldc, int M, int N, int K, double alpha) {
    return GemmF64{A, 1, lda, B, ldb, 1, C, ldc, M, N, K, alpha, nullptr, 0};   // C = A^T B (A is K x M)
}

constexpr int GRAM_ROOM = 16;       // p x p products of tall blocks: room for the parts of their tiles, in results
struct TopWs { double *Y, *Q, *G, *X, *T, *Z, *tmp, *part; size_t part_doubles; size_t bytes; };
TopWs top_ws(void* base, int m, int p) {
    TopWs w{};
    size_t off = 0;
    auto take = [&](size_t count) { double* ptr = base ? reinterpret_cast<double*>(static_cast<char*>(base) + off) : nullptr;
                                    off += align256(count * sizeof(double)); return ptr; };
    w.Y = take((size_t)m * p);
    w.Q = take((size_t)m * p);
    w.G = take((size_t)p * p);
    w.X = take((size_t)p * p);
    w.T = take((size_t)p * p);
    w.Z = take(jacobi_work_bytes(1, p) / sizeof(double));
    w.tmp = take(chol_tmp_doubles(p));
    w.part_doubles = std::max((size_t)GRAM_ROOM * p * p, (size_t)4 * m * p);
    w.part = take(w.part_doubles);
    w.bytes = off;
    return w;
}

// Q <- Y L^{-T} with L L^T = Y^T Y  (one Cholesky-QR pass); the result lands in `out`
int chol_qr(const double* Y, double* out, const TopWs& w, int m, int p, int* bad, hipStream_t s) {
    GemmF64 gram = gemm_tn(Y, p, Y, p, w.G, p, p, p, m, 1.0);
    gram.partial = w.part;
    gram.partial_doubles = w.part_doubles;
    gram.symmetric = 1;
    hipError_t e = launch_gemm_f64(gram, s);
    if (e != hipSuccess) return MLA_ERR_HIP;
    e = launch_chol_inverse(w.G, w.X, w.tmp, p, bad, s);
    if (e != hipSuccess) return MLA_ERR_HIP;
    GemmF64 q = gemm_nt(Y, p, w.X, p, out, p, m, p, p, 1.0);
    q.lower = 1;
    return st(launch_gemm_f64(q, s));
}

// The symmetric matrix whose leading eigenvectors are wanted: S [m x m], or C^T C / n by its factor C [n x m] (Z: n x p of
// scratch), with or without K = C C^T / n [n x n] (Z may lie over K)
struct Symmetric {
    const double* S;
    const double* C;
    int n;
    double* Z;
    const double* K = nullptr;
};

// Y = S Q
hipError_t apply(const Symmetric& a, const double* Q, double* Y, const TopWs& w, int m, int p, hipStream_t s) {
    auto product = [&](GemmF64 g) { g.partial = w.part; g.partial_doubles = w.part_doubles; return launch_gemm_f64(g, s); };
    if (a.S) return product(gemm_nn(a.S, m, Q, p, Y, p, m, p, m, 1.0));
    hipError_t e = product(gemm_nn(a.C, m, Q, p, a.Z, p, a.n, p, m, 1.0));
    return e != hipSuccess ? e : product(gemm_tn(a.C, m, a.Z, p, Y, p, m, p, a.n, 1.0 / (double)a.n));
}

int top_eig(const Symmetric& S, const double* Q0, double* evals, double* R, const TopWs& w, int* info,
            int m, int r, int p, int iters, hipStream_t s) {
    hipError_t e = launch_fill_int(info, 0, 2, s);
    if (e != hipSuccess) return MLA_ERR_HIP;
    int rc;
    // orthonormal start block (two passes: the start block is the caller's and may be badly conditioned)
    if ((rc = chol_qr(Q0, w.Y, w, m, p, info, s)) != MLA_OK) return rc;
    if ((rc = chol_qr(w.Y, w.Q, w, m, p, info, s)) != MLA_OK) return rc;
    auto product = [&](GemmF64 g) { g.partial = w.part; g.partial_doubles = w.part_doubles; return launch_gemm_f64(g, s); };
    if (S.K) {      // S^iters Q spans what C^T K^(iters - 1) (C Q) does: all steps but the ends of the first and the last among n rows
        e = product(gemm_nn(S.C, m, w.Q, p, w.Y, p, S.n, p, m, 1.0));
        for (int it = 1; e == hipSuccess && it < iters; ++it) {
            if ((rc = chol_qr(w.Y, w.Q, w, S.n, p, info, s)) != MLA_OK) return rc;
            e = product(gemm_nn(S.K, S.n, w.Q, p, w.Y, p, S.n, p, S.n, 1.0));
        }
        if (e != hipSuccess) return MLA_ERR_HIP;
        if ((rc = chol_qr(w.Y, w.Q, w, S.n, p, info, s)) != MLA_OK) return rc;
        e = product(gemm_tn(S.C, m, w.Q, p, w.Y, p, m, p, S.n, 1.0));
        if (e != hipSuccess) return MLA_ERR_HIP;
        if ((rc = chol_qr(w.Y, w.Q, w, m, p, info, s)) != MLA_OK) return rc;
    } else {
        for (int it = 0; it < iters; ++it) {
            e = apply(S, w.Q, w.Y, w, m, p, s);
            if (e != hipSuccess) return MLA_ERR_HIP;
            if ((rc = chol_qr(w.Y, w.Q, w, m, p, info, s)) != MLA_OK) return rc;
        }
    }
    // second pass restores orthonormality to rounding level before the Rayleigh-Ritz step
    if ((rc = chol_qr(w.Q, w.Y, w, m, p, info, s)) != MLA_OK) return rc;
    // T = Q^T S Q (S by its factor: (C Q)^T (C Q) / n), T = Z diag(evals) Z^T, R = Q Z[:, :r]
    if (S.S) {
        e = apply(S, w.Y, w.Q, w, m, p, s);
        if (e == hipSuccess) e = product(gemm_tn(w.Y, p, w.Q, p, w.T, p, p, p, m, 1.0));
    } else {
        e = product(gemm_nn(S.C, m, w.Y, p, S.Z, p, S.n, p, m, 1.0));
        GemmF64 ritz = gemm_tn(S.Z, p, S.Z, p, w.T, p, p, p, S.n, 1.0 / (double)S.n);
        ritz.symmetric = 1;
        if (e == hipSuccess) e = product(ritz);
    }
    if (e != hipSuccess) return MLA_ERR_HIP;
    e = launch_symmetrise(w.T, p, s);
    if (e != hipSuccess) return MLA_ERR_HIP;
    e = launch_jacobi(w.T, evals, w.Z, info + 1, 1, p, p > 128 && iters > 0 ? ritz_max_sweeps(p) : JACOBI_MAX_SWEEPS, s,
                      JacobiSpare{w.G, w.part, w.part_doubles});
    if (e != hipSuccess) return MLA_ERR_HIP;
    return st(launch_gemm_f64(gemm_nn(w.Y, p, w.T, p, R, r, m, r, p, 1.0), s));
}

struct LayerWs {
    double *K, *sigma_work, *W_K_rot, *C, *norms, *S, *W_cat;
    void* top; size_t top_bytes;
    size_t bytes;
};
LayerWs layer_ws(void* base, int n, int D, int g, int d, int M, int keep, int p) {
    LayerWs w{};
    size_t off = 0;
    auto take = [&](size_t count) { double* ptr = base ? reinterpret_cast<double*>(static_cast<char*>(base) + off) : nullptr;
                                    off += align256(count * sizeof(double)); return ptr; };
    const size_t gd = (size_t)g * d, mj = 2 * gd - (size_t)keep * (d / M), Mg = (size_t)M * g;
    w.K = take((size_t)n * gd);
    w.sigma_work = take(jacobi_work_bytes(d / (2 * M), (int)Mg) / sizeof(double));
    w.W_K_rot = take(gd * D);
    w.C = take((size_t)n * mj);
    w.norms = take(2 * (size_t)n);
    w.S = take(mj * mj);
    w.W_cat = take(mj * D);
    w.top_bytes = top_ws(nullptr, (int)mj, p).bytes;
    w.top = base ? static_cast<char*>(base) + off : nullptr;
    off += w.top_bytes;
    w.bytes = off;
    return w;
}

bool layer_shape_ok(int n, int D, int g, int h, int d, int M, int keep, int r_kv, int p) {
    if (n <= 0 || D <= 0 || g <= 0 || h <= 0 || d <= 0 || M <= 0 || r_kv <= 0 || p <= 0) return false;
    if (d % 2 || (d / 2) % M || h % g || g < 2 || keep < 1 || keep > M) return false;
    const long mj = 2L * g * d - (long)keep * (d / M);
    return r_kv <= p && p <= mj;
}

}  // namespace

extern "C" {

int mla_conv_project(const double* X, const double* W, double* Y, int n, int D, int m, int ldy, void* hip_stream) {
    if (!X || !W || !Y) return MLA_ERR_NULL;
    if (n <= 0 || D <= 0 || m <= 0 || ldy < m) return MLA_ERR_SHAPE;
    return st(launch_gemm_f64(gemm_nt(X, D, W, D, Y, ldy, n, m, D, 1.0), static_cast<hipStream_t>(hip_stream)));
}

int mla_conv_rope_moments(const double* K, double* sigma, int n, int g, int d, int M, void* hip_stream) {
    if (!K || !sigma) return MLA_ERR_NULL;
    if (n <= 0 || g <= 0 || d <= 0 || M <= 0 || d % 2 || (d / 2) % M) return MLA_ERR_SHAPE;
    if ((long)M * g > MOMENT_MAX_MG) return MLA_ERR_UNSUPPORTED;
    return st(launch_rope_moments(K, sigma, n, g, d, M, static_cast<hipStream_t>(hip_stream)));
}

size_t mla_conv_sym_eig_workspace_bytes(int batch, int m) {
    if (batch <= 0 || m < 2 || m > EIG_MAX_M) return 0;
    return jacobi_work_bytes(batch, m);
}

int mla_conv_sym_eig(double* A, double* evals, double* work, size_t work_bytes, int* info,
                     int batch, int m, int max_sweeps, void* hip_stream) {
    if (!A || !evals || !info) return MLA_ERR_NULL;
    if (batch <= 0 || m < 2 || max_sweeps <= 0) return MLA_ERR_SHAPE;
    if (m > EIG_MAX_M || batch > 65535) return MLA_ERR_UNSUPPORTED;
    if (!work || work_bytes < mla_conv_sym_eig_workspace_bytes(batch, m)) return MLA_ERR_WORKSPACE;
    return st(launch_jacobi(A, evals, work, info, batch, m, max_sweeps, static_cast<hipStream_t>(hip_stream)));
}

int mla_conv_rotate_rows(const double* W, const double* U, double* W_out, int g, int d, int M, int keep, int cols, void* hip_stream) {
    if (!W || !U || !W_out) return MLA_ERR_NULL;
    if (g <= 0 || d <= 0 || M <= 0 || cols <= 0 || d % 2 || (d / 2) % M || keep < 1 || keep > M || W == W_out) return MLA_ERR_SHAPE;
    if ((long)M * g > MOMENT_MAX_MG || (cols + 31) / 32 > 65535) return MLA_ERR_UNSUPPORTED;
    return st(launch_rotate_rows(W, U, W_out, g, d, M, keep, cols, static_cast<hipStream_t>(hip_stream)));
}

int mla_conv_kv_balance(const double* K_nope, int ldk, const double* V, int ldv, double* alpha,
                        double* row_norms, int n, int a, int b, void* hip_stream) {
    if (!K_nope || !V || !alpha || !row_norms) return MLA_ERR_NULL;
    if (n <= 0 || a <= 0 || b <= 0 || ldk < a || ldv < b) return MLA_ERR_SHAPE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    hipError_t e = launch_row_norms(K_nope, ldk, a, V, ldv, b, row_norms, n, s);
    if (e != hipSuccess) return MLA_ERR_HIP;
    return st(launch_alpha(row_norms, alpha, n, s));
}

int mla_conv_joint_moment(const double* K_nope, int ldk, const double* V, int ldv, const double* alpha,
                          double* C, double* S, int n, int a, int b, void* hip_stream) {
    if (!K_nope || !V || !alpha || !C || !S) return MLA_ERR_NULL;
    if (n <= 0 || a <= 0 || b <= 0 || ldk < a || ldv < b) return MLA_ERR_SHAPE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int m = a + b;
    hipError_t e = launch_balance(K_nope, ldk, V, ldv, alpha, C, n, a, b, s);
    if (e != hipSuccess) return MLA_ERR_HIP;
    GemmF64 moment = gemm_tn(C, m, C, m, S, m, m, m, n, 1.0 / (double)n);
    moment.symmetric = 1;
    return st(launch_gemm_f64(moment, s));
}

size_t mla_conv_top_eig_workspace_bytes(int m, int p) {
    if (m <= 0 || p <= 0 || p > m || p > TOP_MAX_P) return 0;
    return top_ws(nullptr, m, p).bytes;
}

int mla_conv_top_eig(const double* S, const double* Q0, double* evals, double* R,
                     void* workspace, size_t workspace_bytes, int* info,
                     int m, int r, int p, int iters, void* hip_stream) {
    if (!S || !Q0 || !evals || !R || !info) return MLA_ERR_NULL;
    if (m <= 0 || r <= 0 || p < r || p > m || iters < 0 || p < 2) return MLA_ERR_SHAPE;
    if (p > TOP_MAX_P) return MLA_ERR_UNSUPPORTED;
    if (!workspace || workspace_bytes < mla_conv_top_eig_workspace_bytes(m, p)) return MLA_ERR_WORKSPACE;
    return top_eig(Symmetric{S, nullptr, 0, nullptr}, Q0, evals, R, top_ws(workspace, m, p), info, m, r, p, iters, static_cast<hipStream_t>(hip_stream));
}

size_t mla_conv_apply_workspace_bytes(int m, int p) {
    if (m <= 0 || p <= 0) return 0;
    return (size_t)4 * m * p * sizeof(double);
}

int mla_conv_apply(const double* S, const double* Q, double* Y, void* workspace, size_t workspace_bytes,
                   int m, int p, void* hip_stream) {
    if (!S || !Q || !Y) return MLA_ERR_NULL;
    if (m <= 0 || p <= 0 || Q == Y) return MLA_ERR_SHAPE;
    GemmF64 g = gemm_nn(S, m, Q, p, Y, p, m, p, m, 1.0);
    if (workspace && workspace_bytes >= 2 * (size_t)m * p * sizeof(double)) {
        g.partial = static_cast<double*>(workspace);
        g.partial_doubles = workspace_bytes / sizeof(double);
    }
    return st(launch_gemm_f64(g, static_cast<hipStream_t>(hip_stream)));
}

size_t mla_convert_layer_workspace_bytes(int n, int D, int g, int h, int d, int M, int keep, int r_kv, int p) {
    if (!layer_shape_ok(n, D, g, h, d, M, keep, r_kv, p) || p > TOP_MAX_P || (long)M * g > MOMENT_MAX_MG) return 0;
    return layer_ws(nullptr, n, D, g, d, M, keep, p).bytes;
}

int mla_convert_layer(const double* X, const double* W_K, const double* W_V, const double* Q0,
                      double* W_KR, double* W_QR, double* W_DKV, double* W_UK, double* W_UV,
                      double* alpha, double* evals_rope, double* U, double* evals_joint, double* R_KV,
                      void* workspace, size_t workspace_bytes, int* info,
                      int n, int D, int g, int h, int d, int M, int keep, int r_kv, int p, int iters,
                      void* hip_stream) {
    if (!X || !W_K || !W_V || !Q0 || !W_KR || !W_QR || !W_DKV || !W_UK || !W_UV || !alpha || !evals_rope ||
        !U || !evals_joint || !R_KV || !info) return MLA_ERR_NULL;
    if (!layer_shape_ok(n, D, g, h, d, M, keep, r_kv, p) || iters < 0 || p < 2) return MLA_ERR_SHAPE;
    if (p > TOP_MAX_P || (long)M * g > MOMENT_MAX_MG || (long)M * g < 2) return MLA_ERR_UNSUPPORTED;
    if (!workspace || workspace_bytes < mla_convert_layer_workspace_bytes(n, D, g, h, d, M, keep, r_kv, p)) return MLA_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const LayerWs w = layer_ws(workspace, n, D, g, d, M, keep, p);
    const int gd = g * d, groups = d / (2 * M), Mg = M * g;
    const int d_rope = keep * (d / M);        // width of the RoPE key
    const int a = gd - d_rope, mj = a + gd;   // NoPE key, joint NoPE-key + value space
    hipError_t e;
#define MLA_TRY(call) do { e = (call); if (e != hipSuccess) return MLA_ERR_HIP; } while (0)
    // scratch of the products: the moment before it is there and after its last use
    const size_t s_doubles = (size_t)mj * mj;
    auto product = [&](GemmF64 p) { p.partial = w.S; p.partial_doubles = s_doubles; return launch_gemm_f64(p, s); };
    // Sec. 4.1 / App. B: key activations before RoPE, their per-group moments, the bases U
    MLA_TRY(product(gemm_nt(X, D, W_K, D, w.K, gd, n, gd, D, 1.0)));
    MLA_TRY(launch_rope_moments(w.K, U, n, g, d, M, s));
    const size_t bases = (size_t)groups * Mg * Mg;
    MLA_TRY(launch_jacobi(U, evals_rope, w.sigma_work, info, groups, Mg, JACOBI_MAX_SWEEPS, s,
                          s_doubles > bases ? JacobiSpare{w.S, w.S + bases, s_doubles - bases} : JacobiSpare{}));
    // Sec. 4.2: rotate W^K; the RoPE key: W_KR = the first d_rope rows, W_QR = the same rows of the rotated selectors (W^UK_i)^T
    MLA_TRY(launch_rotate_rows(W_K, U, w.W_K_rot, g, d, M, keep, D, s));
    MLA_TRY(launch_copy_scaled(w.W_K_rot, D, W_KR, D, d_rope, D, nullptr, 0, s));
    MLA_TRY(launch_gather_w_qr(U, W_QR, g, h, d, M, keep, s));
    // Sec. 4.3: activations of the NoPE key (the key activations rotated) and of the values, alpha
    MLA_TRY(launch_rotate_columns(w.K, U, w.C, mj, n, g, d, M, keep, s));
    MLA_TRY(product(gemm_nt(X, D, W_V, D, w.C + a, mj, n, gd, D, 1.0)));
    MLA_TRY(launch_row_norms(w.C, mj, a, w.C + a, mj, gd, w.norms, n, s));
    MLA_TRY(launch_alpha(w.norms, alpha, n, s));
    // App. D.2: balanced activations, their moment, its leading eigenvectors
    MLA_TRY(launch_balance(w.C, mj, w.C + a, mj, alpha, w.C, n, a, gd, s));
    const TopWs top = top_ws(w.top, mj, p);
    // The power iteration needs the moment S = C^T C / n only in products with a block, 2 m^2 p operations each; by the factor they
    // take 4 n m p and S itself (n m^2) is not formed, but a step has one product more, which costs about 12 us (8e8 operations)
    // whatever its size.  Ms a layer by the factor / by S (20 iterations unless said): m = 8128, p = 768, 4096
    // tokens 69.3 / 75.0 (these with slower solvers); m = 4032, p = 560: 1024 19.7 / 22.9, 2048 23.4 / 23.9, 2300 25.8 / 25.5; m = 1984, p = 320: 512 9.13 / 9.31,
    // 768 9.46 / 9.44, 1100 9.90 / 9.61; 4 iterations 768 6.89 / 6.97, 1100 7.12 / 7.14, 1400 7.27 / 7.26; m = 480, p = 80: 64 2.92 / 2.92,
    // 256 3.12 / 2.93.
    // Fewer tokens than dimensions: with K = C C^T / n (n^2 m, at three quarters of the other products' rate: equal tiles in rounds that
    // do not come out even), S^iters Q = C^T K^(iters - 1) C Q / n, so that all steps but the ends of the first and the last are
    // products of 2 n^2 p among n rows, as their orthonormal blocks are.  A Cholesky pass more of the m rows takes 3e7 p operations'
    // time, and a step or three among n rows do not make up for it and for the launch of K: never one, and 2.4e9 more up to four.
    // The better of the others / by K, ms: 8128, 768, 4096 tokens 63.4 / 42.8 (with slower solvers); 4032, 768: 2000 tokens 20.2 / 15.6, 3000
    // 22.3 / 18.6, 3800 22.6 / 22.9 (not taken); 1984, 64, 1000 tokens: 20 iterations 2.47 / 2.18, 4 1.450 / 1.445 and 3 1.419 / 1.458 (neither
    // taken), 1 1.436 / 1.524.
    Symmetric moment{nullptr, w.C, n, w.S};
    const double by_factor = (4.0 * iters + 2.0) * n * mj * p + 1.0 * n * p * p + 8e8 * iters;
    const double by_moment = 1.0 * n * mj * mj + (2.0 * iters + 2.0) * mj * mj * p + 2.0 * mj * p * p;
    const double by_tokens = 1.3 * n * n * mj + 2.0 * (iters - 1) * n * n * p + 6.0 * n * mj * p + 1.0 * n * p * p +
                             2.0 * (mj - 1.0 * iters * (mj - n)) * p * p + 3e7 * p + (iters <= 4 ? 2.4e9 : 0.0);
    if (iters > 1 && n >= p && n < mj && by_tokens < std::min(by_moment, by_factor)) {
        GemmF64 cct = gemm_nt(w.C, mj, w.C, mj, w.S, n, n, n, mj, 1.0 / (double)n);
        cct.symmetric = 1;
        // (scratch for its shares: what S would have taken beyond K, unless n is nearly m)
        const size_t beyond = s_doubles - (size_t)n * n;
        cct.partial = beyond > top.part_doubles ? w.S + (size_t)n * n : top.part;
        cct.partial_doubles = std::max(beyond, top.part_doubles);
        MLA_TRY(launch_gemm_f64(cct, s));
        moment.K = w.S;
    } else if (by_moment <= by_factor || (size_t)n * p > s_doubles) {
        GemmF64 ctc = gemm_tn(w.C, mj, w.C, mj, w.S, mj, mj, mj, n, 1.0 / (double)n);
        ctc.symmetric = 1;
        ctc.partial = top.part;
        ctc.partial_doubles = top.part_doubles;
        MLA_TRY(launch_gemm_f64(ctc, s));
        moment = Symmetric{w.S, nullptr, 0, nullptr};
    }
    int rc = top_eig(moment, Q0, evals_joint, R_KV, top, info + groups, mj, r_kv, p, iters, s);
    if (rc != MLA_OK) return rc;
    // W^DKV' = R^T [W^DK_NoPE / alpha ; W^DV]
    MLA_TRY(launch_copy_scaled(w.W_K_rot + (size_t)d_rope * D, D, w.W_cat, D, a, D, alpha, 2, s));
    MLA_TRY(launch_copy_scaled(W_V, D, w.W_cat + (size_t)a * D, D, gd, D, nullptr, 0, s));
    MLA_TRY(product(gemm_tn(R_KV, r_kv, w.W_cat, D, W_DKV, D, r_kv, D, mj, 1.0)));
    // W^UK'_i = alpha W^UK_NoPE,i R_K: the rows of R_K rotated back, for the heads that read them
    MLA_TRY(launch_rotate_back(R_KV, U, W_UK, g, h, d, M, keep, r_kv, alpha, s));
    // W^UV'_i = W^UV_i R_V: the rows of R_V that belong to the group of head i, transposed
    MLA_TRY(launch_gather_w_uv(R_KV, W_UV, g, h, d, a, r_kv, s));
#undef MLA_TRY
    return MLA_OK;
}

}  // extern "C"
