// Many load cases at once: up to 64 independent GMRES(m) recurrences (the
// method of Sec. 5.2 for each right-hand side) whose matrix products are one
// multi-right-hand-side product per iteration (k_gemm_f32 / k_gemm_f64), so
// the matrix is read once per iteration for all load cases.
//
// FP64 mode: the product uses the FP64 matrix on the FP64 matrix cores.
// Mixed mode: the inner product is the FP32 matrix (far entries and the FP32
// heads of the near entries) on the FP32 matrix cores, FP32 operands and
// accumulation, plus the FP64 constraint rows (a K-split row product); an outer FP64 iterative
// refinement recomputes the residual with the exact FP64-accumulated product
// of the mixed operator (FP32 matrix widened + FP64 near remainders), so the
// FP32 rounding of the inner products does not limit the final residual.
//
// Each recurrence keeps its own basis, Hessenberg matrix and rotations
// (independent, not block, Krylov spaces: identical or proportional
// right-hand sides cannot break them down).  Orthogonalisation is CGS2 in
// FP64 on the device; the host reads one Hessenberg column per recurrence
// and iteration.
//
// The order of the FP64 sums is part of the mixed mode's results: an ulp in a
// basis vector flips some FP32 roundings of the next product's input, and from
// there the recurrences part by the FP32 products' own noise (1e-9 to 1e-8 of
// the solution, all of it within the tolerance).  So the mixed mode keeps one
// order, whatever FP64 mode does: dot products split by their number
// (dot_split), partials summed one after another (SERIAL), norms by the same
// two kernels.
#include <cmath>
#include <vector>

#include "bem_device.h"

namespace bem {

void launch_gemm_f32(bem_ctx* c, const float* A, int64_t lda, int64_t M, int64_t K, const float* Zt, int64_t ldz,
                     int ncols, double* Y, int64_t ldy, bool accumulate);
void launch_gemm_f64(bem_ctx* c, const void* A, bool a_is_f32, int64_t lda, int64_t M, int64_t K, const double* Zt,
                     int64_t ldz, int ncols, double* Y, int64_t ldy, bool accumulate, double alpha);
void launch_gemm_rows(bem_ctx* c, const double* A, int64_t lda, int64_t M, int64_t K, const double* Zn, int ncols,
                      double* Y, int64_t ldy, bool accumulate, double alpha);

namespace {

constexpr int BR = 64;   // right-hand sides per batch

// Zt32/Zt64[r][i] and Zn64[i][r] from src[r * sstride + i]; zero padding
__global__ __launch_bounds__(256) void k_b_prep(const double* __restrict__ src, int64_t sstride, int nr, int64_t n,
                                                int64_t ld, float* __restrict__ zt32,
                                                double* __restrict__ zt64, double* __restrict__ zn64) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int r = blockIdx.y;
    if (i >= ld) return;
    double v = 0.0;
    if (r < nr && i < n) v = src[(int64_t)r * sstride + i];
    if (zt32) zt32[(int64_t)r * ld + i] = (float)v;
    if (zt64) zt64[(int64_t)r * ld + i] = v;
    if (zn64) zn64[i * BR + r] = v;
}

// W[r][i] += sum_e val[e] * Zn[col[e]][r] for the near entries of row i < N (one wave per row)
__global__ __launch_bounds__(256) void k_b_near(const int64_t* __restrict__ nptr, const int32_t* __restrict__ ncol,
                                                const double* __restrict__ nval, int64_t N,
                                                const double* __restrict__ zn64, int nr, double* __restrict__ W,
                                                int64_t ld) {
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int r = threadIdx.x & 63;
    if (i >= N) return;
    double s = 0.0;
    for (int64_t e = nptr[i]; e < nptr[i + 1]; ++e) s = fma(nval[e], zn64[(int64_t)ncol[e] * BR + r], s);
    if (r < nr) W[(int64_t)r * ld + i] += s;
}

// part[(r * m1 + k) * G + b] = sum over block b's slice of V[(r * m1 + k) * ld + i] * W[r * ld + i].
// A block takes up to four k, so that W is read once for them and four loads of V are in flight
// (one k a block: 26 us for 27 x 64 vectors of 7,713).
constexpr int DOT_K = 4;

__global__ __launch_bounds__(256) void k_b_dots(const double* __restrict__ V, int m1, int64_t ld, int64_t n,
                                                int kcount, const double* __restrict__ W, double* __restrict__ part,
                                                int G) {
    const int k0 = blockIdx.y * DOT_K, r = blockIdx.z;
    const double* w = W + (int64_t)r * ld;
    const double* v[DOT_K];
    double s[DOT_K];
#pragma unroll
    for (int q = 0; q < DOT_K; ++q) {
        v[q] = V + ((int64_t)r * m1 + (k0 + q < kcount ? k0 + q : k0)) * ld;
        s[q] = 0.0;
    }
    if (k0 + 1 == kcount) {
        for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < n; t += (int64_t)G * 256) s[0] = fma(v[0][t], w[t], s[0]);
    } else {
        for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < n; t += (int64_t)G * 256) {
            const double x = w[t];
#pragma unroll
            for (int q = 0; q < DOT_K; ++q) s[q] = fma(v[q][t], x, s[q]);
        }
    }
    __shared__ double red[DOT_K][4];
#pragma unroll
    for (int q = 0; q < DOT_K; ++q) {
        s[q] = wave_sum(s[q]);
        if ((threadIdx.x & 63) == 0) red[q][threadIdx.x >> 6] = s[q];
    }
    __syncthreads();
    const int q = threadIdx.x;
    if (q < DOT_K && k0 + q < kcount)
        part[((int64_t)r * m1 + k0 + q) * G + blockIdx.x] = (red[q][0] + red[q][1]) + (red[q][2] + red[q][3]);
}

// nrm[r * nstride] = sqrt(sum_b part), one wave per vector; SERIAL: the sum one after another
template <bool SERIAL>
__global__ __launch_bounds__(64) void k_b_norm(const double* __restrict__ part, int G, double* __restrict__ nrm,
                                               int nstride) {
    const double* p = part + (int64_t)blockIdx.x * G;
    double s = 0.0;
    if constexpr (SERIAL) {
        if (threadIdx.x == 0)
#pragma unroll 8
            for (int b = 0; b < G; ++b) s += p[b];
    } else {
        for (int b = threadIdx.x; b < G; b += 64) s += p[b];
        s = wave_sum(s);
    }
    if (threadIdx.x == 0) nrm[(int64_t)blockIdx.x * nstride] = sqrt(s);
}

// W[r] -= sum_k h[r][k] V[r][k] with h[r][k] the sum of the G partials of k_b_dots, taken by every block in
// the same order; block 0 of a vector sets Hcol[r][k] to it or adds it.  norm: also the partials of
// |W[r]|^2 of the result, norm[r gridDim.x + block].  SERIAL: the partials one after another, a lane a
// sum.  (A launch of its own for the sums took 5.7 us, three times an iteration.)
template <bool SERIAL>
__global__ __launch_bounds__(256) void k_b_orth(const double* __restrict__ V, int m1, int64_t ld, int64_t n, int kcount,
                                                const double* __restrict__ part, int G, double* __restrict__ Hcol,
                                                int hstride, int accumulate, double* __restrict__ W,
                                                double* __restrict__ norm) {
    __shared__ double hl[256], red[4];
    const int tid = threadIdx.x, r = blockIdx.y;
    const int64_t i = (int64_t)blockIdx.x * 256 + tid;
    double* w = W + (int64_t)r * ld;
    double s = i < n ? w[i] : 0.0;
    for (int k0 = 0; k0 < kcount; k0 += 256) {
        const int nk = kcount - k0 < 256 ? kcount - k0 : 256;
        constexpr int LS = SERIAL ? 1 : 8;   // lanes a sum
        for (int k = tid / LS; k < ((nk + 256 / LS - 1) / (256 / LS)) * (256 / LS); k += 256 / LS) {
            double a = 0.0;
            if (k < nk)
#pragma unroll 8
                for (int b = tid % LS; b < G; b += LS) a += part[((int64_t)r * m1 + k0 + k) * G + b];
#pragma unroll
            for (int o = LS / 2; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
            if (k < nk && tid % LS == 0) {
                hl[k] = a;
                double* H = Hcol + (int64_t)r * hstride + k0 + k;
                if (blockIdx.x == 0) *H = accumulate ? *H + a : a;
            }
        }
        __syncthreads();
        if (i < n) {
            const double* v = V + ((int64_t)r * m1 + k0) * ld + i;
#pragma unroll 8
            for (int k = 0; k < nk; ++k) s -= hl[k] * v[(int64_t)k * ld];
        }
        __syncthreads();
    }
    if (i < n) w[i] = s;
    if (!norm) return;
    const double q = wave_sum(s * s);
    if ((tid & 63) == 0) red[tid >> 6] = q;
    __syncthreads();
    if (tid == 0) norm[(int64_t)r * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// The next basis vectors out[r] = W[r] / |W[r]| and the next product's inputs out / d in the layouts asked for
// (see k_b_prep; rows past nr and entries past n stay zero).  |W[r]|: from the NP partials of its square, or
// nrm[r nstride] (NP = 0); where it is zero out[r] is left as it is.  col: block 0 of a vector hands its
// column Hcol[r][0..j], |W[r]| and then `id` to the host.
__global__ __launch_bounds__(256) void k_b_next(const double* __restrict__ W, int64_t ld, const double* __restrict__ parts,
                                                int NP, const double* __restrict__ nrm, int nstride, int64_t n,
                                                const double* __restrict__ d, double* __restrict__ out,
                                                int64_t ostride, float* __restrict__ zt32, double* __restrict__ zt64,
                                                double* __restrict__ zn64, const double* __restrict__ Hcol, int j,
                                                double* __restrict__ col, uint64_t* flag, uint64_t id) {
    __shared__ double vl;
    const int r = blockIdx.y;
    if (threadIdx.x < 64) {
        double a = 0.0;
        if (NP > 0) {
            for (int b = threadIdx.x; b < NP; b += 64) a += parts[(int64_t)r * NP + b];
            a = sqrt(wave_sum(a));
        } else {
            a = nrm[(int64_t)r * nstride];
        }
        if (threadIdx.x == 0) vl = a;
    }
    __syncthreads();
    const double v = vl;
    if (col && blockIdx.x == 0) {
        double* c = col + (int64_t)r * nstride;
        for (int k = threadIdx.x; k <= j; k += 256) host_put(c + k, Hcol[(int64_t)r * nstride + k]);
        if (threadIdx.x == 0) host_put(c + j + 1, v);
        host_done();
        __syncthreads();
        if (threadIdx.x == 0) host_flag(flag + r, id);
    }
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    double* op = out + (int64_t)r * ostride + i;
    const double o = v != 0.0 ? W[(int64_t)r * ld + i] / v : *op;
    if (v != 0.0) *op = o;
    const double z = o / d[i];
    if (zt32) zt32[(int64_t)r * ld + i] = (float)z;
    if (zt64) zt64[(int64_t)r * ld + i] = z;
    if (zn64) zn64[i * BR + r] = z;
}

// R[r] = B[r] - W[r]
__global__ __launch_bounds__(256) void k_b_residual(const double* __restrict__ B, const double* W, int64_t ld,
                                                    int64_t n, double* R) {   // R may be W
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int r = blockIdx.y;
    if (i < n) R[(int64_t)r * ld + i] = B[(int64_t)r * ld + i] - W[(int64_t)r * ld + i];
}

// X[r] += (sum_{k < jend[r]} y[r][k] V[r][k]) / d
__global__ __launch_bounds__(256) void k_b_update_x(const double* __restrict__ V, int m1, int64_t ld, int64_t n,
                                                    const double* __restrict__ y, const int32_t* __restrict__ jend,
                                                    const double* __restrict__ d, double* __restrict__ X) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int r = blockIdx.y;
    if (i >= n) return;
    double s = 0.0;
    for (int k = 0; k < jend[r]; ++k) s = fma(y[r * m1 + k], V[((int64_t)r * m1 + k) * ld + i], s);
    X[(int64_t)r * ld + i] += s / d[i];
}

__global__ __launch_bounds__(256) void k_b_fill(double* __restrict__ X, int64_t count, double v) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) X[i] = v;
}

__global__ __launch_bounds__(256) void k_b_add(double* __restrict__ X, const double* __restrict__ D, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) X[i] += D[i];
}

struct BW {
    bem_ctx* c;
    int nr, m, m1, G;
    int64_t n, N, ld;
    hipStream_t s;
    double *V, *W, *part, *h, *Hcol, *y;
    int32_t* jend;
    float* zt32;
    double *zt64, *zn64;
    double* host;     // pinned
    double* col;      // a column per vector in coherent host memory,
    uint64_t* flag;   // and the number of the iteration that filled it
    dim3 gv() const { return dim3((unsigned)ceil_div(n, 256), (unsigned)nr); }
};

// the input layouts that product() reads: inner FP32 vectors, FP64 ones, and FP64 ones interleaved for the
// near remainders and the constraint rows of the mixed operator
float* in32(const BW& w, bool exact) { return w.c->opt.precision == BEM_MIXED && !exact ? w.zt32 : nullptr; }
double* in64(const BW& w, bool exact) { return in32(w, exact) ? nullptr : w.zt64; }
double* in_rows(const BW& w, bool exact) {
    return w.c->opt.precision == BEM_MIXED && (exact || w.n > w.N) ? w.zn64 : nullptr;
}

// W = A z for the vectors in the input layouts, inner (mixed: FP32 cores) or exact
void product(BW& w, bool exact) {
    bem_ctx* c = w.c;
    const bool mixed = c->opt.precision == BEM_MIXED;
    if (!mixed) {
        launch_gemm_f64(c, c->A64.p, false, w.ld, w.n, w.ld, w.zt64, w.ld, w.nr, w.W, w.ld, false, 1.0);
        return;
    }
    if (!exact) {
        launch_gemm_f32(c, c->A32.as<float>(), w.ld, w.N, w.ld, w.zt32, w.ld, w.nr, w.W, w.ld, false);
    } else {
        launch_gemm_f64(c, c->A32.p, true, w.ld, w.N, w.ld, w.zt64, w.ld, w.nr, w.W, w.ld, false, 1.0);
        // FP64 remainders of the near entries
        hipLaunchKernelGGL(k_b_near, dim3((unsigned)ceil_div(w.N, 4)), dim3(256), 0, w.s, c->near_ptr.as<int64_t>(),
                           c->near_col.as<int32_t>(), c->near_val.as<double>(), w.N, w.zn64, w.nr, w.W, w.ld);
        BEM_CHECK_LAUNCH();
    }
    if (w.n > w.N)   // constraint rows (FP64, a few)
        launch_gemm_rows(c, c->A64.as<double>(), w.ld, w.n - w.N, w.ld, w.zn64, w.nr, w.W + w.N, w.ld, false, 1.0);
}

// W = A * src for the nr vectors (stride sstride)
void apply(BW& w, const double* src, int64_t sstride, bool exact) {
    hipLaunchKernelGGL(k_b_prep, dim3((unsigned)ceil_div(w.ld, 256), BR), dim3(256), 0, w.s, src, sstride, w.nr, w.n,
                       w.ld, in32(w, exact), in64(w, exact), in_rows(w, exact));
    BEM_CHECK_LAUNCH();
    product(w, exact);
}

// blocks per dot product of `ndots`: about 2048 blocks per launch in total, each at least a few waves of work
int dot_split(const BW& w, int ndots) {
    const int64_t g = 2048 / std::max(ndots, 1);
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, w.G));
}

// norms of the nr vectors v[r * ld] into dst[r * hs]
void queue_norms(BW& w, const double* v, double* dst) {
    const int G = dot_split(w, w.nr), hs = w.m + 2;
    hipLaunchKernelGGL(k_b_dots, dim3(G, 1, w.nr), dim3(256), 0, w.s, v, 1, w.ld, w.n, 1, v, w.part, G);
    BEM_CHECK_LAUNCH();
    auto kernel = w.c->opt.precision == BEM_MIXED ? k_b_norm<true> : k_b_norm<false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)w.nr), dim3(64), 0, w.s, w.part, G, dst, hs);
    BEM_CHECK_LAUNCH();
}

// norms of the nr vectors v[r * ld] into w.h[r * hs] and to the host
void norms(BW& w, const double* v, std::vector<double>& out) {
    const int hs = w.m + 2;
    queue_norms(w, v, w.h);
    BEM_HIP(hipMemcpyAsync(w.host, w.h, sizeof(double) * w.nr * hs, hipMemcpyDeviceToHost, w.s));
    BEM_HIP(hipStreamSynchronize(w.s));
    out.resize(w.nr);
    for (int r = 0; r < w.nr; ++r) out[r] = w.host[r * hs];
}

// waits until every vector's column of iteration `id` is with the host; errors of the stream are raised
void wait_columns(const BW& w, uint64_t id) {
    for (int r = 0; r < w.nr; ++r)
        for (int64_t spin = 1; __atomic_load_n(w.flag + r, __ATOMIC_ACQUIRE) < id; ++spin) {
            if ((spin & 0xffff) != 0) continue;
            const hipError_t e = hipStreamQuery(w.s);
            if (e == hipErrorNotReady) continue;
            BEM_HIP(e);
            if (__atomic_load_n(w.flag + r, __ATOMIC_ACQUIRE) < id)
                throw Error(BEM_ERR_HIP, "GMRES iteration ended without its columns");
        }
}

// Batched GMRES on A x_r = b_r: x is zero on entry, and w.h holds the norms of b (also in bnorm).
// Returns the number of iterations; rel[r] gets the final relative residual.
int bgmres(BW& w, const double* B, double* X, double tol, int max_iter, bool exact_apply, std::vector<double>& rel,
           std::vector<double>& bnorm) {
    bem_ctx* c = w.c;
    const int nr = w.nr, m = w.m, m1 = w.m1, hs = m + 2;
    const bool mixed = c->opt.precision == BEM_MIXED;   // see the head of the file
    const double* d = c->diag.as<double>();
    std::vector<double> H((size_t)nr * (m + 1) * m), cs((size_t)nr * m), sn((size_t)nr * m), g((size_t)nr * (m + 1)),
        yv((size_t)nr * m1);
    std::vector<int32_t> jend(nr), stopped(nr), done(nr);
    int iters = 0;
    std::vector<double> beta(nr);
    for (;;) {
        // residuals B - A X and their norms, then V[r][0] = residual / beta[r]; for the zero guess they are
        // B and bnorm, which the caller has just taken (w.h)
        const double* res = B;
        beta = bnorm;
        if (iters > 0) {
            apply(w, X, w.ld, exact_apply);
            hipLaunchKernelGGL(k_b_residual, w.gv(), dim3(256), 0, w.s, B, w.W, w.ld, w.n, w.W);
            BEM_CHECK_LAUNCH();
            res = w.W;
            norms(w, res, beta);
        }
        bool all_done = true;
        for (int r = 0; r < nr; ++r) {
            rel[r] = bnorm[r] > 0.0 ? beta[r] / bnorm[r] : 0.0;
            done[r] = (bnorm[r] == 0.0 || rel[r] <= tol);
            if (!done[r]) all_done = false;
        }
        if (all_done || iters >= max_iter) break;
        hipLaunchKernelGGL(k_b_next, w.gv(), dim3(256), 0, w.s, res, w.ld, w.h, 0, w.h, hs, w.n, d, w.V,
                           (int64_t)m1 * w.ld, in32(w, exact_apply), in64(w, exact_apply), in_rows(w, exact_apply),
                           w.Hcol, 0, (double*)nullptr, (uint64_t*)nullptr, (uint64_t)0);
        BEM_CHECK_LAUNCH();
        product(w, exact_apply);
        std::fill(H.begin(), H.end(), 0.0);
        std::fill(g.begin(), g.end(), 0.0);
        for (int r = 0; r < nr; ++r) {
            g[(size_t)r * (m + 1)] = beta[r];
            jend[r] = 0;
            stopped[r] = done[r];
        }
        double r_last = 1.0, r_prev = 1.0;
        for (int r = 0; r < nr; ++r) r_last = r_prev = std::max(r == 0 ? 0.0 : r_last, rel[r]);
        for (int j = 0; j < m; ++j) {
            KTimer tj(c, "bgmres_iter");
            // W = A (V[:, j] / d) is on its way
            const int G = dot_split(w, (mixed ? j + 1 : (int)ceil_div(j + 1, DOT_K)) * nr);
            const int GB = mixed ? 0 : (int)ceil_div(w.n, 256);
            double* norm = w.part + (size_t)nr * m1 * w.G;
            for (int pass = 0; pass < 2; ++pass) {
                hipLaunchKernelGGL(k_b_dots, dim3(G, ceil_div(j + 1, DOT_K), nr), dim3(256), 0, w.s, w.V, m1, w.ld,
                                   w.n, j + 1, w.W, w.part, G);
                BEM_CHECK_LAUNCH();
                hipLaunchKernelGGL((mixed ? k_b_orth<true> : k_b_orth<false>), w.gv(), dim3(256), 0, w.s, w.V, m1, w.ld,
                                   w.n, j + 1, w.part, G, w.Hcol, hs, pass, w.W,
                                   pass == 1 && !mixed ? norm : (double*)nullptr);
                BEM_CHECK_LAUNCH();
            }
            if (mixed) queue_norms(w, w.W, w.Hcol + j + 1);
            const uint64_t id = ++c->gm_seq;
            hipLaunchKernelGGL(k_b_next, w.gv(), dim3(256), 0, w.s, w.W, w.ld, norm, GB, w.Hcol + j + 1, hs, w.n, d,
                               w.V + (int64_t)(j + 1) * w.ld, (int64_t)m1 * w.ld, in32(w, exact_apply),
                               in64(w, exact_apply), in_rows(w, exact_apply), w.Hcol, j, w.col, w.flag, id);
            BEM_CHECK_LAUNCH();
            // the next product runs while the host reads the columns, unless the residuals so far say that
            // this iteration ends the solve (a product in vain costs more than the wait)
            const bool more = j + 1 < m && iters + 1 < max_iter, ahead = more && r_last * (r_last / r_prev) > tol;
            if (ahead) product(w, exact_apply);
            wait_columns(w, id);
            ++iters;
            bool all_stopped = true;
            for (int r = 0; r < nr; ++r) {
                if (stopped[r]) continue;
                double* Hr = H.data() + (size_t)r * (m + 1) * m;
                double* cr = cs.data() + (size_t)r * m;
                double* sr = sn.data() + (size_t)r * m;
                double* gr = g.data() + (size_t)r * (m + 1);
                for (int k = 0; k <= j + 1; ++k) Hr[(size_t)k * m + j] = w.col[r * hs + k];
                const double hn = w.col[r * hs + j + 1];
                for (int k = 0; k < j; ++k) {
                    const double a = Hr[(size_t)k * m + j], b = Hr[(size_t)(k + 1) * m + j];
                    Hr[(size_t)k * m + j] = cr[k] * a + sr[k] * b;
                    Hr[(size_t)(k + 1) * m + j] = -sr[k] * a + cr[k] * b;
                }
                const double a = Hr[(size_t)j * m + j], b = Hr[(size_t)(j + 1) * m + j];
                const double rr = std::sqrt(a * a + b * b);
                cr[j] = a / rr;
                sr[j] = b / rr;
                Hr[(size_t)j * m + j] = rr;
                Hr[(size_t)(j + 1) * m + j] = 0.0;
                gr[j + 1] = -sr[j] * gr[j];
                gr[j] = cr[j] * gr[j];
                jend[r] = j + 1;
                if (std::fabs(gr[j + 1]) / bnorm[r] <= tol || hn == 0.0) stopped[r] = 1;
                if (!stopped[r]) all_stopped = false;
            }
            if (all_stopped || iters >= max_iter) break;
            r_prev = r_last;
            r_last = 0.0;   // the largest residual still above the tolerance
            for (int r = 0; r < nr; ++r)
                if (!stopped[r]) r_last = std::max(r_last, std::fabs(g[(size_t)r * (m + 1) + j + 1]) / bnorm[r]);
            if (!ahead && more) product(w, exact_apply);
        }
        // y_r from the triangular systems, then X_r += V_r y_r / d
        for (int r = 0; r < nr; ++r) {
            const double* Hr = H.data() + (size_t)r * (m + 1) * m;
            const double* gr = g.data() + (size_t)r * (m + 1);
            double* yr = yv.data() + (size_t)r * m1;
            for (int k = jend[r] - 1; k >= 0; --k) {
                double sacc = gr[k];
                for (int q = k + 1; q < jend[r]; ++q) sacc -= Hr[(size_t)k * m + q] * yr[q];
                yr[k] = sacc / Hr[(size_t)k * m + k];
            }
        }
        std::copy(yv.begin(), yv.end(), w.host);
        BEM_HIP(hipMemcpyAsync(w.y, w.host, sizeof(double) * nr * m1, hipMemcpyHostToDevice, w.s));
        BEM_HIP(hipMemcpyAsync(w.jend, jend.data(), sizeof(int32_t) * nr, hipMemcpyHostToDevice, w.s));
        hipLaunchKernelGGL(k_b_update_x, w.gv(), dim3(256), 0, w.s, w.V, m1, w.ld, w.n, w.y, w.jend, d, X);
        BEM_CHECK_LAUNCH();
        BEM_HIP(hipStreamSynchronize(w.s));   // host staging and jend are reused
    }
    return iters;
}

}  // namespace

// Y[r * n + i] = (A X)[r][i] for nr <= 64 vectors X[r * n + i], exact FP64-accumulated product of the
// assembled operator on the matrix cores (the mixed operator's FP32 entries are widened exactly).
void batched_apply_exact(bem_ctx* c, int nr, const double* X, double* Y) {
    BW w;
    w.c = c;
    w.nr = nr;
    w.n = c->n;
    w.N = c->nb;
    w.ld = c->ld;
    w.s = c->stream;
    const size_t ld = (size_t)w.ld;
    c->bg_W.alloc(sizeof(double) * 64 * ld * 3);
    c->bg_z.alloc(sizeof(float) * BR * ld + sizeof(double) * BR * ld * 2);
    w.W = c->bg_W.as<double>();
    w.zt32 = c->bg_z.as<float>();
    w.zt64 = reinterpret_cast<double*>(w.zt32 + BR * ld);
    w.zn64 = w.zt64 + BR * ld;
    apply(w, X, w.n, true);
    for (int r = 0; r < nr; ++r)
        BEM_HIP(hipMemcpyAsync(Y + (int64_t)r * w.n, w.W + (int64_t)r * w.ld, sizeof(double) * w.n,
                               hipMemcpyDeviceToDevice, w.s));
}

// Solve for nr <= 64 right-hand sides B[r * ld + i] (device); X[r * ld + i] receives the solutions.
int gmres_solve_batched(bem_ctx* c, int nr, const double* B, double* X, double tol, int max_iter, int* iters_out,
                        double* relres_out, int* refinements_out) {
    BW w;
    w.c = c;
    w.nr = nr;
    w.m = c->opt.restart;
    w.m1 = w.m + 1;
    w.n = c->n;
    w.N = c->nb;
    w.ld = c->ld;
    w.s = c->stream;
    w.G = (int)std::min<int64_t>(ceil_div(w.n, 256), 128);
    const size_t ld = (size_t)w.ld;
    c->bg_V.alloc(sizeof(double) * nr * w.m1 * ld);
    c->bg_W.alloc(sizeof(double) * nr * ld * 3);
    c->bg_part.alloc(sizeof(double) * nr * ((size_t)w.m1 * w.G + (size_t)ceil_div(w.n, 256)));   // and the norms'
    c->bg_small.alloc(sizeof(double) * (size_t)nr * (w.m + 2) * 3 + sizeof(int32_t) * 64);
    c->bg_z.alloc(sizeof(float) * BR * ld + sizeof(double) * BR * ld * 2);
    c->host_stage.alloc(sizeof(double) * std::max<size_t>(4096, (size_t)nr * (w.m + 2) + 64));
    w.V = c->bg_V.as<double>();
    w.W = c->bg_W.as<double>();
    double* R = w.W + nr * ld;
    double* D = R + nr * ld;
    w.part = c->bg_part.as<double>();
    w.h = c->bg_small.as<double>();
    w.Hcol = w.h + (size_t)nr * (w.m + 2);
    w.y = w.Hcol + (size_t)nr * (w.m + 2);
    w.jend = reinterpret_cast<int32_t*>(w.y + (size_t)nr * (w.m + 2));
    w.zt32 = c->bg_z.as<float>();
    w.zt64 = reinterpret_cast<double*>(w.zt32 + BR * ld);
    w.zn64 = w.zt64 + BR * ld;
    w.host = c->host_stage.as<double>();
    const size_t cols = (size_t)nr * (w.m + 2);
    gmres_host(c, BR + cols);
    w.flag = c->gm_host.as<uint64_t>();
    w.col = c->gm_host.as<double>() + BR;
    // zero the Z buffers once: rows >= nr and entries past n stay zero
    const int64_t zwords = (int64_t)BR * ld / 2 * 5;
    hipLaunchKernelGGL(k_b_fill, dim3((unsigned)ceil_div(zwords, 256)), dim3(256), 0, w.s,
                       reinterpret_cast<double*>(w.zt32), zwords, 0.0);
    BEM_CHECK_LAUNCH();
    std::vector<double> bnorm(nr), rel(nr);
    norms(w, B, bnorm);
    const int64_t total = (int64_t)nr * w.ld;
    hipLaunchKernelGGL(k_b_fill, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, w.s, X, total, 0.0);
    BEM_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_b_fill, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, w.s, D, total, 0.0);
    BEM_CHECK_LAUNCH();
    int iters = 0, refinements = 0;
    if (c->opt.precision == BEM_FP64) {
        iters = bgmres(w, B, X, tol, max_iter, true, rel, bnorm);
    } else {
        // FP64 iterative refinement around the FP32-core inner solves
        for (;;) {
            apply(w, X, w.ld, true);
            hipLaunchKernelGGL(k_b_residual, w.gv(), dim3(256), 0, w.s, B, w.W, w.ld, w.n, R);
            BEM_CHECK_LAUNCH();
            std::vector<double> rn;
            norms(w, R, rn);
            double worst = 0.0;
            for (int r = 0; r < nr; ++r) {
                rel[r] = bnorm[r] > 0.0 ? rn[r] / bnorm[r] : 0.0;
                worst = std::max(worst, rel[r]);
            }
            if (worst <= tol || iters >= max_iter || refinements >= 20) break;
            // inner solve of A D = R on the FP32 cores to the digits still missing, but not below 1e-4:
            // FP32-accumulated products over ~10^4 terms carry ~1e-6..1e-5 relative noise, and an
            // inner target near that floor stalls GMRES
            std::vector<double> rr(nr);
            const double inner = std::min(0.1, std::max(1e-4, 0.3 * tol / std::max(worst, 1e-300)));
            iters += bgmres(w, R, D, inner, max_iter - iters, false, rr, rn);
            hipLaunchKernelGGL(k_b_add, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, w.s, X, D, total);
            BEM_CHECK_LAUNCH();
            hipLaunchKernelGGL(k_b_fill, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, w.s, D, total, 0.0);
            BEM_CHECK_LAUNCH();
            ++refinements;
        }
    }
    double worst = 0.0;
    for (int r = 0; r < nr; ++r) worst = std::max(worst, rel[r]);
    *iters_out = iters;
    *relres_out = worst;
    *refinements_out = refinements;
    return worst <= tol ? 0 : 1;
}

}  // namespace bem
