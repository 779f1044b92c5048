// Restarted GMRES(m) with right diagonal (Jacobi) preconditioning (Sec. 5.2:
// GMRES with a diagonal preconditioner), classical Gram-Schmidt applied
// twice, Givens rotations and a zero initial guess.  The Krylov basis,
// the dot products and the updates live on the device in FP64; the host
// keeps the (m+1) x m Hessenberg matrix and the rotations and reads one
// column (j + 2 doubles) per iteration.  The last kernel of an iteration puts
// the column and the iteration's number into coherent host memory, and the
// next iteration is queued before the host waits for it, unless the residuals
// so far say that this one ends the solve (an iteration queued in vain costs
// a product).  The mixed mode wraps GMRES on the mixed operator in FP64
// iterative refinement.
//
// An iteration at small n is bound by its launches (2-3 us of work in each,
// 4-5 us to queue one), so up to GM_SUM vector blocks the sums over a dot
// product's partials are taken by the kernels that use them and the second
// dot products by the first update: 5 launches where separate sums take 9.
// Above it every block would read as many partials as vector entries.  Small
// systems take one launch (k_arnoldi).  1,280 unknowns, 13 iterations, with
// assembly and evaluation: 1.05 ms before, 0.56 with five launches, 0.48 with
// one; 19,733 unknowns, 61 iterations: 31.0 -> 29.3 ms, of which 27.7 in the
// products.
#include <algorithm>
#include <cmath>
#include <vector>

#include "bem_device.h"

namespace bem {
namespace {

// part[k * G + b] = sum over block b's slice of V[k][i] * w[i]
__global__ __launch_bounds__(256) void k_dots(const double* __restrict__ V, int64_t vstride, int64_t n,
                                              const double* __restrict__ w, double* __restrict__ part, int G) {
    const int k = blockIdx.y;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double s = 0.0;
    for (int64_t t = i; t < n; t += (int64_t)G * 256) s = fma(V[k * vstride + t], w[t], s);
    s = wave_sum(s);
    __shared__ double red[4];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[(int64_t)k * G + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// h[k] = sum_b part[k * G + b];  H[k] (+)= h[k].  One wave per k: lane l sums b = l, l + 64, ...
// in order, then a fixed-order butterfly (a thread summing all G partials in turn was a chain of
// G dependent adds behind their loads).  host (one k): the result, then `id`, also to the host.
__global__ __launch_bounds__(64) void k_reduce_parts(const double* __restrict__ part, int G, int kcount,
                                                     double* __restrict__ h, double* __restrict__ Hcol, int accumulate,
                                                     int take_sqrt, double* host, uint64_t* flag, uint64_t id) {
    const int k = blockIdx.x;
    if (k >= kcount) return;
    double s = 0.0;
    for (int b = threadIdx.x; b < G; b += 64) s += part[(int64_t)k * G + b];
    s = wave_sum(s);
    if (threadIdx.x != 0) return;
    if (take_sqrt) s = sqrt(s);
    h[k] = s;
    if (Hcol) Hcol[k] = accumulate ? Hcol[k] + s : s;
    if (host) {
        host_put(host, s);
        host_done();
        host_flag(flag, id);
    }
}

constexpr int64_t GM_SUM = 128;   // vector blocks of 256 (see the head of the file)

// w -= sum_k h[k] V[k], 256 elements a block, the products of a block dealt to four groups of 256
// threads (and its sums to 16 waves): a launch has few blocks, and their chains of loads are what
// it takes.  SUM: h[k] is the sum of the partials src[k G ..], taken by every block in the same
// order, and block 0 adds it to Hcol[k] (or sets it); else h = src.
// dots: the partials of V[k] . w of the result, dots[k gridDim.x + block]; norm: those of |w|^2.
template <bool SUM>
__global__ __launch_bounds__(1024) void k_orth(const double* __restrict__ V, int64_t vstride, int64_t n, int kcount,
                                               const double* __restrict__ src, int G, double* __restrict__ Hcol,
                                               int accumulate, double* __restrict__ w, double* __restrict__ dots,
                                               double* __restrict__ norm) {
    __shared__ double hl[256], wl[256], red[3][256];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, e = tid & 255, q = tid >> 8;
    const int64_t i0 = (int64_t)blockIdx.x * 256, i = i0 + e;
    double s = (q == 0 && i < n) ? w[i] : 0.0;
    for (int k0 = 0; k0 < kcount; k0 += 256) {
        const int nk = kcount - k0 < 256 ? kcount - k0 : 256;
        if constexpr (SUM) {
            for (int k = wv; k < nk; k += 16) {
                double a = 0.0;
                for (int b = lane; b < G; b += 64) a += src[(int64_t)(k0 + k) * G + b];
                a = wave_sum(a);
                if (lane == 0) {
                    hl[k] = a;
                    if (blockIdx.x == 0) Hcol[k0 + k] = accumulate ? Hcol[k0 + k] + a : a;
                }
            }
        } else {
            if (tid < nk) hl[tid] = src[k0 + tid];
        }
        __syncthreads();
        if (i < n) {
#pragma unroll 8
            for (int k = q; k < nk; k += 4) s -= hl[k] * V[(int64_t)(k0 + k) * vstride + i];
        }
        __syncthreads();
    }
    if (q > 0) red[q - 1][e] = s;
    __syncthreads();
    if (q == 0) {
        s = (s + red[0][e]) + (red[1][e] + red[2][e]);
        if (i < n) w[i] = s;
        wl[e] = s;   // 0 past the end
    }
    __syncthreads();
    if (dots) {
        for (int k = wv; k < kcount; k += 16) {
            const double* v = V + (int64_t)k * vstride + i0;
            double a = 0.0;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (i0 + 64 * c + lane < n) a = fma(v[64 * c + lane], wl[64 * c + lane], a);
            a = wave_sum(a);
            if (lane == 0) dots[(int64_t)k * gridDim.x + blockIdx.x] = a;
        }
    }
    if (norm && wv == 0) {
        double a = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) a = fma(wl[64 * c + lane], wl[64 * c + lane], a);
        a = wave_sum(a);
        if (lane == 0) norm[blockIdx.x] = a;
    }
}

// The next Krylov vector out = w / |w| and the product's input z = out / d of the next iteration
// (both left untouched if the norm is zero).  |w|: from the NP partials of its square, or *nrm (NP = 0).
// host: block 0 hands the column Hcol[0..j], |w| and then `id` to the host.
__global__ __launch_bounds__(256) void k_scale_div(const double* w, const double* __restrict__ parts, int NP,
                                                   const double* __restrict__ nrm, const double* __restrict__ d,
                                                   int64_t n, double* out, double* __restrict__ z,   // out may be w
                                                   const double* __restrict__ Hcol, int j, double* __restrict__ host,
                                                   uint64_t* flag, uint64_t id) {
    __shared__ double vl;
    if (threadIdx.x < 64) {
        double a = 0.0;
        if (NP > 0) {
            for (int b = threadIdx.x; b < NP; b += 64) a += parts[b];
            a = sqrt(wave_sum(a));
        } else {
            a = *nrm;
        }
        if (threadIdx.x == 0) vl = a;
    }
    __syncthreads();
    const double v = vl;
    if (host && blockIdx.x == 0) {
        for (int k = threadIdx.x; k <= j; k += 256) host_put(host + k, Hcol[k]);
        if (threadIdx.x == 0) host_put(host + j + 1, v);
        host_done();
        __syncthreads();
        if (threadIdx.x == 0) host_flag(flag, id);
    }
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n || v == 0.0) return;
    const double o = w[i] / v;
    out[i] = o;
    z[i] = o / d[i];
}

constexpr int GM_ONE_N = 2048;        // vector length and
constexpr int64_t GM_ONE = 20480;     // basis entries up to which one block takes the orthogonalisation

// The whole iteration behind the product by one block: w orthogonalised twice against V[0..kc), the next
// Krylov vector and the product's input from it, its column to the host.  w stays in LDS; a wave
// takes a dot product, a thread the updates of its entries.  One CU reads the basis four times, some
// 8 us at GM_ONE entries, against four launches.  Solves of 80, 320 and 1,280 unknowns: 168 -> 140,
// 208 -> 174, 399 -> 340 us.  GM_ONE: the time of 26 solves (13 meshes of 80 to 2,562 unknowns in both bases,
// tolerances 1e-6 and 1e-10, 2 to 42 iterations) over that without this kernel, geometric mean, is 0.842 with
// 8,192 entries, 0.833 with 12,288, 0.835 with 16,384, 0.832 with 20,480, 0.835 with 24,576, 0.839 with
// 32,768 and 0.851 with 49,152: level from 12,288 to 24,576.  At 3,682 unknowns it gains nothing.
__global__ __launch_bounds__(1024) void k_arnoldi(const double* __restrict__ V, int64_t vstride, int n, int kc,
                                                  const double* __restrict__ w, const double* __restrict__ d,
                                                  double* __restrict__ out, double* __restrict__ z,
                                                  double* __restrict__ host, uint64_t* flag, uint64_t id) {
    __shared__ double wl[GM_ONE_N], hl[GM_ONE_N], hs[GM_ONE_N], red[16];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (int i = tid; i < n; i += 1024) wl[i] = w[i];
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
        for (int k = wv; k < kc; k += 16) {
            const double* v = V + (int64_t)k * vstride;
            double a = 0.0;
#pragma unroll 8
            for (int i = lane; i < n; i += 64) a = fma(v[i], wl[i], a);
            a = wave_sum(a);
            if (lane == 0) {
                hl[k] = a;
                hs[k] = pass == 0 ? a : hs[k] + a;
            }
        }
        __syncthreads();
        for (int i = tid; i < n; i += 1024) {
            double s = wl[i];
#pragma unroll 8
            for (int k = 0; k < kc; ++k) s -= hl[k] * V[(int64_t)k * vstride + i];
            wl[i] = s;
        }
        __syncthreads();
    }
    double q = 0.0;
    for (int i = tid; i < n; i += 1024) q = fma(wl[i], wl[i], q);
    q = wave_sum(q);
    if (lane == 0) red[wv] = q;
    __syncthreads();
    q = 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) q += red[u];
    const double nrm = sqrt(q);
    for (int k = tid; k < kc; k += 1024) host_put(host + k, hs[k]);
    if (tid == 0) host_put(host + kc, nrm);
    host_done();
    __syncthreads();
    if (tid == 0) host_flag(flag, id);
    if (nrm == 0.0) return;
    for (int i = tid; i < n; i += 1024) {
        const double o = wl[i] / nrm;
        out[i] = o;
        z[i] = o / d[i];
    }
}

// r = b - Ax
__global__ __launch_bounds__(256) void k_residual(const double* __restrict__ b, const double* __restrict__ Ax, int64_t n,
                                                  double* __restrict__ r) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) r[i] = b[i] - Ax[i];
}

// x += (sum_k y[k] V[k]) / d
__global__ __launch_bounds__(256) void k_update_x(const double* __restrict__ V, int64_t vstride, int64_t n, int kcount,
                                                  const double* __restrict__ y, const double* __restrict__ d,
                                                  double* __restrict__ x) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    double s = 0.0;
    for (int k = 0; k < kcount; ++k) s = fma(y[k], V[k * vstride + i], s);
    x[i] += s / d[i];
}

__global__ __launch_bounds__(256) void k_fill(double* __restrict__ x, int64_t n, double v) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) x[i] = v;
}

__global__ __launch_bounds__(256) void k_axpy(double* __restrict__ x, const double* __restrict__ d, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) x[i] += d[i];
}

__global__ __launch_bounds__(256) void k_copy(const double* __restrict__ a, int64_t n, double* __restrict__ b) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) b[i] = a[i];
}

struct Work {
    bem_ctx* c;
    int64_t n, vs;   // length and padded stride of Krylov vectors
    int m, G;
    double *V, *w, *z, *h, *part, *part2, *Hcol, *misc;
    double* host;    // pinned host staging
    double* col;     // two columns in coherent host memory,
    double* norm;    // a norm,
    uint64_t* flag;  // and the numbers of the iterations and the norm that filled them
    hipStream_t s;
    bool transpose = false;   // solve with A^T (same Jacobi diagonal)
    dim3 g1() const { return dim3((unsigned)ceil_div(n, 256)); }
};

// Waits until the host's word `flag` has reached `id`; errors of the stream are raised.
void wait_flag(Work& W, const uint64_t* flag, uint64_t id) {
    for (int64_t spin = 1; __atomic_load_n(flag, __ATOMIC_ACQUIRE) < id; ++spin) {
        if ((spin & 0xffff) != 0) continue;
        const hipError_t e = hipStreamQuery(W.s);
        if (e == hipErrorNotReady) continue;
        BEM_HIP(e);
        if (__atomic_load_n(flag, __ATOMIC_ACQUIRE) < id) throw Error(BEM_ERR_HIP, "GMRES kernels ended without their answer");
    }
}

// |v| into W.misc and, numbered by the value returned, to the host
uint64_t queue_norm(Work& W, const double* v) {
    const uint64_t id = ++W.c->gm_seq;
    hipLaunchKernelGGL(k_dots, dim3(W.G, 1), dim3(256), 0, W.s, v, (int64_t)0, W.n, v, W.part, W.G);
    BEM_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_reduce_parts, dim3(1), dim3(64), 0, W.s, W.part, W.G, 1, W.misc, (double*)nullptr, 0, 1, W.norm,
                       W.flag + 2, id);
    BEM_CHECK_LAUNCH();
    return id;
}

double host_norm(Work& W, const double* v) {
    wait_flag(W, W.flag + 2, queue_norm(W, v));
    return *W.norm;
}

// Queue iteration j: w = A z, orthogonalised twice against V[0..j], V[j + 1] and the next z from it, its
// column to the host.  Returns the iteration's number.
uint64_t queue_iteration(Work& W, int j) {
    bem_ctx* c = W.c;
    const int64_t n = W.n;
    const int GB = (int)ceil_div(n, 256);
    const int kc = j + 1;
    KTimer tj(c, "gmres_iter");
    if (W.transpose)
        launch_matvec_t(c, W.z, W.w, W.s);
    else
        launch_matvec(c, W.z, W.w, W.s);
    KTimer to(c, "gmres_ortho");
    const uint64_t id = ++c->gm_seq;
    double* next = W.V + (int64_t)kc * W.vs;
    double* col = W.col + (j & 1) * (W.m + 2);
    if (n <= GM_ONE_N && kc <= GM_ONE_N && n * kc <= GM_ONE) {
        hipLaunchKernelGGL(k_arnoldi, dim3(1), dim3(1024), 0, W.s, W.V, W.vs, (int)n, kc, W.w, c->diag.as<double>(), next,
                           W.z, col, W.flag + (j & 1), id);
        BEM_CHECK_LAUNCH();
        return id;
    }
    const bool sum = GB <= GM_SUM;
    // blocks per dot product: one element per thread, fewer where there are many products
    const int G = std::min(W.G, std::max(8, 1024 / kc));
    hipLaunchKernelGGL(k_dots, dim3(G, kc), dim3(256), 0, W.s, W.V, W.vs, n, W.w, W.part, G);
    BEM_CHECK_LAUNCH();
    double* none = nullptr;
    if (sum) {
        hipLaunchKernelGGL(k_orth<true>, dim3(GB), dim3(1024), 0, W.s, W.V, W.vs, n, kc, W.part, G, W.Hcol, 0, W.w,
                           W.part2, none);
        BEM_CHECK_LAUNCH();
        hipLaunchKernelGGL(k_orth<true>, dim3(GB), dim3(1024), 0, W.s, W.V, W.vs, n, kc, W.part2, GB, W.Hcol, 1, W.w,
                           none, W.part);
        BEM_CHECK_LAUNCH();
    } else {
        for (int pass = 0; pass < 2; ++pass) {
            if (pass == 1) {
                hipLaunchKernelGGL(k_dots, dim3(G, kc), dim3(256), 0, W.s, W.V, W.vs, n, W.w, W.part, G);
                BEM_CHECK_LAUNCH();
            }
            hipLaunchKernelGGL(k_reduce_parts, dim3((unsigned)kc), dim3(64), 0, W.s, W.part, G, kc, W.h, W.Hcol, pass, 0,
                               none, (uint64_t*)nullptr, (uint64_t)0);
            BEM_CHECK_LAUNCH();
            hipLaunchKernelGGL(k_orth<false>, dim3(GB), dim3(1024), 0, W.s, W.V, W.vs, n, kc, W.h, 0, W.Hcol, 0, W.w,
                               none, pass == 1 ? W.part2 : none);
            BEM_CHECK_LAUNCH();
        }
        hipLaunchKernelGGL(k_reduce_parts, dim3(1), dim3(64), 0, W.s, W.part2, GB, 1, W.Hcol + kc, none, 0, 1, none,
                           (uint64_t*)nullptr, (uint64_t)0);
        BEM_CHECK_LAUNCH();
    }
    hipLaunchKernelGGL(k_scale_div, dim3(GB), dim3(256), 0, W.s, W.w, W.part, sum ? GB : 0, W.Hcol + kc, c->diag.as<double>(),
                       n, next, W.z, W.Hcol, j, col, W.flag + (j & 1), id);
    BEM_CHECK_LAUNCH();
    return id;
}

// The first Krylov vector r / |r| (|r| in W.misc) and iteration 0 from it.
uint64_t queue_start(Work& W, const double* r) {
    hipLaunchKernelGGL(k_scale_div, W.g1(), dim3(256), 0, W.s, r, W.misc, 0, W.misc, W.c->diag.as<double>(), W.n, W.V, W.z,
                       W.Hcol, 0, (double*)nullptr, (uint64_t*)nullptr, (uint64_t)0);
    BEM_CHECK_LAUNCH();
    return queue_iteration(W, 0);
}

// One GMRES solve of A x = b (x overwritten; zero initial guess).
int gmres_core(Work& W, const double* b, double* x, double tol, int max_iter, int* iters_out, double* relres_out) {
    bem_ctx* c = W.c;
    const int64_t n = W.n;
    const int m = W.m;
    const double* d = c->diag.as<double>();
    hipLaunchKernelGGL(k_fill, W.g1(), dim3(256), 0, W.s, x, n, 0.0);
    BEM_CHECK_LAUNCH();
    // the first iteration is queued before the host has |b|
    const uint64_t norm_id = queue_norm(W, b);
    uint64_t id = queue_start(W, b);
    std::vector<double> H((size_t)(m + 1) * m), cs(m), sn(m), g(m + 1), y(m + 1);
    wait_flag(W, W.flag + 2, norm_id);
    const double bnorm = *W.norm;
    int iters = 0;
    double relres = 0.0;
    bool converged = false;
    if (bnorm == 0.0) {
        BEM_HIP(hipStreamSynchronize(W.s));   // the iteration on its way writes to host memory
        *iters_out = 0;
        *relres_out = 0.0;
        return 0;
    }
    for (;;) {
        // r = b - A x and its norm; b itself for the zero guess, no product needed
        const double* r = b;
        double beta = bnorm;
        if (iters > 0) {
            if (W.transpose)
                launch_matvec_t(c, x, W.w, W.s);
            else
                launch_matvec(c, x, W.w, W.s);
            hipLaunchKernelGGL(k_residual, W.g1(), dim3(256), 0, W.s, b, W.w, n, W.V);
            BEM_CHECK_LAUNCH();
            r = W.V;
            beta = host_norm(W, r);
        }
        relres = beta / bnorm;
        if (relres <= tol) {
            converged = true;
            break;
        }
        if (iters >= max_iter) break;
        if (iters > 0) id = queue_start(W, r);
        std::fill(g.begin(), g.end(), 0.0);
        std::fill(H.begin(), H.end(), 0.0);
        g[0] = beta;
        int jend = 0;
        uint64_t id_next = 0;
        double r_last = relres, r_prev = relres;
        for (int j = 0; j < m; ++j) {
            // the residual this iteration leads to if it falls by the last one's factor
            const bool more = j + 1 < m && iters + 1 < max_iter, ahead = more && r_last * (r_last / r_prev) > tol;
            if (ahead) id_next = queue_iteration(W, j + 1);
            wait_flag(W, W.flag + (j & 1), id);
            const double* col = W.col + (j & 1) * (W.m + 2);
            for (int k = 0; k <= j + 1; ++k) H[(size_t)k * m + j] = col[k];
            const double hn = col[j + 1];
            for (int k = 0; k < j; ++k) {
                const double a = H[(size_t)k * m + j], bb = H[(size_t)(k + 1) * m + j];
                H[(size_t)k * m + j] = cs[k] * a + sn[k] * bb;
                H[(size_t)(k + 1) * m + j] = -sn[k] * a + cs[k] * bb;
            }
            const double a = H[(size_t)j * m + j], bb = H[(size_t)(j + 1) * m + j];
            const double r = std::sqrt(a * a + bb * bb);
            cs[j] = a / r;
            sn[j] = bb / r;
            H[(size_t)j * m + j] = r;
            H[(size_t)(j + 1) * m + j] = 0.0;
            g[j + 1] = -sn[j] * g[j];
            g[j] = cs[j] * g[j];
            ++iters;
            jend = j + 1;
            r_prev = r_last;
            r_last = std::fabs(g[j + 1]) / bnorm;
            if (r_last <= tol || iters >= max_iter || hn == 0.0) break;
            id = ahead || !more ? id_next : queue_iteration(W, j + 1);
        }
        for (int k = jend - 1; k >= 0; --k) {
            double sacc = g[k];
            for (int q = k + 1; q < jend; ++q) sacc -= H[(size_t)k * m + q] * y[q];
            y[k] = sacc / H[(size_t)k * m + k];
        }
        for (int k = 0; k < jend; ++k) W.host[k] = y[k];
        BEM_HIP(hipMemcpyAsync(W.h, W.host, sizeof(double) * jend, hipMemcpyHostToDevice, W.s));
        hipLaunchKernelGGL(k_update_x, W.g1(), dim3(256), 0, W.s, W.V, W.vs, n, jend, W.h, d, x);
        BEM_CHECK_LAUNCH();
    }
    if (iters == 0) BEM_HIP(hipStreamSynchronize(W.s));   // as above
    *iters_out = iters;
    *relres_out = relres;
    return converged ? 0 : 1;
}

}  // namespace

// Coherent host memory of at least `words` 64-bit words: the host sees what a kernel stores there while
// later kernels run.  Its first words hold iteration numbers, which only grow, and start at 0.
void gmres_host(bem_ctx* c, size_t words) {
    c->gm_host.alloc(sizeof(uint64_t) * words, hipHostMallocCoherent);
    std::fill_n(c->gm_host.as<uint64_t>(), c->gm_host.bytes / sizeof(uint64_t), (uint64_t)0);
}

static void setup_work(bem_ctx* c, Work& W) {
    W.c = c;
    W.n = c->n;
    W.vs = c->ld;
    W.m = c->opt.restart;
    W.G = (int)std::min<int64_t>(ceil_div(c->n, 256), 1024);
    W.s = c->stream;
    c->gm_V.alloc(sizeof(double) * (size_t)W.vs * (W.m + 1));
    c->gm_w.alloc(sizeof(double) * W.vs);
    c->gm_z.alloc(sizeof(double) * W.vs);
    c->gm_h.alloc(sizeof(double) * (W.m + 2) * 2);
    // dot partials; those of the second products (GB <= GM_SUM) or the norm's GB
    const int64_t GB = ceil_div(c->n, 256), p1 = (int64_t)W.G * (W.m + 1);
    c->gm_part.alloc(sizeof(double) * (size_t)(p1 + std::max(GB, std::min(GB, GM_SUM) * (W.m + 1))));
    c->gm_r.alloc(sizeof(double) * W.vs * 3);
    W.V = c->gm_V.as<double>();
    W.w = c->gm_w.as<double>();
    W.z = c->gm_z.as<double>();
    W.h = c->gm_h.as<double>();
    W.Hcol = W.h + (W.m + 2);
    W.part = c->gm_part.as<double>();
    W.part2 = W.part + p1;
    W.misc = c->gm_r.as<double>() + 2 * W.vs;
    W.host = c->host_stage.as<double>();
    gmres_host(c, 4 + 2 * (size_t)(W.m + 2));
    W.flag = c->gm_host.as<uint64_t>();
    W.norm = c->gm_host.as<double>() + 3;
    W.col = c->gm_host.as<double>() + 4;
}

// A^T x = b (FP64 operator only): the adjoint solve of the gradient.
int gmres_solve_t(bem_ctx* c, const double* b, double* x, double tol, int max_iter, int* iters, double* relres) {
    if (c->opt.precision != BEM_FP64) throw Error(BEM_ERR_INVALID, "the adjoint solve needs precision FP64");
    Work W;
    setup_work(c, W);
    W.transpose = true;
    return gmres_core(W, b, x, tol, max_iter, iters, relres);
}

int gmres_solve(bem_ctx* c, const double* b, double* x, double tol, int max_iter, int* iters, double* relres,
                int* refinements_out) {
    *refinements_out = 0;
    Work W;
    setup_work(c, W);
    if (c->opt.precision == BEM_FP64) return gmres_core(W, b, x, tol, max_iter, iters, relres);

    // Mixed mode: FP64 iterative refinement around GMRES on the mixed operator.
    double* r = c->gm_r.as<double>();
    double* dx = r + W.vs;
    hipLaunchKernelGGL(k_fill, W.g1(), dim3(256), 0, W.s, x, W.n, 0.0);
    BEM_CHECK_LAUNCH();
    const double bnorm = host_norm(W, b);
    int total = 0, refinements = 0;
    double rel = 0.0;
    if (bnorm == 0.0) {
        *iters = 0;
        *relres = 0.0;
        return 0;
    }
    hipLaunchKernelGGL(k_copy, W.g1(), dim3(256), 0, W.s, b, W.n, r);
    BEM_CHECK_LAUNCH();
    for (;;) {
        rel = host_norm(W, r) / bnorm;
        if (rel <= tol || total >= max_iter || refinements >= 50) break;
        int it = 0;
        double rr = 0.0;
        const double inner = std::max(1e-4, 0.5 * tol / rel);
        gmres_core(W, r, dx, inner, max_iter - total, &it, &rr);
        total += it;
        ++refinements;
        hipLaunchKernelGGL(k_axpy, W.g1(), dim3(256), 0, W.s, x, dx, W.n);
        BEM_CHECK_LAUNCH();
        launch_matvec(c, x, W.w, W.s);
        hipLaunchKernelGGL(k_residual, W.g1(), dim3(256), 0, W.s, b, W.w, W.n, r);
        BEM_CHECK_LAUNCH();
    }
    *iters = total;
    *relres = rel;
    *refinements_out = refinements;
    return rel <= tol ? 0 : 1;
}

}  // namespace bem
