// Matrix-free potential and field at arbitrary points (the field formula
// that closes Sec. 2; "E surface" of Sec. 5.2).
//
// FP64:
// k_ev_far:  one point per lane, panel records read at wave-uniform addresses (scalar
//   registers); regular pairs by the 7-point rule about the centroid, the others as bit
//   masks (Sec. 4 marks and defers them).  The panel range is split over blockIdx.y so that
//   few points still fill the GPU; each split writes its own partial sums.
// k_ev_near: one wave per point: the partial sums and the point's near pairs (closed forms,
//   one pair per lane, straight from the masks), summed over the wave in a fixed order, plus
//   the exterior jump sigma n / 2 for on-surface points.
// MIXED (FP32 far field):
// k_eval_mask: Sec. 4 classification of (point, panel) pairs, panel-stationary
//   lanes, one 64-bit ballot per (point, 64-panel group); compacted to a CSR near list.
// k_eval_far:  target-stationary: one lane per point, panel tiles staged in
//   LDS and read by broadcast; 7-point rule for regular pairs, near pairs
//   masked by select.
// k_eval_finish: k_ev_near's sums from the CSR list.
#include <algorithm>

#include "bem_device.h"
#include "median_device.h"

namespace bem {
namespace {

constexpr int EV_TILE = 64;
constexpr int EV_MASK_PTS = 64;

__global__ __launch_bounds__(256) void k_eval_mask(const double* __restrict__ far64, int64_t Np, int64_t N, int64_t P,
                                                   const double* __restrict__ pts, const int32_t* __restrict__ on_panel,
                                                   uint64_t* __restrict__ mask) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool valid = j < N;
    const bool wave_live = ((j & ~(int64_t)63) < N);
    const double ccx = far64[(int64_t)(FR_CC + 0) * Np + j];
    const double ccy = far64[(int64_t)(FR_CC + 1) * Np + j];
    const double ccz = far64[(int64_t)(FR_CC + 2) * Np + j];
    const double rr = far64[(int64_t)FR_RR * Np + j];
    const int64_t p0 = (int64_t)blockIdx.y * EV_MASK_PTS;
    const int64_t p1 = p0 + EV_MASK_PTS < P ? p0 + EV_MASK_PTS : P;
    for (int64_t p = p0; p < p1; ++p) {
        const double x0 = pts[3 * p], x1 = pts[3 * p + 1], x2 = pts[3 * p + 2];
        const int64_t op = on_panel ? on_panel[p] : -1;
        const bool reg = is_regular(x0 - ccx, x1 - ccy, x2 - ccz, rr) && (j != op);
        const uint64_t m = __ballot(valid && !reg);
        if (wave_live && (threadIdx.x & 63) == 0) mask[(j >> 6) * P + p] = m;
    }
}

// bad[0]: a coordinate of the P points is not finite; bad[1]: an on_panel entry is outside [-1, N).
// (bad: coherent host memory, zero on entry.)
__global__ __launch_bounds__(256) void k_check_points(int64_t P, int64_t N, const double* __restrict__ pts,
                                                      const int32_t* __restrict__ on_panel, int32_t* bad) {
    bool b0 = false, b1 = false;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < 3 * P; i += (int64_t)gridDim.x * 256) {
        b0 = b0 || !isfinite(pts[i]);
        if (on_panel && i < P) b1 = b1 || on_panel[i] < -1 || on_panel[i] >= N;
    }
    if (b0) __hip_atomic_store(bad, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (b1) __hip_atomic_store(bad + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

constexpr int EV_C = 32;    // panels per mask word
constexpr int EV_H = 16;    // panels per half word: what a range of k_ev_far is a multiple of
constexpr int EV_Q = 128;   // near pairs per round of a wave in k_ev_near

// Up to 256 points (one per lane) against the panels [span y, span (y + 1)) of the records `rec`
// (densities in them): part[y][p] = (phi, E), and the bit masks of the pairs that are not regular,
// mask[p][half word].  on_panel: the point's own panel counts as not regular.  PHI false: no potential.
// Bound by FP64 issue; the next panel's record is requested before a panel's arithmetic.  E at 19,732
// centroids: 1.71 ms and 0.14 ms of k_ev_near; node by node over LDS tiles it took 2.30 ms, and 0.35 ms
// more for a mask pass of its own and the near list with its wait of the host.  1000 points against
// 2,192 panels: 21 + 25 us, before 180.
template <bool PHI>
__global__ __launch_bounds__(256) void k_ev_far(const double* __restrict__ rec, int64_t N, int64_t P, int64_t span,
                                                int64_t KS, const double* __restrict__ pts,
                                                const int32_t* __restrict__ on_panel, double* __restrict__ part,
                                                uint16_t* __restrict__ mask) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool live = p < P;
    const int64_t pc = live ? p : P - 1;
    const double p0 = pts[3 * pc], p1 = pts[3 * pc + 1], p2 = pts[3 * pc + 2];
    const int op = on_panel ? on_panel[pc] : -1;
    const int j0 = (int)((int64_t)blockIdx.y * span);
    const int j1 = (int)(j0 + span < N ? j0 + span : N);
    const MedConst k = med_consts();
    double phi = 0.0, e0 = 0.0, e1 = 0.0, e2 = 0.0;
    uint32_t word = 0;
    auto fetch = [&](int j, double (&v)[MED_REC]) {
        const double* r = rec + (int64_t)MED_REC * (j < j1 ? j : j1 - 1);
#pragma unroll
        for (int c = 0; c < MED_REC; ++c) v[c] = r[c];
    };
    auto panel = [&](int j, const double (&v)[MED_REC]) {
        const double t0 = p0 - v[0], t1 = p1 - v[1], t2 = p2 - v[2];
        const double T = __fma_rn(t0, t0, __fma_rn(t1, t1, t2 * t2));
        bool reg = T > v[MD_REACH];
        if (!reg) reg = is_regular(p0 - v[MD_CC], p1 - v[MD_CC + 1], p2 - v[MD_CC + 2], v[MD_RR]);
        if (reg && j != op) {
            const double pa = __fma_rn(t0, v[3], __fma_rn(t1, v[4], t2 * v[5]));
            const double pb = __fma_rn(t0, v[6], __fma_rn(t1, v[7], t2 * v[8]));
            const double pc2 = -(pa + pb);
            const double r2[7] = {T,
                                  __fma_rn(-2.0, pa, T + v[9]),
                                  __fma_rn(-2.0, pb, T + v[10]),
                                  __fma_rn(-2.0, pc2, T + v[11]),
                                  __fma_rn(k.m2rho, pa, __fma_rn(k.rho2, v[9], T)),
                                  __fma_rn(k.m2rho, pb, __fma_rn(k.rho2, v[10], T)),
                                  __fma_rn(k.m2rho, pc2, __fma_rn(k.rho2, v[11], T))};
            const double sg = v[MD_DENS];
            double g[7];
            if constexpr (PHI) {
                double ir[7];
#pragma unroll
                for (int q = 0; q < 7; ++q) {
                    ir[q] = rsqrt_pos(r2[q]);
                    g[q] = ir[q] * (ir[q] * ir[q]);
                }
                phi = __fma_rn(sg,
                               __fma_rn(k.kap0, ir[0], __fma_rn(k.kap, (ir[4] + ir[5]) + ir[6], (ir[1] + ir[2]) + ir[3])),
                               phi);
            } else {
#pragma unroll
                for (int q = 0; q < 7; ++q) g[q] = med_r3(r2[q], k);
            }
            const double G = __fma_rn(k.kap0, g[0], __fma_rn(k.kap, (g[4] + g[5]) + g[6], (g[1] + g[2]) + g[3]));
            const double h0 = __fma_rn(k.kaprho, g[4], g[1]), h1 = __fma_rn(k.kaprho, g[5], g[2]);
            const double h2 = __fma_rn(k.kaprho, g[6], g[3]);
            const double sG = sg * G, s0 = sg * (h2 - h0), s1 = sg * (h2 - h1);
            e0 = __fma_rn(sG, t0, __fma_rn(s0, v[3], __fma_rn(s1, v[6], e0)));
            e1 = __fma_rn(sG, t1, __fma_rn(s0, v[4], __fma_rn(s1, v[7], e1)));
            e2 = __fma_rn(sG, t2, __fma_rn(s0, v[5], __fma_rn(s1, v[8], e2)));
        } else {
            word |= 1u << (j & (EV_H - 1));
        }
        if ((j & (EV_H - 1)) == EV_H - 1 || j == j1 - 1) {   // j0 is a multiple of EV_H
            uint16_t* h = mask + 2 * p * KS + j / EV_H;
            if (live) h[0] = (uint16_t)word;
            if (live && j == (int)N - 1 && (j & (EV_C - 1)) < EV_H) h[1] = 0;   // the last word's other half
            word = 0;
        }
    };
    double vA[MED_REC], vB[MED_REC];
    fetch(j0, vA);
    for (int j = j0; j < j1; j += 2) {
        wait_scalar();
        fetch(j + 1, vB);
        panel(j, vA);
        wait_scalar();
        fetch(j + 2, vA);
        if (j + 1 < j1) panel(j + 1, vB);
    }
    if (!live) return;
    double* o = part + ((int64_t)blockIdx.y * P + p) * 4;
    o[0] = phi;
    o[1] = e0;
    o[2] = e1;
    o[3] = e2;
}

// One wave per point: see the head of the file.  phi_out may be nullptr (K ranges of partial sums).
__global__ __launch_bounds__(256) void k_ev_near(int64_t P, int64_t K, int64_t KS, const double* __restrict__ part,
                                                 const uint32_t* __restrict__ mask, const double* __restrict__ tri64,
                                                 const double* __restrict__ sigma, const double* __restrict__ pts,
                                                 const int32_t* __restrict__ on_panel, double* __restrict__ phi_out,
                                                 double* __restrict__ E_out) {
    __shared__ int32_t list[4][EV_Q];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t p = (int64_t)blockIdx.x * 4 + wv;
    if (p >= P) return;   // no barrier below: each wave works alone
    const uint32_t* mrow = mask + p * KS;
    double phi = 0.0, e0 = 0.0, e1 = 0.0, e2 = 0.0;
    for (int64_t r = lane; r < K; r += 64) {
        const double* o = part + (r * P + p) * 4;
        phi += o[0];
        e0 += o[1];
        e1 += o[2];
        e2 += o[3];
    }
    const double x0 = pts[3 * p], x1 = pts[3 * p + 1], x2 = pts[3 * p + 2];
    const int64_t op = on_panel ? on_panel[p] : -1;
    int cnt = 0;
    for (int64_t w = lane; w < KS; w += 64) cnt += __popc(mrow[w]);
    int incl = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    const int total = __shfl(incl, 63, 64), last = incl;   // the lane's marks are [last - cnt, last) of the list
    int pos = incl - cnt;
    int64_t w = lane;
    uint32_t word = w < KS ? mrow[w] : 0;
    for (int base = 0; base < total; base += EV_Q) {
        const int end = last < base + EV_Q ? last : base + EV_Q;   // the lane goes on where its last round ended
        for (; pos < end; ++pos) {
            while (word == 0) word = mrow[w += 64];
            list[wv][pos - base] = (int32_t)(w * EV_C + __builtin_ctz(word));
            word &= word - 1;
        }
        wave_sync();
        const int nq = total - base < EV_Q ? total - base : EV_Q;
        for (int q = lane; q < nq; q += 64) {
            const int64_t j = list[wv][q];
            double S, F0, F1, F2;
            flat_tri_SF<true, true>(tri64 + (int64_t)TRI_REC * j, x0, x1, x2, j == op, S, F0, F1, F2);
            const double s = sigma[j];
            phi = fma(s, S, phi);
            e0 = fma(s, F0, e0);
            e1 = fma(s, F1, e1);
            e2 = fma(s, F2, e2);
        }
        wave_sync();
    }
    phi = wave_sum(phi);
    e0 = wave_sum(e0);
    e1 = wave_sum(e1);
    e2 = wave_sum(e2);
    if (lane != 0) return;
    if (op >= 0) {
        const double* T = tri64 + (int64_t)TRI_REC * op;
        const double hs = 0.5 * sigma[op];
        e0 += hs * T[TR_N + 0];
        e1 += hs * T[TR_N + 1];
        e2 += hs * T[TR_N + 2];
    }
    if (phi_out) phi_out[p] = phi;
    E_out[3 * p] = e0;
    E_out[3 * p + 1] = e1;
    E_out[3 * p + 2] = e2;
}

__global__ __launch_bounds__(256) void k_eval_far(const double* __restrict__ far64, const float* __restrict__ farR,
                                                  int64_t Np, int64_t N, int64_t span,
                                                  const double* __restrict__ sigma, int64_t P,
                                                  const double* __restrict__ pts, const int32_t* __restrict__ on_panel,
                                                  double* __restrict__ part) {
    __shared__ float tq[EV_TILE][4 * 7];      // node xyz + weight
    __shared__ double tc[EV_TILE][5];     // circumcentre, (eta R)^2, sigma
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool pv = p < P;
    const int64_t pc = pv ? p : P - 1;
    const double x0 = pts[3 * pc], x1 = pts[3 * pc + 1], x2 = pts[3 * pc + 2];
    const int64_t op = on_panel ? on_panel[pc] : -1;
    const float xr0 = (float)x0, xr1 = (float)x1, xr2 = (float)x2;
    double phi = 0.0, e0 = 0.0, e1 = 0.0, e2 = 0.0;
    const int64_t j_beg = (int64_t)blockIdx.y * span;
    const int64_t j_end = j_beg + span < N ? j_beg + span : N;
    for (int64_t t0 = j_beg; t0 < j_end; t0 += EV_TILE) {
        __syncthreads();
        // stage EV_TILE panels: 28 node values + 5 classification values each
        for (int e = threadIdx.x; e < EV_TILE * 33; e += 256) {
            const int pj = e % EV_TILE, comp = e / EV_TILE;
            const int64_t j = t0 + pj;   // < Np: span is a multiple of EV_TILE and Np >= N rounded up
            if (comp < 28)
                tq[pj][comp] = farR[(int64_t)comp * Np + j];
            else if (comp < 32)
                tc[pj][comp - 28] = far64[(int64_t)comp * Np + j];
            else
                tc[pj][4] = (j < N) ? sigma[j] : 0.0;
        }
        __syncthreads();
        const int cnt = (int)((j_end - t0) < EV_TILE ? (j_end - t0) : EV_TILE);
        for (int pj = 0; pj < cnt; ++pj) {
            const int64_t j = t0 + pj;
            const bool reg = is_regular(x0 - tc[pj][0], x1 - tc[pj][1], x2 - tc[pj][2], tc[pj][3]) && (j != op);
            float sp = 0, f0 = 0, f1 = 0, f2 = 0;
#pragma unroll
            for (int q = 0; q < 7; ++q) {
                const float dx = xr0 - tq[pj][q], dy = xr1 - tq[pj][7 + q], dz = xr2 - tq[pj][14 + q];
                const float r2 = dx * dx + dy * dy + dz * dz;
                const float ir = rsqrt_pos(r2);
                const float t = tq[pj][21 + q] * ir;
                sp += t;
                const float t3 = t * ir * ir;
                f0 += t3 * dx;
                f1 += t3 * dy;
                f2 += t3 * dz;
            }
            const double s = reg ? tc[pj][4] : 0.0;
            phi = fma(s, (double)(reg ? sp : (float)0), phi);
            e0 = fma(s, (double)(reg ? f0 : (float)0), e0);
            e1 = fma(s, (double)(reg ? f1 : (float)0), e1);
            e2 = fma(s, (double)(reg ? f2 : (float)0), e2);
        }
    }
    if (pv) {
        double* o = part + ((int64_t)blockIdx.y * P + p) * 4;
        o[0] = phi;
        o[1] = e0;
        o[2] = e1;
        o[3] = e2;
    }
}

__global__ __launch_bounds__(256) void k_eval_finish(const double* __restrict__ part, int KS, int64_t P,
                                                     const int64_t* __restrict__ nptr, const int32_t* __restrict__ ncol,
                                                     const double* __restrict__ tri64, const double* __restrict__ sigma,
                                                     const double* __restrict__ pts, const int32_t* __restrict__ on_panel,
                                                     double* __restrict__ phi_out, double* __restrict__ E_out) {
    const int64_t p = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // wave-uniform
    const int lane = threadIdx.x & 63;
    if (p >= P) return;
    double phi = 0.0, e0 = 0.0, e1 = 0.0, e2 = 0.0;
    for (int k = lane; k < KS; k += 64) {
        const double* o = part + ((int64_t)k * P + p) * 4;
        phi += o[0];
        e0 += o[1];
        e1 += o[2];
        e2 += o[3];
    }
    const double x0 = pts[3 * p], x1 = pts[3 * p + 1], x2 = pts[3 * p + 2];
    const int64_t op = on_panel ? on_panel[p] : -1;
    for (int64_t e = nptr[p] + lane; e < nptr[p + 1]; e += 64) {
        const int64_t j = ncol[e];
        double S, F0, F1, F2;
        flat_tri_SF<true, true>(tri64 + (int64_t)TRI_REC * j, x0, x1, x2, j == op, S, F0, F1, F2);
        const double s = sigma[j];
        phi = fma(s, S, phi);
        e0 = fma(s, F0, e0);
        e1 = fma(s, F1, e1);
        e2 = fma(s, F2, e2);
    }
    phi = wave_sum(phi);
    e0 = wave_sum(e0);
    e1 = wave_sum(e1);
    e2 = wave_sum(e2);
    if (lane != 0) return;
    if (op >= 0) {
        const double* T = tri64 + (int64_t)TRI_REC * op;
        const double hs = 0.5 * sigma[op];
        e0 += hs * T[TR_N + 0];
        e1 += hs * T[TR_N + 1];
        e2 += hs * T[TR_N + 2];
    }
    if (phi_out) phi_out[p] = phi;
    E_out[3 * p] = e0;
    E_out[3 * p + 1] = e1;
    E_out[3 * p + 2] = e2;
}

}  // namespace

void launch_point_mask(bem_ctx* c, int64_t P, const double* pts, const int32_t* on_panel, uint64_t* mask) {
    if (P == 0) return;
    const int64_t Np = (int64_t)(c->far64.bytes / (sizeof(double) * FAR_REC));
    dim3 grid((unsigned)(Np / 256), (unsigned)ceil_div(P, EV_MASK_PTS));
    hipLaunchKernelGGL(k_eval_mask, grid, dim3(256), 0, c->stream, c->far64.as<double>(), Np, c->N, P, pts, on_panel,
                       mask);
    BEM_CHECK_LAUNCH();
}

// K ranges of the panel split of the far pass for P points: about the tuned number of blocks
// (default 2048); span (panels per range) is a multiple of `unit`.
static int64_t eval_split(const bem_ctx* c, int64_t P, int64_t unit, int64_t* span) {
    const int64_t N = c->N;
    const int64_t pb = ceil_div(P, 256);
    int64_t KS = c->tune_eval_blocks / pb;
    if (KS < 1) KS = 1;
    if (KS > ceil_div(N, unit)) KS = ceil_div(N, unit);
    if (KS > 65535) KS = 65535;   // the grid's second dimension
    *span = ceil_div(ceil_div(N, KS), unit) * unit;
    return ceil_div(N, *span);
}

// FP64: points in batches whose masks stay within 256 MiB
static void launch_eval64(bem_ctx* c, const double* sigma, int64_t P, const double* pts, const int32_t* on_panel,
                          double* phi, double* E) {
    const int64_t N = c->N, W = ceil_div(N, EV_C);
    launch_median_records(c, sigma, c->ev_rec);
    const int64_t B = std::min<int64_t>(P, std::max<int64_t>(1024, ((int64_t)256 << 20) / (4 * W)));
    for (int64_t p0 = 0; p0 < P; p0 += B) {
        const int64_t nb = std::min<int64_t>(B, P - p0);
        int64_t span = 0;
        const int64_t K = eval_split(c, nb, EV_H, &span);
        c->ev_part.alloc(sizeof(double) * 4 * (size_t)(K * nb));
        c->ev_mask.alloc(sizeof(uint32_t) * (size_t)(W * nb));
        const double* bp = pts + 3 * p0;
        const int32_t* bo = on_panel ? on_panel + p0 : nullptr;
        {
            KTimer t(c, "eval_far");
            const dim3 grid((unsigned)ceil_div(nb, 256), (unsigned)K);
            if (phi)
                hipLaunchKernelGGL(k_ev_far<true>, grid, dim3(256), 0, c->stream, c->ev_rec.as<double>(), N, nb, span, W,
                                   bp, bo, c->ev_part.as<double>(), c->ev_mask.as<uint16_t>());
            else
                hipLaunchKernelGGL(k_ev_far<false>, grid, dim3(256), 0, c->stream, c->ev_rec.as<double>(), N, nb, span, W,
                                   bp, bo, c->ev_part.as<double>(), c->ev_mask.as<uint16_t>());
            BEM_CHECK_LAUNCH();
        }
        {
            KTimer t(c, "eval_near");
            hipLaunchKernelGGL(k_ev_near, dim3((unsigned)ceil_div(nb, 4)), dim3(256), 0, c->stream, nb, K, W,
                               c->ev_part.as<double>(), c->ev_mask.as<uint32_t>(), c->tri64.as<double>(), sigma, bp, bo,
                               phi ? phi + p0 : nullptr, E + 3 * p0);
            BEM_CHECK_LAUNCH();
        }
    }
}

void launch_check_points(bem_ctx* c, int64_t P, const double* pts, const int32_t* on_panel, int32_t* bad) {
    hipLaunchKernelGGL(k_check_points, dim3((unsigned)std::min<int64_t>(ceil_div(3 * P, 256), 1024)), dim3(256), 0,
                       c->stream, P, c->N, pts, on_panel, bad);
    BEM_CHECK_LAUNCH();
}

void launch_eval(bem_ctx* c, const double* sigma, int64_t P, const double* pts, const int32_t* on_panel, double* phi,
                 double* E) {
    if (P == 0) return;
    if (c->opt.precision == BEM_FP64) {
        launch_eval64(c, sigma, P, pts, on_panel, phi, E);
        return;
    }
    const int64_t N = c->N;
    const int64_t nblk = ceil_div(N, 64);
    c->ev_mask.alloc(sizeof(uint64_t) * nblk * P);
    {
        KTimer t(c, "eval_mask");
        launch_point_mask(c, P, pts, on_panel, c->ev_mask.as<uint64_t>());
    }
    int64_t nnz = 0;
    launch_near_csr(c, c->ev_mask.as<uint64_t>(), P, c->ev_ptr, c->ev_row, c->ev_col, &nnz, "eval_near_csr");
    int64_t span = 0;
    const int64_t KS = eval_split(c, P, EV_TILE, &span);
    c->ev_part.alloc(sizeof(double) * 4 * KS * P);
    {
        KTimer t(c, "eval_far");
        const int64_t Np = (int64_t)(c->far64.bytes / (sizeof(double) * FAR_REC));
        hipLaunchKernelGGL(k_eval_far, dim3((unsigned)ceil_div(P, 256), (unsigned)KS), dim3(256), 0, c->stream,
                           c->far64.as<double>(), c->far32.as<float>(), Np, N, span, sigma, P, pts, on_panel,
                           c->ev_part.as<double>());
        BEM_CHECK_LAUNCH();
    }
    {
        KTimer t(c, "eval_near");
        hipLaunchKernelGGL(k_eval_finish, dim3((unsigned)ceil_div(P, 4)), dim3(256), 0, c->stream,
                           c->ev_part.as<double>(), (int)KS, P, c->ev_ptr.as<int64_t>(), c->ev_col.as<int32_t>(),
                           c->tri64.as<double>(), sigma, pts, on_panel, phi, E);
        BEM_CHECK_LAUNCH();
    }
}

}  // namespace bem
