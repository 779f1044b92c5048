// Reverse sweep of the field lines for the gradient of the streamer integrals
// (Sec. 1, Eq. Breakdowncrit), and field + field Jacobian at collocation points.
//
// The forward tracer (RK4 on dx/ds = dir E/|E| with the integral carried as an
// extra state) is differentiated step by step in reverse order.  Step n from
// x_n evaluates E at the stage points X_1..X_4; its reverse needs E and the
// Jacobian H = dE/dx at the same points, and then runs the adjoint of the step:
//   kbar_s  = h c_s xbar,           c = (1, 2, 2, 1) / 6
//   for s = 4..1:
//     ebar_s = dir (kbar_s - e_s (e_s . kbar_s)) / |E_s| + g h c_s alpha'(|E_s|) e_s
//     Xbar_s = H_s ebar_s;  xbar += Xbar_s;  kbar_{s-1} += (h, h/2, h/2)_s Xbar_s
// with e_s = E_s / |E_s| and g = dJ/dI of the line.  ebar_s is the sensitivity
// of J to the field value at X_s; the pairs (X_s, ebar_s) are written out for
// the charge and geometry terms.  Regular/near classification and the number
// of accepted steps are those of the forward run.
//
// E and H at a step's stage points depend on x_n alone, which the forward run
// left, and not on the adjoint state.  So they are taken for all steps of all
// lines together, stage by stage, as one batch of points (105,000 for 128
// coaxial lines, where a sweep step by step has at most 128 points a pass and
// 8,000 passes one after another); only the recursion in xbar, a few hundred
// operations a step, then runs along each line.
//
//  k_sp_far     - (256 points x panel range) blocks, one point per lane, panel
//                 records read at wave-uniform addresses: E and H of the regular
//                 pairs by the 7-point rule about the centroid (median_device.h),
//                 near pairs as bit masks.
//  k_sp_near    - one wave per point: the ranges' partial sums, the near pairs by
//                 the closed forms differentiated with dual numbers (one pair per
//                 lane), and the next stage's point.
//  k_sp_adjoint - one wave per line: the recursion above, 16 steps' fields staged
//                 in LDS at a time.
#include <algorithm>
#include <climits>

#include "adjoint_device.h"
#include "median_device.h"

namespace bem {
namespace {

constexpr int SP_T = 256;   // points per block of k_sp_far
constexpr int SP_C = 32;    // panels per mask word
constexpr int SP_NC = 9;    // E (3) + H (xx, yy, zz, xy, xz, yz)
constexpr int SP_Q = 128;   // near pairs per round of a wave in k_sp_near
constexpr int SP_STEPS = 16;   // steps of a line staged at a time in k_sp_adjoint

struct LAArgs {
    double h, dir, a, e0, p;
};

__device__ __noinline__ double la_pow(double d, double p) { return pow(d, p); }

// alpha'(e) for alpha = a max(e - e0, 0)^p
__device__ __forceinline__ double la_dalpha(const LAArgs& a, double e) {
    const double d = e - a.e0;
    if (!(d > 0.0)) return 0.0;
    return a.a * a.p * (a.p == 2.0 ? d : la_pow(d, a.p - 1.0));
}

// E and H of the regular pairs of up to 256 points (one per lane, at pts[pstride p]) with the panels
// [span y, span (y + 1)) of the records `rec` (densities in them): part[y][p][9], and the bit masks
// of the other pairs, mask[p][word].  Bound by FP64 issue: 15 FP64 instructions to test a pair and 175
// for a regular one's sums (the node-by-node form takes 245 in all).
__global__ __launch_bounds__(SP_T) void k_sp_far(const double* __restrict__ rec, int64_t N, int64_t P, int64_t span,
                                                 int64_t KS, const double* __restrict__ pts, int64_t pstride,
                                                 double* __restrict__ part, uint32_t* __restrict__ mask) {
    const int64_t p = (int64_t)blockIdx.x * SP_T + threadIdx.x;
    const bool live = p < P;
    const int64_t pc = live ? p : P - 1;
    const double p0 = pts[pstride * pc], p1 = pts[pstride * pc + 1], p2 = pts[pstride * pc + 2];
    const int64_t j0 = (int64_t)blockIdx.y * span;
    const int64_t j1 = j0 + span < N ? j0 + span : N;
    const MedConst k = med_consts();
    double acc[SP_NC];
#pragma unroll
    for (int c = 0; c < SP_NC; ++c) acc[c] = 0.0;
    uint32_t word = 0;
    for (int64_t j = j0; j < j1; ++j) {
        const double* r = rec + MED_REC * j;
        double v[MED_REC];
#pragma unroll
        for (int c = 0; c < MED_REC; ++c) v[c] = r[c];
        const double t0 = p0 - v[0], t1 = p1 - v[1], t2 = p2 - v[2];
        const double T = __fma_rn(t0, t0, __fma_rn(t1, t1, t2 * t2));
        bool reg = T > v[MD_REACH];
        if (!reg) reg = is_regular(p0 - v[MD_CC], p1 - v[MD_CC + 1], p2 - v[MD_CC + 2], v[MD_RR]);
        if (reg) {
            const double m00 = v[3], m01 = v[4], m02 = v[5], m10 = v[6], m11 = v[7], m12 = v[8];
            const double pa = __fma_rn(t0, m00, __fma_rn(t1, m01, t2 * m02));
            const double pb = __fma_rn(t0, m10, __fma_rn(t1, m11, t2 * m12));
            const double pc2 = -(pa + pb);
            double g[7], u[7];   // r^-3 and r^-5 at c, c + m_i, c + rho m_i
            med_r3r5(T, g[0], u[0]);
            med_r3r5(__fma_rn(-2.0, pa, T + v[9]), g[1], u[1]);
            med_r3r5(__fma_rn(-2.0, pb, T + v[10]), g[2], u[2]);
            med_r3r5(__fma_rn(-2.0, pc2, T + v[11]), g[3], u[3]);
            med_r3r5(__fma_rn(k.m2rho, pa, __fma_rn(k.rho2, v[9], T)), g[4], u[4]);
            med_r3r5(__fma_rn(k.m2rho, pb, __fma_rn(k.rho2, v[10], T)), g[5], u[5]);
            med_r3r5(__fma_rn(k.m2rho, pc2, __fma_rn(k.rho2, v[11], T)), g[6], u[6]);
            const double sg = v[MD_DENS];
            // E = G t - (h_0 - h_2) m_0 - (h_1 - h_2) m_1
            const double G = __fma_rn(k.kap0, g[0], __fma_rn(k.kap, (g[4] + g[5]) + g[6], (g[1] + g[2]) + g[3]));
            const double h0 = __fma_rn(k.kaprho, g[4], g[1]), h1 = __fma_rn(k.kaprho, g[5], g[2]);
            const double h2 = __fma_rn(k.kaprho, g[6], g[3]);
            const double sG = sg * G, s0 = sg * (h2 - h0), s1 = sg * (h2 - h1);
            acc[0] = __fma_rn(sG, t0, __fma_rn(s0, m00, __fma_rn(s1, m10, acc[0])));
            acc[1] = __fma_rn(sG, t1, __fma_rn(s0, m01, __fma_rn(s1, m11, acc[1])));
            acc[2] = __fma_rn(sG, t2, __fma_rn(s0, m02, __fma_rn(s1, m12, acc[2])));
            // H = G I - 3 sum w r^-5 d d^T with d = t - c_q m_i: A t t^T - (t V^T + V t^T) + m m^T terms,
            // A = sum u, V = sum_i B_i m_i, B_i = sum c u, C_i = sum c^2 u
            const double s3 = -3.0 * sg;
            const double A = s3 * __fma_rn(k.kap0, u[0], __fma_rn(k.kap, (u[4] + u[5]) + u[6], (u[1] + u[2]) + u[3]));
            const double B0 = __fma_rn(k.kaprho, u[4], u[1]), B1 = __fma_rn(k.kaprho, u[5], u[2]);
            const double B2 = __fma_rn(k.kaprho, u[6], u[3]);
            const double C0 = s3 * __fma_rn(k.kaprho2, u[4], u[1]), C1 = s3 * __fma_rn(k.kaprho2, u[5], u[2]);
            const double C2 = s3 * __fma_rn(k.kaprho2, u[6], u[3]);
            const double b0 = s3 * (B2 - B0), b1 = s3 * (B2 - B1), hA = 0.5 * A;
            // t W^T + W t^T with W = A t / 2 - V
            const double W0 = __fma_rn(hA, t0, __fma_rn(b0, m00, b1 * m10));
            const double W1 = __fma_rn(hA, t1, __fma_rn(b0, m01, b1 * m11));
            const double W2 = __fma_rn(hA, t2, __fma_rn(b0, m02, b1 * m12));
            const double a0 = C0 + C2, a1 = C1 + C2;
            const double P0 = __fma_rn(a0, m00, C2 * m10), P1 = __fma_rn(a0, m01, C2 * m11),
                         P2 = __fma_rn(a0, m02, C2 * m12);
            const double Q0 = __fma_rn(a1, m10, C2 * m00), Q1 = __fma_rn(a1, m11, C2 * m01),
                         Q2 = __fma_rn(a1, m12, C2 * m02);
            acc[3] = __fma_rn(2.0 * t0, W0, __fma_rn(m00, P0, __fma_rn(m10, Q0, acc[3] + sG)));
            acc[4] = __fma_rn(2.0 * t1, W1, __fma_rn(m01, P1, __fma_rn(m11, Q1, acc[4] + sG)));
            acc[5] = __fma_rn(2.0 * t2, W2, __fma_rn(m02, P2, __fma_rn(m12, Q2, acc[5] + sG)));
            acc[6] = __fma_rn(t0, W1, __fma_rn(t1, W0, __fma_rn(m00, P1, __fma_rn(m10, Q1, acc[6]))));
            acc[7] = __fma_rn(t0, W2, __fma_rn(t2, W0, __fma_rn(m00, P2, __fma_rn(m10, Q2, acc[7]))));
            acc[8] = __fma_rn(t1, W2, __fma_rn(t2, W1, __fma_rn(m01, P2, __fma_rn(m11, Q2, acc[8]))));
        } else {
            word |= 1u << (int)(j & (SP_C - 1));
        }
        if ((j & (SP_C - 1)) == SP_C - 1 || j == j1 - 1) {   // j0 is a multiple of SP_C
            if (live) mask[p * KS + j / SP_C] = word;
            word = 0;
        }
    }
    if (!live) return;
    double* o = part + ((int64_t)blockIdx.y * P + p) * SP_NC;
#pragma unroll
    for (int c = 0; c < SP_NC; ++c) o[c] = acc[c];
}

// One wave per point: E and H from the K ranges' partial sums (in order) and the near pairs (panel
// row0 + p left out when rows), written to out[ostride p].  stage 0..2: also the next stage's point,
// x + (h / 2 or h) dir E / |E|, three doubles after the point's own (x the first stage's).
__global__ __launch_bounds__(256, 2) void k_sp_near(int64_t P, int64_t K, int64_t KS, const double* __restrict__ part,
                                                 const uint32_t* __restrict__ mask, const double* __restrict__ tri64,
                                                 const double* __restrict__ sigma, bool rows, int64_t row0,
                                                 double* __restrict__ pts, int64_t pstride, int stage, double h,
                                                 double dir, double* __restrict__ out, int64_t ostride) {
    __shared__ int32_t list[4][SP_Q];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t p = (int64_t)blockIdx.x * 4 + wv;
    if (p >= P) return;   // no barrier below: each wave works alone
    const double* x = pts + pstride * p;
    const double p0 = x[0], p1 = x[1], p2 = x[2];
    const int64_t skip = rows ? row0 + p : -1;
    double acc[SP_NC];
#pragma unroll
    for (int c = 0; c < SP_NC; ++c) acc[c] = 0.0;
    for (int64_t r = lane; r < K; r += 64) {
        const double* o = part + (r * P + p) * SP_NC;
#pragma unroll
        for (int c = 0; c < SP_NC; ++c) acc[c] += o[c];
    }
    const uint32_t* mrow = mask + p * KS;
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
    for (int base = 0; base < total; base += SP_Q) {
        const int end = last < base + SP_Q ? last : base + SP_Q;   // the lane goes on where its last round ended
        for (; pos < end; ++pos) {
            while (word == 0) word = mrow[w += 64];
            list[wv][pos - base] = (int32_t)(w * SP_C + __builtin_ctz(word));
            word &= word - 1;
        }
        wave_sync();
        const int nq = total - base < SP_Q ? total - base : SP_Q;
        for (int q = lane; q < nq; q += 64) {
            const int j = list[wv][q];
            if (j == skip) continue;
            double Fv[3], Jac[3][3];
            tri_F_dx(tri64 + (int64_t)TRI_REC * j, p0, p1, p2, Fv, Jac);
            const double sg = sigma[j];
            acc[0] = fma(sg, Fv[0], acc[0]);
            acc[1] = fma(sg, Fv[1], acc[1]);
            acc[2] = fma(sg, Fv[2], acc[2]);
            acc[3] = fma(sg, Jac[0][0], acc[3]);
            acc[4] = fma(sg, Jac[1][1], acc[4]);
            acc[5] = fma(sg, Jac[2][2], acc[5]);
            acc[6] = fma(sg, 0.5 * (Jac[0][1] + Jac[1][0]), acc[6]);
            acc[7] = fma(sg, 0.5 * (Jac[0][2] + Jac[2][0]), acc[7]);
            acc[8] = fma(sg, 0.5 * (Jac[1][2] + Jac[2][1]), acc[8]);
        }
        wave_sync();
    }
#pragma unroll
    for (int c = 0; c < SP_NC; ++c) acc[c] = wave_sum(acc[c]);
    if (lane != 0) return;
    double* o = out + ostride * p;
#pragma unroll
    for (int c = 0; c < SP_NC; ++c) o[c] = acc[c];
    if (stage < 0 || stage > 2) return;
    const double m = sqrt(acc[0] * acc[0] + acc[1] * acc[1] + acc[2] * acc[2]);
    const double cb = (stage == 2) ? h : 0.5 * h;
    double* xs = pts + pstride * p;
    const double* x0 = xs - 3 * stage;   // the step's own point
    xs[3] = x0[0] + cb * dir * acc[0] / m;
    xs[4] = x0[1] + cb * dir * acc[1] / m;
    xs[5] = x0[2] + cb * dir * acc[2] / m;
}

// the first stage point of every step of line lines[blockIdx.x]: its x_n
__global__ __launch_bounds__(256) void k_sp_points(const int32_t* __restrict__ lines, const int32_t* __restrict__ ns,
                                                   const double* __restrict__ path, int64_t pstride,
                                                   const int64_t* __restrict__ sbase, double* __restrict__ SX) {
    const int64_t l = lines[blockIdx.x];
    for (int64_t e = threadIdx.x; e < 3 * (int64_t)ns[l]; e += 256) {
        const int64_t n = e / 3, k = e % 3;
        SX[3 * (sbase[l] + 4 * n) + k] = path[l * pstride + e];
    }
}

// The reverse recursion of line lines[blockIdx.x], one wave: lane = (step, stage) of a chunk of
// SP_STEPS steps prepares what does not depend on the adjoint state, lane 0 runs the chunk's steps
// backwards, and the lanes write the field sensitivities.  A chain of about 60 dependent FP64
// operations a step; EH[(record - r0)][9].
__global__ __launch_bounds__(64) void k_sp_adjoint(const int32_t* __restrict__ lines, const int32_t* __restrict__ ns,
                                                   const int64_t* __restrict__ sbase, int64_t r0, LAArgs a,
                                                   const double* __restrict__ EH, const double* __restrict__ gI,
                                                   double* __restrict__ SE, double* __restrict__ x0bar) {
    __shared__ double su[SP_STEPS][4][11];   // e (3), 1 / |E|, g c_s alpha', H (6)
    __shared__ double se[SP_STEPS][4][3];
    const int lane = threadIdx.x;
    const int64_t l = lines[blockIdx.x];
    const int32_t n1 = ns[l];
    const double h = a.h, g = gI[l];
    const double cst[4] = {h / 6.0, h / 3.0, h / 3.0, h / 6.0};
    const double cback[4] = {0.0, 0.5 * h, 0.5 * h, h};   // X_s = x + cback[s] k_{s-1}
    double xb0 = 0.0, xb1 = 0.0, xb2 = 0.0;
    for (int32_t hi = n1; hi > 0; hi -= SP_STEPS) {
        const int32_t lo = hi > SP_STEPS ? hi - SP_STEPS : 0;
        const int ks = lane >> 2, st = lane & 3;
        const int64_t r = sbase[l] + 4 * (int64_t)(lo + ks) + st;
        if (lo + ks < hi) {
            const double* e = EH + (r - r0) * SP_NC;
            const double e0 = e[0], e1 = e[1], e2 = e[2];
            const double m = sqrt(e0 * e0 + e1 * e1 + e2 * e2);
            const double im = 1.0 / m;
            double* o = su[ks][st];
            o[0] = e0 * im;
            o[1] = e1 * im;
            o[2] = e2 * im;
            o[3] = im;
            o[4] = g * cst[st] * la_dalpha(a, m);
#pragma unroll
            for (int c = 0; c < 6; ++c) o[5 + c] = e[3 + c];
        }
        __syncthreads();
        if (lane == 0) {
            for (int q = hi - lo - 1; q >= 0; --q) {
                double kb[4][3];
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    kb[s][0] = cst[s] * xb0;
                    kb[s][1] = cst[s] * xb1;
                    kb[s][2] = cst[s] * xb2;
                }
#pragma unroll
                for (int s = 3; s >= 0; --s) {
                    const double* o = su[q][s];
                    const double u0 = o[0], u1 = o[1], u2 = o[2], im = o[3], ga = o[4];
                    const double uk = u0 * kb[s][0] + u1 * kb[s][1] + u2 * kb[s][2];
                    const double eb0 = a.dir * (kb[s][0] - u0 * uk) * im + ga * u0;
                    const double eb1 = a.dir * (kb[s][1] - u1 * uk) * im + ga * u1;
                    const double eb2 = a.dir * (kb[s][2] - u2 * uk) * im + ga * u2;
                    const double X0 = o[5] * eb0 + o[8] * eb1 + o[9] * eb2;
                    const double X1 = o[8] * eb0 + o[6] * eb1 + o[10] * eb2;
                    const double X2 = o[9] * eb0 + o[10] * eb1 + o[7] * eb2;
                    xb0 += X0;
                    xb1 += X1;
                    xb2 += X2;
                    if (s > 0) {
                        kb[s - 1][0] += cback[s] * X0;
                        kb[s - 1][1] += cback[s] * X1;
                        kb[s - 1][2] += cback[s] * X2;
                    }
                    se[q][s][0] = eb0;
                    se[q][s][1] = eb1;
                    se[q][s][2] = eb2;
                }
            }
        }
        __syncthreads();
        if (lo + ks < hi) {
#pragma unroll
            for (int c = 0; c < 3; ++c) SE[3 * r + c] = se[ks][st][c];
        }
        __syncthreads();
    }
    if (lane == 0) {
        x0bar[3 * l] = xb0;
        x0bar[3 * l + 1] = xb1;
        x0bar[3 * l + 2] = xb2;
    }
}

// E and H of one load case at P points pts[pstride p] (rec: its records): out[ostride p] (see k_sp_near)
void sp_fields(bem_ctx* c, const double* rec, const double* sigma, int64_t P, double* pts, int64_t pstride, bool rows,
               int64_t row0, int stage, double h, double dir, double* out, int64_t ostride) {
    const int64_t N = c->N, KS = ceil_div(N, SP_C);
    const int64_t pb = ceil_div(P, SP_T);
    // panel ranges for about 2048 blocks, of 64 panels at least
    int64_t K = std::max<int64_t>(1, std::min<int64_t>(2048 / pb, ceil_div(N, 64)));
    const int64_t span = ceil_div(ceil_div(N, K), SP_C) * SP_C;
    K = ceil_div(N, span);
    c->ad_part.alloc(sizeof(double) * SP_NC * (size_t)(K * P) + sizeof(uint32_t) * (size_t)(KS * P));
    double* part = c->ad_part.as<double>();
    uint32_t* mask = reinterpret_cast<uint32_t*>(part + SP_NC * (size_t)(K * P));
    hipLaunchKernelGGL(k_sp_far, dim3((unsigned)pb, (unsigned)K), dim3(SP_T), 0, c->stream, rec, N, P, span, KS, pts,
                       pstride, part, mask);
    BEM_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_sp_near, dim3((unsigned)ceil_div(P, 4)), dim3(256), 0, c->stream, P, K, KS, part, mask,
                       c->tri64.as<double>(), sigma, rows, row0, pts, pstride, stage, h, dir, out, ostride);
    BEM_CHECK_LAUNCH();
}

// points of one batch: grad_batch, and masks within 256 MiB
int64_t sp_batch(const bem_ctx* c, int64_t P) {
    const int64_t KS = ceil_div(c->N, SP_C);
    const int64_t fit = std::max<int64_t>(1024, ((int64_t)256 << 20) / (4 * KS));
    return std::min<int64_t>(P, std::min<int64_t>(fit, c->grad_batch));
}

}  // namespace

// Reverse sweep over the lines whose forward run left n_steps and path (stride pstride); order:
// the lines by load case (those of case r from obeg[r] on, host and device), their stage records
// one after another in this order, sbase[l] + 4 n + s (rbeg[r]: the first record of case r).
// Writes SX, SE and x0bar[l] (adjoint of the start; 0 where no step was accepted).
void launch_reverse_sweep(bem_ctx* c, int32_t nrhs, const double* sol, const std::vector<int32_t>& order,
                          const std::vector<int64_t>& obeg, const int32_t* d_order, const std::vector<int32_t>& h_ns,
                          const std::vector<int64_t>& h_sbase, const int32_t* ns, const double* path, int64_t pstride,
                          const bem_trace_params* tp, const double* gI, const int64_t* sbase, double* SX, double* SE,
                          double* x0bar) {
    KTimer t(c, "grad_reverse");
    LAArgs a;
    a.h = tp->h;
    a.dir = tp->direction >= 0 ? 1.0 : -1.0;
    a.a = tp->alpha_a;
    a.e0 = tp->alpha_e0;
    a.p = tp->alpha_p;
    // lines whose fields are held at a time: at most about a million steps (288 bytes each), eight
    // batches of points
    const int64_t held = 8 * (int64_t)c->grad_batch;
    for (int32_t r = 0; r < nrhs; ++r) {
        const int64_t o1 = obeg[r + 1];
        if (obeg[r] == o1) continue;
        const double* sigma = sol + (int64_t)r * c->n;
        launch_median_records(c, sigma, c->ad_rec);
        for (int64_t oa = obeg[r]; oa < o1;) {
            int64_t ob = oa, steps = 0;
            while (ob < o1 && (ob == oa || steps + h_ns[order[ob]] <= held)) steps += h_ns[order[ob++]];
            const int64_t r0 = h_sbase[order[oa]];
            if (steps > 0) {
                hipLaunchKernelGGL(k_sp_points, dim3((unsigned)(ob - oa)), dim3(256), 0, c->stream, d_order + oa, ns,
                                   path, pstride, sbase, SX);
                BEM_CHECK_LAUNCH();
                c->ad_state.alloc(sizeof(double) * SP_NC * 4 * (size_t)steps);
                double* EH = c->ad_state.as<double>();
                const int64_t B = sp_batch(c, steps);
                for (int64_t q = 0; q < steps; q += B) {
                    const int64_t nb = std::min<int64_t>(B, steps - q);
                    for (int s = 0; s < 4; ++s)
                        sp_fields(c, c->ad_rec.as<double>(), sigma, nb, SX + 3 * (r0 + 4 * q + s), 12, false, 0, s,
                                  a.h, a.dir, EH + SP_NC * (4 * q + s), 4 * SP_NC);
                }
            }
            hipLaunchKernelGGL(k_sp_adjoint, dim3((unsigned)(ob - oa)), dim3(64), 0, c->stream, d_order + oa, ns, sbase,
                               r0, a, c->ad_state.as<double>(), gI, SE, x0bar);
            BEM_CHECK_LAUNCH();
            oa = ob;
        }
    }
}

// E and H (9 values per row, without the row's own panel) at the centroids pts of rows
// [0, P) of the collocation system, for charge sigma; out [P][9].
void launch_rows_EH(bem_ctx* c, const double* sigma, int64_t P, double* pts, double* out) {
    if (P == 0) return;
    KTimer t(c, "grad_rows_EH");
    launch_median_records(c, sigma, c->ad_rec);
    const int64_t B = sp_batch(c, P);
    for (int64_t p0 = 0; p0 < P; p0 += B)
        sp_fields(c, c->ad_rec.as<double>(), sigma, std::min<int64_t>(B, P - p0), pts + 3 * p0, 3, true, p0, -1, 0.0, 1.0,
                  out + SP_NC * p0, SP_NC);
}

}  // namespace bem
