// Nodal piecewise-linear basis with vertex collocation (Sec. 3; the matrix of
// Eq. Matrix).  sigma_h = sum_k u_k psi_k with psi_k the hat of vertex k;
// row i collocates at vertex x_i, so
//   v_ik = sum over the triangles tau holding k of int lambda_k^tau(y) / (4 pi |x_i - y|) dS,
// lambda_k^tau being tau's barycentric coordinate of k.  Conductor and
// floating-conductor bodies; a floating body's row is its net charge.
//
// Assembly keeps the collision-free ownership of Sec. 4 (each collocation
// point owns its row) at wave granularity: the 64 lanes of a wave are 64
// consecutive rows, while the column and the triangle are wave-uniform, so
// triangle records arrive through the scalar cache and every lane adds into
// its own row only.  A column is summed over the fan of its vertex (a CSR
// built at create), so each entry is written once, with no read-modify-write
// and no atomics; the price is that a regular (row, triangle) pair is
// integrated once per vertex of the triangle.  16 columns per wave are staged
// in LDS and leave as 128-byte row segments (64 bytes when the rows are stored
// in FP32, MIXED precision).  This pass takes the regular
// pairs only; the near-singular and singular ones (a small fraction, each a
// long closed form) follow in a second pass with one wave per row, which adds
// all three hats of the near triangles into its row, so the first pass keeps
// few registers and many waves in flight.
#include <cmath>
#include <type_traits>

#include "bem_device.h"
#include "median_device.h"
#include "nodal_device.h"

namespace bem {
namespace {

// Closed form of int lambda_c(y) / (4 pi |x - y|) dS over the flat triangle T
// (16-double exact-geometry record) for its local vertex c.  With rho the foot
// point of x on the plane and w the height,
//   lambda_c(y) = lambda_c(rho) + g_c . (y - rho),  g_c = n x (v_{c+2} - v_{c+1}) / (2A),
//   int 1/R dS = sum_e t f_e - |w| Omega                 (unit density),
//   int (y - rho)/R dS = sum_e m_e int_e R dl,  int_e R dl = (s+ R+ - s- R- + R0^2 f_e)/2,
// the second by the divergence theorem in the plane (the in-plane gradient of
// R is (y - rho)/R); edge notation and Omega as in flat_tri_SF.  vtx: x is a
// vertex of T, so w = 0 and rho = x; on the two edges that end at x, t = R0 = 0
// and their t f_e and R0^2 f_e terms vanish in the limit (f_e itself is
// infinite there), so they are skipped.
__device__ __forceinline__ void hat_edges(const double* __restrict__ T, double x0, double x1, double x2, bool vtx,
                                          double& I0, double& r0, double& r1, double& r2, double& J0, double& J1,
                                          double& J2) {
    const double n0 = T[TR_N + 0], n1 = T[TR_N + 1], n2 = T[TR_N + 2];
    const double w = vtx ? 0.0 : (x0 - T[0]) * n0 + (x1 - T[1]) * n1 + (x2 - T[2]) * n2;
    r0 = x0 - w * n0;
    r1 = x1 - w * n1;
    r2 = x2 - w * n2;
    const double aw = fabs(w);
    double V[3][3], Rv[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        V[k][0] = T[3 * k] - x0;
        V[k][1] = T[3 * k + 1] - x1;
        V[k][2] = T[3 * k + 2] - x2;
        Rv[k] = sqrt(V[k][0] * V[k][0] + V[k][1] * V[k][1] + V[k][2] * V[k][2]);
    }
    double st = 0.0;
    J0 = J1 = J2 = 0.0;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const int b = (e + 1) % 3;
        const double ax = T[3 * e], ay = T[3 * e + 1], az = T[3 * e + 2];
        double l0 = T[3 * b] - ax, l1 = T[3 * b + 1] - ay, l2 = T[3 * b + 2] - az;
        const double len = sqrt(l0 * l0 + l1 * l1 + l2 * l2);
        const double il = 1.0 / len;
        l0 *= il; l1 *= il; l2 *= il;
        const double m0 = l1 * n2 - l2 * n1, m1 = l2 * n0 - l0 * n2, m2 = l0 * n1 - l1 * n0;
        const double q0 = ax - r0, q1 = ay - r1, q2 = az - r2;
        const double sm = q0 * l0 + q1 * l1 + q2 * l2;
        const double sp = sm + len;
        const double t = q0 * m0 + q1 * m1 + q2 * m2;
        const double Rm = Rv[e], Rp = Rv[b];
        double er = 0.5 * (sp * Rp - sm * Rm);
        if (!(vtx && (Rm == 0.0 || Rp == 0.0))) {
            double f;
            if (sm < 0.0 && sp > 0.0)   // foot within the edge's span (see flat_tri_SF)
                f = log((Rp + sp) * (Rm - sm) / (t * t + w * w));
            else if (sp + sm > 0.0)
                f = log((Rp + sp) / (Rm + sm));
            else
                f = log((Rm - sm) / (Rp - sp));
            st += t * f;
            er += 0.5 * (t * t + w * w) * f;
        }
        J0 += m0 * er;
        J1 += m1 * er;
        J2 += m2 * er;
    }
    double omega = 0.0;
    if (!vtx) {
        const double c0 = V[1][1] * V[2][2] - V[1][2] * V[2][1];
        const double c1 = V[1][2] * V[2][0] - V[1][0] * V[2][2];
        const double c2 = V[1][0] * V[2][1] - V[1][1] * V[2][0];
        const double triple = V[0][0] * c0 + V[0][1] * c1 + V[0][2] * c2;
        const double d01 = V[0][0] * V[1][0] + V[0][1] * V[1][1] + V[0][2] * V[1][2];
        const double d02 = V[0][0] * V[2][0] + V[0][1] * V[2][1] + V[0][2] * V[2][2];
        const double d12 = V[1][0] * V[2][0] + V[1][1] * V[2][1] + V[1][2] * V[2][2];
        const double den = Rv[0] * Rv[1] * Rv[2] + d01 * Rv[2] + d02 * Rv[1] + d12 * Rv[0];
        omega = 2.0 * atan2(fabs(triple), den);
    }
    I0 = st - aw * omega;
}

// Local corner of the triangle T at x, by position: within 1e-13 of T's longest edge; -1 if none
// (a vertex of another body that coincides with a corner of T)
__device__ __forceinline__ int coincident_corner(const double* __restrict__ T, double x0, double x1, double x2) {
    double L2 = 0.0;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const int b = (e + 1) % 3;
        const double d0 = T[3 * b] - T[3 * e], d1 = T[3 * b + 1] - T[3 * e + 1], d2 = T[3 * b + 2] - T[3 * e + 2];
        const double l2 = d0 * d0 + d1 * d1 + d2 * d2;
        L2 = l2 > L2 ? l2 : L2;
    }
    const double tol2 = 1e-26 * L2;
#pragma unroll
    for (int cv = 0; cv < 3; ++cv) {
        const double d0 = x0 - T[3 * cv], d1 = x1 - T[3 * cv + 1], d2 = x2 - T[3 * cv + 2];
        if (d0 * d0 + d1 * d1 + d2 * d2 <= tol2) return cv;
    }
    return -1;
}

// lambda_c(rho) I0 + g_c . J over 4 pi (see hat_edges)
__device__ __forceinline__ double hat_value(const double* __restrict__ T, int c, double I0, double r0, double r1,
                                           double r2, double J0, double J1, double J2) {
    const double n0 = T[TR_N + 0], n1 = T[TR_N + 1], n2 = T[TR_N + 2];
    const double* p = T + 3 * ((c + 1) % 3);
    const double* q = T + 3 * ((c + 2) % 3);
    const double a0 = p[0] - r0, a1 = p[1] - r1, a2 = p[2] - r2;
    const double b0 = q[0] - r0, b1 = q[1] - r1, b2 = q[2] - r2;
    const double two_area = 2.0 * T[TR_A];
    // barycentric coordinate of rho: signed area of (p, q, rho) over A
    const double lam = (n0 * (a1 * b2 - a2 * b1) + n1 * (a2 * b0 - a0 * b2) + n2 * (a0 * b1 - a1 * b0)) / two_area;
    // g = n x (q - p)
    const double e0 = q[0] - p[0], e1 = q[1] - p[1], e2 = q[2] - p[2];
    const double g0 = n1 * e2 - n2 * e1, g1 = n2 * e0 - n0 * e2, g2 = n0 * e1 - n1 * e0;
    return (lam * I0 + (g0 * J0 + g1 * J1 + g2 * J2) / two_area) * INV4PI;
}

// The rule's barycentric coordinate of local vertex c at node q (node order of
// the panel records: centroid, then the orbits (a, a, 1 - 2a) for a = a1, a2
// with the odd coordinate last, middle, first).
struct NodeBary {
    double b[7];
    __device__ NodeBary(int c) {
        const double s15 = sqrt(15.0);
        const double a1 = (6.0 - s15) / 21.0, a2 = (6.0 + s15) / 21.0;
        b[0] = 1.0 / 3.0;
#pragma unroll
        for (int q = 1; q <= 3; ++q) b[q] = (c == 3 - q) ? 1.0 - 2.0 * a1 : a1;
#pragma unroll
        for (int q = 4; q <= 6; ++q) b[q] = (c == 6 - q) ? 1.0 - 2.0 * a2 : a2;
    }
};

// Regular pairs of the vertex rows (KP false) or of the centroid rows below (KP true: x the centroid of
// triangle trow[i], the kernel n . (x - y)/|x - y|^3 in place of 1/|x - y|).
// One wave: rows i0 + lane, the 16 columns of column group cg (neighbouring vertices).  The wave walks the
// distinct triangles that hold a vertex of the group (ascending), evaluates the 7-point
// rule once per triangle and adds each hat whose vertex is in the group into that column's
// LDS slot, so a pair costs about 1.7 visits instead of one per vertex of the triangle.
// The four waves of a block take the same columns on four row tiles, so three of four
// record loads hit the scalar cache.  1-D grid of n_rt x n_cg blocks (row tiles of 256
// rows, n_cg a multiple of 8): blocks are dealt to the 8 XCDs in turn, so block b runs on
// XCD b % 8, and each XCD sweeps all row tiles of one column group before the next,
// keeping that group's records in its own L2; it takes consecutive groups, whose columns
// share lines of the matrix.
// The rule is the form about the centroid (density one in the records).  Corner k's hat is 1/3 at the
// centroid and 1/3 + s (delta_ik - 1/3) at the node on corner i's median (s the median's scale, s rho
// on the second orbit), so with f_q the kernel at the nodes, U = sum w f and h_i = w_1 f_1i + rho w_2
// f_2i its integral is U / 3 + s (h_k - (h_0 + h_1 + h_2) / 3).  A corner lies within reach of its
// triangle, so corners are looked for only there.  Bound by FP64 issue; the next triangle's record is
// requested before a triangle's arithmetic.  9,036 vertices, 18,064 triangles: 1.17 ms; node by node, with
// groups of consecutive vertices (2.03 visits) and no request ahead, 1.77.
// NODES (MIXED, whose products take FP32 inputs and carry an ulp of the operator into the solutions of
// several load cases: gmres_batched.hip): node by node over the records pan64, every sum in the nodes' order.
template <class T, bool KP, bool NODES>   // T: stored type, double (FP64) or float (MIXED)
__global__ __launch_bounds__(256) void k_nodal_regular(int64_t nr, int64_t nv, int64_t ld, int64_t n_rt,
                                                       const double* __restrict__ vert,
                                                       const int32_t* __restrict__ trow,
                                                       const int32_t* __restrict__ tri,
                                                       const int32_t* __restrict__ grp_col,
                                                       const int32_t* __restrict__ grp_ptr,
                                                       const int32_t* __restrict__ grp_tri,
                                                       const uint32_t* __restrict__ grp_loc,
                                                       const double* __restrict__ rec,
                                                       const double* __restrict__ pan64,
                                                       const double* __restrict__ tri64, T* __restrict__ A) {
    constexpr int PF = MD_REACH + 1;             // the part of a record that every pair reads
    __shared__ double tile[4][NODAL_COLS][65];   // padded: the row-segment reads stride 65
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t b = blockIdx.x, xcd = b & 7, slot = b >> 3;
    const int64_t cg = xcd * ((int64_t)gridDim.x / (8 * n_rt)) + slot / n_rt, rt = slot % n_rt;
    const int64_t i0 = (rt * 4 + wv) * 64;
    const int64_t i = i0 + lane;
    const int64_t ic = i < nr ? i : nr - 1;
    const int64_t own = KP ? trow[ic] : -1;
    const double* X = KP ? tri64 + (int64_t)TRI_REC * own : vert + 3 * ic;
    const double x0 = X[KP ? TR_C : 0], x1 = X[KP ? TR_C + 1 : 1], x2 = X[KP ? TR_C + 2 : 2];
    const double n0 = KP ? X[TR_N] : 0.0, n1 = KP ? X[TR_N + 1] : 0.0, n2 = KP ? X[TR_N + 2] : 0.0;
    const int64_t j0 = cg * NODAL_COLS;
#pragma unroll
    for (int cc = 0; cc < NODAL_COLS; ++cc) tile[wv][cc][lane] = 0.0;
    const int32_t e0 = j0 < nv ? grp_ptr[cg] : 0, e1 = j0 < nv ? grp_ptr[cg + 1] : 0;
    MedConst k = med_consts();
    // in vector registers: two records and the pointers fill the scalar ones
    asm volatile("" : "+v"(k.m2rho), "+v"(k.rho2), "+v"(k.kap), "+v"(k.kap0), "+v"(k.kaprho), "+v"(k.c1875), "+v"(k.rho));
    auto visit = [&](int64_t t, uint32_t loc, const double (&v)[PF]) {
        const double t0 = x0 - v[0], t1 = x1 - v[1], t2 = x2 - v[2];
        const double TT = __fma_rn(t0, t0, __fma_rn(t1, t1, t2 * t2));
        bool reg = TT > v[MD_REACH];
        if (!reg) {   // near and singular pairs are left to k_nodal_near (same predicate)
            const double* r = rec + (int64_t)MED_REC * t;
            reg = is_regular(x0 - r[MD_CC], x1 - r[MD_CC + 1], x2 - r[MD_CC + 2], r[MD_RR]);
            if constexpr (KP) {
                reg = reg && t != own;
            } else {
                const int32_t* tv = tri + 3 * t;
                reg = reg && tv[0] != i && tv[1] != i && tv[2] != i;
            }
        }
        if (!reg) return;
        const double pa = __fma_rn(t0, v[3], __fma_rn(t1, v[4], t2 * v[5]));
        const double pb = __fma_rn(t0, v[6], __fma_rn(t1, v[7], t2 * v[8]));
        const double pc = -(pa + pb);
        const double r2[7] = {TT,
                              __fma_rn(-2.0, pa, TT + v[9]),
                              __fma_rn(-2.0, pb, TT + v[10]),
                              __fma_rn(-2.0, pc, TT + v[11]),
                              __fma_rn(k.m2rho, pa, __fma_rn(k.rho2, v[9], TT)),
                              __fma_rn(k.m2rho, pb, __fma_rn(k.rho2, v[10], TT)),
                              __fma_rn(k.m2rho, pc, __fma_rn(k.rho2, v[11], TT))};
        double f[7];
        if constexpr (KP) {
            const double nt = __fma_rn(n0, t0, __fma_rn(n1, t1, n2 * t2));
            const double na = __fma_rn(n0, v[3], __fma_rn(n1, v[4], n2 * v[5]));
            const double nb = __fma_rn(n0, v[6], __fma_rn(n1, v[7], n2 * v[8]));
            const double nc = -(na + nb);
            f[0] = nt * med_r3(r2[0], k);
            f[1] = (nt - na) * med_r3(r2[1], k);
            f[2] = (nt - nb) * med_r3(r2[2], k);
            f[3] = (nt - nc) * med_r3(r2[3], k);
            f[4] = __fma_rn(-k.rho, na, nt) * med_r3(r2[4], k);
            f[5] = __fma_rn(-k.rho, nb, nt) * med_r3(r2[5], k);
            f[6] = __fma_rn(-k.rho, nc, nt) * med_r3(r2[6], k);
        } else {
#pragma unroll
            for (int q = 0; q < 7; ++q) f[q] = rsqrt_pos(r2[q]);
        }
        const double U = __fma_rn(k.kap0, f[0], __fma_rn(k.kap, (f[4] + f[5]) + f[6], (f[1] + f[2]) + f[3]));
        const double h0 = __fma_rn(k.kaprho, f[4], f[1]), h1 = __fma_rn(k.kaprho, f[5], f[2]);
        const double h2 = __fma_rn(k.kaprho, f[6], f[3]);
        const double hs = v[MD_DENS] * MED_SC;
        const double base = (v[MD_DENS] * (1.0 / 3.0)) * __fma_rn(-MED_SC, (h0 + h1) + h2, U);
        const uint32_t l0 = loc & 0xffu, l1 = (loc >> 8) & 0xffu, l2 = (loc >> 16) & 0xffu;
        if (l0 != 0xffu) tile[wv][l0][lane] += __fma_rn(hs, h0, base);
        if (l1 != 0xffu) tile[wv][l1][lane] += __fma_rn(hs, h1, base);
        if (l2 != 0xffu) tile[wv][l2][lane] += __fma_rn(hs, h2, base);
    };
    if constexpr (NODES) {
        const NodeBary nb0(0), nb1(1), nb2(2);
        for (int32_t e = e0; e < e1; ++e) {
            const int64_t t = grp_tri[e];
            const uint32_t loc = grp_loc[e];
            const double* P = pan64 + (int64_t)FAR_REC * t;
            const int32_t* tv = tri + 3 * t;
            const bool mine = KP ? t == own : (tv[0] == i || tv[1] == i || tv[2] == i);
            if (mine || !is_regular(x0 - P[FR_CC], x1 - P[FR_CC + 1], x2 - P[FR_CC + 2], P[FR_RR])) continue;
            double f[7], w[7];
#pragma unroll
            for (int q = 0; q < 7; ++q) {
                const double d0 = x0 - P[FR_X + q], d1 = x1 - P[FR_Y + q], d2 = x2 - P[FR_Z + q];
                const double ir = rsqrt_pos(d0 * d0 + d1 * d1 + d2 * d2);
                w[q] = P[FR_W + q];
                f[q] = KP ? w[q] * (d0 * n0 + d1 * n1 + d2 * n2) * (ir * ir * ir) : ir;
            }
            auto hat = [&](uint32_t l, const NodeBary& nb) {
                if (l == 0xffu) return;
                double s = 0.0;
#pragma unroll
                for (int q = 0; q < 7; ++q) s += KP ? f[q] * nb.b[q] : w[q] * nb.b[q] * f[q];
                tile[wv][l][lane] += s;
            };
            hat(loc & 0xffu, nb0);
            hat((loc >> 8) & 0xffu, nb1);
            hat((loc >> 16) & 0xffu, nb2);
        }
    } else if (e0 < e1) {
        auto fetch = [&](int64_t t, double (&v)[PF]) {
            const double* r = rec + (int64_t)MED_REC * t;
#pragma unroll
            for (int c = 0; c < PF; ++c) v[c] = r[c];
        };
        auto at = [&](int32_t e) { return e < e1 ? e : e1 - 1; };
        double vA[PF], vB[PF];
        int32_t tA = grp_tri[e0], tB = grp_tri[at(e0 + 1)];
        uint32_t lA = grp_loc[e0], lB = grp_loc[at(e0 + 1)];
        fetch(tA, vA);
        for (int32_t e = e0; e < e1; e += 2) {
            wait_scalar();
            const int32_t tC = grp_tri[at(e + 2)], tD = grp_tri[at(e + 3)];
            const uint32_t lC = grp_loc[at(e + 2)], lD = grp_loc[at(e + 3)];
            fetch(tB, vB);
            visit(tA, lA, vA);
            wait_scalar();
            fetch(tC, vA);
            if (e + 1 < e1) visit(tB, lB, vB);
            tA = tC;
            tB = tD;
            lA = lC;
            lB = lD;
        }
    }
    __syncthreads();
    const int cc = lane % NODAL_COLS;
    if (j0 + cc >= nv) return;
    const int64_t jj = grp_col[j0 + cc];
#pragma unroll 4
    for (int s = 0; s < NODAL_COLS; ++s) {
        const int r = lane / NODAL_COLS + 64 / NODAL_COLS * s;
        if (i0 + r < nr) A[(i0 + r) * ld + jj] = (T)tile[wv][cc][r];
    }
}

// Bound of each chunk of 64 consecutive triangles: a centre and a radius such
// that every point within eta R of a circumcentre of the chunk lies in the ball
// (radius = max |cc - centre| + eta R), so a ball of rows apart from it by more
// than the two radii makes only regular pairs with the chunk.
// One wave per chunk.
__global__ __launch_bounds__(256) void k_nodal_chunk_bounds(int64_t N, int64_t Np, const double* __restrict__ far64,
                                                            double* __restrict__ cb) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, ch = t >> 6;
    if (ch * 64 >= N) return;   // whole waves
    const bool live = t < N;
    double c[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) c[k] = live ? far64[(int64_t)(FR_CC + k) * Np + t] : 0.0;
    const double inv = 1.0 / (double)(N - ch * 64 < 64 ? N - ch * 64 : 64);
    double d2 = 0.0, m[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        m[k] = wave_sum(c[k]) * inv;
        d2 += (c[k] - m[k]) * (c[k] - m[k]);
    }
    double r = live ? sqrt(d2) + sqrt(far64[(int64_t)FR_RR * Np + t]) : 0.0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double v = __shfl_xor(r, o, 64);
        r = v > r ? v : r;
    }
    if ((threadIdx.x & 63) != 0) return;
    cb[4 * ch] = m[0];
    cb[4 * ch + 1] = m[1];
    cb[4 * ch + 2] = m[2];
    cb[4 * ch + 3] = r;
}

constexpr int NN_H = 256;   // slots of a wave's column table (192 columns at most: 64 triangles a round)

// Near-singular and singular pairs of one row, by one wave: the vertex rows (KP false: x the vertex
// i, hats by hat_edges) or the centroid rows below (KP true: x the centroid of triangle trow[i] with
// its normal, the hats' normal field).
// The lanes test 64 chunk bounds at a time; of the chunks within reach they classify the 64 triangles
// with the predicate of the regular pass, and the near ones queue up, ascending.  A round takes 64 of
// them, one closed form per lane.  Their hats meet in the row's entries, up to six triangles an entry:
// the round's distinct columns go into a table in LDS, and each column's lane adds its hats in the
// triangles' order, rounding to the stored type after each, as one lane walking the triangles would
// (so FP32 rows hold the same bits).  One lane per row, the earlier form, ran each closed form for a
// few lanes at a time and had 141 waves for 9,036 rows: 4.0 ms, where this takes 0.24 (0.39 with 192
// registers, two waves a SIMD, one chunk of triangles at a time and every column walking the whole round).
template <class T, bool KP>
__global__ __launch_bounds__(64, 3) void k_nodal_near(int64_t nr, int64_t ld, int64_t N, int64_t Np,
                                                   const int32_t* __restrict__ row_order,
                                                   const double* __restrict__ vert, const int32_t* __restrict__ trow,
                                                   const int32_t* __restrict__ tri, const double* __restrict__ far64,
                                                   const double* __restrict__ cb, const double* __restrict__ tri64,
                                                   T* __restrict__ A) {
    __shared__ int32_t lt[192];            // near triangles waiting, ascending
    __shared__ int32_t hkey[NN_H], used[192], s_used;
    __shared__ uint32_t hits[2][NN_H];     // a column's triangles of the round
    __shared__ uint32_t eslot[64];         // slots of a triangle's three columns, 8 bits each
    __shared__ double ev[3][64];
    const int lane = threadIdx.x;
    // blocks go to the 8 XCDs in turn: XCD x takes a contiguous part of the rows' spatial order, so
    // that neighbours' triangle records share its L2
    const int64_t per = (nr + 7) / 8, sx = (int64_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if ((int64_t)(blockIdx.x >> 3) >= per || sx >= nr) return;
    const int64_t i = KP ? sx : row_order[sx];
    const int64_t own = KP ? trow[i] : -1;
    const double* Tx = tri64 + (int64_t)TRI_REC * (KP ? own : 0);
    const double x0 = KP ? Tx[TR_C] : vert[3 * i], x1 = KP ? Tx[TR_C + 1] : vert[3 * i + 1],
                 x2 = KP ? Tx[TR_C + 2] : vert[3 * i + 2];
    T* row = A + i * ld;
    const int64_t nch = (N + 63) >> 6;
    int m = 0;             // triangles waiting
    int64_t cbase = -64;
    uint64_t todo = 0;     // chunks of [cbase, cbase + 64) within reach, not yet classified
    auto near_of = [&](int64_t t) {   // t >= N: some triangle's answer
        t = t < N ? t : N - 1;
        const double c0 = far64[(int64_t)(FR_CC + 0) * Np + t], c1 = far64[(int64_t)(FR_CC + 1) * Np + t],
                     c2 = far64[(int64_t)(FR_CC + 2) * Np + t], rr = far64[(int64_t)FR_RR * Np + t];
        if constexpr (KP) {
            return !is_regular(x0 - c0, x1 - c1, x2 - c2, rr) && t != own;
        } else {
            const int32_t v0 = tri[3 * t], v1 = tri[3 * t + 1], v2 = tri[3 * t + 2];
            return !is_regular(x0 - c0, x1 - c1, x2 - c2, rr) || v0 == i || v1 == i || v2 == i;
        }
    };
    auto below = [&](uint64_t w) {   // bits of w below this lane
        return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(w >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)w, 0u));
    };
    for (;;) {
        while (m < 64) {
            while (todo == 0 && cbase + 64 < nch) {
                cbase += 64;
                const int64_t ch = cbase + lane;
                bool in = false;
                if (ch < nch) {
                    const double* Bd = cb + 4 * ch;
                    const double e0 = Bd[0] - x0, e1 = Bd[1] - x1, e2 = Bd[2] - x2;
                    const double reach = Bd[3] * (1.0 + 1e-9) + 1e-300;
                    in = !(e0 * e0 + e1 * e1 + e2 * e2 > reach * reach);
                }
                todo = __ballot(in);
            }
            if (todo == 0) break;
            // two chunks at a time, their loads in flight together
            const int64_t ta = (cbase + __builtin_ctzll(todo)) * 64 + lane;
            todo &= todo - 1;
            const int64_t tb = todo != 0 ? (cbase + __builtin_ctzll(todo)) * 64 + lane : N;
            todo &= todo - 1;   // 0 stays 0
            bool na = near_of(ta), nb = near_of(tb);
            na = na && ta < N;
            nb = nb && tb < N;
            const uint64_t ma = __ballot(na), mb = __ballot(nb);
            if (na) lt[m + below(ma)] = (int32_t)ta;
            m += __popcll(ma);
            if (nb) lt[m + below(mb)] = (int32_t)tb;
            m += __popcll(mb);
        }
        if (m == 0) break;
        const int n = m < 64 ? m : 64;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NN_H / 64; ++k) {
            hkey[lane + 64 * k] = -1;
            hits[0][lane + 64 * k] = 0;
            hits[1][lane + 64 * k] = 0;
        }
        if (lane == 0) s_used = 0;
        __syncthreads();
        if (lane < n) {
            const int64_t t = lt[lane];
            const double* Tr = tri64 + (int64_t)TRI_REC * t;
            uint32_t slots = 0;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int32_t col = tri[3 * t + c];
                uint32_t h = ((uint32_t)col * 2654435761u) >> 24;
                for (;;) {   // fewer columns than slots: a free or equal one is found
                    const int32_t k = atomicCAS(&hkey[h], -1, col);
                    if (k == -1) used[atomicAdd(&s_used, 1)] = (int32_t)h;
                    if (k == -1 || k == col) break;
                    h = (h + 1) & (NN_H - 1);
                }
                atomicOr(&hits[lane >> 5][h], 1u << (lane & 31));
                slots |= h << (8 * c);
            }
            eslot[lane] = slots;
            double out[3] = {0.0, 0.0, 0.0};
            if constexpr (KP) {
                nodal_tri_hats_nE(Tr, x0, x1, x2, Tx[TR_N], Tx[TR_N + 1], Tx[TR_N + 2], out);
            } else {
                bool vtx = tri[3 * t] == i || tri[3 * t + 1] == i || tri[3 * t + 2] == i;
                // a vertex of another body at x (bodies that touch): the singular closed form at
                // that vertex's own position
                double xs0 = x0, xs1 = x1, xs2 = x2;
                if (!vtx) {
                    const int cv = coincident_corner(Tr, x0, x1, x2);
                    if (cv >= 0) {
                        vtx = true;
                        xs0 = Tr[TR_V + 3 * cv];
                        xs1 = Tr[TR_V + 3 * cv + 1];
                        xs2 = Tr[TR_V + 3 * cv + 2];
                    }
                }
                double I0, r0, r1, r2, J0, J1, J2;
                hat_edges(Tr, xs0, xs1, xs2, vtx, I0, r0, r1, r2, J0, J1, J2);
#pragma unroll
                for (int c = 0; c < 3; ++c) out[c] = hat_value(Tr, c, I0, r0, r1, r2, J0, J1, J2);
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) ev[c][lane] = out[c];
        }
        __syncthreads();
        for (int u = lane; u < s_used; u += 64) {
            const uint32_t h = (uint32_t)used[u];
            T* out = row + hkey[h];
            double y = (double)*out;
            uint64_t w = (uint64_t)hits[1][h] << 32 | hits[0][h];
            while (w) {
                const int e = __builtin_ctzll(w);
                w &= w - 1;
                const uint32_t sl = eslot[e];
                const int c = (sl & 0xffu) == h ? 0 : ((sl >> 8) & 0xffu) == h ? 1 : 2;
                y = (double)(T)(y + ev[c][e]);
            }
            *out = (T)y;
        }
        const int left = m - n;
        const int32_t mv0 = lt[64 + lane], mv1 = lt[128 + lane];
        __syncthreads();   // and the row's entries are there for the next round's columns
        if (lane < left) lt[lane] = mv0;
        if (64 + lane < left) lt[64 + lane] = mv1;
        __syncthreads();
        m = left;
    }
}

// ---- rows that need n . E (interface vertices, literal Final4, sheets) ----------------
// A vertex of flat panels has no normal, so those rows take the normal field at the
// centroids x_T of triangles T (normal n_T): Kc[r][k] = n_T . (field of hat k over every
// triangle but T at x_T) for the centroid rows r (trow[r] = T), row stride ld.  T itself adds
// nothing (in its plane the field of its own density has no normal component).

// Interface vertex rows (Eq. nonconductors at the vertex, taken as the hat-weighted mean over
// the vertex's triangles T of the condition at x_T): one block per interface vertex i,
//   A[i][k] = sum_{T in fan(i)} (a_T/3)/m_i [ (eps+ - eps-) Kc[crow(T)][k]
//                                             + (eps+ + eps-)/2 [k in T]/3 ],
// m_i = sum over the fan of a_T/3; fan order, so the sums are reproducible.  Columns k < nv.
template <class TT>
__global__ __launch_bounds__(256) void k_nodal_iface_rows(int64_t nv, int64_t ld, const int32_t* __restrict__ iface_v,
                                                          const int32_t* __restrict__ fan_ptr,
                                                          const int32_t* __restrict__ fan,
                                                          const int32_t* __restrict__ tri,
                                                          const int32_t* __restrict__ tri_crow,
                                                          const int32_t* __restrict__ vert_body,
                                                          const double* __restrict__ epsp,
                                                          const double* __restrict__ epsm,
                                                          const double* __restrict__ tri64,
                                                          const double* __restrict__ mass,
                                                          const double* __restrict__ Kc, TT* __restrict__ A) {
    const int64_t i = iface_v[blockIdx.x];
    const int32_t bd = vert_body[i];
    const double dk = epsp[bd] - epsm[bd], hs = 0.5 * (epsp[bd] + epsm[bd]) / 3.0;
    const double inv_m = 1.0 / mass[i];
    const int32_t f0 = fan_ptr[i], f1 = fan_ptr[i + 1];
    for (int64_t k = threadIdx.x; k < nv; k += 256) {
        double acc = 0.0;
        for (int32_t e = f0; e < f1; ++e) {
            const int64_t t = fan[e] >> 2;
            const double wT = tri64[(int64_t)TRI_REC * t + TR_A] / 3.0 * inv_m;
            const int32_t* tv = tri + 3 * t;
            const double self = (tv[0] == k || tv[1] == k || tv[2] == k) ? hs : 0.0;
            acc += wT * (dk * Kc[(int64_t)tri_crow[t] * ld + k] + self);
        }
        A[i * ld + k] = (TT)acc;
    }
}

// Rows of floating bodies with a normal-field term (literal Eq. Final4, sheets), the centroid
// rule over the body's triangles: row f (stored at row0 + f)
//   A[k] = sum_{T in f} (a_T/area_f) [ c_kp Kc[crow(T)][k] + c_self [k in T]/3 ]
//        = c_kp sum_T (a_T/area_f) Kc[crow(T)][k] + c_self m_k/area_f [k on f],
// over the body's contiguous centroid rows [cr0, cr1) in order; 0 in columns >= nv; Jacobi
// diagonal 1 (the entry is 0).  grid (column chunks, bodies in the list).
__global__ __launch_bounds__(256) void k_nodal_kp_body_rows(int64_t nv, int64_t ld, int64_t row0,
                                                            const int32_t* __restrict__ flist,
                                                            const int32_t* __restrict__ frange,
                                                            const double* __restrict__ fcoef,
                                                            const int32_t* __restrict__ trow,
                                                            const int32_t* __restrict__ vert_body,
                                                            const int32_t* __restrict__ fidx,
                                                            const double* __restrict__ tri64,
                                                            const double* __restrict__ mass,
                                                            const double* __restrict__ Af,
                                                            const double* __restrict__ Kc, double* __restrict__ A,
                                                            double* __restrict__ diag) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int32_t f = flist[blockIdx.y];
    if (k >= ld) return;
    const double inv_a = 1.0 / Af[f];
    const double cs = fcoef[2 * f], ck = fcoef[2 * f + 1];
    double acc = 0.0;
    if (k < nv) {
        double s = 0.0;
        for (int32_t r = frange[2 * f]; r < frange[2 * f + 1]; ++r)
            s += tri64[(int64_t)TRI_REC * trow[r] + TR_A] * Kc[(int64_t)r * ld + k];
        acc = ck * s * inv_a + (fidx[vert_body[k]] == f ? cs * mass[k] * inv_a : 0.0);
    }
    A[(row0 + f) * ld + k] = acc;
    if (k == 0) diag[nv + f] = 1.0;
}

// Jacobi diagonal of the vertex rows
template <class T>
__global__ __launch_bounds__(256) void k_nodal_diag(int64_t nv, int64_t ld, const T* __restrict__ A,
                                                    double* __restrict__ diag) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < nv) diag[i] = (double)A[i * ld + i];
}

// columns [nv, ld) of the vertex rows: -1 in the column of the row's floating body, else 0
template <class T>
__global__ __launch_bounds__(256) void k_nodal_tail(int64_t nv, int64_t ld, const int32_t* __restrict__ vert_body,
                                                    const int32_t* __restrict__ body_kind,
                                                    const int32_t* __restrict__ fidx, T* __restrict__ A) {
    const int64_t ncol = ld - nv;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= nv * ncol) return;
    const int64_t i = t / ncol, k = t % ncol;
    const int32_t b = vert_body[i];
    A[i * ld + nv + k] = (T)((body_kind[b] == BEM_FLOATING && fidx[b] == k) ? -1.0 : 0.0);
}

// m_k = int psi_k dS = sum over the fan of k of area / 3
__global__ __launch_bounds__(256) void k_nodal_mass(int64_t nv, const int32_t* __restrict__ fan_ptr,
                                                    const int32_t* __restrict__ fan, const double* __restrict__ tri64,
                                                    double* __restrict__ mass) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= nv) return;
    double s = 0.0;
    for (int32_t e = fan_ptr[k]; e < fan_ptr[k + 1]; ++e) s += tri64[(int64_t)TRI_REC * (fan[e] >> 2) + TR_A];
    mass[k] = s / 3.0;
}

// area of floating body f (one block each): sum of m_k over its vertices, fixed order
__global__ __launch_bounds__(256) void k_nodal_body_area(int64_t nv, const int32_t* __restrict__ vert_body,
                                                         const int32_t* __restrict__ fidx,
                                                         const double* __restrict__ mass, double* __restrict__ Af) {
    __shared__ double red[4];
    const int f = blockIdx.x;
    double s = 0.0;
    for (int64_t k = threadIdx.x; k < nv; k += 256)
        if (fidx[vert_body[k]] == f) s += mass[k];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) Af[f] = (red[0] + red[1]) + (red[2] + red[3]);
}

// row nv + f (stored at row0 + f): m_k / area_f on the vertices of floating body f, 0
// elsewhere (all ld columns); its Jacobi diagonal is 1 (the entry is 0)
__global__ __launch_bounds__(256) void k_nodal_constraint(int64_t nv, int64_t row0, int64_t ld, int32_t n_float,
                                                          const int32_t* __restrict__ vert_body,
                                                          const int32_t* __restrict__ fidx,
                                                          const double* __restrict__ mass,
                                                          const double* __restrict__ Af, double* __restrict__ A,
                                                          double* __restrict__ diag) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (int64_t)n_float * ld) return;
    const int64_t f = t / ld, k = t % ld;
    A[(row0 + f) * ld + k] = (k < nv && fidx[vert_body[k]] == f) ? mass[k] / Af[f] : 0.0;
    if (k == 0) diag[nv + f] = 1.0;
}

// phi and E at volume points from vertex densities (the field formula closing
// Sec. 2): 64 points per block, the triangles split over the 4 waves, partial
// sums folded in LDS.  Regular pairs by the 7-point rule with the density at the
// nodes, the others by nodal_tri_phiE.  grid (point tiles, load cases); phi or E
// may be null.
__global__ __launch_bounds__(256) void k_nodal_field(int64_t P, const double* __restrict__ pts, int64_t N,
                                                     const int32_t* __restrict__ tri,
                                                     const double* __restrict__ pan64,
                                                     const double* __restrict__ tri64,
                                                     const double* __restrict__ sol, int64_t n,
                                                     double* __restrict__ phi, double* __restrict__ E) {
    __shared__ double part[4][4][64];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t p = (int64_t)blockIdx.x * 64 + lane;
    const int64_t pc = p < P ? p : P - 1;
    const double x0 = pts[3 * pc], x1 = pts[3 * pc + 1], x2 = pts[3 * pc + 2];
    const double* u = sol + (int64_t)blockIdx.y * n;
    const double s15 = sqrt(15.0);
    const double a1 = (6.0 - s15) / 21.0, a2 = (6.0 + s15) / 21.0;
    const double b1 = 1.0 - 2.0 * a1, b2 = 1.0 - 2.0 * a2;
    const int64_t per = (N + 3) / 4;
    const int64_t t0 = wv * per, t1 = t0 + per < N ? t0 + per : N;
    double ph = 0.0, e0 = 0.0, e1 = 0.0, e2 = 0.0;
    for (int64_t t = t0; t < t1; ++t) {
        const int32_t* tv = tri + 3 * t;
        const double u0 = u[tv[0]], u1 = u[tv[1]], u2 = u[tv[2]];
        const double* Pr = pan64 + (int64_t)FAR_REC * t;
        if (is_regular(x0 - Pr[FR_CC], x1 - Pr[FR_CC + 1], x2 - Pr[FR_CC + 2], Pr[FR_RR])) {
            // density at the nodes: centroid, then the orbits (a, a, 1 - 2a), odd coordinate last, middle, first
            const double sq[7] = {(u0 + u1 + u2) / 3.0,
                                  a1 * u0 + a1 * u1 + b1 * u2, a1 * u0 + b1 * u1 + a1 * u2, b1 * u0 + a1 * u1 + a1 * u2,
                                  a2 * u0 + a2 * u1 + b2 * u2, a2 * u0 + b2 * u1 + a2 * u2, b2 * u0 + a2 * u1 + a2 * u2};
#pragma unroll
            for (int q = 0; q < 7; ++q) {
                const double d0 = x0 - Pr[FR_X + q], d1 = x1 - Pr[FR_Y + q], d2 = x2 - Pr[FR_Z + q];
                const double ir = rsqrt_pos(d0 * d0 + d1 * d1 + d2 * d2);
                const double c = Pr[FR_W + q] * sq[q] * ir;
                const double c3 = c * ir * ir;
                ph += c;
                e0 += c3 * d0;
                e1 += c3 * d1;
                e2 += c3 * d2;
            }
        } else {
            nodal_tri_phiE(tri64 + (int64_t)TRI_REC * t, x0, x1, x2, u0, u1, u2, ph, e0, e1, e2);
        }
    }
    part[0][wv][lane] = ph;
    part[1][wv][lane] = e0;
    part[2][wv][lane] = e1;
    part[3][wv][lane] = e2;
    __syncthreads();
    if (wv == 0 && p < P) {
        const int64_t o = (int64_t)blockIdx.y * P + p;
        double r[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = (part[c][0][lane] + part[c][1][lane]) + (part[c][2][lane] + part[c][3][lane]);
        if (phi) phi[o] = r[0];
        if (E) {
            E[3 * o] = r[1];
            E[3 * o + 1] = r[2];
            E[3 * o + 2] = r[3];
        }
    }
}

// Panel records of a nodal density for the field-line passes: the copy of each
// record (both layouts) with node weight q scaled by the density at node q,
// sum_c b_qc u_c, so that the constant-basis far kernels, run with a density of
// one per panel, sum the nodal density's far field.  Padding panels keep their
// zero weights.
__global__ __launch_bounds__(256) void k_nodal_records(int64_t N, int64_t Np, const int32_t* __restrict__ tri,
                                                       const double* __restrict__ pan64, const double* __restrict__ u,
                                                       double* __restrict__ npan, double* __restrict__ nfar,
                                                       double* __restrict__ ones) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= Np) return;
    double sq[7] = {1.0, 1.0, 1.0, 1.0, 1.0, 1.0, 1.0};
    if (j < N) {
        const double u0 = u[tri[3 * j]], u1 = u[tri[3 * j + 1]], u2 = u[tri[3 * j + 2]];
        const double s15 = sqrt(15.0);
        const double a1 = (6.0 - s15) / 21.0, a2 = (6.0 + s15) / 21.0;
        const double b1 = 1.0 - 2.0 * a1, b2 = 1.0 - 2.0 * a2;
        sq[0] = (u0 + u1 + u2) / 3.0;
        sq[1] = a1 * u0 + a1 * u1 + b1 * u2;
        sq[2] = a1 * u0 + b1 * u1 + a1 * u2;
        sq[3] = b1 * u0 + a1 * u1 + a1 * u2;
        sq[4] = a2 * u0 + a2 * u1 + b2 * u2;
        sq[5] = a2 * u0 + b2 * u1 + a2 * u2;
        sq[6] = b2 * u0 + a2 * u1 + a2 * u2;
    }
#pragma unroll
    for (int k = 0; k < FAR_REC; ++k) {
        double v = pan64[(int64_t)FAR_REC * j + k];
        if (k >= FR_W && k < FR_W + 7) v *= sq[k - FR_W];
        npan[(int64_t)FAR_REC * j + k] = v;
        nfar[(int64_t)k * Np + j] = v;
    }
    ones[j] = 1.0;
}

}  // namespace

void launch_nodal_records(bem_ctx* c, const double* u) {
    const int64_t Np = (int64_t)(c->far64.bytes / (sizeof(double) * FAR_REC));
    c->nod_pan64.alloc(sizeof(double) * FAR_REC * (size_t)Np);
    c->nod_far64.alloc(sizeof(double) * FAR_REC * (size_t)Np);
    c->nod_ones.alloc(sizeof(double) * (size_t)Np);
    hipLaunchKernelGGL(k_nodal_records, dim3((unsigned)ceil_div(Np, 256)), dim3(256), 0, c->stream, c->N, Np,
                       c->tri.as<int32_t>(), c->pan64.as<double>(), u, c->nod_pan64.as<double>(),
                       c->nod_far64.as<double>(), c->nod_ones.as<double>());
    BEM_CHECK_LAUNCH();
}

template <class T>
static void nodal_assemble_t(bem_ctx* c, T* A, double* Atail, int64_t tail_row0) {
    const int64_t nv = c->n_vert, ld = c->ld;
    hipStream_t s = c->stream;
    const int64_t n_rt = ceil_div(nv, 256), n_cg = ceil_div(ceil_div(nv, NODAL_COLS), 8) * 8;
    if (n_rt * n_cg > ((int64_t)1 << 31) - 1) throw Error(BEM_ERR_INVALID, "too many vertices for the LINEAR basis");
    constexpr bool NODES = std::is_same<T, float>::value;
    if (!NODES) launch_median_records(c, nullptr, c->ev_rec);
    hipLaunchKernelGGL((k_nodal_regular<T, false, NODES>), dim3((unsigned)(n_rt * n_cg)), dim3(256), 0, s, nv, nv, ld, n_rt,
                       c->vert.as<double>(), (const int32_t*)nullptr, c->tri.as<int32_t>(), c->grp_col.as<int32_t>(),
                       c->grp_ptr.as<int32_t>(), c->grp_tri.as<int32_t>(), c->grp_loc.as<uint32_t>(), c->ev_rec.as<double>(),
                       c->pan64.as<double>(), c->tri64.as<double>(), A);
    BEM_CHECK_LAUNCH();
    const int64_t Np = (int64_t)(c->far64.bytes / (sizeof(double) * FAR_REC));
    const int64_t nch = ceil_div(c->N, 64);
    c->nodal_bounds.alloc(sizeof(double) * 4 * (size_t)nch);
    hipLaunchKernelGGL(k_nodal_chunk_bounds, dim3((unsigned)ceil_div(c->N, 256)), dim3(256), 0, s, c->N, Np,
                       c->far64.as<double>(), c->nodal_bounds.as<double>());
    BEM_CHECK_LAUNCH();
    hipLaunchKernelGGL((k_nodal_near<T, false>), dim3((unsigned)(ceil_div(nv, 8) * 8)), dim3(64), 0, s, nv, ld, c->N, Np,
                       c->row_order.as<int32_t>(), c->vert.as<double>(), (const int32_t*)nullptr, c->tri.as<int32_t>(),
                       c->far64.as<double>(), c->nodal_bounds.as<double>(), c->tri64.as<double>(), A);
    BEM_CHECK_LAUNCH();
    const int64_t nc = (int64_t)c->h_crow_tri.size(), niv = (int64_t)c->h_iface_v.size();
    const bool need_mass = c->n_float > 0 || niv > 0;
    double* mass = nullptr;
    if (need_mass) {
        c->nodal_mass.alloc(sizeof(double) * (size_t)(nv + c->n_float));
        mass = c->nodal_mass.as<double>();
        hipLaunchKernelGGL(k_nodal_mass, dim3((unsigned)ceil_div(nv, 256)), dim3(256), 0, s, nv,
                           c->fan_ptr.as<int32_t>(), c->fan.as<int32_t>(), c->tri64.as<double>(), mass);
        BEM_CHECK_LAUNCH();
    }
    if (nc > 0) {
        // normal-field rows at the centroids, then the interface vertex rows from them
        double* Kc = c->nod_Kc.as<double>();
        const int64_t n_rtc = ceil_div(nc, 256);
        if (n_rtc * n_cg > ((int64_t)1 << 31) - 1) throw Error(BEM_ERR_INVALID, "too many centroid rows");
        hipLaunchKernelGGL((k_nodal_regular<double, true, NODES>), dim3((unsigned)(n_rtc * n_cg)), dim3(256), 0, s, nc, nv, ld,
                           n_rtc, (const double*)nullptr, c->nod_trow.as<int32_t>(), c->tri.as<int32_t>(),
                           c->grp_col.as<int32_t>(), c->grp_ptr.as<int32_t>(), c->grp_tri.as<int32_t>(),
                           c->grp_loc.as<uint32_t>(), c->ev_rec.as<double>(), c->pan64.as<double>(),
                           c->tri64.as<double>(), Kc);
        BEM_CHECK_LAUNCH();
        hipLaunchKernelGGL((k_nodal_near<double, true>), dim3((unsigned)(ceil_div(nc, 8) * 8)), dim3(64), 0, s, nc, ld,
                           c->N, Np, (const int32_t*)nullptr, (const double*)nullptr, c->nod_trow.as<int32_t>(),
                           c->tri.as<int32_t>(), c->far64.as<double>(), c->nodal_bounds.as<double>(),
                           c->tri64.as<double>(), Kc);
        BEM_CHECK_LAUNCH();
        if (niv > 0) {
            hipLaunchKernelGGL(k_nodal_iface_rows<T>, dim3((unsigned)niv), dim3(256), 0, s, nv, ld,
                               c->nod_iface_v.as<int32_t>(), c->fan_ptr.as<int32_t>(), c->fan.as<int32_t>(),
                               c->tri.as<int32_t>(), c->nod_tri_crow.as<int32_t>(), c->vert_body.as<int32_t>(),
                               c->body_epsp.as<double>(), c->body_epsm.as<double>(), c->tri64.as<double>(), mass, Kc,
                               A);
            BEM_CHECK_LAUNCH();
        }
    }
    hipLaunchKernelGGL(k_nodal_diag<T>, dim3((unsigned)ceil_div(nv, 256)), dim3(256), 0, s, nv, ld, A,
                       c->diag.as<double>());
    BEM_CHECK_LAUNCH();
    if (ld > nv) {
        hipLaunchKernelGGL(k_nodal_tail<T>, dim3((unsigned)ceil_div(nv * (ld - nv), 256)), dim3(256), 0, s, nv, ld,
                           c->vert_body.as<int32_t>(), c->body_kind.as<int32_t>(), c->body_fidx.as<int32_t>(), A);
        BEM_CHECK_LAUNCH();
    }
    if (c->n_float > 0) {
        double* Af = mass + nv;
        hipLaunchKernelGGL(k_nodal_body_area, dim3((unsigned)c->n_float), dim3(256), 0, s, nv,
                           c->vert_body.as<int32_t>(), c->body_fidx.as<int32_t>(), mass, Af);
        BEM_CHECK_LAUNCH();
        hipLaunchKernelGGL(k_nodal_constraint, dim3((unsigned)ceil_div((int64_t)c->n_float * ld, 256)), dim3(256), 0,
                           s, nv, tail_row0, ld, c->n_float, c->vert_body.as<int32_t>(), c->body_fidx.as<int32_t>(),
                           mass, Af, Atail, c->diag.as<double>());
        BEM_CHECK_LAUNCH();
        if (!c->h_flt_kp.empty()) {   // rows with a K' term replace their net-charge rows
            hipLaunchKernelGGL(k_nodal_kp_body_rows, dim3((unsigned)ceil_div(ld, 256), (unsigned)c->h_flt_kp.size()),
                               dim3(256), 0, s, nv, ld, tail_row0, c->nod_flist.as<int32_t>(),
                               c->nod_frange.as<int32_t>(), c->flt_coef.as<double>(), c->nod_trow.as<int32_t>(),
                               c->vert_body.as<int32_t>(), c->body_fidx.as<int32_t>(), c->tri64.as<double>(), mass, Af,
                               c->nod_Kc.as<double>(), Atail, c->diag.as<double>());
            BEM_CHECK_LAUNCH();
        }
    }
}

void launch_nodal_assemble(bem_ctx* c) {
    KTimer kt(c, "nodal_assemble");
    if (c->opt.precision == BEM_MIXED)   // vertex rows FP32 in A32, constraint rows FP64 from row 0 of A64
        nodal_assemble_t<float>(c, c->A32.as<float>(), c->A64.as<double>(), 0);
    else
        nodal_assemble_t<double>(c, c->A64.as<double>(), c->A64.as<double>(), c->n_vert);
}

void launch_nodal_field(bem_ctx* c, int32_t nrhs, const double* sol, int64_t P, const double* pts, double* phi,
                        double* E) {
    KTimer kt(c, "nodal_field");
    if (P == 0) return;
    for (int32_t r0 = 0; r0 < nrhs; r0 += 65535) {   // load cases on grid.y
        const int32_t nr = nrhs - r0 < 65535 ? nrhs - r0 : 65535;
        hipLaunchKernelGGL(k_nodal_field, dim3((unsigned)ceil_div(P, 64), (unsigned)nr), dim3(256), 0, c->stream, P,
                           pts, c->N, c->tri.as<int32_t>(), c->pan64.as<double>(), c->tri64.as<double>(),
                           sol + (int64_t)r0 * c->n, c->n, phi ? phi + (int64_t)r0 * P : nullptr,
                           E ? E + (int64_t)r0 * P * 3 : nullptr);
        BEM_CHECK_LAUNCH();
    }
}

}  // namespace bem
