// Field lines and the streamer integral by clusters of blocks that stay on the GPU for the whole
// run (Sec. 1, Eq. Breakdowncrit; RK4 on dx/ds = dir E/|E|): the default layout in FP64, but for many
// lines with many near panels each (lc_slower).
//
// A cluster is B blocks on the CUs of one XCD.  Block k of a cluster holds the panels j = k, k + B,
// ... in its LDS for the whole call; line l belongs to cluster l mod NC and sits in one of the
// cluster's slots until it stops, when the next of the cluster's lines takes the slot.  All of a
// cluster's live lines advance by one field evaluation per turn:
//  1. every block evaluates its panels at the query points of all live lines: its threads are
//     lines x panels at any live count, so few lines and many lines both fill them.  Regular pairs
//     by the 7-point rule (Sec. 4); the others are held back per wave and done after them by the
//     closed forms, over four lanes a pair;
//  2. a block's partial field of each line (and the first panel a step's segment hits) goes out
//     as one record, and every block reads the B records of every line and adds them in rank
//     order, so all blocks of the cluster hold the same field to the bit;
//  3. every block runs the RK4 stage machine of all lines, one line per lane, and keeps the
//     lines' state in its LDS; block 0 of the cluster writes the results.
// There is one exchange per turn and no launch, no live list in memory, no partial rows and near
// masks to write and read back, and no panel record is read from memory.  Which cluster holds a
// line and in which order its sums are taken depend on the call's arguments alone, so runs are
// bitwise reproducible.
//
// The records carry the signal themselves (three buffers used in turn, every word a sentinel at
// the start; see k_lf_loop in trace_fused.hip): a block puts the sentinel back into its own
// records of the turn before the last once it has read those of the last turn, and its next
// records go out after those stores have landed.  Every wait is bounded (spin_limit polls); at the
// bound the block raises err and leaves, and so, at their own bounds, do the blocks that wait for
// it.  The grid must be resident at once (cooperative launch).
//
// Regular pairs take the 7-point rule about the panel's centroid (median_device.h): 104 FP64
// instructions a pair (7 of them v_rsq_f64) where the node-by-node form takes 129, and 14 values of
// its record where that one reads 32.
//
// What bounds a turn (19,732 panels): the FP64 instructions of the regular pairs while many lines
// are live (27 lines a cluster: 18.4 us of 24), the latency of near pairs (2.0 us), exchange (2.3)
// and step (1.2) when few are.  A run of the benchmark's 256 lines went from 167-187 to 107-117 ms,
// one line from 36 to 20; 16 lines of 200 steps on 1,280 panels from 13.8 to 4.6.  Measured and not
// kept: records read by atomics at the XCD's own L2 (loads at that scope may hit a CU's stale
// cache; 60 to 560 us a turn); one record word of all blocks side by side (8 to 14 us of exchange:
// blocks writing into one cache line wait for each other); the records of the next round of panels
// requested a round ahead (256 registers, 22.1 against 18.9 us); 16 waves a block (186 against 181
// ms for 1024 lines).
#include <algorithm>
#include <climits>
#include <cmath>

#include "bem_device.h"
#include "median_device.h"
#include "nodal_device.h"
#include "trace_device.h"

#include <hip/hip_ext.h>

namespace bem {
namespace {

constexpr int LC_PW = 8;             // waves of a block that read records
constexpr int LC_S = 64;             // line slots of a cluster
constexpr int LC_XCD_CUS = 32;       // CUs of an XCD
// Doubles per panel: a stride of 36 banks, so lanes on consecutive panels do not collide in LDS.
constexpr int LC_REC = MED_REC;
constexpr int LC_Q = 192;            // near pairs a wave holds back (at most 64 + two rounds of 64)
constexpr int LC_NONE = 255;         // end of a thread's chain of held pairs
constexpr int LC_WORDS = 4;          // record words of a line: field (3) and hit parameter (the hit panel in
                                     // place of the field where there is a hit)

// "not written yet" (trace_fused.hip): a signalling NaN that no arithmetic result can equal
constexpr unsigned long long LC_SENT = 0x7FF4C0DE5EA1ED00ull;
__device__ __forceinline__ bool lc_is_sent(double v) {
    return (unsigned long long)__double_as_longlong(v) == LC_SENT;
}

struct LCArgs {
    const double* image;   // [B][P][LC_REC] panel records, panel j = i B + k at [k][i]
    const double* sw;      // densities x w_1 area / 4 pi of several load cases, [rhs][B][P]; or, nodal
                           // basis, the nodal density's three values a panel (k_lc_nodal); or nullptr
    const int32_t* ntri;   // nodal basis: vertices of each triangle
    int64_t N, P;          // panels, panels per block at most
    const double* tri64;
    const int32_t* tri_body;
    const int32_t* body_kind;
    const double* sol;
    int64_t n;
    const int32_t* line_rhs;
    const double* starts;
    int64_t L;
    int32_t NC;            // clusters
    int32_t nrhs;
    LBArgs a;
    int32_t* n_steps;
    int32_t* stop_code;
    double* integral;
    uint8_t* exceeds;
    double* path;
    int64_t pstride;
    unsigned long long* counts;   // near, regular pairs of this call, zero at the start
    double* buf;           // [3][NC][B][LC_S][LC_WORDS] records, every word the sentinel at the start
    int32_t* err;          // set where a wait reached its bound
    uint32_t spin_limit;
    unsigned long long* kts;
};

// Records are exchanged with loads and stores at agent scope: seen across CUs and XCDs without
// writing back or invalidating a cache.
__device__ __forceinline__ double lc_load(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void lc_store(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// two words at once, same scope (each 8-byte word is whole, the two need not be of one time)
__device__ __forceinline__ d2v lc_load2(__amdgpu_buffer_rsrc_t rs, int word) {
    typedef int i4 __attribute__((ext_vector_type(4)));
    const i4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, word * 8, 0, 16);   // sc1
    return d2v{__hiloint2double(v.y, v.x), __hiloint2double(v.w, v.z)};
}

// (t, j) of the first hit: smaller t, then smaller j
__device__ __forceinline__ void lc_first(double& t, int& j, double t2, int j2) {
    if (t2 < t || (t2 == t && j2 < j)) {
        t = t2;
        j = j2;
    }
}

// the value of another lane of the same group of four (quad_perm: no LDS round trip)
template <int CTRL>
__device__ __forceinline__ int quad_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double quad_d(double v) {
    const long long u = __double_as_longlong(v);
    const unsigned lo = (unsigned)quad_i<CTRL>((int)(unsigned)(u & 0xffffffffll));
    const unsigned hi = (unsigned)quad_i<CTRL>((int)(unsigned)((unsigned long long)u >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
constexpr int QUAD_1 = 0xB1, QUAD_2 = 0x4E;   // quad_perm [1,0,3,2] and [2,3,0,1]: lane ^ 1, lane ^ 2

// What a regular pair needs first: t = x - c and |t|^2.
struct LCPoint {
    double t0, t1, t2, T;
};
template <int M>
__device__ __forceinline__ LCPoint lc_point(const double (&v)[M], double p0, double p1, double p2) {
    LCPoint p{p0 - v[0], p1 - v[1], p2 - v[2], 0.0};
    p.T = __fma_rn(p.t0, p.t0, __fma_rn(p.t1, p.t1, p.t2 * p.t2));
    return p;
}
// One regular pair: the field of the panel with record v at the point, times its density, added
// to a.  A lane whose pair is not regular (or that has none) takes a density of 0 at a distance
// that keeps every term finite, so that the pairs of a wave run without a branch.
__device__ __forceinline__ void lc_pair(const double (&v)[14], const LCPoint& p, bool on, const MedConst& kc,
                                        double& a0, double& a1, double& a2) {
    const double T = on ? p.T : 1.0e60;
    const double sg = on ? v[12] : 0.0;
    const double pa = __fma_rn(p.t0, v[3], __fma_rn(p.t1, v[4], p.t2 * v[5]));
    const double pb = __fma_rn(p.t0, v[6], __fma_rn(p.t1, v[7], p.t2 * v[8]));
    const double pc = -(pa + pb);
    const double g10 = med_r3(__fma_rn(-2.0, pa, T + v[9]), kc);
    const double g11 = med_r3(__fma_rn(-2.0, pb, T + v[10]), kc);
    const double g12 = med_r3(__fma_rn(-2.0, pc, T + v[11]), kc);
    const double g20 = med_r3(__fma_rn(kc.m2rho, pa, __fma_rn(kc.rho2, v[9], T)), kc);
    const double g21 = med_r3(__fma_rn(kc.m2rho, pb, __fma_rn(kc.rho2, v[10], T)), kc);
    const double g22 = med_r3(__fma_rn(kc.m2rho, pc, __fma_rn(kc.rho2, v[11], T)), kc);
    const double g0 = med_r3(T, kc);
    const double G = __fma_rn(kc.kap0, g0, __fma_rn(kc.kap, (g20 + g21) + g22, (g10 + g11) + g12));
    const double h0 = __fma_rn(kc.kaprho, g20, g10), h1 = __fma_rn(kc.kaprho, g21, g11);
    const double h2 = __fma_rn(kc.kaprho, g22, g12);
    const double sG = sg * G, s0 = sg * (h2 - h0), s1 = sg * (h2 - h1);
    a0 = __fma_rn(sG, p.t0, __fma_rn(s0, v[3], __fma_rn(s1, v[6], a0)));
    a1 = __fma_rn(sG, p.t1, __fma_rn(s0, v[4], __fma_rn(s1, v[7], a1)));
    a2 = __fma_rn(sG, p.t2, __fma_rn(s0, v[5], __fma_rn(s1, v[8], a2)));
}

// The same for a nodal density: at the nodes c, c + m_i, c + rho m_i it is n0, n0 + d_i, n0 + rho d_i
// (times w_1 area / 4 pi), with n0 its mean over the corners, d_i = s (u_i - mean), d_2 = -d_0 - d_1.
__device__ __forceinline__ void lc_pair_nodal(const double (&v)[16], const LCPoint& p, bool on, const MedConst& kc,
                                              double& a0, double& a1, double& a2) {
    const double T = on ? p.T : 1.0e60;
    const double n0 = on ? v[12] : 0.0, d0 = on ? v[14] : 0.0, d1 = on ? v[15] : 0.0;
    const double d2 = -(d0 + d1);
    const double pa = __fma_rn(p.t0, v[3], __fma_rn(p.t1, v[4], p.t2 * v[5]));
    const double pb = __fma_rn(p.t0, v[6], __fma_rn(p.t1, v[7], p.t2 * v[8]));
    const double pc = -(pa + pb);
    const double g10 = (n0 + d0) * med_r3(__fma_rn(-2.0, pa, T + v[9]), kc);
    const double g11 = (n0 + d1) * med_r3(__fma_rn(-2.0, pb, T + v[10]), kc);
    const double g12 = (n0 + d2) * med_r3(__fma_rn(-2.0, pc, T + v[11]), kc);
    const double g20 = __fma_rn(kc.rho, d0, n0) * med_r3(__fma_rn(kc.m2rho, pa, __fma_rn(kc.rho2, v[9], T)), kc);
    const double g21 = __fma_rn(kc.rho, d1, n0) * med_r3(__fma_rn(kc.m2rho, pb, __fma_rn(kc.rho2, v[10], T)), kc);
    const double g22 = __fma_rn(kc.rho, d2, n0) * med_r3(__fma_rn(kc.m2rho, pc, __fma_rn(kc.rho2, v[11], T)), kc);
    const double g0 = n0 * med_r3(T, kc);
    const double G = __fma_rn(kc.kap0, g0, __fma_rn(kc.kap, (g20 + g21) + g22, (g10 + g11) + g12));
    const double h0 = __fma_rn(kc.kaprho, g20, g10), h1 = __fma_rn(kc.kaprho, g21, g11);
    const double h2 = __fma_rn(kc.kaprho, g22, g12);
    const double s0 = h2 - h0, s1 = h2 - h1;
    a0 = __fma_rn(G, p.t0, __fma_rn(s0, v[3], __fma_rn(s1, v[6], a0)));
    a1 = __fma_rn(G, p.t1, __fma_rn(s0, v[4], __fma_rn(s1, v[7], a1)));
    a2 = __fma_rn(G, p.t2, __fma_rn(s0, v[5], __fma_rn(s1, v[8], a2)));
}

// Field of unit density on the flat triangle T at x by the closed form of flat_tri_SF, over four
// lanes of a quad: lane e < 3 takes edge e (its logarithm, square roots and quotients), the solid
// angle from the distances of the three; lane 3 repeats edge 2 and adds nothing.  One lane a pair
// is a chain of three logarithms, seven square roots and eight divisions; this is a third of it.
// All four lanes return the sum.
// A call, not inlined: inlined it takes the kernel past the registers that three waves a SIMD leave.
struct LCVec3 {
    double x, y, z;
};
__device__ __noinline__ LCVec3 lc_tri_F(const double* __restrict__ T, int e4, double x0, double x1, double x2) {
    const int e = e4 < 2 ? e4 : 2, b = e == 2 ? 0 : e + 1;
    const double n0 = T[TR_N + 0], n1 = T[TR_N + 1], n2 = T[TR_N + 2];
    const double ax = T[3 * e], ay = T[3 * e + 1], az = T[3 * e + 2];
    const double bx = T[3 * b], by = T[3 * b + 1], bz = T[3 * b + 2];
    const double two_area = 2.0 * T[TR_A];
    const double V0 = ax - x0, V1 = ay - x1, V2 = az - x2, U0 = bx - x0, U1 = by - x1, U2 = bz - x2;
    // the height over the plane, from the first vertex in every lane
    const double w = (x0 - T[0]) * n0 + (x1 - T[1]) * n1 + (x2 - T[2]) * n2;
    const double r0 = x0 - w * n0, r1 = x1 - w * n1, r2 = x2 - w * n2;
    double l0 = bx - ax, l1 = by - ay, l2 = bz - az;
    const double len = sqrt(l0 * l0 + l1 * l1 + l2 * l2);
    const double il = 1.0 / len;
    l0 *= il; l1 *= il; l2 *= il;
    const double m0 = l1 * n2 - l2 * n1, m1 = l2 * n0 - l0 * n2, m2 = l0 * n1 - l1 * n0;
    const double q0 = ax - r0, q1 = ay - r1, q2 = az - r2;
    const double sm = q0 * l0 + q1 * l1 + q2 * l2;
    const double sp = sm + len;
    const double t = q0 * m0 + q1 * m1 + q2 * m2;
    const double Rm = sqrt(V0 * V0 + V1 * V1 + V2 * V2);
    constexpr int NEXT = 1 | (2 << 2) | (0 << 4) | (0 << 6);   // lanes 1, 2, 0 (lane 3 as lane 2)
    constexpr int PREV = 2 | (0 << 2) | (1 << 4) | (1 << 6);
    const double Rp = quad_d<NEXT>(Rm), Ro = quad_d<PREV>(Rm);   // at b and at the third vertex
    const bool span = sm < 0.0 && sp > 0.0, fwd = sp + sm > 0.0;
    const double num = span ? (Rp + sp) * (Rm - sm) : (fwd ? Rp + sp : Rm - sm);
    const double den = span ? t * t + w * w : (fwd ? Rm + sm : Rp - sp);
    double f = log(num / den);
    // solid angle: [r1 r2 r3] = -2 A w, and the quad's sum of (r_e . r_e+1) R_e+2
    double dr = (V0 * U0 + V1 * U1 + V2 * U2) * Ro;
    if (e4 == 3) {
        f = 0.0;
        dr = 0.0;
    }
    double F0 = m0 * f, F1 = m1 * f, F2 = m2 * f;
    F0 += quad_d<QUAD_1>(F0);
    F1 += quad_d<QUAD_1>(F1);
    F2 += quad_d<QUAD_1>(F2);
    dr += quad_d<QUAD_1>(dr);
    F0 += quad_d<QUAD_2>(F0);
    F1 += quad_d<QUAD_2>(F1);
    F2 += quad_d<QUAD_2>(F2);
    dr += quad_d<QUAD_2>(dr);
    const double omega = 2.0 * atan2(two_area * fabs(w), Rm * Rp * Ro + dr);
    const double sg = (w > 0.0) ? omega : ((w < 0.0) ? -omega : 0.0);
    return LCVec3{(F0 + sg * n0) * INV4PI, (F1 + sg * n1) * INV4PI, (F2 + sg * n2) * INV4PI};
}

// Field of the linear density with corner values u on the flat triangle T, one lane a pair (a call:
// see lc_tri_F)
__device__ __noinline__ LCVec3 lc_nodal_E(const double* __restrict__ T, double x0, double x1, double x2, double u0,
                                          double u1, double u2) {
    LCVec3 E{0.0, 0.0, 0.0};
    double ph = 0.0;
    nodal_tri_phiE(T, x0, x1, x2, u0, u1, u2, ph, E.x, E.y, E.z);
    return E;
}

// Cluster and rank of a block.  Consecutive block ids go to the 8 XCDs in turn: cluster cl takes ids = cl
// mod 8 (B of the ids on that XCD, where a cluster is a part of one).  Where the clusters do not deal
// out evenly to 8 (a part of the GPU with fewer CUs), they take the ids in turn among themselves.
struct LCPlace {
    int cl, k;
};
__host__ __device__ constexpr LCPlace lc_place(int id, int NC, int B) {
    const int xg = NC % 8 == 0 ? 8 : NC, xi = id % xg, xm = id / xg;
    return LCPlace{xi + xg * (xm / B), xm % B};
}
// every (cluster, rank) by exactly one block, whatever the number of clusters
constexpr bool lc_places_all(int NC, int B) {
    bool seen[64 * 32] = {};
    for (int id = 0; id < NC * B; ++id) {
        const LCPlace p = lc_place(id, NC, B);
        if (p.cl < 0 || p.cl >= NC || p.k < 0 || p.k >= B || seen[p.cl * B + p.k]) return false;
        seen[p.cl * B + p.k] = true;
    }
    return true;
}
constexpr bool lc_places_all() {
    for (int xcds = 1; xcds <= 16; ++xcds)
        for (int B = 8; B <= LC_XCD_CUS; B *= 2)
            if (!lc_places_all(xcds * (LC_XCD_CUS / B), B)) return false;
    return true;
}
static_assert(lc_places_all(), "blocks of the cluster layout");

// W: waves of a block; B: blocks of a cluster; RES: the block's panels in LDS (else read from the image each turn);
// SW: densities from the records (0), of several load cases from LDS (1) or from memory (2);
// NODAL: the density is the nodal one (its three values a panel where SW 1, 2 read load cases')
template <int W, int B, bool RES, int SW, bool NODAL>
__global__ __launch_bounds__(64 * W) void k_lc_trace(LCArgs P) {
    constexpr int LC_W = W, LC_T = 64 * W;
    constexpr int LC_NE = LC_T / 4;   // near pairs evaluated at a time, four lanes each
    extern __shared__ __attribute__((aligned(16))) double lrec[];   // RES: [Pk][LC_REC]; SW 1: [rhs][P]
    // state of the cluster's lines, every block its own copy, all computed alike
    __shared__ double sx[3][LC_S], sy[3][LC_S], sks[3][LC_S], sas[LC_S], sI[LC_S];
    __shared__ int32_t sns[LC_S], sline[LC_S], sphase[LC_S], srhs[LC_S], slot_of[LC_S];
    // far sums by thread, then (once this block's records are out) field sums by wave
    __shared__ double red[3][LC_T];
    double(*psum)[3][LC_S] = reinterpret_cast<double(*)[3][LC_S]>(&red[0][0]);
    __shared__ double nres[3][LC_NE];
    __shared__ uint32_t nq[LC_W][LC_Q];
    __shared__ int32_t nqc[LC_W];
    __shared__ unsigned long long hitT[LC_S], hitP[LC_S];   // first hit of the segment: parameter (as bits) ..
    __shared__ int32_t hitJ[LC_S];                          // .. and panel
    __shared__ int32_t s_nl, s_next, s_abort, s_more, s_hit, s_rec_hit, s_changed;
    static_assert(LC_PW * LC_S <= LC_T, "the field sums fit the far sums' place");

    kclock_start(P.kts);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const LCPlace place = lc_place((int)blockIdx.x, P.NC, B);
    const int cl = place.cl, k = place.k;
    const int64_t nlines = cl < P.L ? (P.L - cl + P.NC - 1) / P.NC : 0;   // lines cl, cl + NC, ...
    if (nlines == 0) {   // uniform over the cluster
        kclock_stop(P.kts);
        return;
    }
    const int Pk = (int)((P.N - k + B - 1) / B);   // panels k, k + B, ...
    const double* img = P.image + (int64_t)k * P.P * LC_REC;
    if constexpr (RES) {
        const d2v* s = reinterpret_cast<const d2v*>(img);
        d2v* d = reinterpret_cast<d2v*>(lrec);
        for (int e = tid; e < Pk * (LC_REC / 2); e += LC_T) d[e] = s[e];
    }
    double* lsw = lrec + (RES ? P.P * LC_REC : 0);
    if constexpr (SW == 1) {
        for (int r = 0; r < P.nrhs; ++r)
            for (int i = tid; i < Pk; i += LC_T) lsw[r * P.P + i] = P.sw[((int64_t)r * B + k) * P.P + i];
    }
    int nl = (int)(nlines < LC_S ? nlines : LC_S);
    if (tid < nl) {
        const int64_t l = cl + (int64_t)P.NC * tid;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double v = P.starts[3 * l + c];
            sx[c][tid] = v;
            sy[c][tid] = v;
            if (P.path && k == 0) P.path[l * P.pstride + c] = v;
        }
        sI[tid] = 0.0;
        sas[tid] = 0.0;
        sns[tid] = 0;
        sphase[tid] = 0;
        sline[tid] = (int32_t)l;
        srhs[tid] = P.line_rhs ? P.line_rhs[l] : 0;
        slot_of[tid] = tid;
    }
    if (tid < LC_S) {
        hitT[tid] = (unsigned long long)__double_as_longlong(2.0);
        hitP[tid] = hitT[tid];
        hitJ[tid] = INT_MAX;
    }
    if (tid == 0) {
        s_nl = nl;
        s_next = nl;
        s_abort = 0;
        s_more = 0;
        s_hit = 0;
        s_rec_hit = 0;
    }
    __syncthreads();
    const MedConst kc = med_consts();
    unsigned long long pairs = 0, nears = 0;   // this block's (thread 0)
    int nl1 = 0, nl2 = 0;   // live counts of the previous two turns
    const int64_t rstride = (int64_t)LC_S * LC_WORDS;   // one block's records of a turn
    const int64_t bstride = (int64_t)P.NC * B * rstride;
    double* bw = P.buf + (int64_t)cl * (B * rstride);             // this turn's records of the cluster ..
    double *bn = bw + bstride, *bp = bw + 2 * bstride;            // .. the next turn's, the last turn's
    // threads [0, nl PB) are nl lines x PB panels: at least 87 % of the block at every nl > 4
    int PB = 1, pi = 0, li = 0, sl = 0, lq = 1;
    bool changed = true;
    for (int turn = 0;; turn = turn < 2 ? turn + 1 : 2) {
        // the sentinel back into this block's records of the turn before the last: every block
        // has read them (it has written those of the last turn since)
        if (turn == 2) {
            double* br = bn + k * rstride;
            for (int e = tid; e < nl2 * LC_WORDS; e += LC_T)
                lc_store(br + e, __longlong_as_double((long long)LC_SENT));
        }
        // ---- 1. this block's panels at every live line's query point ----
        if (changed) {
            PB = LC_T / nl;
            pi = tid / nl;
            li = tid - pi * nl;
            sl = slot_of[li];
            lq = 1;
            while ((8 << lq) * nl <= LC_T && lq < 6) ++lq;   // 4 nl words x 2^lq lanes fit the block
        }
        const bool has = pi < PB;
        const double p0 = sy[0][sl], p1 = sy[1][sl], p2 = sy[2][sl];
        const double* gsw = SW == 2 ? P.sw + ((int64_t)srhs[sl] * B + k) * P.P : nullptr;
        const int lo = SW == 1 ? srhs[sl] * (int)P.P : 0;
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, b0 = 0.0, b1 = 0.0, b2 = 0.0;
        // output word (li, c) of this thread in the sums below, over Q lanes
        const int Q = 1 << lq, oq = tid & (Q - 1), ow = tid >> lq, oc = ow & 3, ol = ow >> 2;
        int base = 0;   // uniform over the wave, which stops where its held pairs fill up
        for (;;) {
            uint32_t* q = nq[wv];
            int qn = 0, mine = LC_NONE;   // pairs held by the wave; the last one held for this thread
            const double* recs = RES ? lrec : img;
            // what every pair reads of a record: centroid, medians, their squares, density, reach
            constexpr int NV = NODAL ? 16 : 14;
            auto fetch = [&](int i, double (&v)[NV]) {
                const double* r = recs + i * LC_REC;
#pragma unroll
                for (int c = 0; c < 12; ++c) v[c] = r[c];
                v[12] = SW == 0 ? r[12] : (SW == 1 ? lsw[lo + i] : gsw[i]);
                v[13] = r[13];
                if constexpr (NODAL) {
                    v[14] = SW == 1 ? lsw[P.P + i] : gsw[B * P.P + i];
                    v[15] = SW == 1 ? lsw[2 * P.P + i] : gsw[2 * B * P.P + i];
                }
            };
            auto pair = [&](const double (&v)[NV], const LCPoint& p, bool on, double& x, double& y, double& z) {
                if constexpr (NODAL)
                    lc_pair_nodal(v, p, on, kc, x, y, z);
                else
                    lc_pair(v, p, on, kc, x, y, z);
            };
            // regular or not (Sec. 4): |t|^2 above the record's reach settles it (the circumcentre's
            // distance is then certainly above eta R); below, the test itself.  A pair that is not
            // is held back.
            auto test = [&](bool ok, int i, const LCPoint& p, double reach) {
                bool reg = p.T > reach;
                if (__ballot(ok && !reg)) {
                    if (ok && !reg) {
                        const double* r = recs + i * LC_REC;
                        reg = is_regular(p0 - r[14], p1 - r[15], p2 - r[16], r[17]);
                    }
                    const bool near = ok && !reg;
                    const uint64_t m = __ballot(near);
                    const int pos = qn + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                    if (near) {
                        q[pos] = ((uint32_t)mine << 22) | ((uint32_t)li << 16) | (uint32_t)i;
                        mine = pos;
                    }
                    qn += __popcll(m);
                }
                return ok && reg;
            };
            // two panels a thread and round (their chains of dependent instructions overlap)
            while (base + PB < Pk && qn <= LC_Q - 128) {
                const int iA = base + pi, iB = iA + PB;
                base += 2 * PB;
                const bool okB = has && iB < Pk;
                double vA[NV], vB[NV];
                fetch(has ? iA : 0, vA);
                fetch(okB ? iB : 0, vB);
                const LCPoint pA = lc_point(vA, p0, p1, p2), pB = lc_point(vB, p0, p1, p2);
                const bool onA = test(has, iA, pA, vA[13]), onB = test(okB, iB, pB, vB[13]);
                pair(vA, pA, onA, a0, a1, a2);
                pair(vB, pB, onB, b0, b1, b2);
            }
            if (base + PB >= Pk && base < Pk && qn <= LC_Q - 128) {   // a last single round
                const int iA = base + pi;
                base += PB;
                const bool okA = has && iA < Pk;
                double vA[NV];
                fetch(okA ? iA : 0, vA);
                const LCPoint pA = lc_point(vA, p0, p1, p2);
                pair(vA, pA, test(okA, iA, pA, vA[13]), a0, a1, a2);
            }
            if (lane == 0) {
                nqc[wv] = qn;
                if (base < Pk) s_more = 1;
            }
            __syncthreads();
            // near pairs of all waves, LC_NE at a time from the last to the first; each thread adds
            // those held for it, from its last to its first
            int tot = 0, before[LC_W], own = 0;
#pragma unroll
            for (int u = 0; u < LC_W; ++u) {
                before[u] = tot;
                if (u == wv) own = tot;
                tot += nqc[u];
            }
            nears += (unsigned long long)tot;
            for (int eb = tot > 0 ? (tot - 1) / LC_NE * LC_NE : -1; eb >= 0; eb -= LC_NE) {
                const int e = eb + (tid >> 2);
                double th = -1.0;
                int eli = 0, ej = 0;
                if (e < tot) {
                    int u = 0, off = 0;
#pragma unroll
                    for (int v = 1; v < LC_W; ++v)
                        if (e >= before[v]) {
                            u = v;
                            off = before[v];
                        }
                    const uint32_t en = nq[u][e - off];
                    eli = (int)((en >> 16) & 63u);
                    ej = (int)(en & 0xffffu) * B + k;
                    const int es = slot_of[eli];
                    const double* Tj = P.tri64 + (int64_t)TRI_REC * ej;
                    const double y0 = sy[0][es], y1 = sy[1][es], y2 = sy[2][es];
                    if constexpr (NODAL) {
                        if ((tid & 3) == 0) {
                            const int32_t* tv = P.ntri + 3 * (int64_t)ej;
                            const LCVec3 f = lc_nodal_E(Tj, y0, y1, y2, P.sol[tv[0]], P.sol[tv[1]], P.sol[tv[2]]);
                            nres[0][tid >> 2] = f.x;
                            nres[1][tid >> 2] = f.y;
                            nres[2][tid >> 2] = f.z;
                        }
                    } else {
                        const double sg = P.sol[(int64_t)srhs[es] * P.n + ej];
                        const LCVec3 f = lc_tri_F(Tj, tid & 3, y0, y1, y2);
                        if ((tid & 3) == 0) {
                            nres[0][tid >> 2] = sg * f.x;
                            nres[1][tid >> 2] = sg * f.y;
                            nres[2][tid >> 2] = sg * f.z;
                        }
                    }
                    if (sphase[es] == 4 && (tid & 3) == 0) {
                        const double x0 = sx[0][es], x1 = sx[1][es], x2 = sx[2][es];
                        th = lb_segment_tri(Tj, x0, x1, x2, y0 - x0, y1 - x1, y2 - x2);
                        if (th >= 0.0) s_hit = 1;
                    }
                }
                __syncthreads();
                while (mine != LC_NONE && own + mine >= eb) {
                    const int r = own + mine - eb;
                    a0 += nres[0][r];
                    a1 += nres[1][r];
                    a2 += nres[2][r];
                    mine = (int)(q[mine] >> 22);
                }
                if (s_hit) {   // uniform; rare: the first hit by (parameter, panel)
                    const unsigned long long tb = (unsigned long long)__double_as_longlong(th + 0.0);
                    if (th >= 0.0) atomicMin(&hitT[eli], tb);
                    __syncthreads();
                    if (tid < nl && hitT[tid] != hitP[tid]) {
                        hitP[tid] = hitT[tid];
                        hitJ[tid] = INT_MAX;
                    }
                    __syncthreads();
                    if (th >= 0.0 && tb == hitT[eli]) atomicMin(&hitJ[eli], ej);
                }
                if (eb > 0) __syncthreads();
            }
            if (s_more == 0) break;   // uniform: written before the barrier above
            __syncthreads();
            if (tid == 0) s_more = 0;
            __syncthreads();
        }
        red[0][tid] = a0 + b0;
        red[1][tid] = a1 + b1;
        red[2][tid] = a2 + b2;
        pairs += (unsigned long long)nl * (unsigned long long)Pk;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the sentinels of this turn have landed
        __syncthreads();
        // ---- 2. the block's records out, every block's records in ----
        if (ol < nl) {
            double v = 0.0;
            if (oc < 3)
                for (int u = oq; u < PB; u += Q) v += red[oc][u * nl + ol];
            for (int o = 1; o < Q; o <<= 1) v += __shfl_xor(v, o, 64);
            if (s_hit) {
                if (oc == 3) v = __longlong_as_double((long long)hitT[ol]);
                else if (oc == 0 && hitJ[ol] != INT_MAX) v = (double)hitJ[ol];
            } else if (oc == 3) {
                v = 2.0;
            }
            if (oq == 0) lc_store(bw + k * rstride + ow, v);
        }
        __syncthreads();   // red is read, psum takes its place
        bool ok = true;
        {
            // wave w < PW: ranks [w R, (w + 1) R); a lane: two words of each
            constexpr int R = B / LC_PW;
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(bw, 0, (int)(B * rstride * 8), 0x00020000);
            for (int e = lane; wv < LC_PW && e < ((2 * nl + 63) & ~63); e += 64) {
                const bool mine = e < 2 * nl;
                const int w0 = wv * R * (int)rstride + (mine ? 2 * e : 0);
                d2v v[R];
                uint32_t polls = 0;
                for (;;) {
                    asm volatile("" ::: "memory");   // the loads stay in the loop
                    bool w = false;
#pragma unroll
                    for (int b = 0; b < R; ++b) v[b] = lc_load2(rs, w0 + b * (int)rstride);
#pragma unroll
                    for (int b = 0; b < R; ++b) w |= lc_is_sent(v[b].x) || lc_is_sent(v[b].y);
                    if (__ballot(w) == 0) break;   // uniform over the wave
                    if (++polls > P.spin_limit) {
                        ok = false;
                        break;
                    }
                }
                d2v sum = v[0];
                bool hit = v[0].y < 2.0;
#pragma unroll
                for (int b = 1; b < R; ++b) {
                    sum += v[b];
                    hit |= v[b].y < 2.0;
                }
                if (mine) {
                    const int l4 = e >> 1;
                    if (e & 1) {
                        psum[wv][2][l4] = sum.x;
                        if (hit) s_rec_hit = 1;
                    } else {
                        psum[wv][0][l4] = sum.x;
                        psum[wv][1][l4] = sum.y;
                    }
                }
            }
        }
        if (!ok && lane == 0) {   // the records are left unused and the run ends
            s_abort = 1;
            __hip_atomic_store(P.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (s_abort) break;   // uniform over the block
        // ---- 3. the stage machine, one line per lane of wave 0 ----
        if (wv == 0) {
            const bool act = lane < nl;
            const int s = slot_of[act ? lane : 0];
            bool live = false;
            if (act) {
                const LBArgs& a = P.a;
                const double h = a.h;
                const int phase = sphase[s];
                const int64_t l = sline[s];
                double F0 = psum[0][0][lane], F1 = psum[0][1][lane], F2 = psum[0][2][lane];
#pragma unroll
                for (int u = 1; u < LC_PW; ++u) {
                    F0 += psum[u][0][lane];
                    F1 += psum[u][1][lane];
                    F2 += psum[u][2][lane];
                }
                const double y0 = sy[0][s], y1 = sy[1][s], y2 = sy[2][s];
                double x0 = sx[0][s], x1 = sx[1][s], x2 = sx[2][s], I = sI[s];
                int32_t ns = sns[s];
                int code = -1;   // -1: the line goes on
                if (phase == 4) {
                    int jb = INT_MAX;
                    if (s_rec_hit) {   // some line's segment hit a panel: this one's first hit, if any
                        double tb = 2.0;
                        for (int b = 0; b < B; ++b) {
                            const double* r = bw + b * rstride + lane * LC_WORDS;
                            const double t = lc_load(r + 3);
                            if (t < 2.0) lc_first(tb, jb, t, (int)lc_load(r));
                        }
                    }
                    if (jb != INT_MAX) {   // the step's segment hit a panel: the step is discarded
                        const int32_t kd = P.body_kind[P.tri_body[jb]];
                        code = (kd == BEM_DIRICHLET) ? BEM_STOP_DIRICHLET
                                                     : ((kd == BEM_FLOATING) ? BEM_STOP_FLOATING : BEM_STOP_INTERFACE);
                    } else {   // accepted: its end point becomes the line's point
                        I = I + h / 6.0 * sas[s];
                        x0 = y0;
                        x1 = y1;
                        x2 = y2;
                        ++ns;
                        if (P.path && k == 0) {
                            P.path[l * P.pstride + 3 * ns + 0] = x0;
                            P.path[l * P.pstride + 3 * ns + 1] = x1;
                            P.path[l * P.pstride + 3 * ns + 2] = x2;
                        }
                        if (ns >= a.max_steps) code = BEM_STOP_MAXSTEPS;
                    }
                }
                if (code < 0) {
                    const double m = sqrt(F0 * F0 + F1 * F1 + F2 * F2);
                    const double im = a.dir / m;
                    const double d0 = F0 * im, d1 = F1 * im, d2 = F2 * im;
                    const double al = lb_alpha(a, m);
                    const bool first = phase == 0 || phase == 4, mid = phase == 1 || phase == 2;
                    // weights of the stages: k1 1, k2 and k3 2, k4 1
                    const double wk = mid ? 2.0 : 1.0;
                    const double c0 = first ? 0.0 : sks[0][s], c1 = first ? 0.0 : sks[1][s],
                                 c2 = first ? 0.0 : sks[2][s], cs = first ? 0.0 : sas[s];
                    const double k0 = c0 + wk * d0, k1 = c1 + wk * d1, k2 = c2 + wk * d2, as = cs + wk * al;
                    const double step = (phase == 3) ? h / 6.0 : ((phase == 2) ? h : 0.5 * h);
                    const double z0 = x0 + step * (phase == 3 ? k0 : d0), z1 = x1 + step * (phase == 3 ? k1 : d1),
                                 z2 = x2 + step * (phase == 3 ? k2 : d2);
                    if (first) {
                        if (!isfinite(m))
                            code = BEM_STOP_NONFINITE;
                        else if (m < a.e_min)
                            code = BEM_STOP_WEAK;
                    } else if (phase == 3 && !(isfinite(z0) && isfinite(z1) && isfinite(z2))) {
                        code = BEM_STOP_NONFINITE;
                    }
                    if (code < 0) {
                        sx[0][s] = x0; sx[1][s] = x1; sx[2][s] = x2;
                        sy[0][s] = z0; sy[1][s] = z1; sy[2][s] = z2;
                        sks[0][s] = k0; sks[1][s] = k1; sks[2][s] = k2;
                        sas[s] = as;
                        sI[s] = I;
                        sns[s] = ns;
                        sphase[s] = first ? 1 : phase + 1;
                    }
                }
                live = code < 0;
                if (!live && k == 0) {
                    P.n_steps[l] = ns;
                    P.stop_code[l] = code;
                    if (P.integral) P.integral[l] = I;
                    if (P.exceeds) P.exceeds[l] = (I > a.k_str) ? 1 : 0;
                }
            }
            // a stopped line's slot takes the cluster's next line
            const uint64_t dead = __ballot(act && !live);
            if (lane == 0) s_changed = 0;
            if (dead) {
                const int nx = s_next;
                const int64_t qi = nx + __popcll(dead & ((1ull << lane) - 1));
                if (act && !live && qi < nlines) {
                    const int64_t l = cl + (int64_t)P.NC * qi;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const double v = P.starts[3 * l + c];
                        sx[c][s] = v;
                        sy[c][s] = v;
                        if (P.path && k == 0) P.path[l * P.pstride + c] = v;
                    }
                    sI[s] = 0.0;
                    sas[s] = 0.0;
                    sns[s] = 0;
                    sphase[s] = 0;
                    sline[s] = (int32_t)l;
                    srhs[s] = P.line_rhs ? P.line_rhs[l] : 0;
                    live = true;
                }
                const uint64_t alive = __ballot(live);
                if (live) slot_of[__popcll(alive & ((1ull << lane) - 1))] = s;
                if (lane == 0) {
                    s_changed = 1;
                    s_next = nx + __popcll(dead);
                    s_nl = __popcll(alive);
                }
            }
        }
        if (s_hit && wv == 1) {   // uniform over the wave: the hit records cleared for the next turn
            hitT[lane] = (unsigned long long)__double_as_longlong(2.0);
            hitP[lane] = hitT[lane];
            hitJ[lane] = INT_MAX;
        }
        __syncthreads();
        if (tid == 0) {   // read again only after the next turn's barriers
            s_hit = 0;
            s_rec_hit = 0;
        }
        nl2 = nl1;
        nl1 = nl;
        nl = s_nl;
        changed = s_changed != 0;
        if (nl == 0) break;
        double* const t = bp;   // the records of the last turn but one are free for the turn after the next
        bp = bw;
        bw = bn;
        bn = t;
    }
    if (tid == 0) {
        atomicAdd(P.counts, nears);
        atomicAdd(P.counts + 1, pairs - nears);
    }
    kclock_stop(P.kts);
}

// the records' words to the sentinel, the call's pair counts and the error flag to zero
__global__ __launch_bounds__(256) void k_lc_fill(int64_t m, unsigned long long* __restrict__ v,
                                                 unsigned long long* __restrict__ counts, int32_t* __restrict__ err) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < m; i += (int64_t)gridDim.x * 256) v[i] = LC_SENT;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        counts[0] = counts[1] = 0;
        err[0] = 0;
    }
}

__global__ void k_lc_count(const unsigned long long* __restrict__ counts, unsigned long long* __restrict__ total) {
    if (threadIdx.x < 2) total[threadIdx.x] += counts[threadIdx.x];
}

__global__ __launch_bounds__(256) void k_lc_density(int64_t N, int64_t P, int B, const double* __restrict__ tri64,
                                                    const double* __restrict__ sol, int64_t n,
                                                    double* __restrict__ sw) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x, rhs = blockIdx.y;
    if (j >= N) return;
    sw[(rhs * B + j % B) * P + j / B] = sol[rhs * n + j] * (MED_W1 * INV4PI * tri64[(int64_t)TRI_REC * j + TR_A]);
}

// The nodal density's values of each panel, times w_1 area / 4 pi: its mean, and s (u_i - mean) of
// corners 0 and 1, as three "load cases" of k_lc_density's layout.
__global__ __launch_bounds__(256) void k_lc_nodal(int64_t N, int64_t P, int B, const double* __restrict__ tri64,
                                                  const int32_t* __restrict__ tri, const double* __restrict__ u,
                                                  double* __restrict__ sw) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= N) return;
    const double w = MED_W1 * INV4PI * tri64[(int64_t)TRI_REC * j + TR_A];
    const double u0 = u[tri[3 * j]], u1 = u[tri[3 * j + 1]], u2 = u[tri[3 * j + 2]];
    const double mean = (u0 + u1 + u2) / 3.0;
    double* o = sw + (j % B) * P + j / B;
    o[0] = w * mean;
    o[B * P] = w * (MED_SC * (u0 - mean));
    o[2 * B * P] = w * (MED_SC * (u1 - mean));
}

// cnt[block]: pairs of the block's panels with the S sampled starts that are not regular
__global__ __launch_bounds__(256) void k_lc_near(const double* __restrict__ far64, int64_t Np, int64_t N, int64_t L,
                                                 int S, const double* __restrict__ starts, int32_t* cnt) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;   // < Np
    const double c0 = far64[(int64_t)FR_CC * Np + j], c1 = far64[(int64_t)(FR_CC + 1) * Np + j],
                 c2 = far64[(int64_t)(FR_CC + 2) * Np + j], rr = far64[(int64_t)FR_RR * Np + j];
    int n = 0;
    for (int s = 0; s < S; ++s) {
        const double* x = starts + 3 * ((int64_t)s * L / S);
        n += __popcll(__ballot(j < N && !is_regular(x[0] - c0, x[1] - c1, x[2] - c2, rr)));
    }
    __shared__ int red[4];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(cnt + blockIdx.x, red[0] + red[1] + red[2] + red[3], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
}

// 8 and 16 blocks a cluster only with everything in LDS (launch_trace_cluster)
template <int W, bool ND>
const void* lc_kernel_of(int B, bool res, int sw) {
#define BEM_LC(BB, RES, SW) reinterpret_cast<const void*>(&k_lc_trace<W, BB, RES, SW, ND>)
    if constexpr (!ND) {
        if (sw == 0) return B == 8 ? BEM_LC(8, true, 0) : (B == 16 ? BEM_LC(16, true, 0) : (res ? BEM_LC(32, true, 0) : BEM_LC(32, false, 0)));
    }
    if (sw == 1) return B == 8 ? BEM_LC(8, true, 1) : (B == 16 ? BEM_LC(16, true, 1) : BEM_LC(32, true, 1));
    return res ? BEM_LC(32, true, 2) : BEM_LC(32, false, 2);
#undef BEM_LC
}
const void* lc_kernel(int W, int B, bool res, int sw, bool nodal) {
    if (nodal) return lc_kernel_of<8, true>(B, res, sw);
    return W == 8 ? lc_kernel_of<8, false>(B, res, sw) : lc_kernel_of<12, false>(B, res, sw);
}

// Whether L lines take less time in the two-kernel layout.  There a line and stage cost more by themselves
// (partial fields and marks through memory, two launches for all lines); here the near pairs, a quad
// of lanes each on the few waves of a block, and where 8 blocks hold the panels the regular pairs do.  In ns
// a line and stage, with v near pairs, measured from 80 to 65,216 panels, eta 6 to 60 (v 80 to 5,600) and 256 to
// 65,536 lines: the two-kernel layout is ahead where 0.054 v + 0.0024 N (past 8 blocks 0.0003 N, where the
// records come from memory 0.0005 N) is above 11 +
// 360,000 / L^1.5, with the nodal basis (near pairs one lane of a quad each) where 0.137 v + 0.0025 N
// (0.001 N) is above 15 + 300,000 / L^1.5.  ms, this layout and the other: 2,192 panels, v 299, 4096 lines of
// 20 steps 12.3 and 10.1, of 1024 lines (40 steps) 6.9 and 7.2; v 1175, 1024 lines 18.2 and 11.5; nodal, 3,816
// panels, v 100, 4096 lines 14.3 and 11.2.  Lines keep about as many near panels as their starts have, so v is
// taken at 64 of the starts.
bool lc_slower(bem_ctx* c, int64_t L, const double* starts, int B, bool res, bool nodal) {
    if (L < 256) return false;
    const double per_near = nodal ? 0.137 : 0.054, l = (double)L;
    const double per_panel = B == 8 ? (nodal ? 0.0025 : 0.0024) : nodal ? 0.001 : res ? 0.0003 : 0.0005;
    const double v0 = ((nodal ? 15.0 + 3.0e5 / (l * std::sqrt(l)) : 11.0 + 3.6e5 / (l * std::sqrt(l))) -
                       per_panel * (double)c->N) / per_near;
    if (v0 >= (double)c->N) return false;
    if (v0 <= 0.0) return true;
    constexpr int S = 64;
    const int64_t Np = (int64_t)(c->far64.bytes / (sizeof(double) * FAR_REC)), nb = ceil_div(c->N, 256);
    c->check_host.alloc(sizeof(int32_t) * (size_t)nb, hipHostMallocCoherent);
    hipLaunchKernelGGL(k_lc_near, dim3((unsigned)nb), dim3(256), 0, c->stream, c->far64.as<double>(), Np, c->N, L, S,
                       starts, c->check_host.as<int32_t>());
    BEM_CHECK_LAUNCH();
    BEM_HIP(hipStreamSynchronize(c->stream));
    int64_t n = 0;
    const volatile int32_t* cnt = c->check_host.as<int32_t>();
    for (int64_t b = 0; b < nb; ++b) n += cnt[b];
    return (double)n > v0 * S;
}

}  // namespace

TraceCluster launch_trace_cluster(bem_ctx* c, int32_t nrhs, const double* sol, int64_t L, const int32_t* line_rhs,
                                  const double* starts, const bem_trace_params* tp, int32_t* n_steps,
                                  int32_t* stop_code, double* path, double* integral, uint8_t* exceeds) {
    if (c->tune_trace_cluster == 0) return TraceCluster::NOT_TAKEN;
    if (c->coop_launch < 0) {
        int v = 0;
        BEM_HIP(hipDeviceGetAttribute(&v, hipDeviceAttributeCooperativeLaunch, c->device));
        c->coop_launch = v ? 1 : 0;
    }
    int cus = 0;
    BEM_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device));
    if (c->coop_launch == 0 || cus < LC_XCD_CUS) return TraceCluster::NOT_TAKEN;
    const int64_t N = c->N;
    if (!line_rhs) nrhs = 1;   // every line takes the first load case
    // nodal basis (one load case; FP64 in either precision): three density values a panel
    const bool nodal = c->opt.basis == BEM_BASIS_LINEAR;
    if (nodal && nrhs > 1) return TraceCluster::NOT_TAKEN;
    const int nd = nodal ? 3 : nrhs;
    // blocks per cluster: as few as hold the panels (and the load cases' densities) in LDS.  Fewer
    // blocks exchange faster and leave more clusters to share the lines (us a turn, 1,280 panels,
    // 16 lines: 6.4 with 8 blocks, 7.7 with 32; 7,712 panels, 16 load cases x 64 lines: 187 ms a
    // run with 16, which hold the densities too, 204 with 8, 208 with 32).  Where 32 do not hold
    // them the densities, then the records, are read from memory each turn.
    auto lds_room = [nodal](int waves) {   // LDS of a CU less what the kernel itself takes
        hipFuncAttributes fa;
        BEM_HIP(hipFuncGetAttributes(&fa, lc_kernel(waves, 32, true, nodal ? 1 : 0, nodal)));
        return (size_t)160 * 1024 - fa.sharedSizeBytes - 16;
    };
    const size_t room = lds_room(8);
    const size_t per_panel = sizeof(double) * LC_REC, per_dens = nd > 1 ? sizeof(double) * (size_t)nd : 0;
    int B = c->tune_trace_blocks > 0 ? c->tune_trace_blocks : 8;
    while (B < 32 && (per_panel + per_dens) * (size_t)ceil_div(N, B) > room) B *= 2;
    const int NC = cus / LC_XCD_CUS * (LC_XCD_CUS / B);
    const int64_t P = ceil_div(N, B);
    if (P > 65535) return TraceCluster::NOT_TAKEN;   // a held pair carries its panel's index in 16 bits
    const bool res = per_panel * (size_t)P <= room;
    // nodal panels beyond LDS: their records and densities from memory each turn lose to the two-kernel
    // layout where the pairs take the time (54,882 panels, 256 lines of 200 steps: 69.7 against 62.2 ms)
    if (nodal && !res && L > (int64_t)NC * 8) return TraceCluster::NOT_TAKEN;
    if (c->tune_trace_blocks == 0 && lc_slower(c, L, starts, B, res, nodal)) return TraceCluster::NOT_TAKEN;
    const int sw = nd == 1 ? 0 : (res && (per_panel + per_dens) * (size_t)P <= room ? 1 : 2);
    const size_t dyn = res ? (per_panel + (sw == 1 ? per_dens : 0)) * (size_t)P : 0;
    // waves per block: 8 are the faster exchange and step (1 line, 19,732 panels: equal; 8 lines,
    // 2,192 panels: 19.0 against 20.8 ms a run), 12 fill the SIMDs better where the pairs take the
    // time (19,732 panels, 256 lines: 52.0 against 53.7 ms, 1024 lines: 181 against 192) and LDS has
    // room for their own arrays too
    const int W = !nodal && L > (int64_t)NC * 8 && dyn <= lds_room(12) ? 12 : 8;
    const void* f = lc_kernel(W, B, res, sw, nodal);
    // the attribute is the process's, not this call's: always the most that a CU has, so that no other
    // thread's call finds less than it needs
    if (dyn > 0) BEM_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_room(W)));
    int per_cu = 0;
    BEM_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, 64 * W, dyn));
    if (per_cu < 1) return TraceCluster::NOT_TAKEN;

    KTimer t(c, "trace");
    LCArgs A;
    const int64_t words = 3 * (int64_t)NC * LC_S * LC_WORDS * B;
    c->lc_buf.alloc(sizeof(double) * (size_t)(words + 8));
    c->lc_image.alloc(sizeof(double) * (size_t)(B * P) * (LC_REC + (nd > 1 ? nd : 0)));
    A.image = c->lc_image.as<double>();
    A.sw = nd > 1 ? c->lc_image.as<double>() + (size_t)(B * P) * LC_REC : nullptr;
    A.buf = c->lc_buf.as<double>();
    A.counts = reinterpret_cast<unsigned long long*>(A.buf + words);
    A.err = reinterpret_cast<int32_t*>(A.counts + 2);
    hipLaunchKernelGGL(k_lc_fill, dim3(256), dim3(256), 0, c->stream, words,
                       reinterpret_cast<unsigned long long*>(A.buf), A.counts, A.err);
    BEM_CHECK_LAUNCH();
    launch_median_records(c, nd > 1 ? nullptr : sol, c->lc_image, B, P);
    if (nodal) {
        hipLaunchKernelGGL(k_lc_nodal, dim3((unsigned)ceil_div(N, 256)), dim3(256), 0, c->stream, N, P, B,
                           c->tri64.as<double>(), c->tri.as<int32_t>(), sol, const_cast<double*>(A.sw));
        BEM_CHECK_LAUNCH();
    } else if (nrhs > 1) {
        hipLaunchKernelGGL(k_lc_density, dim3((unsigned)ceil_div(N, 256), (unsigned)nrhs), dim3(256), 0, c->stream, N,
                           P, B, c->tri64.as<double>(), sol, c->n, const_cast<double*>(A.sw));
        BEM_CHECK_LAUNCH();
    }
    A.N = N;
    A.P = P;
    A.tri64 = c->tri64.as<double>();
    A.tri_body = c->tri_body.as<int32_t>();
    A.body_kind = c->body_kind.as<int32_t>();
    A.sol = sol;
    A.n = c->n;
    A.line_rhs = nrhs > 1 ? line_rhs : nullptr;
    A.starts = starts;
    A.L = L;
    A.NC = NC;
    A.nrhs = nd;
    A.ntri = c->tri.as<int32_t>();
    A.a.h = tp->h;
    A.a.e_min = tp->e_min;
    A.a.dir = tp->direction >= 0 ? 1.0 : -1.0;
    A.a.a = tp->alpha_a;
    A.a.e0 = tp->alpha_e0;
    A.a.p = tp->alpha_p;
    A.a.k_str = tp->k_str;
    A.a.max_steps = tp->max_steps;
    A.n_steps = n_steps;
    A.stop_code = stop_code;
    A.integral = integral;
    A.exceeds = exceeds;
    A.path = path;
    A.pstride = 3 * ((int64_t)tp->max_steps + 1);
    A.spin_limit = (uint32_t)c->tune_trace_spin;
    kclock_begin(c, 1);
    A.kts = kclock_slot(c, "trace_pass");
    hipEvent_t ea = nullptr, eb = nullptr;
    const bool timed = c->profiling == 1;
    if (timed) {
        timing_events(c, &ea, &eb);
        BEM_HIP(hipEventRecord(ea, c->stream));
    }
    void* kargs[] = {&A};
    const hipError_t le =
        hipLaunchCooperativeKernel(f, dim3((unsigned)(NC * B)), dim3((unsigned)(64 * W)), kargs, (unsigned)dyn, c->stream);
    if (le != hipSuccess) {   // refused (nothing launched): the caller takes another layout
        (void)hipGetLastError();
        if (timed) {
            c->event_pool.push_back(ea);
            c->event_pool.push_back(eb);
        }
        kclock_end(c);
        return TraceCluster::NOT_TAKEN;
    }
    if (timed) {
        BEM_HIP(hipEventRecord(eb, c->stream));
        push_timing(c, "trace_pass", ea, eb);
    }
    ++c->trace_pass_launches;
    kclock_end(c);
    c->host_stage.alloc(sizeof(int32_t) * 64);
    int32_t* host = c->host_stage.as<int32_t>() + 32;
    BEM_HIP(hipMemcpyAsync(host, A.err, sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    BEM_HIP(hipStreamSynchronize(c->stream));
    // a wait reached its bound (another kernel held CUs that a cluster's blocks needed for seconds): the
    // caller runs the lines again, one pass after another, in launches whose blocks wait for nothing
    if (*host != 0) return TraceCluster::GAVE_UP;
    hipLaunchKernelGGL(k_lc_count, dim3(1), dim3(64), 0, c->stream, A.counts,
                       reinterpret_cast<unsigned long long*>(c->counters.p) + 2);
    BEM_CHECK_LAUNCH();
    return TraceCluster::DONE;
}

}  // namespace bem
