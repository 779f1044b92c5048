// The 7-point rule about the panel's centroid c (Sec. 4, regular pairs).  The rule's nodes are c and
// c + m_i, c + rho m_i on the three medians (m_i = s (v_i - c), s = 1 - 3 a_1, rho = (1 - 3 a_2) / s,
// m_0 + m_1 + m_2 = 0), so with t = x - c, T = |t|^2 and p_i = t . m_i the squared node distances are
// T, T - 2 p_i + |m_i|^2 and T - 2 rho p_i + rho^2 |m_i|^2: two operations a node instead of six, and
// sums over the nodes of w f(r) d (d = t - c_q m_i) take the nodes' f alone: t sum w f - sum_i m_i (sum
// c_q w f).  On a regular pair a node is at least (eta - 1) R away (R the circumradius) and |m_i| below R,
// so a squared distance comes from numbers at most (1 + 1 / (eta - 1))^2 times its own size: 1.44 at the
// usual eta = 6, 9 at 1.5.  At eta = 1 the panel's shape bounds that; on the meshes of the tests the results
// are then 1e-15 of the largest from the node-by-node form's.
#pragma once

#include "bem_device.h"

namespace bem {

// record of a panel: [0] c, [3] m_0, [6] m_1, [9] |m_i|^2, density x w_1 area / 4 pi, the squared
// distance from c beyond which a point is certainly regular, circumcentre, (eta R)^2
constexpr int MED_REC = 18;
constexpr int MD_DENS = 12, MD_REACH = 13, MD_CC = 14, MD_RR = 17;

constexpr double MED_S15 = 3.8729833462074168852;   // sqrt(15)
constexpr double MED_A1 = (6.0 - MED_S15) / 21.0, MED_A2 = (6.0 + MED_S15) / 21.0;
constexpr double MED_W1 = (155.0 - MED_S15) / 1200.0, MED_W2 = (155.0 + MED_S15) / 1200.0;
constexpr double MED_SC = 1.0 - 3.0 * MED_A1;               // medians' scale
constexpr double MED_RHO = (1.0 - 3.0 * MED_A2) / MED_SC;

// weights over w_1: kap0 of the centroid, kap of the second orbit; and the rule's other constants,
// held in registers (none is an inline FP64 constant; left as literals they are rebuilt at every use)
struct MedConst {
    double m2rho, rho2, kap, kap0, kaprho, kaprho2, c15, c1875, rho;
};
__device__ __forceinline__ MedConst med_consts() {
    MedConst k{-2.0 * MED_RHO,           MED_RHO * MED_RHO,  MED_W2 / MED_W1, 0.225 / MED_W1, MED_W2 / MED_W1 * MED_RHO,
               MED_W2 / MED_W1 * MED_RHO * MED_RHO, 1.5, 1.875, MED_RHO};
    asm volatile("" : "+s"(k.m2rho), "+s"(k.rho2), "+s"(k.kap), "+s"(k.kap0), "+s"(k.kaprho), "+s"(k.kaprho2),
                 "+v"(k.c15), "+s"(k.c1875), "+s"(k.rho));
    return k;
}

// Waits for this wave's scalar loads (and LDS operations) so far.  Scalar loads return out of order, so
// a wait for one is a wait for all: a loop that requests the next record ahead has to wait for the
// current one before that request, or it waits for both.
__device__ __forceinline__ void wait_scalar() { __builtin_amdgcn_s_waitcnt(0xC07F); }   // lgkmcnt(0)

// r^-3 from r^2: from the hardware estimate y of r^-1 (relative error about 2^-24), e = 1 - r^2 y^2
// and y^3 (1 + 3/2 e + 15/8 e^2 + O(e^3)): truncation below 2^-68
__device__ __forceinline__ double med_r3(double r2, const MedConst& k) {
    const double y = __builtin_amdgcn_rsq(r2);
    const double y2 = y * y;
    const double e = __fma_rn(-r2, y2, 1.0);
    const double y3 = y2 * y;
    return __fma_rn(y3 * e, __fma_rn(e, k.c1875, k.c15), y3);
}
// r^-3 and r^-5
__device__ __forceinline__ void med_r3r5(double r2, double& r3, double& r5) {
    const double ir = rsqrt_pos(r2);
    const double ir2 = ir * ir;
    r3 = ir * ir2;
    r5 = r3 * ir2;
}

}  // namespace bem
