// group.hpp -- one MPPI sample on a group of eight lanes: lane j holds
// joint j (j = 0..6) and lane 7 the end-effector frame.  The per-step work
// of Sec. III-A/B is spread over the group so that the chain of one
// sample's step is shorter than on one lane:
//
//   kinematics   every lane forms its joint transform Rp_j Rz(q_j), r_j
//                (lane 7: the fixed EE transform) and an inclusive scan of
//                transform compositions over the group gives every link
//                frame (R_j, p_j) at once, the EE pose in lane 7;
//   velocities   motion subspaces S_j = (z_j, (p_j - O) x z_j) in Pluecker
//                coordinates about one point O for all links (the step's
//                EE point, so that the distal links keep short moment
//                arms), where moving between links needs no transform, so
//                link twists are prefix sums
//                V_j = sum_{i<=j} S_i qd_i and velocity-product
//                accelerations prefix sums of V_i x S_i qd_i (gravity as
//                the base acceleration);
//   bias forces  f_j = I_j A_j + V_j x* I_j V_j (Newton-Euler per link, at
//                its CoM; lane 7 carries the negated wall wrench) and suffix sums
//                give h_j = S_j . sum_{i>=j} f_i, i.e. h(q, qd) of Eq. 5
//                less the external torque;
//   inertia      composite-rigid-body inertias Ic_j = sum_{i>=j} I_i
//                (suffix sums of the ten inertia parameters about O) give
//                the joint-space inertia M_ij = S_i . Ic_j S_j (i <= j),
//                the matrix of Eq. 8 plus the armature diagonal, row j in
//                lane j;
//   solve        the rows are gathered through the group's LDS area and
//                every lane factors M = L D L^T (no pivoting: M is SPD)
//                and solves Eq. 6 for the whole qdd; lane j keeps qdd_j;
//   force        (Eqs. 12-13) with J the EE Jacobian about the EE point
//                (columns (z_j, (p_j - p_ee) x z_j), short moment arms
//                where the estimate is taken) and M = L D L^T:
//                lane r (r < 6) solves L y = (row r of J)^T, lane 6
//                L y = tau_F, and D^-1/2 y is column j of [A^T | y'] with
//                J M^-1 J^T = A A^T and J M^-1 tau_F = A y'; transposed
//                through LDS, so that lane j holds joint j's row, the
//                least-squares solution of A^T x = y' by modified
//                Gram-Schmidt takes its products as sums over the group
//                (three DPP adds each; 19 % fewer instructions of the cost
//                part than with column j in lane j and the pivot column
//                broadcast) and ends in a back substitution in every lane
//                -- without forming J M^-1 J^T, whose condition number (the
//                square of A's) exceeds 1 / u32 near kinematic
//                singularities;
//   cost         lane 7 adds the pose and force terms of Eqs. 9-13, lanes
//                0..6 their joint's limit and torque terms (Eq. 14), and
//                the collision pairs of Eq. 15 are dealt over the eight
//                lanes; the group sums its lanes once, after the horizon.
//
// The code is written per lane against a group object G that provides the
// cross-lane moves (shr<D>: value of lane j - D, 0 for j < D; shr_one<D>:
// the same with 1 for j < D; add_shr<D> /
// add_shl<D>: x plus the value of lane j - D / j + D, plus 0 where there
// is none; bcast<K>: of lane K), sum (over the group, the same bits in every
// lane), sync() (orders the
// group's LDS area) and shm (that area, kGxCount values).  On the device G
// is eight lanes of a row of 16, two groups interleaved (joint j in lane
// 2 j + p), so that DPP row shifts by 2 D stay within a group and fill the
// lanes without a source with 0, and a shift-and-add is one instruction; a
// host emulation runs the same code on eight threads in lockstep at every
// cross-lane move.
#pragma once

#include "rollout.hpp"

namespace mppi {

constexpr int kGroup = 8;
// Group LDS area (values of the rollout type).  The part that the cost part
// of a step reads comes first: the update kernels, whose dynamics wave is
// one step ahead of the cost wave, keep two of it (kGxPart values each) and
// one of the rest, which only the dynamics part touches.
constexpr int kGxSF = 0;                   // [8][6]: S_j
constexpr int kGxTf = kGxSF + 8 * 6;       // [8]: tau_F
constexpr int kGxH = kGxTf + 8;            // [8][12]: handoff to the cost part: p_j, q, qd, v, h_c, m_c
                                           // (lanes 0..6); lane 7: p_ee, R_ee
constexpr int kGxOm = kGxH + 8 * 12;       // [8][8]: the LDL^T factor of M (row i: L below the diagonal,
                                           // 1 / d_i on it), then L^-1 [J^T | tau_F] (row i: joint i)
constexpr int kGxPart = kGxOm + 8 * 8;     // 216
constexpr int kGxRow = kGxPart;            // [8][8]: M row j up to the diagonal
constexpr int kGxRhs = kGxRow + 8 * 8;     // [8]: tau - h
constexpr int kGxRows = 8 * 8 + 8;         // 72
constexpr int kGxCount = kGxPart + kGxRows;   // 288
// Strides between the areas of a wave's groups.  A step's reads are uniform
// over a group (eight addresses per wave, 16 bytes each) or lane by lane
// within its area (the collision pairs' segment ends): the eight areas start
// on distinct banks with strides of an odd number of 32-byte units.
template <typename R> constexpr int gx_pad(int n) { return sizeof(R) == 4 ? (n + 7) / 16 * 16 + 8 : (n + 3) / 8 * 8 + 4; }
template <typename R> constexpr int kGxStride = gx_pad<R>(kGxCount);                        // one area
template <typename R> constexpr int kGxPairStride = gx_pad<R>(2 * kGxPart + kGxRows);       // two cost parts, one set of rows
static_assert(kGxStride<float> >= kGxCount && kGxStride<double> >= kGxCount, "area size");
static_assert(kGxPairStride<float> >= 2 * kGxPart + kGxRows && kGxPairStride<double> >= 2 * kGxPart + kGxRows,
              "area size");

// Per-lane constants of the group rollout (lane 7: the EE frame, massless).
template <typename R> struct GroupLink {
    R Rp[9], rp[3];   // joint frame in the parent frame (lane 7: R_ee, r_ee)
    R Ic[6], com[3], m, arm;
    R qmin, qmax, qdmax, taumax, qrest;
    R sigma, sig_c;   // sampling scale of this joint (0 in lane 7)
    R live;           // 1 for a joint, 0 for lane 7
};

template <typename R> MPPI_HD void group_link(const ModelM<R>& M, const CostM<R>& C, int j, GroupLink<R>& G)
{
    const bool live = j < NJ;
    const LinkM<R>& L = M.L[live ? j : NJ - 1];
#pragma unroll
    for (int a = 0; a < 9; ++a) G.Rp[a] = live ? L.Rp[a] : M.Ree[a];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        G.rp[a] = live ? L.rp[a] : M.ree[a];
        G.com[a] = live ? L.com[a] : R(0);
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) G.Ic[a] = live ? L.Ic[a] : R(0);
    G.m = live ? L.m : R(0);
    G.arm = live ? L.arm : R(0);
    G.qmin = L.qmin; G.qmax = L.qmax; G.qdmax = L.qdmax; G.taumax = L.taumax;
    G.qrest = C.q_rest[live ? j : NJ - 1];
    G.sigma = live ? C.sigma[j] : R(0);
    G.sig_c = live ? C.sig_c[j] : R(0);
    G.live = live ? R(1) : R(0);
}

// This lane's normal of step t: Philox call j / 4 of the counter (c, t, k,
// tick), Box-Muller pair (j / 2) mod 2, cosine (even j) or sine branch --
// the same u32 words and the same arithmetic as normals8, one normal per lane.
template <typename R> MPPI_HD R group_normal(uint64_t seed, uint32_t tick, uint32_t k, uint32_t t, int j)
{
    uint32_t x0 = (uint32_t)(j >> 2), x1 = t, x2 = k, x3 = tick;
    philox10(x0, x1, x2, x3, (uint32_t)seed, (uint32_t)(seed >> 32));
    const bool hi = (j >> 1) & 1;
    R z0, z1;
    box_muller_pair<R>(hi ? x2 : x0, hi ? x3 : x1, z0, z1);
    return (j & 1) ? z1 : z0;
}

// the perturbation recursion of noise_step for this lane's joint
template <typename R> MPPI_HD R group_noise_step(R rho, const GroupLink<R>& L, R z, R du, int t)
{
    return (t == 0 || rho == R(0)) ? L.sigma * z : rho * du + L.sig_c * z;
}

// ---------------------------------------------------------------------------
// scans over the group
// ---------------------------------------------------------------------------
// inclusive prefix composition of (Q, t) (child frame in the parent frame):
// (Qa, ta) o (Qb, tb) = (Qa Qb, Qa tb + ta), earlier joints on the left;
// lanes j < D compose with the identity (I, 0) that the shift leaves them
template <int D, typename R, class G> MPPI_HD void scan_frames(const G& g, R* Q, R* t)
{
    R Qp[9], tp[3];
#pragma unroll
    for (int a = 0; a < 9; ++a)
        Qp[a] = (a % 4 == 0) ? g.template shr_one<D>(Q[a]) : g.template shr<D>(Q[a]);
#pragma unroll
    for (int a = 0; a < 3; ++a) tp[a] = g.template shr<D>(t[a]);
    R nt[3];
    mv3(Qp, t, nt);
    t[0] = nt[0] + tp[0]; t[1] = nt[1] + tp[1]; t[2] = nt[2] + tp[2];
    mm3(Qp, Q, Q);
}
// Inclusive prefix and suffix sums over the group (Hillis-Steele: three
// shift-and-add rounds, lanes past the ends adding 0)
template <int N, typename R, class G> MPPI_HD void prefix_sum(const G& g, R* x)
{
#pragma unroll
    for (int a = 0; a < N; ++a) x[a] = g.template add_shr<1>(x[a]);
#pragma unroll
    for (int a = 0; a < N; ++a) x[a] = g.template add_shr<2>(x[a]);
#pragma unroll
    for (int a = 0; a < N; ++a) x[a] = g.template add_shr<4>(x[a]);
}
template <int N, typename R, class G> MPPI_HD void suffix_sum(const G& g, R* x)
{
#pragma unroll
    for (int a = 0; a < N; ++a) x[a] = g.template add_shl<1>(x[a]);
#pragma unroll
    for (int a = 0; a < N; ++a) x[a] = g.template add_shl<2>(x[a]);
#pragma unroll
    for (int a = 0; a < N; ++a) x[a] = g.template add_shl<4>(x[a]);
}

// EE pose of the group: lane j gets its link frame (lane 7: R_ee, p_ee)
template <typename R, class G> MPPI_HD void group_fk(const G& g, const GroupLink<R>& L, R q, R* Q, R* p)
{
    R c, s;
    sincos_(q, &s, &c);
    joint_rot(L.Rp, c, s, Q);
    p[0] = L.rp[0]; p[1] = L.rp[1]; p[2] = L.rp[2];
    scan_frames<1>(g, Q, p);
    scan_frames<2>(g, Q, p);
    scan_frames<4>(g, Q, p);
}

// The cost weights that the group's running and terminal costs use at
// every step, held in registers: reads from the cost copy in LDS inside the
// EE lane's branch would each wait for their own round trip.
template <typename R> struct GroupCostW {
    R W_pos[3], W_ori[3], W_force[6], W_reg[6];
    R w_q, w_qd, w_post, w_tau;
    int has_ori, force_mode;
};
template <typename R> MPPI_HD void group_cost_w(const CostM<R>& C, GroupCostW<R>& w)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) { w.W_pos[a] = C.W_pos[a]; w.W_ori[a] = C.W_ori[a]; }
#pragma unroll
    for (int a = 0; a < 6; ++a) { w.W_force[a] = C.W_force[a]; w.W_reg[a] = C.W_reg[a]; }
    w.w_q = C.w_q; w.w_qd = C.w_qd; w.w_post = C.w_post; w.w_tau = C.w_tau;
    w.has_ori = C.has_ori;
    w.force_mode = C.force_mode;
}

// pose terms of Eqs. 9-11 from the EE frame (R_ee = R_n R_ee,fixed)
template <typename R> MPPI_HD R pose_cost(const GroupCostW<R>& W, const TargetM<R>& tg, const R* pee, const R* Re)
{
    R s = W.W_pos[0] * sq(tg.p_des[0] - pee[0]) + W.W_pos[1] * sq(tg.p_des[1] - pee[1]) +
          W.W_pos[2] * sq(tg.p_des[2] - pee[2]);
    if (W.has_ori) {
        R Rerr[9], rho[3];
        mm3(tg.RdT, Re, Rerr);
        so3_log(Rerr, rho);
        s += W.W_ori[0] * rho[0] * rho[0] + W.W_ori[1] * rho[1] * rho[1] + W.W_ori[2] * rho[2] * rho[2];
    }
    return s;
}
// this lane's joint-limit, velocity-limit and posture terms (Eq. 14 C_joint)
template <typename R> MPPI_HD R joint_cost1(const GroupCostW<R>& W, const GroupLink<R>& L, R q, R qd)
{
    return W.w_q * (sq(hinge(q - L.qmax)) + sq(hinge(L.qmin - q))) + W.w_qd * sq(hinge(abs_(qd) - L.qdmax)) +
           W.w_post * sq(q - L.qrest);
}
// force terms of Eq. 12 (the arithmetic of force_cost)
template <typename R> MPPI_HD R group_force_cost(const GroupCostW<R>& W, const TargetM<R>& tg, const R* F)
{
    R s = R(0);
#pragma unroll
    for (int a = 0; a < 6; ++a) s += W.W_force[a] * sq(tg.F_des[a] - F[a]) + W.W_reg[a] * F[a] * F[a];
    return s;
}

// One modified Gram-Schmidt step of lsq_wrench on the group with joint j's
// row of [A^T | y] in lane j (a[0..5], a[6] = y): the products of column S
// with itself and the later columns are sums over the group, which every
// lane gets, so row S of the triangular factor (Rm[S][c] = q_S . column c,
// Rm[S][6] = q_S . y, q_S the normalised column S) and idg = 1 / |column S|
// end in every lane's registers, and each lane removes the q_S component
// from its entries.
template <int S, typename R, class G> MPPI_HD void group_mgs_step(const G& g, R* a, R (&Rm)[6][NJ], R* idg)
{
    R p[NJ];
#pragma unroll
    for (int c = S; c < NJ; ++c) p[c] = g.sum(a[S] * a[c]);
    const R id = rsqrt_(p[S]);
    idg[S] = id;
    const R q = a[S] * id;
#pragma unroll
    for (int c = S + 1; c < NJ; ++c) {
        Rm[S][c] = p[c] * id;
        a[c] = fma_(-Rm[S][c], q, a[c]);
    }
}

// What a group step leaves for inspection (host checks): lane 7's EE pose,
// the force estimate (FORCE) and this lane's qdd.
template <typename R> struct GroupStepOut {
    R qdd;
    R pee[3], Re[9];
    R F[6];
};

// M = L D L^T (unit lower L, lower triangle in Lm, 1/d in id) of the rows
// gathered in the group area (rows: its kGxRow part), in every lane; b0 (may
// be null): the right-hand side tau - h of the rows.
template <typename R> struct GroupFactor {
    R Lm[NJ][NJ];
    R id[NJ];
};
template <typename R> MPPI_HD void group_factor(const R* rows, GroupFactor<R>& f, R* b0)
{
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
#pragma unroll
        for (int c = 0; c <= i; ++c) f.Lm[i][c] = rows[i * 8 + c];
        if (b0) b0[i] = rows[kGxRhs - kGxRow + i];
    }
#pragma unroll
    for (int k = 0; k < NJ; ++k) {
        f.id[k] = rcp_(f.Lm[k][k]);
        R u[NJ];
#pragma unroll
        for (int i = k + 1; i < NJ; ++i) { u[i] = f.Lm[i][k]; f.Lm[i][k] = u[i] * f.id[k]; }
#pragma unroll
        for (int i = k + 1; i < NJ; ++i)
#pragma unroll
            for (int c = k + 1; c <= i; ++c) f.Lm[i][c] = fma_(-f.Lm[i][k], u[c], f.Lm[i][c]);
    }
}

// Dynamics part of one step (Eqs. 5-6): kinematics, twists, bias forces,
// composite inertias, the rows of M and their right-hand sides in the group
// area X, the factorisation (into *fac when given) and qdd.  Returns this
// lane's qdd (0 in lane 7); p, Q receive this lane's frame (lane 7: the EE
// pose).  tau: this lane's joint torque (sampled torque plus any
// joint-space external torque); v: the sampled torque (tau_F).
// FDYN: the input of the force estimate that the rows do not hold (tau_F)
// is formed here, on the dynamics chain; otherwise group_cost forms it from the handoff.  The
// update kernel chooses FDYN when the cost part also carries the collision
// pairs, so that neither part runs both.
// wrench: when given, a further world wrench [force; moment] at the EE
// point, acting on the EE lane at this step's state (J(q)^T W on the joints).
// rows: the kGxRow part of the area where it is not kept behind X.
template <typename R, bool FORCE, class G, bool FDYN = false, bool HANDOFF = false>
MPPI_HD R group_dynamics(const G& g, const GroupLink<R>& L, const CostM<R>& C, const R* grav, int ext, R q, R qd,
                         R tau, R v, R* X, GroupFactor<R>* fac, R* p, R* Q, const R* wrench = nullptr,
                         R* rows = nullptr)
{
    const int j = g.j;
    const bool ee = j == kGroup - 1;
    if (!rows) rows = X + kGxRow;
    // the wall's constants, read ahead of the chain that uses them
    R wn[3], wd0 = R(0), wk = R(0), wc = R(0);
    if (ext == EXTW_WALL) {
#pragma unroll
        for (int a = 0; a < 3; ++a) wn[a] = C.wall_n[a];
        wd0 = C.wall_d0;
        wk = C.wall_k;
        wc = C.wall_c;
    }
    sched_fence();

    // ---- kinematics: link frames (lane 7: the EE frame)
    group_fk(g, L, q, Q, p);
    // spatial quantities are taken about the EE point O = p_ee of this
    // step (a fixed point in space for the step): the moment arms of the
    // distal links, whose small inertias set the small entries of M, stay
    // at link length, where arms about the world origin would be the reach
    const R pe[3] = {g.template bcast<kGroup - 1>(p[0]), g.template bcast<kGroup - 1>(p[1]),
                     g.template bcast<kGroup - 1>(p[2])};
    const R pr[3] = {p[0] - pe[0], p[1] - pe[1], p[2] - pe[2]};
    // motion subspace about O (lane 7: none); its linear part (p_j - p_ee)
    // x z_j is also the EE Jacobian's linear column about the EE point
    R z[3] = {Q[2] * L.live, Q[5] * L.live, Q[8] * L.live}, pz[3];
    cross3(pr, z, pz);
    // gather S: in FP32 every lane requests all seven slots here, long before
    // the rows of M need them, so that the exchange's round trip overlaps
    // the bias forces and subtree sums; in FP64 the 84 registers would spill
    // (K = 16384, T = 36: 404 us against 330), and they are read with the rows
    R* slot = X + kGxSF + j * 6;
#pragma unroll
    for (int a = 0; a < 3; ++a) { slot[a] = z[a]; slot[3 + a] = pz[a]; }
    g.sync();
    constexpr bool early = sizeof(R) == 4;
    R Sc[NJ][6];
    auto gather = [&] {
#pragma unroll
        for (int c = 0; c < NJ; ++c)
#pragma unroll
            for (int a = 0; a < 6; ++a) Sc[c][a] = X[kGxSF + c * 6 + a];
        sched_fence();   // in one round trip
    };
    if (early) gather();
    // CoM about O, rotational inertia about the CoM in world axes; link
    // inertia about O: mass m, first moment h = m c, rotational I_O
    R cw[3], Ib[6];
    mv3(Q, L.com, cw);
    cw[0] += pr[0]; cw[1] += pr[1]; cw[2] += pr[2];
    congr_sym3<false>(Q, L.Ic, Ib);
    R In[10];   // h[3], m, I_O[6]
    In[0] = L.m * cw[0]; In[1] = L.m * cw[1]; In[2] = L.m * cw[2]; In[3] = L.m;
    {
        const R c00 = cw[0] * cw[0], c11 = cw[1] * cw[1], c22 = cw[2] * cw[2];
        In[4] = Ib[0] + L.m * (c11 + c22);
        In[5] = Ib[1] + L.m * (c00 + c22);
        In[6] = Ib[2] + L.m * (c00 + c11);
        In[7] = Ib[3] - In[0] * cw[1];
        In[8] = Ib[4] - In[0] * cw[2];
        In[9] = Ib[5] - In[1] * cw[2];
    }

    // ---- twists V_j = sum_{i<=j} S_i qd_i
    R Sq[6] = {z[0] * qd, z[1] * qd, z[2] * qd, pz[0] * qd, pz[1] * qd, pz[2] * qd};
    R V[6] = {Sq[0], Sq[1], Sq[2], Sq[3], Sq[4], Sq[5]};
    prefix_sum<6>(g, V);
    // velocity-product accelerations V_j x (S_j qd_j), prefix-summed, plus
    // the base acceleration -g
    R A[6];
    {
        R t1[3], t2[3], t3[3];
        cross3(V, Sq, t1);
        cross3(V, Sq + 3, t2);
        cross3(V + 3, Sq, t3);
        A[0] = t1[0]; A[1] = t1[1]; A[2] = t1[2];
        A[3] = t2[0] + t3[0]; A[4] = t2[1] + t3[1]; A[5] = t2[2] + t3[2];
    }
    prefix_sum<6>(g, A);
    A[3] -= grav[0]; A[4] -= grav[1]; A[5] -= grav[2];

    // ---- link forces about O, by Newton and Euler at the CoM: with its
    // velocity v_c = v + w x c and acceleration a_c = a + al x c + w x v_c,
    // F = m a_c and N = Ib al + w x (Ib w), then (N + c x F, F) -- a third
    // fewer operations than I A + V x* (I V) with the inertia about O
    R f[6];
    {
        auto sym_mul = [](const R* I, const R* x, R* y) {
            y[0] = I[0] * x[0] + I[3] * x[1] + I[4] * x[2];
            y[1] = I[3] * x[0] + I[1] * x[1] + I[5] * x[2];
            y[2] = I[4] * x[0] + I[5] * x[1] + I[2] * x[2];
        };
        R t1[3], t2[3], vc[3], ac[3], Iw[3], Ia[3];
        cross3(V, cw, t1);
        vc[0] = V[3] + t1[0]; vc[1] = V[4] + t1[1]; vc[2] = V[5] + t1[2];
        cross3(A, cw, t1);
        cross3(V, vc, t2);
        ac[0] = A[3] + t1[0] + t2[0]; ac[1] = A[4] + t1[1] + t2[1]; ac[2] = A[5] + t1[2] + t2[2];
        f[3] = L.m * ac[0]; f[4] = L.m * ac[1]; f[5] = L.m * ac[2];
        sym_mul(Ib, V, Iw);
        sym_mul(Ib, A, Ia);
        cross3(V, Iw, t1);
        cross3(cw, f + 3, t2);
        f[0] = Ia[0] + t1[0] + t2[0]; f[1] = Ia[1] + t1[1] + t2[1]; f[2] = Ia[2] + t1[2] + t2[2];
    }
    if (ext == EXTW_WALL) {
        // unilateral spring-damper at the EE point (lane 7's frame origin,
        // the reference point O: the EE point velocity is V's linear part
        // and the wall force has no moment about O)
        const R delta = wd0 - dot3(wn, p);
        const R ddelta = -dot3(wn, V + 3);
        const R mag = hinge(wk * delta + wc * ddelta);
        if (ee) {
            f[3] -= wn[0] * mag; f[4] -= wn[1] * mag; f[5] -= wn[2] * mag;
        }
    }
    if (wrench && ee) {
#pragma unroll
        for (int a = 0; a < 3; ++a) { f[a] -= wrench[3 + a]; f[3 + a] -= wrench[a]; }
    }

    // ---- subtree sums: bias forces and composite inertias
    suffix_sum<6>(g, f);
    suffix_sum<10>(g, In);
    const R hq = dot3(z, f) + dot3(pz, f + 3);
    // Ic S: (I_O w + h x v, m v - h x w) of the subtree
    R Fm[6];
    {
        R hv[3], hw[3];
        cross3(In, pz, hv);
        cross3(In, z, hw);
        Fm[0] = In[4] * z[0] + In[7] * z[1] + In[8] * z[2] + hv[0];
        Fm[1] = In[7] * z[0] + In[5] * z[1] + In[9] * z[2] + hv[1];
        Fm[2] = In[8] * z[0] + In[9] * z[1] + In[6] * z[2] + hv[2];
        Fm[3] = In[3] * pz[0] - hw[0];
        Fm[4] = In[3] * pz[1] - hw[1];
        Fm[5] = In[3] * pz[2] - hw[2];
    }
    if (FORCE && FDYN) {
        // tau_F (less the gravity torque S . Ic (0, -g) when force_mode is 0)
        R tf = v;
        if (C.force_mode == 0) {
            const R ag[3] = {-grav[0], -grav[1], -grav[2]};
            R ha[3];
            cross3(In, ag, ha);
            tf = v - (dot3(z, ha) + In[3] * dot3(pz, ag));
        }
        X[kGxTf + j] = ee ? R(0) : tf;
    }
    if (!early) gather();
    // row j of M up to the diagonal: M_jc = S_c . (Ic S)_j (c <= j), plus
    // the armature; every lane holds all the S_c and multiplies by its own
    // Ic S.  Above the diagonal, and in the EE lane, the same products are
    // not M (nothing reads that part of the rows).
    R row[NJ];
#pragma unroll
    for (int c = 0; c < NJ; ++c) {
        R s = c == j ? L.arm : R(0);
#pragma unroll
        for (int a = 0; a < 6; ++a) s = fma_(Sc[c][a], Fm[a], s);
        row[c] = s;
    }
#pragma unroll
    for (int c = 0; c < NJ; ++c) rows[j * 8 + c] = row[c];
    rows[kGxRhs - kGxRow + j] = tau - hq;
    g.sync();

    // ---- Eq. 6: qdd = L^-T D^-1 L^-1 (tau + tau_ext - h)
    GroupFactor<R> local;
    GroupFactor<R>& F = fac ? *fac : local;
    R b0[NJ], x[NJ];
    group_factor(rows, F, b0);
    // handoff to the cost part: pre-step q, qd, v, the joint origin and the
    // subtree's mass and first moment (lanes 0..6), the EE pose (lane 7);
    // written once the rows are read, so that the row reads do not queue
    // behind these writes
    R* h = X + kGxH + j * 12;
    {
        const R own[9] = {q, qd, v, In[0], In[1], In[2], In[3], Q[7], Q[8]};   // the last two: no one's
#pragma unroll
        for (int a = 0; a < 3; ++a) h[a] = p[a];
#pragma unroll
        for (int a = 0; a < 9; ++a) h[3 + a] = ee ? Q[a] : own[a];
    }
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
        R s = b0[i];
#pragma unroll
        for (int c = 0; c < i; ++c) s = fma_(-F.Lm[i][c], x[c], s);
        x[i] = s;
    }
#pragma unroll
    for (int i = NJ - 1; i >= 0; --i) {
        R s = x[i] * F.id[i];
#pragma unroll
        for (int c = i + 1; c < NJ; ++c) s = fma_(-F.Lm[c][i], x[c], s);
        x[i] = s;
    }
    if (FORCE && HANDOFF && j == 0) {
        // for the cost part (HANDOFF): row i of L below the diagonal and
        // 1 / d_i on it, in the kGxOm rows, so that it does not factorise
        // M again (one lane writes; the other lanes have read M)
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
#pragma unroll
            for (int c = 0; c < i; ++c) X[kGxOm + i * 8 + c] = F.Lm[i][c];
            X[kGxOm + i * 8 + i] = F.id[i];
        }
    }
    R qj = R(0);
#pragma unroll
    for (int i = 0; i < NJ; ++i) qj = (i == j) ? x[i] : qj;
    return qj;
}

// The collision term of Eqs. 14-15: pair i belongs to lane i mod 8 and to
// round i / 8; a lane keeps its pairs of up to four rounds.  A pair past
// n_pairs has a threshold of 0 and never hits.
constexpr int kGxRounds = 32 / kGroup;
template <typename R> struct GroupPairs {
    int a[kGxRounds], b[kGxRounds];   // segments: link s from p_s to p_s+1 (p_7 = p_ee), or obstacle s - 7
    R d2[kGxRounds];                  // squared thresholds
    int rounds;                       // the same in every lane
};

template <typename R> MPPI_HD void group_pairs(const CostM<R>& C, int j, GroupPairs<R>& P)
{
#pragma unroll
    for (int r = 0; r < kGxRounds; ++r) {
        P.a[r] = C.pa[r * kGroup + j];
        P.b[r] = C.pb[r * kGroup + j];
        P.d2[r] = C.dth2[r * kGroup + j];
    }
    P.rounds = uniform_((C.n_pairs + kGroup - 1) / kGroup);
}

// This lane's hits among its pairs of rounds FIRST, FIRST + STEP, ..., from
// the joint origins and the EE point in the handoff.  A segment's ends are
// read at a selected address, not in a branch per kind of segment: lanes of
// one wave hold both kinds (a wave ran the four cases of a pair one after
// another).  With this and the rounds dealt over both waves of a pair of
// waves, K = 4096, T = 18 with 20 pairs takes 46.4 us (59.0 with all rounds
// on the cost wave and the branches; 7 % longer with the first and third
// round on the dynamics wave instead of the second); FP64 79 us (94).
template <int FIRST, int STEP, typename R>
MPPI_HD R group_hits(const GroupPairs<R>& P, const CostM<R>& C, const R* X)
{
    R hits = R(0);
#pragma unroll
    for (int r = FIRST; r < kGxRounds; r += STEP) {
        if (r >= P.rounds) break;
        const bool la = P.a[r] < NJ, lb = P.b[r] < NJ;
        const R* a0 = la ? X + kGxH + P.a[r] * 12 : C.obs[P.a[r] - NJ];
        const R* b0 = lb ? X + kGxH + P.b[r] * 12 : C.obs[P.b[r] - NJ];
        const R* a1 = a0 + (la ? 12 : 3);
        const R* b1 = b0 + (lb ? 12 : 3);
        hits += seg_dist2(a0, a1, b0, b1) < P.d2[r] ? R(1) : R(0);
    }
    return hits;
}

// Cost part of one step: the force estimate of Eq. 13 (FORCE) from the
// factor of M (fac; when null, the one group_dynamics left in X with
// HANDOFF, else M's rows in X factorised again) and the Jacobian rows left
// in X, and this lane's running cost at (x_t, v_t): pose and
// force terms in lane 7 (pee, Re: its EE pose), joint-limit and torque
// terms in lanes 0..6 (the collision term is group_hits').  Uses the kGxOm
// part of X.
template <typename R, bool FORCE, class G, bool FDYN = false, bool HANDOFF = false>
MPPI_HD R group_cost(const G& g, const GroupLink<R>& L, const CostM<R>& C, const GroupCostW<R>& W,
                     const TargetM<R>& tg, const R* grav, R* X, const GroupFactor<R>* fac, R q, R qd, R v,
                     const R* pee, const R* Re, R* Fout = nullptr)
{
    const int j = g.j;
    const bool ee = j == kGroup - 1;
    R sj[6];   // this lane's motion subspace (the gravity torque of tau_F)
#pragma unroll
    for (int a = 0; a < 6; ++a) sj[a] = X[kGxSF + j * 6 + a];
    sched_fence();   // with the handoff reads: one round trip
    R ell = R(0);
    if (FORCE) {
        // tau_F of this lane's joint: v, less the gravity torque
        // S . Ic (0, -g) of the subtree when force_mode is 0
        if (!FDYN) {
            // the gravity torque is formed whatever force_mode says, so that
            // its reads join the step's first batch instead of a branch
            const R* hj = X + kGxH + j * 12;
            const R ag[3] = {-grav[0], -grav[1], -grav[2]};
            R ha[3];
            cross3(hj + 6, ag, ha);
            const R tg0 = v - (dot3(sj, ha) + hj[9] * dot3(sj + 3, ag));
            const R tf = W.force_mode == 0 ? tg0 : v;
            X[kGxTf + j] = ee ? R(0) : tf;
        }
        // row r of the EE Jacobian about p_ee at joint i: z_i (r < 3), then
        // (p_i - p_ee) x z_i, i.e. component r of the motion subspace S_i
        // about the EE point
        const int r = j < 6 ? j : 5;
        R Jr[NJ];
#pragma unroll
        for (int i = 0; i < NJ; ++i) Jr[i] = X[kGxSF + i * 6 + r];
        g.sync();
        GroupFactor<R> local;
        if (!fac && HANDOFF) {
            // the factor that group_dynamics left in the kGxOm rows
#pragma unroll
            for (int i = 0; i < NJ; ++i) {
#pragma unroll
                for (int c = 0; c < i; ++c) local.Lm[i][c] = X[kGxOm + i * 8 + c];
                local.id[i] = X[kGxOm + i * 8 + i];
            }
        } else if (!fac) {
            group_factor(X + kGxRow, local, (R*)nullptr);
        }
        const GroupFactor<R>& Fc = fac ? *fac : local;
        R bF[NJ];
#pragma unroll
        for (int i = 0; i < NJ; ++i) bF[i] = X[kGxTf + i];
        // 1 / d of this lane's joint (lane 7: of joint 6, weighted 0 below)
        const int jr = j < NJ ? j : NJ - 1;
        R idj = Fc.id[0];
        if (!fac && HANDOFF) {
            idj = X[kGxOm + jr * 8 + jr];
        } else {
#pragma unroll
            for (int i = 1; i < NJ; ++i) idj = jr == i ? Fc.id[i] : idj;
        }
        // ---- lane r < 6 solves for row r of J, lane 6 (and 7) for tau_F:
        // with M = L D L^T, column j of L^-1 [J^T | tau_F]
        R col[NJ];
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            R s = j < 6 ? Jr[i] : bF[i];
#pragma unroll
            for (int c = 0; c < i; ++c) s = fma_(-Fc.Lm[i][c], col[c], s);
            col[i] = s;
        }
        // transposed through the group's area: joint j's row in lane j,
        // scaled by D^-1/2 a row of [A^T | y] with Omega = A A^T and
        // J M^-1 tau_F = A y (A^T = D^-1/2 L^-1 J^T)
        g.sync();
#pragma unroll
        for (int i = 0; i < NJ; ++i) X[kGxOm + i * 8 + j] = col[i];
        g.sync();
        R a[NJ];
        const R sD = rsqrt_sqrt_(idj) * L.live;
#pragma unroll
        for (int c = 0; c < NJ; ++c) a[c] = X[kGxOm + jr * 8 + c] * sD;
        // least squares A^T x = y by modified Gram-Schmidt over the lanes
        // (lsq_wrench's factorisation)
        R Rm[6][NJ], idg[6], bb[6];
        group_mgs_step<0>(g, a, Rm, idg);
        group_mgs_step<1>(g, a, Rm, idg);
        group_mgs_step<2>(g, a, Rm, idg);
        group_mgs_step<3>(g, a, Rm, idg);
        group_mgs_step<4>(g, a, Rm, idg);
        group_mgs_step<5>(g, a, Rm, idg);
        // x = Rm^-1 Q^T y in every lane: (moment, force) about p_ee
#pragma unroll
        for (int s = 5; s >= 0; --s) {
            R t = Rm[s][6];
#pragma unroll
            for (int c = s + 1; c < 6; ++c) t = fma_(-Rm[s][c], bb[c], t);
            bb[s] = t * idg[s];
        }
        const R F[6] = {bb[3], bb[4], bb[5], bb[0], bb[1], bb[2]};
        if (ee) ell += group_force_cost(W, tg, F);
        if (Fout) {
#pragma unroll
            for (int a = 0; a < 6; ++a) Fout[a] = F[a];
        }
    }
    if (ee) ell += pose_cost(W, tg, pee, Re);
    else ell += joint_cost1(W, L, q, qd) + W.w_tau * sq(hinge(abs_(v) - L.taumax));
    return ell;
}

// One step of Eqs. 5-7 and the running cost at the pre-step state (x_t,
// v_t) on one group of lanes: returns this lane's share of l_t and sets
// qdd (0 in lane 7).
template <typename R, bool FORCE, class G, bool COLL = false>
MPPI_HD R group_step(const G& g, const GroupLink<R>& L, const CostM<R>& C, const TargetM<R>& tg, const R* grav,
                     int ext, R q, R qd, R tau, R v, R& qdd, GroupStepOut<R>* dbg = nullptr)
{
    GroupFactor<R> fac;
    R p[3], Q[9], F[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
    qdd = group_dynamics<R, FORCE, G, COLL>(g, L, C, grav, ext, q, qd, tau, v, g.shm, &fac, p, Q);
    GroupCostW<R> W;
    group_cost_w(C, W);
    R ell = group_cost<R, FORCE, G, COLL>(g, L, C, W, tg, grav, g.shm, &fac, q, qd, v, p, Q, F);
    if (COLL) {
        g.sync();   // the other lanes' handoff
        GroupPairs<R> gp;
        group_pairs(C, g.j, gp);
        ell += C.w_coll * group_hits<0, 1>(gp, C, g.shm);
    }
    if (dbg) {
        dbg->qdd = qdd;
#pragma unroll
        for (int a = 0; a < 3; ++a) dbg->pee[a] = p[a];
#pragma unroll
        for (int a = 0; a < 9; ++a) dbg->Re[a] = Q[a];
#pragma unroll
        for (int a = 0; a < 6; ++a) dbg->F[a] = F[a];
    }
    return ell;
}

// Terminal cost phi(x_T) = w_T (C_pos + C_ori + C_joint)(x_T): this lane's share.
template <typename R, class G>
MPPI_HD R group_terminal(const G& g, const GroupLink<R>& L, const CostM<R>& C, const TargetM<R>& tg, R q, R qd)
{
    GroupCostW<R> W;
    group_cost_w(C, W);
    R Q[9], p[3];
    group_fk(g, L, q, Q, p);
    const R s = g.j == kGroup - 1 ? pose_cost(W, tg, p, Q) : joint_cost1(W, L, q, qd);
    return C.w_T * s;
}

// One sample's rollout on the group (Eq. 3 with the dynamics of Sec. III-A):
// returns the sample's total cost S_k in every lane.  Us: [T][7] nominal
// torques; te: this lane's joint-space external torque (constant mode);
// noise_out, noise_lds (either may be null): du[t][j] of this lane's joint
// at (7 t + j) * stride (lanes 0..6).  split: each step as its dynamics
// part and then its cost part (group_dynamics, group_cost with the factor
// of M handed over in the group area) instead of group_step.
template <typename R, bool FORCE, class G, typename UT, bool COLL = false>
MPPI_HD R group_rollout(const G& g, const GroupLink<R>& L, const CostM<R>& C, const TargetM<R>& tg,
                        const R* grav, R q, R qd, R te, const UT* Us, int T, uint64_t seed, uint32_t tick,
                        uint32_t k, R* noise_out, size_t noise_stride, R* noise_lds = nullptr, int lds_stride = 0,
                        bool split = false)
{
    const int j = g.j;
    const int jc = j < NJ ? j : NJ - 1;
    const int ext = C.ext_mode == EXTW_WALL ? EXTW_WALL : EXTW_NONE;
    const R dt = C.dt;
    GroupCostW<R> W;
    group_cost_w(C, W);
    GroupPairs<R> gp;
    if (COLL) group_pairs(C, j, gp);
    R du = R(0), S = R(0);
    for (int t = 0; t < T; ++t) {
        const R z = group_normal<R>(seed, tick, k, (uint32_t)t, j);
        du = group_noise_step(C.rho, L, z, du, t);
        if (noise_out && j < NJ) noise_out[(size_t)(t * NJ + j) * noise_stride] = du;
        if (noise_lds && j < NJ) noise_lds[(t * NJ + j) * lds_stride] = du;
        const R v = (R(Us[t * NJ + jc]) + du) * L.live;
        R qdd;
        if (split) {
            // the dynamics and cost parts in sequence, the factor of M
            // handed over through the group area instead of held in
            // registers across the cost part
            R p[3], Q[9];
            qdd = group_dynamics<R, FORCE, G, COLL, true>(g, L, C, grav, ext, q, qd, v + te, v, g.shm, nullptr, p, Q);
            S += group_cost<R, FORCE, G, COLL, true>(g, L, C, W, tg, grav, g.shm, nullptr, q, qd, v, p, Q);
            if (COLL) {
                g.sync();   // the other lanes' handoff
                S += C.w_coll * group_hits<0, 1>(gp, C, g.shm);
            }
        } else {
            S += group_step<R, FORCE, G, COLL>(g, L, C, tg, grav, ext, q, qd, v + te, v, qdd);
        }
        qd += qdd * dt;
        q += qd * dt;
    }
    S += group_terminal(g, L, C, tg, q, qd);
    return g.sum(S);
}

}  // namespace mppi
