// Hand-written adjoint of log|Psi| and E_L (gfx950, FP64): derivatives with
// respect to the primitive exponents, the MO coefficients and the Jastrow
// parameters (Pade b; the e-n and e-e-n parameters of the many-body
// appendix when present) (Methods, eq. nabla_loss needs d log|Psi| / d theta),
// and with respect to the nuclear positions (Methods, eq. force needs
// d E_L / d R and d ln rho / d R = 2 d log|Psi| / d R).
//
// With a_e[m] = d log Sigma / d phi_m(r_e) from the shared stages:
//   d log|Psi| / d theta = sum_e sum_mu t_mu d chi_mu(r_e) / d theta,
//   t_mu = sum_m C[mu][m] a_e[m]  (plus d J / d b for theta = b).
// The kinetic energy is E_kin = -1/2 sum_{e,m} a_e[m] B[e][m] + (Jastrow-only
// terms) with B = lap phi + 2 grad_e J . grad phi, so
//   d E_kin = -1/2 sum_{e,m} [adot_e[m] d phi[e][m] + a_e[m] d B[e][m]],
// where adot = (d^2 log Sigma / d phi d phi) B is the Hessian-vector product
// of log Sigma along B.  adot is the forward-mode derivative of the
// determinant algebra (Gauss-Jordan tables, determinant ratios, cofactors,
// a_e) in the direction phi -> phi + eps B:
//   Tdot = A0^-1 (B - B0 T),  Ainvdot = -A0^-1 B0 A0^-1,
//   rho_dot, Sdot, Cdot from the k <= 2 minors, and
//   adot_e[v] = (Ainvdot^T C + A0^-T Cdot)[e][v] / S - a_e[v] Sdot / S,
//   adot_e[k] = Ainvdot[k][e] - sum_v (Tdot[k][v] a_e[v] + T[k][v] adot_e[v]).
// Moving nucleus alpha moves its AOs: d chi(r - R) / d R = -grad chi, so the
// force terms need AO Hessians and gradients of AO Laplacians.

#include "qmc_walker.h"

namespace qmc {
namespace {

using namespace walker;

struct GradOut {
    double *dlogpsi;     // [W][P] or NULL
    double *deloc_dth;   // [W][P] or NULL
    double *dlogpsi_dR;  // [W][A][3] or NULL
    double *deloc_dR;    // [W][A][3] or NULL
    int n_param;
};

// Doubles from row to row of the main pass: 64 and four more, so that the four
// rows which put_mo_gradient reads at once lie in different banks.
constexpr int kGradRow = kWave + 4;

// LDS of the gradient kernel (doubles).  Per walker, from its base: the
// shared stages' tables (walker_lds, full layout), then the forward-mode
// tables [2][2][n_max][NMO]: Tdot / Ainvdot, and the slot-indexed rows
// (B0 | Z) that Cdot replaces.  Once a_e and its derivative are in registers
// all of it is dead and the wave's rows take the block from its start:
// a [NMO], adot [NMO] and the two rings [kRing] of kGradRow in the main pass;
// after them each walker's positions [LW][3] and e-e-n tables of the Jastrow
// directions, [LW][n_atoms][2 een_n] factors and [LW][n_atoms][kEenGeo]
// geometry.  The per-nucleus results [n_atoms][6] per walker live past the
// end of all.  (CO: 39.6 KB, so four waves share a compute unit; with a row of
// 2 n_ao + 2 NMO doubles per electron for the MO-coefficient products it was
// 49 KB and three.)
template <int NMO>
__host__ __device__ inline int grad_walker(const DevSystem &S) {
    const int nmax = S.n_up > S.n_dn ? S.n_up : S.n_dn;
    const int fwd = walker_lds<NMO>(S) + 4 * nmax * NMO;
    const int jas = 3 * S.LW + S.LW * S.n_atoms * (S.een_n > 0 ? 2 * S.een_n + kEenGeo : 0);
    return ((fwd > jas ? fwd : jas) + 1) & ~1;
}

template <int NMO>
__host__ __device__ inline int grad_wave(const DevSystem &S) {
    const int walkers = S.WPW * grad_walker<NMO>(S), rows = (2 * NMO + 2 * kRing) * kGradRow;
    return walkers > rows ? walkers : rows;
}

template <int NMO>
__host__ __device__ inline size_t grad_lds(const DevSystem &S) {
    return (size_t)grad_wave<NMO>(S) + (size_t)S.WPW * 6 * S.n_atoms;
}

// Derivative of the k <= 2 minor det T[H,P] along Tdot, from a packed
// excitation code (ratio_code).
template <int NMO>
__device__ __forceinline__ double ratio_code_dot(const double *T, const double *Td, uint32_t c) {
    const uint32_t k = c & 3u;
    if (k == 0) return 0.0;
    const int h1 = (c >> 2) & 7, h2 = (c >> 5) & 7, p1 = (c >> 8) & 31, p2 = (c >> 13) & 31;
    const int a = h1 * NMO + p1;
    if (k == 1) return Td[a];
    const int b = h2 * NMO + p2, d = h1 * NMO + p2, e = h2 * NMO + p1;
    return Td[a] * T[b] + T[a] * Td[b] - Td[d] * T[e] - T[d] * Td[e];
}

// Components of one shell, in AO order: fn(c, P, P_x, P_y, P_z, lap P) of the
// monomials P of angular momentum l.
template <typename Fn>
__device__ __forceinline__ void shell_monomials(int l, double dx, double dy, double dz, Fn fn) {
    if (l == 0) {
        fn(0, 1.0, 0.0, 0.0, 0.0, 0.0);
    } else if (l == 1) {
        fn(0, dx, 1.0, 0.0, 0.0, 0.0);
        fn(1, dy, 0.0, 1.0, 0.0, 0.0);
        fn(2, dz, 0.0, 0.0, 1.0, 0.0);
    } else {
        fn(0, dx * dx, 2.0 * dx, 0.0, 0.0, 2.0);
        fn(1, dx * dy, dy, dx, 0.0, 0.0);
        fn(2, dx * dz, dz, 0.0, dx, 0.0);
        fn(3, dy * dy, 0.0, 2.0 * dy, 0.0, 2.0);
        fn(4, dy * dz, 0.0, dz, dy, 0.0);
        fn(5, dz * dz, 0.0, 0.0, 2.0 * dz, 2.0);
    }
}

// Radial sums of one shell: R, R'/r, R'' + (2l+2) R'/r, (R'' - R'/r) / r^2
// and (d/dr of the third) / r.
struct Radial {
    double v, d, l, dd, l1;
};

// What an exponent's derivatives need of the shell: the sums q of t P,
// A1 = td P + t lap P + 2 t grad P . grad J, and B = 2 q d . grad J.
struct ExpoSums {
    double q, A1, B;
};

// One primitive f's share of the radial sums, and its exponent's derivative of
// log|Psi| (gl) and E_L (ge) at this electron.  With fz = df/dzeta
// (normalisation included: fz = f (qn - r) or f (qn - r^2)),
//   gl = fz q,  ge = -1/2 (fz A1 + d(R'/r)/dzeta B + d(R'' + (2l+2) R'/r)/dzeta q).
__device__ __forceinline__ void radial_prim(const DevSystem &S, double2v pe, double qn, int l, int kn, double r,
                                            double r2, double rinv, double rk, const ExpoSums &z, Radial &R, double &gl,
                                            double &ge) {
    const double ex = pe.x;
    if (S.basis == 0) {
        const double f = pe.y * rk * exp_f64(-ex * r);
        const double kr = kn * rinv, g = kr - ex, l2 = (2.0 * l + 2.0) * rinv;
        const double L = g * g - kr * rinv + l2 * g;
        const double Lp = -2.0 * g * kr * rinv + 2.0 * kr * rinv * rinv - l2 * (kr * rinv + g * rinv);
        R.v += f;
        R.d += f * g * rinv;
        R.l += f * L;
        R.dd += f * (g * g - kr * rinv - g * rinv) * rinv * rinv;
        R.l1 += (f * g * L + f * Lp) * rinv;
        const double fz = f * (qn - r);
        gl = fz * z.q;
        ge = -0.5 * (fz * z.A1 + (fz * g - f) * rinv * z.B + (fz * L + f * (-2.0 * g - l2)) * z.q);
    } else {
        const double f = pe.y * exp_f64(-ex * r2);
        const double F = 4.0 * l + 6.0, s = 4.0 * ex * r2 - F, Q = ex * s;  // lap factor Q, 8 ex r^2 - F = 2 s + F
        const double e2 = -2.0 * ex, ef = e2 * f;
        R.v += f;
        R.d += ef;
        R.l += f * Q;
        R.dd += e2 * ef;
        R.l1 += ef * (Q + 2.0 * e2);
        const double fz = f * (qn - r2);
        gl = fz * z.q;
        ge = -0.5 * (fz * (z.A1 + e2 * z.B + Q * z.q) + f * ((2.0 * s + F) * z.q - 2.0 * z.B));
    }
}

// Ends a batch of two table columns whose results are v..: without a line
// between batches the compiler reads the whole table ahead of the
// multiply-adds and spills it.
__device__ __forceinline__ void batch_end(double &v) { asm volatile("" : "+v"(v) : : "memory"); }
template <typename... T>
__device__ __forceinline__ void batch_end(double &v, T &...more) {
    batch_end(v);
    batch_end(more...);
}

__device__ __forceinline__ double power(double r, int kn) {
    double rk = 1.0;
    for (int t = 0; t < kn; ++t) rk *= r;
    return rk;
}

// The MO-coefficient derivatives of four AOs, sum over a walker's electrons
// of chi a (log|Psi|) and chi adot + beta a (E_L), as products of 4 AOs x 4
// electrons x 4 MOs with four walkers to an instruction (lane 16 k + 4 b + i:
// AO i or MO i of walker b at electron k of the step), written straight to
// the outputs.  chi / beta: the ring rows of the four AOs; sA / sAd: rows of
// a and adot per MO.
template <int NMO>
__device__ __forceinline__ void put_mo_gradient(const DevSystem &S, int lane, int64_t wave_first, int64_t W, int mu0,
                                                const double *chi, const double *beta, const double *sA,
                                                const double *sAd, const int (&col_of)[NMO / 4], const GradOut &G) {
    constexpr int MB = NMO / 4;
    const int k = lane >> 4, b = (lane >> 2) & 3, i = lane & 3;
    const int steps = S.LW >= 4 ? S.LW / 4 : 1;  // products per walker
    const int row = ((mu0 + i) & (kRing - 1)) * kGradRow;
    const bool own = S.LW >= 4 || k < S.LW;      // two-lane walkers fill half of the step
    // this lane's result: AO mu0 + k, MO 4 s + i of walker b of the set.  The
    // factors come by scalar loads: a vector load would wait for every store
    // before it.
    const int mu = mu0 + k;
    double f = 0.0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const double ft = const_tab(S.ao_angf)[mu0 + t < S.n_ao ? mu0 + t : 0];
        f = k == t ? ft : f;
    }
    wave_sync();
    for (int set = 0; set < S.WPW / 4; ++set) {
        const int64_t w = wave_first + 4 * set + b;
        double gl[MB], ge[MB];
#pragma unroll
        for (int s = 0; s < MB; ++s) gl[s] = ge[s] = 0.0;
        for (int q = 0; q < steps; ++q) {
            const int col = (4 * set + b) * S.LW + (own ? 4 * q + k : 0);
            double c = chi[row + col], be = beta[row + col], av[MB], ad[MB];
#pragma unroll
            for (int s = 0; s < MB; ++s) {
                av[s] = sA[(4 * s + i) * kGradRow + col];
                ad[s] = sAd[(4 * s + i) * kGradRow + col];
            }
            c = own ? c : 0.0;
            be = own ? be : 0.0;
#pragma unroll
            for (int s = 0; s < MB; ++s) {
                gl[s] = __builtin_amdgcn_mfma_f64_4x4x4f64(c, av[s], gl[s], 0, 0, 0);
                ge[s] = __builtin_amdgcn_mfma_f64_4x4x4f64(c, ad[s], ge[s], 0, 0, 0);
                ge[s] = __builtin_amdgcn_mfma_f64_4x4x4f64(be, av[s], ge[s], 0, 0, 0);
            }
        }
        if (w < W && mu < S.n_ao) {
#pragma unroll
            for (int s = 0; s < MB; ++s) {
                if (col_of[s] >= 0) {
                    const int64_t out = w * G.n_param + S.n_prim + mu * S.n_mo + col_of[s];
                    if (G.dlogpsi) G.dlogpsi[out] = f * gl[s];
                    if (G.deloc_dth) G.deloc_dth[out] = -0.5 * f * ge[s];
                }
            }
        }
    }
    wave_sync();
}

// Sums over a walker's electrons of a derivative of log|Psi| and of E_L.  The
// walker's first lane keeps the first, the first lane of its upper half the
// second (span_sum_pair).  Idle lanes add zeros, whatever they bring (NaN with a
// nucleus at their far point).
struct WalkerOut {
    double *param;  // this lane's row of the parameter output, or NULL
    double *atom;   // this lane's column of the walker's nuclear sums in LDS, or NULL
    int LW;
    bool upper, active;

    __device__ __forceinline__ WalkerOut(const GradOut &G, const Lane &L, int LW_, int64_t w, double *sAtom) {
        LW = LW_;
        active = L.active;
        upper = L.lw >= LW / 2;
        param = atom = nullptr;
        if (L.wvalid && (L.lw == 0 || L.lw == LW / 2)) {
            double *p = upper ? G.deloc_dth : G.dlogpsi;
            if (p) param = p + w * G.n_param;
            atom = sAtom + (upper ? 3 : 0);
        }
    }
    __device__ __forceinline__ void put(int at, double l, double e) const {
        const double v = span_sum_pair(active ? l : 0.0, active ? e : 0.0, LW, upper);
        if (param) param[at] = v;
    }
    __device__ __forceinline__ void add_atom(int a, const double (&l)[3], const double (&e)[3], double f = 1.0) const {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double v = span_sum_pair(active ? f * l[k] : 0.0, active ? f * e[k] : 0.0, LW, upper);
            if (atom) atom[6 * a + k] += v;
        }
    }
};

// A radial function f(|x - c|) added to J: lap f = f'' + 2 f'/r, grad f = f' u.
// Its share of d E_L is -1/2 (f'' + 2 f'/r) - (h . u) f'.
__device__ __forceinline__ double radial_energy(double f1, double f2, double ri, double hu) {
    return -0.5 * f2 - f1 * (ri + hu);
}

// Derivatives with respect to the Jastrow parameters (Pade b; e-n (w0, w1,
// w2) per nucleus; e-e-n (c, a1, b1, a2, b2, a3, b3) per term) and the
// Jastrow's part of the nuclear gradients, added to the walker's sums.  With
// h = grad_e log|Psi| a change dJ of the Jastrow factor changes E_L by
// -1/2 sum_e (lap_e dJ + 2 h_e . grad_e dJ), a functional linear in dJ.
//
// e-e-n: for an own factor o(u) (u the distance of this electron from the
// nucleus, t its unit vector) and a pair factor s(r), w the pair's unit
// vector, the functional of o s is alpha s + (beta . w) s' + gamma (s'' + 2 s'/r),
//   alpha = -1/2 (o'' + 2 o'/u) - o' h . t,  beta = -(o' t + o h),  gamma = -o / 2,
// times the partner's factor p.  So one pass over the partners per term and
// nucleus gives every direction: the parameters c, a1, a2, a3 scale the
// term; the partner's b and nuclear derivative replace p by dp (dg/db = -g^2,
// dp/dR = -p' t_j), b3 replaces s, and the own factor's b and nuclear
// derivative only need the sums A, B, D of jastrow_terms.  A forward-mode
// pass per direction ran the pair loop 48 times for CO with 5 terms; a pass per
// nucleus formed each pair's part twice (134 k cycles of a wave, now 112 k;
// 4099 walkers 284 -> 264 us).
__device__ __forceinline__ void jastrow_derivs(const DevSystem &S, const Lane &L, double x0, double x1, double x2,
                                               const double (&h)[3], const double *sPos, const double *sF,
                                               const double *sG, const GradOut &G, const WalkerOut &out) {
    const bool need_R = G.dlogpsi_dR || G.deloc_dR;
    const int p_b = S.n_prim + S.n_ao * S.n_mo;  // output index of b
    const int p_en = p_b + 1, p_een = p_en + (S.jas_en ? 3 * S.n_atoms : 0);
    const int e_ = L.active ? L.e : 0;  // idle lanes take electron 0's partners
    // ---- Pade b: K = a g, dK/db = -a g^2 ------------------------------------
    double dl = 0.0, de = 0.0;
    {
#pragma unroll 2
        for (int t = 1; t < S.ne; ++t) {
            int lj;
            const int j = partner(S, e_, t, &lj);
            const double d0 = x0 - sPos[3 * lj], d1 = x1 - sPos[3 * lj + 1], d2 = x2 - sPos[3 * lj + 2];
            const Sep s = separation(d0, d1, d2);
            const double a = (j < S.n_up) == (e_ < S.n_up) ? S.a_par : S.a_anti;
            const Pade p = pade(S.b, s.r);
            const double hw = (h[0] * d0 + h[1] * d1 + h[2] * d2) * s.ri;
            dl -= 0.5 * a * p.g * p.g;
            de += radial_energy(-2.0 * a * p.g * p.g1, a * p.q * p.g1 * (6.0 * S.b * p.g - 2.0), s.ri, hw);
        }
    }
    out.put(p_b, dl, de);
    // ---- e-n parameters and nuclear part --------------------------------------
    if (S.jas_en) {
        for (int a = 0; a < S.n_atoms; ++a) {
            double l3[3] = {0.0, 0.0, 0.0}, e3[3] = {0.0, 0.0, 0.0};
            double lr[3] = {0.0, 0.0, 0.0}, er[3] = {0.0, 0.0, 0.0};
            {
                const auto *R = const_tab(S.atoms) + 4 * a;
                const auto *wn = const_tab(S.jas_en) + 3 * a;
                const double d[3] = {x0 - R[0], x1 - R[1], x2 - R[2]};
                const Sep s = separation(d[0], d[1], d[2]);
                const double r = s.r, w0 = wn[0], w1 = wn[1], w2 = wn[2];
                // (the full division as in the value; w2 q first, 2 w2 may overflow)
                const double q = 1.0 / (1.0 + w2 * r), wq = w2 * q;
                const Pade p = {q, r * q, q * q, -2.0 * wq * q * q};
                const double u[3] = {d[0] * s.ri, d[1] * s.ri, d[2] * s.ri};
                const double hu = h[0] * u[0] + h[1] * u[1] + h[2] * u[2];
                // K = (w0 r + w1 r^2) q and its derivatives in r
                const double K = (w0 + w1 * r) * p.g, K1 = (w0 + 2.0 * w1 * r - K * w2) * p.q;
                const double K2 = (2.0 * w1 - 2.0 * K1 * w2) * p.q, K3 = -3.0 * wq * K2;
                // dK/dw0 = g, dK/dw1 = r g, dK/dw2 = -K g
                l3[0] = p.g;
                e3[0] = radial_energy(p.g1, p.g2, s.ri, hu);
                l3[1] = r * p.g;
                e3[1] = radial_energy(p.g + r * p.g1, 2.0 * p.g1 + r * p.g2, s.ri, hu);
                l3[2] = -K * p.g;
                e3[2] = radial_energy(-(K1 * p.g + K * p.g1), -(K2 * p.g + 2.0 * K1 * p.g1 + K * p.g2), s.ri, hu);
                // d/dR_x: K -> -K' u_x; lap -> -(K''' + 2 K''/r - 2 K'/r^2) u_x;
                // grad -> -(K'' - K'/r) u_x u - (K'/r) e_x
                const double kr = K1 * s.ri;
                const double c = 0.5 * (K3 + 2.0 * s.ri * (K2 - kr)) + (K2 - kr) * hu;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    lr[k] = -K1 * u[k];
                    er[k] = c * u[k] + kr * h[k];
                }
            }
            for (int k = 0; k < 3; ++k) out.put(p_en + 3 * a + k, l3[k], e3[k]);
            if (need_R) out.add_atom(a, lr, er);
        }
    }
    // ---- e-e-n parameters and nuclear part --------------------------------------
    // (told to be rare, or the register allocator serves these nested loops before
    // the main pass, which every system runs: Li2 without e-e-n terms 216 against
    // 212 us, many-body CO 271 against 272 us)
    if (__builtin_expect_with_probability(S.een_n > 0, 1, 0.01))
    for (int m = 0; m < S.een_n; ++m) {
        const auto *tm = const_tab(S.jas_een) + 7 * m;
        const double c = tm[0], a1 = tm[1], b1 = tm[2], a2 = tm[3], b2 = tm[4], a3 = tm[5], b3 = tm[6];
        const double kc = c * a1 * a2 * a3;
        // this term with unit coefficients, and the b1, b2, b3 directions
        double l0 = 0.0, e0 = 0.0, lb1 = 0.0, eb1 = 0.0, lb2 = 0.0, eb2 = 0.0, lb3 = 0.0, eb3 = 0.0;
        // NR factors of an own electron: one when f1 = f2 (both roles then share
        // its functional), and two nuclei at a time, which share the pair's part
        auto term = [&](auto roles) {
            constexpr int NR = decltype(roles)::value, NA = NR == 1 ? 2 : 1;
            for (int a0 = 0; a0 < S.n_atoms; a0 += NA) {
                double lr[NA][3] = {}, er[NA][3] = {};
                {
                    double ui[NA], tv[NA][3], ht[NA], al[NA][NR], be[NA][NR][3], ga[NA][NR];
                    Pade q[NA][NR];
                    const double *fj[NA];  // partner 0's table entries of the nucleus
                    bool on[NA];
#pragma unroll
                    for (int n = 0; n < NA; ++n) {
                        on[n] = a0 + n < S.n_atoms;
                        const int a = on[n] ? a0 + n : a0;
                        const double *g = sG + (L.lw * S.n_atoms + a) * kEenGeo;
                        ui[n] = g[4];
                        for (int k = 0; k < 3; ++k) tv[n][k] = g[1 + k];
                        ht[n] = h[0] * tv[n][0] + h[1] * tv[n][1] + h[2] * tv[n][2];
                        // own factor's functional in each role (0: electron i, factor 1)
#pragma unroll
                        for (int r = 0; r < NR; ++r) {
                            const Pade p = pade(r == 0 ? b1 : b2, g[0]);
                            q[n][r] = p;
                            al[n][r] = radial_energy(p.g1, p.g2, ui[n], ht[n]);
                            ga[n][r] = -0.5 * p.g;
                            for (int k = 0; k < 3; ++k) be[n][r][k] = -(p.g1 * tv[n][k] + p.g * h[k]);
                        }
                        fj[n] = sF + (a * S.een_n + m) * 2;
                    }
                    // sums over the partners by role; pl, pe the partner's b
                    double A[NA][2] = {}, B[NA][2][3] = {}, D[NA][2] = {};
                    double pl = 0.0, pe[2] = {0.0, 0.0};
                    for (int t = 1; t < S.ne; ++t) {
                        int lj;
                        const int j = partner(S, e_, t, &lj);
                        const bool first = e_ > j;
                        const double d0 = x0 - sPos[3 * lj], d1 = x1 - sPos[3 * lj + 1], d2 = x2 - sPos[3 * lj + 2];
                        const Sep s = separation(d0, d1, d2);
                        const Pade p3 = pade(b3, s.r);
                        const double w0 = d0 * s.ri, w1 = d1 * s.ri, w2 = d2 * s.ri;
                        const double lap = p3.g2 + 2.0 * p3.g1 * s.ri;
                        // the pair factor along b3: ds = -s^2, ds' = -2 s s', ds'' = q^3 (6 b s - 2)
                        const double s3 = -p3.g * p3.g, s31 = -2.0 * p3.g * p3.g1;
                        const double lap3 = p3.q * p3.g1 * (6.0 * b3 * p3.g - 2.0) + 2.0 * s31 * s.ri;
                        const double v0 = p3.g1 * w0, v1 = p3.g1 * w1, v2 = p3.g1 * w2;
#pragma unroll
                        for (int n = 0; n < NA; ++n) {
                            // partner's factor p, p' = (p / r_aj)^2, dp/db = -p^2
                            const double *gj = sG + (lj * S.n_atoms + (on[n] ? a0 + n : a0)) * kEenGeo;
                            const double pt = fj[n][lj * S.n_atoms * S.een_n * 2 + (first ? 1 : 0)];
                            const double p = on[n] ? pt : 0.0;
                            const double pq = p * gj[4], pd = pq * pq;
                            const int r1 = NR - 1;
                            const double o = first ? q[n][0].g : q[n][r1].g;
                            const double bw = (first ? be[n][0][0] : be[n][r1][0]) * w0 +
                                              (first ? be[n][0][1] : be[n][r1][1]) * w1 +
                                              (first ? be[n][0][2] : be[n][r1][2]) * w2;
                            const double alr = first ? al[n][0] : al[n][r1], gar = first ? ga[n][0] : ga[n][r1];
                            // functional of o s, and of o ds/db3
                            const double es = alr * p3.g + bw * p3.g1 + gar * lap;
                            eb3 += p * (alr * s3 + bw * s31 + gar * lap3);
                            const double op = first ? o * p : 0.0;  // the pair's value is counted at i
                            lb3 += op * s3;
                            const double jv = first ? o * p3.g : 0.0;
                            pl -= p * p * jv;
                            const double pp = p * p * es;
#pragma unroll
                            for (int r = 0; r < 2; ++r) {
                                const double pr = first == (r == 0) ? p : 0.0;
                                A[n][r] += pr * p3.g;
                                B[n][r][0] += pr * v0;
                                B[n][r][1] += pr * v1;
                                B[n][r][2] += pr * v2;
                                D[n][r] += pr * lap;
                                pe[r] -= first == (r == 0) ? pp : 0.0;
                            }
#pragma unroll
                            for (int k = 0; k < 3; ++k) {
                                const double dp = -pd * gj[1 + k];
                                lr[n][k] += dp * jv;
                                er[n][k] += dp * es;
                            }
                        }
                    }
                    // role 0's partners hold factor 2, role 1's factor 1
                    lb2 += pl;
                    eb2 += pe[0];
                    eb1 += pe[1];
#pragma unroll
                    for (int n = 0; n < NA; ++n) {
                        l0 += q[n][0].g * A[n][0];
#pragma unroll
                        for (int r = 0; r < 2; ++r) {
                            const int v = r < NR ? r : 0;
                            const Pade &o = q[n][v];
                            const double *Br = B[n][r], *br = be[n][v];
                            const double bB = br[0] * Br[0] + br[1] * Br[1] + br[2] * Br[2];
                            e0 += al[n][v] * A[n][r] + bB + ga[n][v] * D[n][r];
                            // own b: o -> do = -g^2, do' = -2 g g', do'' = q^3 (6 b g - 2)
                            const double bo = r == 0 ? b1 : b2;
                            const double og = -o.g * o.g, og1 = -2.0 * o.g * o.g1;
                            const double og2 = o.q * o.g1 * (6.0 * bo * o.g - 2.0);
                            const double hB = h[0] * Br[0] + h[1] * Br[1] + h[2] * Br[2];
                            const double tB = tv[n][0] * Br[0] + tv[n][1] * Br[1] + tv[n][2] * Br[2];
                            const double eo = radial_energy(og1, og2, ui[n], ht[n]) * A[n][r] - (og1 * tB + og * hB) -
                                              0.5 * og * D[n][r];
                            if (r == 0) {
                                lb1 += og * A[n][0];
                                eb1 += eo;
                            } else {
                                eb2 += eo;
                            }
                            // own factor's nuclear derivative: du = -t_x, dt = -(e_x - t_x t) / u
                            const double o3 = 6.0 * bo * bo * o.q * o.q * o.g1;
                            const double o1u = o.g1 * ui[n], c2 = o.g2 - o1u;
                            const double ct = (0.5 * (o3 + 2.0 * ui[n] * c2) + c2 * ht[n]) * A[n][r] + c2 * tB +
                                              o.g1 * hB + 0.5 * o.g1 * D[n][r];
#pragma unroll
                            for (int k = 0; k < 3; ++k) {
                                if (r == 0) lr[n][k] -= o.g1 * tv[n][k] * A[n][r];
                                er[n][k] += ct * tv[n][k] + o1u * (A[n][r] * h[k] + Br[k]);
                            }
                        }
                    }
                }
                if (need_R)
#pragma unroll
                    for (int n = 0; n < NA; ++n)
                        if (a0 + n < S.n_atoms) out.add_atom(a0 + n, lr[n], er[n], kc);
            }
        };
        if (a1 == a2 && b1 == b2) term(std::integral_constant<int, 1>());
        else term(std::integral_constant<int, 2>());
        const int at = p_een + 7 * m;
        out.put(at + 0, a1 * a2 * a3 * l0, a1 * a2 * a3 * e0);
        out.put(at + 1, c * a2 * a3 * l0, c * a2 * a3 * e0);
        out.put(at + 2, kc * lb1, kc * eb1);
        out.put(at + 3, c * a1 * a3 * l0, c * a1 * a3 * e0);
        out.put(at + 4, kc * lb2, kc * eb2);
        out.put(at + 5, c * a1 * a2 * l0, c * a1 * a2 * e0);
        out.put(at + 6, kc * lb3, kc * eb3);
    }
}

// RT: arithmetic of the forward evaluation's AO values and MO value
// contraction (double, or float for the mixed FP32 form); everything the
// adjoint adds is FP64.
//
// Bound by latency: the walkers' tables leave one wave per SIMD, so every
// stage keeps its LDS reads in batches (two table columns, all rows of a
// spin), its tables in scalar loads ahead of use, and its contractions on the
// matrix cores (direction B beside the MO values, the AO weights of a and
// adot, the MO-coefficient products).  Two things cost more than the arithmetic
// and are kept out of the main pass: LDS rows 64 doubles apart, whose reads by
// four rows at once met in the same banks (put_mo_gradient 82 k -> 28 k cycles
// of a CO wave with kGradRow), and vector loads behind stores, which wait for
// them.  All outputs, as first written with LDS rows per electron, then with
// the contractions here, then with these two and one reduction per pair of
// results: Li2, 32 768 walkers 542 -> 254 -> 209 us (175 MB written); CO, 8192
// walkers 564 -> 217 -> 161 us; many-body CO, 4099 walkers 2523 -> 349 -> 264 us.
// Idle lanes run unmasked and selects drop their shares: 211, 163 and 266 us.
template <int NMO, typename RT>
__global__ __launch_bounds__(kWave) void k_grad(DevSystem S, const double *__restrict__ X, int64_t W,
                                                GradOut G) {
    extern __shared__ double smem[];
    int64_t w;
    const int64_t wave_first = (int64_t)blockIdx.x * S.WPW;
    Lane L = make_lane(S, wave_first, W, &w);
    double *wsm = smem + L.wloc * grad_walker<NMO>(S);
    const int nmax = S.n_up > S.n_dn ? S.n_up : S.n_dn;
    const int ts = nmax * NMO;                 // doubles per spin table
    double *sT = wsm;                          // T tables (shared stages)
    double *sC = wsm + 2 * ts;                 // cofactor tables (shared stages)
    double *sTD = wsm + walker_lds<NMO>(S);    // Tdot, Ainvdot
    double *sCD = sTD + 2 * ts;                // B0 | Z rows, then Cdot

    double x0 = 0.0, x1 = 0.0, x2 = 0.0;
    if (L.active) {
        const double *p = X + (w * S.ne + L.e) * 3;
        x0 = p[0];
        x1 = p[1];
        x2 = p[2];
    }
    if (!L.active) {
        x0 = 100.0;
        x1 = 100.0;
        x2 = 100.0;
    }


    // ---- shared stages: MO values and direction B, Gauss-Jordan,
    // determinants, a_e ----
    Core<NMO> c;
    double bvec[NMO];
    core_stages<NMO, RT, 0, false, false, false, true>(S, L, wsm, x0, x1, x2, c, smem, &bvec);
    const double gJ[3] = {c.gJ0, c.gJ1, c.gJ2};
    const double *Tg = sT + L.grp * ts;
    const double *Cg = sC + L.grp * ts;
    double *TDg = sTD + L.grp * ts;
    double *CDg = sCD + L.grp * ts;
    const int sl = c.slot < 0 ? 0 : c.slot;
    const int last = L.nsig > 0 ? L.nsig - 1 : 0;  // last slot of this spin

    // ---- forward mode of the determinant algebra along B -----------------
    double adot[NMO];
    auto forward = [&](auto rows_of_spin) {
        constexpr int JMAX = kMaxSpin < NMO ? kMaxSpin : NMO;
        constexpr int KR = decltype(rows_of_spin)::value < JMAX ? decltype(rows_of_spin)::value : JMAX;
        // rows of this spin's tables (the last one again past it, where the
        // factors that multiply it are zero)
        int row[KR];
#pragma unroll
        for (int k = 0; k < KR; ++k) row[k] = (k < last ? k : last) * NMO;
        // slot-indexed rows: reference columns hold B0 = B[e][k], virtual
        // columns hold Z[e][v] = B[e][v] - sum_k B[e][k] T[k][v]
        {
            double bk[KR];
#pragma unroll
            for (int k = 0; k < KR; ++k) bk[k] = k < L.nsig ? bvec[k] : 0.0;
#pragma unroll
            for (int v = 0; v < NMO; v += 2) {
                double z0 = bvec[v], z1 = bvec[v + 1], s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int k = 0; k < KR; ++k) {
                    const double2 t = *(const double2 *)(Tg + row[k] + v);
                    s0 += bk[k] * t.x;
                    s1 += bk[k] * t.y;
                }
                batch_end(s0, s1);
                if (v >= L.nsig) z0 -= s0;
                if (v + 1 >= L.nsig) z1 -= s1;
                if (L.active && c.slot >= 0) *(double2 *)(CDg + c.slot * NMO + v) = make_double2(z0, z1);
            }
        }
        wave_sync();
        // row of this lane's slot: Tdot[s][v] = sum_s' Ainv[s][e(s')] Z[e(s')][v];
        // W[s][k] = (A0^-1 B0)[s][k]; Ainvdot[s][s''] = -sum_k W[s][k] Ainv[k][e(s'')]
        {
            double as[KR], wk[KR], td[NMO];
#pragma unroll
            for (int k = 0; k < KR; ++k) as[k] = k < L.nsig ? Tg[sl * NMO + k] : 0.0;
#pragma unroll
            for (int v = 0; v < NMO; v += 2) {
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int k = 0; k < KR; ++k) {
                    const double2 z = *(const double2 *)(CDg + row[k] + v);
                    s0 += as[k] * z.x;
                    s1 += as[k] * z.y;
                }
                batch_end(s0, s1);
                td[v] = s0;
                td[v + 1] = s1;
            }
#pragma unroll
            for (int k = 0; k < KR; ++k) wk[k] = k < L.nsig ? td[k] : 0.0;
#pragma unroll
            for (int v = 0; v < (KR < NMO ? KR : NMO); v += 2) {
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int k = 0; k < KR; ++k) {
                    const double2 t = *(const double2 *)(Tg + row[k] + v);
                    s0 -= wk[k] * t.x;
                    s1 -= wk[k] * t.y;
                }
                batch_end(s0, s1);
                if (v < L.nsig) td[v] = s0;
                if (v + 1 < L.nsig) td[v + 1] = s1;
            }
            if (L.active && c.slot >= 0) {
#pragma unroll
                for (int v = 0; v < NMO; v += 2) *(double2 *)(TDg + c.slot * NMO + v) = make_double2(td[v], td[v + 1]);
            }
        }
        wave_sync();
        for (int q = 2 * L.lw; q < 2 * ts; q += 2 * S.LW) *(double2 *)(sCD + q) = make_double2(0.0, 0.0);
        wave_sync();
        // derivatives of S and of the cofactor tables, from the same records
        // as their values
        const double *Tup = sT, *Tdn = sT + ts, *TDup = sTD, *TDdn = sTD + ts;
        double Sd = 0.0;
        for (int i0 = 0; i0 < S.det_rows; i0 += kRecBatch) {
            uint4v rb[kRecBatch];
#pragma unroll
            for (int u = 0; u < kRecBatch; ++u)
                rb[u] = i0 + u < S.det_rows ? const_tab((const uint4v *)S.det_recs)[(i0 + u) * S.LW + (lane_now() & (S.LW - 1))]
                                            : uint4v{0, 0, 0, 0};
#pragma unroll
            for (int u = 0; u < kRecBatch; ++u) {
                const uint4v r = rb[u];
                const double ru = ratio_code(Tup, r.z, NMO, 0), rd = ratio_code(Tdn, r.w, NMO, 0);
                Sd += __hiloint2double((int)r.y, (int)r.x) *
                      (ratio_code_dot<NMO>(Tup, TDup, r.z) * rd + ru * ratio_code_dot<NMO>(Tdn, TDdn, r.w));
            }
        }
        {
            double acc = 0.0;
            for (int i0 = 0; i0 < S.cof_rows; i0 += kRecBatch) {
                uint4v rb[kRecBatch];
#pragma unroll
                for (int u = 0; u < kRecBatch; ++u)
                    rb[u] = i0 + u < S.cof_rows ? const_tab((const uint4v *)S.cof_recs)[(i0 + u) * S.LW + (lane_now() & (S.LW - 1))]
                                                : uint4v{0, 0, 0, 0};
#pragma unroll
                for (int u = 0; u < kRecBatch; ++u) {
                    const uint4v r = rb[u];
                    const int spin = (r.w >> 1) & 1;
                    const double *Ts = spin ? Tdn : Tup, *TDs = spin ? TDdn : TDup;
                    const double *To = spin ? Tup : Tdn, *TDo = spin ? TDup : TDdn;
                    const uint32_t cc = r.z >> 18, oc = r.z & 0x3FFFFu;
                    const int at = ((cc >> 2) & 7) * NMO + (cc >> 5);
                    const double sgn = (cc & 3) == 0 ? 0.0 : ((cc & 3) == 1 ? 1.0 : -1.0);
                    const double cof = (cc & 3) == 0 ? 1.0 : sgn * Ts[at];
                    const double cofd = sgn * TDs[at];
                    acc += __hiloint2double((int)r.y, (int)r.x) *
                           (ratio_code_dot<NMO>(To, TDo, oc) * cof + ratio_code(To, oc, NMO, 0) * cofd);
                    if (r.w & 1u) {
                        sCD[spin * ts + ((r.w >> 2) & 7) * NMO + (r.w >> 5)] = acc;
                        acc = 0.0;
                    }
                }
            }
        }
        const double Sdot = walker_sum(Sd, S.LW);
        wave_sync();
        // adot: virtual orbitals, then the reference ones
        double ainv[KR], ainvd[KR], hk[KR];
#pragma unroll
        for (int k = 0; k < KR; ++k) {
            const double t = Tg[row[k] + sl], td = TDg[row[k] + sl];
            ainv[k] = (k < L.nsig && L.active) ? t : 0.0;
            ainvd[k] = (k < L.nsig && L.active) ? td : 0.0;
            hk[k] = 0.0;
        }
        const double Sinv = 1.0 / c.Ssum;
#pragma unroll
        for (int v = 0; v < NMO; v += 2) {
            double s0 = 0.0, s1 = 0.0;
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                const double2 cv = *(const double2 *)(Cg + row[k] + v), dv = *(const double2 *)(CDg + row[k] + v);
                s0 += ainvd[k] * cv.x + ainv[k] * dv.x;
                s1 += ainvd[k] * cv.y + ainv[k] * dv.y;
            }
            batch_end(s0, s1);
            adot[v] = v >= L.nsig ? (s0 - c.av[v] * Sdot) * Sinv : 0.0;
            adot[v + 1] = v + 1 >= L.nsig ? (s1 - c.av[v + 1] * Sdot) * Sinv : 0.0;
        }
#pragma unroll
        for (int v = 0; v < NMO; v += 2) {
            const double a0 = v >= L.nsig ? c.av[v] : 0.0, a1 = v + 1 >= L.nsig ? c.av[v + 1] : 0.0;
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                const double2 t = *(const double2 *)(Tg + row[k] + v), td = *(const double2 *)(TDg + row[k] + v);
                hk[k] += td.x * a0 + t.x * adot[v] + td.y * a1 + t.y * adot[v + 1];
            }
#pragma unroll
            for (int k = 0; k < KR; ++k) batch_end(hk[k]);
        }
#pragma unroll
        for (int k = 0; k < KR; ++k) adot[k] = k < L.nsig ? ainvd[k] - hk[k] : adot[k];
    };
    if (S.G <= 2) forward(std::integral_constant<int, 2>());
    else if (S.G == 4) forward(std::integral_constant<int, 4>());
    else forward(std::integral_constant<int, 8>());
    wave_sync();  // the walkers' tables become the wave's rows
    L = make_lane(S, wave_first, W, &w, lane_now());
    double *sAtom = smem + grad_wave<NMO>(S) + L.wloc * 6 * S.n_atoms;  // [n_atoms][6]: dlogpsi/dR, dE/dR
    for (int q = L.lw; q < 6 * S.n_atoms; q += S.LW) sAtom[q] = 0.0;
    const WalkerOut out(G, L, S.LW, w, sAtom);

    // ---- main gradient pass over the AOs ----------------------------------
    // Per shell the AO weights t (of a) and td (of adot) meet the monomials
    // first, in sums that every radial derivative and every exponent shares;
    // chi and beta = lap chi + 2 grad J . grad chi take the weights' ring rows
    // for the MO-coefficient products of each four AOs.
    double *sA = smem, *sAd = sA + NMO * kGradRow, *ringT = sAd + NMO * kGradRow, *ringD = ringT + kRing * kGradRow;
    AoWeights<NMO, kGradRow> wt(S, L.lane, sA, ringT, c.av), wd(S, L.lane, sAd, ringD, adot);
    // rows of idle lanes are zero in the products over a walker's electrons
    wave_sync();
#pragma unroll
    for (int m = 0; m < NMO; ++m) {
        sA[m * kGradRow + L.lane] = L.active ? c.av[m] : 0.0;
        sAd[m * kGradRow + L.lane] = L.active ? adot[m] : 0.0;
    }
    wave_sync();
    double gS[3] = {0.0, 0.0, 0.0};
    int col_of[NMO / 4];  // caller's columns of the MOs whose derivatives this lane writes, -1: padding
#pragma unroll
    for (int s = 0; s < NMO / 4; ++s) {
        const int m = 4 * s + (L.lane & 3);
        const int col = const_tab(S.mo_perm)[m < S.n_mo ? m : 0];
        col_of[s] = m < S.n_mo ? col : -1;
    }
    {
        int p = 0, mu = 0, done = 0, atom = -1;
        double lr[3] = {0.0, 0.0, 0.0}, er[3] = {0.0, 0.0, 0.0};
        AtomGeo<double> a;
        a.dx = a.dy = a.dz = a.r2 = 0.0;
        double r = 0.0, rinv = 0.0, gd = 0.0;
        auto put_atom = [&]() {
            if (atom < 0) return;
            out.add_atom(atom, lr, er);
            for (int k = 0; k < 3; ++k) lr[k] = er[k] = 0.0;
        };
        for (int sh = 0; sh < S.n_shells; ++sh) {
            const int4v si = shell_info(S, sh);
            const int nc = (si.y + 1) * (si.y + 2) / 2;
            if (si.x != atom) {  // shells of one atom share the geometry
                put_atom();
                atom = si.x;
                a.set(S, atom, x0, x1, x2);
                r = sqrt(a.r2);
                rinv = 1.0 / r;
                gd = gJ[0] * a.dx + gJ[1] * a.dy + gJ[2] * a.dz;
            }
            wt.need(mu + nc);
            wd.need(mu + nc);
            // sums over the components: t P, t grad P, t lap P, t (Hess P) grad J,
            // td P, td grad P
            double q = 0.0, qv[3] = {0.0, 0.0, 0.0}, qL = 0.0, qh[3] = {0.0, 0.0, 0.0};
            double qd = 0.0, qdv[3] = {0.0, 0.0, 0.0};
            if (si.y == 0) {
                q = wt(mu);
                qd = wd(mu);
            } else if (si.y == 1) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    qv[k] = wt(mu + k);
                    qdv[k] = wd(mu + k);
                }
                q = qv[0] * a.dx + qv[1] * a.dy + qv[2] * a.dz;
                qd = qdv[0] * a.dx + qdv[1] * a.dy + qdv[2] * a.dz;
            } else {
                // symmetric matrix of t: 2 t on the diagonal, t off it
                auto quad = [&](const AoWeights<NMO, kGradRow> &wx, double &s, double (&sv)[3], double &tr, double (&M)[6]) {
                    const double xx = wx(mu), xy = wx(mu + 1), xz = wx(mu + 2), yy = wx(mu + 3), yz = wx(mu + 4),
                                 zz = wx(mu + 5);
                    M[0] = 2.0 * xx, M[1] = xy, M[2] = xz, M[3] = 2.0 * yy, M[4] = yz, M[5] = 2.0 * zz;
                    sv[0] = M[0] * a.dx + M[1] * a.dy + M[2] * a.dz;
                    sv[1] = M[1] * a.dx + M[3] * a.dy + M[4] * a.dz;
                    sv[2] = M[2] * a.dx + M[4] * a.dy + M[5] * a.dz;
                    s = 0.5 * (sv[0] * a.dx + sv[1] * a.dy + sv[2] * a.dz);
                    tr = M[0] + M[3] + M[5];
                };
                double M[6], Md[6], trd;
                quad(wt, q, qv, qL, M);
                quad(wd, qd, qdv, trd, Md);
                qh[0] = M[0] * gJ[0] + M[1] * gJ[1] + M[2] * gJ[2];
                qh[1] = M[1] * gJ[0] + M[3] * gJ[1] + M[4] * gJ[2];
                qh[2] = M[2] * gJ[0] + M[4] * gJ[1] + M[5] * gJ[2];
            }
            const double qg = qv[0] * gJ[0] + qv[1] * gJ[1] + qv[2] * gJ[2];
            // one pass over the primitives: radial sums and exponent derivatives
            const ExpoSums z = {q, qd + qL + 2.0 * qg, 2.0 * gd * q};
            const double rk = S.basis == 0 ? power(r, si.z) : 1.0;
            Radial R = {0.0, 0.0, 0.0, 0.0, 0.0};
            for (int i = 0; i < si.w; ++i) {
                double gl, ge;
                radial_prim(S, prim_info(S, p + i), const_tab(S.prim_qn)[p + i], si.y, si.z, r, a.r2, rinv, rk, z, R,
                            gl, ge);
                out.put(p + i, gl, ge);
            }
            p += si.w;
            {
                const double d[3] = {a.dx, a.dy, a.dz};
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    // sums of t grad chi, td grad chi, t (Hess chi) grad J, t grad lap chi
                    const double tg = R.v * qv[k] + R.d * q * d[k], tdg = R.v * qdv[k] + R.d * qd * d[k];
                    const double th = R.v * qh[k] + R.d * (gd * qv[k] + d[k] * qg + q * gJ[k]) + R.dd * q * gd * d[k];
                    const double t3 = (R.d * qL + R.l1 * q) * d[k] + R.l * qv[k];
                    gS[k] += tg;
                    lr[k] -= tg;
                    er[k] += 0.5 * tdg + th + 0.5 * t3;
                }
            }
            // chi and beta into the ring rows whose weights are spent
            const double Xr = R.l + 2.0 * R.d * gd;
            shell_monomials(si.y, a.dx, a.dy, a.dz, [&](int cc, double P, double Px, double Py, double Pz, double PL) {
                const int at = ((mu + cc) & (kRing - 1)) * kGradRow + L.lane;
                const double chi = P * R.v;
                const double be = P * Xr + R.v * (PL + 2.0 * (gJ[0] * Px + gJ[1] * Py + gJ[2] * Pz));
                ringT[at] = L.active ? chi : 0.0;
                ringD[at] = L.active ? be : 0.0;
            });
            mu += nc;
            for (; mu - done >= 4; done += 4)
                put_mo_gradient<NMO>(S, L.lane, wave_first, W, done, ringT, ringD, sA, sAd, col_of, G);
        }
        put_atom();
        if (done < mu) {
            for (int z = mu; z & 3; ++z) {
                ringT[(z & (kRing - 1)) * kGradRow + L.lane] = 0.0;
                ringD[(z & (kRing - 1)) * kGradRow + L.lane] = 0.0;
            }
            put_mo_gradient<NMO>(S, L.lane, wave_first, W, done, ringT, ringD, sA, sAd, col_of, G);
        }
    }
    // e-n attraction
    for (int a = 0; a < S.n_atoms; ++a) {
        double er[3];
        const auto *A = const_tab(S.atoms) + 4 * a;
        const double d[3] = {x0 - A[0], x1 - A[1], x2 - A[2]};
        const double rr = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
        const double f = -A[3] / (rr * rr * rr);
        for (int k = 0; k < 3; ++k) er[k] = f * d[k];
        const double none[3] = {0.0, 0.0, 0.0};
        out.add_atom(a, none, er);
    }

    // ---- Jastrow parameters and the Jastrow part of the nuclear gradients ---
    wave_sync();  // the rings and rows are no longer read
    {
        L = make_lane(S, wave_first, W, &w, lane_now());
        double *sP = smem + L.wloc * grad_walker<NMO>(S);   // [LW][3]
        double *sF = sP + 3 * S.LW;                         // [LW][n_atoms][2 een_n]
        double *sG = sF + S.LW * S.n_atoms * 2 * S.een_n;   // [LW][n_atoms][kEenGeo]
        sP[3 * L.lw + 0] = x0;
        sP[3 * L.lw + 1] = x1;
        sP[3 * L.lw + 2] = x2;
        een_table_fill<true>(S, L, x0, x1, x2, sF, sG);
        wave_sync();
        const double h[3] = {gJ[0] + gS[0], gJ[1] + gS[1], gJ[2] + gS[2]};
        jastrow_derivs(S, L, x0, x1, x2, h, sP, sF, sG, G, out);
    }
    wave_sync();  // the nuclear sums of both halves of a walker's lanes
    if (L.wvalid && L.lw == 0) {
        // nuclear gradients, with the n-n repulsion
        for (int a = 0; a < S.n_atoms; ++a) {
            const double *A = S.atoms + 4 * a;
            double nn[3] = {0.0, 0.0, 0.0};
            for (int b2 = 0; b2 < S.n_atoms; ++b2) {
                if (b2 == a) continue;
                const double *B = S.atoms + 4 * b2;
                const double d[3] = {A[0] - B[0], A[1] - B[1], A[2] - B[2]};
                const double rr = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
                for (int k = 0; k < 3; ++k) nn[k] -= A[3] * B[3] * d[k] / (rr * rr * rr);
            }
            for (int k = 0; k < 3; ++k) {
                if (G.dlogpsi_dR) G.dlogpsi_dR[(w * S.n_atoms + a) * 3 + k] = sAtom[6 * a + k];
                if (G.deloc_dR) G.deloc_dR[(w * S.n_atoms + a) * 3 + k] = sAtom[6 * a + 3 + k] + nn[k];
            }
        }
    }
}

}  // namespace

template <int NMO>
static hipError_t launch_grad_t(const DevSystem &S, const double *X, int64_t W, const GradOut &G, bool mixed,
                                hipStream_t st) {
    const int64_t blocks = (W + S.WPW - 1) / S.WPW;
    const size_t lds = grad_lds<NMO>(S) * sizeof(double);
    if (mixed)
        hipLaunchKernelGGL((k_grad<NMO, float>), dim3((unsigned)blocks), dim3(kWave), lds, st, S, X, W, G);
    else
        hipLaunchKernelGGL((k_grad<NMO, double>), dim3((unsigned)blocks), dim3(kWave), lds, st, S, X, W, G);
    return hipGetLastError();
}

// LDS by which a system is admitted: what the kernel takes, and at least a row
// of chi, beta, a and adot per electron and the two-component e-e-n tables.
// The kernel no longer holds these; they stay in the limit so that the systems
// a caller sees refused do not depend on the kernel's layout.
size_t grad_lds_bytes(const DevSystem &S) {
    const size_t rows = (size_t)S.LW * 2 * (S.n_ao + S.nmo_pad);
    const size_t een = (size_t)S.LW * (3 + 2 * S.n_atoms * (2 * S.een_n + kEenGeo));
    const size_t admit = S.WPW * ((rows > een ? rows : een) + 6 * S.n_atoms);
    size_t all = 0;
    switch (S.nmo_pad) {
#define QMC_LDS(N) \
    case N: all = grad_lds<N>(S); break;
        QMC_LDS(4) QMC_LDS(8) QMC_LDS(12) QMC_LDS(16) QMC_LDS(20) QMC_LDS(24) QMC_LDS(32)
#undef QMC_LDS
    }
    return (all > admit ? all : admit) * sizeof(double);
}

hipError_t launch_grad(const DevSystem &S, const double *X, int64_t W, double *dlogpsi,
                       double *deloc_dth, double *dlogpsi_dR, double *deloc_dR, int n_param, bool mixed,
                       hipStream_t st) {
    GradOut G{dlogpsi, deloc_dth, dlogpsi_dR, deloc_dR, n_param};
    switch (S.nmo_pad) {
        case 4: return launch_grad_t<4>(S, X, W, G, mixed, st);
        case 8: return launch_grad_t<8>(S, X, W, G, mixed, st);
        case 12: return launch_grad_t<12>(S, X, W, G, mixed, st);
        case 16: return launch_grad_t<16>(S, X, W, G, mixed, st);
        case 20: return launch_grad_t<20>(S, X, W, G, mixed, st);
        case 24: return launch_grad_t<24>(S, X, W, G, mixed, st);
        case 32: return launch_grad_t<32>(S, X, W, G, mixed, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace qmc
