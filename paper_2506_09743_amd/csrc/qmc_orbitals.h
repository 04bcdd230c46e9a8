// Orbital stages of the walker evaluation: MO values of every electron
// (pass 1) and the contraction of the AO derivatives with the adjoint vector
// (pass 2).  Included by qmc_walker.h.
//
// Both contract the wave's 64 electrons (one per lane) with the same small
// AO x MO matrix C.  The matrix cores take it: every coefficient is loaded
// once per wave into a lane register as the A operand of 4 x 4 products,
// instead of once per multiply-add through the scalar cache, whose reads (a
// row per AO, two waves of them per electron) the wave waited for.
//   FP64  v_mfma_f64_4x4x4_4b: lane 16 k + 4 b + i gives A[i][k] (the same
//         for every block b) and B[k][4 b + j], and gets D[k -> row][4 b + j];
//         one instruction is 4 rows x 16 electrons x 4 terms.  It runs at the
//         vector unit's FP64 rate (19 cycles against 17 for the same 256
//         multiply-adds) and is bit for bit the chain of fused multiply-adds
//         in ascending k.
//   FP32  v_mfma_f32_4x4x1_16b: lane 4 b + j gives B[j] = its own electron's
//         value and gets its own electron's 4 rows; one fused multiply-add
//         per element, bit for bit fmaf (11 cycles against 19).
// Measured for CO (28 AOs x 20 MOs, 45 primitives; cycles of one wave with
// about one wave per SIMD): pass 1 44 k -> 19 k, pass 2 42 k -> 20 k; a
// 65 536-walker step 280 -> 234 us together with the elimination and adjoint
// stages' batched LDS reads.  What bounds them now is FP64 vector work, the
// exponentials first.
// The 64 electrons sit in four groups of 16 lanes; operands and results of
// the FP64 products change between "electron per lane" and "row k per lane
// group" through rows of 64 doubles in LDS, a row per AO or MO.
#pragma once

namespace qmc {
namespace walker {

// LDS rows of 64 doubles that the FP64 stages need: a ring of kRing rows for
// AO values or weights (at most 3 + 6 rows are pending at a time), and one
// row per MO while the lanes exchange MO values or adjoint vectors.
constexpr int kRing = 16;

template <int NMO>
constexpr size_t orbital_lds_bytes() {
    return (size_t)(NMO > kRing ? NMO : kRing) * kWave * sizeof(double);
}

// Up to this many MOs (H2-sized systems) the vector unit contracts directly:
// a row is one scalar load of 32 bytes and 4 multiply-adds, less than the
// exchange through LDS costs a lone wave (1024 H2 walkers, 200 steps: 1.30 ms
// so, 1.41 ms through the matrix cores).
constexpr int kFewMO = 4;

// Displacement from the current atom, in the arithmetic of the AO values
// (formed in FP64).
template <typename RT>
struct AtomGeo {
    RT dx, dy, dz, r2;
    __device__ __forceinline__ void set(const DevSystem &S, int a, double x0, double x1, double x2) {
        const auto *A = const_tab(S.atoms) + 4 * a;
        dx = RT(x0 - A[0]);
        dy = RT(x1 - A[1]);
        dz = RT(x2 - A[2]);
        r2 = dx * dx + dy * dy + dz * dz;
    }
};

// Contraction of AO rows with C, one value per electron and AO, in AO order:
// out_m = sum_mu C[mu][m] row_mu.  Rows enter an LDS ring as they are made
// and leave it four at a time; the C rows of the next four are already in
// registers.  Every lane of the wave must use it alike; buf:
// orbital_lds_bytes<NMO>() of LDS.
template <int NMO>
struct MoRows {
    static constexpr int MB = NMO / 4;
    double *buf;
    const __attribute__((address_space(4))) double *Ap;
    int lane, mu, done;  // rows written, rows contracted
    double A[MB], acc[MB][4];

    __device__ __forceinline__ MoRows(const DevSystem &S, int lane_, double *buf_)
        : buf(buf_), lane(lane_), mu(0), done(0) {
        Ap = const_tab(S.mo_a) + ((lane >> 4) * 4 + (lane & 3)) * MB;
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            A[m] = Ap[m];
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[m][t] = 0.0;
        }
    }
    __device__ __forceinline__ void push(double v) {
        buf[(mu & (kRing - 1)) * kWave + lane] = v;
        ++mu;
    }
    __device__ __forceinline__ void contract() {
        const int g = lane >> 4, j = lane & 15;
        wave_sync();
        double B[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) B[t] = buf[((done + g) & (kRing - 1)) * kWave + 16 * t + j];
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[m][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(A[m], B[t], acc[m][t], 0, 0, 0);
        done += 4;
        Ap += 4 * NMO;
#pragma unroll
        for (int m = 0; m < MB; ++m) A[m] = Ap[m];
    }
    // at the end of each shell, of nc rows
    __device__ __forceinline__ void flush(int) {
        while (mu - done >= 4) contract();
    }
    __device__ __forceinline__ void finish(double (&out)[NMO]) {
        const int g = lane >> 4, j = lane & 15;
        while (mu & 3) push(0.0);  // the table's rows are zero there
        if (done < mu) contract();
        wave_sync();
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int t = 0; t < 4; ++t) buf[(4 * m + g) * kWave + 16 * t + j] = acc[m][t];
        wave_sync();
#pragma unroll
        for (int m = 0; m < NMO; ++m) out[m] = buf[m * kWave + lane];
        wave_sync();
    }
};

// The same on the vector unit (kFewMO).  The shell's first row of C moves once
// per shell, by flush, and not by the pushes: a pointer that the branches over s,
// p and d shells advance by different amounts was compiled without its step in the
// d branch, and the next shell read C at a stale address (qmc_grad faulted for
// any system of at most 4 MOs with a shell behind a d shell).
template <>
struct MoRows<kFewMO> {
    const __attribute__((address_space(4))) double *row;
    int c;  // component within the shell
    double acc[kFewMO];

    __device__ __forceinline__ MoRows(const DevSystem &S, int, double *) : row(const_tab(S.mo)), c(0) {
#pragma unroll
        for (int m = 0; m < kFewMO; ++m) acc[m] = 0.0;
    }
    __device__ __forceinline__ void push(double v) {
#pragma unroll
        for (int m = 0; m < kFewMO; ++m) acc[m] += v * row[c * kFewMO + m];
        ++c;
    }
    __device__ __forceinline__ void flush(int nc) {
        row += nc * kFewMO;
        c = 0;
    }
    __device__ __forceinline__ void finish(double (&out)[kFewMO]) {
#pragma unroll
        for (int m = 0; m < kFewMO; ++m) out[m] = acc[m];
    }
};

// Pass 1 in FP64: phi_m(r_e) = sum_mu C[mu][m] chi_mu(r_e) of the lane's
// electron.  Every lane of the wave must call it.
template <int NMO, bool VK>
__device__ __forceinline__ void mo_values_f64(const DevSystem &S, int lane, double *buf, double x0, double x1,
                                              double x2, double (&phi)[NMO]) {
    MoRows<NMO> rows(S, lane, buf);
    int p = 0, atom = -1;
    AtomGeo<double> a;
    double r = 0.0;
    for (int sh = 0; sh < S.n_shells; ++sh) {
        const int4v si = shell_info(S, sh);
        if (si.x != atom) {  // shells of one atom share the geometry
            atom = si.x;
            a.set(S, atom, x0, x1, x2);
            if (S.basis == 0) r = sqrt(a.r2);
        }
        double R, Rd, Rl;
        shell_radial<double, false, VK>(S, p, si.w, si.y, si.z, r, a.r2, 0.0, R, Rd, Rl);
        p += si.w;
        if (si.y == 0) {
            rows.push(R);
        } else if (si.y == 1) {
            rows.push(a.dx * R);
            rows.push(a.dy * R);
            rows.push(a.dz * R);
        } else {  // xx, xy, xz, yy, yz, zz
            rows.push(a.dx * a.dx * R);
            rows.push(a.dx * a.dy * R);
            rows.push(a.dx * a.dz * R);
            rows.push(a.dy * a.dy * R);
            rows.push(a.dy * a.dz * R);
            rows.push(a.dz * a.dz * R);
        }
        rows.flush((si.y + 1) * (si.y + 2) / 2);
    }
    rows.finish(phi);
}

// MO values and the direction B[e][m] = sum_mu C[mu][m] (lap chi + 2 grad J .
// grad chi) of the adjoint in one pass over the shells (gJ: grad_e J).  The
// values round as mo_values_f64's.  buf: twice orbital_lds_bytes<NMO>().
template <int NMO>
__device__ __forceinline__ void mo_values_direction(const DevSystem &S, int lane, double *buf, double x0, double x1,
                                                    double x2, const double (&gJ)[3], double (&phi)[NMO],
                                                    double (&bvec)[NMO]) {
    MoRows<NMO> chi(S, lane, buf), beta(S, lane, buf + (NMO > kRing ? NMO : kRing) * kWave);
    int p = 0, atom = -1;
    AtomGeo<double> a;
    double r = 0.0, rinv = 0.0, gd = 0.0;
    for (int sh = 0; sh < S.n_shells; ++sh) {
        const int4v si = shell_info(S, sh);
        if (si.x != atom) {
            atom = si.x;
            a.set(S, atom, x0, x1, x2);
            if (S.basis == 0) {
                r = sqrt(a.r2);
                rinv = 1.0 / r;
            }
            gd = gJ[0] * a.dx + gJ[1] * a.dy + gJ[2] * a.dz;
        }
        // R as a chain of fused multiply-adds (as without derivatives), R'/r and
        // R'' + (2l+2) R'/r
        double R = 0.0, Rd = 0.0, Rl = 0.0;
        if (S.basis == 0) {
            double rk = 1.0;
            for (int t = 0; t < si.z; ++t) rk *= r;
            const double kr = si.z * rinv, l2 = (2.0 * si.y + 2.0) * rinv;
            for (int q = 0; q < si.w; ++q) {
                const double2v pe = prim_info(S, p + q);
                const double e = exp_f64(-pe.x * r), cr = pe.y * rk, f = cr * e, g = kr - pe.x;
                R = __builtin_fma(cr, e, R);
                Rd += f * g * rinv;
                Rl += f * (g * g - kr * rinv + l2 * g);
            }
        } else {
            const double fl = 4.0 * si.y + 6.0;
            auto add = [&](double2v pe, double e) {
                const double f = pe.y * e, u = pe.x * f;
                R = __builtin_fma(pe.y, e, R);
                Rd -= 2.0 * u;
                Rl += u * (4.0 * pe.x * a.r2 - fl);
            };
            int q = 0;
            for (; q + 1 < si.w; q += 2) {
                const double2v pa = prim_info(S, p + q), pb = prim_info(S, p + q + 1);
                const double ea = exp_f64(-pa.x * a.r2), eb = exp_f64(-pb.x * a.r2);
                add(pa, ea);
                add(pb, eb);
            }
            if (q < si.w) {
                const double2v pa = prim_info(S, p + q);
                add(pa, exp_f64(-pa.x * a.r2));
            }
        }
        p += si.w;
        const double X = Rl + 2.0 * Rd * gd, R2 = 2.0 * R;
        if (si.y == 0) {
            chi.push(R);
            beta.push(X);
        } else if (si.y == 1) {
            chi.push(a.dx * R);
            chi.push(a.dy * R);
            chi.push(a.dz * R);
            beta.push(a.dx * X + R2 * gJ[0]);
            beta.push(a.dy * X + R2 * gJ[1]);
            beta.push(a.dz * X + R2 * gJ[2]);
        } else {  // xx, xy, xz, yy, yz, zz
            chi.push(a.dx * a.dx * R);
            chi.push(a.dx * a.dy * R);
            chi.push(a.dx * a.dz * R);
            chi.push(a.dy * a.dy * R);
            chi.push(a.dy * a.dz * R);
            chi.push(a.dz * a.dz * R);
            beta.push(a.dx * a.dx * X + R2 * (1.0 + 2.0 * a.dx * gJ[0]));
            beta.push(a.dx * a.dy * X + R2 * (a.dy * gJ[0] + a.dx * gJ[1]));
            beta.push(a.dx * a.dz * X + R2 * (a.dz * gJ[0] + a.dx * gJ[2]));
            beta.push(a.dy * a.dy * X + R2 * (1.0 + 2.0 * a.dy * gJ[1]));
            beta.push(a.dy * a.dz * X + R2 * (a.dz * gJ[1] + a.dy * gJ[2]));
            beta.push(a.dz * a.dz * X + R2 * (1.0 + 2.0 * a.dz * gJ[2]));
        }
        const int nc = (si.y + 1) * (si.y + 2) / 2;
        chi.flush(nc);
        beta.flush(nc);
    }
    chi.finish(phi);
    beta.finish(bvec);
}

// Pass 1 of the mixed FP32 form: AO values in FP32, one fused multiply-add
// per AO and MO in AO order.  Every lane of the wave must call it.
template <int NMO>
__device__ __forceinline__ void mo_values_f32(const DevSystem &S, int lane, double x0, double x1, double x2,
                                              float (&phi)[NMO]) {
    constexpr int MB = NMO / 4;
    const auto *Ap = const_tab(S.mo_fa) + (lane & 3) * MB;
    floatx4_t acc[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[m] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    int p = 0, atom = -1;
    AtomGeo<float> a;
    float r = 0.f;
    auto rows = [&](auto nc, auto value, int np, int l, int kn) {
        constexpr int NC = decltype(nc)::value;
        float A[NC][MB];  // in flight while the radial part is evaluated
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int m = 0; m < MB; ++m) A[c][m] = Ap[c * NMO + m];
        Ap += NC * NMO;
        float R, Rd, Rl;
        shell_radial<float, false>(S, p, np, l, kn, r, a.r2, 0.f, R, Rd, Rl);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const float v = value(c, R);
#pragma unroll
            for (int m = 0; m < MB; ++m) acc[m] = __builtin_amdgcn_mfma_f32_4x4x1f32(A[c][m], v, acc[m], 0, 0, 0);
        }
    };
    for (int sh = 0; sh < S.n_shells; ++sh) {
        const int4v si = shell_info(S, sh);
        if (si.x != atom) {
            atom = si.x;
            a.set(S, atom, x0, x1, x2);
            r = sqrt(a.r2);
        }
        if (si.y == 0) {
            rows(std::integral_constant<int, 1>(), [&](int, float R) { return R; }, si.w, si.y, si.z);
        } else if (si.y == 1) {
            rows(std::integral_constant<int, 3>(),
                 [&](int c, float R) { return (c == 0 ? a.dx : (c == 1 ? a.dy : a.dz)) * R; }, si.w, si.y, si.z);
        } else {  // xx, xy, xz, yy, yz, zz
            rows(std::integral_constant<int, 6>(),
                 [&](int c, float R) {
                     const float u = (c < 3) ? a.dx : (c < 5 ? a.dy : a.dz);
                     const float v = (c == 0) ? a.dx : (c == 1 || c == 3) ? a.dy : a.dz;
                     return (u * v) * R;
                 },
                 si.w, si.y, si.z);
        }
        p += si.w;
    }
#pragma unroll
    for (int m = 0; m < NMO; ++m) phi[m] = acc[m / 4][m % 4];
}

// AO weights t_mu = sum_m C[mu][m] a_e[m] of the lane's electron, four rows
// at a time into a ring of LDS rows; the C rows of the next four are already
// in registers.
template <int NMO, int ROW = kWave>
struct AoWeights {
    static constexpr int MB = NMO / 4;
    double *buf;
    const __attribute__((address_space(4))) double *Ap;
    int lane, avail;
    double A[MB], B[MB][4];

    // xbuf: [NMO][64] for the exchange of av, free afterwards; ring: [kRing][ROW]
    // (may overlap xbuf)
    __device__ __forceinline__ AoWeights(const DevSystem &S, int lane_, double *xbuf, double *ring,
                                         const double (&av)[NMO])
        : buf(ring), lane(lane_), avail(0) {
        const int g = lane >> 4, j = lane & 15;
        Ap = const_tab(S.mo_a) + ((lane & 3) * 4 + g) * MB;
#pragma unroll
        for (int s = 0; s < MB; ++s) A[s] = Ap[s];
        wave_sync();
#pragma unroll
        for (int m = 0; m < NMO; ++m) xbuf[m * kWave + lane] = av[m];
        wave_sync();
#pragma unroll
        for (int s = 0; s < MB; ++s)
#pragma unroll
            for (int t = 0; t < 4; ++t) B[s][t] = xbuf[(4 * s + g) * kWave + 16 * t + j];
        wave_sync();
    }
    // rows up to `end` (at most kRing - 3 past the oldest still wanted)
    __device__ __forceinline__ void need(int end) {
        while (avail < end) {
            const int g = lane >> 4, j = lane & 15;
            double d[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < MB; ++s)
#pragma unroll
                for (int t = 0; t < 4; ++t) d[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(A[s], B[s][t], d[t], 0, 0, 0);
            Ap += 4 * NMO;
#pragma unroll
            for (int s = 0; s < MB; ++s) A[s] = Ap[s];
#pragma unroll
            for (int t = 0; t < 4; ++t) buf[((avail + g) & (kRing - 1)) * ROW + 16 * t + j] = d[t];
            avail += 4;
        }
        wave_sync();
    }
    __device__ __forceinline__ double operator()(int mu) const { return buf[(mu & (kRing - 1)) * ROW + lane]; }
};

template <int ROW>
struct AoWeights<kFewMO, ROW> {
    const __attribute__((address_space(4))) double *C;
    const double (&av)[kFewMO];
    __device__ __forceinline__ AoWeights(const DevSystem &S, int, double *, double *, const double (&av_)[kFewMO])
        : C(const_tab(S.mo)), av(av_) {}
    __device__ __forceinline__ void need(int) {}
    __device__ __forceinline__ double operator()(int mu) const {
        double t = 0.0;
#pragma unroll
        for (int m = 0; m < kFewMO; ++m) t += C[mu * kFewMO + m] * av[m];
        return t;
    }
};

// Pass 2: grad_e Sigma / Sigma and lap_e Sigma / Sigma.  With a_e[m] =
// d log Sigma / d phi_m(r_e) and t_mu = sum_m C[mu][m] a_e[m], both are
// sum_mu t_mu (grad, lap) chi_mu(r_e); for chi = P R:
//   grad chi = R grad P + P (R'/r) d,   lap chi = R lap P + P (R'' + (2l+2) R'/r).
// This contraction is the Jacobi trace: the weights t and the products
// t (grad, lap) chi are FP64 in every form; RT is the arithmetic of the AO
// derivative factors (FP32 in the mixed forms).  In FP64 the components of a
// shell are summed first: with q = sum_c t_c P_c, the shell adds (R'/r) q d +
// R sum_c t_c grad P_c and (R'' + (2l+2) R'/r) q + R sum_c t_c lap P_c, and
// the factors of d meet once per atom.  Every lane of the wave must call it;
// buf: orbital_lds_bytes<NMO>() of LDS.
template <int NMO, typename RT, bool VK>
__device__ __forceinline__ void sigma_derivs(const DevSystem &S, int lane, double *buf, double x0, double x1,
                                             double x2, const double (&av)[NMO], double &g0, double &g1, double &g2,
                                             double &lap) {
    AoWeights<NMO> w(S, lane, buf, buf, av);
    int p = 0, mu = 0, atom = -1;
    double G0 = 0.0, G1 = 0.0, G2 = 0.0, L = 0.0, gd = 0.0;
    AtomGeo<RT> a;
    a.dx = a.dy = a.dz = a.r2 = RT(0);
    RT r = RT(0), rinv = RT(0);
    for (int sh = 0; sh < S.n_shells; ++sh) {
        const int4v si = shell_info(S, sh);
        if (si.x != atom) {  // shells of one atom share the geometry
            if constexpr (sizeof(RT) == sizeof(double)) {
                G0 += gd * a.dx;
                G1 += gd * a.dy;
                G2 += gd * a.dz;
                gd = 0.0;
            }
            atom = si.x;
            a.set(S, atom, x0, x1, x2);
            if (sizeof(RT) != sizeof(double) || S.basis == 0) {
                r = sqrt(a.r2);
                rinv = RT(1) / r;
            }
        }
        RT Rv, Rd, Rl;
        shell_radial<RT, true, VK>(S, p, si.w, si.y, si.z, r, a.r2, rinv, Rv, Rd, Rl);
        p += si.w;
        const int nc = (si.y + 1) * (si.y + 2) / 2;
        w.need(mu + nc);
        if constexpr (sizeof(RT) == sizeof(double)) {
            double q;
            if (si.y == 0) {
                q = w(mu);
            } else if (si.y == 1) {
                const double t0 = w(mu), t1 = w(mu + 1), t2 = w(mu + 2);
                q = t0 * a.dx + t1 * a.dy + t2 * a.dz;
                G0 += Rv * t0;
                G1 += Rv * t1;
                G2 += Rv * t2;
            } else {
                const double xx = w(mu), xy = w(mu + 1), xz = w(mu + 2), yy = w(mu + 3), yz = w(mu + 4),
                             zz = w(mu + 5);
                const double u0 = 2.0 * xx * a.dx + xy * a.dy + xz * a.dz;
                const double u1 = xy * a.dx + 2.0 * yy * a.dy + yz * a.dz;
                const double u2 = xz * a.dx + yz * a.dy + 2.0 * zz * a.dz;
                q = 0.5 * (u0 * a.dx + u1 * a.dy + u2 * a.dz);
                G0 += Rv * u0;
                G1 += Rv * u1;
                G2 += Rv * u2;
                L += 2.0 * Rv * (xx + yy + zz);
            }
            gd += Rd * q;
            L += Rl * q;
        } else {
            for (int c = 0; c < nc; ++c) {
                const double t = w(mu + c);
                // monomial, its gradient and Laplacian
                RT P, Px, Py, Pz, PL;
                if (si.y == 0) {
                    P = RT(1); Px = Py = Pz = PL = RT(0);
                } else if (si.y == 1) {
                    P = c == 0 ? a.dx : (c == 1 ? a.dy : a.dz);
                    Px = c == 0 ? RT(1) : RT(0);
                    Py = c == 1 ? RT(1) : RT(0);
                    Pz = c == 2 ? RT(1) : RT(0);
                    PL = RT(0);
                } else {
                    // xx, xy, xz, yy, yz, zz
                    const int iu = (c < 3) ? 0 : (c < 5 ? 1 : 2);
                    const int iv = (c == 0) ? 0 : (c == 1 || c == 3) ? 1 : 2;
                    const RT u = iu == 0 ? a.dx : (iu == 1 ? a.dy : a.dz);
                    const RT v = iv == 0 ? a.dx : (iv == 1 ? a.dy : a.dz);
                    P = u * v;
                    Px = (iu == 0 ? v : RT(0)) + (iv == 0 ? u : RT(0));
                    Py = (iu == 1 ? v : RT(0)) + (iv == 1 ? u : RT(0));
                    Pz = (iu == 2 ? v : RT(0)) + (iv == 2 ? u : RT(0));
                    PL = iu == iv ? RT(2) : RT(0);
                }
                const RT PRd = P * Rd;
                G0 += t * double(Rv * Px + PRd * a.dx);
                G1 += t * double(Rv * Py + PRd * a.dy);
                G2 += t * double(Rv * Pz + PRd * a.dz);
                L += t * double(Rv * PL + P * Rl);
            }
        }
        mu += nc;
    }
    if constexpr (sizeof(RT) == sizeof(double)) {
        G0 += gd * a.dx;
        G1 += gd * a.dy;
        G2 += gd * a.dz;
    }
    g0 = G0;
    g1 = G1;
    g2 = G2;
    lap = L;
    wave_sync();
}

}  // namespace walker
}  // namespace qmc
