// Device-side building blocks of the walker evaluation, shared by the
// evaluation / Metropolis kernels and the gradient kernel of libqmc.
//
// Work decomposition.  One wave of 64 lanes holds 64 / (2G) walkers; each
// walker owns 2G consecutive lanes, G per spin, and lane i of a spin group
// owns electron i of that spin.  A lane evaluates its electron's atomic
// orbitals and molecular orbitals in registers, the Slater matrices are
// factorised across the lanes of a group (row = electron), and the walker's
// scalars are reduced across its lanes with cross-lane shuffles.  Walkers
// never interact, so a walker's results do not depend on its neighbours.
//
// Kinetic energy (appendix on local energies).  With Psi = exp(J) Sigma the
// Laplacian splits into lap J + |grad J|^2 + 2 grad J . grad Sigma / Sigma +
// lap Sigma / Sigma.  Because every determinant is linear in the row of one
// electron, grad_e Sigma / Sigma = sum_m a_e[m] grad phi_m(r_e) and
// lap_e Sigma / Sigma = sum_m a_e[m] lap phi_m(r_e) with a_e[m] =
// d log Sigma / d phi_m(r_e) (this is the per-electron Jacobi trace of
// eq. claudia_trace summed over the CI expansion).  a_e follows from the
// low-rank excited-determinant algebra of eq. table: with T = A0^-1 Phi,
// every excited determinant is D0 det T[H,P] (k <= 2), Sigma = D0 S with
// S = sum_n d_n det T_up[H,P] det T_dn[H,P], and the CI-weighted cofactors
// C = dS/dT give a_e[v] = (A0^-T C)[e,v] / S on virtual orbitals and
// a_e[k] = A0^-1[k,e] - (A0^-T C T^T)[e,k] / S on reference orbitals.
// Only A0 is ever inverted, as in the paper's accelerated scheme.
#pragma once

#include "qmc_device.h"
#include "qmc_exp.h"

#include <math.h>

#include <type_traits>

namespace qmc {
namespace walker {

// Determinant and cofactor records fetched per batch.
constexpr int kRecBatch = 4;

// The system tables never change while a kernel runs: read through the
// constant address space, a load whose address is the same on every lane
// becomes a scalar load, and no load is held back by the LDS exchanges
// between it and its use.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *const_tab(const T *p) {
    return (const __attribute__((address_space(4))) T *)p;
}
typedef double double2v __attribute__((ext_vector_type(2)));
typedef int int4v __attribute__((ext_vector_type(4)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int4v shell_info(const DevSystem &S, int sh) {  // atom, l, kn, nprim
    return const_tab((const int4v *)S.shells)[sh];
}
__device__ __forceinline__ double2v prim_info(const DevSystem &S, int p) {  // exponent, coefficient
    return const_tab((const double2v *)S.prims)[p];
}

// Orders a wave's LDS accesses across its lanes: the work-group is one wave,
// whose LDS instructions execute in order, so only the compiler has to keep
// them so.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Cross-lane exchange within a row of 16 lanes by DPP moves (no LDS round
// trip).  Walkers (LW <= 16 lanes) and spin groups (G <= 8 lanes) are
// aligned to their power-of-two size, so these steps never leave them:
// kSwap1 pairs lane ^ 1 and kSwap2 lane ^ 2 (quad permutes), kHalfMirror
// pairs lane i with 7 - i in each 8-lane half (the other quad), kMirror
// pairs lane i with 15 - i (the other half).  Applied in this order a
// reduction pairs the same partial results as an xor butterfly, and every
// lane of the span ends with the same value.  Callers run them with all
// lanes of the wave active.
constexpr int kSwap1 = 0xB1, kSwap2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;

template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    return __hiloint2double(dpp_i<CTRL>(__double2hiint(v)), dpp_i<CTRL>(__double2loint(v)));
}

// Sum over an aligned span of n = 1, 2, 4, 8 or 16 lanes.
__device__ __forceinline__ double span_sum(double v, int n) {
    if (n > 1) v += dpp_d<kSwap1>(v);
    if (n > 2) v += dpp_d<kSwap2>(v);
    if (n > 4) v += dpp_d<kHalfMirror>(v);
    if (n > 8) v += dpp_d<kMirror>(v);
    return v;
}

// Two sums over an aligned span of n = 2, 4, 8 or 16 lanes for little more than
// one: the span's halves exchange first, so that the lower half ends with the
// sum of a and the upper half (`upper`) with that of b.
__device__ __forceinline__ double span_sum_pair(double a, double b, int n, bool upper) {
    double v = upper ? b : a;
    const double o = upper ? a : b;
    if (n > 8) {
        v += dpp_d<kMirror>(o);
        v += dpp_d<kHalfMirror>(v);
    } else if (n > 4) {
        v += dpp_d<kHalfMirror>(o);
    } else if (n > 2) {
        v += dpp_d<kSwap2>(o);
    } else {
        v += dpp_d<kSwap1>(o);
    }
    if (n > 4) v += dpp_d<kSwap2>(v);
    if (n > 2) v += dpp_d<kSwap1>(v);
    return v;
}

__device__ __forceinline__ int span_sum_i(int v, int n) {
    if (n > 1) v += dpp_i<kSwap1>(v);
    if (n > 2) v += dpp_i<kSwap2>(v);
    if (n > 4) v += dpp_i<kHalfMirror>(v);
    if (n > 8) v += dpp_i<kMirror>(v);
    return v;
}

__device__ __forceinline__ uint32_t span_max_u(uint32_t v, int n) {
    if (n > 1) v = max(v, (uint32_t)dpp_i<kSwap1>((int)v));
    if (n > 2) v = max(v, (uint32_t)dpp_i<kSwap2>((int)v));
    if (n > 4) v = max(v, (uint32_t)dpp_i<kHalfMirror>((int)v));
    if (n > 8) v = max(v, (uint32_t)dpp_i<kMirror>((int)v));
    return v;
}

__device__ __forceinline__ double span_max(double v, int n) {
    if (n > 1) v = fmax(v, dpp_d<kSwap1>(v));
    if (n > 2) v = fmax(v, dpp_d<kSwap2>(v));
    if (n > 4) v = fmax(v, dpp_d<kHalfMirror>(v));
    if (n > 8) v = fmax(v, dpp_d<kMirror>(v));
    return v;
}

// Largest cand over the span, ties to the lower index cl; the result is the
// same on every lane of the span.
template <int CTRL>
__device__ __forceinline__ void argmax_step(double &cand, int &cl) {
    const double oc = dpp_d<CTRL>(cand);
    const int ol = dpp_i<CTRL>(cl);
    if (oc > cand || (oc == cand && ol < cl)) {
        cand = oc;
        cl = ol;
    }
}

__device__ __forceinline__ void span_argmax(double &cand, int &cl, int n) {
    if (n > 1) argmax_step<kSwap1>(cand, cl);
    if (n > 2) argmax_step<kSwap2>(cand, cl);
    if (n > 4) argmax_step<kHalfMirror>(cand, cl);
    if (n > 8) argmax_step<kMirror>(cand, cl);
}

// Sum over the LW lanes of a walker.
__device__ __forceinline__ double walker_sum(double v, int LW) { return span_sum(v, LW); }

__device__ __forceinline__ int walker_sum_i(int v, int LW) { return span_sum_i(v, LW); }

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint32_t lo0 = 0xD2511F53u * c[0], hi0 = __umulhi(0xD2511F53u, c[0]);
        const uint32_t lo1 = 0xCD9E8D57u * c[2], hi1 = __umulhi(0xCD9E8D57u, c[2]);
        const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = lo1;
        c[2] = n2;
        c[3] = lo0;
    }
}

struct Lane {
    int lane;    // 0..63
    int wloc;    // walker slot in the wave
    int lw;      // lane within walker, 0..LW-1
    int grp;     // 0 spin up, 1 spin down
    int i;       // index within the spin group
    int e;       // electron index within the walker
    int nsig;    // electrons of this spin
    int gbase;   // first lane of the group
    bool wvalid; // walker index < W
    bool active; // owns a real electron of a valid walker
};

// The lane's index, formed anew where it stands.  The compiler has moved a value
// kept across a divergent block to the accumulation registers at the block's
// end, before the masked lanes were back, which leaves it undefined in them.
// So indexes that idle lanes load global tables with are taken from here, idle
// lanes run the pair loops with the others instead of being masked, and
// what they hold is dropped by selects.
__device__ __forceinline__ int lane_now() {
    int z = 0;
    asm volatile("" : "+s"(z));
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, z));
}

__device__ __forceinline__ Lane make_lane(const DevSystem &S, int64_t wave_first_walker, int64_t W,
                                          int64_t *walker, int lane = threadIdx.x) {
    Lane L;
    L.lane = lane;
    L.wloc = L.lane / S.LW;
    L.lw = L.lane % S.LW;
    L.grp = L.lw / S.G;
    L.i = L.lw % S.G;
    L.nsig = L.grp == 0 ? S.n_up : S.n_dn;
    L.e = L.grp == 0 ? L.i : S.n_up + L.i;
    L.gbase = L.lane - L.i;
    const int64_t w = wave_first_walker + L.wloc;
    *walker = w;
    L.wvalid = (L.wloc < S.WPW) && (w < W);
    L.active = L.wvalid && (L.i < L.nsig);
    return L;
}

// Determinant ratio from a packed excitation code (rank | h1 << 2 |
// h2 << 5 | p1 << 8 | p2 << 13); T rows of `ts` columns starting at column
// c0 (particles are virtual orbitals, p >= c0).
__device__ __forceinline__ double ratio_code(const double *T, uint32_t c, int ts, int c0) {
    const uint32_t k = c & 3u;
    if (k == 0) return 1.0;
    const int h1 = (c >> 2) & 7, h2 = (c >> 5) & 7, p1 = ((c >> 8) & 31) - c0, p2 = ((c >> 13) & 31) - c0;
    const double a = T[h1 * ts + p1];
    if (k == 1) return a;
    return a * T[h2 * ts + p2] - T[h1 * ts + p2] * T[h2 * ts + p1];
}

// d = a * b + c as one three-address FMA: the constant c is not copied into
// the accumulator of a two-address FMA before every use.  VK: c in vector
// registers (the kernels that loop over steps at one wave per SIMD have
// those to spare, and hoist more scalars out of the loop than fit), else in
// scalar ones.
template <bool VK>
__device__ __forceinline__ double fma_c(double a, double b, double c) {
    double d;
    if constexpr (VK) asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    else asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}

// exp(x) in FP64 (qmc_exp.h), its polynomial's multiply-adds as
// three-address FMAs.
template <bool VK = false>
__device__ __forceinline__ double exp_f64(double x) { return exp_cody_waite(x, fma_c<VK>); }

// 1 / x for x well inside the exponent range (the Pade-type denominators
// 1 + b r >= 1, elimination pivots): the hardware reciprocal estimate refined
// by two Newton steps, within an ulp or so of the quotient.
__device__ __forceinline__ double rcp_ge1(double x) {
    double y = __builtin_amdgcn_rcp(x);
    double e = __builtin_fma(-x, y, 1.0);
    y = __builtin_fma(y, e, y);
    e = __builtin_fma(-x, y, 1.0);
    return __builtin_fma(y, e, y);
}

// a / b given y, 1 / b within an ulp or so: one residual step gives the
// rounded quotient (a == b gives exactly 1).  b well inside the exponent
// range.
__device__ __forceinline__ double div_by_rcp(double a, double b, double y) {
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-q, b, a), y, q);
}

template <typename RT, bool VK>
__device__ __forceinline__ RT rt_exp(RT x) {
    if constexpr (sizeof(RT) == sizeof(double)) return exp_f64<VK>(x);
    // FP32: the hardware base-2 exponential of x log2(e)
    else return __builtin_amdgcn_exp2f(x * 1.44269504088896341f);
}

// Radial part of one shell at distance r: R, and with DERIV also R'/r and
// R'' + (2l+2) R'/r.  Slater R = sum_p c_p r^kn exp(-zeta_p r), so R'/R =
// kn/r - zeta; Gaussian R = sum_p c_p exp(-alpha_p r^2), so R'/r = -2 alpha R
// and R'' + (2l+2) R'/r = (4 alpha^2 r^2 - (4l+6) alpha) R.  The primitive
// coefficients carry the radial normalisation.
template <typename RT, bool DERIV, bool VK = false>
__device__ __forceinline__ void shell_radial(const DevSystem &S, int p, int np, int l, int kn, RT r,
                                             RT r2, RT rinv, RT &Rv, RT &Rd, RT &Rl) {
    Rv = RT(0);
    Rd = RT(0);
    Rl = RT(0);
    if (S.basis == 0) {
        const RT fl = RT(2 * l + 2);
        RT rk = RT(1);
        for (int t = 0; t < kn; ++t) rk *= r;
        for (int q = 0; q < np; ++q) {
            const double2v pe = prim_info(S, p + q);
            const RT ex = RT(pe.x);
            const RT f = RT(pe.y) * rk * rt_exp<RT, VK>(-ex * r);
            Rv += f;
            if (DERIV) {
                const RT g = RT(kn) * rinv - ex;
                Rd += f * g * rinv;
                Rl += f * (g * g - RT(kn) * rinv * rinv + fl * g * rinv);
            }
        }
    } else {
        const RT fl = RT(4 * l + 6);
        auto add = [&](double2v pe, RT e) {
            const RT ex = RT(pe.x);
            const RT f = RT(pe.y) * e;
            Rv += f;
            if (DERIV) {
                Rd -= RT(2) * ex * f;
                Rl += f * (RT(4) * ex * ex * r2 - fl * ex);
            }
        };
        // two at a time: one scalar load and two independent exponentials
        int q = 0;
        for (; q + 1 < np; q += 2) {
            const double2v pa = prim_info(S, p + q), pb = prim_info(S, p + q + 1);
            const RT ea = rt_exp<RT, VK>(-RT(pa.x) * r2), eb = rt_exp<RT, VK>(-RT(pb.x) * r2);
            add(pa, ea);
            add(pb, eb);
        }
        if (q < np) {
            const double2v pa = prim_info(S, p + q);
            add(pa, rt_exp<RT, VK>(-RT(pa.x) * r2));
        }
    }
}

// ---- BF16 matrix-core contractions (mixed form) ------------------------------
// A wave applies the fixed 32 x 32 matrix M = C^T (MO values from AO values)
// to one 32-vector per lane with v_mfma_f32_16x16x32_bf16:
// output tile t (16 rows of M) times the vectors of lane quarter q (16 lanes)
// is one MFMA.  Vectors are staged through LDS so that lane 16 g + j supplies
// elements 8 g .. 8 g + 7 of lane 16 q + j's vector; the 16 x 16 result lands
// as rows 4 g .. 4 g + 3 in lane 16 g + j and goes back through LDS to the
// lane that owns the vector.  SPLIT = 3 writes every operand as a sum of a
// high and a low BF16 part and forms hi*hi + hi*lo + lo*hi (about 16
// significant bits); SPLIT = 1 uses the high parts only.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
constexpr int kStageK = 32;      // padded vector length
constexpr int kRowB = 40;        // bf16 per staged row (80 B, 16-byte aligned)
constexpr int kRowF = 36;        // floats per result row (144 B)
constexpr int kStageBytes = 2 * kWave * kRowB * 2 + kWave * kRowF * 4;

struct Stage {
    __bf16 *hi, *lo;  // [64][kRowB]
    float *out;       // [64][kRowF]
};

__device__ __forceinline__ Stage make_stage(void *base) {
    Stage st;
    st.hi = (__bf16 *)base;
    st.lo = st.hi + kWave * kRowB;
    st.out = (float *)(st.lo + kWave * kRowB);
    return st;
}

__device__ __forceinline__ void stage_put(const Stage &st, int lane, int k, float v) {
    const __bf16 h = (__bf16)v;
    st.hi[lane * kRowB + k] = h;
    st.lo[lane * kRowB + k] = (__bf16)(v - (float)h);
}

// out[lane][o] = sum_k M[o][k] v_lane[k] for o < 16 NT.
template <int NT, int SPLIT>
__device__ __forceinline__ void mfma_apply(const DevSystem &S, const Stage &st, int lane) {
    const int g = lane >> 4, j = lane & 15;
    bf16x8_t ahi[NT], alo[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const uint4 h = S.mfma_tab[(t * 2 + 0) * kWave + lane];
        const uint4 l = S.mfma_tab[(t * 2 + 1) * kWave + lane];
        ahi[t] = __builtin_bit_cast(bf16x8_t, h);
        alo[t] = __builtin_bit_cast(bf16x8_t, l);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int src = (16 * q + j) * kRowB + 8 * g;
        const bf16x8_t bh = *(const bf16x8_t *)(st.hi + src);
        const bf16x8_t bl = *(const bf16x8_t *)(st.lo + src);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[t], bh, acc, 0, 0, 0);
            if (SPLIT == 3) {
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[t], bl, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo[t], bh, acc, 0, 0, 0);
            }
            *(floatx4_t *)(st.out + (16 * q + j) * kRowF + 16 * t + 4 * g) = acc;
        }
    }
}

// Pass 1 on the matrix cores: AO values in FP32, staged as BF16 parts, MO
// values phi[m] = sum_mu C[mu][m] chi_mu with FP32 accumulation.  Every lane
// of the wave must call it.
template <int NMO, int SPLIT>
__device__ __forceinline__ void mo_values_mfma(const DevSystem &S, int lane, void *stage_base, double x0,
                                               double x1, double x2, float (&phi)[NMO]) {
    const Stage st = make_stage(stage_base);
    int p = 0, mu = 0;
    int atom = -1;
    float dx = 0.f, dy = 0.f, dz = 0.f, r2 = 0.f, r = 0.f;
    for (int sh = 0; sh < S.n_shells; ++sh) {
        const int4v si = shell_info(S, sh);
        if (si.x != atom) {  // shells of one atom share the geometry
            atom = si.x;
            const auto *A = const_tab(S.atoms) + 4 * atom;
            dx = float(x0 - A[0]);
            dy = float(x1 - A[1]);
            dz = float(x2 - A[2]);
            r2 = dx * dx + dy * dy + dz * dz;
            r = sqrtf(r2);
        }
        float Rv, Rd, Rl;
        shell_radial<float, false>(S, p, si.w, si.y, si.z, r, r2, 0.f, Rv, Rd, Rl);
        p += si.w;
        const int nc = (si.y + 1) * (si.y + 2) / 2;
        for (int c = 0; c < nc; ++c, ++mu) {
            float P;
            if (si.y == 0) P = 1.f;
            else if (si.y == 1) P = c == 0 ? dx : (c == 1 ? dy : dz);
            else {
                const float u = (c < 3) ? dx : (c < 5 ? dy : dz);
                const float v = (c == 0) ? dx : (c == 1 || c == 3) ? dy : dz;
                P = u * v;
            }
            stage_put(st, lane, mu, P * Rv);
        }
    }
    for (int k = mu; k < kStageK; ++k) stage_put(st, lane, k, 0.f);
    wave_sync();
    mfma_apply<(NMO + 15) / 16, SPLIT>(S, st, lane);
    wave_sync();
#pragma unroll
    for (int m = 0; m < NMO; ++m) phi[m] = st.out[lane * kRowF + m];
    wave_sync();
}

}  // namespace walker
}  // namespace qmc

#include "qmc_orbitals.h"

namespace qmc {
namespace walker {

// LDS of one walker (doubles): T tables [2][nmax][cols] at 0 (nmax =
// max(n_up, n_dn)) and the cofactor tables [2][nmax][cregion] after them,
// both written from the determinant stage on.  FULL layout (the adjoint's):
// cols = NMO, the T rows holding A0^-1 in their reference columns.  Compact
// layout (the evaluation and Metropolis kernels'): only the columns from
// c0 = min(n_up, n_dn), rounded down to even so that rows are read and
// written two columns at a time, the ones the ratios and cofactors read; A0^-1
// passes through the cofactor region (cregion = max(cols, nmax) per row)
// before the cofactors accumulate there.  Before the determinant stage the
// same space holds the e-e-n factor table (een_table doubles at 0, when
// e-e-n terms exist) and the positions [LW][3] + pivot rows [2][NMO] at
// pos_offset.
// Doubles of e-e-n geometry per lane and nucleus: r, the unit vector from
// the nucleus, 1 / r.
constexpr int kEenGeo = 5;

__host__ __device__ inline int een_table(const DevSystem &S) {
    return S.LW * S.n_atoms * 2 * S.een_n;
}

// Doubles of the e-e-n tables by which the explicit and backflow methods admit a
// system: the factors and every lane's geometry.  The tables no longer hold the
// geometry here; it stays in the limit so that the systems a caller sees refused
// do not depend on the kernels' layout.
inline int een_admit(const DevSystem &S) {
    return S.een_n > 0 ? S.LW * S.n_atoms * (2 * S.een_n + kEenGeo) + 3 * S.LW : 0;
}

template <int NMO, bool FULL = true>
__host__ __device__ inline int tab_c0(const DevSystem &S) {
    return FULL ? 0 : (S.n_up < S.n_dn ? S.n_up : S.n_dn) & ~1;
}

template <int NMO, bool FULL = true>
__host__ __device__ inline int tab_cols(const DevSystem &S) {
    return NMO - tab_c0<NMO, FULL>(S);
}

template <int NMO, bool FULL = true>
__host__ __device__ inline int tab_cregion(const DevSystem &S) {
    const int nmax = S.n_up > S.n_dn ? S.n_up : S.n_dn, cols = tab_cols<NMO, FULL>(S);
    return FULL ? cols : (cols > nmax ? cols : (nmax + 1) & ~1);
}

template <int NMO, bool FULL = true>
__host__ __device__ inline int pos_offset(const DevSystem &S) {
    const int nmax = S.n_up > S.n_dn ? S.n_up : S.n_dn;
    const int t = 2 * nmax * tab_cols<NMO, FULL>(S), f = een_table(S);
    return ((f > t ? f : t) + 3 * S.LW + 1) / 2 * 2 - 3 * S.LW;  // the pivot rows are 16-byte aligned
}

template <int NMO, bool FULL = true>
__host__ __device__ inline int walker_lds(const DevSystem &S) {
    const int nmax = S.n_up > S.n_dn ? S.n_up : S.n_dn;
    const int tc = 2 * nmax * (tab_cols<NMO, FULL>(S) + tab_cregion<NMO, FULL>(S));
    const int pp = pos_offset<NMO, FULL>(S) + 3 * S.LW + 2 * NMO;
    return ((tc > pp ? tc : pp) + 1) & ~1;  // 16-byte aligned rows
}

// ---- Jastrow stage -----------------------------------------------------------
// Separation of two points: r, 1 / r.  The hardware reciprocal root with one
// third-order step, and r corrected by its residual: the root within half an
// ulp or so, its reciprocal within an ulp, without the scaling and division
// of the full-range functions.  The refinement forms 0 * inf at r = 0 (an
// electron on a nucleus, or on another one, where every Jastrow term is finite)
// and at an infinite r; the division fix-up puts in the values of r2 / 1 and
// 1 / r2 there, 0 and inf.  (Many-body CO block of 16 384 walkers, 10 steps:
// 1105 us without it, 1113 so, 1156 by a comparison and selects.)
struct Sep {
    double r, ri;
};

__device__ __forceinline__ Sep separation(double d0, double d1, double d2) {
    const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
    double y = __builtin_amdgcn_rsq(r2);
    const double e = __builtin_fma(-(r2 * y), y, 1.0);
    y = __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
    double r = r2 * y;
    r = __builtin_fma(__builtin_fma(-r, r, r2), 0.5 * y, r);
    return {__builtin_amdgcn_div_fixup(r, 1.0, r2), __builtin_amdgcn_div_fixup(y, r2, 1.0)};
}

// Partner t = 1 .. N_e - 1 of electron e, cyclic, and its lane in the walker:
// every lane has N_e - 1 partners, none of them itself, so the pair loops
// have no idle trip.
__device__ __forceinline__ int partner(const DevSystem &S, int e, int t, int *lane) {
    int j = e + t;
    if (j >= S.ne) j -= S.ne;
    *lane = j < S.n_up ? j : S.G + (j - S.n_up);
    return j;
}

// g(r) = r / (1 + b r), the radial form of every Pade-type factor, with
// q = 1 / (1 + b r): g = r q, g' = q^2, g'' = -2 b q^3.
struct Pade {
    double q, g, g1, g2;
};

__device__ __forceinline__ Pade pade(double b, double r) {
    const double q = rcp_ge1(1.0 + b * r), q2 = q * q;
    return {q, r * q, q2, -2.0 * b * q2 * q};
}

// What the partners of the lane's electron read in the e-e-n terms: per
// nucleus a and term the factors g(b1; r_a), g(b2; r_a) (sF, [een_n][2]); with
// GEO (the adjoint) also its geometry (r_a, the unit vector from the nucleus,
// 1 / r_a: sG, [kEenGeo]).
template <bool GEO>
__device__ __forceinline__ void een_table_fill(const DevSystem &S, const Lane &L, double x0, double x1, double x2,
                                               double *sF, double *sG) {
    if (S.een_n == 0) return;
    for (int a = 0; a < S.n_atoms; ++a) {
        const auto *R = const_tab(S.atoms) + 4 * a;
        const double e0 = x0 - R[0], e1 = x1 - R[1], e2 = x2 - R[2];
        const Sep s = separation(e0, e1, e2);
        if constexpr (GEO) {
            double *g = sG + (L.lw * S.n_atoms + a) * kEenGeo;
            g[0] = s.r;
            g[1] = e0 * s.ri;
            g[2] = e1 * s.ri;
            g[3] = e2 * s.ri;
            g[4] = s.ri;
        }
        double *f = sF + (L.lw * S.n_atoms + a) * 2 * S.een_n;
        for (int m = 0; m < S.een_n; ++m) {
            const auto *t = const_tab(S.jas_een) + 7 * m;
            f[2 * m] = s.r * rcp_ge1(1.0 + t[2] * s.r);
            f[2 * m + 1] = s.r * rcp_ge1(1.0 + t[4] * s.r);
        }
    }
}

struct JasTerms {
    double J, g0, g1, g2, lap;
    double vpot;  // Coulomb terms of the electron
};

// Jastrow factor (eq. jastrow: Pade e-e kernel of eq. pade_kernel, e-n and
// e-e-n kernels of the many-body appendix) of the lane's electron: its share
// of J, grad_e J and lap_e J, and its Coulomb terms (eq. Hmol: half of each
// e-e pair, the e-n attraction).  sPos holds the walker's positions, sF the
// e-e-n factors of een_table_fill.  Idle lanes take electron 0's partners and
// return zeros.
__device__ __forceinline__ JasTerms jastrow_terms(const DevSystem &S, const Lane &L, double x0, double x1, double x2,
                                                  const double *sPos, const double *sF) {
    JasTerms o = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const int e = L.active ? L.e : 0;
    const bool up = e < S.n_up;
#pragma unroll 2
    for (int t = 1; t < S.ne; ++t) {
        int lj;
        const int j = partner(S, e, t, &lj);
        const double d0 = x0 - sPos[3 * lj], d1 = x1 - sPos[3 * lj + 1], d2 = x2 - sPos[3 * lj + 2];
        const Sep s = separation(d0, d1, d2);
        const double a = (j < S.n_up) == up ? S.a_par : S.a_anti;
        const Pade p = pade(S.b, s.r);
        const double k1 = a * p.g1, kr = k1 * s.ri;
        o.J += 0.5 * a * p.g;
        o.g0 += kr * d0;
        o.g1 += kr * d1;
        o.g2 += kr * d2;
        o.lap += a * p.g2 + 2.0 * kr;
        o.vpot += 0.5 * s.ri;
    }
    for (int a = 0; a < S.n_atoms; ++a) {
        const auto *R = const_tab(S.atoms) + 4 * a;
        const double d0 = x0 - R[0], d1 = x1 - R[1], d2 = x2 - R[2];
        const Sep s = separation(d0, d1, d2);
        o.vpot -= R[3] * s.ri;
        if (S.jas_en) {
            // e-n kernel K = N / D, N = w0 r + w1 r^2, D = 1 + w2 r:
            // K' = (N' - K D') / D and K'' = (N'' - 2 K' D') / D.  One division
            // per nucleus, so the full one: D may be past the largest double.
            const auto *w = const_tab(S.jas_en) + 3 * a;
            const double q = 1.0 / (1.0 + w[2] * s.r);
            const double K = (w[0] + w[1] * s.r) * s.r * q;
            const double K1 = (w[0] + 2.0 * w[1] * s.r - K * w[2]) * q;
            const double K2 = (2.0 * w[1] - 2.0 * K1 * w[2]) * q;
            const double kr = K1 * s.ri;
            o.J += K;
            o.g0 += kr * d0;
            o.g1 += kr * d1;
            o.g2 += kr * d2;
            o.lap += K2 + 2.0 * kr;
        }
    }
    // e-e-n kernel: for the ordered pair (i, j), i > j, the term is
    // c f1(r_ai) f2(r_aj) f3(r_ij), f_k = a_k g(b_k).  This electron takes
    // the role of i against lower-numbered partners and of j against higher
    // ones; its own factor carries the derivatives, the partner's is a value
    // from the table.  Per term, nucleus and role the partners enter through
    // five sums only,
    //   A = sum p s,  B = sum p s' w,  D = sum p (s'' + 2 s' / r)
    // (p the partner's factor, s = g(b3; r_ij), w the unit vector from the
    // partner), so the own factor's derivatives are formed once per role, not
    // once per partner.  A term symmetric in its electrons (f1 = f2, the
    // physical choice) has one role, in which every pair's value is met twice.
    // (CO, 5 symmetric terms: with a factor pair per partner this stage took
    // 75 k cycles of one wave, half of the step.)
    for (int m = 0; m < S.een_n; ++m) {
        const auto *tm = const_tab(S.jas_een) + 7 * m;
        const double b3 = tm[6], kc = tm[0] * tm[1] * tm[3] * tm[5];
        auto term = [&](auto roles) {
            constexpr int NR = decltype(roles)::value;
            for (int a0 = 0; a0 < S.n_atoms; a0 += 2) {  // two nuclei share a pair's s
                const int na = a0 + 1 < S.n_atoms ? 2 : 1;
                double A[2][NR], B[2][NR][3], D[2][NR];  // [nucleus][role]
#pragma unroll
                for (int n = 0; n < 2; ++n)
#pragma unroll
                    for (int r = 0; r < NR; ++r) A[n][r] = B[n][r][0] = B[n][r][1] = B[n][r][2] = D[n][r] = 0.0;
#pragma unroll 2
                for (int t = 1; t < S.ne; ++t) {
                    int lj;
                    const int j = partner(S, e, t, &lj);
                    const bool first = e > j;
                    const double d0 = x0 - sPos[3 * lj], d1 = x1 - sPos[3 * lj + 1], d2 = x2 - sPos[3 * lj + 2];
                    const Sep s = separation(d0, d1, d2);
                    const Pade p = pade(b3, s.r);
                    const double sr = p.g1 * s.ri, sd = p.g2 + 2.0 * sr;
                    const double *f = sF + ((lj * S.n_atoms + a0) * S.een_n + m) * 2 + (first ? 1 : 0);
#pragma unroll
                    for (int n = 0; n < 2; ++n) {
                        const double pv = f[n < na ? n * 2 * S.een_n : 0];
#pragma unroll
                        for (int r = 0; r < NR; ++r) {
                            const double pr = NR == 1 || first == (r == 0) ? pv : 0.0;
                            const double ps = pr * sr;
                            A[n][r] += pr * p.g;
                            B[n][r][0] += ps * d0;
                            B[n][r][1] += ps * d1;
                            B[n][r][2] += ps * d2;
                            D[n][r] += pr * sd;
                        }
                    }
                }
#pragma unroll
                for (int n = 0; n < 2; ++n) {
                    if (n >= na) break;
                    const auto *R = const_tab(S.atoms) + 4 * (a0 + n);
                    const double d0 = x0 - R[0], d1 = x1 - R[1], d2 = x2 - R[2];
                    const Sep u = separation(d0, d1, d2);
#pragma unroll
                    for (int r = 0; r < NR; ++r) {
                        const Pade q = pade(r == 0 ? tm[2] : tm[4], u.r);
                        const double k0 = kc * q.g, k1 = kc * q.g1, k2 = kc * q.g2, kr = k1 * u.ri;
                        const double dB = d0 * B[n][r][0] + d1 * B[n][r][1] + d2 * B[n][r][2];
                        if (r == 0) o.J += (NR == 1 ? 0.5 : 1.0) * k0 * A[n][r];
                        o.g0 += kr * A[n][r] * d0 + k0 * B[n][r][0];
                        o.g1 += kr * A[n][r] * d1 + k0 * B[n][r][1];
                        o.g2 += kr * A[n][r] * d2 + k0 * B[n][r][2];
                        o.lap += (k2 + 2.0 * kr) * A[n][r] + 2.0 * kr * dB + k0 * D[n][r];
                    }
                }
            }
        };
        if (tm[1] == tm[3] && tm[2] == tm[4]) term(std::integral_constant<int, 1>());
        else term(std::integral_constant<int, 2>());
    }
    auto own = [&](double v) { return L.active ? v : 0.0; };
    return {own(o.J), own(o.g0), own(o.g1), own(o.g2), own(o.lap), own(o.vpot)};
}

// Per-lane results of the stages every evaluation shares.
template <int NMO>
struct Core {
    double J, gJ0, gJ1, gJ2, lapJ, vpot;  // this electron's Jastrow and Coulomb terms
    int slot;                             // Gauss-Jordan slot of this electron
    double Ssum, logD_up, logD_dn, sgn_up, sgn_dn;
    int sing_walker;                      // > 0: a reference matrix is exactly singular
    double av[NMO];                       // a_e[m] = d log Sigma / d phi_m(r_e)
    double bgS0, bgS1, bgS2, blap;        // backflow: grad_e Sigma / Sigma, lap Sigma / Sigma share
};

// Jastrow and Coulomb terms, pass 1 (MO values), in-place Gauss-Jordan of
// the reference matrices, determinant ratios, S, cofactor tables and the
// adjoint vector a_e.  Every lane of the wave must call it (it exchanges
// through LDS).  On return the walker's LDS holds the T tables
// [2][nmax][NMO] at wsm and the cofactor tables right after them.
template <int NMO>
__device__ __forceinline__ void explicit_dets(const DevSystem &S, const Lane &L, double *wsm,
                                              const double (&phi)[NMO], Core<NMO> &c);

// Backflow: grad and Laplacian of Sigma of the backflow-transformed
// determinants (eq. nabla_d), every configuration explicitly.  Every lane of
// the block must call it.  sPos holds the walker's bare positions.
template <int NMO, bool LR, int CAP>
__device__ __forceinline__ void backflow_dets(const DevSystem &S, const Lane &L, double *wsm, double *sPos,
                                              double x0, double x1, double x2, double *buf, Core<NMO> &c);

template <int NMO, bool LR>
__host__ __device__ inline int bf_pos_offset(const DevSystem &S);

// In-place Gauss-Jordan of the spin group's reference matrix, a row per lane
// (NMO entries, this electron's MO values).  Pivot column j (reference orbital
// j after the create-time column permutation) is overwritten by the inverse,
// so at the end the row of slot s holds A0^-1[s][slot(e)] in the columns < n
// and T[s][v] = (A0^-1 Phi)[s][v] in the virtual columns.
// A step's chain is: largest |a[j]| of the rows left, that row through LDS, one
// reciprocal, one multiply-add per column.  The largest is taken on one word
// per lane (the upper bits of |a[j]|, then the lower lane), three cross-lane
// maxima.  inv_cnt: inversions of the row permutation (slot s <- electron row)
// at this lane, to be summed over the group.  piv_row: NMO doubles of LDS per
// group, 16-byte aligned.
template <int NMO>
__device__ __forceinline__ void eliminate(const DevSystem &S, const Lane &L, double (&a)[NMO], int nmax,
                                          double *piv_row, int &slot, int &inv_cnt, double &dprod, bool &singular) {
    constexpr int JMAX = kMaxSpin < NMO ? kMaxSpin : NMO;
    bool done = !L.active;
    slot = -1;
    inv_cnt = 0;
    dprod = 1.0;
    singular = false;
#pragma unroll
    for (int j = 0; j < JMAX; ++j) {
        if (j >= nmax) break;
        const bool work = j < L.nsig;
        uint32_t key = 0;  // 8 or more for a non-zero candidate
        if (work && !done && a[j] != 0.0) {
            const uint32_t hi = (uint32_t)__double2hiint(a[j]) & 0x7FFFFFF8u;
            key = (hi > 8u ? hi : 8u) | (uint32_t)(7 - L.i);
        }
        key = span_max_u(key, S.G);
        const int cl = 7 - (int)(key & 7u);
        const bool is_piv = key >= 8u && L.i == cl;
        if (is_piv) {
#pragma unroll
            for (int m = 0; m < NMO; m += 2) *(double2 *)(piv_row + m) = make_double2(a[m], a[m + 1]);
        }
        // rows left above the pivot's: its row permutation's inversions
        if (key >= 8u && !done && L.i < cl) ++inv_cnt;
        wave_sync();
        // the pivot from the published row (none: the column is zero, or NaN)
        const double piv = key >= 8u ? piv_row[j] : 0.0;
        const bool ok = fabs(piv) > 0.0;
        if (work && !ok) singular = true;
        if (work) dprod *= piv;
        // multiplier as in Doolittle elimination: equal rows cancel exactly
        const double y = rcp_ge1(piv);
        double inv = div_by_rcp(1.0, piv, y), f = div_by_rcp(a[j], piv, y);
        // (a pivot at the ends of the exponent range takes the full division)
        const uint32_t top = (uint32_t)__double2hiint(piv) & 0x7FFFFFFFu;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(ok && top - 0x03C00000u > 0x78400000u) != 0, 0)) {
            inv = 1.0 / piv;
            f = a[j] / piv;
        }
        if (is_piv) {  // this row is scaled in place
#pragma unroll
            for (int m = 0; m < NMO; ++m) a[m] *= inv;
            a[j] = inv;
            done = true;
            slot = j;
        } else if (ok) {
#pragma unroll
            for (int m = 0; m < NMO; m += 2) {
                const double2 pr = *(const double2 *)(piv_row + m);
                a[m] -= f * pr.x;
                a[m + 1] -= f * pr.y;
            }
            a[j] = -f;
        }
        wave_sync();
    }
}

// PSI: stop once log|Psi| is known (no cofactor tables, no adjoint vector):
// the values a finite-difference kinetic energy needs.  RT is the arithmetic
// of the AO evaluation and MF the MO contraction of pass 1 (FP64 when RT is
// double).  FULLT: the full table layout (walker_lds<NMO, true>), which the
// adjoint reads, and its direction B into *bvec; otherwise the compact one.
// VK: see fma_c.
template <int NMO, typename RT, int MF = 0, bool EXPL = false, int BF = 0, bool PSI = false,
          bool FULLT = false, bool VK = false>
__device__ __forceinline__ void core_stages(const DevSystem &S, const Lane &L, double *wsm, double &x0,
                                            double &x1, double &x2, Core<NMO> &c, void *stage = nullptr,
                                            double (*bvec)[NMO] = nullptr) {
    // the compact layout serves the low-rank Metropolis and evaluation
    // kernels (fewer LDS bytes per wave, more waves per CU)
    constexpr bool kFull = FULLT || EXPL || BF;
    const int nmax = S.n_up > S.n_dn ? S.n_up : S.n_dn;
    const int c0 = tab_c0<NMO, kFull>(S), ts = tab_cols<NMO, kFull>(S);
    const int tstride = nmax * ts;                           // doubles per spin T table
    const int cstride = nmax * tab_cregion<NMO, kFull>(S);   // doubles per spin cofactor table
    double *sT = wsm;                        // [2][nmax][ts]
    double *sC = sT + 2 * tstride;           // [2][nmax][cregion / nmax] after the elimination
    // [LW][3] before the elimination (with backflow: after the backflow tables)
    double *sPos = wsm + (BF ? bf_pos_offset<NMO, !EXPL>(S) : pos_offset<NMO, kFull>(S));
    double *sPiv = sPos + 3 * S.LW;          // [2][NMO] during it
    // e-e-n table before the elimination: per lane [n_atoms][een_n][2]
    // factor values (f1, f2) of its electron
    double *sF = wsm;
    double *Tg = sT + L.grp * tstride;
    double *Cg = sC + L.grp * cstride;
    double *piv_row = sPiv + L.grp * NMO;

    if (!L.active) {  // a far point keeps idle lanes finite
        x0 = 100.0;
        x1 = 100.0;
        x2 = 100.0;
    }
    sPos[3 * L.lw + 0] = x0;
    sPos[3 * L.lw + 1] = x1;
    sPos[3 * L.lw + 2] = x2;
    een_table_fill<false>(S, L, x0, x1, x2, sF, nullptr);
    wave_sync();

    // ---- Jastrow and Coulomb terms of this electron (FP64) ----------------
    const JasTerms jt = jastrow_terms(S, L, x0, x1, x2, sPos, sF);
    const double J = jt.J, gJ0 = jt.g0, gJ1 = jt.g1, gJ2 = jt.g2, lapJ = jt.lap, vpot = jt.vpot;

    c.J = J;
    c.gJ0 = gJ0;
    c.gJ1 = gJ1;
    c.gJ2 = gJ2;
    c.lapJ = lapJ;
    c.vpot = vpot;

    if constexpr (BF) {
        backflow_dets<NMO, !EXPL, (BF == 1 ? kSmallCfgBF : kMaxCfgBF)>(S, L, wsm, sPos, x0, x1, x2,
                                                                             (double *)stage, c);
        return;
    }

    // ---- pass 1: MO values of this electron ------------------------------
    // (the LDS stage of the contractions overlays the walkers' tables, whose
    // positions the pair loop has read)
    double a[NMO];
    if constexpr (FULLT) {
        // the adjoint's direction B beside the values
        wave_sync();
        const double gj[3] = {gJ0, gJ1, gJ2};
        mo_values_direction<NMO>(S, L.lane, (double *)stage, x0, x1, x2, gj, a, *bvec);
        if constexpr (sizeof(RT) != sizeof(double)) {
            float phi[NMO];
            mo_values_f32<NMO>(S, L.lane, x0, x1, x2, phi);
#pragma unroll
            for (int m = 0; m < NMO; ++m) a[m] = double(phi[m]);
        }
    } else if constexpr (sizeof(RT) == sizeof(double)) {
        wave_sync();
        double phi[NMO];
        mo_values_f64<NMO, VK>(S, L.lane, (double *)stage, x0, x1, x2, phi);
#pragma unroll
        for (int m = 0; m < NMO; ++m) a[m] = phi[m];
    } else if constexpr (MF > 0) {
        // the staging area overlays the walkers' tables: wait for the
        // position reads of the pair loop first
        wave_sync();
        float phi[NMO];
        mo_values_mfma<NMO, MF>(S, L.lane, stage, x0, x1, x2, phi);
#pragma unroll
        for (int m = 0; m < NMO; ++m) a[m] = double(phi[m]);
    } else {
        float phi[NMO];
        mo_values_f32<NMO>(S, L.lane, x0, x1, x2, phi);
#pragma unroll
        for (int m = 0; m < NMO; ++m) a[m] = double(phi[m]);
    }
    if constexpr (EXPL) {
        explicit_dets<NMO>(S, L, wsm, a, c);
        return;
    }

    // ---- elimination of the reference matrix ------------------------------
    constexpr int JMAX = kMaxSpin < NMO ? kMaxSpin : NMO;
    int slot, inv_cnt;
    double dprod;
    bool singular;
    eliminate<NMO>(S, L, a, nmax, piv_row, slot, inv_cnt, dprod, singular);
    // compact layout: the reference part of each slot's row (A0^-1) goes
    // to the cofactor region for a moment, and each lane keeps its column
    double ainv[JMAX];
    if (L.active && slot >= 0) {
#pragma unroll
        for (int m = 0; m < NMO; m += 2)
            if (m >= c0) *(double2 *)(Tg + slot * ts + m - c0) = make_double2(a[m], a[m + 1]);
        if constexpr (!kFull) {
#pragma unroll
            for (int k = 0; k < JMAX; ++k)
                if (k < nmax) Cg[slot * nmax + k] = a[k];
        }
    }
    if constexpr (!kFull) {
        wave_sync();
        const int sl = slot < 0 ? 0 : slot;
#pragma unroll
        for (int k = 0; k < JMAX; ++k) {
            const double t = Cg[(k < nmax ? k : 0) * nmax + sl];
            ainv[k] = (k < L.nsig && L.active) ? t : 0.0;
        }
        wave_sync();
    }
    // Permutation parity (slot s <- electron row): inversions within the group.
    inv_cnt = span_sum_i(inv_cnt, S.G);
    const double det_sign = ((inv_cnt & 1) ? -1.0 : 1.0) * (dprod < 0.0 ? -1.0 : 1.0);
    const double det_log = log(fabs(dprod));
    // the shared region now becomes the cofactor tables: zero them
    for (int q = 2 * L.lw; q < 2 * cstride; q += 2 * S.LW) *(double2 *)(sC + q) = make_double2(0.0, 0.0);
    wave_sync();

    const int wb = L.lane - L.lw;
    const double logD_up = __shfl(det_log, wb), logD_dn = __shfl(det_log, wb + S.G);
    const double sgn_up = __shfl(det_sign, wb), sgn_dn = __shfl(det_sign, wb + S.G);
    const int sing_walker = walker_sum_i(singular ? 1 : 0, S.LW);

    // ---- S = sum_n d_n det T_up[H,P] det T_dn[H,P] ----------------------
    // records are loaded kRecBatch at a time so their latencies overlap
    const double *Tup = sT, *Tdn = sT + tstride;
    const int lw = lane_now() & (S.LW - 1);
    double Sp = 0.0;
    for (int i0 = 0; i0 < S.det_rows; i0 += kRecBatch) {
        uint4v rb[kRecBatch];
#pragma unroll
        for (int u = 0; u < kRecBatch; ++u)
            rb[u] = i0 + u < S.det_rows ? const_tab((const uint4v *)S.det_recs)[(i0 + u) * S.LW + lw] : uint4v{0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < kRecBatch; ++u) {
            const uint4v r = rb[u];
            Sp += __hiloint2double((int)r.y, (int)r.x) * ratio_code(Tup, r.z, ts, c0) * ratio_code(Tdn, r.w, ts, c0);
        }
    }
    const double Ssum = walker_sum(Sp, S.LW);
    if constexpr (PSI) {
        c.slot = slot;
        c.Ssum = Ssum;
        c.logD_up = logD_up;
        c.logD_dn = logD_dn;
        c.sgn_up = sgn_up;
        c.sgn_dn = sgn_dn;
        c.sing_walker = sing_walker;
        wave_sync();  // the tables are reused by the next evaluation
        return;
    }

    // ---- cofactor tables C_sigma[k][v] = dS / dT_sigma[k][v] ---------------
    // each lane runs its own list of contributions (same length on every
    // lane) and writes an entry after its last contribution
    {
        double acc = 0.0;
        for (int i0 = 0; i0 < S.cof_rows; i0 += kRecBatch) {
            uint4v rb[kRecBatch];
#pragma unroll
            for (int u = 0; u < kRecBatch; ++u)
                rb[u] = i0 + u < S.cof_rows ? const_tab((const uint4v *)S.cof_recs)[(i0 + u) * S.LW + lw] : uint4v{0, 0, 0, 0};
#pragma unroll
            for (int u = 0; u < kRecBatch; ++u) {
                const uint4v r = rb[u];  // an all-zero padding record adds 0 and never flushes
                const int spin = (r.w >> 1) & 1;
                const double *Ts = spin ? Tdn : Tup, *To = spin ? Tup : Tdn;
                const uint32_t cc = r.z >> 18;
                const double tv = Ts[((cc >> 2) & 7) * ts + (cc >> 5) - c0];
                const double cof = (cc & 3) == 0 ? 1.0 : ((cc & 3) == 1 ? tv : -tv);
                acc += __hiloint2double((int)r.y, (int)r.x) * ratio_code(To, r.z & 0x3FFFFu, ts, c0) * cof;
                if (r.w & 1u) {
                    sC[spin * cstride + ((r.w >> 2) & 7) * ts + (r.w >> 5) - c0] = acc;
                    acc = 0.0;
                }
            }
        }
    }
    wave_sync();

    // ---- a_e = d log Sigma / d phi(r_e) ------------------------------------
    // virtual orbitals: a_e[v] = (A0^-T C)[e][v] / S (C vanishes on the
    // reference columns); reference orbitals: a_e[k] = A0^-1[k][e] -
    // sum_v T[k][v] a_e[v].
    double (&av)[NMO] = c.av;
    {
        if constexpr (kFull) {
            const int sl = slot < 0 ? 0 : slot;
#pragma unroll
            for (int k = 0; k < JMAX; ++k) {
                ainv[k] = 0.0;
                if (k < nmax) {
                    const double t = Tg[k * ts + sl];
                    ainv[k] = (k < L.nsig && L.active) ? t : 0.0;
                }
            }
        }
        const double Sinv = 1.0 / Ssum;
        // two columns at a time with every row's reads in one batch; KR, the
        // rows read, is G (rows past nmax repeat the last one, their a_e
        // column is zero)
        auto adjoint = [&](auto rows) {
            constexpr int KR = decltype(rows)::value < JMAX ? decltype(rows)::value : JMAX;
            const double *row[KR];
#pragma unroll
            for (int k = 0; k < KR; ++k) row[k] = Cg + (k < nmax ? k : nmax - 1) * ts - c0;
#pragma unroll
            for (int v = 0; v < NMO; v += 2) {
                double a0 = 0.0, a1 = 0.0;
                if (v >= c0) {
#pragma unroll
                    for (int k = 0; k < KR; ++k) {
                        const double2 cv = *(const double2 *)(row[k] + v);
                        a0 += ainv[k] * cv.x;
                        a1 += ainv[k] * cv.y;
                    }
                }
                av[v] = a0 * Sinv;
                av[v + 1] = a1 * Sinv;
            }
            double h[KR];
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                row[k] += Tg - Cg;
                h[k] = 0.0;
            }
#pragma unroll
            for (int v = 0; v < NMO; v += 2) {
                if (v >= c0) {
#pragma unroll
                    for (int k = 0; k < KR; ++k) {
                        const double2 tv = *(const double2 *)(row[k] + v);
                        h[k] += tv.x * av[v];
                        h[k] += tv.y * av[v + 1];
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < KR; ++k) av[k] = (k < L.nsig) ? ainv[k] - h[k] : av[k];
        };
        if (S.G <= 2) adjoint(std::integral_constant<int, 2>());
        else if (S.G == 4) adjoint(std::integral_constant<int, 4>());
        else adjoint(std::integral_constant<int, 8>());
    }

    c.slot = slot;
    c.Ssum = Ssum;
    c.logD_up = logD_up;
    c.logD_dn = logD_dn;
    c.sgn_up = sgn_up;
    c.sgn_dn = sgn_dn;
    c.sing_walker = sing_walker;
}

// ---- explicit determinants (comparison method) ---------------------------
// Every distinct spin configuration c of the CI expansion is factorised on
// its own: A_c[e][k] = phi_{occ_c[k]}(r_e) (rows = electrons of the spin,
// columns = the configuration's orbital slots) by the same in-place
// Gauss-Jordan across the spin group as the reference matrix of the
// low-rank path.  Sigma = sum_n d_n D_up D_dn, and
// a_e[m] = d log Sigma / d phi_m(r_e) = sum_c W_c (A_c^-1)[k][e] for
// m = occ_c[k], W_c = (sum over the determinants using c of d_n D_other)
// D_c / Sigma.  This is the work the low-rank scheme of eq. table avoids:
// one factorisation per configuration instead of one per spin.

// LDS of one walker for the explicit method (doubles): MO rows [LW][NMO],
// adjoint rows [LW][NMO], per configuration (log|D|, sign, weight)
// [2][n_cfg_max][3], inverse table [2][kMaxSpin][kMaxSpin], pivot rows
// [2][kMaxSpin]; the Jastrow stage's tables and positions come first and
// are dead by then.
template <int NMO>
__host__ __device__ inline int walker_lds_explicit(const DevSystem &S) {
    const int ex = 2 * S.LW * NMO + 6 * S.n_cfg_max + 2 * kMaxSpin * kMaxSpin + 2 * kMaxSpin;
    const int js = pos_offset<NMO>(S) + 3 * S.LW;
    return ex > js ? ex : js;
}

__device__ __forceinline__ double walker_max(double v, int LW) { return span_max(v, LW); }

// In-place Gauss-Jordan of the group's n x n matrix held as one row per
// lane (a[k], k < n; entries beyond n are zero).  Pivot columns are
// overwritten by the inverse exactly as for the reference matrix; slot is
// the pivot step that consumed this lane's row.  Every lane of the block
// runs the same nmax steps (block barriers inside).
__device__ __forceinline__ void group_gauss_jordan(const DevSystem &S, const Lane &L, double (&a)[kMaxSpin],
                                                   int n, int nmax, bool live, double *piv_row, int &slot,
                                                   double &dprod, bool &singular) {
    bool done = !L.active || !live;
    slot = -1;
    dprod = 1.0;
    singular = false;
#pragma unroll
    for (int j = 0; j < kMaxSpin; ++j) {
        if (j >= nmax) break;
        const bool work = live && j < n;
        double cand = (work && !done) ? fabs(a[j]) : -1.0;
        int cl = L.i;
        span_argmax(cand, cl, S.G);
        const bool ok = work && cand > 0.0;
        if (work && !ok) singular = true;
        const bool is_piv = ok && L.active && L.i == cl;
        if (is_piv) {
#pragma unroll
            for (int m = 0; m < kMaxSpin; ++m) piv_row[m] = a[m];
            const double inv = 1.0 / a[j];
#pragma unroll
            for (int m = 0; m < kMaxSpin; ++m) a[m] *= inv;
            a[j] = inv;
            done = true;
            slot = j;
        }
        wave_sync();
        const double piv = ok ? piv_row[j] : 0.0;
        if (work) dprod *= piv;
        if (ok && L.active && !is_piv) {
            const double f = a[j] / piv;
#pragma unroll
            for (int m = 0; m < kMaxSpin; ++m) a[m] -= f * piv_row[m];
            a[j] = -f;
        }
        wave_sync();
    }
}

// Sign of the row permutation (slot s <- electron row) within the group.
__device__ __forceinline__ double group_parity(const DevSystem &S, const Lane &L, int slot) {
    int inv_cnt = 0;
    for (int ip = 0; ip < S.G; ++ip) {
        const int so = __shfl(slot, L.gbase + ip);
        if (L.active && ip > L.i && so >= 0 && so < slot) ++inv_cnt;
    }
    inv_cnt = span_sum_i(inv_cnt, S.G);
    return (inv_cnt & 1) ? -1.0 : 1.0;
}

template <int NMO>
__device__ __forceinline__ void explicit_dets(const DevSystem &S, const Lane &L, double *wsm,
                                              const double (&phi)[NMO], Core<NMO> &c) {
    const int nmax = S.n_up > S.n_dn ? S.n_up : S.n_dn;
    double *sPhi = wsm;                                   // [LW][NMO]
    double *sA = sPhi + S.LW * NMO;                       // [LW][NMO]
    double *sCfg = sA + S.LW * NMO;                       // [2][n_cfg_max][3]
    double *sInv = sCfg + 6 * S.n_cfg_max;                // [2][kMaxSpin][kMaxSpin]
    double *sPv = sInv + 2 * kMaxSpin * kMaxSpin;         // [2][kMaxSpin]
    double *inv_g = sInv + L.grp * kMaxSpin * kMaxSpin;
    double *piv_g = sPv + L.grp * kMaxSpin;
    double *cfg_g = sCfg + L.grp * S.n_cfg_max * 3;
    const int *occ_g = S.cfg_occ + L.grp * S.n_cfg_max * kMaxSpin;
    const int ncfg_g = L.grp == 0 ? S.n_cfg_up : S.n_cfg_dn;
    const int ncmax = S.n_cfg_up > S.n_cfg_dn ? S.n_cfg_up : S.n_cfg_dn;

    wave_sync();  // the Jastrow stage's tables are no longer read
#pragma unroll
    for (int m = 0; m < NMO; ++m) {
        sPhi[L.lw * NMO + m] = phi[m];
        sA[L.lw * NMO + m] = 0.0;
    }
    wave_sync();

    // pass A: log|D_c| and sign of every configuration of this spin
    for (int q = 0; q < ncmax; ++q) {
        const bool live = q < ncfg_g;
        const int *occ = occ_g + (live ? q : 0) * kMaxSpin;
        double a[kMaxSpin];
#pragma unroll
        for (int k = 0; k < kMaxSpin; ++k)
            a[k] = (L.active && live && k < L.nsig) ? sPhi[L.lw * NMO + occ[k]] : 0.0;
        int slot;
        double dprod;
        bool singular;
        group_gauss_jordan(S, L, a, L.nsig, nmax, live, piv_g, slot, dprod, singular);
        const double par = group_parity(S, L, slot);
        if (live && L.i == 0) {
            cfg_g[3 * q] = singular ? -INFINITY : log(fabs(dprod));
            cfg_g[3 * q + 1] = singular ? 0.0 : par * (dprod < 0.0 ? -1.0 : 1.0);
        }
    }
    wave_sync();

    // common shifts, Sigma / (e^mu e^md)
    const int lw = lane_now() & (S.LW - 1);
    double mu = -INFINITY, md = -INFINITY;
    for (int q = lw; q < S.n_cfg_up; q += S.LW) mu = fmax(mu, sCfg[3 * q]);
    for (int q = lw; q < S.n_cfg_dn; q += S.LW) md = fmax(md, sCfg[3 * (S.n_cfg_max + q)]);
    mu = walker_max(mu, S.LW);
    md = walker_max(md, S.LW);
    const bool none = mu == -INFINITY || md == -INFINITY;
    double Sp = 0.0;
    if (!none)
        for (int n = lw; n < S.n_det_x; n += S.LW) {
            const int2 dc = S.det_cfg[n];
            const double *u = sCfg + 3 * dc.x, *v = sCfg + 3 * (S.n_cfg_max + dc.y);
            Sp += S.ci_x[n] * u[1] * v[1] * exp((u[0] - mu) + (v[0] - md));
        }
    const double Ssum = walker_sum(Sp, S.LW);
    const bool zero = none || Ssum == 0.0 || !isfinite(Ssum);

    // weights W_c (the lanes split both spins' configurations)
    for (int q = lw; q < S.n_cfg_up + S.n_cfg_dn; q += S.LW) {
        const int sp = q < S.n_cfg_up ? 0 : 1;
        const int cq = sp ? q - S.n_cfg_up : q;
        double *own = sCfg + 3 * (sp * S.n_cfg_max + cq);
        const double m_own = sp ? md : mu, m_oth = sp ? mu : md;
        double acc = 0.0;
        const int *off = S.cfg_off + sp * (S.n_cfg_max + 1);
        for (int t = off[cq]; t < off[cq + 1]; ++t) {
            const int2 e = S.cfg_use[t];
            const double *o = sCfg + 3 * ((1 - sp) * S.n_cfg_max + e.y);
            acc += S.ci_x[e.x] * o[1] * exp(o[0] - m_oth);
        }
        own[2] = zero ? 0.0 : acc * own[1] * exp(own[0] - m_own) / Ssum;
    }
    wave_sync();

    // pass B: a_e accumulated from each weighted inverse
    for (int q = 0; q < ncmax; ++q) {
        const bool in = q < ncfg_g;
        const double wq = in ? cfg_g[3 * q + 2] : 0.0;
        const bool live = in && wq != 0.0;
        const int *occ = occ_g + (in ? q : 0) * kMaxSpin;
        double a[kMaxSpin];
#pragma unroll
        for (int k = 0; k < kMaxSpin; ++k)
            a[k] = (L.active && live && k < L.nsig) ? sPhi[L.lw * NMO + occ[k]] : 0.0;
        int slot;
        double dprod;
        bool singular;
        group_gauss_jordan(S, L, a, L.nsig, nmax, live, piv_g, slot, dprod, singular);
        if (live && L.active && slot >= 0) {
#pragma unroll
            for (int k = 0; k < kMaxSpin; ++k) inv_g[slot * kMaxSpin + k] = a[k];
        }
        wave_sync();
        if (live && L.active && slot >= 0) {
            for (int k = 0; k < L.nsig; ++k) sA[L.lw * NMO + occ[k]] += wq * inv_g[k * kMaxSpin + slot];
        }
        wave_sync();
    }
#pragma unroll
    for (int m = 0; m < NMO; ++m) c.av[m] = sA[L.lw * NMO + m];
    c.slot = -1;
    c.Ssum = Ssum;
    c.logD_up = mu;
    c.logD_dn = md;
    c.sgn_up = 1.0;
    c.sgn_dn = 1.0;
    c.sing_walker = zero ? 1 : 0;
}

}  // namespace walker
}  // namespace qmc

#include "qmc_backflow.h"
