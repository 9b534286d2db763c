// Device code shared by the pair-sweep kernels (all-pairs and cell list):
// pair arithmetic, fixed-order workgroup reductions and the per-tile and
// per-cluster epilogues that finish a sweep once every partial sum of a tile
// (or every tile of a cluster) has arrived.
#pragma once

#include <type_traits>

#include "../../include/scmd.h"
#include "bath.h"
#include "scmd_internal.h"

namespace scmd {
namespace dev {

constexpr double kSelfR2 = 1.0e300;
constexpr float kSelfR2f = 1.0e30f;

// 1/x in double: hardware estimate (about 2^-23 relative) refined by one
// Newton-Raphson step e = 1 - x y, y += y e (relative error ~ e^2).
__device__ __forceinline__ double rcp_nr(double x) {
    double y = __builtin_amdgcn_rcp(x);
    double e = __builtin_fma(-x, y, 1.0);
    return __builtin_fma(y, e, y);
}

// 1/sqrt(x) in double: hardware estimate refined by one Newton-Raphson step
// y <- y (3/2 - (x/2) y^2) (relative error ~ 1.5 e^2).
__device__ __forceinline__ double rsq_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
    double hx = 0.5 * x;
    double e = __builtin_fma(-hx, y * y, 1.5);
    return y * e;
}

// r[k][i] = b[i]^e[k] for E exponents at once (they share the squarings of b,
// which is overwritten): wave-uniform exponents, so every test is a scalar
// branch, taken once for all N values.
template <typename T, int N, int E>
__device__ __forceinline__ void powers(T (&b)[N], int (&e)[E], T (&r)[E][N]) {
    int all = 0;
#pragma unroll
    for (int k = 0; k < E; ++k) {
        all |= e[k];
#pragma unroll
        for (int i = 0; i < N; ++i) r[k][i] = T(1);
    }
    for (;;) {
#pragma unroll
        for (int k = 0; k < E; ++k) {
            if (e[k] & 1) {
#pragma unroll
                for (int i = 0; i < N; ++i) r[k][i] *= b[i];
            }
            e[k] >>= 1;
        }
        all >>= 1;
        if (all == 0) break;
#pragma unroll
        for (int i = 0; i < N; ++i) b[i] *= b[i];
    }
}

// General exponents, N pairs at a time: u^m from r^2 (in double also for the
// mixed form, which then works in single precision).
template <int PREC, int N>
__device__ __forceinline__ void generic_density(const double (&r2)[N], const PotConst &pc, double (&t)[N]) {
    using T = std::conditional_t<PREC == SCMD_FP64, double, float>;
    T b[N], r[1][N];
    const bool even = (pc.m & 1) == 0;  // even m: powers of 1/r^2
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if constexpr (PREC == SCMD_FP64)
            b[i] = even ? rcp_nr(r2[i]) : rsq_nr(r2[i]);
        else
            b[i] = even ? __builtin_amdgcn_rcpf((float)r2[i]) : __builtin_amdgcn_rsqf((float)r2[i]);
    }
    int e[1] = {even ? pc.m >> 1 : pc.m};
    powers<T, N, 1>(b, e, r);
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = (double)r[0][i];
}

// The force coefficients u^(m+2) [A u^(n-m) - P_i - P_j] and, with EN, u^n.
template <int PREC, int N, bool EN>
__device__ __forceinline__ void generic_force(const double (&r2)[N], double ci, const double (&pj)[N], float cif,
                                              const float (&pjf)[N], const PotConst &pc, float Af, double (&f)[N],
                                              double (&un)[N]) {
    using T = std::conditional_t<PREC == SCMD_FP64, double, float>;
    constexpr int E = EN ? 3 : 2;
    T b[N], r[E][N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if constexpr (PREC == SCMD_FP64)
            b[i] = rsq_nr(r2[i]);
        else
            b[i] = __builtin_amdgcn_rsqf((float)r2[i]);
    }
    int e[E];
    e[0] = pc.m + 2;
    e[1] = pc.n - pc.m;
    if constexpr (EN) e[2] = pc.n;
    powers<T, N, E>(b, e, r);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if constexpr (PREC == SCMD_FP64)
            f[i] = r[0][i] * (__builtin_fma(pc.A, r[1][i], ci) - pj[i]);
        else
            f[i] = (double)(r[0][i] * (__builtin_fmaf(Af, r[1][i], cif) - pjf[i]));
        if constexpr (EN) un[i] = (double)r[2][i];
    }
}

// ---------------------------------------------------------------------------
// Density term: acc += u^m (minus rc^-m inside the cutoff when CUT), u = 1/r.
// MASK: the pair is void (self pair or outside the cutoff) when `off`.
// ---------------------------------------------------------------------------
template <int PREC, bool GEN, bool MASK, bool CUT>
__device__ __forceinline__ void density_pair(double dx, double dy, double dz, bool self, double &acc,
                                             const PotConst &pc) {
    if constexpr (PREC == SCMD_FP64) {
        double r2 = __builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz));
        bool off = false;
        if constexpr (CUT) off = !(r2 < pc.rc2);
        if constexpr (MASK) off = off || self;
        if constexpr (MASK || CUT) r2 = off ? kSelfR2 : r2;
        double t;
        if constexpr (!GEN) {
            double w = rcp_nr(r2);  // u^2
            t = w * w * w;
        } else {
            double x[1] = {r2}, y[1];
            generic_density<PREC, 1>(x, pc, y);
            t = y[0];
        }
        if constexpr (CUT) {
            acc += off ? 0.0 : t - pc.inv_rc_m;
        } else {
            acc += t;
        }
    } else {
        // mixed: r_i - r_j and r^2 in double (the cutoff decision matches the
        // double path), the powers in single precision, the sum in double
        const double r2d = __builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz));
        bool off = false;
        if constexpr (CUT) off = !(r2d < pc.rc2);
        if constexpr (MASK) off = off || self;
        float r2 = (float)r2d;
        if constexpr (MASK || CUT) r2 = off ? kSelfR2f : r2;
        double t;
        if constexpr (!GEN) {
            float w = __builtin_amdgcn_rcpf(r2);
            t = (double)(w * w * w);
        } else {
            double x[1] = {(double)r2}, y[1];
            generic_density<PREC, 1>(x, pc, y);
            t = y[0];
        }
        if constexpr (CUT) {
            acc += off ? 0.0 : t - pc.inv_rc_m;
        } else {
            acc += t;
        }
    }
}

// ---------------------------------------------------------------------------
// Force and pair-energy terms:
//   F_i += u^(m+2) [A u^(n-m) - P_i - P_j] (r_i - r_j),  eu += u^n (- rc^-n).
// ci = -P_i, pj = P_j (single-precision copies for the mixed form).
//
// The FP64 (n, m) = (9, 6) form works with w = 2u: the Newton step for
// 1/sqrt(r^2) written without its factor 1/2, w = y (3 - r^2 y^2), is exactly
// twice y (3/2 - (r^2/2) y^2) (scaling by 2 commutes with rounding), so one
// multiply per pair drops out.  With A/8 in place of A every later product
// is an exact power-of-two multiple of the unscaled one: the force sums come
// out 2^8 and the u^n sums 2^9 times too large, and unscale_force() divides
// them out once per sum.  The results are bitwise those of the form with u.
// ---------------------------------------------------------------------------
template <int PREC, bool GEN>
struct ForceScale {
    static constexpr double f = 1.0, e = 1.0;
};
template <>
struct ForceScale<SCMD_FP64, false> {
    static constexpr double f = 1.0 / 256.0, e = 1.0 / 512.0;
};

template <int PREC, bool GEN>
__device__ __forceinline__ void unscale_force(double &fx, double &fy, double &fz, double &eu) {
    if constexpr (ForceScale<PREC, GEN>::f != 1.0) {
        fx *= ForceScale<PREC, GEN>::f;
        fy *= ForceScale<PREC, GEN>::f;
        fz *= ForceScale<PREC, GEN>::f;
        eu *= ForceScale<PREC, GEN>::e;
    }
}

// 2/sqrt(x) from the hardware estimate and one Newton step (see above).
__device__ __forceinline__ double rsq2_nr(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    return y * __builtin_fma(-x, y * y, 3.0);
}

template <int PREC, bool GEN, bool MASK, bool CUT, bool EN = true>
__device__ __forceinline__ void force_pair(double dx, double dy, double dz, bool self, double ci, double pj,
                                           float cif, float pjf, double &fx, double &fy, double &fz, double &eu,
                                           const PotConst &pc, float Af) {
    if constexpr (PREC == SCMD_FP64) {
        double r2 = __builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz));
        bool off = false;
        if constexpr (CUT) off = !(r2 < pc.rc2);
        if constexpr (MASK) off = off || self;
        if constexpr (MASK || CUT) r2 = off ? kSelfR2 : r2;
        double f, un;
        if constexpr (!GEN) {
            const double w = rsq2_nr(r2);  // 2u
            const double w2 = w * w;
            const double w3 = w2 * w;
            const double w4 = w2 * w2;
            const double w8 = w4 * w4;
            const double q = __builtin_fma(pc.A8, w3, ci) - pj;
            f = w8 * q;   // 2^8 x the force coefficient
            if constexpr (EN) un = w8 * w;  // 2^9 u^n
        } else {
            double x[1] = {r2}, p[1] = {pj}, g[1], e[1];
            float pf[1] = {pjf};
            generic_force<PREC, 1, EN>(x, ci, p, cif, pf, pc, Af, g, e);
            f = g[0];
            if constexpr (EN) un = e[0];
        }
        fx = __builtin_fma(f, dx, fx);
        fy = __builtin_fma(f, dy, fy);
        fz = __builtin_fma(f, dz, fz);
        if constexpr (!EN) {
        } else if constexpr (CUT) {
            eu += off ? 0.0 : un - (GEN ? pc.inv_rc_n : pc.inv_rc_n512);
        } else {
            eu += un;
        }
    } else {
        const double r2d = __builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz));
        bool off = false;
        if constexpr (CUT) off = !(r2d < pc.rc2);
        if constexpr (MASK) off = off || self;
        float r2 = (float)r2d;
        if constexpr (MASK || CUT) r2 = off ? kSelfR2f : r2;
        double fd, un;
        if constexpr (!GEN) {
            float u = __builtin_amdgcn_rsqf(r2);
            float u2 = u * u;
            float u3 = u2 * u;
            float u4 = u2 * u2;
            float u8 = u4 * u4;
            float q = __builtin_fmaf(Af, u3, cif) - pjf;
            fd = (double)(u8 * q);
            if constexpr (EN) un = (double)(u8 * u);
        } else {
            double x[1] = {(double)r2}, p[1] = {pj}, g[1], e[1];
            float pf[1] = {pjf};
            generic_force<PREC, 1, EN>(x, ci, p, cif, pf, pc, Af, g, e);
            fd = g[0];
            if constexpr (EN) un = e[0];
        }
        fx = __builtin_fma(fd, dx, fx);
        fy = __builtin_fma(fd, dy, fy);
        fz = __builtin_fma(fd, dz, fz);
        if constexpr (!EN) {
        } else if constexpr (CUT) {
            eu += off ? 0.0 : un - pc.inv_rc_n;
        } else {
            eu += un;
        }
    }
}

// ---------------------------------------------------------------------------
// The terms of one pair from its r^2 (no mask, no cutoff): what one atom's sum
// and the other's share.
// ---------------------------------------------------------------------------
// u^m.
template <int PREC, bool GEN>
__device__ __forceinline__ double density_term(double r2, const PotConst &pc) {
    if constexpr (GEN) {
        double x[1] = {r2}, t[1];
        generic_density<PREC, 1>(x, pc, t);
        return t[0];
    } else if constexpr (PREC == SCMD_FP64) {
        const double w = rcp_nr(r2);
        return w * w * w;
    } else {
        const float w = __builtin_amdgcn_rcpf((float)r2);
        return (double)(w * w * w);
    }
}

// The density terms of N = 2 or 4 pairs ((n, m) = (9, 6)).  In double one
// reciprocal of the product of the r^2 serves them all, 1/a = (1/ab) b: three
// multiplies per added pair in place of a v_rcp_f64 (16 cycles) and its Newton
// step.  The products round more often, so the step is taken to second order
// (y (1 + e + e^2)), which removes the bias of the first-order one.  us per step,
// one reciprocal per pair / shared: 48,077 atoms 1415 / 1386, 256 clusters 968 /
// 953, 15,000 atoms 172.2 / 167.9, 3001 atoms 23.7 / 23.2; density error against
// 80-bit sums (rms over nine sizes) 3.7e-16 / 2.6e-16.
// A product that leaves the range (a pair at r = 0, four beyond ~1e38 A) makes all
// its terms NaN: sums that are not finite are taken again pair by pair when an atom
// is finished.
template <int PREC, int N>
__device__ __forceinline__ void density_terms(const double (&r2)[N], double (&t)[N], const PotConst &pc) {
    static_assert(N == 2 || N == 4, "pairs or pairs of pairs");
    if constexpr (PREC == SCMD_FP64) {
        const double ab = r2[0] * r2[1], cd = N == 4 ? r2[N - 2] * r2[N - 1] : 1.0;
        const double all = N == 4 ? ab * cd : ab;
        const double y0 = __builtin_amdgcn_rcp(all);
        const double e = __builtin_fma(-all, y0, 1.0);
        const double y = __builtin_fma(y0, __builtin_fma(e, e, e), y0);
        const double yab = N == 4 ? y * cd : y, ycd = y * ab;
        const double w0 = yab * r2[1], w1 = yab * r2[0];
        t[0] = w0 * w0 * w0;
        t[1] = w1 * w1 * w1;
        if constexpr (N == 4) {
            const double w2 = ycd * r2[3], w3 = ycd * r2[2];
            t[2] = w2 * w2 * w2;
            t[3] = w3 * w3 * w3;
        }
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = density_term<PREC, false>(r2[i], pc);
    }
}

// The force coefficient (scaled as in force_pair) and, with EN, u^n.
template <int PREC, bool GEN, bool EN>
__device__ __forceinline__ void force_coef(double r2, double ci, double pj, float cif, float pjf, double &f,
                                           double &un, const PotConst &pc, float Af) {
    if constexpr (GEN) {
        double x[1] = {r2}, p[1] = {pj}, g[1], e[1];
        float pf[1] = {pjf};
        generic_force<PREC, 1, EN>(x, ci, p, cif, pf, pc, Af, g, e);
        f = g[0];
        if constexpr (EN) un = e[0];
    } else if constexpr (PREC == SCMD_FP64) {
        const double w = rsq2_nr(r2);  // 2u
        const double w2 = w * w;
        const double w3 = w2 * w;
        const double w4 = w2 * w2;
        const double w8 = w4 * w4;
        const double q = __builtin_fma(pc.A8, w3, ci) - pj;
        f = w8 * q;
        if constexpr (EN) un = w8 * w;
    } else {
        const float u = __builtin_amdgcn_rsqf((float)r2);
        const float u2 = u * u;
        const float u3 = u2 * u;
        const float u4 = u2 * u2;
        const float u8 = u4 * u4;
        const float q = __builtin_fmaf(Af, u3, cif) - pjf;
        f = (double)(u8 * q);
        if constexpr (EN) un = (double)(u8 * u);
    }
}

// Four partners of one atom, in order (no mask, no cutoff).  General exponents
// take them together, which shares the exponent tests among four pairs and
// gives the power chains four independent values: a 3001-atom evaluation with
// (12, 6) took 20.4 + 44.0 us (density, force sweep) pair by pair.
template <int PREC, bool GEN>
__device__ __forceinline__ void density_quad(const double4 &qi, const double4 (&a)[4], double &acc,
                                             const PotConst &pc) {
    double r2[4], t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double dx = qi.x - a[i].x, dy = qi.y - a[i].y, dz = qi.z - a[i].z;
        r2[i] = __builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz));
    }
    if constexpr (GEN) {
        generic_density<PREC, 4>(r2, pc, t);
    } else {
        density_terms<PREC, 4>(r2, t, pc);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) acc += t[i];
}

template <int PREC, bool GEN, bool EN>
__device__ __forceinline__ void force_quad(const double4 &qi, const double4 (&a)[4], double ci, float cif, double &fx,
                                           double &fy, double &fz, double &eu, const PotConst &pc, float Af) {
    if constexpr (!GEN) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            force_pair<PREC, GEN, false, false, EN>(qi.x - a[i].x, qi.y - a[i].y, qi.z - a[i].z, false, ci, a[i].w, cif,
                                                    (float)a[i].w, fx, fy, fz, eu, pc, Af);
    } else {
        double dx[4], dy[4], dz[4], r2[4], pj[4], f[4], un[4];
        float pjf[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            dx[i] = qi.x - a[i].x;
            dy[i] = qi.y - a[i].y;
            dz[i] = qi.z - a[i].z;
            r2[i] = __builtin_fma(dx[i], dx[i], __builtin_fma(dy[i], dy[i], dz[i] * dz[i]));
            pj[i] = a[i].w;
            pjf[i] = (float)a[i].w;
        }
        generic_force<PREC, 4, EN>(r2, ci, pj, cif, pjf, pc, Af, f, un);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            fx = __builtin_fma(f[i], dx[i], fx);
            fy = __builtin_fma(f[i], dy[i], fy);
            fz = __builtin_fma(f[i], dz[i], fz);
            if constexpr (EN) eu += un[i];
        }
    }
}

// ---------------------------------------------------------------------------
// Workgroup helpers
// ---------------------------------------------------------------------------
// Fixed-shape tree sum over a workgroup of BLOCK threads (deterministic).
// sh needs BLOCK doubles.  Every thread of the workgroup must call it.
template <int BLOCK>
__device__ __forceinline__ double block_sum(double v, double *sh) {
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
#pragma unroll
    for (int s = BLOCK / 2; s > 0; s >>= 1) {
        if (t < s) sh[t] += sh[t + s];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

// Sum of `n` consecutive slots of a partial array (fixed order, loads issued
// ahead of the adds).
__device__ __forceinline__ double sum_slots(const double *__restrict__ p, int n, size_t stride) {
    double s = 0.0;
    int k = 0;
    for (; k + 4 <= n; k += 4) {
        const double a = p[(size_t)k * stride];
        const double b = p[(size_t)(k + 1) * stride];
        const double c = p[(size_t)(k + 2) * stride];
        const double d = p[(size_t)(k + 3) * stride];
        s += a;
        s += b;
        s += c;
        s += d;
    }
    for (; k < n; ++k) s += p[(size_t)k * stride];
    return s;
}

// ---------------------------------------------------------------------------
// Epilogues
// ---------------------------------------------------------------------------
struct DensityOut {
    const double4 *rp;  // positions
    double4 *xp;        // positions + P, read by the force sweep
    double *rho;
    double *tile_sums;
};

// Finish one atom of the density sweep from its complete sum of u^m; q is
// its position.
__device__ __forceinline__ double density_atom_at(int i, double s, const double4 &q, const DensityOut &o,
                                                  const PotConst &pc) {
    const double r = pc.am * s;
    const double sq = sqrt(r);
    const double psi = r > 0.0 ? 1.0 / sq : 0.0;
    o.rho[i] = r;
    o.xp[i] = make_double4(q.x, q.y, q.z, pc.Pscale * psi);
    return -pc.eps_c * sq;  // embedding energy of atom i
}

__device__ __forceinline__ double density_atom(int i, double s, const DensityOut &o, const PotConst &pc) {
    return density_atom_at(i, s, o.rp[i], o, pc);
}

struct ForceOut {
    double4 *f;
    double4 *v;
    double *tile_sums;
    double h;
    int advance;
    // row sweeps of a single cluster whose drift ran inside the density
    // sweep: the force epilogue also applies the thermostat factor st->lambda
    // and the first half-kick, and stores the drifted positions in rp
    int fused;
    const ClusterState *st;
    double4 *rp;
    double2 *dpv;  // drift inputs of the next step (p, v); Langevin: the drifted (r, v)
    double dth;    // dt h
    // bath epilogue of clusters in a Langevin bath: their baths, the run's step index
    const ClusterDesc *cd;
    int local;
    double dt, mass_u;
    int bath;  // clusters in a Langevin bath: 0 none, 1 all, 2 some (read per cluster)
};

struct FinalizeArgs {
    const ClusterDesc *cd;
    ClusterState *st;
    const double *tile_sums;
    int *flag;
    double mass_u, dt;
    int advance;
    int step_add;    // completed steps since st.step was last stored (ramp index = st.step + step_add)
    int store_step;  // 1: store st.step + step_add
};

// Finish one atom of the force sweep: store F and the site pair energy,
// second half-kick when advancing; returns (pair energy, v^2) through refs.
// vi is the atom's current velocity.
__device__ __forceinline__ void force_atom_v(int i, double fx, double fy, double fz, double eu, double4 vi,
                                             const ForceOut &o, const PotConst &pc, double &epair, double &v2) {
#pragma clang fp contract(off)
    const double ei = pc.half_eps_an * eu;
    o.f[i] = make_double4(fx, fy, fz, ei);
    if (o.advance) {
        vi.x = vi.x + o.h * fx;
        vi.y = vi.y + o.h * fy;
        vi.z = vi.z + o.h * fz;
        o.v[i] = vi;
    }
    epair += ei;
    v2 += vi.x * vi.x + vi.y * vi.y + vi.z * vi.z;
}

__device__ __forceinline__ void force_atom(int i, double fx, double fy, double fz, double eu, const ForceOut &o,
                                           const PotConst &pc, double &epair, double &v2) {
    force_atom_v(i, fx, fy, fz, eu, o.v[i], o, pc, epair, v2);
}

// Kinetic energy (eV) and temperature of a cluster from its sum of v^2.
struct KinT {
    double ke, T;
};
__device__ __forceinline__ KinT kinetic_temperature(const ClusterDesc &d, double mass_u, double v2) {
#pragma clang fp contract(off)
    const double ke = 0.5 * mass_u * v2 * kEvPerUA2Fs2;
    const double T = d.ndof > 0 ? 2.0 * ke / ((double)d.ndof * kBoltzmannEv) : 0.0;
    return KinT{ke, T};
}

// Thermostat factor after a step whose ramp index is step_now, at
// temperature T; *ttarget receives the target (0 without thermostat).  The
// Langevin bath acts inside the drift: its factor is 1.
__device__ __forceinline__ double thermostat_lambda(const ClusterDesc &d, double dt, double T, int64_t step_now,
                                                    double *ttarget) {
#pragma clang fp contract(off)
    double lam = 1.0;
    *ttarget = 0.0;
    if (d.kind == SCMD_LANGEVIN) *ttarget = ramp_target(d, step_now);
    if (d.kind == SCMD_BERENDSEN) {
        const double tt = ramp_target(d, step_now);
        *ttarget = tt;
        if (T > 0.0) {
            const double x = 1.0 + (dt / d.tau) * (tt / T - 1.0);
            lam = x > 0.0 ? sqrt(x) : 0.0;
        }
    }
    return lam;
}

// Fixed-order totals of a cluster's tile sums: threads 0..255 add every
// 256th tile, each of the four wavefronts folds its lanes with wave_total,
// and the four wavefront sums are added as (w0 + w1) + (w2 + w3).  Any
// workgroup of >= 256 threads gets the same bits; every thread must call it.
// sh needs 12 doubles.  With V2_ONLY only the v^2 column is read (the others
// come back as 0).
// Sum of a double over the 64 lanes of a fully active wavefront with DPP
// moves, in one fixed order: pairs and quads (quad_perm), 8 and 16 lanes
// (row_half_mirror, row_mirror), then the four rows of 16 (row_bcast15 into
// rows 1 and 3, row_bcast31 into rows 2 and 3); lane 63 ends with
// (r0 + r1) + (r2 + r3) and its value is returned to every lane.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add_src(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xF, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_total(double x) {
    x += dpp_add_src<0xB1, 0xF>(x);
    x += dpp_add_src<0x4E, 0xF>(x);
    x += dpp_add_src<0x141, 0xF>(x);
    x += dpp_add_src<0x140, 0xF>(x);
    x += dpp_add_src<0x142, 0xA>(x);
    x += dpp_add_src<0x143, 0xC>(x);
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), 63);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), 63);
    return __hiloint2double(hi, lo);
}

constexpr int kTotBlock = 256;
template <bool V2_ONLY>
__device__ __forceinline__ void cluster_totals(const ClusterDesc &d, const double *tile_sums, double *sh,
                                               double &emb, double &epair, double &v2) {
    emb = epair = v2 = 0.0;
    const int t = threadIdx.x;
    if (t < kTotBlock) {
        // thread t adds slots t, t + kTotBlock, ... in that order; the loads
        // of kTotU of them are issued together (the cell list has thousands
        // of slots per cluster)
        constexpr int kTotU = 8;
        for (int k0 = t; k0 < d.ntiles; k0 += kTotU * kTotBlock) {
            double e[kTotU], p[kTotU], w[kTotU];
#pragma unroll
            for (int u = 0; u < kTotU; ++u) {
                const int k = k0 + u * kTotBlock;
                e[u] = p[u] = w[u] = 0.0;
                if (k < d.ntiles) {
                    const double *ts = tile_sums + (size_t)(d.tile0 + k) * kTileSums;
                    if constexpr (!V2_ONLY) {
                        e[u] = ts[0];
                        p[u] = ts[1];
                    }
                    w[u] = ts[2];
                }
            }
#pragma unroll
            for (int u = 0; u < kTotU; ++u) {
                if (k0 + u * kTotBlock < d.ntiles) {
                    if constexpr (!V2_ONLY) {
                        emb += e[u];
                        epair += p[u];
                    }
                    v2 += w[u];
                }
            }
        }
    }
    if constexpr (!V2_ONLY) {
        emb = wave_total(emb);
        epair = wave_total(epair);
    }
    v2 = wave_total(v2);
    if (t < kTotBlock && (t & 63) == 0) {
        const int w = t >> 6;
        sh[w] = emb;
        sh[4 + w] = epair;
        sh[8 + w] = v2;
    }
    __syncthreads();
    emb = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    epair = (sh[4] + sh[5]) + (sh[6] + sh[7]);
    v2 = (sh[8] + sh[9]) + (sh[10] + sh[11]);
    __syncthreads();
}

// The non-finite flag sits in host memory: a plain store, visible to the host
// once the stream is synchronised.
__device__ __forceinline__ void raise_flag(int *flag) {
    __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Per-cluster finish, run by one whole workgroup (>= 256 threads): the
// totals of the tile sums, then temperature and the Berendsen factor.  Every
// workgroup that runs it for the same cluster and arguments gets the same
// result bit for bit; only a `writer` stores the cluster state (st.step only
// with store_step).  Returns the cluster's current thermostat factor to
// thread 0.  sh needs 12 doubles.
__device__ inline double cluster_finalize(int c, const FinalizeArgs &o, double *sh, bool writer) {
    // no contraction: the same rounding in every kernel that inlines this
#pragma clang fp contract(off)
    const ClusterDesc d = o.cd[c];
    double emb, epair, v2;
    cluster_totals<false>(d, o.tile_sums, sh, emb, epair, v2);
    if (threadIdx.x != 0) return 1.0;
    ClusterState s = o.st[c];
    const KinT kt = kinetic_temperature(d, o.mass_u, v2);
    double lam = s.lambda;
    const int64_t step_now = s.step + o.step_add;
    if (o.store_step) s.step = step_now;
    if (o.advance) {
        lam = thermostat_lambda(d, o.dt, kt.T, step_now, &s.ttarget);
        s.lambda = lam;
    }
    s.epot = emb + epair;
    s.ekin = lam * lam * kt.ke;
    s.temp = lam * lam * kt.T;
    if (!isfinite(s.epot) || !isfinite(s.ekin)) {
        s.nonfinite = 1;
        if (writer) raise_flag(o.flag);
    }
    if (writer) o.st[c] = s;
    return s.lambda;
}

// ---------------------------------------------------------------------------
// Drift folded into a density sweep, and the matching force epilogues (row and
// split symmetric sweeps; see Drift in scmd_internal.h)
// ---------------------------------------------------------------------------
struct DriftArgs {
    int mode, local;
    int bath;  // clusters in a Langevin bath: 0 none, 1 all, 2 some (read per cluster)
    const double4 *v, *f;
    const double2 *dpv;
    ClusterState *st;
    const double *tile_sums;
    const ClusterDesc *cd;
    double mass_u, dt, h, dth;
    int *flag;  // non-finite flag
};

// Drifted position p + (dt lambda) v with p = r + (dt h) F (Drift).
// Mode 1 reads r, v, F (x, y, z) and forms p; mode 2 reads p, v from the
// three pairs (px, py), (pz, vx), (vy, vz) stored per atom.
struct PV {
    double px, py, pz, vx, vy, vz;
};
__device__ __forceinline__ double4 xyz(const double4 *__restrict__ p, int a) {
    const double *q = reinterpret_cast<const double *>(p + a);
    return make_double4(q[0], q[1], q[2], 0.0);
}
__device__ __forceinline__ double pcomp(double r, double f, double dth) {
#pragma clang fp contract(off)
    return r + dth * f;
}
__device__ __forceinline__ PV pv_from_rvf(const double4 *__restrict__ r, const double4 *__restrict__ v,
                                          const double4 *__restrict__ f, int a, double dth) {
    const double4 ra = xyz(r, a), va = xyz(v, a), fa = xyz(f, a);
    return PV{pcomp(ra.x, fa.x, dth), pcomp(ra.y, fa.y, dth), pcomp(ra.z, fa.z, dth), va.x, va.y, va.z};
}
__device__ __forceinline__ PV pv_load(const double2 *__restrict__ d, int a) {
    const double2 q0 = d[3 * a], q1 = d[3 * a + 1], q2 = d[3 * a + 2];
    return PV{q0.x, q0.y, q1.x, q1.y, q2.x, q2.y};
}
__device__ __forceinline__ double4 drifted(const PV &q, double dtl) {
#pragma clang fp contract(off)
    return make_double4(q.px + dtl * q.vx, q.py + dtl * q.vy, q.pz + dtl * q.vz, 0.0);
}

// Whether cluster c of a launch that drifts is in a Langevin bath.
__device__ __forceinline__ bool in_bath(int c, const DriftArgs &da) {
    return da.bath == 1 || (da.bath == 2 && da.cd[c].kind == SCMD_LANGEVIN);
}

// The thermostat factor of cluster c for a drift (mode 1: as stored; mode 2:
// the previous step's factor, finished here from the cluster's v^2 tile sums in
// the finalize's order, and stored by the one workgroup with `writer`).  A
// cluster in a Langevin bath has its drifted (r, v) stored already: factor 0
// (the row sweeps take p + 0 v = p).  REPORT: the writer reports a kinetic energy
// that is not finite, which the factor may hide from the run's last step (the row
// sweeps and resident runs look at their last step only).  Whole workgroups of
// >= 256 threads; sh needs 12 doubles.
template <bool REPORT>
__device__ __forceinline__ double drift_factor(int c, const DriftArgs &da, bool bath, double *sh, bool writer) {
    if (bath) return 0.0;
    ClusterState *sc = da.st + c;
    if (da.mode != 2) return sc->lambda;
    const ClusterDesc d = da.cd[c];
    double e0, e1, v2;
    cluster_totals<true>(d, da.tile_sums, sh, e0, e1, v2);
    const KinT kt = kinetic_temperature(d, da.mass_u, v2);
    double tt;
    const double lam = thermostat_lambda(d, da.dt, kt.T, sc->step + da.local, &tt);
    if (writer && threadIdx.x == 0) {
        sc->lambda = lam;
        if (REPORT && !isfinite(kt.ke)) raise_flag(da.flag);
    }
    return lam;
}

// Drifted position of atom i (indices into the context's arrays) in the
// symmetric sweeps: r + dt (lambda v + h F) in the drift kernel's order, or in
// a bath the drifted r stored with dpv.  The row sweeps' p + (dt lambda) v
// form saves a third of the bytes where every workgroup loads every atom, but
// rounds twice at the size of r; here each item loads few atoms.
__device__ __forceinline__ double4 drifted_atom(const double4 *__restrict__ rp, int i, const DriftArgs &da, bool bath,
                                                double lam) {
#pragma clang fp contract(off)
    if (bath) {
        const double2 q0 = da.dpv[3 * (size_t)i], q1 = da.dpv[3 * (size_t)i + 1];
        return make_double4(q0.x, q0.y, q1.x, 0.0);
    }
    const double4 r = xyz(rp, i), v = xyz(da.v, i), f = xyz(da.f, i);
    const double vx = lam * v.x + da.h * f.x, vy = lam * v.y + da.h * f.y, vz = lam * v.z + da.h * f.z;
    return make_double4(r.x + da.dt * vx, r.y + da.dt * vy, r.z + da.dt * vz, 0.0);
}

// Force epilogue of a step whose drift ran inside the density sweep: the
// velocity gets the thermostat factor and the first half-kick with the old
// force (as in the drift kernel), then the second half-kick with the new one;
// the drifted position r (x, y, z of the density output) is stored.
template <bool STORE_PV>
__device__ __forceinline__ void force_atom_fused(int i, double fx, double fy, double fz, double eu, const double4 &r,
                                                 const double4 &v_old, const double4 &f_old, double lam,
                                                 const ForceOut &o, const PotConst &pc, double &epair, double &v2) {
#pragma clang fp contract(off)
    const double ei = pc.half_eps_an * eu;
    const double4 fo = f_old;
    double4 vi = v_old;
    vi.x = lam * vi.x;
    vi.y = lam * vi.y;
    vi.z = lam * vi.z;
    vi.x = vi.x + o.h * fo.x;
    vi.y = vi.y + o.h * fo.y;
    vi.z = vi.z + o.h * fo.z;
    o.f[i] = make_double4(fx, fy, fz, ei);
    vi.x = vi.x + o.h * fx;
    vi.y = vi.y + o.h * fy;
    vi.z = vi.z + o.h * fz;
    o.v[i] = vi;
    o.rp[i] = make_double4(r.x, r.y, r.z, 0.0);
    if constexpr (STORE_PV) {  // drift inputs of the next step: p = r + (dt h) F, v
        double2 *d = o.dpv + 3 * (size_t)i;
        d[0] = make_double2(r.x + o.dth * fx, r.y + o.dth * fy);
        d[1] = make_double2(r.z + o.dth * fz, vi.x);
        d[2] = make_double2(vi.y, vi.z);
    }
    epair += ei;
    v2 += vi.x * vi.x + vi.y * vi.y + vi.z * vi.z;
}

// Langevin epilogue (a cluster in a bath): the stored post-bath velocity gets
// the second half-kick; then the first half-kick of the next step with the
// same force and that step's A, O, A (bath.h), whose drifted (r, v) are
// stored for the next density sweep.  The order of operations is the same as
// in the drift kernel.
__device__ __forceinline__ void force_atom_bath(int i, double fx, double fy, double fz, double eu, const double4 &r,
                                                const double4 &v_bath, const double3 &xi_next, double c2_next,
                                                const ClusterDesc &d, const ForceOut &o, const PotConst &pc,
                                                double &epair, double &v2) {
#pragma clang fp contract(off)
    const double ei = pc.half_eps_an * eu;
    double4 vi = v_bath;
    vi.x = vi.x + o.h * fx;
    vi.y = vi.y + o.h * fy;
    vi.z = vi.z + o.h * fz;
    o.f[i] = make_double4(fx, fy, fz, ei);
    o.v[i] = vi;
    o.rp[i] = make_double4(r.x, r.y, r.z, 0.0);
    epair += ei;
    v2 += vi.x * vi.x + vi.y * vi.y + vi.z * vi.z;
    double4 rn = make_double4(r.x, r.y, r.z, 0.0);
    vi.x = vi.x + o.h * fx;
    vi.y = vi.y + o.h * fy;
    vi.z = vi.z + o.h * fz;
    // this is step st->step + local + 1 of the cluster; prepare the next one
    bath_drift_xi(d, c2_next, xi_next, o.dt, rn, vi);
    double2 *q = o.dpv + 3 * (size_t)i;
    q[0] = make_double2(rn.x, rn.y);
    q[1] = make_double2(rn.z, vi.x);
    q[2] = make_double2(vi.y, vi.z);
}

// What the force epilogues read of their own atom before its sums are known:
// position and velocity (bath: the post-bath velocity stored with the drifted
// position), the old force, and in a bath the noise and its amplitude of the
// next step.
struct FusedAtom {
    double4 r, v, f;
    double3 xi;
    double c2;
};
__device__ __forceinline__ FusedAtom fused_atom_load(int i, int c, bool bath, const double4 *__restrict__ xp,
                                                     const ForceOut &o) {
    FusedAtom a;
    a.r = a.v = a.f = make_double4(0, 0, 0, 0);
    a.xi = make_double3(0.0, 0.0, 0.0);
    a.c2 = 0.0;
    if (o.fused) a.r = xp[i];
    if (bath) {
        const double2 *q = o.dpv + 3 * (size_t)i;
        const double2 q1 = q[1], q2 = q[2];
        a.v = make_double4(q1.y, q2.x, q2.y, 0.0);
        const int64_t next = o.st[c].step + o.local + 2;
        a.xi = bath_noise(o.cd[c].seed, next, i - o.cd[c].off);
        a.c2 = bath_c2(o.cd[c], next, o.mass_u);
    } else {
        a.v = o.v[i];
        if (o.fused) a.f = o.f[i];
    }
    return a;
}

// Host: the arguments of the folded drift and of the force epilogues.
inline DriftArgs drift_args(const SweepBuffers &B, const StepArgs &a, const Drift &dr) {
    return DriftArgs{dr.mode, dr.local, dr.bath, B.v, B.f,  B.dpv,      a.st,
                     B.tile_sums, a.cd, a.mass_u, a.dt, a.h, a.dt * a.h, a.flag};
}
// (the fused epilogue stores the drifted positions: rp is the context's
// writable position array, which the sweeps otherwise only read)
inline ForceOut fused_force_out(const SweepBuffers &B, const StepArgs &a, int fused, int local, int bath) {
    return ForceOut{B.f,   B.v,        B.tile_sums, a.h,   a.advance, fused,    a.st, const_cast<double4 *>(B.rp),
                    B.dpv, a.dt * a.h, a.cd,        local, a.dt,      a.mass_u, bath};
}

// ---------------------------------------------------------------------------
// Cell-list check (see CellCheck): per atom, then merged per workgroup.
// ---------------------------------------------------------------------------
// Doubles compared as signed 64-bit integers: flip the magnitude bits of
// negative values (an involution, so the same map decodes).
__device__ __forceinline__ long long ord_encode(double d) {
    const long long b = __double_as_longlong(d);
    return b >= 0 ? b : b ^ 0x7FFFFFFFFFFFFFFFLL;
}
__device__ __forceinline__ double ord_decode(long long b) {
    return __longlong_as_double(b >= 0 ? b : b ^ 0x7FFFFFFFFFFFFFFFLL);
}

struct CellBox {
    double m[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    bool moved = false;
};

__device__ __forceinline__ void cell_check_atom(const CellCheck &cc, int i, const double4 &q, CellBox &b) {
    const double4 o = cc.ref[i];
    const double ex = q.x - o.x, ey = q.y - o.y, ez = q.z - o.z;
    b.moved = b.moved || !(ex * ex + ey * ey + ez * ez <= cc.thr2);
    cc.rs[cc.slot_of[i]] = q;
    b.m[0] = fmin(b.m[0], q.x);
    b.m[1] = fmin(b.m[1], q.y);
    b.m[2] = fmin(b.m[2], q.z);
    b.m[3] = fmax(b.m[3], q.x);
    b.m[4] = fmax(b.m[4], q.y);
    b.m[5] = fmax(b.m[5], q.z);
}

// Every thread of the workgroup (BLOCK threads) calls this once with its
// accumulated box; min/max are exact, so neither the reduction order nor
// the atomic merge order matters.  sh: 6 x BLOCK/64 doubles.
template <int BLOCK>
__device__ __forceinline__ void cell_check_merge(const CellCheck &cc, int cluster, CellBox &b, double *sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            b.m[d] = fmin(b.m[d], __shfl_xor(b.m[d], o, 64));
            b.m[3 + d] = fmax(b.m[3 + d], __shfl_xor(b.m[3 + d], o, 64));
        }
    }
    if (__ballot(b.moved) != 0ull && lane == 0) atomicOr(cc.flag, 1);
    if (lane == 0)
        for (int d = 0; d < 6; ++d) sh[d * (BLOCK / 64) + w] = b.m[d];
    __syncthreads();
    if (threadIdx.x < 6) {
        const int d = threadIdx.x;
        double v = sh[d * (BLOCK / 64)];
        for (int k = 1; k < BLOCK / 64; ++k)
            v = d < 3 ? fmin(v, sh[d * (BLOCK / 64) + k]) : fmax(v, sh[d * (BLOCK / 64) + k]);
        if (d < 3) atomicMin(&cc.box[6 * cluster + d], ord_encode(v));
        else atomicMax(&cc.box[6 * cluster + d], ord_encode(v));
    }
}

}  // namespace dev
}  // namespace scmd
