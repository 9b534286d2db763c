// Resident runs of small clusters: one workgroup per cluster advances it by
// any number of steps in one launch, the cluster held in registers and LDS.
//
// A step of a small cluster on the row sweeps is two launches that each last
// little longer than an empty one (Ni147: 9.6 us, a 3.3 us floor per launch):
// nothing is gained by spreading 10,731 pairs over 256 CUs.  Here one CU does all of
// them and a barrier takes the place of a launch.  That CU's FP64 rate is then the
// bound, so every unordered pair is evaluated once: S neighbouring lanes work for
// atom i; lane s meets the atoms i + k (mod n) of the offsets k = 1 + s, 1 + s + S,
// ... <= (n - 1) / 2, adds the term to its own sum and leaves it in LDS for the other
// (row k, its atom), and after a barrier it collects what the pairs (i - k, i) left.
// For even n the offset n / 2 meets every pair from both ends.  Positions are stored
// twice in a row, so i + k never wraps; the S lanes add their sums with DPP and all
// of them carry the atom's state.  Everything is in a fixed order: results do not
// depend on how a run is cut into launches, nor on evaluations between its calls,
// which run here too.  kResidentMax gives the times.
//
// The scheme is the paper's (Sec. 2 "Computational approach": the densities of
// Eq. (rho), then the forces of Eq. (SC), velocity-Verlet or the Langevin bath).
#include "sweep_common.h"

namespace scmd {
namespace {

using namespace dev;

constexpr int kResBlock = 768;           // 12 wavefronts; four per SIMD fit (128 VGPRs), so small clusters share a CU
constexpr int kResPlane = 2 * kResidentMax;  // entries of a position plane

struct ResidentArgs {
    const ClusterDesc *cd;
    ClusterState *st;
    int *flag;
    double4 *rp, *v, *f;
    double *rho;
    double mass_u, dt, h;
    int nsteps;  // 0: evaluate only
};

// Lanes per atom: as many as the block holds, up to the 16 of a DPP row.
constexpr int resident_lanes(int n) { return n > 96 ? 4 : n > 48 ? 8 : 16; }
static_assert(kResidentMax * resident_lanes(kResidentMax) <= kResBlock && 96 * 8 <= kResBlock && 48 * 16 <= kResBlock,
              "the lanes of the largest cluster of each width fill at most a block");
// Fixed part of the LDS in doubles: two planes of double2, noise, its amplitude
// (padded) and the wavefront sums.
constexpr int kResNoise = 4 * kResPlane, kResAmp = kResNoise + 3 * kResidentMax, kResSums = kResAmp + 2,
              kResTerms = kResSums + 3 * (kResBlock / 64);
// Pair terms left for the other atom: (n - 1) / 2 offsets of n atoms.
__host__ __device__ constexpr int resident_terms(int n) { return n > 1 ? (n - 1) / 2 * n : 0; }
constexpr int resident_lds(int n) { return (kResTerms + resident_terms(n)) * (int)sizeof(double); }

// Sum over the S lanes of an atom, in every one of them.
template <int S>
__device__ __forceinline__ double lane_sum(double x) {
    x += dpp_add_src<0xB1, 0xF>(x);
    x += dpp_add_src<0x4E, 0xF>(x);
    if constexpr (S >= 8) x += dpp_add_src<0x141, 0xF>(x);
    if constexpr (S >= 16) x += dpp_add_src<0x140, 0xF>(x);
    return x;
}

// Density sum of atom i over the lane's pairs; every thread of the workgroup
// (one barrier inside).
template <int PREC, bool GEN, int S>
__device__ __forceinline__ double resident_density(int n, int i, int s, const double2 *xy, double *terms,
                                                   const PotConst &pc) {
    const double2 *zp = xy + kResPlane;
    const int K = (n - 1) / 2;
    const double2 p0 = xy[i];
    const double pz = zp[i].x;
    double acc = 0.0;
    auto term = [&](int j) {
        const double2 q0 = xy[j];
        const double dx = p0.x - q0.x, dy = p0.y - q0.y, dz = pz - zp[j].x;
        return density_term<PREC, GEN>(__builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz)), pc);
    };
    double *row = terms + s * n;
    {
        // two offsets at a time, their terms stored after both are known: a
        // store between them would hold the second's loads back.  j mod n is
        // the smaller of j and j - n as unsigned numbers.
        double *out = row;
        int j = i + 1 + s, k = 1 + s;
        for (; k + S <= K; k += 2 * S, j += 2 * S, out += 2 * S * n) {
            const double u = term(j), w = term(j + S);
            acc += u;
            acc += w;
            out[min((unsigned)j, (unsigned)(j - n))] = u;
            out[S * n + min((unsigned)(j + S), (unsigned)(j + S - n))] = w;
        }
        if (k <= K) {
            const double u = term(j);
            acc += u;
            out[min((unsigned)j, (unsigned)(j - n))] = u;
        }
        if ((n & 1) == 0 && s == 0) acc += term(i + n / 2);
    }
    __syncthreads();
    const double *in = row + i;
#pragma unroll 4
    for (int k = 1 + s; k <= K; k += S, in += S * n) acc += *in;
    return lane_sum<S>(acc);
}

// Force (and, with EN, 2^9 u^n) sums of atom i; one barrier inside.
template <int PREC, bool GEN, bool EN, int S>
__device__ __forceinline__ void resident_force(int n, int i, int s, const double2 *xy, double *terms,
                                               const PotConst &pc, double (&a)[4]) {
    const double2 *zp = xy + kResPlane;
    const float Af = (float)pc.A;
    const int K = (n - 1) / 2;
    const double2 p0 = xy[i], p1 = zp[i];
    const double ci = -p1.y;
    const float cif = (float)ci;
    a[0] = a[1] = a[2] = a[3] = 0.0;
    auto pair = [&](const double2 &q0, const double2 &q1, double weight) {
        const double dx = p0.x - q0.x, dy = p0.y - q0.y, dz = p1.x - q1.x;
        double c, un;
        force_coef<PREC, GEN, EN>(__builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz)), ci, q1.y, cif, (float)q1.y, c,
                                  un, pc, Af);
        a[0] = __builtin_fma(c, dx, a[0]);
        a[1] = __builtin_fma(c, dy, a[1]);
        a[2] = __builtin_fma(c, dz, a[2]);
        if constexpr (EN) a[3] += weight * un;
        // single precision subtracts P_i, then P_j: the other atom's own
        // rounding, as the one-sided sweeps have it
        if constexpr (PREC != SCMD_FP64)
            force_coef<PREC, GEN, false>(__builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz)), -q1.y, p1.y,
                                         -(float)q1.y, -cif, c, un, pc, Af);
        return c;
    };
    double *row = terms + s * n;
    {
        double *out = row;
        int j = i + 1 + s, k = 1 + s;
        for (; k + S <= K; k += 2 * S, j += 2 * S, out += 2 * S * n) {
            const double2 q0 = xy[j], q1 = zp[j], q2 = xy[j + S], q3 = zp[j + S];
            const double c0 = pair(q0, q1, 2.0), c1 = pair(q2, q3, 2.0);
            out[min((unsigned)j, (unsigned)(j - n))] = c0;
            out[S * n + min((unsigned)(j + S), (unsigned)(j + S - n))] = c1;
        }
        if (k <= K) out[min((unsigned)j, (unsigned)(j - n))] = pair(xy[j], zp[j], 2.0);
        if ((n & 1) == 0 && s == 0) pair(xy[i + n / 2], zp[i + n / 2], 1.0);
    }
    __syncthreads();
    const double *in = row + i;
    const double2 *q = xy + (i + n - 1 - s);  // the atom i - k, in the second copy
#pragma unroll 2
    for (int k = 1 + s; k <= K; k += S, q -= S, in += S * n) {
        const double c = *in;
        a[0] = __builtin_fma(c, p0.x - q->x, a[0]);
        a[1] = __builtin_fma(c, p0.y - q->y, a[1]);
        a[2] = __builtin_fma(c, p1.x - q[kResPlane].x, a[2]);
    }
#pragma unroll
    for (int w = 0; w < (EN ? 4 : 3); ++w) a[w] = lane_sum<S>(a[w]);
    unscale_force<PREC, GEN>(a[0], a[1], a[2], a[3]);
}

template <int PREC, bool GEN, int S>
__global__ __launch_bounds__(kResBlock, 4) void k_resident(ResidentArgs o, PotConst pc) {
    extern __shared__ double2 lds_res[];
    const int c = blockIdx.x;
    const ClusterDesc d = o.cd[c];
    const int n = d.n, t = threadIdx.x, lane = t & 63, wave = t >> 6, waves = blockDim.x >> 6;
    double2 *const xy = lds_res, *const zp = xy + kResPlane;
    double *const lds = reinterpret_cast<double *>(lds_res);
    double *const noise = lds + kResNoise, *const amp = lds + kResAmp, *const wsum = lds + kResSums;
    double *const terms = lds + kResTerms;
    const bool bath = d.kind == SCMD_LANGEVIN;
    // lane s of atom i; threads past the atoms idle: they follow atom 0 from
    // past the last offset and own nothing
    const bool active = t / S < n;
    const int i = active ? t / S : 0, s = active ? t % S : n;
    const bool owner = active && s == 0;
    const int a = d.off + i;
    double4 r = make_double4(0, 0, 0, 0), v = r, f = r;
    double rho = 0.0, emb = 0.0, epair = 0.0, v2 = 0.0;
    if (active) {
        r = o.rp[a];
        v = o.v[a];
        f = o.f[a];
    }
    const int64_t step0 = o.st[c].step;
    double lam = o.st[c].lambda;
    // the bath's noise is drawn a step ahead, one atom per thread, by the last
    // wavefronts (the idle threads are among them)
    const int drawer = t - (int)(blockDim.x - ((n + 63) & ~63));
    auto draw = [&](int64_t step) {
        if (bath && drawer >= 0 && drawer < n) {
            const double3 xi = bath_noise(d.seed, step, drawer);
            noise[3 * drawer] = xi.x;
            noise[3 * drawer + 1] = xi.y;
            noise[3 * drawer + 2] = xi.z;
            if (drawer == 0) *amp = bath_c2(d, step, o.mass_u);
        }
    };
    // sums over the owners, in wavefront order, for every thread after a barrier
    auto total = [&](double x, int slot) {
        x = wave_total(owner ? x : 0.0);
        if (lane == 0) wsum[slot * (kResBlock / 64) + wave] = x;
    };
    auto gathered = [&](int slot) {
        double x = wsum[slot * (kResBlock / 64)];
        for (int w = 1; w < waves; ++w) x += wsum[slot * (kResBlock / 64) + w];
        return x;
    };
    if (o.nsteps > 0) draw(step0 + 1);
    __syncthreads();
    for (int k = o.nsteps > 0 ? 1 : 0; k <= o.nsteps; ++k) {
        const bool last = k == o.nsteps;
        {
#pragma clang fp contract(off)
            if (k > 0) {  // pending thermostat factor, first half-kick, move
                v.x = lam * v.x;
                v.y = lam * v.y;
                v.z = lam * v.z;
                v.x = v.x + o.h * f.x;
                v.y = v.y + o.h * f.y;
                v.z = v.z + o.h * f.z;
                if (bath) {
                    bath_drift_xi(d, *amp, make_double3(noise[3 * i], noise[3 * i + 1], noise[3 * i + 2]), o.dt, r, v);
                } else {
                    r.x = r.x + o.dt * v.x;
                    r.y = r.y + o.dt * v.y;
                    r.z = r.z + o.dt * v.z;
                }
            }
            if (owner) {
                xy[i] = xy[i + n] = make_double2(r.x, r.y);
                zp[i] = zp[i + n] = make_double2(r.z, 0.0);
            }
        }
        __syncthreads();
        if (!last) draw(step0 + k + 1);
        rho = pc.am * resident_density<PREC, GEN, S>(n, i, s, xy, terms, pc);
        {
            const double sq = sqrt(rho);
            const double psi = rho > 0.0 ? 1.0 / sq : 0.0;
            emb = -pc.eps_c * sq;
            if (owner) zp[i].y = zp[i + n].y = pc.Pscale * psi;
        }
        __syncthreads();
        // the pair energy only on the run's last step
        double g[4];
        if (last)
            resident_force<PREC, GEN, true, S>(n, i, s, xy, terms, pc, g);
        else
            resident_force<PREC, GEN, false, S>(n, i, s, xy, terms, pc, g);
        {
#pragma clang fp contract(off)
            epair = pc.half_eps_an * g[3];
            f = make_double4(g[0], g[1], g[2], epair);
            if (k > 0) {
                v.x = v.x + o.h * f.x;
                v.y = v.y + o.h * f.y;
                v.z = v.z + o.h * f.z;
            }
            v2 = v.x * v.x + v.y * v.y + v.z * v.z;
        }
        if (!last) {
            lam = 1.0;
            if (d.kind == SCMD_BERENDSEN) total(v2, 2);
            __syncthreads();  // also: every wavefront is done with the positions
            if (d.kind == SCMD_BERENDSEN) {
                double tt;
                lam = thermostat_lambda(d, o.dt, kinetic_temperature(d, o.mass_u, gathered(2)).T, step0 + k, &tt);
            }
        }
    }
    if (owner) {
        o.rp[a] = r;
        o.v[a] = v;
        o.f[a] = f;
        o.rho[a] = rho;
    }
    total(emb, 0);
    total(epair, 1);
    total(v2, 2);
    __syncthreads();
    if (t == 0) {  // as the per-cluster finalize
#pragma clang fp contract(off)
        ClusterState q = o.st[c];
        const KinT kt = kinetic_temperature(d, o.mass_u, gathered(2));
        if (o.nsteps > 0) {
            q.step = step0 + o.nsteps;
            q.lambda = thermostat_lambda(d, o.dt, kt.T, q.step, &q.ttarget);
        }
        q.epot = gathered(0) + gathered(1);
        q.ekin = q.lambda * q.lambda * kt.ke;
        q.temp = q.lambda * q.lambda * kt.T;
        if (!isfinite(q.epot) || !isfinite(q.ekin)) {
            q.nonfinite = 1;
            raise_flag(o.flag);
        }
        o.st[c] = q;
    }
}

template <int PREC, bool GEN, int S>
hipError_t launch_s(const ResidentArgs &o, int nclusters, int nmax, const PotConst &pc, hipStream_t s) {
    const int bytes = resident_lds(nmax);
    hipError_t e = allow_lds(k_resident<PREC, GEN, S>, bytes, resident_lds(kResidentMax));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_resident<PREC, GEN, S>), dim3(nclusters), dim3((nmax * S + 63) / 64 * 64), bytes, s, o, pc);
    return hipGetLastError();
}

template <int PREC, bool GEN>
hipError_t launch(const ResidentArgs &o, int nclusters, int nmax, const PotConst &pc, hipStream_t s) {
    switch (resident_lanes(nmax)) {
        case 4: return launch_s<PREC, GEN, 4>(o, nclusters, nmax, pc, s);
        case 8: return launch_s<PREC, GEN, 8>(o, nclusters, nmax, pc, s);
        default: return launch_s<PREC, GEN, 16>(o, nclusters, nmax, pc, s);
    }
}

}  // namespace

static_assert(resident_lds(kResidentMax) <= 160 * 1024, "a resident cluster fills the LDS of a CU");

hipError_t launch_resident(const SweepBuffers &B, const StepArgs &a, int nclusters, int nmax, int nsteps,
                           const PotConst &pc, int precision, hipStream_t s) {
    if (nmax < 1 || nmax > kResidentMax || pc.cut) return hipErrorInvalidValue;
    (void)hipGetLastError();
    const ResidentArgs o{a.cd, a.st, a.flag, const_cast<double4 *>(B.rp), B.v, B.f, B.rho, a.mass_u, a.dt, a.h, nsteps};
    if (precision == SCMD_FP64)
        return pc.generic ? launch<SCMD_FP64, true>(o, nclusters, nmax, pc, s)
                          : launch<SCMD_FP64, false>(o, nclusters, nmax, pc, s);
    return pc.generic ? launch<SCMD_MIXED, true>(o, nclusters, nmax, pc, s)
                      : launch<SCMD_MIXED, false>(o, nclusters, nmax, pc, s);
}

}  // namespace scmd
