// Symmetric (Newton's third law) all-pairs sweeps for large clusters.
//
// Both sweeps of the paper's scheme (Sec. 2.1 Eqs. (SC), (rho); Sec. 2
// "Computational approach") are symmetric in i and j: (a/r_ij)^m enters
// rho_i and rho_j alike, and the force term of a pair acts with opposite
// signs on i and j.  Here every unordered pair is evaluated once.
//
// Atoms of a cluster are cut into 64-atom tiles; IPT consecutive tiles form
// a group that sits in one wavefront (lane l owns atom l of each of the
// group's tiles).  A work item is one group against a run of later tiles:
// each j tile is loaded one atom per lane and then rotated through the
// wavefront with DPP wave_ror:1 64 times, so that every lane meets every j
// atom; the j tile carries its own force (or density) accumulators along.
// Pairs inside a group are done by a separate diagonal item, in which the
// group's own tiles rotate past it the same way: a pair of different tiles
// is evaluated once (its j sums return to their home lanes after the 64
// rotations and join the i sums of their tile), a pair inside one tile
// one-sidedly from both ends.
//
// An item is run by NW wavefronts: each takes 64 / NW of the rotations of
// every j tile (wavefront w starts with the tile already rotated by
// w 64 / NW), and the wavefronts' sums are added in LDS in wavefront order, so
// an item's partials are the same size whatever NW is (sym_waves() chooses).
//
// Outputs are partial sums: the i side per item, the j side per (group,
// tile).  The reduce kernels add, for every atom, its group's i-side items in
// item order and then the j-side partials of every earlier group in group
// order: the result is deterministic.  Pair energy: each unordered pair adds
// 2 u^n to the i side (pairs inside a tile add u^n per ordered pair), so
// E_pair = (eps/2) a^n sum over all atoms, as in the one-sided sweeps.
#include "sweep_common.h"

namespace scmd {
namespace {

using namespace dev;

// Lane l receives the value of lane l-1 (mod 64): DPP wave_ror:1.  Every
// source lane is valid, so no "old" value is needed (bound_ctrl set).
__device__ __forceinline__ double ror1(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0x13C, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0x13C, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// i atoms of the group held by this lane.
template <int IPT>
struct IGroup {
    double x[IPT], y[IPT], z[IPT], c[IPT];  // c = -P_i
    int gi[IPT];
};

template <int IPT, typename AT>
__device__ __forceinline__ void load_group(const SymItem &it, const SymTile *__restrict__ tiles, AT &&at, double far,
                                           IGroup<IPT> &G) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int p = 0; p < IPT; ++p) {
        G.gi[p] = -1;
        G.x[p] = G.y[p] = G.z[p] = -far;
        G.c[p] = 0.0;
        if (p < it.ng) {
            const SymTile t = tiles[it.t0 + p];
            if (lane < t.ni) {
                G.gi[p] = t.i0 + lane;
                const double4 q = at(G.gi[p]);
                G.x[p] = q.x;
                G.y[p] = q.y;
                G.z[p] = q.z;
                G.c[p] = -q.w;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Force sweep
// ---------------------------------------------------------------------------
template <int PREC, bool EN>
__device__ __forceinline__ void sym_force_pair(double dx, double dy, double dz, double ci, double pj, float cif,
                                               float pjf, double &fx, double &fy, double &fz, double &eu,
                                               double &gx, double &gy, double &gz, const PotConst &pc, float Af) {
    double f, un;
    force_coef<PREC, false, EN>(__builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz)), ci, pj, cif, pjf, f, un, pc, Af);
    fx = __builtin_fma(f, dx, fx);
    fy = __builtin_fma(f, dy, fy);
    fz = __builtin_fma(f, dz, fz);
    gx = __builtin_fma(-f, dx, gx);
    gy = __builtin_fma(-f, dy, gy);
    gz = __builtin_fma(-f, dz, gz);
    if constexpr (EN) eu += un;
}

// The wavefront of the item this thread belongs to (uniform per wavefront).
template <int NW>
__device__ __forceinline__ int item_wave() {
    return NW == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// Sums of Q slices of IPT * 64 doubles over the item's wavefronts, in wavefront
// order, stored at out[q * IPT * 64 + k].  v(q, p) is this lane's value of
// slice q, tile p; sh holds 2 * NW * IPT * 64 doubles, free on entry.
template <int NW, int IPT, int Q, typename V>
__device__ __forceinline__ void store_item_sums(double *__restrict__ out, double *sh, int wave, V &&v) {
    const int lane = threadIdx.x & 63;
    constexpr int S = IPT * 64;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if constexpr (NW == 1) {
#pragma unroll
            for (int p = 0; p < IPT; ++p) out[q * S + p * 64 + lane] = v(q, p);
        } else {
            double *buf = sh + (q & 1) * NW * S;
#pragma unroll
            for (int p = 0; p < IPT; ++p) buf[wave * S + p * 64 + lane] = v(q, p);
            __syncthreads();
            for (int k = threadIdx.x; k < S; k += 64 * NW) {
                double t = buf[k];
#pragma unroll
                for (int w = 1; w < NW; ++w) t += buf[w * S + k];
                out[q * S + k] = t;
            }
        }
    }
}

// EN: accumulate and store the pair energy (u^n); without it (steps whose
// energies nobody reads) the energy partials are neither summed nor stored.
template <int IPT, int PREC, bool EN, int NW>
__global__ __launch_bounds__(64 * NW) void k_sym_force(const SymItem *__restrict__ items,
                                                       const int32_t *__restrict__ order,
                                                       const SymTile *__restrict__ tiles,
                                                       const double4 *__restrict__ xp, double *__restrict__ ipart,
                                                       double *__restrict__ jpart, PotConst pc) {
    constexpr int RW = 64 / NW;             // rotations per wavefront
    constexpr int SI = NW * IPT * 64, SJ = NW * 3 * 64;
    __shared__ double sh[NW == 1 ? 1 : 2 * (SI > SJ ? SI : SJ)];
    __shared__ double2 jtile[NW == 1 ? 1 : 2 * 256];
    const SymItem it = items[order[blockIdx.x]];
    const int lane = threadIdx.x & 63, wave = item_wave<NW>();
    const int rot0 = wave * RW;
    const float Af = (float)pc.A;
    IGroup<IPT> G;
    load_group<IPT>(it, tiles, [&](int i) { return xp[i]; }, kFar, G);
    float cif[IPT];
    double fx[IPT], fy[IPT], fz[IPT], eu[IPT];
#pragma unroll
    for (int p = 0; p < IPT; ++p) {
        fx[p] = fy[p] = fz[p] = eu[p] = 0.0;
        cif[p] = (float)G.c[p];
    }
    if (it.b0 == it.b1) {
        // diagonal item: the group's own tile b rotates past tiles p <= b
        double eus[IPT];  // energy of the pairs of different tiles (counted twice below)
#pragma unroll
        for (int p = 0; p < IPT; ++p) eus[p] = 0.0;
#pragma unroll
        for (int b = 0; b < IPT; ++b) {
            if (b < it.ng) {
                const bool own = G.gi[b] >= 0;  // past the tile's atoms: the j sentinel
                double xj = own ? G.x[b] : kFar, yj = own ? G.y[b] : kFar, zj = own ? G.z[b] : kFar;
                double pj = own ? -G.c[b] : 0.0;
                if constexpr (NW > 1) {
                    const int from = (lane - rot0) & 63;
                    xj = __shfl(xj, from, 64);
                    yj = __shfl(yj, from, 64);
                    zj = __shfl(zj, from, 64);
                    pj = __shfl(pj, from, 64);
                }
                double gx = 0.0, gy = 0.0, gz = 0.0;
                // rotation k: lane l meets atom l - k of tile b; k = 0 is the
                // self pair inside tile b
                auto step = [&](bool with_own_tile) {
                    const float pjf = (float)pj;
#pragma unroll
                    for (int p = 0; p < IPT; ++p) {
                        if (p < b) {
                            sym_force_pair<PREC, EN>(G.x[p] - xj, G.y[p] - yj, G.z[p] - zj, G.c[p], pj, cif[p], pjf,
                                                     fx[p], fy[p], fz[p], eus[p], gx, gy, gz, pc, Af);
                        } else if (p == b && with_own_tile) {
                            double hx = 0.0, hy = 0.0, hz = 0.0;  // one-sided: no j sums
                            sym_force_pair<PREC, EN>(G.x[p] - xj, G.y[p] - yj, G.z[p] - zj, G.c[p], pj, cif[p], pjf,
                                                     fx[p], fy[p], fz[p], eu[p], hx, hy, hz, pc, Af);
                        }
                    }
                    xj = ror1(xj);
                    yj = ror1(yj);
                    zj = ror1(zj);
                    pj = ror1(pj);
                    gx = ror1(gx);
                    gy = ror1(gy);
                    gz = ror1(gz);
                };
                step(NW > 1 && wave != 0);
#pragma unroll 2
                for (int k = 1; k < RW; ++k) step(true);
                // the j sums go back to their home lanes (64 rotations bring
                // them there by themselves)
                if constexpr (NW > 1) {
                    const int at = (lane + rot0 + RW) & 63;
                    gx = __shfl(gx, at, 64);
                    gy = __shfl(gy, at, 64);
                    gz = __shfl(gz, at, 64);
                }
                fx[b] += gx;
                fy[b] += gy;
                fz[b] += gz;
            }
        }
#pragma unroll
        for (int p = 0; p < IPT; ++p) eu[p] += 2.0 * eus[p];
    } else {
        // NW > 1: the item's wavefronts share the j tile in LDS, every atom
        // twice, so that the atom lane l meets at rotation k, (l - k) mod 64,
        // is entry l + 64 - k of both arrays and no index wraps; only the sums
        // rotate by DPP.  The next tile's atoms travel while one is worked on.
        const int dst = (lane - rot0 - RW) & 63;  // atom whose sums this lane ends with
        SymTile t = tiles[it.b0];
        auto fetch = [&](const SymTile &u) {
            return lane < u.ni ? xp[u.i0 + lane] : make_double4(kFar, kFar, kFar, 0.0);
        };
        auto put = [&](int b, const double4 &q) {
            double2 *t0 = jtile + (b & 1) * 256;
            t0[lane] = t0[64 + lane] = make_double2(q.x, q.y);
            t0[128 + lane] = t0[192 + lane] = make_double2(q.z, q.w);
        };
        double4 nxt = make_double4(kFar, kFar, kFar, 0.0);
        if (wave == 0) nxt = fetch(t);
        if constexpr (NW > 1) {
            if (wave == 0) put(it.b0, nxt);
            __syncthreads();
        }
        for (int b = it.b0; b < it.b1; ++b) {
            double xj = nxt.x, yj = nxt.y, zj = nxt.z, pj = nxt.w;
            const int jslot = t.jbase + it.g;
            if (b + 1 < it.b1) {
                t = tiles[b + 1];
                if (wave == 0) nxt = fetch(t);
            }
            const double2 *jt = jtile + (NW > 1 ? (b & 1) * 256 + lane + 64 - rot0 : 0);
            double gx = 0.0, gy = 0.0, gz = 0.0;
#pragma unroll(IPT == 2 ? 4 : 2)
            for (int k = 0; k < RW; ++k) {
                if constexpr (NW > 1) {
                    const double2 q0 = jt[-k], q1 = jt[128 - k];
                    xj = q0.x;
                    yj = q0.y;
                    zj = q1.x;
                    pj = q1.y;
                }
                const float pjf = (float)pj;
#pragma unroll
                for (int p = 0; p < IPT; ++p) {
                    sym_force_pair<PREC, EN>(G.x[p] - xj, G.y[p] - yj, G.z[p] - zj, G.c[p], pj, cif[p], pjf, fx[p], fy[p],
                                         fz[p], eu[p], gx, gy, gz, pc, Af);
                }
                if constexpr (NW == 1) {
                    xj = ror1(xj);
                    yj = ror1(yj);
                    zj = ror1(zj);
                    pj = ror1(pj);
                }
                gx = ror1(gx);
                gy = ror1(gy);
                gz = ror1(gz);
            }
            double ge = 0.0;
            unscale_force<PREC, false>(gx, gy, gz, ge);
            double *out = jpart + (size_t)jslot * 3 * 64;
            if constexpr (NW == 1) {
                out[lane] = gx;
                out[64 + lane] = gy;
                out[128 + lane] = gz;
            } else {
                // two buffers in turn: a wavefront reaches this one again only
                // past the next tile's barrier, when all have read it
                double *buf = sh + (b & 1) * SJ;
                buf[wave * 192 + dst] = gx;
                buf[wave * 192 + 64 + dst] = gy;
                buf[wave * 192 + 128 + dst] = gz;
                if (wave == 0 && b + 1 < it.b1) put(b + 1, nxt);
                __syncthreads();
                if (threadIdx.x < 192) {
                    double v = buf[threadIdx.x];
#pragma unroll
                    for (int w = 1; w < NW; ++w) v += buf[w * 192 + threadIdx.x];
                    out[threadIdx.x] = v;
                }
            }
        }
#pragma unroll
        for (int p = 0; p < IPT; ++p) eu[p] *= 2.0;  // each unordered pair once
        if constexpr (NW > 1) __syncthreads();
    }
#pragma unroll
    for (int p = 0; p < IPT; ++p) unscale_force<PREC, false>(fx[p], fy[p], fz[p], eu[p]);
    // steps without the pair energy leave its slot unwritten (the reduce of
    // such a step does not read it)
    store_item_sums<NW, IPT, EN ? 4 : 3>(ipart + (size_t)it.slot * 4 * 64 * IPT, sh, wave, [&](int q, int p) {
        return q == 0 ? fx[p] : q == 1 ? fy[p] : q == 2 ? fz[p] : eu[p];
    });
}

// ---------------------------------------------------------------------------
// Density sweep
// ---------------------------------------------------------------------------
// With four wavefronts the sweep can also drift the atoms it loads
// (da.mode != 0, see Drift): every item finishes its cluster's thermostat
// factor for itself, and the cluster's first item stores it.
template <int IPT, int PREC, int NW>
__global__ __launch_bounds__(64 * NW) void k_sym_density(const SymItem *__restrict__ items,
                                                         const int32_t *__restrict__ order,
                                                         const SymTile *__restrict__ tiles,
                                                         const double4 *__restrict__ rp, double *__restrict__ ipart,
                                                         double *__restrict__ jpart, PotConst pc, DriftArgs da) {
    constexpr int RW = 64 / NW;
    constexpr int SI = NW * IPT * 64;
    constexpr int SHARE = IPT < 4 ? 2 : 4;  // pairs that share a reciprocal
    __shared__ double sh[NW == 1 ? 1 : 2 * SI];
    __shared__ double jtile[NW == 1 ? 1 : 2 * 384];
    const SymItem it = items[order[blockIdx.x]];
    const int lane = threadIdx.x & 63, wave = item_wave<NW>();
    const int rot0 = wave * RW;
    double lam = 1.0;
    bool bath = false;
    if constexpr (NW > 1) {
        if (da.mode != 0) {
            __shared__ double sh_tot[12];
            bath = in_bath(it.c, da);
            lam = drift_factor<true>(it.c, da, bath, sh_tot, it.first != 0);
        }
    }
    auto position = [&](int i) {
        if constexpr (NW > 1) {
            if (da.mode != 0) return drifted_atom(rp, i, da, bath, lam);
        }
        return rp[i];
    };
    auto square = [](double dx, double dy, double dz) {
        return __builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz));
    };
    auto pair_term = [&](double dx, double dy, double dz) { return density_term<PREC, false>(square(dx, dy, dz), pc); };
    IGroup<IPT> G;
    load_group<IPT>(it, tiles, position, kFarShared, G);
    double acc[IPT];
#pragma unroll
    for (int p = 0; p < IPT; ++p) acc[p] = 0.0;
    if (it.b0 == it.b1) {
        // diagonal item (as in the force sweep): tile b rotates past tiles p <= b
#pragma unroll
        for (int b = 0; b < IPT; ++b) {
            if (b < it.ng) {
                const bool own = G.gi[b] >= 0;
                double xj = own ? G.x[b] : kFarShared, yj = own ? G.y[b] : kFarShared, zj = own ? G.z[b] : kFarShared;
                if constexpr (NW > 1) {
                    const int from = (lane - rot0) & 63;
                    xj = __shfl(xj, from, 64);
                    yj = __shfl(yj, from, 64);
                    zj = __shfl(zj, from, 64);
                }
                double rj = 0.0;
                auto step = [&](bool with_own_tile) {
#pragma unroll
                    for (int p = 0; p < IPT; ++p) {
                        if (p < b) {
                            const double t6 = pair_term(G.x[p] - xj, G.y[p] - yj, G.z[p] - zj);
                            acc[p] += t6;
                            rj += t6;
                        } else if (p == b && with_own_tile) {
                            acc[p] += pair_term(G.x[p] - xj, G.y[p] - yj, G.z[p] - zj);
                        }
                    }
                    xj = ror1(xj);
                    yj = ror1(yj);
                    zj = ror1(zj);
                    rj = ror1(rj);
                };
                step(NW > 1 && wave != 0);
#pragma unroll 2
                for (int k = 1; k < RW; ++k) step(true);
                if constexpr (NW > 1) rj = __shfl(rj, (lane + rot0 + RW) & 63, 64);
                acc[b] += rj;
            }
        }
    } else {
        // the j tile in LDS as in the force sweep
        const int dst = (lane - rot0 - RW) & 63;
        SymTile t = tiles[it.b0];
        auto fetch = [&](const SymTile &u) {
            return lane < u.ni ? position(u.i0 + lane) : make_double4(kFarShared, kFarShared, kFarShared, 0.0);
        };
        auto put = [&](int b, const double4 &q) {
            double *t0 = jtile + (b & 1) * 384;
            t0[lane] = t0[64 + lane] = q.x;
            t0[128 + lane] = t0[192 + lane] = q.y;
            t0[256 + lane] = t0[320 + lane] = q.z;
        };
        double4 nxt = make_double4(kFarShared, kFarShared, kFarShared, 0.0);
        if (wave == 0) nxt = fetch(t);
        if constexpr (NW > 1) {
            if (wave == 0) put(it.b0, nxt);
            __syncthreads();
        }
        for (int b = it.b0; b < it.b1; ++b) {
            double xj = nxt.x, yj = nxt.y, zj = nxt.z;
            const int jslot = t.jbase + it.g;
            if (b + 1 < it.b1) {
                t = tiles[b + 1];
                if (wave == 0) nxt = fetch(t);
            }
            const double *jt = jtile + (NW > 1 ? (b & 1) * 384 + lane + 64 - rot0 : 0);
            double rj = 0.0;
#pragma unroll(IPT == 2 ? 4 : 2)
            for (int k = 0; k < RW; ++k) {
                if constexpr (NW > 1) {
                    xj = jt[-k];
                    yj = jt[128 - k];
                    zj = jt[256 - k];
                }
#pragma unroll
                for (int p = 0; p < IPT; p += SHARE) {
                    double r2[SHARE], t6[SHARE];
#pragma unroll
                    for (int q = 0; q < SHARE; ++q) r2[q] = square(G.x[p + q] - xj, G.y[p + q] - yj, G.z[p + q] - zj);
                    density_terms<PREC, SHARE>(r2, t6, pc);
#pragma unroll
                    for (int q = 0; q < SHARE; ++q) {
                        acc[p + q] += t6[q];
                        rj += t6[q];
                    }
                }
                if constexpr (NW == 1) {
                    xj = ror1(xj);
                    yj = ror1(yj);
                    zj = ror1(zj);
                }
                rj = ror1(rj);
            }
            if constexpr (NW == 1) {
                jpart[(size_t)jslot * 64 + lane] = rj;
            } else {
                double *buf = sh + (b & 1) * NW * 64;
                buf[wave * 64 + dst] = rj;
                if (wave == 0 && b + 1 < it.b1) put(b + 1, nxt);
                __syncthreads();
                if (threadIdx.x < 64) {
                    double v = buf[threadIdx.x];
#pragma unroll
                    for (int w = 1; w < NW; ++w) v += buf[w * 64 + threadIdx.x];
                    jpart[(size_t)jslot * 64 + threadIdx.x] = v;
                }
            }
        }
        if constexpr (NW > 1) __syncthreads();
    }
    store_item_sums<NW, IPT, 1>(ipart + (size_t)it.slot * 64 * IPT, sh, wave, [&](int, int p) { return acc[p]; });
}

// ---------------------------------------------------------------------------
// Reduce + finish: one workgroup of 512 threads per 64-atom tile.  Thread
// (g8, lane), g8 = 0..7, adds the tile's i-side items k and j-side partials
// g with k, g = g8 (mod 8) (items first, each run in increasing order); the
// eight sums are combined in g8 order, so the result is deterministic.
// Q = 1: density; Q = 4: force and pair energy (the energy only when the
// sweep accumulated it, EN; otherwise it is zero and was not stored).
// ---------------------------------------------------------------------------
constexpr int kSymRed = 512;
constexpr int kSymRedGroups = kSymRed / 64;

template <int IPT, int Q, bool EN>
__device__ __forceinline__ void sym_sums(const SymTile &t, const double *__restrict__ ipart,
                                         const double *__restrict__ jpart, double *sh) {
    const int lane = threadIdx.x & 63, g8 = threadIdx.x >> 6;
    constexpr int QI = (Q == 4 && !EN) ? 3 : Q;  // i-side values read
    constexpr int QJ = Q == 4 ? 3 : 1;           // the j side carries no energy
    double s[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) s[q] = 0.0;
    if (lane < t.ni) {
        for (int k = g8; k < t.nitems; k += kSymRedGroups) {
            const double *p = ipart + (size_t)(t.item0 + k) * Q * 64 * IPT + t.p * 64 + lane;
#pragma unroll
            for (int q = 0; q < QI; ++q) s[q] += p[(size_t)q * IPT * 64];
        }
        for (int g = g8; g < t.nj; g += kSymRedGroups) {
            const double *p = jpart + ((size_t)(t.jbase + g) * QJ) * 64 + lane;
#pragma unroll
            for (int q = 0; q < QJ; ++q) s[q] += p[q * 64];
        }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) sh[(g8 * Q + q) * 64 + lane] = s[q];
    __syncthreads();
    if (g8 == 0) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            double v = sh[q * 64 + lane];
            for (int gg = 1; gg < kSymRedGroups; ++gg) v += sh[(gg * Q + q) * 64 + lane];
            sh[q * 64 + lane] = v;
        }
    }
    __syncthreads();
}

// shared: the sweep's pairs shared reciprocals (double).  A product of r^2 that
// left the range then made all its terms NaN: a sum that is not finite is taken
// again here, pair by pair, so that only pairs bad by themselves spoil it.  (Voting
// on it and repeating the item inside the sweep cost 0.3 to 0.9 % of a step.)
template <int IPT>
__global__ __launch_bounds__(kSymRed) void k_sym_density_reduce(const SymTile *__restrict__ tiles,
                                                                const double *__restrict__ ipart,
                                                                const double *__restrict__ jpart, DensityOut o,
                                                                PotConst pc, DriftArgs da, bool shared) {
    __shared__ double sh[kSymRedGroups * 64];
    const SymTile t = tiles[blockIdx.x];
    const bool bath = da.mode != 0 && in_bath(t.c, da);
    const double lam = da.mode != 0 ? da.st[t.c].lambda : 1.0;
    // an atom's position, as the sweep had it
    auto position = [&](int i) { return da.mode != 0 ? drifted_atom(o.rp, i, da, bath, lam) : o.rp[i]; };
    // fetched ahead of the sums
    double4 q = make_double4(0, 0, 0, 0);
    if (threadIdx.x < t.ni) q = position(t.i0 + threadIdx.x);
    sym_sums<IPT, 1, false>(t, ipart, jpart, sh);
    if (threadIdx.x >= 64) return;
    double emb = 0.0;
    if (threadIdx.x < t.ni) {
        double u6 = sh[threadIdx.x];
        if (shared && !isfinite(u6)) {
            const int i = t.i0 + threadIdx.x, a = da.cd[t.c].off, b = a + da.cd[t.c].n;
            u6 = 0.0;
            for (int j = a; j < b; ++j) {
                const double4 p = position(j);
                const double dx = q.x - p.x, dy = q.y - p.y, dz = q.z - p.z;
                if (j != i)
                    u6 += density_term<SCMD_FP64, false>(__builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz)), pc);
            }
        }
        // sums of sentinels alone (5e-227 each, a few hundred at most; a pair 1e12
        // A apart gives 1e-72): the atom has no neighbour
        emb = density_atom_at(t.i0 + threadIdx.x, u6 < 1.0e-220 ? 0.0 : u6, q, o, pc);
    }
    emb = wave_total(emb);
    if (threadIdx.x == 0) o.tile_sums[(size_t)blockIdx.x * kTileSums + 0] = emb;
}

template <int IPT, bool EN>
__global__ __launch_bounds__(kSymRed) void k_sym_force_reduce(const SymTile *__restrict__ tiles,
                                                              const double *__restrict__ ipart,
                                                              const double *__restrict__ jpart,
                                                              const double4 *__restrict__ xp, ForceOut o,
                                                              PotConst pc) {
    __shared__ double sh[kSymRedGroups * 4 * 64];
    const SymTile t = tiles[blockIdx.x];
    const int l = threadIdx.x;
    const int i = t.i0 + l;
    // the epilogue's own-atom loads and, in a bath, the next step's noise do
    // not depend on the sums: they are issued ahead of them
    const bool bath = o.fused && (o.bath == 1 || (o.bath == 2 && o.cd[t.c].kind == SCMD_LANGEVIN));
    FusedAtom a;
    if (l < t.ni) a = fused_atom_load(i, t.c, bath, xp, o);
    sym_sums<IPT, 4, EN>(t, ipart, jpart, sh);
    if (l >= 64) return;
    double epair = 0.0, v2 = 0.0;
    if (l < t.ni) {
        const double fx = sh[l], fy = sh[64 + l], fz = sh[128 + l], eu = sh[192 + l];
        if (bath)
            force_atom_bath(i, fx, fy, fz, eu, a.r, a.v, a.xi, a.c2, o.cd[t.c], o, pc, epair, v2);
        else if (o.fused)
            force_atom_fused<false>(i, fx, fy, fz, eu, a.r, a.v, a.f, o.st[t.c].lambda, o, pc, epair, v2);
        else
            force_atom_v(i, fx, fy, fz, eu, a.v, o, pc, epair, v2);
    }
    epair = wave_total(epair);
    v2 = wave_total(v2);
    if (l == 0) {
        o.tile_sums[(size_t)blockIdx.x * kTileSums + 1] = epair;
        o.tile_sums[(size_t)blockIdx.x * kTileSums + 2] = v2;
    }
}

template <int IPT, int PREC, int NW>
hipError_t launch_ipt(bool force, int stage, bool energy, const SymLaunch &L, const SweepBuffers &B,
                      const ForceOut &fo, const DriftArgs &da, const PotConst &pc, hipStream_t s) {
    (void)hipGetLastError();
    const dim3 block(64 * NW);
    if (stage == 0 && L.nitems > 0) {
        if (force && energy)
            hipLaunchKernelGGL((k_sym_force<IPT, PREC, true, NW>), dim3(L.nitems), block, 0, s, L.items, L.order,
                               L.tiles, B.xp, L.ipart, L.jpart, pc);
        else if (force)
            hipLaunchKernelGGL((k_sym_force<IPT, PREC, false, NW>), dim3(L.nitems), block, 0, s, L.items, L.order,
                               L.tiles, B.xp, L.ipart, L.jpart, pc);
        else
            hipLaunchKernelGGL((k_sym_density<IPT, PREC, NW>), dim3(L.nitems), block, 0, s, L.items, L.order, L.tiles,
                               B.rp, L.ipart, L.jpart, pc, da);
    }
    if (stage == 1 && L.ntiles > 0) {
        if (force) {
            if (energy)
                hipLaunchKernelGGL((k_sym_force_reduce<IPT, true>), dim3(L.ntiles), dim3(kSymRed), 0, s, L.tiles,
                                   L.ipart, L.jpart, B.xp, fo, pc);
            else
                hipLaunchKernelGGL((k_sym_force_reduce<IPT, false>), dim3(L.ntiles), dim3(kSymRed), 0, s, L.tiles,
                                   L.ipart, L.jpart, B.xp, fo, pc);
        } else {
            const DensityOut o{B.rp, B.xp, B.rho, B.tile_sums};
            hipLaunchKernelGGL((k_sym_density_reduce<IPT>), dim3(L.ntiles), dim3(kSymRed), 0, s, L.tiles, L.ipart,
                               L.jpart, o, pc, da, PREC == SCMD_FP64);
        }
    }
    return hipGetLastError();
}

template <int PREC>
hipError_t dispatch_ipt(bool force, int stage, bool energy, const SymLaunch &L, const SweepBuffers &B,
                        const ForceOut &fo, const DriftArgs &da, const PotConst &pc, hipStream_t s) {
#define SCMD_SYM(I, W) launch_ipt<I, PREC, W>(force, stage, energy, L, B, fo, da, pc, s)
    // the folded drift needs the workgroup-wide totals of four wavefronts
    if (L.waves != sym_waves(L.ipt) || (L.waves == 1 && (da.mode != 0 || fo.fused))) return hipErrorInvalidValue;
    switch (L.ipt) {
        case 2: return SCMD_SYM(2, 4);
        case 4: return SCMD_SYM(4, 4);
        case 8: return SCMD_SYM(8, 1);
        default: return hipErrorInvalidValue;
    }
#undef SCMD_SYM
}

}  // namespace

hipError_t launch_sym_density(const SymLaunch &L, const SweepBuffers &B, const StepArgs &a, const Drift &dr,
                              const PotConst &pc, int precision, int stage, hipStream_t s) {
    if (pc.generic || pc.cut) return hipErrorInvalidValue;
    const DriftArgs da = drift_args(B, a, dr);
    return precision == SCMD_FP64 ? dispatch_ipt<SCMD_FP64>(false, stage, true, L, B, ForceOut{}, da, pc, s)
                                  : dispatch_ipt<SCMD_MIXED>(false, stage, true, L, B, ForceOut{}, da, pc, s);
}

hipError_t launch_sym_force(const SymLaunch &L, const SweepBuffers &B, const StepArgs &a, int fused, int local,
                            int bath, const PotConst &pc, int precision, int stage, hipStream_t s) {
    if (pc.generic || pc.cut) return hipErrorInvalidValue;
    const ForceOut fo = fused_force_out(B, a, fused, local, bath);
    const bool energy = a.energy != 0;
    return precision == SCMD_FP64
               ? dispatch_ipt<SCMD_FP64>(true, stage, energy, L, B, fo, DriftArgs{}, pc, s)
               : dispatch_ipt<SCMD_MIXED>(true, stage, energy, L, B, fo, DriftArgs{}, pc, s);
}

}  // namespace scmd
