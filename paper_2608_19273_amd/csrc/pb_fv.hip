// pb_fv.hip -- fused first-order Rusanov finite-volume step on a patch batch
// (the FV composition of paper Sec. II-A, Eq. (3): source term, face fluxes
// from the two adjacent cell values, update), one launch per time step.
//
// Work decomposition (MI355X): a work-group of up to 256 threads (as many
// waves as a plane fills) owns one z-slab of one patch or a run of planes and
// marches through it plane by plane.  Thread t owns column
// (x, y) = (t % p, t / p).  For each plane the work-group
//   1. stores its cells' Q and per-cell aux (1/rho, p, c ...) in LDS, and the
//      4p face-halo cells of the plane, read straight from the face
//      neighbours' interiors (this is the halo gather, fused into the tile
//      load: no halo array ever exists in HBM);
//   2. after one barrier, evaluates the x and y face fluxes from LDS and the
//      z face flux from registers (the lower z face is carried over from the
//      previous plane, so every z face is evaluated once);
//   3. updates the cell, stores it, and (CFL mode) folds the largest speed of
//      the new state into a per-thread maximum.
// LDS is double-buffered by plane parity, so one barrier per plane suffices.
// At the end the work-group reduces its maxima (wave shuffle, then LDS) and
// folds them into the hand-over to the call's next step (FvChain), so dt never
// leaves the device.
#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

#include "pb_common.h"
#include "pb_physics.h"

namespace pb {

namespace {

template <class Ph, typename T>
__device__ __forceinline__ void load_cell(const T *__restrict__ q, const double *__restrict__ ex,
                                          long long off, long long C, long long c, double *out,
                                          double *e)
{
    constexpr int N = Ph::N;
    const T *base = q + off * N + c;
#pragma unroll
    for (int v = 0; v < N; ++v) out[v] = (double)base[(long long)v * C];
    if (Ph::E) e[0] = ex[off + c];
}

template <class Ph, int DIM>
__device__ __forceinline__ void cell_speeds(const Ph &ph, const double *q, const double *a,
                                            double *lm)
{
    lm[0] = fmax(lm[0], ph.template eig<0>(q, a));
    lm[1] = fmax(lm[1], ph.template eig<1>(q, a));
    if (DIM == 3) lm[2] = fmax(lm[2], ph.template eig<2>(q, a));
}

// Largest speeds of a freshly written cell, for the next step's dt only: the
// aux evaluation uses the reciprocal / rsqrt estimates refined by Newton
// steps (a max over cells needs no correctly rounded quotient).
template <class Ph, int DIM>
__device__ __forceinline__ void cell_speeds_fast(const Ph &ph, const double *q, double *lm)
{
    constexpr int AA = Ph::A > 0 ? Ph::A : 1;
    double a[AA], e[1] = {0.0};
    ph.aux_fast(q, e, a);
    cell_speeds<Ph, DIM>(ph, q, a, lm);
}

}  // namespace

// raw (storage-type) values of one cell: N unknowns plus the extra input
template <class Ph, typename T>
struct RawCell {
    T q[Ph::N];
    double e;
};

template <class Ph, typename T>
__device__ __forceinline__ void issue_load(const T *__restrict__ q, const double *__restrict__ ex,
                                           long long off, long long C, long long c, RawCell<Ph, T> &r)
{
    const T *base = q + off * Ph::N + c;
#pragma unroll
    for (int v = 0; v < Ph::N; ++v) r.q[v] = base[(long long)v * C];
    if (Ph::E) r.e = ex[off + c];
}

template <class Ph, typename T>
__device__ __forceinline__ void unpack(const RawCell<Ph, T> &r, double *q, double *e)
{
#pragma unroll
    for (int v = 0; v < Ph::N; ++v) q[v] = (double)r.q[v];
    e[0] = Ph::E ? r.e : 0.0;
}

template <class Ph, int D>
__device__ __forceinline__ void phys_flux_or_zero(const Ph &ph, const double *q, const double *a, double *F)
{
    if (Ph::kFlux) {
        ph.template flux<D>(q, a, F);
    } else {
#pragma unroll
        for (int v = 0; v < Ph::N; ++v) F[v] = 0.0;
    }
}

// Keeps the compiler from fusing a flux's last product into a later sum, so that
// every place that adds this flux adds the same bits.  Components that are
// components of Q (Euler's mass flux) are left alone: as values of their own they
// would take registers of their own (five steps of 693 patches of 13^3 in FP32
// storage: 175 us with them, 172 without and with no such rounding at all).
template <class Ph> struct FluxCopies { static constexpr int n = 0; };
template <int DIM> struct FluxCopies<Euler<DIM>> { static constexpr int n = 1; };
template <class Ph>
__device__ __forceinline__ void flux_as_rounded(double *F)
{
#pragma unroll
    for (int v = FluxCopies<Ph>::n; v < Ph::N; ++v) __asm__("" : "+v"(F[v]));
}

// The aux values an x or y neighbour's flux and speed read, which the plane
// kernel passes through LDS: all of them, except for SRHD, whose direction d
// reads p, v_d and lambda_d only, so v_z and lambda_z stay in the z carry
// (10 instead of 12 values per cell: three work-groups fit a CU's LDS).
template <class Ph> struct PlaneAux {
    static constexpr int n = Ph::A;
    static __device__ __forceinline__ constexpr int idx(int j) { return j; }
};
template <> struct PlaneAux<Srhd> {
    static constexpr int n = 5;
    static __device__ __forceinline__ constexpr int idx(int j) { return j < 3 ? j : j + 1; }   // p, v_x, v_y, l_x, l_y
};

// Work schedule of the plane-march kernel.  Slab mode (plan.planes == 0):
// work-group (unit) u marches slab u % n_slabs of patch u / n_slabs (a slab
// can start beyond the last plane of a patch smaller than the batch maximum:
// such a unit only takes part in the reductions).  Balanced mode (uniform
// patch size p, plan.planes = K p planes in patch order): the grid is a
// chosen number of work-groups per CU (those that fit at once: no second
// round) and work-group r marches the planes
// [r T / G, (r + 1) T / G) of that sequence, one segment per patch it
// crosses, so every work-group moves the same number of planes and the last
// round of a grid of whole patches, partly filled, disappears.  Column mode
// (plan.runs): unit u marches runs[u].z planes starting at plane runs[u].y of
// patch runs[u].x and continuing, without a restart, into the +z neighbour
// (the z halo between consecutive patches of a run is the plane the march
// has just processed: it is never read twice).
struct FvPlan {
    int n_units, n_slabs, slab, remap;
    long long planes;   // balanced mode: total planes (0: slab mode)
    const int4 *runs;   // column mode (non-null): unit u marches runs[u] = (patch, first plane, planes)
};

// the largest p + 2 of a work-group of so many waves
constexpr int kPlanePH[5] = {0, 10, 13, 15, kFvPmax + 2};

template <class Ph, int DIM, typename T, bool kLam, int WV>
__global__ __launch_bounds__(kWave *WV) __attribute__((amdgpu_waves_per_eu(3))) void fv_step_kernel(
    const T *__restrict__ qin, T *__restrict__ qout, const double *__restrict__ ex,
    const PatchDev *__restrict__ patches, FvPlan plan, Ctrl *__restrict__ ctrl, int slot_in, double dt_fixed, FvChain chain, Ph ph)
{
    constexpr int N = Ph::N, A = Ph::A, AP = PlaneAux<Ph>::n, W = N + AP, AA = A > 0 ? A : 1;
    constexpr int PH = kPlanePH[WV];
    constexpr bool kOneWave = WV < 4;
    constexpr int DZ = DIM == 3 ? 2 : 1;   // z direction index (unused in 2D)
    __shared__ double lds[2][W][PH * PH];

    const int t = threadIdx.x;
    const int unit = plan.remap ? xcd_remap(blockIdx.x, plan.n_units) : (int)blockIdx.x;
    const double dt = step_dt<DIM, kLam, (Ph::E > 0), kWave * WV>(ctrl, slot_in, dt_fixed, chain);
    double lm[3] = {0.0, 0.0, 0.0};
    bool bad = false;
    int parity = 0;   // LDS buffer of the next plane (alternates over every plane the work-group marches)

    // one segment: n planes starting at plane z0 of patch k, continuing into
    // the +z neighbour at the patch's top (the patches of a run share p)
    auto segment = [&](int k, int z0, int n) {
    const int p = patches[k].p;
    const long long C = (DIM == 3) ? (long long)p * p * p : (long long)p * p;

    const bool work = n > 0;
    const bool active = work && t < p * p;
    const int x = active ? t % p : 0, y = active ? t / p : 0;
    const int li = (y + 1) * PH + (x + 1);

    // face-halo cell of each plane: of four waves, wave w serves side w (-x,
    // +x, -y, +y), so the extra loads and aux evaluations spread over all of
    // them; of fewer waves the last, which has lanes without a cell of their
    // own, serves all 4p cells
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int side = kOneWave ? lane / p : wave, j = kOneWave ? lane - side * p : lane;
    const bool halo = work && (kOneWave ? wave == WV - 1 && side < 4 : j < p);
    int hsrc = 0, hdst = 0;
    if (halo) {
        int hx, hy, sx, sy;
        if (side == 0)      { hx = -1; hy = j;  sx = p - 1; sy = j;     }
        else if (side == 1) { hx = p;  hy = j;  sx = 0;     sy = j;     }
        else if (side == 2) { hx = j;  hy = -1; sx = j;     sy = p - 1; }
        else                { hx = j;  hy = p;  sx = j;     sy = 0;     }
        hsrc = sy * p + sx;
        hdst = (hy + 1) * PH + (hx + 1);
    }
    const long long cxy = (long long)y * p + x;
    const long long pp = (long long)p * p;
    // where the halo cell of patch kk's plane 0 is: four waves, the first cell
    // of the neighbour on the wave's side; one wave, the byte offset of the
    // lane's cell from the state's start (32 bits, one register)
    using HaloOff = std::conditional_t<kOneWave, unsigned, long long>;
    auto halo_off = [&](int kk) -> HaloOff {
        const PatchDev &Q = patches[kk];
        if constexpr (!kOneWave) {
            return patches[Q.nbr[side]].off;
        } else {
            const unsigned o0 = (unsigned)patches[Q.nbr[0]].off, o1 = (unsigned)patches[Q.nbr[1]].off,
                           o2 = (unsigned)patches[Q.nbr[2]].off, o3 = (unsigned)patches[Q.nbr[3]].off;
            const unsigned o = !halo || side == 0 ? o0 : side == 1 ? o1 : side == 2 ? o2 : o3;
            return (o * N + hsrc) * (unsigned)sizeof(T);
        }
    };
    auto halo_load = [&](HaloOff off, int z, RawCell<Ph, T> &r) {
        if constexpr (!kOneWave) {
            issue_load<Ph>(qin, ex, off, C, (long long)z * pp + hsrc, r);
        } else {
            const unsigned o = off + (unsigned)(z * (int)pp) * (unsigned)sizeof(T);
#pragma unroll
            for (int v = 0; v < N; ++v)
                r.q[v] = *reinterpret_cast<const T *>(reinterpret_cast<const char *>(qin + (long long)v * C) + o);
        }
    };
    int kc = k;
    // the current patch and its +z neighbour (the run's next patch): cell
    // offsets of the patch and of the wave's halo-side neighbour (lanes
    // without a halo cell load cell 0 of that neighbour and drop it)
    long long offc = patches[k].off;
    HaloOff hoffc = halo_off(k);
    double hr_ = 0.5 * dt * patches[k].inv_dx;   // the face sums below are doubled
    int kn = (DIM == 3) ? patches[k].nbr[5] : k;
    long long offn = patches[kn].off;
    HaloOff hoffn = halo_off(kn);
    int zl = z0;   // the current plane's z inside the current patch

    // per thread, two sets that swap roles from plane to plane (the loop runs
    // two planes per trip, so nothing is copied between them): a plane's
    // values (q, a), its z flux and speed (fz, lz), and the doubled flux and
    // fluctuation of its lower z face (fs, dn)
    struct Carry {
        double q[N], a[AA], fz[N], fs[N], dn[N];
        double lz;
    };
    Carry cA, cB;
    double e[1];
    double *qc = cA.q, *ac = cA.a, *fzc = cA.fz, *fs2l = cA.fs, *dn2l = cA.dn;
    double &lzc = cA.lz;
    lzc = 0.0;
    // one-plane prefetch (raw storage-type values): the own column for plane
    // z+1 and the halo cell for plane z.  One plane ahead is as fast as two or
    // three, and with the next plane's flux evaluated after the x and y
    // directions the kernel fits in 3 waves per SIMD without spilling.
    RawCell<Ph, T> rnA, hrA;

    // plane zl + d (d = 0, 1, 2; p >= 2) of the run: the current patch or the next
    auto own_plane_off = [&](int zz) -> long long { return zz >= p ? offn : offc; };
    auto own_plane_c = [&](int zz) -> long long { return (zz >= p ? zz - p : zz) * pp + cxy; };

    // Every lane issues every load (idle lanes at a valid address they do not
    // use), and the prefetch at the slab's top reloads a plane in reach
    // instead of skipping: a load under a divergent or conditional branch
    // makes the compiler copy its target registers at the join, which waits
    // for the load right there and empties the prefetch ring.
    if (work) {
        RawCell<Ph, T> rc;
        issue_load<Ph>(qin, ex, offc, C, z0 * pp + cxy, rc);
        if (DIM == 3) {
            RawCell<Ph, T> rm;
            const long long om = (z0 == 0) ? patches[patches[k].nbr[4]].off : offc;
            const int zm = (z0 == 0) ? p - 1 : z0 - 1;
            issue_load<Ph>(qin, ex, om, C, zm * pp + cxy, rm);
            issue_load<Ph>(qin, ex, own_plane_off(z0 + 1), C, own_plane_c(z0 + 1), rnA);
            double qm[N], am[AA], fzm[N];
            unpack<Ph>(rm, qm, e);
            // The face below the run's first plane is evaluated as the faces
            // inside a run: the z fluxes are rounded before they are added,
            // whichever products the compiler would fuse into the sum here or
            // there, so that a seam changes no bit of the results.
            ph.aux(qm, e, am);
            phys_flux_or_zero<Ph, DZ>(ph, qm, am, fzm);
            flux_as_rounded<Ph>(fzm);
            unpack<Ph>(rc, qc, e);
            ph.aux(qc, e, ac);
            phys_flux_or_zero<Ph, DZ>(ph, qc, ac, fzc);
            flux_as_rounded<Ph>(fzc);
            lzc = ph.template eig<DZ>(qc, ac);
            rusanov_face2<Ph, DZ>(ph, qm, fzm, ph.template eig<DZ>(qm, am), qc, fzc, lzc, fs2l, dn2l);
        } else {
            unpack<Ph>(rc, qc, e);
            ph.aux(qc, e, ac);
        }
    }
    if (work) {
        halo_load(hoffc, z0, hrA);
    }

    // run plane i (at zl of the current patch): consumes rn (own plane i+1)
    // and hr (halo of plane i), then refills them with planes i+2 and i+1,
    // clamped to the plane after the run and to the run's last plane
    auto plane = [&](int i, RawCell<Ph, T> &rn, RawCell<Ph, T> &hr, Carry &cur, Carry &nxt) {
        const double *qc = cur.q, *ac = cur.a, *fzc = cur.fz, *fs2l = cur.fs, *dn2l = cur.dn;
        const double lzc = cur.lz;
        double(*buf)[PH * PH] = lds[parity];
        parity ^= 1;
        double hq[N], he[1];
        unpack<Ph>(hr, hq, he);
        {
            const int zh = zl + min(1, n - 1 - i);
            halo_load(zh >= p ? hoffn : hoffc, zh >= p ? zh - p : zh, hr);
        }
        if (halo) {
            double ha[AA];
            ph.aux(hq, he, ha);
#pragma unroll
            for (int v = 0; v < N; ++v) buf[v][hdst] = hq[v];
#pragma unroll
            for (int j = 0; j < AP; ++j) buf[N + j][hdst] = ha[PlaneAux<Ph>::idx(j)];
        }
        if (active) {
#pragma unroll
            for (int v = 0; v < N; ++v) buf[v][li] = qc[v];
#pragma unroll
            for (int j = 0; j < AP; ++j) buf[N + j][li] = ac[PlaneAux<Ph>::idx(j)];
        }
        lds_barrier();   // (no thread reads what another writes to global memory)
        double acc2[N];
#pragma unroll
        for (int v = 0; v < N; ++v) acc2[v] = 0.0;
        if (active) {
            {
                double qL[N], aL[AA], qR[N], aR[AA];
#pragma unroll
                for (int v = 0; v < N; ++v) { qL[v] = buf[v][li - 1]; qR[v] = buf[v][li + 1]; }
#pragma unroll
                for (int a = 0; a < AA; ++a) { aL[a] = 0.0; aR[a] = 0.0; }
#pragma unroll
                for (int j = 0; j < AP; ++j) {
                    aL[PlaneAux<Ph>::idx(j)] = buf[N + j][li - 1];
                    aR[PlaneAux<Ph>::idx(j)] = buf[N + j][li + 1];
                }
                rusanov_pair2<Ph, 0>(ph, qL, aL, qc, ac, qR, aR, acc2);
            }
            {
                double qL[N], aL[AA], qR[N], aR[AA];
#pragma unroll
                for (int v = 0; v < N; ++v) { qL[v] = buf[v][li - PH]; qR[v] = buf[v][li + PH]; }
#pragma unroll
                for (int a = 0; a < AA; ++a) { aL[a] = 0.0; aR[a] = 0.0; }
#pragma unroll
                for (int j = 0; j < AP; ++j) {
                    aL[PlaneAux<Ph>::idx(j)] = buf[N + j][li - PH];
                    aR[PlaneAux<Ph>::idx(j)] = buf[N + j][li + PH];
                }
                rusanov_pair2<Ph, 1>(ph, qL, aL, qc, ac, qR, aR, acc2);
            }
        }
        // the next plane's primitives, flux and speed, after the x and y
        // directions: fewer values are live at once (3 waves per SIMD)
        double *qn = nxt.q, *an = nxt.a, *fzn = nxt.fz;
        double &lzn = nxt.lz;
        lzn = 0.0;
        if (DIM == 3) {
            unpack<Ph>(rn, qn, e);
            const int z2 = zl + min(2, n - i);
            issue_load<Ph>(qin, ex, own_plane_off(z2), C, own_plane_c(z2), rn);
            ph.aux(qn, e, an);
            phys_flux_or_zero<Ph, DZ>(ph, qn, an, fzn);
            flux_as_rounded<Ph>(fzn);   // (see the first plane)
            lzn = ph.template eig<DZ>(qn, an);
        }
        if (active) {
            if (DIM == 3) {
                double *fs2u = nxt.fs, *dn2u = nxt.dn;
                rusanov_face2<Ph, DZ>(ph, qc, fzc, lzc, qn, fzn, lzn, fs2u, dn2u);
#pragma unroll
                for (int v = 0; v < N; ++v) acc2[v] += (fs2u[v] - fs2l[v]) + (dn2u[v] + dn2l[v]);
            }
            double S[N];
            if (Ph::kSrc) {
                ph.source(qc, ac, S);
            } else {
#pragma unroll
                for (int v = 0; v < N; ++v) S[v] = 0.0;
            }
            double qw[N];
            T *dst = qout + offc * N + zl * pp + cxy;
#pragma unroll
            for (int v = 0; v < N; ++v) {
                const double nv = v < N - Ph::M ? qc[v] - hr_ * acc2[v] + dt * S[v] : qc[v];   // material: carried
                const T st = (T)nv;
                __builtin_nontemporal_store(st, dst + (long long)v * C);
                qw[v] = (double)st;
                bad |= !isfinite(qw[v]);
            }
            if (kLam) cell_speeds_fast<Ph, DIM>(ph, qw, lm);
        }
    };
    // after plane i: the run continues in the +z neighbour at the patch's top
    // (already the source of the loads issued for its first planes)
    auto advance = [&](int i) {
        if (DIM == 3 && ++zl == p && i + 1 < n) {
            if (chain.seen) {
                count_patch(ctrl, chain, kc, bad);
                bad = false;
                kc = kn;
            }
            zl = 0;
            offc = offn;
            hoffc = hoffn;
            hr_ = 0.5 * dt * patches[kn].inv_dx;
            kn = patches[kn].nbr[5];
            offn = patches[kn].off;
            hoffn = halo_off(kn);
        }
    };

    int i = 0;
    for (; i + 1 < n; i += 2) {
        plane(i, rnA, hrA, cA, cB);
        advance(i);
        plane(i + 1, rnA, hrA, cB, cA);
        advance(i + 1);
    }
    if (i < n) plane(i, rnA, hrA, cA, cB);
    if (DIM == 3 && chain.seen) {
        count_patch(ctrl, chain, kc, bad);
        bad = false;
    }
    };

    if (DIM == 3 && plan.runs) {
        const int4 r = plan.runs[unit];
        segment(r.x, r.y, r.z);
    } else if (DIM == 3 && plan.planes > 0) {
        // balanced mode: a contiguous run of planes (every patch has p planes)
        const int p = patches[0].p;
        const long long G = plan.n_units;
        long long s = plan.planes * unit / G;
        const long long s1 = plan.planes * (unit + 1) / G;
        while (s < s1) {
            const int k = (int)(s / p);
            const int za = (int)(s - (long long)k * p);
            const int zb = (int)min((long long)p, za + (s1 - s));
            segment(k, za, zb - za);
            s += zb - za;
        }
    } else {
        const int k = unit / plan.n_slabs, sl = unit - k * plan.n_slabs;
        const int p = patches[k].p;
        const int z0 = (DIM == 3) ? sl * plan.slab : 0;
        const int z1 = (DIM == 3) ? min(p, z0 + plan.slab) : 1;
        segment(k, min(z0, z1), max(0, z1 - z0));
    }
    finish_step<DIM, kLam, kWave * WV>(ctrl, slot_in, dt, lm, bad, chain);
}

// ---------------------------------------------------------------------------
// DMA-fed variant of the same step (3D, no extra per-cell input, p a
// multiple of 4): the state planes do not pass through registers.  Each
// plane of the slab (interior p x p cells and the four face-halo strips read
// from the neighbours) is copied HBM/L2 -> LDS by the gfx950 global->LDS DMA
// loads three planes ahead into a ring of four plane buffers, so about three
// planes of loads per work-group are always in flight and the waves only
// compute.  Interior and +-y strips move in 16-byte pieces, the strided
// +-x strips as 4-byte words.  Per plane z the work-group
//   1. writes the aux of its cells (computed one plane earlier) and of the
//      halo cells (computed now from the halo strips in LDS) to LDS;
//   2. waits for the DMA of plane z+1 (exact vmcnt: only the DMA and stores
//      issued after it may still be in flight) and meets at a bare barrier;
//   3. issues the DMA of plane z+3 into the buffer plane z-1 used;
//   4. evaluates the faces and updates the cell exactly as fv_step_kernel.
// The plane loop is dispatched on z % 4 to four copies of the body, each
// naming its buffers statically, so the compiler can tell the ring's buffers
// apart and does not wait for DMA into a buffer it is not reading.
namespace {

constexpr int kDmaNP = kFvPmax * kFvPmax + 4 * kFvPmax;   // slots per unknown and plane

// the wave index, as a value the compiler knows is the same in every lane
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

// wait until at most n of this wave's vector-memory operations are in flight
__device__ __forceinline__ void wait_vm(int n)
{
    switch (n) {
    case 0: __builtin_amdgcn_s_waitcnt(0x0070); break;
    case 1: __builtin_amdgcn_s_waitcnt(0x0071); break;
    case 2: __builtin_amdgcn_s_waitcnt(0x0072); break;
    case 3: __builtin_amdgcn_s_waitcnt(0x0073); break;
    case 4: __builtin_amdgcn_s_waitcnt(0x0074); break;
    case 5: __builtin_amdgcn_s_waitcnt(0x0075); break;
    case 6: __builtin_amdgcn_s_waitcnt(0x0076); break;
    case 7: __builtin_amdgcn_s_waitcnt(0x0077); break;
    case 8: __builtin_amdgcn_s_waitcnt(0x0078); break;
    case 9: __builtin_amdgcn_s_waitcnt(0x0079); break;
    case 10: __builtin_amdgcn_s_waitcnt(0x007a); break;
    case 11: __builtin_amdgcn_s_waitcnt(0x007b); break;
    case 12: __builtin_amdgcn_s_waitcnt(0x007c); break;
    case 13: __builtin_amdgcn_s_waitcnt(0x007d); break;
    case 14: __builtin_amdgcn_s_waitcnt(0x007e); break;
    default: __builtin_amdgcn_s_waitcnt(0x007f); break;   // 15 (larger counts are clamped down: still safe)
    }
}

// the bare work-group barrier (no memory fence: callers wait for what they need)
__device__ __forceinline__ void bare_barrier() { __asm__ volatile("s_barrier" ::: "memory"); }

// DMA of one plane (plane index zl inside the source patch `own` for the
// interior; the halo strips from the face neighbours) into buf[N][kDmaNP].
// Jobs: per unknown `ji` interior pieces of 1 KB, one +-x job, one +-y job;
// job k runs on wave k % 4.  Every wave issues the same number of DMA
// instructions in every plane (lanes without data are masked).
__device__ __forceinline__ void dma_plane(void *buf_v, const void *q_v, int esz, int N, long long C, int p,
                                          long long own, const long long *onb, int zl, int ji, int w)
{
    char *buf = static_cast<char *>(buf_v);
    const char *q = static_cast<const char *>(q_v);
    const int epp = 16 / esz;   // elements per 16-byte piece
    const int dpe = esz / 4;    // 4-byte words per element
    const int L = threadIdx.x & 63;
    const long long pp = (long long)p * p;
    const int J = N * (ji + 2);
    for (int k = w; k < J; k += 4) {
        const int v = k / (ji + 2), r = k - v * (ji + 2);
        char *dst = buf + (long long)v * kDmaNP * esz;
        const long long row = (long long)v * C + zl * pp;   // element offset of the plane row in a patch block
        if (r < ji) {
            const int piece = 64 * r + L;
            if (piece * epp < pp)
                dma_to_lds16(q + (own * N + row + (long long)piece * epp) * esz, dst + 1024 * r);
        } else if (r == ji) {
            const int j = L / dpe, word = L - j * dpe;
            if (j < 2 * p) {
                const int side = j / p, yy = j - side * p;
                const long long e = onb[side] * N + row + (long long)yy * p + (side == 0 ? p - 1 : 0);
                dma_to_lds4(q + e * esz + 4 * word, dst + pp * esz);
            }
        } else {
            const int pps = p / epp;   // pieces per strip
            if (L < 2 * pps) {
                const int side = L / pps, kk = L - side * pps;
                const long long e = onb[2 + side] * N + row + (long long)(side == 0 ? p - 1 : 0) * p + kk * epp;
                dma_to_lds16(q + e * esz, dst + (pp + 2 * p) * esz);
            }
        }
    }
}

}  // namespace

template <class Ph, typename T, bool kLam>
__global__ __launch_bounds__(kFvThreads, 2) void fv_step_dma_kernel(
    const T *__restrict__ qin, T *__restrict__ qout, const PatchDev *__restrict__ patches, int n_units,
    int n_slabs, int slab, int remap, Ctrl *__restrict__ ctrl, int slot_in, double dt_fixed, FvChain chain, Ph ph)
{
    constexpr int N = Ph::N, A = Ph::A, AA = A > 0 ? A : 1;
    static_assert(Ph::E == 0, "the DMA variant has no extra per-cell input");
    __shared__ T sq0[N * kDmaNP], sq1[N * kDmaNP], sq2[N * kDmaNP], sq3[N * kDmaNP];
    __shared__ double sa[2][AA][kDmaNP];

    const int t = threadIdx.x, w = wave_index();
    const int unit = remap ? xcd_remap(blockIdx.x, n_units) : (int)blockIdx.x;
    const int k = unit / n_slabs, sl = unit - k * n_slabs;
    const PatchDev P = patches[k];
    const int p = P.p;
    const long long C = (long long)p * p * p, pp = (long long)p * p;
    long long onb[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) onb[f] = patches[P.nbr[f]].off;
    const int z0 = sl * slab, z1 = min(p, z0 + slab);
    const bool work = z0 < p;
    const bool active = work && t < pp;
    const int x = active ? t % p : 0, y = active ? t / p : 0;
    const double dt = step_dt<3, kLam, (Ph::E > 0)>(ctrl, slot_in, dt_fixed, chain);
    const double hr_ = 0.5 * dt * P.inv_dx;
    // LDS slots of the cell and its four in-plane neighbours (halo strips
    // follow the p x p interior: -x, +x, -y, +y, p cells each)
    const int li = y * p + x;
    const int lxm = x == 0 ? (int)pp + y : li - 1, lxp = x == p - 1 ? (int)pp + p + y : li + 1;
    const int lym = y == 0 ? (int)pp + 2 * p + x : li - p, lyp = y == p - 1 ? (int)pp + 3 * p + x : li + p;
    // halo cells whose aux this thread evaluates: wave w serves strip w
    const int j = t & 63;
    const bool halo = work && j < p;
    const int hslot = (int)pp + w * p + j;
    // DMA instructions per wave and plane, and stores per wave and plane
    const int ji = (int)((pp * (long long)sizeof(T) + 1023) / 1024);
    const int J = N * (ji + 2);
    const int dw = (J - w + 3) / 4;
    const int sw = (64 * w < pp) ? N : 0;

    double lm[3] = {0.0, 0.0, 0.0};
    bool bad = false;
    if (work) {
        double qc[N], ac[AA], fzc[N], fs2l[N], dn2l[N], e[1] = {0.0};
        double lzc = 0.0;
        auto src_of = [&](int zz) __device__ -> long long { return zz >= p ? onb[5] : P.off; };
        auto dma = [&](int zz) __device__ {   // plane zz into ring buffer zz % 4
            T *b = (zz & 3) == 0 ? sq0 : (zz & 3) == 1 ? sq1 : (zz & 3) == 2 ? sq2 : sq3;
            dma_plane(b, qin, (int)sizeof(T), N, C, p, src_of(zz), onb, zz >= p ? zz - p : zz, ji, w);
        };
        auto d_of = [&](int zz) __device__ { return zz <= z1 ? dw : 0; };
        // the plane below the slab (for the first z face): a register load,
        // issued before the DMA so that waiting for it leaves the DMA in flight
        double qm[N];
        if (active) {
            const long long om = (z0 == 0) ? onb[4] : P.off;
            const int zm = (z0 == 0) ? p - 1 : z0 - 1;
            const T *b = qin + om * N + (long long)zm * pp + li;
#pragma unroll
            for (int v = 0; v < N; ++v) qm[v] = (double)b[(long long)v * C];
        }
        dma(z0);
        if (z0 + 1 <= z1) dma(z0 + 1);
        if (z0 + 2 <= z1) dma(z0 + 2);
        wait_vm(d_of(z0 + 1) + d_of(z0 + 2));
        bare_barrier();
        if (active) {
            const T *cb = (z0 & 3) == 0 ? sq0 : (z0 & 3) == 1 ? sq1 : (z0 & 3) == 2 ? sq2 : sq3;
#pragma unroll
            for (int v = 0; v < N; ++v) qc[v] = (double)cb[v * kDmaNP + li];
            double am[AA], fzm[N];
            ph.aux(qm, e, am);
            phys_flux_or_zero<Ph, 2>(ph, qm, am, fzm);
            ph.aux(qc, e, ac);
            phys_flux_or_zero<Ph, 2>(ph, qc, ac, fzc);
            lzc = ph.template eig<2>(qc, ac);
            rusanov_face2<Ph, 2>(ph, qm, fzm, ph.template eig<2>(qm, am), qc, fzc, lzc, fs2l, dn2l);
        }

        auto plane = [&](auto bufc, int z) __device__ {
            constexpr int B = decltype(bufc)::value;
            T *cur = B == 0 ? sq0 : B == 1 ? sq1 : B == 2 ? sq2 : sq3;
            T *nxt = B == 3 ? sq0 : B == 0 ? sq1 : B == 1 ? sq2 : sq3;
            T *prv = B == 1 ? sq0 : B == 2 ? sq1 : B == 3 ? sq2 : sq3;   // buffer of plane z-1 (= z+3)
            double(*sab)[kDmaNP] = sa[z & 1];
            // 1. aux of this plane's cells and halo cells to LDS
            if (active) {
#pragma unroll
                for (int a = 0; a < A; ++a) sab[a][li] = ac[a];
            }
            if (halo) {
                double hq[N], ha[AA];
#pragma unroll
                for (int v = 0; v < N; ++v) hq[v] = (double)cur[v * kDmaNP + hslot];
                ph.aux(hq, e, ha);
#pragma unroll
                for (int a = 0; a < A; ++a) sab[a][hslot] = ha[a];
            }
            // 2. plane z+1 landed (all but the DMA and stores issued after it)
            wait_vm(d_of(z + 2) + sw * min(2, z - z0));
            __builtin_amdgcn_s_waitcnt(0xc07f);   // this wave's LDS writes done
            bare_barrier();
            // 3. prefetch plane z+3 into the buffer plane z-1 used
            if (z + 3 <= z1)
                dma_plane(prv, qin, (int)sizeof(T), N, C, p, src_of(z + 3), onb, z + 3 >= p ? z + 3 - p : z + 3, ji, w);
            // 4. faces and update
            if (active) {
                double qn[N], an[AA], fzn[N];
#pragma unroll
                for (int v = 0; v < N; ++v) qn[v] = (double)nxt[v * kDmaNP + li];
                ph.aux(qn, e, an);
                phys_flux_or_zero<Ph, 2>(ph, qn, an, fzn);
                const double lzn = ph.template eig<2>(qn, an);
                double acc2[N];
#pragma unroll
                for (int v = 0; v < N; ++v) acc2[v] = 0.0;
                {
                    double qL[N], aL[AA], qR[N], aR[AA];
#pragma unroll
                    for (int v = 0; v < N; ++v) { qL[v] = (double)cur[v * kDmaNP + lxm]; qR[v] = (double)cur[v * kDmaNP + lxp]; }
#pragma unroll
                    for (int a = 0; a < A; ++a) { aL[a] = sab[a][lxm]; aR[a] = sab[a][lxp]; }
                    rusanov_pair2<Ph, 0>(ph, qL, aL, qc, ac, qR, aR, acc2);
                }
                {
                    double qL[N], aL[AA], qR[N], aR[AA];
#pragma unroll
                    for (int v = 0; v < N; ++v) { qL[v] = (double)cur[v * kDmaNP + lym]; qR[v] = (double)cur[v * kDmaNP + lyp]; }
#pragma unroll
                    for (int a = 0; a < A; ++a) { aL[a] = sab[a][lym]; aR[a] = sab[a][lyp]; }
                    rusanov_pair2<Ph, 1>(ph, qL, aL, qc, ac, qR, aR, acc2);
                }
                {
                    double fs2u[N], dn2u[N];
                    rusanov_face2<Ph, 2>(ph, qc, fzc, lzc, qn, fzn, lzn, fs2u, dn2u);
#pragma unroll
                    for (int v = 0; v < N; ++v) {
                        acc2[v] += (fs2u[v] - fs2l[v]) + (dn2u[v] + dn2l[v]);
                        fs2l[v] = fs2u[v];
                        dn2l[v] = dn2u[v];
                    }
                }
                double S[N];
                if (Ph::kSrc) {
                    ph.source(qc, ac, S);
                } else {
#pragma unroll
                    for (int v = 0; v < N; ++v) S[v] = 0.0;
                }
                double qw[N];
                T *dst = qout + P.off * N + (long long)z * pp + li;
#pragma unroll
                for (int v = 0; v < N; ++v) {
                    const double nv = v < N - Ph::M ? qc[v] - hr_ * acc2[v] + dt * S[v] : qc[v];   // material: carried
                    const T st = (T)nv;
                    __builtin_nontemporal_store(st, dst + (long long)v * C);
                    qw[v] = (double)st;
                    bad |= !isfinite(qw[v]);
                }
                if (kLam) cell_speeds_fast<Ph, 3>(ph, qw, lm);
#pragma unroll
                for (int v = 0; v < N; ++v) { qc[v] = qn[v]; fzc[v] = fzn[v]; }
#pragma unroll
                for (int a = 0; a < A; ++a) ac[a] = an[a];
                lzc = lzn;
            }
        };
        for (int z = z0; z < z1; ++z) {
            switch (z & 3) {
            case 0: plane(std::integral_constant<int, 0>(), z); break;
            case 1: plane(std::integral_constant<int, 1>(), z); break;
            case 2: plane(std::integral_constant<int, 2>(), z); break;
            default: plane(std::integral_constant<int, 3>(), z); break;
            }
        }
        // no DMA may still write LDS when the work-group ends
        wait_vm(0);
    }
    finish_step<3, kLam>(ctrl, slot_in, dt, lm, bad, chain);
}

// ---------------------------------------------------------------------------
// Small patches (3D, one p for the whole batch, p^3 <= 256).  The plane march
// leaves most of a work-group idle when p^2 is small (9 of 256 threads for
// p = 3).  Here a work-group takes groups of G whole patches, one thread per
// cell, and goes from group to group while the batch lasts:
//   1. every thread puts its cell's Q and aux into LDS, and (kSelf false) the
//      work-group does the same for the G * 6p^2 face-halo cells read from the
//      neighbours (the halo gather, again fused into the load).  Slots: the
//      G p^3 cells, then per patch and face the p^2 halo cells;
//   2. the loads of the next group go out, and after one barrier every thread
//      evaluates the three directions in the difference form of the plane
//      kernel from its six face neighbours, updates, stores and keeps the
//      speeds of the new state.
// kSelf: every patch is periodic on itself, so a face neighbour is a cell of
// the same patch in LDS: nothing is loaded or evaluated twice.  With one p the
// patches lie one after the other, so the group gives every address but the
// neighbours' indexes, which are loaded two groups ahead.
// Bound: vector issue and LDS, each busy 60 % of the time between the barriers.
// 8694 patches of 6^3 (1.9 M cells, 150 MB): 36 us per step with kSelf, 54 us
// (8000 of them) without, 24 us at the copy rate; one group per work-group, halo
// cells loaded and evaluated in every case: 62 us.
constexpr int kSmallHalo = 2;   // halo cells per thread, at most

// doubles per LDS slot: Q and aux of one cell side by side, so that a
// neighbour's are immediate offsets of one address; odd, so that consecutive
// slots start in different banks
template <class Ph> constexpr int kSmallSlot = (Ph::N + Ph::A) | 1;

// patches per group: as many as the threads, the halo loads and the LDS hold
template <class Ph>
int small_group(int p)
{
    const int box = (p + 2) * (p + 2) * (p + 2);
    return std::max(1, std::min({kFvThreads / (p * p * p), kSmallHalo * kFvThreads / (6 * p * p),
                                 (int)(kFvSmallLds / ((Ph::N + Ph::A) * box * sizeof(double)))}));
}

template <class Ph, typename T, bool kLam, bool kSelf>
__global__ __launch_bounds__(kFvThreads, kSelf ? 4 : 3) void fv_small_kernel(
    const T *__restrict__ qin, T *__restrict__ qout, const double *__restrict__ ex,
    const PatchDev *__restrict__ patches, int K, int p, int G, int n_groups, Ctrl *__restrict__ ctrl, int slot_in,
    double dt_fixed, FvChain chain, Ph ph)
{
    constexpr int N = Ph::N, A = Ph::A, AA = A > 0 ? A : 1, W = kFvThreads / kWave, SW = kSmallSlot<Ph>;
    extern __shared__ double box[];   // [slots][SW]
    __shared__ int sbad[2][W];
    const int t = threadIdx.x;
    const int P2 = p * p, P3 = P2 * p, HP = 6 * P2, NC = G * P3;
    const int g = t / P3, l = t - g * P3;
    const int x = l % p, y = (l / p) % p, z = l / P2;
    const double dt = step_dt<3, kLam, (Ph::E > 0)>(ctrl, slot_in, dt_fixed, chain);
    const int grid = (int)gridDim.x, first = xcd_remap(blockIdx.x, grid);

    // LDS slots of the six face neighbours (threads beyond the group's cells: slot 0)
    int nb[6];
    {
        const int c[3] = {x, y, z}, st[3] = {1, p, P2};
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const int d = f >> 1, s = f & 1, e = s ? p - 1 : 0;
            const int in = t + (s ? st[d] : -st[d]);
            const int wrap = t + (s ? -(p - 1) : p - 1) * st[d];
            const int ij = d == 0 ? z * p + y : d == 1 ? z * p + x : y * p + x;
            nb[f] = c[d] != e ? in : kSelf ? wrap : NC + (g * 6 + f) * P2 + ij;
            nb[f] = t < NC ? nb[f] * SW : 0;
        }
    }
    // this thread's halo cells (the cell of slot NC + t + 256 k): group-local
    // patch and face (index into the neighbour table), source cell
    int hpf[kSmallHalo], hcell[kSmallHalo];
    if (!kSelf) {
#pragma unroll
        for (int k = 0; k < kSmallHalo; ++k) {
            const int h = t + k * kFvThreads;
            const int gg = h / HP, r = h - gg * HP, f = r / P2, ij = r - f * P2, i = ij % p, j = ij / p;
            const int from = (f & 1) ? 0 : p - 1, d = f >> 1;
            hpf[k] = h < G * HP ? gg * 8 + f : -1;
            hcell[k] = d == 0 ? (j * p + i) * p + from : d == 1 ? (j * p + from) * p + i : (from * p + j) * p + i;
        }
    }
    // the loads in flight: this thread's cell and halo cells of the next
    // group, and the halo cells' source patches of the one after it.  Lanes
    // without a cell load the group's first one (no load sits in a divergent
    // branch).
    RawCell<Ph, T> rc, rh[kSelf ? 1 : kSmallHalo];
    int hn[kSmallHalo] = {0, 0};
    double idx = 0.0, idn = 0.0;
    auto load_nbr = [&](int grp) {
        if (kSelf) return;
#pragma unroll
        for (int k = 0; k < kSmallHalo; ++k) {
            const int gg = hpf[k] >> 3, f = hpf[k] & 7, kk = grp * G + gg;
            hn[k] = patches[hpf[k] >= 0 && kk < K ? kk : 0].nbr[hpf[k] >= 0 ? f : 0];
        }
    };
    auto load_group = [&](int grp) {
        const int k = grp * G + g;
        const bool on = t < NC && k < K;
        const long long off = (long long)(on ? k : grp * G) * P3;
        idn = patches[on ? k : grp * G].inv_dx;
        issue_load<Ph>(qin, ex, off, P3, on ? l : 0, rc);
        if (!kSelf) {
#pragma unroll
            for (int h = 0; h < kSmallHalo; ++h)
                issue_load<Ph>(qin, ex, (long long)hn[h] * P3, P3, hpf[h] >= 0 ? hcell[h] : 0, rh[h]);
        }
    };

    double lm[3] = {0.0, 0.0, 0.0};
    int grp = first;
    if (grp < n_groups) {
        load_nbr(grp);
        load_group(grp);
        load_nbr(min(grp + grid, n_groups - 1));
    }
    for (int it = 0; grp < n_groups; grp += grid, it ^= 1) {
        const int k = grp * G + g;
        const bool active = t < NC && k < K;
        double qc[N], ac[AA], e[1] = {0.0};
        unpack<Ph>(rc, qc, e);
        ph.aux(qc, e, ac);
        idx = idn;
        if (t < NC) {
#pragma unroll
            for (int v = 0; v < N; ++v) box[t * SW + v] = qc[v];
#pragma unroll
            for (int a = 0; a < A; ++a) box[t * SW + N + a] = ac[a];
        }
        if (!kSelf) {
#pragma unroll
            for (int h = 0; h < kSmallHalo; ++h) {
                if (h * kFvThreads >= G * HP) continue;   // (the same for the whole work-group)
                double hq[N], ha[AA], he[1] = {0.0};
                unpack<Ph>(rh[h], hq, he);
                ph.aux(hq, he, ha);
                if (hpf[h] >= 0) {
                    const int d = (NC + t + h * kFvThreads) * SW;
#pragma unroll
                    for (int v = 0; v < N; ++v) box[d + v] = hq[v];
#pragma unroll
                    for (int a = 0; a < A; ++a) box[d + N + a] = ha[a];
                }
            }
        }
        // (the last group is loaded again at the end, unused)
        load_group(min(grp + grid, n_groups - 1));
        load_nbr(min(grp + 2 * grid, n_groups - 1));
        lds_barrier();   // (no thread reads what another writes to global memory)
        bool bad = false;
        if (active) {
            double acc2[N];
#pragma unroll
            for (int v = 0; v < N; ++v) acc2[v] = 0.0;
            auto dirn = [&](auto D, int sl, int sr) {
                double qL[N], aL[AA], qR[N], aR[AA];
#pragma unroll
                for (int v = 0; v < N; ++v) { qL[v] = box[sl + v]; qR[v] = box[sr + v]; }
#pragma unroll
                for (int a = 0; a < A; ++a) { aL[a] = box[sl + N + a]; aR[a] = box[sr + N + a]; }
                // (one direction's reads at a time: all of them would not fit the registers)
                __builtin_amdgcn_sched_barrier(0);
                rusanov_pair2<Ph, decltype(D)::value>(ph, qL, aL, qc, ac, qR, aR, acc2);
            };
            dirn(std::integral_constant<int, 0>(), nb[0], nb[1]);
            dirn(std::integral_constant<int, 1>(), nb[2], nb[3]);
            dirn(std::integral_constant<int, 2>(), nb[4], nb[5]);
            double S[N];
            if (Ph::kSrc) {
                ph.source(qc, ac, S);
            } else {
#pragma unroll
                for (int v = 0; v < N; ++v) S[v] = 0.0;
            }
            const double hr_ = 0.5 * dt * idx;
            T *dst = qout + (long long)k * P3 * N + l;
            double qw[N];
#pragma unroll
            for (int v = 0; v < N; ++v) {
                const T st = (T)(v < N - Ph::M ? qc[v] - hr_ * acc2[v] + dt * S[v] : qc[v]);
                __builtin_nontemporal_store(st, dst + (long long)v * P3);
                qw[v] = (double)st;
                bad |= !isfinite(qw[v]);
            }
            if (kLam) cell_speeds_fast<Ph, 3>(ph, qw, lm);
        }
        // groups with a NaN or infinity are counted one by one
        const bool any = __ballot(bad) != 0;
        if ((t & (kWave - 1)) == 0) sbad[it][t / kWave] = any;
        lds_barrier();   // the group's LDS is free for the next one
        if (t == 0) {
            int b = 0;
            for (int w = 0; w < W; ++w) b |= sbad[it][w];
            if (b) atomicAdd(&ctrl->nonfinite, 1ull);
        }
    }
    finish_step<3, kLam>(ctrl, slot_in, dt, lm, false, chain);
}

// Largest speeds of the current state (first step of a call in CFL mode):
// work-group u takes patches u, u + gridDim.x, ... and stores its maxima as
// partials; work-group 0 clears slot 0 of the hand-over lines.
template <class Ph, int DIM, typename T>
__global__ __launch_bounds__(kFvThreads) void fv_lambda_kernel(const T *__restrict__ q,
                                                               const PatchDev *__restrict__ patches, int K,
                                                               double *__restrict__ part,
                                                               unsigned long long *__restrict__ lines, int n_lines,
                                                               Ph ph)
{
    constexpr int N = Ph::N, A = Ph::A;
    double lm[3] = {0.0, 0.0, 0.0};
    double e[1] = {0.0};
    for (int k = blockIdx.x; k < K; k += gridDim.x) {
        const PatchDev &P = patches[k];
        const int p = P.p;
        const long long C = (DIM == 3) ? (long long)p * p * p : (long long)p * p;
        for (long long c = threadIdx.x; c < C; c += blockDim.x) {
            double qc[N], ac[A > 0 ? A : 1];
            load_cell<Ph>(q, (const double *)nullptr, P.off, C, c, qc, e);
            ph.aux(qc, e, ac);
            cell_speeds<Ph, DIM>(ph, qc, ac, lm);
        }
    }
    store_partial<DIM>(part, lm, blockIdx.x, gridDim.x);
    if (blockIdx.x == 0 && (int)threadIdx.x < n_lines) {
#pragma unroll
        for (int d = 0; d < 3; ++d) lines[16 * threadIdx.x + d] = 0ull;
    }
}

// two ranges of words to zero with vector stores (no memset node, so this is
// safe inside captured graphs)
__global__ void zero_kernel(unsigned *a, int na, unsigned *b, int nb)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < na + nb; i += gridDim.x * blockDim.x)
        (i < na ? a[i] : b[i - na]) = 0u;
}

// ------------------------------------------------------------------ host --

// (cached per device)
pb_status device_cus(int *out)
{
    static std::mutex mu;
    static std::vector<std::pair<int, int>> cache;
    int dev = 0;
    PB_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> g(mu);
    for (const auto &e : cache)
        if (e.first == dev) { *out = e.second; return PB_OK; }
    int cus = 0;
    PB_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    cache.push_back({dev, std::max(1, cus)});
    *out = std::max(1, cus);
    return PB_OK;
}

FvChain fv_chain(const pb_batch *b, int step, double cfl, bool by_patch)
{
    const WsLayout L = ws_layout(b->pde, b->dim, b->h, b->total_cells, b->N, b->storage, b->K);
    // the set alternates with the state buffer that the step reads
    auto set = [&](int i) { return reinterpret_cast<unsigned *>(b->ws + L.seen) + (size_t)i * seen_words(b->K); };
    return FvChain{step, cfl, b->dxmin, reinterpret_cast<unsigned long long *>(b->ws + L.lines), L.n_lines,
                   reinterpret_cast<const double *>(b->ws + L.part),
                   b->pde == PB_PDE_SRHD ? c2p_units(b) : std::min(b->K, kLamUnits),
                   by_patch ? set(b->cur ^ (step & 1)) : nullptr, set(b->cur ^ (step & 1) ^ 1), seen_words(b->K)};
}

// Waves of a plane-march work-group: as many as the largest plane fills, so
// that small planes don't hold registers and LDS for waves without cells.
// What bounds these planes is the chain from barrier to barrier, and more
// work-groups per CU overlap more of them.  Five steps of 693 patches, us with
// always four waves and with this, FP64: 13^3 234 and 227, 11^3 171 and 160,
// 9^3 138 and 122, 7^3 96 and 70; FP32 storage: 204 and 172, 150 and 117, 128
// and 93, 95 and 67.  The halo cells are then one wave's, each lane with a
// neighbour of its own: 32-bit offsets keep that in registers (with 64-bit ones
// 24 to 70 spilled, and 13^3 in FP64 took 259 us), so the state must be
// smaller than 4 GiB.  SRHD stays with four waves: two offsets per lane (the
// pressures), and its steps got slower (8^3 213 to 262 us).
static int plane_waves(const pb_batch *b)
{
    if (b->dim != 3 || b->pde == PB_PDE_SRHD) return 4;
    const size_t bytes = (size_t)b->total_cells * b->N * (b->storage == PB_STORE_FP32 ? 4 : 8);
    return bytes >> 32 ? 4 : (b->pmax * b->pmax + kWave - 1) / kWave;
}

namespace {

template <class Ph, int DIM, typename T>
pb_status launch_typed(pb_batch *b, const Ph &ph, const void *qin, void *qout, int slot_in, int step,
                       double dt_fixed, double cfl, hipStream_t s)
{
    const int slab = (DIM == 3) ? (b->fv_slab > 0 ? std::min(b->fv_slab, b->pmax) : b->pmax) : 1;
    const int n_slabs = (DIM == 3) ? (b->pmax + slab - 1) / slab : 1;
    int n_units = b->K * n_slabs;
    Ctrl *ctrl = reinterpret_cast<Ctrl *>(b->ws);
    const WsLayout L = ws_layout(b->pde, b->dim, b->h, b->total_cells, b->N, b->storage, b->K);
    // in CFL mode the steps of a call hand the speed maxima to each other
    const FvChain chain = fv_chain(b, step, cfl, DIM == 3 && b->fv_runs.w < 0);
    const T *qi = static_cast<const T *>(qin);
    T *qo = static_cast<T *>(qout);
    const double *ex = Ph::E ? reinterpret_cast<const double *>(b->ws + L.pres)
                             : nullptr;
    if constexpr (DIM == 3) {
      if (fv_small_eligible(b)) {
        const int p = b->p[0], G = small_group<Ph>(p), n_groups = (b->K + G - 1) / G;
        const size_t lds = (size_t)kSmallSlot<Ph> * G * (p * p * p + (b->self ? 0 : 6 * p * p)) * sizeof(double);
        int cus = 0;
        pb_status st = device_cus(&cus);
        if (st != PB_OK) return st;
        // work-groups that are resident at once (by registers four or three, or
        // as many as the LDS holds)
        const int per_cu = (int)std::max<size_t>(1, std::min<size_t>(b->self ? 4 : 3, (size_t)160 * 1024 / (lds + 512)));
        const int nwg = std::min(n_groups, per_cu * cus);
        const bool lam = !(dt_fixed > 0.0) && Ph::E == 0;
        auto go = [&](auto kern) {
            launch_main(b, kern, dim3(nwg), dim3(kFvThreads), lds, s, qi, qo, ex, b->d_patches, b->K, p, G, n_groups,
                        ctrl, slot_in, dt_fixed, chain, ph);
        };
        if constexpr (Ph::E > 0) {   // SRHD: dt comes from the con2prim pass
            b->self ? go(fv_small_kernel<Ph, T, false, true>) : go(fv_small_kernel<Ph, T, false, false>);
        } else if (b->self) {
            lam ? go(fv_small_kernel<Ph, T, true, true>) : go(fv_small_kernel<Ph, T, false, true>);
        } else {
            lam ? go(fv_small_kernel<Ph, T, true, false>) : go(fv_small_kernel<Ph, T, false, false>);
        }
        PB_HIP(hipGetLastError());
        return PB_OK;
      }
    }
    // the plane-march kernel: slab units, column runs along +z chains, or
    // the balanced plane schedule over the work-groups that are resident at
    // once (uniform p)
    FvPlan plan{n_units, n_slabs, slab, b->fv_xcd_remap, 0, nullptr};
    const int wv = plane_waves(b);
    auto plane_kernel = [&](auto kern) -> pb_status {
        if (DIM == 3 && b->fv_runs.d) {   // (built for the current tuning only)
            plan.runs = static_cast<const int4 *>(b->fv_runs.d);
            plan.n_units = b->fv_runs.n;
        } else if (DIM == 3 && b->fv_persist > 0 && b->uniform_p) {
            int cus = 0;
            pb_status st = device_cus(&cus);
            if (st != PB_OK) return st;
            const long long slots = (long long)b->fv_persist * cus;
            const long long planes = (long long)b->K * b->p[0];
            plan.planes = planes;
            plan.n_units = (int)std::min<long long>(slots, planes);
        }
        launch_main(b, kern, dim3(plan.n_units), dim3(kWave * wv), 0, s, qi, qo, ex, b->d_patches, plan, ctrl,
                    slot_in, dt_fixed, chain, ph);
        return PB_OK;
    };
    auto plane_waves_kernel = [&](auto lam) -> pb_status {
        constexpr bool kLam = decltype(lam)::value;
        if constexpr (DIM == 3 && Ph::E == 0) {
            switch (wv) {
            case 1: return plane_kernel(fv_step_kernel<Ph, DIM, T, kLam, 1>);
            case 2: return plane_kernel(fv_step_kernel<Ph, DIM, T, kLam, 2>);
            case 3: return plane_kernel(fv_step_kernel<Ph, DIM, T, kLam, 3>);
            }
        }
        return plane_kernel(fv_step_kernel<Ph, DIM, T, kLam, 4>);
    };
    pb_status lst = PB_OK;
    if constexpr (Ph::E > 0) {  // SRHD: dt comes from the con2prim pass
        lst = plane_waves_kernel(std::false_type());
    } else if (DIM == 3 && b->fv_dma && fv_dma_eligible(b)) {
        if (dt_fixed > 0.0)
            launch_main(b, fv_step_dma_kernel<Ph, T, false>, dim3(n_units), dim3(kFvThreads), 0, s, qi, qo,
                               b->d_patches, n_units, n_slabs, slab, b->fv_xcd_remap, ctrl, slot_in, dt_fixed,
                               chain, ph);
        else
            launch_main(b, fv_step_dma_kernel<Ph, T, true>, dim3(n_units), dim3(kFvThreads), 0, s, qi, qo,
                               b->d_patches, n_units, n_slabs, slab, b->fv_xcd_remap, ctrl, slot_in, dt_fixed,
                               chain, ph);
    } else {
        lst = dt_fixed > 0.0 ? plane_waves_kernel(std::false_type()) : plane_waves_kernel(std::true_type());
    }
    if (lst != PB_OK) return lst;
    PB_HIP(hipGetLastError());
    return PB_OK;
}

template <class Ph, int DIM, typename T>
pb_status launch_lambda_typed(pb_batch *b, const Ph &ph, const void *q, hipStream_t s)
{
    const WsLayout L = ws_layout(b->pde, b->dim, b->h, b->total_cells, b->N, b->storage, b->K);
    double *part = reinterpret_cast<double *>(b->ws + L.part);
    const int units = std::min(b->K, kLamUnits);
    hipLaunchKernelGGL((fv_lambda_kernel<Ph, DIM, T>), dim3(units), dim3(kFvThreads), 0, s, static_cast<const T *>(q),
                       b->d_patches, b->K, part, reinterpret_cast<unsigned long long *>(b->ws + L.lines), L.n_lines,
                       ph);
    PB_HIP(hipGetLastError());
    return PB_OK;
}

// dispatch on (pde, dim, storage); F is a generic lambda taking (phys, dim tag, T tag)
template <class F>
pb_status dispatch(pb_batch *b, F &&f)
{
    const bool f32 = b->storage == PB_STORE_FP32;
    const double *pr = b->params.data();
    switch (b->pde) {
    case PB_PDE_ADVECTION_F: {
        AdvF ph{{pr[0], pr[1], pr[2]}, pr[3]};
        if (b->dim == 2) return f32 ? f(ph, std::integral_constant<int, 2>(), float()) : f(ph, std::integral_constant<int, 2>(), double());
        return f32 ? f(ph, std::integral_constant<int, 3>(), float()) : f(ph, std::integral_constant<int, 3>(), double());
    }
    case PB_PDE_ADVECTION_B: {
        AdvB ph{{pr[0], pr[1], pr[2]}, pr[3]};
        if (b->dim == 2) return f32 ? f(ph, std::integral_constant<int, 2>(), float()) : f(ph, std::integral_constant<int, 2>(), double());
        return f32 ? f(ph, std::integral_constant<int, 3>(), float()) : f(ph, std::integral_constant<int, 3>(), double());
    }
    case PB_PDE_ADVECTION_VAR:
        if (b->dim == 2) {
            AdvVar<2> ph{pr[0]};
            return f32 ? f(ph, std::integral_constant<int, 2>(), float()) : f(ph, std::integral_constant<int, 2>(), double());
        } else {
            AdvVar<3> ph{pr[0]};
            return f32 ? f(ph, std::integral_constant<int, 3>(), float()) : f(ph, std::integral_constant<int, 3>(), double());
        }
    case PB_PDE_EULER:
        if (b->dim == 2) {
            Euler<2> ph{pr[0]};
            return f32 ? f(ph, std::integral_constant<int, 2>(), float()) : f(ph, std::integral_constant<int, 2>(), double());
        } else {
            Euler<3> ph{pr[0]};
            return f32 ? f(ph, std::integral_constant<int, 3>(), float()) : f(ph, std::integral_constant<int, 3>(), double());
        }
    case PB_PDE_SRHD: {
        Srhd ph{pr[0]};
        if (f32) return f(ph, std::integral_constant<int, 3>(), float());
        return f(ph, std::integral_constant<int, 3>(), double());
    }
    default:
        set_error("fv_rusanov_step: PDE not supported by the finite-volume kernel");
        return PB_EUNSUPPORTED;
    }
}

}  // namespace

// Column runs: the +z link k -> s = nbr[k][+z] holds where s's -z neighbour
// is k and both patches have the same p (>= 2 for the FV march, >= 4 for the
// FD march, whose window reaches 4 planes ahead), so the march reads s's
// first planes as the continuation of k's column.  Links form chains and
// cycles; each gets a number of runs proportional to its planes (at least
// one; at most one per plane for FV, per patch for FD), about w work-groups
// per CU in total, and runs of one chain split its planes as evenly as
// integers allow.  Units are ordered layer-major: the lowest run of every
// chain (chains by their smallest patch index), then every chain's second
// run, and so on.  With the XCD remap an XCD then holds the runs of one
// height layer over a block of neighbouring chains of a grid in patch order
// (several whole rows of them), which start at equal heights, march in step
// and find their x and y neighbours' planes in the same L2.  (Chain after
// chain gave each XCD every layer of fewer chains, two rows on the headline
// grid, so half the y-halo strips came from other XCDs: HBM reads 1.48x
// the algorithmic reads instead of 1.16x.)
//
// The library's own split (`fit`; no tuning asks for another) gives a chain
// its share rounded down, so that all runs are resident at once, and lets the
// FD runs be shorter than a patch where whole patches leave CUs without work.
// Independent patches between half and all of the resident work-groups thus get
// one run each.  Ten steps of 16^3 patches with one run each and with two, us:
// 400 patches 436 and 455, 512 439 and 471, 600 570 and 541, 700 592 and 616, 767
// 621 and 655 (384: 424 and 363, and two is what they get); 13^3 520 392 and 406,
// 1000 532 and 644; 8^3 1030 217 and 193, 1500 260 and 278, 2000 302 and 325.
std::vector<int4> column_runs(int kind, int K, const int *p, const int *nbr, int w, int cus, bool fit)
{
    const int pmin = kind == 0 ? 2 : 4;
    std::vector<int> succ(K, -1), pred(K, -1);
    for (int k = 0; k < K; ++k) {
        const int s = nbr[6 * k + 5];
        if (p[k] >= pmin && p[s] == p[k] && nbr[6 * s + 4] == k) {
            succ[k] = s;
            pred[s] = k;
        }
    }
    std::vector<std::vector<int>> chains;
    std::vector<char> seen(K, 0);
    for (int k = 0; k < K; ++k) {   // open chains, from their first patch
        if (pred[k] >= 0) continue;
        chains.emplace_back();
        for (int j = k; j >= 0; j = succ[j]) {
            seen[j] = 1;
            chains.back().push_back(j);
        }
    }
    for (int k = 0; k < K; ++k) {   // cycles, from their smallest patch
        if (seen[k]) continue;
        chains.emplace_back();
        int j = k;
        do {
            seen[j] = 1;
            chains.back().push_back(j);
            j = succ[j];
        } while (j != k);
    }
    std::vector<std::pair<int, int>> order;   // (smallest patch, chain)
    for (int c = 0; c < (int)chains.size(); ++c)
        order.push_back({*std::min_element(chains[c].begin(), chains[c].end()), c});
    std::sort(order.begin(), order.end());
    long long total = 0;
    for (const auto &c : chains) total += (long long)c.size() * p[c[0]];
    const double slots = (double)w * cus;
    std::vector<std::vector<int4>> per;   // the runs of each chain, bottom to top
    size_t rm = 0;
    for (const auto &o : order) {
        const std::vector<int> &c = chains[o.second];
        const int pc = p[c[0]];
        const long long planes = (long long)c.size() * pc;
        const long long rmax = kind == 0 || fit ? planes : (long long)c.size();
        const double share = slots * (double)planes / (double)total;
        const long long r = std::max(1LL, std::min(rmax, fit ? (long long)(share + 1e-9) : std::llround(share)));
        per.emplace_back();
        for (long long j = 0; j < r; ++j) {
            const long long s0 = j * planes / r, s1 = (j + 1) * planes / r;
            per.back().push_back(make_int4(c[s0 / pc], (int)(s0 % pc), (int)(s1 - s0), 0));
        }
        rm = std::max(rm, per.back().size());
    }
    // layer-major: the first run of every chain, then every second run, ...
    std::vector<int4> runs;
    for (size_t j = 0; j < rm; ++j)
        for (const auto &v : per)
            if (j < v.size()) runs.push_back(v[j]);
    return runs;
}

// Work-groups per CU of the library's own split: as many as make three waves
// per SIMD (plane_waves), but two of single waves, whose runs get too short
// (3072 patches of 8^3, us per step: 52.8 with twelve per CU, 40.4 with eight,
// 44.4 with six; 1728 of 11^3 in FP32 with six, five, four of two waves 38, 42,
// 41).
int fv_own_per_cu(const pb_batch *b)
{
    const int waves = plane_waves(b);
    return waves == 1 ? 8 : 12 / waves;
}

namespace {

// w < 0: the library's own split, -w work-groups per CU
pb_status build_table(pb_batch *b, pb_batch::RunTable &tab, int kind, int w, bool applies)
{
    if (tab.w == w && (tab.d || w == 0 || !applies)) return PB_OK;
    tab.w = 0;
    if (tab.d) {
        PB_HIP(hipFree(tab.d));
        tab.d = nullptr;
        tab.n = 0;
    }
    if (w == 0 || !applies) {
        tab.w = w;
        return PB_OK;
    }
    int cus = 0;
    pb_status st = device_cus(&cus);
    if (st != PB_OK) return st;
    const std::vector<int4> runs = column_runs(kind, b->K, b->p.data(), b->nbr.data(), std::abs(w), cus, w < 0);
    if ((long long)runs.size() > max_units(b->K)) { set_error("column runs exceed the partial buffers"); return PB_EINVAL; }
    void *d = nullptr;
    PB_HIP(hipMalloc(&d, runs.size() * sizeof(int4)));
    if (hipMemcpy(d, runs.data(), runs.size() * sizeof(int4), hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipFree(d);
        set_error("hipMemcpy of the column runs failed");
        return PB_EHIP;
    }
    tab.d = d;
    tab.n = (int)runs.size();
    tab.w = w;
    return PB_OK;
}

}  // namespace

pb_status runs_prepare(pb_batch *b)
{
    // FV: without a tuning, runs that fill the device's three work-groups per
    // CU once.  16^3 patches, FP64, us per step with one work-group per patch
    // and with these runs: 8 patches 27.9 and 6.8, 64 28.7 and 11.0, 256 33.0
    // and 28.6, 1024 87.4 and 83.3, 2048 163 and 159; 1728 patches of 8^3 50.9
    // and 42.4; relativistic, 2048 of 16^3, 316 and 304 with the con2prim pass.
    // (Larger patches than the plane kernels take have no split of their own:
    // the batch exists, its steps are refused.)
    const bool own = b->fv_slab == 0 && b->fv_persist == 0 && b->fv_column == 0 && !b->fv_dma && !fv_small_eligible(b) &&
                     b->pde != PB_PDE_LINSYM && b->pmax <= kFvPmax;
    pb_status st = build_table(b, b->fv_runs, 0, own ? -fv_own_per_cu(b) : b->fv_column, b->dim == 3);
    if (st != PB_OK) return st;
    // (no FD table for a batch whose FD steps are refused: most of them have a
    // halo of 1; creating 2048 patches of 16^3 takes 0.1 ms less)
    const bool fd = b->dim == 3 && b->pde == PB_PDE_EULER && b->h >= 3 && b->storage == PB_STORE_FP64;
    int w = b->fd_column;
    if (fd && w == 2 && b->pmax <= kFvPmax) {
        // the default: runs shorter than a patch where the batch has fewer
        // patches than resident work-groups.  A step of 16^3 patches with
        // whole patches and with these runs: 1 patch 157 and 34 us, 64 168 and
        // 68, 256 184 and 163, 384 257 and 218 (7 planes of start-up per run
        // against CUs without work; runs of at least 2, 3 or 4 planes were no
        // better for any of these).
        int cus = 0;
        if ((st = device_cus(&cus)) != PB_OK) return st;
        if (b->K < 2 * cus) w = -2;
    }
    return build_table(b, b->fd_runs, 1, w, fd);
}

bool fv_small_eligible(const pb_batch *b)
{
    return b->dim == 3 && b->uniform_p && b->p[0] * b->p[0] * b->p[0] <= kFvThreads;
}

bool fv_dma_eligible(const pb_batch *b)
{
    if (b->dim != 3 || b->pde == PB_PDE_SRHD || b->pde == PB_PDE_LINSYM) return false;
    for (int pk : b->p)
        if (pk % 4 != 0 || pk > kFvPmax) return false;
    for (int i = 0; i < 2; ++i)
        if (reinterpret_cast<uintptr_t>(b->state[i]) % 16 != 0) return false;
    return true;
}

pb_status launch_fv_step(pb_batch *b, const void *qin, void *qout, int slot_in, int step, double dt_fixed,
                         double cfl, hipStream_t s)
{
    return dispatch(b, [&](const auto &ph, auto dimc, auto tt) -> pb_status {
        using Ph = std::decay_t<decltype(ph)>;
        using T = decltype(tt);
        constexpr int DIM = decltype(dimc)::value;
        return launch_typed<Ph, DIM, T>(b, ph, qin, qout, slot_in, step, dt_fixed, cfl, s);
    });
}

pb_status launch_fv_lambda(pb_batch *b, const void *q, hipStream_t s)
{
    return dispatch(b, [&](const auto &ph, auto dimc, auto tt) -> pb_status {
        using Ph = std::decay_t<decltype(ph)>;
        using T = decltype(tt);
        constexpr int DIM = decltype(dimc)::value;
        if constexpr (Ph::E > 0) {
            set_error("internal: SRHD speeds come from the con2prim pass");
            return PB_EINVAL;
        } else {
            return launch_lambda_typed<Ph, DIM, T>(b, ph, q, s);
        }
    });
}

static pb_status launch_zero(pb_batch *b, bool ctrl, hipStream_t s)
{
    const WsLayout L = ws_layout(b->pde, b->dim, b->h, b->total_cells, b->N, b->storage, b->K);
    const int na = ctrl ? (int)(sizeof(Ctrl) / 4) : 0, nb = 2 * seen_words(b->K);
    hipLaunchKernelGGL(zero_kernel, dim3(std::min((na + nb + 255) / 256, 256)), dim3(256), 0, s,
                       reinterpret_cast<unsigned *>(b->ws), na, reinterpret_cast<unsigned *>(b->ws + L.seen), nb);
    PB_HIP(hipGetLastError());
    return PB_OK;
}

pb_status launch_ctrl_init(pb_batch *b, hipStream_t s) { return launch_zero(b, true, s); }

pb_status launch_seen_init(pb_batch *b, hipStream_t s) { return launch_zero(b, false, s); }

}  // namespace pb
