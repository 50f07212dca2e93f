// pb_common.h -- internal declarations shared by the library's translation
// units (host runtime and HIP kernels).  Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cstdint>
#include <exception>
#include <new>
#include <string>
#include <tuple>
#include <vector>

#include "../../include/patchhip.h"

namespace pb {

constexpr int kWave = 64;
constexpr int kFvThreads = 256;   // one 16x16 plane per work-group
constexpr int kFvPmax = 16;

// One patch as the kernels see it (48 bytes, 16-aligned).
struct alignas(16) PatchDev {
    long long off;   // first cell of the patch (cells, not elements)
    int p;           // cells per direction
    int nbr[6];      // face neighbours -x,+x,-y,+y,-z,+z
    int pad;
    double inv_dx;   // 1 / dx
};
static_assert(sizeof(PatchDev) == 48, "PatchDev layout");

// Control block at the start of the workspace (256 bytes).
struct Ctrl {
    double dt[2];                       // step sizes, ping-ponged by step parity
    unsigned long long reserved[4];
    unsigned long long nonfinite;       // units that produced NaN/Inf
    unsigned long long c2p_cells;
    unsigned long long c2p_fail;
    unsigned long long c2p_iters;
    unsigned long long c2p_fallback;
    unsigned int c2p_maxit;
    unsigned int pad0;
    unsigned long long pad[20];
};
static_assert(sizeof(Ctrl) == 256, "Ctrl layout");

// thread-local error text
void set_error(const std::string &msg);
pb_status hip_fail(hipError_t e, const char *what);

// Every C-ABI entry point runs its body between PB_API_BEGIN and PB_API_END,
// so no C++ exception (a failed host allocation, a thread that could not
// start) crosses the C boundary: it becomes PB_ENOMEM or PB_EINVAL with a
// message.
pb_status api_fail(const char *what, pb_status st) noexcept;
#define PB_API_BEGIN try {
#define PB_API_END                                                                                    \
    }                                                                                                 \
    catch (const std::bad_alloc &) { return ::pb::api_fail("out of host memory", PB_ENOMEM); }        \
    catch (const std::exception &e_) { return ::pb::api_fail(e_.what(), PB_EINVAL); }               \
    catch (...) { return ::pb::api_fail("unexpected host error", PB_EINVAL); }

#define PB_HIP(call)                                          \
    do {                                                      \
        hipError_t e_ = (call);                               \
        if (e_ != hipSuccess) return ::pb::hip_fail(e_, #call); \
    } while (0)

// ------------------------------------------------------------ device utils

__device__ __forceinline__ double wave_max(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
    return v;
}

// the value of the lane that a DPP control selects
template <int CTRL>
__device__ __forceinline__ double dpp(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// the same in the rows of ROWS; the other rows keep their own value
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_rows(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp((int)b, (int)b, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// largest value of each eight lanes, in all of them (no LDS traffic)
__device__ __forceinline__ double max8(double v)
{
    v = fmax(v, dpp<0x141>(v));   // mirrored in the eight
    v = fmax(v, dpp<0x1b>(v));    // mirrored in the four
    return fmax(v, dpp<0xb1>(v)); // neighbours swapped
}

// largest value of a wave, in its last lane
__device__ __forceinline__ double wave_max_last(double v)
{
    v = max8(v);
    v = fmax(v, dpp<0x140>(v));                  // mirrored in the row of 16
    v = fmax(v, dpp_rows<0x142, 0xa>(v));        // last lane of rows 0, 2 to rows 1, 3
    return fmax(v, dpp_rows<0x143, 0xc>(v));     // last lane of row 1 to rows 2, 3
}

// Work-group order -> unit order such that the units one XCD runs (the
// hardware deals work-groups round-robin over the 8 XCDs) are consecutive:
// neighbouring patches then share that XCD's L2 for their halo reads.
// Global -> LDS DMA (gfx950 global_load_lds_dword / _dwordx4): every active
// lane copies 4 / 16 bytes from its global address to lds + 4 / 16 * lane.
// The destination is wave-uniform (M0).  They are issued from inline
// assembly on purpose: the compiler then does not add conservative waits for
// them before unrelated LDS reads (its alias tracking of such copies gives up
// when a kernel has many of them), and the callers wait explicitly
// (s_waitcnt vmcnt) before they read the copied data.  The instructions have
// no register results; the memory clobber keeps LDS accesses in order.
__device__ __forceinline__ unsigned lds_address(const void *p)
{
    return (unsigned)(size_t)((__attribute__((address_space(3))) const void *)p);
}

__device__ __forceinline__ void dma_to_lds16(const void *g, const void *lds)
{
    const unsigned a = __builtin_amdgcn_readfirstlane(lds_address(lds));
    __asm__ volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(a), "v"(g) : "memory", "m0");
}

__device__ __forceinline__ void dma_to_lds4(const void *g, const void *lds)
{
    const unsigned a = __builtin_amdgcn_readfirstlane(lds_address(lds));
    __asm__ volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" : : "s"(a), "v"(g) : "memory", "m0");
}

// Work-group max of lm[0..DIM) stored as this unit's partial (plain stores,
// no atomics and no fence: the kernel boundary makes them visible to the
// reduction kernel that follows).  Layout: part[d * n_units + unit].
template <int DIM>
__device__ __forceinline__ void store_partial(double *__restrict__ part, const double *lm, int unit,
                                              int n_units)
{
    __shared__ double red[3][kFvThreads / kWave];
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
        const double m = wave_max(lm[d]);
        if (lane == 0) red[d][w] = m;
    }
    __syncthreads();
    if (t < DIM) {
        double m = red[t][0];
        for (int i = 1; i < (int)(blockDim.x / kWave); ++i) m = fmax(m, red[t][i]);
        part[(long long)t * n_units + unit] = m;
    }
}

// Hand-over of the CFL maxima between the FV steps of one call, with no
// reduction kernel.  The call's first kernel stores the largest speeds of the
// starting state as at most kLamUnits partials [DIM][n_part]; step 0 reduces
// them in every work-group.  Step i folds the largest speeds of its new state
// into slot i % 3 by atomicMax on the IEEE-754 bit patterns: exact and
// independent of the order, since the maxima are >= 0 and never NaN (fmax
// from 0 drops NaN speeds) and such doubles order as their bit patterns.  Step
// i > 0 takes dt from slot (i - 1) % 3.  Both form dt = cfl / sum_d Lambda_d /
// dx_min as the reduction kernel does, and work-group 0 records it in
// ctrl->dt[slot] for the host.  Slot 0 is cleared by the call's first kernel
// and slot (i + 1) % 3 by work-group 0 of step i: last written two steps
// before and last read one step before, by kernels that have finished.
// A slot has up to kLines cache lines of its own and a work-group folds into
// one of them.  One line for everything took about 1.6 ns per atomic (42 us
// of a 116 us step of 8694 work-groups); eight lines that hold all three
// slots were no better where the work-groups read one slot while others fold
// into the next (132 us): a slot's lines are read or folded into, not both.
constexpr int kLamUnits = 1024;
constexpr int kC2pUnits = 2048;   // SRHD: partials of the con2prim pass
constexpr int kLines = 8;
struct FvChain {
    int step;
    double cfl, dxmin;
    unsigned long long *lines;   // [3 slots][n_lines][16], direction d at d
    int n_lines;                 // a power of two, at most kLines
    const double *part;          // step 0 (SRHD: every step): the partials
    int n_part;
    // one bit per patch: counted as not finite in this step, where the
    // library's own split deals a patch to several work-groups and counts by
    // patches (else null: the work-groups are counted).  The other set, the
    // next step's, is cleared.
    unsigned *seen, *seen_next;
    int n_seen;                  // words of a set
};

// counts patch k once per step if a lane of the wave saw a NaN or infinity
__device__ __forceinline__ void count_patch(Ctrl *ctrl, const FvChain &c, int k, bool bad)
{
    if (__ballot(bad) == 0 || (threadIdx.x & (kWave - 1)) != 0) return;
    const unsigned bit = 1u << (k & 31);
    if (!(atomicOr(&c.seen[k >> 5], bit) & bit)) atomicAdd(&ctrl->nonfinite, 1ull);
}

template <int DIM>
__device__ __forceinline__ double chain_dt(const double *lam, const FvChain &c)
{
    double den = 0.0;
#pragma unroll
    for (int d = 0; d < DIM; ++d) den += lam[d] / c.dxmin;
    return c.cfl / den;
}

// largest value of each row of the partials [DIM][n_part], in each of the
// work-group's T threads
template <int DIM, int T>
__device__ __forceinline__ void part_max(const FvChain &c, double *lam)
{
    __shared__ double red[DIM][T / kWave];
    const int t = threadIdx.x, lane = t & (kWave - 1);
    // eight loads per row in flight at a time: past the end the last entry again
    for (int i0 = t; i0 < c.n_part + t; i0 += 8 * T) {
        double v[DIM][8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int i = min(i0 + j * T, c.n_part - 1);
#pragma unroll
            for (int d = 0; d < DIM; ++d) v[d][j] = c.part[d * c.n_part + i];
        }
#pragma unroll
        for (int d = 0; d < DIM; ++d)
#pragma unroll
            for (int j = 0; j < 8; ++j) lam[d] = fmax(lam[d], v[d][j]);
    }
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
        lam[d] = wave_max(lam[d]);
        if (lane == 0) red[d][t / kWave] = lam[d];
    }
    __syncthreads();
#pragma unroll
    for (int d = 0; d < DIM; ++d)
#pragma unroll
        for (int w = 0; w < T / kWave; ++w) lam[d] = fmax(lam[d], red[d][w]);
}

// Adds the con2prim statistics of a step (rows 3-7 of its partials [8][n_part]:
// iterations, failures, largest iteration count, fallbacks, cells) to the
// control block; one work-group of the launch calls it.  Sums of integers
// held exactly in doubles: the order does not matter.
template <int T>
__device__ __forceinline__ void add_c2p_stats(Ctrl *ctrl, const FvChain &c)
{
    const int lane = threadIdx.x & (kWave - 1);
    for (int r = 3 + (int)threadIdx.x / kWave; r < 8; r += T / kWave) {
        double v = 0.0;
        for (int i = lane; i < c.n_part; i += kWave) {
            const double u = c.part[r * c.n_part + i];
            v = r == 5 ? fmax(v, u) : v + u;
        }
        for (int o = 32; o > 0; o >>= 1) {
            const double u = __shfl_xor(v, o, kWave);
            v = r == 5 ? fmax(v, u) : v + u;
        }
        if (lane != 0) continue;
        if (r == 3) ctrl->c2p_iters += (unsigned long long)v;
        if (r == 4) ctrl->c2p_fail += (unsigned long long)v;
        if (r == 5) ctrl->c2p_maxit = max(ctrl->c2p_maxit, (unsigned)v);
        if (r == 6) ctrl->c2p_fallback += (unsigned long long)v;
        if (r == 7) ctrl->c2p_cells += (unsigned long long)v;
    }
}

// the step's dt: fixed, from the call's starting state, handed over from the
// previous step of the call, or (kC2p: SRHD) from the partials of the con2prim
// pass before it, whose statistics work-group 0 also adds up.  Every thread of
// the work-group calls it.
template <int DIM, bool kLam, bool kC2p = false, int T = kFvThreads>
__device__ __forceinline__ double step_dt(Ctrl *ctrl, int slot_in, double dt_fixed, const FvChain &c)
{
    double lam[DIM];
#pragma unroll
    for (int d = 0; d < DIM; ++d) lam[d] = 0.0;
    if constexpr (kC2p) {
        if (blockIdx.x == 0) add_c2p_stats<T>(ctrl, c);
        if (dt_fixed > 0.0) return dt_fixed;
        part_max<DIM, T>(c, lam);
        const double dt = chain_dt<DIM>(lam, c);
        if (blockIdx.x == 0 && threadIdx.x == 0) ctrl->dt[slot_in] = dt;
        return dt;
    }
    if (!kLam) return dt_fixed;
    if (c.step == 0) {
        part_max<DIM, T>(c, lam);
    } else {
        static_assert(kLines == 8, "one line per lane of eight");
        const int lane = threadIdx.x & (kWave - 1);
        const unsigned long long *l = c.lines + 16 * ((c.step + 2) % 3 * c.n_lines + (lane & (c.n_lines - 1)));
#pragma unroll
        for (int d = 0; d < DIM; ++d) lam[d] = max8(__longlong_as_double((long long)l[d]));
    }
    return chain_dt<DIM>(lam, c);
}

// Work-group barrier for the LDS exchange only: wait for this wave's LDS
// writes, then the bare barrier instruction (the compiler memory clobber
// keeps LDS accesses on their side of it).  __syncthreads() would also wait
// for every global load and store the wave has in flight (its fence covers
// global memory), draining the prefetch of the next planes and the stores of
// the last one at every barrier.  Only for kernels in which no thread reads
// global data another thread of the launch writes.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0), vmcnt and expcnt unconstrained
    __asm__ volatile("s_barrier" ::: "memory");
}

// Classical RK4 with stage values y1 = Q0 + dt/2 k1, y2 = Q0 + dt/2 k2,
// y3 = Q0 + dt k3 and no running sum of the k: the new state is
//   Q0 + ((y1 - Q0) + 2 (y2 - Q0) + (y3 - Q0)) / 3 + dt/6 k4,
// so stages 1-3 read Q0 and write one array each, and only the last stage
// reads y1, y2 and its own y3: 13 passes over the state per step instead of
// the 16 of a running sum, with two roundings of the sum instead of four.
__device__ __forceinline__ double rk_base(double q0, double y1, double y2, double y3)
{
    return q0 + ((y1 - q0) + 2.0 * (y2 - q0) + (y3 - q0)) * (1.0 / 3.0);
}

// End of a step's work-group: counts it in ctrl->nonfinite if a lane saw a
// NaN or infinity (bad: not already counted by patches), folds its cells' largest speeds into the hand-over and
// records the step's dt for the host (see FvChain).  The exchange between the
// lanes runs on DPP moves and the one barrier waits for LDS only, so that the
// work-group's last stores drain after it has ended its own work.
template <int DIM, bool kLam, int T = kFvThreads>
__device__ __forceinline__ void finish_step(Ctrl *ctrl, int slot_in, double dt, const double *lm, bool bad,
                                            const FvChain &c)
{
    constexpr int W = T / kWave;
    __shared__ double red[DIM][W];
    __shared__ int sbad[W];
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    const bool any = __ballot(bad) != 0;
    if (lane == 0) sbad[w] = any;
    if (kLam) {
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
            const double m = wave_max_last(lm[d]);
            if (lane == kWave - 1) red[d][w] = m;
        }
    }
    lds_barrier();
    if (t == 0) {
        int b = 0;
        for (int i = 0; i < W; ++i) b |= sbad[i];
        if (b) atomicAdd(&ctrl->nonfinite, 1ull);
        if (kLam && blockIdx.x == 0) ctrl->dt[slot_in] = dt;
    }
    if (blockIdx.x == 0)
        for (int i = t; i < c.n_seen; i += T) c.seen_next[i] = 0u;
    if (kLam && t < DIM) {
        double m = red[t][0];
        for (int i = 1; i < W; ++i) m = fmax(m, red[t][i]);
        atomicMax(c.lines + 16 * (c.step % 3 * c.n_lines + (blockIdx.x & (c.n_lines - 1))) + t,
                  (unsigned long long)__double_as_longlong(m));
    }
    if (kLam && blockIdx.x == 0 && t < c.n_lines) {
#pragma unroll
        for (int d = 0; d < 3; ++d) c.lines[16 * ((c.step + 1) % 3 * c.n_lines + t) + d] = 0ull;
    }
}

__device__ __forceinline__ int xcd_remap(int bid, int n)
{
    const int q = n >> 3, r = n & 7;
    const int x = bid & 7, j = bid >> 3;
    return x * q + (x < r ? x : r) + j;
}

}  // namespace pb

// ------------------------------------------------------------------------
// Host runtime object (defined here so that every translation unit of the
// library can read it).
struct pb_batch {
    int dim = 0, K = 0, N = 0, h = 0, pde = 0, storage = 0;
    std::vector<int> p;
    std::vector<double> dx;
    std::vector<int> nbr;
    std::vector<double> params;
    void *state[2] = {nullptr, nullptr};
    int cur = 0;
    char *ws = nullptr;
    size_t ws_bytes = 0;
    hipStream_t stream = nullptr;
    long long total_cells = 0;
    double dxmin = 0.0;
    int pmax = 0;
    bool uniform_p = true;
    bool self = false;   // every patch is its own neighbour on every face
    pb::PatchDev *d_patches = nullptr;
    long long steps = 0;
    double last_dt_host = 0.0;
    // tuning
    int fv_slab = 0;
    int fv_xcd_remap = 1;
    int fd_xcd_remap = 1;
    int fd_wg_per_cu = 2;
    int fd_ws = 1;   // linear-system FD: wave-specialised kernel
    int fv_dma = 0;
    int fv_persist = 0;   // FV 3D, one p: > 0 = balanced plane schedule over this many work-groups per CU
    int fv_column = 0;    // FV 3D: > 0 = column runs along +z chains, about this many work-groups per CU
    int fd_column = 2;    // Euler FD: likewise (runs of whole patches at least); 0 = one work-group per patch
    // column-run tables (int4: patch, first plane, planes, 0; one per unit)
    // of the FV and the Euler FD plane kernels, and the w each was built for
    // (w < 0: the library's own split, fitted to the device)
    struct RunTable {
        void *d = nullptr;
        int n = 0, w = 0;
    };
    RunTable fv_runs, fd_runs;
    // SRHD guess mode
    int guess = PB_GUESS_PLAIN;
    const pb_mlp *mlp = nullptr;
    bool pres_valid = false;         // SRHD: the workspace holds a previous pressure
    // FD: tile work list (largest patches first) and the B_d matrices
    bool fd_ready = false;
    void *d_fd_mem = nullptr;        // one allocation that holds every table below
    void *d_fd_items = nullptr;
    void *d_fd_ws_items = nullptr;   // per-tile geometry of the wave-specialised kernel
    int fd_n_items = 0;
    void *d_fd_boxes = nullptr;      // 128-cell boxes of the box kernel
    int fd_n_boxes = 0;
    void *d_fd_boxA = nullptr;       // A operands of the box kernel
    double *d_fd_B = nullptr;
    double *d_fd_A = nullptr;        // A operands of the one-wave-per-tile FD kernel
    // graph cache
    struct GraphEntry {
        int kind, n_steps, parity_cur;
        double key0, key1, key2;
        int key3;
        hipGraphExec_t exec;
    };
    std::vector<GraphEntry> graphs;
    hipStream_t capture_stream = nullptr;
    int last_slot = 0;
    // event timing of the step kernels (eager mode only): one event pair per
    // launch, or in span mode one pair per run of back-to-back launches of
    // the FV step kernel (the first launch's start, the last launch's end)
    bool profiling = false, prof_span = false;
    int prof_n = 0;                 // completed event pairs
    long long prof_launches = 0;    // launches those pairs cover
    long long prof_pending = 0;     // launches of the pair still open
    std::vector<hipEvent_t> prof_ev[2];
    // events the next main-kernel launch sets from its own start and end
    // (null: that end is not recorded)
    hipEvent_t kev[2] = {nullptr, nullptr};
};

namespace pb {
// workspace sub-ranges (byte offsets), from the batch description
struct WsLayout {
    size_t ctrl = 0;       // Ctrl
    size_t part = 0;       // per-unit partials [8][units]: speeds (3), con2prim stats (5)
    size_t lines = 0;      // FV hand-over lines (FvChain), in the tail of the partials: no step uses both
    int n_lines = 0;
    size_t seen = 0;       // FvChain::seen: two sets of (K + 31) / 32 words, between the partials in use and the lines
    size_t pres = 0;       // SRHD: pressure per cell (double)
    size_t yA = 0, yB = 0; // FD: stage buffers
    size_t total = 0;
};
// the FD step's two stage buffers exist for the linear system and for 3D
// Euler batches whose halo reaches the FD stencil (h >= 3)
inline bool fd_buffers(int pde, int dim, int h)
{
    return pde == PB_PDE_LINSYM || (pde == PB_PDE_EULER && dim == 3 && h >= 3);
}
WsLayout ws_layout(int pde, int dim, int h, long long total_cells, int N, int storage, int K);
// largest number of work units any launch uses (partials are sized for it)
inline long long max_units(int K) { return (long long)K * kFvPmax; }
inline int seen_words(int K) { return (K + 31) / 32; }

// launches a step's main kernel (the FV step, an FD stage) with its arguments
// converted to the kernel's parameter types; when the batch is profiling, the
// dispatch itself sets the events it is given to its start and end
// (hipExtLaunchKernel), so a pair on one launch times the kernel alone,
// without the launch gap or the dt reduction that may follow it on the stream
template <typename... P, typename... Args>
inline void launch_main(const pb_batch *b, void (*kern)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t s,
                        Args... args)
{
    static_assert(sizeof...(P) == sizeof...(Args), "kernel argument count");
    std::tuple<P...> a{static_cast<P>(args)...};
    void *ptrs[sizeof...(P)];
    std::apply([&ptrs](auto &...x) { int i = 0; ((ptrs[i++] = static_cast<void *>(&x)), ...); }, a);
    if (b->kev[0] || b->kev[1])
        (void)hipExtLaunchKernel(reinterpret_cast<const void *>(kern), grid, block, ptrs, lds, s, b->kev[0],
                                 b->kev[1], 0);
    else
        (void)hipLaunchKernel(reinterpret_cast<const void *>(kern), grid, block, ptrs, lds, s);
}

// launchers (implemented in the kernel translation units)
// largest speeds of state q: partials for the first step of a call
pb_status launch_fv_lambda(pb_batch *b, const void *q, hipStream_t s);
// the hand-over of the batch for step `step` of a call
FvChain fv_chain(const pb_batch *b, int step, double cfl, bool by_patch);
// compute units of the current device
pb_status device_cus(int *out);
pb_status launch_fv_step(pb_batch *b, const void *qin, void *qout, int slot_in, int step, double dt_fixed,
                         double cfl, hipStream_t s);
// con2prim pass of state q: pressures, and partials (largest speeds,
// statistics) that the FV step after it reduces
pb_status launch_srhd_c2p(pb_batch *b, const void *q, hipStream_t s);
// the number of those partials per row
int c2p_units(const pb_batch *b);
// one stage of the linear system's step: `out` from Q0 and the stage input y
// (stage 0: Q0 itself); the last RK4 stage also reads the earlier stages'
// values y1 and y2, and out may be y1
pb_status launch_fd_stage(pb_batch *b, int stage, int rk_stages, const void *q0, const void *y, const void *y1,
                          const void *y2, void *out, double dt, double sigma, hipStream_t s);
// one stage of step `step` of a call of the Euler FD4 + KO6 scheme, with the
// buffers of launch_fd_stage (dt handed from step to step as in the FV path
// unless dt_fixed > 0)
pb_status launch_fd_euler_stage(pb_batch *b, int stage, int rk_stages, const void *q0, const void *y, const void *y1,
                                const void *y2, void *out, int step, double dt_fixed, double cfl, double sigma,
                                hipStream_t s);
// the whole step in one launch, where every patch is its own neighbour and
// p^3 <= 256
bool fd_self_eligible(const pb_batch *b);
pb_status launch_fd_euler_self(pb_batch *b, int rk_stages, const void *q0, void *out, int step, double dt_fixed,
                               double cfl, double sigma, hipStream_t s);
// the DMA-fed FV kernel applies to this batch (3D, no extra per-cell input,
// every p a multiple of 4, 16-byte aligned state buffers)
bool fv_dma_eligible(const pb_batch *b);
// the small-patch FV kernel applies (3D, one p, p^3 <= 256 threads); its
// work-groups take as many patches as fit 256 threads and an LDS box of
// (p+2)^3 slots of N + A doubles per patch within kFvSmallLds bytes
constexpr size_t kFvSmallLds = 64 * 1024;
bool fv_small_eligible(const pb_batch *b);
// the column runs (patch, first plane, planes, 0) of a 3D batch with
// neighbour table nbr [K][6], about w work-groups per CU on `cus` CUs.
// kind 0 (FV): links between patches of one p >= 2, runs of any length;
// kind 1 (Euler FD, halo 3): links between patches of one p >= 4, runs of
// whole patches at least.
std::vector<int4> column_runs(int kind, int K, const int *p, const int *nbr, int w, int cus, bool fit);
// work-groups per CU of the library's own split of an FV batch
int fv_own_per_cu(const pb_batch *b);
// (re)builds the column-run tables for b->fv_column and b->fd_column (a
// table is freed when its w is 0 or does not apply); host call, done when
// the batch is created and when its tuning is set, never inside a capture
pb_status runs_prepare(pb_batch *b);
// dt of an FD step: dt_fixed if > 0, else cfl / sum_d (rho(B_d) / dx_min)
double fd_dt(const pb_batch *b, double cfl, double dt_fixed);
// uploads the FD work list and B_d (library-owned; done once, before any capture)
pb_status fd_prepare(pb_batch *b);
pb_status launch_ctrl_init(pb_batch *b, hipStream_t s);
// clears both sets of FvChain::seen (after steps that did not alternate the state buffers)
pb_status launch_seen_init(pb_batch *b, hipStream_t s);
}  // namespace pb
