// 1D lines: whole SSP-RK3 steps in one launch (gfx950).
//
// A 1D grid has too little work per Runge-Kutta stage to pay for a launch:
// its gap, the read of the control record and the load latency cost more
// than the stage.  Here one launch runs all three stages of a step.  A
// workgroup owns a tile of the line and keeps it in LDS: stage s forms the
// tile's cells and REACH (2 - s) more on either side (Tile1D), so the tile
// needs nothing from its neighbours until the step is over.  The state
// alternates between U and U1 with the step parity, because neighbouring
// tiles still read the old state while a tile writes the new one.
//
// Per stage a thread first forms one midpoint flux (its six nodes and the
// Roe quantities of the middle two come from LDS), then, after a barrier,
// one cell's difference, stage update, check and Roe quantities.  Those
// (velocity, pressure, enthalpy, sqrt(rho)) are formed once per cell and
// stage, where a stage kernel without them forms them twice per midpoint
// and once more for the node flux and the check.  Every value is formed by
// the operations of the single stage, in the same order: the same bits.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>

#include "wcnst.h"
#include "wcnst_device.hpp"
#include "wcnst_host.hpp"

namespace wcnst {

// Most threads of a workgroup that holds a whole line.
template <int SYS>
constexpr int LINE_SOLO_THREADS = SYS == SYS_EULER ? 256 : 1024;

// Threads of a tile, and positions it has room for.
constexpr int tile_threads(LineTiles t)
{
    return t == LineTiles::WAVES_2 ? 2 * WAVE : (t == LineTiles::WAVES_1 ? WAVE : TILE_THREADS);
}
constexpr int tile_cap(LineTiles t)
{
    return t == LineTiles::WIDE ? LINE_CAP : (t == LineTiles::PAIR ? PAIR_CAP : tile_threads(t));
}

// Wavefronts per SIMD the tile kernels are held to (168 registers for Euler).
template <int SYS>
constexpr int LINE_WAVES = SYS == SYS_EULER ? 3 : 4;

// Doubles of one position in LDS: three stage states, the midpoint flux,
// the Roe quantities (Euler) and the node flux (MND, HWCNS).
template <int SYS, int NV, int DIFF>
struct LineLds {
    static constexpr int AUX = SYS == SYS_EULER ? 4 : 0;
    static constexpr int NODE = DIFF == DIFF_MD ? 0 : NV;
    static constexpr int PER = 4 * NV + AUX + NODE;
    double* d;
    int cap;
    int cur = 0;  // state(0): the step's start; state(1), state(2): its first two stages
    __device__ double* state(int k) const { return d + (size_t)(k == 2 ? 2 : k ^ cur) * NV * cap; }
    __device__ double* flux() const { return d + (size_t)3 * NV * cap; }
    __device__ double* aux() const { return d + (size_t)4 * NV * cap; }
    __device__ double* node() const { return d + (size_t)(4 * NV + AUX) * cap; }
};

// Position q of the state in S and, for Euler, its Roe quantities.
template <int SYS, int NV, class L>
__device__ __forceinline__ void put_position(const L& lds, double* S, int q, const double (&o)[NV],
                                             const Node<NV>& N)
{
#pragma unroll
    for (int v = 0; v < NV; ++v) S[v * lds.cap + q] = o[v];
    if constexpr (SYS == SYS_EULER) {
        double* a = lds.aux();
        a[q] = N.u;
        a[lds.cap + q] = N.p;
        a[2 * lds.cap + q] = N.H;
        a[3 * lds.cap + q] = N.s;
    }
}

// One stage of the tile, between two barriers of the caller.  Stage 2 writes the
// tile's cells to out when it is given (a tile of many), else, as the
// other stages, to LDS (in place of the first stage: ghosts still read the
// step's start at their source cell while that cell's thread writes).  bad: key of this thread's first non-physical cell
// (~0 if none); speed: CFL speed bits of its cells after stage 2.
// THREADS (0: any): every thread of so many has at most one midpoint and one
// position.
// PAIR (with THREADS, Euler): two threads a midpoint, one side each, for lines that
// leave most SIMDs a wavefront at most: a midpoint's chain (4400 cycles of a
// stage's 6200) loses three of its six interpolations, for half as many
// midpoints to a wavefront.
template <int SYS, int NV, int FLUX, int SCHEME, bool CHAR, int DIFF, int THREADS, bool PAIR>
__device__ __forceinline__ void line_stage(const Tile1D<DIFF>& T, const LineLds<SYS, NV, DIFF>& lds, int stage,
                                           double dt, long long step, const Params& P, double* __restrict__ out,
                                           unsigned long long& bad, unsigned long long& speed)
{
    constexpr int G = Tile1D<DIFF>::G;
    const int tid = (int)threadIdx.x, nt = THREADS ? THREADS : (int)blockDim.x, cap = lds.cap;
    const int a = T.A(stage), base = T.base();
    const double* S = lds.state(stage);
    double* F = lds.flux();
    double* fn = lds.node();
    const double* aux = lds.aux();
    if constexpr (PAIR) {
        const int i = tid >> 1;
        const bool right = tid & 1;
        if (i < T.faces(stage)) {
            const int q = a - G - 2 + i - base;
            double n[5][NV], f[NV];
#pragma unroll
            for (int m = 0; m < 5; ++m)
#pragma unroll
                for (int v = 0; v < NV; ++v) n[m][v] = S[v * cap + (right ? q + 5 - m : q + m)];
            Node<NV> A, B;
            A.u = aux[q + 2];
            A.H = aux[2 * cap + q + 2];
            A.s = aux[3 * cap + q + 2];
            B.u = aux[q + 3];
            B.p = aux[cap + q + 3];
            B.H = aux[2 * cap + q + 3];
            B.s = aux[3 * cap + q + 3];
            face_flux_pair<NV, FLUX, SCHEME, CHAR>(n, right, P, f,
                                                   [&](Eigen<NV>& E) { roe_average<NV>(A, B, P.gamma, E); });
            if constexpr (DIFF == DIFF_MND) {
                // (the right lane's centre is node j+1)
                double g[NV];
                node_flux<NV>(n[2], B, g);
                if (right) {
#pragma unroll
                    for (int v = 0; v < NV; ++v) fn[v * cap + i] = g[v];
                }
            }
            if (!right) {
#pragma unroll
                for (int v = 0; v < NV; ++v) F[v * cap + i] = f[v];
            }
        }
    }
    for (int i = tid; !PAIR && i < T.faces(stage); i += nt) {
        const int q = a - G - 2 + i - base;  // node j-2 of midpoint j = a - G + i
        double s[6][NV];
#pragma unroll
        for (int m = 0; m < 6; ++m)
#pragma unroll
            for (int v = 0; v < NV; ++v) s[m][v] = S[v * cap + q + m];
        RegStencil<NV> st{s};
        double f[NV];
        unsigned fb;
        if constexpr (SYS == SYS_EULER) {
            Node<NV> A, B;
            A.u = aux[q + 2];
            A.H = aux[2 * cap + q + 2];
            A.s = aux[3 * cap + q + 2];
            B.u = aux[q + 3];
            B.p = aux[cap + q + 3];
            B.H = aux[2 * cap + q + 3];
            B.s = aux[3 * cap + q + 3];
            face_flux<SYS, NV, FLUX, SCHEME, CHAR>(st, P, f, fb,
                                                   [&](Eigen<NV>& E) { roe_average<NV>(A, B, P.gamma, E); });
            if constexpr (DIFF == DIFF_MND) {
                // the flux of node j+1, which cell a + i's difference and
                // that of cell a + i - 2 take
                double g[NV];
                node_flux<NV>(s[3], B, g);
#pragma unroll
                for (int v = 0; v < NV; ++v) fn[v * cap + i] = g[v];
            }
        } else {
            face_flux<SYS, NV, FLUX, SCHEME, CHAR>(st, P, f, fb);
            if constexpr (DIFF == DIFF_MND) {
                double g[NV];
                node_flux<SYS, NV>(s[3], P, g);
                fn[i] = g[0];
            }
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) F[v * cap + i] = f[v];
        if constexpr (THREADS != 0) break;
    }
    if constexpr (DIFF == DIFF_HW) {
        // node fluxes a-2 .. b+1
        for (int i = tid; i < T.B(stage) - a + 4; i += nt) {
            const int q = a - 2 + i - base;
            double u[NV], g[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) u[v] = S[v * cap + q];
            if constexpr (SYS == SYS_EULER) {
                Node<NV> N;
                N.u = aux[q];
                N.p = aux[cap + q];
                node_flux<NV>(u, N, g);
            } else {
                node_flux<SYS, NV>(u, P, g);
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) fn[v * cap + i] = g[v];
        }
    }
    __syncthreads();
    const double* S0 = lds.state(0);
    double* So = lds.state(stage == 2 ? 1 : stage + 1);
    const int lo = out ? T.A(stage) : T.out_lo(stage), hi = out ? T.B(stage) : T.out_hi(stage);
    for (int p = lo + tid; p < hi; p += nt) {
        int c = p;
        const bool ghost = T.ghosts && (p < 0 || p >= P.nx);
        if (any_lane(ghost)) c = T.source(p, P.bc_x);
        const int k = c - a, q = c - base;
        double R[NV], u[NV], un[NV], o[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const double* f = F + v * cap + k;
            const double* g = fn + v * cap + k;
            if constexpr (DIFF == DIFF_MD) R[v] = md(P.c1x, P.c2x, P.c3x, f[0], f[1], f[2], f[3], f[4], f[5]);
            else if constexpr (DIFF == DIFF_HW)
                R[v] = hwcns(P.c1x, P.c2x, P.c3x, f[0], f[1], g[0], g[1], g[3], g[4]);
            else R[v] = mnd(P.c1x, P.c2x, P.c3x, f[0], f[1], f[2], f[3], g[0], g[2]);
            u[v] = S[v * cap + q];
            un[v] = S0[v * cap + q];
        }
        rk_combine<NV>(stage, dt, u, un, R, o);
        if (P.bc_x >= BC_REFLECT && any_lane(ghost)) {
            const int kind = T.ghosts ? ghost_kind(p, P.nx, P.bc_x) : GH_COPY;
#pragma unroll
            for (int v = 0; v < NV; ++v) o[v] = ghost_value(kind, v, 1, o[v], P.fixed_x);
        }
        Node<NV> N;
        if constexpr (SYS == SYS_EULER) node_quantities<NV>(o, P.gamma, N);
        if (out) {
#pragma unroll
            for (int v = 0; v < NV; ++v) store_agent(&out[(size_t)v * P.nx + p], o[v]);
        } else {
            put_position<SYS, NV>(lds, So, p - base, o, N);
        }
        if (p >= T.c0 && p < T.c1) {
            bool b;
            if constexpr (SYS == SYS_EULER) b = node_bad<NV>(o, N);
            else b = cell_bad<SYS, NV>(o, P);
            if (any_lane(b) && b) {
                const unsigned long long key = ((unsigned long long)(step * 3 + stage) << 36) | (unsigned long long)p;
                bad = key < bad ? key : bad;
            }
            if (stage == 2) {
                double sp;
                if constexpr (SYS == SYS_EULER) sp = node_speed<NV>(N, P);
                else sp = cell_speed<SYS, NV>(o, P);
                const unsigned long long bits = (unsigned long long)__double_as_longlong(sp);
                speed = bits > speed ? bits : speed;
            }
        }
        if constexpr (THREADS != 0) break;
    }
}

// Loads the tile's positions (cells, ghosts) from U and forms their Roe
// quantities.  (No barrier.)  THREADS: at most two positions per thread, both
// loads in flight, then the caller's (read) and the weight table.
template <int SYS, int NV, int DIFF, int THREADS, class READ>
__device__ __forceinline__ void line_load(const Tile1D<DIFF>& T, const LineLds<SYS, NV, DIFF>& lds,
                                          const double* __restrict__ U, const Params& P, const READ& read)
{
    const int base = T.base(), n = T.positions();
    const auto store = [&](int i, double (&u)[NV]) {
        const int p = base + i;
        if (P.bc_x >= BC_REFLECT && any_lane(p < 0 || p >= P.nx)) {
            const int kind = ghost_kind(p, P.nx, P.bc_x);
#pragma unroll
            for (int v = 0; v < NV; ++v) u[v] = ghost_value(kind, v, 1, u[v], P.fixed_x);
        }
        Node<NV> N;
        if constexpr (SYS == SYS_EULER) node_quantities<NV>(u, P.gamma, N);
        put_position<SYS, NV>(lds, lds.state(0), i, u, N);
    };
    const auto fetch = [&](int i, double (&u)[NV]) {
        const int p = base + i;
        int c = p;
        if (any_lane(p < 0 || p >= P.nx)) c = ghost_map(p, P.nx, P.bc_x);
#pragma unroll
        for (int v = 0; v < NV; ++v) u[v] = U[(size_t)v * P.nx + c];
    };
    if constexpr (THREADS != 0) {
        const int i = (int)threadIdx.x, k = i + THREADS;
        double u[2][NV];
        if (i < n) fetch(i, u[0]);
        if (k < n) fetch(k, u[1]);
        read();
        put_weight_table(THREADS - WAVE);
#pragma unroll 1
        for (int m = 0; m < 2; ++m) {
            if (m * THREADS + i >= n) break;
            double t[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) t[v] = m ? u[1][v] : u[0][v];
            store(m * THREADS + i, t);
        }
    } else {
        for (int i = (int)threadIdx.x; i < n; i += (int)blockDim.x) {
            double u[NV];
            fetch(i, u);
            store(i, u);
        }
    }
}

// Maximum over the wavefront of a bit pattern, in lane 63: data-parallel
// moves within and across the rows of 16 lanes (about 30 cycles a step,
// where an exchange through the LDS crossbar takes about 90).
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp_max(unsigned long long m)
{
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)m, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(m >> 32), CTRL, ROWS, 0xf, false);
    const unsigned long long o = ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
    return o > m ? o : m;
}

__device__ __forceinline__ unsigned long long line_wave_max(unsigned long long m)
{
    m = dpp_max<0x111, 0xf>(m);  // row_shr 1, 2, 4, 8: lane 15 of each row
    m = dpp_max<0x112, 0xf>(m);
    m = dpp_max<0x114, 0xf>(m);
    m = dpp_max<0x118, 0xf>(m);
    m = dpp_max<0x142, 0xa>(m);  // row_bcast 15 into rows 1 and 3
    m = dpp_max<0x143, 0xc>(m);  // row_bcast 31 into rows 2 and 3
    return m;
}

// dt of the step from (t, max CFL speed), or false at the final time.
__device__ __forceinline__ bool line_dt(const LineStep& A, double t, unsigned long long smax_bits, double& dt)
{
    const bool fin = isfinite(A.t_final);
    if (fin && A.t_final - t <= 1e-12 * A.t_final) return false;
    dt = A.fixed_dt > 0.0 ? A.fixed_dt : A.cfl / __longlong_as_double((long long)smax_bits);
    if (fin && dt > A.t_final - t) dt = A.t_final - t;
    return true;
}

// One SSP-RK3 step of tile t of a line cut every w cells: in -> out.
template <int SYS, int NV, int FLUX, int SCHEME, bool CHAR, int DIFF, bool AHEAD, LineTiles TILES>
__device__ __forceinline__ void line_tile_step(const double* __restrict__ in, double* __restrict__ out,
                                               Ctrl* __restrict__ ctrl, const Params& P, const LineStep& A, int t,
                                               int w, double* mem)
{
    const Tile1D<DIFF> T(t, w, P.nx, P.bc_x);
    const LineLds<SYS, NV, DIFF> lds{mem, tile_cap(TILES)};
    constexpr int THREADS = tile_threads(TILES);
    // Every workgroup takes the same decision from the record: an earlier
    // step's failure and the final time are fixed when the launch starts
    // (a failure in this launch has a key of this step; the status follows
    // in the next launch).  AHEAD: read with the state, in one round trip
    // (Shu-Osher 2048 cells 40.1 -> 39.3 ms); the multi-line launch, which has
    // its table entry to wait for, measured 1 % slower so.
    long long step = 0;
    double time = 0.0;
    unsigned long long key = 0, sp0 = 0, sp1 = 0, sp2 = 0;
    int done = 0, status = 0;
    const auto record = [&]() {
        const StepRec* cur = &ctrl->rec[A.parity];
        step = cur->step;
        time = cur->t;
        key = ctrl->bad_key;
        sp0 = ctrl->speed[0];
        sp1 = ctrl->speed[1];
        sp2 = ctrl->speed[2];
        done = ctrl->done;
        status = ctrl->status;
    };
    if constexpr (AHEAD) {
        line_load<SYS, NV, DIFF, THREADS>(T, lds, in, P, record);
    } else {
        line_load<SYS, NV, DIFF, THREADS>(T, lds, in, P, [] {});
        record();
    }
    const bool lead = t == 0 && threadIdx.x == 0;
    if (done != 0 || status != 0) return;
    if (key != ~0ull && bad_stage_of(key, step) > 2u) {
        if (lead) ctrl->status = (int)WCNST_E_NONPHYSICAL;
        return;
    }
    const int cell = speed_slot(step), next = cell == 2 ? 0 : cell + 1, after = next == 2 ? 0 : next + 1;
    double dt;
    if (!line_dt(A, time, cell == 0 ? sp0 : (cell == 1 ? sp1 : sp2), dt)) {
        if (lead) ctrl->done = 1;
        return;
    }
    if (lead) {
        StepRec* nx = &ctrl->rec[A.parity ^ 1];
        ctrl->rec[A.parity].dt = dt;
        nx->t = time + dt;
        nx->dt = 0.0;
        nx->step = step + 1;
        nx->smax_bits = 0ull;
        ctrl->speed[after] = 0ull;
    }
    __syncthreads();
    unsigned long long bad = ~0ull, speed = 0ull;
#pragma unroll
    for (int stage = 0; stage < 3; ++stage) {
        line_stage<SYS, NV, FLUX, SCHEME, CHAR, DIFF, THREADS, TILES == LineTiles::PAIR>(
            T, lds, stage, dt, step, P, stage == 2 ? out : nullptr, bad, speed);
        __syncthreads();
    }
    if (bad != ~0ull) atomicMin(&ctrl->bad_key, bad);
    // one CFL speed per workgroup: the waves' maxima meet in LDS (the last
    // stage has read the fluxes)
    unsigned long long* red = reinterpret_cast<unsigned long long*>(lds.flux());
    speed = line_wave_max(speed);
    if ((threadIdx.x & (WAVE - 1)) == WAVE - 1) red[threadIdx.x / WAVE] = speed;
    __syncthreads();
    if (threadIdx.x == 0) {
        speed = red[0];
        for (int w = 1; w < THREADS / WAVE; ++w) speed = red[w] > speed ? red[w] : speed;
        unsigned long long* dst = &ctrl->speed[next];
        // the record only grows during the launch: a workgroup whose
        // maximum it already holds skips the atomic
        if (__hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < speed) atomicMax(dst, speed);
    }
}

template <int SYS, int NV, int FLUX, int SCHEME, bool CHAR, int DIFF, LineTiles TILES>
__global__ void __launch_bounds__(TILE_THREADS, LINE_WAVES<SYS>)
line_step(const double* __restrict__ in, double* __restrict__ out, Ctrl* __restrict__ ctrl, Params P, LineStep A,
          int width)
{
    __shared__ double mem[LineLds<SYS, NV, DIFF>::PER * tile_cap(TILES)];
    line_tile_step<SYS, NV, FLUX, SCHEME, CHAR, DIFF, true, TILES>(in, out, ctrl, P, A, (int)blockIdx.x, width, mem);
}

// A uniform pointer known to point to device memory (the statement keeps the
// two casts from cancelling).
template <class T>
__device__ __forceinline__ T* in_global(T* p)
{
    auto g = (__attribute__((address_space(1))) T*)p;
    asm("" : "+s"(g));
    return (T*)g;
}

// One step of many independent 1D Euler lines: block b takes a tile of the
// grid map[b] of the table (a search over the table without a map).
template <int FLUX, int SCHEME, bool CHAR, LineTiles TILES>
__global__ void __launch_bounds__(tile_threads(TILES), LINE_WAVES<SYS_EULER>)
line_step_multi(const ReqGrid* __restrict__ reqs, const int* __restrict__ map, int nreq, int tick_step)
{
    __shared__ double mem[LineLds<SYS_EULER, 3, DIFF_MND>::PER * tile_cap(TILES)];
    // the tiles of one XCD are one contiguous run of the table's tiles
    const int b = xcd_order((int)blockIdx.x, 0, (int)gridDim.x);
    int row = 0;
    if (map) {
        row = map[b];
    } else {
        int hi = nreq - 1;
        while (row < hi) {
            const int mid = (row + hi + 1) >> 1;
            if (reqs[mid].blk0 <= b) row = mid;
            else hi = mid - 1;
        }
    }
    ReqGrid R = reqs[row];
    // the fields the tile and its loads need, in one round trip
    asm volatile("" : "+s"(R.U), "+s"(R.U1), "+s"(R.ctrl), "+s"(R.P.nx), "+s"(R.P.bc_x), "+s"(R.blk0), "+s"(R.width),
                 "+s"(R.parity0), "+s"(R.home));
    LineStep A;
    A.t_final = R.t_final;
    A.cfl = R.cfl;
    A.fixed_dt = 0.0;
    A.parity = (R.parity0 + tick_step) & 1;
    const bool at_home = A.parity == R.home;
    // (pointers read from a table are generic; an access through one counts
    // with the LDS accesses too, and each of these would wait for all)
    double *U = in_global(R.U), *U1 = in_global(R.U1);
    line_tile_step<SYS_EULER, 3, FLUX, SCHEME, CHAR, DIFF_MND, false, TILES>(
        at_home ? U : U1, at_home ? U1 : U, in_global(R.ctrl), R.P, A, b - R.blk0, R.width, mem);
}

// Many steps of a short line in one launch: one workgroup holds the whole
// line in LDS (positions: nx + 2 REACH, `cap` of them in the dynamic LDS) and
// loops over stages and steps, with barriers only.  Up to max_steps steps
// from the current record, fewer at the final time or a failure; the state
// and the record are written back as the steps of line_step and line_settle
// leave them (a failure in the first two stages leaves the step's start).
// open: start of a call (the speed of the state at hand is formed, done
// cleared, the step counter remembered).
template <int SYS, int NV, int FLUX, int SCHEME, bool CHAR, int DIFF>
__global__ void __launch_bounds__(LINE_SOLO_THREADS<SYS>)
line_solo(double* __restrict__ U, Ctrl* __restrict__ ctrl, Params P, LineStep A, int max_steps, int open, int cap)
{
    extern __shared__ double mem[];
    __shared__ unsigned long long red[3];  // step n's maximum in red[n % 3]
    __shared__ unsigned long long first_bad;
    const int tid = (int)threadIdx.x;
    const Tile1D<DIFF> T(0, P.nx, P.nx, P.bc_x);
    LineLds<SYS, NV, DIFF> lds{mem, cap};
    line_load<SYS, NV, DIFF, 0>(T, lds, U, P, [] {});
    int p = A.parity;
    const long long step0 = ctrl->rec[p].step;
    double time = ctrl->rec[p].t, before = time, dt = 0.0;
    unsigned long long smax = ctrl->speed[speed_slot(step0)];
    if (ctrl->status != 0 || (!open && ctrl->done != 0)) {  // (one workgroup: uniform)
        if (open && tid == 0) {
            ctrl->done = 0;
            ctrl->call_step0 = max(ctrl->rec[0].step, ctrl->rec[1].step);
        }
        return;
    }
    if (tid == 0) first_bad = ~0ull;
    if (tid < 3) red[tid] = 0ull;
    init_weight_table();  // (its barrier also publishes the positions)
    const auto wg_max = [&](unsigned long long m, int slot) {
        m = line_wave_max(m);
        if ((tid & (WAVE - 1)) == WAVE - 1) atomicMax(&red[slot], m);
        __syncthreads();
        return red[slot];
    };
    if (open) {
        unsigned long long m = 0ull;
        const double* S = lds.state(0);
        for (int c = tid; c < P.nx; c += (int)blockDim.x) {
            double u[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) u[v] = S[v * cap + Tile1D<DIFF>::REACH + c];
            const unsigned long long b = (unsigned long long)__double_as_longlong(cell_speed<SYS, NV>(u, P));
            m = b > m ? b : m;
        }
        smax = wg_max(m, 2);
    }
    int n = 0, done = 0, slot = 0;
    unsigned long long key = ~0ull;
#pragma unroll 1
    while (n < max_steps) {
        if (!line_dt(A, time, smax, dt)) {
            done = 1;
            break;
        }
        unsigned long long bad = ~0ull, speed = 0ull;
        bool whole = true;
        const int next = slot == 2 ? 0 : slot + 1;
#pragma unroll
        for (int stage = 0; stage < 3; ++stage) {
            if (stage == 2 && first_bad != ~0ull) {
                whole = false;
                break;
            }
            line_stage<SYS, NV, FLUX, SCHEME, CHAR, DIFF, 0, false>(T, lds, stage, dt, step0 + n, P, nullptr, bad, speed);
            if (bad != ~0ull) atomicMin(&first_bad, bad);
            if (stage == 0 && tid == 0) red[next] = 0ull;
            if (stage < 2) __syncthreads();
        }
        before = time;
        time = time + dt;
        smax = wg_max(speed, slot);  // (its barrier publishes the last stage)
        if (whole) lds.cur ^= 1;
        slot = next;
        n += 1;
        key = first_bad;
        if (key != ~0ull) break;
    }
    const double* S = lds.state(0);
    if (n > 0)
        for (int c = tid; c < P.nx; c += (int)blockDim.x)
#pragma unroll
            for (int v = 0; v < NV; ++v) U[(size_t)v * P.nx + c] = S[v * cap + Tile1D<DIFF>::REACH + c];
    if (tid != 0) return;
    if (open) ctrl->call_step0 = step0;
    ctrl->done = done;
    if (key != ~0ull) {
        ctrl->bad_key = key;
        ctrl->status = (int)WCNST_E_NONPHYSICAL;
    }
    p ^= n & 1;
    const long long step = step0 + n;
    if (n > 0) {
        ctrl->rec[p ^ 1].t = before;
        ctrl->rec[p ^ 1].dt = dt;
        ctrl->rec[p ^ 1].step = step - 1;
        ctrl->rec[p ^ 1].smax_bits = 0ull;
        ctrl->rec[p].t = time;
        ctrl->rec[p].dt = 0.0;
        ctrl->rec[p].step = step;
    }
    ctrl->rec[p].smax_bits = smax;
    for (int k = 0; k < 3; ++k) ctrl->speed[k] = k == speed_slot(step) ? smax : 0ull;
}

// Ends a run of line steps: the newest state into U (it is in U1 when its
// parity is not `home`), the status of a failure in the last step, and the
// speed into the newest record.  A step that failed in its first or second
// stage leaves U at the step's start.  A call that took no step (one on a
// line that had failed before, or of no steps) has nothing to end: U is the
// caller's, and U1 may hold a step that was rejected.
__device__ __forceinline__ void settle_line(Ctrl* ctrl, double* __restrict__ U, const double* __restrict__ U1,
                                            size_t n, int home, int blk, int nblk)
{
    // (independent reads, issued together)
    const long long s0 = ctrl->rec[0].step, s1 = ctrl->rec[1].step, begun = ctrl->call_step0;
    const unsigned long long key = ctrl->bad_key;
    const int p = s0 >= s1 ? 0 : 1;
    const long long step = p ? s1 : s0;
    if (step == begun) return;
    // (the newest record is the one that a failed step opened)
    const int at = key != ~0ull && bad_stage_of(key, step - 1) != 2u ? p ^ 1 : p;
    if (at != home)
        for (size_t i = (size_t)blk * blockDim.x + threadIdx.x; i < n; i += (size_t)nblk * blockDim.x) U[i] = U1[i];
    if (blk == 0 && threadIdx.x == 0) {
        if (key != ~0ull) ctrl->status = (int)WCNST_E_NONPHYSICAL;
        ctrl->rec[p].smax_bits = ctrl->speed[speed_slot(step)];
    }
}

__global__ void __launch_bounds__(256) line_settle(Ctrl* ctrl, double* U, const double* U1, long long n, int home)
{
    settle_line(ctrl, U, U1, (size_t)n, home, (int)blockIdx.x, (int)gridDim.x);
}

// Grid (rows, blocks per row).
__global__ void __launch_bounds__(256) line_settle_multi(const ReqGrid* __restrict__ reqs)
{
    const ReqGrid& R = reqs[blockIdx.x];
    settle_line(R.ctrl, R.U, R.U1, (size_t)3 * R.P.nx, R.home, (int)blockIdx.y, (int)gridDim.y);
}

}  // namespace wcnst

using namespace wcnst;

// --------------------------------------------------------------- launchers

int wcnst_line_width(int diff, int nx, bool pair)
{
    if (pair) return line_tile_width<DIFF_MND, true>(nx);
    return diff == WCNST_MD ? line_tile_width<DIFF_MD>(nx)
                            : (diff == WCNST_HWCNS ? line_tile_width<DIFF_HW>(nx) : line_tile_width<DIFF_MND>(nx));
}

int wcnst_line_tiles(int diff, int nx, bool pair)
{
    const int w = wcnst_line_width(diff, nx, pair);
    return (nx + w - 1) / w;
}

// Two threads a midpoint while that leaves the launch within one workgroup
// per CU, where a step lasts as long as one wavefront's chain: 2048 cells 11.2
// -> 9.7 us, 27 000 (248 tiles) 11.1 -> 9.7; 30 000 (276) 11.4 -> 11.8, 110 000
// 14.9 -> 19.2 (Shu-Osher states; a Sod tube of 27 904 cells takes 11.3).  For
// MND: the right lane's centre node is the one whose node flux MND takes; MD and
// HWCNS lines keep a thread a midpoint, and pairs are not written for them.
bool wcnst_line_pair(long long tiles) { return tiles <= WCNST_PAIR_TILES; }

// A launch of more lines than a CU's four full tiles hold at once, all of
// which fit a workgroup of one or two wavefronts whole, takes such workgroups:
// of the four wavefronts of a full tile those lines leave two or three idle in
// their places on the CU.  Us a step, full tiles -> these: 4096 lines of 16
// cells 68.1 -> 42.8, of 56 68.7 -> 45.3, of 57 69.7 -> 57.8, of 120 84.2 ->
// 69.8; 2000 of 32 37.1 -> 26.9; 1000 lines gain nothing (18.8; 5 cells 20.2
// -> 22.5).
LineTiles wcnst_line_shape(int lines, long long pair_tiles, int longest)
{
    if (wcnst_line_pair(pair_tiles)) return LineTiles::PAIR;
    const int positions = longest + 2 * Tile1D<DIFF_MND>::REACH;
    if (lines <= 4 * WCNST_PAIR_TILES || positions > 2 * WAVE) return LineTiles::WIDE;
    return positions <= WAVE ? LineTiles::WAVES_1 : LineTiles::WAVES_2;
}

namespace {

struct LineLaunch {
    const wcnst_desc* d;
    const Params* P;
    Ctrl* ctrl;
    const double* in;
    double* out;
    LineStep A;
    hipStream_t st;
    int solo_steps = 0;  // > 0: that many steps in one workgroup, in place
    int open = 0;

    template <int SYS, int NV, int FLUX, int SCHEME, bool CHAR, int DIFF>
    void solo() const
    {
        const int cap = d->nx + 2 * Tile1D<DIFF>::REACH;
        const int threads = std::min(LINE_SOLO_THREADS<SYS>, (cap + WAVE - 1) / WAVE * WAVE);
        const size_t bytes = sizeof(double) * (size_t)cap * LineLds<SYS, NV, DIFF>::PER;
        hipLaunchKernelGGL((line_solo<SYS, NV, FLUX, SCHEME, CHAR, DIFF>), dim3(1), dim3((unsigned)threads), bytes, st,
                           out, ctrl, *P, A, solo_steps, open, cap);
    }
    template <int SYS, int NV, int FLUX, int SCHEME, bool CHAR>
    void diff() const
    {
        if (solo_steps > 0) {
            if (d->diff == WCNST_MD) solo<SYS, NV, FLUX, SCHEME, CHAR, DIFF_MD>();
            else if (d->diff == WCNST_HWCNS) solo<SYS, NV, FLUX, SCHEME, CHAR, DIFF_HW>();
            else solo<SYS, NV, FLUX, SCHEME, CHAR, DIFF_MND>();
            return;
        }
        if (d->diff == WCNST_MD) tiles<SYS, NV, FLUX, SCHEME, CHAR, DIFF_MD, false>();
        else if (d->diff == WCNST_HWCNS) tiles<SYS, NV, FLUX, SCHEME, CHAR, DIFF_HW, false>();
        else if (SYS == SYS_EULER && wcnst_line_pair(wcnst_line_tiles(d->diff, d->nx, true)))
            tiles<SYS, NV, FLUX, SCHEME, CHAR, DIFF_MND, SYS == SYS_EULER>();
        else tiles<SYS, NV, FLUX, SCHEME, CHAR, DIFF_MND, false>();
    }
    template <int SYS, int NV, int FLUX, int SCHEME, bool CHAR, int DIFF, bool PAIR>
    void tiles() const
    {
        constexpr LineTiles TILES = PAIR ? LineTiles::PAIR : LineTiles::WIDE;
        hipLaunchKernelGGL((line_step<SYS, NV, FLUX, SCHEME, CHAR, DIFF, TILES>),
                           dim3((unsigned)wcnst_line_tiles(d->diff, d->nx, PAIR)), dim3(tile_threads(TILES)), 0, st, in,
                           out, ctrl, *P, A, wcnst_line_width(d->diff, d->nx, PAIR));
    }
    template <int SYS, int NV, int FLUX, bool CHAR>
    void scheme() const
    {
        switch (d->scheme) {
        case WCNST_LINEAR: diff<SYS, NV, FLUX, SCH_LINEAR, CHAR>(); break;
        case WCNST_JS: diff<SYS, NV, FLUX, SCH_JS, CHAR>(); break;
        case WCNST_Z: diff<SYS, NV, FLUX, SCH_Z, CHAR>(); break;
        default:
            if (d->q == 6) diff<SYS, NV, FLUX, SCH_TENO, CHAR>();
            else diff<SYS, NV, FLUX, SCH_TENO_Q, CHAR>();
            break;
        }
    }
    template <int FLUX>
    void euler() const
    {
        if (d->charwise) scheme<SYS_EULER, 3, FLUX, true>();
        else scheme<SYS_EULER, 3, FLUX, false>();
    }
    void run() const
    {
        if (d->system == WCNST_ADVECTION) scheme<SYS_ADV, 1, FLUX_ROE, false>();
        else if (d->system == WCNST_BURGERS) {
            if (d->flux == WCNST_LF) scheme<SYS_BURG, 1, FLUX_LF, false>();
            else scheme<SYS_BURG, 1, FLUX_ROE, false>();
        } else if (d->flux == WCNST_LF) euler<FLUX_LF>();
        else if (d->flux == WCNST_VANLEER) euler<FLUX_VL>();
        else euler<FLUX_ROE>();
    }
};

struct MultiLaunch {
    const wcnst_desc* d;
    const ReqGrid* reqs;
    const int* map;
    int nreq, nblocks, tick_step;
    LineTiles shape;
    hipStream_t st;

    template <int FLUX, int SCHEME, bool CHAR>
    void go() const
    {
        if (shape == LineTiles::PAIR) run<FLUX, SCHEME, CHAR, LineTiles::PAIR>();
        else if (shape == LineTiles::WAVES_1) run<FLUX, SCHEME, CHAR, LineTiles::WAVES_1>();
        else if (shape == LineTiles::WAVES_2) run<FLUX, SCHEME, CHAR, LineTiles::WAVES_2>();
        else run<FLUX, SCHEME, CHAR, LineTiles::WIDE>();
    }
    template <int FLUX, int SCHEME, bool CHAR, LineTiles TILES>
    void run() const
    {
        hipLaunchKernelGGL((line_step_multi<FLUX, SCHEME, CHAR, TILES>), dim3((unsigned)nblocks),
                           dim3(tile_threads(TILES)), 0, st, reqs, map, nreq, tick_step);
    }
    template <int FLUX, bool CHAR>
    void scheme() const
    {
        switch (d->scheme) {
        case WCNST_LINEAR: go<FLUX, SCH_LINEAR, CHAR>(); break;
        case WCNST_JS: go<FLUX, SCH_JS, CHAR>(); break;
        case WCNST_Z: go<FLUX, SCH_Z, CHAR>(); break;
        default:
            if (d->q == 6) go<FLUX, SCH_TENO, CHAR>();
            else go<FLUX, SCH_TENO_Q, CHAR>();
            break;
        }
    }
    template <int FLUX>
    void chars() const
    {
        if (d->charwise) scheme<FLUX, true>();
        else scheme<FLUX, false>();
    }
};

}  // namespace

hipError_t wcnst_launch_line_step(const wcnst_desc* d, const Params& P, Ctrl* ctrl, const double* in, double* out,
                                  const LineStep& A, hipStream_t st)
{
    LineLaunch{d, &P, ctrl, in, out, A, st}.run();
    return hipGetLastError();
}

// One workgroup is ahead of a launch per step while its wavefronts have a
// SIMD each (Euler: 4; us a step of 200 cells with MD 8.95 against 10.74, HWCNS
// 9.33 against 10.95; MND 9.23 against 9.31, its tiles taking two threads a
// midpoint; 312 cells with MND 13.0 against 12.0 for tiles of one) or their
// stage is short (scalar systems: 1000 cells 5.2 us against 6.9, 1500 6.6,
// 2000 8.4).
bool wcnst_line_solo(const wcnst_desc* d)
{
    if (d->ndim != 1) return false;
    const int reach = d->diff == WCNST_MD ? Tile1D<DIFF_MD>::REACH
                                          : (d->diff == WCNST_HWCNS ? Tile1D<DIFF_HW>::REACH : Tile1D<DIFF_MND>::REACH);
    return d->nx + 2 * reach <= (d->system == WCNST_EULER ? 256 : 1536);
}

hipError_t wcnst_launch_line_solo(const wcnst_desc* d, const Params& P, Ctrl* ctrl, double* U, const LineStep& A,
                                  int steps, bool open, hipStream_t st)
{
    LineLaunch L{d, &P, ctrl, U, U, A, st};
    L.solo_steps = steps;
    L.open = open ? 1 : 0;
    L.run();
    return hipGetLastError();
}

hipError_t wcnst_launch_line_multi(const wcnst_desc* d, const void* reqs, const int* map, int nreq, int nblocks,
                                   int tick_step, LineTiles shape, hipStream_t st)
{
    const MultiLaunch L{d, (const ReqGrid*)reqs, map, nreq, nblocks, tick_step, shape, st};
    if (d->flux == WCNST_LF) L.chars<FLUX_LF>();
    else if (d->flux == WCNST_VANLEER) L.chars<FLUX_VL>();
    else L.chars<FLUX_ROE>();
    return hipGetLastError();
}

hipError_t wcnst_launch_line_settle(Ctrl* ctrl, double* U, const double* U1, long long n, int home, hipStream_t st)
{
    const long long blocks = (n + 1023) / 1024;
    hipLaunchKernelGGL(line_settle, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(256), 0, st, ctrl, U, U1, n,
                       home);
    return hipGetLastError();
}

hipError_t wcnst_launch_line_settle_multi(const void* reqs, int nreq, hipStream_t st)
{
    if (nreq <= 0) return hipSuccess;
    hipLaunchKernelGGL(line_settle_multi, dim3((unsigned)nreq, 8), dim3(256), 0, st, (const ReqGrid*)reqs);
    return hipGetLastError();
}
