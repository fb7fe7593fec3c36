// Host-side helpers shared by the translation units of libwcnst.
#pragma once

#include <hip/hip_runtime.h>

#include <stddef.h>

#include "wcnst.h"

// Records a thread-local message (read by wcnst_last_error) and returns st.
wcnst_status wcnst_fail(wcnst_status st, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
wcnst_status wcnst_check_desc(const wcnst_desc* d);
int wcnst_desc_nvar(const wcnst_desc* d);
// WCNST_OK when d has the scheme parameters of a (flux, scheme, charwise,
// q, gamma, C_T, C, epsilons, difference).
wcnst_status wcnst_check_same_scheme(const wcnst_desc& a, const wcnst_desc& d);
size_t wcnst_align256(size_t b);

namespace wcnst {
struct Params;
struct Ctrl;
struct LineStep;
}
// Solver parameters of a validated descriptor (spacing, Eq. (5) coefficients).
void wcnst_make_params(const wcnst_desc* d, wcnst::Params* out);

// Multi-grid launches: bytes of one control block; reset it to t = 0 and
// accumulate the CFL speed of U (1D or 2D Euler grid d) for step 0; one
// stage of every 2D grid of a ReqGrid table (nblocks = total segments of ty
// rows).
size_t wcnst_ctrl_bytes();
hipError_t wcnst_launch_init_grid(const wcnst_desc* d, const double* U, void* ctrl, hipStream_t st);
// general: some grid of the table has reflecting / fixed sides or gravity
// (the tables then take the stage kernels that handle them).
// map (nullable): the table row of every block (wcnst_launch_block_map);
// without one each block searches the table.
struct MultiShape {
    int ty;        // rows per segment
    bool general;  // as above
    bool brief;    // whole short segments (wcnst_short_segments)
};
hipError_t wcnst_launch_multi(const wcnst_desc* d, const void* reqs, const int* map, int nreq, int nblocks, int stage,
                              int tick_step, MultiShape m, hipStream_t st);
// 1D lines.  Cells per tile and tiles (workgroups) of a line; one whole SSP-RK3 step of one
// line, in -> out, or of every 1D Euler line of a ReqGrid table (nblocks =
// total tiles), whose state alternates between U and U1 with the step
// parity; and the end of a run of steps: the newest state into U (from U1
// where the newest record's parity is not the line's home parity), the
// status of a failure in the last step, the CFL speed into the newest record.
// (pair: tiles of two threads a midpoint, MND only, for which wcnst_line_pair
// has the rule, from the launch's tiles at that width).
int wcnst_line_width(int diff, int nx, bool pair);
int wcnst_line_tiles(int diff, int nx, bool pair);
constexpr int WCNST_PAIR_TILES = 256;  // the CUs of the device this is built for
bool wcnst_line_pair(long long tiles);
// The tiles of a multi-line launch: a thread a midpoint, two, or a thread a
// midpoint in workgroups of one or two wavefronts that hold short lines whole.
enum class LineTiles { WIDE, PAIR, WAVES_1, WAVES_2 };
// The rule, from the number of lines, their tiles of two threads a midpoint
// and the longest.
LineTiles wcnst_line_shape(int lines, long long pair_tiles, int longest);
hipError_t wcnst_launch_line_step(const wcnst_desc* d, const wcnst::Params& P, wcnst::Ctrl* ctrl, const double* in,
                                  double* out, const wcnst::LineStep& A, hipStream_t st);
hipError_t wcnst_launch_line_multi(const wcnst_desc* d, const void* reqs, const int* map, int nreq, int nblocks,
                                   int tick_step, LineTiles shape, hipStream_t st);
// Whether one workgroup runs the whole line, and up to `steps` steps of it in
// one launch, in place (open: the start of a solve or step call; nothing
// else has to be launched before it).
bool wcnst_line_solo(const wcnst_desc* d);
hipError_t wcnst_launch_line_solo(const wcnst_desc* d, const wcnst::Params& P, wcnst::Ctrl* ctrl, double* U,
                                  const wcnst::LineStep& A, int steps, bool open, hipStream_t st);
hipError_t wcnst_launch_line_settle(wcnst::Ctrl* ctrl, double* U, const double* U1, long long n, int home,
                                    hipStream_t st);
hipError_t wcnst_launch_line_settle_multi(const void* reqs, int nreq, hipStream_t st);
// One persistent launch that runs the nreq 1D grids of a table to their
// final times (or max_steps more steps): per_group grids per workgroup of
// `waves` wavefronts (at most 8 each).
hipError_t wcnst_launch_persist(const wcnst_desc* d, const void* reqs, int nreq, int per_group, int waves,
                                long long max_steps, bool general, hipStream_t st);
// Fill the block map of a table of nreq rows and `total` blocks (map: total
// ints; the rows' blk0 ascending from 0).
hipError_t wcnst_launch_block_map(const void* reqs, int nreq, int total, int* map, hipStream_t st);
// true when d has sides other than periodic / zero gradient, or gravity
bool wcnst_general_bc(const wcnst_desc* d);
// Wavefronts of the current device at two per SIMD (four SIMDs per CU).
int wcnst_wave_slots();
// Rows per 2D segment (1 to 12, or a multiple of four up to 64) when the
// caller fixes none, for a launch over the grids (strips[i], rows[i]), i < n,
// on a device of `slots` wavefronts (2 per SIMD): the height minimising a
// cost fitted to measured stage times.  Never changes results.
int wcnst_auto_rows(const int* strips, const int* rows, int n, int slots);
// Rows that a workgroup takes where the caller asks for segments of ty rows:
// ty, or, of heights too low for the wavefronts of a workgroup, several
// adjoining segments where the same fit has that faster.
int wcnst_joined_rows(int ty, const int* strips, const int* rows, int n, int slots);
// Whether a launch of `groups` segments of ty rows works them whole (twelve
// wavefronts each) or by turns of four rows: the cheaper by the same fit.
bool wcnst_short_segments(long long groups, int ty, int slots);
// wcnst_launch_init_grid for every grid of a ReqGrid table (one launch).
hipError_t wcnst_launch_multi_init(int ndim, const void* reqs, int nreq, hipStream_t st);

#define WCNST_HIP_TRY(expr)                                                                \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                              \
            return wcnst_fail(WCNST_E_HIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
    } while (0)
