// Private definitions shared by the library's host and device sources.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gapsim.h"

namespace gs {

// Workgroup barrier for LDS only: __syncthreads also waits for every global load
// and store the wave has under way (their data would be visible to the other
// waves), which costs a round trip per barrier where none of it is exchanged.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int MAXM = GS_MAX_MESH;
constexpr uint32_t NO_ID = 0xFFFFFFFFu;
// fixed-point charge weights: a macroparticle is 2^F units
constexpr int F32_BITS = 24;
constexpr int F64_BITS = 44;
// tallies per gap, filled by the push and folded into the state by the field solve
enum {
  T_ABS = 0,      // [s*2 + wall], 4 entries
  T_EMIT = 4,     // [wall], 2 entries
  T_INJ = 6,
  T_PUSHED = 7,   // live particles pushed
  T_N = 8
};
// A gap's tallies, and on small grids its node sums, lie in rows: workgroups whose
// blockIdx differs modulo the rows add to different ones, and the field solve takes
// their sum.  Additions of many workgroups to one address are done one after the
// other, 24 ns each (568 workgroups adding 513 nodes: 15.1 us to one row, 4.9 us to
// four, 3.7 us to eight, while the field solve reads and clears a row more for each).
constexpr int TALLY_ROWS = 4;   // 128 bytes apart
constexpr int TALLY_ROW = 16;
constexpr int ACC_ROWS = 4;
// node k of row r, counted from ACC_ROWS times the gap's node offset: runs of 32
// nodes, so that the rows spread over the memory channels
__host__ __device__ inline int acc_row_at(int k, int r) { return (k & ~31) * ACC_ROWS + r * 32 + (k & 31); }
// Grids and contexts whose node sums have rows.  With more nodes the additions are
// bound by their number (4097 nodes, 256 workgroups: 8.8 us to one row, 7.8 to four);
// with more gaps, or fewer slots than 256 tiles of 2048, a gap has few workgroups, and
// the field solve's reads cost more (1e5 particles, 256 cells: 19.6 us a step, 19.3
// with one row; 1e6 particles, 512 cells: 28.6 and 37.6).  Gaps of 6e5 particles on 512
// cells, us a step with rows and with one: 4 gaps 34.4 and 42.4, 8 gaps 46.0 and 48.3, 16
// gaps 56.9 and 56.7; on 2500 cells 47.2 and 49.3, 51.1 and 51.4, 66.3 and 64.4.
constexpr int ACC_ROWS_NMAX = 2559, ACC_ROWS_GAPS = 8;
constexpr int64_t ACC_ROWS_SLOTS = 1 << 19;

// Per-gap constants (read-only on the device).
struct GapConst {
  int32_t N;          // cells
  int32_t M, g;       // meshes, gap mesh
  int32_t see_law, see_max;
  int32_t see_yield, pad_y;
  int32_t Z[2];
  int32_t beam_side;  // GS_BEAM_CIRCUIT or GS_BEAM_GROUND
  int64_t beam_n;     // ions per step without a schedule
  int64_t sched_base, sched_len;  // the gap's beam schedule in DevPtrs::sched (len 0: none)
  int64_t cap[2];
  int64_t pbase[2];   // first particle slot of species s
  int64_t nbase;      // offset of the node arrays (N + 1 entries)
  int64_t evbase;     // first slot of the gap's absorbed-ion event list
  int64_t evcap;      // its capacity
  int64_t ebase;      // offset of the binary32/64 field table (N + 2 entries)
  int64_t hbase[2];   // first counter of species s in the cell-sort bin arrays
                      // (room for ceil(N / SORT_BIN_MIN) bins per species)
  uint64_t seed;
  double d, dx, A, eps0, dt, cgap, c_par;
  double rdx, reps0;   // reciprocals (see div_by): 1 / dx, 1 / eps0,
  double rdt, rev, rE0, rmass[2];  // 1 / dt, 1 / ev, 1 / see_E0, 1 / mass
  double s0;           // sheet charge per unit of Z: weight * q_unit [C/m^2]
  double alpha[2];     // Z q dt^2 / (m dx): velocity change in cells/step per V/m
  double mass[2], ev;
  double see_amp, see_E0, see_E;
  double see_poly[6], see_pEmax;  // GS_YIELD_POLY: coefficients in powers of E / 1 keV, E clamp [eV]
  double see_mu, see_sig;         // GS_SEE_LOGNORMAL: ln E ~ N(mu, sig^2), E in eV
  double beam_Emin, beam_Emax;
  double beam_layer;  // [m]; 0: one step of flight
  double v_ref;
  double src_dc, src_amp, src_w, src_phase;
  // strict: D = sL h + sR D1 - sS q1 + sb Vs - sz phi0     (h = 15 D1 - 7 D2 + D3)
  double sL[MAXM * MAXM], sR[MAXM * MAXM], sS[MAXM * MAXM], sb[MAXM], sz[MAXM];
  // weak: D* = wL h + wR D1 - wS q1 + wb Vs
  double wL[MAXM * MAXM], wR[MAXM * MAXM], wS[MAXM * MAXM], wb[MAXM];
  // T' itself (loop equations in volts for the Newton residual)
  double Tp[MAXM * MAXM];
  // Newton on u = (V, I_0..I_{M-1}): the residual is affine in u, so its
  // Jacobian J is constant; Jinv row-major (M+1)^2
  double Jinv[(MAXM + 1) * (MAXM + 1)];
};

// Per-gap mutable state (device).
struct GapState {
  int64_t level;        // last solved level (-1 before the first step)
  int64_t seen_epoch;   // compaction epoch already applied to this gap
  int64_t count[2];     // slots the current push sweeps, per species
  int64_t live[2];      // live particles after the last push, per species
  int64_t next_id;      // next particle id
  int64_t beam_id0;     // id of beam particle 0 of the current push
  int64_t beam_now;     // beam ions of the current push
  double qprev[MAXM];   // loop charges q^{n-1}
  double dq[3][MAXM];   // increments D^{n-1}, D^{n-2}, D^{n-3}
  double sigma_prev, qcirc_prev;
  // u = (V, I) history for the Newton guess
  double uh[3][MAXM + 1];
  // diagnostics of the last solved level
  double t, phi0, sigma, qcirc, qcirc_star, qconv, e_ground;
  double qcirc_step;    // Q_circ* of this level minus Q_circ of the one before
  double q_space;       // A times the integral of rho over the gap at this level
  double q[MAXM], I[MAXM];
  int64_t abs_last[4], emit_last[2], inj_last, pushed_last;
  int64_t abs_cum[4], emit_cum[2], inj_cum, pushed_cum;
  int32_t newton_last, newton_fb_last;
  int64_t newton_total, newton_fallbacks;
  int32_t newton_max, newton_levels;  // most corrections at one level; Newton levels solved
  double newton_r0, newton_r;
  double guess[MAXM + 1];  // the u the last Newton solve started from
  double mlp_prop[3];      // the guess network's proposal at the last solve (used or not)
  // ring of the last 8 levels' (V, I_0, I_1, sigma, Q_abs, Q_em): the guess
  // network's input; hist_head is the slot the next level goes to
  double hist[8][6];
  int32_t hist_head, pad1;
};

// An ion absorbed by an electrode, waiting for its secondary emission.
struct Event {
  double u;       // impact velocity in cells per step
  uint32_t ref;   // in a push workgroup's LDS queue: the ion's slot in its region;
                  // in the gap's overflow list: the ion's id (a compaction may move
                  // the slot before the field kernel emits).  The id keys the draws.
  uint32_t wall;
};

// What a push reads of a gap before and while it streams the particles, written
// by the field solve: constants and the step's counts in two cache lines, so
// that a workgroup starts after one round trip instead of one per structure.
struct PushHead {
  int64_t count[2];   // slots to sweep, per species
  int64_t beam_now, beam_id0, level;
  int64_t pbase[2], nbase, ebase, evbase, evcap;
  double alpha[2];
  int32_t N, Z[2];
  int32_t see;        // absorbed ions free electrons
  int64_t pad;
};
static_assert(sizeof(PushHead) == 128, "two cache lines");

// Where a gap is read to, in pinned host memory.
struct ReadBack {
  unsigned long long tally[TALLY_ROWS * TALLY_ROW], next_count[2];
  unsigned long long umax[2];  // time-step check: largest |u| per species (bits)
  unsigned int cmax, pad;      //   most electrons in one cell
  GapState s;
};

// Context-wide device pointers handed to kernels.
struct DevPtrs {
  const GapConst *gc;
  GapState *gs;
  PushHead *head;                  // [G]
  // particle slots, two buffers selected by compaction epoch parity
  void *X[2], *U[2];
  uint32_t *ID[2];
  unsigned long long *next_count;  // [G][2] append cursor
  unsigned long long *cursor;      // [G][2] slot count after the compaction or sort in progress
  unsigned long long *tally;       // [G][TALLY_ROWS][TALLY_ROW], T_N of a row used
  unsigned long long *acc;         // node charge accumulators, int64 two's complement
  unsigned long long *acc_rows;    // more rows of them for the push's sums, or null (see acc_row_at)
  double *rho64, *E64;             // node and half-grid arrays (nbase offsets, both)
  void *ehat;                      // field table for the push, binary32 or binary64
  int64_t *epoch;                  // compaction epoch (device)
  unsigned int *err;               // [0] flags, [1] gap of first error
  unsigned int *steal;             // the push's pool counter, cleared by the field solve
  unsigned int *push_done;         // push workgroups done: a top counter and 32 group
                                   // counters, 128 bytes apart (the last resets them)
  // the field solve's hand-offs between its kernels: the prefix sums of the
  // cell terms within chunks of FCN nodes (per node), the chunks' totals and
  // weighted sums [G][NCHMAX][2], their offsets [G][NCHMAX], sigma [G]
  double *fsl, *fpart, *foff, *fsig;
  Event *ev;                       // absorbed-ion events, per-gap lists
  unsigned long long *ev_count;    // [G]
  unsigned long long *ev_done;     // [G] events of the list already emitted by k_emit
  // periodic cell sort: live particles per bin, then per-bin write cursors
  unsigned long long *hist, *bcur;
  // in-place compaction: live particles per tile (then their prefix), at
  // tcnt[pbase / 64 + k] for tile k of a region; holes below the live count
  int *tcnt;
  unsigned long long *fill_h;  // [G][2]
  unsigned long long *live;    // a bit per slot, 64 per word from pbase / 64
  int *wrank;                  // per word past the live count: tail rank of its first live slot
  const int64_t *sched;            // beam schedules of all gaps (GapConst::sched_base)
  // exchange with an external circuit engine (field mode 2), in pinned host
  // memory the device maps: ext_v[g] the engine's gap voltage for the level
  // being solved (read), ext_phi[g] the electrode potential it gave (written)
  const double *ext_v;
  double *ext_phi;
  // mapped host word: the events the last push left in the gaps' lists (an
  // upper bound when k_emit wrote it), which the host reads to choose who
  // emits the next push's lists
  unsigned long long *list_seen;
  ReadBack *rb;                    // (mapped) read-back buffer of the time-step check
  unsigned long long *dt_max;      // time-step check: largest |u| bits per species, then the
                                   // electrons per cell (zero between checks)
  Event *ovf;                      // push workgroups' events past their LDS queues: room for ovq
  int64_t ovf_wgs;                 //   events of each of ovf_wgs workgroups and for as many LDS
  int64_t ovq;                     //   queues (k_push divides it)
  // Newton guess network: bfloat16 weights (flat layout of gs_mlp_dev.h) and
  // the normalisation block; null until weights are set
  const uint16_t *mlp_w;
  const double *mlp_norm;
  // sample recording for training: level n of gap g goes to sample
  // (n - rec_level0) * G + g when that is below rec_cap
  float *rec_x;  // [rec_cap][48] raw features
  float *rec_y;  // [rec_cap][3] raw targets u* - u_extrapolated
  int64_t rec_cap, rec_level0;
};

enum { ERR_CAPACITY = 1u, ERR_BADINJECT = 2u, ERR_NOCONV = 4u };

// Nodes per chunk of the field solve's density and table kernels, and the
// chunks of the largest gap (16384 cells: nodes 0..16384).
constexpr int FCN = 1024;
constexpr int NCHMAX = 16384 / FCN + 1;

// Smallest cell-sort bin (cells per bin): bounds the bin arrays and the LDS of
// the sort kernels (16384 cells -> 4096 bins per species).
constexpr int SORT_BIN_MIN = 4;

// Absorbed-ion events a push workgroup queues in LDS.
constexpr int EVQ = 128;
// Absorbed-ion events a push workgroup keeps in its global overflow region
// (past these they go to the gap's list, emitted by k_emit after the push):
// from OVQ_MIN to OVQ_MAX, in proportion to the emitting gaps' ion slots.  A
// position in the gap's list costs each wave that needs one a returning atomic
// on the gap's counter, and at some 1e5 overflowing events a step those
// serialise; the regions are sized so that a push rarely needs the list.
constexpr int OVQ_MIN = 1024, OVQ_MAX = 8192;


struct LaunchCfg {
  int block;         // push block size
  int tile;          // particles per tile
  int grid;          // push blocks
  int nmax;          // largest n_cells of the context
  int fp64;          // particle precision
  int wide;          // binary32: 64-bit LDS deposit cells (else 32-bit cells with carries)
  int compact_grid;  // compaction blocks
  int ppt;           // particles per thread per chunk (one or two 16-byte vectors)
  int sort_bin;      // cells per bin of the periodic counting sort that replaces the
                     // compaction (0: plain compaction); with it the push queues no
                     // events past its LDS queue and k_emit emits them after the push
  int steal;         // the last 1/steal of each push workgroup's tiles go to a pool
                     // that workgroups done with their own draw from (0: none)
  int stream;        // push particle stream: STREAM_RR round-robin tile order,
                     // STREAM_NT non-temporal binary32 loads and stores
  int max_wgs;       // tiles of the regions' slots: more push blocks would find nothing to do
  int min_wgs;       // a single gap's push may use as few workgroups as this (see k_push)
  int masks;         // per launch: the push writes the live masks of the words
                     // below each region's count, and the compaction that follows
                     // takes them instead of reading those positions
  int lists;         // per launch: the push's last workgroup emits the gaps'
                     // lists of absorbed ions (else k_emit does, after the push)
};
constexpr int STREAM_RR = 1, STREAM_NT = 2;

// launchers (gs_kernels.hip)
// Optional timing: when `a` is set, the start and end of the launched kernel(s)
// are recorded into these events by the dispatch packets themselves
// (hipExtLaunchKernel), so the elapsed time holds no launch latency.
struct KTime {
  hipEvent_t a = nullptr, b = nullptr;
};

hipError_t launch_field(const DevPtrs &p, int G, int mode, int guess, double newton_tol,
                        int newton_maxit, int fp64, int nmax, hipStream_t s, KTime t = {});
hipError_t launch_push(const DevPtrs &p, int G, const LaunchCfg &lc, hipStream_t s, KTime t = {});
// its instantiations, compiled in units of their own
hipError_t launch_push_f64(const DevPtrs &p, int G, const LaunchCfg &lc, hipStream_t s, KTime t);
hipError_t launch_push_f32w(const DevPtrs &p, int G, const LaunchCfg &lc, hipStream_t s, KTime t);
hipError_t launch_push_f32c(const DevPtrs &p, int G, const LaunchCfg &lc, hipStream_t s, KTime t);
hipError_t launch_push_f32w_nt(const DevPtrs &p, int G, const LaunchCfg &lc, hipStream_t s, KTime t);
hipError_t launch_push_f32c_nt(const DevPtrs &p, int G, const LaunchCfg &lc, hipStream_t s, KTime t);
hipError_t launch_compact(const DevPtrs &p, int G, const LaunchCfg &lc, hipStream_t s, KTime t = {});
// the cell sort (count, scan, scatter, commit), in place of launch_compact
hipError_t launch_sort(const DevPtrs &p, int G, const LaunchCfg &lc, hipStream_t s, KTime t = {});
// secondary emission of every gap's queued events, many workgroups (after a push)
hipError_t launch_emit(const DevPtrs &p, int G, int fp64, int grid, hipStream_t s, KTime t = {});
hipError_t launch_inject(const DevPtrs &p, int gap, int species, long long n, const double *x_dev,
                         const double *v_dev, long long id0, int N, int ncu, int fp64, hipStream_t s);
// the potential of a gap's last level, to host memory the device maps
hipError_t launch_phi(const DevPtrs &p, int gap, double *phi, hipStream_t s);
// time-step check: largest |u| per species (bit patterns of non-negative floats,
// max-reduced as unsigned integers) and the most electrons in one cell of one gap,
// to the read-back buffer
hipError_t launch_dt_scan(const DevPtrs &p, int gap, int N, int fp64, int ncu, hipStream_t s);
// guess network (gs_mlp.hip): y[n][3] = net(x[n][48]) with bfloat16 weights W (finite: all of them are)
hipError_t launch_mlp_forward(const uint16_t *W, bool finite, const float *x, long long n, float *y, int ncu,
                              hipStream_t s);
size_t push_lds_bytes(int nmax, int fp64, int G, int wide);
size_t sort_lds_bytes(int G, int nmax, int bin);

}  // namespace gs
