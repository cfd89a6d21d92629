// Internal structures shared by the kernels (lbm_kernels.hip) and the runtime (lbm_capi.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_lattice.h"

namespace lbm {

enum Side { XMIN = 0, XMAX = 1, YMIN = 2, YMAX = 3 };
enum Bc { BC_PERIODIC = 0, BC_ZG = 1, BC_NRBC = 2, BC_NRBC_A = 3 };

// Sides with the characteristic fill (the perfectly non-reflecting LODI boundary, or CBC (A)).
inline __host__ __device__ bool is_char_bc(int b) { return b == BC_NRBC || b == BC_NRBC_A; }
enum Storage { ST_F64 = 0, ST_F32 = 1, ST_F16 = 2 };

// Device descriptor of one run.  Lives in device memory (one per run); kernels receive an
// array of pointers to descriptors, so a single run and a batch share every kernel.
//
// Grid: Nx x Ny nodes; population i of node (x, y) is f[par][i * plane + y * pitch + x].  With
// the row layout (default) the q population rows of one grid row are adjacent (plane = padded
// row, pitch = q padded rows), which keeps the pulls of a tile inside a few MiB of address
// space; with the plane layout `plane` is a whole padded plane and `pitch` a padded row.
// Arrays of per-pair and per-shell constants are sized for the largest stencil (D2Q37).
// Frame: the nodes outside the fast interior rectangle [fx0,fx1) x [fy0,fy1), i.e. a frame of
// depth gxm/gxp/gym/gyp on the four sides.  The ring is the outer part of the frame with depth 3
// on characteristic (NRBC) sides only: the boundary nodes that need the FP64 characteristic
// fill, handled by the first blocks of the boundary launches.  Strips of a frame-shaped region
// are numbered bottom strip, top strip, left strip, right strip (row-major inside each strip).
// Frame index t, which Q and the moment strips U use: the ring nodes first, t = their ring index
// in [0, ring_n); then, from ann0 (ring_n rounded up to 64) on, the other frame nodes, numbered
// as the strips of the annulus between the ring's inner rectangle and the fast rectangle (depths
// axm/axp/aym/ayp); the ring_n..ann0 gap is unused.  A frame thread touches its own Q/U entries
// with unit stride, and the ring blocks and the frame blocks share no cache line of Q or U.
// Without a ring the numbering is the frame's own strip numbering.
struct alignas(256) RunDev {
    int Nx, Ny, pitch, storage;
    long long plane;          // element stride between populations of one node
    long long fsize;          // elements of one population buffer
    long long qplane;         // elements per component plane of Q and U
    int gxm, gxp, gym, gyp;   // frame depths
    int Wxm, Wxp, Wym, Wyp;   // PML width per side (0 if none)
    int W, qd, open_x, open_y;
    int bc[4];
    int fx0, fx1, fy0, fy1;   // fast rectangle
    int frame_n, has_q, ring_n, pml_terms;   // pml_terms: PML moments in the NRBC target
    int rxm, rxp, rym, ryp;   // characteristic-boundary ring depths (3 on NRBC sides, else 0)
    int axm, axp, aym, ayp;   // depths of the frame's annulus off the ring
    int ann0, ann_n;          // first frame index and count of the frame nodes off the ring
    int tiles_x[3], tiles_y[3];   // bulk tiles for tile widths 64, 128, 256
    // two-step passes (core_strips = 0: the run takes single steps only).  The bands hold the level
    // between of the frame and of the interior within 2 reach of it: a row band (bT rows below the
    // top edge, then bB above the bottom one, every column) and a column band (bR columns, then bL,
    // the rows off the frame's y strips), both with the q population rows of a row adjacent.
    int core_strips, shell_n;     // strips of the two-step tiles; nodes of the shell
    int bL, bR, bB, bT;
    int m_row, l_row;             // elements of a population row of the row and the column band
    long long l_first, msize;     // first element of the column band; elements of both
    // state
    void *f[2];
    void *M;                  // bands of the two-step passes (or NULL)
    void *Q;                  // [q][qplane] in the compute type
    double *U[2];             // [4][qplane]: rho, ux, uy, T (absolute values)
    void *G;                  // [q][rplane] compute type: post-boundary populations of the ring
    double *P;                // [4][rplane]: characteristic targets formed by k_target (if tgt_pre)
    long long rplane;
    int par, tgt_pre;         // tgt_pre: NRBC targets formed by k_target (PML moments or CBC (A))
    long long step, limit;    // a run is active while step < limit
    // constants (double and float copies)
    double omega, rho0, u0x, u0y, T0, th0, b0, r0x, r0y, sigma_max, inv_W2, scale, inv_scale;
    double H0rest, H0e[NPAIR_MAX], H0o[NPAIR_MAX], E2_0[NSHELL_MAX], O1_0[NSHELL_MAX];
    double xx0, xy0, yy0, k2a0, k10, eq0[NEQ];   // FP64 storage: the mean state's polynomial coefficients over rho
    float omega_f, rho0_f, u0x_f, u0y_f, th0_f, b0_f, r0x_f, r0y_f, T0_f, scale_f, inv_scale_f;
    float H0rest_f, H0e_f[NPAIR_MAX], H0o_f[NPAIR_MAX], E2_0_f[NSHELL_MAX], O1_0_f[NSHELL_MAX];
#ifdef LBM_BOUNDS
    unsigned oob;             // bounds-checked build: nonzero once a kernel met an index out of range
#endif
};

// Launch decomposition of a set of runs: prefix[k] = first block of run k, prefix[n] = total.
// Classes: the interior tiles; the frame launch (ring blocks, then frame blocks); the phase-A
// launch (ring blocks, then frame blocks if the run has a PML); the characteristic targets of
// runs that select the PML moments (ring blocks).
// Two-step passes add the two-step tiles and the second step's frame launch (ring, frame and shell
// blocks); a small frame is launched in blocks that split the populations (ring, then frame), phase A likewise.
enum Cls { CLS_BULK = 0, CLS_FRAME = 1, CLS_A = 2, CLS_TGT = 3, CLS_CORE = 4, CLS_FRAME2 = 5, CLS_SPLIT = 6, CLS_A_SPLIT = 7, NCLS = 8 };
struct KernelSet;

// Position of a sub-step in its batch: time steps and population buffer swaps since its start.
struct Sub { int steps, flips; };
struct LaunchSet {
    const KernelSet *ks;      // kernels of the runs' velocity stencil (one stencil per set)
    RunDev *const *runs;      // device array of descriptor pointers
    const int *prefix[NCLS];  // device prefix arrays per class
    int blocks[NCLS];         // total blocks per class
    int nruns;
    int poison = 0;           // debug canary: NaN-fill each step's destination buffers first
    int split = -1;           // fused grid: phase-A blocks after split/8 of the tiles; -1 default
    int core_rows = 0;        // rows of a two-step tile; 0: the set takes single steps only
    bool split_small = false; // boundary launches of single steps split a node's populations over 4 waves
    bool stream_frame = true; // the frame kernel of single steps streams its stores (FP32, FP16)
};

// Two-step tiles: CORE_X columns of the level between, CORE_R rows per turn (one wave each); they
// advance core_out columns by two steps.  CORE_PAD: LDS elements before and after the rows, which
// the lanes that advance no node may read.
constexpr int CORE_X = 64, CORE_R = 4, CORE_PAD = 8, CORE_LINE = 64;
// Columns a tile advances: whole CORE_LINE-byte pieces of a population row, from a column that starts one.
constexpr int core_out(int reach, int es) { return (CORE_X - 2 * reach) * es / CORE_LINE * CORE_LINE / es; }
inline __host__ __device__ int core_x0(int fx0, int reach, int es) { return (fx0 + reach) * es / CORE_LINE * CORE_LINE / es; }
// LDS rows of a tile: CORE_R per population, and one more for each row pulled two turns later.
constexpr int core_lds_rows(const LatticeInfo &l) {
    int n = 0;
    for (int i = 0; i < l.q; ++i) {
        const int delay = l.ey(i) + reach_of(l);
        n += CORE_R + (delay > CORE_R ? delay - CORE_R : 0);
    }
    return n;
}
// Tiles a compute unit holds (160 KiB of LDS, allotted in 1280 bytes; at most 4 waves per SIMD)
// and their waves per SIMD, which bound the kernel's registers.
constexpr int core_tiles_per_cu(const LatticeInfo &l, int es) {
    const int bytes = ((core_lds_rows(l) * CORE_X + 2 * CORE_PAD) * es + 1279) / 1280 * 1280;
    return 163840 / bytes < 4 ? 163840 / bytes : 4;
}
constexpr int core_waves(const LatticeInfo &l, int es) { return core_tiles_per_cu(l, es) * CORE_R / 4; }

constexpr int FRAME_BLOCK = 256;
// Ring nodes per block of the boundary launches: one active wave per 256-thread block, so the
// ring's few, poorly coalesced waves (a 3-wide strip puts ~21 grid rows in one wave) land on
// different compute units instead of sharing one unit's memory pipeline four at a time.
constexpr int RING_BLOCK = 64;
// Nodes per block of the boundary kernels that split their populations over its 4 waves, and the most
// such blocks of a launch set for which they are taken (256 CUs times those a CU holds at once; a
// second round of blocks costs more than the split gains).  Frame launch and fused launch together,
// us, split and not, below and above the line: D2Q37 FP64 340^2 33.7, 37.0, 490^2 (720 blocks) 53.6,
// 52.4; FP32 490^2 33.5, 37.5, 740^2 (1100) 54.6, 52.1; D2Q17 FP64 490^2 28.0, 29.3, 560^2 (810)
// 33.1, 32.7; FP32 640^2 24.5, 26.4, 880^2 (1260) 36.7, 37.9.
// Without characteristic sides no long FP64 chain is shortened, and a state that the L2s hold answers
// a lone wave soon enough, so there the line is lower the smaller the interior is.  us per step, whole
// nodes and split, at (blocks, interior nodes / 256): D2Q37 FP32 ZG with 60 cells of layer (608, 38)
// 17.3, 19.5; channel 52 cells deep (984, 90) 22.5, 25.4; 15 cells (608, 709) 32.1, 32.9; 20 cells
// (488, 474) 26.8, 24.0; 10 cells (536, 1418) 42.4, 37.7; FP16 (608, 38) 17.1, 19.6, (960, 99) 17.9,
// 21.8; D2Q17 FP64 (456, 91) 14.2, 15.1, (608, 709) 27.3, 25.6, FP32 (688, 969) 19.5, 20.8, FP16 (456,
// 91) 12.4, 11.8, (608, 709) 15.3, 16.5.  With a ring D2Q37 FP32 (984, 90) 31.6, 25.7, D2Q17 FP16
// (1104, 969) 21.1, 19.5, (1184, 241) 18.9, 19.8; FP64 D2Q37, whose line is lower already, (456, 91)
// 24.5, 23.2.  D2Q37 FP32 beside a large interior: (952, 1904) 52.0, 55.2, 832^2 ring (900, 2480)
// 57.9, 61.1, ZG 57.0, 58.1, (696, 3891) 86.5, 76.8.
constexpr int SPLIT_BLOCK = 64;
constexpr int split_most(int q, int elem, bool ring, long long interior) {
    const int most = 256 * (q == 37 ? (elem == 8 ? 2 : elem == 4 && interior > 256 * 1024 ? 3 : 4)
                            : q == 17 ? (elem == 8 ? 3 : 5) : 0);
    const long long line = ring                  ? 1024 + interior / 1024
                           : elem < 8            ? (q == 37 ? 416 + interior / 1024 : 448 + interior / 2048)
                           : q == 37             ? most
                                                 : 384 + interior / 512;
    return line < most ? (int)line : most;
}
static_assert(SPLIT_BLOCK == RING_BLOCK, "the split launch has the ring's blocks");

// Whether the frame kernel of single steps streams its stores, for a set whose populations have this
// many bytes (two levels, without padding); tall: more than twice as many rows as columns.  FP64 does.  FP32 and FP16 rows of the side strips start
// and end inside 64-byte pieces, which the cache joins with their neighbours' when they are ordinary
// stores; but those push out what the next step reads, while the state is about what the L2s hold (32
// MB), and in FP16 cost the next grid more than they save once it is past the Infinity Cache.  us per
// step, streaming and ordinary: D2Q9 FP32 89 x 1335 (9 MB) 14.9, 15.6, D2Q37 FP32 591 x 145 (25 MB)
// 21.8, 22.7 and 370^2 (41 MB) 27.7, 28.6, D2Q17 FP32 89 x 1335 (16 MB) 19.9, 20.6; D2Q37 FP32 130 x
// 1266 (49 MB) 41.3, 36.8, 576^2 ZG (98 MB) 38.0, 39.7, 1032^2 (315 MB) 87.1, 83.6, D2Q17 1032^2 (145
// MB) 43.9, 41.9, 280 x 3580 (136 MB) 68.8, 61.5, D2Q9 820^2 (48 MB) 22.8, 23.5.  FP16 D2Q37 470^2 (33 MB) 37.2, 37.7, D2Q9 1032^2
// (38 MB) 22.4, 19.2, D2Q17 1764^2 (212 MB) 66.6, 58.3, D2Q37 1764^2 (461 MB) 159.2, 152.9; 2064^2 ZG
// (630 MB) 184.7, 191.0, D2Q17 4112^2 ZG (1150 MB) 248.4, 255.3, with a ring even (1177 MB 284.4, 284.4).
constexpr bool frame_streams(int elem, size_t bytes, bool tall) {
    return elem == 8 || (elem == 4 ? bytes < (tall ? 48000000 : 130000000) : bytes < 36000000 || bytes >= 500000000);
}

// Blocks of a run in the boundary launches: ring blocks, then frame blocks, each count rounded up
// to a multiple of 8.  Blocks are dealt round-robin to the 8 XCDs, so every run's frame blocks
// then start on the first XCD and can be remapped XCD by XCD (neighbouring strip rows, which
// share pulled rows and Q planes, on one XCD and its L2); the padding blocks exit at once.
__host__ __device__ inline int ring_block_count(int ring_n) {
    return ((ring_n + RING_BLOCK - 1) / RING_BLOCK + 7) & ~7;
}
__host__ __device__ inline int frame_block_count(int frame_n) {
    return ((frame_n + FRAME_BLOCK - 1) / FRAME_BLOCK + 7) & ~7;
}

// Kernel launchers of one velocity stencil (lbm_kernels.hip, compiled once per stencil).  All
// enqueue on `s` and return the HIP status of the launch.
// phase_a: characteristic fill of the ring and PML auxiliary update; frame: phase B (collision)
// of every frame node, ring included; target: characteristic targets with the PML moments.
struct KernelSet {
    int q;
    // step kernels of sub-step ks of a batch (parity par + ks; active while step + ks < limit)
    hipError_t (*phase_a)(const LaunchSet &L, int storage, Sub ks, hipStream_t s);
    // frame, phase_a_bulk and bulk take optional events a and b (both or neither), attached to
    // the dispatch: they take the kernel's own start and end time
    hipError_t (*frame)(const LaunchSet &L, int storage, Sub ks, hipStream_t s, hipEvent_t a,
                        hipEvent_t b);
    hipError_t (*target)(const LaunchSet &L, int storage, Sub ks, hipStream_t s);
    // phase A and the bulk tiles in one launch
    hipError_t (*phase_a_bulk)(const LaunchSet &L, int storage, int tx, Sub ks, hipStream_t s,
                               hipEvent_t a, hipEvent_t b);
    hipError_t (*bulk)(const LaunchSet &L, int storage, int tx, Sub ks, hipStream_t s,
                       hipEvent_t a, hipEvent_t b);
    // end of a batch of n sub-steps with `flips` buffer swaps: step counters and parities advance
    hipError_t (*advance)(const LaunchSet &L, int n, int flips, hipStream_t s);
    hipError_t (*set_limit)(RunDev *run, long long limit, hipStream_t s);
    hipError_t (*set_limits)(RunDev *const *runs, const long long *limits, int n, hipStream_t s);
    hipError_t (*init)(RunDev *run, int storage, int Nx, int Ny, const double *rho,
                       const double *ux, const double *uy, const double *T, float *absmax,
                       hipStream_t s);
    hipError_t (*moments)(RunDev *run, int storage, int Nx, int Ny, double *rho, double *ux,
                          double *uy, double *T, hipStream_t s);
    hipError_t (*export_f)(RunDev *run, int storage, int Nx, int Ny, const double *fbar,
                           double *out, hipStream_t s);
    // Q of every frame node into a full grid (nt: the frame index extent, ann0 + ann_n)
    hipError_t (*export_q)(RunDev *run, int storage, int nt, double *out, hipStream_t s);
    hipError_t (*check)(RunDev *run, int storage, int Nx, int Ny, int *flag, hipStream_t s);
    hipError_t (*err_rows)(const double *rho, const double *ux, const double *T, int Nx,
                           int x0, int y0, int lx, int ly, const double *rr, const double *ru,
                           const double *rt, double *partials, hipStream_t s);
    // the sums of err_rows over the moments of the run's current state, formed in the kernel
    hipError_t (*err_rows_state)(RunDev *run, int storage, int x0, int y0, int lx, int ly,
                                 const double *rr, const double *ru, const double *rt,
                                 double *partials, hipStream_t s);
    hipError_t (*err_final)(const double *partials, int nrows, double *out, hipStream_t s);
    // debug canary of sub-step ks: NaN into the buffers the step writes in full (every active run)
    hipError_t (*poison)(const LaunchSet &L, int storage, Sub ks, hipStream_t s);
    // two time steps from sub-step k1 on, one pass over the interior
    hipError_t (*two_steps)(const LaunchSet &L, int storage, Sub k1, hipStream_t s);
};

namespace k37 { extern const KernelSet kernels; }
namespace k17 { extern const KernelSet kernels; }
namespace k9 { extern const KernelSet kernels; }

}  // namespace lbm
