// Internal device descriptors and kernel entry points of libyeeopt (not part
// of the public ABI).  Host runtime and kernels share these layouts.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#define YO_MAX_PORTS 8
#define YO_MAX_SLOTS 32
#define YO_TY 4           // rows per wave
#define YO_TY2 6          // rows per wave of the two-step region's taller tiles
#define YO_MAX_WPB 8      // waves per block of the step kernel: 4 or 8
#define YO_PAIR_TY 2      // whole-grid tiles: rows per wave,
#define YO_PAIR_W 8       // waves per block,
#define YO_PAIR_GROUP 32  // tiles that consecutive blocks take for one right-hand side

// Field arrays carry a ghost row on either side of y.  A row of nx cells is cut
// into ns strips of 60, each in a segment of nc x 64 floats, the components of a
// strip side by side: component c of cell (x, j, k), j in [-1, ny], of an array
// with nc components sits at
//   (((k * (ny + 1) + (j + 1)) * ns + s) * nc + c) * 64 + 2 + x - 60 s,
// s = x / 60 (row ny of a plane is row -1 of the next, a ghost of both).  The 2
// floats on either side of the 60 are pads: the lanes of a wave that own no cell
// of its strip lie over them and store values nobody reads, so that every row of
// a strip is stored in whole 128-byte lines (stores of 240-byte rows across
// lines reached 2.8 TB/s, of whole lines 4.7), and a component's offset from a
// strip's first is a constant of the instruction.
// The state of one right-hand side and buffer is one such array with nc = 6
// (Ex Ey Ez Ht_x Ht_y Ht_z), kappa one with nc = 3.  Ghost rows are zero and
// never written, and columns and planes outside the grid are read past the
// buffer (zero), which realises the perfect-conductor box (values outside the
// grid read as zero) without branches.
#define YO_SW 60          // cells per strip
#define YO_LEAD 2         // pad floats (halo lanes) before them

struct YoPlaneD {
    int axis, index, lo0, lo1, n0, n1;
};

// One right-hand side: its own field state, absorbing-layer memories, DFT
// sums, source plane and per-step phase table.
struct YoRhsD {
    // state buffers, layout above, nc = 6 (E then Ht): two, which a launch that
    // advances the state swaps, or with time blocking asked for three (nbuf), the
    // state after step s in F[s % 3]
    float *F[3];
    // CPML memories: one slot of psi_slot floats per state buffer, of each axis
    // four values (the two of E's components, the two of Ht's): axis a's at
    // float offset psi_off[a]; rows of the y- and z-slabs ([nz][Wy], [Wz][ny]) as
    // the field rows' strips with nc = 4, those of the x-slabs
    // [side][nz][ny][4][lo], or [nz][ny][4][lo + hi] where the slabs differ
    float *psi;
    float2 *dft_box;         // [3][bz][by][bx]
    float2 *dft_mon;         // concatenated port planes [2][n1][n0]
    float *dft_mid;          // E after a pair's first step: the box, then the port planes
    const float4 *steptab;   // [n_steps]: source signal (x, y) at (n+1/2)dt, (cos, sin) at n dt
    const float2 *src_j;     // [2][n1][n0], nullptr if no source
    YoPlaneD src;
    int win_start, win_len;
    float ginv[4];           // inverse Gram matrix of the steady-state fit
    int freq;
    int n_dft;               // frequencies this right-hand side's DFT accumulates (1, or all under a pulse)
    const float4 *dfttab;    // DFT phases (.z, .w) of frequency f at step n: dfttab[f * n_steps + n]
    int box_fstride;         // float2 entries from one frequency's DFT box to the next
    int mon_fstride;         // the same for the port planes
    int src_nc;              // component planes of the source (see YoPlanD::mon_nc)
    int pad2;
};

// One plan (one geometry): shared material and geometry description.
struct YoPlanD {
    int nx, ny, nz, ns;      // ns: strips per row
    float sx, sy, sz, pad0;
    int plo[3], phi[3];      // PML cells low/high per axis
    const float *kappa;      // ghost layout (ghosts zero)
    const float4 *kplane;    // [nz]: a plane's one kappa per component, .w 1 (0: it has no one value)
    const float4 *prof[3];   // per axis [n_a][2]: (b, c, 1/kappa, 0) at the E, then at the Ht sites
    unsigned psi_off[3], psi_slot;   // floats
    int psi_xrow, psi_xw, psi_xside;  // x-slab rows: floats per row, per value, and to the high slab
    int box[6];              // x0 y0 z0 bx by bz
    int n_ports;
    int n_steps;
    int dft_stride;          // the DFT adds E^n of the steps n divisible by it (1: every step)
    int nbuf;                // state buffers per right-hand side (2 or 3)
    int r2[6];               // two-step region [x0, x1) x [y0, y1) x [z0, z1) (empty: x1 <= x0)
    YoPlaneD ports[YO_MAX_PORTS];
    int mon_off[YO_MAX_PORTS];
    int mon_total;
    // device counters of this plan: steps, launches of the run that took any, and
    // for the forward and the adjoint right-hand sides the buffer their state is in
    int *step_ctr;
    int n_rhs;
    // component planes of a port's monitor (and of its adjoint source): 2 =
    // the tangential E on the plane; 5 = those, the normal E half a cell past
    // the plane, and the tangential E one cell past it
    int mon_nc;
    const YoRhsD *rhs;       // [n_rhs]
};

// A tile is one wave's work (or, in the cooperative layout, one block's):
// owned x in [x0, x0+xn) (xn <= 60), rows [j0, j0+jn) (jn <= YO_TY, or
// YO_TY * waves per block), planes [k0, k1).  Packed as int4
// (x0 | xn << 16, j0 | jn << 16, k0 | k1 << 16, tile class); k1 may need all of
// its 16 bits.
__host__ __device__ inline int yo_high(int v) { return (int)((unsigned)v >> 16); }
struct YoSlot {
    const YoPlanD *plan;
    const int4 *tiles;       // tile list of this launch's class
    int rhs0, nrhs;
    int ntile, nzc;          // tiles; whole-grid tiles: z-chunks of each
};

struct YoStepArgs {
    int n_slots;
    int k_offset;            // steps into the chunk; step = counter + k_offset
    int b_offset;            // launches into the chunk that advanced the state
    int total_waves;
    int wpb;                 // waves per block (4 or 8)
    int prefix[YO_MAX_SLOTS + 1];
    YoSlot slot[YO_MAX_SLOTS];
};

// Work list of the small per-step kernels (DFT accumulation and source
// injection): per slot, the plan, its right-hand side range and the number
// of points per right-hand side.
struct YoAuxArgs {
    int n_slots;
    int k_offset;
    int b_offset;
    int pair;                // k_dft: after a pair of steps, adding both
    int total_blocks;
    int prefix[YO_MAX_SLOTS + 1];   // blocks
    const YoPlanD *plan[YO_MAX_SLOTS];
    int rhs0[YO_MAX_SLOTS], nrhs[YO_MAX_SLOTS];
    int npts[YO_MAX_SLOTS];         // points per right-hand side
};

struct YoCtrArgs {
    int n;
    int add;                 // steps the launches before took, or 0: a reset
    int pairs;               // they went two per launch, an odd last one alone
    const YoPlanD *plan[YO_MAX_SLOTS];
    int which[YO_MAX_SLOTS]; // sides selected
};

// A ghost-layout array on one side of a copy: F[*now], of the buffers of a
// right-hand side the one that holds its state (known on the device only, as
// a caller may replay launches it captured), or F[0] without `now`.
struct YoGhost {
    float *F[3];
    const int *now;
};

// Parametrization buffers of one plan.
struct YoChainBufs {
    int md, nd, mc, nc, S, U, V, G0, G1;   // G0 = md+4 (x), G1 = nd+4 (y)
    int tmax;                               // filter taps per sub-pixel (max)
    float eps_core, eps_clad, delta;
    // filter tables
    int *tap_lo_x, *tap_n_x, *tap_lo_y, *tap_n_y;   // [S md], [S nd]
    float *tap_w_x, *tap_w_y;                        // [S md][tmax], [S nd][tmax]
    float *tapt_x, *tapt_y;                          // [rmax_x][mc], [rmax_y][nc]: a control's weights from its first sub-pixel on
    int *urange_x, *urange_y;                        // per control: [2] first/last sub-pixel
    // forward state
    float *mask;      // [V][U]
    float *rho;       // [V][U]
    float *tanh_;     // [S nd][S md]
    float *P, *Q, *R; // [3][G1][G0]
    float *aux;       // [6][G1][G0]: n2x n2y Gx_x Gy_x Gx_y Gy_y
    // backward
    float *gPQ;       // [6][G1][G0]: gP(x,y,z) gQ(x,y,z)
    float *gG;        // [4][G1][G0]: gGx_x gGy_x gGx_y gGy_y
    float *gR;        // [2][G1][G0]
    float *gphi;      // [S nd][S md]
    float *tmp;       // [S nd][mc], or forward [nc][S md] (yo_filter_by_rows)
    // morphological filters (n_morph = 0: none; rho = the Eq. (3) projection)
    int n_morph;      // stages
    unsigned mdil;    // bit k set: stage k dilates, else erodes
    int n_mtaps;      // disc taps
    float malpha;     // sharpness
    float minv;       // 1 / n_mtaps
    int mrad;         // the disc's radius in whole sub-pixels
    int *mwid;        // [2 mrad + 1]: largest |dx| of each of its rows (-1: none)
    float *mcan;      // [n_morph + 1][V][U]: stage inputs, then the last output
    float *msum;      // [n_morph][S nd][S md]: each stage's kernel sums
    float *tanh2;     // [S nd][S md]: tanh of the projection after the stages
    float *mg;        // [2][S nd][S md]: gradients between stages
};

// Is the filter's x pass made once for each control row, in a launch of its own?
// Not where there are more of those than sub-pixel rows that could share them:
// each sub-pixel then filters its own, and no rows are kept.  Nor where a
// sub-pixel has few taps: of a radius up to 2 (tmax 6) the launch costs more than
// it saves below some 700x700 sub-pixels (yo_set_design whole, one pass and two:
// 96x96 at radius 1.5 12.5 and 16.0 us, at 3 17.0 and 15.7; 600x600 at 2 17.9 and
// 18.4; 1200x1200 at 1.5 32.0 and 29.8).
inline bool yo_filter_by_rows(int nc, int nud, int nvd, int tmax)
{
    return nc <= nvd && (tmax > 6 || (size_t)nud * nvd >= (size_t)1 << 19);
}

// ---- kernel launchers ----
// pm: 0 = interior tiles (no CPML code), 1 = interior tiles plus tiles inside
// the x-slabs only (the x-axis CPML code), 7 = CPML tiles with the code of all
// three axes, 8 = CPML tiles each running its own class's code (int4 .w);
// coop: one tile per block, its waves stacked in y (tiles of YO_TY * wpb
// rows); prefetch: operands of the next plane loaded during this one
// rows: rows per wave, YO_TY, or YO_TY2 for the shell (pm 7 or 8, not coop)
hipError_t yo_launch_step(int pm, bool coop, bool prefetch, const YoStepArgs &args, int blocks,
                          hipStream_t s, int rows = YO_TY);
// two steps per sweep over the tiles of the two-step region (independent
// waves); zslab: the tiles of the z-slabs under it, with z-axis CPML code;
// rows: rows per wave, YO_TY, or YO_TY2 for the region itself; coop: one
// tile per block, its waves stacked in y and sharing rows through LDS
hipError_t yo_launch_step2(bool zslab, int rows, bool coop, const YoStepArgs &args, int blocks,
                           hipStream_t s);
// two steps over whole-grid tiles (one block each, YO_PAIR_W waves); shell:
// tiles with x- or y-slabs, source planes or the grid's first column or row
// gen: 1 planes normal to y or z, 2 and more than 32 x-slab columns in a strip
hipError_t yo_launch_pair(bool shell, bool dft, int gen, const YoStepArgs &args, int blocks, hipStream_t s);
// one step over the same tiles (all of them)
hipError_t yo_launch_one(const YoStepArgs &args, int blocks, hipStream_t s);
hipError_t yo_launch_dft(const YoAuxArgs &args, hipStream_t s);
hipError_t yo_launch_source(const YoAuxArgs &args, hipStream_t s);
hipError_t yo_launch_ctr(const YoCtrArgs &args, hipStream_t s);
hipError_t yo_launch_fill(float *p, size_t n, float v, hipStream_t s);
// dense [ncomp][nz][ny][nx] <-> components c0 .. c0+ncomp-1 of a ghost-layout
// array with nc components
hipError_t yo_launch_to_ghost(const float *dense, const YoGhost &ghost, int ncomp, int c0, int nc, int nz,
                              int ny, int nx, int ns, hipStream_t s);
// a background: kappa and its kplane (planes k_lo .. k_hi are taken as not
// uniform), and the n values of the canvas' mask
hipError_t yo_launch_background(const float *dense, float *kappa, float4 *kplane, int nz, int ny, int nx, int ns,
                                int k_lo, int k_hi, const float *mask, float *mask_out, size_t n, hipStream_t s);
hipError_t yo_launch_from_ghost(const YoGhost &ghost, float *dense, int ncomp, int c0, int nc, int nz,
                                int ny, int nx, int ns, hipStream_t s);
// in-place phasor fit of n complex sums; sets *bad to 1 if a result is not
// finite (*bad is left alone otherwise)
hipError_t yo_launch_finalize(float2 *a, size_t n, float g00, float g01, float g10, float g11,
                              int *bad, hipStream_t s);
// modal coefficients, out [n_src][n_ports][n_freq]
struct YoAlphaArgs {
    const float2 *mon;         // port planes of output right-hand side r at mon_stride r
    const float2 *w;           // weights (of frequency f at w_fstride f)
    size_t mon_stride, w_fstride;
    int mon_off[YO_MAX_PORTS], w_off[YO_MAX_PORTS], n[YO_MAX_PORTS];
    int n_src, n_ports, n_freq;
    float2 *out;
};
hipError_t yo_launch_alpha(const YoAlphaArgs &a, hipStream_t s);
hipError_t yo_launch_chain_forward(const YoChainBufs &c, const float *C, float beta,
                                   float *kappa, int ny, int ns, int i0, int j0,
                                   int k_lo, int k_hi, hipStream_t s);
#define YO_MAX_GF 32
#define YO_MAX_GA 64
#define YO_MAX_FREQ 16
struct YoGradArgs {
    const float2 *EF[YO_MAX_GF];   // forward box phasors, index f*n_src + s
    const float2 *EA[YO_MAX_GA];   // adjoint box phasors, index f*n_ports + p
    float sinth[YO_MAX_FREQ];      // sin(w dt / 2) per frequency
    const float2 *coef;            // [n_src][n_ports][n_freq]
    const float *kappa;            // ghost layout
    float *gbox;                   // [3][bz][by][bx] dF/dkappa
    int n_src, n_ports, n_freq;
    int ns, ny;
    int box[6];
};
hipError_t yo_launch_grad_assemble(const YoGradArgs &a, hipStream_t s);
// dF/dkappa on the box (planes z0 .. z0 + bz - 1) to dF/dC
hipError_t yo_launch_chain_vjp(const YoChainBufs &c, const float *gbox, int z0, int bz, int k_lo, int k_hi,
                               float beta, float *dFdC, hipStream_t s);
// grey fraction of the design area: rho in (lo, hi) as tanh in (tlo, thi);
// count: YO_GRAY_BLOCKS ints
#define YO_GRAY_BLOCKS 16
#define YO_MAX_DISC 32    // largest disc radius, sub-pixels
hipError_t yo_launch_unbinarity(const YoChainBufs &c, float tlo, float thi, int *count, float *out,
                                hipStream_t s);
hipError_t yo_launch_adam(float *C, const float *G, float *M, float *V, int n, float lr, float b1, float b2,
                          float eps, float inv1, float inv2, hipStream_t s);
// floats from the start of a row's component 0 to cell x in an array of nc
// components (see the layout above)
__host__ __device__ inline int yo_col(int x, int nc)
{
    const int s = x / YO_SW;
    return s * 64 * nc + YO_LEAD + (x - s * YO_SW);
}

// ghost-layout offset of component c of (x, j, k) in an array of nc components
__host__ __device__ inline size_t yo_off(int c, int x, int j, int k, int ny, int ns, int nc)
{
    return ((size_t)k * (ny + 1) + (size_t)(j + 1)) * ns * 64 * nc + (size_t)(yo_col(x, nc) + 64 * c);
}
