// Device helpers shared by the time-stepping kernels.
#pragma once

#include "yo_internal.h"

namespace {

// Neighbour exchange along x with DPP whole-wave shifts (one VALU move, no
// LDS round trip).  The lane with no neighbour gets 0; those are halo lanes,
// whose results are never used.
__device__ __forceinline__ float shfl_next(float v)   // value of lane+1 (wave_shl:1)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ float shfl_prev(float v)   // value of lane-1 (wave_shr:1)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Raw buffer access: the resource (base, size) and the row offset are
// wave-uniform scalars, the only per-lane operand is the column offset, so a
// load costs no vector address arithmetic.  Reads past the buffer return 0.
typedef __amdgpu_buffer_rsrc_t Rsrc;
__device__ __forceinline__ Rsrc rsrc_of(const float *p, size_t n_floats)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), (short)0,
                                             (int)(n_floats * sizeof(float)), 0x00020000);
}
__device__ __forceinline__ float bload(Rsrc r, int voff, int soff)
{
    return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ __forceinline__ void bstore(float v, Rsrc r, int voff, int soff)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), r, voff, soff, 0);
}

// Store of a new field value: no wave of this launch reads it again, so it
// is marked non-temporal (cache-policy bit 1) to leave the caches to the
// halo rows and planes that neighbouring tiles do re-read.  (The CPML
// memories keep the default policy: marked the same way, measured slower.)
__device__ __forceinline__ void bstore_nt(float v, Rsrc r, int voff, int soff)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), r, voff, soff, 2);
}

__device__ __forceinline__ int slab_index(int u, int n, int lo, int hi)
{
    if (u < 0 || u >= n) return -1;
    if (u < lo) return u;
    if (u >= n - hi) return u - (n - hi) + lo;
    return -1;
}

// one CPML-modified difference: psi_new = b psi_old + c d, returns d/k + psi_new
struct Cpml {
    float b, c, ki;
};
__device__ __forceinline__ Cpml cpml_at(const float *prof, int n, int which, int u)
{
    // prof layout [6][n]: bE cE kiE bH cH kiH ; which = 0 (E sites) or 3 (H sites)
    Cpml p;
    p.b = prof[(which + 0) * n + u];
    p.c = prof[(which + 1) * n + u];
    p.ki = prof[(which + 2) * n + u];
    return p;
}
__device__ __forceinline__ float pml_diff(float d, const Cpml &p, float psi_old, float &psi_new)
{
    psi_new = fmaf(p.b, psi_old, p.c * d);
    return fmaf(d, p.ki, psi_new);
}

__device__ __forceinline__ int sel3(int a, int v0, int v1, int v2)
{
    return a == 0 ? v0 : (a == 1 ? v1 : v2);
}

__device__ __forceinline__ float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ Cpml lane_cpml(const Cpml &c, int l)
{
    Cpml o;
    o.b = lane_value(c.b, l);
    o.c = lane_value(c.c, l);
    o.ki = lane_value(c.ki, l);
    return o;
}

// CPML memory slots of each axis, as first components (two components per
// slot): with two state buffers, E one slot (0) read and written in place
// and Ht two (2, 4) by step parity, since halo rows recompute Ht from the
// old step's memory while its owner writes the new one; with three state
// buffers (two steps per launch) three slots each, E at 0, 2, 4 and Ht at
// 6, 8, 10, the step's memories in slot step % 3: a two-step launch reads
// slot n % 3 around its cells and writes slot (n + 2) % 3 of its own while
// single steps write (n + 1) % 3.
__device__ __forceinline__ void cpml_slots(int nbuf, int step, int &qEo, int &qEn, int &qHo, int &qHn)
{
    if (nbuf == 3) {
        const int s0 = step % 3, s1 = (step + 1) % 3;
        qEo = 2 * s0;
        qEn = 2 * s1;
        qHo = 6 + 2 * s0;
        qHn = 6 + 2 * s1;
    } else {
        const int par = step & 1;
        qEo = qEn = 0;
        qHo = 2 + 2 * par;
        qHn = 2 + 2 * (par ^ 1);
    }
}

// What a lane does of a row: the byte offset of its column in a row for loads
// (past every buffer for columns outside the grid: they read zero) and for
// stores, that of its column inside the x-slabs (negative outside), whether
// it owns the column and whether it stores (own, or a pad column of the
// strip: see yo_col).
struct LaneX {
    int xl, xs, px;
    bool own, st;
};
constexpr int kFar = (int)0x80000000;   // past every buffer (all are below 2 GiB)

// lead: lanes before the first owned column (columns x0 - lead + lane)
__device__ __forceinline__ LaneX lane_x(const YoPlanD &P, int x0, int xn, int lane, int lead)
{
    LaneX L;
    const int x = x0 - lead + lane;
    const bool in = x >= 0 && x < P.nx && lane <= lead + xn;
    L.own = lane >= lead && lane < lead + xn;
    L.xl = in ? yo_col(x, P.sw, P.slead) * (int)sizeof(float) : kFar;
    // position in the strip that holds the tile: the lanes over its pad
    // columns store too (values nobody reads), so that a whole strip's row is
    // stored in whole 128-byte lines.  A line stored in part costs about four
    // line transfers here: tiles of 60 columns at plain offsets streamed 2.8
    // TB/s, the same columns in strips with stored pads 4.7 TB/s (a copy: 4.8)
    const int s = x0 / P.sw, pos = x0 - s * P.sw + lane;   // slead == lead in the strip layout
    const bool pad = P.strips && (pos < lead || pos >= lead + P.sw || x >= P.nx) && pos < 64 &&
                     64 * s + pos < P.nxp && lane < xn + 2 * lead + (x >= P.nx ? 64 : 0);
    L.st = L.own || pad;
    L.xs = pad ? (64 * s + pos) * (int)sizeof(float) : L.xl;
    L.px = -1;
    return L;
}

__device__ __forceinline__ void block_sync_lds()
{
    // LDS-only ordering: outstanding global loads and stores stay in flight
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace
