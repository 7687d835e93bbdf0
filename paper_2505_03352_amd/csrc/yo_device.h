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
__device__ __forceinline__ Rsrc rsrc_of(const float *p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float bload(Rsrc r, int voff, unsigned soff)
{
    return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, (int)soff, 0));
}
__device__ __forceinline__ void bstore(float v, Rsrc r, int voff, unsigned soff)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), r, voff, (int)soff, 0);
}

// Store of a new field value: no wave of this launch reads it again, so it
// is marked non-temporal (cache-policy bit 1) to leave the caches to the
// halo rows and planes that neighbouring tiles do re-read.  (The CPML
// memories keep the default policy: marked the same way, measured slower.)
__device__ __forceinline__ void bstore_nt(float v, Rsrc r, int voff, unsigned soff)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), r, voff, (int)soff, 2);
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
__device__ __forceinline__ Cpml cpml_at(const float4 *prof, int which, int u)   // which: 0 E sites, 1 Ht sites
{
    const float4 v = prof[2 * u + which];
    return Cpml{v.x, v.y, v.z};
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

// The buffer (and CPML memory slot) that holds the state at the launch, and
// the one it goes to when the launch advances it by `adv` steps.
__device__ __forceinline__ int buf_now(const YoPlanD &P, int step, int b_offset)
{
    return P.nbuf == 3 ? step % 3 : (P.step_ctr[1] + b_offset) & 1;
}
template <class PP>   // PP: pointer to a YoPlanD in global or constant memory
__device__ __forceinline__ int buf_next(PP P, int now, int adv)
{
    return P->nbuf == 3 ? (now + adv) % 3 : now ^ 1;
}

// bytes of one array of nc components
template <class PP>
__device__ __forceinline__ unsigned array_bytes(PP P, int nc)
{
    return (unsigned)((P->nz * (P->ny + 1) + 1) * P->ns) * (unsigned)(64 * nc * sizeof(float));
}

// one slot of a right-hand side's CPML memories
template <class PP>
__device__ __forceinline__ Rsrc psi_rsrc(PP P, const float *psi, int slot)
{
    return rsrc_of(psi + (size_t)slot * P->psi_slot, 4u * P->psi_slot);
}

// Lane offsets past every buffer (all are below 4 GiB less 4 KiB): loads give
// zero, stores are dropped.  Component offsets are added to it.
constexpr int kFar = (int)0xfffff000u;

// What a lane does of a row of a tile (columns x0 - 2 + lane): the byte offset
// of its column for loads from the state, kappa and the rows of CPML memories
// (past the buffer for columns outside the grid or past the halo lanes) and
// for stores to the state and the memories, and whether it owns the column.
// Stores also go to the pads of the tile's strip, so that a whole strip's row
// is stored in whole 128-byte lines.  A line stored in part costs about four
// line transfers here: tiles of 60 columns at plain offsets streamed 2.8 TB/s,
// the same columns in strips with stored pads 4.7 TB/s (a copy: 4.8).
struct LaneX {
    int x;
    int xl, xk, xp;
    int xs, xps;
    int px;               // byte offset in an x-slab memory row (negative outside the slabs)
    bool own, st;
};
template <class PP>
__device__ __forceinline__ LaneX lane_x(PP P, int x0, int xn, int lane)
{
    LaneX L;
    const int x = x0 - YO_LEAD + lane;
    L.x = x;
    const bool in = x >= 0 && x < P->nx && lane < xn + 2 * YO_LEAD;
    L.own = lane >= YO_LEAD && lane < YO_LEAD + xn;
    L.xl = in ? yo_col(x, 6) * 4 : kFar;
    L.xk = in ? yo_col(x, 3) * 4 : kFar;
    L.xp = in ? yo_col(x, 4) * 4 : kFar;
    const int s = x0 / YO_SW, pos = x0 - s * YO_SW + lane;   // place in the tile's strip
    // (past the grid's last column up to the end of its line)
    // (both within the strip: further lanes' places are the next component's)
    const bool pad = pos < 64 && (((pos < YO_LEAD || pos >= YO_LEAD + YO_SW) && lane < xn + 2 * YO_LEAD) ||
                                  (x >= P->nx && pos < ((YO_LEAD + P->nx - s * YO_SW + 31) & ~31)));
    L.st = L.own || pad;
    L.xs = pad ? (s * 384 + pos) * 4 : (L.own ? L.xl : kFar);
    L.xps = pad ? (s * 256 + pos) * 4 : (L.own ? L.xp : kFar);
    L.px = -1;
    return L;
}

// the lane's place in the x-slabs' memories, and their coefficients there
template <class PP>
__device__ __forceinline__ void lane_xslab(PP P, LaneX &L, Cpml &cxE, Cpml &cxH)
{
    if (L.xl == kFar || slab_index(L.x, P->nx, P->plo[0], P->phi[0]) < 0) return;
    L.px = (L.x < P->plo[0] ? L.x : P->psi_xside + L.x - (P->nx - P->phi[0])) * 4;
    cxE = cpml_at(P->prof[0], 0, L.x);
    cxH = cpml_at(P->prof[0], 1, L.x);
}

__device__ __forceinline__ void block_sync_lds()
{
    // LDS-only ordering: outstanding global loads and stores stay in flight
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace
