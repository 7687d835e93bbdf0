// Fused single Yee steps for gfx950 in launches by tile class, and two steps
// over the region clear of slabs and planes: what yo_time_kernel and the tuner
// measure, and what runs where single-step launches are timed and in plans whose
// CPML memories pass 4 GiB (build_layout); the stepping itself is yo_pair.hip's.
// A single step is two launches over every selected right-hand side of every plan
// in the call: the interior tiles (clear of every absorbing slab, no CPML code)
// and the CPML shell; each advances its tiles by one full step (Ht half step, then
// E step).  The soft current source follows.  Also the running DFT (design box and
// port planes) around the steps, and the step counters.
//
// Update (paper Sec. 2: time-harmonic sources, steady-state phasors):
//   Ht^{n+1/2} = Ht^{n-1/2} - curl_e E^n                        (forward differences)
//   E^{n+1}    = E^n + kappa curl_h Ht^{n+1/2} - kappa j^{n+1/2} (backward differences)
// every difference along axis a scaled by S_a = c dt / d_a; in a CPML slab
// the difference d becomes d/k + psi with psi <- b psi + c d.
//
// Work decomposition (one wave = 64 lanes):
//   * lane l handles x = x0 - 2 + l.  Lanes 2..xn+1 own their cells; the
//     lanes on either side are halo lanes whose values reach the owners
//     through DPP whole-wave shifts.
//   * a wave owns rows j0..j0+jn-1 (jn <= 4) and recomputes the Ht of row
//     j0-1, which the E update of row j0 needs (or, in cooperative blocks,
//     takes it and the E row above from its neighbours through LDS).
//   * a wave marches z-planes k0..k1-1, carrying E of the next plane and the
//     Ht of the previous plane in registers; it starts one plane early to
//     recompute Ht(k0-1).
// A step reads the state buffer of step n and writes that of step n+1, and
// likewise the slots of the CPML memories, so a halo recompute reads old values
// no other wave overwrites in this launch, and every recomputed halo value is
// bitwise equal to the one its owner stores (same expression, same inputs, no
// contraction).  Every load is unconditional: rows outside the grid are ghost
// rows, columns and planes outside it are read past the buffer; all zero.
//
// A CPML tile's class (bit a: it meets the absorbing slab of axis a) picks
// an instantiation with the CPML code of exactly those axes, or the shell
// runs the code of all three.
//
// Launch: blocks of 4 (or 8) waves, dispatched round-robin over the 8 XCDs;
// the block index is remapped so each XCD receives one contiguous run of
// tiles and neighbouring tiles (sharing halo rows) meet in the same L2.
#include "yo_device.h"

namespace {

// What the CPML code needs of the plan and the right-hand side, read once
// per tile before any store (a store to global memory would otherwise make
// the compiler reload the descriptors with vector loads and wait for them),
// plus the y and z profile coefficients of the tile's rows and planes, one
// row (plane) per lane, taken out with readlane when used.
struct CpmlCtx {
    int ny, nz, ns;
    int plo[3], phi[3], W[3];
    unsigned so[3];          // each axis' memories in a slot, bytes
    int xrow, xw;            // x-slab rows: bytes per row and per value
    Rsrc po, pn;             // this right-hand side's CPML memories, the slots read and written
    Cpml cyE, cyH;           // lane l: row j0 - 1 + l
    Cpml czE, czH;           // lane l: plane k0 - 1 + l
    int j0m, k0m;            // j0 - 1, k0 - 1
};

// Byte offset of the memories of axis A at row j of plane k within a slot, the
// wave-uniform part; false when the row is outside the axis' slabs (x-slab:
// the lane part decides).
template <int A>
__device__ __forceinline__ bool psi_at(const CpmlCtx &C, int j, int k, unsigned &o)
{
    if (A == 0) {
        o = (unsigned)(k * C.ny + j) * C.xrow;
        return true;
    }
    if (A == 1) {
        const int py = slab_index(j, C.ny, C.plo[1], C.phi[1]);
        o = (unsigned)((k * C.W[1] + py) * C.ns) * 1024u;
        return py >= 0;
    }
    const int pz = slab_index(k, C.nz, C.plo[2], C.phi[2]);
    o = (unsigned)((pz * C.ny + j) * C.ns) * 1024u;
    return pz >= 0;
}

// CPML corrections of the six differences of one Ht site row (row j, plane
// k): each difference inside an absorbing slab of its axis becomes d/kp + psi
// with psi <- b psi + c d.  Ht's memories are read from one slot and written
// to another (halo rows recompute Ht, reading psi of the old step); only the
// owner writes the new value.  PRE: the old values were loaded with the
// plane's fields (q[axis][component]); else they are loaded here.
template <int A, bool PRE>
__device__ __forceinline__ void psi_pair(const CpmlCtx &C, int v, int j, int k, const LaneX &L, const Cpml &c,
                                         bool store, const float (&q)[2], float &d0, float &d1)
{
    unsigned o;
    if (!psi_at<A>(C, j, k, o)) return;
    if (A == 0 && L.px < 0) return;
    const int vl = A == 0 ? L.px : L.xp + 256 * v, st = A == 0 ? C.xw : 256;
    const unsigned ov = A == 0 ? o + v * C.xw : o;
    float n0, n1;
    d0 = pml_diff(d0, c, PRE ? q[0] : bload(C.po, vl, C.so[A] + ov), n0);
    d1 = pml_diff(d1, c, PRE ? q[1] : bload(C.po, vl, C.so[A] + ov + st), n1);
    if (store) {
        const int vs = A == 0 ? L.px : L.xps + 256 * v;
        bstore(n0, C.pn, vs, C.so[A] + ov);
        bstore(n1, C.pn, vs, C.so[A] + ov + st);
    }
}

template <int PM, bool PRE>
__device__ __forceinline__ void h_cpml(const CpmlCtx &C, int j, int k, const LaneX &L, const Cpml &cxH, bool own_row,
                                       const float (&q)[3][2], float &dxEz, float &dxEy, float &dyEz,
                                       float &dyEx, float &dzEy, float &dzEx)
{
    if (j < 0 || j >= C.ny || k < 0) return;
    if (PM & 1)   // Hy, Hz
        psi_pair<0, PRE>(C, 2, j, k, L, cxH, own_row && L.own, q[0], dxEz, dxEy);
    if (PM & 2)   // Hx, Hz
        psi_pair<1, PRE>(C, 2, j, k, L, lane_cpml(C.cyH, j - C.j0m), own_row && L.st, q[1], dyEz, dyEx);
    if (PM & 4)   // Hx, Hy
        psi_pair<2, PRE>(C, 2, j, k, L, lane_cpml(C.czH, k - C.k0m), own_row && L.st, q[2], dzEy, dzEx);
}

// CPML corrections of the six differences of one owned E site row, from the
// slot of the state read to that of the state written.  PRE as for h_cpml.
template <int PM, bool PRE>
__device__ __forceinline__ void e_cpml(const CpmlCtx &C, int j, int k, const LaneX &L, const Cpml &cxE,
                                       const float (&q)[3][2], float &dxHz, float &dxHy, float &dyHz,
                                       float &dyHx, float &dzHy, float &dzHx)
{
    if (PM & 1)   // Ey, Ez
        psi_pair<0, PRE>(C, 0, j, k, L, cxE, L.own, q[0], dxHz, dxHy);
    if (PM & 2)   // Ex, Ez
        psi_pair<1, PRE>(C, 0, j, k, L, lane_cpml(C.cyE, j - C.j0m), L.st, q[1], dyHz, dyHx);
    if (PM & 4)   // Ex, Ey
        psi_pair<2, PRE>(C, 0, j, k, L, lane_cpml(C.czE, k - C.k0m), L.st, q[2], dzHy, dzHx);
}

// Old CPML memories v, v + 1 (0: E's, 2: Ht's) of every axis in PM at one
// row, or 0 where `use` is false or the lane is outside the slab (its offset
// is past the buffer, so the load moves no data and the loads need no branch).
template <int PM>
__device__ __forceinline__ void psi_preload(const CpmlCtx &C, int v, int j, int k, const LaneX &L, bool use,
                                            float (&out)[3][2])
{
    unsigned o;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (!(PM & (1 << a))) continue;
        bool in = a == 0 ? psi_at<0>(C, j, k, o) : a == 1 ? psi_at<1>(C, j, k, o) : psi_at<2>(C, j, k, o);
        in = in && use;
        const int vl = !in ? kFar : a == 0 ? (L.px >= 0 ? L.px : kFar) : L.xp + 256 * v;
        const unsigned so = in ? C.so[a] + o + (a == 0 ? v * C.xw : 0) : 0u, st = !in ? 0u : a == 0 ? C.xw : 256u;
        out[a][0] = bload(C.po, vl, so);
        out[a][1] = bload(C.po, vl, so + st);
    }
}

// Exchange slots of a cooperative block, per plane parity and wave: Ex and
// Ez of the wave's first row (next plane), Ht_x and Ht_z of its last row.
#define YO_XS_FLOATS (2 * YO_MAX_WPB * 4 * 64)

// One wave's share of a tile.  COOP = false: the tile is the wave's own
// (rows j0 .. j0+jn-1); the wave loads the E rows above and below and
// recomputes the Ht row below.  COOP = true: the tile is the block's, its
// waves are stacked in y (wave w owns rows J0 + w TY ...), and neighbouring
// waves hand each other the one row they share through LDS: Ex, Ez of the
// row above and Ht_x, Ht_z of the row below.  Only the block's bottom wave
// recomputes the Ht row below the block and only its top wave loads the E
// row above it; one barrier per plane.
template <int TY, int PM, bool COOP, bool PF>
__device__ __forceinline__ void wave_step(const YoPlanD &P, const YoRhsD &R, const int now,
                                          const int4 t, const int w, const int lane, float *xs)
{
    const int ny = P.ny, nz = P.nz;
    const int rows = ny + 1;
    const unsigned gs = 1536u * P.ns;                         // state of one row, bytes (kappa: half)
    const int nxt = buf_next(&P, now, 1);
    const Rsrc Fo = rsrc_of(R.F[now], array_bytes(&P, 6));
    const Rsrc Fn = rsrc_of(R.F[nxt], array_bytes(&P, 6));
    const Rsrc K = rsrc_of(P.kappa, array_bytes(&P, 3));
    const float sx = P.sx, sy = P.sy, sz = P.sz;

    const int x0 = t.x & 0xffff, xn = t.x >> 16;
    const int J0 = t.y & 0xffff, JN = t.y >> 16;
    const int k0 = t.z & 0xffff, k1 = yo_high(t.z);
    const int j0 = COOP ? J0 + w * TY : J0;
    const int jn = COOP ? clampi(JN - w * TY, 0, TY) : JN;
    const bool bottom = !COOP || w == 0;
    const bool top = !COOP || JN - w * TY <= TY;        // no rows of the tile above this wave
    if (COOP && jn == 0) {
        // past the tile's last row: nothing to compute, but keep the barriers
        for (int k = k0 - 1; k < k1; ++k) block_sync_lds();
        return;
    }
    // this wave's slots; a neighbour's are 4 * 64 floats below or above
    float *const xme = COOP ? xs + w * 4 * 64 + lane : nullptr;
    auto xslot = [&](int pp, int dw, int c) -> float & {
        return xme[(pp * YO_MAX_WPB + dw) * 4 * 64 + c * 64];
    };
    // lanes past the halo lane after the last owned one take no part: their
    // column offset lies past every buffer, so their loads move no data (a
    // narrow strip costs only its own columns)
    LaneX L = lane_x(&P, x0, xn, lane);
    const int x = L.x;
    const int xo = L.xl, xh = L.xl + 768, xs_ = L.xs;
    const bool st_x = L.st;
    // wave-uniform byte offsets of row (j, k) in the state and kappa arrays, and
    // the lane's for loads from plane k (past the buffer outside the grid)
    auto ro = [&](int j, int k) -> unsigned {
        return (unsigned)(clampi(k, 0, nz - 1) * rows + (clampi(j, -1, ny) + 1)) * gs;
    };
    auto at = [&](int v, int k) -> int { return k >= 0 && k < nz ? v : kFar; };
    auto rk = [&](int j, int k) -> unsigned { return ro(j, k) >> 1; };

    // ---- CPML data (CPML classes only), read before any store ----
    Cpml cxE = {1.0f, 0.0f, 1.0f}, cxH = {1.0f, 0.0f, 1.0f};
    CpmlCtx C;
    if (PM) {
        C.ny = ny; C.nz = nz; C.ns = P.ns;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            C.plo[a] = P.plo[a];
            C.phi[a] = P.phi[a];
            C.W[a] = P.plo[a] + P.phi[a];
            C.so[a] = 4u * P.psi_off[a];
        }
        C.xrow = P.psi_xrow * 4;
        C.xw = P.psi_xw * 4;
        C.po = psi_rsrc(&P, R.psi, now);
        C.pn = psi_rsrc(&P, R.psi, nxt);
        C.j0m = j0 - 1;
        C.k0m = k0 - 1;
        const Cpml one = {1.0f, 0.0f, 1.0f};
        C.cyE = C.cyH = C.czE = C.czH = one;
        if ((PM & 2) && lane <= TY) {
            const int jj = j0 - 1 + lane;
            if (jj >= 0 && jj < ny && slab_index(jj, ny, P.plo[1], P.phi[1]) >= 0) {
                C.cyE = cpml_at(P.prof[1], 0, jj);
                C.cyH = cpml_at(P.prof[1], 1, jj);
            }
        }
        if (PM & 4) {
            const int kk = k0 - 1 + lane;
            if (kk >= 0 && kk < k1 && slab_index(kk, nz, P.plo[2], P.phi[2]) >= 0) {
                C.czE = cpml_at(P.prof[2], 0, kk);
                C.czH = cpml_at(P.prof[2], 1, kk);
            }
        }
        if (PM & 1) lane_xslab(&P, L, cxE, cxH);
    }

    float Ec[3][TY + 2], Enx[3][TY + 2];
    float Hp[2][TY];          // Ht_x, Ht_y of the previous plane, rows j0..j0+TY-1
    float Hc[3][TY + 1];      // Ht of the current plane, rows j0-1..j0+TY-1
    float Ho_[3][TY + 1], Kv[3][TY];

    // Plane k works on E(k) in Ec, E(k+1) in Enx, old Ht(k) in Ho_ and
    // kappa(k) in Kv.  PF (prefetch): those are in registers when plane k
    // starts, and the loads for plane k+1 are issued before plane k's stores,
    // because the vector-memory counter also counts stores and a wait placed
    // after them would wait for the stores too.  Without PF a plane loads its
    // own operands (fewer registers, more waves to hide the latency).
    // rows a wave never loads (the row below unless bottom, the row above
    // unless top) are filled from neighbours or never read
    auto load_plane = [&](int k, float (&en)[3][TY + 2], float (&ho)[3][TY + 1],
                          float (&kv)[3][TY]) {
        const int ve = at(xo, k + 1), vh = at(xh, k), vk = at(L.xk, k);
#pragma unroll
        for (int r = 1; r <= TY; ++r) {
            const int o = ro(j0 - 1 + r, k + 1);
#pragma unroll
            for (int c = 0; c < 3; ++c) en[c][r] = bload(Fo, ve + 256 * c, o);
        }
#pragma unroll
        for (int r = 1; r <= TY; ++r) {
            const int o = ro(j0 - 1 + r, k);
#pragma unroll
            for (int c = 0; c < 3; ++c) ho[c][r] = bload(Fo, vh + 256 * c, o);
        }
#pragma unroll
        for (int r = 1; r <= TY; ++r) {
            const int o = rk(j0 - 1 + r, k);
#pragma unroll
            for (int c = 0; c < 3; ++c) kv[c][r - 1] = bload(K, vk + 256 * c, o);
        }
        // last, so that the branches do not blur the wait counts of the rest
        if (bottom) {
            const int oe = ro(j0 - 1, k + 1), oh = ro(j0 - 1, k);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                en[c][0] = bload(Fo, ve + 256 * c, oe);
                ho[c][0] = bload(Fo, vh + 256 * c, oh);
            }
        }
        if (top) {
            // only Ex and Ez of the row above enter (as y-differences)
            const int o = ro(j0 + TY, k + 1);
            en[0][TY + 1] = bload(Fo, ve, o);
            en[2][TY + 1] = bload(Fo, ve + 512, o);
        }
    };

#pragma unroll
    for (int c = 0; c < 3; ++c) {
        Ec[c][0] = Enx[c][0] = Ho_[c][0] = Hc[c][0] = 0.0f;
        Ec[c][TY + 1] = Enx[c][TY + 1] = 0.0f;
    }
#pragma unroll
    for (int r = 0; r < TY + 2; ++r) {
        if (r == 0 && !bottom) continue;
        const int o = ro(j0 - 1 + r, k0 - 1);
#pragma unroll
        for (int c = 0; c < 3; ++c) Ec[c][r] = bload(Fo, at(xo, k0 - 1) + 256 * c, o);
    }
#pragma unroll
    for (int r = 0; r < TY; ++r) { Hp[0][r] = 0.0f; Hp[1][r] = 0.0f; }
    if (PF) load_plane(k0 - 1, Enx, Ho_, Kv);

    for (int k = k0 - 1; k < k1; ++k) {
        const bool own_k = (k >= k0);
        float Enx2[3][TY + 2], Ho2[3][TY + 1], Kv2[3][TY];
        if (PF) {
            // unconditional (the last plane re-reads itself) so the wait counts stay exact
            load_plane(k + 1 < k1 ? k + 1 : k, Enx2, Ho2, Kv2);
        } else {
            load_plane(k, Enx, Ho_, Kv);
        }
        // CPML tiles without prefetch: the plane's old CPML memories are
        // loaded here with its fields, so one wait covers both
        constexpr bool PRE = PM != 0 && !PF;
        float qH[TY + 1][3][2], qE[TY][3][2];
        if constexpr (PRE) {
            const bool kin = k >= 0 && k < nz;
#pragma unroll
            for (int r = 0; r <= TY; ++r) {
                const int j = j0 - 1 + r;
                const bool use = (r > 0 || bottom) && kin && j >= 0 && j < ny;
                psi_preload<PM>(C, 2, j, k, L, use, qH[r]);
            }
#pragma unroll
            for (int r = 1; r <= TY; ++r) {
                const bool use = k >= k0 && r <= jn;
                psi_preload<PM>(C, 0, j0 - 1 + r, k, L, use, qE[r - 1]);
            }
        }
        const int pp = k & 1;
        if (COOP) {
            // E of plane k+1, first row: the wave below's row above
            xslot(pp, 0, 0) = Enx[0][1];
            xslot(pp, 0, 1) = Enx[2][1];
        }

        // ---------------- Ht at plane k, rows j0-1 .. j0+TY-1 ----------------
#pragma unroll
        for (int r = 0; r <= TY; ++r) {
            if (r == 0 && !bottom) continue;
            const int j = j0 - 1 + r;
            const float ez_i1 = shfl_next(Ec[2][r]);
            const float ey_i1 = shfl_next(Ec[1][r]);
            float dyEz = Ec[2][r + 1] - Ec[2][r];
            float dzEy = Enx[1][r] - Ec[1][r];
            float dzEx = Enx[0][r] - Ec[0][r];
            float dxEz = ez_i1 - Ec[2][r];
            float dxEy = ey_i1 - Ec[1][r];
            float dyEx = Ec[0][r + 1] - Ec[0][r];
            const bool own_row = own_k && (r >= 1) && (r <= jn);
            if (PM) h_cpml<PM, PRE>(C, j, k, L, cxH, own_row, qH[r], dxEz, dxEy, dyEz, dyEx, dzEy, dzEx);
            const float hx = Ho_[0][r] - fmaf(sy, dyEz, -(sz * dzEy));
            const float hy = Ho_[1][r] - fmaf(sz, dzEx, -(sx * dxEz));
            const float hz = Ho_[2][r] - fmaf(sx, dxEy, -(sy * dyEx));
            Hc[0][r] = hx;
            Hc[1][r] = hy;
            Hc[2][r] = hz;
            if (own_row && st_x) {
                const unsigned o = ro(j, k);
                bstore_nt(hx, Fn, xs_ + 768, o);
                bstore_nt(hy, Fn, xs_ + 1024, o);
                bstore_nt(hz, Fn, xs_ + 1280, o);
            }
        }
        if (COOP) {
            xslot(pp, 0, 2) = Hc[0][TY];
            xslot(pp, 0, 3) = Hc[2][TY];
            block_sync_lds();
            if (!bottom) {
                Hc[0][0] = xslot(pp, -1, 2);
                Hc[2][0] = xslot(pp, -1, 3);
            }
            if (!top) {
                Enx[0][TY + 1] = xslot(pp, 1, 0);
                Enx[2][TY + 1] = xslot(pp, 1, 1);
            }
        }
        // ---------------- E at plane k, rows j0 .. j0+jn-1 ----------------
#pragma unroll
        for (int r = 1; r <= TY; ++r) {
            const int j = j0 - 1 + r;
            const float hz_im = shfl_prev(Hc[2][r]);
            const float hy_im = shfl_prev(Hc[1][r]);
            if (!own_k || r > jn) continue;
            float dyHz = Hc[2][r] - Hc[2][r - 1];
            float dzHy = Hc[1][r] - Hp[1][r - 1];
            float dzHx = Hc[0][r] - Hp[0][r - 1];
            float dxHz = Hc[2][r] - hz_im;
            float dxHy = Hc[1][r] - hy_im;
            float dyHx = Hc[0][r] - Hc[0][r - 1];
            if (PM) e_cpml<PM, PRE>(C, j, k, L, cxE, qE[r - 1], dxHz, dxHy, dyHz, dyHx, dzHy, dzHx);
            float ex = fmaf(Kv[0][r - 1], fmaf(sy, dyHz, -(sz * dzHy)), Ec[0][r]);
            float ey = fmaf(Kv[1][r - 1], fmaf(sz, dzHx, -(sx * dxHz)), Ec[1][r]);
            float ez = fmaf(Kv[2][r - 1], fmaf(sx, dxHy, -(sy * dyHx)), Ec[2][r]);
            // perfect conductor: tangential E on the planes i=0, j=0, k=0
            ex = (j == 0 || k == 0) ? 0.0f : ex;
            ey = (x == 0 || k == 0) ? 0.0f : ey;
            ez = (x == 0 || j == 0) ? 0.0f : ez;
            if (st_x) {
                const unsigned o = ro(j, k);
                bstore_nt(ex, Fn, xs_, o);
                bstore_nt(ey, Fn, xs_ + 256, o);
                bstore_nt(ez, Fn, xs_ + 512, o);
            }
        }
#pragma unroll
        for (int r = 1; r <= TY; ++r) {
            Hp[0][r - 1] = Hc[0][r];
            Hp[1][r - 1] = Hc[1][r];
        }
#pragma unroll
        for (int r = 0; r < TY + 2; ++r) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                Ec[c][r] = Enx[c][r];
                if (PF) Enx[c][r] = Enx2[c][r];
            }
        }
        if (PF) {
#pragma unroll
            for (int r = 0; r <= TY; ++r) {
#pragma unroll
                for (int c = 0; c < 3; ++c) Ho_[c][r] = Ho2[c][r];
            }
#pragma unroll
            for (int r = 0; r < TY; ++r) {
#pragma unroll
                for (int c = 0; c < 3; ++c) Kv[c][r] = Kv2[c][r];
            }
        }
    }
}

// PM = YO_PM_ANY: tiles of every CPML class in one launch, each tile's class
// (int4 .w) selecting its code.
#define YO_PM_ANY 8
template <int PM, bool COOP, bool PF, int TY>
__device__ __forceinline__ void tile_step(const YoPlanD &P, const YoRhsD &R, int now, const int4 t,
                                          int w, int lane, float *xs)
{
    if constexpr (PM == YO_PM_ANY) {
        switch (t.w) {
        case 1: wave_step<TY, 1, COOP, PF>(P, R, now, t, w, lane, xs); break;
        case 2: wave_step<TY, 2, COOP, PF>(P, R, now, t, w, lane, xs); break;
        case 3: wave_step<TY, 3, COOP, PF>(P, R, now, t, w, lane, xs); break;
        case 4: wave_step<TY, 4, COOP, PF>(P, R, now, t, w, lane, xs); break;
        case 5: wave_step<TY, 5, COOP, PF>(P, R, now, t, w, lane, xs); break;
        case 6: wave_step<TY, 6, COOP, PF>(P, R, now, t, w, lane, xs); break;
        case 7: wave_step<TY, 7, COOP, PF>(P, R, now, t, w, lane, xs); break;
        default: wave_step<TY, 0, COOP, PF>(P, R, now, t, w, lane, xs); break;
        }
    } else {
        wave_step<TY, PM, COOP, PF>(P, R, now, t, w, lane, xs);
    }
}

// TY: rows per wave (YO_TY; YO_TY2 for the taller shell tiles)
template <int PM, bool COOP, bool PF, int TY = YO_TY>
__global__ __launch_bounds__(64 * YO_MAX_WPB) void k_yee_step(const YoStepArgs a)
{
    const int nb = gridDim.x, b = blockIdx.x;
    const int q = nb >> 3, rem = nb & 7, xcd = b & 7, pos = b >> 3;
    const int lb = (xcd < rem) ? xcd * (q + 1) + pos : rem * (q + 1) + (xcd - rem) * q + pos;
    const int wpb = a.wpb;
    // the wave index is the same in every lane: say so, so that everything
    // derived from it (slot, tile, row offsets) lives in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane(lb * wpb + (int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    // every early exit below is uniform over the block (slot prefixes are
    // whole blocks), as the cooperative variant's barriers require
    if (wave >= a.total_waves) return;
    int s = 0;
    while (s + 1 < a.n_slots && wave >= a.prefix[s + 1]) ++s;
    const YoSlot sl = a.slot[s];
    const YoPlanD &P = *sl.plan;
    const int step = *P.step_ctr + a.k_offset;
    if (step >= P.n_steps) return;
    const int now = buf_now(P, step, a.b_offset);
    const int local = wave - a.prefix[s];
    if (COOP) {
        // one tile per block; consecutive blocks take the same tile for the
        // next right-hand sides, which share kappa
        __shared__ float xs[YO_XS_FLOATS];
        const int blk = local / wpb;
        const int w = local - blk * wpb;
        const int r = sl.rhs0 + blk % sl.nrhs;
        const int ti = blk / sl.nrhs;
        if (ti >= sl.ntile) return;
        tile_step<PM, true, PF, TY>(P, P.rhs[r], now, sl.tiles[ti], w, lane, xs);
    } else {
        // A block's waves take consecutive tiles (neighbouring x-strips of
        // the same rows) of one right-hand side, so together they stream
        // contiguous row segments and share the cache lines at the strips'
        // edges; consecutive blocks take the same tiles for the next
        // right-hand sides, which share kappa.
        const int grp = local / (wpb * sl.nrhs);
        const int in_grp = local - grp * (wpb * sl.nrhs);
        const int r = sl.rhs0 + in_grp / wpb;
        const int ti = grp * wpb + in_grp % wpb;
        if (ti >= sl.ntile) return;
        tile_step<PM, false, PF, TY>(P, P.rhs[r], now, sl.tiles[ti], 0, lane, nullptr);
    }
}

// ---------------------------------------------------------------------------
// Two steps per sweep (temporal blocking) for the tiles of the two-step region
// R2 (YoPlanD::r2), which lies two cells clear of every absorbing slab and of
// every source plane, so neither step needs CPML code or a source term there.
// A wave owns x in [x0, x0+xn) (xn <= 60; lane l holds x = x0 - 2 + l), rows
// j0..j0+jn-1 (jn <= TY) and planes k0..k1-1, reads the state after step n
// (buffer n % 3) and writes the state after step n+2 (buffer (n+2) % 3),
// recomputing from step n's values everything the second step needs around
// its cells: step n+1 on lanes 1..62, rows j0-1..j0+TY and planes k0-1..k1,
// step n+1's Ht on one more lane, row and plane below.  Marching up z, it
// takes step n+1 at plane k and step n+2 at plane k-1 in the same pass (a
// wavefront in z-t), so each plane's state is read once for both steps.
// The cells of R2's outermost layer also get their step-n+1 state written
// (buffer (n+1) % 3): the single steps of the tiles around R2 read it.
// Every value is computed with the expression and the operand order of the
// single-step kernel, so the two paths give bitwise the same fields.
// ZP: the tiles of the z-slabs under R2's x-y footprint (planes down to 0 and
// up to nz - 1), with the z-axis CPML code of the single-step kernel: a wave
// reads the memories of slot n % 3 around its cells, keeps step n+1's new
// ones in registers for the second step, and writes slot (n+2) % 3 of its own
// cells and, for R2's outermost layer, the Ht memories of step n+1 (slot
// (n+1) % 3), which the single steps around read.  Planes past the grid are
// the perfect conductor's zeros.
// COOP: the tile is the block's, its waves stacked in y (wave w owns rows
// J0 + w TY ...); each wave loads its own rows of step n and the rows it
// shares with the waves below and above come through LDS (E^n of the two
// rows below and above, Ht^{n-1/2} of the two below and one above; one
// barrier per plane, two parities), so only the block's bottom and top
// waves load the block's halo rows.
template <int TY, bool ZP, bool COOP = false>
__device__ __forceinline__ void wave_step2(const YoPlanD &P, const YoRhsD &R, const int step,
                                           const int4 t, const int w, const int wpb, const int lane,
                                           float *xs)
{
    const int ny = P.ny, nz = P.nz;
    const int rows = ny + 1;
    const unsigned gs = 1536u * P.ns;
    const int nb = P.nbuf;
    const Rsrc FA = rsrc_of(R.F[step % nb], array_bytes(&P, 6));          // after step n
    const Rsrc FB = rsrc_of(R.F[(step + 1) % nb], array_bytes(&P, 6));    // after n+1 (rim)
    const Rsrc FC = rsrc_of(R.F[(step + 2) % nb], array_bytes(&P, 6));    // after n+2
    const Rsrc K = rsrc_of(P.kappa, array_bytes(&P, 3));
    const float sx = P.sx, sy = P.sy, sz = P.sz;

    const int x0 = t.x & 0xffff, xn = t.x >> 16;
    const int J0 = t.y & 0xffff, JN = t.y >> 16;
    const int k0 = t.z & 0xffff, k1 = yo_high(t.z);
    const int j0 = COOP ? J0 + w * TY : J0;
    const int jn = COOP ? clampi(JN - w * TY, 0, TY) : JN;
    const bool bottom = !COOP || w == 0;
    const bool top = !COOP || JN - w * TY <= TY;        // no rows of the tile above this wave
    if (COOP && jn == 0) {
        // past the tile's last row: nothing to compute, but keep the barriers
        for (int k = k0 - 2; k <= k1; ++k) block_sync_lds();
        return;
    }
    // exchange slots of this wave (20 per parity: E^n rows TY, TY+1 and Ht
    // rows TY, TY+1 for the wave above; E^n row 2, row 3's Ex and Ez, and Ht
    // row 2 for the wave below); a neighbour's are 20 * 64 floats away
    float *const xme = COOP ? xs + w * 20 * 64 + lane : nullptr;
    auto xslot = [&](int pp, int dw, int q) -> float & {
        return xme[(pp * wpb + dw) * 20 * 64 + q * 64];
    };
    const LaneX L = lane_x(&P, x0, xn, lane);
    const int x = L.x, xo = L.xl, xh = L.xl + 768, xs_ = L.xs;
    const bool own_x = L.own, st_x = L.st;
    // R2's outermost layer, whose step-n+1 state the tiles around R2 read
    const int ra0 = P.r2[0], ra1 = P.r2[1], rb0 = P.r2[2], rb1 = P.r2[3], rc0 = P.r2[4], rc1 = P.r2[5];
    const bool rim_x = own_x && (x == ra0 || x == ra1 - 1);
    // z-axis CPML memories (ZP): the slots of the three states, and byte offsets
    // of the memories at row j of slab plane pz
    const int zlo = P.plo[2], zhi = P.phi[2];
    const Rsrc P0 = psi_rsrc(&P, R.psi, step % 3), P1 = psi_rsrc(&P, R.psi, (step + 1) % 3),
               P2 = psi_rsrc(&P, R.psi, (step + 2) % 3);
    auto zo = [&](int pz, int j) -> unsigned {
        return 4u * P.psi_off[2] + (unsigned)((pz * ny + j) * P.ns) * 1024u;
    };
    auto ro = [&](int j, int k) -> unsigned {
        return (unsigned)(clampi(k, 0, nz - 1) * rows + (clampi(j, -1, ny) + 1)) * gs;
    };
    auto at = [&](int v, int k) -> int { return k >= 0 && k < nz ? v : kFar; };
    auto rk = [&](int j, int k) -> unsigned { return ro(j, k) >> 1; };
    // row index r: j = j0 - 2 + r
    constexpr int NE = TY + 4;     // E^n rows 0..TY+3 (the last: Ex and Ez only)
    constexpr int NH = TY + 3;     // Ht^{n-1/2} and Ht^{n+1/2} rows 0..TY+2
    float Ec[3][NE], Enx[3][NE];   // E^n at planes k and k+1
    float Ho[3][NH];               // Ht^{n-1/2} at plane k
    float Hh[3][NH], Hhp[3][NH];   // Ht^{n+1/2} at planes k and k-1
    float Kc[3][NH], Kp[3][NH];    // kappa at planes k and k-1 (rows 1..TY+2)
    float E1c[3][NH], E1p[3][NH];  // E^{n+1} at planes k and k-1 (rows 1..TY+2)
    float H2[3][NH], H2p[2][NH];   // Ht^{n+3/2} at planes k-1 and k-2 (rows 1..TY+1)
    // ZP: z memories of step n+1 (Ht rows 0..TY+2, E rows 1..TY+2) at
    // planes k and k-1, with the planes' coefficients
    float qH1[2][NH], qH1p[2][NH], qE1[2][NH], qE1p[2][NH];
    Cpml czH = {1.0f, 0.0f, 1.0f}, czE = czH, czHp = czH, czEp = czH;
    int pzp = -1;

    // all: every row from memory; else (COOP) the rows a neighbour passes on
    // are left for the exchange
    auto load_e = [&](int k, float (&e)[3][NE], bool all) {
#pragma unroll
        for (int r = 0; r < NE; ++r) {
            if (COOP && !all && ((r < 2 && !bottom) || (r >= TY + 2 && !top))) continue;
            const unsigned o = ro(j0 - 2 + r, k);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if (r == NE - 1 && c == 1) { e[c][r] = 0.0f; continue; }
                e[c][r] = bload(FA, at(xo, k) + 256 * c, o);
            }
        }
    };
    load_e(k0 - 2, Ec, true);
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int r = 0; r < NH; ++r) Hhp[c][r] = E1p[c][r] = Kp[c][r] = H2[c][r] = 0.0f;
#pragma unroll
    for (int r = 0; r < NH; ++r) {
        H2p[0][r] = H2p[1][r] = 0.0f;
        qH1[0][r] = qH1[1][r] = qE1[0][r] = qE1[1][r] = 0.0f;
    }

    for (int k = k0 - 2; k <= k1; ++k) {
        load_e(k + 1, Enx, false);
#pragma unroll
        for (int r = 0; r < NH; ++r) {
            if (COOP && ((r < 2 && !bottom) || (r >= TY + 2 && !top))) continue;
            const unsigned o = ro(j0 - 2 + r, k);
#pragma unroll
            for (int c = 0; c < 3; ++c) Ho[c][r] = bload(FA, at(xh, k) + 256 * c, o);
        }
        if (COOP) {
            // the rows the neighbours share, then theirs
            const int pp = k & 1;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                xslot(pp, 0, c) = Enx[c][TY];
                xslot(pp, 0, 3 + c) = Enx[c][TY + 1];
                xslot(pp, 0, 6 + c) = Ho[c][TY];
                xslot(pp, 0, 9 + c) = Ho[c][TY + 1];
                xslot(pp, 0, 12 + c) = Enx[c][2];
                xslot(pp, 0, 17 + c) = Ho[c][2];
            }
            xslot(pp, 0, 15) = Enx[0][3];
            xslot(pp, 0, 16) = Enx[2][3];
            block_sync_lds();
            if (!bottom) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    Enx[c][0] = xslot(pp, -1, c);
                    Enx[c][1] = xslot(pp, -1, 3 + c);
                    Ho[c][0] = xslot(pp, -1, 6 + c);
                    Ho[c][1] = xslot(pp, -1, 9 + c);
                }
            }
            if (!top) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    Enx[c][TY + 2] = xslot(pp, 1, 12 + c);
                    Ho[c][TY + 2] = xslot(pp, 1, 17 + c);
                }
                Enx[0][TY + 3] = xslot(pp, 1, 15);
                Enx[1][TY + 3] = 0.0f;
                Enx[2][TY + 3] = xslot(pp, 1, 16);
            }
        }
        // ZP: plane k's z coefficients (its memories of step n, slot n % 3,
        // are loaded where used)
        const int pz = ZP ? slab_index(k, nz, zlo, zhi) : -1;
        if (ZP && pz >= 0) {
            czH = cpml_at(P.prof[2], 1, k);
            czE = cpml_at(P.prof[2], 0, k);
        }
        const bool do_e1 = k >= k0 - 1;
        if (do_e1) {
#pragma unroll
            for (int r = 1; r < NH; ++r) {
                const unsigned o = rk(j0 - 2 + r, k);
#pragma unroll
                for (int c = 0; c < 3; ++c) Kc[c][r] = bload(K, at(L.xk, k) + 256 * c, o);
            }
        }
        // ---- step n+1's Ht at plane k, rows 0..TY+2 ----
#pragma unroll
        for (int r = 0; r < NH; ++r) {
            const float ez_i1 = shfl_next(Ec[2][r]);
            const float ey_i1 = shfl_next(Ec[1][r]);
            const float dyEz = Ec[2][r + 1] - Ec[2][r];
            const float dzEy = Enx[1][r] - Ec[1][r];
            const float dzEx = Enx[0][r] - Ec[0][r];
            const float dxEz = ez_i1 - Ec[2][r];
            const float dxEy = ey_i1 - Ec[1][r];
            const float dyEx = Ec[0][r + 1] - Ec[0][r];
            float dzEy_ = dzEy, dzEx_ = dzEx;
            if (ZP && pz >= 0) {
                const unsigned o = zo(pz, j0 - 2 + r);
                dzEy_ = pml_diff(dzEy, czH, bload(P0, L.xp + 512, o), qH1[0][r]);                       // Hx
                dzEx_ = pml_diff(dzEx, czH, bload(P0, L.xp + 768, o), qH1[1][r]);   // Hy
            }
            Hh[0][r] = Ho[0][r] - fmaf(sy, dyEz, -(sz * dzEy_));
            Hh[1][r] = Ho[1][r] - fmaf(sz, dzEx_, -(sx * dxEz));
            Hh[2][r] = Ho[2][r] - fmaf(sx, dxEy, -(sy * dyEx));
            if (ZP && k < 0) Hh[0][r] = Hh[1][r] = Hh[2][r] = 0.0f;   // ghost plane
        }
        if (do_e1) {
            // ---- step n+1's E at plane k, rows 1..TY+2 ----
            const bool own_k = k >= k0 && k < k1;
            const bool rim_k = k == rc0 || k == rc1 - 1;
#pragma unroll
            for (int r = 1; r < NH; ++r) {
                const int j = j0 - 2 + r;
                const float hz_im = shfl_prev(Hh[2][r]);
                const float hy_im = shfl_prev(Hh[1][r]);
                const float dyHz = Hh[2][r] - Hh[2][r - 1];
                const float dzHy = Hh[1][r] - Hhp[1][r];
                const float dzHx = Hh[0][r] - Hhp[0][r];
                const float dxHz = Hh[2][r] - hz_im;
                const float dxHy = Hh[1][r] - hy_im;
                const float dyHx = Hh[0][r] - Hh[0][r - 1];
                float dzHy_ = dzHy, dzHx_ = dzHx;
                if (ZP && pz >= 0) {
                    const unsigned o = zo(pz, j);
                    dzHy_ = pml_diff(dzHy, czE, bload(P0, L.xp, o), qE1[0][r]);                       // Ex
                    dzHx_ = pml_diff(dzHx, czE, bload(P0, L.xp + 256, o), qE1[1][r]);   // Ey
                }
                float ex = fmaf(Kc[0][r], fmaf(sy, dyHz, -(sz * dzHy_)), Ec[0][r]);
                float ey = fmaf(Kc[1][r], fmaf(sz, dzHx_, -(sx * dxHz)), Ec[1][r]);
                float ez = fmaf(Kc[2][r], fmaf(sx, dxHy, -(sy * dyHx)), Ec[2][r]);
                ex = (j == 0 || k == 0) ? 0.0f : ex;
                ey = (x == 0 || k == 0) ? 0.0f : ey;
                ez = (x == 0 || j == 0) ? 0.0f : ez;
                if (ZP && (k < 0 || k >= nz)) ex = ey = ez = 0.0f;   // ghost planes stay zero
                E1c[0][r] = ex;
                E1c[1][r] = ey;
                E1c[2][r] = ez;
                // the step-n+1 state of R2's outermost layer
                const bool own_r = r >= 2 && r - 2 < jn;
                if (own_k && own_r && ((st_x && (rim_k || j == rb0 || j == rb1 - 1)) || rim_x)) {
                    const unsigned o = ro(j, k);
                    bstore_nt(ex, FB, xs_, o);
                    bstore_nt(ey, FB, xs_ + 256, o);
                    bstore_nt(ez, FB, xs_ + 512, o);
                    bstore_nt(Hh[0][r], FB, xs_ + 768, o);
                    bstore_nt(Hh[1][r], FB, xs_ + 1024, o);
                    bstore_nt(Hh[2][r], FB, xs_ + 1280, o);
                    if (ZP && pz >= 0) {
                        bstore(qH1[0][r], P1, L.xps + 512, zo(pz, j));
                        bstore(qH1[1][r], P1, L.xps + 768, zo(pz, j));
                    }
                }
            }
        }
        if (k >= k0) {
            // ---- step n+2 at plane km = k-1: Ht rows 1..TY+1, E rows 2..TY+1 ----
            const int km = k - 1;
#pragma unroll
            for (int r = 1; r <= TY + 1; ++r) {
                const float ez_i1 = shfl_next(E1p[2][r]);
                const float ey_i1 = shfl_next(E1p[1][r]);
                const float dyEz = E1p[2][r + 1] - E1p[2][r];
                const float dzEy = E1c[1][r] - E1p[1][r];
                const float dzEx = E1c[0][r] - E1p[0][r];
                const float dxEz = ez_i1 - E1p[2][r];
                const float dxEy = ey_i1 - E1p[1][r];
                const float dyEx = E1p[0][r + 1] - E1p[0][r];
                float dzEy_ = dzEy, dzEx_ = dzEx;
                if (ZP && pzp >= 0) {
                    float n0, n1;
                    dzEy_ = pml_diff(dzEy, czHp, qH1p[0][r], n0);   // Hx
                    dzEx_ = pml_diff(dzEx, czHp, qH1p[1][r], n1);   // Hy
                    if (st_x && r >= 2 && r - 2 < jn && km >= k0 && km < k1) {
                        const int j = j0 - 2 + r;
                        bstore(n0, P2, L.xps + 512, zo(pzp, j));
                        bstore(n1, P2, L.xps + 768, zo(pzp, j));
                    }
                }
                H2[0][r] = Hhp[0][r] - fmaf(sy, dyEz, -(sz * dzEy_));
                H2[1][r] = Hhp[1][r] - fmaf(sz, dzEx_, -(sx * dxEz));
                H2[2][r] = Hhp[2][r] - fmaf(sx, dxEy, -(sy * dyEx));
                if (ZP && km < 0) H2[0][r] = H2[1][r] = H2[2][r] = 0.0f;   // ghost plane
            }
            if (km >= k0) {
#pragma unroll
                for (int r = 2; r <= TY + 1; ++r) {
                    const int j = j0 - 2 + r;
                    const float hz_im = shfl_prev(H2[2][r]);
                    const float hy_im = shfl_prev(H2[1][r]);
                    if (r - 2 >= jn) continue;
                    const float dyHz = H2[2][r] - H2[2][r - 1];
                    const float dzHy = H2[1][r] - H2p[1][r];
                    const float dzHx = H2[0][r] - H2p[0][r];
                    const float dxHz = H2[2][r] - hz_im;
                    const float dxHy = H2[1][r] - hy_im;
                    const float dyHx = H2[0][r] - H2[0][r - 1];
                    float dzHy_ = dzHy, dzHx_ = dzHx;
                    if (ZP && pzp >= 0) {
                        float n0, n1;
                        dzHy_ = pml_diff(dzHy, czEp, qE1p[0][r], n0);   // Ex
                        dzHx_ = pml_diff(dzHx, czEp, qE1p[1][r], n1);   // Ey
                        if (st_x) {
                            bstore(n0, P2, L.xps, zo(pzp, j));
                            bstore(n1, P2, L.xps + 256, zo(pzp, j));
                        }
                    }
                    float ex = fmaf(Kp[0][r], fmaf(sy, dyHz, -(sz * dzHy_)), E1p[0][r]);
                    float ey = fmaf(Kp[1][r], fmaf(sz, dzHx_, -(sx * dxHz)), E1p[1][r]);
                    float ez = fmaf(Kp[2][r], fmaf(sx, dxHy, -(sy * dyHx)), E1p[2][r]);
                    ex = (j == 0 || km == 0) ? 0.0f : ex;
                    ey = (x == 0 || km == 0) ? 0.0f : ey;
                    ez = (x == 0 || j == 0) ? 0.0f : ez;
                    if (st_x) {
                        const unsigned o = ro(j, km);
                        bstore_nt(ex, FC, xs_, o);
                        bstore_nt(ey, FC, xs_ + 256, o);
                        bstore_nt(ez, FC, xs_ + 512, o);
                        bstore_nt(H2[0][r], FC, xs_ + 768, o);
                        bstore_nt(H2[1][r], FC, xs_ + 1024, o);
                        bstore_nt(H2[2][r], FC, xs_ + 1280, o);
                    }
                }
            }
#pragma unroll
            for (int r = 1; r <= TY + 1; ++r) {
                H2p[0][r] = H2[0][r];
                H2p[1][r] = H2[1][r];
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
#pragma unroll
            for (int r = 0; r < NE; ++r) Ec[c][r] = Enx[c][r];
#pragma unroll
            for (int r = 0; r < NH; ++r) {
                Hhp[c][r] = Hh[c][r];
                E1p[c][r] = E1c[c][r];
                Kp[c][r] = Kc[c][r];
            }
        }
        if (ZP) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int r = 0; r < NH; ++r) {
                    qH1p[c][r] = qH1[c][r];
                    qE1p[c][r] = qE1[c][r];
                }
            czHp = czH;
            czEp = czE;
            pzp = pz;
        }
    }
}

template <bool ZP, int TY, bool COOP>
__global__ __launch_bounds__(64 * YO_MAX_WPB) void k_yee_step2(const YoStepArgs a)
{
    const int nb = gridDim.x, b = blockIdx.x;
    const int q = nb >> 3, rem = nb & 7, xcd = b & 7, pos = b >> 3;
    const int lb = (xcd < rem) ? xcd * (q + 1) + pos : rem * (q + 1) + (xcd - rem) * q + pos;
    const int wpb = a.wpb;
    const int wave = __builtin_amdgcn_readfirstlane(lb * wpb + (int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    if (wave >= a.total_waves) return;
    int s = 0;
    while (s + 1 < a.n_slots && wave >= a.prefix[s + 1]) ++s;
    const YoSlot sl = a.slot[s];
    const YoPlanD &P = *sl.plan;
    const int step = *P.step_ctr + a.k_offset;
    // the host schedules a pair only where both steps remain
    if (step + 1 >= P.n_steps) return;
    const int local = wave - a.prefix[s];
    if (COOP) {
        // one tile per block; consecutive blocks take the same tile for the
        // next right-hand sides (every early exit above is uniform over the
        // block, as the barriers require)
        extern __shared__ float xs2[];
        const int blk = local / wpb;
        const int w = local - blk * wpb;
        const int r = sl.rhs0 + blk % sl.nrhs;
        const int ti = blk / sl.nrhs;
        if (ti >= sl.ntile) return;
        wave_step2<TY, ZP, true>(P, P.rhs[r], step, sl.tiles[ti], w, wpb, lane, xs2);
        return;
    }
    const int grp = local / (wpb * sl.nrhs);
    const int in_grp = local - grp * (wpb * sl.nrhs);
    const int r = sl.rhs0 + in_grp / wpb;
    const int ti = grp * wpb + in_grp % wpb;
    if (ti >= sl.ntile) return;
    wave_step2<TY, ZP, false>(P, P.rhs[r], step, sl.tiles[ti], 0, wpb, lane, nullptr);
}

// locate point q of slot s in the aux work list: whole blocks per right-hand
// side, so that its descriptor is the block's
__device__ __forceinline__ bool aux_point(const YoAuxArgs &a, int &s, int &r, int &q)
{
    const int blk = blockIdx.x;
    s = 0;
    while (s + 1 < a.n_slots && blk >= a.prefix[s + 1]) ++s;
    const int per = (a.npts[s] + 255) / 256;
    if (per <= 0) return false;
    const int lb = blk - a.prefix[s], rr = lb / per;
    r = a.rhs0[s] + rr;
    q = (lb - rr * per) * 256 + (int)threadIdx.x;
    return rr < a.nrhs[s] && q < a.npts[s];
}

// Component plane tt of a port or source plane (normal `axis`, cell index
// `index`): 0, 1 the tangential E (t1, t2) on the plane; 2 the normal E
// (its sites lie half a cell past the plane, stored at the same index);
// 3, 4 the tangential E on the next plane.
__device__ __forceinline__ void plane_component(int axis, int index, int tt, int &c, int &idx)
{
    c = tt == 2 ? axis : (axis + 1 + (tt < 2 ? tt : tt - 3)) % 3;
    idx = index + (tt >= 3 ? 1 : 0);
}

// Running DFT of E^n: S += E^n exp(+i w n dt) on the design box (3 components)
// and the port planes (2 tangential components), for each frequency the
// right-hand side accumulates; under a pulse with a DFT stride m > 1 only the
// steps divisible by m add.  Called before step n, or, with a.pair, after the
// launch that took steps n and n + 1: E^n is still in its buffer, E^{n+1} in
// dft_mid, and each sum is read and written once for both.
__global__ __launch_bounds__(256) void k_dft(const YoAuxArgs a)
{
    int s, r, q;
    if (!aux_point(a, s, r, q)) return;
    const YoPlanD &P = *a.plan[s];
    const int step = *P.step_ctr + a.k_offset;
    if (step >= P.n_steps) return;
    const YoRhsD &R = P.rhs[r];
    auto takes = [&](int n) {
        const int w = n - R.win_start;
        return w >= 0 && w < R.win_len && !(P.dft_stride > 1 && n % P.dft_stride);
    };
    const bool d0 = takes(step), d1 = a.pair && takes(step + 1);
    if (!d0 && !d1) return;
    const float *F = R.F[buf_now(P, step, a.b_offset)];
    const int bx = P.box[3], by = P.box[4], bz = P.box[5];
    const int bsz = bx * by * bz;
    const float e1 = d1 ? R.dft_mid[q] : 0.0f;
    float e;
    float2 *acc;
    int fstride;
    if (q < 3 * bsz) {
        const int c = q / bsz, rem = q - c * bsz;
        const int bk = rem / (bx * by), rem2 = rem - bk * bx * by;
        const int bj = rem2 / bx, bi = rem2 - bj * bx;
        e = F[yo_off(c, P.box[0] + bi, P.box[1] + bj, P.box[2] + bk, P.ny, P.ns, 6)];
        acc = R.dft_box + q;
        fstride = R.box_fstride;
    } else {
        const int qm = q - 3 * bsz;
        int p = 0;
        while (p + 1 < P.n_ports && qm >= P.mon_off[p + 1]) ++p;
        const YoPlaneD pl = P.ports[p];
        const int loc = qm - P.mon_off[p];
        const int plane = pl.n0 * pl.n1;
        const int tt = loc / plane, rem = loc - tt * plane;
        const int b = rem / pl.n0, ai = rem - b * pl.n0;
        int c, idx;
        plane_component(pl.axis, pl.index, tt, c, idx);
        const int cx = sel3(pl.axis, idx, pl.lo0 + ai, pl.lo0 + ai);
        const int cy = sel3(pl.axis, pl.lo0 + ai, idx, pl.lo1 + b);
        const int cz = sel3(pl.axis, pl.lo1 + b, pl.lo1 + b, idx);
        e = F[yo_off(c, cx, cy, cz, P.ny, P.ns, 6)];
        acc = R.dft_mon + qm;
        fstride = R.mon_fstride;
    }
    // four frequencies' sums and phases loaded together: one after another their
    // round trips were most of the kernel's time
    const int nf = R.n_dft;
    for (int f0 = 0; f0 < nf; f0 += 4) {
        float2 v[4], p0[4], p1[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int f = f0 + i;
            if (f >= nf) break;
            const float4 *st = R.dfttab + (size_t)f * P.n_steps + step;
            v[i] = acc[(size_t)f * fstride];
            if (d0) p0[i] = make_float2(st[0].z, st[0].w);
            if (d1) p1[i] = make_float2(st[1].z, st[1].w);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (f0 + i >= nf) break;
            if (d0) {
                v[i].x = fmaf(e, p0[i].x, v[i].x);
                v[i].y = fmaf(e, p0[i].y, v[i].y);
            }
            if (d1) {
                v[i].x = fmaf(e1, p1[i].x, v[i].x);
                v[i].y = fmaf(e1, p1[i].y, v[i].y);
            }
            acc[(size_t)(f0 + i) * fstride] = v[i];
        }
    }
}

// Soft current source of step n (called after step n): E^{n+1} -= kappa j^{n+1/2}
// on the right-hand side's source plane.
__global__ __launch_bounds__(256) void k_source(const YoAuxArgs a)
{
    int s, r, q;
    if (!aux_point(a, s, r, q)) return;
    const YoPlanD &P = *a.plan[s];
    const int step = *P.step_ctr + a.k_offset;
    if (step >= P.n_steps) return;
    const YoRhsD &R = P.rhs[r];
    if (!R.src_j) return;
    const YoPlaneD pl = R.src;
    const int plane = pl.n0 * pl.n1;
    if (q >= R.src_nc * plane) return;
    const float4 st = R.steptab[step];
    const int tt = q / plane, rem = q - tt * plane;
    const int b = rem / pl.n0, ai = rem - b * pl.n0;
    int c, idx;
    plane_component(pl.axis, pl.index, tt, c, idx);
    const int cx = sel3(pl.axis, idx, pl.lo0 + ai, pl.lo0 + ai);
    const int cy = sel3(pl.axis, pl.lo0 + ai, idx, pl.lo1 + b);
    const int cz = sel3(pl.axis, pl.lo1 + b, pl.lo1 + b, idx);
    const size_t o = yo_off(c, cx, cy, cz, P.ny, P.ns, 6);
    const float2 jv = R.src_j[q];
    const float j = fmaf(jv.x, st.x, jv.y * st.y);
    float *F = R.F[buf_next(&P, buf_now(P, step, a.b_offset), 1)];
    F[o] = fmaf(-P.kappa[yo_off(c, cx, cy, cz, P.ny, P.ns, 3)], j, F[o]);
}

// The counters after the launches of a.add steps, of which those within the
// plan's run took place, or at a reset.  Each side keeps its own buffer: the
// number of swaps depends on how a run was cut into calls, and a side's state
// stays where its run left it while the other side runs.
__global__ void k_ctr(const YoCtrArgs a)
{
    const int i = threadIdx.x;
    if (i >= a.n) return;
    const YoPlanD &P = *a.plan[i];
    int *c = P.step_ctr;
    if (!a.add) c[0] = c[1] = 0;
    const int left = max(P.n_steps - c[0], 0);
    const int paired = a.pairs ? a.add & ~1 : 0;
    const int two = min(paired, left) / 2, one = clampi(left - paired, 0, a.add - paired);
    c[0] += a.add;
    c[1] += two + one;
    for (int q = 0; q < 2; ++q)
        if (a.which[i] >> q & 1)
            c[2 + q] = !a.add ? 0 : (c[2 + q] + (P.nbuf == 3 ? 2 * two : two) + one) % P.nbuf;
}

}  // namespace

template <int PM, bool COOP, bool PF, int TY = YO_TY>
static void launch_one(const YoStepArgs &args, int blocks, hipStream_t s)
{
    hipLaunchKernelGGL((k_yee_step<PM, COOP, PF, TY>), dim3(blocks), dim3(64 * args.wpb), 0, s, args);
}

template <int PM>
static void launch_pm(bool coop, bool pf, const YoStepArgs &args, int blocks, hipStream_t s)
{
    if (coop) {
        if (pf) launch_one<PM, true, true>(args, blocks, s);
        else launch_one<PM, true, false>(args, blocks, s);
    } else {
        if (pf) launch_one<PM, false, true>(args, blocks, s);
        else launch_one<PM, false, false>(args, blocks, s);
    }
}

hipError_t yo_launch_step(int pm, bool coop, bool prefetch, const YoStepArgs &args, int blocks,
                          hipStream_t s, int rows)
{
    if (blocks <= 0) return hipSuccess;
    if (args.wpb != 4 && args.wpb != 8) return hipErrorInvalidValue;
    if (rows == YO_TY2) {
        // taller tiles: the CPML shell's independent waves only
        if (coop) return hipErrorInvalidValue;
        if (pm == YO_PM_ANY && prefetch) launch_one<YO_PM_ANY, false, true, YO_TY2>(args, blocks, s);
        else if (pm == YO_PM_ANY) launch_one<YO_PM_ANY, false, false, YO_TY2>(args, blocks, s);
        else if (pm == 7 && prefetch) launch_one<7, false, true, YO_TY2>(args, blocks, s);
        else if (pm == 7) launch_one<7, false, false, YO_TY2>(args, blocks, s);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    if (rows != YO_TY) return hipErrorInvalidValue;
    switch (pm) {
    case 0: launch_pm<0>(coop, prefetch, args, blocks, s); break;
    case 1: launch_pm<1>(coop, prefetch, args, blocks, s); break;
    case 7: launch_pm<7>(coop, prefetch, args, blocks, s); break;
    case YO_PM_ANY: launch_pm<YO_PM_ANY>(coop, prefetch, args, blocks, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t yo_launch_step2(bool zslab, int rows, bool coop, const YoStepArgs &args, int blocks,
                           hipStream_t s)
{
    if (blocks <= 0) return hipSuccess;
    if (args.wpb != 4 && args.wpb != 8) return hipErrorInvalidValue;
    const dim3 g(blocks), b(64 * args.wpb);
    // cooperative: 20 exchange slots of 64 floats per wave and parity
    const size_t lds = (size_t)2 * args.wpb * 20 * 64 * sizeof(float);
    if (zslab && rows == YO_TY && !coop)
        hipLaunchKernelGGL((k_yee_step2<true, YO_TY, false>), g, b, 0, s, args);
    else if (!zslab && rows == YO_TY && !coop)
        hipLaunchKernelGGL((k_yee_step2<false, YO_TY, false>), g, b, 0, s, args);
    else if (!zslab && rows == YO_TY2 && !coop)
        hipLaunchKernelGGL((k_yee_step2<false, YO_TY2, false>), g, b, 0, s, args);
    else if (!zslab && rows == YO_TY && coop)
        hipLaunchKernelGGL((k_yee_step2<false, YO_TY, true>), g, b, lds, s, args);
    else if (!zslab && rows == YO_TY2 && coop)
        hipLaunchKernelGGL((k_yee_step2<false, YO_TY2, true>), g, b, lds, s, args);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t yo_launch_dft(const YoAuxArgs &args, hipStream_t s)
{
    if (args.total_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_dft, dim3(args.total_blocks), dim3(256), 0, s, args);
    return hipGetLastError();
}

hipError_t yo_launch_source(const YoAuxArgs &args, hipStream_t s)
{
    if (args.total_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_source, dim3(args.total_blocks), dim3(256), 0, s, args);
    return hipGetLastError();
}

hipError_t yo_launch_ctr(const YoCtrArgs &args, hipStream_t s)
{
    hipLaunchKernelGGL(k_ctr, dim3(1), dim3(64), 0, s, args);
    return hipGetLastError();
}
