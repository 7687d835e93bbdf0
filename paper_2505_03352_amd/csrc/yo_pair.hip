// The time stepping: two Yee steps per launch over the whole grid, absorbing
// layers and sources inside (temporal blocking), or one.  Update, layout and
// expressions as in yo_step.hip, whose single steps these equal bitwise.
//
// A block of W waves marches up z over one strip of columns (yo_col) and a
// stack of W TY rows, TY a wave; per plane k it takes, from the state after
// step n,
//   S1  Ht^{n+1/2} at plane k      (E^n at k and k+1, Ht^{n-1/2} at k)
//   S2  E^{n+1}    at plane k      (kappa, Ht^{n+1/2} at k and k-1)
//   S3  Ht^{n+3/2} at plane k-1    (E^{n+1} at k-1 and k)
//   S4  E^{n+2}    at plane k-1    (kappa, Ht^{n+3/2} at k-1 and k-2)
// and stores S3 and S4, so a plane's state is read once and written once for
// two steps; a step alone is S1 and S2, stored.  Each row is worked on by one
// wave; the one row a stage needs of the neighbouring wave (above for Ht, below
// for E) comes through LDS, with two barriers per plane.  The rows at the
// block's ends (two below, two above) and the lanes at the strip's (two on
// either side) are recomputed from their own loads and not stored, as are the
// two planes below and one above a z-chunk.
//
// What bounds it: on large grids the traffic between the L2s and memory.  Per
// cell and pair of steps 24 bytes of state in, times 16/12 rows and 64/60
// columns, 24 out and, in planes of more than one kappa, 12 of kappa in;
// counted on 320x240x96 with 6 right-hand sides before kappa's planes: 3.2 GB
// in and 1.4 GB out in 850 us, 5.4 TB/s, no more shared in the L2s than that.
// On small ones the latency of a plane (4 us of a block alone on its CU, 6.5 of
// two): nearly as many scalar as vector instructions, and a quarter to half of
// the waves' time in waits.  Two rows a wave and eight waves keep the kernel at
// 128 registers (16 waves per CU, two blocks).
// Measured per step of the pair (HIP events; in brackets the two-step interior
// with a one-step shell it replaced):
//   600x400x120, 25 right-hand sides 5.0 ms (11.0), 6.3 ps per cell-update clear
//   of the slabs and 8.9 in them; 430x450x64, 6: 655 us (1390); 320x240x96, 6:
//   391 us (871); 91x103x88, 2: 27 us (142).  kappa loaded in every plane: 5.35
//   ms, 753, 425 and 27 us.
// Other shapes, when these stood at 5.8 ms, 463 and 32 us: 3 rows a wave 5.9 ms,
// 562 and 48 us; 4 rows and 4 waves 6.5 ms, 536 and 35 us; 16 waves of 2 rows
// 6.3 ms, 587 and 48 us.  At 5.8 ms, 423 and 27 us: 16 waves of one row 5.7 ms,
// 529 and 29 us (for the clear tiles alone, or 3 rows there: 1 to 2 % of the
// first); the next plane's operands loaded ahead of this one's stores 447 and 29
// us (spills); streaming loads 6.9 ms, 475 and 35 us; the clear tiles' code for
// the clear tiles of a mixed launch 431 and 27 us.
#include "yo_device.h"

namespace {

// Scalar loads of data no kernel of this launch writes.  `opaque` keeps such
// loads, and uniform tests, where they are used: hoisted out of the march they
// would not fit the scalar registers.
template <class T> using Const = const __attribute__((address_space(4))) T *;
template <class T>
__device__ __forceinline__ Const<T> constant(const T *p)
{
    return (Const<T>)(uintptr_t)p;
}
template <class T> using Global = __attribute__((address_space(1))) T *;
template <class T>
__device__ __forceinline__ T opaque(T v)
{
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ Cpml cpml_uniform(const float4 *prof, int which, int u)
{
    Const<float> p = (Const<float>)(uintptr_t)(prof + 2 * u + which);
    return Cpml{p[0], p[1], p[2]};
}

// tile flags (uniform): rows r owned, in the y-slabs, in the grid
enum { F_OWN = 0, F_YSLAB = 4, F_IN = 8, F_X = 1 << 12, F_SRC = 1 << 13, F_X0 = 1 << 14, F_Y0 = 1 << 15,
       F_BOX = 16, F_MON = 1 << 20 };

// CP: tiles that meet the x- or y-slabs, a source plane or the grid's first
// column or row; else only the z-slabs' code is there.  DFT: E^{n+1} of the
// design box and the port planes is stored for the running DFT.  GEN: 1 planes
// normal to y or z too, 2 and up to 64 x-slab columns in a strip, else 32
// (kernels of their own: the code costs the others registers, the columns LDS).  ONE: S1 and S2 only, stored:
// one step.
template <int TY, int W, bool CP, bool DFT, int GEN, bool ONE>
__device__ __forceinline__ void wave_pair(const Const<YoPlanD> P, const Const<YoRhsD> R, const int step, const int now,
                                          const int4 t, const int w, const int lane, float *lds)
{
    const int ny = P->ny, nz = P->nz;
    const unsigned gs = 1536u * P->ns, pstr = (unsigned)(ny + 1) * gs;   // state of a row, of a plane, bytes
    const unsigned ps = 1024u * P->ns;                                   // CPML memories of a row
    const int nxt = buf_next(P, now, ONE ? 1 : 2);
    const Rsrc FA = rsrc_of(R->F[now], array_bytes(P, 6));   // after step n
    const Rsrc FC = rsrc_of(R->F[nxt], array_bytes(P, 6));   // after step n+2
    const Rsrc KR = rsrc_of(P->kappa, array_bytes(P, 3));
    const Rsrc PS = rsrc_of(R->psi, 4u * P->nbuf * P->psi_slot);   // every slot
    const Const<float> kplane = (Const<float>)(uintptr_t)P->kplane;
    const float sx = P->sx, sy = P->sy, sz = P->sz;
    const int x0 = t.x & 0xffff, xn = t.x >> 16;
    const int J0 = t.y & 0xffff, JN = t.y >> 16;
    const int k0 = t.z & 0xffff, k1 = yo_high(t.z);
    const int jb = J0 - 2 + w * TY;        // this wave's first row
    LaneX L = lane_x(P, x0, xn, lane);
    const int xl = L.xl, xk = L.xk, xp = L.xp;
    const int xs = L.st ? L.xs : kFar, xps = L.st ? L.xps : kFar;   // stores of lanes that store nothing are dropped

    // absorbing layers: x per lane, y per row, z per plane
    const int ylo = P->plo[1], zlo = P->plo[2], zhi = P->phi[2];
    const int yh0 = ny - P->phi[1];                          // first row of the high y-slab
    Cpml cxE = {1.0f, 0.0f, 1.0f}, cxH = cxE;
    int xi = 0;
    if (CP && (t.w & 1)) {
        lane_xslab(P, L, cxE, cxH);
        // the lane's place among the strip's slab columns
        const unsigned long long m = __ballot(L.px >= 0);
        xi = L.px >= 0 ? __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0)) : 0;
    }
    const bool ylow = jb < ylo;
    const int py0 = ylow ? jb : jb - yh0 + ylo;             // slab row of row 0
    int fl0 = 0;
    unsigned rb[TY];
#pragma unroll
    for (int r = 0; r < TY; ++r) {
        const int j = jb + r;
        rb[r] = (unsigned)(clampi(j, -1, ny) + 1) * gs;
        if (j >= J0 && j < J0 + JN) fl0 |= 1 << (F_OWN + r);
        if (j >= 0 && j < ny) fl0 |= 1 << (F_IN + r);
        if (CP && j >= 0 && j < ny && (j < ylo || j >= yh0)) fl0 |= 1 << (F_YSLAB + r);
        if (DFT && j >= J0 && j < J0 + JN && j >= P->box[1] && j < P->box[1] + P->box[4]) fl0 |= 1 << (F_BOX + r);
        if (CP && j == 0) fl0 |= F_Y0;
    }
    if (CP && (t.w & 1)) fl0 |= F_X;
    if (CP && x0 == 0) fl0 |= F_X0;
    if (CP) {
        // the source plane and this wave's rows
        const int sp = R->src.index, lo0 = R->src.lo0, n0 = R->src.n0;
        if (GEN && R->src.axis) {
            const bool y = R->src.axis == 1;
            const int ja = y ? sp : R->src.lo1, jn = y ? 2 : R->src.n1;
            if (R->src_j && lo0 < x0 + xn + 2 && lo0 + n0 > x0 - 2 && jb < ja + jn && jb + TY > ja) fl0 |= F_SRC;
        } else if (R->src_j && sp + (R->src_nc == 5 ? 1 : 0) >= x0 - 2 && sp <= x0 + xn + 1 && jb < lo0 + n0 && jb + TY > lo0)
            fl0 |= F_SRC;
    }
    if constexpr (DFT) {
        const bool xbox = x0 < P->box[0] + P->box[3] && x0 + xn > P->box[0];
        if (!xbox) fl0 &= ~(0xf << F_BOX);
        for (int q = 0; CP && q < P->n_ports; ++q) {
            const int ix = P->ports[q].index, lo0 = P->ports[q].lo0, n0 = P->ports[q].n0;
            if (GEN && P->ports[q].axis) {
                const bool y = P->ports[q].axis == 1;
                const int ja = y ? ix : P->ports[q].lo1, jn = y ? 2 : P->ports[q].n1;
                if (lo0 < x0 + xn && lo0 + n0 > x0 && jb < ja + jn && jb + TY > ja) fl0 |= F_MON;
            } else if (ix + (P->mon_nc == 5) >= x0 && ix < x0 + xn && jb < lo0 + n0 && jb + TY > lo0)
                fl0 |= F_MON;
        }
    }
    const unsigned zb0 = 4u * (P->psi_off[2] + now * P->psi_slot), zb2 = 4u * (P->psi_off[2] + nxt * P->psi_slot);
    const unsigned yb0 = 4u * (P->psi_off[1] + now * P->psi_slot), yb2 = 4u * (P->psi_off[1] + nxt * P->psi_slot);
    const unsigned xb0 = 4u * (P->psi_off[0] + now * P->psi_slot), xb2 = 4u * (P->psi_off[0] + nxt * P->psi_slot);
    const unsigned ypl = (unsigned)(ylo + P->phi[1]) * ps;   // a plane's y-slab rows
    const unsigned xrow = 4u * P->psi_xrow, xw = 4u * P->psi_xw;
    const float4 *profy = P->prof[1], *profz = P->prof[2];

    // LDS: rows for the neighbouring waves (12 slots of W x 64), then the
    // memories of step n+1 that the second step reads one plane later: y-slab
    // rows (block row, value, plane parity), x-slab columns (row, value, parity)
    float *const ex = lds + lane;
    auto slot = [&](int q, int ww) -> float & { return ex[(q * W + ww) * 64]; };
    constexpr int XL = GEN == 2 ? 64 : 32;
    float *const ystash = lds + 12 * W * 64 + w * TY * 4 * 2 * 64 + lane;
    float *const xstash = lds + 12 * W * 64 + W * TY * 4 * 2 * 64 + w * TY * 4 * 2 * XL + xi;
    auto yst = [&](int r, int v, int par) -> float & { return ystash[((r * 4 + v) * 2 + par) * 64]; };
    auto xst = [&](int r, int v, int par) -> float & { return xstash[((r * 4 + v) * 2 + par) * XL]; };

    // by plane parity: E^n, Ht^{n+1/2}, E^{n+1}, kappa, Ht^{n+3/2} and the z
    // memories of step n+1 (the second of a plane's two is the plane before)
    float E0[2][3][TY], H[2][3][TY], E1_[2][3][TY], K[2][3][TY], H2_[2][3][TY];
    float zH_[2][2][TY], zE_[2][2][TY];
    const int kb = k0 == 0 ? 0 : k0 - (ONE ? 1 : 2);
#pragma unroll
    for (int r = 0; r < TY; ++r) {
        const unsigned o = (unsigned)kb * pstr + rb[r];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            E0[0][c][r] = bload(FA, xl + 256 * c, o);
            H[1][c][r] = E1_[1][c][r] = K[1][c][r] = 0.0f;
        }
        H2_[1][0][r] = H2_[1][1][r] = 0.0f;
    }
    slot(2 * (kb & 1), w) = E0[0][0][0];
    slot(2 * (kb & 1) + 1, w) = E0[0][2][0];
    slot(4 + 2 * ((kb - 1) & 1), w) = 0.0f;
    slot(4 + 2 * ((kb - 1) & 1) + 1, w) = 0.0f;
    block_sync_lds();

    fl0 = __builtin_amdgcn_readfirstlane(fl0);
    const int wu = w + 1 < W ? w + 1 : w, wd = w > 0 ? w - 1 : 0;
    int k = kb;
    // one plane; the arrays are those of plane k and of plane k-1, which the
    // next call swaps (so nothing is copied from plane to plane)
    auto plane = [&](float (&Ec)[3][TY], float (&En)[3][TY], float (&Hc)[3][TY], float (&Hp)[3][TY],
                     float (&E1)[3][TY], float (&E1p)[3][TY], float (&Kc)[3][TY], float (&Kp)[3][TY],
                     float (&H2)[3][TY], float (&H2p)[3][TY], float (&zH)[2][TY], float (&zHp)[2][TY],
                     float (&zE)[2][TY], float (&zEp)[2][TY]) {
        const int fl = opaque(fl0);
        const int par = k & 1;
        const int km = k - 1;
        const int pz = slab_index(k, nz, zlo, zhi), pzm = slab_index(km, nz, zlo, zhi);
        const bool kin = k < nz, kmin = km >= 0;   // k >= 0 always, km < nz
        const bool kuni = kin && kplane[4 * min(k, nz - 1) + 3] != 0.0f;
        const bool ownk = km >= k0 && km < k1;
        auto own1 = [&](int r) { return k >= k0 && (fl >> (F_OWN + r) & 1); };   // a step alone: k < k1
        {
            // planes past the grid read zero (past the buffer), and so does kappa
            // where the plane has one value per component
            const unsigned oh = (unsigned)min(k, nz - 1) * pstr, oe = (unsigned)min(k + 1, nz - 1) * pstr;
            const int ve = k + 1 < nz ? xl : kFar, vh = kin ? xl + 768 : kFar, vk = kin && !kuni ? xk : kFar;
#pragma unroll
            for (int r = 0; r < TY; ++r) {
                const unsigned e = oe + rb[r], h = oh + rb[r], q = h >> 1;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    En[c][r] = bload(FA, ve + 256 * c, e);
                    Hc[c][r] = bload(FA, vh + 256 * c, h);
                    Kc[c][r] = bload(KR, vk + 256 * c, q);
                }
            }
        }
        // old memories, loaded with the plane's fields so that one wait covers
        // all: z; x and y (E, E, Ht, Ht)
        if (pz >= 0) {
#pragma unroll
            for (int r = 0; r < TY; ++r) {
                const unsigned o = zb0 + (unsigned)(pz * ny + clampi(jb + r, 0, ny - 1)) * ps;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    zE[c][r] = bload(PS, xp + 256 * c, o);
                    zH[c][r] = bload(PS, xp + 512 + 256 * c, o);
                }
            }
        }
        float qx[CP ? 4 : 1][TY], qy[CP ? 4 : 1][TY];
        if constexpr (CP) {
            if ((fl & F_X) && kin) {
                const int pv = L.px >= 0 ? L.px : kFar;
#pragma unroll
                for (int r = 0; r < TY; ++r) {
                    const unsigned o = xb0 + (unsigned)(k * ny + clampi(jb + r, 0, ny - 1)) * xrow;
#pragma unroll
                    for (int v = 0; v < 4; ++v) qx[v][r] = bload(PS, pv, o + v * xw);
                }
            }
#pragma unroll
            for (int r = 0; r < TY; ++r)
                if ((fl >> (F_YSLAB + r) & 1) && kin) {
                    const unsigned o = yb0 + (unsigned)k * ypl + (unsigned)(py0 + r) * ps;
#pragma unroll
                    for (int v = 0; v < 4; ++v) qy[v][r] = bload(PS, xp + 256 * v, o);
                }
        }
        slot(2 * (par ^ 1), w) = En[0][0];
        slot(2 * (par ^ 1) + 1, w) = En[2][0];

        // ---- S1 ----
        Cpml cz;
        if (pz >= 0) cz = cpml_uniform(profz, 1, k);
        const float exu = slot(2 * par, wu), ezu = slot(2 * par + 1, wu);
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const float eu0 = r + 1 < TY ? Ec[0][r + 1 < TY ? r + 1 : r] : exu;
            const float eu2 = r + 1 < TY ? Ec[2][r + 1 < TY ? r + 1 : r] : ezu;
            float dyEz = eu2 - Ec[2][r];
            float dzEy = En[1][r] - Ec[1][r];
            float dzEx = En[0][r] - Ec[0][r];
            float dxEz = shfl_next(Ec[2][r]) - Ec[2][r];
            float dxEy = shfl_next(Ec[1][r]) - Ec[1][r];
            float dyEx = eu0 - Ec[0][r];
            if constexpr (CP) {
                if ((fl & F_X) && kin && (fl >> (F_IN + r) & 1)) {
                    if (L.px >= 0) {
                        float n0, n1;
                        dxEz = pml_diff(dxEz, cxH, qx[2][r], n0);
                        dxEy = pml_diff(dxEy, cxH, qx[3][r], n1);
                        if constexpr (ONE) {
                            if (own1(r) && L.own) {
                                const unsigned o = xb2 + (unsigned)(k * ny + jb + r) * xrow;
                                bstore(n0, PS, L.px, o + 2 * xw);
                                bstore(n1, PS, L.px, o + 3 * xw);
                            }
                        } else {
                            xst(r, 0, par) = n0;
                            xst(r, 1, par) = n1;
                        }
                    }
                }
                if ((fl >> (F_YSLAB + r) & 1) && kin) {
                    const Cpml cy = cpml_uniform(profy, 1, jb + r);
                    float n0, n1;
                    dyEz = pml_diff(dyEz, cy, qy[2][r], n0);
                    dyEx = pml_diff(dyEx, cy, qy[3][r], n1);
                    if constexpr (ONE) {
                        if (own1(r)) {
                            const unsigned o = yb2 + (unsigned)k * ypl + (unsigned)(py0 + r) * ps;
                            bstore(n0, PS, xps + 512, o);
                            bstore(n1, PS, xps + 768, o);
                        }
                    } else {
                        yst(r, 0, par) = n0;
                        yst(r, 1, par) = n1;
                    }
                }
            }
            if (pz >= 0 && (fl >> (F_IN + r) & 1)) {
                dzEy = pml_diff(dzEy, cz, zH[0][r], zH[0][r]);
                dzEx = pml_diff(dzEx, cz, zH[1][r], zH[1][r]);
                if (ONE && own1(r)) {
                    const unsigned o = zb2 + (unsigned)(pz * ny + jb + r) * ps;
                    bstore(zH[0][r], PS, xps + 512, o);
                    bstore(zH[1][r], PS, xps + 768, o);
                }
            }
            Hc[0][r] = Hc[0][r] - fmaf(sy, dyEz, -(sz * dzEy));
            Hc[1][r] = Hc[1][r] - fmaf(sz, dzEx, -(sx * dxEz));
            Hc[2][r] = Hc[2][r] - fmaf(sx, dxEy, -(sy * dyEx));
        }
        // (a step alone has no second barrier: slots by parity)
        const int s8 = ONE ? 8 + 2 * par : 8;
        slot(s8, w) = Hc[0][TY - 1];
        slot(s8 + 1, w) = Hc[2][TY - 1];
        block_sync_lds();

        // ---- S2 ----
        if (kuni) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const unsigned v = __float_as_uint(kplane[4 * k + c]), kl = xk != kFar ? v : 0u;
#pragma unroll
                for (int r = 0; r < TY; ++r)
                    Kc[c][r] = __uint_as_float(__float_as_uint(Kc[c][r]) | ((fl >> (F_IN + r) & 1) ? kl : 0u));
            }
        }
        if (pz >= 0) cz = cpml_uniform(profz, 0, k);
        const float hxd = slot(s8, wd), hzd = slot(s8 + 1, wd);
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const float hd0 = r > 0 ? Hc[0][r > 0 ? r - 1 : 0] : hxd;
            const float hd2 = r > 0 ? Hc[2][r > 0 ? r - 1 : 0] : hzd;
            float dyHz = Hc[2][r] - hd2;
            float dzHy = Hc[1][r] - Hp[1][r];
            float dzHx = Hc[0][r] - Hp[0][r];
            float dxHz = Hc[2][r] - shfl_prev(Hc[2][r]);
            float dxHy = Hc[1][r] - shfl_prev(Hc[1][r]);
            float dyHx = Hc[0][r] - hd0;
            if constexpr (CP) {
                if ((fl & F_X) && kin && (fl >> (F_IN + r) & 1)) {
                    if (L.px >= 0) {
                        float n0, n1;
                        dxHz = pml_diff(dxHz, cxE, qx[0][r], n0);
                        dxHy = pml_diff(dxHy, cxE, qx[1][r], n1);
                        if constexpr (ONE) {
                            if (own1(r) && L.own) {
                                const unsigned o = xb2 + (unsigned)(k * ny + jb + r) * xrow;
                                bstore(n0, PS, L.px, o);
                                bstore(n1, PS, L.px, o + xw);
                            }
                        } else {
                            xst(r, 2, par) = n0;
                            xst(r, 3, par) = n1;
                        }
                    }
                }
                if ((fl >> (F_YSLAB + r) & 1) && kin) {
                    const Cpml cy = cpml_uniform(profy, 0, jb + r);
                    float n0, n1;
                    dyHz = pml_diff(dyHz, cy, qy[0][r], n0);
                    dyHx = pml_diff(dyHx, cy, qy[1][r], n1);
                    if constexpr (ONE) {
                        if (own1(r)) {
                            const unsigned o = yb2 + (unsigned)k * ypl + (unsigned)(py0 + r) * ps;
                            bstore(n0, PS, xps, o);
                            bstore(n1, PS, xps + 256, o);
                        }
                    } else {
                        yst(r, 2, par) = n0;
                        yst(r, 3, par) = n1;
                    }
                }
            }
            if (pz >= 0 && (fl >> (F_IN + r) & 1)) {
                dzHy = pml_diff(dzHy, cz, zE[0][r], zE[0][r]);
                dzHx = pml_diff(dzHx, cz, zE[1][r], zE[1][r]);
                if (ONE && own1(r)) {
                    const unsigned o = zb2 + (unsigned)(pz * ny + jb + r) * ps;
                    bstore(zE[0][r], PS, xps, o);
                    bstore(zE[1][r], PS, xps + 256, o);
                }
            }
            E1[0][r] = fmaf(Kc[0][r], fmaf(sy, dyHz, -(sz * dzHy)), Ec[0][r]);
            E1[1][r] = fmaf(Kc[1][r], fmaf(sz, dzHx, -(sx * dxHz)), Ec[1][r]);
            E1[2][r] = fmaf(Kc[2][r], fmaf(sx, dxHy, -(sy * dyHx)), Ec[2][r]);
        }
        // perfect conductor: tangential E on the planes x = 0, y = 0, z = 0
        auto conductor = [&](int kk, float (&e)[3][TY]) {
            if (kk == 0) {
#pragma unroll
                for (int r = 0; r < TY; ++r) e[0][r] = e[1][r] = 0.0f;
            }
            if constexpr (CP) {
                if (fl & F_X0) {
#pragma unroll
                    for (int r = 0; r < TY; ++r) {
                        e[1][r] = L.x == 0 ? 0.0f : e[1][r];
                        e[2][r] = L.x == 0 ? 0.0f : e[2][r];
                    }
                }
                if (fl & F_Y0) {
#pragma unroll
                    for (int r = 0; r < TY; ++r)
                        if (jb + r == 0) e[0][r] = e[2][r] = 0.0f;
                }
            }
        };
        // the soft current source of one step on E after it
        auto source = [&](int kk, int n, float (&e)[3][TY], const float (&kv)[3][TY]) {
            if (!CP || !(fl & F_SRC)) return;
            Const<YoRhsD> Rc = opaque(R);
            const int lo1 = Rc->src.lo1, n1 = Rc->src.n1;
            if (!(GEN && Rc->src.axis) && (kk < lo1 || kk >= lo1 + n1)) return;
            const int lo0 = Rc->src.lo0, n0 = Rc->src.n0, snc = Rc->src_nc;
            Const<float> st = (Const<float>)(uintptr_t)(Rc->steptab + n);
            const float stx = st[0], sty = st[1];
            const int pl = n0 * n1, d = L.x - Rc->src.index;
            if constexpr (GEN > 0) {
                // any normal: the place across the plane and in it, and the
                // plane's component that goes to each of E's (-1: none)
                const Global<const float2> sj = (Global<const float2>)(uintptr_t)Rc->src_j;
                const int ax = Rc->src.axis, ix = Rc->src.index;
#pragma unroll
                for (int r = 0; r < TY; ++r) {
                    const int j = jb + r;
                    const int dn = (ax == 0 ? L.x : ax == 1 ? j : kk) - ix;
                    const int a = (ax == 0 ? j : L.x) - lo0, b = (ax == 2 ? j : kk) - lo1;
                    if (!(dn == 0 || (snc == 5 && dn == 1)) || a < 0 || a >= n0 || b < 0 || b >= n1) continue;
                    const Global<const float2> q = sj + b * n0 + a;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const int m = (c - ax + 3) % 3;
                        const int t = m == 0 ? (snc == 5 && dn == 0 ? 2 : -1) : m - 1 + (dn ? 3 : 0);
                        if (t >= 0)
                            e[c][r] = fmaf(-kv[c][r], fmaf(q[t * pl].x, stx, q[t * pl].y * sty), e[c][r]);
                    }
                }
                return;
            }
            if (!(d == 0 || (snc == 5 && d == 1))) return;
            const Global<const float2> sj = (Global<const float2>)(uintptr_t)Rc->src_j;
#pragma unroll
            for (int r = 0; r < TY; ++r) {
                const int a = jb + r - lo0;
                if (a < 0 || a >= n0) continue;
                const Global<const float2> q = sj + (kk - lo1) * n0 + a;
                const Global<const float2> qy = q + (d ? 3 : 0) * pl, qz = q + (d ? 4 : 1) * pl;
                e[1][r] = fmaf(-kv[1][r], fmaf(qy->x, stx, qy->y * sty), e[1][r]);
                e[2][r] = fmaf(-kv[2][r], fmaf(qz->x, stx, qz->y * sty), e[2][r]);
                if (snc == 5 && d == 0) {
                    const Global<const float2> qx_ = q + 2 * pl;
                    e[0][r] = fmaf(-kv[0][r], fmaf(qx_->x, stx, qx_->y * sty), e[0][r]);
                }
            }
        };
        conductor(k, E1);
        source(k, step, E1, Kc);
        if constexpr (ONE) {
            if (k < k0) return;
            const unsigned o = (unsigned)k * pstr;
#pragma unroll
            for (int r = 0; r < TY; ++r) {
                if (!(fl >> (F_OWN + r) & 1)) continue;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    bstore_nt(E1[c][r], FC, xs + 256 * c, o + rb[r]);
                    bstore_nt(Hc[c][r], FC, xs + 768 + 256 * c, o + rb[r]);
                }
            }
            return;
        }
        if constexpr (DFT) {
            // E^{n+1} on this tile's cells of the design box and the port planes,
            // for the running DFT (k_dft, which adds both steps after this launch)
            if (k >= k0 && k < k1 && (fl & (0xf << F_BOX | F_MON))) {
                Const<YoPlanD> Pc = opaque(P);
                const Global<float> mid = (Global<float>)(uintptr_t)opaque(R)->dft_mid;
                const int bx = Pc->box[3], by = Pc->box[4], bz = Pc->box[5], bk = k - Pc->box[2];
                const int bi = L.x - Pc->box[0];
                if (bk >= 0 && bk < bz && (fl & 0xf << F_BOX) && L.own && bi >= 0 && bi < bx) {
#pragma unroll
                    for (int r = 0; r < TY; ++r) {
                        if (!(fl >> (F_BOX + r) & 1)) continue;
                        const int o = (bk * by + jb + r - Pc->box[1]) * bx + bi;
#pragma unroll
                        for (int c = 0; c < 3; ++c) mid[c * bz * by * bx + o] = E1[c][r];
                    }
                }
                if (CP && (fl & F_MON)) {
                    const Global<float> mon = mid + 3 * bz * by * bx;
                    const int np = Pc->n_ports, nc = Pc->mon_nc;
                    for (int q = 0; q < np; ++q) {
                        const int lo0 = Pc->ports[q].lo0, n0 = Pc->ports[q].n0, n1 = Pc->ports[q].n1;
                        const int bk1 = k - Pc->ports[q].lo1, d = L.x - Pc->ports[q].index;
                        if constexpr (GEN > 0) {
                            const int ax = Pc->ports[q].axis, ix = Pc->ports[q].index, pl = n0 * n1;
#pragma unroll
                            for (int r = 0; r < TY; ++r) {
                                const int j = jb + r;
                                const int dn = (ax == 0 ? L.x : ax == 1 ? j : k) - ix;
                                const int a = (ax == 0 ? j : L.x) - lo0, b = (ax == 2 ? j : k) - Pc->ports[q].lo1;
                                if (!L.own || !(fl >> (F_OWN + r) & 1) || !(dn == 0 || (nc == 5 && dn == 1)) || a < 0 ||
                                    a >= n0 || b < 0 || b >= n1)
                                    continue;
                                const int o = Pc->mon_off[q] + b * n0 + a;
#pragma unroll
                                for (int c = 0; c < 3; ++c) {
                                    const int m = (c - ax + 3) % 3;
                                    const int t = m == 0 ? (nc == 5 && dn == 0 ? 2 : -1) : m - 1 + (dn ? 3 : 0);
                                    if (t >= 0) mon[o + t * pl] = E1[c][r];
                                }
                            }
                            continue;
                        }
                        if (bk1 < 0 || bk1 >= n1 || !L.own || !(d == 0 || (nc == 5 && d == 1))) continue;
                        const int pl = n0 * n1, o = Pc->mon_off[q] + bk1 * n0;
#pragma unroll
                        for (int r = 0; r < TY; ++r) {
                            const int a = jb + r - lo0;
                            if (!(fl >> (F_OWN + r) & 1) || a < 0 || a >= n0) continue;
                            mon[o + (d ? 3 : 0) * pl + a] = E1[1][r];
                            mon[o + (d ? 4 : 1) * pl + a] = E1[2][r];
                            if (nc == 5 && d == 0) mon[o + 2 * pl + a] = E1[0][r];
                        }
                    }
                }
            }
        }
        slot(4 + 2 * par, w) = E1[0][0];
        slot(4 + 2 * par + 1, w) = E1[2][0];

        // ---- S3 at plane k-1 ----
        if (pzm >= 0) cz = cpml_uniform(profz, 1, km);
        const float fxu = slot(4 + 2 * (par ^ 1), wu), fzu = slot(4 + 2 * (par ^ 1) + 1, wu);
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const float eu0 = r + 1 < TY ? E1p[0][r + 1 < TY ? r + 1 : r] : fxu;
            const float eu2 = r + 1 < TY ? E1p[2][r + 1 < TY ? r + 1 : r] : fzu;
            float dyEz = eu2 - E1p[2][r];
            float dzEy = E1[1][r] - E1p[1][r];
            float dzEx = E1[0][r] - E1p[0][r];
            float dxEz = shfl_next(E1p[2][r]) - E1p[2][r];
            float dxEy = shfl_next(E1p[1][r]) - E1p[1][r];
            float dyEx = eu0 - E1p[0][r];
            const bool own = ownk && (fl >> (F_OWN + r) & 1);
            if constexpr (CP) {
                if ((fl & F_X) && kmin && (fl >> (F_IN + r) & 1)) {
                    if (L.px >= 0) {
                        float n0, n1;
                        dxEz = pml_diff(dxEz, cxH, xst(r, 0, par ^ 1), n0);
                        dxEy = pml_diff(dxEy, cxH, xst(r, 1, par ^ 1), n1);
                        if (own && L.own) {
                            const unsigned o = xb2 + (unsigned)(km * ny + jb + r) * xrow;
                            bstore(n0, PS, L.px, o + 2 * xw);
                            bstore(n1, PS, L.px, o + 3 * xw);
                        }
                    }
                }
                if ((fl >> (F_YSLAB + r) & 1) && kmin) {
                    const Cpml cy = cpml_uniform(profy, 1, jb + r);
                    float n0, n1;
                    dyEz = pml_diff(dyEz, cy, yst(r, 0, par ^ 1), n0);
                    dyEx = pml_diff(dyEx, cy, yst(r, 1, par ^ 1), n1);
                    if (own) {
                        const unsigned o = yb2 + (unsigned)km * ypl + (unsigned)(py0 + r) * ps;
                        bstore(n0, PS, xps + 512, o);
                        bstore(n1, PS, xps + 768, o);
                    }
                }
            }
            if (pzm >= 0 && (fl >> (F_IN + r) & 1)) {
                float n0, n1;
                dzEy = pml_diff(dzEy, cz, zHp[0][r], n0);
                dzEx = pml_diff(dzEx, cz, zHp[1][r], n1);
                if (own) {
                    const unsigned o = zb2 + (unsigned)(pzm * ny + jb + r) * ps;
                    bstore(n0, PS, xps + 512, o);
                    bstore(n1, PS, xps + 768, o);
                }
            }
            H2[0][r] = Hp[0][r] - fmaf(sy, dyEz, -(sz * dzEy));
            H2[1][r] = Hp[1][r] - fmaf(sz, dzEx, -(sx * dxEz));
            H2[2][r] = Hp[2][r] - fmaf(sx, dxEy, -(sy * dyEx));
        }
        slot(10, w) = H2[0][TY - 1];
        slot(11, w) = H2[2][TY - 1];
        block_sync_lds();

        // ---- S4 at plane k-1 ----
        if (!ownk || !(fl & ((1 << TY) - 1))) return;
        if (pzm >= 0) cz = cpml_uniform(profz, 0, km);
        const float gxd = slot(10, wd), gzd = slot(11, wd);
        float E2[3][TY];
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const float hd0 = r > 0 ? H2[0][r > 0 ? r - 1 : 0] : gxd;
            const float hd2 = r > 0 ? H2[2][r > 0 ? r - 1 : 0] : gzd;
            float dyHz = H2[2][r] - hd2;
            float dzHy = H2[1][r] - H2p[1][r];
            float dzHx = H2[0][r] - H2p[0][r];
            float dxHz = H2[2][r] - shfl_prev(H2[2][r]);
            float dxHy = H2[1][r] - shfl_prev(H2[1][r]);
            float dyHx = H2[0][r] - hd0;
            const bool own = fl >> (F_OWN + r) & 1;
            if constexpr (CP) {
                if ((fl & F_X) && own) {
                    if (L.px >= 0) {
                        float n0, n1;
                        dxHz = pml_diff(dxHz, cxE, xst(r, 2, par ^ 1), n0);
                        dxHy = pml_diff(dxHy, cxE, xst(r, 3, par ^ 1), n1);
                        if (L.own) {
                            const unsigned o = xb2 + (unsigned)(km * ny + jb + r) * xrow;
                            bstore(n0, PS, L.px, o);
                            bstore(n1, PS, L.px, o + xw);
                        }
                    }
                }
                if ((fl >> (F_YSLAB + r) & 1) && own) {
                    const Cpml cy = cpml_uniform(profy, 0, jb + r);
                    float n0, n1;
                    dyHz = pml_diff(dyHz, cy, yst(r, 2, par ^ 1), n0);
                    dyHx = pml_diff(dyHx, cy, yst(r, 3, par ^ 1), n1);
                    const unsigned o = yb2 + (unsigned)km * ypl + (unsigned)(py0 + r) * ps;
                    bstore(n0, PS, xps, o);
                    bstore(n1, PS, xps + 256, o);
                }
            }
            if (pzm >= 0 && own) {
                float n0, n1;
                dzHy = pml_diff(dzHy, cz, zEp[0][r], n0);
                dzHx = pml_diff(dzHx, cz, zEp[1][r], n1);
                const unsigned o = zb2 + (unsigned)(pzm * ny + jb + r) * ps;
                bstore(n0, PS, xps, o);
                bstore(n1, PS, xps + 256, o);
            }
            E2[0][r] = fmaf(Kp[0][r], fmaf(sy, dyHz, -(sz * dzHy)), E1p[0][r]);
            E2[1][r] = fmaf(Kp[1][r], fmaf(sz, dzHx, -(sx * dxHz)), E1p[1][r]);
            E2[2][r] = fmaf(Kp[2][r], fmaf(sx, dxHy, -(sy * dyHx)), E1p[2][r]);
        }
        conductor(km, E2);
        source(km, step + 1, E2, Kp);
        const unsigned om = (unsigned)km * pstr;
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            if (!(fl >> (F_OWN + r) & 1)) continue;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                bstore_nt(E2[c][r], FC, xs + 256 * c, om + rb[r]);
                bstore_nt(H2[c][r], FC, xs + 768 + 256 * c, om + rb[r]);
            }
        }
    };
    for (;;) {
        plane(E0[0], E0[1], H[0], H[1], E1_[0], E1_[1], K[0], K[1], H2_[0], H2_[1], zH_[0], zH_[1], zE_[0], zE_[1]);
        if (++k > k1 - ONE) break;
        plane(E0[1], E0[0], H[1], H[0], E1_[1], E1_[0], K[1], K[0], H2_[1], H2_[0], zH_[1], zH_[0], zE_[1], zE_[0]);
        if (++k > k1 - ONE) break;
    }
}

template <int TY, int W, bool CP, bool DFT, int GEN, bool ONE>
__global__ __launch_bounds__(64 * W, 4) void k_yee_pair(const YoStepArgs a)
{
    const int nb = gridDim.x, b = blockIdx.x;
    const int q = nb >> 3, rem = nb & 7, xcd = b & 7, pos = b >> 3;
    const int lb = (xcd < rem) ? xcd * (q + 1) + pos : rem * (q + 1) + (xcd - rem) * q + pos;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    // every early exit is uniform over the block, as the barriers require
    const int wave0 = lb * W;
    if (wave0 >= a.total_waves) return;
    int s = 0;
    while (s + 1 < a.n_slots && wave0 >= a.prefix[s + 1]) ++s;
    const YoSlot sl = a.slot[s];
    const Const<YoPlanD> P = constant(sl.plan);
    const int step = *constant(P->step_ctr) + a.k_offset;
    // the host schedules a pair only where both steps remain
    if (step + (ONE ? 0 : 1) >= P->n_steps) return;
    const int now = P->nbuf == 3 ? step % 3 : (constant(P->step_ctr)[1] + a.b_offset) & 1;
    const int blk = (wave0 - a.prefix[s]) / W;
    // consecutive blocks take neighbouring strips of the same rows (whose row
    // segments are neighbours in memory) of one right-hand side, then the same
    // tiles of the next one, which share kappa
    // (order alone, 600x400x120 with 25 right-hand sides: 6.4 to 7.3 ms per step
    // with one tile after another over the right-hand sides, 5.8 in groups)
    const int G = YO_PAIR_GROUP;
    const int g = blk / (G * sl.nrhs), in_g = blk - g * (G * sl.nrhs);
    const int gsz = min(G, sl.ntile * sl.nzc - g * G);
    if (gsz <= 0) return;
    const int r = sl.rhs0 + in_g / gsz;
    // the tile's chunk of planes, chunks outermost
    const int ti = g * G + in_g % gsz, zc = ti / sl.ntile;
    const int kq = P->nz / sl.nzc, kr = P->nz % sl.nzc;
    const int k0 = zc * kq + min(zc, kr), k1 = k0 + kq + (zc < kr);
    extern __shared__ float lds[];
    const Const<int> tp = (Const<int>)(uintptr_t)(sl.tiles + ti - zc * sl.ntile);
    wave_pair<TY, W, CP, DFT, GEN, ONE>(P, constant(P->rhs + r), step, now, int4{tp[0], tp[1], k0 | k1 << 16, tp[3]}, w, lane, lds);
}

}  // namespace

hipError_t yo_launch_pair(bool shell, bool dft, int gen, const YoStepArgs &args, int blocks, hipStream_t s)
{
    if (blocks <= 0) return hipSuccess;
    if (args.wpb != YO_PAIR_W) return hipErrorInvalidValue;
    constexpr int T = YO_PAIR_TY, W = YO_PAIR_W;
    const size_t lds = sizeof(float) * 12 * W * 64;
    // (two blocks per CU with 32 x-slab columns a strip, one with 64)
    const size_t lds_shell = lds + sizeof(float) * W * T * 4 * 2 * (64 + (gen == 2 ? 64 : 32));
    auto go = [&](auto kernel, size_t bytes) {
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * W), bytes, s, args);
        return hipGetLastError();
    };
    if (!shell) return dft ? go(k_yee_pair<T, W, false, true, 0, false>, lds) : go(k_yee_pair<T, W, false, false, 0, false>, lds);
    if (gen == 2)
        return dft ? go(k_yee_pair<T, W, true, true, 2, false>, lds_shell) : go(k_yee_pair<T, W, true, false, 2, false>, lds_shell);
    if (gen == 1)
        return dft ? go(k_yee_pair<T, W, true, true, 1, false>, lds_shell) : go(k_yee_pair<T, W, true, false, 1, false>, lds_shell);
    return dft ? go(k_yee_pair<T, W, true, true, 0, false>, lds_shell) : go(k_yee_pair<T, W, true, false, 0, false>, lds_shell);
}

hipError_t yo_launch_one(const YoStepArgs &args, int blocks, hipStream_t s)
{
    if (blocks <= 0) return hipSuccess;
    if (args.wpb != YO_PAIR_W) return hipErrorInvalidValue;
    constexpr int T = YO_PAIR_TY, W = YO_PAIR_W;
    hipLaunchKernelGGL((k_yee_pair<T, W, true, false, 1, true>), dim3(blocks), dim3(64 * W),
                       sizeof(float) * 12 * W * 64, s, args);
    return hipGetLastError();
}
