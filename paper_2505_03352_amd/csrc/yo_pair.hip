// Two Yee steps per launch over the whole grid (temporal blocking with the
// absorbing layers and the sources inside).  Update, layout and expressions
// as in yo_step.hip, whose single steps these two equal bitwise.
//
// A block of W waves marches up z over one strip of columns (yo_col) and a
// stack of W TY rows, TY a wave; per plane k it takes, from the state after
// step n,
//   S1  Ht^{n+1/2} at plane k      (E^n at k and k+1, Ht^{n-1/2} at k)
//   S2  E^{n+1}    at plane k      (kappa, Ht^{n+1/2} at k and k-1)
//   S3  Ht^{n+3/2} at plane k-1    (E^{n+1} at k-1 and k)
//   S4  E^{n+2}    at plane k-1    (kappa, Ht^{n+3/2} at k-1 and k-2)
// and stores S3 and S4, so a plane's state is read once and written once for
// two steps.  Each row is worked on by one wave; the one row a stage needs of
// the neighbouring wave (above for Ht, below for E) comes through LDS, with
// two barriers per plane.  The rows at the block's ends (two below, two
// above) and the lanes at the strip's (two on either side) are recomputed
// from their own loads and not stored, as are the two planes below and one
// above a z-chunk.
//
// What bounds it: memory traffic (per cell and pair of steps 24 bytes in and
// 24 out, times 16/12 rows and 64/60 columns on the way in) and, below about
// a chip full of blocks, the latency of one plane.  Two rows a wave and eight
// waves keep the kernel at 128 registers (16 waves per CU, two blocks).
// Measured per step of the pair (HIP events):
//   600x400x120, 25 right-hand sides 5.8 ms (two-step interior and one-step
//   shell at the start of this work: 11.0), 7.4 ps per cell-update clear of
//   the slabs, 10 in them; 320x240x96, 6: 463 us (871); 91x103x88, 2: 32 us
//   (142).  3 rows a wave: 5.9 ms, 562 us, 48 us; 4 rows and 4 waves: 6.5 ms,
//   536 us, 35 us; 16 waves of 2 rows: 6.3 ms, 587 us, 48 us; loading the next
//   plane's operands during S4: no faster (8.3 against 8.4 ps).
#include "yo_device.h"

namespace {

// scalar loads of data no kernel of this launch writes
typedef const __attribute__((address_space(4))) float *ConstF;
__device__ __forceinline__ Cpml cpml_uniform(const float *prof, int n, int which, int u)
{
    ConstF p = (ConstF)(uintptr_t)prof;
    Cpml c;
    c.b = p[(which + 0) * n + u];
    c.c = p[(which + 1) * n + u];
    c.ki = p[(which + 2) * n + u];
    return c;
}

// CP: tiles that meet the x- or y-slabs, or a source plane; else only the
// z-slabs' code is there
template <int TY, int W, bool CP>
__device__ __forceinline__ void wave_pair(const YoPlanD &P, const YoRhsD &R, const int step, const int4 t,
                                          const int w, const int lane, float *lds)
{
    const int nx = P.nx, ny = P.ny, nz = P.nz, nxp = P.nxp;
    const int rows = ny + 2;
    const size_t groups = (size_t)(nz + 2) * rows;
    const int rowb = nxp * (int)sizeof(float);
    const int s0 = step % 3, s2 = (step + 2) % 3;         // buffers and CPML memory slots
    const Rsrc FA = rsrc_of(R.F[s0], 6 * groups * nxp);   // after step n
    const Rsrc FC = rsrc_of(R.F[s2], 6 * groups * nxp);   // after step n+2
    const Rsrc KR = rsrc_of(P.kappa, 3 * groups * nxp);
    const Rsrc PS = rsrc_of(R.psi, (size_t)P.psi_total);
    const float sx = P.sx, sy = P.sy, sz = P.sz;
    const int x0 = t.x & 0xffff, xn = t.x >> 16;
    const int J0 = t.y & 0xffff, JN = t.y >> 16;
    const int k0 = t.z & 0xffff, k1 = t.z >> 16;
    const int jb = J0 - 2 + w * TY;        // this wave's first row
    LaneX L = lane_x(P, x0, xn, lane, 2);
    const int x = x0 - 2 + lane;
    const bool xin = x >= 0 && x < nx && x <= x0 + xn + 1;
    const int xl = xin ? yo_col(x, P.sw, P.slead) * (int)sizeof(float) : kFar;
    const int xst = L.st ? L.xs : kFar;    // stores of lanes that store nothing are dropped
    const bool x_first = x == 0;

    // absorbing layers: x per lane (the tile's flag uniform), y per row, z per plane
    const bool xc = CP && (t.w & 1), yc = CP && (t.w & 2);
    int px = -1, xi = 0;
    Cpml cxE = {1.0f, 0.0f, 1.0f}, cxH = cxE;
    if (xc) {
        const int u = xin ? slab_index(x, nx, P.plo[0], P.phi[0]) : -1;
        if (u >= 0) {
            px = (x < P.plo[0] ? x : P.psi_xside + x - (nx - P.phi[0])) * (int)sizeof(float);
            xi = u;
            cxE = cpml_at(P.prof[0], nx, 0, x);
            cxH = cpml_at(P.prof[0], nx, 3, x);
        }
    }
    const float *profy = P.prof[1], *profz = P.prof[2];
    const int ylo = P.plo[1], yhi = P.phi[1], zlo = P.plo[2], zhi = P.phi[2];
    const int Wy = ylo + yhi, xrp = P.psi_xrp;
    const int ox = P.psi_off[0], oy = P.psi_off[1], oz = P.psi_off[2];
    const int nx1 = P.psi_n[0], ny1 = P.psi_n[1], nz1 = P.psi_n[2];
    auto ax = [&](int q, int k, int j) { return (ox + q * nx1 + (k * ny + j) * xrp) * (int)sizeof(float); };
    auto ay = [&](int q, int k, int py) { return (oy + q * ny1 + (k * Wy + py) * nxp) * (int)sizeof(float); };
    auto az = [&](int q, int pz, int j) { return (oz + q * nz1 + (pz * ny + j) * nxp) * (int)sizeof(float); };

    // the source plane (normal to x) and this tile
    const YoPlaneD sp = R.src;
    const bool src_on = CP && R.src_j != nullptr && sp.index + (R.src_nc == 5 ? 1 : 0) >= x0 - 2 &&
                        sp.index <= x0 + xn + 1 && jb < sp.lo0 + sp.n0 && jb + TY > sp.lo0;
    const float2 *sj = R.src_j;
    const int snc = R.src_nc;
    float4 st0 = {0, 0, 0, 0}, st1 = st0;
    if (src_on) {
        st0 = R.steptab[step];
        st1 = R.steptab[step + 1];
    }

    // LDS: rows for the neighbouring waves (12 slots of W x 64), then the
    // memories of step n+1 that the second step reads one plane later: y-slab
    // rows (slab row, value, plane parity), x-slab columns (row, value, parity)
    float *const xs = lds + lane;
    auto slot = [&](int q, int ww) -> float & { return xs[(q * W + ww) * 64]; };
    float *const ystash = lds + 12 * W * 64 + lane;
    float *const xstash = lds + 12 * W * 64 + YO_PAIR_YROWS * 4 * 2 * 64 + w * TY * 4 * 2 * 32;
    auto yst = [&](int sr, int v, int par) -> float & { return ystash[((sr * 4 + v) * 2 + par) * 64]; };
    auto xst_ = [&](int r, int v, int par) -> float & { return xstash[((r * 4 + v) * 2 + par) * 32 + xi]; };

    // byte offsets: of row r within a plane of the state (half that for kappa), and
    // which rows this block owns
    const int pstr = rows * 6 * rowb;
    int rb[TY], own_rows = 0;
#pragma unroll
    for (int r = 0; r < TY; ++r) {
        rb[r] = (clampi(jb + r, -1, ny) + 1) * 6 * rowb;
        if (jb + r >= J0 && jb + r < J0 + JN) own_rows |= 1 << r;
    }

    // by plane parity: E^n, Ht^{n+1/2}, E^{n+1}, kappa, Ht^{n+3/2} and the z
    // memories of step n+1 (the second of a plane's two is the plane before)
    float E0[2][3][TY], H[2][3][TY], E1_[2][3][TY], K[2][3][TY], H2_[2][3][TY];
    float zH_[2][2][TY], zE_[2][2][TY];
    const int kb = k0 == 0 ? 0 : k0 - 2;
#pragma unroll
    for (int r = 0; r < TY; ++r) {
        const int o = (kb + 1) * pstr + rb[r];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            E0[0][c][r] = bload(FA, xl, c * rowb + o);
            H[1][c][r] = E1_[1][c][r] = K[1][c][r] = 0.0f;
        }
        H2_[1][0][r] = H2_[1][1][r] = 0.0f;
        zH_[1][0][r] = zH_[1][1][r] = zE_[1][0][r] = zE_[1][1][r] = 0.0f;
    }
    slot(2 * (kb & 1), w) = E0[0][0][0];
    slot(2 * (kb & 1) + 1, w) = E0[0][2][0];
    slot(4 + 2 * ((kb - 1) & 1), w) = 0.0f;
    slot(4 + 2 * ((kb - 1) & 1) + 1, w) = 0.0f;
    block_sync_lds();

    // loads of plane k's operands: E^n of plane k+1, Ht and kappa of plane k
    auto load_plane = [&](int k, float (&en)[3][TY], float (&hc)[3][TY], float (&kc)[3][TY]) {
        const int oh = (k + 1) * pstr, oe = k + 1 > nz ? oh : oh + pstr;
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const int e = oe + rb[r], h = oh + rb[r] + 3 * rowb, q = (oh + rb[r]) >> 1;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                en[c][r] = bload(FA, xl, c * rowb + e);
                hc[c][r] = bload(FA, xl, c * rowb + h);
                kc[c][r] = bload(KR, xl, c * rowb + q);
            }
        }
    };
    int k = kb;
    // one plane; the arrays are those of plane k and of plane k-1, which the
    // next call swaps (so nothing is copied from plane to plane)
    auto plane = [&](float (&Ec)[3][TY], float (&En)[3][TY], float (&Hc)[3][TY], float (&Hp)[3][TY],
                     float (&E1)[3][TY], float (&E1p)[3][TY], float (&Kc)[3][TY], float (&Kp)[3][TY],
                     float (&H2)[3][TY], float (&H2p)[3][TY], float (&zH)[2][TY], float (&zHp)[2][TY],
                     float (&zE)[2][TY], float (&zEp)[2][TY]) {
        const int par = k & 1;
        const int km = k - 1;
        const int pz = slab_index(k, nz, zlo, zhi), pzm = slab_index(km, nz, zlo, zhi);
        const bool kin = k >= 0 && k < nz, kmin = km >= 0 && km < nz;
        load_plane(k, En, Hc, Kc);
        if (pz >= 0) {
#pragma unroll
            for (int r = 0; r < TY; ++r) {
                const int j = clampi(jb + r, 0, ny - 1);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    zH[c][r] = bload(PS, xl, az(6 + 2 * s0 + c, pz, j));
                    zE[c][r] = bload(PS, xl, az(2 * s0 + c, pz, j));
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < TY; ++r) zH[0][r] = zH[1][r] = zE[0][r] = zE[1][r] = 0.0f;
        }
        // old memories of the x- and y-slabs (H, H, E, E), loaded with the
        // plane's fields so that one wait covers all
        float qx[CP ? 4 : 1][TY], qy[CP ? 4 : 1][TY];
        if constexpr (CP) {
            if (xc && kin) {
                const int pv = px >= 0 ? px : kFar;
#pragma unroll
                for (int r = 0; r < TY; ++r) {
                    const int j = clampi(jb + r, 0, ny - 1);
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        qx[c][r] = bload(PS, pv, ax(6 + 2 * s0 + c, k, j));
                        qx[2 + c][r] = bload(PS, pv, ax(2 * s0 + c, k, j));
                    }
                }
            }
            if (yc && kin) {
#pragma unroll
                for (int r = 0; r < TY; ++r) {
                    const int py = slab_index(jb + r, ny, ylo, yhi);
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        qy[c][r] = bload(PS, py >= 0 ? xl : kFar, ay(6 + 2 * s0 + c, k, py >= 0 ? py : 0));
                        qy[2 + c][r] = bload(PS, py >= 0 ? xl : kFar, ay(2 * s0 + c, k, py >= 0 ? py : 0));
                    }
                }
            }
        }
        slot(2 * (par ^ 1), w) = En[0][0];
        slot(2 * (par ^ 1) + 1, w) = En[2][0];

        // ---- S1 ----
        Cpml cz = {1.0f, 0.0f, 1.0f};
        if (pz >= 0) cz = cpml_uniform(profz, nz, 3, k);
        const int wu = w + 1 < W ? w + 1 : w;
        const float exu = slot(2 * par, wu), ezu = slot(2 * par + 1, wu);
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const int j = jb + r;
            const float eu0 = r + 1 < TY ? Ec[0][r + 1 < TY ? r + 1 : r] : exu;
            const float eu2 = r + 1 < TY ? Ec[2][r + 1 < TY ? r + 1 : r] : ezu;
            float dyEz = eu2 - Ec[2][r];
            float dzEy = En[1][r] - Ec[1][r];
            float dzEx = En[0][r] - Ec[0][r];
            float dxEz = shfl_next(Ec[2][r]) - Ec[2][r];
            float dxEy = shfl_next(Ec[1][r]) - Ec[1][r];
            float dyEx = eu0 - Ec[0][r];
            const bool jin = j >= 0 && j < ny;
            if (xc && kin && jin && px >= 0) {
                float n0, n1;
                dxEz = pml_diff(dxEz, cxH, qx[0][r], n0);
                dxEy = pml_diff(dxEy, cxH, qx[CP ? 1 : 0][r], n1);
                xst_(r, 0, par) = n0;
                xst_(r, 1, par) = n1;
            }
            if (yc && kin) {
                const int py = slab_index(j, ny, ylo, yhi);
                if (py >= 0) {
                    const Cpml cy = cpml_uniform(profy, ny, 3, j);
                    const int sr = j < ylo ? j : j - (ny - yhi);
                    float n0, n1;
                    dyEz = pml_diff(dyEz, cy, qy[0][r], n0);
                    dyEx = pml_diff(dyEx, cy, qy[CP ? 1 : 0][r], n1);
                    yst(sr, 0, par) = n0;
                    yst(sr, 1, par) = n1;
                }
            }
            if (pz >= 0 && jin) {
                dzEy = pml_diff(dzEy, cz, zH[0][r], zH[0][r]);
                dzEx = pml_diff(dzEx, cz, zH[1][r], zH[1][r]);
            }
            Hc[0][r] = Hc[0][r] - fmaf(sy, dyEz, -(sz * dzEy));
            Hc[1][r] = Hc[1][r] - fmaf(sz, dzEx, -(sx * dxEz));
            Hc[2][r] = Hc[2][r] - fmaf(sx, dxEy, -(sy * dyEx));
        }
        slot(8, w) = Hc[0][TY - 1];
        slot(9, w) = Hc[2][TY - 1];
        block_sync_lds();

        // ---- S2 ----
        if (pz >= 0) cz = cpml_uniform(profz, nz, 0, k);
        const int wd = w > 0 ? w - 1 : 0;
        const float hxd = slot(8, wd), hzd = slot(9, wd);
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const int j = jb + r;
            const float hd0 = r > 0 ? Hc[0][r > 0 ? r - 1 : 0] : hxd;
            const float hd2 = r > 0 ? Hc[2][r > 0 ? r - 1 : 0] : hzd;
            float dyHz = Hc[2][r] - hd2;
            float dzHy = Hc[1][r] - Hp[1][r];
            float dzHx = Hc[0][r] - Hp[0][r];
            float dxHz = Hc[2][r] - shfl_prev(Hc[2][r]);
            float dxHy = Hc[1][r] - shfl_prev(Hc[1][r]);
            float dyHx = Hc[0][r] - hd0;
            const bool jin = j >= 0 && j < ny;
            if (xc && kin && jin && px >= 0) {
                float n0, n1;
                dxHz = pml_diff(dxHz, cxE, qx[CP ? 2 : 0][r], n0);
                dxHy = pml_diff(dxHy, cxE, qx[CP ? 3 : 0][r], n1);
                xst_(r, 2, par) = n0;
                xst_(r, 3, par) = n1;
            }
            if (yc && kin) {
                const int py = slab_index(j, ny, ylo, yhi);
                if (py >= 0) {
                    const Cpml cy = cpml_uniform(profy, ny, 0, j);
                    const int sr = j < ylo ? j : j - (ny - yhi);
                    float n0, n1;
                    dyHz = pml_diff(dyHz, cy, qy[CP ? 2 : 0][r], n0);
                    dyHx = pml_diff(dyHx, cy, qy[CP ? 3 : 0][r], n1);
                    yst(sr, 2, par) = n0;
                    yst(sr, 3, par) = n1;
                }
            }
            if (pz >= 0 && jin) {
                dzHy = pml_diff(dzHy, cz, zE[0][r], zE[0][r]);
                dzHx = pml_diff(dzHx, cz, zE[1][r], zE[1][r]);
            }
            float ex = fmaf(Kc[0][r], fmaf(sy, dyHz, -(sz * dzHy)), Ec[0][r]);
            float ey = fmaf(Kc[1][r], fmaf(sz, dzHx, -(sx * dxHz)), Ec[1][r]);
            float ez = fmaf(Kc[2][r], fmaf(sx, dxHy, -(sy * dyHx)), Ec[2][r]);
            E1[0][r] = CP && j == 0 ? 0.0f : ex;
            E1[1][r] = CP && x_first ? 0.0f : ey;
            E1[2][r] = CP && (x_first || j == 0) ? 0.0f : ez;
        }
        if (k == 0) {   // perfect conductor (x = 0 and y = 0: CP tiles only)
#pragma unroll
            for (int r = 0; r < TY; ++r) E1[0][r] = E1[1][r] = 0.0f;
        }
        // the soft current source of step n on E^{n+1}
        auto source = [&](int kk, const float4 &st, float (&e)[3][TY], const float (&kv)[3][TY]) {
            if (!src_on || kk < sp.lo1 || kk >= sp.lo1 + sp.n1) return;
            const int pl = sp.n0 * sp.n1, d = x - sp.index;
            if (!(d == 0 || (snc == 5 && d == 1))) return;
#pragma unroll
            for (int r = 0; r < TY; ++r) {
                const int a = jb + r - sp.lo0;
                if (a < 0 || a >= sp.n0) continue;
                const float2 *q = sj + (kk - sp.lo1) * sp.n0 + a;
                const float2 jy = q[(d ? 3 : 0) * pl], jz = q[(d ? 4 : 1) * pl];
                e[1][r] = fmaf(-kv[1][r], fmaf(jy.x, st.x, jy.y * st.y), e[1][r]);
                e[2][r] = fmaf(-kv[2][r], fmaf(jz.x, st.x, jz.y * st.y), e[2][r]);
                if (snc == 5 && d == 0) {
                    const float2 jx = q[2 * pl];
                    e[0][r] = fmaf(-kv[0][r], fmaf(jx.x, st.x, jx.y * st.y), e[0][r]);
                }
            }
        };
        source(k, st0, E1, Kc);
        slot(4 + 2 * par, w) = E1[0][0];
        slot(4 + 2 * par + 1, w) = E1[2][0];

        // ---- S3 at plane k-1 ----
        const bool ownk = km >= k0 && km < k1;
        if (pzm >= 0) cz = cpml_uniform(profz, nz, 3, km);
        const float fxu = slot(4 + 2 * (par ^ 1), wu), fzu = slot(4 + 2 * (par ^ 1) + 1, wu);
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const int j = jb + r;
            const float eu0 = r + 1 < TY ? E1p[0][r + 1 < TY ? r + 1 : r] : fxu;
            const float eu2 = r + 1 < TY ? E1p[2][r + 1 < TY ? r + 1 : r] : fzu;
            float dyEz = eu2 - E1p[2][r];
            float dzEy = E1[1][r] - E1p[1][r];
            float dzEx = E1[0][r] - E1p[0][r];
            float dxEz = shfl_next(E1p[2][r]) - E1p[2][r];
            float dxEy = shfl_next(E1p[1][r]) - E1p[1][r];
            float dyEx = eu0 - E1p[0][r];
            const bool jin = j >= 0 && j < ny;
            const bool own = ownk && (own_rows >> r & 1);
            if (xc && kmin && jin && px >= 0) {
                float n0, n1;
                dxEz = pml_diff(dxEz, cxH, xst_(r, 0, par ^ 1), n0);
                dxEy = pml_diff(dxEy, cxH, xst_(r, 1, par ^ 1), n1);
                if (own && L.own) {
                    bstore(n0, PS, px, ax(6 + 2 * s2, km, j));
                    bstore(n1, PS, px, ax(6 + 2 * s2 + 1, km, j));
                }
            }
            if (yc && kmin) {
                const int py = slab_index(j, ny, ylo, yhi);
                if (py >= 0) {
                    const Cpml cy = cpml_uniform(profy, ny, 3, j);
                    const int sr = j < ylo ? j : j - (ny - yhi);
                    float n0, n1;
                    dyEz = pml_diff(dyEz, cy, yst(sr, 0, par ^ 1), n0);
                    dyEx = pml_diff(dyEx, cy, yst(sr, 1, par ^ 1), n1);
                    if (own) {
                        bstore(n0, PS, xst, ay(6 + 2 * s2, km, py));
                        bstore(n1, PS, xst, ay(6 + 2 * s2 + 1, km, py));
                    }
                }
            }
            if (pzm >= 0 && jin) {
                float n0, n1;
                dzEy = pml_diff(dzEy, cz, zHp[0][r], n0);
                dzEx = pml_diff(dzEx, cz, zHp[1][r], n1);
                if (own) {
                    bstore(n0, PS, xst, az(6 + 2 * s2, pzm, j));
                    bstore(n1, PS, xst, az(6 + 2 * s2 + 1, pzm, j));
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
        if (pzm >= 0) cz = cpml_uniform(profz, nz, 0, km);
        const float gxd = slot(10, wd), gzd = slot(11, wd);
        float E2[3][TY];
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const int j = jb + r;
            const float hd0 = r > 0 ? H2[0][r > 0 ? r - 1 : 0] : gxd;
            const float hd2 = r > 0 ? H2[2][r > 0 ? r - 1 : 0] : gzd;
            float dyHz = H2[2][r] - hd2;
            float dzHy = H2[1][r] - H2p[1][r];
            float dzHx = H2[0][r] - H2p[0][r];
            float dxHz = H2[2][r] - shfl_prev(H2[2][r]);
            float dxHy = H2[1][r] - shfl_prev(H2[1][r]);
            float dyHx = H2[0][r] - hd0;
            const bool own = ownk && (own_rows >> r & 1);
            if (xc && own && px >= 0) {
                float n0, n1;
                dxHz = pml_diff(dxHz, cxE, xst_(r, 2, par ^ 1), n0);
                dxHy = pml_diff(dxHy, cxE, xst_(r, 3, par ^ 1), n1);
                if (L.own) {
                    bstore(n0, PS, px, ax(2 * s2, km, j));
                    bstore(n1, PS, px, ax(2 * s2 + 1, km, j));
                }
            }
            if (yc && own) {
                const int py = slab_index(j, ny, ylo, yhi);
                if (py >= 0) {
                    const Cpml cy = cpml_uniform(profy, ny, 0, j);
                    const int sr = j < ylo ? j : j - (ny - yhi);
                    float n0, n1;
                    dyHz = pml_diff(dyHz, cy, yst(sr, 2, par ^ 1), n0);
                    dyHx = pml_diff(dyHx, cy, yst(sr, 3, par ^ 1), n1);
                    bstore(n0, PS, xst, ay(2 * s2, km, py));
                    bstore(n1, PS, xst, ay(2 * s2 + 1, km, py));
                }
            }
            if (pzm >= 0 && own) {
                float n0, n1;
                dzHy = pml_diff(dzHy, cz, zEp[0][r], n0);
                dzHx = pml_diff(dzHx, cz, zEp[1][r], n1);
                bstore(n0, PS, xst, az(2 * s2, pzm, j));
                bstore(n1, PS, xst, az(2 * s2 + 1, pzm, j));
            }
            float ex = fmaf(Kp[0][r], fmaf(sy, dyHz, -(sz * dzHy)), E1p[0][r]);
            float ey = fmaf(Kp[1][r], fmaf(sz, dzHx, -(sx * dxHz)), E1p[1][r]);
            float ez = fmaf(Kp[2][r], fmaf(sx, dxHy, -(sy * dyHx)), E1p[2][r]);
            E2[0][r] = CP && j == 0 ? 0.0f : ex;
            E2[1][r] = CP && x_first ? 0.0f : ey;
            E2[2][r] = CP && (x_first || j == 0) ? 0.0f : ez;
        }
        if (km == 0) {
#pragma unroll
            for (int r = 0; r < TY; ++r) E2[0][r] = E2[1][r] = 0.0f;
        }
        source(km, st1, E2, Kp);
        if (ownk) {
            const int om = (km + 1) * pstr;
#pragma unroll
            for (int r = 0; r < TY; ++r) {
                if (!(own_rows >> r & 1)) continue;
                const int o = om + rb[r];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    bstore_nt(E2[c][r], FC, xst, c * rowb + o);
                    bstore_nt(H2[c][r], FC, xst, (3 + c) * rowb + o);
                }
            }
        }
    };
    for (;;) {
        plane(E0[0], E0[1], H[0], H[1], E1_[0], E1_[1], K[0], K[1], H2_[0], H2_[1], zH_[0], zH_[1], zE_[0], zE_[1]);
        if (++k > k1) break;
        plane(E0[1], E0[0], H[1], H[0], E1_[1], E1_[0], K[1], K[0], H2_[1], H2_[0], zH_[1], zH_[0], zE_[1], zE_[0]);
        if (++k > k1) break;
    }
}

template <int TY, int W, bool CP>
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
    const YoPlanD &P = *sl.plan;
    const int step = *P.step_ctr + a.k_offset;
    // the host schedules a pair only where both steps remain
    if (step + 1 >= P.n_steps) return;
    const int blk = (wave0 - a.prefix[s]) / W;
    // consecutive blocks take neighbouring strips of the same rows (whose row
    // segments are neighbours in memory) of one right-hand side, then the same
    // tiles of the next one, which share kappa
    // (order alone, 600x400x120 with 25 right-hand sides: 6.4 to 7.3 ms per step
    // with one tile after another over the right-hand sides, 5.8 in groups)
    const int G = YO_PAIR_GROUP;
    const int g = blk / (G * sl.nrhs), in_g = blk - g * (G * sl.nrhs);
    const int gsz = min(G, sl.ntile - g * G);
    if (gsz <= 0) return;
    const int r = sl.rhs0 + in_g / gsz;
    const int ti = g * G + in_g % gsz;
    extern __shared__ float lds[];
    wave_pair<TY, W, CP>(P, P.rhs[r], step, sl.tiles[ti], w, lane, lds);
}

}  // namespace

hipError_t yo_launch_pair(bool shell, const YoStepArgs &args, int blocks, hipStream_t s)
{
    if (blocks <= 0) return hipSuccess;
    if (args.wpb != YO_PAIR_W) return hipErrorInvalidValue;
    const size_t lds = sizeof(float) * 12 * YO_PAIR_W * 64;
    const size_t lds_shell = lds + sizeof(float) * (YO_PAIR_YROWS * 4 * 2 * 64 + YO_PAIR_W * YO_PAIR_TY * 4 * 2 * 32);
    const dim3 g(blocks), b(64 * YO_PAIR_W);
    if (shell) hipLaunchKernelGGL((k_yee_pair<YO_PAIR_TY, YO_PAIR_W, true>), g, b, lds_shell, s, args);
    else hipLaunchKernelGGL((k_yee_pair<YO_PAIR_TY, YO_PAIR_W, false>), g, b, lds, s, args);
    return hipGetLastError();
}
