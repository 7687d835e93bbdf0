// Parametrization chain (paper Sec. 3) and its vector-Jacobian product, plus
// the small kernels around the time stepping: fills, pitched copies, the
// steady-state fit, the modal overlap and the Eq. (1) gradient assembly.
// All of this is 2-D or plane-sized work next to the 3-D time stepping; the
// kernels are plain one-thread-per-output gathers (no atomics, fixed
// summation order, so results do not depend on scheduling).
#include <algorithm>
#include <type_traits>

#include "yo_internal.h"

namespace {

constexpr int BS = 256;

inline int nblk(size_t n) { return (int)((n + BS - 1) / BS); }

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// ------------------------------------------------------------- utilities
__global__ void k_fill(float *p, size_t n, float v)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// dense [ncomp][nz][ny][nx] -> components c0.. of a ghost-layout array of nc
// components (interior only; ghosts untouched).  Flat over the dense array, so
// that its side is whole lines; indices fit 32 bits (the library's grids have
// under 2^31 values in three components), 64-bit divisions here cost more than
// the copy.  Plane: of kappa, also each plane's first cell, and a mark that k_kplane
// clears.
template <bool Plane>
__global__ void k_to_ghost(const float *src, const YoGhost to, unsigned n, int c0, int nc, unsigned nz, unsigned ny,
                           unsigned nx, int ns, float4 *kplane)
{
    float *dst = to.F[to.now ? *to.now : 0];
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const unsigned row = i / nx, x = i - row * nx;
        const unsigned pl = row / ny, y = row - pl * ny;
        const unsigned q = pl / nz, z = pl - q * nz;
        dst[yo_off(c0 + (int)q, (int)x, (int)y, (int)z, (int)ny, ns, nc)] = src[i];
        if (Plane && !x && !y) {
            float *e = reinterpret_cast<float *>(kplane + z);
            e[q] = src[i];
            if (!q) e[3] = 1.0f;
        }
    }
}

__global__ void k_from_ghost(const YoGhost from, float *dst, unsigned n, int c0, int nc, unsigned nz, unsigned ny,
                             unsigned nx, int ns)
{
    const float *src = from.F[from.now ? *from.now : 0];
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const unsigned row = i / nx, x = i - row * nx;
        const unsigned pl = row / ny, y = row - pl * ny;
        const unsigned q = pl / nz, z = pl - q * nz;
        dst[i] = src[yo_off(c0 + (int)q, (int)x, (int)y, (int)z, (int)ny, ns, nc)];
    }
}

// Which planes hold one value per component: blocks that compare a plane's cells
// with its first bit by bit, a wave per row, strips (yo_col) side by side, a lane
// a column, and clear the plane's mark where one differs.  (600x400x120: 400 us
// with one block a plane.)  The canvas' mask is copied on the way (two launches
// fewer: 13 us of yo_set_background on 30x26x18 cells, not 18).
__global__ __launch_bounds__(BS) void k_kplane(const float *kappa, float4 *kplane, int ny, int nx, int ns, int k_lo,
                                               int k_hi, const float *mask, float *mask_out, size_t n)
{
    for (size_t i = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * BS + threadIdx.x; i < n;
         i += (size_t)gridDim.x * gridDim.y * BS)
        mask_out[i] = mask[i];
    const int k = blockIdx.x, lane = threadIdx.x & 63;
    if (k >= k_lo && k <= k_hi) {
        if (!blockIdx.y && !threadIdx.x) kplane[k].w = 0.0f;
        return;
    }
    const float *v = kappa + yo_off(0, 0, 0, k, ny, ns, 3);
    const unsigned first[3] = {__float_as_uint(v[0]), __float_as_uint(v[64]), __float_as_uint(v[128])};
    bool differs = false;
    for (int y = blockIdx.y * (BS / 64) + (threadIdx.x >> 6); y < ny; y += gridDim.y * (BS / 64)) {
        const float *row = kappa + yo_off(0, 0, y, k, ny, ns, 3) - YO_LEAD;
        for (int s = 0; s < ns; ++s) {
            const bool in = lane >= YO_LEAD && lane < YO_LEAD + YO_SW && s * YO_SW + lane - YO_LEAD < nx;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const unsigned u = __float_as_uint(row[(s * 3 + c) * 64 + lane]);
                differs = differs || (in && u != first[c]);
            }
        }
    }
    if (differs) kplane[k].w = 0.0f;
}

// Ehat = (g00 Re S + g01 Im S) + i (g10 Re S + g11 Im S): least-squares
// amplitude/phase from the DFT sums S = sum E^n exp(+i w n dt).  Any
// non-finite phasor (all-ones exponent bits) sets *bad to 1: one atomic per
// wave that holds one.
__global__ void k_finalize(float2 *a, size_t n, float g00, float g01, float g10, float g11, int *bad)
{
    unsigned int nonfinite = 0u;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        const float2 s = a[i];
        const float2 e = make_float2(fmaf(g00, s.x, g01 * s.y), fmaf(g10, s.x, g11 * s.y));
        a[i] = e;
        nonfinite |= (__float_as_uint(e.x) & 0x7f800000u) == 0x7f800000u;
        nonfinite |= (__float_as_uint(e.y) & 0x7f800000u) == 0x7f800000u;
    }
    const unsigned long long m = __ballot(nonfinite != 0u);
    if ((threadIdx.x & 63) == 0 && m) atomicOr(bad, 1);
}

// alpha = sum w * Ehat over one port plane, a block per source, port and
// frequency; fixed-order tree
__global__ void k_alpha(const YoAlphaArgs a)
{
    __shared__ float sr[BS], si[BS];
    const int f = blockIdx.x % a.n_freq, sp = blockIdx.x / a.n_freq;
    const int p = sp % a.n_ports, src = sp / a.n_ports;
    const float2 *e = a.mon + a.mon_stride * (size_t)(f * a.n_src + src) + a.mon_off[p];
    const float2 *w = a.w + a.w_fstride * (size_t)f + a.w_off[p];
    const int n = a.n[p];
    float ar = 0.0f, ai = 0.0f;
    for (int i = threadIdx.x; i < n; i += BS) {
        const float2 u = w[i], b = e[i];
        ar = fmaf(u.x, b.x, fmaf(-u.y, b.y, ar));
        ai = fmaf(u.x, b.y, fmaf(u.y, b.x, ai));
    }
    sr[threadIdx.x] = ar;
    si[threadIdx.x] = ai;
    __syncthreads();
    for (int s = BS / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            sr[threadIdx.x] += sr[threadIdx.x + s];
            si[threadIdx.x] += si[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) a.out[blockIdx.x] = make_float2(sr[0], si[0]);
}

// ------------------------------------------------------------- forward chain
// Eq. (2) with the truncated Gaussian basis (separable taps with clamped
// control indices).  First along x: tmp[b][ud], a control row at each
// sub-pixel column (shared by the S nd / nc times 2r sub-pixel rows that read
// it: one pass over the controls per sub-pixel took 17 us at 400x400
// sub-pixels and r = 3, the two passes 8 together; yo_filter_by_rows says where).
__device__ __forceinline__ float filter_x(const YoChainBufs &c, const float *C, int b, int ud)
{
    const int xlo = c.tap_lo_x[ud], xn = c.tap_n_x[ud];
    float row = 0.0f;
    for (int tx = 0; tx < xn; ++tx) {
        const int a = clampi(xlo + tx, 0, c.mc - 1);
        row = fmaf(c.tap_w_x[ud * c.tmax + tx], C[b * c.mc + a], row);
    }
    return row;
}

__global__ void k_filter_x(YoChainBufs c, const float *C)
{
    const int nud = c.S * c.md;
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i >= c.nc * nud) return;
    const int b = i / nud;
    c.tmp[i] = filter_x(c, C, b, i - b * nud);
}

// Then along y and the tanh projection Eq. (3)/(6) into the canvas `out`,
// whose margin takes the background fill.  Rows: x is done (tmp), else C's rows
// are filtered here.
template <bool Rows>
__global__ void k_project(YoChainBufs c, const float *C, float beta, float *out)
{
    const int n = c.U * c.V;
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i >= n) return;
    const int v = i / c.U, u = i - v * c.U;
    const int nud = c.S * c.md, ud = u - 2 * c.S, vd = v - 2 * c.S;
    if (ud < 0 || ud >= nud || vd < 0 || vd >= c.S * c.nd) {
        out[i] = c.mask[i];
        return;
    }
    const int ylo = c.tap_lo_y[vd], yn = c.tap_n_y[vd];
    float phi = 0.0f;
    for (int ty = 0; ty < yn; ++ty) {
        const int b = clampi(ylo + ty, 0, c.nc - 1);
        phi = fmaf(c.tap_w_y[vd * c.tmax + ty], Rows ? c.tmp[b * nud + ud] : filter_x(c, C, b, ud), phi);
    }
    phi -= 0.5f;
    const float t = tanhf(beta * phi);
    c.tanh_[vd * nud + ud] = t;
    out[i] = 0.5f * (1.0f + t);
}

// The disc sums of the morphological stages: a block takes a tile of 64 x 16
// sub-pixels, with the disc's radius around it in LDS, each thread four
// neighbours of a row, which share the values a row of the disc passes over.
// The sums run over the taps row by row in the order of the tap table
// (mirrored in the transpose).  The tile's exponentials (or quotients) are
// taken once each, not once per tap: at a radius of 10 (317 taps) and 416x416
// sub-pixels a stage took 80 us (its transpose 75) with both done per tap.
// Rows of odd pitch keep the four rows a wave reads in different banks.
// Small discs wait for single reads: with the rows of one and three taps in loops
// and one tile value in flight at a time four stages of 13 taps took 43.4 us with
// the rest of yo_set_design (a thread and an exponential per tap: 38.6), now 38.4.
constexpr int MTX = 64, MTY = 16;
template <bool mirror>
__device__ __forceinline__ void disc_sums(const float *tile, int R, const int *wid, int lx, int ly, float (&acc)[4])
{
    const int pitch = (MTX + 2 * R) | 1;
    acc[0] = acc[1] = acc[2] = acc[3] = 0.0f;
    for (int dy = -R; dy <= R; ++dy) {
        const int w = wid[dy + R];
        if (w < 0) continue;
        const float *row = tile + (ly + R + (mirror ? -dy : dy)) * pitch + lx + R;
        // the 2w + 4 values of the row under the four discs, in the taps' order
        const int dir = mirror ? -1 : 1;
        const float *x = row + (mirror ? w + 3 : -w);
        auto tap = [&](int j, int i, int n) {     // value j of the row, disc i; n values a disc
            const int d = mirror ? 3 - i : i;
            if (j >= d && j - d < n) acc[i] += x[dir * j];
        };
        // (rows too short for the shared middle, at lengths the compiler knows: their
        // reads are in flight together)
        auto few = [&](auto n) {
#pragma unroll
            for (int j = 0; j < n() + 3; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) tap(j, i, n());
        };
        if (w < 2) {
            if (w) few(std::integral_constant<int, 3>());
            else few(std::integral_constant<int, 1>());
            continue;
        }
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) tap(j, i, 5);
#pragma unroll 4
        for (int j = 3; j <= 2 * w; ++j) {
            const float v = x[dir * j];
            acc[0] += v;
            acc[1] += v;
            acc[2] += v;
            acc[3] += v;
        }
#pragma unroll
        for (int j = 1; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if ((mirror ? 3 - i : i) >= j) acc[i] += x[dir * (2 * w + j)];
    }
}

// Eqs. (4)-(5): one soft dilation or erosion of the canvas `in` with the
// normalised disc (mean over the taps), on the design area; taps are
// clamped into the canvas, so near the design edge they read the fixed
// margin.  Exponents are shifted so every term is at most one:
// dilation 1 + log(mean e^{a(rho-1)}) / a, erosion -log(mean e^{-a rho}) / a
// (the same values as Eqs. (4)-(5)).  The mean is kept for the transpose.
__global__ __launch_bounds__(BS) void k_morph(YoChainBufs c, const float *in, float *out, float *sum, int dilate)
{
    extern __shared__ float tile[];
    __shared__ int wid[2 * YO_MAX_DISC + 1];
    const int R = c.mrad, pitch = (MTX + 2 * R) | 1;
    const int u0 = blockIdx.x * MTX, v0 = blockIdx.y * MTY;
    const float a = c.malpha;
    for (int i = threadIdx.x; i < 2 * R + 1; i += BS) wid[i] = c.mwid[i];
#pragma unroll 4
    for (int i = threadIdx.x; i < pitch * (MTY + 2 * R); i += BS) {
        const int ty = i / pitch, tx = i - ty * pitch;
        const float r = in[clampi(v0 + ty - R, 0, c.V - 1) * c.U + clampi(u0 + tx - R, 0, c.U - 1)];
        tile[i] = dilate ? expf(a * (r - 1.0f)) : expf(-a * r);
    }
    __syncthreads();
    const int lx = (threadIdx.x & 15) * 4, ly = threadIdx.x >> 4;
    float acc[4];
    disc_sums<false>(tile, R, wid, lx, ly, acc);
    const int v = v0 + ly, vd = v - 2 * c.S;
    if (v >= c.V) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int u = u0 + lx + q, ud = u - 2 * c.S, i = v * c.U + u;
        if (u >= c.U) break;
        if (ud < 0 || ud >= c.S * c.md || vd < 0 || vd >= c.S * c.nd) {
            out[i] = c.mask[i];
            continue;
        }
        const float m = acc[q] * c.minv;
        sum[vd * (c.S * c.md) + ud] = m;
        const float l = logf(m) / a;
        out[i] = dilate ? 1.0f + l : -l;
    }
}

// The projection after the morphological stages, Eq. (6):
// rho = (1 + tanh(beta (rho~ - 1/2))) / 2 on the design area.
__global__ void k_morph_project(YoChainBufs c, const float *in, float beta)
{
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i >= c.U * c.V) return;
    const int v = i / c.U, u = i - v * c.U;
    const int ud = u - 2 * c.S, vd = v - 2 * c.S;
    if (ud < 0 || ud >= c.S * c.md || vd < 0 || vd >= c.S * c.nd) {
        c.rho[i] = c.mask[i];
        return;
    }
    const float t = tanhf(beta * (in[i] - 0.5f));
    c.tanh2[vd * (c.S * c.md) + ud] = t;
    c.rho[i] = 0.5f * (1.0f + t);
}

// Eq. (8): S x S box means centred on each E component (E_x window shifted
// half a cell in x, E_y in y), of 1/eps, eps and rho.
__global__ void k_box(YoChainBufs c)
{
    const int gsz = c.G0 * c.G1;
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i >= 3 * gsz) return;
    const int comp = i / gsz, pix = i - comp * gsz;
    const int n = pix / c.G0, m = pix - n * c.G0;
    const int half = c.S / 2;
    const int shx = comp == 0 ? half : 0, shy = comp == 1 ? half : 0;
    const float de = c.eps_core - c.eps_clad;
    float p = 0.0f, q = 0.0f, r = 0.0f;
    for (int b = 0; b < c.S; ++b) {
        const int v = clampi(c.S * n + shy + b, 0, c.V - 1);
        for (int a = 0; a < c.S; ++a) {
            const int u = clampi(c.S * m + shx + a, 0, c.U - 1);
            const float rho = c.rho[v * c.U + u];
            const float eps = fmaf(de, rho, c.eps_clad);
            p += 1.0f / eps;
            q += eps;
            r += rho;
        }
    }
    const float inv = 1.0f / (float)(c.S * c.S);
    c.P[i] = p * inv;
    c.Q[i] = q * inv;
    c.R[i] = r * inv;
}

__device__ __forceinline__ void sobel(const float *R, int G0, int G1, int n, int m, float &gx,
                                      float &gy)
{
    const float w[3] = {1.0f, 2.0f, 1.0f};
    float sx = 0.0f, sy = 0.0f;
#pragma unroll
    for (int dn = -1; dn <= 1; ++dn) {
#pragma unroll
        for (int dm = -1; dm <= 1; ++dm) {
            const float v = R[clampi(n + dn, 0, G1 - 1) * G0 + clampi(m + dm, 0, G0 - 1)];
            sx = fmaf(w[dn + 1] * (float)dm, v, sx);
            sy = fmaf(w[dm + 1] * (float)dn, v, sy);
        }
    }
    gx = sx * 0.125f;
    gy = sy * 0.125f;
}

// Sobel normals, Eq. (7), extrusion through the slab into the 3-D kappa.
__global__ void k_smooth(YoChainBufs c, float *kappa, int ny, int ns, int i0,
                         int j0, int k_lo, int k_hi)
{
    const int wm = c.md + 2, wn = c.nd + 2;
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i >= wm * wn) return;
    const int n = 1 + i / wm, m = 1 + i % wm;
    const int gsz = c.G0 * c.G1;
    const int pix = n * c.G0 + m;
    float gxx, gyx, gxy, gyy;
    sobel(c.R, c.G0, c.G1, n, m, gxx, gyx);             // on the E_x grid
    sobel(c.R + gsz, c.G0, c.G1, n, m, gxy, gyy);       // on the E_y grid
    const float n2x = gxx * gxx / (gxx * gxx + gyx * gyx + c.delta);
    const float n2y = gyy * gyy / (gxy * gxy + gyy * gyy + c.delta);
    const float kx = fmaf(n2x, c.P[pix], (1.0f - n2x) / c.Q[pix]);
    const float ky = fmaf(n2y, c.P[gsz + pix], (1.0f - n2y) / c.Q[gsz + pix]);
    const float kzi = 1.0f / c.Q[2 * gsz + pix];
    const float kzf = 0.5f * (c.P[2 * gsz + pix] + 1.0f / c.eps_clad);
    c.aux[0 * gsz + pix] = n2x;
    c.aux[1 * gsz + pix] = n2y;
    c.aux[2 * gsz + pix] = gxx;
    c.aux[3 * gsz + pix] = gyx;
    c.aux[4 * gsz + pix] = gxy;
    c.aux[5 * gsz + pix] = gyy;
    const int x = i0 - 2 + m, y = j0 - 2 + n;
    for (int k = k_lo; k <= k_hi; ++k) {
        kappa[yo_off(0, x, y, k, ny, ns, 3)] = kx;
        kappa[yo_off(1, x, y, k, ny, ns, 3)] = ky;
    }
    for (int k = k_lo; k < k_hi; ++k) kappa[yo_off(2, x, y, k, ny, ns, 3)] = kzi;
    kappa[yo_off(2, x, y, k_lo - 1, ny, ns, 3)] = kzf;
    kappa[yo_off(2, x, y, k_hi, ny, ns, 3)] = kzf;
}

// ------------------------------------------------------------- Eq. (1)
// dF/deps_c(r) = sum_{f,s,p} 2 Re[coef_{s,p,f} (-2 i sin theta_f) E_F E_A]
//             = sum 4 sin theta_f Im[coef E_F E_A];  dF/dkappa = -dF/deps / kappa^2
// One thread per box value, which reads its n_freq (n_src + n_ports) phasors
// (one per in-plane cell, looping over components and planes, left the chip
// idle: 388 us on a 252x152x13 box with 5 wavelengths and 1 + 4 phasors each,
// 311 MB).
__global__ __launch_bounds__(BS) void k_grad(const YoGradArgs a)
{
    const int bx = a.box[3], by = a.box[4], bz = a.box[5];
    const int o = blockIdx.x * BS + threadIdx.x;
    if (o >= 3 * bx * by * bz) return;
    const int row = o / bx, bi = o - row * bx;
    const int pl = row / by, bj = row - pl * by;
    const int c = pl / bz, bk = pl - c * bz;
    float ge = 0.0f;
    for (int f = 0; f < a.n_freq; ++f) {
        const float s4 = 4.0f * a.sinth[f];
        for (int s = 0; s < a.n_src; ++s) {
            const float2 ef = a.EF[f * a.n_src + s][o];
#pragma unroll 4
            for (int p = 0; p < a.n_ports; ++p) {
                const float2 ea = a.EA[f * a.n_ports + p][o];
                const float2 cf = a.coef[(s * a.n_ports + p) * a.n_freq + f];
                // prod = ef * ea
                const float pr = fmaf(ef.x, ea.x, -ef.y * ea.y);
                const float pi = fmaf(ef.x, ea.y, ef.y * ea.x);
                // Im(cf * prod)
                const float im = fmaf(cf.x, pi, cf.y * pr);
                ge = fmaf(s4, im, ge);
            }
        }
    }
    const float kap = a.kappa[yo_off(c, a.box[0] + bi, a.box[1] + bj, a.box[2] + bk, a.ny, a.ns, 3)];
    a.gbox[o] = -ge / (kap * kap);
}

// ------------------------------------------------------------- chain VJP
// Transpose of the extrusion through the slab (dF/dkappa on the box summed
// over the E_x planes, the E_y planes, the interior and the face E_z), then
// the Eq. (7) partials and the normal-vector partials (written region only).
__global__ void k_vjp_pointwise(YoChainBufs c, const float *gbox, int z0, int bz, int k_lo, int k_hi)
{
    const int gsz = c.G0 * c.G1;
    const int pix = blockIdx.x * BS + threadIdx.x;
    if (pix >= gsz) return;
    const int n = pix / c.G0, m = pix - n * c.G0;
    const bool w = (n >= 1 && n <= c.nd + 2 && m >= 1 && m <= c.md + 2);
    float gP[3] = {0, 0, 0}, gQ[3] = {0, 0, 0}, gG[4] = {0, 0, 0, 0};
    if (w) {
        // box cell (bi, bj) is component-grid pixel (bi + 1, bj + 1)
        const int bx = c.md + 2, by = c.nd + 2, i = (n - 1) * bx + m - 1;
        const size_t cs = (size_t)bx * by * bz;
        float gm[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int bk = 0; bk < bz; ++bk) {
            const int z = z0 + bk;
            const size_t o = (size_t)bk * bx * by + i;
            const float g0 = gbox[o], g1 = gbox[cs + o], g2 = gbox[2 * cs + o];
            if (z >= k_lo && z <= k_hi) {
                gm[0] += g0;
                gm[1] += g1;
            }
            if (z >= k_lo && z < k_hi) gm[2] += g2;
            if (z == k_lo - 1 || z == k_hi) gm[3] += g2;
        }
        for (int comp = 0; comp < 2; ++comp) {
            const float g = gm[comp];
            const float n2 = c.aux[comp * gsz + pix];
            const float Gx = c.aux[(2 + 2 * comp) * gsz + pix];
            const float Gy = c.aux[(3 + 2 * comp) * gsz + pix];
            const float P = c.P[comp * gsz + pix], Q = c.Q[comp * gsz + pix];
            gP[comp] = g * n2;
            gQ[comp] = -g * (1.0f - n2) / (Q * Q);
            const float gn = g * (P - 1.0f / Q);
            const float D = Gx * Gx + Gy * Gy + c.delta;
            const float D2 = D * D;
            if (comp == 0) {
                gG[0] = gn * 2.0f * Gx * (Gy * Gy + c.delta) / D2;
                gG[1] = -gn * 2.0f * Gy * Gx * Gx / D2;
            } else {
                gG[3] = gn * 2.0f * Gy * (Gx * Gx + c.delta) / D2;
                gG[2] = -gn * 2.0f * Gx * Gy * Gy / D2;
            }
        }
        const float Qz = c.Q[2 * gsz + pix];
        gP[2] = 0.5f * gm[3];
        gQ[2] = -gm[2] / (Qz * Qz);
    }
    for (int k = 0; k < 3; ++k) {
        c.gPQ[k * gsz + pix] = gP[k];
        c.gPQ[(3 + k) * gsz + pix] = gQ[k];
    }
    for (int k = 0; k < 4; ++k) c.gG[k * gsz + pix] = gG[k];
}

// Transpose of the clamped Sobel stencils: gather every (pixel, tap) whose
// clamped source is this pixel.
__global__ void k_vjp_sobel(YoChainBufs c)
{
    const int gsz = c.G0 * c.G1;
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i >= 2 * gsz) return;
    const int comp = i / gsz, pix = i - comp * gsz;
    const int nq = pix / c.G0, mq = pix - nq * c.G0;
    const float *gx = c.gG + (2 * comp) * gsz;
    const float *gy = c.gG + (2 * comp + 1) * gsz;
    const float w[3] = {1.0f, 2.0f, 1.0f};
    float acc = 0.0f;
    for (int n = nq - 1; n <= nq + 1; ++n) {
        if (n < 0 || n >= c.G1) continue;
        for (int m = mq - 1; m <= mq + 1; ++m) {
            if (m < 0 || m >= c.G0) continue;
            const float ax = gx[n * c.G0 + m], ay = gy[n * c.G0 + m];
            for (int dn = -1; dn <= 1; ++dn) {
                if (clampi(n + dn, 0, c.G1 - 1) != nq) continue;
                for (int dm = -1; dm <= 1; ++dm) {
                    if (clampi(m + dm, 0, c.G0 - 1) != mq) continue;
                    acc = fmaf(w[dn + 1] * (float)dm * 0.125f, ax, acc);
                    acc = fmaf(w[dm + 1] * (float)dn * 0.125f, ay, acc);
                }
            }
        }
    }
    c.gR[i] = acc;
}

// number of window sub-pixels of pixel m (shift sh) that clamp onto u
__device__ __forceinline__ int win_count(int m, int sh, int S, int u, int n_hr)
{
    int cnt = 0;
    for (int a = 0; a < S; ++a) cnt += (clampi(S * m + sh + a, 0, n_hr - 1) == u);
    return cnt;
}

// Transpose of the box means to the canvas, the density mix and the
// derivative (beta/2)(1 - t^2) of the last projection (t = its tanh values)
// on the design area, into gout [S nd][S md].
__global__ void k_vjp_canvas(YoChainBufs c, float beta, const float *tproj, float *gout)
{
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i >= c.U * c.V) return;
    const int v = i / c.U, u = i - v * c.U;
    const int ud = u - 2 * c.S, vd = v - 2 * c.S;
    if (ud < 0 || ud >= c.S * c.md || vd < 0 || vd >= c.S * c.nd) return;
    const int gsz = c.G0 * c.G1;
    const int half = c.S / 2;
    const float invS2 = 1.0f / (float)(c.S * c.S);
    float gi = 0.0f, ge = 0.0f, gr = 0.0f;
    for (int comp = 0; comp < 3; ++comp) {
        const int shx = comp == 0 ? half : 0, shy = comp == 1 ? half : 0;
        const int mc0 = (u - shx) / c.S, nc0 = (v - shy) / c.S;
        for (int n = nc0 - 1; n <= nc0 + 1; ++n) {
            if (n < 0 || n >= c.G1) continue;
            const int cy = win_count(n, shy, c.S, v, c.V);
            if (!cy) continue;
            for (int m = mc0 - 1; m <= mc0 + 1; ++m) {
                if (m < 0 || m >= c.G0) continue;
                const int cx = win_count(m, shx, c.S, u, c.U);
                if (!cx) continue;
                const float wgt = (float)(cx * cy) * invS2;
                const int pix = n * c.G0 + m;
                gi = fmaf(wgt, c.gPQ[comp * gsz + pix], gi);
                ge = fmaf(wgt, c.gPQ[(3 + comp) * gsz + pix], ge);
                if (comp < 2) gr = fmaf(wgt, c.gR[comp * gsz + pix], gr);
            }
        }
    }
    const float de = c.eps_core - c.eps_clad;
    const float eps = fmaf(de, c.rho[i], c.eps_clad);
    const float grho = fmaf(gi, -de / (eps * eps), fmaf(ge, de, gr));
    const float t = tproj[vd * (c.S * c.md) + ud];
    gout[vd * (c.S * c.md) + ud] = grho * 0.5f * beta * (1.0f - t * t);
}

// Transpose of a morphological stage: d rho~(x) / d rho(x') = e(x') / (n
// mean(x)) for every tap with x + delta = x', e the stage's shifted
// exponential, so the gradient at x' gathers q = g / mean over x = x' - delta
// (the disc is symmetric) within the design area (taps that were clamped land
// in the margin, which has no gradient).  With tproj, the Eq. (3)
// projection's derivative follows.
__global__ __launch_bounds__(BS) void k_morph_vjp(YoChainBufs c, const float *g_, const float *sum, const float *in,
                                                  int dilate, const float *tproj, float beta, float *gout)
{
    extern __shared__ float tile[];
    __shared__ int wid[2 * YO_MAX_DISC + 1];
    const int nud = c.S * c.md, nvd = c.S * c.nd;
    const int R = c.mrad, pitch = (MTX + 2 * R) | 1;
    const int u0 = blockIdx.x * MTX, v0 = blockIdx.y * MTY;
    for (int i = threadIdx.x; i < 2 * R + 1; i += BS) wid[i] = c.mwid[i];
#pragma unroll 4
    for (int i = threadIdx.x; i < pitch * (MTY + 2 * R); i += BS) {
        const int ty = i / pitch, tx = i - ty * pitch;
        const int vq = v0 + ty - R, uq = u0 + tx - R;
        const bool in_area = vq >= 0 && vq < nvd && uq >= 0 && uq < nud;
        tile[i] = in_area ? g_[vq * nud + uq] / sum[vq * nud + uq] : 0.0f;
    }
    __syncthreads();
    const int lx = (threadIdx.x & 15) * 4, ly = threadIdx.x >> 4;
    float acc[4];
    disc_sums<true>(tile, R, wid, lx, ly, acc);
    const int vd = v0 + ly;
    if (vd >= nvd) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int ud = u0 + lx + q, i = vd * nud + ud;
        if (ud >= nud) break;
        const float r = in[(vd + 2 * c.S) * c.U + ud + 2 * c.S];
        const float e = dilate ? expf(c.malpha * (r - 1.0f)) : expf(-c.malpha * r);
        float g = e * acc[q] * c.minv;
        if (tproj) {
            const float t = tproj[i];
            g *= 0.5f * beta * (1.0f - t * t);
        }
        gout[i] = g;
    }
}

// Transpose of the separable filter, x then y, with each control's weights
// side by side (tapt; summed on the host where taps were clamped onto it).
// Searched among the sub-pixels' taps instead, each pass took 21 to 48 us.
__global__ void k_vjp_filter_x(YoChainBufs c)   // tmp[vd][a] = sum_ud gphi W_x(ud, a)
{
    const int i = blockIdx.x * BS + threadIdx.x;
    const int nvd = c.S * c.nd, nud = c.S * c.md;
    if (i >= nvd * c.mc) return;
    const int vd = i / c.mc, a = i - vd * c.mc;
    const int u0 = c.urange_x[2 * a], n = c.urange_x[2 * a + 1] - u0 + 1;
    const float *w = c.tapt_x + a, *g = c.gphi + vd * nud + u0;
    float acc = 0.0f;
#pragma unroll 8
    for (int t = 0; t < n; ++t) acc = fmaf(w[t * c.mc], g[t], acc);
    c.tmp[i] = acc;
}

__global__ void k_vjp_filter_y(YoChainBufs c, float *dFdC)
{
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i >= c.nc * c.mc) return;
    const int b = i / c.mc, a = i - b * c.mc;
    const int v0 = c.urange_y[2 * b], n = c.urange_y[2 * b + 1] - v0 + 1;
    const float *w = c.tapt_y + b, *g = c.tmp + v0 * c.mc + a;
    float acc = 0.0f;
#pragma unroll 8
    for (int t = 0; t < n; ++t) acc = fmaf(w[t * c.nc], g[t * c.mc], acc);
    dFdC[i] = acc;
}

// Unbinarity (Sec. 4): grey sub-pixels of the design area, those whose
// final density lies strictly between the two thresholds, given as tanh
// values of the last projection (rho = (1 + t) / 2).  YO_GRAY_BLOCKS blocks
// leave a count each and one wave adds them: an atomic per wave on one counter
// took 30 us for 400x400 sub-pixels.
__global__ __launch_bounds__(1024) void k_gray_count(YoChainBufs c, const float *tproj, float tlo, float thi,
                                                     int *count)
{
    __shared__ int part[16];
    const int n = c.S * c.md * c.S * c.nd;
    int mine = 0;
    for (int i = blockIdx.x * 1024 + threadIdx.x; i < n; i += YO_GRAY_BLOCKS * 1024)
        mine += tproj[i] > tlo && tproj[i] < thi;
    for (int o = 32; o > 0; o >>= 1) mine += __shfl_down(mine, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < 16; ++w) t += part[w];
        count[blockIdx.x] = t;
    }
}

__global__ void k_gray_finish(const int *count, float inv_total, float *out)
{
    int t = threadIdx.x < YO_GRAY_BLOCKS ? count[threadIdx.x] : 0;
    for (int o = 32; o > 0; o >>= 1) t += __shfl_down(t, o);
    if (threadIdx.x == 0) out[0] = (float)t * inv_total;
}

// Adam (Sec. 4, Eqs. (10)-(11)) on the controls: M, V moving averages of the
// gradient and its square; the update divides the bias-corrected first
// moment by the square root of the bias-corrected second plus eps.
// inv1 = 1 / (1 - b1^i), inv2 = 1 / (1 - b2^i) for step i (from the host).
__global__ void k_adam(float *C, const float *G, float *M, float *V, int n, float lr, float b1,
                       float b2, float eps, float inv1, float inv2)
{
    const int i = blockIdx.x * BS + threadIdx.x;
    if (i >= n) return;
    const float g = G[i];
    const float m = fmaf(b1, M[i], (1.0f - b1) * g);
    const float v = fmaf(b2, V[i], (1.0f - b2) * (g * g));
    M[i] = m;
    V[i] = v;
    C[i] = C[i] - lr * ((m * inv1) / (sqrtf(v * inv2) + eps));
}

}  // namespace

hipError_t yo_launch_fill(float *p, size_t n, float v, hipStream_t s)
{
    if (!n) return hipSuccess;
    int blocks = nblk(n);
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill, dim3(blocks), dim3(BS), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t yo_launch_to_ghost(const float *dense, const YoGhost &ghost, int ncomp, int c0, int nc, int nz,
                              int ny, int nx, int ns, hipStream_t s)
{
    const size_t n = (size_t)ncomp * nz * ny * nx;
    if (!n) return hipSuccess;
    int blocks = nblk(n);
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_to_ghost<false>, dim3(blocks), dim3(BS), 0, s, dense, ghost, (unsigned)n, c0, nc,
                       (unsigned)nz, (unsigned)ny, (unsigned)nx, ns, (float4 *)nullptr);
    return hipGetLastError();
}

hipError_t yo_launch_background(const float *dense, float *kappa, float4 *kplane, int nz, int ny, int nx, int ns,
                                int k_lo, int k_hi, const float *mask, float *mask_out, size_t n, hipStream_t s)
{
    const size_t m = (size_t)3 * nz * ny * nx;
    hipLaunchKernelGGL(k_to_ghost<true>, dim3(std::min(nblk(m), 65536)), dim3(BS), 0, s, dense, YoGhost{{kappa}, nullptr},
                       (unsigned)m, 0, 3, (unsigned)nz, (unsigned)ny, (unsigned)nx, ns, kplane);
    hipLaunchKernelGGL(k_kplane, dim3(nz, 16), dim3(BS), 0, s, (const float *)kappa, kplane, ny, nx, ns, k_lo, k_hi, mask,
                       mask_out, n);
    return hipGetLastError();
}

hipError_t yo_launch_from_ghost(const YoGhost &ghost, float *dense, int ncomp, int c0, int nc, int nz,
                                int ny, int nx, int ns, hipStream_t s)
{
    const size_t n = (size_t)ncomp * nz * ny * nx;
    if (!n) return hipSuccess;
    int blocks = nblk(n);
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_from_ghost, dim3(blocks), dim3(BS), 0, s, ghost, dense, (unsigned)n, c0, nc,
                       (unsigned)nz, (unsigned)ny, (unsigned)nx, ns);
    return hipGetLastError();
}

hipError_t yo_launch_finalize(float2 *a, size_t n, float g00, float g01, float g10, float g11,
                              int *bad, hipStream_t s)
{
    if (!n) return hipSuccess;
    int blocks = nblk(n);
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_finalize, dim3(blocks), dim3(BS), 0, s, a, n, g00, g01, g10, g11, bad);
    return hipGetLastError();
}

hipError_t yo_launch_alpha(const YoAlphaArgs &a, hipStream_t s)
{
    const int n = a.n_src * a.n_ports * a.n_freq;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_alpha, dim3(n), dim3(BS), 0, s, a);
    return hipGetLastError();
}

static dim3 morph_grid(int nu, int nv) { return dim3((nu + MTX - 1) / MTX, (nv + MTY - 1) / MTY); }
static size_t morph_lds(const YoChainBufs &c) { return sizeof(float) * ((MTX + 2 * c.mrad) | 1) * (MTY + 2 * c.mrad); }

hipError_t yo_launch_chain_forward(const YoChainBufs &c, const float *C, float beta, float *kappa,
                                   int ny, int ns, int i0, int j0, int k_lo,
                                   int k_hi, hipStream_t s)
{
    const size_t UV = (size_t)c.U * c.V;
    const size_t DD = (size_t)c.S * c.md * c.S * c.nd;
    float *rho = c.n_morph ? c.mcan : c.rho;
    if (yo_filter_by_rows(c.nc, c.S * c.md, c.S * c.nd, c.tmax)) {
        hipLaunchKernelGGL(k_filter_x, dim3(nblk((size_t)c.nc * c.S * c.md)), dim3(BS), 0, s, c, C);
        hipLaunchKernelGGL(k_project<true>, dim3(nblk(UV)), dim3(BS), 0, s, c, C, beta, rho);
    } else {
        hipLaunchKernelGGL(k_project<false>, dim3(nblk(UV)), dim3(BS), 0, s, c, C, beta, rho);
    }
    for (int k = 0; k < c.n_morph; ++k)
        hipLaunchKernelGGL(k_morph, morph_grid(c.U, c.V), dim3(BS), morph_lds(c), s, c, c.mcan + k * UV, c.mcan + (k + 1) * UV,
                           c.msum + k * DD, (int)((c.mdil >> k) & 1u));
    if (c.n_morph)
        hipLaunchKernelGGL(k_morph_project, dim3(nblk(UV)), dim3(BS), 0, s, c, c.mcan + c.n_morph * UV, beta);
    hipLaunchKernelGGL(k_box, dim3(nblk((size_t)3 * c.G0 * c.G1)), dim3(BS), 0, s, c);
    hipLaunchKernelGGL(k_smooth, dim3(nblk((size_t)(c.md + 2) * (c.nd + 2))), dim3(BS), 0, s, c,
                       kappa, ny, ns, i0, j0, k_lo, k_hi);
    return hipGetLastError();
}

hipError_t yo_launch_grad_assemble(const YoGradArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(k_grad, dim3(nblk((size_t)3 * a.box[3] * a.box[4] * a.box[5])), dim3(BS), 0, s, a);
    return hipGetLastError();
}

hipError_t yo_launch_chain_vjp(const YoChainBufs &c, const float *gbox, int z0, int bz, int k_lo, int k_hi,
                               float beta, float *dFdC, hipStream_t s)
{
    const size_t gsz = (size_t)c.G0 * c.G1;
    hipLaunchKernelGGL(k_vjp_pointwise, dim3(nblk(gsz)), dim3(BS), 0, s, c, gbox, z0, bz, k_lo, k_hi);
    hipLaunchKernelGGL(k_vjp_sobel, dim3(nblk(2 * gsz)), dim3(BS), 0, s, c);
    const size_t UV = (size_t)c.U * c.V;
    const size_t DD = (size_t)c.S * c.md * c.S * c.nd;
    float *g = c.n_morph ? c.mg : c.gphi;
    hipLaunchKernelGGL(k_vjp_canvas, dim3(nblk(UV)), dim3(BS), 0, s, c, beta, c.n_morph ? c.tanh2 : c.tanh_, g);
    for (int k = c.n_morph - 1; k >= 0; --k) {
        float *next = k == 0 ? c.gphi : (g == c.mg ? c.mg + DD : c.mg);
        hipLaunchKernelGGL(k_morph_vjp, morph_grid(c.S * c.md, c.S * c.nd), dim3(BS), morph_lds(c), s, c,
                           (const float *)g, (const float *)(c.msum + k * DD), (const float *)(c.mcan + k * UV),
                           (int)((c.mdil >> k) & 1u), k == 0 ? (const float *)c.tanh_ : (const float *)nullptr,
                           beta, next);
        g = next;
    }
    hipLaunchKernelGGL(k_vjp_filter_x, dim3(nblk((size_t)c.S * c.nd * c.mc)), dim3(BS), 0, s, c);
    hipLaunchKernelGGL(k_vjp_filter_y, dim3(nblk((size_t)c.nc * c.mc)), dim3(BS), 0, s, c, dFdC);
    return hipGetLastError();
}

hipError_t yo_launch_unbinarity(const YoChainBufs &c, float tlo, float thi, int *count, float *out,
                                hipStream_t s)
{
    const size_t n = (size_t)c.S * c.md * c.S * c.nd;
    hipLaunchKernelGGL(k_gray_count, dim3(YO_GRAY_BLOCKS), dim3(1024), 0, s, c,
                       (const float *)(c.n_morph ? c.tanh2 : c.tanh_), tlo, thi, count);
    hipLaunchKernelGGL(k_gray_finish, dim3(1), dim3(64), 0, s, count, (float)(1.0 / (double)n), out);
    return hipGetLastError();
}

hipError_t yo_launch_adam(float *C, const float *G, float *M, float *V, int n, float lr, float b1, float b2,
                          float eps, float inv1, float inv2, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_adam, dim3(nblk((size_t)n)), dim3(BS), 0, s, C, G, M, V, n, lr, b1, b2, eps, inv1,
                       inv2);
    return hipGetLastError();
}
