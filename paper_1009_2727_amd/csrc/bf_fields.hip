// bf_fields.hip -- grid kernels of the boosted-frame PIC step for gfx950.
//
//  * k_faraday: B^{n-1/2} -> B^{n+1/2} with the Cole-Karkkainen operator
//    Delta* = (alpha + beta S^1) Delta (Sec. 4.2, 2D: the y neighbours folded into the centre
//    and S^1 a full-cell transverse shift) applied to Friedman's
//    Etilde = (1+theta/4) E^n - 1/2 E^{n-1} + (1/2-theta/4) Ebar (Sec. 4.3, Eq.
//    Faraday_Friedman, indices shifted by one), split-field PML (Appendix II) on the borders.
//  * k_ampere: Yee Ampere E^{n+1} = E^n + dt (curl B^{n+1/2} - J) with the PML split.
//    k_faraday, first in the step, clears the raw current the deposit accumulates into.
//  * k_filter_ampere: the current filter (Sec. 4.1) for unit-stride passes and Ampere in one
//    launch; other stride masks take the line filter of bf_sim3.hip on the grid seen with one y
//    plane, then k_ampere.
//  * k_stations: lab-frame stations (Sec. 3.2).
//  * k_rho: charge density for the Gauss diagnostic.
//
// Each stored cell has one owner thread that writes every component there, so ping-pong targets
// receive a value for every cell (cells outside a component's update range are copied).
#include "bf_kernels.h"

namespace bf {

// One FDX x FDZ tile (bx, by) of stored cells, one thread per cell.  The workgroup stages
// Friedman's Etilde of the tile with a one-cell border in LDS, so it is made once per cell instead
// of once per stencil point; the owner of a cell writes the new Ebar.  Outside a non-periodic axis
// Etilde is 0 and the transverse terms of Delta* vanish with it.  Bound by L2/Infinity Cache
// traffic (18 words per cell): 30 us on 256 x 4096 cells with Friedman, 2.7 TB/s; 52 us with
// Etilde made at every stencil point (72 loads per cell).
constexpr int FDX = FARADAY_TX, FDZ = FARADAY_TZ, FDP = FDX + 2, FDN = FDP * (FDZ + 2);

template <typename R, bool FRIED>
__device__ __forceinline__ void faraday_block(const Geo& g, const FieldSet<R>& f, const PmlTab<R>& pm,
                                              R dt, R a2, R b2, R th, R idx, R idz, int bx, int by)
{
    __shared__ R sT[3][FDN];
    const int x0 = bx * FDX, z0 = by * FDZ;
    for (int q = threadIdx.x; q < FDN; q += 256) {
        const int a = q % FDP, b = q / FDP;
        int i = x0 - 1 + a, k = z0 - 1 + b;
        const bool own = a >= 1 && a <= FDX && b >= 1 && b <= FDZ && i < g.Sx && k < g.Sz;
        if (g.perx) i = i < 0 ? i + g.Sx : (i >= g.Sx ? i % g.Sx : i);
        if (g.perz) k = k < 0 ? k + g.Sz : (k >= g.Sz ? k % g.Sz : k);
        const bool in = i >= 0 && i < g.Sx && k >= 0 && k < g.Sz;
        const long o = in ? gofs(g, i, k) : 0;
#pragma unroll
        for (int c = 0; c < 3; c++) {
            R e = f.E[c][o];
            if constexpr (FRIED) {
                const R eo = f.Eo[c][o], eb = f.Eb[c][o];
                const R ebn = (R(1) - R(0.5) * th) * eo + R(0.5) * th * eb;
                e = (R(1) + R(0.25) * th) * e - R(0.5) * eo + (R(0.5) - R(0.25) * th) * ebn;
                if (own) f.Ebn[c][o] = ebn;
            }
            sT[c][q] = in ? e : R(0);
        }
    }
    __syncthreads();
    const int tx = threadIdx.x % FDX, tz = threadIdx.x / FDX;
    const int i = x0 + tx, k = z0 + tz;
    if (i >= g.Sx || k >= g.Sz) return;
    const long o = gofs(g, i, k);
    const int t = (tz + 1) * FDP + tx + 1;
    // differences towards the half node above the cell, at the cell shifted by s
    auto DX = [&](int c, int s) -> R { return (sT[c][t + s + 1] - sT[c][t + s]) * idx; };
    auto DZ = [&](int c, int s) -> R { return (sT[c][t + s + FDP] - sT[c][t + s]) * idz; };
    // transverse neighbours (outside a non-periodic axis the term is zero)
    const bool zu = g.perz || k + 1 < g.Sz, zd = g.perz || k > 0, xu = g.perx || i + 1 < g.Sx, xd = g.perx || i > 0;
    auto DXs = [&](int c) -> R {   // Delta*_x at (i + 1/2, k)
        R v = a2 * DX(c, 0);
        if (b2 != R(0)) v += b2 * ((zu ? DX(c, FDP) : R(0)) + (zd ? DX(c, -FDP) : R(0)));
        return v;
    };
    auto DZs = [&](int c) -> R {   // Delta*_z at (i, k + 1/2)
        R v = a2 * DZ(c, 0);
        if (b2 != R(0)) v += b2 * ((xu ? DZ(c, 1) : R(0)) + (xd ? DZ(c, -1) : R(0)));
        return v;
    };
    const int xmax_n = smax(g.Sx, g.perx, 0), xmax_h = smax(g.Sx, g.perx, 1);
    const int zmax_n = smax(g.Sz, g.perz, 0), zmax_h = smax(g.Sz, g.perz, 1);
    // B_x (node x, half z): dB/dt = + Delta*_z E_y
    {
        R b = f.B[0][o];
        if (i <= xmax_n && k <= zmax_h) {
            R d = DZs(1);
            b = pm.xi[1][1][k] * b + pm.c[1][1][k] * d;
        }
        f.Bn[0][o] = b;
    }
    // B_z (half x, node z): dB/dt = - Delta*_x E_y
    {
        R b = f.B[2][o];
        if (i <= xmax_h && k <= zmax_n) {
            R d = -DXs(1);
            b = pm.xi[0][1][i] * b + pm.c[0][1][i] * d;
        }
        f.Bn[2][o] = b;
    }
    // B_y (half x, half z): dB/dt = + Delta*_x E_z - Delta*_z E_x, split in the PML
    {
        R b = f.B[1][o];
        if (i <= xmax_h && k <= zmax_h) {
            R dX = DXs(2);
            R dZ = -DZs(0);
            const bool sx = pm.on[0][1][i], sz = pm.on[1][1][k];
            if (!sx && !sz) {
                b = b + dt * (dX + dZ);
            } else {
                R px = f.Byx[o], pz = b - px;
                px = pm.xi[0][1][i] * px + pm.c[0][1][i] * dX;
                pz = pm.xi[1][1][k] * pz + pm.c[1][1][k] * dZ;
                f.Byx[o] = px;
                b = px + pz;
            }
        }
        f.Bn[1][o] = b;
    }
    // the raw current of the previous step is cleared here, at the start of the step, so that
    // it stays readable between steps
    for (int c = 0; c < 3; c++) f.J[c][o] = R(0);
}

template <typename R, bool FRIED>
__global__ void __launch_bounds__(256) k_faraday(Geo g, FieldSet<R> f, PmlTab<R> pm, R dt, R a2,
                                                 R b2, R th, R idx, R idz)
{
    faraday_block<R, FRIED>(g, f, pm, dt, a2, b2, th, idx, idz, blockIdx.x, blockIdx.y);
}

// E^{n+1} of stored cell (i, k) from the current j[3] there
template <typename R>
__device__ __forceinline__ void ampere_cell(const Geo& g, const FieldSet<R>& f, const PmlTab<R>& pm,
                                            R dt, R idx, R idz, int i, int k, const R j[3])
{
    const long o = gofs(g, i, k);
    const int xlo_n = g.perx ? 0 : 1, zlo_n = g.perz ? 0 : 1;
    const int xhi = g.perx ? g.Sx - 1 : g.Sx - 2, zhi = g.perz ? g.Sz - 1 : g.Sz - 2;
    // B one cell below along x and z; 0 beyond a non-periodic edge
    const bool bx = i > 0 || g.perx, bz = k > 0 || g.perz;
    const long oxm = bx ? gofs(g, i > 0 ? i - 1 : g.Sx - 1, k) : o, ozm = bz ? gofs(g, i, k > 0 ? k - 1 : g.Sz - 1) : o;
    const R By = f.Bn[1][o], Byx = bx ? f.Bn[1][oxm] : R(0), Byz = bz ? f.Bn[1][ozm] : R(0);
    const R Bz = f.Bn[2][o], Bzx = bx ? f.Bn[2][oxm] : R(0);
    const R Bx = f.Bn[0][o], Bxz = bz ? f.Bn[0][ozm] : R(0);
    // E_x (half x, node z): dE/dt = - Delta_z B_y - J_x
    {
        R e = f.E[0][o];
        if (i <= xhi && k >= zlo_n && k <= zhi) {
            R d = -(By - Byz) * idz - j[0];
            e = pm.xi[1][0][k] * e + pm.c[1][0][k] * d;
        }
        f.Eo[0][o] = e;
    }
    // E_z (node x, half z): dE/dt = + Delta_x B_y - J_z
    {
        R e = f.E[2][o];
        if (i >= xlo_n && i <= xhi && k <= zhi) {
            R d = (By - Byx) * idx - j[2];
            e = pm.xi[0][0][i] * e + pm.c[0][0][i] * d;
        }
        f.Eo[2][o] = e;
    }
    // E_y (node, node): dE/dt = - Delta_x B_z + Delta_z B_x - J_y, split in the PML
    {
        R e = f.E[1][o];
        if (i >= xlo_n && i <= xhi && k >= zlo_n && k <= zhi) {
            R dX = -(Bz - Bzx) * idx - j[1];
            R dZ = (Bx - Bxz) * idz;
            const bool sx = pm.on[0][0][i], sz = pm.on[1][0][k];
            if (!sx && !sz) {
                e = e + dt * (dX + dZ);
            } else {
                R px = f.Eyx[o], pz = e - px;
                px = pm.xi[0][0][i] * px + pm.c[0][0][i] * dX;
                pz = pm.xi[1][0][k] * pz + pm.c[1][0][k] * dZ;
                f.Eyx[o] = px;
                e = px + pz;
            }
        }
        f.Eo[1][o] = e;
    }
}

template <typename R>
__device__ __forceinline__ void ampere_block(const Geo& g, const FieldSet<R>& f, const PmlTab<R>& pm,
                                             R dt, R idx, R idz, int bx, int by)
{
    const int i = bx * 64 + (threadIdx.x & 63);
    const int k = by * 4 + (threadIdx.x >> 6);
    if (i >= g.Sx || k >= g.Sz) return;
    const long o = gofs(g, i, k);
    const R j[3] = {f.Jf[0][o], f.Jf[1][o], f.Jf[2][o]};
    ampere_cell<R>(g, f, pm, dt, idx, idz, i, k, j);
}

template <typename R>
__global__ void __launch_bounds__(256) k_ampere(Geo g, FieldSet<R> f, PmlTab<R> pm, R dt, R idx,
                                                R idz)
{
    ampere_block<R>(g, f, pm, dt, idx, idz, blockIdx.x, blockIdx.y);
}

// ---- current filter and Ampere in one launch ----------------------------------------------
// A sequence of unit-stride passes along an axis is one symmetric stencil of 2 RC + 1 taps; the
// zeros held outside a component's range after every pass equal that stencil applied to the
// line continued oddly about the positions just outside (filt_pos).  A workgroup owns a TX x TZ
// tile of stored cells: it stages the three raw currents with a halo of RC cells, applies the x
// stencil into a second LDS tile, the z stencil into registers, writes the filtered current and
// advances E with it.  A component's last half node on its own non-periodic axis is copied along
// that axis: J_x's from the raw column, J_z's as the x stencil of the raw row.
// Bound by the latency of its loads on small grids and by L2/Infinity Cache traffic on large
// ones.  It replaces two launches of the line filter (a barrier per pass, one intermediate in
// HBM) and k_ampere: 36 us against 68 us on 256 x 4096 cells with reach 5, 10 us against 34 us
// on 75 x 1691.
// The 64 x 16 tile reads each current 1.9 times (RC = 5), the 32 x 8 tile 3 times; the small one
// is taken where the large one would leave CUs idle.
__device__ __forceinline__ int filt_pos(int p, int S, int hi, int per, int& sg)
{
    sg = 1;
    if (per) {
        p %= S;
        return p < 0 ? p + S : p;
    }
    if (p >= 0 && p <= hi) return p;
    const int q = p < 0 ? -2 - p : 2 * (hi + 1) - p;
    sg = (p == -1 || p == hi + 1 || q < 0 || q > hi) ? 0 : -1;
    return sg ? q : 0;
}

template <int RC, int TX, int TZ, typename R>
__global__ void __launch_bounds__(256) k_filter_ampere(Geo g, FieldSet<R> f, PmlTab<R> pm, Stencil2 st, R dt, R idx,
                                                       R idz)
{
    constexpr int AX = TX + 2 * RC, AZ = TZ + 2 * RC, NQ = TX * TZ / 256;
    __shared__ R sA[3][AZ * AX];
    __shared__ R sB[3][AZ * TX];
    __shared__ int ci[2][AX];              // column of each staged position under the continuation
    __shared__ long ri[2][AZ];             // offset of its row
    __shared__ R cs[2][AX], rs[2][AZ];     // ... and its sign; [0]: the component that ends a half node early
    const int x0 = (int)blockIdx.x * TX, z0 = (int)blockIdx.y * TZ;
    // last filtered position of J_x, J_y, J_z along x and z
    const int hx[3] = {g.perx ? g.Sx - 1 : g.Sx - 2, g.Sx - 1, g.Sx - 1};
    const int hz[3] = {g.Sz - 1, g.Sz - 1, g.perz ? g.Sz - 1 : g.Sz - 2};
    R c[RC + 1];
#pragma unroll
    for (int m = 0; m <= RC; m++) c[m] = (R)st.c[m];
    for (int q = threadIdx.x; q < 2 * (AX + AZ); q += 256) {
        int sg;
        if (q < 2 * AX) {
            const int h = q / AX, a = q % AX;
            ci[h][a] = filt_pos(x0 - RC + a, g.Sx, hx[h], g.perx, sg);
            cs[h][a] = (R)sg;
        } else {
            const int h = (q - 2 * AX) / AZ, b = (q - 2 * AX) % AZ;
            ri[h][b] = gofs(g, 0, filt_pos(z0 - RC + b, g.Sz, hz[2 - 2 * h], g.perz, sg));
            rs[h][b] = (R)sg;
        }
    }
    __syncthreads();
    // component 0 ends a half node early along x, component 2 along z
#pragma unroll 4
    for (int q = threadIdx.x; q < AZ * AX; q += 256) {
        const int a = q % AX, b = q / AX;
        const int i0 = ci[0][a], i1 = ci[1][a];
        const long k0 = ri[0][b], k1 = ri[1][b];
        const R x0s = cs[0][a], x1s = cs[1][a], z0s = rs[0][b], z1s = rs[1][b];
        sA[0][q] = x0s * z1s * f.J[0][k1 + i0];
        sA[1][q] = x1s * z1s * f.J[1][k1 + i1];
        sA[2][q] = x1s * z0s * f.J[2][k0 + i1];
    }
    __syncthreads();
    for (int q = threadIdx.x; q < AZ * TX; q += 256) {
        const int a = q % TX, b = q / TX;
#pragma unroll
        for (int m = 0; m < 3; m++) {
            const R* r = sA[m] + b * AX + a + RC;
            R v = R(0);          // outermost taps first: the small terms before the large ones
#pragma unroll
            for (int t = RC; t >= 1; t--) v += c[t] * (r[-t] + r[t]);
            v += c[0] * r[0];
            if (m == 0 && x0 + a == hx[0] + 1) {   // the copied half node of J_x
                v = x0 + a < g.Sx ? rs[1][b] * f.J[0][ri[1][b] + x0 + a] : R(0);
            }
            sB[m][q] = v;
        }
    }
    __syncthreads();
    const int tx = threadIdx.x % TX, tz = threadIdx.x / TX;
#pragma unroll
    for (int n = 0; n < NQ; n++) {
        const int i = x0 + tx, b = tz + n * (256 / TX), k = z0 + b;
        if (i >= g.Sx || k >= g.Sz) continue;
        R j[3];
#pragma unroll
        for (int m = 0; m < 3; m++) {
            const R* r = sB[m] + (b + RC) * TX + tx;
            R v = R(0);
#pragma unroll
            for (int t = RC; t >= 1; t--) v += c[t] * (r[-t * TX] + r[t * TX]);
            v += c[0] * r[0];
            j[m] = v;
        }
        if (k == hz[2] + 1) {                      // the copied half node of J_z
            R v = R(0);
            for (int t = -RC; t <= RC; t++) {
                int sx;
                const int q = filt_pos(i + t, g.Sx, hx[2], g.perx, sx);
                if (sx) v += c[t < 0 ? -t : t] * (R)sx * f.J[2][gofs(g, q, k)];
            }
            j[2] = v;
        }
        const long o = gofs(g, i, k);
#pragma unroll
        for (int m = 0; m < 3; m++) f.Jf[m][o] = j[m];
        ampere_cell<R>(g, f, pm, dt, idx, idz, i, k, j);
    }
}

// ---- momentum-conserving gather: fields to the nodes -------------------------------------
// Each component of E^n and of B^n = (B^{n-1/2} + B^{n+1/2}) / 2 becomes, at node (i, k), the
// mean of its values at the Yee locations around the node along its staggered axes: E_x (i -+
// 1/2, k), E_z (i, k -+ 1/2), B_x (i, k -+ 1/2), B_y the four (i -+ 1/2, k -+ 1/2), B_z (i -+ 1/2,
// k); E_y sits on the node.  Locations beyond a non-periodic edge read 0.
template <typename R>
__global__ void __launch_bounds__(256) k_nodes(Geo g, FieldSet<R> f)
{
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    const int k = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (i >= g.Sx || k >= g.Sz) return;
    const int il = swrap(i - 1, g.Sx, g.perx), kl = swrap(k - 1, g.Sz, g.perz);
    auto at = [&](const R* a, int ii, int kk) { return (ii < 0 || kk < 0) ? R(0) : a[gofs(g, ii, kk)]; };
    auto bn = [&](int c, int ii, int kk) { return R(0.5) * (at(f.B[c], ii, kk) + at(f.Bn[c], ii, kk)); };
    const long o = gofs(g, i, k);
    f.G[0][o] = R(0.5) * (at(f.E[0], il, k) + at(f.E[0], i, k));
    f.G[1][o] = f.E[1][o];
    f.G[2][o] = R(0.5) * (at(f.E[2], i, kl) + at(f.E[2], i, k));
    f.G[3][o] = R(0.5) * (bn(0, i, kl) + bn(0, i, k));
    f.G[4][o] = R(0.25) * ((bn(1, il, kl) + bn(1, i, kl)) + (bn(1, il, k) + bn(1, i, k)));
    f.G[5][o] = R(0.5) * (bn(2, il, k) + bn(2, i, k));
}

template <typename R>
void launch_nodes(const Geo& g, const FieldSet<R>& f, hipStream_t s)
{
    dim3 grid((g.Sx + 63) / 64, (g.Sz + 3) / 4);
    hipLaunchKernelGGL((k_nodes<R>), grid, dim3(256), 0, s, g, f);
}

// ---- batched runs: one launch per phase over the cell blocks of all runs ---------------------
template <typename R>
__global__ void __launch_bounds__(256) k_faraday_batch(const FaradayDesc<R>* __restrict__ d, QueueRef q)
{
    int r = 0;
    for (int k = 0;; k++) {
        const int it = stride_item(q, k);
        if (it < 0) return;
        r = run_of(q, it, r);
        const FaradayDesc<R>& D = d[r];
        const int local = it - q.off[r];
        if (D.fried)
            faraday_block<R, true>(D.g, D.f, D.pm, D.dt, D.a2, D.b2, D.th, D.idx, D.idz, local % D.gx,
                                   local / D.gx);
        else
            faraday_block<R, false>(D.g, D.f, D.pm, D.dt, D.a2, D.b2, D.th, D.idx, D.idz, local % D.gx,
                                    local / D.gx);
    }
}

template <typename R>
__global__ void __launch_bounds__(256) k_ampere_batch(const AmpereDesc<R>* __restrict__ d, QueueRef q)
{
    int r = 0;
    for (int k = 0;; k++) {
        const int it = stride_item(q, k);
        if (it < 0) return;
        r = run_of(q, it, r);
        const AmpereDesc<R>& D = d[r];
        const int local = it - q.off[r];
        ampere_block<R>(D.g, D.f, D.pm, D.dt, D.idx, D.idz, local % D.gx, local / D.gx);
    }
}


// ---- stations ----------------------------------------------------------------------------
template <typename R>
__device__ double bilin(const Geo& g, const R* a, int hx, int hz, double xc, double zc)
{
    double xs = xc - 0.5 * hx, zs = zc - 0.5 * hz;
    int jx = (int)floor(xs), jz = (int)floor(zs);
    double fx = xs - jx, fz = zs - jz;
    double v = 0.0;
    for (int p = 0; p < 2; p++)
        for (int q = 0; q < 2; q++) {
            int i = swrap(jx + p + g.Px, g.Sx, g.perx), k = swrap(jz + q + g.Pz, g.Sz, g.perz);
            if (i < 0 || k < 0) continue;
            v += (p ? fx : 1.0 - fx) * (q ? fz : 1.0 - fz) * (double)a[gofs(g, i, k)];
        }
    return v;
}

template <typename R>
__global__ void k_stations(Geo g, FieldSet<R> f, StationParams sp, double* rec, int* counts)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= sp.n) return;
    double zb = sp.zlab[q] / sp.gamma - sp.beta * sp.t;     // boosted position
    double zc = (zb - sp.shift * sp.dz_um) / sp.dz_um;     // window cells
    int n = counts[q];
    if (zc < 0.0 || zc >= (double)g.Nz || n >= sp.cap) return;
    double xc = sp.xc;
    double E0 = bilin(g, f.E[0], 1, 0, xc, zc), E1 = bilin(g, f.E[1], 0, 0, xc, zc),
           E2 = bilin(g, f.E[2], 0, 1, xc, zc);
    double B0 = 0.5 * (bilin(g, f.B[0], 0, 1, xc, zc) + bilin(g, f.Bn[0], 0, 1, xc, zc));
    double B1 = 0.5 * (bilin(g, f.B[1], 1, 1, xc, zc) + bilin(g, f.Bn[1], 1, 1, xc, zc));
    double B2 = 0.5 * (bilin(g, f.B[2], 1, 0, xc, zc) + bilin(g, f.Bn[2], 1, 0, xc, zc));
    double ga = sp.gamma, be = sp.beta;
    double* r = rec + ((long)q * sp.cap + n) * 7;
    r[0] = ga * (sp.t + be * zb);
    r[1] = ga * (E0 + be * B1);
    r[2] = ga * (E1 - be * B0);
    r[3] = E2;
    r[4] = ga * (B0 - be * E1);
    r[5] = ga * (B1 + be * E0);
    r[6] = B2;
    counts[q] = n + 1;
}

// ---- charge density (diagnostic, FP64) -------------------------------------------------------
__device__ __forceinline__ double s3d(double r)
{
    double a = fabs(r);
    if (a < 1.0) return 2.0 / 3.0 - a * a + 0.5 * a * a * a;
    if (a < 2.0) { double b = 2.0 - a; return b * b * b / 6.0; }
    return 0.0;
}

__device__ void rho_add(const Geo& g, double* rho, double qw, double x, double z)
{
    int i0 = (int)floor(x), k0 = (int)floor(z);
    for (int a = -1; a <= 2; a++) {
        double sx = s3d(x - (i0 + a));
        int si = swrap(i0 + a + g.Px, g.Sx, g.perx);
        if (si < 0 || sx == 0.0) continue;
        for (int b = -1; b <= 2; b++) {
            double sz = s3d(z - (k0 + b));
            int sk = swrap(k0 + b + g.Pz, g.Sz, g.perz);
            if (sk < 0 || sz == 0.0) continue;
            atomicAdd(&rho[(long)sk * g.Sx + si], qw * sx * sz);
        }
    }
}

template <typename R>
__global__ void k_rho(Geo g, ElectronArrays<R> e, int ne, IonArrays<R> ion, int ni, double zsh,
                      const double* xm, int na, double xa_home0, double za, double aw,
                      double inv_cell, double* rho)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < ne) {
        double w = (double)e.w[p];
        if (w != 0.0) rho_add(g, rho, -w * inv_cell, e.x[p], e.z[p]);
    } else if (p < ne + ni) {
        int q = p - ne;
        double w = (double)ion.w[q];
        if (w != 0.0) rho_add(g, rho, w * inv_cell, ion.x[q], ion.z0[q] - zsh);
    } else if (p < ne + ni + na) {
        int q = p - ne - ni;
        rho_add(g, rho, -aw * inv_cell, xm[q], za);
        rho_add(g, rho, aw * inv_cell, xa_home0 + q, za);
    }
}

__global__ void k_fill_int(int* p, int n, int v)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ---- launchers ------------------------------------------------------------------------------
template <typename R>
void launch_faraday_batch(const FaradayDesc<R>* d, const QueueRef& q, int nblocks, hipStream_t s)
{
    if (q.total > 0)
        hipLaunchKernelGGL((k_faraday_batch<R>), dim3(nblocks), dim3(256), 0, s, d, q);
}

template <typename R>
void launch_ampere_batch(const AmpereDesc<R>* d, const QueueRef& q, int nblocks, hipStream_t s)
{
    if (q.total > 0)
        hipLaunchKernelGGL((k_ampere_batch<R>), dim3(nblocks), dim3(256), 0, s, d, q);
}



template <typename R>
void launch_faraday(const Geo& g, const FieldSet<R>& f, const PmlTab<R>& pm, const SolverCoef& c,
                    hipStream_t s)
{
    dim3 grid((g.Sx + FDX - 1) / FDX, (g.Sz + FDZ - 1) / FDZ);
    if (c.theta > 0.0)
        hipLaunchKernelGGL((k_faraday<R, true>), grid, dim3(256), 0, s, g, f, pm, (R)c.dt, (R)c.a2,
                           (R)c.b2, (R)c.theta, (R)c.idx, (R)c.idz);
    else
        hipLaunchKernelGGL((k_faraday<R, false>), grid, dim3(256), 0, s, g, f, pm, (R)c.dt, (R)c.a2,
                           (R)c.b2, (R)c.theta, (R)c.idx, (R)c.idz);
}

template <typename R>
void launch_ampere(const Geo& g, const FieldSet<R>& f, const PmlTab<R>& pm, const SolverCoef& c,
                   hipStream_t s)
{
    dim3 grid((g.Sx + 63) / 64, (g.Sz + 3) / 4);
    hipLaunchKernelGGL((k_ampere<R>), grid, dim3(256), 0, s, g, f, pm, (R)c.dt, (R)c.idx, (R)c.idz);
}

template <int RC, int TX, int TZ, typename R>
static void filter_ampere(const Geo& g, const FieldSet<R>& f, const PmlTab<R>& pm, const Stencil2& st,
                          const SolverCoef& c, hipStream_t s)
{
    const dim3 grid((g.Sx + TX - 1) / TX, (g.Sz + TZ - 1) / TZ);
    hipLaunchKernelGGL((k_filter_ampere<RC, TX, TZ, R>), grid, dim3(256), 0, s, g, f, pm, st, (R)c.dt, (R)c.idx,
                       (R)c.idz);
}

template <int RC, typename R>
static void filter_ampere(const Geo& g, const FieldSet<R>& f, const PmlTab<R>& pm, const Stencil2& st,
                          const SolverCoef& c, hipStream_t s)
{
    // the large tile from two workgroups per CU on
    if ((long)((g.Sx + 63) / 64) * ((g.Sz + 15) / 16) >= 512) filter_ampere<RC, 64, 16, R>(g, f, pm, st, c, s);
    else filter_ampere<RC, 32, 8, R>(g, f, pm, st, c, s);
}

template <typename R>
void launch_filter_ampere(const Geo& g, const FieldSet<R>& f, const PmlTab<R>& pm, const Stencil2& st,
                          const SolverCoef& c, hipStream_t s)
{
    switch (st.reach) {
    case 1: filter_ampere<1, R>(g, f, pm, st, c, s); break;
    case 2: filter_ampere<2, R>(g, f, pm, st, c, s); break;
    case 3: filter_ampere<3, R>(g, f, pm, st, c, s); break;
    case 4: filter_ampere<4, R>(g, f, pm, st, c, s); break;
    case 5: filter_ampere<5, R>(g, f, pm, st, c, s); break;
    case 6: filter_ampere<6, R>(g, f, pm, st, c, s); break;
    }
}

template <typename R>
void launch_stations(const Geo& g, const FieldSet<R>& f, const StationParams& sp, double* rec,
                     int* counts, hipStream_t s)
{
    if (sp.n <= 0) return;
    hipLaunchKernelGGL((k_stations<R>), dim3(1), dim3(64), 0, s, g, f, sp, rec, counts);
}

template <typename R>
void launch_rho(const Geo& g, const ElectronArrays<R>& e, int ne, const IonArrays<R>& ion, int ni,
                double zsh, const double* xm, int na, double xa_home0, double za, double aw,
                double inv_cell, double* rho, hipStream_t s)
{
    int n = ne + ni + na;
    if (n <= 0) return;
    hipLaunchKernelGGL((k_rho<R>), dim3((n + 255) / 256), dim3(256), 0, s, g, e, ne, ion, ni, zsh, xm,
                       na, xa_home0, za, aw, inv_cell, rho);
}

__global__ void k_rho_beam(Geo g, BeamArrays b, int n, double inv_cell, double* rho)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n || b.state[p] == 2) return;
    const double x = b.x[p], z = b.z[p];
    if (!g.perx && (x < 0.0 || x >= (double)g.Nx)) return;
    if (!g.perz && (z < 0.0 || z >= (double)g.Nz)) return;
    rho_add(g, rho, -b.w[p] * inv_cell, x, z);
}

void launch_rho_beam(const Geo& g, const BeamArrays& b, int n, double inv_cell, double* rho, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_rho_beam, dim3((n + 255) / 256), dim3(256), 0, s, g, b, n, inv_cell, rho);
}

void launch_fill_int(int* p, int n, int v, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_fill_int, dim3((n + 255) / 256), dim3(256), 0, s, p, n, v);
}

#define BF_INST(R)                                                                                 \
    template void launch_faraday<R>(const Geo&, const FieldSet<R>&, const PmlTab<R>&,              \
                                    const SolverCoef&, hipStream_t);                               \
    template void launch_nodes<R>(const Geo&, const FieldSet<R>&, hipStream_t);                       \
    template void launch_ampere<R>(const Geo&, const FieldSet<R>&, const PmlTab<R>&,               \
                                   const SolverCoef&, hipStream_t);                                \
    template void launch_filter_ampere<R>(const Geo&, const FieldSet<R>&, const PmlTab<R>&,        \
                                          const Stencil2&, const SolverCoef&, hipStream_t);        \
    template void launch_faraday_batch<R>(const FaradayDesc<R>*, const QueueRef&, int, hipStream_t); \
    template void launch_ampere_batch<R>(const AmpereDesc<R>*, const QueueRef&, int, hipStream_t);   \
    template void launch_stations<R>(const Geo&, const FieldSet<R>&, const StationParams&,         \
                                     double*, int*, hipStream_t);                                  \
    template void launch_rho<R>(const Geo&, const ElectronArrays<R>&, int, const IonArrays<R>&,    \
                                int, double, const double*, int, double, double, double, double,   \
                                double*, hipStream_t);
BF_INST(float)
BF_INST(double)

}  // namespace bf
