// One or more time steps of small and middle-sized lattices, all rows of a tile at once.
//
// The update is k_step's (lb_kernels.hip): pull, density, 9-point stencils, collision
// (lb_collide.h), with the same expressions in the same order, so that the results are bitwise
// those of k_step and k_step2.  Those kernels march a strip of lanes down the rows of a tile, which
// is the cheapest in reads and registers once a launch has several workgroups for every CU, but
// makes a chain of one or two collisions and barriers per row: on a lattice that cannot fill the
// chip, the chain is all the time there is.  Here every node of a tile has its own lane: a wave
// holds 64 columns of one row (so the row's descriptors stay in scalar registers), a workgroup up
// to 16 rows, and the only chain is load, density, barrier, collision.
//
// NS steps per launch.  A tile whose last step stores w x h nodes collides (w + 2 H) x (h + 2 H)
// nodes in the first, H = 2 (NS - 1): each step loses two nodes at each edge (the stencil's and the
// pull's neighbour).  The first step also needs the densities of the ring around its nodes, which a
// few of the waves pull as well.  Between steps the post-collision populations pass through LDS.
// Replicas whose row fits 64 columns are tiled by whole rows (columns wrap inside the tile, no loss
// in x).  Tiles of 128 or 256 columns were slower at every size.
//
// What bounds it: below ~2^17 nodes the chain of a launch (~2 us to the first collision, then 1.5 us
// a step in FP32, 3 us in FP64: the collision's own dependent instructions); from ~2^19 nodes VALU
// issue, the lost rows included (2048 x 400 in FP32: 24.4 us for 10.3 M wave instructions per two
// steps).  Measured, us per step, k_step2's 16-row tiles before and these after: 64^2 FP64 41 / 3.6,
// 128^2 FP32 24 / 2.6, 512^2 FP32 23.6 / 6.0, 2048 x 400 FP32 24.8 / 12.2, FP64 45 / 23.6,
// 1500 x 1101 FP32 30.6 / 21.1.

#include "lb_collide.h"
#include "lb_internal.h"
#include "lb_rng.h"

namespace lbf {

constexpr int TX = 64;        // columns of a tile: a wave
constexpr int DW = TX + 2;    // slots of a density row

// CACHED: stores go through the caches (the next step's reads find them there) instead of carrying
// the nontemporal policy.
// Waves per SIMD: with the launch bound alone the compiler aims at one workgroup of 1024 and parks values
// in the accumulation registers; asked for 8 (6 in FP64) it fits 54 to 56 vector registers without them, 18
// instructions less per node (2048 x 400 12.55 -> 12.18 us per step, 1500 x 1101 21.38 -> 21.10).
template <typename S, typename R, bool PLAIN, bool CN, int NS, bool CACHED>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(sizeof(S) == 8 ? 6 : 8)))
    k_tile(const RepDesc *__restrict__ reps, const unsigned long long *__restrict__ tdev, const S *__restrict__ fin,
           S *__restrict__ fout, const Tile *__restrict__ table, int nrep, int ntiles, int toff,
           const S *__restrict__ xi, long long xi_plane, unsigned *__restrict__ flags)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int H = 2 * (NS - 1);
    constexpr unsigned ES = sizeof(S);
    const int lx = threadIdx.x & 63;
    const int ly = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);   // row: uniform per wave
    const int TY = blockDim.x >> 6;

    // consecutive tiles on one XCD (workgroup i runs on XCD i mod 8)
    const int per = (ntiles + 7) >> 3;
    const int b = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
    if (b >= ntiles) return;
    // the replica whose tiles include b (table[r].x0: index of its first tile)
    int rep = 0, first = 0;
    if (nrep > 1) {
        int hi = nrep - 1;
        while (rep < hi) {
            const int mid = (rep + hi + 1) >> 1;
            if (table[mid].x0 <= b) rep = mid;
            else hi = mid - 1;
        }
        first = table[rep].x0;
    }
    const RepDesc &d = reps[rep];
    const Consts<R> &c = consts<R>(d);
    const VConsts<R> vk = vconsts<R>(c);
    const int nx = d.nx, ny = d.ny;
    const unsigned long long t = tdev[0] + (unsigned long long)toff;
    const bool whole = nx <= TX;
    const int wout = whole ? nx : TX - 2 * H, hout = TY - 2 * H;
    const int strips = whole ? 1 : (nx + (TX - 2 * H) - 1) / (TX - 2 * H);
    const int band = (b - first) / strips, strip = (b - first) - band * strips;
    const int x0 = strip * wout, y0 = band * hout;
    const int h = min(hout, ny - y0);      // stored rows
    const int rows = h + 2 * H;            // collided rows of the first step, [0, rows) of the tile
    const unsigned nxb = (unsigned)nx * ES, rowb = 9u * nxb;
    const S *__restrict__ P = fin + d.off;
    S *__restrict__ Qo = fout + d.off;

    auto wrapx = [nx](int v) { return v < 0 ? v + nx : (v >= nx ? v - nx : v); };
    auto wrapy = [ny](int v) {   // uniform; more than one period only for lattices of a few rows
        while (v < 0) v += ny;
        while (v >= ny) v -= ny;
        return v;
    };
    auto row_of = [&](int y) { return row_rsrc(P + (unsigned long long)(unsigned)y * (9ull * nx), rowb); };

    // the lane's column (lanes past a whole row repeat column 0 and never store)
    const int xw = whole ? (lx < nx ? lx : 0) : wrapx(x0 - H + lx);
    const unsigned c0 = (unsigned)xw * ES, cm = (unsigned)(xw == 0 ? nx - 1 : xw - 1) * ES,
                   cp = (unsigned)(xw == nx - 1 ? 0 : xw + 1) * ES;
    // populations pulled at row yy, this lane's column
    auto pull = [&](int yy, R f[Q]) {
        const int y = wrapy(yy);
        const auto rm = row_of(y == 0 ? ny - 1 : y - 1), rz = row_of(y), rp = row_of(y == ny - 1 ? 0 : y + 1);
        f[0] = (R)bld<S>(rz, c0, 0);
        f[1] = (R)bld<S>(rz, cm, nxb);
        f[2] = (R)bld<S>(rm, c0, 2 * nxb);
        f[3] = (R)bld<S>(rz, cp, 3 * nxb);
        f[4] = (R)bld<S>(rp, c0, 4 * nxb);
        f[5] = (R)bld<S>(rm, cm, 5 * nxb);
        f[6] = (R)bld<S>(rm, cp, 6 * nxb);
        f[7] = (R)bld<S>(rp, cp, 7 * nxb);
        f[8] = (R)bld<S>(rp, cm, 8 * nxb);
    };

    // LDS: densities of rows -1 .. rows (row r at (r + 1) DW, column x at x + 1), then, between
    // steps, populations 1..8 of the tile's rows (population i at (i - 1) TY TX)
    R *D = reinterpret_cast<R *>(smem_raw);
    S *F = reinterpret_cast<S *>(D + (TY + 2) * DW);
    const int xl = whole ? (lx == 0 ? nx - 1 : lx - 1) : lx - 1;   // neighbour columns inside the tile
    const int xr = whole ? (lx == nx - 1 ? 0 : lx + 1) : lx + 1;
    const bool lane_on = !whole || lx < nx;
    // a density into row r; in a whole row the end columns also fill the slots beyond the other end
    auto put = [&](int r, R v) {
        R *row = D + (r + 1) * DW + 1;
        if (lane_on) row[lx] = v;
        if (whole) {
            if (lx == 0) row[nx] = v;
            if (lx == nx - 1) row[-1] = v;
        }
    };

    const bool live = ly < rows;           // uniform per wave
    const int yb = y0 - H;                 // lattice row of the tile's row 0
    R f[Q];
    {
        R g[Q], e[Q];
        // the ring: rows -1 and `rows` by the waves of rows 0 and rows - 1, and (strips) columns -1
        // and TX by the lanes of one wave of row 1 (row 0 when it is the only one)
        const bool top = live && ly == 0, bottom = live && ly == rows - 1;
        const bool sides = !whole && ly == (rows > 1 ? 1 : 0);
        const int sr = (lx >> 1) - 1;
        const bool side_on = sides && sr <= rows;
        if (live) pull(yb + ly, f);
        if (top || bottom) pull(top ? yb - 1 : yb + rows, g);
        if (side_on) {
            const int sx = wrapx(lx & 1 ? x0 - H + TX : x0 - H - 1);
            const int yz = wrapy(yb + sr), ym = yz == 0 ? ny - 1 : yz - 1, yp = yz == ny - 1 ? 0 : yz + 1;
            const long long pitch = 9ll * nx;
            const int sm = sx == 0 ? nx - 1 : sx - 1, sp = sx == nx - 1 ? 0 : sx + 1;
            const S *Pm = P + ym * pitch, *Pz = P + yz * pitch, *Pp = P + yp * pitch;
            e[0] = (R)Pz[sx];
            e[1] = (R)Pz[nx + sm];
            e[2] = (R)Pm[2 * nx + sx];
            e[3] = (R)Pz[3 * nx + sp];
            e[4] = (R)Pp[4 * nx + sx];
            e[5] = (R)Pm[5 * nx + sm];
            e[6] = (R)Pm[6 * nx + sp];
            e[7] = (R)Pp[7 * nx + sp];
            e[8] = (R)Pp[8 * nx + sm];
        }
        if (live) put(ly, dens9<R, PLAIN>(f, c));
        if (top || bottom) put(top ? -1 : rows, dens9<R, PLAIN>(g, c));
        if (side_on) D[(sr + 1) * DW + (lx & 1 ? TX + 1 : 0)] = dens9<R, PLAIN>(e, c);
        if (rows == 1 && live) {   // the only row pulls both ring rows
            pull(yb + rows, g);
            put(rows, dens9<R, PLAIN>(g, c));
        }
    }
    __syncthreads();

    unsigned st = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        // step t + s collides rows [2 s, rows - 2 s)
        const bool on = ly >= 2 * s && ly < rows - 2 * s;
        if (on) {
            const R *Dz = D + (ly + 1) * DW + 1 + lx, *Dp = Dz + DW, *Dm = Dz - DW;
            R lap, gx, gy;
            stencil9<R>(Dz[0], Dz[1], Dz[-1], Dp[0], Dp[1], Dp[-1], Dm[0], Dm[1], Dm[-1], lap, gx, gy);
            if (PLAIN) {
#pragma unroll
                for (int i = 0; i < Q; ++i) f[i] -= c.sub[i];
            }
            const unsigned y = (unsigned)wrapy(yb + ly);
            R xi4 = 0, xi9 = 0;
            if (CN && d.noise == 2) {
                const S *__restrict__ xp = xi + s * xi_plane + 2 * (d.xi_off + (long long)y * nx + xw);
                xi4 = (R)xp[0];
                xi9 = (R)xp[1];
            }
            st |= collide<R, CN>(f, lap, gx, gy, c, vk, d.noise, y * (unsigned)nx + (unsigned)xw, d.rep_id, t + s,
                                 d.seed_lo, d.seed_hi, xi4, xi9);
#pragma unroll
            for (int i = 0; i < Q; ++i) f[i] = (R)(S)(PLAIN ? add_rn<R>(f[i], c.sub[i]) : f[i]);
        }
        if (s == NS - 1) {
            const int xs = x0 - H + lx;
            const bool store = on && (whole ? lx < nx : lx >= H && lx < TX - H && xs < nx);
            if (on) {
                const auto W = row_rsrc(Qo + (unsigned long long)(unsigned)(y0 + ly - H) * (9ull * nx), rowb);
                if (store) {
#pragma unroll
                    for (int i = 0; i < Q; ++i) bst<S, CACHED>(W, c0, i * nxb, (S)f[i]);
                    if (st) atomicOr(flags, st);
                }
            }
        } else {
            const int plane = TY * TX;
            if (on) {
                S *Fo = F + ly * TX + lx;
#pragma unroll
                for (int i = 1; i < Q; ++i) Fo[(i - 1) * plane] = (S)f[i];
            }
            __syncthreads();
            // pull of step t + s + 1, rows [2 s + 1, rows - 2 s - 1)
            const bool pl = ly >= 2 * s + 1 && ly < rows - 2 * s - 1;
            if (pl) {
                const S *Fz = F + ly * TX, *Fm = Fz - TX, *Fp = Fz + TX;
                f[1] = (R)Fz[xl];
                f[2] = (R)Fm[plane + lx];
                f[3] = (R)Fz[2 * plane + xr];
                f[4] = (R)Fp[3 * plane + lx];
                f[5] = (R)Fm[4 * plane + xl];
                f[6] = (R)Fm[5 * plane + xr];
                f[7] = (R)Fp[6 * plane + xr];
                f[8] = (R)Fp[7 * plane + xl];
                put(ly, dens9<R, PLAIN>(f, c));
            }
            __syncthreads();
        }
    }
}

size_t tile_lds_bytes(int precision, int ns, int ty)
{
    const size_t e = precision == 0 ? 8 : 4;
    return e * ((size_t)(ty + 2) * DW + (ns > 1 ? (size_t)8 * ty * TX : 0));
}

template <typename S, typename R, bool PLAIN, bool CN, int NS> static hipError_t set_tile_limit()
{
    const int bytes = (int)tile_lds_bytes(sizeof(S) == 8 ? 0 : 1, NS, TILE_MAX_TY);
    hipError_t e = hipFuncSetAttribute((const void *)k_tile<S, R, PLAIN, CN, NS, false>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)k_tile<S, R, PLAIN, CN, NS, true>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    return e;
}

// only the FP64 variants of two steps can need more than 64 KB
hipError_t set_tile_lds_limit()
{
    hipError_t e = set_tile_limit<double, double, false, false, 2>();
    return e == hipSuccess ? set_tile_limit<double, double, false, true, 2>() : e;
}

long long tile_count(int nx, int ny, int ns, int ty)
{
    const int hx = 2 * (ns - 1), w = nx <= TX ? nx : TX - 2 * hx, h = ty - 2 * hx;
    return (long long)((nx + w - 1) / w) * ((ny + h - 1) / h);
}

template <typename S, typename R, bool PLAIN, bool CN, int NS> static void launch_tile_t(const TileLaunch &a, hipStream_t s)
{
    const size_t lds = tile_lds_bytes(sizeof(S) == 8 ? 0 : 1, NS, a.ty);
    const dim3 grid((unsigned)((a.ntiles + 7) / 8 * 8)), block(TX * a.ty);
    if (a.cached)
        hipLaunchKernelGGL((k_tile<S, R, PLAIN, CN, NS, true>), grid, block, lds, s, a.reps, a.tdev, (const S *)a.fin,
                           (S *)a.fout, a.table, a.nrep, a.ntiles, a.toff, (const S *)a.xi, (long long)a.xi_plane, a.flags);
    else
        hipLaunchKernelGGL((k_tile<S, R, PLAIN, CN, NS, false>), grid, block, lds, s, a.reps, a.tdev, (const S *)a.fin,
                           (S *)a.fout, a.table, a.nrep, a.ntiles, a.toff, (const S *)a.xi, (long long)a.xi_plane, a.flags);
}

template <typename S, typename R, bool PLAIN> static void launch_tile_ns(const TileLaunch &a, hipStream_t s)
{
    if (a.ns == 1)
        a.xi ? launch_tile_t<S, R, PLAIN, true, 1>(a, s) : launch_tile_t<S, R, PLAIN, false, 1>(a, s);
    else if (a.ns == 2)
        a.xi ? launch_tile_t<S, R, PLAIN, true, 2>(a, s) : launch_tile_t<S, R, PLAIN, false, 2>(a, s);
    else if constexpr (sizeof(S) == 4)
        launch_tile_t<S, R, PLAIN, false, 4>(a, s);
}

bool tile_has_kernel(int precision, int ns, bool correlated)
{
    return ns == 1 || ns == 2 || (ns == 4 && precision != 0 && !correlated);
}

hipError_t launch_tile(int precision, const TileLaunch &a, hipStream_t s)
{
    if (!tile_has_kernel(precision, a.ns, a.xi != nullptr) || a.ty <= 4 * (a.ns - 1) || a.ty > TILE_MAX_TY)
        return hipErrorInvalidValue;
    if (precision == 0)
        launch_tile_ns<double, double, false>(a, s);
    else if (a.plain)
        launch_tile_ns<float, float, true>(a, s);
    else
        launch_tile_ns<float, float, false>(a, s);
    return hipGetLastError();
}

}  // namespace lbf
