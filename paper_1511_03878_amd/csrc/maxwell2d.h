// Bodies of the 2-D field update: the fused Yee update (strips by marching
// waves, or tiles) and the passes of the sixth-order solver.
//
// Yee: all three sweeps on a strip or a TX x TY tile of nodes, held in registers
// or LDS: B^{n+1/2} = B^n - dt/2 curl E^n, E^{n+1} = E^n + dt (curl B^{n+1/2} -
// J^{n+1/2}), B^{n+1} = B^{n+1/2} - dt/2 curl E^{n+1}.  B updates use forward
// differences of E and E updates backward differences of B, so a one-node
// halo on every side is enough for the three sweeps.  On an open x axis the
// E update at the faces needs By and Bz half a cell outside; they follow from
// the first-order characteristic (Silver-Mueller) condition at the face and
// time n + 1/2 combined with the 1-D Yee update (r = dt/dx, B_1 the first
// inside dual B, E^n the face E):
//   x = 0, incident Ey_i, Ez_i:  Bz = (4 Ey_i - 2 Ey^n - (1 - r) B_1) / (1 + r)
//                                By = (2 Ez^n - (1 - r) B_1 - 4 Ez_i) / (1 + r)
//   x = L, outflow:              Bz = (2 Ey^n - (1 - r) B_1) / (1 + r)
//                                By = (-2 Ez^n - (1 - r) B_1) / (1 + r)
// The kernel reads E^n, B^n from one field buffer and writes E^{n+1},
// B^{n+1} to the other (tiles read halos of their neighbours, which must not
// have been advanced yet).  It also accumulates the field energy of E^n, B^n
// over the tile's own nodes and clears the tile of the J buffer the next step
// deposits into.
#pragma once

#include "kernels.h"

namespace pic {

// Field of a 2-D Gaussian beam at the x = 0 face at time t and transverse
// position y.  L = {a0, omega0, w0, tau, t0, x_focus, y_center, phase}.
// Paraxial beam in one transverse dimension: waist w0 at x_focus, Rayleigh
// length z_R = omega0 w0^2 / 2; at the face (distance s = -x_focus from the
// waist) the spot is w0 sqrt(1 + (s / z_R)^2), the wavefront curvature
// s / (s^2 + z_R^2), the Gouy shift atan(s / z_R) / 2, and the amplitude
// a0 omega0 sqrt(w0 / spot).  Envelope exp(-2 ln2 ((t - t0) / tau)^2), tau the
// intensity FWHM; carrier sin(omega0 (t - t0) - omega0 y'^2 curv / 2 +
// Gouy + phase), y' = y - y_center.  Evaluated in FP64.
inline __device__ double beam_field(const double L[8], double t, double y)
{
    const double om = L[1], w0 = L[2], s = -L[5];
    const double zr = 0.5 * om * w0 * w0;
    const double spot = w0 * sqrt(1.0 + (s / zr) * (s / zr));
    const double curv = s / (s * s + zr * zr);
    const double gouy = 0.5 * atan2(s, zr);
    const double yr = y - L[6], tr = (t - L[4]) / L[3];
    const double env = exp(-2.0 * M_LN2 * tr * tr);
    const double prof = exp(-(yr / spot) * (yr / spot));
    const double ph = om * (t - L[4]) - 0.5 * om * yr * yr * curv + gouy + L[7];
    return L[0] * om * sqrt(w0 / spot) * env * prof * sin(ph);
}

// Workgroup b of g that share the tiles.  Workgroups are dispatched to the 8
// XCDs in turn (workgroup b to XCD b % 8), and each XCD has its own L2.  Renumbering the workgroups XCD-major gives
// every XCD a contiguous band of tiles, so the halo rows and columns a tile
// shares with its neighbours are mostly fetched into the same L2.
__device__ __forceinline__ int xcd_block(int b, int g)
{
    return (g & 7) ? b : (b & 7) * (g >> 3) + (b >> 3);
}

// The Silver-Mueller ghosts in one stated form (see curl2), at x = 0 (E face
// values, B first inside) and x = L.
template <typename T>
__device__ __forceinline__ T ghost_lo_bz(T ey, T b, T eyi, T r, T ir)
{
    return fma(-(T(1) - r), b, T(4) * eyi - T(2) * ey) * ir;
}
template <typename T>
__device__ __forceinline__ T ghost_lo_by(T ez, T b, T ezi, T r, T ir)
{
    return fma(T(-4), ezi, fma(ez, T(2), -((T(1) - r) * b))) * ir;
}
template <typename T>
__device__ __forceinline__ T ghost_hi(T e, T b, T r, T ir)  // e = Ey (Bz) or -Ez (By)
{
    return fma(e, T(2), -((T(1) - r) * b)) * ir;
}

// Incident Ey, Ez at the x = 0 face of step ls, row gj.
template <typename T>
__device__ __forceinline__ void incident_field(const SimDev<T> &S, int64_t ls, int gj, T &eyi, T &ezi)
{
    eyi = ezi = T(0);
    if (ls < S.laser_steps) {
        if (S.laser_ey) eyi = glb(S.laser_ey)[ls * S.n[1] + gj];
        if (S.laser_ez) ezi = glb(S.laser_ez)[ls * S.n[1] + gj];
    }
    if (S.nlaser) {
        const double t = ((double)ls + 0.5) * S.wdt;
        double ey = 0.0, ez = 0.0;
        for (int l = 0; l < S.nlaser; ++l) {
            if (S.las_pol[l] == 1) ey += beam_field(S.las[l], t, ((double)gj + 0.5) * S.dd[1]);
            else ez += beam_field(S.las[l], t, (double)gj * S.dd[1]);
        }
        eyi += (T)ey;
        ezi += (T)ez;
    }
}

// Yee tiles of workgroup b of g (256 threads).
template <typename T, int TX, int TY>
__device__ __forceinline__ void yee2d_tiles(const SimDev<T> *__restrict__ sims, int nsims,
                                            const int *__restrict__ tile_prefix, int total, int wg, int nwg)
{
    constexpr int W = TX + 3, H = TY + 3, NB = W * H;
    constexpr int NE = (TX + 1) * (TY + 1);  // nodes of sweep 2
    __shared__ T sE[3][NB], sB[3][NB];
    __shared__ double s_red[4];
    const int tid = threadIdx.x;

    for (int tile = xcd_block(wg, nwg); tile < total; tile += nwg) {
        const int s = find_sim(tile_prefix, nsims, tile);
        const SimDev<T> &S = sims[s];
        if (!glb(S.st)->active || S.morder == 6) continue;
        const int lt = tile - tile_prefix[s];
        const int n0 = S.n[0], n1 = S.n[1], fn0 = S.fn[0], fn1 = S.fn[1];
        const int per0 = S.periodic[0], per1 = S.periodic[1];
        const int ntx = (fn0 + TX - 1) / TX;
        const int X0 = (lt % ntx) * TX, Y0 = (lt / ntx) * TY;
        const int64_t stepn = glb(S.st)->step;
        T *const *Jc = S.J[stepn & 1];
        T *const *Jn = S.J[(stepn + 1) & 1];
        T *const *Fc = S.F[stepn & 1];
        T *const *Fn = S.F[(stepn + 1) & 1];

        // ---- load nodes [X0-1, X0+TX+1] x [Y0-1, Y0+TY+1] -------------------
        // All loads of the tile are issued before the first LDS write, from an
        // index that is always in range (a node that does not exist reads node
        // 0 and the value is dropped afterwards), so no load sits behind a
        // branch and each thread keeps all its requests in flight.  J is read
        // straight into the registers of the thread that uses it in sweep 2.
        // staggering: Ex (d,p) Ey (p,d) Ez (p,p) Bx (p,d) By (d,p) Bz (d,d)
        struct Idx {
            int64_t dp, pd, pp, dd;
        };
        auto node_idx = [&](int a, int b) {
            const int gi = X0 - 1 + a, gj = Y0 - 1 + b;
            // nodes more than one past the last stored node feed no update
            // (tiles may be wider than the grid); they stay zero
            const bool need = gi <= fn0 + 1 && gj <= fn1 + 1;
            const int ip = need ? axis_node(gi, n0, per0, 0) : -1;
            const int id = need ? axis_node(gi, n0, per0, 1) : -1;
            const int jp = need ? axis_node(gj, n1, per1, 0) : -1;
            const int jd = need ? axis_node(gj, n1, per1, 1) : -1;
            Idx r;
            r.dp = (id >= 0 && jp >= 0) ? id + (int64_t)fn0 * jp : -1;
            r.pd = (ip >= 0 && jd >= 0) ? ip + (int64_t)fn0 * jd : -1;
            r.pp = (ip >= 0 && jp >= 0) ? ip + (int64_t)fn0 * jp : -1;
            r.dd = (id >= 0 && jd >= 0) ? id + (int64_t)fn0 * jd : -1;
            return r;
        };
        auto ld = [&](T *f, int64_t k) {
            const T x = glb(f)[k >= 0 ? k : 0];
            return k >= 0 ? x : T(0);
        };
        constexpr int NIT = (NB + 255) / 256;
        constexpr int NJT = (NE + 255) / 256;
        T v[NIT][6];
        T jv[NJT][3];
        double esum = 0.0;
#pragma unroll
        for (int r = 0; r < NIT; ++r) {
            const int t = min(tid + 256 * r, NB - 1);
            const Idx q = node_idx(t % W, t / W);
            v[r][0] = ld(Fc[0], q.dp);
            v[r][1] = ld(Fc[1], q.pd);
            v[r][2] = ld(Fc[2], q.pp);
            v[r][3] = ld(Fc[3], q.pd);
            v[r][4] = ld(Fc[4], q.dp);
            v[r][5] = ld(Fc[5], q.dd);
        }
#pragma unroll
        for (int r = 0; r < NJT; ++r) {
            const int t = min(tid + 256 * r, NE - 1);
            const Idx q = node_idx(1 + t % (TX + 1), 1 + t / (TX + 1));
            jv[r][0] = ld(Jc[0], q.dp);
            jv[r][1] = ld(Jc[1], q.pd);
            jv[r][2] = ld(Jc[2], q.pp);
        }
#pragma unroll
        for (int r = 0; r < NIT; ++r) {
            const int t = tid + 256 * r;
            if (t >= NB) break;
            const int a = t % W, b = t / W;
            const int gi = X0 - 1 + a, gj = Y0 - 1 + b;
            const bool own = a >= 1 && a <= TX && b >= 1 && b <= TY && gi < fn0 && gj < fn1;
            sE[0][t] = v[r][0]; sE[1][t] = v[r][1]; sE[2][t] = v[r][2];
            sB[0][t] = v[r][3]; sB[1][t] = v[r][4]; sB[2][t] = v[r][5];
            if (own) {
                // invalid (outside) nodes were loaded as zero, so they add nothing
#pragma unroll
                for (int c = 0; c < 6; ++c) esum += (double)v[r][c] * (double)v[r][c];
            }
        }
        __syncthreads();

        const T dt = S.dt, h = T(0.5) * S.dt;
        const T ix = T(1) / S.d[0], iy = T(1) / S.d[1];

        // ---- sweep 1: B^{n+1/2} on a in [0, TX+1], b in [0, TY+1] -----------
        for (int t = tid; t < (TX + 2) * (TY + 2); t += 256) {
            const int a = t % (TX + 2), b = t / (TX + 2);
            const int c = b * W + a;
            sB[0][c] -= h * (sE[2][c + W] - sE[2][c]) * iy;
            sB[1][c] += h * (sE[2][c + 1] - sE[2][c]) * ix;
            sB[2][c] -= h * curl2(sE[1][c + 1] - sE[1][c], ix, sE[0][c + W] - sE[0][c], iy);
        }
        __syncthreads();

        // ---- Silver-Mueller ghosts on an open x axis -------------------------
        if (!per0) {
            const T r = dt * ix;
            const T ir = T(1) / (T(1) + r);
            if (X0 == 0) {
                for (int b = tid; b < H; b += 256) {
                    T eyi, ezi;
                    incident_field(S, stepn, wrap_idx(Y0 - 1 + b, n1), eyi, ezi);
                    const int c = b * W;  // a = 0 is x-node -1 (dual -1/2 for By, Bz)
                    sB[2][c] = ghost_lo_bz(sE[1][c + 1], sB[2][c + 1], eyi, r, ir);
                    sB[1][c] = ghost_lo_by(sE[2][c + 1], sB[1][c + 1], ezi, r, ir);
                }
            }
            const int ag = n0 - X0 + 1;  // local column of dual x index n0 (x = L + 1/2)
            if (ag >= 1 && ag <= TX + 1) {
                for (int b = tid; b < H; b += 256) {
                    const int c = b * W + ag;
                    sB[2][c] = ghost_hi(sE[1][c], sB[2][c - 1], r, ir);
                    sB[1][c] = ghost_hi(-sE[2][c], sB[1][c - 1], r, ir);
                }
            }
            __syncthreads();
        }

        // ---- sweep 2: E^{n+1} on a in [1, TX+1], b in [1, TY+1] -------------
#pragma unroll
        for (int r = 0; r < NJT; ++r) {
            const int t = tid + 256 * r;
            if (t >= NE) break;
            const int a = 1 + t % (TX + 1), b = 1 + t / (TX + 1);
            const int c = b * W + a;
            sE[0][c] += dt * ((sB[2][c] - sB[2][c - W]) * iy - jv[r][0]);
            sE[1][c] += dt * (-(sB[2][c] - sB[2][c - 1]) * ix - jv[r][1]);
            sE[2][c] += dt * (curl2(sB[1][c] - sB[1][c - 1], ix, sB[0][c] - sB[0][c - W], iy) - jv[r][2]);
        }
        __syncthreads();

        // ---- sweep 3: B^{n+1} on the tile's own nodes, then write back -------
        for (int t = tid; t < TX * TY; t += 256) {
            const int a = 1 + t % TX, b = 1 + t / TX;
            const int gi = X0 + a - 1, gj = Y0 + b - 1;
            if (gi >= fn0 || gj >= fn1) continue;
            const int c = b * W + a;
            const T bx = sB[0][c] - h * (sE[2][c + W] - sE[2][c]) * iy;
            const T by = sB[1][c] + h * (sE[2][c + 1] - sE[2][c]) * ix;
            const T bz = sB[2][c] - h * curl2(sE[1][c + 1] - sE[1][c], ix, sE[0][c + W] - sE[0][c], iy);
            // own nodes are inside the periodic range; on an open axis the dual
            // components stop one node short
            const bool dx_ok = per0 || gi <= n0 - 1;
            const int64_t k = gi + (int64_t)fn0 * gj;
            glb(Fn[1])[k] = sE[1][c];
            glb(Fn[2])[k] = sE[2][c];
            glb(Fn[3])[k] = bx;
            glb(Jn[1])[k] = T(0);
            glb(Jn[2])[k] = T(0);
            if (dx_ok) {
                glb(Fn[0])[k] = sE[0][c];
                glb(Fn[4])[k] = by;
                glb(Fn[5])[k] = bz;
                glb(Jn[0])[k] = T(0);
            }
        }

        // ---- field energy of E^n, B^n ----------------------------------------
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) esum += __shfl_xor(esum, o, 64);
        if ((tid & 63) == 0) s_red[tid >> 6] = esum;
        __syncthreads();
        if (tid == 0)
            glb(S.upart)[lt] = 0.5 * S.vcell * (s_red[0] + s_red[1] + s_red[2] + s_red[3]);
        __syncthreads();
    }
}

// The same update by waves that march along y (the default; the tiles serve
// the presets that the tuner tries).  A wave takes a strip of kStripCols x
// S.yee_bz nodes, one column per lane (lane 0 the column before the strip, lanes
// 62 and 63 the two after it), keeps the rows of the three sweeps in registers,
// reads x neighbours from the neighbouring lane, and has the next four rows in
// flight while it updates one; no LDS, no barrier.  The tiles load, update and
// store in turn with two workgroups per CU (197 VGPRs), so latency bounds them;
// this kernel runs at 4.1 TB/s from HBM (4096 x 1024 nodes; a copy of as many
// arrays runs at 5.2 - 6.5) and 5.1 from the last-level cache.  us per launch,
// tiles / strips, FP32: 4096 x 1024 99 / 73, 2048 x 1024 52 / 29, 1024 x 1024
// 26 / 18; FP64: 163 / 141, 90 / 72, 38 / 32.  In the step: 4096 x 1024 laser
// box 321 -> 288 us, 1536 x 384 102 -> 94.  Rows per strip: 16 take 80 us at
// 4096 x 1024 (too few waves), 6 take 74; 56 columns, which makes rows of
// stores start on 32 bytes, 75.  Rows are read and written through buffer
// descriptors whose bounds check drops the lanes that have no node (and reads
// zero for them), so no access sits behind a branch.
constexpr int kMarchAhead = 4;

// Descriptor of a row of n nodes; offsets in bytes, kNoNode is past every row
// (a grid has at most 2^30 cells and 4 rows or more: rows up to 2^31 + 8 bytes).
constexpr uint32_t kNoNode = 0xfffffff0u;
template <typename T>
struct RowBuf {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ RowBuf(const T *row, int n)
        : r(__builtin_amdgcn_make_buffer_rsrc((void *)row, 0, (int)((uint32_t)n * (uint32_t)sizeof(T)), 0x00027000))
    {
    }
    __device__ __forceinline__ T load(uint32_t off) const
    {
        if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
        else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    }
    __device__ __forceinline__ void store(uint32_t off, T x) const
    {
        if constexpr (sizeof(T) == 4) {
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), r, off, 0, 0);
        } else {
            typedef uint32_t W2 __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(W2, x), r, off, 0, 0);
        }
    }
};

// Strips of workgroup wg of nwg (256 threads, a strip per wave).
template <typename T>
__device__ __forceinline__ void yee2d_march(const SimDev<T> *__restrict__ sims, int nsims,
                                            const int *__restrict__ tile_prefix, int total, int wg, int nwg)
{
    const int ln = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int tile = kStripsPerWg * xcd_block(wg, nwg) + wv; tile < total; tile += kStripsPerWg * nwg) {
        const int s = find_sim(tile_prefix, nsims, tile);
        const SimDev<T> &S = sims[s];
        if (!glb(S.st)->active || S.morder == 6) continue;
        const int lt = tile - tile_prefix[s];
        const int n0 = S.n[0], n1 = S.n[1], fn0 = S.fn[0];
        const int per0 = S.periodic[0];  // (y is periodic in 2-D)
        const int ntx = (fn0 + kStripCols - 1) / kStripCols;
        const int X0 = (lt % ntx) * kStripCols, Y0 = (lt / ntx) * S.yee_bz;
        const int rows = min(S.yee_bz, n1 - Y0);
        const int64_t stepn = glb(S.st)->step;
        T *const *Jc = S.J[stepn & 1];
        T *const *Jn = S.J[(stepn + 1) & 1];
        T *const *Fc = S.F[stepn & 1];
        T *const *Fn = S.F[(stepn + 1) & 1];

        // byte offsets of the lane's column in a row, for primal and dual x;
        // columns more than one past the last stored node feed no update
        const int gi = X0 - 1 + ln;
        const int ip = gi <= fn0 + 1 ? axis_node(gi, n0, per0, 0) : -1;
        const int id = gi <= fn0 + 1 ? axis_node(gi, n0, per0, 1) : -1;
        const uint32_t op = ip >= 0 ? (uint32_t)ip * (uint32_t)sizeof(T) : kNoNode;
        const uint32_t od = id >= 0 ? (uint32_t)id * (uint32_t)sizeof(T) : kNoNode;
        const bool own = ln >= 1 && ln <= kStripCols && gi < fn0;
        const uint32_t wp = own ? op : kNoNode, wd = own ? od : kNoNode;
        // staggering: Ex (d,p) Ey (p,d) Ez (p,p) Bx (p,d) By (d,p) Bz (d,d)
        struct Row {
            T e[3], b[3], j[3];
        };
        // row b of the strip is row Y0 - 1 + b of the grid: E of rows 0 .. rows + 2,
        // B up to rows + 1, J up to rows + 1 from 1 (others read as zero, from an
        // empty descriptor)
        auto load_row = [&](int b, Row &r) {
            int gj = Y0 - 1 + min(b, rows + 2);
            gj += gj < 0 ? n1 : 0;
            gj -= gj >= n1 ? n1 : 0;
            const int64_t ro = (int64_t)fn0 * gj;
            const int ne = b <= rows + 2 ? fn0 : 0, nb = b <= rows + 1 ? fn0 : 0, nj = b >= 1 ? nb : 0;
            r.e[0] = RowBuf<T>(Fc[0] + ro, ne).load(od);
            r.e[1] = RowBuf<T>(Fc[1] + ro, ne).load(op);
            r.e[2] = RowBuf<T>(Fc[2] + ro, ne).load(op);
            r.b[0] = RowBuf<T>(Fc[3] + ro, nb).load(op);
            r.b[1] = RowBuf<T>(Fc[4] + ro, nb).load(od);
            r.b[2] = RowBuf<T>(Fc[5] + ro, nb).load(od);
            r.j[0] = RowBuf<T>(Jc[0] + ro, nj).load(od);
            r.j[1] = RowBuf<T>(Jc[1] + ro, nj).load(op);
            r.j[2] = RowBuf<T>(Jc[2] + ro, nj).load(op);
        };
        const bool lo = !per0 && X0 == 0;
        // incident field of row ln (evaluated first: it takes many registers)
        T eyi = T(0), ezi = T(0);
        if (lo && ln < rows + 2) incident_field(S, stepn, wrap_idx(Y0 - 1 + ln, n1), eyi, ezi);
        Row r0, cur, nxt, ring[kMarchAhead];
        load_row(0, r0);
        load_row(1, cur);
        load_row(2, nxt);
#pragma unroll
        for (int u = 0; u < kMarchAhead; ++u) load_row(3 + u, ring[u]);

        const T dt = S.dt, h = T(0.5) * S.dt;
        const T ix = T(1) / S.d[0], iy = T(1) / S.d[1];
        const T sm = dt * ix, ism = T(1) / (T(1) + sm);
        const int ag = per0 ? -1 : n0 - X0 + 1;  // lane of dual x index n0 (x = L + 1/2)
        auto up = [&](T x) { return __shfl_down(x, 1); };  // value of the next column
        auto dn = [&](T x) { return __shfl_up(x, 1); };    // ... of the previous one

        // the three sweeps on a row; e, en: E of the row and of the next
        double esum = 0.0;
        auto b_half = [&](const T b[3], const T e[3], const T en[3], T o[3]) {
            o[0] = b[0] - h * (en[2] - e[2]) * iy;
            o[1] = b[1] + h * (up(e[2]) - e[2]) * ix;
            o[2] = b[2] - h * curl2(up(e[1]) - e[1], ix, en[0] - e[0], iy);
        };
        // B^{n+1/2} of the row in c (row number b), with ghosts and field energy
        auto sweep1 = [&](int b, const Row &c, const Row &n, T o[3]) {
            b_half(c.b, c.e, n.e, o);
            if (lo) {
                const T ey = up(c.e[1]), ez = up(c.e[2]), bz = up(o[2]), by = up(o[1]);
                const T iy_ = __shfl(eyi, b), iz_ = __shfl(ezi, b);
                if (ln == 0) {
                    o[2] = ghost_lo_bz(ey, bz, iy_, sm, ism);
                    o[1] = ghost_lo_by(ez, by, iz_, sm, ism);
                }
            }
            if (ag >= 1 && ag <= kStripCols + 1) {
                const T bz = dn(o[2]), by = dn(o[1]);
                if (ln == ag) {
                    o[2] = ghost_hi(c.e[1], bz, sm, ism);
                    o[1] = ghost_hi(-c.e[2], by, sm, ism);
                }
            }
            double en = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) en += squares2((double)c.e[k], (double)c.b[k]);
            esum += own && b <= rows ? en : 0.0;
        };
        // E^{n+1} of the row in c from B^{n+1/2} of it (bh) and of the previous row
        auto sweep2 = [&](const Row &c, const T bh[3], const T bp[3], T o[3]) {
            o[0] = c.e[0] + dt * ((bh[2] - bp[2]) * iy - c.j[0]);
            o[1] = c.e[1] + dt * (-(bh[2] - dn(bh[2])) * ix - c.j[1]);
            o[2] = c.e[2] + dt * (curl2(bh[1] - dn(bh[1]), ix, bh[0] - bp[0], iy) - c.j[2]);
        };

        T bh[3], bp[3], ec[3];  // B^{n+1/2} and E^{n+1} of the row to write, B of the one before
        b_half(r0.b, r0.e, cur.e, bp);
        sweep1(1, cur, nxt, bh);
        sweep2(cur, bh, bp, ec);
        for (int b0 = 1; b0 <= rows; b0 += kMarchAhead) {
#pragma unroll
            for (int u = 0; u < kMarchAhead; ++u) {
                const int b = b0 + u;  // row to write; nxt holds row b + 1, ring[u] row b + 2
                if (b > rows) break;
                T bn[3], en[3], o[3];
                sweep1(b + 1, nxt, ring[u], bn);
                sweep2(nxt, bn, bh, en);
                b_half(bh, ec, en, o);
                const int64_t ro = (int64_t)fn0 * (Y0 - 1 + b);
                RowBuf<T>(Fn[0] + ro, fn0).store(wd, ec[0]);
                RowBuf<T>(Fn[1] + ro, fn0).store(wp, ec[1]);
                RowBuf<T>(Fn[2] + ro, fn0).store(wp, ec[2]);
                RowBuf<T>(Fn[3] + ro, fn0).store(wp, o[0]);
                RowBuf<T>(Fn[4] + ro, fn0).store(wd, o[1]);
                RowBuf<T>(Fn[5] + ro, fn0).store(wd, o[2]);
                RowBuf<T>(Jn[0] + ro, fn0).store(wd, T(0));
                RowBuf<T>(Jn[1] + ro, fn0).store(wp, T(0));
                RowBuf<T>(Jn[2] + ro, fn0).store(wp, T(0));
                nxt = ring[u];
                load_row(b + 2 + kMarchAhead, ring[u]);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    ec[k] = en[k];
                    bh[k] = bn[k];
                }
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) esum += __shfl_xor(esum, o, 64);
        if (ln == 0) glb(S.upart)[lt] = 0.5 * S.vcell * esum;
    }
}

// Sixth-order staggered field solver (2-D, periodic axes): the same three
// sweeps as three passes over the tiles of the Yee decomposition (so the
// per-tile energy partials line up), one node per thread iteration, the
// neighbours read from global memory (L2 hits).  The derivative at a half
// point comes from the three node pairs around it with the weights that cancel
// the h^2 and h^4 terms of the Taylor series: 75/64, -25/384, 3/640.
// PASS 0: B^{n+1/2} from E^n into the other buffer, energy of E^n, B^n;
// PASS 1: E^{n+1} from B^{n+1/2} and J, clears the other J buffer;
// PASS 2: B^{n+1} from E^{n+1}, in place (it reads E only).
template <typename T, int PASS>
__device__ __forceinline__ void hi2d_tiles(const SimDev<T> *__restrict__ sims, int nsims,
                                           const int *__restrict__ tile_prefix, int total, int TX, int TY,
                                           int wg, int nwg)
{
    __shared__ double s_red[4];
    const int tid = threadIdx.x;
    constexpr T c1 = T(75.0 / 64.0), c2 = T(-25.0 / 384.0), c3 = T(3.0 / 640.0);
    for (int tile = xcd_block(wg, nwg); tile < total; tile += nwg) {
        const int s = find_sim(tile_prefix, nsims, tile);
        const SimDev<T> &S = sims[s];
        if (!glb(S.st)->active || S.morder != 6) continue;
        const int lt = tile - tile_prefix[s];
        const int n0 = S.n[0], n1 = S.n[1];
        const int ntx = (n0 + TX - 1) / TX;
        const int X0 = (lt % ntx) * TX, Y0 = (lt / ntx) * TY;
        const int64_t stepn = glb(S.st)->step;
        T *const *Fc = S.F[stepn & 1];
        T *const *Fn = S.F[(stepn + 1) & 1];
        const T dt = S.dt, h = T(0.5) * S.dt;
        const T ix = T(1) / S.d[0], iy = T(1) / S.d[1];
        double esum = 0.0;
        for (int t = tid; t < TX * TY; t += 256) {
            const int gi = X0 + t % TX, gj = Y0 + t / TX;
            if (gi >= n0 || gj >= n1) continue;
            const int64_t k = gi + (int64_t)n0 * gj;
            // value of array f at node (gi + di, gj + dj), periodic (|d| <= 3 <= n)
            auto node = [&](const T *f, int di, int dj) {
                int a = gi + di, b = gj + dj;
                a += a < 0 ? n0 : 0;
                a -= a >= n0 ? n0 : 0;
                b += b < 0 ? n1 : 0;
                b -= b >= n1 ? n1 : 0;
                return glb(f)[a + (int64_t)n0 * b];
            };
            // forward difference (half point after the node) and backward
            // (half point before it) along x (ax = 0) or y (ax = 1)
            auto dfw = [&](const T *f, int ax) {
                const int u = ax == 0, v = ax == 1;
                return sum3(c1, node(f, u, v) - node(f, 0, 0), c2, node(f, 2 * u, 2 * v) - node(f, -u, -v), c3,
                            node(f, 3 * u, 3 * v) - node(f, -2 * u, -2 * v));
            };
            auto dbw = [&](const T *f, int ax) {
                const int u = ax == 0, v = ax == 1;
                return sum3(c1, node(f, 0, 0) - node(f, -u, -v), c2, node(f, u, v) - node(f, -2 * u, -2 * v), c3,
                            node(f, 2 * u, 2 * v) - node(f, -3 * u, -3 * v));
            };
            if constexpr (PASS == 0 || PASS == 2) {
                T *const *E = PASS == 0 ? Fc : Fn;
                const T bx0 = glb(PASS == 0 ? Fc[3] : Fn[3])[k];
                const T by0 = glb(PASS == 0 ? Fc[4] : Fn[4])[k];
                const T bz0 = glb(PASS == 0 ? Fc[5] : Fn[5])[k];
                const T bx = bx0 - h * dfw(E[2], 1) * iy;
                const T by = by0 + h * dfw(E[2], 0) * ix;
                const T bz = bz0 - h * curl2(dfw(E[1], 0), ix, dfw(E[0], 1), iy);
                if constexpr (PASS == 0) {
                    const T ex = glb(Fc[0])[k], ey = glb(Fc[1])[k], ez = glb(Fc[2])[k];
                    esum += squares6(ex, ey, ez, bx0, by0, bz0);
                }
                glb(Fn[3])[k] = bx;
                glb(Fn[4])[k] = by;
                glb(Fn[5])[k] = bz;
            } else {
                T *const *Jc = S.J[stepn & 1];
                T *const *Jn = S.J[(stepn + 1) & 1];
                const T ex = glb(Fc[0])[k] + dt * (dbw(Fn[5], 1) * iy - glb(Jc[0])[k]);
                const T ey = glb(Fc[1])[k] + dt * (-dbw(Fn[5], 0) * ix - glb(Jc[1])[k]);
                const T ez = glb(Fc[2])[k] + dt * (curl2(dbw(Fn[4], 0), ix, dbw(Fn[3], 1), iy) - glb(Jc[2])[k]);
                glb(Fn[0])[k] = ex;
                glb(Fn[1])[k] = ey;
                glb(Fn[2])[k] = ez;
                glb(Jn[0])[k] = T(0);
                glb(Jn[1])[k] = T(0);
                glb(Jn[2])[k] = T(0);
            }
        }
        if constexpr (PASS == 0) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) esum += __shfl_xor(esum, o, 64);
            if ((tid & 63) == 0) s_red[tid >> 6] = esum;
            __syncthreads();
            if (tid == 0)
                glb(S.upart)[lt] = 0.5 * S.vcell * (s_red[0] + s_red[1] + s_red[2] + s_red[3]);
            __syncthreads();
        }
    }
}

}  // namespace pic
