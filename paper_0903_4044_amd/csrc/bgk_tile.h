// bgk_tile.h -- the streaming kernel on tiles of cells (k_tile), for one- and
// two-dimensional kinds.  Same pass, inputs and outputs as k_stream (see
// bgk_device.h); there every cell relaxes the 4 or 7 stencil inputs of each
// velocity itself, here a workgroup relaxes each cell of a tile and of its
// halo once and the stencils read the relaxed values from LDS.
//
// In one and two dimensions bound by the memory traffic: 1024 x 48^3 FP32
// moves 0.93 GB (1.03 times f's read and write) in 184 to 198 us, 128^2 x 24^3
// 2.26 GB (1.25 times: halo rows read again, spilled registers) in 462 to 480,
// 64 cavities 62 GB (1.32 times) in 12.1 ms, 4.7 to 5.2 TB/s where a large copy
// reaches 4.9.  The issue of vector instructions is not far behind: 49 per
// element in 2D (76 in k_stream, most of them its seven relaxations and their
// table loads), with the loads of the next plane in flight.  In k_stream these
// passes took 272 us, 790 us and 19.6 ms.  160^2 x 20^3 FP32 558 to 585 us,
// 1096 there; 48^2 x 24^3 FP64 154 us, 272; recording on 64^2 x 24^3 FP32 199,
// 231.
#pragma once

#include "bgk_device.h"

namespace bgk {

// A tile is TX x TY cells, four consecutive cells of a row per wave.  The LDS
// plane holds the tile and two halo cells on every side, position
// (y + 2 HY) * PITCH + x + 2; each position holds one value per lane.
// Waves per workgroup: in 2D the halo of 8 x 8 cells doubles the relaxed
// values, that of 8 x 4 cells makes it 2.5 times (float: 499 against 554 us a
// step on 128^2 x 24^3); in FP64 the two LDS planes of 8 x 8 cells and the
// registers of 16 waves do not fit.  In 1D the halo is small and the short
// workgroups balance better (1024 x 48^3: 203 us a step with 4 waves, 212
// with 8, 210 with 16).
template <typename real, int DIM>
struct TileShape {
    static constexpr int NW = DIM == 1 ? 4 : sizeof(real) == 4 ? 16 : 8;
    static constexpr int TX = DIM == 1 ? 4 * NW : 8, TY = DIM == 1 ? 1 : NW / 2;
    static constexpr int HY = DIM == 1 ? 0 : 2;
    static constexpr int PITCH = TX + 4, NPOS = PITCH * (TY + 2 * HY);
    // rows of a wave: four cells, YH y-halo positions (2D; the 4 TX of them
    // shared out evenly), two x-halo positions
    static constexpr int YH = DIM == 1 ? 0 : 4 * TX / NW, RPW = 4 + YH + 2, NROW = NW * RPW;
    static constexpr int NG = DIM == 1 ? 0 : 2 * TY + 2 * TX;    // wall entries of a tile: left, right, bottom, top faces
    static constexpr int NZT = NROW + NG + (NROW + NG) % 2;      // z-table columns
};

// One row of a tile: the cell whose h is read (offset in the instance, in
// elements) and the entry that relaxes it; at a ghost position also the ghost
// entry's z-table column and the velocities that take it (code: 0 none, 1 all
// (k_tile3 only), 2 v_x > 0, 3 v_x <= 0, 4 v_y > 0, 5 v_y <= 0).
struct TileRow { uint32_t off; int par, gpar, gcol, code; };

template <typename real, int DIM>
__host__ __device__ constexpr size_t tile_buffer() { return (size_t)TileShape<real, DIM>::NPOS * 64 * sizeof(real); }

// Dynamic LDS: two planes of relaxed values, the z tables [plane][column][2],
// the planes' (mass share or v_z, energy) weights.
struct TileLds { size_t zt, w, total; };

template <typename real, int DIM>
__host__ __device__ inline TileLds tile_lds(const Geo &g)
{
    TileLds L;
    L.zt = 2 * tile_buffer<real, DIM>();
    L.w = L.zt + (size_t)(g.nvz + 1) * TileShape<real, DIM>::NZT * 2 * sizeof(real);
    L.w = (L.w + 15) & ~(size_t)15;
    L.total = L.w + (size_t)2 * (g.nvz + 1) * sizeof(double);
    return L;
}

// Sums over the wave of 4 x N values (v[cell][q]): afterwards every lane of
// the 16-lane row r holds in out[q] the total of cell tile_row_cell(r).  Two
// half exchanges (each adds two values' halves and keeps one of them per
// lane) and a sum inside the row: 21 N operations instead of 4 N full
// butterflies.
__device__ __forceinline__ double swap_add32(double x, double y)
{
    const unsigned long long a = (unsigned long long)__double_as_longlong(x), b = (unsigned long long)__double_as_longlong(y);
    auto lo = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false);
    auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
    return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ double swap_add16(double x, double y)
{
    const unsigned long long a = (unsigned long long)__double_as_longlong(x), b = (unsigned long long)__double_as_longlong(y);
    auto lo = __builtin_amdgcn_permlane16_swap((unsigned)a, (unsigned)b, false, false);
    auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
    return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ int tile_row_cell(int r) { return (r >> 1) | ((r & 1) << 1); }

template <typename real, int DIM, bool NTSTORE, bool REC>
__global__ void __attribute__((amdgpu_flat_work_group_size(64 * TileShape<real, DIM>::NW, 64 * TileShape<real, DIM>::NW), amdgpu_waves_per_eu(sizeof(real) == 4 ? 4 : 2)))
    k_tile(Args A, const real *__restrict__ src, real *__restrict__ dst, const real *__restrict__ params,
           double *__restrict__ partial)
{
    using S = TileShape<real, DIM>;
    using R2 = vec_t<real, 2>;
    constexpr int RPW = S::RPW, NACC = 9, NTH = 64 * S::NW;
    constexpr uint32_t RB = 64 * sizeof(real);             // bytes of one position
    constexpr uint32_t BUF = (uint32_t)tile_buffer<real, DIM>();
    constexpr uint32_t ZR = S::NZT * 2 * sizeof(real);      // bytes of one plane of the z tables
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ TileRow s_row[S::NROW];
    __shared__ double s_acc[4 * S::NW][NACC];
    const Geo &g = A.g;
    const TileLds Lo = tile_lds<real, DIM>(g);
    unsigned char *const zt = smem + Lo.zt;
    double *const wt = reinterpret_cast<double *>(smem + Lo.w);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nitems = A.nttiles * A.vsplit;
    const int Lq = xcd_remap(blockIdx.x, nitems);
    int tq, ch;
    {
        constexpr int SB = 64;  // tiles of a superblock, walked chunk by chunk
        const int sb = Lq / (SB * A.vsplit), c0 = sb * SB, n = min(SB, A.nttiles - c0), k = Lq - c0 * A.vsplit;
        ch = k / n;
        tq = c0 + (k - ch * n);
    }
    int lo = 0, hi = A.ninst;  // inst[lo].ttile0 <= tq < inst[hi].ttile0
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (A.inst[mid].ttile0 <= tq) lo = mid; else hi = mid;
    }
    const Inst &I = A.inst[lo];
    const int tpr = (I.nx + S::TX - 1) / S::TX, tpc = (I.ny + S::TY - 1) / S::TY;
    const int tt = strip_tile(tq - I.ttile0, tpr, tpc, 2);
    const int ty = tt / tpr, x0 = (tt - ty * tpr) * S::TX, y0 = ty * S::TY;

    // ---- rows and tables of the tile
    for (int r = tid; r < S::NROW; r += NTH) {
        const int w = r / RPW, k = r - w * RPW;
        int px, py;  // position in the tile
        if (k < 4) {
            px = DIM == 1 ? 4 * w + k : 4 * (w & 1) + k;
            py = DIM == 1 ? 0 : w >> 1;
        } else if (k < 4 + S::YH) {
            const int j = w * S::YH + k - 4, l = j / S::TX;  // line l: y = -2, -1, TY, TY + 1
            px = j - l * S::TX;
            py = l < 2 ? l - 2 : S::TY + l - 2;
        } else {
            const int side = w & 1;
            px = side ? S::TX + k - 4 - S::YH : k - 6 - S::YH;
            py = DIM == 1 ? 0 : w >> 1;
        }
        const int x = x0 + px, y = y0 + py;
        const bool ox = x < 0 || x >= I.nx, oy = y < 0 || y >= I.ny;
        // (positions outside along two directions, in the halo and outside the
        // domain across it, or outside along a direction the instance does not
        // stream along, are never read as such: the clamped cell)
        int cx = min(max(x, 0), I.nx - 1), cy = min(max(y, 0), I.ny - 1);
        TileRow t;
        t.gpar = -1;
        t.gcol = 0;
        t.code = 0;
        if (I.kind == KIND_PER1 || I.kind == KIND_PER2) {
            cx = (x % I.nx + I.nx) % I.nx;
            if (inst_dim(I) >= 2) cy = (y % I.ny + I.ny) % I.ny;
        } else if (I.kind == KIND_SHOCK) {
            // (the far field's entry, whose c0 is 0, in place of the cell's: every velocity takes it)
        } else if (ox ? !oy && py >= 0 && py < S::TY : oy && px >= 0 && px < S::TX) {
            const int wl = ox ? (x < 0 ? 0 : 1) : (y < 0 ? 2 : 3);
            t.gpar = I.pseudo0 + wall_offset(I, wl) + (ox ? cy : cx);
            t.gcol = S::NROW + (wl == 0 ? py : wl == 1 ? S::TY + py : wl == 2 ? 2 * S::TY + px : 2 * S::TY + S::TX + px);
            t.code = wl + 2;
        }
        t.par = I.kind == KIND_SHOCK && ox ? I.pseudo0 + (x < 0 ? 0 : 1) : I.cell0 + cy * I.nx + cx;
        t.off = (uint32_t)(cy * I.nx + cx) * (uint32_t)g.nv;
        s_row[r] = t;
    }
    for (int k = tid; k < g.nvz; k += NTH) {
        const ZW w = zweights(g, k);
        wt[2 * k] = g.red ? w.m : w.z;
        wt[2 * k + 1] = w.zz;
    }
    for (int k = tid; k < 4 * S::NW * NACC; k += NTH) (&s_acc[0][0])[k] = 0.0;
    __syncthreads();
    {
        const float inv = 1.0f / (float)g.nvz;
        for (int t = tid; t < S::NROW * g.nvz; t += NTH) {
            const int r = (int)(((float)t + 0.5f) * inv), z = t - r * g.nvz;
            const TileRow &row = s_row[r];
            const real *E = params + (long long)row.par * g.pe + g.tz + 2 * z;
            *reinterpret_cast<R2 *>(zt + z * ZR + r * 2 * sizeof(real)) = *reinterpret_cast<const R2 *>(E);
            if (row.code) {
                const real *G = params + (long long)row.gpar * g.pe + g.tz + 2 * z;
                *reinterpret_cast<R2 *>(zt + z * ZR + row.gcol * 2 * sizeof(real)) = *reinterpret_cast<const R2 *>(G);
            }
        }
    }
    __syncthreads();

    // ---- this wave's rows
    uint32_t roff[RPW];     // byte offset of the row's h in the instance
    int gm = 0;             // rows with a ghost part
    // double: the ghost's column behind the row's own, in bytes (in float these
    // scalars cost vector registers that are not there: 128^2 x 24^3 496 us a
    // step without them, 624 with; 48^2 x 24^3 FP64 177 without, 167 with)
    int dcol[sizeof(real) == 8 ? RPW : 1];
    bool out[4];            // cells inside the instance
    const TileRow *const rows = s_row + wave * RPW;
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        roff[r] = __builtin_amdgcn_readfirstlane(rows[r].off) * (uint32_t)sizeof(real);
        if (DIM == 2 && __builtin_amdgcn_readfirstlane(rows[r].code)) gm |= 1 << r;
        if constexpr (sizeof(real) == 8)
            dcol[r] = (__builtin_amdgcn_readfirstlane(rows[r].gcol) - (wave * RPW + r)) * 2 * (int)sizeof(real);
    }
    const int cx0 = x0 + (DIM == 1 ? 4 * wave : 4 * (wave & 1)), cy0 = y0 + (DIM == 1 ? 0 : wave >> 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = cy0 < I.ny && cx0 + i < I.nx;
    // Tiles with cells outside the instance or a halo that reaches over a wall.
    // Of the whole tile and not of the wave alone: the planes' barriers then
    // stand in control flow that the workgroup shares.  (Waves of such a tile
    // without ghosts of their own take the longer path too; they would wait for
    // the others at each barrier.  One loop with the barrier between the phases'
    // own branches spills: 128^2 x 24^3 FP32 552 us a step, 504 with this.)
    const bool walls = I.kind == KIND_CAVITY;
    const int reach = walls ? 2 : 0;
    // (forced into a scalar register: three spilled registers fewer)
    const bool edge = __builtin_amdgcn_readfirstlane(
        (int)(x0 + S::TX + reach > I.nx || (walls && x0 == 0) ||
              (DIM == 2 && (y0 + S::TY + reach > I.ny || (walls && y0 == 0))))) != 0;
    const bool wall = cx0 == 0 || cx0 + 4 >= I.nx || cy0 == 0 || cy0 + 1 >= I.ny;  // the wave has wall cells
    const bool xh = DIM == 2 || wave < 2;  // the wave has x-halo rows
    real c0[RPW];                           // the rows' c0 (wave-uniform)
    float chi[4], clo[4];                   // the cells' c0 - 1 as two-float sums
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        const real *E = params + (long long)__builtin_amdgcn_readfirstlane(rows[r].par) * g.pe;
        if constexpr (sizeof(real) == 4) {
            auto uni = [](float x) {
                return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
            };
            c0[r] = uni(E[0]);
            if (r < 4) {
                const double c = *reinterpret_cast<const double *>(E + 2) - 1.0;
                chi[r] = uni((float)c);
                clo[r] = uni((float)(c - (double)(float)c));
            }
        } else {
            c0[r] = E[0];
            if (r < 4) chi[r] = clo[r] = 0.0f;
        }
    }
    const real *base = src + I.f0;
    const uint32_t ibytes = (uint32_t)((long long)I.ncell * g.nv * sizeof(real));
    const __amdgpu_buffer_rsrc_t frs = make_rsrc(base, ibytes), ors = make_rsrc(dst + I.f0, ibytes);
    // (the instance's branch record, a byte per velocity; its address from I at
    // every store would be loaded again each time, the record may alias it)
    const __amdgpu_buffer_rsrc_t rrs = make_rsrc(REC ? A.rec + I.f0 : nullptr, REC ? ibytes / (uint32_t)sizeof(real) : 0u);
    const bool lim = I.minmod != 0;
    const uint32_t key = sizeof(real) == 4 ? pass_key(A.pass, 0) : 0u;
    const uint32_t zstep = (uint32_t)g.npl * (uint32_t)sizeof(real);
    const uint32_t lb = (uint32_t)lane * (uint32_t)sizeof(real);
    // LDS addresses: this lane's slot at the wave's first cell, halo rows
    const int cpos = DIM == 1 ? 4 * wave + 2 : ((wave >> 1) + 2) * S::PITCH + 4 * (wave & 1) + 2;
    const uint32_t aw = (uint32_t)cpos * RB + lb;
    const int yl = wave * S::YH / S::TX;
    const uint32_t ay = DIM == 1 ? 0u : (uint32_t)((yl < 2 ? yl : S::TY + yl) * S::PITCH + wave * S::YH - yl * S::TX + 2) * RB + lb;
    const uint32_t ax = (uint32_t)((DIM == 1 ? 0 : ((wave >> 1) + 2) * S::PITCH) + ((wave & 1) ? S::TX + 2 : 0)) * RB + lb;
    const uint32_t az = (uint32_t)(wave * RPW) * (uint32_t)(2 * sizeof(real));  // z-table column of the wave's first row

    const int npg = (g.npl + 63) >> 6;
    const int pg1 = (int)((long long)(ch + 1) * npg / A.vsplit);
    const float inv_nvx = 1.0f / (float)g.nvx;
    for (int pg = (int)((long long)ch * npg / A.vsplit); pg < pg1; ++pg) {
        const int pr = pg * 64 + lane, p = min(pr, g.npl - 1);
        const bool valid = pr < g.npl;
        const int jy = (int)(((float)p + 0.5f) * inv_nvx), jx = p - jy * g.nvx;
        const double vx = vnode(g, 0, jx), vy = vnode(g, 1, jy);
        const bool nx_ = !(vx > 0.0), ny_ = !(vy > 0.0);
        const real Cx = (real)(fabs(vx) * I.cx), Cy = (real)(fabs(vy) * I.cy);
        const real kx = lim ? (real)0.5 * ((real)1 - Cx) : (real)0, ky = lim ? (real)0.5 * ((real)1 - Cy) : (real)0;
        const uint32_t pb = (uint32_t)p * (uint32_t)sizeof(real);
        // upwind taps of this lane: k = -2, -1, +1 cells along x and y
        uint32_t xr[3], yr[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const int k = m == 0 ? -2 : m == 1 ? -1 : 1;
            xr[m] = aw + (uint32_t)((nx_ ? -k : k) * (int)RB);
            yr[m] = DIM == 1 ? aw : aw + (uint32_t)((ny_ ? -k : k) * (int)(S::PITCH * RB));
        }
        auto emits = [&](int code) {
            return (code == 2 && !nx_) || (code == 3 && nx_) || (code == 4 && !ny_) || (code == 5 && ny_);
        };
        real ha[RPW];  // h of the plane in flight
        auto load = [&](real (&h)[RPW], int z) {
            const uint32_t zo = (uint32_t)min(z, g.nvz - 1) * zstep;
#pragma unroll
            for (int r = 0; r < RPW; ++r) {
                if (r >= 4 + S::YH && !xh) continue;
                h[r] = buf_ld<real>(frs, pb, roff[r] + zo);
            }
        };
        load(ha, 0);
        int em = 0;  // rows whose ghost entry this lane takes
        real l1[RPW], l2[RPW];
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            const int par = __builtin_amdgcn_readfirstlane(rows[r].par);
            const real *E = params + (long long)par * g.pe;
            if (gm >> r & 1)
                if (emits(__builtin_amdgcn_readfirstlane(rows[r].code))) {
                    E = params + (long long)__builtin_amdgcn_readfirstlane(rows[r].gpar) * g.pe;
                    em |= 1 << r;
                }
            l1[r] = E[g.tx1 + jx] * E[g.ty1 + jy];
            l2[r] = E[g.tx2 + jx] * E[g.ty2 + jy];
        }
        double A0[4], Az[4], Azz[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) A0[i] = Az[i] = Azz[i] = 0.0;
        uint32_t hash[4];
        auto plane = [&](int z, real (&h)[RPW], auto odd_c, auto edge_c) {
            constexpr bool EDGE = decltype(edge_c)::value;
            constexpr uint32_t B = decltype(odd_c)::value ? BUF : 0u;
            constexpr bool ODD = decltype(odd_c)::value;
            const unsigned char *Z = zt + (uint32_t)z * ZR + az;
            real h0[4], u0[4], dm[4];
            // the rows' z-table pairs first (a read per row between the writes
            // would wait for each one's LDS latency)
            constexpr int HALF = (RPW + 1) / 2;
#pragma unroll
            for (int b0 = 0; b0 < RPW; b0 += HALF) {
            R2 ab[HALF];
#pragma unroll
            for (int q = 0; q < HALF && b0 + q < RPW; ++q) {
                const int r = b0 + q;
                const unsigned char *zp = Z + r * 2 * sizeof(real);
                if constexpr (sizeof(real) == 8) {
                    if (EDGE) zp += dcol[r] & ((em << (31 - r)) >> 31);
                } else if (EDGE && (gm >> r & 1)) {
                    const int d = __builtin_amdgcn_readfirstlane(rows[r].gcol) - (wave * RPW + r);
                    if (em >> r & 1) zp += d * 2 * (int)sizeof(real);
                }
                ab[q] = *reinterpret_cast<const R2 *>(zp);
            }
#pragma unroll
            for (int q = 0; q < HALF && b0 + q < RPW; ++q) {
                const int r = b0 + q;
                if (r >= 4 + S::YH && !xh) continue;
                const real M = l1[r] * ab[q][0] + l2[r] * ab[q][1];
                const real cr = EDGE && (em >> r & 1) ? (real)0 : c0[r];
                const real u = cr * h[r] + M;
                const uint32_t a = r < 4 ? aw + r * RB : r < 4 + S::YH ? ay + (r - 4) * RB : ax + (r - 4 - S::YH) * RB;
                *reinterpret_cast<real *>(smem + a + B) = u;
                if (r < 4) {
                    h0[r] = h[r];
                    u0[r] = u;
                    if constexpr (sizeof(real) == 4) dm[r] = __builtin_fmaf(chi[r], h[r], __builtin_fmaf(clo[r], h[r], M));
                }
            }
            }
            load(h, z + 1);
            __syncthreads();
            const double w1 = wt[2 * z], w2 = wt[2 * z + 1];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (EDGE && !out[i]) continue;
                auto lds = [&](uint32_t a) { return *reinterpret_cast<const real *>(smem + a + i * RB + B); };
                auto fdiff = [&](real um2, real um1, real up1, real k) {
                    const real d0 = u0[i] - um1;
                    return fmadd(k, minmod3(up1 - u0[i], d0) - minmod3(d0, um1 - um2), d0);
                };
                const real xm2 = lds(xr[0]), xm1 = lds(xr[1]), xp1 = lds(xr[2]);
                const real fx = fdiff(xm2, xm1, xp1, kx);
                real s = Cx * fx;
                real ym2 = 0, ym1 = 0, yp1 = 0, dy = 0;
                if constexpr (DIM == 2) {
                    ym2 = lds(yr[0]);
                    ym1 = lds(yr[1]);
                    yp1 = lds(yr[2]);
                    dy = Cy * fdiff(ym2, ym1, yp1, ky);
                }
                const uint32_t cb = roff[i] + (uint32_t)z * zstep;
                if constexpr (REC) {
                    const real d0 = u0[i] - xm1;
                    uint32_t code = mm_code<real>(d0, xm1 - xm2) | mm_code<real>(xp1 - u0[i], d0) << 2;
                    if constexpr (DIM == 2) {
                        const real e0 = u0[i] - ym1;
                        code |= (mm_code<real>(e0, ym1 - ym2) | mm_code<real>(yp1 - u0[i], e0) << 2) << 4;
                    }
                    __builtin_amdgcn_raw_buffer_store_b8((unsigned char)code, rrs, p, (int)(cb / (uint32_t)sizeof(real)), 0);
                }
                double rd;
                if constexpr (sizeof(real) == 4) {
                    s = DIM == 2 ? __builtin_fmaf(Cx, fx, dy) : s;
                    const float d = dm[i] - s;
                    // one hash per plane pair (even plane: low 16 bits)
                    if constexpr (!ODD) hash[i] = hash32((cb / 4u + (uint32_t)p) ^ key);
                    const uint32_t r16 = ODD ? hash[i] >> 16 : hash[i] & 0xffffu;
                    unsigned long long b = (unsigned long long)__double_as_longlong((double)h0[i] + (double)d);
                    b += (unsigned long long)r16 << 13;
                    b &= ~((1ull << 29) - 1ull);
                    rd = __longlong_as_double((long long)b);
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, (float)rd), ors, (int)pb, (int)cb,
                                                          NTSTORE ? 2 : 0);
                } else {
                    rd = u0[i] - s - dy;
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(vec_t<uint32_t, 2>, rd), ors, (int)pb, (int)cb,
                                                          NTSTORE ? 2 : 0);
                }
                A0[i] += rd;
                Az[i] = __builtin_fma(w1, rd, Az[i]);
                Azz[i] = __builtin_fma(w2, rd, Azz[i]);
            }
        };
        if (edge) {
            for (int z = 0; z < g.nvz; z += 2) {
                plane(z, ha, std::false_type{}, std::true_type{});
                if (z + 1 < g.nvz) plane(z + 1, ha, std::true_type{}, std::true_type{});
            }
        } else {
            for (int z = 0; z < g.nvz; z += 2) {
                plane(z, ha, std::false_type{}, std::false_type{});
                if (z + 1 < g.nvz) plane(z + 1, ha, std::true_type{}, std::false_type{});
            }
        }
        // the last plane's buffer may be read while the next group writes the
        // other one only if that is not the same buffer
        if (g.nvz & 1) __syncthreads();
        // fold into the cells' sums: the five moments, and for wall cells the
        // half-range fluxes (nothing reads those of other cells)
        const double fvx = vnode(g, 0, jx), fvy = vnode(g, 1, jy);
        double v[4][NACC];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (!valid) A0[i] = Az[i] = Azz[i] = 0.0;
            double t[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) t[q] = 0.0;
            if (g.red) fold_column(t, fvx, fvy, Az[i], 0.0, Azz[i]);
            else fold_column(t, fvx, fvy, A0[i], Az[i], Azz[i]);
#pragma unroll
            for (int q = 0; q < NACC; ++q) v[i][q] = t[q];
        }
        double mine = 0.0;
        auto total = [&](int q) {
            const double s = wave_sum<16>(swap_add16(swap_add32(v[0][q], v[1][q]), swap_add32(v[2][q], v[3][q])));
            if ((lane & 15) == q) mine = s;
        };
#pragma unroll
        for (int q = 0; q < 5; ++q) total(q);
        if (wall)
#pragma unroll
            for (int q = 5; q < NACC; ++q) total(q);
        if ((lane & 15) < NACC) s_acc[4 * wave + tile_row_cell(lane >> 4)][lane & 15] += mine;
    }
    {
        const int i = tile_row_cell(lane >> 4), q = lane & 15;
        const bool in = cy0 < I.ny && cx0 + i < I.nx;
        if (in && q < NQ) {
            const long long gc = I.cell0 + (long long)cy0 * I.nx + cx0 + i;
            partial[(gc * A.vsplit + ch) * NQ + q] = q < NACC ? s_acc[4 * wave + i][q] : 0.0;
        }
    }
}

// ---------------------------------------------------------------- three dimensions
// The same on tiles of 4 x 4 x 4 cells, float: wave w holds two x lines (y, z)
// = (2 (w & 1) + ln, w >> 1) of the tile and relaxes 16 rows a line and plane:
// its four cells, two halo cells on either side of the line, and four cells
// each of one line of the y and z halos.  64 + 192 relaxed values for 64
// outputs, 4 relaxations per output instead of 10.  Eight waves of 250
// registers (the rows' Maxwellian factors, the loads in flight and the FP64
// sums of 8 cells; with 16 waves of 4 cells a third of them spills) and one LDS
// plane (64 KB; two do not fit beside the z tables), so two barriers a plane.
// Tiles at a boundary (EDGE) and inner ones run as kernels of their own: the
// ghosts' selection compiled into one kernel with the inner path spills both.
// Bound by the issue of vector instructions (53 to 60 per output, 55% of the
// cycles at two waves a SIMD) and the barriers.  48^3 cells x 16^3 FP32: 1.03 ms
// (1000 inner tiles) + 1.04 (728 at the walls) a pass, 3.55 in k_stream;
// 48^3 x 12^3 a step 1.30 ms, 3.97; 36 x 28 x 32 x 20^3 1.71, 2.29.
struct Tile3 {
    static constexpr int T = 4, NW = 8, RPW = 32, NROW = NW * RPW;  // cells per side, waves, rows
    // LDS positions: the lines' 8 cells each, then the y and the z halo lines
    static constexpr int YH = 128, ZH = 192, NPOS = 256;
};

// Tiles along an axis of n cells whose halo lies inside (the second to the
// last but one or two).
__host__ __device__ inline int tile3_inner(int n) { return n < 10 ? 0 : (n - 6) / 4; }

// (edge: z tables of two entries a row, the cell's and its ghost's)
__host__ __device__ inline TileLds tile3_lds(const Geo &g, bool edge)
{
    TileLds L;
    L.zt = (size_t)Tile3::NPOS * 64 * sizeof(float);
    L.w = L.zt + (size_t)g.nvz * Tile3::NROW * (edge ? 4 : 2) * sizeof(float);
    L.w = (L.w + 15) & ~(size_t)15;
    L.total = L.w + (size_t)2 * g.nvz * sizeof(double);
    return L;
}

template <bool NTSTORE, bool EDGE>
__global__ void __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
    k_tile3(Args A, const float *__restrict__ src, float *__restrict__ dst, const float *__restrict__ params,
            double *__restrict__ partial)
{
    using S = Tile3;
    using R2 = vec_t<float, 2>;
    constexpr int RPW = S::RPW, NTH = 64 * S::NW;
    constexpr uint32_t RB = 64 * sizeof(float);          // bytes of one position
    constexpr uint32_t ZC = (EDGE ? 4 : 2) * sizeof(float), ZR = S::NROW * ZC;  // bytes of one row and one plane of the z tables
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ TileRow s_row[S::NROW];
    __shared__ double s_acc[S::T * S::T * S::T][NQ];
    __shared__ __align__(16) float s_c0[S::NROW];
    __shared__ __align__(16) uint32_t s_off[S::NROW];
    const Geo &g = A.g;
    const TileLds Lo = tile3_lds(g, EDGE);
    unsigned char *const zt = smem + Lo.zt;
    double *const wt = reinterpret_cast<double *>(smem + Lo.w);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nitems = A.nttiles * A.vsplit;
    const int Lq = xcd_remap(blockIdx.x, nitems);
    int tq, ch;
    {
        constexpr int SB = 64;  // tiles of a superblock, walked chunk by chunk
        const int sb = Lq / (SB * A.vsplit), c0 = sb * SB, n = min(SB, A.nttiles - c0), k = Lq - c0 * A.vsplit;
        ch = k / n;
        tq = c0 + (k - ch * n);
    }
    auto first = [&](int i) { return EDGE ? A.inst[i].ttile0 : A.inst[i].itile0; };
    int lo = 0, hi = A.ninst;  // first(lo) <= tq < first(hi)
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first(mid) <= tq) lo = mid; else hi = mid;
    }
    const Inst &I = A.inst[lo];
    const int tpr = (I.nx + 3) / 4, tpc = (I.ny + 3) / 4;
    const int ix = tile3_inner(I.nx), iy = tile3_inner(I.ny), iz = tile3_inner(I.nz);
    int tx, ty, tz, q = tq - first(lo);
    if constexpr (!EDGE) {  // the inner box, in strips four tiles wide layer by layer
        tz = 1 + q / (ix * iy);
        const int tt = strip_tile(q - (tz - 1) * ix * iy, ix, iy, 4);
        ty = 1 + tt / ix;
        tx = 1 + tt - (ty - 1) * ix;
    } else {  // layer by layer, row by row: all but the inner box
        const bool box = ix > 0 && iy > 0 && iz > 0;
        const int tl = tpr * tpc, ring = box ? tl - ix * iy : tl, il = box ? iz : 0;
        if (q < tl) tz = 0;
        else if (q < tl + il * ring) { tz = 1 + (q - tl) / ring; q -= tl + (tz - 1) * ring; }
        else { tz = 1 + il + (q - tl - il * ring) / tl; q -= tl + il * ring + (tz - 1 - il) * tl; }
        if (tz < 1 || tz > il || q < tpr) { ty = q / tpr; tx = q - ty * tpr; }
        else if (q < tpr + iy * (tpr - ix)) {
            ty = 1 + (q - tpr) / (tpr - ix);
            tx = q - tpr - (ty - 1) * (tpr - ix);
            if (tx > 0) tx += ix;
        } else {
            q -= tpr + iy * (tpr - ix);
            ty = 1 + iy + q / tpr;
            tx = q - (ty - 1 - iy) * tpr;
        }
    }
    const int x0 = tx * 4, y0 = ty * 4, z0 = tz * 4;

    // ---- rows and tables of the tile
    for (int r = tid; r < S::NROW; r += NTH) {
        const int w = r / 16, k = r - w * 16, hl = (w & 3) < 2 ? (w & 3) - 2 : (w & 3) + 2, hz = (w >> 2) < 2 ? (w >> 2) - 2 : (w >> 2) + 2;
        const int px = k < 4 ? k : k < 8 ? (k < 6 ? k - 6 : k - 2) : k & 3;
        const int py = k >= 8 && k < 12 ? hl : w & 3, pz = k >= 12 ? hz : w >> 2;
        const int x = x0 + px, y = y0 + py, z = z0 + pz;
        const bool ox = x < 0 || x >= I.nx, oy = y < 0 || y >= I.ny, oz = z < 0 || z >= I.nz;
        // (positions never read as such, outside along a direction in which no
        // cell of the tile reads them, are the clamped cell)
        int cx = min(max(x, 0), I.nx - 1), cy = min(max(y, 0), I.ny - 1), cz = min(max(z, 0), I.nz - 1);
        TileRow t;
        t.gpar = -1;
        t.gcol = 0;
        t.code = 0;
        const int dim = inst_dim(I);
        if (I.kind == KIND_PER1 || I.kind == KIND_PER2 || I.kind == KIND_PER3) {
            cx = (x % I.nx + I.nx) % I.nx;
            if (dim >= 2) cy = (y % I.ny + I.ny) % I.ny;
            if (dim >= 3) cz = (z % I.nz + I.nz) % I.nz;
        } else if (I.kind == KIND_SHOCK) {
            if (ox && k < 8) {
                t.gpar = I.pseudo0 + (x < 0 ? 0 : 1);
                t.code = 1;
            }
        } else if ((int)ox + (int)oy + (int)oz == 1 && (ox ? k < 8 : oy ? k < 4 || (k >= 8 && k < 12) : k < 4 || k >= 12) &&
                   !(oz && dim < 3)) {
            const int wl = ox ? (x < 0 ? 0 : 1) : oy ? (y < 0 ? 2 : 3) : (z < 0 ? 4 : 5);
            const int face = ox ? cz * I.ny + cy : oy ? cz * I.nx + cx : cy * I.nx + cx;
            t.gpar = I.pseudo0 + wall_offset(I, wl) + face;
            t.code = wl + 2;
        }
        const int cell = (cz * I.ny + cy) * I.nx + cx;
        t.par = I.cell0 + cell;
        t.off = (uint32_t)cell * (uint32_t)g.nv * (uint32_t)sizeof(float);
        s_row[r] = t;
        s_c0[r] = params[(long long)t.par * g.pe];
        s_off[r] = t.off;
    }
    for (int k = tid; k < g.nvz; k += NTH) {
        const ZW w = zweights(g, k);
        wt[2 * k] = w.z;
        wt[2 * k + 1] = w.zz;
    }
    for (int k = tid; k < S::T * S::T * S::T * NQ; k += NTH) (&s_acc[0][0])[k] = 0.0;
    __syncthreads();
    {
        const float inv = 1.0f / (float)g.nvz;
        for (int t = tid; t < S::NROW * g.nvz; t += NTH) {
            const int r = (int)(((float)t + 0.5f) * inv), z = t - r * g.nvz;
            const TileRow &row = s_row[r];
            const float *E = params + (long long)row.par * g.pe + g.tz + 2 * z;
            *reinterpret_cast<R2 *>(zt + z * ZR + r * ZC) = *reinterpret_cast<const R2 *>(E);
            if constexpr (EDGE) {
                const float *G = row.code ? params + (long long)row.gpar * g.pe + g.tz + 2 * z : E;
                *reinterpret_cast<R2 *>(zt + z * ZR + r * ZC + sizeof(R2)) = *reinterpret_cast<const R2 *>(G);
            }
        }
    }
    __syncthreads();

    // ---- this wave's rows
    int gm = 0, zm = 0;     // rows with a ghost part; those across z
    bool out[8];            // cells inside the instance
    const TileRow *const rows = s_row + wave * RPW;
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        const int code = __builtin_amdgcn_readfirstlane(rows[r].code);
        if (code) gm |= 1 << r;
        if (code >= 6) zm |= 1 << r;
    }
    // lines 2 wave and 2 wave + 1 of the tile: y = wy + ln, z = wz
    const int wy = 2 * (wave & 1), wz = wave >> 1, gy = y0 + wy, gz = z0 + wz;
    const int hy = y0 + (wy < 2 ? wy - 2 : wy + 2), hz = z0 + (wz < 2 ? wz - 2 : wz + 2);  // its halo lines (y and z)
    float chi[8], clo[8];   // the cells' c0 - 1 as two-float sums
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        out[i] = gz < I.nz && gy + (i >> 2) < I.ny && x0 + (i & 3) < I.nx;
        const float *E = params + (long long)__builtin_amdgcn_readfirstlane(rows[16 * (i >> 2) + (i & 3)].par) * g.pe;
        auto uni = [](float x) {
            return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
        };
        const double c = *reinterpret_cast<const double *>(E + 2) - 1.0;
        chi[i] = uni((float)c);
        clo[i] = uni((float)(c - (double)(float)c));
    }
    // byte offsets of h in the instance: the wave's first line, and the lines of
    // its halo rows (interior tiles, where each is four cells in a row)
    const uint32_t cs = (uint32_t)g.nv * (uint32_t)sizeof(float), ls = (uint32_t)I.nx * cs;
    auto cell_at = [&](int y, int z) { return (uint32_t)((z * I.ny + y) * I.nx + x0) * cs; };
    const uint32_t o0 = cell_at(gy, gz), oy = cell_at(hy, gz), oz = cell_at(gy, hz);
    const uint32_t ibytes = (uint32_t)((long long)I.ncell * g.nv * sizeof(float));
    const __amdgpu_buffer_rsrc_t frs = make_rsrc(src + I.f0, ibytes), ors = make_rsrc(dst + I.f0, ibytes);
    const bool lim = I.minmod != 0;
    const double czz = I.cz;
    const uint32_t key = pass_key(A.pass, 0);
    const uint32_t zstep = (uint32_t)g.npl * (uint32_t)sizeof(float);
    const uint32_t lb = (uint32_t)lane * (uint32_t)sizeof(float);
    // LDS addresses: this lane's slot at the wave's first cell, its halo rows
    const uint32_t aw = (uint32_t)(wave * 16 + 2) * RB + lb;
    const uint32_t ay = (uint32_t)(S::YH + wave * 8) * RB + lb, az = (uint32_t)(S::ZH + wave * 8) * RB + lb;
    auto yat = [&](int ln, int k) {  // the line's neighbour at y + k
        const int q = wy + ln + k;
        const int p = q >= 0 && q < 4 ? (wz * 4 + q) * 8 + 2 : S::YH + (wz * 4 + (q < 0 ? q + 2 : q - 2)) * 4;
        return (uint32_t)p * RB + lb;
    };
    auto zat = [&](int ln, int k) {  // at z + k
        const int q = wz + k;
        const int p = q >= 0 && q < 4 ? (q * 4 + wy + ln) * 8 + 2 : S::ZH + ((q < 0 ? q + 2 : q - 2) * 4 + wy + ln) * 4;
        return (uint32_t)p * RB + lb;
    };
    const uint32_t zcol = (uint32_t)(wave * RPW) * ZC;  // z-table place of the wave's first row

    const int npg = (g.npl + 63) >> 6;
    const int pg1 = (int)((long long)(ch + 1) * npg / A.vsplit);
    const float inv_nvx = 1.0f / (float)g.nvx;
    for (int pg = (int)((long long)ch * npg / A.vsplit); pg < pg1; ++pg) {
        const int pr = pg * 64 + lane, p = min(pr, g.npl - 1);
        const bool valid = pr < g.npl;
        const int jy = (int)(((float)p + 0.5f) * inv_nvx), jx = p - jy * g.nvx;
        const double vx = vnode(g, 0, jx), vy = vnode(g, 1, jy);
        const bool nx_ = !(vx > 0.0), ny_ = !(vy > 0.0);
        const float Cx = (float)(fabs(vx) * I.cx), Cy = (float)(fabs(vy) * I.cy);
        const float kx = lim ? 0.5f * (1.0f - Cx) : 0.0f, ky = lim ? 0.5f * (1.0f - Cy) : 0.0f;
        const uint32_t pb = (uint32_t)p * (uint32_t)sizeof(float);
        // upwind taps of this lane: k = -2, -1, +1 cells along x and y (those
        // along z follow the plane's sign)
        uint32_t xr[3], yr[2][3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const int k = m == 0 ? -2 : m == 1 ? -1 : 1;
            xr[m] = aw + (uint32_t)((nx_ ? -k : k) * (int)RB);
            yr[0][m] = ny_ ? yat(0, -k) : yat(0, k);
            yr[1][m] = ny_ ? yat(1, -k) : yat(1, k);
        }
        float ha[RPW];  // h of the plane in flight
        // (an address that the compiler takes for new at each plane: it otherwise
        // keeps the loop-invariant table entries read from it in registers)
        auto fresh = [](uint32_t o) {
            asm volatile("" : "+v"(o));
            return o;
        };
        auto load = [&](int z) {
            const uint32_t zo = (uint32_t)min(z, g.nvz - 1) * zstep;
            const uint32_t *const off = s_off + fresh((uint32_t)(wave * RPW));
#pragma unroll
            for (int r = 0; r < RPW; ++r) {
                if constexpr (EDGE) {
                    ha[r] = buf_ld<float>(frs, pb + off[r], zo);
                } else {
                    const int k = r & 15;
                    const uint32_t o = (k < 4 ? o0 + k * cs : k < 6 ? o0 - (6 - k) * cs : k < 8 ? o0 + (k - 2) * cs
                                        : k < 12 ? oy + (k - 8) * cs : oz + (k - 12) * cs) + (r >> 4) * ls;
                    ha[r] = buf_ld<float>(frs, pb, o + zo);
                }
            }
        };
        load(0);
        int em = 0;  // rows whose ghost entry this lane takes
        float l1[RPW], l2[RPW];
        auto entry = [&](int r, bool zpos) {
            const float *E = params + (long long)__builtin_amdgcn_readfirstlane(rows[r].par) * g.pe;
            em &= ~(1 << r);
            if (gm >> r & 1) {
                const int code = __builtin_amdgcn_readfirstlane(rows[r].code);
                if (code == 1 || (code == 2 && !nx_) || (code == 3 && nx_) || (code == 4 && !ny_) || (code == 5 && ny_) ||
                    (code == 6 && zpos) || (code == 7 && !zpos)) {
                    E = params + (long long)__builtin_amdgcn_readfirstlane(rows[r].gpar) * g.pe;
                    em |= 1 << r;
                }
            }
            l1[r] = E[g.tx1 + jx] * E[g.ty1 + jy];
            l2[r] = E[g.tx2 + jx] * E[g.ty2 + jy];
        };
#pragma unroll
        for (int r = 0; r < RPW; ++r) entry(r, g.zneg == 0);
        double A0[8], Az[8], Azz[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) A0[i] = Az[i] = Azz[i] = 0.0;
        // the sum over the wave's lanes of four cells' values, one per 16-lane row
        auto sum4 = [&](double a, double b, double c, double d) {
            return wave_sum<16>(swap_add16(swap_add32(a, b), swap_add32(c, d)));
        };
        double *const acc = s_acc[8 * wave + tile_row_cell(lane >> 4)];  // (line 1: 4 NQ further)
        uint32_t hash[8];
        auto plane = [&](int z, auto odd_c) {
            constexpr bool ODD = decltype(odd_c)::value;
            if (z == g.zneg) {  // from here on v_z > 0
                if (EDGE) {  // the half-range flux of v_z < 0
#pragma unroll
                    for (int ln = 0; ln < 2; ++ln) {
                        const double *a = Az + 4 * ln;
                        const double s = sum4(valid ? a[0] : 0.0, valid ? a[1] : 0.0, valid ? a[2] : 0.0, valid ? a[3] : 0.0);
                        if ((lane & 15) == 9) acc[4 * NQ * ln + 9] -= s;
                    }
                }
                if (EDGE && zm)
#pragma unroll
                    for (int r = 0; r < RPW; ++r)
                        if (zm >> r & 1) entry(r, true);
            }
            const bool zpos = z >= g.zneg;
            const unsigned char *Z = zt + (uint32_t)z * ZR + zcol;
            float h0[8], dm[8];
            using R4 = vec_t<float, 4>;
#pragma unroll
            for (int b0 = 0; b0 < RPW; b0 += 4) {
                __builtin_amdgcn_sched_barrier(0);  // (all rows' table values at once would not fit the registers)
                R2 ab[4];
                const R4 c0 = *reinterpret_cast<const R4 *>(s_c0 + wave * RPW + b0);
                int gh[4];  // all bits set: this lane takes the row's ghost entry
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int r = b0 + q;
                    gh[q] = EDGE ? (em << (31 - r)) >> 31 : 0;
                    ab[q] = *reinterpret_cast<const R2 *>(Z + r * ZC - gh[q] * (int)sizeof(R2));
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int r = b0 + q;
                    const float M = l1[r] * ab[q][0] + l2[r] * ab[q][1];
                    const float cq = c0[q];  // (0 for a ghost)
                    const float cr = EDGE ? __builtin_bit_cast(float, __builtin_bit_cast(int, cq) & ~gh[q]) : cq;
                    if ((r & 15) < 4) {
                        const int i = (r >> 4) * 4 + (r & 3);
                        h0[i] = ha[r];
                        dm[i] = __builtin_fmaf(chi[i], ha[r], __builtin_fmaf(clo[i], ha[r], M));
                    }
                    ha[r] = cr * ha[r] + M;  // (h becomes u)
                }
            }
            __syncthreads();  // the previous plane's values are read
#pragma unroll
            for (int r = 0; r < RPW; ++r) {
                const int k = r & 15, ln = r >> 4;
                const uint32_t a = k < 4 ? aw + (8 * ln + k) * RB : k < 6 ? aw + (8 * ln + k - 6) * RB : k < 8 ? aw + (8 * ln + k - 2) * RB
                                 : k < 12 ? ay + (4 * ln + k - 8) * RB : az + (4 * ln + k - 12) * RB;
                *reinterpret_cast<float *>(smem + a) = ha[r];
            }
            load(z + 1);
            __syncthreads();
            const double w1 = wt[2 * z], w2 = wt[2 * z + 1];
            const float Cz = (float)(fabs(w1) * czz), kz = lim ? 0.5f * (1.0f - Cz) : 0.0f;
            uint32_t zr[2][3];
#pragma unroll
            for (int ln = 0; ln < 2; ++ln) {
                zr[ln][0] = zpos ? zat(ln, -2) : zat(ln, 2);
                zr[ln][1] = zpos ? zat(ln, -1) : zat(ln, 1);
                zr[ln][2] = zpos ? zat(ln, 1) : zat(ln, -1);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                constexpr uint32_t LB = 8 * RB;  // from line to line
                const int ln = i >> 2, x = i & 3;
                if (x % 2 == 0) __builtin_amdgcn_sched_barrier(0);
                auto lds = [&](uint32_t a) { return *reinterpret_cast<const float *>(smem + a + x * RB); };
                const float u0 = lds(aw + ln * LB);
                auto fdiff = [&](float um2, float um1, float up1, float k) {
                    const float d0 = u0 - um1;
                    return fmadd(k, minmod3(up1 - u0, d0) - minmod3(d0, um1 - um2), d0);
                };
                const float fx = fdiff(lds(xr[0] + ln * LB), lds(xr[1] + ln * LB), lds(xr[2] + ln * LB), kx);
                float dy = Cy * fdiff(lds(yr[ln][0]), lds(yr[ln][1]), lds(yr[ln][2]), ky);
                dy = __builtin_fmaf(Cz, fdiff(lds(zr[ln][0]), lds(zr[ln][1]), lds(zr[ln][2]), kz), dy);
                const uint32_t cb = o0 + ln * ls + x * cs + (uint32_t)z * zstep;
                const float d = dm[i] - __builtin_fmaf(Cx, fx, dy);
                // one hash per plane pair (even plane: low 16 bits)
                if constexpr (!ODD) hash[i] = hash32((cb / 4u + (uint32_t)p) ^ key);
                const uint32_t r16 = ODD ? hash[i] >> 16 : hash[i] & 0xffffu;
                unsigned long long b = (unsigned long long)__double_as_longlong((double)h0[i] + (double)d);
                b += (unsigned long long)r16 << 13;
                b &= ~((1ull << 29) - 1ull);
                const double rd = __longlong_as_double((long long)b);
                if (!EDGE || out[i])
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, (float)rd), ors, (int)pb, (int)cb,
                                                          NTSTORE ? 2 : 0);
                A0[i] += rd;
                Az[i] = __builtin_fma(w1, rd, Az[i]);
                Azz[i] = __builtin_fma(w2, rd, Azz[i]);
            }
        };
        for (int z = 0; z < g.nvz; z += 2) {
            plane(z, std::false_type{});
            if (z + 1 < g.nvz) plane(z + 1, std::true_type{});
        }
        // fold into the cells' sums: the five moments, and for wall cells the
        // half-range fluxes (nothing reads those of other cells)
        const double fvx = vnode(g, 0, jx), fvy = vnode(g, 1, jy);
#pragma unroll
        for (int ln = 0; ln < 2; ++ln) {
            double v[4][NQ];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int i = 4 * ln + x;
                if (!valid) A0[i] = Az[i] = Azz[i] = 0.0;
#pragma unroll
                for (int q = 0; q < NQ; ++q) v[x][q] = 0.0;
                // (9: added where v_z changes sign; 10: completed when written)
                fold_column(v[x], fvx, fvy, A0[i], Az[i], Azz[i], 0.0, Az[i]);
            }
            double mine = 0.0;
            auto total = [&](int q) {
                const double s = sum4(v[0][q], v[1][q], v[2][q], v[3][q]);
                if ((lane & 15) == q) mine = s;
            };
#pragma unroll
            for (int q = 0; q < 5; ++q) total(q);
            if (EDGE)
#pragma unroll
                for (int q = 5; q < NQ; ++q)
                    if (q != 9) total(q);
            if ((lane & 15) < NQ) acc[4 * NQ * ln + (lane & 15)] += mine;
        }
    }
    // (lane 10 of a row completes its sum with the one that lane 9 left in LDS)
    __syncthreads();
#pragma unroll
    for (int ln = 0; ln < 2; ++ln) {
        const int i = tile_row_cell(lane >> 4), q = lane & 15;
        if (q < NQ && gz < I.nz && gy + ln < I.ny && x0 + i < I.nx) {
            const long long gc = I.cell0 + ((long long)gz * I.ny + gy + ln) * I.nx + x0 + i;
            const double *s = s_acc[8 * wave + 4 * ln + i];
            // (no plane with v_z > 0: slot 9 was never split off, all of slot 10 is its)
            partial[(gc * A.vsplit + ch) * NQ + q] = q < 9 ? s[q] : g.zneg < g.nvz ? (q == 10 ? s[10] + s[9] : s[9])
                                                     : q == 9 ? -s[10] : 0.0;
        }
    }
}

}  // namespace bgk
