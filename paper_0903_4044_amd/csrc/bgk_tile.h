// bgk_tile.h -- the streaming kernel on tiles of cells (k_tile), for one- and
// two-dimensional kinds.  Same pass, inputs and outputs as k_stream (see
// bgk_device.h); there every cell relaxes the 4 or 7 stencil inputs of each
// velocity itself, here a workgroup relaxes each cell of a tile and of its
// halo once and the stencils read the relaxed values from LDS.
//
// Bound by the issue of vector instructions: k_stream spends ~76 per element
// on 2D grids, most of them on the seven relaxations and their table loads;
// here a plane of 64 (jx, jy) of 4 cells takes ~180 (45 per element) with the
// loads of the next plane in flight.  128^2 x 24^3 FP32: 510 us a pass for the
// 1.81 GB of f (3.5 TB/s), 790 in k_stream; 160^2 x 20^3 595 (2.8 TB/s), 1096;
// 48 cavities of up to 160^2 8.4 ms, 13.2; 48^2 x 24^3 FP64 159 us (3.2 TB/s),
// 272; 1024 x 48^3 FP32 217 us (4.2 TB/s), 272; recording on 64^2 x 24^3
// FP32 201, 231.
#pragma once

#include "bgk_device.h"

namespace bgk {

// A tile is TX x TY cells, four consecutive cells of a row per wave.  The LDS
// plane holds the tile and two halo cells on every side, position
// (y + 2 HY) * PITCH + x + 2; each position holds one value per lane.
// Waves per workgroup: in 2D the halo of 8 x 8 cells doubles the relaxed
// values, that of 8 x 4 cells makes it 2.5 times (float: 519 against 577 us a
// step on 128^2 x 24^3); in FP64 the two LDS planes of 8 x 8 cells and the
// registers of 16 waves do not fit.  In 1D the halo is small and the short
// workgroups balance better (1024 x 48^3: 224 us a step with 4 waves, 240
// with 8, 255 with 16).
template <typename real, int DIM>
struct TileShape {
    static constexpr int NW = DIM == 1 ? 4 : sizeof(real) == 4 ? 16 : 8;
    static constexpr int TX = DIM == 1 ? 4 * NW : 8, TY = DIM == 1 ? 1 : NW / 2;
    static constexpr int HY = DIM == 1 ? 0 : 2;
    static constexpr int PITCH = TX + 4, NPOS = PITCH * (TY + 2 * HY);
    // rows of a wave: four cells, YH y-halo positions (2D; the 4 TX of them
    // shared out evenly), two x-halo positions
    static constexpr int YH = DIM == 1 ? 0 : 4 * TX / NW, RPW = 4 + YH + 2, NROW = NW * RPW;
    static constexpr int NG = 2 * TY + (DIM == 1 ? 0 : 2 * TX);  // ghost entries of a tile: left, right, bottom, top faces
    static constexpr int NZT = NROW + NG + (NROW + NG) % 2;      // z-table columns
};

// One row of a tile: the cell whose h is read (offset in the instance, in
// elements) and the entry that relaxes it; at a ghost position also the ghost
// entry's z-table column and the velocities that take it (code: 0 none, 1 all,
// 2 v_x > 0, 3 v_x <= 0, 4 v_y > 0, 5 v_y <= 0).
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
            if (ox) {
                t.gpar = I.pseudo0 + (x < 0 ? 0 : 1);
                t.gcol = S::NROW + (x < 0 ? 0 : S::TY);
                t.code = 1;
            }
        } else if (ox ? !oy && py >= 0 && py < S::TY : oy && px >= 0 && px < S::TX) {
            const int wl = ox ? (x < 0 ? 0 : 1) : (y < 0 ? 2 : 3);
            t.gpar = I.pseudo0 + wall_offset(I, wl) + (ox ? cy : cx);
            t.gcol = S::NROW + (wl == 0 ? py : wl == 1 ? S::TY + py : wl == 2 ? 2 * S::TY + px : 2 * S::TY + S::TX + px);
            t.code = wl + 2;
        }
        t.par = I.cell0 + cy * I.nx + cx;
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
    bool out[4];            // cells inside the instance
    const TileRow *const rows = s_row + wave * RPW;
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        roff[r] = __builtin_amdgcn_readfirstlane(rows[r].off) * (uint32_t)sizeof(real);
        if (__builtin_amdgcn_readfirstlane(rows[r].code)) gm |= 1 << r;
    }
    const int cx0 = x0 + (DIM == 1 ? 4 * wave : 4 * (wave & 1)), cy0 = y0 + (DIM == 1 ? 0 : wave >> 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = cy0 < I.ny && cx0 + i < I.nx;
    const bool edge = gm != 0 || !(out[0] && out[1] && out[2] && out[3]);
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
            return code == 1 || (code == 2 && !nx_) || (code == 3 && nx_) || (code == 4 && !ny_) || (code == 5 && ny_);
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
                if (EDGE && (gm >> r & 1)) {
                    const int dcol = __builtin_amdgcn_readfirstlane(rows[r].gcol) - (wave * RPW + r);
                    if (em >> r & 1) zp += dcol * 2 * (int)sizeof(real);
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

}  // namespace bgk
