// Cell sweeps: MicSA on bit planes with a row's 32 sites of one parity in
// one register, several sweeps per launch, the neighbours exchanged through
// LDS.  One form serves a whole small lattice per work-group (any number of
// sweeps per launch) and tiles of a large one (T sweeps per launch, rings
// recomputed), for any row length.
//
// Planes (per lattice; cell = row * W + w, row = y + Ly z, W = ceil(Kx / 32)
// words per row and parity; bit b of word w is site k = 32 w + b of the
// row's parity-p sites, x = 2k + ((p + y + z) & 1)):
//   spin[l][p][cell]         dem0/dem1[l][p][cell]  the daemon level's bits
//   bond[l / bdiv][d][cell]  coupling of the even site's bond in direction d
// With Lx a multiple of 128 these are the multispin planes (msc_kernels.hpp)
// read as 32-bit words.
//
// A thread owns NR cells for the whole launch: both parities' spins, the
// level bits and all twelve coupling words (six of the even sites, six of
// the odd ones, gathered once) stay in registers.  A half sweep reads four
// LDS words (the rows y +- 1 and z +- 1 of the other parity; the x
// neighbours are the thread's own word and the same word rotated, or one
// more LDS word where a row has several), runs the bit-sliced Creutz move
// (24 three-input operations for 32 sites) and publishes one word; one
// barrier per half sweep.
//
// Tiles.  A work-group owns TY rows x TZ planes and computes on EY x EZ,
// GY = 2T (or 0: the whole side, periodic) more rows on each side and GZ
// planes likewise: half sweep h of the launch is right on all but the outer
// h + 1 rows and planes, so the owned ones are right after 2T.  Rows and
// planes at the edge read themselves in place of a neighbour they do not
// have; nobody uses what that gives.
//
// Walkers (Sec. 2.6).  With one per site the wandering is along x: a row's
// levels move by 0 or 1 site into the other parity's words, in registers,
// the bits that cross from word to word exchanged through LDS.  With several
// families (Sec. 2.8; also several daemons per site) a launch covers at most
// one sweep of each: a family's levels are loaded for its sweep, displaced by
// the wandering it owes since its last one, and stored after it, so that no
// wandering is a pass of its own.
//
// Refresh levels (Sec. 2.7) depend on the refresh index and temperature
// only: k_cells_draw draws those of many refreshes in one launch on the
// whole device, and the sweep reads them (loaded a refresh ahead).
//
// Bound: instruction issue where the device is full (a half of 32 sites is
// about 36 VALU instructions per wave, 24 of them the move), else the chain
// of one half: LDS reads, the move, the write, a barrier, 0.12 us with one
// wave and 0.25 us with sixteen.  Measured against the byte-wise LDS sweeps
// this replaced (us per sweep, refreshes left out, one MI355X): 8^3 0.25
// (4.5), 16^3 0.32, with a logged row 0.36 (4.2), 64 x 32^3 0.52 (9.9), 256 x
// 64^3 1.7 = 39600 updates/ns; against one or two byte sweeps per launch: 64^3 x
// 2 1.19 (3.6), 104 x 90 x 70 x 4 2.56 (10.5).  The VALU is busy 67 % of a launch
// of 512 lattices of 32^3, 39 % of 256^3 (where waves wait 64 % of their time
// for memory, LDS and barriers) and 19 % of 64^3 x 2 (128 work-groups of short
// launches).  Four cells per thread do not fit 128 registers: 1 to 21 spill,
// up to 57 with a walker per site, so that plans take three there for long calls
// of rows of several words (three spill 10 to 23).
#pragma once
#include "bitplane_kernels.hpp"
#include "byte_kernels.hpp"

namespace micsa {

constexpr int kCellLanes = 1024;   // work-group size at most
constexpr int kCellMaxNR = 4;      // cells per thread at most

struct CellGeom {
    Geom g;
    int32_t W;      // words per row and parity
    int32_t bdiv;   // lattices that share one set of coupling planes (consecutive ones)
    int64_t plane;  // cells = rows * W
};

__device__ __forceinline__ uint32_t cell_mask(int nv) { return nv >= 32 ? 0xFFFFFFFFu : (1u << nv) - 1u; }

// ------------------------------------------------------ 32-site Creutz move
__device__ __forceinline__ uint32_t maj32(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}

// The Creutz move on 32 sites: u[0..5] are the unsatisfied-bond
// bits; returns the accepted flips and updates the level bits.
__device__ __forceinline__ uint32_t cell_move(const uint32_t (&u)[6], uint32_t& m0, uint32_t& m1)
{
    const uint32_t s1 = xor3(u[0], u[1], u[2]), c1 = maj32(u[0], u[1], u[2]);
    const uint32_t s2 = xor3(u[3], u[4], u[5]), c2 = maj32(u[3], u[4], u[5]);
    const uint32_t k0 = s1 & s2;
    const uint32_t u1 = xor3(c1, c2, k0), u2 = maj32(c1, c2, k0);
    const uint32_t x0 = __builtin_amdgcn_bitop3_b32(s1, m0, s2, 0x69);   // ~(m0 ^ s1 ^ s2) = ~w0
    const uint32_t cw0 = __builtin_amdgcn_bitop3_b32(s1, m0, s2, 0x48);  // m0 & (s1 ^ s2)
    const uint32_t w1 = xor3(m1, u1, cw0), cw1 = maj32(m1, u1, cw0);
    const uint32_t p = __builtin_amdgcn_bitop3_b32(w1, x0, w1, 0x30);    // w1 & w0
    const uint32_t r = __builtin_amdgcn_bitop3_b32(w1, x0, w1, 0xF3);    // w1 | w0
    const uint32_t acc = __builtin_amdgcn_bitop3_b32(u2, p, cw1, 0x16);  // ~(u2 & cw1) & (u2 ^ cw1 ^ p)
    const uint32_t v = __builtin_amdgcn_bitop3_b32(u2, r, cw1, 0x48);    // (u2 ^ cw1) & r
    m0 = (acc & x0) | (~acc & m0);
    m1 = (acc & v) | (~acc & m1);
    return acc;
}

// ------------------------------------------------------------------- draws
// v shifted up by one with the lane's bit of a lane mask coming in: one
// add-with-carry.
__device__ __forceinline__ void cell_push(uint32_t& v, uint64_t mask)
{
    uint64_t carry;
    asm("v_addc_co_u32_e64 %0, %1, %2, %2, %3" : "=v"(v), "=s"(carry) : "v"(v), "s"(mask));
}

// Both parities' levels of word w of a row: 32 sites of each, 16 Philox
// calls (nv / 2 for a shorter word).  The bits enter from the top word's end,
// one add-with-carry each.
__device__ __forceinline__ void cell_draw(const Geom& g, int row, int w, int nv, uint32_t fam_off, uint32_t rho,
                                          uint32_t r, uint32_t sw, uint32_t t0, uint32_t t1, uint32_t t2,
                                          uint32_t (&d0)[2], uint32_t (&d1)[2])
{
    const uint32_t base = (uint32_t)(((int64_t)g.Lx * row) >> 2) + fam_off + 16u * (uint32_t)w;
    uint32_t a0 = 0, a1 = 0, b0 = 0, b1 = 0;  // even-x and odd-x sites
    auto push = [&](uint32_t& l0, uint32_t& l1, uint32_t u) {
        const uint64_t p0 = __ballot(u > t0), p1 = __ballot(u > t1), p2 = __ballot(u > t2);
        cell_push(l1, p1);
        cell_push(l0, p0 ^ p1 ^ p2);
    };
    for (int c = (nv >> 1) - 1; c >= 0; --c) {
        const u32x4 o = philox10(base + (uint32_t)c, rho, r, sw, g.key0, g.key1);
        push(a0, a1, o.v2);
        push(b0, b1, o.v3);
        push(a0, a1, o.v0);
        push(b0, b1, o.v1);
    }
    const int y = row % g.Ly, z = row / g.Ly;
    const bool q = (y + z) & 1;  // parity of the row's even-x sites
    d0[0] = q ? b0 : a0;
    d1[0] = q ? b1 : a1;
    d0[1] = q ? a0 : b0;
    d1[1] = q ? a1 : b1;
}

// A slice of drawn refreshes: refresh j of the slice (index rho0 + j) has its
// level planes at dr0 / dr1 + j * stride words, laid out [lattice][p][cell].
struct CellDraw {
    CellGeom cg;
    uint32_t *dr0, *dr1;
    uint32_t *fam0[6], *fam1[6];  // several families: the planes of each (n = 1), in place of dr0 / dr1
    int32_t families;             // grid.y runs over lattice * families + family
    const DaemonThresholds* dth;  // the schedule's table
    int64_t rho0, stride;
    int32_t n, L;
};

// Thread per (refresh, cell) of lattice l, grid-stride.  Bound: the Philox
// multiplications (quarter rate).
__device__ __forceinline__ void cells_draw_body(const CellDraw& D, int lf, int64_t first, int64_t step)
{
    const CellGeom& cg = D.cg;
    const int l = lf / D.families, fam = lf - l * D.families;
    uint32_t* const o0 = D.families > 1 ? D.fam0[fam] : D.dr0;
    uint32_t* const o1 = D.families > 1 ? D.fam1[fam] : D.dr1;
    const int64_t total = (int64_t)D.n * cg.plane;
    for (int64_t i = first; i < total; i += step) {
        const int j = (int)(i / cg.plane);
        const int64_t cell = i - (int64_t)j * cg.plane;
        const int row = (int)(cell / cg.W), w = (int)(cell - (int64_t)row * cg.W);
        const DaemonThresholds th = D.dth[D.rho0 + j];
        uint32_t d0[2], d1[2];
        cell_draw(cg.g, row, w, min(32, cg.g.Kx - 32 * w), (uint32_t)fam * (uint32_t)(cg.g.Nh / 2), (uint32_t)(D.rho0 + j), (uint32_t)(l % cg.g.R),
                  stream_word(kStreamDaemon, (uint32_t)(l / cg.g.R)), (uint32_t)(th.t0 - 1u), (uint32_t)(th.t1 - 1u),
                  (uint32_t)(th.t2 - 1u), d0, d1);
        const int64_t at = (int64_t)j * D.stride + (int64_t)l * 2 * cg.plane + cell;
        o0[at] = d0[0];
        o1[at] = d1[0];
        o0[at + cg.plane] = d0[1];
        o1[at + cg.plane] = d1[1];
    }
}

__global__ void __launch_bounds__(256) k_cells_draw(CellDraw D)
{
    cells_draw_body(D, blockIdx.y, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x);
}

// The canonical baselines draw a uniform u per site and half sweep (Philox
// (h >> 2, 2k + p, r, stream | s), word h & 3, h the parity-split index) and
// compare it with a table that falls with its index, so that the whole
// comparison is one small number per site, drawn here for many sweeps at once:
//   ALG 1, heat bath: c = #{v : u < tau[v]}, 0..7; the spin becomes 1 iff its
//     count v of neighbours with J s = -1 is at least c.  Three bits.
//   ALG 2, Metropolis: theta[0..3] take every move, c = #{q in 4..6 : u <
//     theta[q]}; a spin with u unsatisfied bonds (q = 6 - u) flips iff
//     u + c >= 3.  Two bits.
// Planes: dr + ((it * 2 + p) * K + i) * L * plane + l * plane + cell, K bits.
struct CellCanon {
    CellGeom cg;
    uint32_t* dr;
    const HeatBathThresholds* tab;  // the schedule's table, an entry per refresh
    int64_t k0;                     // first sweep
    int32_t n, period, L, gamma;
};

__device__ __forceinline__ int64_t cell_refresh_index(int64_t k, int32_t P)
{
    return P >= 1 ? k / P : 63 - __clzll((unsigned long long)(k + 1));
}

// The table of a half sweep: u < t as u <= t - 1, or never for t = 0 (t may be 2^32).
struct CellTable {
    uint32_t t[7];
    uint64_t on[7];
    bool some_never;  // the smallest is 0 (the scalar unit is near its rate: no masks without it)
};

__device__ __forceinline__ void cell_table(const HeatBathThresholds& th, CellTable& T)
{
#pragma unroll
    for (int v = 0; v < 7; ++v) {
        T.t[v] = (uint32_t)(th.tau[v] - (th.tau[v] ? 1u : 0u));
        T.on[v] = th.tau[v] ? ~0ull : 0ull;
    }
    T.some_never = th.tau[6] == 0;
}

// The comparisons of a cell's 4 n4 sites, the words of base + n4 - 1 .. base.
template <int ALG, int K>
__device__ __forceinline__ void cell_compare(const CellTable& T, uint32_t base, int n4, uint32_t time, uint32_t rep,
                                             uint32_t sw, uint32_t key0, uint32_t key1, uint32_t (&b)[K])
{
#pragma unroll
    for (int i = 0; i < K; ++i) b[i] = 0;
    auto push = [&](uint32_t u) {
        uint64_t M[7];
#pragma unroll
        for (int v = ALG == 1 ? 0 : 4; v < 7; ++v) M[v] = __ballot(u <= T.t[v]);
        if (T.some_never)
#pragma unroll
            for (int v = ALG == 1 ? 0 : 4; v < 7; ++v) M[v] &= T.on[v];
        if (ALG == 1) {
            cell_push(b[0], M[0] ^ M[1] ^ M[2] ^ M[3] ^ M[4] ^ M[5] ^ M[6]);
            cell_push(b[1], (M[1] & ~M[3]) | M[5]);
            cell_push(b[K - 1], M[3]);
        } else {
            cell_push(b[0], M[4] ^ M[5] ^ M[6]);
            cell_push(b[1], M[5]);
        }
    };
    for (int c = n4 - 1; c >= 0; --c) {
        const u32x4 o = philox10(base + (uint32_t)c, time, rep, sw, key0, key1);
        push(o.v3);
        push(o.v2);
        push(o.v1);
        push(o.v0);
    }
}

// Thread per cell of lattice blockIdx.y and half sweep blockIdx.z (uniform, so
// that its table is too), grid-stride.
template <int ALG>
__global__ void __launch_bounds__(64) k_cells_draw_canonical(CellCanon D)
{
    constexpr int K = ALG == 1 ? 3 : 2;
    const CellGeom& cg = D.cg;
    const int l = blockIdx.y;
    const uint32_t rep = (uint32_t)(l % cg.g.R);
    const uint32_t sw = stream_word(ALG == 1 ? kStreamHeatBath : kStreamMetropolis, (uint32_t)(l / cg.g.R));
    const int64_t k = D.k0 + (blockIdx.z >> 1);
    const uint32_t time = (uint32_t)(2 * k + (blockIdx.z & 1));
    CellTable T;
    cell_table(D.tab[cell_refresh_index(k / D.gamma, D.period)], T);
    for (int64_t cell = (int64_t)blockIdx.x * 64 + threadIdx.x; cell < cg.plane; cell += (int64_t)gridDim.x * 64) {
        const int64_t row = cg.W == 1 ? cell : cell / cg.W;  // (a division is a good part of a short row's work)
        const int w = (int)(cell - row * cg.W), n4 = min(32, cg.g.Kx - 32 * w) >> 2;
        uint32_t b[K];
        cell_compare<ALG, K>(T, (uint32_t)((row * cg.g.Kx + 32 * w) >> 2), n4, time, rep, sw, cg.g.key0, cg.g.key1, b);
#pragma unroll
        for (int i = 0; i < K; ++i)
            D.dr[((int64_t)blockIdx.z * K + i) * D.L * cg.plane + (int64_t)l * cg.plane + cell] = b[i];
    }
}

// ------------------------------------------------------------------ sweeps
struct CellTile {
    int32_t TY, TZ;    // owned rows and planes
    int32_t GY, GZ;    // ring rows and planes on each side (0: the whole side, periodic)
    int32_t EY, EZ;    // rows and planes computed on
    int32_t nty, ntz;  // tiles
    float inv_EYW, inv_W, inv_Ly, inv_Lz;  // reciprocals of EY W, W, Ly, Lz
};

// a / n for 0 <= a < 2^22 with inv = 1.0f / n: the product is off by less
// than one, put right by a step either way.
__device__ __forceinline__ int cell_div(int a, int n, float inv)
{
    int q = (int)((float)a * inv);
    const int r = a - q * n;
    q += r >= n ? 1 : 0;
    return r < 0 ? q - 1 : q;
}

// v mod n for |v| < 2^22.
__device__ __forceinline__ int cell_wrap(int v, int n, float inv)
{
    int r = v - (int)floorf((float)v * inv) * n;
    r += r < 0 ? n : 0;
    return r >= n ? r - n : r;
}


struct CellSweep {
    CellGeom cg;
    CellTile f;
    const uint32_t *s_in, *d0_in, *d1_in, *bond;
    uint32_t *s_out, *d0_out, *d1_out;  // may be the inputs where a tile is a whole lattice
    const uint32_t *dr0, *dr1;          // drawn levels of the launch's first refresh
    int64_t dr_stride;              // words from one refresh's levels to the next's
    unsigned long long* tally;
    uint32_t* log;       // logged launches: [row][lattices][lanes], see k_cells_log_rows; or null
    int64_t k0;          // first sweep index
    int32_t n;           // sweeps
    int32_t ref0;        // first refresh sweep of the launch, counted from k0 (>= n: none)
    int32_t period;      // refresh period, 0: before sweeps k with k + 1 a power of two
    int32_t log_stride;  // sweeps between logged rows
    int32_t log_first;   // sweeps until the launch's first one
    int32_t lattices;
    float inv_bdiv;      // 1 / cg.bdiv
    int32_t wander0;     // walkers, one per site: parity of the wandering owed at the start, or -1
    const HeatBathThresholds* tab;  // baselines that draw in place: the schedule's table (ref0: its next entry)
    int32_t gamma;                  // and the sweeps of a timestep
};

// Several families: the levels of each sweep of the launch (in and out), the
// direction of its family and the parity of the wandering it owes (-1: none).
struct CellFamilies {
    const uint32_t *in0[6], *in1[6];
    uint32_t *out0[6], *out1[6];
    int32_t dir[6], owed[6];
};

// Sweeps from one refresh (at k) to the next.
__device__ __forceinline__ int64_t cell_refresh_gap(int64_t k, int32_t P) { return P >= 1 ? P : k + 1; }

// Sum over a wave, in lane 63 (DPP: shifts by 1, 2, 4, 8 within rows of 16,
// then the rows' totals broadcast upwards).
__device__ __forceinline__ uint32_t wave_sum_dpp(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, true);  // row 0 -> 1, 2 -> 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, true);  // rows 0, 1 -> 2, 3
    return v;
}

// Maximum over a wave of values >= 0, the same in every lane.
__device__ __forceinline__ int wave_max_dpp(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, true));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, true));
    return __builtin_amdgcn_readlane(v, 63);
}

// XM: how a row's x neighbours are found.  0: the row is one word (rotate
// within its Kx bits); 1: several full words (funnel shift with the next or
// previous one); 2: several words, the last one short.
// ALG 0: MicSA; 1, 2: the heat bath and Metropolis on drawn planes; 3: walkers,
// one per site; 4: daemons or walkers in several families (F).
// RING: tiles with rings (a branch per half sweep costs a whole lattice 5 %).
// DRAW: a baseline that draws its comparisons in the half sweep that uses them.
template <int NR, int XM, int ALG, bool RING, bool DRAW = false>
__device__ __forceinline__ void cells_body(const CellSweep& J, const CellFamilies* F, int l, int ty, int tz,
                                           uint32_t* lds)
{
    constexpr int CAP = NR * kCellLanes;  // LDS words of one parity's plane
    constexpr bool LEVELS = ALG == 0 || ALG == 3;  // one family, in registers for the whole launch
    constexpr bool CANON = ALG == 1 || ALG == 2;
    const CellGeom& cg = J.cg;
    const Geom& g = cg.g;
    const CellTile& f = J.f;
    const int W = XM == 0 ? 1 : cg.W;
    const int t = threadIdx.x, B = blockDim.x;
    const int y0 = ty * f.TY, z0 = tz * f.TZ;
    const int EYW = f.EY * W, C = EYW * f.EZ;
    const int ownY = min(f.TY, g.Ly - y0), ownZ = min(f.TZ, g.Lz - z0);

    uint32_t s[2][NR], m0[2][NR], m1[2][NR];  // by parity
    uint32_t j[2][NR][6];                     // couplings: x same k, x shifted, y + 1, y - 1, z + 1, z - 1
    int iyp[NR], iym[NR], izp[NR], izm[NR];   // LDS words of the neighbours
    int adj[2][NR];                           // XM > 0: the other x word of each parity's sites
    uint32_t sa[NR], sb[NR], sc[2][NR], sd[2][NR], nvs[NR], nvps[NR];
    uint32_t gyp[NR], gym[NR], gzp[NR], gzm[NR], gxn[NR], gxp[NR];  // families: byte steps to the neighbour cells
    bool qq[NR];
    uint32_t gi[NR];                          // byte offset of the cell in a plane (fewer than 2^30 cells)
    uint32_t own = 0, valid = 0;              // bit i: cell i is owned / exists
    // Half sweeps of the launch that the wave's i-th cells take part in: a cell
    // n rows inside a ringed edge matters up to half sweep n (what is further out
    // is never read again by a cell that matters), a lane without one never.
    // (Skipped waves: 2 x 64^3 in tiles of 32 x 32 cells with rings of 12 rows
    // 1.37 -> 1.28 us per sweep, 104 x 90 x 70 x 4 3.0 -> 2.9.)
    int last[NR];
    // uniform plane addresses; a lane adds a 32-bit byte offset
    const int64_t lp = (int64_t)l * 2 * cg.plane;
    auto at = [](const uint32_t* base, uint32_t off) {
        return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(base) + off);
    };
    auto put = [](uint32_t* base, uint32_t off, uint32_t v) {
        *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(base) + off) = v;
    };
    const uint32_t* const bl = J.bond + (int64_t)cell_div(l, cg.bdiv, J.inv_bdiv) * 6 * cg.plane;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int c = t + i * B;
        const bool ok = c < C;
        const int cc = ok ? c : 0;  // a lane without a cell reads cell 0's neighbours, writes its own word
        const int ez = cell_div(cc, EYW, f.inv_EYW), rem = cc - ez * EYW;
        const int ey = XM == 0 ? rem : cell_div(rem, W, f.inv_W), w = XM == 0 ? 0 : rem - ey * W;
        const int y = cell_wrap(y0 - f.GY + ey, g.Ly, f.inv_Ly), z = cell_wrap(z0 - f.GZ + ez, g.Lz, f.inv_Lz);
        iyp[i] = cc + (ey + 1 < f.EY ? W : (f.GY ? 0 : W - EYW));
        iym[i] = cc + (ey > 0 ? -W : (f.GY ? 0 : EYW - W));
        izp[i] = cc + (ez + 1 < f.EZ ? EYW : (f.GZ ? 0 : EYW - C));
        izm[i] = cc + (ez > 0 ? -EYW : (f.GZ ? 0 : C - EYW));
        const int wn = w + 1 == W ? 0 : w + 1, wp = w == 0 ? W - 1 : w - 1;
        const int q = (y + z) & 1;
        qq[i] = q;
        const int nv = min(32, g.Kx - 32 * w), nvp = min(32, g.Kx - 32 * wp);
        nvs[i] = (uint32_t)nv;
        nvps[i] = (uint32_t)nvp;
        // the shifted x neighbour of a parity-p site is at k + 1 (q ^ p = 1) or k - 1
        if (XM == 0) {
            sa[i] = q ? 1u : (uint32_t)(g.Kx - 1);
        } else {
            adj[0][i] = cc + (q ? wn : wp) - w;
            adj[1][i] = cc + (q ? wp : wn) - w;
            sa[i] = q ? 1u : 0u;
            sb[i] = 1u - sa[i];
            sc[0][i] = q ? 0u : (uint32_t)(nvp - 1);
            sd[0][i] = q ? (uint32_t)(nv - 1) : 0u;
            sc[1][i] = q ? (uint32_t)(nvp - 1) : 0u;
            sd[1][i] = q ? 0u : (uint32_t)(nv - 1);
        }
        const int ZS = g.Ly * W;  // cells of a plane z
        const int me = z * ZS + y * W + w;
        gi[i] = (uint32_t)me << 2;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            s[p][i] = at(J.s_in + lp + p * cg.plane, gi[i]);
            m0[p][i] = LEVELS ? at(J.d0_in + lp + p * cg.plane, gi[i]) : 0u;
            m1[p][i] = LEVELS ? at(J.d1_in + lp + p * cg.plane, gi[i]) : 0u;
        }
        auto bd = [&](int d, int cell) { return at(bl + (int64_t)d * cg.plane, (uint32_t)cell << 2); };
        const uint32_t jpx = bd(kPx, me), jmx = bd(kMx, me);
        const uint32_t jA = q ? jmx : jpx, jB = q ? jpx : jmx;
        j[0][i][0] = jA;
        j[0][i][1] = jB;
        j[0][i][2] = bd(kPy, me);
        j[0][i][3] = bd(kMy, me);
        j[0][i][4] = bd(kPz, me);
        j[0][i][5] = bd(kMz, me);
        // an odd site's coupling is its even neighbour's in the opposite direction
        j[1][i][0] = jA;
        {
            uint32_t N = jB;
            if (XM > 0) {
                const uint32_t Np = bd(kPx, me + wp - w), Nm = bd(kMx, me + wn - w);
                N = q ? Np : Nm;
            }
            j[1][i][1] = (q ? (jB << 1) | (N >> (nvp - 1)) : (jB >> 1) | (N << (nv - 1))) & cell_mask(nv);
        }
        const int syp = y + 1 == g.Ly ? W - ZS : W, sym = y == 0 ? ZS - W : -W;
        const int szp = z + 1 == g.Lz ? ZS - (int)cg.plane : ZS, szm = z == 0 ? (int)cg.plane - ZS : -ZS;
        j[1][i][2] = bd(kMy, me + syp);
        j[1][i][3] = bd(kPy, me + sym);
        j[1][i][4] = bd(kMz, me + szp);
        j[1][i][5] = bd(kPz, me + szm);
        gyp[i] = (uint32_t)syp << 2;
        gym[i] = (uint32_t)sym << 2;
        gzp[i] = (uint32_t)szp << 2;
        gzm[i] = (uint32_t)szm << 2;
        gxn[i] = (uint32_t)(wn - w) << 2;
        gxp[i] = (uint32_t)(wp - w) << 2;
        const bool o = ok && (unsigned)(ey - f.GY) < (unsigned)ownY && (unsigned)(ez - f.GZ) < (unsigned)ownZ;
        own |= (o ? 1u : 0u) << i;
        valid |= (ok ? 1u : 0u) << i;
        int inside = INT32_MAX;
        if (f.GY) inside = min(ey, f.EY - 1 - ey);
        if (f.GZ) inside = min(inside, min(ez, f.EZ - 1 - ez));
        last[i] = RING ? wave_max_dpp(ok ? inside : 0) : INT32_MAX;
        lds[c] = s[0][i];
        lds[CAP + c] = s[1][i];
    }
    auto levels = [&]() {
        int v = 0;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int n = __popc(m0[0][i]) + __popc(m0[1][i]) + 2 * (__popc(m1[0][i]) + __popc(m1[1][i]));
            v += (own >> i) & 1u ? n : 0;
        }
        return v;
    };
    // valid bits of cell i's word: the same for every cell unless the rows
    // have a short last word
    const uint32_t mask01 = XM == 0 ? cell_mask(g.Kx) : 0xFFFFFFFFu;
    auto msk = [&](int i) { return XM == 2 ? cell_mask((int)nvs[i]) : mask01; };
    // the levels of the next refresh, loaded ahead of it (with three or four
    // cells per thread the registers are needed elsewhere: loaded at it)
    constexpr bool AHEAD = LEVELS && NR <= 2;
    uint32_t r0[2][NR], r1[2][NR];
    int64_t dr = 0;
    auto fetch = [&]() {
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                r0[p][i] = at(J.dr0 + dr + lp + p * cg.plane, gi[i]);
                r1[p][i] = at(J.dr1 + dr + lp + p * cg.plane, gi[i]);
            }
    };
    int64_t ref = J.ref0;
    if (AHEAD) fetch();  // (with no refresh in the launch the addresses are still good)
    // MicSA: levels in, minus levels out, of the owned sites; else a quarter of
    // their energy change
    int taken = LEVELS ? levels() : 0;
    // the baselines' drawn bits of the next half sweep, loaded during this one
    constexpr int K = ALG == 1 ? 3 : 2;
    uint32_t nx[NR][K];
    const int64_t lplane = (int64_t)J.lattices * cg.plane;
    const uint32_t* cd = CANON && !DRAW ? J.dr0 + (int64_t)l * cg.plane : nullptr;
    int halves = 2 * J.n;
    auto fetch_half = [&](int h) {
        if (DRAW) return;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            if (RING && last[i] < h) continue;
#pragma unroll
            for (int b = 0; b < K; ++b) nx[i][b] = at(cd + b * lplane, gi[i]);
        }
        --halves;
        cd += halves > 0 ? K * lplane : 0;  // (past the last half: the same addresses again)
    };
    if (CANON) fetch_half(1);
    CellTable table{};  // of the sweep under way, where the comparisons are drawn here
    const uint32_t rep = DRAW ? (uint32_t)(l % g.R) : 0u;
    const uint32_t stream = DRAW ? stream_word(ALG == 1 ? kStreamHeatBath : kStreamMetropolis, (uint32_t)(l / g.R)) : 0u;
    // families: the next sweep's levels at the places they come from (and the
    // adjacent words of the same row, for a move along x), loaded a sweep ahead
    uint32_t n0[2][NR], n1[2][NR], a0[2][NR], a1[2][NR];
    auto fetch_family = [&](int it) {
        const int dir = F->dir[it], owed = F->owed[it];
        const int axis = dir >> 1, sgn = (dir & 1) ? -1 : 1;
        const uint32_t *b0 = F->in0[it] + lp, *b1 = F->in1[it] + lp;
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                // a site of the wandering's parity takes the level one step along the
                // direction, a site of the other parity one step against it, both from
                // the other parity's plane
                const int toward = p == owed ? sgn : -sgn;
                uint32_t off = gi[i];
                if (owed >= 0 && axis == 1) off += toward > 0 ? gyp[i] : gym[i];
                if (owed >= 0 && axis == 2) off += toward > 0 ? gzp[i] : gzm[i];
                const int64_t pl = (owed >= 0 ? 1 - p : p) * cg.plane;
                n0[p][i] = at(b0 + pl, off);
                n1[p][i] = at(b1 + pl, off);
                if (XM > 0) {
                    const uint32_t side = gi[i] + (toward > 0 ? gxn[i] : gxp[i]);
                    a0[p][i] = at(b0 + pl, side);
                    a1[p][i] = at(b1 + pl, side);
                }
            }
    };
    auto take_family = [&](int it) {
        const int dir = F->dir[it], owed = F->owed[it];
        const bool alongx = owed >= 0 && (dir >> 1) == 0;
        const int sgn = (dir & 1) ? -1 : 1;
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                uint32_t v0 = n0[p][i], v1 = n1[p][i];
                if (alongx) {
                    // x +- 1 of a site at x = 2k + q is index k + q (forwards) or k + q - 1
                    const int q = (qq[i] ? 1 : 0) ^ p;
                    const int toward = p == owed ? sgn : -sgn;
                    const int shift = toward > 0 ? q : q - 1;
                    const uint32_t c0 = XM == 0 ? v0 : a0[p][i], c1 = XM == 0 ? v1 : a1[p][i];
                    const uint32_t nv = nvs[i], nvp = XM == 0 ? nv : nvps[i];
                    const uint32_t s0 = toward > 0 ? (v0 >> 1) | (c0 << (nv - 1)) : (v0 << 1) | (c0 >> (nvp - 1));
                    const uint32_t s1 = toward > 0 ? (v1 >> 1) | (c1 << (nv - 1)) : (v1 << 1) | (c1 >> (nvp - 1));
                    v0 = shift ? s0 & cell_mask((int)nv) : v0;
                    v1 = shift ? s1 & cell_mask((int)nv) : v1;
                }
                m0[p][i] = v0;
                m1[p][i] = v1;
            }
    };
    if (ALG == 4) fetch_family(0);
    // walkers, one per site: the wandering of parity w, within each row
    auto wander = [&](auto wc) {
        constexpr int w = decltype(wc)::value;
        uint32_t* edge = lds + 2 * CAP;
        if (XM > 0) {
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const uint32_t top = nvs[i] - 1;
                edge[t + i * B] = (m0[1 - w][i] & 1u) | ((m1[1 - w][i] & 1u) << 1) |
                                  (((m0[w][i] >> top) & 1u) << 2) | (((m1[w][i] >> top) & 1u) << 3);
            }
            lds_barrier();
        }
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const uint32_t f0 = m0[1 - w][i], f1 = m1[1 - w][i], g0 = m0[w][i], g1 = m1[w][i];
            uint32_t fd0, fd1, gu0, gu1;  // f a site down, g a site up
            if (XM == 0) {
                const uint32_t top = (uint32_t)g.Kx - 1u;
                fd0 = (f0 >> 1) | (f0 << top);
                fd1 = (f1 >> 1) | (f1 << top);
                gu0 = (g0 << 1) | (g0 >> top);
                gu1 = (g1 << 1) | (g1 >> top);
            } else {
                // the row's next and previous words (adj holds both, by the row's offset)
                const uint32_t en = edge[qq[i] ? adj[0][i] : adj[1][i]], ep = edge[qq[i] ? adj[1][i] : adj[0][i]];
                const uint32_t top = nvs[i] - 1;
                fd0 = (f0 >> 1) | ((en & 1u) << top);
                fd1 = (f1 >> 1) | (((en >> 1) & 1u) << top);
                gu0 = (g0 << 1) | ((ep >> 2) & 1u);
                gu1 = (g1 << 1) | ((ep >> 3) & 1u);
            }
            const bool moved = w ? !qq[i] : qq[i];  // the sites of parity w sit at odd x
            const uint32_t mk = msk(i);
            m0[w][i] = moved ? fd0 & mk : f0;
            m1[w][i] = moved ? fd1 & mk : f1;
            m0[1 - w][i] = moved ? gu0 & mk : g0;
            m1[1 - w][i] = moved ? gu1 & mk : g1;
        }
    };
    auto wander_parity = [&](int w) {
        if (w)
            wander(std::integral_constant<int, 1>{});
        else
            wander(std::integral_constant<int, 0>{});
    };
    if (ALG == 3 && J.wander0 >= 0) wander_parity(J.wander0);
    lds_barrier();

    // the x neighbour word of parity p's sites other than the one at the same k
    auto shifted = [&](int i, int p) -> uint32_t {
        const uint32_t o = s[1 - p][i];
        if (XM == 0) {
            const uint32_t c = (uint32_t)g.Kx - sa[i], a = p ? c : sa[i], b = p ? sa[i] : c;
            return ((o >> a) | (o << b)) & mask01;
        }
        const uint32_t N = lds[(1 - p) * CAP + adj[p][i]];
        const bool up = p ? !qq[i] : qq[i];
        if (XM == 1) return __builtin_amdgcn_alignbit(up ? N : o, up ? o : N, up ? 1u : 31u);
        const uint32_t a = p ? sb[i] : sa[i], b = p ? sa[i] : sb[i];
        return (((o >> a) << b) | ((N >> sc[p][i]) << sd[p][i])) & msk(i);
    };
    auto unsat = [&](int i, int p, uint32_t (&u)[6]) {
        const uint32_t* oth = lds + (1 - p) * CAP;
        const uint32_t S = s[p][i];
        u[2] = xor3(S, oth[iyp[i]], j[p][i][2]);
        u[3] = xor3(S, oth[iym[i]], j[p][i][3]);
        u[4] = xor3(S, oth[izp[i]], j[p][i][4]);
        u[5] = xor3(S, oth[izm[i]], j[p][i][5]);
        u[0] = xor3(S, s[1 - p][i], j[p][i][0]);
        u[1] = xor3(S, shifted(i, p), j[p][i][1]);
    };
    // Logged sweeps: a lane stores its unsatisfied bonds (each counted at its even
    // end) and, above bit 16, its level sum; k_cells_log_rows adds the lanes.
    // The bonds are those that the next even half finds before it moves anything,
    // so a logged sweep costs a few counts and a store: 0.36 us at 16^3, 0.32 not
    // logged (0.69 with the fields formed once more and the lanes summed here).
    uint32_t* logto = J.log ? J.log + (int64_t)l * B + t : nullptr;
    uint32_t logD = 0;
    bool pend = false;  // a sweep has ended whose row is not yet written
    int to_log = J.log_first;
    auto bonds = [&](int i, const uint32_t (&u)[6]) {
        uint32_t n = 0;
#pragma unroll
        for (int d = 0; d < 6; ++d) n += (uint32_t)__popc(u[d] & msk(i));
        return (valid >> i) & 1u ? n : 0u;
    };
    auto write_row = [&](uint32_t U) {
        *logto = U | logD;
        logto += (int64_t)J.lattices * B;
        pend = false;
    };
    auto half = [&](auto pc, int h) {  // half sweep h of the launch, from 1
        constexpr int p = decltype(pc)::value;
        uint32_t U = 0;
        uint32_t cur[NR][K];
        if (CANON && DRAW) {
#pragma unroll
            for (int i = 0; i < NR; ++i)  // (gi: the cell's byte offset; one word per row)
                cell_compare<ALG, K>(table, (gi[i] >> 2) * (uint32_t)(g.Kx >> 2), g.Kx >> 2,
                                     (uint32_t)(2 * J.k0) + (uint32_t)(h - 1), rep, stream, g.key0, g.key1, cur[i]);
        } else if (CANON) {
#pragma unroll
            for (int i = 0; i < NR; ++i)
#pragma unroll
                for (int b = 0; b < K; ++b) cur[i][b] = nx[i][b];
            fetch_half(h + 1);
        }
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            if (RING && last[i] < h) continue;
            uint32_t u[6];
            unsat(i, p, u);
            if (p == 0 && pend) U += bonds(i, u);
            if (!CANON) {
                s[p][i] ^= cell_move(u, m0[p][i], m1[p][i]);
            } else {
                const uint32_t s1 = xor3(u[0], u[1], u[2]), c1 = maj32(u[0], u[1], u[2]);
                const uint32_t s2 = xor3(u[3], u[4], u[5]), c2 = maj32(u[3], u[4], u[5]);
                const uint32_t u0 = s1 ^ s2, k0 = s1 & s2;
                const uint32_t u1 = xor3(c1, c2, k0), u2 = maj32(c1, c2, k0);  // unsatisfied bonds
                uint32_t f;
                if (ALG == 2) {
                    // u + c >= 3: u2, or u1 u0 + c1 c0 carries past 2
                    const uint32_t a = cur[i][1], b = cur[i][0];
                    f = u2 | (u1 & a) | ((u1 | a) & (u0 | b));
                } else {
                    // v = u for a spin 0, 6 - u for a spin 1; 6 - u has the bits
                    // ~(u2 | (u1 & u0)), ~(u1 ^ u0), u0
                    const uint32_t S = s[p][i];
                    const uint32_t d1 = ~(u1 ^ u0), d2 = ~(u2 | (u1 & u0));
                    const uint32_t v0 = u0, v1 = (S & d1) | (~S & u1), v2 = (S & d2) | (~S & u2);
                    const uint32_t b0 = ~v0 & cur[i][0];
                    const uint32_t b1 = maj32(~v1, cur[i][1], b0);
                    const uint32_t b2 = maj32(~v2, cur[i][K - 1], b1);  // v < c
                    f = S ^ ~b2;                                        // the spin becomes ~(v < c)
                }
                if (XM == 0 || XM == 2) f &= msk(i);
                // dH = 12 - 4 u per flip
                const int e = 3 * __popc(f) - __popc(f & u0) - 2 * __popc(f & u1) - 4 * __popc(f & u2);
                taken += (own >> i) & 1u ? e : 0;
                s[p][i] ^= f;
            }
            lds[p * CAP + t + i * B] = s[p][i];
        }
        if (p == 0 && pend) write_row(U);
        lds_barrier();
    };

    for (int it = 0; it < J.n; ++it) {
        if (ALG == 3 && it > 0 && it != ref) wander_parity((int)((J.k0 + it - 1) & 1));
        if (ALG == 4) {
            take_family(it);
            fetch_family(it + 1 < J.n ? it + 1 : it);
            taken += levels();
        }
        if (LEVELS && it == ref) {
            taken -= levels();
            if (!AHEAD) fetch();
#pragma unroll
            for (int i = 0; i < NR; ++i)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    m0[p][i] = r0[p][i];
                    m1[p][i] = r1[p][i];
                }
            taken += levels();
            ref += cell_refresh_gap(J.k0 + it, J.period);
            // no branch around the loads: they stay in flight until the next refresh
            dr += ref < J.n ? J.dr_stride : 0;
            if (AHEAD) fetch();
        }
        if (CANON && DRAW && (it == 0 || it == ref || J.period < 1)) {
            cell_table(J.tab[cell_refresh_index((J.k0 + it) / J.gamma, J.period)], table);
            if (it == ref) ref += (int64_t)J.period * J.gamma;
        }
        half(std::integral_constant<int, 0>{}, 2 * it + 1);
        half(std::integral_constant<int, 1>{}, 2 * it + 2);
        if (ALG == 4) {
            taken -= levels();
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                if (!((own >> i) & 1u)) continue;
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    put(F->out0[it] + lp + p * cg.plane, gi[i], m0[p][i]);
                    put(F->out1[it] + lp + p * cg.plane, gi[i], m1[p][i]);
                }
            }
        }
        if (J.log && --to_log == 0) {
            to_log = J.log_stride;
            uint32_t D = 0;
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const int n = __popc(m0[0][i]) + __popc(m0[1][i]) + 2 * (__popc(m1[0][i]) + __popc(m1[1][i]));
                D += (valid >> i) & 1u ? (uint32_t)n : 0u;
            }
            logD = D << 16;
            pend = true;
        }
    }
    if (pend) {
        uint32_t U = 0;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            uint32_t u[6];
            unsat(i, 0, u);
            U += bonds(i, u);
        }
        write_row(U);
    }
    if (LEVELS) taken -= levels();
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if (!((own >> i) & 1u)) continue;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            put(J.s_out + lp + p * cg.plane, gi[i], s[p][i]);
            if (LEVELS) put(J.d0_out + lp + p * cg.plane, gi[i], m0[p][i]);
            if (LEVELS) put(J.d1_out + lp + p * cg.plane, gi[i], m1[p][i]);
        }
    }
    // a wave's sum fits 32 bits (at most 64 lanes x 4 cells x 64 sites x 3, per refresh met)
    const int sum = (int)wave_sum_dpp((uint32_t)taken);
    if ((t & 63) == 63 && sum != 0)
        atomicAdd(&J.tally[(int64_t)l * kSlots + ((ty + tz * f.nty + (t >> 6)) % kSlots)],
                  (unsigned long long)(4ll * sum));
}

// Grid (tiles along y, tiles along z, lattices).
template <int NR, int XM, int ALG, bool RING>
__global__ void __launch_bounds__(kCellLanes) k_cells_sweep(CellSweep J)
{
    __shared__ uint32_t lds[(ALG == 3 && XM > 0 ? 3 : 2) * NR * kCellLanes];
    cells_body<NR, XM, ALG, RING>(J, nullptr, blockIdx.z, blockIdx.x, blockIdx.y, lds);
}

// The baselines on whole lattices of one word per row, drawing as they go
// (with four cells per thread 12 or 13 registers spill).
template <int NR, int ALG>
__global__ void __launch_bounds__(kCellLanes) k_cells_sweep_drawing(CellSweep J)
{
    __shared__ uint32_t lds[2 * NR * kCellLanes];
    cells_body<NR, 0, ALG, false, true>(J, nullptr, blockIdx.z, 0, 0, lds);
}

template <int NR, int XM>
__global__ void __launch_bounds__(kCellLanes) k_cells_sweep_families(CellSweep J, CellFamilies F)
{
    __shared__ uint32_t lds[2 * NR * kCellLanes];
    cells_body<NR, XM, 4, true>(J, &F, blockIdx.z, blockIdx.x, blockIdx.y, lds);
}

// Rows of a logged launch: entry e = row * lattices + lattice of `out` gets the
// unsatisfied bonds and the level sum from its lanes' words; the baselines,
// which neither hold nor change the levels, get the sum from its slots.  A wave
// per entry.
__global__ void __launch_bounds__(256) k_cells_log_rows(const uint32_t* __restrict__ raw, int64_t n, int lanes,
                                                        const unsigned long long* __restrict__ levels, int lattices,
                                                        long long* __restrict__ out)
{
    const int64_t e = blockIdx.x * 4ll + (threadIdx.x >> 6);
    if (e >= n) return;
    const int lane = threadIdx.x & 63;
    long long U = 0, D = levels ? (long long)levels[(e % lattices) * kSlots + lane] : 0;
    for (int k = lane; k < lanes; k += 64) {
        const uint32_t v = raw[e * lanes + k];
        U += v & 0xFFFFu;
        D += v >> 16;
    }
    U = wave_sum64(U);
    D = wave_sum64(D);
    if (lane == 0) {
        out[2 * e] = U;
        out[2 * e + 1] = D;
    }
}

// The batched launches of the serving pool: whole lattices of different jobs,
// each with its own shape, schedule and sweep index, a work-group per item.
// Table entries are uniform per work-group.  (The draw keeps its copy of an
// entry, whose family pointers it indexes, in 232 B of scratch per lane.)
struct CellItem {
    int32_t job, lattice;
};

template <int NR, int XM>
__global__ void __launch_bounds__(kCellLanes) k_cells_sweep_batch(const CellSweep* __restrict__ jobs,
                                                                  const CellItem* __restrict__ items)
{
    __shared__ uint32_t lds[2 * NR * kCellLanes];
    const CellItem it = items[blockIdx.x];
    const CellSweep J = jobs[it.job];
    cells_body<NR, XM, 0, false>(J, nullptr, it.lattice, 0, 0, lds);
}

__global__ void __launch_bounds__(256) k_cells_draw_batch(const CellDraw* __restrict__ jobs,
                                                          const CellItem* __restrict__ items)
{
    const CellItem it = items[blockIdx.y];
    const CellDraw D = jobs[it.job];
    cells_draw_body(D, it.lattice, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x);
}

// ------------------------------------------------- planes <-> other layouts
// Bit 0 of each byte of a word as four bits, and back.
__device__ __forceinline__ uint32_t gather4(uint32_t w) { return ((w & 0x01010101u) * 0x01020408u) >> 24; }
__device__ __forceinline__ uint32_t spread4(uint32_t n) { return ((n & 0xFu) * 0x00204081u) & 0x01010101u; }

// Byte layout -> planes, thread per (lattice, cell): 32 bytes of each parity.
// Coupling planes are written by the first lattice of each set.
struct CellLevels {
    uint32_t *d0[6], *d1[6];  // level planes of each family
    int32_t families;
};

__global__ void __launch_bounds__(256) k_cells_pack(CellGeom cg, const uint8_t* __restrict__ spin_b,
                                                    const uint8_t* __restrict__ dem_b, uint32_t* __restrict__ spin,
                                                    CellLevels lv, uint32_t* __restrict__ bond)
{
    const Geom& g = cg.g;
    const int64_t cell = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int l = blockIdx.y;
    if (cell >= cg.plane) return;
    const int64_t row = cell / cg.W;
    const int w = (int)(cell - row * cg.W);
    const int n4 = min(32, g.Kx - 32 * w) >> 2;
    const int64_t h = row * g.Kx + 32 * w;
    const int64_t at = (int64_t)l * 2 * cg.plane + cell;
    const uint32_t *ev = reinterpret_cast<const uint32_t*>(spin_b + (int64_t)l * 2 * g.Nh + h),
                   *od = reinterpret_cast<const uint32_t*>(spin_b + ((int64_t)l * 2 + 1) * g.Nh + h);
    uint32_t se = 0, so = 0, jb[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        if (v >= n4) break;
        const uint32_t a = ev[v], b = od[v];
        se |= gather4(a) << (4 * v);
        so |= gather4(b) << (4 * v);
#pragma unroll
        for (int k = 0; k < 6; ++k) jb[k] |= gather4(a >> (1 + k)) << (4 * v);
    }
    spin[at] = se;
    spin[at + cg.plane] = so;
    if (l % cg.bdiv == 0)
#pragma unroll
        for (int k = 0; k < 6; ++k) bond[((int64_t)(l / cg.bdiv) * 6 + k) * cg.plane + cell] = jb[k];
    for (int f = 0; f < lv.families; ++f)
        for (int p = 0; p < 2; ++p) {
            const uint32_t* m = reinterpret_cast<const uint32_t*>(
                dem_b + (((int64_t)l * lv.families + f) * 2 + p) * g.Nh + h);
            uint32_t e0 = 0, e1 = 0;
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                if (v >= n4) break;
                const uint32_t c = m[v];
                e0 |= gather4(c) << (4 * v);
                e1 |= gather4(c >> 1) << (4 * v);
            }
            lv.d0[f][at + p * cg.plane] = e0;
            lv.d1[f][at + p * cg.plane] = e1;
        }
}

__global__ void __launch_bounds__(256) k_cells_unpack(CellGeom cg, const uint32_t* __restrict__ spin, CellLevels lv,
                                                      const uint32_t* __restrict__ bond,
                                                      uint8_t* __restrict__ spin_b, uint8_t* __restrict__ dem_b)
{
    const Geom& g = cg.g;
    const int64_t cell = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int l = blockIdx.y;
    if (cell >= cg.plane) return;
    const int64_t row = cell / cg.W;
    const int w = (int)(cell - row * cg.W);
    const int n4 = min(32, g.Kx - 32 * w) >> 2;
    const int64_t h = row * g.Kx + 32 * w;
    const int64_t at = (int64_t)l * 2 * cg.plane + cell;
    uint32_t *ev = reinterpret_cast<uint32_t*>(spin_b + (int64_t)l * 2 * g.Nh + h),
             *od = reinterpret_cast<uint32_t*>(spin_b + ((int64_t)l * 2 + 1) * g.Nh + h);
    const uint32_t se = spin[at], so = spin[at + cg.plane];
    uint32_t jb[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) jb[k] = bond[((int64_t)(l / cg.bdiv) * 6 + k) * cg.plane + cell];
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        if (v >= n4) break;
        uint32_t a = spread4(se >> (4 * v));
#pragma unroll
        for (int k = 0; k < 6; ++k) a |= spread4(jb[k] >> (4 * v)) << (1 + k);
        ev[v] = a;
        od[v] = spread4(so >> (4 * v));
    }
    for (int f = 0; f < lv.families; ++f)
        for (int p = 0; p < 2; ++p) {
            uint32_t* m = reinterpret_cast<uint32_t*>(dem_b + (((int64_t)l * lv.families + f) * 2 + p) * g.Nh + h);
            const uint32_t e0 = lv.d0[f][at + p * cg.plane], e1 = lv.d1[f][at + p * cg.plane];
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                if (v >= n4) break;
                m[v] = spread4(e0 >> (4 * v)) | (spread4(e1 >> (4 * v)) << 1);
            }
        }
}

// Bit-plane layout (a word holds one site of 64 lattices) -> planes.  A wave
// per (word lattice, parity, cell), a lane per lattice: the site's word is
// uniform, so it is a lane mask, and one add-with-carry shifts each lane's
// bit in.  Lattice (s, r) is plane set s R + r; the coupling planes of a
// sample (cg.bdiv = R) are written by its replica 0.
__device__ __forceinline__ uint32_t cell_bits(const uint64_t* __restrict__ w, int nv)
{
    uint32_t v = 0;
    for (int k = nv - 1; k >= 0; --k) v = v + v + (__builtin_amdgcn_inverse_ballot_w64(w[k]) ? 1u : 0u);
    return v;
}

__global__ void __launch_bounds__(256) k_cells_pack_bits(GeomB gb, CellGeom cg, const uint64_t* __restrict__ bspin,
                                                         const uint64_t* __restrict__ bm0,
                                                         const uint64_t* __restrict__ bm1,
                                                         const uint64_t* __restrict__ Jw, uint32_t* __restrict__ spin,
                                                         uint32_t* __restrict__ d0, uint32_t* __restrict__ d1,
                                                         uint32_t* __restrict__ bond)
{
    const Geom& g = cg.g;
    const int wl = blockIdx.y;
    const int64_t i = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (i >= 2 * cg.plane) return;
    const int p = i >= cg.plane ? 1 : 0;
    const int64_t cell = i - p * cg.plane, row = cell / cg.W;
    const int w = (int)(cell - row * cg.W), nv = min(32, g.Kx - 32 * w);
    const int64_t h = row * g.Kx + 32 * w, at = ((int64_t)wl * 2 + p) * g.Nh + h;
    const uint32_t vs = cell_bits(bspin + at, nv), v0 = cell_bits(bm0 + at, nv), v1 = cell_bits(bm1 + at, nv);
    int s, r;
    const bool live = bp_lattice(gb, wl, lane_id(), s, r);
    const int64_t l = (int64_t)s * g.R + r, to = (l * 2 + p) * cg.plane + cell;
    if (live) {
        spin[to] = vs;
        d0[to] = v0;
        d1[to] = v1;
    }
    if (p == 0)
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            const uint32_t b = cell_bits(Jw + ((int64_t)bp_cset(gb, wl) * 6 + d) * g.Nh + h, nv);
            if (live && r == 0) bond[((int64_t)s * 6 + d) * cg.plane + cell] = b;
        }
}

// Planes -> bit-plane layout: a ballot per site, kept by the lane that
// stores the site's word (lanes of no lattice hold 0).
__global__ void __launch_bounds__(256) k_cells_unpack_bits(GeomB gb, CellGeom cg, const uint32_t* __restrict__ spin,
                                                           const uint32_t* __restrict__ d0,
                                                           const uint32_t* __restrict__ d1,
                                                           uint64_t* __restrict__ bspin, uint64_t* __restrict__ bm0,
                                                           uint64_t* __restrict__ bm1)
{
    const Geom& g = cg.g;
    const int wl = blockIdx.y, lane = lane_id();
    const int64_t i = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (i >= 2 * cg.plane) return;
    const int p = i >= cg.plane ? 1 : 0;
    const int64_t cell = i - p * cg.plane, row = cell / cg.W;
    const int w = (int)(cell - row * cg.W), nv = min(32, g.Kx - 32 * w);
    int s, r;
    const bool live = bp_lattice(gb, wl, lane, s, r);
    const int64_t from = live ? (((int64_t)s * g.R + r) * 2 + p) * cg.plane + cell : 0;
    const uint32_t vs = live ? spin[from] : 0u, v0 = live ? d0[from] : 0u, v1 = live ? d1[from] : 0u;
    uint64_t os = 0, o0 = 0, o1 = 0;
    for (int k = 0; k < nv; ++k) {
        const uint64_t bs = __ballot((vs >> k) & 1u), b0 = __ballot((v0 >> k) & 1u), b1 = __ballot((v1 >> k) & 1u);
        os = lane == k ? bs : os;
        o0 = lane == k ? b0 : o0;
        o1 = lane == k ? b1 : o1;
    }
    if (lane < nv) {
        const int64_t at = ((int64_t)wl * 2 + p) * g.Nh + row * g.Kx + 32 * w + lane;
        bspin[at] = os;
        bm0[at] = o0;
        bm1[at] = o1;
    }
}

// -------------------------------------------------------------- reductions
// KIND 0: unsatisfied bonds of lattice l (each at its even end); 1: level
// sum; 2: sites where replicas a and b of sample blockIdx.y differ.  Grid
// (blocks, lattices or samples), grid-stride over the cells.  Up to kSlots
// blocks store their slot each, and the first one zeros the others: a read of
// a small lattice is this launch and a copy.
template <int KIND>
__global__ void __launch_bounds__(256) k_cells_count(CellGeom cg, const uint32_t* __restrict__ spin, CellLevels lv,
                                                     const uint32_t* __restrict__ bond, int a, int b,
                                                     unsigned long long* __restrict__ out)
{
    const Geom& g = cg.g;
    const int l = blockIdx.y;
    const int64_t lp = (int64_t)l * 2 * cg.plane, lb = (int64_t)(l / cg.bdiv) * 6 * cg.plane;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    int v = 0;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < cg.plane; c += step) {
        if (KIND == 1) {
            for (int f = 0; f < lv.families; ++f)
                v += __popc(lv.d0[f][lp + c]) + __popc(lv.d0[f][lp + cg.plane + c]) +
                     2 * (__popc(lv.d1[f][lp + c]) + __popc(lv.d1[f][lp + cg.plane + c]));
        } else if (KIND == 2) {
            const int64_t pa = ((int64_t)l * g.R + a) * 2 * cg.plane + c, pb = ((int64_t)l * g.R + b) * 2 * cg.plane + c;
            v += __popc(spin[pa] ^ spin[pb]) +
                 __popc(spin[pa + cg.plane] ^ spin[pb + cg.plane]);
        } else {
            const int row = (int)(c / cg.W), w = (int)(c - (int64_t)row * cg.W);
            const int z = row / g.Ly, y = row - z * g.Ly, q = (y + z) & 1;
            const int nv = min(32, g.Kx - 32 * w);
            auto od = [&](int yy, int zz, int ww) {
                return spin[lp + cg.plane + ((int64_t)zz * g.Ly + yy) * cg.W + ww];
            };
            auto bd = [&](int d) { return bond[lb + (int64_t)d * cg.plane + c]; };
            const uint32_t S = spin[lp + c], O = od(y, z, w);
            const int wn = w + 1 == cg.W ? 0 : w + 1, wp = w == 0 ? cg.W - 1 : w - 1;
            const uint32_t N = od(y, z, q ? wn : wp);
            const uint32_t X = q ? (O >> 1) | (N << (nv - 1)) : (O << 1) | (N >> (min(32, g.Kx - 32 * wp) - 1));
            const uint32_t m = cell_mask(nv);
            v += __popc((S ^ O ^ bd(q ? kMx : kPx)) & m) + __popc((S ^ X ^ bd(q ? kPx : kMx)) & m) +
                 __popc((S ^ od(y + 1 == g.Ly ? 0 : y + 1, z, w) ^ bd(kPy)) & m) +
                 __popc((S ^ od(y == 0 ? g.Ly - 1 : y - 1, z, w) ^ bd(kMy)) & m) +
                 __popc((S ^ od(y, z + 1 == g.Lz ? 0 : z + 1, w) ^ bd(kPz)) & m) +
                 __popc((S ^ od(y, z == 0 ? g.Lz - 1 : z - 1, w) ^ bd(kMz)) & m);
        }
    }
    unsigned long long* const to = out + (int64_t)l * kSlots;
    if (gridDim.x > (unsigned)kSlots) {  // slots set to zero beforehand
        block_add(to, v);
        return;
    }
    __shared__ long long part[4];
    const long long s = wave_sum64(v);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0)
        to[blockIdx.x] = (unsigned long long)(part[0] + part[1] + part[2] + part[3]);
    else if (blockIdx.x == 0 && threadIdx.x >= gridDim.x && threadIdx.x < (unsigned)kSlots)
        to[threadIdx.x] = 0;
}

}  // namespace micsa
