// Kernels of the equilibrium workload of App. C: one Gaussian sample, runs x
// 2 replicas x M temperatures, continuous walkers (gamma = 1) refreshed every
// EMCS, Houdayer cluster moves between the replicas and parallel tempering.
//
// Energy mesh: couplings, energies and walkers are integers in units of
// 2^-17 (the paper allows walkers on a fine energy mesh, Sec. 2.3), so the
// Creutz move is exact integer arithmetic.
//
// Exponential on the mesh: P(n) = (1 - q) q^n, q = exp(-lambda 2^-17), drawn
// as four independent base-256 digits, digit d by inverse CDF on word d of
// one Philox output: c_d = #{v : w_d >= t_d[v]} with the table t_d[0..254]
// computed on the host.  Every t_d[v] lies in [2^24, 2^32] (the most likely
// value of a digit has probability >= 1/256), so the device holds
// t_d[v] - 1 in 32 bits (w >= t <=> w > t - 1), plus an indexed-search guide
// (Chen and Asau, 1974): for each top byte b of w the range [lo, hi] of
// counts the words of that bucket can have, so a draw costs one guide read
// and, in most buckets, no or one threshold compare.  The walkers use
// lambda = beta_t; the Metropolis update (a fresh walker per attempt,
// Sec. 2.3) and the tempering swaps (lambda = beta_t - beta_{t+1}) only
// need "n >= k", which is decided digit by digit from the top with at most
// two table reads per digit.
//
// Layout in HBM (per run u, replica a, slot c of the replica group):
//   rows[u][a][c][r]   one 64-bit word per lattice row r = y + Ly z: bit x
//                      is the spin bit sigma of site x + Lx r (Lx <= 64)
//   perm[u][a][t]      slot holding the configuration at temperature t
//   E[u][a][c]         energy of slot c (units of 2^-17), refreshed every EMCS
//   rec[x * R0 + r]    per-site coupling record (x-major so that the threads
//                      of consecutive rows read consecutive records):
//                      J+x, J+y, J+z, J-x, J-y, J-z, their sum, 0
// Tempering exchanges slots in perm; configurations never move.
//
// Work split of k_pt_emcs: one work-group per (temperature, run) holds both
// replicas of that temperature (Houdayer needs the pair); thread rr owns
// lattice row rr % R0 of replica rr / R0, so the x-neighbours of a site are
// bits of the thread's own word and the y/z-neighbours are the same bit of
// four other row words.  Forward-X wandering moves walkers within a row
// only, so every walker stays with the thread that owns its row.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "philox.hpp"

namespace micsa {

constexpr int kPtBlock = 256;
// u32 words per exponential table: [d * 256 + v] = t_d[v] - 1 (v < 255),
// then 4 x 256 guides as u16 lo | hi << 8 at byte offset 4096 + 2 (d * 256 + b)
constexpr int kPtTable = 1536;
enum : uint32_t { kStreamPtWalker = 6u, kStreamPtMetropolis = 7u, kStreamPtHoudayer = 8u, kStreamPtSwap = 9u,
                  kStreamPtSpin = 10u };

struct PtGeom {
    int32_t Lx, Ly, Lz;
    int32_t R0;  // rows per lattice
    int32_t N;
    int32_t M;     // temperatures
    int32_t runs;
    int32_t S;     // sweeps per EMCS
    uint32_t key0, key1;
    uint64_t xmask;  // the low Lx bits
};

__device__ __forceinline__ int32_t bit_mask(uint64_t w, int x) { return -(int32_t)((w >> x) & 1u); }

__device__ __forceinline__ uint64_t rot_up(uint64_t m, const PtGeom& g)  // bit x <- bit x - 1
{
    return ((m << 1) | (m >> (g.Lx - 1))) & g.xmask;
}
__device__ __forceinline__ uint64_t rot_down(uint64_t m, const PtGeom& g)  // bit x <- bit x + 1
{
    return ((m >> 1) | (m << (g.Lx - 1))) & g.xmask;
}

// The four digits of a draw: digit d is the number of thresholds below word d.
// The guide's lower bound and one compare settle nearly every word (the buckets
// of the low digits hold about one threshold each), so the four go side by
// side without a branch; what is left lies in a steep digit's last bucket,
// whose counts fall off geometrically, and goes on in growing steps.  (Digit after
// digit by bisection, each waiting for its own LDS reads, the draws of 16 M
// walkers took 67 us.)  Entry 255 of a digit is the largest word.
__device__ __forceinline__ int32_t exp_draw4(const uint32_t* tab, const u32x4& w)
{
    const uint32_t ws[4] = {w.v0, w.v1, w.v2, w.v3};
    uint32_t gb[4], t[4];
    int32_t n[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) gb[d] = ((const uint16_t*)(tab + 1024))[d * 256 + (ws[d] >> 24)];
#pragma unroll
    for (int d = 0; d < 4; ++d) t[d] = tab[d * 256 + (gb[d] & 255u)];
#pragma unroll
    for (int d = 0; d < 4; ++d) n[d] = (int32_t)(gb[d] & 255u) + (ws[d] > t[d] ? 1 : 0);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        int32_t hi = (int32_t)(gb[d] >> 8), step = 1;
        if (ws[d] > t[d])
            while (n[d] < hi) {
                const int32_t m = min(n[d] + step, hi) - 1;
                const bool above = ws[d] > tab[d * 256 + m];
                n[d] = above ? m + 1 : n[d];
                hi = above ? hi : m;
                step = above ? 2 * step : 1;
            }
    }
    return n[0] + (n[1] << 8) + (n[2] << 16) + (n[3] << 24);
}

// n >= k for the mesh exponential n drawn from words w.  Digit d of n
// exceeds k_d iff w_d >= t_d[k_d] (k_d <= 254) and falls below k_d iff
// w_d < t_d[k_d - 1] (k_d >= 1); equal digits pass to the next one.
__device__ __forceinline__ bool exp_at_least(const uint32_t* tab, const u32x4& w, int64_t k)
{
    if (k <= 0) return true;
    if (k >= (int64_t)1 << 32) return false;
    const uint32_t ws[4] = {w.v0, w.v1, w.v2, w.v3};
#pragma unroll
    for (int d = 3; d >= 0; --d) {
        const int32_t kd = (int32_t)((k >> (8 * d)) & 255);
        const uint32_t* td = tab + d * 256;
        if (kd <= 254 && ws[d] > td[kd]) return true;
        if (kd >= 1 && ws[d] <= td[kd - 1]) return false;
    }
    return true;
}

// Energy of one row's forward bonds: -sum J s_x s_y = sum J (2 d - 1),
// d = sigma_x XOR sigma_y.
template <bool JL>
__device__ __forceinline__ int32_t row_energy(const PtGeom& g, const int4* rec, int r, uint64_t row, uint64_t ryp,
                                              uint64_t rzp)
{
    const uint64_t dx = row ^ rot_down(row, g), dy = row ^ ryp, dz = row ^ rzp;
    int32_t e = 0;
    for (int x = 0; x < g.Lx; ++x) {
        const int4 a = rec[2 * (x * g.R0 + r)];
        e += (2 * (a.x & bit_mask(dx, x)) - a.x) + (2 * (a.y & bit_mask(dy, x)) - a.y) +
             (2 * (a.z & bit_mask(dz, x)) - a.z);
    }
    return e;
}

struct PtRowNb {
    int r, yp, ym, zp, zm;  // row indices of the row and its y/z neighbours
    int y, z;
};

__device__ __forceinline__ PtRowNb pt_row_nb(const PtGeom& g, int r)
{
    PtRowNb n;
    n.r = r;
    n.y = r % g.Ly;
    n.z = r / g.Ly;
    const int yp = n.y + 1 == g.Ly ? 0 : n.y + 1, ym = n.y == 0 ? g.Ly - 1 : n.y - 1;
    const int zp = n.z + 1 == g.Lz ? 0 : n.z + 1, zm = n.z == 0 ? g.Lz - 1 : n.z - 1;
    n.yp = yp + g.Ly * n.z;
    n.ym = ym + g.Ly * n.z;
    n.zp = n.y + g.Ly * zp;
    n.zm = n.y + g.Ly * zm;
    return n;
}

// LDS carve-up of k_pt_emcs (bytes): tables, coupling records (JL), spin
// rows of both replicas, walkers (ALGO 0), Houdayer rows and scan scratch.
struct PtLds {
    uint32_t tab, rec, rows, walk, mark, diff, scan, misc, total;
};

__host__ __device__ inline PtLds pt_lds_layout(const PtGeom& g, bool jl, bool walkers)
{
    PtLds l;
    uint32_t o = 0;
    l.tab = o;
    o += kPtTable * 4;
    l.rec = o;
    o += jl ? (uint32_t)g.N * 32u : 0u;
    l.rows = o;
    o += (uint32_t)g.R0 * 16u;
    l.walk = o;
    o += walkers ? (uint32_t)g.N * 8u : 0u;
    l.mark = o;
    o += (uint32_t)g.R0 * 8u;
    l.diff = o;
    o += (uint32_t)g.R0 * 8u;
    l.scan = o;
    o += kPtBlock * 4u;
    l.misc = o;
    o += 64u;
    l.total = o;
    return l;
}

// One EMCS of the fixed-temperature moves (walkers: ALGO 0; Metropolis:
// ALGO 1), then the Houdayer move (HOUD) and both replicas' energies.
// Grid (M, runs); block kPtBlock; dynamic LDS pt_lds_layout(g, JL, ALGO == 0).
template <int ALGO, bool HOUD, bool JL>
__global__ __launch_bounds__(kPtBlock) void k_pt_emcs(PtGeom g, const int4* __restrict__ grec,
                                                        uint64_t* __restrict__ spins,
                                                        const int32_t* __restrict__ perm, int64_t* __restrict__ E,
                                                        const uint32_t* __restrict__ wtab, uint32_t e)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const PtLds L = pt_lds_layout(g, JL, ALGO == 0);
    uint32_t* tab = (uint32_t*)(lds + L.tab);
    const int4* rec = JL ? (const int4*)(lds + L.rec) : grec;
    uint64_t* rows = (uint64_t*)(lds + L.rows);  // [2][R0]
    int32_t* walk = (int32_t*)(lds + L.walk);    // [2][Lx][R0]
    uint64_t* mark = (uint64_t*)(lds + L.mark);
    uint64_t* diff = (uint64_t*)(lds + L.diff);
    int32_t* scan = (int32_t*)(lds + L.scan);
    int32_t* misc = (int32_t*)(lds + L.misc);
    unsigned long long* esum = (unsigned long long*)(lds + L.misc + 16);

    const int t = blockIdx.x, run = blockIdx.y, tid = threadIdx.x;
    const int R0 = g.R0, nrow = 2 * R0;
    const int32_t slot0 = perm[((int64_t)run * 2 + 0) * g.M + t];
    const int32_t slot1 = perm[((int64_t)run * 2 + 1) * g.M + t];
    uint64_t* g0 = spins + (((int64_t)run * 2 + 0) * g.M + slot0) * R0;
    uint64_t* g1 = spins + (((int64_t)run * 2 + 1) * g.M + slot1) * R0;
    const uint32_t sw = (uint32_t)run;

    for (int k = tid; k < kPtTable; k += kPtBlock) tab[k] = wtab[(int64_t)t * kPtTable + k];
    if (JL)
        for (int k = tid; k < 2 * g.N; k += kPtBlock) ((int4*)(lds + L.rec))[k] = grec[k];
    for (int k = tid; k < R0; k += kPtBlock) {
        rows[k] = g0[k];
        rows[R0 + k] = g1[k];
    }
    if (tid < 2) esum[tid] = 0ull;
    __syncthreads();

    if (ALGO == 0) {  // walkers drawn at beta_t (one Philox output per site)
        for (int rr = tid; rr < nrow; rr += kPtBlock) {
            const int rep = rr >= R0, r = rr - rep * R0;
            for (int x = 0; x < g.Lx; ++x) {
                const uint32_t i = (uint32_t)(x + g.Lx * r);
                const u32x4 w = philox10(i, e, (uint32_t)(2 * t + rep), stream_word(kStreamPtWalker, sw), g.key0,
                                         g.key1);
                walk[(rep * g.Lx + x) * R0 + r] = exp_draw4(tab, w);
            }
        }
    }

    for (int s = 0; s < g.S; ++s) {
        for (int p = 0; p < 2; ++p) {
            for (int rr = tid; rr < nrow; rr += kPtBlock) {
                const int rep = rr >= R0, r = rr - rep * R0;
                const PtRowNb nb = pt_row_nb(g, r);
                const uint64_t* rw = rows + rep * R0;
                const uint64_t row = rw[r];
                const uint64_t xp = rot_down(row, g), xm = rot_up(row, g);
                const uint64_t yp = rw[nb.yp], ym = rw[nb.ym], zp = rw[nb.zp], zm = rw[nb.zm];
                uint64_t flips = 0;
                for (int x = (p + nb.y + nb.z) & 1; x < g.Lx; x += 2) {
                    const int4 a = rec[2 * (x * R0 + r)], b = rec[2 * (x * R0 + r) + 1];
                    // h = sum J s = Jsum - 2 sum over neighbours with sigma = 1
                    const int32_t up = (a.x & bit_mask(xp, x)) + (a.y & bit_mask(yp, x)) + (a.z & bit_mask(zp, x)) +
                                       (a.w & bit_mask(xm, x)) + (b.x & bit_mask(ym, x)) + (b.y & bit_mask(zm, x));
                    const int32_t h2 = 2 * (b.z - 2 * up);  // 2 h
                    const int32_t own = bit_mask(row, x);
                    const int32_t dH = (h2 ^ own) - own;    // 2 s h, s = -1 when sigma = 1
                    bool acc;
                    if (ALGO == 0) {
                        int32_t* wp = walk + (rep * g.Lx + x) * R0 + r;
                        const int32_t n = *wp;
                        acc = n - dH >= 0;
                        if (acc) *wp = n - dH;
                    } else {
                        const uint32_t i = (uint32_t)(x + g.Lx * r);
                        const u32x4 w = philox10(i, e * (uint32_t)g.S + (uint32_t)s, (uint32_t)(2 * t + rep),
                                                 stream_word(kStreamPtMetropolis, sw), g.key0, g.key1);
                        acc = exp_at_least(tab, w, dH);
                    }
                    flips |= (uint64_t)acc << x;
                }
                rows[rep * R0 + r] = row ^ flips;
            }
            __syncthreads();
        }
        if (ALGO == 0) {  // forward-X wandering of the sites of parity s & 1 (row-local)
            for (int rr = tid; rr < nrow; rr += kPtBlock) {
                const int rep = rr >= R0, r = rr - rep * R0;
                const int y = r % g.Ly, z = r / g.Ly;
                int32_t* wr = walk + rep * g.Lx * R0 + r;
                for (int x = ((s & 1) + y + z) & 1; x < g.Lx; x += 2) {
                    const int xn = x + 1 == g.Lx ? 0 : x + 1;
                    const int32_t tmp = wr[x * R0];
                    wr[x * R0] = wr[xn * R0];
                    wr[xn * R0] = tmp;
                }
            }
        }
    }

    if (HOUD) {
        // differing sites per row, in site order: prefix over contiguous row chunks
        const int chunk = (R0 + kPtBlock - 1) / kPtBlock;
        int32_t mine = 0;
        for (int r = tid * chunk; r < min(R0, (tid + 1) * chunk); ++r) {
            const uint64_t d = (rows[r] ^ rows[R0 + r]) & g.xmask;
            diff[r] = d;
            mark[r] = 0;
            mine += __popcll(d);
        }
        scan[tid] = mine;
        __syncthreads();
        for (int off = 1; off < kPtBlock; off <<= 1) {  // inclusive scan
            const int32_t v = tid >= off ? scan[tid - off] : 0;
            __syncthreads();
            scan[tid] += v;
            __syncthreads();
        }
        const int32_t count = scan[kPtBlock - 1];
        if (count > 0) {
            const uint32_t u = philox10((uint32_t)t, e, 0u, stream_word(kStreamPtHoudayer, sw), g.key0, g.key1).v0;
            const int32_t k = (int32_t)(((uint64_t)u * (uint64_t)count) >> 32);
            const int32_t before = scan[tid] - mine;
            if (k >= before && k < scan[tid]) {  // the chosen site is in this thread's chunk
                int32_t left = k - before;
                for (int r = tid * chunk; r < min(R0, (tid + 1) * chunk); ++r) {
                    uint64_t d = diff[r];
                    const int32_t c = __popcll(d);
                    if (left < c) {
                        for (; left > 0; --left) d &= d - 1;  // drop the lower set bits
                        mark[r] = d & (~d + 1);
                        break;
                    }
                    left -= c;
                }
            }
            // grow the cluster to the connected component of the chosen site
            for (;;) {
                __syncthreads();
                if (tid == 0) misc[0] = 0;
                __syncthreads();
                for (int r = tid; r < R0; r += kPtBlock) {
                    const PtRowNb nb = pt_row_nb(g, r);
                    const uint64_t d = diff[r], m = mark[r];
                    uint64_t m2 = d & (m | mark[nb.yp] | mark[nb.ym] | mark[nb.zp] | mark[nb.zm]);
                    for (;;) {  // close along the row
                        const uint64_t m3 = d & (m2 | rot_up(m2, g) | rot_down(m2, g));
                        if (m3 == m2) break;
                        m2 = m3;
                    }
                    if (m2 != m) {
                        mark[r] = m2;
                        misc[0] = 1;
                    }
                }
                __syncthreads();
                if (misc[0] == 0) break;
            }
            for (int r = tid; r < R0; r += kPtBlock) {
                rows[r] ^= mark[r];
                rows[R0 + r] ^= mark[r];
            }
            __syncthreads();
        }
    }

    // write back and energies
    for (int rr = tid; rr < nrow; rr += kPtBlock) {
        const int rep = rr >= R0, r = rr - rep * R0;
        const PtRowNb nb = pt_row_nb(g, r);
        const uint64_t* rw = rows + rep * R0;
        const int32_t er = row_energy<JL>(g, rec, r, rw[r], rw[nb.yp], rw[nb.zp]);
        atomicAdd(&esum[rep], (unsigned long long)(int64_t)er);
        (rep ? g1 : g0)[r] = rw[r];
    }
    __syncthreads();
    if (tid == 0) {
        E[((int64_t)run * 2 + 0) * g.M + slot0] = (int64_t)esum[0];
        E[((int64_t)run * 2 + 1) * g.M + slot1] = (int64_t)esum[1];
    }
}

// ---------------------------------------------------------------------------
// Register-resident variant for rows of LX <= 32 sites (LX a compile-time
// constant) and 2 * Ly * Lz <= 1024: a work-group holds G temperatures (both
// replicas each) and every thread owns exactly one row of one replica, so
// the walkers of a row live in VGPRs, split by parity class (wk0: the
// row's even sites x = 2j + ((y+z) & 1), wk1: its odd sites), and every bit
// test uses a constant offset.  Forward-X wandering pairs site j of the
// moving class with site j (or j + 1 when the class starts at x = 1) of the
// other class, all within the row.
// It runs the Metropolis sweeps, and the walkers of lattices whose field tables
// (k_pt_emcs_tab) exceed LDS.  Metropolis is held to 64 registers, so that
// two work-groups share a compute unit (10^3 with Houdayer moves: 605 us per
// EMCS, 790 with one); with those moves 22 spill.
// LDS: tables [G][kPtTable] u32 | records [N][2] int4 | rows [G][2][R0] u32 |
//      mark, diff [G][R0] u32 | energies [G][2] u64; the Houdayer move
//      keeps the neighbour rows [R0] 4 x u16 over the tables.
struct PtRegLds {
    uint32_t tab, rec, rows, mark, diff, esum, total;
};

__host__ __device__ inline PtRegLds pt_reg_layout(const PtGeom& g, int G)
{
    PtRegLds l;
    uint32_t o = 0;
    l.tab = o;
    o += (uint32_t)G * kPtTable * 4u;
    l.rec = o;
    o += (uint32_t)g.N * 32u;
    l.rows = o;
    o += (uint32_t)G * 2u * g.R0 * 4u;
    l.mark = o;
    o += (uint32_t)G * g.R0 * 4u;
    l.diff = o;
    o += (uint32_t)G * g.R0 * 4u;
    o = (o + 7u) & ~7u;
    l.esum = o;
    o += (uint32_t)G * 16u;
    l.total = o;
    return l;
}

template <int LX>
__device__ __forceinline__ uint32_t rot_down32(uint32_t m)  // bit x <- bit x + 1
{
    constexpr uint32_t MASK = LX == 32 ? 0xFFFFFFFFu : ((1u << LX) - 1u);
    return ((m >> 1) | (m << (LX - 1))) & MASK;
}
template <int LX>
__device__ __forceinline__ uint32_t rot_up32(uint32_t m)  // bit x <- bit x - 1
{
    constexpr uint32_t MASK = LX == 32 ? 0xFFFFFFFFu : ((1u << LX) - 1u);
    return ((m << 1) | (m >> (LX - 1))) & MASK;
}

// The cyclic runs of the row d that hold a bit of m (m within d): the carry of
// d + m runs through a run's bits above its lowest mark, and those of the
// reversed words through the bits below; two copies of the row side by side
// make the runs that cross its end whole.
template <int LX>
__device__ __forceinline__ uint32_t row_fill(uint32_t d, uint32_t m)
{
    static_assert(2 * LX <= 32, "two copies of a row in a word");
    constexpr uint32_t MASK = (1u << LX) - 1u;
    const uint32_t dd = d | (d << LX), mm = m | (m << LX);
    const uint32_t up = dd & (~(dd + mm) | mm);
    const uint32_t rd = __brev(dd), rm = __brev(mm);
    const uint32_t f = up | __brev(rd & (~(rd + rm) | rm));
    return (f | (f >> LX)) & MASK;
}

// A row's marks grown by its neighbours' and closed along the row.
template <int LX>
__device__ __forceinline__ bool grow_row(uint32_t* mq, int r, uint32_t d, ushort4 n)
{
    const uint32_t m = mq[r];
    const uint32_t m2 = row_fill<LX>(d, d & (m | mq[n.x] | mq[n.y] | mq[n.z] | mq[n.w]));
    if (m2 == m) return false;
    mq[r] = m2;
    return true;
}

// Houdayer's move of temperatures t0 .. t0 + G of a run: a site drawn among
// those where the replicas differ (diff: a word per row), and its connected
// component in mark (zero on entry).  One wave per temperature: prefix over
// the rows in site order, then growth with no barrier (the wave alone writes
// the temperature's marks, and a wave's LDS accesses are in order).  All waves
// growing together, with three barriers a round and the rows closed bit by
// bit, took 100 of an EMCS's 363 us at 10^3.  nbr: rows along +y, -y, +z, -z.
template <int LX>
__device__ __forceinline__ void houdayer_grow(const PtGeom& g, int G, int t0, uint32_t run, uint32_t e,
                                              const uint32_t* diff, uint32_t* mark, const ushort4* nbr)
{
    const int R0 = g.R0, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nwave = blockDim.x >> 6;
    const int chunk = (R0 + 63) / 64;
    for (int q = wave; q < G; q += nwave) {
        if (t0 + q >= g.M) continue;
        const uint32_t* dq = diff + q * R0;
        uint32_t* mq = mark + q * R0;
        int32_t mine = 0;
        for (int rr = lane * chunk; rr < min(R0, (lane + 1) * chunk); ++rr) mine += __popc(dq[rr]);
        int32_t incl = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t v = __shfl_up(incl, off, 64);
            if (lane >= off) incl += v;
        }
        const int32_t count = __shfl(incl, 63, 64);
        if (count == 0) continue;
        const uint32_t u = philox10((uint32_t)(t0 + q), e, 0u, stream_word(kStreamPtHoudayer, run), g.key0, g.key1).v0;
        const int32_t k = (int32_t)(((uint64_t)u * (uint64_t)count) >> 32);
        const int32_t before = incl - mine;
        if (k >= before && k < incl) {
            int32_t left = k - before;
            for (int rr = lane * chunk; rr < min(R0, (lane + 1) * chunk); ++rr) {
                uint32_t d = dq[rr];
                const int32_t c = __popc(d);
                if (left < c) {
                    for (; left > 0; --left) d &= d - 1;
                    mq[rr] = d & (~d + 1u);
                    break;
                }
                left -= c;
            }
        }
        // up to four rows per lane held, so that their reads overlap
        ushort4 n[4];
        uint32_t d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int rr = min(lane + 64 * i, R0 - 1);
            n[i] = nbr[rr];
            d[i] = dq[rr];
        }
        bool grown;
        do {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            grown = false;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int rr = lane + 64 * i;
                if (rr < R0) grown |= grow_row<LX>(mq, rr, d[i], n[i]);
            }
            for (int rr = lane + 256; rr < R0; rr += 64) grown |= grow_row<LX>(mq, rr, dq[rr], nbr[rr]);
        } while (__any(grown));
    }
}

__device__ __forceinline__ int32_t sbit(uint32_t w, int pos)  // 0 or -1
{
    return __builtin_amdgcn_sbfe((int32_t)w, pos, 1);
}

template <int LX, int ALGO, int P>
__device__ __forceinline__ void reg_half(const PtGeom& g, const int4* rec, uint32_t* rows, int base, int r,
                                         const PtRowNb& nb, int32_t (&wk)[LX / 2], const uint32_t* tab, uint32_t e,
                                         int s, int t, int rep, uint32_t run)
{
    constexpr int K = LX / 2;
    const int R0 = g.R0;
    const int xs = (P + nb.y + nb.z) & 1;  // first x of this class in the row
    const uint32_t own = rows[base + r];
    const uint32_t wo = own >> xs, wxp = rot_down32<LX>(own) >> xs, wxm = rot_up32<LX>(own) >> xs;
    const uint32_t wyp = rows[base + nb.yp] >> xs, wym = rows[base + nb.ym] >> xs;
    const uint32_t wzp = rows[base + nb.zp] >> xs, wzm = rows[base + nb.zm] >> xs;
    const int4* rc = rec + 2 * (xs * R0 + r);
    uint32_t flips = 0;
    // the walker path unrolls (walkers in registers); the Metropolis path
    // keeps one generator output live at a time
    constexpr int kUnroll = ALGO == 0 ? K : 1;
#pragma unroll kUnroll
    for (int j = 0; j < K; ++j) {
        const int4 a = rc[4 * R0 * j], b = rc[4 * R0 * j + 1];
        const int32_t up = (a.x & sbit(wxp, 2 * j)) + (a.y & sbit(wyp, 2 * j)) + (a.z & sbit(wzp, 2 * j)) +
                           (a.w & sbit(wxm, 2 * j)) + (b.x & sbit(wym, 2 * j)) + (b.y & sbit(wzm, 2 * j));
        const int32_t h2 = 2 * (b.z - 2 * up);
        const int32_t m = sbit(wo, 2 * j);
        const int32_t dH = (h2 ^ m) - m;
        bool acc;
        if (ALGO == 0) {
            const int32_t n = wk[j], nn = n - dH;
            acc = nn >= 0;
            wk[j] = acc ? nn : n;
        } else {
            const uint32_t i = (uint32_t)(2 * j + xs + LX * r);
            const u32x4 w = philox10(i, e * (uint32_t)g.S + (uint32_t)s, (uint32_t)(2 * t + rep),
                                     stream_word(kStreamPtMetropolis, run), g.key0, g.key1);
            acc = exp_at_least(tab, w, dH);
        }
        flips |= acc ? (1u << (2 * j)) : 0u;
    }
    rows[base + r] = own ^ (flips << xs);
}

// Forward-X wandering of the sites of class PW: site j of class PW at
// x = 2j + xs swaps with site j + xs of the other class (periodic).
template <int K>
__device__ __forceinline__ void reg_wander(int32_t (&A)[K], int32_t (&B)[K], int xs)
{
    int32_t nA[K], nB[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
        nA[j] = xs ? B[(j + 1) % K] : B[j];
        nB[j] = xs ? A[(j + K - 1) % K] : A[j];
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
        A[j] = nA[j];
        B[j] = nB[j];
    }
}

// Grid (ceil(M / G), runs); block 64 * ceil(2 G R0 / 64) <= 1024 threads;
// dynamic LDS pt_reg_layout(g, G).
template <int LX, int ALGO, bool HOUD>
__global__ __launch_bounds__(1024, ALGO == 1 ? 8 : 4) void k_pt_emcs_reg(PtGeom g, int G, const int4* __restrict__ grec,
                                                      uint64_t* __restrict__ spins, const int32_t* __restrict__ perm,
                                                      int64_t* __restrict__ E, const uint32_t* __restrict__ wtab,
                                                      uint32_t e)
{
    constexpr int K = LX / 2;
    constexpr uint32_t MASK = LX == 32 ? 0xFFFFFFFFu : ((1u << LX) - 1u);
    extern __shared__ __align__(16) unsigned char lds[];
    const PtRegLds L = pt_reg_layout(g, G);
    uint32_t* tabs = (uint32_t*)(lds + L.tab);
    int4* rec = (int4*)(lds + L.rec);
    uint32_t* rows = (uint32_t*)(lds + L.rows);
    uint32_t* mark = (uint32_t*)(lds + L.mark);
    uint32_t* diff = (uint32_t*)(lds + L.diff);
    unsigned long long* esum = (unsigned long long*)(lds + L.esum);
    ushort4* nbr = (ushort4*)(lds + L.tab);

    const int R0 = g.R0, tid = threadIdx.x, nthr = blockDim.x;
    const int tl = tid / (2 * R0), rem = tid - tl * 2 * R0;
    const int rep = rem >= R0, r = rem - rep * R0;
    const int t0 = blockIdx.x * G, t = t0 + tl;
    const int run = blockIdx.y;
    const uint32_t sw = (uint32_t)run;
    const bool live = tl < G && t < g.M;
    const int base = (tl * 2 + rep) * R0;

    for (int k = tid; k < G * kPtTable; k += nthr) {
        const int tg = t0 + k / kPtTable;
        tabs[k] = tg < g.M ? wtab[(int64_t)tg * kPtTable + k % kPtTable] : 0u;
    }
    for (int k = tid; k < 2 * g.N; k += nthr) rec[k] = grec[k];
    int32_t slot = 0;
    uint64_t* grow = nullptr;
    if (live) {
        slot = perm[((int64_t)run * 2 + rep) * g.M + t];
        grow = spins + (((int64_t)run * 2 + rep) * g.M + slot) * R0 + r;
        rows[base + r] = (uint32_t)*grow;
    }
    if (tid < 2 * G) esum[tid] = 0ull;
    const PtRowNb nb = pt_row_nb(g, live ? r : 0);
    __syncthreads();

    const uint32_t* tab = tabs + (live ? tl : 0) * kPtTable;
    int32_t wk0[K], wk1[K];
#pragma unroll
    for (int j = 0; j < K; ++j) wk0[j] = wk1[j] = 0;
    if (ALGO == 0 && live) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int xs = (c + nb.y + nb.z) & 1;
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const uint32_t i = (uint32_t)(2 * j + xs + LX * r);
                const u32x4 w = philox10(i, e, (uint32_t)(2 * t + rep), stream_word(kStreamPtWalker, sw), g.key0,
                                         g.key1);
                (c == 0 ? wk0 : wk1)[j] = exp_draw4(tab, w);
            }
        }
    }

    for (int s = 0; s < g.S; ++s) {
        if (live) reg_half<LX, ALGO, 0>(g, rec, rows, base, r, nb, wk0, tab, e, s, t, rep, sw);
        __syncthreads();
        if (live) reg_half<LX, ALGO, 1>(g, rec, rows, base, r, nb, wk1, tab, e, s, t, rep, sw);
        __syncthreads();
        if (ALGO == 0) {
            if ((s & 1) == 0)
                reg_wander<K>(wk0, wk1, (nb.y + nb.z) & 1);
            else
                reg_wander<K>(wk1, wk0, (1 + nb.y + nb.z) & 1);
        }
    }

    if (HOUD) {
        // (the tables are no longer read; the first R0 threads own the rows of a temperature)
        if (tid < R0) nbr[tid] = make_ushort4((uint16_t)nb.yp, (uint16_t)nb.ym, (uint16_t)nb.zp, (uint16_t)nb.zm);
        if (live && rep == 0) {
            diff[tl * R0 + r] = (rows[base + r] ^ rows[base + R0 + r]) & MASK;
            mark[tl * R0 + r] = 0u;
        }
        __syncthreads();
        houdayer_grow<LX>(g, G, t0, sw, e, diff, mark, nbr);
        __syncthreads();
        if (live) rows[base + r] ^= mark[tl * R0 + r];
        __syncthreads();
    }

    if (live) {
        const uint32_t own = rows[base + r];
        const uint32_t dx = own ^ rot_down32<LX>(own), dy = own ^ rows[base + nb.yp], dz = own ^ rows[base + nb.zp];
        int32_t en = 0;
#pragma unroll
        for (int x = 0; x < LX; ++x) {
            const int4 a = rec[2 * (x * R0 + r)];
            en += (2 * (a.x & sbit(dx, x)) - a.x) + (2 * (a.y & sbit(dy, x)) - a.y) + (2 * (a.z & sbit(dz, x)) - a.z);
        }
        atomicAdd(&esum[tl * 2 + rep], (unsigned long long)(int64_t)en);
        *grow = own;
    }
    __syncthreads();
    if (live && r == 0) E[((int64_t)run * 2 + rep) * g.M + slot] = (int64_t)esum[tl * 2 + rep];
}

// ---------------------------------------------------------------------------
// Table variant for rows of LX <= 16 sites: the field of a site from two reads.
// A work-group holds G temperatures (both replicas each), a thread one row of
// one replica, as two words: class c holds the row's sites x = 2j + ((c + q)
// & 1), q = (y + z) & 1 (parity c), site j at bit 4j.  Then the neighbours of a
// class are the other class's words, along y and z at the same j, along x at j
// and j + 1 or j - 1, and three of them combine into an index per nibble:
//   T[c][q * H + h][(2 j + side) * 8 + k] = 2 sum J_d (2 k_d - 1), d = x, y, z
// forward (side 0) or backward (1), k_d = 1 where the bond's spins differ, so
// that n - 2 s h = n + T + T', and a lattice's energy is half the sum of the
// forward entries.  Rows of T are an odd number of words apart, so that lanes
// of consecutive rows start in different banks.
// A walker moves right (RM) or left (LM) by one site each sweep, so half sweep
// 0 takes RM and LM in turn, and the arrays turn by one index every second
// sweep: after even sweeps in rows of q = 1, after odd ones in those of q = 0.
// Threads are ordered by q, so that a wave has one: no lane selects.
// Bound: VALU issue and LDS reads about alike: per site 12 instructions and 2
// reads, where one field from six masked couplings took 35 and two 16-byte
// reads.  200 runs of 40 temperatures of 10^3, 10 sweeps and a Houdayer move:
// 235 us per EMCS (k_pt_emcs_reg 368): 8.5 a sweep (17), 42 the Houdayer move
// (81 to 106), the rest draws, staging and energies.
// The draws' tables and T share LDS, so that two work-groups of 10^3 fit a
// compute unit and one's Houdayer move and draws run under the other's sweeps.
// (Metropolis sweeps need both at once and are bound by their Philox calls: at
// 10^3 they took 695 us here, 562 on the records, k_pt_emcs_reg.)
struct PtTabLds {
    uint32_t tab, T, W, mark, diff, nbr, esum, total;
};

// Words per row of T.
__host__ __device__ constexpr uint32_t pt_tab_stride(int Lx) { return 8u * (uint32_t)Lx + 1u; }

__host__ __device__ inline PtTabLds pt_tab_layout(const PtGeom& g, int G)
{
    PtTabLds l;
    const uint32_t tab = (uint32_t)G * kPtTable * 4u, T = 2u * (uint32_t)g.R0 * pt_tab_stride(g.Lx) * 4u;
    l.tab = l.T = 0;
    uint32_t o = tab > T ? tab : T;
    l.W = o;
    o += (uint32_t)G * 4u * g.R0 * 4u;
    l.mark = o;
    o += (uint32_t)G * g.R0 * 4u;
    l.diff = o;
    o += (uint32_t)G * g.R0 * 4u;
    l.nbr = o;
    o += (uint32_t)g.R0 * 8u;
    l.esum = o;
    o += (uint32_t)G * 16u;
    l.total = o;
    return l;
}

__device__ __forceinline__ uint32_t spread4(uint32_t v)  // bit 2j -> bit 4j, j < 8
{
    v &= 0x5555u;
    v = (v | (v << 8)) & 0x00550055u;
    v = (v | (v << 4)) & 0x05050505u;
    return (v | (v << 2)) & 0x11111111u;
}
__device__ __forceinline__ uint32_t gather2(uint32_t v)  // bit 4j -> bit 2j
{
    v = (v | (v >> 2)) & 0x05050505u;
    v = (v | (v >> 4)) & 0x00550055u;
    return (v | (v >> 8)) & 0x5555u;
}
template <int K>
__device__ __forceinline__ uint32_t nib_next(uint32_t w)  // site j <- site j + 1
{
    return (w >> 4) | ((w & 0xFu) << (4 * K - 4));
}
template <int K>
__device__ __forceinline__ uint32_t nib_prev(uint32_t w)  // site j <- site j - 1
{
    constexpr uint32_t MASK = K == 8 ? 0xFFFFFFFFu : (1u << (4 * K)) - 1u;
    return ((w << 4) & MASK) | (w >> (4 * K - 4));
}

// Indices into T of a row's sites of one class: own word, the other class's
// word of the row, and the neighbour rows' words along +y, +z or -y, -z.
template <int K>
__device__ __forceinline__ uint32_t tab_index(uint32_t own, uint32_t x, uint32_t y, uint32_t z)
{
    return (x | (y << 1) | (z << 2)) ^ (own | (own << 1) | (own << 2));
}

struct PtTabRow {
    unsigned char* lds;
    // byte offsets of class 0 in it: the row's entries of T, its word, and its
    // neighbours' words; and from class 0 to class 1 of T and of W
    uint32_t T, W, yp, ym, zp, zm, cT, cW;
    int q;

    __device__ __forceinline__ uint32_t& at(uint32_t o) const { return *(uint32_t*)(lds + o); }
    // entry idx_j of site j, the nibbles of idx holding one each
    __device__ __forceinline__ int32_t entry(uint32_t row, uint32_t idx, int j, int side) const
    {
        return (int32_t)at(row + (__builtin_amdgcn_ubfe(idx, 4 * j, 3) << 2) + 64 * j + 32 * side);
    }
};

template <int LX, int P>
__device__ __forceinline__ void tab_half(const PtTabRow& a, uint32_t& own, uint32_t other, int32_t (&wk)[LX / 2])
{
    constexpr int K = LX / 2;
    const uint32_t o = P ? 0 : a.cW;  // the other class
    const uint32_t yp = a.at(a.yp + o), ym = a.at(a.ym + o), zp = a.at(a.zp + o), zm = a.at(a.zm + o);
    const bool odd = P ? !a.q : a.q;  // the class starts at x = 1
    const uint32_t xp = odd ? nib_next<K>(other) : other, xm = odd ? other : nib_prev<K>(other);
    const uint32_t F = tab_index<K>(own, xp, yp, zp), B = tab_index<K>(own, xm, ym, zm);
    const uint32_t T = a.T + (P ? a.cT : 0);
    constexpr uint32_t ONES = K == 8 ? 0x11111111u : 0x11111111u & ((1u << (4 * K)) - 1u);
    uint32_t refused = 0;  // bit 4j + 3
    int32_t v[K];
#pragma unroll
    for (int j = 0; j < K; ++j) v[j] = a.entry(T, F, j, 0) + a.entry(T, B, j, 1);
#pragma unroll
    for (int j = K - 1; j >= 0; --j) {
        const int32_t nn = wk[j] + v[j];
        wk[j] = nn >= 0 ? nn : wk[j];
        refused = __builtin_amdgcn_alignbit(refused, (uint32_t)nn, 28);
    }
    own ^= ~(refused >> 3) & ONES;
    a.at(a.W + (P ? a.cW : 0)) = own;
}

// Grid (ceil(M / G), runs); block 128 * ceil(G R0 / 64) <= 1024 threads (whole
// waves of each row parity); dynamic LDS pt_tab_layout(g, G).
template <int LX, bool HOUD>
__global__ __launch_bounds__(1024, LX <= 10 ? 8 : 4) void k_pt_emcs_tab(
    PtGeom g, int G, const uint32_t* __restrict__ gT, uint64_t* __restrict__ spins, const int32_t* __restrict__ perm,
    int64_t* __restrict__ E, const uint32_t* __restrict__ wtab, uint32_t e)
{
    constexpr int K = LX / 2;
    extern __shared__ __align__(16) unsigned char lds[];
    const PtTabLds L = pt_tab_layout(g, G);
    uint32_t* tabs = (uint32_t*)(lds + L.tab);
    uint4* T = (uint4*)(lds + L.T);
    uint32_t* mark = (uint32_t*)(lds + L.mark);
    uint32_t* diff = (uint32_t*)(lds + L.diff);
    unsigned long long* esum = (unsigned long long*)(lds + L.esum);
    ushort4* nbr = (ushort4*)(lds + L.nbr);

    const int R0 = g.R0, H = R0 / 2, Y = g.Ly / 2, tid = threadIdx.x, nthr = blockDim.x;
    const int q = __builtin_amdgcn_readfirstlane(tid >= nthr / 2);
    const int k = tid - q * (nthr / 2);  // (temperature, replica, row of parity q)
    const int tl = k / R0, rep = (k - tl * R0) / H, h = k - (2 * tl + rep) * H;
    const int t0 = blockIdx.x * G, t = t0 + tl, run = blockIdx.y;
    const bool live = tl < G && t < g.M;
    const int z = h / Y, y = 2 * (h - z * Y) + ((q + z) & 1), r = y + g.Ly * z;
    const int yp = y + 1 == g.Ly ? 0 : y + 1, ym = y == 0 ? g.Ly - 1 : y - 1;
    const int zp = z + 1 == g.Lz ? 0 : z + 1, zm = z == 0 ? g.Lz - 1 : z - 1;

    // the draws' tables, and T behind them; the rest of T after the draws
    const int nt = min(G, g.M - t0) * kPtTable / 4, nG = G * kPtTable / 4;  // 16-byte words
    const int nT = 2 * R0 * (int)pt_tab_stride(LX) / 4;                     // (R0 is a multiple of 4)
    for (int i = tid; i < nt; i += nthr) T[i] = ((const uint4*)wtab)[(int64_t)t0 * (kPtTable / 4) + i];
    for (int i = nG + tid; i < nT; i += nthr) T[i] = ((const uint4*)gT)[i];
    if (tid < 2 * G) esum[tid] = 0ull;
    int32_t slot = 0;
    uint64_t* grow = nullptr;
    uint32_t c0 = 0, c1 = 0;
    PtTabRow a;
    a.lds = lds;
    a.cT = 4u * R0 * pt_tab_stride(LX);
    a.cW = 4u * R0;
    a.T = L.T + (live ? 4u * (q * H + h) * pt_tab_stride(LX) : 0u);
    // words [G][2][class][q][H]
    const uint32_t Wl = L.W + (live ? 8u * (2 * tl + rep) * R0 : 0u), Wo = Wl + 4u * (1 - q) * H;
    a.W = Wl + (live ? 4u * (q * H + h) : 0u);
    a.yp = Wo + (live ? 4u * (z * Y + (yp >> 1)) : 0u);
    a.ym = Wo + (live ? 4u * (z * Y + (ym >> 1)) : 0u);
    a.zp = Wo + (live ? 4u * (zp * Y + (y >> 1)) : 0u);
    a.zm = Wo + (live ? 4u * (zm * Y + (y >> 1)) : 0u);
    a.q = q;
    if (live) {
        slot = perm[((int64_t)run * 2 + rep) * g.M + t];
        grow = spins + (((int64_t)run * 2 + rep) * g.M + slot) * R0 + r;
        const uint32_t row = (uint32_t)*grow;
        c0 = spread4(row >> q);
        c1 = spread4(row >> (1 - q));
        a.at(a.W) = c0;
        a.at(a.W + a.cW) = c1;
        if (HOUD && k < H)  // the first replica's rows of the first temperature
            nbr[r] = make_ushort4((uint16_t)(yp + g.Ly * z), (uint16_t)(ym + g.Ly * z), (uint16_t)(y + g.Ly * zp),
                                  (uint16_t)(y + g.Ly * zm));
    }
    __syncthreads();

    const uint32_t* tab = tabs + (live ? tl : 0) * kPtTable;
    int32_t rm[K], lm[K];
#pragma unroll
    for (int j = 0; j < K; ++j) rm[j] = lm[j] = 0;
    if (live) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const uint32_t i = (uint32_t)(2 * j + (c ^ q) + LX * r);
                const u32x4 w = philox10(i, e, (uint32_t)(2 * t + rep), stream_word(kStreamPtWalker, (uint32_t)run),
                                         g.key0, g.key1);
                (c == 0 ? rm : lm)[j] = exp_draw4(tab, w);
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < min(nG, nT); i += nthr) T[i] = ((const uint4*)gT)[i];
    __syncthreads();

    const auto turn = [&] {  // RM to the next index, LM to the one before
        const int32_t last = rm[K - 1], first = lm[0];
#pragma unroll
        for (int j = K - 1; j > 0; --j) rm[j] = rm[j - 1];
        rm[0] = last;
#pragma unroll
        for (int j = 0; j + 1 < K; ++j) lm[j] = lm[j + 1];
        lm[K - 1] = first;
    };
    for (int s = 0; s < g.S; s += 2) {
        if (live) tab_half<LX, 0>(a, c0, c1, rm);
        __syncthreads();
        if (live) tab_half<LX, 1>(a, c1, c0, lm);
        __syncthreads();
        if (s + 1 == g.S) break;
        if (q == 1) turn();
        if (live) tab_half<LX, 0>(a, c0, c1, lm);
        __syncthreads();
        if (live) tab_half<LX, 1>(a, c1, c0, rm);
        __syncthreads();
        if (q == 0) turn();
    }

    if (HOUD) {
        if (live && rep == 0) {
            const uint32_t d0 = c0 ^ a.at(a.W + 2 * a.cW), d1 = c1 ^ a.at(a.W + 3 * a.cW);  // the other replica's row
            diff[tl * R0 + r] = (gather2(d0) << q) | (gather2(d1) << (1 - q));
            mark[tl * R0 + r] = 0u;
        }
        __syncthreads();
        houdayer_grow<LX>(g, G, t0, (uint32_t)run, e, diff, mark, nbr);
        __syncthreads();
        if (live) {
            const uint32_t m = mark[tl * R0 + r];
            c0 ^= spread4(m >> q);
            c1 ^= spread4(m >> (1 - q));
            a.at(a.W) = c0;
            a.at(a.W + a.cW) = c1;
        }
        __syncthreads();
    }

    if (live) {
        const uint32_t x0 = q ? nib_next<K>(c1) : c1, x1 = q ? c0 : nib_next<K>(c0);  // sites one to the right
        const uint32_t F0 = tab_index<K>(c0, x0, a.at(a.yp + a.cW), a.at(a.zp + a.cW));
        const uint32_t F1 = tab_index<K>(c1, x1, a.at(a.yp), a.at(a.zp));
        int32_t en = 0;
#pragma unroll
        for (int j = 0; j < K; ++j)
            en += a.entry(a.T, F0, j, 0) + a.entry(a.T + a.cT, F1, j, 0);
        atomicAdd(&esum[tl * 2 + rep], (unsigned long long)(int64_t)(en / 2));
        *grow = (gather2(c0) << q) | (gather2(c1) << (1 - q));
    }
    __syncthreads();
    if (live && q == 0 && h == 0) E[((int64_t)run * 2 + rep) * g.M + slot] = (int64_t)esum[tl * 2 + rep];
}

// Tempering step: one wave per replica group (run, replica); lane t decides
// pair (t, t+1), first the pairs with t even, then those with t odd.
__global__ __launch_bounds__(256) void k_pt_swap(PtGeom g, int32_t* __restrict__ perm,
                                                 const int64_t* __restrict__ E, int64_t* __restrict__ swaps,
                                                 const uint32_t* __restrict__ ptab, uint32_t e)
{
    __shared__ int32_t sp[4][64];
    __shared__ int64_t se[4][64];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int grp = blockIdx.x * 4 + wv;
    const bool live = grp < 2 * g.runs;
    const int run = grp >> 1, rep = grp & 1;
    if (live && lane < g.M) {
        const int32_t c = perm[(int64_t)grp * g.M + lane];
        sp[wv][lane] = c;
        se[wv][lane] = E[(int64_t)grp * g.M + c];
    }
    const bool pair = live && lane + 1 < g.M;
    u32x4 w{0, 0, 0, 0};
    if (pair)
        w = philox10((uint32_t)lane, e, (uint32_t)rep, stream_word(kStreamPtSwap, (uint32_t)run), g.key0, g.key1);
    __syncthreads();
    for (int ph = 0; ph < 2; ++ph) {
        if (pair && (lane & 1) == ph) {
            const int64_t x = se[wv][lane] - se[wv][lane + 1];
            if (exp_at_least(ptab + (int64_t)lane * kPtTable, w, -x)) {
                const int32_t c = sp[wv][lane];
                sp[wv][lane] = sp[wv][lane + 1];
                sp[wv][lane + 1] = c;
                const int64_t v = se[wv][lane];
                se[wv][lane] = se[wv][lane + 1];
                se[wv][lane + 1] = v;
                swaps[(int64_t)grp * (g.M - 1) + lane] += 1;
            }
        }
        __syncthreads();
    }
    if (live && lane < g.M) perm[(int64_t)grp * g.M + lane] = sp[wv][lane];
}

// Initial spins sigma = bit 31 of word i & 3 of Philox (i >> 2, t, replica,
// 10 << 24 | run) into slot t.  One thread per row; grid covers runs*2*M*R0.
__global__ __launch_bounds__(256) void k_pt_init_spins(PtGeom g, uint64_t* __restrict__ spins)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)g.runs * 2 * g.M * g.R0;
    if (k >= total) return;
    const int r = (int)(k % g.R0);
    const int t = (int)((k / g.R0) % g.M);
    const int rep = (int)((k / ((int64_t)g.R0 * g.M)) % 2);
    const int run = (int)(k / ((int64_t)g.R0 * g.M * 2));
    uint64_t row = 0;
    for (int x = 0; x < g.Lx; ++x) {
        const uint32_t i = (uint32_t)(x + g.Lx * r);
        const u32x4 o = philox10(i >> 2, (uint32_t)t, (uint32_t)rep, stream_word(kStreamPtSpin, (uint32_t)run),
                                 g.key0, g.key1);
        const uint32_t ws[4] = {o.v0, o.v1, o.v2, o.v3};
        row |= (uint64_t)(ws[i & 3] >> 31) << x;
    }
    spins[k] = row;
}

// Reads of runs u0 .. u0 + gridDim.y, a wave per (temperature, run):
// E [run][replica][temperature] through the permutation, and the overlap of
// the two replicas, sum_x s^a s^b = N - 2 (number of differing sites).  The
// rows themselves stay: copying 12.8 MB of them to the host took 2.2 of the
// 3.8 ms of four EMCS and a read at 200 runs of 40 temperatures of 10^3.
__global__ __launch_bounds__(64) void k_pt_read(PtGeom g, int u0, const int32_t* __restrict__ perm,
                                                const int64_t* __restrict__ E, const uint64_t* __restrict__ spins,
                                                int64_t* __restrict__ outE, int64_t* __restrict__ outQ)
{
    const int t = blockIdx.x, lane = threadIdx.x;
    const int64_t b0 = (int64_t)(u0 + blockIdx.y) * 2 * g.M, b1 = b0 + g.M;
    const int64_t s0 = b0 + perm[b0 + t], s1 = b1 + perm[b1 + t];
    int32_t d = 0;
    if (outQ)
        for (int r = lane; r < g.R0; r += 64) d += __popcll((spins[s0 * g.R0 + r] ^ spins[s1 * g.R0 + r]) & g.xmask);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) d += __shfl_xor(d, off, 64);
    if (lane == 0) {
        if (outE) {
            outE[(int64_t)blockIdx.y * 2 * g.M + t] = E[s0];
            outE[((int64_t)blockIdx.y * 2 + 1) * g.M + t] = E[s1];
        }
        if (outQ) outQ[(int64_t)blockIdx.y * g.M + t] = g.N - 2 * (int64_t)d;
    }
}

// Energies of every slot from scratch: grid (M, runs * 2), one block per slot.
__global__ __launch_bounds__(256) void k_pt_energy(PtGeom g, const int4* __restrict__ rec,
                                                   const uint64_t* __restrict__ spins, int64_t* __restrict__ E)
{
    __shared__ unsigned long long acc;
    const int64_t lat = (int64_t)blockIdx.y * g.M + blockIdx.x;  // (run, replica, slot)
    const uint64_t* rw = spins + lat * g.R0;
    if (threadIdx.x == 0) acc = 0ull;
    __syncthreads();
    for (int r = threadIdx.x; r < g.R0; r += blockDim.x) {
        const PtRowNb nb = pt_row_nb(g, r);
        atomicAdd(&acc, (unsigned long long)(int64_t)row_energy<false>(g, rec, r, rw[r], rw[nb.yp], rw[nb.zp]));
    }
    __syncthreads();
    if (threadIdx.x == 0) E[lat] = (int64_t)acc;
}

}  // namespace micsa
