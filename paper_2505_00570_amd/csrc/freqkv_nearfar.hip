// Near/far form of the compression operator: any span n and any retained length Lc from n/5 up, bf16 caches.  Where n is 2 Lc or 4 Lc
// most spans take the form by units instead (freqkv_nearfar_units.hip).
//
// The operator of Sec. 3.3 Eq. 2-3 with the transforms of Appendix A (n-point DCT-II, the Lc lowest
// coefficients, Lc-point inverse, sqrt(Lc/n)) is, entry by entry,
//     M[m][j] = (1/2n) (E(a_m - b_j) + E(a_m + b_j)),   E(t) = sin(Lc t) cot(t/2),
//     a_m = pi (2m+1) / 2Lc,   b_j = pi (2j+1) / 2n,    sin(Lc (a_m -+ b_j)) = (-1)^m cos(Lc b_j),
// that is a Cauchy matrix between the points a_m and b_j with diagonal factors on both sides:
//     M[m][j] = (1/n) (-1)^m K(a_m, b_j) cos(Lc b_j),   K(a, b) = (cot((a-b)/2) + cot((a+b)/2)) / 2.
// Rows that lie close together along the token axis get the exact entries; K between intervals that are apart is
// smooth, so there it is interpolated on Chebyshev points of both intervals (the kernel-independent fast multipole
// scheme with Lagrange polynomials, 8 points per interval, relative error of the far part below 1e-3 of a share
// that is itself 6 % of the result: 1e-6 in all).  Sizes, in span rows:
//     leaf     128 rows: its 8 moments are sum_j L_s(j) cos(Lc b_j) x_j
//     block    4 leaves: 8 moments from its leaves' (coarse level)
//     tile     32 result rows (32 n/Lc span rows): a window of NK leaves with exact entries, 8 local values from the
//              leaves of the neighbouring blocks
//     group    the GT tiles of one step: 8 local values from all the blocks further away
// Per channel that is about 1.3 M multiply-adds at 6083 -> 3041 against 18.5 M for the dense operator, all of them on
// the matrix cores with bf16 operands: the cache values enter as they are (no scale, no conversion, no range guard),
// the exact entries as the sum of two bf16 parts (16 significant bits; the second part only around the tile, where
// entries are large).  The far part has two parts where they cost little, and one elsewhere: the moment tables (a product
// of 8 moments has 16 result rows: the second parts take the other 8), the tables from local values to results (one more
// product per tile) and, with windows of 3 leaves, the tiles' local values (the same product).  So the rms error stays
// below that of a matrix of the operator in fp16, at every ratio: before the result is rounded, on white rows,
// 6083 -> 2737 1.6e-4 of the RMS (fp16 matrix 1.8e-4; with one part throughout the far field 1.9e-4).  On channels of one frequency close to
// the retained length, where the far rows add up in phase, what has one part shows: up to 9.2e-4 of the span's rms there (fp16 matrix
// 1.8e-4), but for the long spans of which SPILL below speaks.
//
// One workgroup owns 32 channels (64 bytes of every row) of one head-tensor and streams the span twice through a ring
// of LDS slots (a leaf each): first for the moments, then for the result rows, which mostly come from the 256 MB memory-side
// cache then, because 256 workgroups x 64 bytes of each row are still in it: that is why a workgroup takes 32 channels and not a whole
// 256-byte row.  What bounds it: where entries repeat from tile to tile (SHIFTS) moving the rows; else the tables, 22 to 36 KB per tile
// and workgroup against 4 KB of rows for each (6083 -> 3041 of 128 head-tensors 120 us where the rows come from HBM, as they do with several
// caches in turn: twice the time of a copy; 100 to 104 us in calls on one cache, whose rows stay in the memory-side cache).  Ownership
// by columns keeps the in-place write free of hazards: rows are written behind the rows still to be read.
//
// Four waves move data (global -> LDS copies, counted by vmcnt), four compute; apart, because the copies and the loads of
// tables come back in one order: a wave that did both would wait for its newest copies in front of every table.
#include "freqkv_nearfar.h"

#include <cmath>
#include <cstring>
#include <type_traits>

namespace freqkv {

namespace {

// Where the exact window of tile t starts (leaf), and whether the ends of the span shifted it.
struct TileAt { int leaf0, clamped; };
__host__ __device__ inline TileAt tile_at(const NfGeom& g, int t)
{
    const int a = (int)((unsigned)(32 * t) * (unsigned)g.n / (unsigned)g.Lc);       // first span row of the tile
    int l = (a - 32) >> 7;                                                           // at least 32 rows on its left
    const int top = g.NL - g.NK;
    TileAt r;
    r.clamped = l < 0 || l > top;
    r.leaf0 = l < 0 ? 0 : (l > top ? top : l);
    return r;
}
// First of the 16-row steps of the window that get the second bf16 part: the tile in their middle.
__host__ __device__ inline int tile_lo_step(const NfGeom& g, int t, int leaf0)
{
    const int a = (int)((unsigned)(32 * t) * (unsigned)g.n / (unsigned)g.Lc), rows = 32 * g.n / g.Lc;
    const int k = (2 * (a - leaf0 * kLeaf) + rows - 16 * g.NLO + 16) >> 5;
    const int top = 8 * g.NK - g.NLO;
    return k < 0 ? 0 : (k > top ? top : k);
}
__host__ __device__ inline int tile_slot(const NfGeom& g, int t)
{
    if (!g.shifts) return t;
    return t < g.tlo ? g.PT + t : (t >= g.thi ? g.PT + g.tlo + (t - g.thi) : t % g.PT);
}
// Are the moments' tables the same for all leaves but the last?  cos(Lc b_j) is cos(phase of the leaf + angle within it), so the cosines and
// sines of the angles within a leaf do for all, and the moments are their products' sum with the phase's cosine and (negative) sine.
// (Not for spans of up to 3 blocks: the second product costs more than the tables' way does, 251 -> 125 rows of 1728 head-tensors 75.5 -> 78.3 us.
// On longer spans it depends on how many copies are in flight: a table per leaf -> shared, rows from HBM, ratio 0.6: 1600 rows of 16, 32, 128, 512
// head-tensors 16.2 -> 16.8, 16.9 -> 17.8, 40.6 -> 40.1, 143.7 -> 142.0 us; 2600 of 16, 32, 64, 256 23.2 -> 24.0, 26.2 -> 26.7, 34.0 -> 33.5, 123.1 -> 119.9; 4092
// of the same 36.1 -> 36.6, 42.1 -> 41.1, 52.2 -> 50.5, 181.9 -> 178.7.  A choice by the size of the call would make its bits depend on it.)
__host__ __device__ inline bool phased(const NfGeom& g) { return g.NK == 2 && !g.shifts && g.NC > g.NB; }
// First block of the neighbourhood that group gr treats leaf by leaf.
__host__ __device__ inline int group_block0(const NfGeom& g, int gr)
{
    const int a = (int)((unsigned)(32 * g.GT * gr) * (unsigned)g.n / (unsigned)g.Lc);
    const int b = (a - 128) >> 9, top = g.NC > g.NB ? g.NC - g.NB : 0;
    return b < 0 ? 0 : (b > top ? top : b);
}

// ------------------------------------------------------------------------------------------
// tables, built on the device in fp64 and rounded once
// ------------------------------------------------------------------------------------------

// K between two positions in span rows; image_only: without its direct term.
__device__ double far_kernel(double a, double b, double n, bool image_only)
{
    const double s = (a + b) / (2.0 * n), d = (a - b) / (2.0 * n);
    double v = cospi(s) / sinpi(s);
    if (!image_only) v += cospi(d) / sinpi(d);
    return 0.5 * v;
}
// Intervals are cut at the end of the span.
__device__ Iv interval(double a, double b, double n)
{
    if (b > n) b = n;
    return Iv{0.5 * (a + b), 0.5 * (b - a)};
}
__device__ Iv leaf_iv(const NfGeom& g, int l) { return interval(128.0 * l, 128.0 * l + 128.0, g.n); }
__device__ Iv block_iv(const NfGeom& g, int b) { return interval(512.0 * b, 512.0 * b + 512.0, g.n); }
__device__ Iv tile_iv(const NfGeom& g, int t)
{
    const double r = (double)g.n / g.Lc;
    return interval(32.0 * t * r, (32.0 * t + 32.0) * r, g.n);
}
__device__ Iv group_iv(const NfGeom& g, int gr)
{
    const double r = (double)g.n / g.Lc, w = 32.0 * g.GT;
    return interval(w * gr * r, (w * gr + w) * r, g.n);
}

// Near entry of result row m and span row j for table slot `slot`.
__device__ double near_entry(const NfGeom& g, int slot, int m_in, int row_in)
{
    int t = slot;
    bool direct = false;                    // a pattern shared by the tiles in the middle: no reflected term
    if (g.shifts) {
        if (slot < g.PT) {
            t = g.tlo + ((slot - g.tlo) % g.PT + g.PT) % g.PT;
            direct = true;
            if (t >= g.thi) return 0.0;
        } else {
            t = slot - g.PT;
            if (t >= g.tlo) t = g.thi + (t - g.tlo);
        }
    }
    const long long n = g.n, Lc = g.Lc, m = 32LL * t + m_in, j = 128LL * tile_at(g, t).leaf0 + row_in;
    if (t >= g.NT || m >= Lc || j >= n) return 0.0;
    double v = entry((2 * m + 1) * n - (2 * j + 1) * Lc, n, Lc);
    if (!direct) v += entry((2 * m + 1) * n + (2 * j + 1) * Lc, n, Lc);
    return v / (2.0 * n);
}

// What the kernel wants to know of tile t, in one scalar load: first leaf of the window, first step with second parts, table
// slot | slot of the wave's next tile (of this task or the next), first block of the next group's neighbourhood.
__device__ u32x2 tile_words(const NfGeom& g, int t)
{
    const int l = tile_at(g, t).leaf0, next = t + kCompute < g.NT ? t + kCompute : t % kCompute;
    return u32x2{(uint32_t)l | (uint32_t)tile_lo_step(g, t, l) << 8 | (uint32_t)tile_slot(g, t) << 16,
                 (uint32_t)tile_slot(g, next) | (uint32_t)group_block0(g, min(t / g.GT + 1, g.NG - 1)) << 16};
}

// One thread per 16 bytes (lane) of a fragment.
__global__ void k_nf_tables(NfGeom g, char* __restrict__ out)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= g.off_w / 16) {
        const long long w = idx - g.off_w / 16;
        u32x2* const words = (u32x2*)(out + g.off_w);
        if (w < g.NT) words[w] = tile_words(g, (int)w);
        else if (w == g.NT) words[w] = u32x2{(uint32_t)group_block0(g, 0), 0u};
        else if (phased(g) && w <= g.NT + g.NL) {            // cosine and sine of the phase at which a leaf begins
            const double t = (double)((256 * (w - g.NT - 1) * g.Lc) % (4LL * g.n)) / (2.0 * g.n);
            words[w] = u32x2{__float_as_uint((float)cospi(t)), __float_as_uint((float)sinpi(t))};
        }
        return;
    }
    const int lane = (int)(idx & 63);
    const long long byte = (idx >> 6) * kFrag;
    const int l32 = lane & 31, hw = lane >> 5, l16 = lane & 15, g4 = lane >> 4;
    const double n = g.n;
    bf16x8 v;
    for (int i = 0; i < 8; ++i) {
        double x = 0.0;
        if (byte < g.off_v) {
            // exact entries: [slot][first parts: 8 NK steps | second parts: NLO steps], 16 rows x 32 results
            const int f = (int)(byte / kFrag), per = 8 * g.NK + g.NLO;
            const int slot = f / per;
            int k = f - slot * per;
            const bool second = k >= 8 * g.NK;
            if (second) {
                int t = slot;
                if (g.shifts) {
                    if (slot < g.PT) t = g.tlo + ((slot - g.tlo) % g.PT + g.PT) % g.PT;
                    else { t = slot - g.PT; if (t >= g.tlo) t = g.thi + (t - g.tlo); }
                }
                k = k - 8 * g.NK + tile_lo_step(g, t, tile_at(g, t).leaf0);
            }
            x = g.out_scale * near_entry(g, slot, l32, 16 * k + 8 * hw + i);
            if (second) x -= first_part(x);
        } else if (byte < g.off_m) {
            // moments: [slot][4 steps of 32 rows], 8 moments (then the second parts of their entries) x 32 rows.  Slots: one per leaf; all
            // leaves but the last | the last; or (phased) cosines of all leaves but the last, from a phase of zero | their sines | the last
            const int f = (int)((byte - g.off_v) / kFrag), slot = f >> 2;
            const int leaf = phased(g) ? (slot == 2 ? g.NL - 1 : 0) : g.v_slots == 2 ? (slot ? g.NL - 1 : 0) : slot;
            const long long j = 128LL * leaf + (f & 3) * 32 + 8 * g4 + i;
            const Iv iv = phased(g) && slot < 2 ? Iv{64.0, 64.0} : leaf_iv(g, leaf);
            if (iv.h > 0 && (j < g.n || (phased(g) && slot < 2))) {
                const long long ph = ((2 * j + 1) * (long long)g.Lc) % (4LL * g.n);      // cos(Lc b_j)
                const double t = (double)ph / (2.0 * n);
                x = lagrange(l16 & 7, (j + 0.5 - iv.c) / iv.h) * (phased(g) && slot == 1 ? sinpi(t) : cospi(t)) / 128.0;
                if (l16 >= 8) x -= first_part(x);
            }
        } else if (byte < g.off_c) {
            // coarse moments of a block from those of its 4 leaves, and their second parts
            const int b = (int)((byte - g.off_m) / kFrag), leaf = 4 * b + g4;
            const Iv lv = leaf_iv(g, leaf), bv = block_iv(g, b);
            if (lv.h > 0) {
                x = lagrange(l16 & 7, (lv.node(i) - bv.c) / bv.h) * 0.25;
                if (l16 >= 8) x -= first_part(x);
            }
        } else if (byte < g.off_f) {
            // local values of two groups from 4 blocks; with spills the second parts behind the first of each pair of groups
            const int kst = g.NCp / 4, kst2 = g.spills ? 2 * kst : kst, f = (int)((byte - g.off_c) / kFrag), fk = f % kst2;
            const int gr = 2 * (f / kst2) + (l16 >> 3), b = 4 * (fk % kst) + g4;
            if (gr < g.NG && b < g.NC) {
                const int b0 = group_block0(g, gr);
                if (b < b0 || b >= b0 + g.NB)
                    x = far_kernel(group_iv(g, gr).node(l16 & 7), block_iv(g, b).node(i), n, false) * 512.0 / n;
                if (fk >= kst) x -= first_part(x);
            }
        } else if (byte < g.off_t) {
            // local values of two tiles from the 4 leaves of a neighbouring block; with spills the second parts behind each fragment
            const int ff = (int)((byte - g.off_f) / kFrag), f = g.spills ? ff / 2 : ff, mt = f / g.NB;
            const int gr = mt / (g.GT / 2), t = 2 * mt + (l16 >> 3);
            const int leaf = 4 * (group_block0(g, gr) + f % g.NB) + g4;
            const Iv lv = leaf_iv(g, leaf);
            if (t < g.NT && lv.h > 0) {
                const TileAt at = tile_at(g, t);
                const bool near = leaf >= at.leaf0 && leaf < at.leaf0 + g.NK;
                const bool shared = g.shifts && t >= g.tlo && t < g.thi;
                if (!near || shared) x = far_kernel(tile_iv(g, t).node(l16 & 7), lv.node(i), n, near) * 128.0 / n;
                if (g.spills && (ff & 1)) x -= first_part(x);
            }
        } else {
            // results of a tile from its 8 local values and the 8 of its group; [any but the last group | the last][tile], then the
            // same again for the second product: with windows of 2 leaves, and with spills, the second parts of all 16; else the second
            // parts of the tile's 8 and, for the second parts of the local values themselves, its first parts once more
            const int ff = (int)((byte - g.off_t) / kFrag), second = ff >= 2 * g.GT, f = ff - second * 2 * g.GT;
            const int gr = f < g.GT ? 0 : g.NG - 1, t = gr * g.GT + f % g.GT, m = 32 * t + l32;
            if (m < g.Lc) {
                const bool tile_twice = second && g.NK == 3 && !g.spills;
                const Iv iv = hw && !tile_twice ? group_iv(g, gr) : tile_iv(g, t);
                x = g.out_scale * lagrange(i, ((m + 0.5) * n / g.Lc - iv.c) / iv.h) * ((m & 1) ? -1.0 : 1.0);
                if (second && !(hw && tile_twice)) x -= first_part(x);
            }
        }
        v[i] = (__bf16)(float)x;
    }
    *(bf16x8*)(out + idx * 16) = v;
}

// ------------------------------------------------------------------------------------------
// the kernel
// ------------------------------------------------------------------------------------------

// NK: leaves per exact window; NLO: 16-row steps of it with a second part; TPW: tiles per computing wave and step.
// SHIFTS: tables of exact entries repeat from tile to tile (NfGeom::shifts) and stay in registers.
// SPILL, for long spans: 512 bytes of moments per leaf would leave the ring too few slots.  LDS keeps those of the last two blocks, for the
// blocks' own; all of them go to memory too, and come back a block at a time into a window of kWin blocks, ahead of the tiles' local
// values.  Such spans have a matrix form of fp16 entries and fp32 sums beside this one, so everything of the far part has two bf16 parts
// here, tables, moments and local values: on channels of one frequency close to the retained length, where the far rows add up in
// phase, the rms error is 0.44e-4 to 0.64e-4 of the span's rms against 0.87e-4 to 1.8e-4 there (with one part 4.9e-4 to 6.5e-4), on white
// rows 0.44e-4 to 0.68e-4 against 0.87e-4 to 1.8e-4.  The second parts cost 10 to 23 % of the time: half of it the products (three for one),
// the groups' local values above all, half the moments' way back and the ring slots that they take.  Against the matrix form: 14813 -> 8887
// rows of 336 head-tensors 14099 -> 1381 us, 16384 -> 14745 of 32 2189 -> 215, 11787 -> 2946 of 8 229 -> 86.  (Without the window, each wave
// requesting what it needs of a group's 12 leaves: 1429, 224 and 90 us.)
// ALL_NEAR, for spans of up to 3 blocks: no block is far from any group, so there are no blocks' moments and the groups' local values stay
// zero.  Two barriers, a load of tables and the blocks' products less between the readings of a task, which takes 3 to 9 us: 255 -> 127 rows of
// 1728 head-tensors 93.5 -> 72.6 us, 469 -> 117 114 -> 98, 599 -> 299 of 480 57.6 -> 50.0, 1020 -> 918 of 1920 455 -> 438.
template <int NK, int NLO, int TPW, bool SHIFTS, bool SPILL, bool ALL_NEAR>
__global__ __launch_bounds__((kCompute + kMovers) * 64, 2)
void k_nearfar(SlabTable tab, NfGeom g, const char* __restrict__ tables, float* __restrict__ tap)
{
    __shared__ __attribute__((aligned(1024))) char smem[kLdsBytes];
    char* const ring = smem;
    char* const mom = smem + g.R * kSlotB;           // [leaf][channel][8] (SPILL: of 8 leaves)
    char* const cloc = mom + g.NLm * kVecB;          // [group]...
    char* const loc = cloc + g.NGp * kVecB;          // [2][tile of the group]..., with TWO_LOC the second parts behind them
    char* const cmom = loc;                          // [block]..., gone before the first local values of tiles come (SPILL: two parts each)
    char* const ltab = loc + g.NX * kVecB;           // moments of an inner leaf (SHIFTS; PHASED: their cosines) | of an inner block | of the last block
    constexpr int GT = kCompute * TPW;
    char* const win = loc + 4 * GT * kVecB;          // SPILL: moments of kWin blocks [block mod kWin][leaf]..., in the place of cmom as well
    constexpr bool TWO_LOC = NK == 3 || SPILL;       // local values of tiles in two parts
    constexpr int MV = SPILL ? 2 : 1;                // vectors of the moments of a leaf or a block: with SPILL first and second parts

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int tph = g.d / kC;                        // tasks per head-tensor

    // Task -> first row of the span at its channels.  The tasks of a head-tensor take consecutive slots of one XCD
    // (workgroups are dealt round-robin to 8): they read the halves of the same 128-byte lines.
    auto task_base = [&](int vb, int* ht_out, int* c0_out) -> char* {
        const int full = g.hts / 8, per_group = 8 * tph;
        int task = vb;
        if (vb < full * per_group) {
            const int grp = vb / per_group, local = vb - grp * per_group;
            task = (grp * 8 + (local & 7)) * tph + (local >> 3);
        }
        const int ht = task / tph, c0 = (task - ht * tph) * kC;
        const int slab = ht / g.hts_per_slab, r = ht - slab * g.hts_per_slab;
        const int b = r / g.n_heads, h = r - b * g.n_heads;
        *ht_out = ht;
        *c0_out = c0;
        return tab.base[slab] + ((long long)b * g.stride_batch + (long long)h * g.stride_head +
                                 (long long)g.S * g.stride_token + c0) * 2;
    };
    const int tasks = g.hts * tph;
    const u32x2* const words = (const u32x2*)(tables + g.off_w);            // of tiles, then the first group's first block
    const uint32_t rowb = (uint32_t)g.stride_token * 2;

    auto wrap = [&](int s) { return s < 0 ? s + g.R : (s >= g.R ? s - g.R : s); };

    // moments of leaves that do not exist stay zero: they meet zero table entries and must be finite
    for (int i = threadIdx.x; i < (g.NLm + g.NGp + g.NX) * (kVecB / 16); i += (kCompute + kMovers) * 64)
        ((u32x4*)mom)[i] = u32x4{0u, 0u, 0u, 0u};
    for (int i = threadIdx.x; i < kTabFrags * 64; i += (kCompute + kMovers) * 64) {
        const int f = i >> 6;
        const int off = f < 4 ? g.off_v + f * kFrag : g.off_m + (f == 4 ? 0 : g.NC - 1) * kFrag;
        ((u32x4*)ltab)[i] = *(const u32x4*)(tables + off + (i & 63) * 16);
    }
    lds_barrier();

    if (wave >= kCompute) {
        // ---- movers.  Leaves go out in the order in which they are used: last to first for the moments, then, since the
        // first R of them are still in the ring, R, R+1, ... for the results (of 48 leaves at 6083 rows 14 stay in the
        // ring, and 16 in registers, see below).  A leaf may take its slot when the steps that used the slot's previous leaf are over, i.e. behind
        // the barrier after them.  Slots are taken in one direction round the ring on the way down and in the other on
        // the way up, so that leaf l and leaf l + R share one.
        // A mover issues little besides copies: its own instructions, branches above all, are what bounds the first reading when
        // rows come from the memory-side cache.  So leaves go out in runs (down, up), from a scalar base.
        const int mv = wave - kCompute;
        const uint32_t ring_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)ring + mv * 32 * kRowB;
        const int row0 = mv * 32 + (lane >> 2);                                               // its row in the first of its two copies
        const uint32_t part = (lane & 3) * 16;
        // Most of a mover's registers are free, and four movers hold 4 blocks in them: the first whole ones behind the leaves that stay
        // in the ring are read from it on the way down (each mover its part) and written back on the way up.  6083 -> 3041 of 128
        // head-tensors: 127 -> 121 us (5 or 6 blocks need more registers than there are); with less to read again than that and a
        // half (spans up to some 4600 rows) the instructions cost what the copies did.
        const bool hold = g.NL - g.R >= 6 * kHeld;
        const int hold0 = hold ? (g.R + 3) / 4 * 4 : g.NL, hold1 = hold ? hold0 + 4 * kHeld : g.NL;
        u32x4 held[kHeld][4][2];
        int copies = 0;                                      // leaves that came from memory
        int issued = 0, slot = 0, dir = 1, vb = blockIdx.x, ht, c0;
        bool down = true;
        int leaf = g.NL - 1, left = g.NL;                                                     // next leaf, leaves left in the run
        const char* src = task_base(vb, &ht, &c0);
        auto issue_until = [&](int limit) {
            while (issued < limit && vb < tasks) {
                const int count = min(limit - issued, left);
                for (int k = 0; k < count; ++k) {
                    const uint32_t to = ring_lds + slot * kSlotB;
                    if (!down && leaf >= hold0 && leaf < hold1) {
                        char* const p = ring + slot * kSlotB + mv * 32 * kRowB + lane * 16;
                        dispatch<kHeld>((leaf - hold0) >> 2, [&](auto b) {
                            dispatch<4>(leaf & 3, [&](auto l) {
                                static_for<2>([&](auto i) { *(u32x4*)(p + i.value * 16 * kRowB) = held[b.value][l.value][i.value]; });
                            });
                        });
                    } else {
                        static_for<2>([&](auto i) {                  // 16 rows each; past the span: its last row again
                            const uint32_t row = (uint32_t)min(leaf * kLeaf + row0 + 16 * i.value, g.n - 1);
                            lds_dma16(to + i.value * 16 * kRowB, src, row * rowb + part);
                        });
                        ++copies;
                    }
                    slot = wrap(slot + dir);
                    leaf += down ? -1 : 1;
                }
                issued += count;
                left -= count;
                if (left) break;
                if (down && g.NL > g.R) {                    // turn round: leaf R goes where leaf 0 is
                    slot = wrap(slot - dir);
                    dir = -dir;
                    down = false;
                    leaf = g.R;
                    left = g.NL - g.R;
                } else {
                    if (down && g.NL == g.R) {
                        slot = wrap(slot - dir);
                        dir = -dir;
                    }
                    down = true;
                    leaf = g.NL - 1;
                    left = g.NL;
                    vb += gridDim.x;
                }
                if (down && vb < tasks) src = task_base(vb, &ht, &c0);
            }
        };
        const bool whole = g.NL < g.R;                       // the span and part of the next one fit the ring
        issue_until(min(g.R, g.NL));
        // of the task: counts at its start; slot of its last leaf and where to go from there; copies up to leaf `end` of the results
        int p0 = 0, d0 = 0, at0 = 0, at_dir = 1;
        auto copied = [&](int end) { return d0 + g.NL + max(0, min(end, hold0) - g.R) + max(0, end - hold1); };
        for (int v = blockIdx.x; v < tasks; v += gridDim.x) {
            int at = wrap(at0 - at_dir * (4 * g.NC - g.NL));         // slot of the block's last leaf
            for (int i = g.NC - 1; i >= 0; --i) {
                wait_copies(copies - (d0 + g.NL - 4 * i));
                lds_barrier();
                issue_until(p0 + min((i == g.NC - 1 ? 0 : g.NL - 4 * (i + 1)) + g.R, g.NL));
                // (there before the next barrier, and so before a copy can take their slots)
                if (4 * i >= hold0 && 4 * i < hold1) {
                    const char* p[4];
                    static_for<4>([&](auto l) { p[l.value] = ring + wrap(at + at_dir * (3 - l.value)) * kSlotB + mv * 32 * kRowB + lane * 16; });
                    dispatch<kHeld>(i - hold0 / 4, [&](auto b) {
                        static_for<4>([&](auto l) {
                            static_for<2>([&](auto k) { held[b.value][l.value][k.value] = *(const u32x4*)(p[l.value] + k.value * 16 * kRowB); });
                        });
                    });
                }
                at = wrap(at + 4 * at_dir);
            }
            lds_barrier();
            if (whole) issue_until(p0 + g.R);
            if constexpr (!ALL_NEAR) {
                lds_barrier();
                lds_barrier();
            }
            if constexpr (SPILL) lds_barrier();
            for (int t = 0; t < g.NT; t += kCompute) {
                const int first = words[t][0] & 255;
                const int end = (int)(words[min(t + kCompute, g.NT) - 1][0] & 255) + NK;
                wait_copies(copies - copied(end));
                lds_barrier();
                // The next task's leaves come in one go in the last step: what the computing waves load of the next tile's tables waits behind
                // every copy that is in flight, step after step, and without tables in flight the copies take what HBM gives (all as soon as their slots are
                // free -> in the last two steps -> in the last one -> all after it: 2044 -> 1226 rows of 256 head-tensors 98.0, 96.4, 93.0, 93.4 us,
                // 2044 -> 1839 124, 119, 116, 117, 4999 -> 2499 of 256 189.9, 186.6, 187.9, -, 6083 -> 3041 of 128 121.1, 119.8, 120.2, 120.3).
                int limit = p0 + (whole ? g.R : g.NL + first);
                if (!SHIFTS && t + kCompute < g.NT) limit = min(limit, p0 + g.NL + max(0, g.NL - g.R));
                issue_until(limit);
            }
            p0 += g.NL + max(0, g.NL - g.R);
            d0 = copied(g.NL);
            at0 = wrap(at0 - at_dir);
            at_dir = -at_dir;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
    }

    // ---- computing waves
    // What a lane derives from its index is recomputed in every step (an opaque copy of the index): kept across the steps, all
    // of it together does not fit the register file, and a spilled register comes back behind the copies in flight.
    int lane_v = lane;
#define NF_LANE()                                                                                                       \
    asm volatile("" : "+v"(lane_v));                                                                                    \
    [[maybe_unused]] const int l32 = lane_v & 31, hw = lane_v >> 5, l16 = lane_v & 15, g4 = lane_v >> 4, vec16 = l16 * 16
    // a fragment: one scalar offset each
    const auto tabs = __builtin_amdgcn_make_buffer_rsrc((void*)tables, 0, g.table_bytes, 0x00020000);
    const int lane16 = lane * 16;
    auto table = [&](int off) { return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(tabs, lane16, off, 0)); };
    auto lds_table = [&](int f) { return *(const bf16x8*)(ltab + f * kFrag + lane * 16); };
    // Moment products have the first parts of the table in result rows 0..7 and the second parts in 8..15: the half-waves add
    // them up, the lower for channels 0..15 (a0), the upper for 16..31 (a1).  [channel][8], 4 per lane.
    [[maybe_unused]] const auto spill = __builtin_amdgcn_make_buffer_rsrc(SPILL ? g.spill + (long long)blockIdx.x * g.spill_bytes : nullptr, 0,
                                                                         SPILL ? g.spill_bytes : 0, 0x00020000);
    // spill_at: where they go in memory as well (SPILL; negative: nowhere)
    auto put_moments = [&](char* vec, f32x4 a0, f32x4 a1, [[maybe_unused]] int spill_at) {
        NF_LANE();
        f32x4 sum;
        static_for<4>([&](auto i) {
            const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a0[i.value]), __float_as_uint(a1[i.value]), false, false);
            sum[i.value] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
        });
        const u32x2 first = pack4(sum);
        *(u32x2*)(vec + hw * 256 + vec16 + (g4 & 1) * 8) = first;
        if constexpr (SPILL) {
            const int at = hw * 256 + vec16 + (g4 & 1) * 8;
            const u32x2 second = pack4(rest(sum, first));
            *(u32x2*)(vec + kVecB + at) = second;
            if (spill_at >= 0) {
                __builtin_amdgcn_raw_buffer_store_b64(first, spill, at, spill_at, 0);
                __builtin_amdgcn_raw_buffer_store_b64(second, spill, at + kVecB, spill_at, 0);
            }
        }
    };
    // all 16 result rows of a product: two vectors (SPILL: their second parts in memory)
    auto put16 = [&](char* vec, int h, f32x4 a, [[maybe_unused]] int spill_at) {
        NF_LANE();
        const u32x2 first = pack4(a);
        *(u32x2*)(vec + (g4 >> 1) * kVecB + h * 256 + vec16 + (g4 & 1) * 8) = first;
        if constexpr (SPILL)
            __builtin_amdgcn_raw_buffer_store_b64(pack4(rest(a, first)), spill, (g4 >> 1) * kVecB + h * 256 + vec16 + (g4 & 1) * 8, spill_at, 0);
    };

    // Tables that change from step to step are fetched one step ahead of their use, into registers: a load queues behind
    // the copies in flight, a step's worth of time.  What does not change sits in LDS or stays in registers.
    // Local values of the tiles of a group from the leaves around it: a wave takes two tiles and a half of the channels, with TPW == 2
    // one half in each of the group's steps (u) from the same tables.  A table is requested again right after its last use.
    // SPILL with TPW == 1: a block's tables at a time, first and second parts of all would not fit the registers.
    constexpr bool ROLL = SPILL && TPW == 1;
    bf16x8 ft[ROLL ? 1 : kNB], ft2[SPILL && !ROLL ? kNB : 1];
    const int mt = TPW == 2 ? wave : wave & 1;
    auto fetch_local = [&](int gr, auto k) {
        constexpr int I = ROLL ? 0 : k.value;
        const int off = g.off_f + ((gr * (GT / 2) + mt) * kNB + k.value) * (MV * kFrag);
        ft[I] = table(off);
        if constexpr (SPILL) ft2[I] = table(off + kFrag);
    };
    bf16x8 lf;
    f32x4 la;
    const int local_at = (lane >> 4) * MV * kVecB + (TPW == 2 ? 0 : wave >> 1) * 256 + (lane & 15) * 16;
    const char* const local_in = (SPILL ? win : mom) + local_at;
    char* const local_out = loc + 2 * mt * kVecB + (lane >> 5) * kVecB + (TPW == 2 ? 0 : wave >> 1) * 256 + (lane & 15) * 16 + (lane >> 4 & 1) * 8;
    // part: of a block's moments (SPILL: the first parts meet both parts of the table, the second the first)
    auto locals_read = [&](int block0, auto u, auto k, auto part) {
        const int block = block0 + k.value, at = SPILL ? (block - block / kWin * kWin) * 4 * MV * kVecB : block0 * 4 * kVecB + k.value * 4 * kVecB;
        lf = *(const bf16x8*)(local_in + at + (TPW == 2 ? u.value * 256 : 0) + part.value * kVecB);
    };
    auto locals_mac = [&](auto k, auto part) {
        constexpr int I = ROLL ? 0 : k.value;
        if constexpr (decltype(k)::value == 0 && part.value == 0) la = f32x4{0.f, 0.f, 0.f, 0.f};
        la = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ft[I], lf, la, 0, 0, 0);
        if constexpr (SPILL && part.value == 0) la = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ft2[I], lf, la, 0, 0, 0);
    };
    // SPILL: a block's moments come back from memory, a leaf to each wave, into a place of the window that holds none in use
    auto window_load = [&](int block) {
        return __builtin_amdgcn_raw_buffer_load_b128(spill, lane * 16, (min(block, g.NC - 1) * 4 + wave) * (2 * kVecB), 0);
    };
    auto window_put = [&](int block, u32x4 x) {
        block = min(block, g.NC - 1);
        *(u32x4*)(win + ((block - block / kWin * kWin) * 4 + wave) * (2 * kVecB) + lane * 16) = x;
    };
    auto locals_put = [&](int gr, auto u) {
        char* const p = local_out + (gr & 1) * (GT * kVecB) + (TPW == 2 ? u.value * 256 : 0);
        const u32x2 first = pack4(la);
        *(u32x2*)p = first;
        if constexpr (TWO_LOC) *(u32x2*)(p + 2 * GT * kVecB) = pack4(rest(la, first));
    };
    auto block_moments = [&](int b) {
        NF_LANE();
        const bf16x8 m = lds_table(b == g.NC - 1 ? 5 : 4);
        f32x4 a[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        static_for<2>([&](auto h) {
            const char* const in = mom + ((SPILL ? 4 * b & 7 : 4 * b) + g4) * (MV * kVecB) + h.value * 256 + vec16;
            a[h.value] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(m, *(const bf16x8*)in, a[h.value], 0, 0, 0);
            if constexpr (SPILL) a[h.value] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(m, *(const bf16x8*)(in + kVecB), a[h.value], 0, 0, 0);
        });
        put_moments(cmom + b * (MV * kVecB), a[0], a[1], -1);
    };
    // PHASED: one pair of tables for all leaves but the last, the cosines' in LDS, the sines' in registers, as is the last leaf's own.  (A
    // table per leaf, requested a step ahead, comes back behind the copies of all the leaves that are in flight, so that the ring did
    // little to hide their way: 6083 -> 3041 of 128 head-tensors 50 000 -> 40 000 cycles for the first reading, 122.6 -> 120.9 us; 4092 -> 2455 of 512
    // 342 -> 336; the errors are the same to four digits.  For windows of 3 leaves there are no registers left.)
    constexpr bool PHASED = NK == 2 && !SHIFTS && !ALL_NEAR;
    bf16x8 vt[4], vs[PHASED ? 4 : 1];                // moments of the wave's next leaf (PHASED: of the last leaf)
    auto fetch_moments = [&](int leaf) {
        const int off = g.off_v + (PHASED ? 2 : SHIFTS ? (leaf == g.NL - 1) : leaf) * 4 * kFrag;
        static_for<4>([&](auto k) { vt[k.value] = table(off + k.value * kFrag); });
    };
    bf16x8 rt[TPW], rt2[TPW];                        // results from local values: first and second product
    auto fetch_results = [&](bool last) {
        static_for<TPW>([&](auto u) {
            const int off = g.off_t + ((last ? GT : 0) + wave + kCompute * u.value) * kFrag;
            rt[u.value] = table(off);
            rt2[u.value] = table(off + 2 * GT * kFrag);
        });
    };
    auto pin_results = [&]() { static_for<TPW>([&](auto u) { pin(rt[u.value]); pin(rt2[u.value]); }); };
    const int top_leaf = 4 * (g.NC - 1) + wave < g.NL ? 4 * (g.NC - 1) + wave : 4 * (g.NC - 2) + wave;   // the wave's first
    // (all of them in flight together, in the order in which they are used)
    if constexpr (PHASED) static_for<4>([&](auto k) { vs[k.value] = table(g.off_v + (4 + k.value) * kFrag); });
    if (top_leaf >= 0) fetch_moments(top_leaf);
    if constexpr (!ROLL) static_for<kNB>([&](auto k) { fetch_local(0, k); });
    fetch_results(g.NG == 1);

    // table of exact entries of the tile at hand, in registers; replaced step by step when the next tile has another
    constexpr int STEPS = 8 * NK + NLO, PER = STEPS * kFrag;
    bf16x8 e[STEPS];
    auto fetch_entries = [&](int slot) { static_for<STEPS>([&](auto k) { e[k.value] = table(slot * PER + k.value * kFrag); }); };
    int cur_slot = -1;
    if (wave < g.NT) {
        cur_slot = (int)(words[wave][0] >> 16);
        fetch_entries(cur_slot);
    }
    if constexpr (PHASED) static_for<4>([&](auto k) { pin(vs[k.value]); });
    if (SHIFTS || PHASED) static_for<4>([&](auto k) { pin(vt[k.value]); });
    pin_results();
    static_for<STEPS>([&](auto k) { pin(e[k.value]); });

    // parts of addresses that depend on the lane
    const char* const tr16 = ring + (8 * (lane >> 5) + (lane >> 2 & 3)) * kRowB + (lane >> 4 & 1) * 32 + (lane & 3) * 8;    // its 8 bytes of a 16-row step
    const char* const far_tile = loc + wave * kVecB + (lane & 31) * 16;
    const char* const far_group = cloc + (lane & 31) * 16;
    const uint32_t row_lane = (uint32_t)(lane & 15) * rowb + (lane >> 4) * 16;

    int ptr = 0, dir = 1;                            // ring slot of the task's first leaf (the span's last), and where to go from there
    for (int vb = blockIdx.x; vb < tasks; vb += gridDim.x) {
        int ht, c0;
        char* const base = task_base(vb, &ht, &c0);
        // ---- moments, from the last leaf to the first: a step is one block, a wave takes one leaf
        {
            int s = wrap(ptr + dir * (g.NL - 1 - 4 * (g.NC - 1) - wave));
            for (int i = g.NC - 1; i >= 0; --i) {
                const int leaf = 4 * i + wave;
                if (SHIFTS && leaf != top_leaf)
                    static_for<4>([&](auto k) { vt[k.value] = lds_table(k.value); });
                [[maybe_unused]] bf16x8 vc[4];
                [[maybe_unused]] u32x2 phase;
                if constexpr (PHASED) {
                    static_for<4>([&](auto k) { vc[k.value] = lds_table(k.value); });
                    phase = words[g.NT + 1 + min(leaf, g.NL - 1)];
                }
                lds_barrier();
                if (leaf < g.NL) {
                    NF_LANE();
                    const char* x = ring + s * kSlotB + (8 * g4 + (l16 >> 2)) * kRowB + (l16 & 3) * 8;   // the lane's 8 bytes of a 32-row step
                    f32x4 a[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
                    bf16x8 xa[4][2];                         // all of the leaf first: one wait for LDS instead of eight
                    static_for<4>([&](auto k) {
                        static_for<2>([&](auto h) {
                            const char* p = x + k.value * 32 * kRowB + h.value * 32;
                            xa[k.value][h.value] = join(read_tr(p), read_tr(p + 4 * kRowB));
                        });
                    });
                    __builtin_amdgcn_sched_barrier(0);
                    auto products = [&](const bf16x8 (&t)[4], f32x4 (&to)[2]) {
                        static_for<4>([&](auto k) {
                            static_for<2>([&](auto h) {
                                to[h.value] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t[k.value], xa[k.value][h.value], to[h.value], 0, 0, 0);
                            });
                        });
                    };
                    if (!PHASED || leaf == g.NL - 1) products(vt, a);
                    if constexpr (PHASED) {
                        if (leaf != g.NL - 1) {
                            f32x4 b[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
                            products(vc, a);
                            products(vs, b);
                            const float c = __uint_as_float(phase[0]), s = __uint_as_float(phase[1]);
                            static_for<2>([&](auto h) { static_for<4>([&](auto r) { a[h.value][r.value] = c * a[h.value][r.value] - s * b[h.value][r.value]; }); });
                        }
                    }
                    put_moments(mom + (SPILL ? leaf & 7 : leaf) * (MV * kVecB), a[0], a[1], leaf * (MV * kVecB));
                    if (!SHIFTS && !PHASED) fetch_moments(leaf >= 4 ? leaf - 4 : top_leaf);
                } else if constexpr (SPILL) {                // (a leaf that does not exist: see above)
                    const f32x4 none = {0.f, 0.f, 0.f, 0.f};
                    put_moments(mom + (leaf & 7) * (MV * kVecB), none, none, leaf * (MV * kVecB));
                }
                if (!ALL_NEAR && i < g.NC - 1 && wave == (i & 3)) block_moments(i + 1);
                s = wrap(s + 4 * dir);
            }
        }
        // ---- local values of the groups from the blocks that are far from them: units of two groups and 16 channels, 2 units
        // of a wave and 4 x 4 blocks at a time, their tables requested together
        if constexpr (!ALL_NEAR) {
            NF_LANE();
            // (SPILL: the tables' first parts meet both parts of the blocks' moments, their second parts, kst fragments on, the first)
            const int q0 = wave >> 1, h = wave & 1, blocks4 = g.NCp / 4, kst = MV * blocks4, mts = g.NGp / 2;
            bf16x8 ct[2][4];
            auto fetch_far = [&](int m0, int k0) {
                static_for<2>([&](auto j) {
                    static_for<4>([&](auto k) {
                        ct[j.value][k.value] = table(g.off_c + (min(m0 + 2 * j.value, mts - 1) * kst + min(k0 + k.value, kst - 1)) * kFrag);
                    });
                });
            };
            if constexpr (SPILL) settle_memory();            // the moments are in memory, for all waves behind the barrier
            fetch_far(q0, 0);
            lds_barrier();
            if (wave == 0) block_moments(0);
            lds_barrier();
            for (int m0 = q0; m0 < mts; m0 += 4) {
                f32x4 a[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
                for (int k0 = 0; k0 < kst; k0 += 4) {
                    static_for<4>([&](auto k) {
                        if (k0 + k.value < kst) {
                            bf16x8 c = {}, c2 = {};              // (behind the last block lies other data, perhaps not finite)
                            const bool second = SPILL && k0 + k.value >= blocks4;
                            const int b = 4 * (second ? k0 + k.value - blocks4 : k0 + k.value) + g4;
                            if (b < g.NC) {
                                const char* const in = cmom + b * (MV * kVecB) + h * 256 + vec16;
                                c = *(const bf16x8*)in;
                                if constexpr (SPILL) c2 = *(const bf16x8*)(in + kVecB);
                            }
                            static_for<2>([&](auto j) { a[j.value] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ct[j.value][k.value], c, a[j.value], 0, 0, 0); });
                            if constexpr (SPILL) {
                                if (!second)
                                    static_for<2>([&](auto j) { a[j.value] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ct[j.value][k.value], c2, a[j.value], 0, 0, 0); });
                            }
                        }
                    });
                    if (k0 + 4 < kst) fetch_far(m0, k0 + 4);
                    else if (m0 + 4 < mts) fetch_far(m0 + 4, 0);
                }
                static_for<2>([&](auto j) {
                    const int m = m0 + 2 * j.value;
                    if (m < mts) put16(cloc + 2 * m * kVecB, h, a[j.value], g.spill_cloc + 2 * m * kVecB);
                });
            }
            if constexpr (SPILL) settle_memory();            // the groups' second parts are in memory
        }
        lds_barrier();
        if constexpr (SPILL) {                               // the first kWin blocks that the groups' neighbourhoods take
            u32x4 x[kWin];
            static_for<kWin>([&](auto i) { x[i.value] = window_load((int)words[g.NT][0] + i.value); });
            static_for<kWin>([&](auto i) { window_put((int)words[g.NT][0] + i.value, x[i.value]); });
            lds_barrier();
        }
        // ... and those of the first group's tiles
        static_for<TPW>([&](auto u) {
            static_for<kNB>([&](auto k) {
                if constexpr (ROLL) fetch_local(0, k);
                static_for<MV>([&](auto part) {
                    locals_read((int)words[g.NT][0], u, k, part);
                    locals_mac(k, part);
                });
                if constexpr (!ROLL) { if (u.value == TPW - 1) fetch_local(g.NG > 1, k); }
            });
            locals_put(0, u);
        });

        // ---- results: a step is one tile per wave, a group TPW steps
        int at_leaf = 0, at_slot = wrap(ptr + dir * g.NLr);      // a leaf and its slot (leaf 0: the last one read)
        if (g.NL >= g.R) {                               // the next task goes on from here: where the leaf behind the last would be
            ptr = wrap(ptr - dir);
            dir = -dir;
        } else {
            ptr = wrap(ptr + dir * g.NL);
        }
        const int up = g.NL >= g.R ? dir : -dir;         // leaf l + 1 sits one slot further on this way
        // Result rows go out through a buffer that ends with the last of them: rows past it are dropped without a branch, which
        // would make every wait for a table expect the stores to be missing and so wait for them too.
        const auto out = __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)((uint32_t)g.Lc * rowb), 0x00020000);
        float* const tp = tap ? tap + ((g.tap_slab0 * g.hts_per_slab + ht) * (long long)g.Lc) * g.d + c0 : nullptr;

        // Rounding and storing a tile, in 7 parts that the next tile's matrix instructions cover.  A lane has result row
        // 32 t + l32, channels 8 q + 4 hw + (0..3) in registers 4 q ..; the half-waves trade, so that the lower keeps channels 0..15
        // of its row and the upper 16..31, then lanes 16 apart, so that one store writes 16 whole 64-byte rows.
        uint32_t w[4][2];
        u32x4 row[2];
        auto finish = [&](f32x16& acc, int t, auto part) {
            constexpr int P = decltype(part)::value;
            if constexpr (P == 0) {
                if (tp) {
                    NF_LANE();
                    if (32 * t + l32 < g.Lc)
                        static_for<16>([&](auto i) { tp[(long long)(32 * t + l32) * g.d + 8 * (i.value / 4) + 4 * hw + i.value % 4] = acc[i.value]; });
                }
            }
            if constexpr (P < 4) {
                w[P][0] = pack2(acc[4 * P], acc[4 * P + 1]);
                w[P][1] = pack2(acc[4 * P + 2], acc[4 * P + 3]);
            } else if constexpr (P == 4) {
                static_for<2>([&](auto q) {
                    static_for<2>([&](auto i) {
                        const auto s = __builtin_amdgcn_permlane32_swap(w[q.value][i.value], w[q.value + 2][i.value], false, false);
                        row[q.value][i.value] = s[0];
                        row[q.value][2 + i.value] = s[1];
                    });
                });
            } else if constexpr (P == 5) {
                static_for<4>([&](auto i) {
                    const auto s = __builtin_amdgcn_permlane16_swap(row[0][i.value], row[1][i.value], false, false);
                    row[0][i.value] = s[0];
                    row[1][i.value] = s[1];
                });
            } else {
                // one path for all tiles: behind a branch, the waits for tables would have to expect the stores to be missing
                static_for<2>([&](auto i) {
                    const int m = 32 * t + 16 * i.value;
                    __builtin_amdgcn_raw_buffer_store_b128(row[i.value], out, (lane & 15) < g.Lc - m ? row_lane + (uint32_t)m * rowb : ~15u, 0, 0);
                });
            }
        };
        // One step of group c, part u: tile t into acc, while the tile before it (tp_, in prev; none: a tile past the end) is stored
        // and the local values of the next group's tiles are computed.
        // (Windows of 3 leaves leave no registers for that: there a tile is stored at the end of its own step.)
        constexpr bool LATE = NK == 2;
        int before = g.NT + kCompute;                    // a tile past the end: nothing to store
        auto step = [&](int c, auto uc, f32x16& acc, f32x16& prev) {
            constexpr int U = decltype(uc)::value;
            const int tl = wave + kCompute * U, t = GT * c + tl;
            // what the step needs to know of its tile: a scalar load, ahead of the barrier (behind it its wait would take in LDS reads)
            const u32x2 word = words[min(t, g.NT - 1)];
            const int next_slot = (int)(word[1] & 0xffff), block0 = (int)(word[1] >> 16), next_group = c + 1 < g.NG ? c + 1 : 0;
            // SPILL: requested ahead of the barrier, where the wave waits anyhow: the second parts of the group's values, for the upper
            // half-wave; the block that the window takes in (TPW == 1: the first of two); ROLL: the first block's tables
            [[maybe_unused]] bf16x8 glo;
            [[maybe_unused]] u32x4 incoming;
            if constexpr (SPILL) {
                if constexpr (ROLL) fetch_local(next_group, IC<0>{});
                glo = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(spill, (lane & 31) * 16, g.spill_cloc + c * kVecB, 0));
                incoming = window_load(block0 + kNB + U);
            }
            lds_barrier();
            if (t >= g.NT) {                             // no tile for this wave in the last step of the task
                if constexpr (LATE) static_for<7>([&](auto p) { finish(prev, before, p); });
                before = t;
                return;
            }
            const int leaf0 = (int)(word[0] & 255), klo = (int)(word[0] >> 8 & 255);
            at_slot = wrap(at_slot + up * (leaf0 - at_leaf));
            at_leaf = leaf0;
            const int s0 = at_slot * kSlotB, s1 = wrap(at_slot + up) * kSlotB, s2 = NK == 3 ? wrap(at_slot + 2 * up) * kSlotB : 0;
            const char *const x0 = tr16 + s0, *const x1 = tr16 + s1, *const x2 = NK == 3 ? tr16 + s2 : nullptr;
            // 8 NK matrix instructions with the first parts, then NLO with the second; operands are read kAhead instructions
            // ahead, and the order is pinned: left alone the compiler reads the whole window first and runs out of registers
            constexpr int kAhead = 3;
            bf16x8 xf[kAhead + 1], far, far2;
            auto fetch_rows = [&](auto kc) {
                constexpr int K = decltype(kc)::value;
                const char* p;
                if constexpr (K < 8 * NK) {
                    p = (K < 8 ? x0 : K < 16 ? x1 : x2) + (K % 8) * 16 * kRowB;
                } else {
                    const int ks = klo + K - 8 * NK;
                    if constexpr (NK == 2)
                        p = tr16 + ((ks >= 8 ? s1 : s0) + (ks & 7) * 16 * kRowB);
                    else                                         // (a choice among three would become an array in scratch memory)
                        p = tr16 + (wrap(at_slot + up * (ks >> 3)) * kSlotB + (ks & 7) * 16 * kRowB);
                }
                xf[K % (kAhead + 1)] = join(read_tr(p), read_tr(p + 4 * kRowB));
            };
            static_for<16>([&](auto r) { acc[r.value] = 0.f; });
            static_for<kAhead>([&](auto k) { fetch_rows(k); });
            static_for<STEPS>([&](auto k) {
                constexpr int K = decltype(k)::value;
                if constexpr (K + kAhead < STEPS) fetch_rows(IC<K + kAhead>{});
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[K % (kAhead + 1)], e[K], acc, 0, 0, 0);
                if constexpr (!SHIFTS) e[K] = table(next_slot * PER + K * kFrag);
                // Local values of the next group (behind the last: of no use, but a branch costs more): reads, products and the result,
                // a few instructions apart.  The tables are requested ahead of the step's stores: their wait then passes over them.
                if constexpr (SPILL) {
                    // a third of the step for each block: reads, products, reads, products; then its tables for the step after (ROLL:
                    // the next block's)
                    constexpr int THIRD = STEPS / kNB, B = K / THIRD, AT = K % THIRD;
                    if constexpr (B < kNB) {
                        if constexpr (AT == THIRD - 6) locals_read(block0, uc, IC<B>{}, IC<0>{});
                        if constexpr (AT == THIRD - 4) locals_mac(IC<B>{}, IC<0>{});
                        if constexpr (AT == THIRD - 3) locals_read(block0, uc, IC<B>{}, IC<1>{});
                        if constexpr (AT == THIRD - 1) {
                            locals_mac(IC<B>{}, IC<1>{});
                            if constexpr (ROLL && B + 1 < kNB) fetch_local(next_group, IC<B + 1>{});
                            if constexpr (!ROLL && U == TPW - 1) fetch_local(c + 2 < g.NG ? c + 2 : 0, IC<B>{});
                            if constexpr (B == kNB - 1) locals_put(c + 1, uc);
                        }
                    }
                    if constexpr (K == STEPS / 2) {
                        window_put(block0 + kNB + U, incoming);
                        if constexpr (TPW == 1) incoming = window_load(block0 + kNB + 1);
                    }
                    if constexpr (TPW == 1 && K == STEPS - 1) window_put(block0 + kNB + 1, incoming);
                } else {
                    constexpr int A = TPW == 2 && U == 0 ? 9 : 2;
                    if constexpr (K >= A && (K - A) % 3 == 0 && (K - A) / 3 < kNB) locals_read(block0, uc, IC<(K - A) / 3>{}, IC<0>{});
                    if constexpr (K >= A + 2 && (K - A) % 3 == 2 && (K - A) / 3 < kNB) {
                        locals_mac(IC<(K - A) / 3>{}, IC<0>{});
                        if constexpr (U == TPW - 1) fetch_local(c + 2 < g.NG ? c + 2 : 0, IC<(K - A) / 3>{});
                    }
                    if constexpr (K == A + 3 * kNB) locals_put(c + 1, uc);
                }
                if constexpr (LATE) {
                    if constexpr (K >= 2 && K < 6) finish(prev, before, IC<K - 2>{});
                    if constexpr (K == 10) finish(prev, before, IC<4>{});
                    if constexpr (K == 12) finish(prev, before, IC<5>{});
                    if constexpr (K == 14) finish(prev, before, IC<6>{});
                }
                // far part: 8 local values of the tile and 8 of its group; for the second product the tile's, first and second parts (SPILL:
                // the same again, and the second parts of all 16 for a third)
                if constexpr (K == STEPS - 5) {
                    const char* const p = far_tile + (c & 1) * (GT * kVecB) + U * (kCompute * kVecB);
                    far = *(const bf16x8*)(lane < 32 ? p : far_group + c * kVecB);
                    if constexpr (SPILL) {
                        far2 = *(const bf16x8*)(p + 2 * GT * kVecB);
                        if (lane >= 32) far2 = glo;
                    } else if constexpr (TWO_LOC) {
                        far2 = *(const bf16x8*)(p + (lane < 32 ? 0 : 2 * GT * kVecB));
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(far, rt[U], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(TWO_LOC && !SPILL ? far2 : far, rt2[U], acc, 0, 0, 0);
            if constexpr (SPILL) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(far2, rt[U], acc, 0, 0, 0);
            if (SHIFTS && next_slot != cur_slot) {           // at the ends of the span only
                fetch_entries(next_slot);
                static_for<STEPS>([&](auto k) { pin(e[k.value]); });
            }
            cur_slot = next_slot;
            before = t;
            if constexpr (!LATE) static_for<7>([&](auto p) { finish(acc, t, p); });
        };
        f32x16 acc0, acc1;
        static_for<16>([&](auto r) { acc0[r.value] = 0.f; acc1[r.value] = 0.f; });
        const int steps = (g.NT + kCompute - 1) / kCompute;
        for (int i = 0; i < steps; i += 2) {
            const int c = TPW == 2 ? i / 2 : i;
            step(c, IC<0>{}, acc0, acc1);
            if (TPW == 1 && g.NG > 1 && c >= g.NG - 2) { fetch_results(c == g.NG - 2); pin_results(); }
            if (i + 1 < steps) {
                step(TPW == 2 ? c : c + 1, IC<TPW - 1>{}, acc1, acc0);
                if (TPW == 1 && c + 1 >= g.NG - 2) { fetch_results(c + 1 == g.NG - 2); pin_results(); }
            }
            if (TPW == 2 && g.NG > 1 && c >= g.NG - 2) { fetch_results(c == g.NG - 2); pin_results(); }
        }
        if constexpr (LATE) {
            if (steps & 1) static_for<7>([&](auto p) { finish(acc0, before, p); });
            else           static_for<7>([&](auto p) { finish(acc1, before, p); });
        }
        if (SHIFTS && top_leaf >= 0) {
            fetch_moments(top_leaf);
            static_for<4>([&](auto k) { pin(vt[k.value]); });
        }
    }
}

#undef NF_LANE

}  // namespace

// Everything that follows from the span alone.  False: no near/far form for this shape.
bool nf_geometry(int n, int Lc, int head_dim, NfGeom* out)
{
    if (head_dim % kC || Lc >= n || n < kNfMinSpan || n > 16384 || 5LL * Lc < n) return false;
    NfGeom g;
    memset(&g, 0, sizeof(g));
    g.n = n; g.Lc = Lc; g.d = head_dim;
    const double tile_rows = 32.0 * n / Lc;
    // The window has 32 rows to spare on the left of a tile and must keep some 24 on its right: 2 leaves up to 72 rows
    // per tile (ratios from 0.44), else 3 (ratios from 0.2: 160 rows).  Second parts around the tile: 8 to 24 rows beyond it on
    // both sides with 6 and 12 steps, 20 or more with 10 (tiles of up to 104 rows, ratios from 0.31).  At ratio 0.25 the
    // rms error on autoregressive rows (0.9) is 0.83e-4 with 10 steps and 0.61e-4 with 12, 0.81e-4 in the fp16 matrix form.
    g.NK = tile_rows <= 72.0 ? 2 : 3;
    g.NLO = g.NK == 2 ? 6 : (tile_rows <= 104.0 ? 10 : 12);
    g.GT = kCompute * (g.NK == 2 ? 2 : 1);
    g.NL = (n + kLeaf - 1) / kLeaf;
    if (g.NL < g.NK) g.NL = g.NK;
    g.NC = (g.NL + 3) / 4;
    g.NT = (Lc + 31) / 32;
    g.NG = (g.NT + g.GT - 1) / g.GT;
    g.NB = kNB;
    g.NCp = g.NC <= 4 ? 4 : (g.NC + 15) / 16 * 16;
    g.NGp = (g.NG + 1) / 2 * 2;
    g.NLm = 4 * (g.NC > g.NB ? g.NC : g.NB);
    // n = s Lc with s = 2 or 4: the exact entries repeat from tile to tile (every PT tiles) but for the reflected term,
    // which then joins the far part except where the reflection of the window is close: at the ends.
    const int s = n / Lc;
    g.shifts = n % Lc == 0 && (s == 2 || s == 4);
    if (g.shifts) {
        g.PT = s == 2 ? 2 : 1;
        g.tlo = 0;
        g.thi = g.NT;
        auto own = [&](int t) {                      // a table of its own: the reflection is close, or the span ends here
            const TileAt at = tile_at(g, t);
            const int a = 32 * t * s, b = a + 32 * s, wa = kLeaf * at.leaf0, wb = wa + kLeaf * g.NK;
            return at.clamped || b > n || wb > n || a + wa < 64 || (n - b) + (n - wb) < 64;
        };
        while (g.tlo < g.thi && own(g.tlo)) ++g.tlo;
        while (g.thi > g.tlo && own(g.thi - 1)) --g.thi;
    }
    // ring: what LDS leaves, and at least the leaves from the first one a step still uses to the last one the next needs
    const int loc_vectors = (g.NK == 2 ? 2 : 4) * g.GT;
    g.NX = g.NCp > loc_vectors ? g.NCp : loc_vectors;
    int need = (int)std::floor((2 * kCompute - 1) * tile_rows / kLeaf) + 1 + g.NK;
    const int turn = (int)std::floor((kCompute * tile_rows + 32.0) / kLeaf) + 2 + 4;   // from a task's last step to the next task's first
    if (need < turn) need = turn;
    if (need < 8) need = 8;
    auto slots_left = [&] { return (kLdsBytes - (g.NLm + g.NGp + g.NX) * kVecB - kTabFrags * kFrag) / kSlotB; };
    g.R = slots_left();
    if (g.R < need && g.NC >= g.NB) {                // in two parts throughout, see the kernel
        g.spills = 1;
        g.spill_cloc = 4 * g.NC * 2 * kVecB;
        g.spill_bytes = g.spill_cloc + g.NGp * kVecB;
        g.NLm = 8 * 2;
        g.NCp = (g.NC + 3) / 4 * 4;
        const int later = 4 * g.GT + kWin * 4 * 2;   // tiles' local values, the window of moments
        g.NX = 2 * g.NCp > later ? 2 * g.NCp : later;
        g.R = slots_left();
    }
    if (g.R < need) return false;
    // By units, where that form exists; but not where this one has two parts throughout, for the error that the matrix form of such
    // spans has: by units 11132 -> 2783 rows would be 5.1e-4 off at the retained length (0.45e-4 here, matrix form 0.9e-4), in 69 us for 84
    // at 12284 -> 3071 of 64 head-tensors (matrix form 687).
    if (!g.spills && nf_unit_geometry(n, Lc, head_dim, out)) return true;
    const int slots = g.shifts ? g.PT + g.tlo + (g.NT - g.thi) : g.NT, parts = g.spills ? 2 : 1;
    g.v_slots = phased(g) ? 3 : g.shifts ? 2 : g.NL;
    g.off_v = slots * (8 * g.NK + g.NLO) * kFrag;
    g.off_m = g.off_v + g.v_slots * 4 * kFrag;
    g.off_c = g.off_m + g.NC * kFrag;
    g.off_f = g.off_c + (g.NGp / 2) * (g.NCp / 4) * parts * kFrag;
    g.off_t = g.off_f + g.NG * (g.GT / 2) * g.NB * parts * kFrag;
    g.off_w = g.off_t + 4 * g.GT * kFrag;
    g.table_bytes = g.off_w + (g.NT + 1 + (phased(g) ? g.NL : 0)) * 8;
    if (g.R > 19) g.R = 19;                          // more copies than that are never in flight
    if (g.NL < g.R && g.R < g.NL + 4) g.R = g.NL;    // no slots over for part of the next task only
    g.NLr = (g.NL - 1) % g.R;
    *out = g;
    return true;
}

hipError_t launch_nf_tables(const NfGeom& g, char* out, hipStream_t st)
{
    if (g.TU) return launch_nf_unit_tables(g, out, st);
    const long long threads = g.off_w / 16 + g.NT + 1 + g.NL;
    hipLaunchKernelGGL(k_nf_tables, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, g, out);
    return hipGetLastError();
}

hipError_t launch_nearfar(const SlabTable& tab, const NfGeom& g, const char* tables, float* tap, unsigned most_wgs, hipStream_t st)
{
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    const unsigned tasks = (unsigned)(g.hts * (g.d / kC)), resident = (unsigned)cus / 8 * 8;
    unsigned grid = resident >= 8 && tasks > resident ? resident : tasks;
    if (g.spills && grid > most_wgs) grid = most_wgs;
    if (!grid || (g.spills && !g.spill)) return hipErrorInvalidValue;
    if (g.TU) return launch_nearfar_units(tab, g, tables, tap, grid, st);
    const dim3 block((kCompute + kMovers) * 64);
    auto launch = [&](auto spills, auto all_near) {
        constexpr bool SPILL = decltype(spills)::value, ALL_NEAR = decltype(all_near)::value;
        if (g.NK == 2) {
            if (g.shifts) hipLaunchKernelGGL((k_nearfar<2, 6, 2, true, SPILL, ALL_NEAR>), dim3(grid), block, 0, st, tab, g, tables, tap);
            else          hipLaunchKernelGGL((k_nearfar<2, 6, 2, false, SPILL, ALL_NEAR>), dim3(grid), block, 0, st, tab, g, tables, tap);
        } else if (g.NLO == 10) {
            hipLaunchKernelGGL((k_nearfar<3, 10, 1, false, SPILL, ALL_NEAR>), dim3(grid), block, 0, st, tab, g, tables, tap);
        } else {
            if (g.shifts) hipLaunchKernelGGL((k_nearfar<3, 12, 1, true, SPILL, ALL_NEAR>), dim3(grid), block, 0, st, tab, g, tables, tap);
            else          hipLaunchKernelGGL((k_nearfar<3, 12, 1, false, SPILL, ALL_NEAR>), dim3(grid), block, 0, st, tab, g, tables, tap);
        }
    };
    if (g.spills)          launch(std::true_type{}, std::false_type{});
    else if (g.NC <= kNB)  launch(std::false_type{}, std::true_type{});
    else                   launch(std::false_type{}, std::false_type{});
    return hipGetLastError();
}

}  // namespace freqkv
