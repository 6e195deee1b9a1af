// Near/far form of the compression operator for spans of n = 2 Lc or 4 Lc rows: one table of exact entries for the whole span.
//
// The operator, its split into exact entries near the diagonal and an interpolated far part, and what the workgroup and its
// waves do are those of freqkv_nearfar.hip (E, K, a_m and b_j as in its header).  What is different here:
//
// *Units.*  Leaves (128 span rows, the sources of 8 moments) start 64 rows ahead of the span: leaf l holds rows
// 128 l - 64 .. 128 l + 63.  A unit is the 64 (n = 2 Lc) or 32 (n = 4 Lc) results that lie in rows 128 u .. 128 u + 127, and its
// exact window is the leaves u and u + 1: 64 rows to spare on both sides.  A tile is 32 results, 2 or 1 to a unit; a wave takes a tile at
// a time, and each fragment of rows that it reads from LDS meets the first and the second parts of its entries.
//
// *Images.*  K has a reflected term, cot((a+b)/2): each row acts a second time, from the other side of the nearer end.  The rows that
// the first and the last leaf have beyond the span hold those images, that is the span's first and last rows in reverse order
// (zeros behind them), and the leaf's moments and the exact entries treat them as rows: with 48 to 64 rows of the span in the last
// leaf no other image is closer than that to any result, so all other images belong to the far part.  So there is one table of
// moments for all leaves, and the exact entries are E(a_m - b_j) alone, the same for every unit: they stay in registers for the life
// of the workgroup, and no wave loads a table of its own at the ends.
//
// *Waves.*  What a wave issues beside its matrix instructions is not hidden behind them (a 32x32x16 product holds its wave for 32 cycles,
// every other instruction for 3 to 6 more), only behind another wave's.  So at ratio 1/2 each SIMD has two computing waves, a tile each, and a
// mover, with 168 registers each; at 1/4, with one tile to a unit, one computing wave and a mover with 256.  A group of 8 tiles takes 2150
// cycles (a wave alone on its SIMD, a tile at a time: 4300; one wave with both tiles of a unit: 3000) of which 1700 are matrix instructions.
//
// *Loads.*  A load of a computing wave waits behind all copies in flight, so no step has any: the far part's tables are the same for all
// inner groups too, because there the images of the neighbourhood are taken with the blocks.  And the compiler must know that none is in
// flight (settle_memory): a wait that it adds for a load on some other path is one for the copies, or for the stores of the last step.
//
// *Error.*  What stands 64 rows from a result already goes through the far part, where the form with a tile at a time has up to 128
// rows more of exact entries.  So the moments' roundings take each other over (pack4_carry), and at ratio 1/4 the groups' local values have
// second parts, for a third product: on channels of one frequency close to the retained length, where the far rows add up in phase, the rms
// error is then 5.7e-4 of the span's rms at 8188 -> 4094 (a tile at a time 6.0e-4), 5.0e-4 (5.3e-4) at 4092 -> 2046, 1.7e-4 (4.2e-4) at 8188 -> 2047
// and 1.8e-4 (2.9e-4) at 4092 -> 1023, on white rows 0.90e-4 (1.04e-4), 0.92e-4 (1.04e-4), 0.43e-4 (0.69e-4) and 0.44e-4 (0.70e-4).  The third product
// and the LDS of the second parts cost 0.5 to 3 % at ratio 1/4, the carries up to 1 %.
//
// Against a tile at a time, same device: 512 head-tensors x 8188 rows 473 -> 448 us, 2048 x 4092 946 -> 863 (bare streams of the same rows
// and results, with the re-read part, take 0.9 and 0.8 of that), 512 x 8188 -> 2047 413 -> 383, 512 x 4092 -> 1023 210 -> 198, but 64 x 4092 ->
// 1023, one task to each compute unit, 26.8 -> 27.3.  What bounds it: the rows that come in for the moments (10 bytes per cycle and compute
// unit, what HBM gives), then rows, results and matrix instructions together; in between 3000 to 4400 cycles of every 55000 or 108000 in
// which the far part is prepared and little moves.
#include "freqkv_nearfar.h"

#include <cmath>
#include <cstring>

namespace freqkv {

namespace {

constexpr int kLead = 64;                 // rows of the first leaf ahead of the span
constexpr int kTab = 7;                   // fragments kept in LDS: moments of a leaf | of the first, an inner, the last block

// exact entries of a unit with TU tiles: 16-row steps with second parts, those around a tile or all
template <int TU> constexpr int kLo = TU == 2 ? 7 : 16;
template <int TU> __host__ __device__ constexpr int lo_step(int tile) { return TU == 2 ? 2 + 5 * tile : 0; }

// ---- tables, built on the device in fp64 and rounded once

// The two terms of K between two positions in span rows.
__device__ double far_term(double q) { return 0.5 * cospi(q) / sinpi(q); }
__device__ double far_direct(double a, double b, double n) { return far_term((a - b) / (2.0 * n)); }
__device__ double far_image(double a, double b, double n) { return far_term((a + b) / (2.0 * n)); }

__device__ Iv leaf_at(int l) { return Iv{128.0 * l, 64.0}; }
// The first and the last leaf, which hold images as well, belong to no block: sources of their own behind the blocks.
__device__ Iv block_at(const NfGeom& g, int b)
{
    const double a = fmax(512.0 * b - kLead, 128.0 - kLead), e = fmin(512.0 * b + 512.0 - kLead, 128.0 * (g.NL - 1) - kLead);
    return Iv{0.5 * (a + e), 0.5 * (e - a)};
}
// Tiles and groups are not cut at the end of the span, so that all have the same tables.
template <int TU> __device__ Iv tile_rows(int t) { const double w = 128.0 / TU; return Iv{w * t + 0.5 * w, 0.5 * w}; }
__device__ Iv group_rows(int c) { return Iv{512.0 * c + 256.0, 256.0}; }

__host__ __device__ inline int near_block0(const NfGeom& g, int c)      // first block of the neighbourhood of group c
{
    const int top = g.NC > kNB ? g.NC - kNB : 0;
    return c < 1 ? 0 : (c - 1 > top ? top : c - 1);
}
// The first and the last group have tables of their own from leaves to tiles: only there are the images of the neighbourhood too close
// to be taken with the blocks.
__host__ __device__ inline bool end_group(const NfGeom& g, int c) { return c == 0 || c == g.NG - 1; }

// Units of 4 leaves that the movers hold at most, each 32 KB of 1.1 MB that a task moves at 8188 rows: 3, 4 at ratio 1/2 448, 442 us, 4, 5, 6, 7 at
// 1/4 384, 386, 379, 387.
template <int TU> constexpr int kUnitHeld = TU == 2 ? 4 : 6;
template <int TU> constexpr int GTiles = kCompute * TU;       // tiles of a group, and computing waves: each takes one

// One thread per 16 bytes (lane) of a fragment.
template <int TU>
__global__ void k_nf_unit_tables(NfGeom g, char* __restrict__ out)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= g.table_bytes / 16) return;
    const int lane = (int)(idx & 63);
    const long long byte = (idx >> 6) * kFrag;
    const int l32 = lane & 31, hw = lane >> 5, l16 = lane & 15, g4 = lane >> 4;
    const double n = g.n;
    bf16x8 v;
    for (int i = 0; i < 8; ++i) {
        double x = 0.0;
        if (byte < g.off_v) {
            // exact entries: [tile][first parts: 16 steps], then [tile][second parts: kLo steps], 16 rows x 32 results
            int f = (int)(byte / kFrag), tile, k;
            const bool second = f >= 16 * TU;
            if (second) { f -= 16 * TU; tile = f / kLo<TU>; k = f % kLo<TU> + lo_step<TU>(tile); }
            else { tile = f / 16; k = f % 16; }
            const long long m = 32 * tile + l32, j = 16 * k + 8 * hw + i - kLead;
            x = g.out_scale * entry((2 * m + 1) * g.n - (2 * j + 1) * (long long)g.Lc, g.n, g.Lc) / (2.0 * n);
            if (second) x -= first_part(x);
        } else if (byte < g.off_m) {
            // moments: [4 steps of 32 rows], 8 moments (then the second parts of their entries) x 32 rows.  cos(Lc b_j) repeats every
            // 4 or 8 rows: any leaf will do.
            const int f = (int)((byte - g.off_v) / kFrag);
            const long long j = 128 - kLead + f * 32 + 8 * g4 + i;
            const Iv iv = leaf_at(1);
            const long long ph = ((2 * j + 1) * (long long)g.Lc) % (4LL * g.n);
            x = lagrange(l16 & 7, (j + 0.5 - iv.c) / iv.h) * cospi((double)ph / (2.0 * n)) / 128.0;
            if (l16 >= 8) x -= first_part(x);
        } else if (byte < g.off_c) {
            // coarse moments of a block from those of its leaves, and their second parts: [first | inner | last]
            const int slot = (int)((byte - g.off_m) / kFrag), b = slot == 0 ? 0 : (slot == 1 ? 1 : g.NC - 1), leaf = 4 * b + g4;
            if (slot == 1 || (leaf > 0 && leaf < g.NL - 1)) {
                const Iv bv = slot == 1 ? Iv{512.0 * b - kLead + 256.0, 256.0} : block_at(g, b);
                x = lagrange(l16 & 7, (leaf_at(leaf).node(i) - bv.c) / bv.h) * 0.25;
                if (l16 >= 8) x -= first_part(x);
            }
        } else if (byte < g.off_f) {
            // local values of two groups from 4 sources: blocks, the first leaf, the last
            const int f = (int)((byte - g.off_c) / kFrag), kst = g.NCp / 4;
            const int c = 2 * (f / kst) + (l16 >> 3), b = 4 * (f % kst) + g4;
            if (c < g.NG && b < g.NC + 2) {
                const int end = b - g.NC, leaf = end > 0 ? g.NL - 1 : 0, b0 = near_block0(g, c), in = end < 0 ? b : leaf / 4;
                const bool far = in < b0 || in >= b0 + kNB;
                const Iv iv = end < 0 ? block_at(g, b) : leaf_at(leaf);
                const double at = group_rows(c).node(l16 & 7), from = iv.node(i);
                if (far && iv.h > 0) x += far_direct(at, from, n);
                if (end < 0 && iv.h > 0 && (far || !end_group(g, c))) x += far_image(at, from, n);
                x *= (end < 0 ? 512.0 : 128.0) / n;
            }
        } else if (byte < g.off_t) {
            // local values of two tiles from the 4 leaves of a neighbouring block: [first group | any in between | last][2 tiles][block]
            const int f = (int)((byte - g.off_f) / kFrag), kind = f / (g.GT / 2 * kNB), mt = f / kNB % (g.GT / 2);
            const int c = kind == 0 ? 0 : (kind == 1 ? 1 : g.NG - 1), t = GTiles<TU> * c + 2 * mt + (l16 >> 3), u = t / TU;
            const int leaf = 4 * (kind == 1 ? f % kNB : near_block0(g, c) + f % kNB) + g4;
            if (kind == 1 || (t < g.NT && leaf < g.NL)) {
                const double at = tile_rows<TU>(t).node(l16 & 7), from = leaf_at(leaf).node(i);
                if (leaf != u && leaf != u + 1) x += far_direct(at, from, n);
                if (kind != 1 && leaf != 0 && leaf != g.NL - 1) x += far_image(at, from, n);
                x *= 128.0 / n;
            }
        } else {
            // results of a tile of a group from its 8 local values and the 8 of its group; then the same again for the second product:
            // with two tiles to a unit the second parts of all 16; with one the second parts of the tile's 8 and, for the second parts of
            // the local values themselves, its first parts once more, and for a third product the group's first and second parts
            const int ff = (int)((byte - g.off_t) / kFrag), product = ff / g.GT, t = ff % g.GT, m = 32 * t + l32;
            const Iv iv = product == 2 || (hw && !(product == 1 && TU == 1)) ? group_rows(0) : tile_rows<TU>(t);
            x = g.out_scale * lagrange(i, ((m + 0.5) * n / g.Lc - iv.c) / iv.h) * ((m & 1) ? -1.0 : 1.0);
            if ((product == 1 && !(hw && TU == 1)) || (product == 2 && hw)) x -= first_part(x);
        }
        v[i] = (__bf16)(float)x;
    }
    *(bf16x8*)(out + idx * 16) = v;
}

// ---- the kernel

// TU: tiles of a unit.
template <int TU>
__global__ __launch_bounds__((GTiles<TU> + kMovers) * 64, TU + 1)
void k_nearfar_units(SlabTable tab, NfGeom g, const char* __restrict__ tables, float* __restrict__ tap)
{
    __shared__ __attribute__((aligned(1024))) char smem[kLdsBytes];
    char* const ring = smem;
    char* const mom = smem + g.R * kSlotB;           // [leaf][channel][8]
    char* const cloc = mom + g.NLm * kVecB;          // [group]...
    constexpr bool TWO_GROUP = TU == 1;              // local values of groups in two parts: all second parts behind all first
    char* const loc = cloc + (TWO_GROUP ? 2 : 1) * g.NGp * kVecB;      // [even group | odd | last][tile of the group]..., with TWO_LOC second parts behind each
    char* const cmom = loc;                          // [block | first leaf | last]..., gone before the first local values of tiles come
    char* const ltab = loc + g.NX * kVecB;           // moments | block moments | with LDS_TABS results from local values
    constexpr int GT = GTiles<TU>, LO = kLo<TU>, kWaves = GT, kThreads = (kWaves + kMovers) * 64;
    constexpr bool TWO_LOC = TU == 1;                // local values of tiles in two parts
    constexpr bool LDS_TABS = TU == 2;               // (three waves to a SIMD: 168 registers)
    constexpr int HELD = kUnitHeld<TU>;              // units of four leaves that the movers hold
    constexpr int LOCB = 8 * kVecB;                  // local values of a group: 8 tiles, or 4 in two parts

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
    const uint32_t rowb = (uint32_t)g.stride_token * 2;

    auto wrap = [&](int s) { return s < 0 ? s + g.R : (s >= g.R ? s - g.R : s); };

    // moments of leaves that do not exist stay zero: they meet zero table entries and must be finite
    for (int i = threadIdx.x; i < (g.NLm + (TWO_GROUP ? 2 : 1) * g.NGp + g.NX) * (kVecB / 16); i += kThreads)
        ((u32x4*)mom)[i] = u32x4{0u, 0u, 0u, 0u};
    for (int i = threadIdx.x; i < kTab * 64; i += kThreads) ((u32x4*)ltab)[i] = *(const u32x4*)(tables + g.off_v + i * 16);
    char* const rt_tab = ltab + kTab * kFrag;        // [first product | second][the tile's part, the same for all | the group's part of each tile]
    constexpr int RT = 512 * (1 + GT);
    if constexpr (LDS_TABS) {
        for (int i = threadIdx.x; i < 2 * RT / 16; i += kThreads) {
            const int second = i >= RT / 16, j = i - second * (RT / 16), part = j / 32;
            ((u32x4*)rt_tab)[i] = *(const u32x4*)(tables + g.off_t + (second * GT + (part ? part - 1 : 0)) * kFrag + (part ? 512 : 0) + (j & 31) * 16);
        }
    }
    settle_memory();
    lds_barrier();

    if (wave >= kWaves) {
        // ---- movers.  Leaves go out in the order in which they are used: last to first for the moments, then, since the
        // first R of them are still in the ring, R, R+1, ... for the results.  A leaf may take its slot when the steps that used the
        // slot's previous leaf are over, i.e. behind the barrier after them.  Slots are taken in one direction round the ring on the
        // way down and in the other on the way up, so that leaf l and leaf l + R share one.
        // A mover issues little besides copies: its own instructions, branches above all, hold up copies and steps, 600 of the 2600 cycles of a
        // step of the results.  So leaves go out in runs (down, up), from a scalar base, held ones four at a time, and the waits are found
        // by a jump (4092 -> 2046 of 16384 head-tensors 6890 -> 6790 us, of 64 29.6 -> 28.9; 8188 -> 2047 of 512 387 -> 382; with four units held, see
        // kUnitHeld, instead of three 28.5, and 8188 -> 4094 of 512 449 -> 443).  With a raised priority they lose what they gain: then their bursts
        // go ahead of what the computing waves read from LDS first (6790 -> 7010).
        const int mv = wave - kWaves;
        const uint32_t ring_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)ring + mv * 32 * kRowB;
        const int row0 = mv * 32 + (lane >> 2);                                               // its row of a leaf in the first of its two copies
        const uint32_t part = (lane & 3) * 16, from0 = (uint32_t)row0 * rowb + part, from1 = from0 + 16 * rowb;
        char* const mine = ring + mv * 32 * kRowB + lane * 16;                                // where it lands, in slot 0
        const int zero0 = 2 * (g.n - (g.NL - 1) * kLeaf + kLead);                             // rows of the last leaf from here on hold nothing
        // Most of a mover's registers are free, and four movers hold units of four leaves in them: read from the ring on the way down (each
        // mover its part) and written back on the way up.  The way up begins with leaf R and goes a unit at a time, so a unit held is one of
        // those: where R is no multiple of 4 it lies in two blocks, and its leaf l is in place l & 3.  The held units lie g.held_every
        // apart, so that what comes from memory in between is asked for all the way up.
        u32x4 held[HELD][4][2];
        const int unit0 = g.R & 3;                           // place of a unit's first leaf
        int held_at[HELD];                                   // first leaves
        static_for<HELD>([&](auto i) { held_at[i.value] = i.value < g.held ? g.held0 + i.value * g.held_every : 1 << 20; });
        int copies = 0;                                      // leaves that came from memory
        int issued = 0, slot = 0, dir = 1, vb = blockIdx.x, ht, c0;
        bool down = true;
        int leaf = g.NL - 1, left = g.NL;                                                     // next leaf, leaves left in the run
        int again = -1;                                      // slot of the last leaf, copied a second time and not yet cut
        const char* src = task_base(vb, &ht, &c0);
        const char* from = nullptr;                          // of the next leaf, if it is an inner one
        const long long leaf_bytes = (long long)kLeaf * rowb;
        auto set_from = [&]() { from = src + ((long long)leaf * kLeaf - kLead) * rowb; };
        set_from();
        // the next `count` leaves, none of them the first or the last, downwards (step -1) or upwards
        auto copy_inner = [&](int count, auto step) {
            for (; count > 0; --count) {
                const uint32_t to = ring_lds + slot * kSlotB;
                lds_dma16(to, from, from0);
                lds_dma16(to + 16 * kRowB, from, from1);
                from += step.value * leaf_bytes;
                slot = wrap(slot + dir);
            }
        };
        auto copy_end = [&](int l) {                         // the first leaf or the last: beyond the ends of the span their images
            static_for<2>([&](auto i) {                      // 16 rows each
                int row = l * kLeaf - kLead + row0 + 16 * i.value;
                row = max(row, ~row);
                row = min(row, 2 * g.n - 1 - row);
                lds_dma16(ring_lds + slot * kSlotB + i.value * 16 * kRowB, src, (uint32_t)row * rowb + part);
            });
            from += down ? -leaf_bytes : leaf_bytes;
            slot = wrap(slot + dir);
        };
        auto issue_until = [&](int limit) {
            while (issued < limit && vb < tasks) {
                int count = min(limit - issued, left);
                issued += count;
                left -= count;
                if (down) {
                    copies += count;
                    if (leaf == g.NL - 1) {
                        copy_end(leaf);
                        --leaf;
                        --count;
                    }
                    const int inner = min(count, leaf);
                    copy_inner(inner, IC<-1>{});
                    leaf -= inner;
                    if (count > inner) copy_end(0);
                } else {
                    for (int m; count > 0; count -= m) {
                        m = min(count, 4 - ((leaf - g.R) & 3));
                        int which = HELD;
                        static_for<HELD>([&](auto b) { which = leaf == held_at[b.value] && m == 4 ? b.value : which; });
                        if (which == HELD) {
                            copies += m;
                            const bool last = leaf + m == g.NL;
                            copy_inner(last ? m - 1 : m, IC<1>{});
                            if (last) {
                                again = slot;
                                copy_end(g.NL - 1);
                            }
                        } else {
                            char* p[4];                      // of the leaf in place l
                            static_for<4>([&](auto l) { p[l.value] = mine + wrap(slot + dir * ((l.value - unit0) & 3)) * kSlotB; });
                            dispatch<HELD>(which, [&](auto b) {
                                static_for<4>([&](auto l) {
                                    static_for<2>([&](auto i) { *(u32x4*)(p[l.value] + i.value * 16 * kRowB) = held[b.value][l.value][i.value]; });
                                });
                            });
                            slot = wrap(slot + 4 * dir);
                            from += 4 * leaf_bytes;
                        }
                        leaf += m;
                    }
                }
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
                    if (vb < tasks) src = task_base(vb, &ht, &c0);
                }
                set_from();
            }
        };
        // the last leaf's rows behind the images (there: this wave's copies of it have landed)
        auto cut = [&](int at) {
            static_for<2>([&](auto i) {
                if (mv * 32 + (lane >> 2) + 16 * i.value >= zero0) *(u32x4*)(mine + at * kSlotB + i.value * 16 * kRowB) = u32x4{0u, 0u, 0u, 0u};
            });
        };
        const bool whole = g.NL < g.R;                       // the span and part of the next one fit the ring
        issue_until(min(g.R, g.NL));
        // of the task: counts at its start; slot of its last leaf and where to go from there; copies up to leaf `end` of the results
        int p0 = 0, d0 = 0, at0 = 0, at_dir = 1;
        auto copied = [&](int end) {
            int c = d0 + g.NL + max(0, end - g.R);
            static_for<HELD>([&](auto i) { c -= between(end - held_at[i.value], 0, 4); });
            return c;
        };
        for (int v = blockIdx.x; v < tasks; v += gridDim.x) {
            int at = wrap(at0 - at_dir * (4 * g.NC - g.NL));         // slot of the block's last leaf
            for (int i = g.NC - 1; i >= 0; --i) {
                wait_copies(copies - (d0 + g.NL - 4 * i));
                if (i == g.NC - 1) cut(at0);
                lds_barrier();
                // held units: this block's places from unit0 on belong to the unit that begins in it, the others to the one before
                static_for<HELD>([&](auto b) {
                    const int begins = 4 * i + unit0 - held_at[b.value];
                    if (begins == 0 || (begins == 4 && unit0)) {
                        static_for<4>([&](auto l) {
                            if ((l.value >= unit0) == (begins == 0)) {
                                const char* const p = mine + wrap(at + at_dir * (3 - l.value)) * kSlotB;
                                static_for<2>([&](auto k) { held[b.value][l.value][k.value] = *(const u32x4*)(p + k.value * 16 * kRowB); });
                            }
                        });
                        asm volatile("; %0" :: "n"(b.value));
                    }
                });
                at = wrap(at + 4 * at_dir);
                lds_barrier();                               // all have read the block: its slots are free
                issue_until(p0 + min(g.NL - 4 * i + g.R, g.NL));
            }
            lds_barrier();
            if (whole) issue_until(p0 + g.R);
            lds_barrier();
            lds_barrier();
            for (int c = 0; c < g.NG; ++c) {
                const int end = min(4 * c + 5, g.NL);
                wait_copies(copies - copied(end));
                if (end == g.NL && again >= 0) {
                    cut(again);
                    again = -1;
                }
                lds_barrier();
                issue_until(p0 + (whole ? g.R : g.NL + 4 * c));
            }
            p0 += g.NL + max(0, g.NL - g.R);
            d0 = copied(g.NL);
            if (g.NL >= g.R) {                               // (as the computing waves' ptr and dir)
                at0 = wrap(at0 - at_dir);
                at_dir = -at_dir;
            } else {
                at0 = wrap(at0 + at_dir * g.NL);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
    }

    // ---- computing waves
    // What a lane derives from its index is recomputed where it is used, from the hardware (the compiler would keep the index, or all that
    // follows from it, in registers): a spilled register comes back behind the copies in flight.
#define NF_LANE()                                                                                                       \
    int lane_v;                                                                                                         \
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane_v));                       \
    [[maybe_unused]] const int l32 = lane_v & 31, hw = lane_v >> 5, l16 = lane_v & 15, g4 = lane_v >> 4, vec16 = l16 * 16
    // a fragment: one scalar offset each
    const auto tabs = __builtin_amdgcn_make_buffer_rsrc((void*)tables, 0, g.table_bytes, 0x00020000);
    auto table = [&](int off) {
        NF_LANE();
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(tabs, lane_v * 16, off, 0));
    };
    // Moment products have the first parts of the table in result rows 0..7 and the second parts in 8..15: the half-waves add
    // them up, the lower for a0, the upper for a1.  [channel][8], 4 per lane.  Of the four roundings each takes over what the one before
    // left: what the moments meet next varies little from one to its neighbour, so that the errors cancel where they used to add up.
    // (25 frequencies from 60 below to 60 above the retained length, rms error over the span's rms: 8188 -> 4094 5.9e-4 -> 5.6e-4, 4092 ->
    // 2046 5.2e-4 -> 4.9e-4, a tile at a time 5.9e-4 and 5.2e-4; white rows 1.0e-4 -> 0.9e-4; no difference in time.)
    auto add_parts = [&](f32x4 a0, f32x4 a1) {
        f32x4 sum;
        static_for<4>([&](auto i) {
            const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a0[i.value]), __float_as_uint(a1[i.value]), false, false);
            sum[i.value] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
        });
        return pack4_carry(sum);
    };
    auto block_moments = [&](int b) {
        NF_LANE();
        const bf16x8 m = *(const bf16x8*)(ltab + (4 + (b == g.NC - 1 ? 2 : (b ? 1 : 0))) * kFrag + lane_v * 16);
        f32x4 a[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        static_for<2>([&](auto h) {
            a[h.value] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(m, *(const bf16x8*)(mom + (4 * b + g4) * kVecB + h.value * 256 + vec16), a[h.value], 0, 0, 0);
        });
        *(u32x2*)(cmom + b * kVecB + hw * 256 + vec16 + (g4 & 1) * 8) = add_parts(a[0], a[1]);
    };

    // A load of a computing wave queues behind the copies in flight, a step's worth of time and more.  So no step loads anything: what it
    // needs is the same for all steps and sits in registers or LDS.
    // Local values of the tiles of a group from the leaves around it: a wave takes two tiles and a half of the channels.
    const int mt = wave % (GT / 2), half0 = wave / (GT / 2);
    auto local_table = [&](int kind, int k) { return table(g.off_f + ((kind * (GT / 2) + mt) * kNB + k) * kFrag); };
    auto local_in = [&](int block0) -> const char* { NF_LANE(); return mom + block0 * 4 * kVecB + g4 * kVecB + half0 * 256 + vec16; };
    auto locals_read = [&](const char* in, auto k) { return *(const bf16x8*)(in + k.value * 4 * kVecB); };
    auto locals_mac = [&](const bf16x8 (&f)[kNB], bf16x8 in, f32x4& a, auto k) {
        a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[k.value], in, k.value ? a : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    };
    auto locals_put = [&](int buf, f32x4 a) {
        NF_LANE();
        char* const p = loc + (2 * mt + hw) * kVecB + half0 * 256 + vec16 + (g4 & 1) * 8 + buf * LOCB;
        const u32x2 first = pack4(a);
        *(u32x2*)p = first;
        if constexpr (TWO_LOC) *(u32x2*)(p + GT * kVecB) = pack4(rest(a, first));
    };
    const int own_wave = wave, own_tile = wave % TU;
    bf16x8 ft[kNB], rt, rt2, rt3;                    // local values of an inner group; results from local values: first, second and third product
    bf16x8 e[16], lo[LO];                            // exact entries, second parts
    static_for<kNB>([&](auto k) { ft[k.value] = local_table(1, k.value); });
    static_for<16>([&](auto k) { e[k.value] = table((own_tile * 16 + k.value) * kFrag); });
    static_for<LO>([&](auto k) { lo[k.value] = table((16 * TU + own_tile * LO + k.value) * kFrag); });
    if constexpr (!LDS_TABS) {
        rt = table(g.off_t + wave * kFrag);
        rt2 = table(g.off_t + (GT + wave) * kFrag);
        rt3 = table(g.off_t + (2 * GT + wave) * kFrag);
        pin(rt);
        pin(rt2);
        pin(rt3);
    }
    static_for<kNB>([&](auto k) { pin(ft[k.value]); });
    static_for<16>([&](auto k) { pin(e[k.value]); });
    static_for<LO>([&](auto k) { pin(lo[k.value]); });

    int ptr = 0, dir = 1;                            // ring slot of the task's first leaf (the span's last), and where to go from there
    for (int vb = blockIdx.x; vb < tasks; vb += gridDim.x) {
        int ht, c0;
        char* const base = task_base(vb, &ht, &c0);
        int wave = own_wave;                             // (opaque: what follows from it would be kept for all tasks, in lanes of registers that are short)
        asm volatile("" : "+s"(wave));
        const int tile = wave % TU;                      // of the unit
        // ---- moments, from the last leaf to the first: a step is one block, a wave takes one leaf, with eight waves half of its channels
        constexpr int H1 = 2 / TU;                       // halves that a wave takes
        const int in_block = wave & 3;
        int s = wrap(ptr + dir * (g.NL - 1 - 4 * (g.NC - 1) - in_block));
        auto block_step = [&](int i) {
            int leaf = 4 * i + in_block;
            asm volatile("" : "+s"(leaf));               // (what follows from it for block 0 would be kept in a register)
            bf16x8 vt[4], xa[4][H1];
            {
                NF_LANE();
                static_for<4>([&](auto k) { vt[k.value] = *(const bf16x8*)(ltab + k.value * kFrag + lane_v * 16); });
            }
            lds_barrier();
            if (leaf < g.NL) {
                NF_LANE();
                const char* x = ring + s * kSlotB + (8 * g4 + (l16 >> 2)) * kRowB + (l16 & 3) * 8 + (wave >> 2) * 32;   // the lane's 8 bytes of a 32-row step
                static_for<4>([&](auto k) {
                    static_for<H1>([&](auto h) {
                        const char* p = x + k.value * 32 * kRowB + h.value * 32;
                        xa[k.value][h.value] = join(read_tr(p), read_tr(p + 4 * kRowB));
                    });
                });
            }
            lds_barrier();                               // the block's slots are free
            if (leaf < g.NL) {
                f32x4 a[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
                static_for<4>([&](auto k) {
                    static_for<H1>([&](auto h) {
                        constexpr int A = H1 == 2 ? h.value : k.value & 1;
                        a[A] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[k.value], xa[k.value][h.value], a[A], 0, 0, 0);
                    });
                });
                if constexpr (H1 == 1) a[0] = a[1] = a[0] + a[1];
                const u32x2 sum = add_parts(a[0], a[1]);     // (with eight waves both halves have the same)
                NF_LANE();
                const int at = (H1 == 2 ? hw : wave >> 2) * 256 + vec16 + (g4 & 1) * 8;
                *(u32x2*)(mom + leaf * kVecB + at) = sum;
                if (leaf == 0) *(u32x2*)(cmom + g.NC * kVecB + at) = sum;
                if (leaf == g.NL - 1) *(u32x2*)(cmom + (g.NC + 1) * kVecB + at) = sum;
            }
            if (i < g.NC - 1 && wave == (i & 3)) block_moments(i + 1);
            s = wrap(s + 4 * dir);
        };
        for (int i = g.NC - 1; i > 0; --i) block_step(i);
        // ---- local values of the groups from the blocks that are far from them: a wave takes half of the channels and every second or fourth
        // pair of groups; tables of KC x 4 blocks at a time, the next ones requested before these are used.  Local values of the first and the last
        // group's tiles from the leaves around them.
        {
            constexpr int KC = 5, BUFS = TU == 2 ? 1 : 3;
            const int h = wave & 1, kst = g.NCp / 4, mts = g.NGp / 2, m0 = wave >> 1;
            constexpr int MS = kWaves / 2;
            const int chunks = (kst + KC - 1) / KC, items = (mts - m0 + MS - 1) / MS * chunks;
            bf16x8 ct[BUFS][KC], fe[2][kNB];
            auto fetch_far = [&](auto buf, int it) {
                const int mf = min(m0 + it / chunks * MS, mts - 1) * kst, kf = it % chunks * KC;
                static_for<KC>([&](auto k) { ct[buf.value][k.value] = table(g.off_c + (mf + min(kf + k.value, kst - 1)) * kFrag); });
            };
            // (requested as early as the registers allow)
            static_for<2>([&](auto i) { static_for<kNB>([&](auto k) { fe[i.value][k.value] = local_table(2 * i.value, k.value); }); });
            block_step(0);
            fetch_far(IC<0>{}, 0);
            lds_barrier();
            if (wave == 0) block_moments(0);
            f32x4 le[2];
            static_for<2>([&](auto end) {
                const char* const in = local_in(near_block0(g, end.value ? g.NG - 1 : 0));
                static_for<kNB>([&](auto k) { locals_mac(fe[end.value], locals_read(in, k), le[end.value], k); });
            });
            __builtin_amdgcn_sched_barrier(0);
            static_for<BUFS - 1>([&](auto i) { fetch_far(IC<i.value + 1>{}, i.value + 1); });
            lds_barrier();
            NF_LANE();
            f32x4 a = {0.f, 0.f, 0.f, 0.f};
            auto far_item = [&](auto buf, int it) {
                const int k0 = it % chunks * KC, m = m0 + it / chunks * MS;
                static_for<KC>([&](auto k) {
                    bf16x8 c = {};                           // (behind the last source lies other data, perhaps not finite)
                    if (4 * (k0 + k.value) + g4 < g.NC + 2) c = *(const bf16x8*)(cmom + (4 * (k0 + k.value) + g4) * kVecB + h * 256 + vec16);
                    a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ct[buf.value][k.value], c, a, 0, 0, 0);
                });
                if (it + BUFS < items) fetch_far(buf, it + BUFS);
                if (k0 + KC >= kst) {                        // all 16 result rows: two groups
                    char* const p = cloc + (2 * m + (g4 >> 1)) * kVecB + h * 256 + vec16 + (g4 & 1) * 8;
                    const u32x2 first = pack4(a);
                    *(u32x2*)p = first;
                    if constexpr (TWO_GROUP) *(u32x2*)(p + g.NGp * kVecB) = pack4(rest(a, first));
                    a = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            };
            for (int it = 0; it < items; it += BUFS)
                static_for<BUFS>([&](auto i) { if (it + i.value < items) far_item(i, it + i.value); });
            lds_barrier();
            locals_put(0, le[0]);
            locals_put(2, le[1]);
            settle_memory();
        }

        // ---- results: a step is one tile per wave, the units of a group
        int at_slot = wrap(ptr + dir * g.NLr);           // slot of leaf 0 (the last one read)
        if (g.NL >= g.R) {                               // the next task goes on from here: where the leaf behind the last would be
            ptr = wrap(ptr - dir);
            dir = -dir;
        } else {
            ptr = wrap(ptr + dir * g.NL);
        }
        const int up = g.NL >= g.R ? dir : -dir;         // leaf l + 1 sits one slot further on this way
        at_slot = wrap(at_slot + up * (wave / TU));
        // Result rows go out through a buffer that ends with the last of them: rows past it are dropped without a branch, which
        // would make every wait for a table expect the stores to be missing and so wait for them too.
        const auto out = __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)((uint32_t)g.Lc * rowb), 0x00020000);
        float* const tp = tap ? tap + ((g.tap_slab0 * g.hts_per_slab + ht) * (long long)g.Lc) * g.d + c0 : nullptr;

        // A lane has result row 32 t + l32, channels 8 q + 4 hw + (0..3) in w[q]; the half-waves trade, so that the lower keeps channels
        // 0..15 of its row and the upper 16..31, then lanes 16 apart, so that one store writes 16 whole 64-byte rows.
        uint32_t w[4][2];
        auto round_tile = [&](const f32x16& acc, int t) {
            if (tp) {
                NF_LANE();
                if (32 * t + l32 < g.Lc)
                    static_for<16>([&](auto i) { tp[(long long)(32 * t + l32) * g.d + 8 * (i.value / 4) + 4 * hw + i.value % 4] = acc[i.value]; });
            }
            static_for<4>([&](auto q) { static_for<2>([&](auto i) { w[q.value][i.value] = pack2(acc[4 * q.value + 2 * i.value], acc[4 * q.value + 2 * i.value + 1]); }); });
        };
        auto store_tile = [&](int t, auto part) {            // in three parts
            constexpr int P = decltype(part)::value;
            auto swap32 = [&](uint32_t& a, uint32_t& b) { const auto s = __builtin_amdgcn_permlane32_swap(a, b, false, false); a = s[0]; b = s[1]; };
            auto swap16 = [&](uint32_t& a, uint32_t& b) { const auto s = __builtin_amdgcn_permlane16_swap(a, b, false, false); a = s[0]; b = s[1]; };
            if constexpr (P == 0) {
                static_for<2>([&](auto q) { static_for<2>([&](auto i) { swap32(w[q.value][i.value], w[q.value + 2][i.value]); }); });
            } else if constexpr (P == 1) {
                static_for<2>([&](auto i) { swap16(w[0][i.value], w[1][i.value]); swap16(w[2][i.value], w[3][i.value]); });
            } else {
                NF_LANE();
                const uint32_t row_lane = (uint32_t)l16 * rowb + g4 * 16;
                static_for<2>([&](auto i) {
                    const int m = 32 * t + 16 * i.value;
                    const u32x4 row = {w[i.value][0], w[i.value][1], w[i.value + 2][0], w[i.value + 2][1]};
                    __builtin_amdgcn_raw_buffer_store_b128(row, out, l16 < g.Lc - m ? row_lane + (uint32_t)m * rowb : ~15u, 0, 0);
                });
            }
        };
        // With one computing wave on a SIMD a tile is stored under the next tile's matrix instructions.
        constexpr bool LATE = TU == 1;
        auto results = [&](auto tile_c) {
            constexpr int V = decltype(tile_c)::value, K0 = lo_step<TU>(V);
            int before = g.NT;                               // tile to be stored: none
            if constexpr (LATE) static_for<4>([&](auto q) { static_for<2>([&](auto i) { w[q.value][i.value] = 0u; }); });
            for (int c = 0; c < g.NG; ++c) {
                const int u = kCompute * c + wave / TU, t = GT * c + wave;
                lds_barrier();
                if (u >= g.NU) break;                        // no unit for this wave in the last step of the task
                NF_LANE();
                const char* const tr16 = ring + (8 * hw + (l16 >> 2)) * kRowB + (g4 & 1) * 32 + (lane_v & 3) * 8;    // its 8 bytes of a 16-row step
                const char* const x0 = tr16 + at_slot * kSlotB;
                const char* const x1 = tr16 + wrap(at_slot + up) * kSlotB;
                at_slot = wrap(at_slot + 4 * up);
                // Row fragments are read kAhead steps ahead, and the order is pinned: left alone the compiler reads the whole window first
                // and runs out of registers.
                constexpr int kAhead = 2;
                bf16x8 xf[kAhead + 1], lf[kNB], far, far2, far3, ra, rb;
                f32x16 acc;
                f32x4 la;
                auto fetch_rows = [&](auto kc) {
                    constexpr int K = decltype(kc)::value;
                    const char* const p = (K < 8 ? x0 : x1) + (K % 8) * 16 * kRowB;
                    xf[K % (kAhead + 1)] = join(read_tr(p), read_tr(p + 4 * kRowB));
                };
                auto mac = [&](bf16x8 x, bf16x8 y) { acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, acc, 0, 0, 0); };
                static_for<16>([&](auto r) { acc[r.value] = 0.f; });
                static_for<kAhead>([&](auto k) { fetch_rows(k); });
                __builtin_amdgcn_sched_barrier(0);
                static_for<16>([&](auto k) {
                    constexpr int K = decltype(k)::value;
                    if constexpr (K + kAhead < 16) fetch_rows(IC<K + kAhead>{});
                    mac(xf[K % (kAhead + 1)], e[K]);
                    if constexpr (K >= K0 && K < K0 + LO) mac(xf[K % (kAhead + 1)], lo[K - K0]);
                    // far part: 8 local values of the tile and 8 of its group; for the second product the tile's, first and second parts; for
                    // the third the group's, second and first
                    if constexpr (K == 4) {
                        NF_LANE();
                        const char* const p = loc + (c == g.NG - 1 && c ? 2 : c & 1) * LOCB + wave * kVecB + l32 * 16;
                        far = *(const bf16x8*)(hw ? cloc + c * kVecB + l32 * 16 : p);
                        far2 = far;
                        if constexpr (TWO_LOC) far2 = *(const bf16x8*)(p + (hw ? GT * kVecB : 0));
                        if constexpr (TWO_GROUP) far3 = *(const bf16x8*)(cloc + (hw ? c : c + g.NGp) * kVecB + l32 * 16);
                        ra = rt;
                        rb = rt2;
                        if constexpr (LDS_TABS) {
                            const char* const q = rt_tab + l32 * 16 + (hw ? (1 + wave) * 512 : 0);
                            ra = *(const bf16x8*)q;
                            rb = *(const bf16x8*)(q + RT);
                        }
                    }
                    if constexpr (K == 7) {
                        mac(far, ra);
                        mac(far2, rb);
                        if constexpr (TWO_GROUP) mac(far3, rt3);
                    }
                    // local values of the next group (an end group has its own already: of no use there, but a branch costs more)
                    if constexpr (K == 9) {
                        const char* const in = local_in(near_block0(g, c + 1));
                        static_for<kNB>([&](auto b) { lf[b.value] = locals_read(in, b); });
                    }
                    if constexpr (K >= 12 && K < 12 + kNB) locals_mac(ft, lf[K - 12], la, IC<K - 12>{});
                    if constexpr (LATE && K >= 1 && K < 4) store_tile(before, IC<K - 1>{});
                    __builtin_amdgcn_sched_barrier(0);
                });
                locals_put(c + 1 & 1, la);
                round_tile(acc, t);
                if constexpr (!LATE) static_for<3>([&](auto p) { store_tile(t, p); });
                before = t;
            }
            if constexpr (LATE) static_for<3>([&](auto p) { store_tile(before, p); });
        };
        if (TU == 1 || tile == 0) results(IC<0>{});
        else results(IC<TU - 1>{});
    }
    settle_memory();
}

#undef NF_LANE

}  // namespace

// Everything that follows from the span alone.  False: no such form (then that of freqkv_nearfar.hip, perhaps).
bool nf_unit_geometry(int n, int Lc, int head_dim, NfGeom* out)
{
    // From 1000 rows at ratio 1/2 and 1500 at 1/4: there the error is no larger than that of a tile at a time, whose end tiles have
    // both terms of K in one rounded entry (1404 -> 351: 1.46e-4 on frequencies close to the retained length against 1.39e-4, 1532 -> 383
    // 1.32e-4 against 1.50e-4), and the time less (1 x 8 heads of 512 rows 8.4 -> 9.2 us, of 1024 rows 11.0 -> 10.9, of 2044
    // 16.6 -> 15.2; 32 x 8 heads of 1024 rows 77 -> 65).
    if (head_dim % kC || n > 16384 || !(n == 2 * Lc ? n >= 1000 : n == 4 * Lc && n >= 1500)) return false;
    const int units = (n + kLeaf - 1) / kLeaf, beyond = units * kLeaf - n;
    if (beyond > 16) return false;                   // 48 to 64 rows of the last leaf are in the span: no other image comes closer to a tile than 32 rows
    NfGeom g;
    memset(&g, 0, sizeof(g));
    g.n = n; g.Lc = Lc; g.d = head_dim;
    g.TU = n == 2 * Lc ? 2 : 1;
    g.NK = 2;
    g.NLO = g.TU == 2 ? kLo<2> : kLo<1>;
    g.GT = kCompute * g.TU;
    g.NU = units;
    g.NL = units + 1;
    g.NC = (g.NL + 3) / 4;
    g.NT = (Lc + 31) / 32;
    g.NG = (units + kCompute - 1) / kCompute;
    g.NB = kNB;
    g.NCp = (g.NC + 2 + 3) / 4 * 4;                  // blocks, first leaf, last
    g.NGp = (g.NG + 1) / 2 * 2;
    g.NLm = 4 * (g.NC > kNB ? g.NC : kNB);
    g.off_v = g.TU * (16 + g.NLO) * kFrag;
    g.off_m = g.off_v + 4 * kFrag;
    g.off_c = g.off_m + 3 * kFrag;
    g.off_f = g.off_c + (g.NGp / 2) * (g.NCp / 4) * kFrag;
    g.off_t = g.off_f + 3 * (g.GT / 2) * kNB * kFrag;
    g.off_w = g.table_bytes = g.off_t + (g.TU == 1 ? 3 : 2) * g.GT * kFrag;
    // ring: what LDS leaves, and at least the five leaves of a step and the four of the next or of the next task's first
    g.NX = g.NCp > 24 ? g.NCp : 24;                  // (three groups' local values take 8 vectors each)
    const int fixed = (g.NLm + (g.TU == 1 ? 2 : 1) * g.NGp + g.NX) * kVecB + kTab * kFrag + (g.TU == 2 ? 2 * 512 * (1 + g.GT) : 0);
    g.R = (kLdsBytes - fixed) / kSlotB;
    if (g.R < 9) return false;
    if (g.R > 19) g.R = 19;                          // more copies than that are never in flight
    if (g.NL < g.R && g.R < g.NL + 4) g.R = g.NL;    // no slots over for part of the next task only
    g.NLr = (g.NL - 1) % g.R;
    // units of four leaves that the movers hold: of those from leaf R on, spread over the rest of the span
    const int held_of = (g.NL - 1 - g.R) / 4;        // (whole ones, without the last leaf, whose rows are cut)
    if (held_of > 0) {
        const int most = g.TU == 2 ? kUnitHeld<2> : kUnitHeld<1>;
        g.held = held_of < most ? held_of : most;
        g.held_every = 4 * (held_of / g.held);
        g.held0 = g.R + g.held_every - 4;
    }
    *out = g;
    return true;
}

hipError_t launch_nf_unit_tables(const NfGeom& g, char* out, hipStream_t st)
{
    const dim3 grid((unsigned)((g.table_bytes / 16 + 255) / 256));
    if (g.TU == 2) hipLaunchKernelGGL((k_nf_unit_tables<2>), grid, dim3(256), 0, st, g, out);
    else           hipLaunchKernelGGL((k_nf_unit_tables<1>), grid, dim3(256), 0, st, g, out);
    return hipGetLastError();
}

hipError_t launch_nearfar_units(const SlabTable& tab, const NfGeom& g, const char* tables, float* tap, unsigned grid, hipStream_t st)
{
    const dim3 block((g.GT + kMovers) * 64);
    if (g.TU == 2) hipLaunchKernelGGL((k_nearfar_units<2>), dim3(grid), block, 0, st, tab, g, tables, tap);
    else           hipLaunchKernelGGL((k_nearfar_units<1>), dim3(grid), block, 0, st, tab, g, tables, tap);
    return hipGetLastError();
}

}  // namespace freqkv
