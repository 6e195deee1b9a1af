// gfx950 kernels for chunk-wise (prefill) attention over the compacted cache.
//
// The tokens of an incoming chunk are the last q_len cached rows; query i sits at in-cache position
// p_i = cur_len - q_len + i and attends to rows [0, p_i]: sinks, compressed rows, the earlier tokens of its
// chunk and itself (Sec. 3.4 Eq. 5).  Keys are cached un-rotated and take the rotary embedding of their
// row index when they are read; queries take the one of p_i (closing paragraph of Sec. 3.4).
//
// Unlike the one-token case this is a dense contraction (q_len x cur_len x d per head, twice), so it runs
// on the matrix cores, as a streaming-softmax attention kernel.  Small passes put the cached operands
// into MFMA fragment order first (all fp16: a bf16 cache value is exact in fp16, and the rotated keys and
// queries keep 11 significant bits instead of 8):
//   k_prefill_cs      cos/sin of (row * theta_j) for every cached row, fp64 angle reduction, fp32 table (kept by the library)
//   k_prefill_prep    Kr = rotate(K) in tiles of 32 keys, [tile][group of 8 channels][key][8]; Vt = V transposed in
//                     tiles of 32 keys, [tile][channel block][k-step][half][channel][8 keys], keys permuted so that a
//                     softmax tile, as the matrix core leaves it in registers, is already the second operand of
//                     the weighted sum
// and k_attend_prefill first builds, per wave, Qr = rotate(q) * log2(e)/sqrt(d) for its 32 queries in
// registers (once), then computes S^T = Kr Qr^T for 32 keys x 32 queries at a time, the running softmax per
// query (a query is a column, so its sum is an in-lane reduction plus one exchange between the two
// half-waves at the end), and O^T += Vt P^T.  Where few workgroups use a tile there is no such pass: k_attend_prefill<.., true> reads the cached
// rows and makes the tiles of them itself, in LDS.
#include "freqkv_internal.h"

namespace freqkv {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

template <int I> struct IC { static constexpr int value = I; };
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (I < N) {
        f(IC<I>{});
        static_for<N, I + 1>(f);
    }
}

constexpr int kD = 128;            // head_dim served by this kernel
constexpr int kKeyTile = 32;       // keys per tile
constexpr int kQPerWave = 32;      // queries per wave
constexpr int kPrefillWaves = 8;   // waves per workgroup of the attention kernel
constexpr int kTileBytes = kKeyTile * kD * 2;   // one Kr or Vt tile, fp16
constexpr float kSlack = 14.0f;    // log2 of the largest un-rescaled softmax weight (an fp16 operand: < 2^16)
constexpr float kWeightLimit = 16384.0f;   // 2^kSlack

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ half2v pack_half2(float a, float b)
{
    f32x2 v = {a, b};
    return __builtin_convertvector(v, half2v);          // round to nearest even, one packed conversion
}

// Cached rows that the attention kernel reads keys and values from, where not from the operands that k_prefill_prep wrote.  The operands' pointers stay among
// the kernel's first arguments: behind all others they came 0.1 us later (365 queries over 365 rows of 8 KV heads 14.40 -> 14.49 us, 335 over 4 x 4 x 335 14.07 -> 14.20).
template <bool DIRECT> struct Rows { void* none; };
template <> struct Rows<true> { SlabTable tab; };

// Workgroups of k_prefill_prep to a unit, some of which may have no tile.
__host__ __device__ inline int prep_tiles(int key_tiles) { return key_tiles < 64 || (-key_tiles & 7) * 14 > key_tiles ? key_tiles : (key_tiles + 7) & ~7; }

// Position of the key that sits at storage index s (0..31) of a Vt tile: the matrix core leaves a
// 32x32 result with register r of a lane in half-wave hw at row 8*(r/4) + 4*hw + r%4; k-step t of the
// weighted sum takes registers 8t .. 8t+7, so storage index s = 16t + 8hw + e holds key
// 16t + 8*(e/4) + 4*hw + e%4.
__device__ __forceinline__ int vt_key(int s)
{
    int t = s >> 4, hw = (s >> 3) & 1, e = s & 7;
    return 16 * t + 8 * (e >> 2) + 4 * hw + (e & 3);
}

}  // namespace

// cs[p][j] = (cos, sin)(p * base^(-2j/d)), p < rows, j < d/2.
__global__ void k_prefill_cs(float2* __restrict__ cs, int rows, int d, double base, int rope)
{
    long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    int half = d / 2;
    if (idx >= (long long)rows * half) return;
    int p = (int)(idx / half), j = (int)(idx - (long long)p * half);
    float2 o = {1.f, 0.f};
    if (rope) {
        double theta = pow(base, -2.0 * (double)j / (double)d);
        double x = (double)p * theta;
        double k = rint(x * 0.15915494309189535);
        double r = fma(-k, 6.283185307179586, x);
        r = fma(-k, 2.4492935982947064e-16, r);
        double s, c;
        sincos(r, &s, &c);
        o.x = (float)c;
        o.y = (float)s;
    }
    cs[idx] = o;
}

// One workgroup per (unit, tile of 32 keys) writes the tile's rotated keys and its transposed values (one launch for both: short
// calls are bound by the launches, and the loads of the two halves overlap).
// Keys: a thread rotates a group of 8 pairs of one row; the group of the lower half and its partner group of the upper half
// come from the same two 16-byte loads.  Kr tile layout (fp16): [group of 8 channels g8 = 0..15][key 0..31][8].
// Values: the 32 x 128 bf16 block is read row by row with 16-byte loads, turned through LDS, and written as the Vt tile.
// Vt tile layout (fp16): [channel block db = 0..3][k-step t = 0..1][half-wave hw = 0..1][channel 0..31][8 keys].
__global__ __launch_bounds__(256) void k_prefill_prep(const PrefillGeom, const float2* __restrict__ cs, _Float16* __restrict__ Kr,
                                                      _Float16* __restrict__ Vt, const SlabTable tab)
{
    const PrefillGeom g = first_argument<decltype(k_prefill_prep)>();
    __shared__ uint32_t sm[kKeyTile][kD / 2 + 1];             // [key][pair of channels], one word of padding per row
    constexpr int half = kD / 2, pgn = half / 8;              // groups of 8 pairs per row
    // Workgroups are dealt round-robin to the 8 XCDs: unit by unit, in multiples of 8, so that the tiles of the same rows of all units go to one, and their cos and
    // sin, as many bytes as a unit's keys and values, come to one L2 instead of all (without the multiples -> with them, whole calls: 301 queries over 5001 rows of 8 KV
    // heads 49.8 -> 48.9 us, 945 over 8 x 2375 27.8 -> 26.7, 300 over 8 x 2500 32.5 -> 31.6, 4190 over 4190 of 32 207.6 -> 204.8).  From 64 tiles on, and with up to a fourteenth of them without a tile:
    // some XCDs have more work than others then (4 layers x 4 x 8 x 1056 rows, 33 tiles, 166 -> 170; 2 x 4 x 8 x 1120 102 -> 104; 2 x 2 x 8 x 2110, 66 tiles, 177.8 -> 179.5).  Row by row, with the units of
    // the same rows next to each other, heads that lie 2 MB apart lose (4 x 8 x 8192 rows, 2000 queries, 874 -> 906; 2 layers, 4000 queries, 735 -> 754).
    const int tiles = prep_tiles(g.key_tiles), tile = blockIdx.x % tiles, unit = blockIdx.x / tiles;
    if (tile >= g.key_tiles) return;
    const int layer = unit / g.units_per_layer;
    const int rem = unit - layer * g.units_per_layer;
    const int b = rem / g.n_kv, kvh = rem - b * g.n_kv;
    const long long head = (long long)b * g.stride_batch + (long long)kvh * g.stride_head;
    const uint16_t* khead = (const uint16_t*)tab.base[2 * layer] + head;
    const uint16_t* vhead = (const uint16_t*)tab.base[2 * layer + 1] + head;
    static_assert(kKeyTile * pgn == 256 && kKeyTile * (kD / 8) == 512, "pieces per thread");
    const int key = threadIdx.x / pgn, pg = threadIdx.x % pgn, j0 = pg * 8;    // the thread's key piece
    const int krow = tile * kKeyTile + key;
    u32x4 lo = {0u, 0u, 0u, 0u}, up = lo, vw[2] = {lo, lo};  // rows beyond cur_len are zero
    float2 c[8];
    if (krow < g.cur_len) {
        const uint16_t* row = khead + (long long)krow * g.stride_token;
        lo = *(const u32x4*)(row + j0);
        up = *(const u32x4*)(row + half + j0);
        const f32x4* cr = (const f32x4*)(cs + (long long)krow * half + j0);
        static_for<4>([&](auto i) {
            const f32x4 x = cr[i.value];
            c[2 * i.value] = {x[0], x[1]};
            c[2 * i.value + 1] = {x[2], x[3]};
        });
    }
    static_for<2>([&](auto i) {
        const int piece = threadIdx.x + 256 * i.value;
        const int row = tile * kKeyTile + piece / (kD / 8);
        if (row < g.cur_len) vw[i.value] = *(const u32x4*)(vhead + (long long)row * g.stride_token + piece % (kD / 8) * 8);
    });
    static_for<2>([&](auto i) {
        const int piece = threadIdx.x + 256 * i.value;
        static_for<4>([&](auto w) { sm[piece / (kD / 8)][piece % (kD / 8) * 4 + w.value] = vw[i.value][w.value]; });
    });
    const long long tile0 = ((long long)unit * g.key_tiles + tile) * (kKeyTile * kD);
    {
        half8 lo8 = {}, up8 = {};
        if (krow < g.cur_len) {
            static_for<4>([&](auto i) {
                const float a0 = bf16_lo(lo[i.value]), a1 = bf16_hi(lo[i.value]);
                const float b0 = bf16_lo(up[i.value]), b1 = bf16_hi(up[i.value]);
                const float2 c0 = c[2 * i.value], c1 = c[2 * i.value + 1];
                // lower half: x_j cos - x_{j+d/2} sin;  upper half: x_{j+d/2} cos + x_j sin
                lo8[2 * i.value]     = (_Float16)(a0 * c0.x - b0 * c0.y);
                lo8[2 * i.value + 1] = (_Float16)(a1 * c1.x - b1 * c1.y);
                up8[2 * i.value]     = (_Float16)(b0 * c0.x + a0 * c0.y);
                up8[2 * i.value + 1] = (_Float16)(b1 * c1.x + a1 * c1.y);
            });
        }
        _Float16* dst = Kr + tile0 + ((long long)pg * kKeyTile + key) * 8;
        *(half8*)dst = lo8;
        *(half8*)(dst + pgn * kKeyTile * 8) = up8;
    }
    __syncthreads();
    // thread = (k-step t, half-wave hw, pair of channels): two adjacent 16-byte groups of the tile
    const int cp = threadIdx.x & 63, hw = (threadIdx.x >> 6) & 1, t = threadIdx.x >> 7;
    half8 lov, hiv;
    static_for<8>([&](auto e) {
        const uint32_t w = sm[vt_key(16 * t + 8 * hw + e.value)][cp];
        lov[e.value] = (_Float16)bf16_lo(w);
        hiv[e.value] = (_Float16)bf16_hi(w);
    });
    const int ch = 2 * cp, db = ch >> 5, dl = ch & 31;
    _Float16* dst = Vt + tile0 + (long long)(((db * 2 + t) * 2 + hw) * 32 + dl) * 8;
    *(half8*)dst = lov;
    *(half8*)(dst + 8) = hiv;
}

// Workgroup = 8 waves = 8 tasks of one KV unit, two waves per SIMD; a task is (query head of the KV group,
// block of 32 queries), heads fastest, so that with 4 query heads per KV head the waves walk the same keys.
// A wave keeps its 32 queries, their 128 x 32 output block and two 32 x 32 score blocks in vector registers
// (under 256 in all, so that two waves share a SIMD and the matrix instructions take all operands from the
// vector registers).
// HALVES == 2, for short calls: a workgroup has 4 tasks, and its first and last four waves (two to a SIMD) take the two halves of the
// keys, each with rings of its own; the halves meet in LDS at the end.  So half as many states go through memory as with as many parts
// of the key range more, or none, and no merging kernel.  With 8 KV heads of 4 query heads 1000 queries on 1000 rows 34.2 us in one stream,
// 24.2 in halves; 100 on 1000 25.2 in 3 parts, 21.8 in 3 parts of halves; prefill_cut has more of them.  A step of one tile of each half takes 1.08
// times that of eight tasks (twice the copies).
// DIRECT: keys and values come from the cached rows; a tile is asked for a step and a half ahead of its use, into registers, and rotated, turned and
// written to LDS between the matrix instructions of the weighted sum.  That is some 50 (in halves 100) vector instructions per thread and step beside some 80,
// and 16 KB (in halves 32) of cos and sin through the 64 bytes per cycle of a compute unit beside 16 (32) of keys and values: 0.24 us per step,
// 0.52 in halves.  (In halves cos and sin that turn on from key to key, from the table every eighth tile, made whole calls up to 9 % shorter, 128 queries over
// 4 x 4 x 6431 rows 41.5 -> 37.8 us, but are up to 7e-7 off where the table's are 3e-8.)  Rows touched
// ahead of time, so that they come from the L2, changed nothing.  prefill_direct says which calls gain by it.
template <int HALVES, bool DIRECT>
__global__ __launch_bounds__(kPrefillWaves * 64, 2)
void k_attend_prefill(const PrefillGeom, const _Float16* __restrict__ Kr, const _Float16* __restrict__ Vt,
                      const uint16_t* __restrict__ q, const float2* __restrict__ cs, uint16_t* __restrict__ out,
                      float* __restrict__ lse, float* __restrict__ part_acc, float2* __restrict__ part_ml, const Rows<DIRECT> rows)
{
    const PrefillGeom g = first_argument<decltype(k_attend_prefill<HALVES, DIRECT>)>();
    constexpr int TASKS = kPrefillWaves / HALVES;                        // of a workgroup
    __shared__ __attribute__((aligned(1024))) char ring[HALVES][2][4][kTileBytes];   // of each half: Kr tiles t+1, t+2, t+3 of step t, Vt tiles t .. t+3
    constexpr int QUERIES = 32 * kD * 2, ORIGIN = HALVES == 1 ? (kD / 2) * 8 : 0;
    __shared__ __attribute__((aligned(1024))) char qsm[TASKS][QUERIES + ORIGIN];     // of each task: its queries, and the angles at its first one (in halves: those in a slot not yet used)
    static_assert(sizeof(ring) + sizeof(qsm) <= 160 * 1024, "a compute unit's LDS, all of it in halves");

    static_assert(kTileBytes % (TASKS * 64 * 16) == 0, "whole 16-byte pieces of a tile per thread");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // scalar: the loop bounds below are per wave
    const int lane = threadIdx.x & 63;
    const int half = wave / TASKS, tw = wave % TASKS;
    auto& ksm = ring[half][0];
    auto& vsm = ring[half][1];
    const int l32 = lane & 31, hw = lane >> 5;
    const int tasks_per_unit = g.G * g.q_blocks;
    const int wgs_per_unit = (tasks_per_unit + TASKS - 1) / TASKS;
    // blockIdx -> (KV unit, workgroup of the unit).  Workgroups are dealt round-robin to the 8 XCDs, so inside a
    // group of 8 units the XCD index picks the unit: all workgroups of a unit run on one XCD and share its L2
    // for the unit's K/V tiles (dealt unit by unit, every XCD fetched every unit: 12.7 GB of fabric reads per
    // launch against 2.2 GB of operands).  The units left over after the last full group are dealt plainly.
    // With the key range in parts, only workgroups that see keys of a part are there, part by part, so that every XCD gets as many
    // (those that saw none used to be launched too, side by side with the others: with an even number of parts some XCDs got
    // two rounds and some half of one: 2118 queries on 4237 rows, 2 KV heads of 2, in 4 parts of 2 halves 56.6 -> 37.7 us).
    int unit, wg_seq, split = 0;
    {
        const int grp = blockIdx.x / (8 * g.wgs);
        int local = blockIdx.x - grp * 8 * g.wgs;
        if (grp < g.units / 8) {
            unit = grp * 8 + (local & 7);
            wg_seq = local >> 3;
        } else {
            local = blockIdx.x - (g.units / 8) * 8 * g.wgs;
            unit = (g.units / 8) * 8 + local / g.wgs;
            wg_seq = local % g.wgs;
        }
        while (split + 1 < g.n_split) {
            const int here = wgs_per_unit - prefill_first_wg(g.cur_len, g.q_len, g.G, wgs_per_unit, TASKS, split * g.split_tiles);
            if (wg_seq < here) break;
            wg_seq -= here;
            ++split;
        }
    }
    // later query blocks see more keys: hand them out first so that the long workgroups start early
    const int wg_in_unit = wgs_per_unit - 1 - wg_seq;
    const int task = wg_in_unit * TASKS + tw;
    const bool active = task < tasks_per_unit;
    const int qb = active ? task / g.G : 0;
    const int gh = active ? task - qb * g.G : 0;
    const long long head = (long long)unit * g.G + gh;             // dense query-head index
    const int q0 = qb * kQPerWave;                                 // first query row of this wave
    const int pos0 = g.cur_len - g.q_len + q0;                     // its in-cache position

    // keys this wave needs: [0, pos0 + 31] cut at cur_len; the workgroup loads up to its largest need
    const int my_last = active ? min(pos0 + kQPerWave - 1, g.cur_len - 1) : -1;
    int my_tiles = (my_last + kKeyTile) / kKeyTile;
    const int full_tiles = active ? (pos0 + 1) / kKeyTile : 0;     // tiles every query of the wave sees whole
    int wg_tiles;
    {
        const int last_task = min(wg_in_unit * TASKS + TASKS - 1, tasks_per_unit - 1);
        const int last_qb = last_task / g.G;
        const int wg_last = min(g.cur_len - g.q_len + last_qb * kQPerWave + kQPerWave - 1, g.cur_len - 1);
        wg_tiles = (wg_last + kKeyTile) / kKeyTile;
    }
    // few workgroups: the key tiles of each are cut into n_split parts, whose states k_prefill_merge brings together
    const int part0 = split * g.split_tiles;
    if (g.n_split > 1) {
        wg_tiles = min(wg_tiles, part0 + g.split_tiles);
        my_tiles = min(my_tiles, wg_tiles);
    }
    const bool seen = my_tiles > part0;                            // the task sees keys of this part
    // this half's tiles: t0 .. t0 + steps - 1, of which there may be one less for the second half
    const int steps = HALVES == 1 ? wg_tiles - part0 : (wg_tiles - part0 + 1) / 2;
    const int t0 = part0 + half * steps, t1 = min(t0 + steps, wg_tiles);
    my_tiles = min(my_tiles, t1);

    f32x16 acc[4];              // O^T: [channel block], 32 channels x 32 queries each
    static_for<4>([&](auto db) { static_for<16>([&](auto r) { acc[db.value][r.value] = 0.f; }); });
    float m = 0.f, lsum = 0.f;  // m: reference point of the lane's query (both half-waves agree); lsum: this half-wave's share
    f32x16 negm;                // -m in every register: the accumulator input of the first score instruction of a tile
    static_for<16>([&](auto r) { negm[r.value] = 0.f; });

    const char *ksrc = nullptr, *vsrc = nullptr;
    if constexpr (!DIRECT) {
        ksrc = (const char*)(Kr + (long long)unit * g.key_tiles * (kKeyTile * kD));
        vsrc = (const char*)(Vt + (long long)unit * g.key_tiles * (kKeyTile * kD));
    }
    constexpr int PIECE = kTileBytes / TASKS;          // of a tile, per wave
    const int tid16 = tw * PIECE + lane * 16;
    // this lane's 16 bytes inside a k-step of a tile (keys in even and odd k-steps; values)
    const int frag[2] = {(hw * kKeyTile + (DIRECT ? l32 ^ 4 * hw : l32)) * 16, (hw * kKeyTile + (DIRECT ? l32 ^ (8 + 4 * hw) : l32)) * 16};
    const int vfrag = (hw * kKeyTile + (DIRECT ? l32 >> 1 | (l32 & 1) << 4 : l32)) * 16;

    // Step t consumes tile t: it computes S(t+1) = Kr(t+1) Qr^T while the softmax of S(t) runs, then
    // O^T += Vt(t) P(t)^T.  Kr(t+3) and Vt(t+3) are requested at the start of step t, straight into their ring
    // slots (whose tiles t-1 were consumed a step ago), and have landed at the barrier that ends it.  Keys are
    // thus two barriers ahead of their use, so that the first fragments of Kr(t+2) can be read before the
    // barrier of step t: the matrix instructions of step t+1 then start right behind it.
    // A tile is copied global -> LDS directly, each wave its 1 KB share (the copy is issued from assembly: the
    // compiler, which cannot tell the ring slots apart, would wait for a copy issued through its builtin in
    // front of the next LDS read; the waits are placed by hand, before each barrier).
    typedef __attribute__((address_space(3))) char* lptr_t;
    const uint32_t k_lds = (uint32_t)(uintptr_t)(lptr_t)ksm[0] + tw * PIECE;
    const uint32_t v_lds = (uint32_t)(uintptr_t)(lptr_t)vsm[0] + tw * PIECE;
    auto dma = [&](uint32_t lds, const char* src, int tile, int slot) {
        static_for<PIECE / 1024>([&](auto i) {
            lds_dma16(lds + (slot & 3) * kTileBytes + i.value * 1024, src + (long long)tile * kTileBytes + tid16 + i.value * 1024);
        });
    };
    auto dma_k = [&](int tile, int slot) { dma(k_lds, ksrc, tile, slot); };
    auto dma_v = [&](int tile, int slot) { dma(v_lds, vsrc, tile, slot); };
    // Copies past the last tile are not branched around: they repeat the last tile into a slot that nobody
    // reads any more, which keeps the loop free of branches.
    const int last_tile = (t1 > t0 ? t1 : wg_tiles) - 1;
    // DIRECT: a thread has its piece of a tile in registers, asked for a step ahead: 4 pairs of a key (in halves of two, 16 rows apart), which it
    // rotates, and 4 (8) keys of two channels, which it turns.  Rows beyond cur_len are read as zero, past the end of the buffer.  Keys lie in LDS at
    // place key ^ 4 (group of 8 channels & 3) of their group, channels at place c / 2 + 16 (c & 1) of their block, so that the writes of
    // a wave go to different banks, as do the reads.
    constexpr int NK = HALVES, P = 4, NV = 4 * HALVES;       // keys, pairs, values per channel of a thread
    struct Staged { u32x2 lo[NK], up[NK]; f32x4 angle[NK][2]; uint32_t v[NV]; } sg;        // angle: (cos, sin) of 4 pairs
    __amdgpu_buffer_rsrc_t kbuf, vbuf, cbuf;
    uint32_t koff = 0, voff = 0, coff = 0, row_bytes = 0;
    char *kput = nullptr, *vput = nullptr;             // in slot 0
    if constexpr (DIRECT) {
        const int layer = unit / g.units_per_layer, rem = unit - layer * g.units_per_layer;
        const int b = rem / g.n_kv, kvh = rem - b * g.n_kv;
        const long long at = (long long)b * g.stride_batch + (long long)kvh * g.stride_head;
        const int size = (int)(((long long)(g.cur_len - 1) * g.stride_token + kD) * 2);
        kbuf = __builtin_amdgcn_make_buffer_rsrc((void*)((const uint16_t*)rows.tab.base[2 * layer] + at), 0, size, kBufferFlags);
        vbuf = __builtin_amdgcn_make_buffer_rsrc((void*)((const uint16_t*)rows.tab.base[2 * layer + 1] + at), 0, size, kBufferFlags);
        cbuf = __builtin_amdgcn_make_buffer_rsrc((void*)cs, 0, g.cur_len * (kD / 2) * 8, kBufferFlags);
        row_bytes = (uint32_t)g.stride_token * 2;
        constexpr int KW = 4 / HALVES;                 // waves, of 8 keys each
        const int key = (lane >> 3) + 8 * (tw % KW), j0 = tw / KW * 32 + (lane & 7) * P, g8 = j0 / 8;
        koff = key * row_bytes + j0 * 2;
        coff = key * (kD / 2 * 8) + j0 * 8;
        kput = ksm[0] + g8 * (kKeyTile * 16) + (key ^ 4 * (g8 & 3)) * 16 + j0 % 8 * 2;
        const int oct = HALVES == 1 ? tw >> 1 : tw, first = HALVES == 1 ? tw & 1 : 0;      // 8 keys of the tile (k-step, half-wave); which 4 of them
        voff = vt_key(8 * oct + 4 * first) * row_bytes + lane * 4;
        vput = vsm[0] + (((lane >> 4) * 4 + oct) * kKeyTile + (lane & 15)) * 16 + first * 8;
    }
    auto cs_at = [&](uint32_t at, f32x4 (&x)[2]) {
        static_for<2>([&](auto i) { x[i.value] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(cbuf, at + i.value * 16, 0, 0)); });
    };
    auto ask_k = [&](Staged& x, int tile) {
        static_for<NK>([&](auto k) { cs_at(coff + (tile * kKeyTile + k.value * 16) * (kD / 2 * 8), x.angle[k.value]); });
        static_for<NK>([&](auto k) {
            const uint32_t at = koff + (tile * kKeyTile + k.value * 16) * row_bytes;
            x.lo[k.value] = __builtin_amdgcn_raw_buffer_load_b64(kbuf, at, 0, 0);
            x.up[k.value] = __builtin_amdgcn_raw_buffer_load_b64(kbuf, at + kD, 0, 0);
        });
    };
    auto ask_v = [&](Staged& x, int tile) {
        static_for<NV>([&](auto e) {
            x.v[e.value] = __builtin_amdgcn_raw_buffer_load_b32(vbuf, voff + (tile * kKeyTile + (e.value / 4 * 8 + e.value % 4)) * row_bytes, 0, 0);
        });
    };
    // (the empty assembly keeps what follows where it stands, behind the matrix instruction before it)
    u32x2 hk[2];                                       // what goes to LDS: lower and upper half of the channels of a key
    uint32_t hv[2][NV / 2];                            // both channels
    auto turn_k = [&](Staged& x, auto k, auto i) {     // two pairs of a key
        constexpr int K = decltype(k)::value, I = decltype(i)::value;
        uint32_t lo = x.lo[K][I], up = x.up[K][I];
        asm volatile("" : "+v"(lo), "+v"(up));
        const float a0 = bf16_lo(lo), a1 = bf16_hi(lo), b0 = bf16_lo(up), b1 = bf16_hi(up);
        const f32x4 c = x.angle[K][I];
        hk[0][I] = __builtin_bit_cast(uint32_t, pack_half2(a0 * c[0] - b0 * c[1], a1 * c[2] - b1 * c[3]));
        hk[1][I] = __builtin_bit_cast(uint32_t, pack_half2(b0 * c[0] + a0 * c[1], b1 * c[2] + a1 * c[3]));
    };
    auto turn_v = [&](Staged& x, auto i) {             // two keys
        asm volatile("" : "+v"(x.v[2 * i.value]), "+v"(x.v[2 * i.value + 1]));
        const uint32_t w0 = x.v[2 * i.value], w1 = x.v[2 * i.value + 1];
        hv[0][i.value] = __builtin_bit_cast(uint32_t, pack_half2(bf16_lo(w0), bf16_lo(w1)));
        hv[1][i.value] = __builtin_bit_cast(uint32_t, pack_half2(bf16_hi(w0), bf16_hi(w1)));
    };
    auto put_k = [&](int slot, auto k) {
        char* const to = kput + (slot & 3) * kTileBytes + k.value * 256;               // (16 keys on: bit 4 of the place is no part of the exchange)
        *(u32x2*)to = hk[0];
        *(u32x2*)(to + kD / 16 * kKeyTile * 16) = hk[1];
    };
    auto put_v = [&](int slot) {
        typedef uint32_t piece_t __attribute__((ext_vector_type(NV / 2)));
        static_for<2>([&](auto c) {
            piece_t w;
            static_for<NV / 2>([&](auto i) { w[i.value] = hv[c.value][i.value]; });
            *(piece_t*)(vput + (slot & 3) * kTileBytes + c.value * 256) = w;
        });
    };
    auto take = [&](Staged& x, int slot) {
        static_for<NK>([&](auto k) {
            static_for<2>([&](auto i) { turn_k(x, k, i); });
            put_k(slot, k);
        });
        static_for<NV / 2>([&](auto i) { turn_v(x, i); });
        put_v(slot);
    };
    // ---- queries of this wave: second operand of S^T = Kr Qr^T, lane = query column, 8 channels per k-step half.
    // Qr = rotate(q at its in-cache position) * log2(e)/sqrt(d), computed here once: the lane's groups of 8 channels in the lower half
    // (k-steps 0..3) and their rotary partners in the upper half (k-steps 4..7) are in its registers together.  A lane wants 16 bytes
    // here and there of a query's row: asked for like that, 64 lines to a load, the start of a workgroup took 7 us.  So rows come in
    // whole, all of them in flight at once, and turn through LDS.  Rows of the block beyond q_len are zero (another row is loaded for
    // them).  A wave without a task asks for no queries: the loads of seven such waves held up the eighth by 1 us.
    // What then bounded the start was cos and sin, 16 KB of them per wave, twice its queries, through the 64 bytes per cycle of a compute unit
    // (128 of 240 to 288 KB), and the turning of them.  The angle of query r of a block that begins at position p is that of p plus that of
    // r: one row of the table per wave (scaled) and its rows 0..31 once per workgroup, in slots of the rings that no copy uses yet, and
    // a complex product per pair in fp32, 1e-7 beside the 5e-4 of the operands' fp16.  The tiles are requested behind the queries, so that
    // they come while these are rotated.  In halves, the two waves of a task take half of the k-steps each and swap them in LDS.
    // Start of a workgroup in halves: 301 queries over 5001 rows 10400 -> 8250 cycles, 300 over 300 9940 -> 7460; in one stream, 4094 over
    // 8192, 12800 -> 12600 (all the queries of 256 workgroups come from memory at once).
    constexpr int NP = 16 / HALVES, NL = 8 / HALVES, NS = 4 / HALVES;   // pieces of 16 bytes of a row, loads, k-steps of the lower half, per wave
    char* const turn = qsm[tw] + half * (32 * NP * 16);                  // 32 rows, piece i of row r in place i ^ (r & 15), in halves i ^ (r / 2 & 7)
    char* const table = ring[0][0][(part0 + 3) & 3];                     // rows 0..15 in this slot of the keys, 16..31 in that of the values
    constexpr int TABLE_HALF = (int)sizeof(ring[0][0]);
    char* const origin = HALVES == 1 ? qsm[tw] + QUERIES : ring[HALVES - 1][0][(part0 + steps + 3) & 3] + wave * (kD / 2) * 8;
    {
        u32x4 rt[2], x[NL];
        float2 o = {0.f, 0.f};
        const int rrow = 4 * wave + (lane >> 5), rpiece = lane & 31;
        static_for<2>([&](auto i) {
            rt[i.value] = *(const u32x4*)(cs + (long long)min(rrow + 2 * i.value, g.cur_len - 1) * (kD / 2) + rpiece * 2);
        });
        const int r0 = lane / NP, pi = lane % NP;
        if (active) {
            o = cs[(long long)pos0 * (kD / 2) + lane];
            const int piece = HALVES == 1 ? pi : (pi & 3) + 4 * half + 8 * (pi >> 2);
            const uint16_t* const qrows = q + (head * g.q_len + q0) * kD + piece * 8;
            const int most = g.q_len - 1 - q0;                    // last row of the block that there is
            static_for<NL>([&](auto j) { x[j.value] = *(const u32x4*)(qrows + (long long)min(64 / NP * j.value + r0, most) * kD); });
        }
        static_for<2>([&](auto i) {
            const int row = rrow + 2 * i.value;
            *(u32x4*)(table + (row >> 4) * TABLE_HALF + (row & 15) * 512 + (rpiece ^ (row & 15)) * 16) = rt[i.value];
        });
        if (active) {
            *(float2*)(origin + lane * 8) = {o.x * g.qscale, o.y * g.qscale};
            static_for<NL>([&](auto j) {
                const int row = 64 / NP * j.value + r0;
                *(u32x4*)(turn + row * (NP * 16) + (pi ^ (HALVES == 1 ? row & 15 : row >> 1 & 7)) * 16) = x[j.value];
            });
        }
    }
    __syncthreads();
    Staged early[3];
    if constexpr (DIRECT) {
        static_for<3>([&](auto i) {
            ask_k(early[i.value], min(t0 + i.value, last_tile));
            ask_v(early[i.value], min(t0 + i.value, last_tile));
        });
    } else {
        static_for<3>([&](auto i) { dma_k(min(t0 + i.value, last_tile), t0 + i.value); });
        static_for<3>([&](auto i) { dma_v(min(t0 + i.value, last_tile), t0 + i.value); });
    }
    half8 qf[8];
    static_for<8>([&](auto s8) { qf[s8.value] = half8{}; });
    if (active) {
        auto get = [&](int i) { return *(const u32x4*)(turn + l32 * (NP * 16) + (i ^ (HALVES == 1 ? l32 & 15 : l32 >> 1 & 7)) * 16); };
        const char* const torigin = origin + (HALVES == 1 ? 0 : half * 256) + hw * 64;
        const char* const trow = table + (l32 >> 4) * TABLE_HALF + (l32 & 15) * 512 + (HALVES == 1 ? 0 : half * 256);
        const int tswap = (4 * hw ^ (l32 & 15)) * 16;
        u32x4 lo[NS], up[NS];
        static_for<NS>([&](auto s) { lo[s.value] = get(2 * s.value + hw); up[s.value] = get(NP / 2 + 2 * s.value + hw); });
        half8 mine[2 * NS];
        const bool there = l32 < g.q_len - q0;
        static_for<NS>([&](auto s) {
            constexpr int S = decltype(s)::value;
            half8 lo8 = {}, up8 = {};
            static_for<4>([&](auto ec) {
                constexpr int E = decltype(ec)::value;
                const f32x4 w = *(const f32x4*)(trow + S / 2 * 256 + ((8 * (S % 2) + E) * 16 ^ tswap)), v = *(const f32x4*)(torigin + S * 128 + E * 16);
                const float2 c0 = {v[0] * w[0] - v[1] * w[1], v[1] * w[0] + v[0] * w[1]}, c1 = {v[2] * w[2] - v[3] * w[3], v[3] * w[2] + v[2] * w[3]};
                const float a0 = bf16_lo(lo[S][E]), a1 = bf16_hi(lo[S][E]);
                const float b0 = bf16_lo(up[S][E]), b1 = bf16_hi(up[S][E]);
                // lower half: x_j cos - x_{j+d/2} sin;  upper half: x_{j+d/2} cos + x_j sin
                lo8[2 * E]     = (_Float16)(a0 * c0.x - b0 * c0.y);
                lo8[2 * E + 1] = (_Float16)(a1 * c1.x - b1 * c1.y);
                up8[2 * E]     = (_Float16)(b0 * c0.x + a0 * c0.y);
                up8[2 * E + 1] = (_Float16)(b1 * c1.x + a1 * c1.y);
            });
            mine[S] = there ? lo8 : half8{};
            mine[NS + S] = there ? up8 : half8{};
        });
        if constexpr (HALVES == 1) {
            static_for<8>([&](auto s8) { qf[s8.value] = mine[s8.value]; });
        } else {
            static_for<4>([&](auto i) { *(half8*)(turn + (i.value * 64 + lane) * 16) = mine[i.value]; });   // (the wave's own rows: it has read them)
        }
    }
    if constexpr (DIRECT) {
        static_for<3>([&](auto i) { take(early[i.value], t0 + i.value); });
        ask_k(sg, min(t0 + 3, last_tile));
        ask_v(sg, min(t0 + 3, last_tile));
    } else {
        // the keys of three tiles and the values of the first have landed, which is what the first step reads; it ends with all of them there
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * (PIECE / 1024)) : "memory");
    }
    __syncthreads();
    if constexpr (HALVES == 2) {
        if (active) {
            static_for<8>([&](auto s8) {
                constexpr int S = decltype(s8)::value % 4;
                qf[s8.value] = *(const half8*)(qsm[tw] + S / 2 * 4096 + ((s8.value / 4 * 2 + S % 2) * 64 + lane) * 16);
            });
        }
    }

    half8 kf[8], vf[8];         // fragments of Kr(t+1) and Vt(t), read from LDS a few matrix instructions ahead
    auto read_k = [&](auto s8, const char* kt) { kf[s8.value] = *(const half8*)(kt + frag[s8.value % 2] + s8.value * (2 * kKeyTile * 16)); };

    // cur holds S(t) - m: the accumulators of the scores start at minus the query's reference point, so the
    // exponent needs no subtraction; nxt receives S(t+1) - m during step t; the two swap roles every step.
    f32x16 cur, nxt;
    static_for<16>([&](auto r) { cur[r.value] = 0.f; });
    if (my_tiles > t0) {
        const char* kt = ksm[t0 & 3];
        static_for<8>([&](auto s8) {
            read_k(s8, kt);
            cur = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[s8.value], qf[s8.value], cur, 0, 0, 0);
        });
        static_for<2>([&](auto s8) { read_k(s8, ksm[(t0 + 1) & 3]); });
    }

    // Causal mask of a tile that reaches past the first query of the wave.
    auto mask_tile = [&](int tile, f32x16& s) {
        const int key_base = tile * kKeyTile;
        const int qpos = pos0 + l32;
        static_for<16>([&](auto r) {
            constexpr int R = decltype(r)::value;
            const int key = key_base + 8 * (R / 4) + 4 * hw + (R % 4);
            if (key > qpos) s[R] = -INFINITY;
        });
    };
    // Moves the reference point m of every query whose largest score in s exceeds it by more than the slack
    // (all of them on the first tile) up to that score: the accumulated sums and the pending scores follow.
    // Returns the lane's shift.  Any reference point gives the same quotient, so the point only has to keep
    // the weights inside the fp16 range.  Rare after the first tiles.
    auto move_refs = [&](f32x16& s, bool all) -> float {
        float v = s[0];
        static_for<16>([&](auto r) { v = fmaxf(v, s[r.value]); });
        const float mx = fmaxf(v, __shfl_xor(v, 32));
        // (a query may see nothing of the first tile of its part: its point stays where it is)
        const bool grow = all ? mx > -INFINITY : mx > kSlack;
        const float delta = grow ? mx : 0.f;
        const float f = exp2_fast(-delta);
        m += delta;
        lsum *= f;
        static_for<4>([&](auto db) { static_for<16>([&](auto r) { acc[db.value][r.value] *= f; }); });
        static_for<16>([&](auto r) { s[r.value] -= delta; });
        static_for<16>([&](auto r) { negm[r.value] = -m; });
        return delta;
    };

    // One step: tile t, whose scores minus m are in s, is consumed while the scores of tile t+1 go to n.
    bool first = true;          // the first tile sets the reference points whatever the scores are
    auto step = [&](int t, f32x16& s, f32x16& n) {
        const bool mine = DIRECT || t < my_tiles;
        if (mine) {
            if (t >= full_tiles) mask_tile(t, s);
            if (first) move_refs(s, true);
            first = false;
        }
        if constexpr (!DIRECT) {
            dma_k(min(t + 3, last_tile), t + 3);
            dma_v(min(t + 3, last_tile), t + 3);
        }
        if (mine) {
            const char* kt = ksm[(t + 1) & 3];            // past the wave's last tile a stale slot: result unused
            const char* vt = vsm[t & 3] + vfrag;
            auto read_v = [&](auto i) { vf[i.value] = *(const half8*)(vt + i.value * (2 * kKeyTile * 16)); };
            // ---- scores of the next tile on the matrix cores, dealt out between the exponentials of this tile
            // on the vector units: per 16-channel step one matrix instruction and two weights, packed to fp16
            // as they are produced; kf[0], kf[1] were read before the barrier
            float ps = 0.f;
            u32x4 pw[2];        // P^T, the second operand of the weighted sum, per k-step
            static_for<8>([&](auto s8) {
                constexpr int S8 = decltype(s8)::value;
                if constexpr (S8 < 6) {
                    read_k(IC<S8 + 2>{}, kt);
                } else {                                   // first k-step of the weighted sum: vf[2*db]
                    read_v(IC<(S8 - 6) * 4>{});
                    read_v(IC<(S8 - 6) * 4 + 2>{});
                }
                n = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[S8], qf[S8], S8 == 0 ? negm : n, 0, 0, 0);
                constexpr int R = 2 * S8;
                const half2v ph = pack_half2(exp2_fast(s[R]), exp2_fast(s[R + 1]));
                ps = __builtin_amdgcn_fdot2(ph, half2v{(_Float16)1, (_Float16)1}, ps, false);   // sums the rounded weights
                pw[R / 8][(R % 8) / 2] = __builtin_bit_cast(uint32_t, ph);
                __builtin_amdgcn_sched_barrier(0);
            });
            // No weight may exceed 2^kSlack (fp16 operands).  That is checked after the fact, on the sum of the
            // lane's 16 weights, which is there anyway (an overflowed weight makes it infinite): if it is too
            // large for some lane, the reference points move, the scores of the next tile, which started from
            // the old ones, follow, and the weights of this tile are computed again.
            if (__builtin_amdgcn_ballot_w64(!(ps <= kWeightLimit)) != 0) {
                const float delta = move_refs(s, false);
                static_for<16>([&](auto r) { n[r.value] -= delta; });
                ps = 0.f;
                static_for<8>([&](auto s8) {
                    constexpr int R = 2 * decltype(s8)::value;
                    const half2v ph = pack_half2(exp2_fast(s[R]), exp2_fast(s[R + 1]));
                    ps = __builtin_amdgcn_fdot2(ph, half2v{(_Float16)1, (_Float16)1}, ps, false);
                    pw[R / 8][(R % 8) / 2] = __builtin_bit_cast(uint32_t, ph);
                });
            }
            lsum += ps;
            // ---- O^T += Vt P^T : 128 channels x 32 queries, contraction over the 32 keys; k-step outermost so
            // that dependent accumulations are four instructions apart
            static_for<2>([&](auto k2) {
                const half8 pf = __builtin_bit_cast(half8, pw[k2.value]);
                static_for<4>([&](auto db) {
                    if constexpr (decltype(k2)::value == 0) read_v(IC<decltype(db)::value * 2 + 1>{});   // second k-step
                    else if constexpr (decltype(db)::value < 2) read_k(db, ksm[(t + 2) & 3]);   // first fragments of the step after
                    acc[db.value] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[db.value * 2 + k2.value], pf, acc[db.value], 0, 0, 0);
                    // tile t+3 goes to LDS between the matrix instructions, and tile t+4 is asked for
                    if constexpr (DIRECT) {
                        constexpr int S = decltype(k2)::value * 4 + decltype(db)::value;
                        if constexpr (HALVES == 1 ? S % 2 == 0 && S < 4 : S < 4) turn_k(sg, IC<S / 2 % HALVES>{}, IC<HALVES == 1 ? S / 2 : S % 2>{});
                        if constexpr (HALVES == 2 && S == 1) put_k(t + 3, IC<0>{});
                        if constexpr (S == 3) {
                            put_k(t + 3, IC<HALVES - 1>{});
                            ask_k(sg, min(t + 4, last_tile));
                        }
                        if constexpr (S >= 4 && S % (2 / HALVES) == 0) turn_v(sg, IC<(S - 4) / (2 / HALVES)>{});
                        if constexpr (S == 7) {
                            put_v(t + 3);
                            ask_v(sg, min(t + 4, last_tile));
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
        }
        if constexpr (!DIRECT) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };
    if constexpr (DIRECT) {
        // the steps that the wave has keys of, then those of the others' alone: in one loop, with a way for either, the compiler moves
        // the registers of the loads in flight about and waits for them
        int t = t0;
        for (; t < my_tiles; t += 2) {
            step(t, cur, nxt);
            if (t + 1 >= my_tiles) { ++t; break; }
            step(t + 1, nxt, cur);
        }
#pragma unroll 1
        for (; t < t0 + steps; ++t) {
            take(sg, t + 3);
            ask_k(sg, min(t + 4, last_tile));
            ask_v(sg, min(t + 4, last_tile));
            __syncthreads();
        }
    } else {
        for (int t = t0; t < t0 + steps; t += 2) {
            step(t, cur, nxt);
            if (t + 1 < t0 + steps) step(t + 1, nxt, cur);
        }
    }

    // ---- normalise and store: lane = query, registers = channels 8*(r/4) + 4*hw + r%4 of each block
    lsum += __shfl_xor(lsum, 32);
    constexpr int NB = 4 / HALVES;                     // channel blocks that a wave finishes
    f32x16 fin[NB];
    if constexpr (HALVES == 1) {
        static_for<4>([&](auto db) { fin[db.value] = acc[db.value]; });
    } else {
        // The two waves of a task finish two channel blocks each, and hand each other the rest.
        // (behind the last step's barrier nobody reads or copies into the rings any more)
        char* const area = &ring[0][0][0][0] + tw * 18 * 1024;
        float2* const ml = (float2*)(area + 16 * 1024) + lane;
        auto give = [&](auto first) {                  // the partner's two blocks
            static_for<2>([&](auto db) {
                static_for<4>([&](auto r4) {
                    constexpr int R = 4 * decltype(r4)::value, B = decltype(first)::value + decltype(db)::value;
                    ((f32x4*)(area + half * 8192))[(db.value * 4 + r4.value) * 64 + lane] = f32x4{acc[B][R], acc[B][R + 1], acc[B][R + 2], acc[B][R + 3]};
                });
            });
        };
        if (half == 0) {
            give(IC<2>{});
            fin[0] = acc[0], fin[1] = acc[1];
        } else {
            give(IC<0>{});
            fin[0] = acc[2], fin[1] = acc[3];
        }
        ml[half * 64] = {m, lsum};
        __syncthreads();
        const float2 o = ml[(1 - half) * 64];
        const float m0 = lsum > 0.f ? m : -1e30f, m1 = o.y > 0.f ? o.x : -1e30f, M = fmaxf(m0, m1);
        const float f0 = exp2_fast(m0 - M), f1 = exp2_fast(m1 - M);
        m = M;
        lsum = lsum * f0 + o.y * f1;
        static_for<2>([&](auto db) {
            static_for<4>([&](auto r4) {
                const f32x4 x = ((const f32x4*)(area + (1 - half) * 8192))[(db.value * 4 + r4.value) * 64 + lane];
                static_for<4>([&](auto i) {
                    constexpr int R = 4 * decltype(r4)::value + decltype(i)::value;
                    fin[db.value][R] = fin[db.value][R] * f0 + x[i.value] * f1;
                });
            });
        });
    }
    if (g.n_split > 1) {
        // the state as it is, in the order of the registers (1 KB per store): [task][part][channel block][register / 4][lane][4]
        if (seen) {
            const long long st = ((long long)unit * tasks_per_unit + task) * g.n_split + split;
            f32x4* o = (f32x4*)part_acc + st * (16 * 64) + half * (NB * 4 * 64) + lane;
            static_for<NB>([&](auto db) {
                static_for<4>([&](auto r4) {
                    constexpr int R = 4 * decltype(r4)::value;
                    o[(db.value * 4 + r4.value) * 64] = f32x4{fin[db.value][R], fin[db.value][R + 1], fin[db.value][R + 2], fin[db.value][R + 3]};
                });
            });
            if (half == 0 && hw == 0) part_ml[st * 32 + l32] = {lsum > 0.f ? m : -1e30f, lsum};
        }
        return;
    }
    if (active) {
        // The results turn in LDS, where the queries did, and leave as whole rows (in halves, as half rows): 8 bytes here and there of 32
        // rows to a store, as the registers have them, took longer: end of a workgroup in halves (300 over 300) 6460 -> 3410 cycles, in one stream 5130 -> 2950.
        const float inv = 1.0f / lsum;
        static_for<NB>([&](auto db) {
            static_for<4>([&](auto r4) {
                constexpr int R = 4 * decltype(r4)::value, I = decltype(db)::value * 4 + decltype(r4)::value;
                f32x2 a = {fin[db.value][R] * inv, fin[db.value][R + 1] * inv};
                f32x2 b = {fin[db.value][R + 2] * inv, fin[db.value][R + 3] * inv};
                u32x2 w;
                w[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(a, bf16x2));
                w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(b, bf16x2));
                *(u32x2*)(turn + l32 * (NP * 16) + (I ^ (HALVES == 1 ? l32 & 15 : l32 >> 1 & 7)) * 16 + hw * 8) = w;
            });
        });
        const int r0 = lane / NP, pi = lane % NP;
        uint16_t* const orow = out + (head * g.q_len + q0) * kD + half * (NB * 32) + pi * 8;
        static_for<NL>([&](auto j) {
            const int row = 64 / NP * j.value + r0;
            const u32x4 w = *(const u32x4*)(turn + row * (NP * 16) + (pi ^ (HALVES == 1 ? row & 15 : row >> 1 & 7)) * 16);
            if (q0 + row < g.q_len) *(u32x4*)(orow + (long long)row * kD) = w;
        });
        if (lse && half == 0 && hw == 0 && q0 + l32 < g.q_len) lse[head * g.q_len + q0 + l32] = 0.6931471805599453f * (m + log2f(lsum));
    }
}

// Merges the parts of the key range (n_split > 1): one workgroup per task, a wave per block of 32 channels, the same lane layout.
__global__ __launch_bounds__(256) void k_prefill_merge(const PrefillGeom, const float* __restrict__ part_acc,
                                                       const float2* __restrict__ part_ml, uint16_t* __restrict__ out,
                                                       float* __restrict__ lse)
{
    const PrefillGeom g = first_argument<decltype(k_prefill_merge)>();
    const int tasks_per_unit = g.G * g.q_blocks;
    const int unit = blockIdx.x / tasks_per_unit, task = blockIdx.x - unit * tasks_per_unit;
    const int db = threadIdx.x >> 6, lane = threadIdx.x & 63, l32 = lane & 31, hw = lane >> 5;
    const int qb = task / g.G, gh = task - qb * g.G, q0 = qb * kQPerWave;
    const int last = min(g.cur_len - g.q_len + q0 + kQPerWave - 1, g.cur_len - 1);
    const int parts = ((last + kKeyTile) / kKeyTile + g.split_tiles - 1) / g.split_tiles;     // parts that some query of the task sees
    const long long st = (long long)blockIdx.x * g.n_split;
    float M = -1e30f, L = 0.f;
    f32x4 o[4] = {};
    // Four parts at a time, all their loads in flight (past the last part its own again, and then not used): one after the other, three parts
    // waited six times for memory.
    for (int s = 0; s < parts; s += 4) {
        float2 ml[4];
        f32x4 x[4][4];
        static_for<4>([&](auto i) { ml[i.value] = part_ml[(st + min(s + i.value, parts - 1)) * 32 + l32]; });
        static_for<4>([&](auto i) {
            const f32x4* a = (const f32x4*)part_acc + (st + min(s + i.value, parts - 1)) * (16 * 64) + db * (4 * 64) + lane;
            static_for<4>([&](auto r4) { x[i.value][r4.value] = a[r4.value * 64]; });
        });
        __builtin_amdgcn_sched_barrier(0);                            // (left alone the compiler has four to six of them in flight)
        float Mn = M;
        static_for<4>([&](auto i) { Mn = fmaxf(Mn, ml[i.value].x); });
        const float old = exp2_fast(M - Mn);
        M = Mn;
        L *= old;
        static_for<4>([&](auto r4) { o[r4.value] *= old; });
        static_for<4>([&](auto i) {
            // (not by a weight of 0, which would make an infinite sum NaN)
            const bool there = s + i.value < parts;
            const float f = exp2_fast(ml[i.value].x - M);
            L = there ? fmaf(ml[i.value].y, f, L) : L;
            static_for<4>([&](auto r4) {
                static_for<4>([&](auto e) {
                    const float sum = fmaf(x[i.value][r4.value][e.value], f, o[r4.value][e.value]);
                    o[r4.value][e.value] = there ? sum : o[r4.value][e.value];
                });
            });
        });
    }
    const int qi = q0 + l32;
    if (qi >= g.q_len) return;
    const long long head = (long long)unit * g.G + gh;
    const float inv = 1.0f / L;
    uint16_t* orow = out + (head * g.q_len + qi) * kD + db * 32 + 4 * hw;
    static_for<4>([&](auto r4) {
        f32x2 a = {o[r4.value][0] * inv, o[r4.value][1] * inv}, b = {o[r4.value][2] * inv, o[r4.value][3] * inv};
        u32x2 w;
        w[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(a, bf16x2));
        w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(b, bf16x2));
        *(u32x2*)(orow + 8 * r4.value) = w;
    });
    if (lse && db == 0 && hw == 0) lse[head * g.q_len + qi] = 0.6931471805599453f * (M + log2f(L));
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------

hipError_t launch_prefill_cs(float2* cs, int rows, int d, double rope_base, int rope, hipStream_t st)
{
    const long long total = (long long)rows * (d / 2);
    hipLaunchKernelGGL(k_prefill_cs, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, cs, rows, d, rope_base, rope);
    return hipGetLastError();
}

hipError_t launch_prefill_prepare(const SlabTable& tab, const PrefillGeom& g, const float2* cs, _Float16* Kr, _Float16* Vt, hipStream_t st)
{
    if (g.d != kD || g.cur_len < 1 || g.q_len < 1 || g.q_len > g.cur_len) return hipErrorInvalidValue;
    if (g.key_tiles * kKeyTile < g.cur_len || g.q_pad < g.q_len || g.q_pad % kQPerWave) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_prefill_prep, dim3((unsigned)((long long)g.units * prep_tiles(g.key_tiles))), dim3(256), 0, st, g, cs, Kr, Vt, tab);
    return hipGetLastError();
}

hipError_t launch_attend_prefill(const PrefillGeom& g, const SlabTable* tab, const _Float16* Kr, const _Float16* Vt, const void* q, const float2* cs,
                                 void* out, float* lse, float* part_acc, float2* part_ml, hipStream_t st)
{
    if (g.d != kD || g.q_blocks * kQPerWave != g.q_pad) return hipErrorInvalidValue;
    if (g.halves != 1 && g.halves != 2) return hipErrorInvalidValue;
    if (tab ? !prefill_direct_fits(g.cur_len, g.stride_token) : !Kr || !Vt) return hipErrorInvalidValue;
    if (g.n_split < 1 || (g.n_split > 1 && (!part_acc || !part_ml || (long long)g.n_split * g.split_tiles < g.key_tiles))) return hipErrorInvalidValue;
    const int tasks = kPrefillWaves / g.halves, wgs_per_unit = (g.G * g.q_blocks + tasks - 1) / tasks;
    PrefillGeom gw = g;
    gw.wgs = 0;
    for (int s = 0; s < g.n_split; ++s) gw.wgs += wgs_per_unit - prefill_first_wg(g.cur_len, g.q_len, g.G, wgs_per_unit, tasks, s * g.split_tiles);
    const dim3 grid((unsigned)((long long)g.units * gw.wgs)), block(kPrefillWaves * 64);
    auto launch = [&](auto kernel, const auto& rows) {
        hipLaunchKernelGGL(kernel, grid, block, 0, st, gw, Kr, Vt, (const uint16_t*)q, cs, (uint16_t*)out, lse, part_acc, part_ml, rows);
    };
    if (tab) {
        const Rows<true> rows = {*tab};
        if (g.halves == 2) launch(k_attend_prefill<2, true>, rows);
        else               launch(k_attend_prefill<1, true>, rows);
    } else {
        const Rows<false> rows = {};
        if (g.halves == 2) launch(k_attend_prefill<2, false>, rows);
        else               launch(k_attend_prefill<1, false>, rows);
    }
    if (g.n_split > 1)
        hipLaunchKernelGGL(k_prefill_merge, dim3((unsigned)((long long)g.units * g.G * g.q_blocks)), dim3(256), 0, st, g, part_acc, part_ml,
                           (uint16_t*)out, lse);
    return hipGetLastError();
}

}  // namespace freqkv
