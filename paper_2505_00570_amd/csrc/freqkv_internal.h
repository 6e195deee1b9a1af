// Internal interface between the host side of libfreqkv (argument checks, plans,
// basis cache, launch sequence) and its gfx950 kernels.  Not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace freqkv {

// One wave copies 64 x 16 bytes global -> LDS without passing registers: lane i reads 16 bytes at its own
// address src and the data lands at LDS byte address lds + 16 i (lds is the same for the whole wave).  The copy
// counts as a vector-memory load (vmcnt); the compiler does not know that it writes LDS, so the kernel waits
// for it by hand (s_waitcnt vmcnt) before the barrier that publishes the data.  M0 carries the LDS address:
// kernels that use this have no other user of M0 (the compiler rejects M0 in a clobber list, so the build
// script checks the generated assembly for that instead).
__device__ __forceinline__ void lds_dma16(uint32_t lds, const void* src)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds), "v"(src) : "memory");
}
// ... from a scalar address and an offset of the lane's own
__device__ __forceinline__ void lds_dma16(uint32_t lds, const void* base, uint32_t offset)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(lds), "v"(offset), "s"(base) : "memory");
}

constexpr int kBufferFlags = 0x00020000;        // fourth word of a buffer's descriptor: raw, 32-bit elements

// What a kernel's arguments take, from its type.
template <class Kernel> struct Arguments;
template <class A, class... More> struct Arguments<void(A, More...)> {
    static_assert(sizeof(A) % 8 == 0 && ((sizeof(More) % 8 == 0) && ...), "sizes add up without gaps");
    typedef A First;
    static constexpr int bytes = (int)(sizeof(A) + (sizeof(More) + ... + 0));
};

// The kernel's first argument, behind a fetch of the cache lines that hold its arguments (the first 256 bytes of them), all lines at once.  Read
// where they are used, one line after the other comes from memory at the start of a kernel, 600 to 900 cycles each: so kernels of a few
// microseconds have their small arguments first, the table of slabs behind them, and take the first from here.  A line is touched at its
// start, which has to lie within the arguments: hence their size from the kernel's type.
template <class Kernel> __device__ __forceinline__ typename Arguments<Kernel>::First first_argument()
{
    typedef typename Arguments<Kernel>::First A;
    constexpr int bytes = Arguments<Kernel>::bytes, lines = ((bytes < 256 ? bytes : 256) + 63) / 64;
    A a = {};
#ifdef __HIP_DEVICE_COMPILE__
    auto* args = (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile(".set fetch_line, 0\n\t"
                 ".rept %1\n\t"
                 "s_load_dword s90, %0, fetch_line\n\t"
                 ".set fetch_line, fetch_line + 64\n\t"
                 ".endr\n\t"
                 "s_waitcnt lgkmcnt(0)" : "+s"(args) : "n"(lines) : "s90");
    __builtin_memcpy(&a, (const __attribute__((address_space(4))) A*)args, sizeof(A));
#endif
    return a;
}

// One launch group addresses at most this many (layer, K|V) slabs; their base
// pointers travel by value in the kernel arguments.
constexpr int kMaxSlabs = 192;

struct SlabTable {
    char* base[kMaxSlabs];
};
// ... of a launch of few slabs, see with_slabs
constexpr int kFewSlabs = 8;
struct FewSlabs {
    char* base[kFewSlabs];
};
struct TailTable {
    int rows[kMaxSlabs];
};

// Tile constants of the fp16-MFMA contraction.
constexpr int kColTile   = 128;   // virtual columns per workgroup tile
constexpr int kKStage    = 32;    // contraction rows staged per pipeline step
constexpr int kRowsFold  = 256;   // rows per parity per workgroup tile (folded variant)
constexpr int kRowsPlain = 512;   // rows per workgroup tile (plain variant)

// Geometry of one pass (by-value kernel argument).
struct Geom {
    int n;               // span length
    int Lc;              // retained length
    int S;               // sink rows
    int d;               // head_dim
    int hts_per_slab;    // batch * n_heads
    int n_heads;
    int ncols;           // virtual columns in this pass = slabs * hts_per_slab * d
    int ncoltiles;       // ceil(ncols / kColTile)
    int fold;            // 1: even/odd folded operator, 0: plain
    int high;            // 0: the Lc lowest coefficients are kept, 1: the highest (ablation variant),
                         // 2: forward transform only, all n coefficients (power spectrum)
    float spec_scale;    // power spectrum: 1 / (batch * head_dim)
    // two-level fold (l2 != 0): this Geom describes one of its two launches
    int l2;              // 0: not used, 1: even part (folded again, n = n0/2, Lc = Lc0/2), 2: odd part (plain)
    int n0, Lc0;         // span and retained length of the full problem
    int H;               // n0/4 rounded up to a pipeline stage: half the contraction length of the odd part
    const _Float16* ebuf; // odd part: fp16 even part E[head-tensor][Lc0/2][d] written by the first launch
    const uint32_t* hmax; // per head-tensor of this pass: largest bf16 magnitude (bit pattern) of its span, or null:
                          // the span is scaled by a power of two on its way into the fp16 workspace (range guard)
    int Kh;              // contraction length: n/2 (fold) or n
    int Kpad;            // Kh rounded up to kKStage
    int nkstages;        // Kpad / kKStage
    int Mh;              // output rows per parity: Lc/2 (fold) or Lc
    int Mpad;            // Mh rounded up to the workgroup tile
    int Grows;           // rows of the stored basis: 2*Mpad (fold) or Mpad
    int nmtiles;         // Mpad / tile rows
    long long stride_batch, stride_head, stride_token;   // elements
    long long tap_slab0; // index of this pass's first slab in the caller's [2][n_layers] order
};

// Byte address of (token 0, channel c) of the head-tensor that owns virtual column vcol.
template <class Slabs>
__device__ __forceinline__ char* column_base(const Slabs& tab, const Geom& g, int vcol,
                                             int elem_bytes, int* ht_out)
{
    int ht   = vcol / g.d;
    int c    = vcol - ht * g.d;
    int slab = ht / g.hts_per_slab;
    int r    = ht - slab * g.hts_per_slab;
    int b    = r / g.n_heads;
    int h    = r - b * g.n_heads;
    if (ht_out) *ht_out = ht;
    long long off = (long long)b * g.stride_batch + (long long)h * g.stride_head + c;
    return tab.base[slab] + off * elem_bytes;
}

enum Variant { kNone = 0, kFoldF16 = 1, kPlainF16 = 2, kF32 = 3, kDrop = 4, kFold2F16 = 5, kFast = 6,
               kNearFar = 7 };   // 7: in the key of its tables and in freqkv_plan_t::runs; Shape::variant is the form without it

// ---- basis construction (fp64 closed form, rounded once) -------------------------
// G: [Kpad/8][Grows][8] fp16.  Folded: rows [0,Mpad) even part, rows [Mpad,2Mpad) odd part.
hipError_t launch_basis_f16(_Float16* G, const Geom& g, int rescale, hipStream_t st);
// Gt: [parity] of Kh x Mpad fp32 (plain: one parity), four consecutive k side by side (f32_at).
hipError_t launch_basis_f32(float* Gt, const Geom& g, int rescale, hipStream_t st);

// Power of two that brings a head-tensor whose largest bf16 magnitude has the bit pattern `amax` into
// [2^11, 2^12): sums of four such values stay far below the fp16 limit, and nothing but values 2^-25 of the
// largest falls into fp16's subnormal range.  Returns the exponent e (scale 2^e); 0 for all-zero, inf or nan.
__device__ __forceinline__ int guard_exponent(uint32_t amax)
{
    const int E = (int)(amax >> 7) & 0xff;
    if (E == 0 || E == 255) return 0;
    int e = 138 - E;
    return e > 120 ? 120 : e;
}
__device__ __forceinline__ float pow2f(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }

// ---- bf16 cache: largest magnitude per head-tensor (zero hmax first), fold/convert the span, contract
hipError_t launch_absmax_bf16(const SlabTable& tab, const Geom& g, uint32_t* hmax, hipStream_t st);

// elem_bytes 4: the cache holds float32 (power spectrum of fp32 caches only)
hipError_t launch_prepare_bf16(const SlabTable& tab, const Geom& g, _Float16* ws, hipStream_t st, int elem_bytes = 2);
// mode 0: rows into the cache; 1: power-spectrum epilogue, tap = spectrum lines [slab][head][n] (atomics);
// 2: even part of the two-level fold, fp16 rows into the buffer passed as tap, nothing else; 3: odd part, combined with g.ebuf into the cache
hipError_t launch_contract_f16(const SlabTable& tab, const Geom& g, const _Float16* G,
                               const _Float16* ws, float* tap, int mode, hipStream_t st);
// two-level fold: gA = geometry of the even-part launch; wsA folded layout (xee | xeo), wsB plain layout (xo)
hipError_t launch_prepare_bf16_l2(const SlabTable& tab, const Geom& gA, _Float16* wsA, _Float16* wsB, hipStream_t st);
hipError_t launch_fill_zero(float* p, size_t count, hipStream_t st);

// ---- fp32 cache ------------------------------------------------------------------------
hipError_t launch_prepare_f32(const SlabTable& tab, const Geom& g, float* ws, hipStream_t st);
hipError_t launch_contract_f32(const SlabTable& tab, const Geom& g, const float* Gt,
                               const float* ws, float* tap, hipStream_t st);

// ---- factored transform (spans n = 4pq, Lc = n/2, bf16 caches): one kernel, no workspace ------------------
// Is there a compiled kernel for this span and head_dim?  (p, q) are the coprime odd factors of n/4, `channels`
// the channels of a head-tensor one workgroup owns (head_dim is a multiple of it).
bool fast_supported(int n, int Lc, int head_dim, int* p, int* q, int* channels);
size_t fast_table_bytes(int n, int head_dim);         // stage matrices in fragment order + the middle step's maps
size_t fast_lds_halfs(int n, int head_dim);           // fp16 values of one workgroup's LDS image (diagnostics)
void fast_build_tables_host(int n, int head_dim, char* out);   // fp64, rounded once; `out` is host memory
// rest_scale: what is left of the operator's 1/n after the scaled stages (1/2; sqrt(n/Lc)/2 without the
// rescale of Eq. 3).  dump/stop: diagnostic, see the kernel; pass nullptr, 0.
hipError_t launch_fast(const SlabTable& tab, const Geom& g, const void* tables, float rest_scale, float* tap,
                       _Float16* dump, int stop, hipStream_t st);

// ---- near/far form (bf16 caches, n/5 <= Lc < n): one kernel, no workspace ------------------------------------
constexpr int kNfMinSpan = 128;
// Geometry (by-value kernel argument); everything but the last block follows from n and Lc.
struct NfGeom {
    int n, Lc;
    int NK, NLO;             // leaves (128 rows) per exact window; its 16-row steps that get a second bf16 part
    int GT;                  // tiles (32 result rows) per step and group
    int NL, NC, NT, NG, NB;  // leaves, blocks of 4 leaves, tiles, groups, blocks of a group's neighbourhood
    int NLm, NCp, NGp, NX;   // leaves, blocks, groups that LDS has room for; vectors where blocks and later tiles go
    int R, NLr;              // ring slots; (NL - 1) mod R
    int shifts, PT, tlo, thi; // exact entries repeat every PT tiles for tiles tlo .. thi-1
    int TU, NU;              // the form by units (freqkv_nearfar_units.hip): tiles per unit, units; TU 0: not that form
    int held, held0, held_every;  // ... units of four leaves that its movers hold in registers: how many, the first one's first leaf, their distance in leaves
    int spills;              // the leaves' moments do not fit LDS: they go through spill, spill_bytes per workgroup
    int spill_bytes;         // (a multiple of 16)
    int spill_cloc;          // ... of these: where the second parts of the groups' local values begin
    char* spill;
    int v_slots;             // moment tables: 2 (all leaves but the last | the last), 3 (cosines | sines | the last) or one per leaf
    int off_v, off_m, off_c, off_f, off_t, off_w, table_bytes;
    int d;
    int S, n_heads, hts_per_slab, hts;
    float out_scale;         // sqrt(n/Lc) without the rescale of Eq. 3, else 1 (in the tables)
    long long stride_batch, stride_head, stride_token, tap_slab0;
};
bool nf_geometry(int n, int Lc, int head_dim, NfGeom* out);
bool nf_unit_geometry(int n, int Lc, int head_dim, NfGeom* out);
hipError_t launch_nf_unit_tables(const NfGeom& g, char* out, hipStream_t st);
hipError_t launch_nearfar_units(const SlabTable& tab, const NfGeom& g, const char* tables, float* tap, unsigned grid, hipStream_t st);
hipError_t launch_nf_tables(const NfGeom& g, char* out, hipStream_t st);
// most_wgs: workgroups that g.spill has room for (if g.spills)
hipError_t launch_nearfar(const SlabTable& tab, const NfGeom& g, const char* tables, float* tap, unsigned most_wgs, hipStream_t st);

// ---- tail move: rows [src, src+rows) -> [dst, dst+rows) of every head-tensor; ranges must not overlap
hipError_t launch_move_rows(const SlabTable& tab, const Geom& g, int elem_bytes, int src_row,
                            int dst_row, int rows, hipStream_t st);
// the first tails.rows[slab] rows from src on -> dst on, for every slab its own count (at most `most`); the ranges of one
// slab may overlap, but not rows that are less than `gap` apart
hipError_t launch_move_tails(const SlabTable& tab, const TailTable& tails, const Geom& g, int elem_bytes, int src_row,
                             int dst_row, int most, int gap, hipStream_t st);

// ---- calibration: plain 16-byte copy; register-only MFMA loop (16 x 32x32x16 f16 per iteration per wave)
hipError_t launch_calib_copy(void* dst, const void* src, size_t bytes, hipStream_t st);
hipError_t launch_calib_mfma(float* out, int blocks, int iters, hipStream_t st);

// ---- decode attention over the compacted cache ---------------------------------------------------
// Geometry of one attention pass (by-value kernel argument).  A "unit" is one (layer, batch, KV head).
// Division of 0 .. 2^31 - 1 by a fixed d, which a kernel would spend some 150 cycles on at its start.  With 2^s < d <= 2^(s+1), factor =
// ceil(2^(32+s) / d) has 32 bits and is less than 2^(s+1) / d too large, which a quotient's floor does not notice: n 2^(s+1) < 2^(32+s).
struct Divisor {
    uint32_t factor, shift;            // factor 0: d is 1
    __host__ __device__ int quotient(int n) const
    {
        return factor ? (int)((uint32_t)(((uint64_t)(uint32_t)n * factor) >> 32) >> shift) : n;
    }
};
inline Divisor divisor(int d)
{
    if (d <= 1) return Divisor{0, 0};
    uint32_t s = 0;
    while ((2u << s) < (uint32_t)d) ++s;
    return Divisor{(uint32_t)((((uint64_t)1 << (32 + s)) + d - 1) / d), s};
}

struct AttGeom {
    int d;                 // head_dim: 64, 128 or 256
    int G;                 // query heads per KV head
    int GT;                // query heads one workgroup handles together: 1, 2 or 4, divides G
    int n_kv;              // KV heads
    int units;             // layers in this pass * batch * n_kv
    int units_per_layer;   // batch * n_kv
    int cur_len;           // cached rows, >= 1 (with cur_lens: the longest sequence's, an upper bound)
    int q_pos;             // in-cache position of the query (with cur_lens: each sequence's last row)
    const int* cur_lens;   // optional device array [batch] of per-sequence cached rows, or null
    int P;                 // rotary pairs per lane, attend_pairs_per_lane(d)
    int n_split;           // row chunks per unit
    int chunk;             // rows per chunk, a multiple of 2 * attend_row_step(d)
    long long stride_batch, stride_head, stride_token;   // elements
    Divisor by_split, by_layer, by_kv, by_q;   // n_split, units_per_layer, n_kv, q_len
    int q_len;             // launch_attend_many: queries of a head, G being that of all heads; else 0
    float qscale;          // log2(e) / sqrt(d)
};

// One rotary pair: its frequency and the rotation that advances the position by attend_row_step(d) rows (the second d/2 entries of a table:
// by twice as many).
struct RopeEntry {
    double theta;
    float cd, sd;
};

// Rotary pairs (and twice as many channels) one lane of the attention kernel owns.
constexpr int attend_pairs_per_lane(int d) { return d > 256 ? 8 : 4; }
// Rows between two consecutive rows handled by one lane group: 4 waves x 64 lanes / (lanes per row).
constexpr int attend_row_step(int d) { return 4 * 64 / (d / (2 * attend_pairs_per_lane(d))); }
// Waves per SIMD the compiler must leave room for (bounds the registers of a lane).
constexpr int attend_min_waves(int elem_bytes, int GT, int P) { return elem_bytes == 2 ? (P == 4 ? (GT == 1 ? 4 : 3) : 2) : (P == 4 ? 2 : 1); }

hipError_t launch_rope_table(RopeEntry* rt, int d, double base, hipStream_t st);
// tab.base[2*i] / [2*i+1]: K / V slab of the pass's i-th layer.  part_acc: [units*G][n_split][d] fp32,
// part_ml: [units*G][n_split][2] fp32 (running maximum in the exp2 domain, sum of weights).
hipError_t launch_attend_partial(const SlabTable& tab, const AttGeom& g, int elem_bytes, const void* q,
                                 const RopeEntry* rt, float* part_acc, float* part_ml, void* out, float* lse, hipStream_t st);
// Several queries of each head, the last q_len rows, bf16 and d = 128: g.G = query heads per KV head * q_len, q and out dense [units][g.G][d].
hipError_t launch_attend_many(const SlabTable& tab, const AttGeom& g, const void* q, const RopeEntry* rt, float* part_acc, float* part_ml, void* out,
                              float* lse, hipStream_t st);
hipError_t launch_attend_merge(const AttGeom& g, int elem_bytes, const float* part_acc, const float* part_ml,
                               void* out, float* lse, hipStream_t st);

// ---- chunk-wise (prefill) attention over the compacted cache ------------------------------------------
struct PrefillGeom {
    int d;                 // head_dim (128)
    int G;                 // query heads per KV head
    int n_kv;
    int units;             // layers in this pass * batch * n_kv
    int units_per_layer;   // batch * n_kv
    int cur_len;           // cached rows, the chunk's tokens included
    int q_len;             // tokens of the chunk = queries per head; they are the last q_len cached rows
    int q_pad;             // q_len rounded up to 32
    int q_blocks;          // q_pad / 32
    int key_tiles;         // ceil(cur_len / 32)
    int n_split;           // parts that the key tiles of a workgroup are cut into, of split_tiles tiles each
    int split_tiles;
    int halves;            // 2: the waves of a workgroup share out the keys of its part in two halves (4 tasks instead of 8)
    int wgs;               // workgroups of a unit, over all parts: those that see keys of them
    long long stride_batch, stride_head, stride_token;   // elements
    float qscale;          // log2(e) / sqrt(d)
};
// First of a unit's `wgs` workgroups of `tasks` tasks each (in the order of their query blocks) that sees the key tile `tile`; the
// later ones do too.
__host__ __device__ inline int prefill_first_wg(int cur_len, int q_len, int G, int wgs, int tasks, int tile)
{
    if (32 * tile >= cur_len) return wgs;
    const int beyond = 32 * tile - (cur_len - q_len);         // of the first query's row
    return beyond > 0 ? beyond / 32 * G / tasks : 0;
}

// cs: [rows][d/2] (cos, sin).
hipError_t launch_prefill_cs(float2* cs, int rows, int d, double rope_base, int rope, hipStream_t st);
// Kr, Vt: [units][key_tiles] tiles of 32 keys x d fp16 in fragment order.
hipError_t launch_prefill_prepare(const SlabTable& tab, const PrefillGeom& g, const float2* cs, _Float16* Kr, _Float16* Vt, hipStream_t st);
// Offsets of a head's rows and of their cos/sin, a tile beyond the last, are within 31 bits (the attention kernel reads the cached rows as a buffer).
inline bool prefill_direct_fits(int cur_len, long long stride_token)
{
    return stride_token < (1LL << 30) && ((long long)cur_len + 32) * (stride_token > 256 ? stride_token : 256) * 2 < (1LL << 31);
}
// With tab, keys and values come from the cached rows, without it from Kr and Vt.
// q: dense [units*G][q_len][d] bf16, rotated inside the attention kernel.  part_acc, part_ml (n_split > 1): per (task, part)
// 32 x d fp32 and 32 x (reference point, sum).
hipError_t launch_attend_prefill(const PrefillGeom& g, const SlabTable* tab, const _Float16* Kr, const _Float16* Vt, const void* q, const float2* cs,
                                 void* out, float* lse, float* part_acc, float2* part_ml, hipStream_t st);

}  // namespace freqkv
