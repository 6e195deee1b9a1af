// gfx950 kernels for decode attention over the compacted cache.
//
// One incoming token attends to every cached row [0, cur_len) of its KV head: sinks, compressed rows
// and the tokens appended since, itself included (Sec. 3.3 Eq. 4, Sec. 3.4 Eq. 5).  Keys are cached
// without the rotary embedding; the key of cache row p is rotated by position p, an index inside the
// cache, when it is read, and the query by its own in-cache position (closing paragraph of Sec. 3.4,
// appendix on key states with RoPE).  Rotary pairing is LLaMA's: channel i turns with channel i + d/2
// by the angle pos * base^(-2i/d).
//
// The work is bound by reading K and V once from HBM, so one or two heads are worked out on the vector ALUs; four
// heads go to the matrix cores, which leaves the vector ALUs half idle.  The kernels:
//   k_attend_partial  one workgroup per (KV head, chunk of rows, group of 1 or 2 query heads that share
//                     the KV head); every lane owns 4 rotary pairs of a row (8 channels), D/8 lanes
//                     share a row, and each such lane group walks its rows with a running
//                     max / sum / weighted-V state (online softmax).  cos/sin of the row position are
//                     advanced by a fixed rotation per step from seeds computed with an fp64 range
//                     reduction, so no table is read in the loop.
//   k_attend_quads    the same for groups of four query heads.
//   k_attend_merge    combines the per-chunk states of a query head and writes the output row (not needed for one chunk).
#include "freqkv_internal.h"

namespace freqkv {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kWaves = 4;
constexpr int kUnroll = 2;          // rows in flight per lane group per loop step (times two: prefetch)
constexpr float kMinusBig = -1.0e30f;
constexpr int kReseed = 32;          // loop steps between exact recomputations of the row cos/sin
constexpr float kSlack = 8.0f;      // log2 of the largest un-rescaled softmax weight

template <int I> struct IC { static constexpr int value = I; };
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (I < N) {
        f(IC<I>{});
        static_for<N, I + 1>(f);
    }
}

// ---- P consecutive channels (P = 4 or 8), as stored and as floats ---------------------------------
template <typename T, int P> struct Raw;
template <> struct Raw<uint16_t, 4> { u32x2 a; };
template <> struct Raw<float, 4>    { f32x4 a; };
template <> struct Raw<uint16_t, 8> { u32x4 a; };
template <> struct Raw<float, 8>    { f32x4 a, b; };

__device__ __forceinline__ void load_raw(const uint16_t* p, Raw<uint16_t, 4>& r) { r.a = *(const u32x2*)p; }
__device__ __forceinline__ void load_raw(const float* p, Raw<float, 4>& r) { r.a = *(const f32x4*)p; }
__device__ __forceinline__ void load_raw(const uint16_t* p, Raw<uint16_t, 8>& r) { r.a = *(const u32x4*)p; }
__device__ __forceinline__ void load_raw(const float* p, Raw<float, 8>& r) { r.a = *(const f32x4*)p; r.b = *(const f32x4*)(p + 4); }

// ... of a buffer, which reads as zero past its end
__device__ __forceinline__ void load_raw(__amdgpu_buffer_rsrc_t b, uint32_t at, Raw<uint16_t, 4>& r) { r.a = __builtin_amdgcn_raw_buffer_load_b64(b, at, 0, 0); }
__device__ __forceinline__ void load_raw(__amdgpu_buffer_rsrc_t b, uint32_t at, Raw<float, 4>& r)
{
    r.a = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(b, at, 0, 0));
}
__device__ __forceinline__ void load_raw(__amdgpu_buffer_rsrc_t b, uint32_t at, Raw<uint16_t, 8>& r) { r.a = __builtin_amdgcn_raw_buffer_load_b128(b, at, 0, 0); }
__device__ __forceinline__ void load_raw(__amdgpu_buffer_rsrc_t b, uint32_t at, Raw<float, 8>& r)
{
    r.a = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(b, at, 0, 0));
    r.b = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(b, at, 16, 0));
}

template <int P> __device__ __forceinline__ void unpack(const Raw<uint16_t, P>& r, float (&f)[P])
{
    static_for<P / 2>([&](auto i) {
        constexpr int I = decltype(i)::value;
        f[2 * I]     = __uint_as_float(r.a[I] << 16);
        f[2 * I + 1] = __uint_as_float(r.a[I] & 0xffff0000u);
    });
}
__device__ __forceinline__ void unpack(const Raw<float, 4>& r, float (&f)[4])
{
    static_for<4>([&](auto i) { f[decltype(i)::value] = r.a[decltype(i)::value]; });
}
__device__ __forceinline__ void unpack(const Raw<float, 8>& r, float (&f)[8])
{
    static_for<4>([&](auto i) { f[i.value] = r.a[i.value]; f[4 + i.value] = r.b[i.value]; });
}

// The upper half-wave of x and the lower of y change places.
__device__ __forceinline__ void swap_halves(u32x4& x, u32x4& y)
{
    static_for<4>([&](auto i) {
        const uint32_t a = x[i.value], b = y[i.value];
        const auto s = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        x[i.value] = s[0];
        y[i.value] = s[1];
    });
}
__device__ __forceinline__ void swap_halves(f32x4& x, f32x4& y)
{
    u32x4 a = __builtin_bit_cast(u32x4, x), b = __builtin_bit_cast(u32x4, y);
    swap_halves(a, b);
    x = __builtin_bit_cast(f32x4, a);
    y = __builtin_bit_cast(f32x4, b);
}
__device__ __forceinline__ void swap_halves(Raw<uint16_t, 8>& x, Raw<uint16_t, 8>& y) { swap_halves(x.a, y.a); }
__device__ __forceinline__ void swap_halves(Raw<float, 8>& x, Raw<float, 8>& y)
{
    swap_halves(x.a, y.a);
    swap_halves(x.b, y.b);
}

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// Lane exchange inside a row of 16 lanes through the data-parallel primitives (no LDS traffic).
template <int CTRL> __device__ __forceinline__ float dpp(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
// Sum over the LPR (4, 8, 16 or 32) adjacent lanes that share a cache row; every lane gets the sum.
template <int LPR> __device__ __forceinline__ float group_sum(float x)
{
    x += dpp<0xB1>(x);                           // quad_perm [1,0,3,2]
    x += dpp<0x4E>(x);                           // quad_perm [2,3,0,1]
    if constexpr (LPR >= 8) x += dpp<0x141>(x);  // mirror inside each half row of 8
    if constexpr (LPR >= 16) x += dpp<0x140>(x); // mirror inside the row of 16
    if constexpr (LPR >= 32) x += __shfl_xor(x, 16);
    return x;
}

// Barrier for what the workgroup keeps in LDS.  (The other one would wait for all loads as well, those of rows past the end of a chunk among
// them, which nobody uses: 2000 cycles at the end of every workgroup.)
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Lane I of each quad, in all four lanes of it.
template <int I> __device__ __forceinline__ float quad_lane(float x) { return dpp<I * 0x55>(x); }

// x op (x of the lane O further or nearer), in every lane; O = 4, 8, 16 or 32.  On the vector units: a shuffle goes through LDS, and
// a chain of them is what the end of a short call waits for.
template <int O, class F> __device__ __forceinline__ float fold(float x, F&& op)
{
    if constexpr (O == 4) {
        return op(x, dpp<0x141>(dpp<0x1B>(x)));  // mirrored in the quad [3,2,1,0], then in the half row
    } else if constexpr (O == 8) {
        return op(x, dpp<0x128>(x));             // the row of 16 turned by 8
    } else if constexpr (O == 16) {
        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return op(__uint_as_float(s[0]), __uint_as_float(s[1]));
    } else {
        static_assert(O == 32);
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return op(__uint_as_float(s[0]), __uint_as_float(s[1]));
    }
}
// Sums of two values over lanes O apart: the lanes without O in their index get that of x, the others that of y.
template <int O> __device__ __forceinline__ float fold_two(float x, float y, [[maybe_unused]] int lane)
{
    if constexpr (O == 4) {
        const bool upper = lane & 4;
        return (upper ? y : x) + dpp<0x141>(dpp<0x1B>(upper ? x : y));
    } else if constexpr (O == 8) {
        const bool upper = lane & 8;
        return (upper ? y : x) + dpp<0x128>(upper ? x : y);
    } else {
        static_assert(O == 16 || O == 32);
        const auto s = O == 16 ? __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false)
                               : __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(s[0]) + __uint_as_float(s[1]);
    }
}
// x of the lane without O in its index and of the one with it, for the two lanes O apart.
struct Pair { float of[2]; };
template <int O> __device__ __forceinline__ Pair both(float x)
{
    if constexpr (O == 16) {
        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return Pair{{__uint_as_float(s[0]), __uint_as_float(s[1])}};
    } else {
        static_assert(O == 4 || O == 8);
        // moved O lanes up into the quads that have O in their index, and down into those that have not
        constexpr int upper = O == 4 ? 0xa : 0xc;
        const int i = __builtin_bit_cast(int, x);
        return Pair{{__builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, 0x110 + O, 0xf, upper, false)),
                     __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, 0x100 + O, 0xf, 0xf ^ upper, false))}};
    }
}
// ... over the lanes O, 2 O, ... 32 apart
template <int O, class F> __device__ __forceinline__ float fold_from(float x, F&& op)
{
    x = fold<O>(x, op);
    if constexpr (O < 32) x = fold_from<2 * O>(x, op);
    return x;
}
// ... over all 64 lanes
template <class F> __device__ __forceinline__ float wave_fold(float x, F&& op)
{
    x = op(x, dpp<0xB1>(x));                     // lanes 1, 2 and 4 apart (quads exchange halves, half rows of 8 mirror)
    x = op(x, dpp<0x4E>(x));
    x = op(x, dpp<0x141>(x));
    return fold_from<8>(x, op);
}
struct Add { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct Max { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };

// Four heads: the score of the row lane / (D / 16) and the head that the lane's place in its quad names, from the products of four rows with the
// channels of its quad.  All quads that share a row get the same bits: where each keeps what it has, two lanes add up the same two
// values.  (D = 256, with S0..S3 the sums of the quads of 16 lanes: turned by 8 first S0 + S2 and S1 + S3.  By 4 first, they would have
// (S0 + S3) + (S2 + S1) or (S1 + S0) + (S3 + S2), and a quad's weights would not be those whose sum divides its results: 2e-5 off for scores of 30.)
template <int D> __device__ __forceinline__ float row_score(f32x4 x, int lane)
{
    if constexpr (D == 64) {
        return fold_two<4>(fold_two<8>(x[0], x[2], lane), fold_two<8>(x[1], x[3], lane), lane);
    } else if constexpr (D == 128) {
        return fold<4>(fold_two<8>(fold_two<16>(x[0], x[2], lane), fold_two<16>(x[1], x[3], lane), lane), Add{});
    } else {
        const float s = fold_two<16>(fold_two<32>(x[0], x[2], lane), fold_two<32>(x[1], x[3], lane), lane);
        const float t = s + dpp<0x128>(s);
        return t + dpp<0x124>(t);
    }
}

// Two adjacent results, rounded once.
__device__ __forceinline__ void store2(uint16_t* p, float a, float b)
{
    f32x2 v = {a, b};
    *(uint32_t*)p = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ void store2(float* p, float a, float b) { *(f32x2*)p = f32x2{a, b}; }

// cos and sin of pos * theta.  The product, its reduction to [-pi/4, pi/4] plus a quadrant and the two
// short Taylor sums (truncation below 2e-9 on that interval) are all in fp64; the results are rounded once.
struct CosSin { float c, s; };
// x is worked out where this stands.
__device__ __forceinline__ void here(float& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ CosSin seed_sincos(double theta, int pos)
{
    double x = (double)pos * theta;
    double k = rint(x * 0.6366197723675814);              // 2/pi
    double r = fma(-k, 1.5707963267948966, x);
    r = fma(-k, 6.123233995736766e-17, r);
    double r2 = r * r;
    // sin r = r (1 - r2/6 + r2^2/120 - r2^3/5040 + r2^4/362880 - r2^5/39916800)
    double ps = -1.0 / 39916800.0;
    ps = fma(ps, r2, 1.0 / 362880.0);
    ps = fma(ps, r2, -1.0 / 5040.0);
    ps = fma(ps, r2, 1.0 / 120.0);
    ps = fma(ps, r2, -1.0 / 6.0);
    ps = fma(ps, r2, 1.0);
    double sr = r * ps;
    // cos r = 1 - r2/2 + r2^2/24 - r2^3/720 + r2^4/40320 - r2^5/3628800 + r2^6/479001600
    double pc = 1.0 / 479001600.0;
    pc = fma(pc, r2, -1.0 / 3628800.0);
    pc = fma(pc, r2, 1.0 / 40320.0);
    pc = fma(pc, r2, -1.0 / 720.0);
    pc = fma(pc, r2, 1.0 / 24.0);
    pc = fma(pc, r2, -0.5);
    double cr = fma(pc, r2, 1.0);
    // add the quadrant back: angle = r + quad * pi/2
    int quad = (int)((long long)k & 3);
    double cs = (quad & 1) ? sr : cr;
    double ss = (quad & 1) ? cr : sr;
    if (quad == 1 || quad == 2) cs = -cs;
    if (quad >= 2) ss = -ss;
    return CosSin{(float)cs, (float)ss};
}

}  // namespace

// theta_j = base^(-2j/d) and the rotation that advances a row position by `step` rows; then the same for twice as many.
__global__ void k_rope_table(RopeEntry* rt, int d, double base, int step)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x, j = i < d / 2 ? i : i - d / 2;
    if (i >= d) return;
    if (i >= d / 2) step *= 2;
    double theta = base > 0.0 ? pow(base, -2.0 * (double)j / (double)d) : 0.0;       // no rotary embedding: every angle is zero
    double sd, cd;
    sincos((double)step * theta, &sd, &cd);
    RopeEntry e;
    e.theta = theta;
    e.cd = (float)cd;
    e.sd = (float)sd;
    rt[i] = e;
}

// The lane's index, counted again: kept across a loop, with what derives from it, it would not fit the registers of the longest kernels.
__device__ __forceinline__ int lane_index()
{
    uint32_t none = 0;
    asm volatile("" : "+v"(none));
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, none));
}

// Workgroups that read the same rows, for query heads beyond those of one, follow each other on one XCD (they are dealt round-robin to 8) and
// find them in its L2 (8 query heads to each of 4 KV heads x 8192 rows x 32 layers 181 -> 159 us, of 8 x 4000 x 32 167 -> 155; with all
// first parts ahead of all second ones, rows came from memory again).
__device__ __forceinline__ void share_out(int parts, int& chunk_id, int& part)
{
    const int chunks = (int)gridDim.x / parts, whole = chunks & ~7, at = chunk_id - whole * parts;
    if (at < 0) {
        const int grp = chunk_id / (8 * parts), local = chunk_id - grp * 8 * parts;
        part = local >> 3;
        chunk_id = grp * 8 + (local & 7);
    } else {
        part = at / (chunks - whole);
        chunk_id = whole + at - part * (chunks - whole);
    }
}

// The end of a chunk, from the states of its lane groups in LDS (red: HSLOTS of them; largest scores and sums of each wave): sums, and the chunk's
// state in memory or (ONE) the results.
template <typename T, int D, int GT, int W, int HSLOTS, bool ONE>
__device__ __forceinline__ void finish_chunk(const float* red, const float (&xm)[GT][W], const float (&xl)[GT][W], int tid, int heads, long long head0,
                                             int split, int n_split, float* __restrict__ part_acc, float* __restrict__ part_ml,
                                             T* __restrict__ out, float* __restrict__ lse)
{
    auto group_ml = [&](int gi, float* M, float* L) {
        *M = xm[gi][0];
        *L = xl[gi][0];
        static_for<W - 1>([&](auto w) { *M = fmaxf(*M, xm[gi][w.value + 1]); *L += xl[gi][w.value + 1]; });
    };
    const long long pidx = head0 * n_split + split;                            // + gi * n_split below
    for (int idx = tid; idx < heads * (D / 2); idx += W * 64) {
        const int gi = idx / (D / 2), ch = 2 * (idx - gi * (D / 2));
        f32x2 sum = {0.f, 0.f};
#pragma unroll
        for (int hs = 0; hs < HSLOTS; ++hs) sum += *(const f32x2*)(red + (hs * GT + gi) * D + ch);
        if constexpr (ONE) {
            float M, L;
            group_ml(gi, &M, &L);
            store2(out + (head0 + gi) * D + ch, sum[0] / L, sum[1] / L);
        } else {
            *(f32x2*)(part_acc + (pidx + (long long)gi * n_split) * D + ch) = sum;
        }
    }
    if (tid < heads) {
        float M, L;
        group_ml(tid, &M, &L);
        if constexpr (ONE) {
            if (lse) lse[head0 + tid] = 0.6931471805599453f * (M + log2f(L));
        } else {
            *(f32x2*)(part_ml + (pidx + (long long)tid * n_split) * 2) = f32x2{M, L};
        }
    }
}

// T: storage type of the cache, the query and the output (uint16_t = bfloat16 bits, or float).
// D: head_dim.  GT: query heads handled together (they share the KV head).  P: rotary pairs per lane
// (the lane owns channels P*l .. P*l+P-1 and their partners D/2 + P*l ..), so D/(2P) lanes share a row.
// ONE: there is one chunk only; the workgroup writes the results itself and no merge kernel runs.
// (Two forms were built and taken back.  Merging by the workgroup that arrives last: the arrival counter of a launch is an
// atomic of many workgroups on 8 XCDs, 28 us for 16 chunks of 8 heads against 19.5 with the second kernel.  Workgroups of
// eight waves: half as many loop steps, but the same time, 14.9 against 15.1 us at 32 chunks.)
// EXACT: no surplus loop step where a chunk has an odd number of them.
template <typename T, int D, int GT, int P, bool ONE, bool EXACT>
__global__ __launch_bounds__(kWaves * 64, attend_min_waves(sizeof(T), GT, P))
void k_attend_partial(const AttGeom, const T* __restrict__ q,
                      const RopeEntry* __restrict__ rt, float* __restrict__ part_acc,
                      float* __restrict__ part_ml, T* __restrict__ out, float* __restrict__ lse, const SlabTable tab)
{
    const AttGeom g = first_argument<decltype(k_attend_partial<T, D, GT, P, ONE, EXACT>)>();
    constexpr int LPR = D / (2 * P);       // lanes per cache row
    constexpr int RPW = 64 / LPR;          // rows per wave per load
    constexpr int STEP = kWaves * RPW;     // rows between two consecutive rows of one lane group
    constexpr int U = kUnroll;
    constexpr int HSLOTS = kWaves * RPW / 2;
    typedef Raw<T, P> RawT;

    __shared__ float red[HSLOTS * GT * D];
    __shared__ __attribute__((aligned(16))) float xm[GT][kWaves];
    __shared__ float xl[GT][kWaves];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = lane % LPR;
    const int slot = lane / LPR;

    int chunk_id = blockIdx.x, part = blockIdx.y;
    if (g.G != GT && gridDim.y == 1) share_out(g.G / GT, chunk_id, part);
    const int unit = g.by_split.quotient(chunk_id);
    const int split = chunk_id - unit * g.n_split;
    const int g0 = part * GT;                         // first query head of this workgroup inside the KV group
    const int layer = g.by_layer.quotient(unit);
    const int rem = unit - layer * g.units_per_layer;
    const int b = g.by_kv.quotient(rem);
    const int kvh = rem - b * g.n_kv;
    const long long head_off = (long long)b * g.stride_batch + (long long)kvh * g.stride_head;
    const T* kbase = (const T*)tab.base[2 * layer] + head_off;
    const T* vbase = (const T*)tab.base[2 * layer + 1] + head_off;

    // Cached rows and query position of this sequence: common to the batch, or per sequence (clamped to
    // [1, g.cur_len] so that every address stays inside the cache whatever the device array holds).
    int cur_len = g.cur_len, q_pos = g.q_pos;
    if (g.cur_lens) {
        cur_len = max(1, min(g.cur_lens[b], g.cur_len));
        q_pos = cur_len - 1;
    }
    const int row0 = split * g.chunk;
    const int row_end = min(row0 + g.chunk, cur_len);   // <= row0 for a chunk beyond a short sequence: no rows
    const int p0 = row0 + wave * RPW + slot;           // first row of this lane group

    // ---- rows of this lane group: p0, p0+STEP, p0+2*STEP, ...
    const int nit = row_end > row0 ? (row_end - row0 + STEP * U - 1) / (STEP * U) : 0;
    // Rows are addressed by 32-bit byte offsets inside the head's slab (uniform base + per-lane offset; the host
    // checks the range).  Of rows past the end of the chunk the values are zero, from past the end of a buffer (times a weight of 0 an infinite
    // value would be NaN), and the keys those of other rows, the last one's at most, and masked in the steps that can contain them: no load is
    // conditional, so the loads in flight can be counted exactly.
    const uint32_t row_bytes = (uint32_t)g.stride_token * (uint32_t)sizeof(T);
    const uint32_t lane_off = (uint32_t)(P * l) * (uint32_t)sizeof(T);
    const int size = (int)((uint32_t)max(row_end - 1, 0) * row_bytes + (uint32_t)(D * sizeof(T)));
    const __amdgpu_buffer_rsrc_t kbuf = __builtin_amdgcn_make_buffer_rsrc((void*)kbase, 0, size, kBufferFlags);
    const __amdgpu_buffer_rsrc_t vbuf = __builtin_amdgcn_make_buffer_rsrc((void*)vbase, 0, size, kBufferFlags);
    uint32_t next_off = (uint32_t)p0 * row_bytes + lane_off;      // first row of the step to be loaded next
    struct Rows { RawT kl[U], kh[U], vl[U], vh[U]; };
    auto issue = [&](Rows& r) {
        static_for<U>([&](auto uu) {
            constexpr int u = decltype(uu)::value;
            const uint32_t at = next_off + (uint32_t)(u * STEP) * row_bytes;
            load_raw(kbuf, at, r.kl[u]);
            load_raw(kbuf, at + D / 2 * (uint32_t)sizeof(T), r.kh[u]);
            load_raw(vbuf, at, r.vl[u]);
            load_raw(vbuf, at + D / 2 * (uint32_t)sizeof(T), r.vh[u]);
        });
        next_off += (uint32_t)(U * STEP) * row_bytes;
    };
    // Frequencies and queries, then the rows of the first step, all requested together ahead of the seeds: loads come back in
    // order.  (A second step of rows is slower, as several workgroups share a compute unit: 32 x
    // 4096 rows of 1 head 16.0 -> 16.9 us, 16 x 4096 of 2 12.1 -> 12.6, 32 x 1000 of 1 9.3 -> 9.9.)
    // (Left alone the compiler puts the rows behind the seeds.)
    RopeEntry re[P];
    RawT qrl[GT], qrh[GT];
    static_for<P>([&](auto jj) { re[jj.value] = rt[P * l + jj.value]; });
    static_for<GT>([&](auto gg) {
        const T* qp = q + ((long long)unit * g.G + g0 + gg.value) * D;
        load_raw(qp + P * l, qrl[gg.value]);
        load_raw(qp + D / 2 + P * l, qrh[gg.value]);
    });
    Rows ra, rb;
    issue(ra);
    __builtin_amdgcn_sched_barrier(0);

    // ---- rotary state of the P pairs this lane owns: pair j couples channels P*l+j and D/2+P*l+j.
    // (c, s) = cos/sin of (row position * theta_j); each processed row advances them by the fixed rotation
    // (cd, sd) of STEP rows, and every kReseed loop steps they are recomputed exactly.
    float c[P], s[P], cd[P], sd[P];
    auto seed_rows = [&](int pos, const RopeEntry (&entries)[P]) {
        static_for<P>([&](auto jj) {
            constexpr int j = decltype(jj)::value;
            const RopeEntry e = entries[j];
            CosSin k0 = seed_sincos(e.theta, pos);
            c[j] = k0.c; s[j] = k0.s;
            cd[j] = e.cd;
            sd[j] = e.sd;
        });
    };
    seed_rows(p0, re);

    // ---- queries: rotated at the query's position, scaled by log2(e)/sqrt(d) so that exp is exp2
    float ql[GT][P], qh[GT][P];
    {
        float qc[P], qs[P];
        static_for<P>([&](auto jj) {
            constexpr int j = decltype(jj)::value;
            CosSin q0 = seed_sincos(re[j].theta, q_pos);
            qc[j] = q0.c; qs[j] = q0.s;
        });
        static_for<GT>([&](auto gg) {
            constexpr int gi = decltype(gg)::value;
            float a[P], bb[P];
            unpack(qrl[gi], a);
            unpack(qrh[gi], bb);
            static_for<P>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                ql[gi][j] = (a[j] * qc[j] - bb[j] * qs[j]) * g.qscale;
                qh[gi][j] = (bb[j] * qc[j] + a[j] * qs[j]) * g.qscale;
            });
        });
    }

    float m[GT], lsum[GT], acc[GT][2 * P];
    static_for<GT>([&](auto gg) {
        constexpr int gi = decltype(gg)::value;
        m[gi] = kMinusBig;
        lsum[gi] = 0.f;
        static_for<2 * P>([&](auto cc) { acc[gi][decltype(cc)::value] = 0.f; });
    });

    // ---- main loop over the rows of this lane group: p0, p0+STEP, p0+2*STEP, ...
    // One step: the U rows in r (loaded a step ago) against the GT queries.
    auto consume = [&](const Rows& r, int it) {
        if (it != 0 && (it & (kReseed - 1)) == 0) {
            RopeEntry again[P];
            static_for<P>([&](auto jj) { again[jj.value] = rt[P * l + jj.value]; });
            seed_rows(p0 + it * U * STEP, again);
        }
        const bool tail = row0 + (it + 1) * U * STEP > row_end;       // same for the whole workgroup

        float sc[U][GT];
        static_for<U>([&](auto uu) {
            constexpr int u = decltype(uu)::value;
            float a[P], bb[P];
            unpack(r.kl[u], a);
            unpack(r.kh[u], bb);
            float part[GT];
            static_for<GT>([&](auto gg) { part[decltype(gg)::value] = 0.f; });
            static_for<P>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                float rl = a[j] * c[j] - bb[j] * s[j];
                float rh = bb[j] * c[j] + a[j] * s[j];
                static_for<GT>([&](auto gg) {
                    constexpr int gi = decltype(gg)::value;
                    part[gi] = fmaf(ql[gi][j], rl, part[gi]);
                    part[gi] = fmaf(qh[gi][j], rh, part[gi]);
                });
                float cn = c[j] * cd[j] - s[j] * sd[j];        // advance the pair's angle by STEP rows
                s[j] = s[j] * cd[j] + c[j] * sd[j];
                c[j] = cn;
            });
            static_for<GT>([&](auto gg) { sc[u][gg.value] = group_sum<LPR>(part[gg.value]); });
            if (tail) {                                        // only the last steps of a chunk can hold rows past its end
                const bool valid = p0 + (it * U + u) * STEP < row_end;
                static_for<GT>([&](auto gg) {
                    constexpr int gi = decltype(gg)::value;
                    sc[u][gi] = valid ? sc[u][gi] : -INFINITY;
                });
            }
        });

        static_for<GT>([&](auto gg) {
            constexpr int gi = decltype(gg)::value;
            // The reference point m of the running softmax only moves when a score exceeds it by more than
            // 2^kSlack; until then weights up to 2^kSlack are accumulated as they are (any reference point
            // gives the same quotient), and the rescaling of the accumulators is skipped for the whole wave.
            float mx = sc[0][gi];
            static_for<U>([&](auto uu) { mx = fmaxf(mx, sc[decltype(uu)::value][gi]); });
            const bool grow = mx > m[gi] + kSlack;
            if (__builtin_amdgcn_ballot_w64(grow) != 0) {
                float mn = grow ? mx : m[gi];
                float f = exp2_fast(m[gi] - mn);
                m[gi] = mn;
                lsum[gi] *= f;
                static_for<2 * P>([&](auto cc) { acc[gi][decltype(cc)::value] *= f; });
            }
            static_for<U>([&](auto uu) {
                constexpr int u = decltype(uu)::value;
                float pw = exp2_fast(sc[u][gi] - m[gi]);
                lsum[gi] += pw;
                float va[P], vb2[P];
                unpack(r.vl[u], va);
                unpack(r.vh[u], vb2);
                static_for<P>([&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    acc[gi][j] = fmaf(pw, va[j], acc[gi][j]);
                    acc[gi][P + j] = fmaf(pw, vb2[j], acc[gi][P + j]);
                });
            });
        });
    };
    // Two register sets take turns: while one step is consumed the loads of the next are in flight.  Without EXACT the step
    // count is rounded up to even; a surplus step sees only rows past the end (weights exactly zero).
    for (int it = 0; it < nit; it += 2) {
        issue(rb);
        consume(ra, it);
        if (EXACT && it + 1 >= nit) break;
        issue(ra);
        consume(rb, it + 1);
    }

    // ---- combine the lane groups of the workgroup
    // 1. common maximum per query head: over the lane groups of a wave by lane swaps, over waves through LDS; then sums, and accumulators
    // rescaled.
    const int ln = lane_index(), tid_end = wave * 64 + ln;
    float scale[GT];
    {
        static_for<GT>([&](auto gg) {
            constexpr int gi = decltype(gg)::value;
            const float mx = fold_from<LPR>(m[gi], Max{});
            if (ln == 0) xm[gi][wave] = mx;
        });
        lds_barrier();
        static_for<GT>([&](auto gg) {
            constexpr int gi = decltype(gg)::value;
            float M = xm[gi][0];
            static_for<kWaves - 1>([&](auto w) { M = fmaxf(M, xm[gi][w.value + 1]); });
            const float f = exp2_fast(m[gi] - M);
            const float ls = fold_from<LPR>(lsum[gi] * f, Add{});
            if (ln == 0) xl[gi][wave] = ls;
            scale[gi] = f;
        });
    }
    // Two neighbouring lane groups are folded into one, the even one keeping the lower half of the channels and the odd one the upper,
    // and park their sums in LDS.
    static_assert(P == 4);
    static_for<GT>([&](auto gg) {
        constexpr int gi = decltype(gg)::value;
        f32x4 sum;
        static_for<P>([&](auto jj) {
            constexpr int j = decltype(jj)::value;
            sum[j] = fold_two<LPR>(acc[gi][j] * scale[gi], acc[gi][P + j] * scale[gi], ln);
        });
        *(f32x4*)(red + ((wave * (RPW / 2) + (ln / LPR >> 1)) * GT + gi) * D + (ln / LPR & 1) * (D / 2) + P * (ln % LPR)) = sum;
    });
    lds_barrier();

    // 2. sum over the parked lane groups; two channels of one query head per thread and pass
    finish_chunk<T, D, GT, kWaves, HSLOTS, ONE>(red, xm, xl, tid_end, GT, (long long)unit * g.G + g0, split, g.n_split, part_acc, part_ml, out, lse);
}

// The same for four query heads that share a KV head, scores and weighted sums on the matrix cores (v_mfma_f32_4x4x1_16b_f32: fp32 products and
// sums; in each quad of lanes the product of 4 values, one per lane, and 4 others, a lane getting the 4 that its own value has part in).
//   keys     a quad of lanes has four rows, each lane 8 rotary pairs of its row; times the head that the lane's place in the quad names they give
//            the lane four scores' shares, summed over the quads by lane exchanges that halve what is left, so that a lane ends with one
//            score and one exponential for every 8 rows of 128 channels.
//   values   a lane has 8 adjacent channels of two rows.
// A key turns by the position of its row less that of the query, which so stays as it is.
// What bounds it: rows; with a workgroup to a compute unit also the time until the first come (4000 cycles) and, one wave to a SIMD hiding nothing, the 1400
// cycles of a step.  Rows asked for 16 bytes a lane, 170 vector instructions instead of 280 per 8 rows, frequencies and queries by whole lines, no rows
// beyond a chunk's end (with keys shared out like values, each lane 4 pairs, dot products on the vector units and a head's softmax to a lane ->
// this, graphs of calls, rows from HBM): 8 KV heads x 6147 rows 13.2 -> 12.4 us, x 3000 10.9 -> 9.9, x 16000 19.9 -> 18.7, 64 x 1000
// 14.2 -> 13.3, 128 x 4096 53.6 -> 51.5; d = 64, 8 x 4000, 9.9 -> 8.6; d = 256 14.8 -> 13.5; fp32 14.7 -> 12.2.  Where a call has the memory to itself for longer the
// sum is what it was: 256 x 8192 183 us, 5.9 TB/s.  Tried: copies into a ring in LDS, no registers for rows in flight (8 x 6147 12.5,
// 256 x 8192 196); waves that take rows apart from each other's (256 x 8192 198); 8 waves (8 x 6147 12.0, as these 11.2 in calls one after the
// other); the same for 1 and 2 heads (8 x 6147 of 1 head 9.1 -> 10.6 on rows in the memory-side cache, 11.5 -> 11.7 from HBM).
// SHORT: chunks of up to 2 kReseed steps.
// MANY: the heads are the queries of a chunk of g.q_len that has just been appended, g.G in all (for each head that shares the KV head all of the chunk), not
// always a multiple of four; each has its own position, by which it is turned, and its own number of rows.
// SETS: sets of four heads that a workgroup has.  Two of them share the rows' loads, unpacking and turning, 120 of 180 vector instructions per 8 rows; the
// results are the same to the bit.  Calls with 8 query heads to a KV head, a set to a workgroup -> two, graphs of calls, rows from HBM: 8 layers x 20 x
// 8 KV heads x 2143 rows 363 -> 291 us, 32 layers x 5 x 4 x 3806 322 -> 278, 5 x 16 x 310 of d = 256 217 -> 182, 8 x 56 x 8 x 488 of d = 64
// 141 -> 117, fp32 56 x 8 x 1476 150 -> 120; two_sets has the others.
// Of bf16 workgroups of one set three fit a compute unit, of the others two.  513 to 768 of them want three (the loop for long chunks had two registers too
// many: 576 workgroups of 4400 rows 267 us, 259 by threes).
template <typename T, bool MANY, int SETS> constexpr bool by_threes() { return sizeof(T) == 2 && SETS == 1 && !MANY; }
template <typename T, int D, bool ONE, bool SHORT, bool MANY, int SETS>
__global__ __launch_bounds__(kWaves * 64, (by_threes<T, MANY, SETS>() ? 3 : 2))
void k_attend_quads(const AttGeom, const T* __restrict__ q, const RopeEntry* __restrict__ rt, float* __restrict__ part_acc,
                    float* __restrict__ part_ml, T* __restrict__ out, float* __restrict__ lse, const SlabTable tab)
{
    const AttGeom g = first_argument<decltype(k_attend_quads<T, D, ONE, SHORT, MANY, SETS>)>();
    constexpr int GT = 4, W = kWaves;
    constexpr int N = 8;                          // channels of a value, and pairs of a key, that a lane has
    constexpr int LPR = D / N, RPW = 64 / LPR;    // lanes that share a value, rows that a wave's lanes have one value of each
    constexpr int SR = 2 * RPW;                   // rows of a wave's step
    constexpr int HSLOTS = W * RPW / 2;
    constexpr int kReseedSteps = 2 * kReseed;
    typedef Raw<T, N> RawN;

    constexpr int EB = D / 2 * (int)sizeof(RopeEntry), QB = SETS * GT * D * (int)sizeof(T), SB = 1024, TABLE = EB < SB ? SB : EB, QUERY = QB < SB ? SB : QB;
    constexpr int ENDS = HSLOTS * GT * D * 4, STARTS = W * (TABLE + QUERY);
    __shared__ __attribute__((aligned(16))) float red[(ENDS > STARTS ? ENDS : STARTS) / 4];
    __shared__ __attribute__((aligned(16))) float xm[GT][W];
    __shared__ float xl[GT][W];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // (neighbours read the same rows, see k_attend_partial)
    int chunk_id = blockIdx.x, part = blockIdx.y;
    if (g.G != SETS * GT && gridDim.y == 1) share_out(MANY ? (g.G + GT - 1) / GT : g.G / (SETS * GT), chunk_id, part);
    const int unit = g.by_split.quotient(chunk_id);
    const int split = chunk_id - unit * g.n_split;
    const int g0 = part * (SETS * GT);                // first query head of this workgroup inside the KV group
    const int layer = g.by_layer.quotient(unit);
    const int rem = unit - layer * g.units_per_layer;
    const int b = g.by_kv.quotient(rem);
    const int kvh = rem - b * g.n_kv;
    const long long head_off = ((long long)b * g.stride_batch + (long long)kvh * g.stride_head) * (long long)sizeof(T);
    const char* const kb = tab.base[2 * layer] + head_off;
    const char* const vb = tab.base[2 * layer + 1] + head_off;
    const long long head0 = (long long)unit * g.G + g0;                        // dense query head
    const int heads = MANY ? min(GT, g.G - g0) : GT;

    int cur_len = g.cur_len, q_pos = g.q_pos;
    if (g.cur_lens) {
        cur_len = max(1, min(g.cur_lens[b], g.cur_len));
        q_pos = cur_len - 1;
    }
    const int row0 = split * g.chunk;
    const int wave_row0 = row0 + wave * SR;
    // MANY: places of the queries in their chunk, of the lane's and the least and the last of the set's, which may go on from the end of one head's
    // chunk to the next head's; the rows that the lane's query sees, and that all of the set see.  No others than a query of the set sees are read.
    const int place = MANY ? g0 + (lane & 3) - g.by_q.quotient(g0 + (lane & 3)) * g.q_len : 0;
    const int place0 = MANY ? g0 - g.by_q.quotient(g0) * g.q_len : 0, past = cur_len - g.q_len + 1;
    const int row_end = min(row0 + g.chunk, MANY ? past + min(place0 + heads, g.q_len) - 1 : cur_len);   // <= row0 for a chunk beyond a short sequence: no rows
    const int limit = MANY ? min(row_end, past + place) : row_end, seen = MANY ? min(row_end, past + (place0 + heads > g.q_len ? 0 : place0)) : row_end;
    const int nit = row_end > row0 ? (row_end - row0 + W * SR - 1) / (W * SR) : 0;

    // ---- what a lane has.  Keys: 8 pairs, 8 piece .. +7, of the row krow of a step; of values 8 channels of the rows vrow and vrow + 1; and the score of
    // row srow.  Keys are requested in pieces of 16 bytes (fp32: 32), a quad of lanes having the same piece of four rows (asked for 8 bytes each,
    // they come at 4.7 TB/s instead of 6.1).  With 64 or 128 channels the lower half-wave has the lower channels of the first half of a step's rows and the upper
    // the upper ones; the next load has the other rows, and the half-waves trade.
    // Rows are addressed by 32-bit byte offsets inside the head's slab (the host checks the range).  Of rows past the end of the chunk the keys are its
    // last row's again, and masked, and the values zero, from past the end of a buffer (times a weight of 0 an infinite value would be NaN): no load is
    // conditional, so the loads in flight can be counted exactly.
    auto piece_of = [](int lane) { return D == 256 ? lane >> 2 : D == 128 ? lane >> 2 & 7 : lane >> 2 & 3; };
    auto krow_of = [](int lane) { return lane / (D / 4) * 4 + (lane & 3); };
    const int piece = piece_of(lane), krow = krow_of(lane), srow = lane / (LPR / 2), vrow = 2 * (lane / LPR);
    const uint32_t row_bytes = (uint32_t)g.stride_token * (uint32_t)sizeof(T);
    const uint32_t last_off = (uint32_t)max(row_end - 1, 0) * row_bytes;
    const uint32_t kfrom = (uint32_t)(D < 256 ? krow & (SR / 2 - 1) : krow) * row_bytes, vfrom = (uint32_t)vrow * row_bytes + (uint32_t)(N * (lane % LPR)) * (uint32_t)sizeof(T);
    const uint32_t kpart = (uint32_t)(N * piece + (D < 256 && lane >= 32 ? D / 2 : 0)) * (uint32_t)sizeof(T);
    const __amdgpu_buffer_rsrc_t vbuf = __builtin_amdgcn_make_buffer_rsrc((void*)vb, 0, (int)(last_off + (uint32_t)(D * sizeof(T))), kBufferFlags);
    uint32_t next_at = (uint32_t)wave_row0 * row_bytes;
    struct Rows { RawN kl, kh, v[2]; };
    auto issue = [&](Rows& r) {
        const uint32_t o = min(next_at + kfrom, last_off) + kpart;
        load_raw((const T*)(kb + o), r.kl);
        if constexpr (D == 256) load_raw((const T*)(kb + o) + D / 2, r.kh);
        else                    load_raw((const T*)(kb + (min(next_at + SR / 2 * row_bytes + kfrom, last_off) + kpart)), r.kh);
        static_for<2>([&](auto u) { load_raw(vbuf, next_at + u.value * row_bytes + vfrom, r.v[u.value]); });
        next_at += (uint32_t)(W * SR) * row_bytes;
    };
    // Frequencies and queries, then the rows of two steps, all requested together ahead of the seeds: loads come back in order.  Each wave asks for
    // whole lines, once, and hands them out through LDS: every lane asking for its own entries, the few lines of the table were
    // what all waves of the device waited for.
    char* const own = (char*)red + wave * (TABLE + QUERY);
    u32x4 line[(TABLE + QUERY) / SB];
    static_for<TABLE / SB>([&](auto j) { line[j.value] = *(const u32x4*)((const char*)(rt + D / 2) + min(j.value * SB + 16 * lane, EB - 16)); });
    static_for<QUERY / SB>([&](auto j) { line[TABLE / SB + j.value] = *(const u32x4*)((const char*)(q + head0 * D) + min(j.value * SB + 16 * lane, (MANY ? heads * (QB / GT) : QB) - 16)); });
    Rows ra, rb;
    issue(ra);
    issue(rb);
    __builtin_amdgcn_sched_barrier(0);
    static_for<(TABLE + QUERY) / SB>([&](auto j) { *(u32x4*)(own + j.value * SB + 16 * lane) = line[j.value]; });
    asm volatile("" ::: "memory");                    // (a wave's LDS instructions take effect in order)

    // ---- the lane's query, scaled by log2(e)/sqrt(d) so that exp is exp2, and the rotary state of its pairs: a pair couples channels j and D/2 + j.
    // (c, s) = cos/sin of ((row position - query position) * theta_j), so that the query stays as it is; each step advances them by the
    // fixed rotation (cd, sd) of its W SR rows, and every kReseedSteps they are recomputed exactly.
    float c[N], s[N], cd[N], sd[N], ql[SETS][N], qh[SETS][N];
    RawN qa[SETS], qb[SETS];
    static_for<SETS>([&](auto h) {
        load_raw((const T*)(own + TABLE) + (h.value * GT + (lane & 3)) * D + N * piece, qa[h.value]);
        load_raw((const T*)(own + TABLE) + (h.value * GT + (lane & 3)) * D + D / 2 + N * piece, qb[h.value]);
    });
    RopeEntry entries[N];
    static_for<N>([&](auto j) { entries[j.value] = ((const RopeEntry*)own)[N * piece + j.value]; });
    static_for<SETS>([&](auto h) {
        unpack(qa[h.value], ql[h.value]);
        unpack(qb[h.value], qh[h.value]);
        static_for<N>([&](auto j) {
            const float x = ql[h.value][j.value] * g.qscale, y = qh[h.value][j.value] * g.qscale;
            const CosSin k0 = MANY ? seed_sincos(entries[j.value].theta, place + 1 - g.q_len) : CosSin{1.f, 0.f};
            ql[h.value][j.value] = MANY ? x * k0.c - y * k0.s : x;
            qh[h.value][j.value] = MANY ? y * k0.c + x * k0.s : y;
        });
    });
    const int kp0 = wave_row0 + krow - q_pos;           // of the lane's key in the first step
    auto seed = [&](const RopeEntry (&entries)[N], int pos) {
        static_for<N>([&](auto j) {
            const CosSin k0 = seed_sincos(entries[j.value].theta, pos);
            c[j.value] = k0.c;
            s[j.value] = k0.s;
        });
    };
    static_for<N>([&](auto j) {
        cd[j.value] = entries[j.value].cd;
        sd[j.value] = entries[j.value].sd;
    });
    seed(entries, kp0);
    // (all of it ahead of the rows: moved into the loop's branch, frequencies and query would be awaited there, behind the rows)
    static_for<N>([&](auto j) {
        constexpr int J = j.value;
        here(c[J]); here(s[J]); here(cd[J]); here(sd[J]);
        static_for<SETS>([&](auto h) { here(ql[h.value][J]); here(qh[h.value][J]); });
    });

    typedef float Acc4 __attribute__((ext_vector_type(4)));
    float qm[SETS], qsum[SETS];                       // of the lane's head in each set
    Acc4 qacc[SETS][N];                               // [channel][head]
    auto start = [&] {
        static_for<SETS>([&](auto h) {
            qm[h.value] = kMinusBig;
            qsum[h.value] = 0.f;
            static_for<N>([&](auto cc) { qacc[h.value][cc.value] = Acc4{0.f, 0.f, 0.f, 0.f}; });
        });
    };
    start();

    // apart: in steps that hold rows which not all queries of the set see, each adds up those that it sees
    auto consume = [&](auto apart, Rows& r, int it) {
        if constexpr (D < 256) swap_halves(r.kl, r.kh);
        float a[N], bb[N];
        unpack(r.kl, a);
        unpack(r.kh, bb);
        // four rows, one to each lane of a quad, times four queries: [row] for the query of the lane
        f32x4 of_rows[SETS];
        static_for<SETS>([&](auto h) { of_rows[h.value] = f32x4{0.f, 0.f, 0.f, 0.f}; });
        static_for<N>([&](auto jj) {
            constexpr int j = jj.value;
            // (which product is rounded by itself is said here: left to the compiler, it is not the same for one set of heads and for two)
            const float lo = fmaf(a[j], c[j], -(bb[j] * s[j])), up = fmaf(bb[j], c[j], a[j] * s[j]);
            static_for<SETS>([&](auto h) { of_rows[h.value] = __builtin_amdgcn_mfma_f32_4x4x1f32(lo, ql[h.value][j], of_rows[h.value], 0, 0, 0); });
            static_for<SETS>([&](auto h) { of_rows[h.value] = __builtin_amdgcn_mfma_f32_4x4x1f32(up, qh[h.value][j], of_rows[h.value], 0, 0, 0); });
            const float cn = fmaf(c[j], cd[j], -(s[j] * sd[j]));
            s[j] = fmaf(s[j], cd[j], c[j] * sd[j]);
            c[j] = cn;
        });
        __builtin_amdgcn_sched_barrier(0);
        const bool tail = row0 + (it + 1) * (W * SR) > seen;
        const bool masked = tail && wave_row0 + it * (W * SR) + srow >= limit;
        Pair weights[SETS];
        static_for<SETS>([&](auto h) {
            float sc = row_score<D>(of_rows[h.value], lane);
            if (masked) sc = -INFINITY;
            // The reference point m of the running softmax only moves when a score exceeds it by more than 2^kSlack, see k_attend_partial.  It is
            // common to the two rows whose values a lane has.
            float& m = qm[h.value];
            const float mx = fold<LPR / 2>(sc, Max{});
            const bool grow = mx > m + kSlack;
            if (__builtin_amdgcn_ballot_w64(grow) != 0) {
                const float mn = grow ? mx : m;
                const float f = exp2_fast(m - mn);
                m = mn;
                qsum[h.value] *= f;
                static_for<GT>([&](auto gg) {
                    const float fh = quad_lane<gg.value>(f);
                    static_for<N>([&](auto cc) { qacc[h.value][cc.value][gg.value] *= fh; });
                });
            }
            const float pw = exp2_fast(sc - m);
            qsum[h.value] += pw;
            weights[h.value] = both<LPR / 2>(pw);
        });
        if constexpr (decltype(apart)::value != 0) {
            if (tail) {
                static_for<2>([&](auto u) {
                    const int row = wave_row0 + it * (W * SR) + vrow + u.value;
                    float va[N];
                    unpack(r.v[u.value], va);
                    static_for<GT>([&](auto gg) {
                        const float w = quad_lane<gg.value>(weights[0].of[u.value]);
                        const bool sees = row < __float_as_int(quad_lane<gg.value>(__int_as_float(limit)));
                        static_for<N>([&](auto cc) {
                            const float sum = qacc[0][cc.value][gg.value];
                            qacc[0][cc.value][gg.value] = sees ? fmaf(w, va[cc.value], sum) : sum;
                        });
                    });
                });
                return;
            }
        }
        static_for<2>([&](auto u) {
            float va[N];
            unpack(r.v[u.value], va);
            static_for<SETS>([&](auto h) {
                static_for<N>([&](auto cc) {
                    qacc[h.value][cc.value] = __builtin_amdgcn_mfma_f32_4x4x1f32(weights[h.value].of[u.value], va[cc.value], qacc[h.value][cc.value], 0, 0, 0);
                });
            });
        });
    };
    auto seed_again = [&](int it) {
        const int ln = lane_index();
        RopeEntry again[N];
        static_for<N>([&](auto j) { again[j.value] = rt[D / 2 + N * piece_of(ln) + j.value]; });
        seed(again, wave_row0 + krow_of(ln) - q_pos + it * (W * SR));
    };
    // Two register sets take turns: while one step is consumed the loads of the next are in flight.  A long chunk has its steps
    // rounded up to an even number; a surplus step sees only rows past the end (weights exactly zero).
    if constexpr (SHORT) {
        for (int it = 0; it < nit; it += 2) {
            consume(IC<0>{}, ra, it);
            if (it + 1 >= nit) break;
            __builtin_amdgcn_sched_barrier(0);
            issue(ra);
            __builtin_amdgcn_sched_barrier(0);
            consume(IC<0>{}, rb, it + 1);
            __builtin_amdgcn_sched_barrier(0);
            issue(rb);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        int it = 0;
        while (true) {
            for (const int end = min(nit, it + kReseedSteps); it < end; it += 2) {
                consume(IC<0>{}, ra, it);
                __builtin_amdgcn_sched_barrier(0);
                issue(ra);
                __builtin_amdgcn_sched_barrier(0);
                consume(IC<0>{}, rb, it + 1);
                __builtin_amdgcn_sched_barrier(0);
                issue(rb);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (it >= nit) break;
            seed_again(it);
        }
    }
    if constexpr (MANY) {
        // A value that is infinite or NaN, in a row that not all queries of the set see, has made the sums of the others NaN, by their weight of 0: sums that are
        // not finite are worked out again, with those rows left out where they are not seen.  (26 queries of 2 heads to each of 2 x 8 KV heads over 335 rows take 10.85 us,
        // 10.8 without this; values looked at in each step 11.2 to 11.3.)
        if (seen < row_end) {
            float none[4] = {0.f, 0.f, 0.f, 0.f};
            static_for<N>([&](auto cc) { static_for<GT>([&](auto gg) { none[gg.value] = fmaf(qacc[0][cc.value][gg.value], 0.f, none[gg.value]); }); });
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(none[0] + none[1] + none[2] + none[3] == 0.f)) != 0, 0)) {
                next_at = (uint32_t)wave_row0 * row_bytes;
                start();
                for (int it = 0; it < nit; ++it) {
                    if (it % kReseedSteps == 0) seed_again(it);
                    issue(ra);
                    consume(IC<1>{}, ra, it);
                }
            }
        }
    }

    // ---- combine the lane groups of the workgroup
    // 1. common maximum per query head: over the lane groups of a wave by lane swaps, over waves through LDS; then sums, and accumulators
    // rescaled, one head to a lane of each quad.
    const int ln = lane_index(), tid_end = wave * 64 + ln;
    static_for<SETS>([&](auto h) {
        if constexpr (h.value > 0) lds_barrier();         // (the set before has been read)
        float scale[GT];
        {
            const float mx = fold_from<LPR>(qm[h.value], Max{});
            if (ln < GT) xm[ln][wave] = mx;
            lds_barrier();
            float M = kMinusBig;
            static_for<W / 4>([&](auto w) {
                const f32x4 of_waves = *(const f32x4*)&xm[ln & 3][4 * w.value];
                M = fmaxf(M, fmaxf(fmaxf(of_waves[0], of_waves[1]), fmaxf(of_waves[2], of_waves[3])));
            });
            const float f = exp2_fast(qm[h.value] - M);
            const float ls = fold_from<LPR / 2>(qsum[h.value] * f, Add{});
            if (ln < GT) xl[ln][wave] = ls;
            static_for<GT>([&](auto gg) { scale[gg.value] = quad_lane<gg.value>(f); });
        }
        // Two neighbouring lane groups are folded into one, the even one keeping the lower half of the lanes' channels and the odd one the upper,
        // and park their sums in LDS.
        static_for<GT>([&](auto gg) {
            constexpr int gi = decltype(gg)::value;
            f32x4 sum;
            static_for<4>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                sum[j] = fold_two<LPR>(qacc[h.value][j][gi] * scale[gi], qacc[h.value][4 + j][gi] * scale[gi], ln);
            });
            *(f32x4*)(red + ((wave * (RPW / 2) + (ln / LPR >> 1)) * GT + gi) * D + N * (ln % LPR) + (ln / LPR & 1) * 4) = sum;
        });
        lds_barrier();

        // 2. sum over the parked lane groups; two channels of one query head per thread and pass
        finish_chunk<T, D, GT, W, HSLOTS, ONE>(red, xm, xl, tid_end, heads, head0 + h.value * GT, split, g.n_split, part_acc, part_ml, out, lse);
    });
}

// One workgroup per query head merges the chunk states, normalises, stores.  D/2 threads cover the channels (two each), and
// kMergeShare such groups of threads take the chunks in turn: what the kernel costs is the chain of loads, so that all of them
// should be in flight (22 chunks of one head: 8.2 us with one load behind the other, see the figures in k_attend_partial).
constexpr int kMergeShare = 4;
template <typename T, int D>
__global__ __launch_bounds__(kMergeShare * D / 2)
void k_attend_merge(const AttGeom, const float* __restrict__ part_acc, const float* __restrict__ part_ml,
                    T* __restrict__ out, float* __restrict__ lse)
{
    const AttGeom g = first_argument<decltype(k_attend_merge<T, D>)>();
    constexpr int NT = kMergeShare * D / 2, NWV = NT / 64;
    __shared__ float wm[NWV], wl[NWV], sh_w[NT];
    __shared__ f32x2 sh_sum[kMergeShare][D / 2];
    const long long head = blockIdx.x;                    // (layer, batch, query head), dense
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int pr = tid % (D / 2), part = tid / (D / 2);
    const f32x2* ml = (const f32x2*)(part_ml + head * g.n_split * 2);
    const float* acc = part_acc + head * g.n_split * D + 2 * pr;
    f32x2 sum = {0.f, 0.f};
    float M = kMinusBig, L = 0.f;
    for (int s0 = 0; s0 < g.n_split; s0 += NT) {          // NT chunks at a time (one pass but for tiny head counts)
        const int here = min(NT, g.n_split - s0);
        // the accumulators of the first chunks are requested ahead of everything else
        f32x2 v[8] = {};
        static_for<8>([&](auto i) {
            if (i.value * kMergeShare < here)
                v[i.value] = *(const f32x2*)(acc + (long long)min(s0 + part + i.value * kMergeShare, g.n_split - 1) * D);
        });
        const f32x2 mine = tid < here ? ml[s0 + tid] : f32x2{kMinusBig, 0.f};
        float mx = mine[0];
        mx = wave_fold(mx, Max{});
        if (lane == 0) wm[wave] = mx;
        __syncthreads();
        float Mn = M;
        static_for<NWV>([&](auto w) { Mn = fmaxf(Mn, wm[w.value]); });
        const float w = tid < here ? exp2_fast(mine[0] - Mn) : 0.f;
        sh_w[tid] = w;
        float ls = mine[1] * w;
        ls = wave_fold(ls, Add{});
        if (lane == 0) wl[wave] = ls;
        __syncthreads();
        const float f = exp2_fast(M - Mn);
        L *= f;
        static_for<NWV>([&](auto i) { L += wl[i.value]; });
        sum[0] *= f;
        sum[1] *= f;
        M = Mn;
        for (int sp0 = part; sp0 < here; sp0 += 8 * kMergeShare) {
            if (sp0 != part)
                static_for<8>([&](auto i) { v[i.value] = *(const f32x2*)(acc + (long long)min(s0 + sp0 + i.value * kMergeShare, g.n_split - 1) * D); });
            static_for<8>([&](auto i) {
                const int sp = sp0 + i.value * kMergeShare;
                if (sp >= here) return;
                const float x = sh_w[sp];
                sum[0] = fmaf(v[i.value][0], x, sum[0]);
                sum[1] = fmaf(v[i.value][1], x, sum[1]);
            });
        }
        __syncthreads();
    }
    sh_sum[part][pr] = sum;
    __syncthreads();
    if (part == 0) {
        static_for<kMergeShare - 1>([&](auto i) { sum[0] += sh_sum[i.value + 1][pr][0]; sum[1] += sh_sum[i.value + 1][pr][1]; });
        store2(out + head * D + 2 * pr, sum[0] / L, sum[1] / L);
        if (lse && pr == 0) lse[head] = 0.6931471805599453f * (M + log2f(L));
    }
}

// ---------------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------------

hipError_t launch_rope_table(RopeEntry* rt, int d, double base, hipStream_t st)
{
    int step = attend_row_step(d);
    hipLaunchKernelGGL(k_rope_table, dim3((d + 63) / 64), dim3(64), 0, st, rt, d, base, step);
    return hipGetLastError();
}

static dim3 partial_grid(const AttGeom& g, int together)
{
    const long long chunks = (long long)g.units * g.n_split, parts = (g.G + together - 1) / together;
    return chunks * parts < 1 << 23 ? dim3((unsigned)(chunks * parts)) : dim3((unsigned)chunks, (unsigned)parts);   // (a launch has up to 2^32 threads per direction)
}

template <typename T, int D, int GT, bool ONE, bool EXACT>
static void launch_partial_o(const SlabTable& tab, const AttGeom& g, const void* q, const RopeEntry* rt, float* part_acc,
                             float* part_ml, void* out, float* lse, hipStream_t st)
{
    const dim3 grid = partial_grid(g, GT);
    hipLaunchKernelGGL((k_attend_partial<T, D, GT, attend_pairs_per_lane(D), ONE, EXACT>), grid, dim3(kWaves * 64), 0, st, g, (const T*)q, rt,
                       part_acc, part_ml, (T*)out, lse, tab);
}

template <typename T, int D, int GT>
static void launch_partial_g(const SlabTable& tab, const AttGeom& g, const void* q, const RopeEntry* rt, float* part_acc,
                             float* part_ml, void* out, float* lse, hipStream_t st)
{
    // Odd numbers of steps up to 23: leaving the last one out gives 4 % and more (7 steps, 28 chunks of 224 rows: 15.1 -> 13.8 us per
    // call); the branch in the loop costs 0.4 % of long chunks.
    const int steps = g.chunk / (kUnroll * attend_row_step(D));
    const bool exact = (steps & 1) && steps < 24;
    if (g.n_split == 1) exact ? launch_partial_o<T, D, GT, true, true>(tab, g, q, rt, part_acc, part_ml, out, lse, st)
                              : launch_partial_o<T, D, GT, true, false>(tab, g, q, rt, part_acc, part_ml, out, lse, st);
    else                exact ? launch_partial_o<T, D, GT, false, true>(tab, g, q, rt, part_acc, part_ml, out, lse, st)
                              : launch_partial_o<T, D, GT, false, false>(tab, g, q, rt, part_acc, part_ml, out, lse, st);
}

template <typename T, int D, bool MANY, int SETS>
static void launch_quads(const SlabTable& tab, const AttGeom& g, const void* q, const RopeEntry* rt, float* part_acc, float* part_ml, void* out,
                         float* lse, hipStream_t st)
{
    const dim3 grid = partial_grid(g, 4 * SETS);
    // Long chunks: more workgroups than three to each compute unit go by twos, held apart by LDS that they do not use, so that the last
    // round has more of them (4400 rows, by threes -> by twos: 800 workgroups 353 -> 328 us, 896 371 -> 362, 1024 397 -> 395, 1280 496 -> 495, 2048 787 -> 780; up to three
    // all are there at once, and 576 of them take 259 instead of 266).
    const unsigned apart = by_threes<T, MANY, SETS>() && (long long)grid.x * grid.y > 3 * 256 ? 40 << 10 : 0;
    const bool brief = g.chunk <= 2 * kReseed * kUnroll * attend_row_step(D);
    auto launch = [&](auto one, auto is_short) {
        hipLaunchKernelGGL((k_attend_quads<T, D, decltype(one)::value != 0, decltype(is_short)::value != 0, MANY, SETS>), grid, dim3(kWaves * 64),
                           decltype(is_short)::value ? 0 : apart, st, g, (const T*)q, rt, part_acc, part_ml, (T*)out, lse, tab);
    };
    if constexpr (SETS > 1) {
        // (left early, as SHORT leaves its loop at an odd step, the loop takes more registers than there are)
        g.n_split == 1 ? launch(IC<1>{}, IC<0>{}) : launch(IC<0>{}, IC<0>{});
    } else if (g.n_split == 1) {
        brief ? launch(IC<1>{}, IC<1>{}) : launch(IC<1>{}, IC<0>{});
    } else {
        brief ? launch(IC<0>{}, IC<1>{}) : launch(IC<0>{}, IC<0>{});
    }
}

// Two sets of four heads to a workgroup: a workgroup takes 1.2 to 1.4 times as long, and there are half as many; an odd number of steps is rounded up.
// Time of one set to a workgroup over that of two (above 1 two are faster; 1 to 11 steps of 2 * attend_row_step(d) rows, much the same for d = 64, 128, 256):
// (profiles/decode_sets.txt)
//   workgroups of two sets                      bf16: 1 step   3     5    even   9, 11      fp32: 1 step   3     5    even   7    9, 11
//   up to 128 (every second compute unit idle; 128 8.3 us for 6.8 at 8 KV heads of 8 x 100 rows)
//   136 to 256 (one to a compute unit)                 0.91  1.00  1.03  1.11  1.06               0.91  0.94  0.93  1.04  1.02  1.09
//   300, 384 (two; of the others three, in fp32 two)   0.83  0.86  0.86  0.97  0.89               0.95  0.91  0.95  1.05  0.98  1.00 (long ones 1.03 to 1.27)
//   400, 500                                           1.02  1.06  1.07  1.21  1.12               1.11  1.06  1.13  1.22  1.16  1.18
//   520, 600 (a few for the second time)               0.85  0.90  0.91  1.03  0.97               0.95  0.98  1.04  1.11  1.07  1.06
//   700; 1000 and 1200                                 0.96  1.04  1.04  1.17  1.09               1.09  1.11  1.17  1.26  1.19  1.19
//   800                                                0.88  0.93  0.96  1.08  0.99               1.02  1.03  1.08  1.17  1.10  1.09
static bool two_sets(const AttGeom& g, int elem_bytes)
{
    if (g.G % 8) return false;
    const long long wgs = (long long)g.units * g.n_split * (g.G / 8);
    const bool f32 = elem_bytes == 4;
    int one = 0;                               // odd numbers of steps up to this have one set
    if (wgs <= 128) return false;
    else if (wgs <= 256) one = f32 ? 5 : 1;
    else if (wgs <= 384) { if (!f32) return false; one = 11; }
    else if (wgs <= 512) one = 0;
    else if (wgs <= 640) one = f32 ? 3 : 9;
    else if (!f32) one = wgs > 768 && wgs <= 896 ? 9 : 1;
    const int rows = kUnroll * attend_row_step(g.d), steps = ((g.chunk < g.cur_len ? g.chunk : g.cur_len) + rows - 1) / rows;
    return steps % 2 == 0 || steps > one;
}

template <typename T, int D>
static hipError_t launch_partial_d(const SlabTable& tab, const AttGeom& g, const void* q, const RopeEntry* rt, float* part_acc,
                                   float* part_ml, void* out, float* lse, hipStream_t st)
{
    switch (g.GT) {
        case 4:
            if (two_sets(g, sizeof(T))) launch_quads<T, D, false, 2>(tab, g, q, rt, part_acc, part_ml, out, lse, st);
            else                        launch_quads<T, D, false, 1>(tab, g, q, rt, part_acc, part_ml, out, lse, st);
            break;
        case 2: launch_partial_g<T, D, 2>(tab, g, q, rt, part_acc, part_ml, out, lse, st); break;
        case 1: launch_partial_g<T, D, 1>(tab, g, q, rt, part_acc, part_ml, out, lse, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_partial_t(const SlabTable& tab, const AttGeom& g, const void* q, const RopeEntry* rt,
                                   float* part_acc, float* part_ml, void* out, float* lse, hipStream_t st)
{
    if (g.P != attend_pairs_per_lane(g.d)) return hipErrorInvalidValue;
    switch (g.d) {
        case 64:  return launch_partial_d<T, 64>(tab, g, q, rt, part_acc, part_ml, out, lse, st);
        case 128: return launch_partial_d<T, 128>(tab, g, q, rt, part_acc, part_ml, out, lse, st);
        case 256: return launch_partial_d<T, 256>(tab, g, q, rt, part_acc, part_ml, out, lse, st);
        default:  return hipErrorInvalidValue;
    }
}

hipError_t launch_attend_partial(const SlabTable& tab, const AttGeom& g, int elem_bytes, const void* q,
                                 const RopeEntry* rt, float* part_acc, float* part_ml, void* out, float* lse, hipStream_t st)
{
    if (g.units < 1 || g.n_split < 1 || g.chunk < 1 || g.cur_len < 1) return hipErrorInvalidValue;
    if ((long long)(g.n_split - 1) * g.chunk >= g.cur_len) return hipErrorInvalidValue;   // no chunk beyond the longest cache
    if ((long long)g.n_split * g.chunk < g.cur_len) return hipErrorInvalidValue;          // chunks cover the cache
    if (g.G % g.GT) return hipErrorInvalidValue;
    if (g.chunk % (kUnroll * attend_row_step(g.d))) return hipErrorInvalidValue;
    return elem_bytes == 2 ? launch_partial_t<uint16_t>(tab, g, q, rt, part_acc, part_ml, out, lse, st)
                           : launch_partial_t<float>(tab, g, q, rt, part_acc, part_ml, out, lse, st);
}

hipError_t launch_attend_many(const SlabTable& tab, const AttGeom& g, const void* q, const RopeEntry* rt, float* part_acc, float* part_ml, void* out,
                              float* lse, hipStream_t st)
{
    if (g.units < 1 || g.n_split < 1 || g.chunk < 1 || g.q_len < 1 || g.q_len > g.cur_len || g.G % g.q_len) return hipErrorInvalidValue;
    if ((long long)(g.n_split - 1) * g.chunk >= g.cur_len || (long long)g.n_split * g.chunk < g.cur_len) return hipErrorInvalidValue;
    if (g.d != 128 || g.GT != 4 || g.cur_lens || g.chunk % (kUnroll * attend_row_step(g.d))) return hipErrorInvalidValue;
    launch_quads<uint16_t, 128, true, 1>(tab, g, q, rt, part_acc, part_ml, out, lse, st);
    return hipGetLastError();
}

hipError_t launch_attend_merge(const AttGeom& g, int elem_bytes, const float* part_acc, const float* part_ml,
                               void* out, float* lse, hipStream_t st)
{
    if (g.n_split < 2) return hipSuccess;                 // the one chunk's workgroup has written the results
    const dim3 grid((unsigned)((long long)g.units * g.G)), block(kMergeShare * g.d / 2);
    auto launch = [&](auto d) {
        constexpr int D = decltype(d)::value;
        if (elem_bytes == 2) hipLaunchKernelGGL((k_attend_merge<uint16_t, D>), grid, block, 0, st, g, part_acc, part_ml, (uint16_t*)out, lse);
        else                 hipLaunchKernelGGL((k_attend_merge<float, D>), grid, block, 0, st, g, part_acc, part_ml, (float*)out, lse);
    };
    switch (g.d) {
        case 64:  launch(IC<64>{}); break;
        case 128: launch(IC<128>{}); break;
        case 256: launch(IC<256>{}); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace freqkv
