// gfx950 kernels for decode attention over the compacted cache.
//
// One incoming token attends to every cached row [0, cur_len) of its KV head: sinks, compressed rows
// and the tokens appended since, itself included (Sec. 3.3 Eq. 4, Sec. 3.4 Eq. 5).  Keys are cached
// without the rotary embedding; the key of cache row p is rotated by position p, an index inside the
// cache, when it is read, and the query by its own in-cache position (closing paragraph of Sec. 3.4,
// appendix on key states with RoPE).  Rotary pairing is LLaMA's: channel i turns with channel i + d/2
// by the angle pos * base^(-2i/d).
//
// The work is bound by reading K and V once from HBM, so scores are worked out on the vector ALUs; the weighted sums of four
// heads go to the matrix cores, which leaves the vector ALUs half idle.  Two kernels:
//   k_attend_partial  one workgroup per (KV head, chunk of rows, group of <= 4 query heads that share
//                     the KV head); every lane owns 4 rotary pairs of a row (8 channels), D/8 lanes
//                     share a row, and each such lane group walks its rows with a running
//                     max / sum / weighted-V state (online softmax).  cos/sin of the row position are
//                     advanced by a fixed rotation per step from seeds computed with an fp64 range
//                     reduction, so no table is read in the loop.
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

__device__ __forceinline__ void load_raw(const uint16_t* p, Raw<uint16_t, 4>& r) { r.a = *(const u32x2*)p; }
__device__ __forceinline__ void load_raw(const float* p, Raw<float, 4>& r) { r.a = *(const f32x4*)p; }

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

// Sums of four values over the LPR adjacent lanes that share a cache row: lane i of each quad gets that of x[i].  The first two steps
// halve what is left to sum.  All quads get the same bits: with S0..S3 the sums of the quads of a row of 16, turned by 8 first each has S0 + S2 or S1 + S3,
// and then the sum of both.  (By 4 first, they would have (S0 + S3) + (S2 + S1) or (S1 + S0) + (S3 + S2), and a quad's weights would not
// be those whose sum divides its results: 2e-5 off for scores of 30.)
template <int LPR> __device__ __forceinline__ float quad_sums(const float (&x)[4], int lane)
{
    const bool odd = lane & 1, high = lane & 2;
    float a = odd ? x[1] : x[0], b = odd ? x[3] : x[2];
    a += dpp<0xB1>(odd ? x[0] : x[1]);           // quad_perm [1,0,3,2]
    b += dpp<0xB1>(odd ? x[2] : x[3]);
    float s = high ? b : a;
    s += dpp<0x4E>(high ? a : b);                // quad_perm [2,3,0,1]
    if constexpr (LPR == 8) {
        s += dpp<0x141>(dpp<0x1B>(s));           // the other quad of the half row: mirrored in the quad [3,2,1,0], then in the half row
    } else {
        static_assert(LPR >= 16);
        s += dpp<0x128>(s);                      // the row of 16 turned by 8 and by 4
        s += dpp<0x124>(s);
        if constexpr (LPR >= 32) s += __shfl_xor(s, 16);
    }
    return s;
}

// x op (x of the lane O further or nearer), in every lane; O = 8, 16 or 32.  On the vector units: a shuffle goes through LDS, and
// a chain of them is what the end of a short call waits for.
template <int O, class F> __device__ __forceinline__ float fold(float x, F&& op)
{
    if constexpr (O == 8) {
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
    if constexpr (O == 8) {
        const bool upper = lane & 8;
        return (upper ? y : x) + dpp<0x128>(upper ? x : y);
    } else {
        static_assert(O == 16 || O == 32);
        const auto s = O == 16 ? __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false)
                               : __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(s[0]) + __uint_as_float(s[1]);
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

// theta_j = base^(-2j/d) and the rotation that advances a row position by `step` rows.
__global__ void k_rope_table(RopeEntry* rt, int d, double base, int step)
{
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= d / 2) return;
    double theta = pow(base, -2.0 * (double)j / (double)d);
    double sd, cd;
    sincos((double)step * theta, &sd, &cd);
    RopeEntry e;
    e.theta = theta;
    e.cd = (float)cd;
    e.sd = (float)sd;
    rt[j] = e;
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
    constexpr bool QUADS = GT == 4;        // see the main loop
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

    // Workgroups that read the same rows, for query heads beyond GT, follow each other on one XCD (they are dealt round-robin to 8) and
    // find them in its L2 (8 query heads to each of 4 KV heads x 8192 rows x 32 layers 181 -> 159 us, of 8 x 4000 x 32 167 -> 155; with all
    // first parts ahead of all second ones, rows came from memory again).
    int chunk_id = blockIdx.x, part = blockIdx.y;
    if (g.G != GT && gridDim.y == 1) {
        const int parts = g.G / GT, chunks = (int)gridDim.x / parts, whole = chunks & ~7, at = chunk_id - whole * parts;
        if (at < 0) {
            const int grp = chunk_id / (8 * parts), local = chunk_id - grp * 8 * parts;
            part = local >> 3;
            chunk_id = grp * 8 + (local & 7);
        } else {
            part = at / (chunks - whole);
            chunk_id = whole + at - part * (chunks - whole);
        }
    }
    const int unit = chunk_id / g.n_split;
    const int split = chunk_id - unit * g.n_split;
    const int g0 = part * GT;                         // first query head of this workgroup inside the KV group
    const int layer = unit / g.units_per_layer;
    const int rem = unit - layer * g.units_per_layer;
    const int b = rem / g.n_kv;
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
    const int last = cur_len - 1;
    // Rows are addressed by 32-bit byte offsets inside the head's slab (uniform base + per-lane offset; the host
    // checks the range).  Rows past the end re-read the last row: no load is conditional, so the loads in
    // flight can be counted exactly; such rows are masked in the steps that can contain them.
    const char* kb = (const char*)kbase;
    const char* vb = (const char*)vbase;
    const uint32_t row_bytes = (uint32_t)g.stride_token * (uint32_t)sizeof(T);
    const uint32_t lane_off = (uint32_t)(P * l) * (uint32_t)sizeof(T);
    const uint32_t last_off = (uint32_t)last * row_bytes + lane_off;
    uint32_t next_off = (uint32_t)p0 * row_bytes + lane_off;      // first row of the step to be loaded next
    struct Rows { RawT kl[U], kh[U], vl[U], vh[U]; };
    auto issue = [&](Rows& r) {
        static_for<U>([&](auto uu) {
            constexpr int u = decltype(uu)::value;
            const uint32_t o = min(next_off + (uint32_t)(u * STEP) * row_bytes, last_off);
            load_raw((const T*)(kb + o), r.kl[u]);
            load_raw((const T*)(kb + o) + D / 2, r.kh[u]);
            load_raw((const T*)(vb + o), r.vl[u]);
            load_raw((const T*)(vb + o) + D / 2, r.vh[u]);
        });
        next_off += (uint32_t)(U * STEP) * row_bytes;
    };
    // Frequencies and queries, then the rows of the first step or (QUADS) two, all requested together ahead of the seeds: loads come back in
    // order.  (With 1 or 2 heads more workgroups share a compute unit, and a step less in flight is faster: 32 x
    // 4096 rows of 1 head 16.9 -> 16.0 us, 16 x 4096 of 2 12.6 -> 12.1, 32 x 1000 of 1 9.9 -> 9.3.)
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
    if constexpr (QUADS) issue(rb);
    __builtin_amdgcn_sched_barrier(0);

    // ---- rotary state of the P pairs this lane owns: pair j couples channels P*l+j and D/2+P*l+j.
    // (c, s) = cos/sin of (row position * theta_j); each processed row advances them by the fixed rotation
    // (cd, sd) of STEP rows, and every kReseed loop steps they are recomputed exactly.
    float c[P], s[P], cd[P], sd[P];
    auto seed_rows = [&](int pos, const RopeEntry (&entries)[P]) {
        static_for<P>([&](auto jj) {
            constexpr int j = decltype(jj)::value;
            const RopeEntry e = entries[j];
            CosSin k0 = seed_sincos(g.rope ? e.theta : 0.0, pos);   // no rotary embedding: every angle is zero
            c[j] = k0.c; s[j] = k0.s;
            cd[j] = g.rope ? e.cd : 1.f;
            sd[j] = g.rope ? e.sd : 0.f;
        });
    };
    seed_rows(p0, re);

    // ---- queries: rotated at the query's position, scaled by log2(e)/sqrt(d) so that exp is exp2
    float ql[GT][P], qh[GT][P];
    {
        float qc[P], qs[P];
        static_for<P>([&](auto jj) {
            constexpr int j = decltype(jj)::value;
            CosSin q0 = seed_sincos(g.rope ? re[j].theta : 0.0, q_pos);
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

    // Four heads: softmax of a row by quads of lanes, a head to each lane, and weighted sums on the matrix cores (v_mfma_f32_4x4x1, fp32 in and
    // out: in each quad the product of 4 weights, one per lane, and 4 values, one per lane; a lane gets the 4 sums of its channel).  What
    // bounds a chunk that has its compute unit to itself is vector issue, 4 cycles per instruction: a step of two rows took 440
    // of them with every lane working out all heads, four exponentials at a quarter of the rate among them, and takes 280, so that rows are
    // what it waits for (1 x 8 KV heads x 6147 rows 14.4 -> 13.2 us per call, with the arguments and the last barrier 12.5; x 16000 20.9 -> 17.9; 32 layers
    // x 8 x 4000 rows with 8 query heads each 152 -> 138).
    typedef float Acc4 __attribute__((ext_vector_type(4)));
    [[maybe_unused]] float qm = kMinusBig, qsum = 0.f;   // of the lane's head
    [[maybe_unused]] Acc4 qacc[2 * P];                   // [channel][head]
    static_for<2 * P>([&](auto cc) { qacc[cc.value] = Acc4{0.f, 0.f, 0.f, 0.f}; });

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

        float sc[U][QUADS ? 1 : GT];
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
            if constexpr (QUADS) sc[u][0] = quad_sums<LPR>(part, lane);
            else static_for<GT>([&](auto gg) { sc[u][gg.value] = group_sum<LPR>(part[gg.value]); });
            if (tail) {                                        // only the last steps of a chunk can hold rows past its end
                const bool valid = p0 + (it * U + u) * STEP < row_end;
                static_for<QUADS ? 1 : GT>([&](auto gg) {
                    constexpr int gi = decltype(gg)::value;
                    sc[u][gi] = valid ? sc[u][gi] : -INFINITY;
                });
            }
        });

        if constexpr (QUADS) {
            // (the reference point as below)
            float mx = sc[0][0];
            static_for<U>([&](auto uu) { mx = fmaxf(mx, sc[uu.value][0]); });
            const bool grow = mx > qm + kSlack;
            if (__builtin_amdgcn_ballot_w64(grow) != 0) {
                const float mn = grow ? mx : qm;
                const float f = exp2_fast(qm - mn);
                qm = mn;
                qsum *= f;
                static_for<GT>([&](auto gg) {
                    const float fh = quad_lane<gg.value>(f);
                    static_for<2 * P>([&](auto cc) { qacc[cc.value][gg.value] *= fh; });
                });
            }
            static_for<U>([&](auto uu) {
                constexpr int u = decltype(uu)::value;
                const float pw = exp2_fast(sc[u][0] - qm);
                qsum += pw;
                float va[P], vb2[P];
                unpack(r.vl[u], va);
                unpack(r.vh[u], vb2);
                static_for<P>([&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    qacc[j] = __builtin_amdgcn_mfma_f32_4x4x1f32(pw, va[j], qacc[j], 0, 0, 0);
                    qacc[P + j] = __builtin_amdgcn_mfma_f32_4x4x1f32(pw, vb2[j], qacc[P + j], 0, 0, 0);
                });
            });
            return;
        }

        static_for<QUADS ? 0 : GT>([&](auto gg) {
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
        if constexpr (!QUADS) issue(rb);
        consume(ra, it);
        if (EXACT && it + 1 >= nit) break;
        issue(ra);
        consume(rb, it + 1);
        if constexpr (QUADS) issue(rb);
    }

    // ---- combine the lane groups of the workgroup
    // 1. common maximum per query head: over the lane groups of a wave by lane swaps, over waves through LDS; then sums, and accumulators
    // rescaled.  (Four heads: still one to a lane of each quad, so once for all four.)
    // (the lane's index is counted again: kept across the loop with what derives from it, it would not fit the registers of the longest kernel)
    uint32_t none = 0;
    asm volatile("" : "+v"(none));
    const int ln = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, none)), tid_end = wave * 64 + ln;
    float scale[GT];
    if constexpr (QUADS) {
        const float mx = fold_from<LPR>(qm, Max{});
        if (ln < 4) xm[ln][wave] = mx;
        lds_barrier();
        const f32x4 of_waves = *(const f32x4*)xm[ln & 3];
        const float f = exp2_fast(qm - fmaxf(fmaxf(of_waves[0], of_waves[1]), fmaxf(of_waves[2], of_waves[3])));
        const float ls = fold_from<LPR>(qsum * f, Add{});
        if (ln < 4) xl[ln][wave] = ls;
        static_for<GT>([&](auto gg) { scale[gg.value] = quad_lane<gg.value>(f); });
    } else {
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
    // and park their sums in LDS.  (With the reference points and sums of four heads worked out at once, where every lane used to do all of
    // them and the swaps folded each value for both groups: 64 rows of 8 KV heads 6.4 -> 5.8 us, 300 9.0 -> 8.4, 6147 13.3 -> 13.0.)
    static_assert(P == 4);
    static_for<GT>([&](auto gg) {
        constexpr int gi = decltype(gg)::value;
        f32x4 sum;
        static_for<P>([&](auto jj) {
            constexpr int j = decltype(jj)::value;
            sum[j] = fold_two<LPR>((QUADS ? qacc[j][gi] : acc[gi][j]) * scale[gi], (QUADS ? qacc[P + j][gi] : acc[gi][P + j]) * scale[gi], ln);
        });
        *(f32x4*)(red + ((wave * (RPW / 2) + (ln / LPR >> 1)) * GT + gi) * D + (ln / LPR & 1) * (D / 2) + P * (ln % LPR)) = sum;
    });
    lds_barrier();

    // 2. sum over the parked lane groups; two channels of one query head per thread and pass
    auto group_ml = [&](int gi, float* M, float* L) {
        *M = xm[gi][0];
        *L = xl[gi][0];
        static_for<kWaves - 1>([&](auto w) { *M = fmaxf(*M, xm[gi][w.value + 1]); *L += xl[gi][w.value + 1]; });
    };
    const long long head0 = (long long)unit * g.G + g0;                        // dense query head of gi = 0
    const long long pidx = head0 * g.n_split + split;                          // + gi * n_split below
    for (int idx = tid_end; idx < GT * D / 2; idx += kWaves * 64) {
        const int gi = idx / (D / 2), ch = 2 * (idx - gi * (D / 2));
        f32x2 sum = {0.f, 0.f};
#pragma unroll
        for (int hs = 0; hs < HSLOTS; ++hs) sum += *(const f32x2*)(red + (hs * GT + gi) * D + ch);
        if constexpr (ONE) {
            float M, L;
            group_ml(gi, &M, &L);
            store2(out + (head0 + gi) * D + ch, sum[0] / L, sum[1] / L);
        } else {
            *(f32x2*)(part_acc + (pidx + (long long)gi * g.n_split) * D + ch) = sum;
        }
    }
    if (tid_end < GT) {
        float M, L;
        group_ml(tid_end, &M, &L);
        f32x2* ml = (f32x2*)(part_ml + (pidx + (long long)tid_end * g.n_split) * 2);
        if constexpr (ONE) {
            if (lse) lse[head0 + tid_end] = 0.6931471805599453f * (M + log2f(L));
        } else {
            *ml = f32x2{M, L};
        }
    }
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
    hipLaunchKernelGGL(k_rope_table, dim3((d / 2 + 63) / 64), dim3(64), 0, st, rt, d, base, step);
    return hipGetLastError();
}

template <typename T, int D, int GT, bool ONE, bool EXACT>
static void launch_partial_o(const SlabTable& tab, const AttGeom& g, const void* q, const RopeEntry* rt, float* part_acc,
                             float* part_ml, void* out, float* lse, hipStream_t st)
{
    const long long chunks = (long long)g.units * g.n_split, parts = g.G / g.GT;
    const dim3 grid = chunks * parts < 1 << 23 ? dim3((unsigned)(chunks * parts)) : dim3((unsigned)chunks, (unsigned)parts);   // (a launch has up to 2^32 threads per direction)
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

template <typename T, int D>
static hipError_t launch_partial_d(const SlabTable& tab, const AttGeom& g, const void* q, const RopeEntry* rt, float* part_acc,
                                   float* part_ml, void* out, float* lse, hipStream_t st)
{
    switch (g.GT) {
        case 4: launch_partial_g<T, D, 4>(tab, g, q, rt, part_acc, part_ml, out, lse, st); break;
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
