// Shared by the two kernels of the near/far form (freqkv_nearfar.hip, freqkv_nearfar_units.hip): sizes, the interpolation, and
// what their waves do between LDS and the matrix cores.
#pragma once
#include "freqkv_internal.h"

namespace freqkv {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

template <int I> struct IC { static constexpr int value = I; };
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (I < N) {
        f(IC<I>{});
        static_for<N, I + 1>(f);
    }
}

// f(IC<i>) for a uniform i in [0, N).  The cases end in different (empty) assembly: merged into one, what they do to the elements of
// an array would keep that array in scratch memory.
template <int N, class F>
__device__ __forceinline__ void dispatch(int i, F&& f)
{
    static_for<N>([&](auto c) {
        if (i == c.value) {
            f(c);
            asm volatile("; %0" :: "n"(c.value));
        }
    });
}

constexpr int kC = 32;                    // channels per workgroup
constexpr int kRowB = kC * 2;             // bytes of one row in a ring slot
constexpr int kLeaf = 128;                // span rows per leaf
constexpr int kSlotB = kLeaf * kRowB;     // bytes of one ring slot
constexpr int kVecB = kC * 8 * 2;         // bytes of 8 moments (or local values) of 32 channels, [channel][8] bf16
constexpr int kFrag = 1024;               // one operand fragment: 64 lanes x 8 bf16
constexpr int kCompute = 4, kMovers = 4;  // waves
constexpr int kNB = 3;                    // blocks of a group's neighbourhood: 512 rows or less, 128 to spare on both sides
constexpr int kWin = kNB + 2;             // blocks whose moments are back in LDS where they go through memory: a group's and those ahead
constexpr int kHeld = 4;                  // blocks that the movers keep in registers
constexpr int kTabFrags = 6;              // table fragments kept in LDS
constexpr int kLdsBytes = 160 * 1024;

// ---- tables
// Chebyshev points of the first kind on [-1, 1] and the Lagrange polynomials on them.
__device__ double cheb(int s) { return cospi((2 * s + 1) / 16.0); }
__device__ double lagrange(int s, double u)
{
    double p = 1.0;
    const double xs = cheb(s);
    for (int q = 0; q < 8; ++q)
        if (q != s) p *= (u - cheb(q)) / (xs - cheb(q));
    return p;
}
// E of the header comment at the angle pi q / (2 n Lc); its limit at zero is 2 Lc.
__device__ double entry(long long q, long long n, long long Lc)
{
    if (q == 0) return 2.0 * (double)Lc;
    const double t = (double)q / (double)(4 * n * Lc);
    return sinpi((double)(q % (4 * n)) / (double)(2 * n)) * cospi(t) / sinpi(t);
}
// Intervals in span rows.
struct Iv {
    double c, h;             // centre, half width; h <= 0: nothing in it
    __device__ double node(int s) const { return c + h * cheb(s); }
};

// What a bf16 holds of x; the rest, rounded in its turn, is its second part.
__device__ double first_part(double x) { return (double)(float)(__bf16)(float)x; }

// ---- kernels
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A uniform x no smaller than lo and no larger than hi, in scalar registers (left alone the compiler takes v_med3 and moves it back).
__device__ __forceinline__ int between(int x, int lo, int hi)
{
    int y = max(__builtin_amdgcn_readfirstlane(x), lo);
    asm("" : "+s"(y));
    return min(y, hi);
}

// Waits until all but the newest `leaves` leaf copies of this wave (2 instructions each) have landed.  The count is an immediate, so this
// jumps to one of 32 waits: found by halves, the branches took a mover some 300 cycles of each step.
__device__ __forceinline__ void wait_copies(int leaves)
{
    // (the jump's base is the instruction behind s_getpc, the table 6 instructions of 4 bytes further on, 8 bytes to an entry)
    leaves = between(leaves, 0, 31);
    asm volatile("s_getpc_b64 s[90:91]\n\t"
                 "s_lshl_b32 s92, %0, 3\n\t"
                 "s_add_u32 s90, s90, s92\n\t"
                 "s_addc_u32 s91, s91, 0\n\t"
                 "s_add_u32 s90, s90, 24\n\t"
                 "s_addc_u32 s91, s91, 0\n\t"
                 "s_setpc_b64 s[90:91]\n\t"
                 ".set nf_wait_n, 0\n\t"
                 ".rept 32\n\t"
                 "s_waitcnt vmcnt(nf_wait_n)\n\t"
                 "s_branch .Lnf_waited_%=\n\t"
                 ".set nf_wait_n, nf_wait_n + 2\n\t"
                 ".endr\n"
                 ".Lnf_waited_%=:"
                 :: "s"(leaves) : "s90", "s91", "s92", "scc", "memory");
}

// A load that only some passes through a loop issue is awaited where it is issued: otherwise the compiler has to expect it in
// flight at every use, and waits there for whatever is really in flight, copies and stores.
__device__ __forceinline__ void pin(bf16x8& v) { asm volatile("" : "+v"(v)); }

// Waits for all loads and stores of the wave, in a form that the compiler takes into account (0: the vector memory counter).  Where
// paths meet it has to expect what any of them has in flight, and would wait for it again and again further on.
__device__ __forceinline__ void settle_memory() { __builtin_amdgcn_s_waitcnt(0x0f70); }

typedef __attribute__((address_space(3))) s16x4* lds_s16x4;

// Four consecutive rows of 16 columns, transposed: lane i of 16 gets column i.  Each lane names the 8 bytes
// (row lane/4, columns 4 (lane%4) ..) that it fetches.
__device__ __forceinline__ s16x4 read_tr(const char* p) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)p); }

__device__ __forceinline__ bf16x8 join(s16x4 a, s16x4 b)
{
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ u32x2 pack4(f32x4 a) { return u32x2{pack2(a[0], a[1]), pack2(a[2], a[3])}; }
// The same with what each rounding leaves passed on to the next: the sum keeps its precision.
__device__ __forceinline__ u32x2 pack4_carry(f32x4 a)
{
    uint32_t q[4];
    float left = 0.f;
    static_for<4>([&](auto i) {
        const float x = a[i.value] + left;
        q[i.value] = __builtin_bit_cast(uint16_t, (__bf16)x);
        left = x - __uint_as_float(q[i.value] << 16);
    });
    return u32x2{q[0] | q[1] << 16, q[2] | q[3] << 16};
}
// What rounding to `first` left of a.
__device__ __forceinline__ f32x4 rest(f32x4 a, u32x2 first)
{
    static_for<4>([&](auto i) {
        a[i.value] -= __uint_as_float(i.value & 1 ? first[i.value / 2] & 0xffff0000u : first[i.value / 2] << 16);
    });
    return a;
}

}  // namespace

}  // namespace freqkv
