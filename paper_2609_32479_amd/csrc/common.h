// Device-side building blocks shared by the library's kernels (gfx950):
// operand types, matrix-core fragments, wave and workgroup synchronisation,
// lane masks of the segmented scans, the tile's hit-slot order, the packing
// of tracks into wave tiles, and the direct-to-LDS weight-stage copy.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(8))) float f32x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

// Matrix-core operand types.  OP_F32: fp32 weights and operands, each the exact
// sum of three bf16 parts (see Frag<OP_F32>).  OP_BF16: bf16 weights and bf16 activation
// operands (v_mfma_f32_32x32x16_bf16).  OP_F16: weights converted to fp16
// (exact for bf16 values in the fp16 normal range) and fp16 activation
// operands (v_mfma_f32_32x32x16_f16).  OP_F32W: fp32 as OP_F32, the same stored weights,
// multiplied by the fp32 instruction (see Frag<OP_F32W>).
// Accumulation is fp32 in all four.
enum { OP_F32 = 0, OP_BF16 = 1, OP_F16 = 2, OP_F32W = 3 };
constexpr bool is_half(int op) { return op == OP_BF16 || op == OP_F16; }

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kRmsEps = 1e-6f;
// The fp32 gate clamps |pre-activation| to 80 and the 16-bit head clamps the
// SiLU exponent to 80 log2(e), so that exp stays finite; the change in the
// result is below exp(-80).
constexpr float kGateClamp = 80.0f * kLog2e;
constexpr int kLdsBytesMax = 160 * 1024;
constexpr int kCopyBytes = 1024;  // one wave-wide 16-byte-per-lane copy

constexpr int cmax(int a, int b) { return a > b ? a : b; }
constexpr int round_up(int v, int m) { return (v + m - 1) / m * m; }

template <int OP> struct Frag;
template <> struct Frag<OP_BF16> {
    typedef bf16x8 T;
    typedef __bf16 E;
    static __device__ __forceinline__ f32x16 mma(T a, T b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ void mma(T a, T b, f32x16 &c, f32x16 &) { c = mma(a, b, c); }
    static __device__ __forceinline__ f32x4 mma16(T a, T b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ T pack(const float *v) {
        f32x8 f = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
        return __builtin_convertvector(f, bf16x8);
    }
};
template <> struct Frag<OP_F16> {
    typedef f16x8 T;
    typedef _Float16 E;
    static __device__ __forceinline__ f32x16 mma(T a, T b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ void mma(T a, T b, f32x16 &c, f32x16 &) { c = mma(a, b, c); }
    static __device__ __forceinline__ f32x4 mma16(T a, T b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ T pack(const float *v) {
        f32x8 f = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
        return __builtin_convertvector(f, f16x8);
    }
};
// fp32 operands on the bf16 matrix cores (the splitting into exact parts that
// extended-precision sums use).  An fp32 value of magnitude 2^-110 or more is exactly
// h + m + l, three bf16 values of 8 significant bits each, h and m rounded, so that |m|
// is at most 2^-8 and |l| 2^-17 of a significand (below 2^-110 l, and then m, lose bits
// that are below bf16's smallest subnormal: at most 2^-134).  A product is taken as its
// six largest part products; of the three left out, m l and l m are together at most
// 2^-24 of the product, l l far below.
// The matrix cores cut a sum off where they add a product to it (a lone product
// added to its own small parts is up to 2 units of 2^-24 off, the fp32 instruction 1), so
// the products h h have a sum of their own, in which few terms are exact, the small ones
// another, and one fp32 addition rounds the two: a row of one term is 0.435 units off in
// the root mean square (fp32 instruction 0.424) and at most 2 (1), of two terms 0.37
// (0.43), of eight 0.25 (0.46), of 128 0.15 (0.47).  In one sum and with h cut off a
// row of one term was 0.69 off and up to 4.2, of eight terms 0.95.  Two-norm errors
// against 64 bits: 65 536 tracks, four layers of 128: 1.9e-7 (one sum 2.9e-7); the
// minGRU of 40 000: 1.5e-7 (3.2e-7).
// Cycles of 16 terms: 192 against 512 of the fp32 instruction.  65 536 tracks through
// the d = 128 encoder take 2.87 ms, 40 000 through the minGRU 3.06 (one sum 2.71 and 2.96,
// the fp32 instruction 5.49 and 6.77).  All eight products above 2^-30, with parts cut
// off: 0.424 units for one term, but 3.60 and 3.81 ms.
struct bf16x8x3 {
    bf16x8 h, m, l;
};
template <> struct Frag<OP_F32> {
    typedef bf16x8x3 T;
    typedef float E;
    // (named by the pipelined layers, which no fp32 kernel has)
    static __device__ f32x16 mma(const T &a, const T &b, f32x16 c);
    // c += the large products, s += the small ones
    static __device__ __forceinline__ void mma(const T &a, const T &b, f32x16 &c, f32x16 &s) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.l, b.h, s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.l, s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.m, s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.h, s, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.h, c, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.m, s, 0, 0, 0);
    }
    // The same with the small products in two sums, which take turns: for a wave that
    // has the SIMD to itself, whose dependent products run at 44 cycles each instead of
    // 32.
    static __device__ __forceinline__ void mma(const T &a, const T &b, f32x16 &c, f32x16 &s, f32x16 &t) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.l, b.h, s, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.l, t, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.m, s, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.h, t, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.m, s, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.h, c, 0, 0, 0);
    }
    static __device__ __forceinline__ T pack(const float *v) {
        typedef float f2 __attribute__((ext_vector_type(2)));
        typedef __bf16 b2 __attribute__((ext_vector_type(2)));
        u32x4 h, m, l;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f2 x = {v[2 * i], v[2 * i + 1]};
            const unsigned hb = __builtin_bit_cast(unsigned, __builtin_convertvector(x, b2));
            const f2 r = {x[0] - __uint_as_float(hb << 16), x[1] - __uint_as_float(hb & 0xffff0000u)};
            const unsigned mb = __builtin_bit_cast(unsigned, __builtin_convertvector(r, b2));
            const float s0 = r[0] - __uint_as_float(mb << 16), s1 = r[1] - __uint_as_float(mb & 0xffff0000u);
            h[i] = hb;
            m[i] = mb;
            l[i] = __builtin_amdgcn_perm(__float_as_uint(s1), __float_as_uint(s0), 0x07060302u);
        }
        return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
    }
};
// fp32 operands that may be infinite, or so large that part products overflow: h m and
// h l of an infinite h are infinite or NaN where the product is neither, and parts of
// different signs overflow to different infinities.  They are put together again and
// multiplied by the fp32 instruction (eight of depth 2, 512 cycles for 16 terms).
// It runs where weights or operands are beyond the limits here, below which no sum of
// up to 384 products can overflow: a handle with such weights takes it throughout, and
// the places that see operands without a bound (the minGRU's input rows, the head's
// pooled and hidden values) look for them, a comparison per eight values.  The
// normalised stream is at most sqrt(d), the states then stay below 2^61 with weights and
// biases below the limits, and sines and cosines are at most 1.
constexpr float kWideWeight = 0x1p27f, kWideBias = 0x1p60f, kWideOperand = 0x1p90f;
template <> struct Frag<OP_F32W> {
    typedef bf16x8x3 T;
    typedef float E;
    static __device__ __forceinline__ float value(const T &x, int e) {
        return ((float)x.l[e] + (float)x.m[e]) + (float)x.h[e];
    }
    static __device__ __forceinline__ f32x16 mma(const T &a, const T &b, f32x16 c) {
#pragma unroll
        for (int e = 0; e < 8; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(value(a, e), value(b, e), c, 0, 0, 0);
        return c;
    }
    static __device__ __forceinline__ void mma(const T &a, const T &b, f32x16 &c, f32x16 &) { c = mma(a, b, c); }
    // (h cut off, so that no finite value becomes infinite; no further parts of infinity)
    static __device__ __forceinline__ T pack(const float *v) {
        T x;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float h = __uint_as_float(__float_as_uint(v[e]) & 0xffff0000u);
            const float r = fabsf(v[e]) == __builtin_inff() ? 0.0f : v[e] - h;
            const float m = __uint_as_float(__float_as_uint(r) & 0xffff0000u);
            x.h[e] = (__bf16)h;
            x.m[e] = (__bf16)m;
            x.l[e] = (__bf16)(r - m);
        }
        return x;
    }
};
// The larger of m and the eight values' magnitudes (NaN, which stays NaN in the part
// products, does not count).
__device__ __forceinline__ float max_abs(float m, const float *v) {
#pragma unroll
    for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(v[e]));
    return m;
}
// The operand's columns or rows (bit i: lanes i and i + 32) that hold a magnitude beyond
// kWideOperand.
__device__ __forceinline__ unsigned wide_mask(float magnitude) {
    const unsigned long long w = __ballot(magnitude >= kWideOperand);
    return unsigned(w) | unsigned(w >> 32);
}
// The operand of this lane's values for the fp32 instruction if its column or row is
// wide, and for the part products if not; 0 for the other, which then adds nothing (the
// weights are finite): a track's bits do not depend on what else lies in its tile.
__device__ __forceinline__ bf16x8x3 take_wide(float *v, bool wide) {
    float w[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        w[e] = wide ? v[e] : 0.0f;
        v[e] = wide ? 0.0f : v[e];
    }
    return Frag<OP_F32W>::pack(w);
}
// On the host: whether any of n weights (or biases) is beyond the limit.
inline bool any_beyond(const float *w, size_t n, float limit) {
    bool any = false;
    for (size_t i = 0; i < n; ++i) any |= !(__builtin_fabsf(w[i]) < limit);  // (no early exit: vectorised)
    return any;
}
// The split of OP_F32 on the host (the weights): the parts' bf16 bits.  From 2^127 on h is
// cut off (rounded it might be infinite); infinity and NaN have no further parts.
struct Bf16Parts {
    uint16_t part[3];
};
inline Bf16Parts bf16_parts(float v) {
    auto bits = [](float x) {
        uint32_t u;
        __builtin_memcpy(&u, &x, 4);
        return u;
    };
    auto value = [](uint32_t u) {
        float x;
        __builtin_memcpy(&x, &u, 4);
        return x;
    };
    // to the nearest bf16, ties to even
    auto near = [](uint32_t u) { return (u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u; };
    uint32_t h = near(bits(v));
    if (!(__builtin_fabsf(v) < 0x1p127f)) {
        if (v != v) return {{0x7fc0, 0, 0}};
        h = bits(v) & 0xffff0000u;
        if (__builtin_isinf(v)) return {{uint16_t(h >> 16), 0, 0}};
    }
    const float r = v - value(h);
    const uint32_t m = near(bits(r));
    return {{uint16_t(h >> 16), uint16_t(m >> 16), uint16_t(bits(r - value(m)) >> 16)}};
}

// exp(x) for |x| <= 80 in fp32: x log2(e) = p + l with the product's and log2(e)'s
// rounding errors in l, p = n + (p - n) with n the nearest whole number (in the low bits
// of q), the hardware's exp2 of (p - n) + l, and n added to the exponent bits.
// 1 / d for 1 <= d <= 2^126: the hardware's reciprocal (1 ulp) and one Newton step, whose
// last operation rounds a value right to 2^-45: the correctly rounded quotient.
// Against 64 bits over |x| <= 80 (4 M arguments) exp is 0.83 ulp off at most and 0.30 in
// the root mean square, the library's figures to the last digit (with exp2 of the
// unreduced product 1.23 and 0.41); of 4 M quotients 1 / (1 + e) none differs from the
// division's.  9 and 3 instructions; the library's forms also cover ranges that a
// clamped argument cannot reach and take about 14 and 11.
__device__ __forceinline__ float exp_clamped(float x) {
#pragma clang fp contract(off)  // (p is the rounded product everywhere)
    constexpr float kLog2eLo = float(1.4426950408889634 - double(kLog2e)), kRound = 0x1.8p23f;
    const float q = fmaf(x, kLog2e, kRound), p = x * kLog2e;
    const float f = (p - (q - kRound)) + fmaf(x, kLog2eLo, fmaf(x, kLog2e, -p));
    return __uint_as_float(__float_as_uint(__builtin_amdgcn_exp2f(f)) + (__float_as_uint(q) << 23));
}
__device__ __forceinline__ float rcp_clamped(float d) {
    const float r = __builtin_amdgcn_rcpf(d);
    return fmaf(fmaf(-d, r, 1.0f), r, r);
}
// v sigmoid(v) = v / (1 + exp(-v)), the exponent clamped (the change is below exp(-80)
// |v|), the quotient with a residual step, which rounds it as the division would (an
// infinite quotient has none).
__device__ __forceinline__ float silu_f32(float v) {
    const float d = 1.0f + exp_clamped(-__builtin_amdgcn_fmed3f(v, -80.0f, 80.0f)), r = rcp_clamped(d);
    const float q = v * r;
    return fabsf(q) < __builtin_inff() ? fmaf(fmaf(-d, q, v), r, q) : q;
}

// N products in a row whose weight fragments come from LDS: step(i, fragment i) for i in
// order, with the fragments of the next DEPTH - 1 steps always on their way (load(i)
// reads one).  The fences keep that order: left to itself the compiler reads two
// fragments, waits for both (an LDS read under load takes longer than two products)
// and only then issues their products.  d = 256, six layers, 262 144 tracks: 18.2 ->
// 17.2 ms with three; d = 128, 500 tracks: 39.2 -> 37.6 us with four.  DEPTH 0: left to
// the compiler (for kernels that have no registers for it).
template <int N, int DEPTH, class Load, class Step>
__device__ __forceinline__ void ring_products(Load load, Step step) {
    if constexpr (DEPTH == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) step(i, load(i));
    } else {
        decltype(load(0)) w[DEPTH];
#pragma unroll
        for (int i = 0; i < DEPTH; ++i)
            if (i < N) w[i] = load(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            step(i, w[i % DEPTH]);
            if (i + DEPTH < N) w[i % DEPTH] = load(i + DEPTH);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The lane index, read afresh: values derived from it are formed where they
// are used instead of being held in registers across the whole kernel.
__device__ __forceinline__ int fresh_lane() {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Lane mask (wave-uniform, 64 bits) of the lanes whose stream has bit p set:
// lanes 0-31 follow b0, lanes 32-63 follow b1.
__device__ __forceinline__ unsigned long long half_mask(unsigned b0, unsigned b1, int p) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 m = {(unsigned)((int)(b0 << (31 - p)) >> 31), (unsigned)((int)(b1 << (31 - p)) >> 31)};
    return __builtin_bit_cast(unsigned long long, m);
}

// v in lanes outside m, 0 in lanes of m: one v_cndmask with the mask in SGPRs.
__device__ __forceinline__ float zero_lanes(float v, unsigned long long m) {
    float r;
    asm("v_cndmask_b32_e64 %0, %1, 0, %2" : "=v"(r) : "v"(v), "s"(m));
    return r;
}

// Tile hit index held in hit slot s (0 <= s < CAP).  Slot s = 32 n + 8 i + 4 g + j
// is row 8 i + 4 g + j of hit tile n in the input projection; that row lands
// in lanes of half g at accumulator register 4 i + j, which is position
// 16 n + 4 i + j of stream g, i.e. tile hit SP * g + 16 n + 4 i + j.
template <int SP>
__device__ __forceinline__ int slot_to_hit(int s) {
    int n = s >> 5, i = (s >> 3) & 3, g = (s >> 2) & 1, j = s & 3;
    return SP * g + 16 * n + 4 * i + j;
}

// Folded slot order of the encoder: stream 0 (lanes 0-31) holds tile rows
// 0 .. SP-1 in register order, stream 1 (lanes 32-63) holds rows 2 SP-1 down to
// SP, i.e. register position p of stream 1 is row 2 SP - 1 - p.  An ascending
// pass over the registers then runs stream 0 forward and stream 1 in reverse,
// and a descending pass the other two directions; both meet at rows SP - 1 and
// SP, so one lane swap carries a track across the streams.
template <int SP>
__device__ __forceinline__ int slot_to_row(int s) {
    const int n = s >> 5, i = (s >> 3) & 3, g = (s >> 2) & 1, j = s & 3;
    const int p = 16 * n + 4 * i + j;
    return g ? 2 * SP - 1 - p : p;
}

// The SP row bits of stream 1 (rows SP .. 2 SP - 1 of a row mask) in register
// order: bit p is row 2 SP - 1 - p.
template <int SP>
__device__ __forceinline__ unsigned stream1_bits(unsigned long long rows) {
    const unsigned hi = unsigned(rows >> SP) & (SP >= 32 ? 0xffffffffu : ((1u << SP) - 1u));
    return __builtin_bitreverse32(hi) >> (32 - SP);
}

// Copy of one weight stage from global memory straight into an LDS slot:
// global_load_lds_dwordx4 moves 16 bytes per lane, 1 KiB per wave
// instruction, into LDS at M0 + 16 * lane.  Each wave copies the pieces
// w, w + WAVES, ...; waves with fewer pieces repeat the last one (same bytes to
// the same place), so every wave issues exactly LPW loads per stage and can
// wait for an older stage with a constant vmcnt.  The instruction is written
// out because the compiler, which cannot tell the ring slots apart, would
// otherwise wait for every such load before each LDS access; the kernel keeps
// the count itself (wait_vmcnt).  The LDS address is an operand bound to M0,
// so the compiler writes M0 itself and knows it is read here; the s_nop is
// the one wait state the hardware needs between that write and the load.
__device__ __forceinline__ void lds_dma16(const void *gsrc, unsigned lds_addr) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :
                 : "v"(gsrc), "{m0}"(__builtin_amdgcn_readfirstlane(lds_addr))
                 : "memory");
}

// slot_lds: LDS byte address of the slot.
template <class C>
__device__ __forceinline__ void copy_stage(const unsigned char *stages, int s, unsigned slot_lds, int wid, int lane) {
    const unsigned char *src = stages + (size_t)s * C::STAGE + lane * 16;
#pragma unroll
    for (int i = 0; i < C::LPW; ++i) {
        int piece = wid + i * C::WAVES;
        piece = piece < C::COPIES ? piece : C::COPIES - 1;
        lds_dma16(src + piece * kCopyBytes, slot_lds + piece * kCopyBytes);
    }
}

// The tracks that a few waves of a workgroup still have to fit between them: the
// first not yet in a tile (t), the end of their range, and for the 64 tracks
// from t on the ones already in a tile or refused (bit i of taken: track t + i).
// Each of those waves keeps the same copy in scalar registers.
struct TrackPool {
    int t, end;
    unsigned long long taken;
    // past the leading tracks that are done
    __device__ __forceinline__ void slide() {
        const int sh = taken == ~0ull ? 64 : __builtin_ctzll(~taken);
        taken = sh == 64 ? 0ull : taken >> sh;
        t += sh;
    }
};

// The offsets of the pool's next window, straight into LDS (win_lds: byte address
// of 2 x 64 ints): track t + lane's, then the one after it.  One wave's job, after
// the barrier that follows a round's packing; in place at the next barrier that
// this wave passes with its loads complete.  (Read by every wave at the start of a
// round they cost it the latency of a first touch.)
constexpr int kWindowBytes = 2 * 64 * 4;
__device__ __forceinline__ void lds_dma4(const void *gsrc, unsigned lds_addr) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dword %0, off"
                 :
                 : "v"(gsrc), "{m0}"(__builtin_amdgcn_readfirstlane(lds_addr))
                 : "memory");
}
__device__ __forceinline__ void prefetch_window(const int *__restrict__ offsets, TrackPool p, unsigned win_lds,
                                                int lane) {
    p.slide();
    const int idx = p.t + lane;
    lds_dma4(offsets + (idx < p.end ? idx : p.end), win_lds);
    lds_dma4(offsets + (idx + 1 < p.end ? idx + 1 : p.end), win_lds + 256);
}

// One tile per wave for TILES waves, from the pool they share.  Each of them runs
// the same packing of all TILES tiles over the same offsets and keeps tile `me`, so
// they agree on the pool's next state without any exchange.  A tile takes the
// oldest track left, then, until it is full: a track that fills its CAP rows
// exactly, else the first that leaves room for the shortest track of the window,
// else the first that fits; up to MAXTR tracks.
// A track's result does not depend on the tile it lands in, so the packing only
// decides how full the tiles are and how many the slowest wave takes.  Each wave
// packing a range of its own first-fit gave, with lengths 8..20 and 262 144
// tracks on 256 workgroups of 12 waves, 41.4 tiles per wave on average but 46 for
// the slowest wave of the launch; the exact fits and pools of 4 waves give 38.6
// and 41.  (Pools of all 12 give 38.3 and 39, but a step of the packing, about 25
// dependent instructions, takes a wave some 300 cycles, and each wave runs the
// steps of its whole pool: they made a round of 12 tiles 2.3 us longer.)
// win: the offsets of the first window (prefetch_window); later ones of the same
// round are read from memory.
// Tracks that cannot be fitted (rows outside [lo, hi), an end before the
// start, no hits, more than CAP) are handed to refuse(bad, empty, too_long: lane
// masks, track index of this lane).  Tile me's track table goes to tab (first
// tile row, length, first hit row, track index: MAXTR ints each), its track count
// to k, its rows to n and the mask of its rows that start a track to smask.
// Returns the number of tiles formed, the same in every wave (0: the pool is empty).
template <int CAP, int MAXTR, int TILES, class Refuse>
__device__ __forceinline__ int pool_pack(const int *__restrict__ offsets, const int *win, TrackPool &p, long long lo,
                                         long long hi, int me, int lane, int *tab, int &k, int &n,
                                         unsigned long long &smask, Refuse refuse) {
    static_assert(CAP <= 64 && MAXTR <= 255, "tile shape");
    typedef unsigned long long u64;
    int my_pos = 0, tiles = 0;  // my_pos: rows + 256 tracks of tile me
    u64 my_rows = 0;
    bool first = true;
    for (;;) {
        // the oldest track left goes into the next tile, so every turn moves on
        p.slide();
        if (tiles >= TILES || p.t >= p.end) break;
        const int idx = p.t + lane;
        const bool in = idx < p.end;
        int off = 0, nxt = 0;
        if (first) {
            off = win[lane];
            nxt = win[64 + lane];
        } else if (in) {
            off = offsets[idx];
            nxt = offsets[idx + 1];
        }
        first = false;
        const u64 fresh = __ballot(in) & ~p.taken;
        const bool bad = nxt < off || (long long)off < lo || (long long)nxt > hi;
        const int len = bad ? -1 : nxt - off;
        u64 av = fresh & __ballot(len > 0 && len <= CAP);
        const u64 refused = fresh & ~av;
        if (refused) {
            const u64 bad_m = refused & __ballot(bad), empty_m = refused & __ballot(len == 0);
            refuse(bad_m, empty_m, refused & ~bad_m & ~empty_m, idx);
            p.taken |= refused;
        }
        if (!av) continue;
        // shortest track of the window: the lowest length bit by bit
        int mn = 0;
#pragma unroll
        for (int b = CAP; b; b >>= 1) mn += (av & __ballot(len < mn + b)) ? 0 : b;
        const bool more = p.end - p.t > 64;
        int place = 0;   // this lane's tile row + 256 x its place in the tile
        u64 my_sel = 0;  // lanes of tile me
        do {
            int room = CAP, pos = 0;
            u64 rows = 0, m = av;
            const u64 before = av;
            do {
                const int i = __builtin_ctzll(m);
                const int li = __builtin_amdgcn_readlane(len, i);
                asm("s_bitset0_b64 %0, %1" : "+s"(av) : "s"(i));
                asm("s_bitset1_b64 %0, %1" : "+s"(rows) : "s"(pos));  // (bit pos % 64: the tile row)
                place = lane == i ? pos : place;
                room -= li;
                pos += li + 256;
                const u64 m1 = av & __ballot(len == room), m2 = av & __ballot(len <= room - mn),
                          m3 = av & __ballot(len <= room);
                m = m1 ? m1 : m2 ? m2 : m3;
            } while (m && pos < 256 * MAXTR);
            const u64 sel = before & ~av;
            p.taken |= sel;
            if (tiles == me) {
                my_sel = sel;
                my_rows = rows;
                my_pos = pos;
            }
            ++tiles;
            // (few candidates left make poor tiles: read on, if there are more)
        } while (tiles < TILES && av && !(more && __builtin_popcountll(av) < 24));
        if ((my_sel >> lane) & 1ull) {
            int *e = tab + (place >> 8);
            e[0] = place & 255;
            e[MAXTR] = len;
            e[2 * MAXTR] = off;
            e[3 * MAXTR] = idx;
        }
    }
    // (uniform already, but not for the compiler)
    k = uniform(my_pos >> 8);
    n = uniform(my_pos & 255);
    smask = (u64)(unsigned)uniform(int(unsigned(my_rows))) |
            ((u64)(unsigned)uniform(int(unsigned(my_rows >> 32))) << 32);
    return uniform(tiles);
}

// First track of group g of ng: the tracks are split into ng contiguous groups
// (one per workgroup) of about equal hit rows.  The result is the number of tracks i with
// offsets[i] < offsets[0] + R g / ng (R: the rows of all tracks), found by a
// 64-ary search that follows the leading run of true probes; that count grows
// with the target for any offsets array, so the groups of consecutive g tile
// [0, n_tracks) even when the offsets are invalid.  Without rows (R <= 0) the
// split is by track count.  Wave-uniform.
__device__ __forceinline__ int group_begin(const int *__restrict__ offsets, int n_tracks, long long g, long long ng,
                                           int lane) {
    if (g <= 0) return 0;
    if (g >= ng) return n_tracks;
    const long long o0 = offsets[0];
    const long long rows = (long long)offsets[n_tracks] - o0;
    if (rows <= 0) return int((long long)n_tracks * g / ng);
    const long long target = o0 + rows * g / ng;
    int lo = 0, hi = n_tracks;  // the count lies in [lo, hi]
    while (hi > lo) {
        const int stride = (hi - lo + 63) / 64;
        const int p = lo + (lane + 1) * stride - 1;  // probes below hi
        const bool below = p < hi && (long long)offsets[p] < target;
        const unsigned long long nb = ~__ballot(below);
        const int c = nb ? __builtin_ctzll(nb) : 64;  // leading true probes
        const int nlo = lo + c * stride;
        const int phi = lo + (c + 1) * stride - 1;  // the first false probe, if any
        hi = phi < hi ? phi : hi;
        lo = nlo < hi ? nlo : hi;
    }
    return lo;
}

// Workgroups of a launch: one per compute unit (the LDS ring and the register
// file are sized for it), and no more than tracks.  group_begin spreads the
// rows over all of them, so a small call takes few tiles on many units instead of
// several in a row on a few.  A tile's walk through the layers is what a small
// call costs: with at least 8 tracks per wave (6 workgroups for 500 tracks) the
// four-layer d = 128 encoder took 243 us for 500 tracks, spread over the chip
// 39 us; from about 20 000 tracks on both rules fill the chip.  Calls on several streams
// then take turns instead of sharing the chip, which costs less than it gains: 3 072
// tracks 290 -> 58 us a call on one stream, on four streams 145 -> 55 us a call (500
// tracks 123 -> 36, 14 000 207 -> 168; the backbone and the fp32 and 64-hit encoders alike).
inline unsigned workgroups(int n_tracks, int cu_count) {
    return (unsigned)(n_tracks < cu_count ? (n_tracks < 1 ? 1 : n_tracks) : cu_count);
}

// Workgroup barrier that orders LDS only (the kernel shares nothing through
// global memory within a workgroup).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// s_waitcnt vmcnt(N) with the other counters left alone (gfx9 encoding).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

}  // namespace
