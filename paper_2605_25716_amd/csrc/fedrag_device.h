// Device-side helpers shared by the gfx950 kernels: storage-type traits, MFMA wrappers, wave helpers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// A kernel starts on a page.  What a short launch waits for first is its own instructions, which many megabytes of keys between two
// launches have pushed out of every cache, and where it lies in the code object decides how many such waits there are: each is
// 0.6 us, and with kernels packed closely a change in the size of any other kernel moved one or two of them into or out of a layer
// of seven launches (117 query rows over two contexts, 32 layers: 1.95 to 2.01 ms between builds of the same kernels).
#define FEDRAG_KERNEL __global__ __attribute__((aligned(4096)))

namespace fedrag {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// 16-bit storage types.  vec8 is the 16-byte MFMA operand (8 contraction elements per lane).
struct BF16 {
    typedef __bf16 elem;
    typedef bf16x8_t vec8;
    typedef bf16x4_t vec4;
    // D(16x16) += A(16x32) . B(32x16); lane l: A row l%16, B column l%16, contraction elements (l/16)*8..+8;
    // D column l%16, rows (l/16)*4..+4.
    static __device__ __forceinline__ f32x4_t mfma16(vec8 a, vec8 b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    // D(32x32) += A(32x16) . B(16x32); lane l: A row l%32, B column l%32, contraction elements (l/32)*8..+8;
    // D column l%32, rows 8*(r/4) + 4*(l/32) + r%4 for r in 0..15.
    static __device__ __forceinline__ f32x16_t mfma32(vec8 a, vec8 b, f32x16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ elem from_float(float x) { return static_cast<__bf16>(x); }
    static __device__ __forceinline__ float to_float(elem x) { return static_cast<float>(x); }
};

struct F16 {
    typedef _Float16 elem;
    typedef f16x8_t vec8;
    typedef f16x4_t vec4;
    static __device__ __forceinline__ f32x4_t mfma16(vec8 a, vec8 b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ f32x16_t mfma32(vec8 a, vec8 b, f32x16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ elem from_float(float x) { return static_cast<_Float16>(x); }
    static __device__ __forceinline__ float to_float(elem x) { return static_cast<float>(x); }
};

template <class V>
__device__ __forceinline__ V zero_vec() {
    V v;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(V) / sizeof(v[0])); ++i) v[i] = 0;
    return v;
}

// Lanes of one wave exchange data through LDS: order this wave's LDS writes before its later LDS reads.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// Max / sum over the lane pairs (l, l ^ 32) and (l, l ^ 16).  The lane-swap instructions exchange half waves (rows of
// 16) between two registers: given the same value twice they leave one register with the lower partner's value in
// both lanes and one with the upper's, without the trip through the LDS crossbar that a shuffle takes.
struct LanePair {
    float lower, upper;
};
__device__ __forceinline__ LanePair lane_pair32(float x) {
    const uint32_t v = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    const uint32_t a = r[0], b = r[1];
    return LanePair{__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)};
}
__device__ __forceinline__ LanePair lane_pair16(float x) {
    const uint32_t v = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const uint32_t a = r[0], b = r[1];
    return LanePair{__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)};
}
__device__ __forceinline__ float xor32_max(float x) { const LanePair p = lane_pair32(x); return fmaxf(p.lower, p.upper); }
__device__ __forceinline__ float xor32_sum(float x) { const LanePair p = lane_pair32(x); return p.lower + p.upper; }
__device__ __forceinline__ float xor16_max(float x) { const LanePair p = lane_pair16(x); return fmaxf(p.lower, p.upper); }
__device__ __forceinline__ float xor32_min(float x) { const LanePair p = lane_pair32(x); return fminf(p.lower, p.upper); }
__device__ __forceinline__ float xor16_min(float x) { const LanePair p = lane_pair16(x); return fminf(p.lower, p.upper); }
__device__ __forceinline__ float xor16_sum(float x) { const LanePair p = lane_pair16(x); return p.lower + p.upper; }

// min / max over aligned groups of N = 8 or 16 consecutive lanes, result in every lane of the group, with data-parallel
// primitives only (no LDS crossbar): exchange inside quads, then mirror the half row (lane k <-> 7 - k: the other
// quad, whose lanes already agree), then mirror the row of 16.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
template <int N, class Op>
__device__ __forceinline__ float group_reduce(float x, Op op) {
    static_assert(N == 8 || N == 16, "groups of 8 or 16 lanes");
    x = op(x, dpp_move<0xB1>(x));   // quad_perm [1,0,3,2]
    x = op(x, dpp_move<0x4E>(x));   // quad_perm [2,3,0,1]
    x = op(x, dpp_move<0x141>(x));  // row_half_mirror
    if (N == 16) x = op(x, dpp_move<0x140>(x));  // row_mirror
    return x;
}
template <int N>
__device__ __forceinline__ float group_max(float x) {
    return group_reduce<N>(x, [](float a, float b) { return fmaxf(a, b); });
}

// The same reduction of a minimum and a maximum at once, one instruction per step and value: the data-parallel move is
// folded into the minimum / maximum (the compiler emits a move, a canonicalising maximum and the operation itself).  A
// register has to be two instructions old before a data-parallel read, which the other value's step and a nop give it.
// One statement from the first step to the last, opened by that wait: the compiler may put a copy of either value before a
// statement and does not look inside it for the distance.
#define FEDRAG_MIN_MAX_STEP(lanes)                                       \
    "v_min_f32_dpp %0, %0, %0 " lanes " row_mask:0xf bank_mask:0xf\n\t" \
    "v_max_f32_dpp %1, %1, %1 " lanes " row_mask:0xf bank_mask:0xf\n\t"
#define FEDRAG_MIN_MAX_OF_8                                         \
    "s_nop 1\n\t" FEDRAG_MIN_MAX_STEP("quad_perm:[1,0,3,2]")        \
    "s_nop 0\n\t" FEDRAG_MIN_MAX_STEP("quad_perm:[2,3,0,1]")        \
    "s_nop 0\n\t" FEDRAG_MIN_MAX_STEP("row_half_mirror")
template <int N>
__device__ __forceinline__ void group_min_max(float& lo, float& hi) {
    static_assert(N == 8 || N == 16, "groups of 8 or 16 lanes");
    if constexpr (N == 8)
        asm(FEDRAG_MIN_MAX_OF_8 "s_nop 1" : "+v"(lo), "+v"(hi));
    else
        asm(FEDRAG_MIN_MAX_OF_8 "s_nop 0\n\t" FEDRAG_MIN_MAX_STEP("row_mirror") "s_nop 1" : "+v"(lo), "+v"(hi));
}
#undef FEDRAG_MIN_MAX_OF_8
#undef FEDRAG_MIN_MAX_STEP

// A code of the transport codec before its truncation: t clamped to [0, levels], NaN to 0 (the median of three with a NaN among
// them is the least of the others).
__device__ __forceinline__ float clamp_code(float t, float levels) { return __builtin_amdgcn_fmed3f(t, 0.0f, levels); }

// Sixteen values in [0, 256) truncated to bytes, value e in byte e % 4 of word e / 4, each conversion writing its byte.  The
// words take turns because a partly written register must not be written again by the next instruction.
__device__ __forceinline__ void bytes_of(const float (&t)[16], uint32_t (&w)[4]) {
    asm("v_cvt_u32_f32_sdwa %0, %4 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %1, %8 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %2, %12 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %3, %16 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %0, %5 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %1, %9 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %2, %13 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %3, %17 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %0, %6 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %1, %10 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %2, %14 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %3, %18 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %0, %7 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %1, %11 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %2, %15 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD\n\t"
        "v_cvt_u32_f32_sdwa %3, %19 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD\n\t"
        "s_nop 1"
        : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
        : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(t[5]), "v"(t[6]), "v"(t[7]), "v"(t[8]), "v"(t[9]),
          "v"(t[10]), "v"(t[11]), "v"(t[12]), "v"(t[13]), "v"(t[14]), "v"(t[15]));
}

// Keep a value's computation above this point: the compiler may otherwise sink pure register arithmetic towards
// its first use (past a barrier, into the next loop iteration), out of the scheduling region it was written for.
template <class V>
__device__ __forceinline__ void pin_here(V& v) {
    asm volatile("" : "+v"(v));
}

// Scalars (a kernel's arguments) that are all in registers from here on: asked for where the code happens to need them they are as
// many trips to memory, one after the other, as there are branches and address computations between, 0.2 us each in a launch
// whose caches are cold.
#define FEDRAG_S(x) "s"(x)
#define FEDRAG_S3(f) "s"((f).m), "s"((f).s), "s"((f).d)  // a FastDiv
#define FEDRAG_HAVE_HERE(...) asm volatile("" ::__VA_ARGS__)

// Transposing LDS read: within each group of 16 lanes, lane j receives element (j % 4) of the 8 bytes addressed
// by lane 4 e + j / 4, for e = 0..3.  With lane s of the group pointing at row (s / 4), columns 4 (s % 4)..+4 of
// a row-major 4 x 16 block, lane j gets column j of the block, rows 0..3.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2_t lds_read_tr16(const char* p) {
    const s16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3)))*)p);
    return __builtin_bit_cast(u32x2_t, v);
}

// exp2(a - b) with the convention that a == -inf gives 0 even when b == -inf.
__device__ __forceinline__ float exp2_diff(float a, float b) {
    return (a == -INFINITY) ? 0.0f : fast_exp2(a - b);
}

// 8x8 transpose of 16-bit elements held as 8 registers-of-8 (in[r][c] -> out[c][r]).
// Each 32-bit word holds two adjacent columns; v_perm_b32 picks halves of two words.
__device__ __forceinline__ void transpose8x8_b16(const u32x4_t in[8], u32x4_t out[8]) {
#pragma unroll
    for (int c2 = 0; c2 < 4; ++c2) {          // word index along the input row = column pair (2*c2, 2*c2+1)
#pragma unroll
        for (int r2 = 0; r2 < 4; ++r2) {      // input row pair (2*r2, 2*r2+1)
            const uint32_t a = in[2 * r2][c2];      // row 2r2   : cols 2c2 (lo), 2c2+1 (hi)
            const uint32_t b = in[2 * r2 + 1][c2];  // row 2r2+1 : same columns
            // out row (=in col) 2c2   : word r2 = { in[2r2][2c2]   (lo), in[2r2+1][2c2]   (hi) }
            // out row          2c2+1 : word r2 = { in[2r2][2c2+1] (lo), in[2r2+1][2c2+1] (hi) }
            out[2 * c2][r2] = __builtin_amdgcn_perm(b, a, 0x05040100u);
            out[2 * c2 + 1][r2] = __builtin_amdgcn_perm(b, a, 0x07060302u);
        }
    }
}

}  // namespace fedrag
