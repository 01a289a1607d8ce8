// Device-side helpers shared by the gfx950 kernels: storage-type conversion and
// wave/block reductions.  Wavefronts are 64 lanes wide.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace icarus {

typedef uint16_t bf16_t;  // raw bfloat16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t v) {
    return __uint_as_float(((uint32_t)v) << 16);
}

// float -> bfloat16, round to nearest even (NaN kept quiet): gfx950 converts two at a time in one instruction.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)lo, (__bf16)hi});
}
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }

template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ float ld(const float *p) { return *p; }
    static __device__ __forceinline__ void st(float *p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
    static __device__ __forceinline__ float ld(const bf16_t *p) { return bf16_to_f32(*p); }
    static __device__ __forceinline__ void st(bf16_t *p, float v) { *p = f32_to_bf16(v); }
};

// FP8 E4M3 (OCP: largest finite value 448, no infinities) cache element.  gfx950's conversion instructions
// implement this format: decode is exact, encode rounds to nearest even and turns magnitudes of 480 and
// more into NaN, so values are clamped to +-448 first.
struct fp8_t { uint8_t v; };
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float fp8_to_f32(uint32_t code) { return __builtin_amdgcn_cvt_pk_f32_fp8(code, false)[0]; }
__device__ __forceinline__ uint32_t f32_to_fp8(float x) {
    if (!(x == x)) return 0x7fu;
    x = fminf(fmaxf(x, -448.f), 448.f);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(x, 0.f, 0, false) & 0xffu;
}

// Cache element access: value = stored element (x scale for FP8 codes).
template <typename KT> struct KVElem {
    static __device__ __forceinline__ float ld(const KT *p, float) { return Elem<KT>::ld(p); }
    static __device__ __forceinline__ void st(KT *p, float v, float) { Elem<KT>::st(p, v); }
};
template <> struct KVElem<fp8_t> {
    static __device__ __forceinline__ float ld(const fp8_t *p, float scale) { return fp8_to_f32(p->v) * scale; }
    static __device__ __forceinline__ void st(fp8_t *p, float v, float scale) { p->v = (uint8_t)f32_to_fp8(v / scale); }
};

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// Sums N values over the wave's 64 lanes (N a power of two up to 64): in each step a lane keeps half of its values and
// sends the other half, so N - 1 + log2(64 / N) exchanges do what N sums of 6 would.  Lane l ends with the sum of
// value l / (64 / N).  By recursion: as a loop over halves the values went through scratch memory where a kernel sums 64.
template <int N, int H = N / 2, int O = 32>
__device__ __forceinline__ float wave_sums(float (&v)[N], int lane) {
    if constexpr (O > 0) {
        const bool hi = lane & O;
        if constexpr (H > 0) {
#pragma unroll
            for (int i = 0; i < H; ++i) {
                const float keep = hi ? v[i + H] : v[i], send = hi ? v[i] : v[i + H];
                v[i] = keep + __shfl_xor(send, O, 64);
            }
        } else {
            v[0] += __shfl_xor(v[0], O, 64);
        }
        return wave_sums<N, H / 2, O / 2>(v, lane);
    }
    return v[0];
}

// One rotated pair.  Which product is rounded before the sum is written out: a cache entry must not depend on which
// of the kernels that append wrote it, and left to the compiler they came out differently.
__device__ __forceinline__ void rotate_pair(float a, float b, float cs, float sn, float *ra, float *rb) {
    *ra = __builtin_fmaf(a, cs, -(b * sn));
    *rb = __builtin_fmaf(a, sn, b * cs);
}

// Block-wide reductions for blocks of up to 1024 threads; `red` is a shared float[16].
// Every thread gets the result.
__device__ __forceinline__ float block_sum(float v, float *red) {
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) red[w] = v;
    __syncthreads();
    float r = 0.f;
    for (int i = 0; i < nw; ++i) r += red[i];
    return r;
}
__device__ __forceinline__ float block_max(float v, float *red) {
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    v = wave_max(v);
    __syncthreads();
    if (lane == 0) red[w] = v;
    __syncthreads();
    float r = red[0];
    for (int i = 1; i < nw; ++i) r = fmaxf(r, red[i]);
    return r;
}

}  // namespace icarus
