// Generic vector kernels for the ICaRus layer step: any shape, storage type float32 or
// bfloat16, fp32 accumulation.  They serve the fp32 configuration and every shape the
// matrix-core kernels do not cover.
#include "device_util.h"
#include "kernels.h"

#include <algorithm>
#include <type_traits>

namespace icarus {

#define DISPATCH_T(bf16, ...)                         \
    do {                                              \
        if (bf16) { typedef bf16_t T; __VA_ARGS__; }  \
        else      { typedef float T;  __VA_ARGS__; }  \
    } while (0)
// T as above; KT: element type of the KV pool (T, or FP8 codes)
#define DISPATCH_TK(bf16, kv8, ...)                                   \
    do {                                                              \
        if (kv8) { typedef fp8_t KT; DISPATCH_T(bf16, __VA_ARGS__); } \
        else if (bf16) { typedef bf16_t T; typedef bf16_t KT; __VA_ARGS__; } \
        else { typedef float T; typedef float KT; __VA_ARGS__; }      \
    } while (0)

// ------------------------------------------------------------------ RMSNorm
template <typename T>
__global__ void __launch_bounds__(256) k_rmsnorm(const T *__restrict__ x, const T *__restrict__ w, T *__restrict__ y,
                                                 int n, float eps) {
    __shared__ float red[16];
    const T *xr = x + (size_t)blockIdx.x * n;
    T *yr = y + (size_t)blockIdx.x * n;
    float ss = 0.f;
    for (int i = threadIdx.x; i < n; i += blockDim.x) { float v = Elem<T>::ld(xr + i); ss += v * v; }
    ss = block_sum(ss, red);
    float inv = rsqrtf(ss / (float)n + eps);
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        Elem<T>::st(yr + i, Elem<T>::ld(xr + i) * inv * Elem<T>::ld(w + i));
}

hipError_t launch_rmsnorm(const Dims &dm, const void *x, const void *w, void *y, int R, int n, hipStream_t st) {
    if (R <= 0) return hipSuccess;
    DISPATCH_T(dm.bf16, hipLaunchKernelGGL(k_rmsnorm<T>, dim3(R), dim3(256), 0, st, (const T *)x, (const T *)w, (T *)y, n, dm.eps));
    return hipGetLastError();
}

// ------------------------------------------------------------------ GEMM  Y = X W^T  (fp32 out)
// 64x64 output tile per 256-thread block, 4x4 outputs per thread, K staged 16 at a time in LDS.
template <typename T>
__global__ void __launch_bounds__(256) k_gemm_generic(const T *__restrict__ X, int ldx, const T *__restrict__ W,
                                                      int M, int N, int K, float *__restrict__ Y, int ldy) {
    __shared__ float Xs[16][65];
    __shared__ float Ws[16][65];
    int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    float acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
    for (int k0 = 0; k0 < K; k0 += 16) {
        for (int e = threadIdx.x; e < 64 * 16; e += 256) {
            int rr = e >> 4, kk = e & 15;
            int m = m0 + rr, n = n0 + rr, k = k0 + kk;
            Xs[kk][rr] = (m < M && k < K) ? Elem<T>::ld(X + (size_t)m * ldx + k) : 0.f;
            Ws[kk][rr] = (n < N && k < K) ? Elem<T>::ld(W + (size_t)n * K + k) : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = Xs[kk][ty * 4 + i]; b[i] = Ws[kk][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int m = m0 + ty * 4 + i, n = n0 + tx * 4 + j;
            if (m < M && n < N) Y[(size_t)m * ldy + n] = acc[i][j];
        }
}

hipError_t launch_gemm_generic(const Dims &dm, const void *X, int ldx, const void *W, int M, int N, int K,
                               float *Y, int ldy, hipStream_t st) {
    if (M <= 0 || N <= 0) return hipSuccess;
    dim3 grid((N + 63) / 64, (M + 63) / 64);
    DISPATCH_T(dm.bf16, hipLaunchKernelGGL(k_gemm_generic<T>, grid, dim3(256), 0, st, (const T *)X, ldx, (const T *)W, M, N, K, Y, ldy));
    return hipGetLastError();
}

// ------------------------------------------------------------------ LoRA shrink / expand
// One block per row; wave w computes t[rr] for rr = w, w+4, ...
template <typename T>
__global__ void __launch_bounds__(256) k_lora_shrink(const T *__restrict__ X, int ldx, const T *__restrict__ A, int K, int r,
                                                     const int32_t *__restrict__ row_model, float *__restrict__ t, float scale) {
    int row = blockIdx.x;
    int j = row_model[row];
    if (j < 0) return;
    const T *xr = X + (size_t)row * ldx;
    const T *Aj = A + (size_t)j * r * K;
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int rr = w; rr < r; rr += 4) {
        float acc = 0.f;
        for (int k = lane; k < K; k += 64) acc += Elem<T>::ld(Aj + (size_t)rr * K + k) * Elem<T>::ld(xr + k);
        acc = wave_sum(acc);
        if (lane == 0) t[(size_t)row * r + rr] = acc * scale;
    }
}

template <typename T>
__global__ void __launch_bounds__(256) k_lora_expand(const float *__restrict__ t, const T *__restrict__ B, int N, int r,
                                                     const int32_t *__restrict__ row_model, float *__restrict__ Y, int ldy) {
    int row = blockIdx.y;
    int j = row_model[row];
    if (j < 0) return;
    int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= N) return;
    const T *Bn = B + ((size_t)j * N + n) * r;
    float acc = 0.f;
    for (int k = 0; k < r; ++k) acc += Elem<T>::ld(Bn + k) * t[(size_t)row * r + k];
    Y[(size_t)row * ldy + n] += acc;
}

hipError_t launch_lora_shrink_generic(const Dims &dm, const void *X, int ldx, const void *A, int K,
                                      const int32_t *row_model, float *t, int R, hipStream_t st) {
    if (R <= 0 || dm.r <= 0) return hipSuccess;
    DISPATCH_T(dm.bf16, hipLaunchKernelGGL(k_lora_shrink<T>, dim3(R), dim3(256), 0, st, (const T *)X, ldx, (const T *)A, K, dm.r, row_model, t, dm.lora_scale));
    return hipGetLastError();
}
hipError_t launch_lora_expand_generic(const Dims &dm, const float *t, const void *B, int N,
                                      const int32_t *row_model, float *Y, int ldy, int R, hipStream_t st) {
    if (R <= 0 || dm.r <= 0) return hipSuccess;
    dim3 grid((N + 255) / 256, R);
    DISPATCH_T(dm.bf16, hipLaunchKernelGGL(k_lora_expand<T>, grid, dim3(256), 0, st, t, (const T *)B, N, dm.r, row_model, Y, ldy));
    return hipGetLastError();
}

// ------------------------------------------------------------------ elementwise epilogues
template <typename T>
__global__ void __launch_bounds__(256) k_resid_store(const T *__restrict__ resid, const float *__restrict__ acc, T *__restrict__ out, size_t total) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < total) Elem<T>::st(out + i, Elem<T>::ld(resid + i) + acc[i]);
}
template <typename T>
__global__ void __launch_bounds__(256) k_silu_mul(const float *__restrict__ g, const float *__restrict__ u, T *__restrict__ h, size_t total) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < total) {
        float a = g[i];
        Elem<T>::st(h + i, a / (1.f + __expf(-a)) * u[i]);
    }
}
hipError_t launch_resid_store(const Dims &dm, const void *resid, const float *acc, void *out, int R, int n, hipStream_t st) {
    size_t total = (size_t)R * n;
    if (!total) return hipSuccess;
    DISPATCH_T(dm.bf16, hipLaunchKernelGGL(k_resid_store<T>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, (const T *)resid, acc, (T *)out, total));
    return hipGetLastError();
}
hipError_t launch_silu_mul(const Dims &dm, const float *gate, const float *up, void *h, int R, int n, hipStream_t st) {
    size_t total = (size_t)R * n;
    if (!total) return hipSuccess;
    DISPATCH_T(dm.bf16, hipLaunchKernelGGL(k_silu_mul<T>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, gate, up, (T *)h, total));
    return hipGetLastError();
}

// ------------------------------------------------------------------ QK-norm + RoPE + paged append
// One block per row.  Heads 0..Hq-1 are q; for encoder rows heads Hq..Hq+Hkv-1 are k and the
// next Hkv are v.  The row arrives as `splits` fp32 slices (split-K partials of the projection
// GEMM, `slice` floats apart) that are summed here.  Angles are computed in double, once per
// row: pos * theta^(-2i/D).

template <typename T, typename KT>
__global__ void __launch_bounds__(256) k_rope_append(const float *__restrict__ qkv, int ldq, int splits, size_t slice,
                                                     const int32_t *__restrict__ row_seq,
                                                     const int32_t *__restrict__ row_model, const int32_t *__restrict__ row_pos,
                                                     const int32_t *__restrict__ bt, int max_blocks, KT *__restrict__ pool,
                                                     T *__restrict__ q_out, int64_t *__restrict__ slot_out, int slot_by_row,
                                                     const T *__restrict__ q_norm, const T *__restrict__ k_norm,
                                                     int Hq, int Hkv, int D, int Bk, double log2_theta, float eps, int qk_norm,
                                                     float k_scale, float v_scale, const int32_t *__restrict__ row_map) {
    extern __shared__ float sm[];  // the row [n_heads * D] | cos, sin [D/2 each] | inv_rms per head [Hq + Hkv]
    // row_map (optional): the projections were computed on a permutation of the call's rows; input row i is the
    // call's row row_map[i], whose metadata it takes and at whose place q is written
    const float *src = qkv + (size_t)blockIdx.x * ldq;
    int row = row_map ? row_map[blockIdx.x] : (int)blockIdx.x;
    int s = row_seq[row], pos = row_pos[row];
    bool enc = row_model[row] < 0;
    int half = D >> 1;
    int n_rot = Hq + (enc ? Hkv : 0), n_heads = Hq + (enc ? 2 * Hkv : 0);
    // With few rows a row's heads are split over gridDim.y workgroups: this one takes heads [h0, h1) of the
    // row's q heads and, on an encoder row, its k and v heads (numbered Hq .. Hq + 2 Hkv - 1).
    const int h0 = (int)((long long)n_heads * blockIdx.y / gridDim.y), h1 = (int)((long long)n_heads * (blockIdx.y + 1) / gridDim.y);
    const int r1 = min(h1, n_rot);  // end of this part's rotated heads
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    float *xr = sm, *cs_t = sm + (size_t)(Hq + 2 * Hkv) * D, *sn_t = cs_t + half, *inv = sn_t + half;
    const bool vec_ok = D % 4 == 0 && ldq % 4 == 0 && slice % 4 == 0;
    if (!vec_ok)
        for (int i = h0 * D + threadIdx.x; i < h1 * D; i += 256) {
            float v = src[i];
            for (int z = 1; z < splits; ++z) v += src[z * slice + i];
            xr[i] = v;
        }
    // rows and slices 16-byte aligned: 16-byte loads, four slices in flight
    for (int i = h0 * D + threadIdx.x * 4; vec_ok && i < h1 * D; i += 1024) {
        float4 v = *(const float4 *)(src + i);
        int z = 1;
        for (; z + 3 < splits; z += 4) {
            const float4 a = *(const float4 *)(src + (size_t)z * slice + i), b = *(const float4 *)(src + (size_t)(z + 1) * slice + i);
            const float4 c4 = *(const float4 *)(src + (size_t)(z + 2) * slice + i), d4 = *(const float4 *)(src + (size_t)(z + 3) * slice + i);
            v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
            v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w;
            v.x += c4.x; v.y += c4.y; v.z += c4.z; v.w += c4.w;
            v.x += d4.x; v.y += d4.y; v.z += d4.z; v.w += d4.w;
        }
        for (; z < splits; ++z) {
            const float4 a = *(const float4 *)(src + (size_t)z * slice + i);
            v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
        }
        *(float4 *)(xr + i) = v;
    }
    for (int i = threadIdx.x; i < half; i += 256) {
        double ang = (double)pos * exp2(-(2.0 * (double)i / (double)D) * log2_theta);
        double sn_d, cs_d;
        sincos(ang, &sn_d, &cs_d);
        cs_t[i] = (float)cs_d;
        sn_t[i] = (float)sn_d;
    }
    __syncthreads();
    if (qk_norm) {
        for (int h = h0 + w; h < r1; h += 4) {
            float ss = 0.f;
            for (int i = lane; i < D; i += 64) { float v = xr[(size_t)h * D + i]; ss += v * v; }
            ss = wave_sum(ss);
            if (lane == 0) inv[h] = rsqrtf(ss / (float)D + eps);
        }
        __syncthreads();
    }
    int64_t slot = 0;
    KT *kdst = nullptr, *vdst = nullptr;
    int off = 0;
    if (enc) {
        int blk = bt[(size_t)s * max_blocks + pos / Bk];
        off = pos % Bk;
        slot = (int64_t)blk * Bk + off;
        kdst = pool + (size_t)blk * Hkv * 2 * Bk * D;
        vdst = kdst;
        if (threadIdx.x == 0 && blockIdx.y == 0 && slot_out) slot_out[slot_by_row ? row : s] = slot;
    }
    for (int idx = h0 * half + threadIdx.x; idx < r1 * half; idx += 256) {
        int h = idx / half, i = idx % half;
        float cs = cs_t[i], sn = sn_t[i];
        float a = xr[(size_t)h * D + i], b = xr[(size_t)h * D + i + half];
        if (qk_norm) {
            const T *nw = h < Hq ? q_norm : k_norm;
            a = a * inv[h] * Elem<T>::ld(nw + i);
            b = b * inv[h] * Elem<T>::ld(nw + i + half);
        }
        float ra, rb;
        rotate_pair(a, b, cs, sn, &ra, &rb);
        if (h < Hq) {
            T *dst = q_out + ((size_t)row * Hq + h) * D;
            Elem<T>::st(dst + i, ra);
            Elem<T>::st(dst + i + half, rb);
        } else {
            KT *dst = kdst + ((size_t)(h - Hq) * 2 + 0) * Bk * D + (size_t)off * D;  // K plane [Bk][D]
            KVElem<KT>::st(dst + i, ra, k_scale);
            KVElem<KT>::st(dst + i + half, rb, k_scale);
        }
    }
    if (enc) {
        const float *vsrc = xr + (size_t)(Hq + Hkv) * D;
        const int v0 = max(h0 - (Hq + Hkv), 0), v1 = h1 - (Hq + Hkv);  // this part's v heads
        for (int idx = v0 * D + threadIdx.x; idx < v1 * D; idx += 256) {
            int h = idx / D, i = idx % D;
            KT *dst = vdst + ((size_t)h * 2 + 1) * Bk * D;  // V plane [D][Bk]
            KVElem<KT>::st(dst + (size_t)i * Bk + off, vsrc[idx], v_scale);
        }
    }
}

hipError_t launch_rope_append(const Dims &dm, const float *qkv, int ldq, int splits, size_t slice, const RowMeta &rm,
                              const int32_t *bt, int max_blocks, void *pool, void *q_out, int64_t *slot_out, int slot_by_row,
                              const void *q_norm, const void *k_norm, int R, hipStream_t st, const int32_t *row_map) {
    if (R <= 0) return hipSuccess;
    size_t shm = sizeof(float) * ((size_t)(dm.Hq + 2 * dm.Hkv) * dm.D + dm.D + dm.Hq + dm.Hkv);
    double l2t = log2(dm.theta);
    if (shm > 160 * 1024) return hipErrorInvalidValue;
    // few rows: several workgroups per row, each with four heads or more
    int parts = 1;
    while (parts < 8 && R * 2 * parts <= 1024 && dm.Hq / (2 * parts) >= 4) parts *= 2;
    DISPATCH_TK(dm.bf16, dm.kv8, {
        if (shm > 64 * 1024) {
            static bool attr_set = false;  // per instantiation
            if (!attr_set) {
                hipError_t e = hipFuncSetAttribute((const void *)k_rope_append<T, KT>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
                if (e != hipSuccess) return e;
                attr_set = true;
            }
        }
        hipLaunchKernelGGL((k_rope_append<T, KT>), dim3(R, parts), dim3(256), shm, st, qkv, ldq, splits, slice, rm.row_seq, rm.row_model,
                           rm.row_pos, bt, max_blocks, (KT *)pool, (T *)q_out, slot_out, slot_by_row, (const T *)q_norm,
                           (const T *)k_norm, dm.Hq, dm.Hkv, dm.D, dm.Bk, l2t, dm.eps, dm.qk_norm, dm.k_scale, dm.v_scale, row_map);
    });
    return hipGetLastError();
}

// four consecutive cache elements (aligned to four elements)
template <typename KT> struct KVElem4;
template <> struct KVElem4<float> {
    static __device__ __forceinline__ void ld(const float *p, float, float (&f)[4]) {
        const float4 v = *(const float4 *)p;
        f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    }
};
template <> struct KVElem4<bf16_t> {
    static __device__ __forceinline__ void ld(const bf16_t *p, float, float (&f)[4]) {
        const uint2 v = *(const uint2 *)p;
        f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
        f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
    }
    static __device__ __forceinline__ void st(bf16_t *p, const float (&f)[4], float) {
        uint2 v;
        v.x = pack_bf16(f[0], f[1]);
        v.y = pack_bf16(f[2], f[3]);
        *(uint2 *)p = v;
    }
};
template <> struct KVElem4<fp8_t> {
    static __device__ __forceinline__ void ld(const fp8_t *p, float scale, float (&f)[4]) {
        const uint32_t v = *(const uint32_t *)p;
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = fp8_to_f32((v >> (8 * e)) & 0xffu) * scale;
    }
    static __device__ __forceinline__ void st(fp8_t *p, const float (&f)[4], float scale) {
        uint32_t v = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) v |= f32_to_fp8(f[e] / scale) << (8 * e);
        *(uint32_t *)p = v;
    }
};

// ------------------------------------------------------------------ the same for prefill chunks
// One workgroup per tile of up to 16 consecutive chunk rows that lie in one KV block (head_dim 128, blocks of 16, bf16
// storage, encoder rows only), or, with few tiles, per tile and share of the heads.  Bound by memory: the row's fp32
// projections in, q and the cache entries out.  A row at a time, each V value was a 2-byte store of its own, 32 bytes
// from the next (the cache holds V transposed), and a rotated pair two more; here a thread rotates four pairs at a time,
// and the tile's V goes through LDS into 16-byte pieces of the transposed plane.  16384 rows x 6144 columns: 169 us ->
// 136 us, 4337 rows 50 -> 34 us, 512 rows x 10240 columns 26 -> 14 us.
// tiles: device, first row | rows << 16.
template <typename KT>
__global__ void __launch_bounds__(256) k_rope_append_tile(const float *__restrict__ qkv, int ldq, int splits, size_t slice,
                                                          const int32_t *__restrict__ tiles, const int32_t *__restrict__ row_seq,
                                                          const int32_t *__restrict__ row_pos, const int32_t *__restrict__ bt,
                                                          int max_blocks, KT *__restrict__ pool, bf16_t *__restrict__ q_out,
                                                          int64_t *__restrict__ slot_out, const bf16_t *__restrict__ q_norm,
                                                          const bf16_t *__restrict__ k_norm, int h_begin, int Hq, int Hkv,
                                                          double log2_theta, float eps, int qk_norm, float k_scale, float v_scale) {
    constexpr int D = 128, half = 64, Bk = 16;
    __shared__ float cs_t[Bk][half], sn_t[Bk][half];
    __shared__ __attribute__((aligned(16))) KT vt[D][Bk + 16 / sizeof(KT)];  // V of one head, transposed; rows 16 bytes apart from full banks
    const int tile = tiles[blockIdx.x], row0 = tile & 0xffff, n = tile >> 16;
    const int s = row_seq[row0], pos0 = row_pos[row0], off0 = pos0 % Bk;
    const int blk = bt[(size_t)s * max_blocks + pos0 / Bk];
    // heads h_begin .. Hq - 1 are q (none for a cache-only call), then Hkv k heads, then Hkv v heads; this workgroup's share
    const int n_rot = Hq + Hkv, n_heads = n_rot + Hkv - h_begin;
    const int h0 = h_begin + (int)((long long)n_heads * blockIdx.y / gridDim.y);
    const int h1 = h_begin + (int)((long long)n_heads * (blockIdx.y + 1) / gridDim.y);
    const int tid = threadIdx.x, t = tid >> 4, l = tid & 15;
    if (h0 < n_rot)
        for (int i = tid; i < n * half; i += 256) {
            const double ang = (double)(pos0 + i / half) * exp2(-(2.0 * (double)(i % half) / (double)D) * log2_theta);
            double sn_d, cs_d;
            sincos(ang, &sn_d, &cs_d);
            cs_t[i / half][i % half] = (float)cs_d;
            sn_t[i / half][i % half] = (float)sn_d;
        }
    if (slot_out && blockIdx.y == 0 && tid < n) slot_out[row0 + tid] = (int64_t)blk * Bk + off0 + tid;
    __syncthreads();
    const bool live = t < n;  // 16 lanes per row; rows past the tile's last repeat it and store nothing
    const float *src = qkv + (size_t)(row0 + min(t, n - 1)) * ldq;
    auto load4 = [&](int col) {
        float4 v = *(const float4 *)(src + col);
        for (int z = 1; z < splits; ++z) {
            const float4 a = *(const float4 *)(src + (size_t)z * slice + col);
            v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
        }
        return v;
    };
    KT *const blk_k = pool + (size_t)blk * Hkv * 2 * Bk * D;
    const int r1 = min(h1, n_rot);
    float4 na = make_float4(0.f, 0.f, 0.f, 0.f), nb = na;  // one head ahead
    if (h0 < r1) { na = load4(h0 * D + 4 * l); nb = load4(h0 * D + half + 4 * l); }
    for (int h = h0; h < r1; ++h) {
        const float4 va = na, vb = nb;
        if (h + 1 < r1) { na = load4((h + 1) * D + 4 * l); nb = load4((h + 1) * D + half + 4 * l); }
        float a[4] = {va.x, va.y, va.z, va.w}, b[4] = {vb.x, vb.y, vb.z, vb.w};
        if (qk_norm) {
            float p[4];  // pair 4 l + e; summed in the order of k_rope_append, which has a pair to a lane
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                p[e] = __builtin_fmaf(b[e], b[e], a[e] * a[e]);
#pragma unroll
                for (int o = 8; o > 0; o >>= 1) p[e] += __shfl_xor(p[e], o, 64);
            }
            const float inv = rsqrtf(((p[0] + p[2]) + (p[1] + p[3])) / (float)D + eps);
            const bf16_t *nw = h < Hq ? q_norm : k_norm;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[e] = a[e] * inv * bf16_to_f32(nw[4 * l + e]);
                b[e] = b[e] * inv * bf16_to_f32(nw[half + 4 * l + e]);
            }
        }
        if (!live) continue;
        float ra[4], rb[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            rotate_pair(a[e], b[e], cs_t[t][4 * l + e], sn_t[t][4 * l + e], &ra[e], &rb[e]);
        }
        if (h < Hq) {
            bf16_t *dst = q_out + ((size_t)(row0 + t) * Hq + h) * D + 4 * l;
            KVElem4<bf16_t>::st(dst, ra, 1.f);
            KVElem4<bf16_t>::st(dst + half, rb, 1.f);
        } else {
            KT *dst = blk_k + (size_t)(h - Hq) * 2 * Bk * D + (size_t)(off0 + t) * D + 4 * l;  // K plane [Bk][D]
            KVElem4<KT>::st(dst, ra, k_scale);
            KVElem4<KT>::st(dst + half, rb, k_scale);
        }
    }
    constexpr int kPer = 16 / sizeof(KT);  // elements of a 16-byte piece: 8 or 16 tokens
    for (int h = max(h0, n_rot); h < h1; ++h) {
        const float4 va = load4(h * D + 4 * l), vb = load4(h * D + half + 4 * l);
        __syncthreads();  // the previous head's pieces have been read
        if (live) {
            const float v[8] = {va.x, va.y, va.z, va.w, vb.x, vb.y, vb.z, vb.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) KVElem<KT>::st(&vt[(e >> 2) * half + 4 * l + (e & 3)][off0 + t], v[e], v_scale);
        }
        __syncthreads();
        KT *dst = blk_k + ((size_t)(h - n_rot) * 2 + 1) * Bk * D;  // V plane [D][Bk]
        for (int i = tid; i < D * Bk / kPer; i += 256) {
            const int d = i / (Bk / kPer), o = i % (Bk / kPer) * kPer;
            if (off0 <= o && off0 + n >= o + kPer) *(uint4 *)(dst + (size_t)d * Bk + o) = *(const uint4 *)&vt[d][o];
            else  // a tile that fills its block in part: only the tokens it has
                for (int e = max(off0, o); e < min(off0 + n, o + kPer); ++e) dst[(size_t)d * Bk + e] = vt[d][e];
        }
    }
}

bool rope_tiles_supported(const Dims &dm, int ldq, size_t slice) {
    return dm.bf16 && dm.D == 128 && dm.Bk == 16 && ldq % 4 == 0 && slice % 4 == 0;
}

// A tile's thread works through its slices, four heads and then V one after the other, 12-22 us however few tiles there
// are; a row at a time, 24-200 rows fill the chip better.  Row kernel -> tiles, 48 heads (q, k and v): 24 rows 4.1 -> 22
// us, 128 rows 7 -> 22, 256 rows 9.3 -> 12.5, 400 rows 11.5 -> 12.0, 600 rows 16.3 -> 14.9; 80 heads: 64 rows 8.3 -> 14.6,
// 128 rows 14 -> 15.5, 256 rows 18.6 -> 11.7; FP8 cache: 256 rows of 48 heads 8.8 -> 13.5, 512 rows 13.0 -> 14.1, 400 rows of
// 80 29.5 -> 14.8.  And a tile takes as long for one row as for sixteen: short chunks go row by row.  48 heads: 1000 tiles of
// one row 25.2 -> 41.0 us, of two 36.3 -> 42.6, of three 47.3 -> 45.3 (500: 28.6 -> 30.4), of four 60.4 -> 47.1; 80 heads: 50.5
// -> 86.3, 77.8 -> 90.7, 113 -> 109, 158 -> 119.
bool rope_tiles_pay(const Dims &dm, int rows, int n_tiles) {
    return (int64_t)rows * (dm.Hq + 2 * dm.Hkv) >= 20480 && (int64_t)rows >= 4 * (int64_t)n_tiles;
}

hipError_t launch_rope_append_tiles(const Dims &dm, const float *qkv, int ldq, int splits, size_t slice, const RowMeta &rm,
                                    const int32_t *tiles, int n_tiles, bool kv_only, const int32_t *bt, int max_blocks, void *pool,
                                    void *q_out, int64_t *slot_out, const void *q_norm, const void *k_norm, hipStream_t st) {
    if (n_tiles <= 0) return hipSuccess;
    if (!rope_tiles_supported(dm, ldq, slice)) return hipErrorInvalidValue;
    const int h_begin = kv_only ? dm.Hq : 0, n_heads = dm.Hq - h_begin + 2 * dm.Hkv;
    int parts = 1;  // few tiles: several workgroups per tile, each with four heads or more
    while (parts < 16 && n_tiles * parts < 1536 && n_heads / (2 * parts) >= 4) parts *= 2;
    auto launch = [&](auto kt) {
        typedef decltype(kt) KT;
        hipLaunchKernelGGL(k_rope_append_tile<KT>, dim3(n_tiles, parts), dim3(256), 0, st, qkv, ldq, splits, slice, tiles, rm.row_seq, rm.row_pos,
                           bt, max_blocks, (KT *)pool, (bf16_t *)q_out, slot_out, (const bf16_t *)q_norm, (const bf16_t *)k_norm, h_begin,
                           dm.Hq, dm.Hkv, log2(dm.theta), dm.eps, dm.qk_norm, dm.k_scale, dm.v_scale);
        return hipGetLastError();
    };
    return dm.kv8 ? launch(fp8_t()) : launch(bf16_t());
}

// What the fused form of the above (gemm_quad.hip) needs of each row: cosines and sines of its 64 angles, and its slot.
__global__ void __launch_bounds__(256) k_rope_table(const int32_t *__restrict__ row_seq, const int32_t *__restrict__ row_pos,
                                                    const int32_t *__restrict__ bt, int max_blocks, int R, double log2_theta,
                                                    float *__restrict__ cs, float *__restrict__ sn, int64_t *__restrict__ slot) {
    constexpr int D = 128, half = 64, Bk = 16;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), i = threadIdx.x & 63;
    if (row >= R) return;
    const int pos = row_pos[row];
    const double ang = (double)pos * exp2(-(2.0 * (double)i / (double)D) * log2_theta);
    double sn_d, cs_d;
    sincos(ang, &sn_d, &cs_d);
    cs[(size_t)row * half + i] = (float)cs_d;
    sn[(size_t)row * half + i] = (float)sn_d;
    if (i == 0) slot[row] = (int64_t)bt[(size_t)row_seq[row] * max_blocks + pos / Bk] * Bk + pos % Bk;
}

hipError_t launch_rope_table(const Dims &dm, const RowMeta &rm, const int32_t *bt, int max_blocks, int R, float *cs, float *sn, int64_t *slot,
                             hipStream_t st) {
    if (R <= 0) return hipSuccess;
    if (dm.D != 128 || dm.Bk != 16) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_rope_table, dim3((R + 3) / 4), dim3(256), 0, st, rm.row_seq, rm.row_pos, bt, max_blocks, R, log2(dm.theta), cs, sn, slot);
    return hipGetLastError();
}

// ------------------------------------------------------------------ attention (one block per row and query head)
// Online softmax over chunks of 1024 cached positions.  Scores: LPT threads per position, each every LPT-th quad of its
// elements.  Output: thread (part, d) adds every parts-th quad of positions to output element d; V^T rows hold a block's
// tokens side by side, so a quad is one load, and neighbouring threads take the quads of a block's row (pl of them, up to four).
// Latency-bound at the sizes this kernel is for, and next by the lines that its loads touch: with a thread per position and
// a part per wave every load touched a line per lane.  Rows x 4 heads x 64, us, that with 256 threads a workgroup / this, float32:
// 3 rows over 128 tokens 9.4 / 8.4, 12 rows over 1000 28.7 / 13.0, 768 rows 253 / 93; bf16 768 rows 240 / 93; FP8 64 rows over 128 10.1 / 8.6,
// 768 rows over 1000 169 / 106.
// KU, VU: loads in flight.  With eight the workgroups in flight were fewer (109-144 registers, now 74-82) and 1024 threads spilled for an FP8
// cache, whose load is four conversions: 768 rows float32 115, bf16 138, FP8 186 us.
// quads: D and Bk are multiples of 4; else one element, one position at a time.
template <typename T, typename KT, int NT, int LPT, bool quads>
__global__ void __launch_bounds__(NT) k_attn_generic(const T *__restrict__ q, const KT *__restrict__ pool,
                                                     const int32_t *__restrict__ bt, int max_blocks,
                                                     const int32_t *__restrict__ row_seq, const int32_t *__restrict__ row_kvlen,
                                                     T *__restrict__ out, int Hq, int Hkv, int D, int Bk, float scale,
                                                     float k_scale, float v_scale, int parts, int pl) {
    constexpr int KU = sizeof(KT) == 1 ? 2 : 4, VU = 4;
    __shared__ __attribute__((aligned(16))) float sc[1024];
    __shared__ size_t soff[1024];  // where a position's V elements are, within its head
    __shared__ float sum[NT];
    __shared__ float red[16];
    extern __shared__ __attribute__((aligned(16))) float qs[];  // [D]
    int row = blockIdx.y, h = blockIdx.x;
    int c = h / (Hq / Hkv);
    int s = row_seq[row], n = row_kvlen[row];
    const int32_t *btr = bt + (size_t)s * max_blocks;
    for (int i = threadIdx.x; i < D; i += NT) qs[i] = Elem<T>::ld(q + ((size_t)row * Hq + h) * D + i);
    __syncthreads();
    const int width = NT / parts;  // all three are powers of two
    const int part = threadIdx.x % pl + pl * (threadIdx.x / (pl * width)), d = threadIdx.x / pl % width;
    const int sub = threadIdx.x % LPT;
    size_t head_stride = (size_t)2 * Bk * D, blk_stride = (size_t)Hkv * head_stride;
    const KT *head = pool + (size_t)c * head_stride;
    float m = -INFINITY, l = 0.f, acc = 0.f;
    for (int c0 = 0; c0 < n; c0 += 1024) {
        int cnt = min(1024, n - c0);
        float lmax = -INFINITY;
        for (int t = threadIdx.x / LPT; t < cnt; t += NT / LPT) {
            int tok = c0 + t;
            const int in_blk = tok % Bk;
            const size_t off = (size_t)btr[tok / Bk] * blk_stride;
            const KT *kr = head + off + (size_t)in_blk * D;
            float dot = 0.f;
            if constexpr (quads) {
#pragma unroll KU
                for (int i = 4 * sub; i < D; i += 4 * LPT) {
                    float kv[4];
                    KVElem4<KT>::ld(kr + i, k_scale, kv);
                    const float4 qv = *(const float4 *)(qs + i);
                    dot += qv.x * kv[0];
                    dot += qv.y * kv[1];
                    dot += qv.z * kv[2];
                    dot += qv.w * kv[3];
                }
            } else {
                for (int i = 0; i < D; ++i) dot += qs[i] * KVElem<KT>::ld(kr + i, k_scale);
            }
#pragma unroll
            for (int o = 1; o < LPT; o *= 2) dot += __shfl_xor(dot, o, 64);  // the threads of a position go round together
            dot *= scale;
            if (sub == 0) {
                sc[t] = dot;
                soff[t] = off + in_blk;
            }
            lmax = fmaxf(lmax, dot);
        }
        float cmax = block_max(lmax, red);  // barriers inside also publish sc[] and soff[]
        float m_new = fmaxf(m, cmax);
        float lsum = 0.f;
        for (int t = threadIdx.x; t < cnt; t += NT) {
            float p = __expf(sc[t] - m_new);
            sc[t] = p;
            lsum += p;
        }
        float csum = block_sum(lsum, red);  // likewise the probabilities
        float alpha = (m == -INFINITY) ? 0.f : __expf(m - m_new);
        l = l * alpha + csum;
        if (d < D) {
            float a = acc * alpha;
            const KT *vd = head + (size_t)Bk * D + (size_t)d * Bk;
            if constexpr (quads) {
#pragma unroll VU
                for (int t = 4 * part; t + 3 < cnt; t += 4 * parts) {
                    float v[4];
                    KVElem4<KT>::ld(vd + soff[t], v_scale, v);
                    const float4 p = *(const float4 *)(sc + t);
                    a += p.x * v[0];
                    a += p.y * v[1];
                    a += p.z * v[2];
                    a += p.w * v[3];
                }
                if (part == 0)  // the last, partial quad: what lies past the context may be anything
                    for (int t = cnt & ~3; t < cnt; ++t) a += sc[t] * KVElem<KT>::ld(vd + soff[t], v_scale);
            } else {
                for (int t = part; t < cnt; t += parts) a += sc[t] * KVElem<KT>::ld(vd + soff[t], v_scale);
            }
            acc = a;
        }
        m = m_new;
        __syncthreads();
    }
    sum[part * width + d] = acc;
    __syncthreads();
    if (threadIdx.x < D) {
        acc = sum[threadIdx.x];
        for (int p = 1; p < parts; ++p) acc += sum[p * width + threadIdx.x];
        Elem<T>::st(out + ((size_t)row * Hq + h) * D + threadIdx.x, l > 0.f ? acc / l : 0.f);
    }
}

// Workgroups up to which each gets a CU, and so 1024 threads (512 where D < 64).  Rows x 4 heads x 64, us with 256 / 1024 threads, float32: 12
// workgroups over 1000 tokens 20.7 / 13.7, 256 over 128 tokens 8.6 / 8.6 and over 1000 29.6 / 18.4, 260 8.4 / 12.8 and 37.4 / 37.8; bf16 256
// 9.5 / 8.5 and 28.8 / 15.2, 260 9.2 / 12.8 and 45.1 / 34.3, 768 10.2 / 18.3 and 49.8 / 51.0; FP8 256 9.6 / 8.4 and 29.8 / 15.2, 260 9.2 / 12.1 and
// 40.4 / 30.7, 768 10.4 / 16.9 and 50.1 / 48.7.
constexpr int kGenericWide = 256;

hipError_t launch_attn_generic(const Dims &dm, const void *q, const void *pool, const int32_t *bt, int max_blocks,
                               const RowMeta &rm, void *out, int R, hipStream_t st) {
    if (R <= 0) return hipSuccess;
    float scale = 1.0f / sqrtf((float)dm.D);
    dim3 grid(dm.Hq, R);
    auto launch = [&](auto nt, auto lpt, auto by_quads) {
        constexpr int NT = decltype(nt)::value, LPT = decltype(lpt)::value;
        constexpr bool quads = decltype(by_quads)::value;
        int parts = 1;
        while (parts < 32 && NT / (2 * parts) >= dm.D) parts *= 2;
        const int pl = std::min(parts, !quads || dm.Bk % 16 == 0 ? 4 : dm.Bk % 8 == 0 ? 2 : 1);  // quads of a block
        DISPATCH_TK(dm.bf16, dm.kv8, hipLaunchKernelGGL((k_attn_generic<T, KT, NT, LPT, quads>), grid, dim3(NT), sizeof(float) * dm.D, st, (const T *)q,
                                                        (const KT *)pool, bt, max_blocks, rm.row_seq, rm.row_kvlen, (T *)out, dm.Hq, dm.Hkv,
                                                        dm.D, dm.Bk, scale, dm.k_scale, dm.v_scale, parts, pl));
        return hipGetLastError();
    };
    constexpr std::integral_constant<int, 1> one;
    constexpr std::integral_constant<int, 2> two;
    constexpr std::integral_constant<int, 4> four;
    constexpr std::integral_constant<int, 256> few;
    constexpr std::true_type by_quads;
    if (dm.D % 4 || dm.Bk % 4) return launch(few, one, std::false_type());
    // A position's address costs each of its threads two divisions, so a short row has fewer of them; and 1024 threads need more rounds to
    // meet than a short row takes.  bf16, us, one thread a position and 256 a workgroup at first / four and 1024 / this: D = 32, 12 rows x
    // 8 heads over 128 tokens 7.8 / 8.5 / 7.5, 768 rows over 1000 154 / 171 / 97; D = 16 the same 7.1 / 8.5 / 7.2 and 67 / 129 / 57; D = 48
    // 9.0 / 8.6 / 7.8 and 302 / 243 / 156; D = 60, 768 rows x 4 heads 225 / 149 / 119 (float32 241 / 120 / 136).
    const bool wide = (int64_t)dm.Hq * R <= kGenericWide;
    if (dm.D < 32) return wide ? launch(std::integral_constant<int, 512>(), one, by_quads) : launch(few, one, by_quads);
    if (dm.D < 64) return wide ? launch(std::integral_constant<int, 512>(), two, by_quads) : launch(few, two, by_quads);
    return wide ? launch(std::integral_constant<int, 1024>(), four, by_quads) : launch(few, four, by_quads);
}

}  // namespace icarus

// ------------------------------------------------------------------ plain copy (counter calibration)
namespace icarus {
__global__ void __launch_bounds__(256) k_bench_copy(const uint4 *__restrict__ src, uint4 *__restrict__ dst, size_t n16) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x, stride = (size_t)gridDim.x * 256;
    for (; i < n16; i += stride) dst[i] = src[i];
}
hipError_t launch_bench_copy(const void *src, void *dst, size_t bytes, hipStream_t st) {
    size_t n16 = bytes / 16;
    if (!n16) return hipSuccess;
    unsigned blocks = (unsigned)std::min<size_t>((n16 + 255) / 256, 256 * 32);
    hipLaunchKernelGGL(k_bench_copy, dim3(blocks), dim3(256), 0, st, (const uint4 *)src, (uint4 *)dst, n16);
    return hipGetLastError();
}

// ------------------------------------------------------------------ streaming read (achievable HBM rate)
// Every wave walks its own contiguous 8 KB chunks (the size of one (block, kv-head) of the cache) in a
// grid-stride order, eight independent 16-byte loads per lane in flight twice over, and folds what it reads
// into one word so that the loads cannot be dropped.  Nothing is stored unless the fold hits one value.
__global__ void __launch_bounds__(256) k_bench_read(const uint4 *__restrict__ src, size_t n_chunks, uint32_t *__restrict__ out) {
    const int lane = threadIdx.x & 63;
    const size_t wave = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6), n_waves = (size_t)gridDim.x * 4;
    uint4 acc = make_uint4(0u, 0u, 0u, 0u);
    uint4 a[8], b[8];
    auto load = [&](size_t c, uint4 (&d)[8]) {
        const uint4 *p = src + c * 512 + lane;
#pragma unroll
        for (int i = 0; i < 8; ++i) d[i] = p[i * 64];
    };
    auto fold = [&](const uint4 (&d)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) { acc.x ^= d[i].x; acc.y ^= d[i].y; acc.z ^= d[i].z; acc.w ^= d[i].w; }
    };
    size_t c = wave;
    if (c < n_chunks) load(c, a);
    for (; c < n_chunks; c += 2 * n_waves) {
        const size_t c1 = c + n_waves, c2 = c + 2 * n_waves;
        if (c1 < n_chunks) load(c1, b);
        fold(a);
        if (c2 < n_chunks) load(c2, a);
        if (c1 < n_chunks) fold(b);
    }
    if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9e3779b9u) out[0] = acc.x;
}
hipError_t launch_bench_read(const void *src, size_t bytes, uint32_t *out, hipStream_t st) {
    const size_t n_chunks = bytes / 8192;
    if (!n_chunks) return hipSuccess;
    unsigned blocks = (unsigned)std::min<size_t>((n_chunks + 3) / 4, 256 * 4);
    hipLaunchKernelGGL(k_bench_read, dim3(blocks), dim3(256), 0, st, (const uint4 *)src, n_chunks, out);
    return hipGetLastError();
}
}  // namespace icarus
