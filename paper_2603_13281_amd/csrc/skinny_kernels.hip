// Vector kernels of the layer step for a handful of rows: any shape, storage type float32 or bfloat16, fp32 accumulation.
//
// With up to kSkinnyRows rows a projection is a few mat-vecs, and what bounds it is latency, not bytes or arithmetic:
// the 64 x 64 tiles of the many-row kernel put a 256-wide layer's projections on 4-11 workgroups, each of which walks K
// sixteen at a time between two barriers (32-94 us a projection, 340 us a step of 3 rows).  Here a wave owns a few
// output columns and all rows: its 64 lanes split K in 16-byte pieces, so a column of 1024 bytes is one load per lane,
// and the sums meet in registers.  The adapter delta, the residual and the SwiGLU product are added where the sum
// is, and one launch serves the projections that read the same rows: 9 launches for that step instead of 18.  A projection
// is a chain of loads and exchanges: the row's model is asked for first, then the pieces of weights and rows, then, while
// those come, the adapter's columns and the residual; the sums of all columns and rows go through the lanes together
// (wave_sums).  Loads behind one another and a sum at a time took 5.4 us for 3 rows, 256 -> 768, and 9.5 for 12 rows, this 4.0
// and 5.8.
#include "device_util.h"
#include "kernels.h"

#include <type_traits>

namespace icarus {

namespace {

// 16 bytes of storage elements as floats
template <typename T> struct Vec16;
template <> struct Vec16<float> {
    static constexpr int N = 4;
    typedef float4 Raw;
    static __device__ __forceinline__ void un(const float4 &v, float (&f)[4]) { f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w; }
};
template <> struct Vec16<bf16_t> {
    static constexpr int N = 8;
    typedef uint4 Raw;
    static __device__ __forceinline__ void un(const uint4 &v, float (&f)[8]) {
        f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
        f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
        f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xffff0000u);
        f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xffff0000u);
    }
};
// one element at a time: rows that are not whole 16-byte pieces
template <typename T> struct Vec1 {
    static constexpr int N = 1;
    typedef T Raw;
    static __device__ __forceinline__ void un(const T &v, float (&f)[1]) { f[0] = Elem<T>::ld(&v); }
};
template <typename V, typename T> __device__ __forceinline__ typename V::Raw ld_raw(const T *p) { return *(const typename V::Raw *)p; }
template <typename V, typename T> __device__ __forceinline__ void ld_vec(const T *p, float (&f)[V::N]) { V::un(ld_raw<V>(p), f); }

// One workgroup per row: y = rmsnorm(x) * wn (NORM), and for a decoder row t[target][row][0..r) = scale * A[model] y (or
// x) for up to two targets; a wave takes every fourth of the targets * r outputs.
template <typename T, typename V, bool NORM>
__global__ void __launch_bounds__(256) k_row_generic(const T *__restrict__ x, int ldx, int K, const T *__restrict__ wn, float eps,
                                                     T *__restrict__ y, const T *__restrict__ A0, const T *__restrict__ A1, int r,
                                                     const int32_t *__restrict__ row_model, float scale, float *__restrict__ t, int R) {
    __shared__ float red[16];
    const int row = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const T *xr = x + (size_t)row * ldx;
    if (NORM) {
        float ss = 0.f;
        for (int k = threadIdx.x * V::N; k < K; k += 256 * V::N) {
            float f[V::N];
            ld_vec<V>(xr + k, f);
#pragma unroll
            for (int e = 0; e < V::N; ++e) ss += f[e] * f[e];
        }
        ss = block_sum(ss, red);
        const float inv = rsqrtf(ss / (float)K + eps);
        T *yr = y + (size_t)row * K;
        for (int k = threadIdx.x; k < K; k += 256) Elem<T>::st(yr + k, Elem<T>::ld(xr + k) * inv * Elem<T>::ld(wn + k));
        __syncthreads();  // the shrink reads the row as stored, from this workgroup's own stores
        xr = yr;
    }
    const int j = A0 ? row_model[row] : -1;
    if (j < 0) return;
    const int n_out = (A1 ? 2 : 1) * r;
    for (int o = w; o < n_out; o += 4) {
        const T *a = (o < r ? A0 : A1) + ((size_t)j * r + (o < r ? o : o - r)) * K;
        float acc = 0.f;
        for (int k = lane * V::N; k < K; k += 64 * V::N) {
            float f[V::N], g[V::N];
            ld_vec<V>(xr + k, f);
            ld_vec<V>(a + k, g);
#pragma unroll
            for (int e = 0; e < V::N; ++e) acc += f[e] * g[e];
        }
        acc = wave_sum(acc);
        if (lane == 0) t[((size_t)(o < r ? 0 : 1) * R + row) * r + (o < r ? o : o - r)] = acc * scale;
    }
}

// Y[R, N] = X W^T (+ the rows' adapter deltas), RM >= R rows.  A wave takes kCols columns; DUAL: kCols / 2 columns of the
// gate and of the up projection.
constexpr int kCols = 4;
struct SkinnyArgs {
    const void *X; int ldx, R, K;
    const void *W[3]; int n_end[3];          // weight segments: columns [n_end[s - 1], n_end[s]) are rows of W[s]; DUAL: gate, up
    const void *B[2]; const float *t; int r; // adapter of the first segment (DUAL: gate, up), t from k_row_generic; null: none
    const int32_t *row_model;
    const void *resid; void *Y; int ldy;     // SKINNY_F32: float Y; else storage Y (SKINNY_RESID: + resid, same stride)
    const void *wn; float eps;               // NORM: the rows are rmsnorm(X) * wn
    const void *A[2]; float scale;           // SHRINK: t = scale * A[model] x, computed here
};

// The row kernel's work in the projection that reads its rows, where that is little: a launch of its own takes 2.4-3.2 us and the next
// one's start.  NORM: every wave sums the squares of the rows that it multiplies anyway, and scales its sums.  SHRINK: wave w multiplies row w
// with the up to eight rows of its model's A, in every workgroup, and the products meet in LDS.
constexpr int kShrinkRank = 8;
template <typename T, typename V, int RM, int MODE, bool NORM = false, bool SHRINK = false>
__global__ void __launch_bounds__(256) k_gemm_skinny(SkinnyArgs a) {
    constexpr bool dual = MODE == SKINNY_DUAL;
    constexpr int ND = dual ? 2 : 1;  // targets with adapters
    __shared__ float ts[SHRINK ? ND * 4 * kShrinkRank : 1];
    constexpr int NO = dual ? kCols / 2 : kCols;  // output columns of a wave
    const int lane = threadIdx.x & 63, N = a.n_end[dual ? 0 : 2];
    const int n0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * NO;
    if (!SHRINK && n0 >= N) return;
    const T *wrow[kCols];
#pragma unroll
    for (int c = 0; c < kCols; ++c) {
        const int n = min(n0 + c % NO, N - 1);  // columns past the last are computed on it and dropped
        if (dual) {
            wrow[c] = (const T *)a.W[c / NO] + (size_t)n * a.K;
        } else {
            const int s = n < a.n_end[0] ? 0 : n < a.n_end[1] ? 1 : 2;
            wrow[c] = (const T *)a.W[s] + (size_t)(n - (s ? a.n_end[s - 1] : 0)) * a.K;
        }
    }
    // sum (column c, row m) ends in lanes (c * RM + m) * kShare and the kShare - 1 after it
    constexpr int kShare = 64 / (kCols * RM);
    const int c = lane / kShare / RM, row = lane / kShare % RM, n = n0 + c;
    const bool mine = c < NO && row < a.R && n < N, first = mine && lane % kShare == 0;
    const int j = mine && (SHRINK || a.t) && n < a.n_end[0] ? a.row_model[row] : -1;
    const T *X = (const T *)a.X;
    int k = lane * V::N;
    typename V::Raw wv[kCols], xv[RM], gv, av[ND][kShrinkRank], dv;
    // SHRINK: this wave's row and its model's A; without one the products are those of a weight row, and dropped
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int model = SHRINK && wave < a.R ? a.row_model[wave] : -1;
    const T *drow = X + (size_t)min(wave, a.R - 1) * a.ldx, *A[ND];
    int astep[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        const bool has = SHRINK && model >= 0 && a.A[d];
        A[d] = has ? (const T *)a.A[d] + (size_t)model * a.r * a.K : wrow[0];
        astep[d] = has ? a.K : 0;
    }
    auto load = [&] {
        if constexpr (NORM) gv = ld_raw<V>((const T *)a.wn + k);
        if constexpr (SHRINK) {
#pragma unroll
            for (int d = 0; d < ND; ++d)
#pragma unroll
                for (int i = 0; i < kShrinkRank; ++i) av[d][i] = ld_raw<V>(A[d] + (size_t)min(i, a.r - 1) * astep[d] + k);
            dv = ld_raw<V>(drow + k);
        }
#pragma unroll
        for (int i = 0; i < kCols; ++i) wv[i] = ld_raw<V>(wrow[i] + k);
#pragma unroll
        for (int m = 0; m < RM; ++m) xv[m] = ld_raw<V>(X + (size_t)min(m, a.R - 1) * a.ldx + k);
    };
    if (k < a.K) load();
    // what is added to the sum is fetched beneath the first pieces
    float res = 0.f, delta[2] = {0.f, 0.f};
    if (MODE == SKINNY_RESID && first) res = Elem<T>::ld((const T *)a.resid + (size_t)row * a.ldy + n);
    float bv[2][kShrinkRank];
    if constexpr (SHRINK) {
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int i = 0; i < kShrinkRank; ++i)
                bv[d][i] = a.B[d] ? Elem<T>::ld((const T *)a.B[d] + ((size_t)max(j, 0) * a.n_end[0] + min(n, a.n_end[0] - 1)) * a.r + min(i, a.r - 1)) : 0.f;
    } else if (j >= 0) {
#pragma unroll
        for (int d = 0; d < (dual ? 2 : 1); ++d) {
            const T *b = (const T *)a.B[d];
            if (!b) continue;
            b += ((size_t)j * a.n_end[0] + n) * a.r;
            const float *tr = a.t + ((size_t)d * a.R + row) * a.r;
            float v = 0.f;
#pragma unroll 8
            for (int i = 0; i < a.r; ++i) v += Elem<T>::ld(b + i) * tr[i];
            delta[d] = v;
        }
    }
    float acc[kCols * RM];
#pragma unroll
    for (int i = 0; i < kCols * RM; ++i) acc[i] = 0.f;
    float ss[RM], dot[ND * kShrinkRank];
#pragma unroll
    for (int m = 0; m < RM; ++m) ss[m] = 0.f;
#pragma unroll
    for (int i = 0; i < ND * kShrinkRank; ++i) dot[i] = 0.f;
    while (k < a.K) {
        float gf[V::N];
        if constexpr (NORM) V::un(gv, gf);
        if constexpr (SHRINK) {
            float xf[V::N];
            V::un(dv, xf);
#pragma unroll
            for (int e = 0; e < V::N; ++e) xf[e] = NORM ? xf[e] * gf[e] : xf[e];
#pragma unroll
            for (int i = 0; i < ND * kShrinkRank; ++i) {
                float af[V::N];
                V::un(av[i / kShrinkRank][i % kShrinkRank], af);
#pragma unroll
                for (int e = 0; e < V::N; ++e) dot[i] += af[e] * xf[e];
            }
        }
#pragma unroll
        for (int m = 0; m < RM; ++m) {
            float xf[V::N];
            V::un(xv[m], xf);
            if constexpr (NORM) {
#pragma unroll
                for (int e = 0; e < V::N; ++e) {
                    ss[m] += xf[e] * xf[e];
                    xf[e] *= gf[e];
                }
            }
#pragma unroll
            for (int i = 0; i < kCols; ++i) {
                float wf[V::N];
                V::un(wv[i], wf);
#pragma unroll
                for (int e = 0; e < V::N; ++e) acc[i * RM + m] += wf[e] * xf[e];
            }
        }
        k += 64 * V::N;
        if (k < a.K) load();
    }
    float sum = wave_sums(acc, lane), up = 0.f, inv = 1.f;
    if constexpr (NORM) {
        inv = rsqrtf(wave_sums(ss, lane) / (float)a.K + a.eps);  // of row lane / (64 / RM)
        sum *= __shfl(inv, row * (64 / RM), 64);
    }
    if constexpr (SHRINK) {
        constexpr int kLanes = 64 / (ND * kShrinkRank);  // that hold the sum of one product
        const int d = lane / kLanes / kShrinkRank, i = lane / kLanes % kShrinkRank;
        float v = wave_sums(dot, lane) * a.scale;
        if constexpr (NORM) v *= __shfl(inv, wave * (64 / RM), 64);
        if (lane % kLanes == 0) ts[(d * 4 + wave) * kShrinkRank + i] = v;
        __syncthreads();
        if (j >= 0) {
#pragma unroll
            for (int d = 0; d < ND; ++d)
#pragma unroll
                for (int x = 0; x < kShrinkRank; ++x)
                    if (x < a.r && a.A[d]) delta[d] += bv[d][x] * ts[(d * 4 + row) * kShrinkRank + x];
        }
    }
    if (dual) up = __shfl_xor(sum, 32, 64) + delta[1];  // the upper half of the lanes holds the up projection
    sum += delta[0];
    if (!first) return;
    if (MODE == SKINNY_F32) ((float *)a.Y)[(size_t)row * a.ldy + n] = sum;
    else if (MODE == SKINNY_RESID) Elem<T>::st((T *)a.Y + (size_t)row * a.ldy + n, res + sum);
    else Elem<T>::st((T *)a.Y + (size_t)row * a.ldy + n, sum / (1.f + __expf(-sum)) * up);
}

template <typename F>
hipError_t with_type(bool bf16, bool vec, F f) {
    if (bf16) return vec ? f(bf16_t(), Vec16<bf16_t>()) : f(bf16_t(), Vec1<bf16_t>());
    return vec ? f(float(), Vec16<float>()) : f(float(), Vec1<float>());
}

bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }
bool whole_pieces(const Dims &dm, int n) { return n % (dm.bf16 ? 8 : 4) == 0; }

}  // namespace

hipError_t launch_row_generic(const Dims &dm, const void *x, int ldx, int K, const void *wn, void *y, const void *A0, const void *A1,
                              const int32_t *row_model, float *t, int R, hipStream_t st) {
    if (R <= 0 || (!wn && !A0)) return hipSuccess;
    const bool vec = whole_pieces(dm, K) && whole_pieces(dm, ldx) && aligned16(x);
    return with_type(dm.bf16, vec, [&](auto tt, auto vv) {
        typedef decltype(tt) T;
        typedef decltype(vv) V;
        if (wn)
            hipLaunchKernelGGL((k_row_generic<T, V, true>), dim3(R), dim3(256), 0, st, (const T *)x, ldx, K, (const T *)wn, dm.eps, (T *)y,
                               (const T *)A0, (const T *)A1, dm.r, row_model, dm.lora_scale, t, R);
        else
            hipLaunchKernelGGL((k_row_generic<T, V, false>), dim3(R), dim3(256), 0, st, (const T *)x, ldx, K, (const T *)nullptr, dm.eps,
                               (T *)nullptr, (const T *)A0, (const T *)A1, dm.r, row_model, dm.lora_scale, t, R);
        return hipGetLastError();
    });
}

// float32 rows of whole 16-byte pieces (in bf16 the projection reads the normalised rows as rounded), with adapters up to four of them, a
// wave each.  Beyond some width what every workgroup does again outweighs the launch, the sooner the more rows there are.  A layer step with
// adapters on q and o, FFN 2.7 times as wide, us, row kernels / fused: 3 rows, 256 columns 46.5 / 36.0, 512 45.1 / 35.1, 1024 52.4 / 43.3, 2048
// 88.7 / 73.0; 12 rows (norm alone) 46.4 / 42.9, 52.1 / 50.3, 72.8 / 75.5, 117 / 125.
// Nine rows and more take the form of 16, whose norm costs it the registers of a second wave on its SIMD (256 instead of 240): beyond a wave to each of the
// 1024 SIMDs, 4096 rows of weights, it loses.  12 rows of 256 / 512 columns, us, row kernel / fused: gate and up of 2 x 2048 49.4 / 47.6 and 52.1 / 50.9,
// 2 x 2560 54.4 / 54.8 and 57.0 / 59.4, 2 x 4096 57.6 / 58.7 and 62.3 / 64.9, 2 x 8192 78.0 / 83.2 and 83.9 / 91.2, 2 x 32768 194 / 226 and 206 / 247; q, k and v
// (gate and up fused in both) of 4096 52.5 / 49.5 and 55 / 52.7, 6144 60.5 / 61.4 and 63.5 / 66.2.  Up to eight rows the fused form is the faster one at all of these.
constexpr int kFusedColumns = 2048, kFusedColumnsMoreRows = 512;
constexpr int kFusedRowsAnyWidth = 8, kFusedWeightRows = 4 * 1024;
bool skinny_takes_rows(const Dims &dm, const SkinnyGemm &g) {
    const bool shrink = g.A[0] || g.A[1];
    if (g.R > kFusedRowsAnyWidth && g.n[0] + g.n[1] + g.n[2] > kFusedWeightRows) return false;
    if (dm.bf16 || g.K > (g.R <= 4 ? kFusedColumns : kFusedColumnsMoreRows) || !whole_pieces(dm, g.K) || !whole_pieces(dm, g.ldx) || !aligned16(g.X) || (g.wn && !aligned16(g.wn))) return false;
    for (int s = 0; s < 3; ++s)
        if (g.W[s] && !aligned16(g.W[s])) return false;
    if ((g.mode == SKINNY_RESID) != !g.wn) return false;
    if (!shrink) return g.wn != nullptr;
    for (int d = 0; d < 2; ++d)
        if (g.A[d] && !aligned16(g.A[d])) return false;
    return g.R <= 4 && dm.r <= kShrinkRank;
}

hipError_t launch_gemm_skinny(const Dims &dm, const SkinnyGemm &g, hipStream_t st) {
    if (g.R <= 0) return hipSuccess;
    if (g.R > kSkinnyRows) return hipErrorInvalidValue;
    SkinnyArgs a{};
    a.X = g.X; a.ldx = g.ldx; a.R = g.R; a.K = g.K;
    const bool dual = g.mode == SKINNY_DUAL;
    bool vec = whole_pieces(dm, g.K) && whole_pieces(dm, g.ldx) && aligned16(g.X);
    int end = 0;
    for (int s = 0; s < 3; ++s) {
        a.W[s] = g.W[s];
        if (g.W[s]) vec = vec && aligned16(g.W[s]);
        if (!dual) end += g.n[s];
        a.n_end[s] = dual ? g.n[0] : end;
    }
    a.B[0] = g.B[0]; a.B[1] = g.B[1]; a.t = !g.A[0] && !g.A[1] && (g.B[0] || g.B[1]) ? g.t : nullptr; a.r = dm.r; a.row_model = g.row_model;
    a.resid = g.resid; a.Y = g.Y; a.ldy = g.ldy;
    a.wn = g.wn; a.eps = dm.eps; a.A[0] = g.A[0]; a.A[1] = g.A[1]; a.scale = dm.lora_scale;
    const bool shrink = g.A[0] || g.A[1];
    const int N = a.n_end[dual ? 0 : 2], per_wg = 4 * (dual ? kCols / 2 : kCols);
    if (N <= 0) return hipSuccess;
    const dim3 grid((N + per_wg - 1) / per_wg);
    if (g.wn || shrink) {
        if (!skinny_takes_rows(dm, g) || !vec) return hipErrorInvalidValue;
        auto rows = [&](auto rm, auto with_shrink) {
            constexpr int RM = decltype(rm)::value;
            constexpr bool SH = decltype(with_shrink)::value;
            switch (g.mode) {
            case SKINNY_F32: hipLaunchKernelGGL((k_gemm_skinny<float, Vec16<float>, RM, SKINNY_F32, true, SH>), grid, dim3(256), 0, st, a); break;
            case SKINNY_RESID:
                if constexpr (SH) hipLaunchKernelGGL((k_gemm_skinny<float, Vec16<float>, RM, SKINNY_RESID, false, true>), grid, dim3(256), 0, st, a);
                break;
            default: hipLaunchKernelGGL((k_gemm_skinny<float, Vec16<float>, RM, SKINNY_DUAL, true, SH>), grid, dim3(256), 0, st, a); break;
            }
            return hipGetLastError();
        };
        if (shrink) return rows(std::integral_constant<int, 4>(), std::true_type());
        if (g.R <= 4) return rows(std::integral_constant<int, 4>(), std::false_type());
        if (g.R <= 8) return rows(std::integral_constant<int, 8>(), std::false_type());
        return rows(std::integral_constant<int, 16>(), std::false_type());
    }
    return with_type(dm.bf16, vec, [&](auto tt, auto vv) {
        typedef decltype(tt) T;
        typedef decltype(vv) V;
        auto rows = [&](auto rm) {
            constexpr int RM = decltype(rm)::value;
            switch (g.mode) {
            case SKINNY_F32: hipLaunchKernelGGL((k_gemm_skinny<T, V, RM, SKINNY_F32>), grid, dim3(256), 0, st, a); break;
            case SKINNY_RESID: hipLaunchKernelGGL((k_gemm_skinny<T, V, RM, SKINNY_RESID>), grid, dim3(256), 0, st, a); break;
            default: hipLaunchKernelGGL((k_gemm_skinny<T, V, RM, SKINNY_DUAL>), grid, dim3(256), 0, st, a); break;
            }
            return hipGetLastError();
        };
        if (g.R <= 4) return rows(std::integral_constant<int, 4>());
        if (g.R <= 8) return rows(std::integral_constant<int, 8>());
        return rows(std::integral_constant<int, 16>());
    });
}

}  // namespace icarus
