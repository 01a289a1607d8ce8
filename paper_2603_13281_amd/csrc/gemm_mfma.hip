// ICaRusLinear on gfx950 matrix cores: one base-weight GEMM over all stacked rows with the
// per-model LoRA delta folded in as extra K-steps (bf16 storage, fp32 accumulation).
//
//   Y[R, N] = X[R, K] . W[N, K]^T  +  T[R, M*r] . Bcat[N, M*r]^T
//
// T is the masked shrink result: T[row, j*r + i] = s * (A_j x_row)_i if row belongs to model j, else 0
// (encoder rows are all zero), so multiplying by the concatenation of every model's B applies to
// each row exactly its own adapter.  The extension costs M*r extra K on top of K (3-5 %) and needs
// no row reordering: the base weights are still read once for all streams (Alg. 2).
//
// Tiling: a workgroup of WAVES_M x WAVES_N waves owns a BM x BN output tile; each wave a
// (BM/WAVES_M) x (BN/WAVES_N) sub-tile of 32x32x16 bf16 MFMAs.  K advances BK at a time through a
// ring of NS LDS stages filled by 16-byte LDS-direct loads (global memory -> LDS without passing
// through registers), so NS-1 slabs are in flight or landed while one is computed and one barrier
// per slab suffices.  Inside LDS the 16-byte chunks of each 256-byte line are XOR-swizzled with
// the line number: the wave-wide loads write 1 KiB contiguously, and the MFMA fragment reads
// (16 bytes per lane, 32 consecutive rows) spread over all banks.  Every load reads an always-valid
// address (rows and columns past the matrix are clamped: they only feed outputs that are never
// stored; chunks that must read as zeros come from a page of zeros), so the K loop is branch-free
// apart from the switch from base-weight slabs to adapter slabs.
//
// MFMA 32x32x16 bf16 operand layout (lane l): A[row l%32][k 8(l/32)..+7], B[k 8(l/32)..+7][col l%32],
// C[row 8(r/4) + 4(l/32) + r%4][col l%32] for accumulator register r = 0..15.
#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "gemm_tile.h"

namespace icarus {

namespace {

constexpr int kKAlign = 64;  // K of every GEMM is a multiple of this

template <int BM, int BN, int BK, int NS, int WAVES_M, int WAVES_N, bool GROUPED>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N) k_gemm_mfma(GemmArgs g) {
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;  // wave tile
    constexpr int TM = WM / 32, TN = WN / 32;            // 32x32 MFMA tiles per wave
    constexpr int CPR = BK / 8;                          // 16-byte chunks per tile row
    constexpr int RPU = 64 / CPR;                        // tile rows per 1 KiB unit (one wave-wide load)
    constexpr int A_LD = BM / RPU / NW, B_LD = BN / RPU / NW;  // loads per wave and slab
    constexpr int NL = A_LD + B_LD;
    constexpr int kBOff = BM * BK * 2, kStage = (BM + BN) * BK * 2;
    static_assert(BM % (RPU * NW) == 0 && BN % (RPU * NW) == 0, "tile / wave mismatch");
    static_assert(TM >= 1 && TN >= 1 && NS >= 2 && NS <= 5 && (NS - 2) * NL < 64, "tile shape");
    extern __shared__ __attribute__((aligned(1024))) char smem[];  // [NS] stages of { A [BM][BK], B [BN][BK] }
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)smem;

    // XCD-aware tile order.  The 8 XCDs take workgroups round-robin and each runs about 32 of them
    // at a time (one per CU).  The tile grid of every K slice is cut into panels of panel_m x panel_n
    // <= 32 tiles; consecutive workgroups of one XCD work on one panel, so that what they stream
    // through that XCD's L2 at any moment is panel_m slabs of X and panel_n slabs of W instead of one
    // of each per tile.  Consecutive panels (on different XCDs at the same time) walk down the rows
    // first, sharing their weight columns in the memory-side cache, then the slices.
    int tile_m, tile_n, kz;
    if (!tile_of_workgroup(g, &tile_m, &tile_n, &kz)) return;
    const int k_begin = kz * g.k_per_split;
    const int k_end = min(g.K_ext, k_begin + g.k_per_split);
    const int nk = (k_end - k_begin + BK - 1) / BK;

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w / WAVES_N, wn = w % WAVES_N;
    // rows [row0, row_end) of this tile, and the weights they are multiplied with
    int row0 = tile_m * BM, row_end = g.R;
    const bf16_t *W0 = g.W[0], *W1 = g.W[1];
    if constexpr (GROUPED) {
        row0 = g.row_tiles[3 * tile_m];
        row_end = g.row_tiles[3 * tile_m + 1];
        const int grp = g.row_tiles[3 * tile_m + 2];
        if (grp > 0) {
            W0 = g.Wg[0] + (size_t)(grp - 1) * g.wg_stride;
            W1 = g.Wg[1] + (size_t)(grp - 1) * g.wg_stride;
        }
    }

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // This lane's part of every wave-wide load: LDS slot `lane` of a 1 KiB unit is 256-byte line
    // lane/16, position lane%16, which (un-swizzled) holds chunk kc/8 of unit row ru.  A wave's units
    // are NW apart (NW even), so the swizzle key of its lines is the same for every unit.  Row
    // sources are fixed for the whole K loop: base-K slabs read pointer + k, the few adapter slabs
    // past K read T (activation side) and the models' B (weight side), or the zero page.
    static_assert(NW % 2 == 0, "swizzle key must not depend on the unit");
    const int lin = lane >> 4, key = (w * 4 + lin) & (CPR - 1);
    const int qd = lin * 16 + ((lane & 15) ^ key);
    const int ru = qd / CPR, kc = (qd % CPR) * 8;
    const bf16_t *zero = (const bf16_t *)g_zero_page;
    const bf16_t *pa[A_LD], *pt[A_LD];
    BRow br[B_LD];
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
        int row = min(row0 + (w + NW * i) * RPU + ru, row_end - 1);  // clamped rows feed outputs that are never stored
        pa[i] = g.X + (size_t)row * g.ldx + kc;
        pt[i] = g.T ? g.T + (size_t)row * g.ldt + kc : zero;
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
        br[i] = b_row<BN, WN>(g, W0, W1, tile_n, (w + NW * i) * RPU + ru);
        br[i].w += kc;
    }
    const int K_base = g.K, mr = g.M_models * g.r, lr = 31 - __clz(max(g.r, 1)), ldt = g.T ? g.ldt : 0;
    const int rmask = g.r - 1;
    const size_t model_stride = (size_t)g.n_seg[0] * g.r;  // elements between consecutive models' B

    const int n_base = min(nk, max(0, (K_base - k_begin) / BK)), turn = gemm_turn(g, tile_n, n_base);
    auto k_of = [&](int kt) { return k_begin + (kt < n_base ? gemm_slab(kt, turn, n_base) : kt) * BK; };
    // enqueue the loads of slab kt into ring stage `stage`
    auto issue = [&](int kt, int stage) {
        const int k0 = k_of(kt);
        const uint32_t la = lds0 + stage * kStage + w * 1024;
        if (k0 < K_base) {  // slab inside the base weights (K is a multiple of the slab)
#pragma unroll
            for (int i = 0; i < A_LD; ++i) dma16(pa[i] + k0, la + i * (NW * 1024));
#pragma unroll
            for (int i = 0; i < B_LD; ++i) dma16(br[i].w + k0, la + kBOff + i * (NW * 1024));
            return;
        }
        const int k2 = k0 - K_base + kc;  // this lane's adapter column (r is a power of two)
#pragma unroll
        for (int i = 0; i < A_LD; ++i) dma16(k2 < ldt ? pt[i] + (k2 - kc) : zero, la + i * (NW * 1024));
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
            int kk = k2 - (br[i].kind == 2 ? mr : 0);
            bool ok = br[i].kind != 0 && kk >= 0 && kk < mr;
            dma16(ok ? br[i].b + (size_t)(kk >> lr) * model_stride + (kk & rmask) : zero, la + kBOff + i * (NW * 1024));
        }
    };

    const int fr = lane & 31, fh = lane >> 5;
    constexpr int KS = BK / 16;
    static_assert(KS % 2 == 0, "the two fragment sets alternate over the K steps of a slab");
    // Two fragment sets used alternately: while the MFMAs of one K step run from one set, the reads of
    // the next step fill the other.  A wave issues in order and an MFMA holds the issue slot until the
    // matrix pipe takes it, so the reads must be issued BEFORE the MFMAs they are to overlap with; the
    // compiler, left alone, sinks them behind the MFMAs to save the second set (measured on a bare loop:
    // 63 % of the matrix pipe's rate with 4 waves per CU, 87 % with the order pinned), hence the
    // scheduling barriers.
    bf16x8 fa[2][TM], fb[2][TN];
    auto read_frags = [&](int stage, int ks, bf16x8 (&af)[TM], bf16x8 (&bfr)[TN]) {
        const char *sA = smem + stage * kStage, *sB = sA + kBOff;
#pragma unroll
        for (int i = 0; i < TM; ++i) af[i] = *(const bf16x8 *)(sA + swz<CPR>(wm * WM + i * 32 + fr, 2 * ks + fh));
#pragma unroll
        for (int j = 0; j < TN; ++j) bfr[j] = *(const bf16x8 *)(sB + swz<CPR>(wn * WN + j * 32 + fr, 2 * ks + fh));
    };
    auto mma = [&](const bf16x8 (&af)[TM], const bf16x8 (&bfr)[TN]) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    };
    // K steps 0 .. KS-2 of the slab in `stage`; set 0 holds step 0 on entry, set 1 holds step KS-1 on exit.
    // A wave issues in order, and an LDS read that the LDS cannot take yet blocks the MFMAs behind it while the
    // matrix pipe runs dry; so each fragment read of the next step sits right behind an MFMA of this one, whose
    // passes cover it (a batch of reads ahead of the MFMAs cost the sum of both).
    auto slab_head = [&](int stage) {
        const char *sA = smem + stage * kStage, *sB = sA + kBOff;
#pragma unroll
        for (int ks = 0; ks + 1 < KS; ++ks) {
            const int cur = ks & 1, nxt = cur ^ 1;
#pragma unroll
            for (int m = 0; m < TM * TN; ++m) {
                const int i = m / TN, j = m % TN;
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][i], fb[cur][j], acc[i][j], 0, 0, 0);
                if (TM * TN >= TM + TN) {
                    if (m < TM) fa[nxt][m] = *(const bf16x8 *)(sA + swz<CPR>(wm * WM + m * 32 + fr, 2 * (ks + 1) + fh));
                    else if (m < TM + TN) fb[nxt][m - TM] = *(const bf16x8 *)(sB + swz<CPR>(wn * WN + (m - TM) * 32 + fr, 2 * (ks + 1) + fh));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (TM * TN < TM + TN) read_frags(stage, ks + 1, fa[nxt], fb[nxt]);  // tiles with fewer MFMAs than fragments
        }
    };
    auto wait_for_slab = [&](int younger) {  // younger: slabs enqueued after the one waited for
        if (NS > 4 && younger >= 3) wait_loads<(NS > 4 ? 3 : 0) * NL>();
        else if (NS > 3 && younger >= 2) wait_loads<(NS > 3 ? 2 : 0) * NL>();
        else if (younger >= 1) wait_loads<NL>();
        else wait_loads<0>();
    };
    // Ring of NS stages.  One barrier per slab, placed before the last 16-wide K step of slab kt is
    // multiplied: by then every wave has read all of slab kt into registers, so after the barrier
    // (which also follows each wave's wait for its own loads of slab kt+1) slab kt+1 is complete
    // in LDS and the stage of slab kt can be refilled with slab kt+NS.  The first fragments of slab
    // kt+1 are fetched right after the barrier and the pending MFMAs of slab kt cover their latency,
    // the refill's issue and the barrier's wake-up.
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < nk) issue(s, s);
    wait_for_slab(min(NS - 2, nk - 1));
    __builtin_amdgcn_s_barrier();
    if (NS - 1 < nk) issue(NS - 1, NS - 1);
    read_frags(0, 0, fa[0], fb[0]);
    int stage = 0, kt = 0;
    // Steady state: the slab to enqueue (kt+NS) lies in the base weights, so the section after the
    // barrier is straight-line code: the first fragments of slab kt+1, then the pending MFMAs of slab
    // kt alternating with the loads of slab kt+NS, so that the matrix pipe is fed while the wave
    // issues its memory instructions.
    const int n_steady = n_base - NS;
    for (; kt < n_steady; ++kt) {
        slab_head(stage);
        const int next = stage + 1 == NS ? 0 : stage + 1;
        wait_loads<(NS - 2) * NL>();
        __builtin_amdgcn_s_barrier();
        read_frags(next, 0, fa[0], fb[0]);
        const int k0 = k_begin + gemm_slab(kt + NS, turn, n_base) * BK;
        const uint32_t la = lds0 + stage * kStage + w * 1024;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < TM * TN; ++t) {
            acc[t / TN][t % TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[1][t / TN], fb[1][t % TN], acc[t / TN][t % TN], 0, 0, 0);
#pragma unroll
            for (int l = t * NL / (TM * TN); l < (t + 1) * NL / (TM * TN); ++l) {
                if (l < A_LD) dma16(pa[l] + k0, la + l * (NW * 1024));
                else dma16(br[l - A_LD].w + k0, la + kBOff + (l - A_LD) * (NW * 1024));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        stage = next;
    }
    for (; kt < nk; ++kt) {  // the last slabs: adapter columns to enqueue, or nothing left to enqueue
        slab_head(stage);
        const int next = stage + 1 == NS ? 0 : stage + 1;
        if (kt + 1 < nk) {
            wait_for_slab(min(NS - 2, nk - 2 - kt));
            __builtin_amdgcn_s_barrier();
            read_frags(next, 0, fa[0], fb[0]);
            __builtin_amdgcn_sched_barrier(0);
            if (kt + NS < nk) issue(kt + NS, stage);
        }
        mma(fa[1], fb[1]);
        __builtin_amdgcn_sched_barrier(0);
        stage = next;
    }

    __syncthreads();  // every wave has left the K loop: the ring is the epilogue's scratch
    static_assert(NW * 32 * (WN + 8) * 4 <= NS * kStage, "epilogue scratch must fit the ring");
    store_wave_tile<32, TM, TN, BN>(g, acc, (float *)smem + w * 32 * (WN + 8), tile_n, kz, row0 + wm * WM, row_end, wn);
}

// Second pass of a split-K GEMM: sum the fp32 partials P[z][row][n] and apply the epilogue.
__global__ void __launch_bounds__(256) k_splitk_reduce(const float *__restrict__ P, int splits, int R, int N, int epi,
                                                       void *__restrict__ Y, int ldy, const bf16_t *__restrict__ resid, int ldr) {
    size_t idx = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (idx >= (size_t)R * N) return;
    int row = (int)(idx / N), n = (int)(idx % N);  // N is a multiple of 4
    float4 v = {0.f, 0.f, 0.f, 0.f};
    for (int z = 0; z < splits; ++z) {
        float4 p = *(const float4 *)(P + ((size_t)z * R + row) * N + n);
        v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
    }
    if (epi == EPI_F32) {
        *(float4 *)((float *)Y + (size_t)row * ldy + n) = v;
    } else {
        const bf16_t *rp = resid + (size_t)row * ldr + n;
        bf16_t *yp = (bf16_t *)Y + (size_t)row * ldy + n;
        const uint2 r = *(const uint2 *)rp;  // rows and columns in fours: 8-byte aligned
        *(uint2 *)yp = make_uint2(pack_bf16(v.x + __uint_as_float(r.x << 16), v.y + __uint_as_float(r.x & 0xffff0000u)),
                                  pack_bf16(v.z + __uint_as_float(r.y << 16), v.w + __uint_as_float(r.y & 0xffff0000u)));
    }
}

// The matrix pipe alone: 8 independent accumulators per wave, operands fixed in registers.
__global__ void __launch_bounds__(256) k_bench_mfma(float *__restrict__ out, int iters) {
    const int lane = threadIdx.x & 63;
    bf16x8 a, b;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        a[e] = (__bf16)(0.001f * (float)((lane + e) % 7));
        b[e] = (__bf16)(0.002f * (float)((lane + 2 * e) % 5));
    }
    f32x16 acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[t], 0, 0, 0);
    }
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) s += acc[t][r];
    out[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
}

template <int BM, int BN, int BK, int NS, int WAVES_M, int WAVES_N, bool GROUPED = false>
hipError_t launch_cfg(GemmArgs g, hipStream_t st) {
    g.m_tiles = GROUPED ? g.n_row_tiles : (g.R + BM - 1) / BM;
    g.n_tiles = 0;
    if (g.mode == GEMM_DUAL) {
        g.n_tiles = (g.n_seg[0] + BN / 2 - 1) / (BN / 2);
    } else {
        for (int s = 0; s < g.nseg; ++s) {
            g.tiles_seg[s] = (g.n_seg[s] + BN - 1) / BN;
            g.n_tiles += g.tiles_seg[s];
        }
    }
    constexpr size_t shm = (size_t)NS * (BM + BN) * BK * sizeof(bf16_t);
    gemm_set_panels(&g, BM, BN, (int)(((size_t)160 << 10) / shm));
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)k_gemm_mfma<BM, BN, BK, NS, WAVES_M, WAVES_N, GROUPED>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    dim3 grid(gemm_grid(g));
    hipLaunchKernelGGL((k_gemm_mfma<BM, BN, BK, NS, WAVES_M, WAVES_N, GROUPED>), grid, dim3(64 * WAVES_M * WAVES_N), shm, st, g);
    return hipGetLastError();
}

// Tile shapes: rows x weight rows of a workgroup, all with 64-wide K slabs (32-wide slabs ask for every 128-byte line of
// a weight row twice, half each time, and stream at about 60 % of the rate).  The first two are k_gemm_mfma (128 x 128 of more than
// one row tile: k_gemm_quad, see in_quadrants), the others k_gemm_quad (192 x 128: gemm_quad.hip may take lower tiles, and see launch_gemm_mfma).  first_us: what a workgroup takes apart from its slabs (start, first slab, epilogue); slab_us: a slab
// with every CU busy, for each of the per_cu workgroups that share one.  The figures are a fit to 5000 timings on
// this GPU (80-4337 rows x the projections of a Llama-3-8B- and a Qwen3-32B-shaped layer x every tile x 1-12 slices; the
// fit is 7-11 % off on average), see gemm_plan and gemm_row_tile.  They are of the kernels before k_gemm_quad, and
// count one 192 x 128 workgroup to a CU where two now fit.  What they are for, the order of the choices, holds for the present ones (144-1100 rows,
// 12 counts, of the four projections of both layers, every tile and slice count timed anew with weights from HBM: the choice is 1.6 % from the fastest on
// average and within 5 % in 87 of 96; 250 rows, 5120 -> 10240 55.9 us where three slices of 160 x 256 take 39.6 + their sums, 512 rows, 14336 -> 4096 74.5
// and 8 of 256 x 256 55.6 + sums); as times they are up to 16 % high.
struct TileShape { int bm, bn, per_cu; float first_us, slab_us; };
constexpr TileShape kTileShape[TILE_KINDS] = {
    {0, 0, 0, 0.f, 0.f},
    {64, 128, 2, 2.0f, 0.77f},
    {128, 128, 1, 3.8f, 0.60f},
    {192, 128, 1, 4.7f, 0.77f},
    {256, 256, 1, 7.8f, 1.65f},
    {192, 256, 1, 10.2f, 1.26f},
    {160, 256, 1, 9.3f, 1.13f},
};

int n_tiles_for(const GemmArgs &g, int bm, int bn) {
    int m_tiles = (g.R + bm - 1) / bm, n_tiles = 0;
    if (g.mode == GEMM_DUAL) return m_tiles * ((g.n_seg[0] + bn / 2 - 1) / (bn / 2));
    for (int s = 0; s < g.nseg; ++s) n_tiles += (g.n_seg[s] + bn - 1) / bn;
    return m_tiles * n_tiles;
}

// Whether the workgroups of a launch take their slabs of the weights from different places along K (gemm_turn), column tile n from
// slab n on.  Started all at the same one, they ask at any moment for the same few columns of every weight row; where the rows
// are a multiple of 4 KB apart that is a few bits of the address, and what the memory channels make of it depends on where the
// matrices lie.  Column tile n + 1 starts one slab behind n, so that an XCD's workgroups still pass over the same slabs of X within a few slabs'
// time (starts a golden section apart were as good up to 64 rows but cost 316 rows, 14336 -> 4096 25 %).  us, same / different starts, weights
// from HBM in 3-13 places: 4096 -> 2 x 14336, 9-64 rows 43.6-60 / 46.8-51, mean 53.4 / 47, 128 rows 58.6 / 54.5, 144 rows 61.2 / 58.5, 316 rows 82.5 / 78; LM head
// 4096 -> 128256, 9 rows 196 / 177, 64 rows 221 / 198; 6144 -> 2 x 8192, 9 rows 56 / 51; 14336 -> 4096 and 4096 -> 4096 in slices equal; 576 and 753 rows equal (bound by
// the matrix cores).  Rows 10 KB apart (5120 -> 2 x 25600) 107.6 / 109.7, 120.4 / 121.5.  Groups of rows with weights of their own, steps of 9-360 rows: 4096 columns within
// the runs' 3 %, 2048 columns, 330 rows 279 / 268.
bool gemm_staggered(const GemmArgs &g) { return g.K % 2048 == 0 && g.R <= 384; }

bool is_quad(int kind) { return kind >= TILE_192x128; }

// Launches of gemm_quad.hip: 128 x 128 tiles too where there is more than one row tile.  A single one waits for its weights and takes the deeper
// ring of k_gemm_mfma, as do groups of rows.
bool in_quadrants(const GemmArgs &g, int tile) {
    return std::max(g.K, g.ldx) <= kQuadMaxK && (is_quad(tile) || (tile == TILE_128 && g.R > 128 && !g.row_tiles));
}

int k_ext_of(const GemmArgs &g) {
    if (g.mode == GEMM_DUAL) return g.K + (g.T ? 2 * g.M_models * g.r : 0);
    return g.K + ((g.T && g.B[0]) ? g.M_models * g.r : 0);
}

// Modelled time of a launch, in us, for tiles with a CU of their own: rounds of workgroups over the 256 CUs; a round that
// leaves CUs idle has faster slabs.
float model_us(const GemmArgs &g, int kind, int splits) {
    const TileShape &t = kTileShape[kind];
    const int slabs = (k_ext_of(g) + kKAlign - 1) / kKAlign, per_slice = (slabs + splits - 1) / splits;
    const int64_t wgs = (int64_t)n_tiles_for(g, t.bm, t.bn) * splits;
    auto round = [&](int64_t n) { return n ? t.first_us + (float)per_slice * t.slab_us * (0.75f + 0.25f * (float)n / 256.f) : 0.f; };
    return (float)(wgs / 256) * round(256) + round(wgs % 256);
}

}  // namespace

// Panels of the XCD-aware tile order (see k_gemm_mfma) for bm x bn tiles, per_cu workgroups to a CU.  The panels of all
// K slices are dealt to the 8 XCDs in turn, so what an XCD gets is a whole number of panels: the shape is the one that
// keeps the fullest XCD's workgroups within the fewest rounds of its 32 CUs, and among those the one that streams the
// fewest bytes per tile through the XCD's L2.  (With panels always as large as the grid allows, 20 column tiles in 12
// slices made 10 panels, two for two of the XCDs and one for the others; 9 row tiles made panels of 8 and 1 rows, which
// alternate over the XCDs: 144 rows, 25600 -> 5120 in 160 x 256 tiles 102 us -> 70 us; 2100 rows, gate/up
// 14336 x 2 in 256 x 256 tiles 579 -> 442 us.)
void gemm_set_panels(GemmArgs *g, int bm, int bn, int per_cu) {
    const int Mt = g->m_tiles, Nt = g->n_tiles, splits = std::max(1, g->splits), cap = 32 * per_cu;
    float best = 0.f;
    g->panel_m = 0;
    for (int m = 1; m <= std::min(Mt, 8); ++m) {
        const int pms = (Mt + m - 1) / m, pm = (Mt + pms - 1) / pms;
        if (pm != m) continue;  // the same height is reached with a smaller m
        for (int n = 1; n <= std::min(Nt, 32 / m); ++n) {
            const int pns = (Nt + n - 1) / n, pn = (Nt + pns - 1) / pns;
            if (pn != n) continue;
            const int64_t fullest = ((int64_t)pms * pns * splits + 7) / 8 * (pm * pn);
            const float load = (float)fullest / (float)cap;  // a last round that is only partly filled is also a faster one
            const float rounds = fullest <= cap ? load : 0.5f * (load + (float)((fullest + cap - 1) / cap));
            const float bytes = (float)(pm * bm + pn * bn) / (float)((bm + bn) * pm * pn);  // of a tile on its own
            float score = rounds * (1.f + 0.5f * bytes);
            if (splits > 1 && pms * pns % 8) score *= 1.06f;  // else an XCD works on the same tiles in every slice
            if (!g->panel_m || score < best) {
                best = score;
                g->panel_m = pm; g->panel_n = pn; g->panels_m = pms; g->n_panels = pms * pns;
            }
        }
    }
    g->inv_panels = gemm_inv(g->n_panels);
    g->inv_panels_m = gemm_inv(g->panels_m);
    g->inv_panel_m = gemm_inv(g->panel_m);
}

bool gemm_mfma_supported(const Dims &dm, int K) {
    bool r_ok = dm.r == 0 || (dm.r >= 8 && (dm.r & (dm.r - 1)) == 0);  // adapter rank: a power of two >= 8
    // every output width must be a multiple of 8 (16-byte stores of the epilogue)
    bool n_ok = dm.d % 8 == 0 && dm.F % 8 == 0 && (dm.Hq * dm.D) % 8 == 0 && (dm.Hkv * dm.D) % 8 == 0;
    return dm.bf16 && K % kKAlign == 0 && r_ok && n_ok;
}

// Tile and number of K slices of a GEMM.
//
// Up to 128 rows the weights' way from HBM is what counts: one row tile, 128 wide (64 x 256 tiles for up to 64 rows of an LM
// head: within 3 % either way at up to two rounds of CUs, 2-10 % slower where the last round is short -- 151936 and 202048 outputs --
// and for K = 4096), and so many slices that about one workgroup per
// CU streams them (more slices were measured: their partial sums cost more than the depth in flight brings; fewer, as
// the model below would have it from timings with cached weights, cost a step of 90 rows 1 %).
//
// Beyond that the choice is the smallest modelled time over the tiles and slice counts (model_us + the partial sums'
// way through memory and, where no later kernel takes the slices as they are, a launch).  Near ties are decided by what
// the model does not know -- how the strides of the slices fall on the HBM channels, what the row kernel after a sliced
// projection pays, what the wide tiles do to the clock -- so the plain choice has a start.  The modelled time has to
// undercut by 3 %: up to 384 rows of a narrow output, 192-row tiles in as many slices as the CUs hold at once; from 1024
// rows, 256 x 256 tiles that fill most of the CUs.  In between, slices have to earn 3 %.
// Measured inside a layer, weights from HBM, consumers of the slices included (5 widths of 2048-8192, 130-32768 rows, QKV, O,
// gate/up, down: 1316 launches, every tile x 1-12 slices): within 0.6 % of the fastest on average, 18 % at worst (252 rows,
// 5120 -> 10240).  Without the start for the plain choice 28 of them were 2-29 % slower than one tile for each range of
// row counts (162 rows, 28672 -> 8192: 152 us in 192 x 256 tiles, 118 us in 192 x 128; 10000 rows, 4096 -> 4096: 349 us in
// 160 x 256, 327 us in 256 x 256); with it 9, by 7 % at most.  The fixed tiles in turn are 10 % from the fastest on
// average (512 rows, 25600 -> 5120: 233 us in 128 x 128 tiles, 144 us in 256 x 256 and 6 slices; 4337 rows, 14336 -> 4096,
// whose 272 tiles of 256 x 256 need two rounds of 256 CUs: 616 us, in 160 x 256 tiles 486 us).
GemmPlan gemm_plan(const GemmArgs &g, int max_splits, bool takes_slices) {
    int n_total = 0;
    for (int s = 0; s < g.nseg; ++s) n_total += g.n_seg[s];
    const int slabs = (k_ext_of(g) + kKAlign - 1) / kKAlign;
    if (g.R <= 128) {
        const int kind = g.R <= 64 ? TILE_64x128 : TILE_128;
        const int tiles = n_tiles_for(g, kTileShape[kind].bm, kTileShape[kind].bn);
        int splits = tiles < 160 ? std::min({max_splits, 256 / tiles, slabs / 4}) : 1;
        return {kind, std::max(1, splits)};
    }
    auto modelled = [&](int kind, int splits) {
        const float mb = (float)g.R * (float)n_total * 4e-6f;  // one slice
        return model_us(g, kind, splits) + (splits > 1 ? mb * splits * 0.38f + (takes_slices ? 0.f : 4.f + mb * 0.2f) : 0.f);
    };
    const bool few = g.R <= 384;
    GemmPlan best{TILE_128, 1};
    float best_us = -1.f;
    if (few && g.mode != GEMM_DUAL && n_tiles_for(g, 192, 256) < 160) {
        const int tiles = n_tiles_for(g, 192, 128);
        best = {TILE_192x128, tiles < 160 ? std::max(1, std::min({max_splits, 256 / tiles, slabs / 4})) : 1};
        best_us = 0.97f * modelled(best.tile, best.splits);
    } else if (g.R >= 1024 && n_tiles_for(g, 256, 256) >= 192) {
        best = {TILE_256x256, 1};
        best_us = 0.97f * modelled(best.tile, best.splits);
    }
    for (int kind = TILE_128; kind < TILE_KINDS; ++kind) {  // several row tiles of 64 would read the weights again
        for (int splits = 1; splits <= max_splits; ++splits) {
            if (splits > 1) {
                const int per = (slabs + splits - 1) / splits;
                if (per < 6) break;
                if ((slabs + per - 1) / per != splits) continue;  // the last slice would be empty
            }
            const float us = modelled(kind, splits) * (splits > 1 && !few && g.R < 1024 ? 1.03f : 1.f);
            if (best_us < 0.f || us < best_us) { best_us = us; best = {kind, splits}; }
        }
    }
    return best;
}

// Tile of a grouped launch: the one whose row tiles together cost the fewest slabs.  off: first row of each group and the end
// of the last.  Each row tile reads its group's weights once, so with a few rows per group the smallest tile that holds most
// groups wins, with hundreds the large one.  Gate and up of 9 groups (4096 -> 2 x 14336), us in 64 x 128 / 128 x 128 / 192 x 128 /
// 256 x 256 tiles: groups of 66 rows 474 / 404 / 449 / 488, one of 300 and eight of 38 rows 392 / 448 / 488 / 559, groups of
// 130 rows 622 / 662 / 471 / 503, of 256 rows 855 / 710 / 863 / 531, of 1024 rows 3037 / 2604 / 2551 / 1785 (2014 in a launch
// of 256 x 256 tiles per group).
int gemm_row_tile(const int *off, int n_groups) {
    int best = TILE_64x128;
    float best_cost = -1.f;
    for (int kind : {TILE_64x128, TILE_128, TILE_192x128, TILE_256x256}) {
        const TileShape &t = kTileShape[kind];
        int64_t tiles = 0;
        for (int j = 0; j < n_groups; ++j) tiles += (off[j + 1] - off[j] + t.bm - 1) / t.bm;
        const float cost = (float)tiles * t.slab_us / (float)(t.bn * t.per_cu);
        if (best_cost < 0.f || cost < best_cost) { best_cost = cost; best = kind; }
    }
    return best;
}
int gemm_tile_rows(int tile) { return kTileShape[tile].bm; }
int gemm_tile_cols(int tile) { return kTileShape[tile].bn; }
bool gemm_tile_marked(int tile) { return tile >= TILE_192x256; }

// K slices of a grouped launch.  With a weight matrix per group it is bound by their way from HBM, like a GEMM of few
// rows, and by the last round: 9 groups x 32 column tiles on 512 workgroup slots leave 32 CUs with twice the work of
// the others (346 rows, 14336 -> 4096: 259 us whole, 207 us in 7 slices + 10 us for their sum).  The smallest modelled time:
// with weights from HBM a 64-row workgroup takes 0.85 us a slab alone on its CU, 1.4 us when two share one (which is HBM's
// rate for 16 KB of weights each), the others a quarter more than slab_us; the slices' way through memory as in gemm_plan.
int gemm_grouped_splits(const GemmArgs &g, int max_splits, bool takes_slices) {
    if (g.mode == GEMM_DUAL) return 1;
    const TileShape &t = kTileShape[g.tile];
    int n_tiles = 0, n_total = 0;
    for (int s = 0; s < g.nseg; ++s) {
        n_tiles += (g.n_seg[s] + t.bn - 1) / t.bn;
        n_total += g.n_seg[s];
    }
    const int slabs = g.K / kKAlign, cap = 256 * t.per_cu;
    const float mb = (float)g.R * (float)n_total * 4e-6f;
    int best = 1;
    float best_us = -1.f;
    for (int splits = 1; splits <= max_splits; ++splits) {
        const int per = (slabs + splits - 1) / splits, wgs = g.n_row_tiles * n_tiles * splits;
        if (splits > 1 && (per < 4 || (slabs + per - 1) / per != splits)) continue;
        auto round = [&](int n) {
            if (n == 0) return 0.f;
            const float slab = t.per_cu == 1 ? 1.25f * t.slab_us : n <= 256 ? 0.85f : 1.4f;
            return t.first_us + (float)per * slab;
        };
        float us = (float)(wgs / cap) * round(cap) + round(wgs % cap);
        if (splits > 1) us += mb * splits * (0.22f + 0.2f) + (takes_slices ? 0.f : 4.f + mb * 0.2f);
        if (best_us < 0.f || us < best_us) { best_us = us; best = splits; }
    }
    return best;
}

hipError_t launch_gemm_mfma(GemmArgs g, hipStream_t st) {
    if (g.R <= 0) return hipSuccess;
    if (g.K % kKAlign) return hipErrorInvalidValue;
    if (g.splits < 1) g.splits = 1;
    if (g.slice_rows < g.R) g.slice_rows = g.R;
    if (g.row_tiles && (g.tile < TILE_64x128 || g.tile > TILE_256x256)) return hipErrorInvalidValue;
    if (g.tile == TILE_AUTO) g.tile = gemm_plan(g, 1, false).tile;
    if (is_quad(g.tile) && std::max(g.K, g.ldx) > kQuadMaxK) {
        if (g.row_tiles) return hipErrorInvalidValue;
        g.tile = TILE_128;
    }
    g.K_ext = k_ext_of(g);
    g.k_per_split = ((g.K_ext + g.splits - 1) / g.splits + kKAlign - 1) / kKAlign * kKAlign;
    g.stagger = gemm_staggered(g) ? gemm_inv(std::min(g.k_per_split, g.K) / kKAlign) : 0u;
    // Tiles of 192 rows by 128 that are needed in full (gemm_quad.hip has lower ones), with adapters: the slabs of adapter columns are
    // code that a workgroup of k_gemm_quad runs once, fetched as it goes (a form with fewer instructions per load but more of them in
    // all took 1.3 us longer still); four such slabs cost 1.3-2 us more there than in this kernel's loop, which only a long K earns back.  us with 8
    // adapters of rank 32, this kernel / that: 171-189 rows, 5120 -> 10240 in 3 slices 38.3 / 40.9, 8192 -> 5120 in 6 32.1 / 34.6; 324-378
    // rows, 8192 -> 5120 in 3 44.0 / 46.6; 370 rows, 20480 -> 5120 in 3 93.3 / 93.8; 171-189 rows, 25600 -> 5120 in 6 83.7 / 81.5.  Rank 16:
    // 180 rows, 4096 -> 6144 in 5 30.4 / 25.7; 370 rows, 4096 -> 4096 in 4 35.0 / 29.9.
    const int cols = g.K_ext - g.K;
    if (g.tile == TILE_192x128 && !g.row_tiles && g.mode == GEMM_PLAIN && g.R > 160 * ((g.R + 191) / 192) && cols >= 256 && g.K <= 64 * cols)
        return launch_cfg<192, 128, 64, 3, 2, 2>(g, st);
    if (in_quadrants(g, g.tile)) return launch_gemm_quad(g, st);
    switch (g.tile) {
    case TILE_64x128: return g.row_tiles ? launch_cfg<64, 128, 64, 3, 2, 2, true>(g, st) : launch_cfg<64, 128, 64, 3, 2, 2>(g, st);
    case TILE_128: return g.row_tiles ? launch_cfg<128, 128, 64, 4, 2, 2, true>(g, st) : launch_cfg<128, 128, 64, 4, 2, 2>(g, st);
    default: return hipErrorInvalidValue;
    }
}

bool gemm_qkv_fused(const GemmArgs &g, GemmPlan plan) {
    return plan.splits == 1 && in_quadrants(g, plan.tile) && g.nseg == 3 && !g.T && !g.row_tiles;
}
hipError_t launch_gemm_qkv(GemmArgs g, const QkvStore &e, hipStream_t st) {
    if (g.R <= 0) return hipSuccess;
    if (g.K % kKAlign || !gemm_qkv_fused(g, {g.tile, g.splits})) return hipErrorInvalidValue;
    g.slice_rows = g.R;
    g.K_ext = g.k_per_split = g.K;
    g.stagger = gemm_staggered(g) ? gemm_inv(g.K / kKAlign) : 0u;
    return launch_gemm_quad_qkv(g, e, st);
}

hipError_t launch_splitk_reduce(const float *P, int splits, int R, int N, int epi, void *Y, int ldy, const void *resid,
                                int ldr, hipStream_t st) {
    size_t quads = (size_t)R * N / 4;
    if (!quads) return hipSuccess;
    hipLaunchKernelGGL(k_splitk_reduce, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, st, P, splits, R, N, epi, Y, ldy,
                       (const bf16_t *)resid, ldr);
    return hipGetLastError();
}

hipError_t launch_bench_mfma(float *out, int waves, int iters, hipStream_t st) {
    hipLaunchKernelGGL(k_bench_mfma, dim3(waves / 4), dim3(256), 0, st, out, iters);
    return hipGetLastError();
}

}  // namespace icarus
