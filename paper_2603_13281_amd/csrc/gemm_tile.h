// Parts shared by the LDS-direct GEMM kernels (gemm_mfma.hip, gemm_quad.hip): the weight row a tile row reads, the 16-byte
// LDS-direct load and its waits, the swizzled place of a chunk in LDS, and the epilogue.
#pragma once
#include "device_util.h"
#include "kernels.h"

namespace icarus {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

namespace {

// Per-thread description of one 16-byte load of the weight (B) tile, fixed for the whole K loop.
struct BRow {
    const bf16_t *w;   // weight row + chunk offset: base-K loads are w + k
    const bf16_t *b;   // adapter B of this output column: &B[0][n][0] + chunk offset inside a model
    int kind;          // 0: no adapter columns; 1: adapter range [0, M*r); 2: range [M*r, 2*M*r) (up rows)
};

// LDS B-row b of weight tile tile_n -> weight row.  DUAL: a tile covers BN/2 output columns; inside
// each wave column of WN LDS rows the first WN/2 are gate rows and the next WN/2 the up rows of the
// same WN/2 output columns.
// W0, W1: weights of segment 0 (DUAL: gate, up), which in a grouped launch are the row group's.
template <int BN, int WN>
__device__ __forceinline__ BRow b_row(const GemmArgs &g, const bf16_t *W0, const bf16_t *W1, int tile_n, int b) {
    BRow o;
    if (g.mode == GEMM_DUAL) {
        int wn = b / WN, j = (b % WN) / (WN / 2), nn = b % (WN / 2);
        int n = min(tile_n * (BN / 2) + wn * (WN / 2) + nn, g.n_seg[0] - 1);
        o.w = (j ? W1 : W0) + (size_t)n * g.K;
        const bf16_t *B = j ? g.B[1] : g.B[0];
        o.kind = (g.T && B) ? 1 + j : 0;
        o.b = o.kind ? B + (size_t)n * g.r : o.w;
        return o;
    }
    // plain: up to three weight segments stacked along N; tiles never straddle segments
    int t = tile_n;
    const bf16_t *W = W0;
    int n_seg = g.n_seg[0];
    bool first = true;
    if (g.nseg > 1 && t >= g.tiles_seg[0]) {
        t -= g.tiles_seg[0]; W = g.W[1]; n_seg = g.n_seg[1]; first = false;
        if (g.nseg > 2 && t >= g.tiles_seg[1]) { t -= g.tiles_seg[1]; W = g.W[2]; n_seg = g.n_seg[2]; }
    }
    int n = min(t * BN + b, n_seg - 1);
    o.w = W + (size_t)n * g.K;
    o.kind = (first && g.T && g.B[0]) ? 1 : 0;
    o.b = o.kind ? g.B[0] + (size_t)n * g.r : o.w;
    return o;
}

// Slabs of base weights, n_base of them, are taken from slab `turn` on, around the end: tile_n modulo their number, or 0 (GemmArgs::stagger).
__device__ __forceinline__ int gemm_turn(const GemmArgs &g, int tile_n, int n_base) { return (int)__umulhi((uint32_t)tile_n * g.stagger, (uint32_t)n_base); }
__device__ __forceinline__ int gemm_slab(int kt, int turn, int n_base) {
    const int at = kt + turn;
    return at < n_base ? at : at - n_base;
}

// 256 bytes of zeros: the source of LDS-direct loads that must read as zeros (adapter columns a
// row does not have, padding past the last adapter column).
__device__ uint4 g_zero_page[16];

// 16-byte LDS-direct load: lane i of the wave copies 16 bytes from its own global address g to LDS
// byte address lds_base + 16 i (lds_base wave-uniform).  The data bypasses the registers and the
// load stays in flight, counted by vmcnt, until it has been written to LDS.  Written as inline
// assembly so that the compiler does not tie later LDS reads to it with a full vmcnt(0) wait: the
// pipeline below waits explicitly.  m0 carries the LDS base; nothing else in these kernels uses m0.
__device__ __forceinline__ void dma16(const void *g, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(g) : "memory");
}

// s_waitcnt immediate (gfx9 encoding) for vmcnt <= N and lgkmcnt == 0: all LDS reads of the wave
// have returned and at most N of its global loads are still in flight.
constexpr int waitcnt_vm_lgkm0(int n) { return (n & 15) | (7 << 4) | (0 << 8) | ((n >> 4) << 14); }

template <int N>
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(N)); }

// Byte offset of 16-byte chunk c of tile row `row` inside an operand's LDS stage.  Rows are stored
// densely (CPR chunks each); inside every 256-byte line (one pass over the 64 banks) the chunk
// position is XOR-ed with the low bits of the line number, so that the 16-byte fragment reads of
// 16 consecutive rows, which the LDS serves together, fall into 16 different bank groups.
template <int CPR>
__device__ __forceinline__ int swz(int row, int c) {
    int q = row * CPR + c, line = q >> 4, p = q & 15;
    return (line << 8) + ((p ^ (line & (CPR - 1))) << 4);
}

// Epilogue of a wave that holds TM x TN MFMA tiles of MF x MF (wave wm, wn of the tile at tile_n, its rows from wrow0 on, below row_end).
// Accumulator register r of MFMA tile (i, j) is row 8(r/4) + 4(lane/32) + r%4, column lane%32: a lane owns single columns, which
// would make 2-byte stores.  Each wave therefore turns 32 rows of its tile at a time through scr, its own 32 x (WN + 8) floats of
// LDS, and reads them back row-major, 8 columns per lane, for 16- and 32-byte global accesses.
template <int MF, int TM, int TN, int BN, typename Acc>
__device__ __forceinline__ void store_wave_tile(const GemmArgs &g, const Acc (&acc)[TM][TN], float *scr, int tile_n, int kz, int wrow0,
                                                int row_end, int wn) {
    constexpr int WN = MF * TN, IG = 32 / MF;  // columns of the wave; MFMA row tiles of a 32-row group
    const int lane = threadIdx.x & 63;
    constexpr int kGroups = (TM + IG - 1) / IG;  // with an odd number of 16-row tiles the last one is half a group
    constexpr bool kMayBeDual = TN % 2 == 0;
    const bool dual = kMayBeDual && g.mode == GEMM_DUAL;
    constexpr int kEs = WN + 8;  // scratch row stride in floats: rows 4 apart fall into different bank halves
    const int col_l = lane % MF;
    auto row_of = [&](int ii, int r) { return MF == 32 ? 8 * (r >> 2) + (lane >> 5) * 4 + (r & 3) : ii * 16 + (lane >> 4) * 4 + r; };
    int seg = 0, t = tile_n, col_base = 0;
    if (!dual)
        while (seg + 1 < g.nseg && t >= g.tiles_seg[seg]) { t -= g.tiles_seg[seg]; col_base += g.n_seg[seg]; ++seg; }
    const int wcols = dual ? WN / 2 : WN;                                   // output columns of this wave
    const int n_wave = dual ? tile_n * (BN / 2) + wn * (WN / 2) : t * BN + wn * WN;  // first of them, inside the segment
    const int n_lim = g.n_seg[dual ? 0 : seg];
    const int lpr = wcols / 8, rpp = 64 / lpr;                              // lanes per row, rows per pass
    const int rr0 = lane / lpr, c8 = (lane % lpr) * 8;
    // The residual rows of the next 32-row group are requested before this group is turned through
    // LDS, so that their latency (HBM: another kernel wrote them) is not paid once per pass.
    constexpr int kPasses = WN / 16;  // passes over a 32-row group when the wave's columns are all outputs
    const bool with_resid = !dual && g.epi != EPI_F32;
    uint4 rres[2][kPasses];
    auto load_resid = [&](int i, uint4 (&dst)[kPasses]) {
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            const int row = wrow0 + i * 32 + rr0 + p * rpp, n_in = n_wave + c8;
            dst[p] = (row < row_end && n_in < n_lim) ? *(const uint4 *)(g.resid + (size_t)row * g.ldr + col_base + n_in) : make_uint4(0u, 0u, 0u, 0u);
        }
    };
    if (with_resid) load_resid(0, rres[0]);
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
        const int rows_here = min(32, (TM - i * IG) * MF);
        if (with_resid && i + 1 < kGroups) load_resid(i + 1, rres[(i + 1) & 1]);
        if (dual) {
            if constexpr (kMayBeDual) {
#pragma unroll
                for (int j = 0; j < TN / 2; ++j)
#pragma unroll
                    for (int q = 0; q < IG * (MF * MF / 64); ++q) {
                        const int ii = q % IG, r = q / IG;
                        if (i * IG + ii >= TM) continue;
                        float gt = acc[i * IG + ii][j][r], up = acc[i * IG + ii][j + TN / 2][r];
                        scr[row_of(ii, r) * kEs + j * MF + col_l] = gt * __builtin_amdgcn_rcpf(1.f + __expf(-gt)) * up;  // 1 ulp reciprocal: the result is rounded to bf16
                    }
            }
        } else {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < IG * (MF * MF / 64); ++q)
                    if (i * IG + q % IG < TM) scr[row_of(q % IG, q / IG) * kEs + j * MF + col_l] = acc[i * IG + q % IG][j][q / IG];
        }
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            const int rr = rr0 + p * rpp;
            if (rr >= rows_here) break;  // the fused gate/up tile has half the output columns: half the passes
            const int row = wrow0 + i * 32 + rr, n_in = n_wave + c8;
            if (row >= row_end || n_in >= n_lim) continue;  // output widths are multiples of 8
            const float4 a = *(const float4 *)(scr + rr * kEs + c8), b = *(const float4 *)(scr + rr * kEs + c8 + 4);
            float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            const int n = col_base + n_in;
            if (!dual && g.epi == EPI_F32) {
                float *yp = (float *)g.Y + ((size_t)kz * g.slice_rows + row) * g.ldy + n;
                *(float4 *)yp = a;
                *(float4 *)(yp + 4) = b;
                continue;
            }
            if (!dual) {  // EPI_BF16_RESID
                const uint4 rv = rres[i & 1][p];
                const uint32_t rw[4] = {rv.x, rv.y, rv.z, rv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[2 * e] += __uint_as_float(rw[e] << 16);
                    v[2 * e + 1] += __uint_as_float(rw[e] & 0xffff0000u);
                }
            }
            uint4 o;
            o.x = pack_bf16(v[0], v[1]);
            o.y = pack_bf16(v[2], v[3]);
            o.z = pack_bf16(v[4], v[5]);
            o.w = pack_bf16(v[6], v[7]);
            *(uint4 *)((bf16_t *)g.Y + (size_t)row * g.ldy + n) = o;
        }
    }
}

}  // namespace
}  // namespace icarus
