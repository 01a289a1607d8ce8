// ICaRusLinear (see gemm_mfma.hip) for more than 128 rows: tiles of 256 weight rows x 256, 192 or 160 stacked rows, for the
// projections of a prefill chunk and the wide ones of a decode batch, and of 128 x 192, 160 or 128 for the narrow ones.  Below: the
// epilogue of the QKV projection, which appends to the cache.
//
// Bound: the matrix cores, and the power they draw.  Eight waves sit 2 x 4 over a wide tile; over a narrow one four sit 2 x 2, which
// leaves room for a second workgroup on its CU, or eight 4 x 2 where there is none (see launch_any); a wave owns (BM / 2) x 64 outputs, or
// (BM / 4) x 64, in 16x16x32 bf16 MFMAs.  K advances 64 columns (whole 128-byte lines of every row) at a time through two LDS stages filled by
// LDS-direct loads.  What a slab's loads get is time: with the fragments read K step by K step, as in gemm_mfma.hip, every
// part of a stage is in use until the last step, and a load has three quarters of a slab to arrive; measured at 16384 x 28672 x
// 4096 the 256 x 256 loop waited for its loads more than for anything else (matrix pipe busy 64 % of the cycles).  Here a wave
// works through the four quadrants of its tile instead (two halves of its rows x two of its columns), each over all 64
// columns of the slab: it reads half an operand at once, into registers, and that half of the stage is free for the slab
// after next.  A load has one and a half slabs to arrive, with the same two stages.  A quadrant is a phase:
//
//      slab        even                                    odd
//      multiplied  X0 W0   X0 W1   X1 W1   X1 W0           X0 W1   X0 W0   X1 W0   X1 W1
//      read        W1      X1      X0'     W1'             W0      X1      X0''    W0''         ' of the next slab
//      requested   X0      W0      W1      X1              X0      W1      W0      X1           of the slab after next
//
// so each half is read once and at most one half of every operand is read ahead (64 + 32 fragment registers beside 128
// accumulators in the 256-row tile).  What a phase requests was read in the phase before or earlier; a barrier after every
// second phase says that all waves are done with it, and that the loads of all waves for the next two phases have landed.
// MFMAs of 16x16x32 draw less power than 32x32x16 for the same work (half the accumulator traffic), and power is what is
// left: the clock settles at 1.83 GHz with the pipe busy 81 % of the cycles, against 1.65 GHz and 73 % in 32x32x16.
// Measured (us, the kernel this one replaced / this one): 16384 rows, gate and up of 4096 -> 2 x 14336 in 256 x 256 tiles
// 2987 / 2557 (1.50 PFLOP/s), 14336 -> 4096 1500 / 1275; 4337 rows, 14336 -> 4096 in 160 x 256 484 / 397; 753 rows, gate and
// up in 192 x 256 175 / 149; 316 rows in 160 x 256 84 / 75.  Narrow tiles: 753 rows, 14336 -> 4096 in 2 slices 102 / 96; 316 rows,
// 14336 -> 4096 in 4 slices 58.7 / 53.5; 144 rows, 8192 -> 5120 in 6 slices 34.4 / 32.2.  Not kept: four waves of 128 x 128 (a third fewer LDS reads, one wave
// a SIMD; 0-4 % slower), three stages of 160-row tiles (0-7 % slower), raised priority around the MFMAs (1 % slower).
//
// MFMA 16x16x32 bf16 operand layout (lane l): A[row l%16][k 8(l/16)..+7], B[k 8(l/16)..+7][col l%16],
// C[row 4(l/16) + r][col l%16] for accumulator register r = 0..3.
#include "gemm_tile.h"

namespace icarus {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// dma16 with the address in two parts, a wave-uniform base and the lane's byte offset from it: stepping along K costs no
// vector instruction
__device__ __forceinline__ void dma16_at(const void *base, uint32_t off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(off), "s"(base) : "memory");
}

template <int V> struct Int { static constexpr int value = V; };

// MT0, MT1: 16-row tiles of a wave in the two halves of its rows
template <int MT0, int MT1, int WAVES_N, int WAVES_M>
struct QuadShape {
    static constexpr int BM = 16 * WAVES_M * (MT0 + MT1), BN = 64 * WAVES_N, BK = 64;
    static constexpr int kXStage = BM * BK * 2, kWStage = BN * BK * 2, kStages = 2 * (kXStage + kWStage);  // LDS: two stages of X, two of W,
    static constexpr int kScratch = WAVES_M * WAVES_N * 32 * 72 * 4;                                          // then the epilogue's scratch
    static constexpr int kLds = kStages > kScratch ? kStages : kScratch;
};

// Epilogue of the QKV projection: a head is the columns of two neighbouring waves, which meet in LDS 32 rows at a time.  Of a q or k
// head each wave takes half of those rows, a lane eight pairs of one; the sums of the QK-norm run in the order of
// k_rope_append_tile.  Of a v head a wave takes its own columns, a lane one of them, and whole pieces of eight tokens of the transposed
// plane go out at once.
// The projections used to go out and in again in float32 (403 MB of 16384 rows each way) around a kernel of its own.  Projection + append, us,
// before / now with the table of the rows' angles: 16384 rows, 48 heads 640 + 136 / 594 + 8 (256 x 256), 753 rows 53.6 + 13.2 / 57.2 + 4.9, 512
// rows of 80 heads 67.9 + 12.2 / 68.2 + 4.8 (192 x 128).  The angles are fetched a group ahead: where they were asked for, 753 rows took
// 64 us.
template <int TM, int BN>
__device__ __forceinline__ void store_qkv_tile(const GemmArgs &g, const QkvStore &e, const f32x4 (&acc)[TM][4], float *scratch, int w, int wn,
                                               int tile_n, int wrow0, int row_end) {
    constexpr int kEs = 64 + 8, kScr = 32 * kEs, kPlane = 16 * 128;
    const int lane = threadIdx.x & 63, half = wn & 1;
    const int t1 = tile_n - g.tiles_seg[0], t2 = t1 - g.tiles_seg[1];
    const int seg = t1 < 0 ? 0 : t2 < 0 ? 1 : 2, t = t1 < 0 ? tile_n : t2 < 0 ? t1 : t2;
    const int head = (t * BN + wn * 64) >> 7;
    const bool there = head < (seg == 0 ? e.Hq : e.Hkv);
    float *own = scratch + w * kScr;
    const float *lo = scratch + (w - half) * kScr, *hi = lo + kScr;
    const int c = lane & 7;  // the pairs of a lane: 8 c and the seven after it
    // angles and slots of a group are requested while the one before it is stored
    float cs[2][8], sn[2][8];
    int64_t slot[2];
    auto fetch = [&](int i) {
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            const int row = min(wrow0 + 32 * i + (seg < 2 ? 16 * half + 8 * pass + (lane >> 3) : lane & 31), row_end - 1);
            if (seg > 0) slot[pass] = e.slot[row];
            if (seg < 2)
#pragma unroll
                for (int x = 0; x < 8; x += 4) {
                    *(float4 *)(cs[pass] + x) = *(const float4 *)(e.cs + (size_t)row * 64 + 8 * c + x);
                    *(float4 *)(sn[pass] + x) = *(const float4 *)(e.sn + (size_t)row * 64 + 8 * c + x);
                }
        }
    };
    fetch(0);
    const bf16_t *nw = seg == 0 ? e.q_norm : seg == 1 ? e.k_norm : nullptr;
    uint4 nlo = make_uint4(0u, 0u, 0u, 0u), nhi = nlo;
    if (nw) { nlo = *(const uint4 *)(nw + 8 * c); nhi = *(const uint4 *)(nw + 64 + 8 * c); }
    auto element = [](uint4 v, int x) {
        const uint32_t u = x < 2 ? v.x : x < 4 ? v.y : x < 6 ? v.z : v.w;
        return __uint_as_float(x & 1 ? u & 0xffff0000u : u << 16);
    };
#pragma unroll
    for (int i = 0; i < (TM + 1) / 2; ++i) {
        const int first = wrow0 + 32 * i, n = min(min(32, (TM - 2 * i) * 16), row_end - first);
        if (i > 0) __syncthreads();
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (2 * i + ii < TM) own[(ii * 16 + (lane >> 4) * 4 + r) * kEs + j * 16 + (lane & 15)] = acc[2 * i + ii][j][r];
        __syncthreads();
        if (!there) continue;
        if (seg < 2) {
            float ra[2][8], rb[2][8];
#pragma unroll
            for (int pass = 0; pass < 2; ++pass) {
                const int rr = 16 * half + 8 * pass + (lane >> 3);
                float a[8], b[8];
#pragma unroll
                for (int x = 0; x < 8; x += 4) {
                    *(float4 *)(a + x) = *(const float4 *)(lo + rr * kEs + 8 * c + x);
                    *(float4 *)(b + x) = *(const float4 *)(hi + rr * kEs + 8 * c + x);
                }
                if (nw) {
                    float p[8];
#pragma unroll
                    for (int x = 0; x < 8; ++x) {
                        p[x] = __builtin_fmaf(b[x], b[x], a[x] * a[x]);
#pragma unroll
                        for (int o = 4; o > 0; o >>= 1) p[x] += __shfl_xor(p[x], o, 64);
                    }
                    const float inv = rsqrtf((((p[0] + p[4]) + (p[2] + p[6])) + ((p[1] + p[5]) + (p[3] + p[7]))) / 128.f + e.eps);
#pragma unroll
                    for (int x = 0; x < 8; ++x) {
                        a[x] = a[x] * inv * element(nlo, x);
                        b[x] = b[x] * inv * element(nhi, x);
                    }
                }
#pragma unroll
                for (int x = 0; x < 8; ++x) rotate_pair(a[x], b[x], cs[pass][x], sn[pass][x], &ra[pass][x], &rb[pass][x]);
            }
            const int64_t at[2] = {slot[0], slot[1]};
            if (i + 1 < (TM + 1) / 2) fetch(i + 1);
#pragma unroll
            for (int pass = 0; pass < 2; ++pass) {
                const int rr = 16 * half + 8 * pass + (lane >> 3), row = first + rr;
                if (rr >= n) continue;
                auto pack = [](const float (&v)[8]) { return make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7])); };
                auto pack8 = [&](const float (&v)[8]) {
                    uint32_t u[2] = {0u, 0u};
#pragma unroll
                    for (int x = 0; x < 8; ++x) u[x >> 2] |= f32_to_fp8(v[x] / e.k_scale) << (8 * (x & 3));
                    return make_uint2(u[0], u[1]);
                };
                if (seg == 0) {
                    bf16_t *dst = e.q + ((size_t)row * e.Hq + head) * 128 + 8 * c;
                    *(uint4 *)dst = pack(ra[pass]);
                    *(uint4 *)(dst + 64) = pack(rb[pass]);
                } else {
                    const size_t dst = ((size_t)(at[pass] >> 4) * e.Hkv + head) * 2 * kPlane + (size_t)(at[pass] & 15) * 128 + 8 * c;
                    if (e.kv8) {
                        *(uint2 *)((uint8_t *)e.pool + dst) = pack8(ra[pass]);
                        *(uint2 *)((uint8_t *)e.pool + dst + 64) = pack8(rb[pass]);
                    } else {
                        *(uint4 *)((bf16_t *)e.pool + dst) = pack(ra[pass]);
                        *(uint4 *)((bf16_t *)e.pool + dst + 64) = pack(rb[pass]);
                    }
                }
            }
        } else {
            const int d = half * 64 + lane, slot_lo = (int)slot[0], slot_hi = (int)(slot[0] >> 32);
            auto slot_of = [&](int r) { return (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane(slot_hi, r) << 32 | (uint32_t)__builtin_amdgcn_readlane(slot_lo, r)); };
            // bit r: row r + 1 has the slot after row r's (entries of a call may share a block, with rows of others between theirs)
            const int lo_after = __shfl_down(slot_lo, 1, 64), hi_after = __shfl_down(slot_hi, 1, 64);
            const uint64_t in_line = __ballot(hi_after == slot_hi && lo_after == slot_lo + 1);
            if (i + 1 < (TM + 1) / 2) fetch(i + 1);
            for (int r = 0; r < n;) {
                const int64_t first_slot = slot_of(r);
                const size_t dst = (((size_t)(first_slot >> 4) * e.Hkv + head) * 2 + 1) * kPlane + (size_t)d * 16 + (size_t)(first_slot & 15);
                if (!(first_slot & 7) && r + 8 <= n && (in_line >> r & 0x7f) == 0x7f) {
                    float v[8];
#pragma unroll
                    for (int x = 0; x < 8; ++x) v[x] = own[(r + x) * kEs + lane];
                    if (e.kv8) {
                        uint32_t u[2] = {0u, 0u};
#pragma unroll
                        for (int x = 0; x < 8; ++x) u[x >> 2] |= f32_to_fp8(v[x] / e.v_scale) << (8 * (x & 3));
                        *(uint2 *)((uint8_t *)e.pool + dst) = make_uint2(u[0], u[1]);
                    } else {
                        *(uint4 *)((bf16_t *)e.pool + dst) =
                            make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
                    }
                    r += 8;
                } else {
                    const float v = own[r * kEs + lane];
                    if (e.kv8) ((uint8_t *)e.pool)[dst] = (uint8_t)f32_to_fp8(v / e.v_scale);
                    else ((bf16_t *)e.pool)[dst] = f32_to_bf16(v);
                    ++r;
                }
            }
        }
    }
}

// e: the epilogue's arguments where it is that of the QKV projection (QKV), else null.  TURN: workgroups may start at different places along K (gemm_turn).
template <int MT0, int MT1, int WAVES_N, int WAVES_M, bool GROUPED, bool QKV, bool TURN>
__device__ __forceinline__ void quad_tile(const GemmArgs &g, const QkvStore *e) {
    using Shape = QuadShape<MT0, MT1, WAVES_N, WAVES_M>;
    constexpr int NW = WAVES_M * WAVES_N, BM = Shape::BM, BN = Shape::BN, BK = Shape::BK;
    constexpr int WM = BM / WAVES_M, WN = 64, NT = 2, KS = BK / 32;
    constexpr int kRow = BK * 2;                          // bytes of a tile row in LDS
    constexpr int kXStage = Shape::kXStage, kWStage = Shape::kWStage, kBOff = 2 * kXStage;
    constexpr int LDW = 4 / WAVES_M, LDX0 = 2 * MT0 / WAVES_N, LDX1 = 2 * MT1 / WAVES_N;        // loads of a wave for a half of W, for the halves of X;
    constexpr bool kOdd0 = 2 * MT0 % WAVES_N != 0, kOdd1 = 2 * MT1 % WAVES_N != 0;    // an odd number of row tiles leaves four units over
    constexpr int kPair0 = LDW + LDX0, kPair1 = LDW + LDX1;                   // loads of a wave in the first, the second two phases of a slab: at least
    constexpr int kSlab = kPair0 + kPair1 + (kOdd0 && kOdd1 ? 1 : 0);
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)smem;
    int tile_m, tile_n, kz;
    if (!tile_of_workgroup(g, &tile_m, &tile_n, &kz)) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w / WAVES_N, wn = w % WAVES_N;
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
    // The tile's weight rows, from n0 on.  Fused: the first halves of the waves' columns are gate rows, the second halves the up
    // rows of the same outputs.
    const bool dual = g.mode == GEMM_DUAL;
    int n0 = tile_n * (BN / 2), n_lim = g.n_seg[0];
    bool adp0 = g.T && g.B[0], adp1 = g.T && g.B[1];  // the halves of W have adapter columns (fused: gate and up rows, else the same)
    if (!dual) {
        int t = tile_n;
        W1 = W0;
        adp1 = adp0;
        if (g.nseg > 1 && t >= g.tiles_seg[0]) {
            t -= g.tiles_seg[0]; W0 = W1 = g.W[1]; n_lim = g.n_seg[1]; adp0 = adp1 = false;
            if (g.nseg > 2 && t >= g.tiles_seg[1]) { t -= g.tiles_seg[1]; W0 = W1 = g.W[2]; n_lim = g.n_seg[2]; }
        }
        n0 = t * BN;
    }
    const int k_begin = kz * g.k_per_split;
    const int k_end = min(adp0 || adp1 ? g.K_ext : g.K, k_begin + g.k_per_split);
    const int nk = (k_end - k_begin + BK - 1) / BK;            // slabs of this slice (none: it stores zeros)
    const int n_base = min(nk, max(0, (g.K - k_begin) / BK));  // of them base weights

    // Halves travel in units of 1 KiB (8 rows), each one wave-wide load: lane l fills 256-byte line l / 16 of the unit, position
    // l % 16, which un-swizzled is a chunk of one of the unit's two rows of that line.
    // This lane's part of unit u of a half: row of the half, 16-byte chunk.  Worked out again where it is needed (the lane's
    // number passes through an empty asm): kept over the K loop, the rows would cost it registers that it does not have.
    struct Place { int hr, kc; };
    auto place = [&](int u, bool again) {
        int l = lane;
        if (again) asm volatile("" : "+v"(l));
        const int lin = l >> 4, qd = lin * 16 + ((l & 15) ^ ((u * 4 + lin) & 7));
        return Place{u * 8 + qd / 8, qd % 8 * 8};
    };
    auto x_row = [&](int h, int hr) {
        const int per = h ? 16 * MT1 : 16 * MT0;
        return min(row0 + hr / per * WM + h * (16 * MT0) + hr % per, row_end - 1);
    };
    auto w_row = [&](int h, int hr) { return min(n0 + (dual ? hr : hr / (WN / 2) * WN + h * (WN / 2) + hr % (WN / 2)), n_lim - 1); };
    // unit i of this wave in a half of X: w + NW i, and of the four units left over by an odd number of row tiles one for each
    // of waves 0-3 (first half) or 4-7 (second half; 0-3 again where only that half has them)
    auto x_unit = [&](int h, int i) { return i < (h ? LDX1 : LDX0) ? w + NW * i : NW * i + (w & 3); };
    auto x_has = [&](int h) { return h ? kOdd1 && (kOdd0 ? w >= 4 : w < 4) : kOdd0 && w < 4; };
    const char *xb = (const char *)(g.X + (size_t)row0 * g.ldx + k_begin);
    const char *wb0 = (const char *)(W0 + (size_t)n0 * g.K + k_begin), *wb1 = (const char *)(W1 + (size_t)n0 * g.K + k_begin);
    uint32_t xo[2][LDX0 + LDX1 + 1], wo[2][LDW];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < (h ? LDX1 + kOdd1 : LDX0 + kOdd0); ++i) {
            const Place p = place(x_unit(h, i), false);
            xo[h][i] = (uint32_t)((x_row(h, p.hr) - row0) * (uint32_t)g.ldx + p.kc) * 2u;
        }
#pragma unroll
        for (int i = 0; i < LDW; ++i) {
            const Place p = place(w + NW * i, false);
            wo[h][i] = (uint32_t)((w_row(h, p.hr) - n0) * (uint32_t)g.K + p.kc) * 2u;
        }
    }
    const int turn = TURN ? gemm_turn(g, tile_n, n_base) : 0;
    auto place_of = [&](int kt) { return TURN ? gemm_slab(kt, turn, n_base) : kt; };
    // part: 0, 1 the halves of X; 2, 3 those of W
    auto part_lds = [&](int P, int S) { return P >= 2 ? kBOff + S * kWStage + (P & 1) * (kWStage / 2) : S * kXStage + P * (16 * WAVES_M * MT0 * kRow); };
    // load i of a part, of the slab of base weights at place kt along K (gemm_slab)
    auto load_one = [&](auto Part, auto Stage, int kt, int i) {
        constexpr int P = decltype(Part)::value, S = decltype(Stage)::value;
        if constexpr (P < 2) {
            if (i < (P ? LDX1 : LDX0) || x_has(P)) dma16_at(xb + (size_t)kt * kRow, xo[P][i], lds0 + part_lds(P, S) + x_unit(P, i) * 1024);
        } else dma16_at((P & 1 ? wb1 : wb0) + (size_t)kt * kRow, wo[P & 1][i], lds0 + part_lds(P, S) + (w + NW * i) * 1024);
    };
    auto n_loads = [](int P) { return P >= 2 ? LDW : P ? LDX1 + kOdd1 : LDX0 + kOdd0; };
    // all of a part, of any slab
    auto load_part = [&](auto Part, auto Stage, int kt) {
        constexpr int P = decltype(Part)::value, S = decltype(Stage)::value;
        if (kt < n_base) {
#pragma unroll
            for (int i = 0; i < n_loads(P); ++i) load_one(Part, Stage, place_of(kt), i);
            return;
        }
        const int mr = g.M_models * g.r;
        const bf16_t *zero = (const bf16_t *)g_zero_page;
#pragma unroll
        for (int i = 0; i < n_loads(P); ++i) {
            const int u = P < 2 ? x_unit(P, i) : w + NW * i;
            if (P < 2 && i >= (P ? LDX1 : LDX0) && !x_has(P)) continue;
            const bf16_t *p = zero;
            const Place at = place(u, true);
            const int k2 = k_begin + kt * BK - g.K + at.kc;
            if constexpr (P < 2) {
                if (g.T && k2 < g.ldt) p = g.T + (size_t)x_row(P, at.hr) * g.ldt + k2;
            } else {
                const int kk = k2 - (dual && (P & 1) ? mr : 0), lr = 31 - __clz(max(g.r, 1));
                if ((P & 1 ? adp1 : adp0) && kk >= 0 && kk < mr)
                    p = ((dual && (P & 1)) ? g.B[1] : g.B[0]) + (size_t)w_row(P & 1, at.hr) * g.r + (size_t)(kk >> lr) * g.n_seg[0] * g.r + (kk & (g.r - 1));
            }
            dma16(p, lds0 + part_lds(P, S) + u * 1024);
        }
    };

    f32x4 acc[MT0 + MT1][2 * NT];
#pragma unroll
    for (int i = 0; i < MT0 + MT1; ++i)
#pragma unroll
        for (int j = 0; j < 2 * NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
    bf16x8 fa0[KS][MT0], fa1[KS][MT1], fb[2][KS][NT];
    // where this lane reads the first 16 rows of a part of its wave, in stage 0
    int rx0[KS], rx1[KS], rw[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const int at = swz<8>(lane & 15, 4 * ks + (lane >> 4));
        rx0[ks] = at + wm * 16 * MT0 * kRow;
        rx1[ks] = at + wm * 16 * MT1 * kRow;
        rw[ks] = at + wn * (WN / 2) * kRow + kBOff;
    }
    // fragment f of a part
    auto read_one = [&](auto Part, auto Stage, int f) {
        constexpr int P = decltype(Part)::value, S = decltype(Stage)::value;
        if constexpr (P == 0) fa0[f / MT0][f % MT0] = *(const bf16x8 *)(smem + rx0[f / MT0] + part_lds(P, S) + (f % MT0) * (16 * kRow));
        else if constexpr (P == 1) fa1[f / MT1][f % MT1] = *(const bf16x8 *)(smem + (MT0 == MT1 ? rx0 : rx1)[f / MT1] + part_lds(P, S) + (f % MT1) * (16 * kRow));
        else fb[P - 2][f / NT][f % NT] = *(const bf16x8 *)(smem + rw[f / NT] + (part_lds(P, S) - kBOff) + (f % NT) * (16 * kRow));
    };
    auto n_frags = [](int P) { return KS * (P >= 2 ? NT : P ? MT1 : MT0); };
    // One phase: quadrant (A, B) of the wave tile over the 64 columns of the slab; meanwhile part RD is read from
    // stage RS and part LP of slab lk (at its place along K) requested into stage LS.
    auto phase = [&](auto A, auto B, auto RD, auto RS, auto LP, auto LS, auto hot, int lk, int at) {
        constexpr int a = decltype(A)::value, b = decltype(B)::value, MT = a ? MT1 : MT0, kMul = MT * NT * KS;
        constexpr int rn = kMul / 2, l0 = kMul / 2, nl = n_loads(decltype(LP)::value), nrd = n_frags(decltype(RD)::value);
#pragma unroll
        for (int m = 0; m < kMul; ++m) {
            const int ks = m / (MT * NT), i = m % (MT * NT) / NT, j = m % NT;
            f32x4 &c = acc[a * MT0 + i][b * NT + j];
            if constexpr (a == 0) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa0[ks][i], fb[b][ks][j], c, 0, 0, 0);
            else c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa1[ks][i], fb[b][ks][j], c, 0, 0, 0);
#pragma unroll
            for (int f = 0; f < nrd; ++f)
                if (f * rn / nrd == m) read_one(RD, RS, f);
            if constexpr (decltype(hot)::value) {
#pragma unroll
                for (int l = 0; l < nl; ++l)
                    if (l0 + l * (kMul - l0) / nl == m) load_one(LP, LS, at, l);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (!decltype(hot)::value) {
            if (lk < nk) load_part(LP, LS, lk);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // Every wave has read what the phases before read, and at most n loads of this wave are still in flight.
    auto sync = [&](auto n) {
        wait_loads<decltype(n)::value>();
        __builtin_amdgcn_s_barrier();
    };
    constexpr Int<0> I0; constexpr Int<1> I1; constexpr Int<2> I2; constexpr Int<3> I3;
    if (nk > 0) {
        load_part(I0, I0, 0); load_part(I2, I0, 0); load_part(I3, I0, 0); load_part(I1, I0, 0);
        if (nk > 1) { load_part(I0, I1, 1); load_part(I3, I1, 1); load_part(I2, I1, 1); load_part(I1, I1, 1); }
        if (nk > 1) sync(Int<kSlab>());
        else sync(I0);
#pragma unroll
        for (int f = 0; f < n_frags(0); ++f) read_one(I0, I0, f);
#pragma unroll
        for (int f = 0; f < n_frags(2); ++f) read_one(I2, I0, f);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        int kt = 0;
        // One slab, in stage S; F: the half of W that is multiplied first (0 in even slabs, 1 in odd ones), L: the other one.
        auto slab = [&](auto S, auto hot) {
            constexpr bool H = decltype(hot)::value;
            constexpr Int<decltype(S)::value> F; constexpr Int<1 - F.value> L, N;  // N: the next slab's stage
            constexpr Int<F.value + 2> WF; constexpr Int<L.value + 2> WL;
            const int at = place_of(kt + 2);
            const bool there1 = H || kt + 1 < nk, there2 = H || kt + 2 < nk;
            phase(I0, F, WL, S, I0, S, hot, kt + 2, at);
            phase(I0, L, I1, S, WF, S, hot, kt + 2, at);
            if (there2) sync(Int<kSlab>());
            else if (there1) sync(Int<kPair1>());
            else sync(I0);
            phase(I1, L, I0, N, WL, S, hot, kt + 2, at);
            phase(I1, F, WL, N, I1, S, hot, kt + 2, at);
            if (there2) sync(Int<kSlab>());
            else sync(I0);
            ++kt;
        };
        while (kt + 4 <= n_base) {
            slab(I0, Int<1>());
            slab(I1, Int<1>());
        }
        while (kt < nk) {
            slab(I0, Int<0>());
            if (kt < nk) slab(I1, Int<0>());
        }
    }
    __syncthreads();  // every wave has left the K loop: the stages are the epilogue's scratch
    static_assert(NW * 32 * (WN + 8) * 4 <= Shape::kLds, "epilogue scratch must fit");
    if constexpr (QKV) store_qkv_tile<MT0 + MT1, BN>(g, *e, acc, (float *)smem, w, wn, tile_n, row0 + wm * WM, row_end);
    else store_wave_tile<16, MT0 + MT1, 2 * NT, BN>(g, acc, (float *)smem + w * 32 * (WN + 8), tile_n, kz, row0 + wm * WM, row_end, wn);
}

// 256 x 256 tiles turn in an instance of their own: launches bound by the matrix cores took 0.4 % for the three scalar instructions a slab, but those
// of 193-256 rows wait for their weights.  us, same / different starts: LM head 4096 -> 128256, 193 rows 264 / 249, 256 rows 282 / 260; gate and
// up 8192 -> 2 x 28672, 193 rows 210 / 207, 224 rows 225 / 212, 256 rows 227 / 217 (means of two GPUs, 2-8 % each);
// a token step of one layer and that head, 194 rows 536 / 507, 230 rows 566 / 536.
// Not in slices of K: 8192 -> 10240 in 6, 220 rows 45.6 / 57.7, 256 rows 47.5 / 57.
constexpr bool turns(int row_tiles) { return row_tiles < 8; }

template <int MT0, int MT1, int WAVES_N, int WAVES_M, bool GROUPED, bool TURN>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N, WAVES_M * WAVES_N == 8 ? 1 : 2) k_gemm_quad(GemmArgs g) {
    quad_tile<MT0, MT1, WAVES_N, WAVES_M, GROUPED, false, TURN>(g, nullptr);
}

template <int MT0, int MT1, int WAVES_N, int WAVES_M>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N, WAVES_M * WAVES_N == 8 ? 1 : 2) k_gemm_quad_qkv(GemmArgs g, QkvStore e) {
    quad_tile<MT0, MT1, WAVES_N, WAVES_M, false, true, turns(MT0 + MT1)>(g, &e);
}

template <int MT0, int MT1, int WAVES_N, bool GROUPED, int WAVES_M = 2, bool TURN = turns(MT0 + MT1)>
hipError_t launch_quad(GemmArgs g, hipStream_t st, const QkvStore *e = nullptr) {
    using Shape = QuadShape<MT0, MT1, WAVES_N, WAVES_M>;
    constexpr int BM = Shape::BM, BN = Shape::BN;
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
    gemm_set_panels(&g, BM, BN, WAVES_M * WAVES_N == 8 ? 1 : 2);
    dim3 grid(gemm_grid(g));
    if constexpr (!GROUPED)
        if (e) {
            static bool qkv_set = false;
            if (!qkv_set) {
                hipError_t rc = hipFuncSetAttribute((const void *)k_gemm_quad_qkv<MT0, MT1, WAVES_N, WAVES_M>, hipFuncAttributeMaxDynamicSharedMemorySize, Shape::kLds);
                if (rc != hipSuccess) return rc;
                qkv_set = true;
            }
            hipLaunchKernelGGL((k_gemm_quad_qkv<MT0, MT1, WAVES_N, WAVES_M>), grid, dim3(64 * WAVES_M * WAVES_N), Shape::kLds, st, g, *e);
            return hipGetLastError();
        }
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t rc = hipFuncSetAttribute((const void *)k_gemm_quad<MT0, MT1, WAVES_N, WAVES_M, GROUPED, TURN>, hipFuncAttributeMaxDynamicSharedMemorySize, Shape::kLds);
        if (rc != hipSuccess) return rc;
        attr_set = true;
    }
    hipLaunchKernelGGL((k_gemm_quad<MT0, MT1, WAVES_N, WAVES_M, GROUPED, TURN>), grid, dim3(64 * WAVES_M * WAVES_N), Shape::kLds, st, g);
    return hipGetLastError();
}

int gemm_col_tiles(const GemmArgs &g, int bn) {
    if (g.mode == GEMM_DUAL) return (2 * g.n_seg[0] + bn - 1) / bn;
    int n = 0;
    for (int s = 0; s < g.nseg; ++s) n += (g.n_seg[s] + bn - 1) / bn;
    return n;
}

hipError_t launch_any(const GemmArgs &g, const QkvStore *e, hipStream_t st) {
    switch (g.tile) {
    case TILE_192x128: {
        if (g.row_tiles) return launch_quad<3, 3, 2, true>(g, st);
        // As many lower tiles, if they hold the rows: no MFMAs for padding (316 rows in tiles of 192 / 160: 14336 -> 4096 in 4
        // slices 54.4 / 53.5 us, 4096 -> 4096 28.5 / 26.7; 144 rows, 8192 -> 5120 in 6 slices 34.4 / 32.2)
        const int tiles = (g.R + 191) / 192;
        // Eight waves in place of four where a workgroup has its CU to itself: two waves a SIMD, each half as high, hide each other's
        // reads and barriers for a third more of those reads.  us: QKV of 753 rows (192 workgroups) 58.4 / 54.6, of 512 rows x 10240 (240) 68.7 / 67.3,
        // 360 rows, 4096 -> 4096 in 4 slices 24.6 / 22.7, 14336 -> 4096 53.7 / 52.7.  In layers of four widths (2048-5120), weights from HBM, 135-1100 rows,
        // prefill and decode with 8 adapters: 91 launches of 192-row tiles 3835 / 3741 us together, single ones up to 4 % either way (in a loop of one
        // launch some are: 384 rows, 8192 -> 5120 in 3 slices 39.2 / 40.2).  129-160 rows a tile keep four waves of 160; eight of 192 took 1-3 %
        // longer: prefill of 140 rows 180 / 184.5, 158 rows 183 / 190.5, 318 rows 246 / 249.5, decode of 261 and 288 rows 269 / 272.5, 272 / 275.
        const int cols = gemm_col_tiles(g, 128);
        if (tiles * cols * g.splits <= 256) {
            if (g.R <= 128 * tiles) return launch_quad<1, 1, 2, false, 4>(g, st, e);
            if (g.R > 160 * tiles) return launch_quad<2, 1, 2, false, 4>(g, st, e);
        }
        if (g.R <= 128 * tiles) return launch_quad<2, 2, 2, false>(g, st, e);
        return g.R <= 160 * tiles ? launch_quad<3, 2, 2, false>(g, st, e) : launch_quad<3, 3, 2, false>(g, st, e);
    }
    case TILE_256x256:
        if (g.row_tiles) return launch_quad<4, 4, 4, true>(g, st);
        return g.stagger && g.splits == 1 && !e ? launch_quad<4, 4, 4, false, 2, true>(g, st) : launch_quad<4, 4, 4, false>(g, st, e);
    // 753 rows, 4096 -> 4096, in k_gemm_mfma / here with four waves / with eight 45.7 / 45.5 / 43.1 us; the 286 launches of the layers above 7574 / 7589 / 7349
    case TILE_128: return launch_quad<1, 1, 2, false, 4>(g, st, e);
    case TILE_192x256: return launch_quad<3, 3, 4, false>(g, st, e);
    case TILE_160x256: return launch_quad<3, 2, 4, false>(g, st, e);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace
hipError_t launch_gemm_quad(const GemmArgs &g, hipStream_t st) { return launch_any(g, nullptr, st); }
hipError_t launch_gemm_quad_qkv(const GemmArgs &g, const QkvStore &e, hipStream_t st) { return launch_any(g, &e, st); }

}  // namespace icarus
