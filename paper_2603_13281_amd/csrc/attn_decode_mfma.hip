// Shared-KV paged GQA decode attention on gfx950 matrix cores (bf16 storage, head_dim 128,
// block_size 16).
//
// All stacked queries of one sequence that share a kv-head -- (1 + m_s) streams x g heads --
// form the N dimension of the MFMA tiles, so each KV block is fetched from HBM once for all
// of the sequence's models.  A workgroup (4 waves) owns one kv-head of one equal share of the
// call's cached tokens and walks the share's pieces (token ranges of one sequence each) in turn.
// Per 32-token group a wave computes
//     S^T[32 tok x G]  = K[32 tok x 128] . Q^T          (A = K straight from global memory)
//     O^T[128 x G]    += V^T[128 x 32 tok] . P^T         (A = V^T straight from global memory)
// with an online softmax on the S^T accumulators.  The cache layout (K token-major, V
// transposed inside the block) makes every global load a 128-bit load that lands directly in
// MFMA operand registers: no LDS staging and no register shuffles for P.
//
// Work split inside the workgroup:
//   up to 3 query tiles (G <= 48): the four waves take the chunk's groups w, w+4, ... with all tiles;
//   4 or 5 query tiles (G <= 80):  the O^T accumulators of all tiles do not fit one wave, so waves
//     0,1 take tiles [0, NA) and waves 2,3 tiles [NA, NA+NB), each pair splitting the groups two
//     ways.  A group is then loaded by two waves; the second load is served by the caches.
//
// MFMA 16x16x32 bf16 operand layout (lane l, q = l / 16):
//   A[row l%16][k 8q..8q+7], B[k 8q..8q+7][col l%16], C[row 4q+i][col l%16] (i = 0..3).
// Token <-> tile-row mapping inside a 32-token group (two KV blocks), chosen so that the 8
// P values a lane owns after the two S^T tiles are 8 consecutive tokens of one block:
//   S^T tile t, row 4q'+i'  <->  block q'/2, token-in-block 8(q'%2) + 4t + i'
//   PV contraction index k = 8q + 4t + i  <->  block q/2, token-in-block 8(q%2) + 4t + i.
#include "device_util.h"
#include "kernels.h"

#include <type_traits>

namespace icarus {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

namespace {

constexpr int kD = 128;       // head_dim
constexpr int kBk = 16;       // tokens per block
constexpr int kGrp = 32;      // tokens per wave iteration (two blocks)
constexpr int kKS = kD / 32;  // k-steps of the QK^T contraction
constexpr int kDT = kD / 16;  // d tiles of the PV product
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kSlack = 8.f;  // log2 units a score may exceed the softmax reference before it is moved
constexpr int kAttnMaxChunk = 16384;  // tokens per workgroup chunk, at most
constexpr size_t kRingBytes = (size_t)2 * 4 * 16 * 64 * 16;  // shared KV ring: 2 rounds x 4 groups x 16 KB

struct KVFrag {
    bf16x8 k[2][kKS];  // k[t][ks]: A operand of S^T tile t, k-step ks
    bf16x8 v[kDT];     // v[dt]:    A operand of O^T tile dt
};

__device__ __forceinline__ bf16x8 zero8() {
    bf16x8 z;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.f;
    return z;
}

// Issue the 16 loads of one 32-token group.  blk0/blk1: physical block ids (wave-uniform).
__device__ __forceinline__ void load_group(KVFrag &f, const bf16_t *__restrict__ pool, int blk0, int blk1, int c, int Hkv,
                                           int lane) {
    const int m = lane & 15, q = lane >> 4;
    const size_t head_stride = (size_t)2 * kBk * kD;
    // K rows: lane m reads block m/8, token-in-block 8((m/4)%2) + 4t + m%4, d = 32ks + 8q
    const bf16_t *kb = pool + ((size_t)((m >> 3) ? blk1 : blk0) * Hkv + c) * head_stride;
    const int tok0 = 8 * ((m >> 2) & 1) + (m & 3);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks)
            f.k[t][ks] = *(const bf16x8 *)(kb + (size_t)(tok0 + 4 * t) * kD + 32 * ks + 8 * q);
    // V^T rows: lane reads block q/2, d = 16dt + m, tokens 8(q%2) .. +7
    const bf16_t *vb = pool + ((size_t)((q >> 1) ? blk1 : blk0) * Hkv + c) * head_stride + (size_t)kBk * kD;
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt) f.v[dt] = *(const bf16x8 *)(vb + (size_t)(16 * dt + m) * kBk + 8 * (q & 1));
}

// The O^T accumulators live in the accumulation registers, where the matrix cores update them in place.  The
// rare rescale (a moved softmax reference) multiplies copies in ordinary registers; left to itself the
// compiler then keeps the accumulators of the common path in ordinary registers too and moves all of them
// across for every group.  An empty statement that demands its operand in an accumulation register, placed
// where the two paths meet, keeps the copies inside the rare branch.
#define ICARUS_IN_ACC(x) asm volatile("" : "+a"(x))

// Where the decode walks keep the wave's Q fragments: in registers when the wave has two or three query tiles (a
// wave issues in order and is alone on its SIMD, so a fragment read in front of the MFMAs that need it stalls it for
// the read's whole latency, up to twelve times per group); with one tile they stay in LDS, which keeps that
// instantiation at two workgroups per CU.
template <int NT>
constexpr bool kQInRegs = NT > 1;

// Per-wave running state for NT query tiles.
template <int NT>
struct State {
    f32x4 o[kDT][NT];  // O^T accumulators: [d 16dt + 4q + i][query 16qt + l%16]
    float m[NT];       // running max (log2 domain), uniform over the 4 lanes sharing a query
    float l[NT];       // running sum, per-lane partial (reduced over q at the end)
};

// One 32-token group: S^T, online softmax, PV, one 16-query tile at a time so that only one
// tile's scores are live.  Uses the first N tiles of st.  Q fragments of those tiles (B operands): qr, in
// registers, or qlds, in LDS as [qt][ks][lane] (see kQInRegs).
// tail == false: all 32 tokens are valid for every query.
// tail == true:  `left` tokens of the chunk remain from this group's first token on (for the row
//   with the longest context); query tile qt of this lane may attend only to the first
//   left - stag[qt] of them (stag: how many positions the lane's query row ends before the last
//   row -- 0 at decode, the causal stagger of a prefill chunk).
template <int NT, int N, bool tail>
__device__ __forceinline__ void compute_group(State<NT> &st, KVFrag &f, const bf16x8 (&qr)[NT][kKS], const bf16x8 *__restrict__ qlds, int left,
                                              const int (&stag)[NT], float scale_log2, int lane) {
    const int q = lane >> 4;
    // token index inside the group of S^T element (tile t, register i) on this lane: tbase + 4t + i
    const int tbase = 16 * (q >> 1) + 8 * (q & 1);
    if (tail) {
        // stale cache bytes past the end may hold anything: zero those V columns (scores are masked below)
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (tbase + e >= left) f.v[dt][e] = (__bf16)0.f;
    }
#pragma unroll
    for (int qt = 0; qt < N; ++qt) {
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) ICARUS_IN_ACC(st.o[dt][qt]);
        f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {
            const bf16x8 qv = kQInRegs<NT> ? qr[qt][ks] : qlds[(qt * kKS + ks) * 64 + lane];
            s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.k[0][ks], qv, s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.k[1][ks], qv, s1, 0, 0, 0);
        }
        // raw scores; the softmax scale (> 0) is applied to their maximum and inside the exponent's fused
        // multiply-add, not to each score
        float sv[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sv[i] = s0[i];
            sv[4 + i] = s1[i];
        }
        if (tail) {
            const int lim = left - stag[qt];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (tbase + e >= lim) sv[e] = -INFINITY;
        }
        float mx = sv[0];
#pragma unroll
        for (int e = 1; e < 8; ++e) mx = fmaxf(mx, sv[e]);
        mx *= scale_log2;
        // st.m is a reference exponent, not necessarily the exact running max: it moves (and the
        // accumulators are rescaled) only when some score exceeds it by more than kSlack, so
        // p = 2^(s - m) stays below 2^kSlack and the common case needs no cross-lane exchange.
        if (__any(mx > st.m[qt] + kSlack)) {
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float m_old = st.m[qt];
            const float m_new = fmaxf(m_old, mx);
            st.m[qt] = m_new;
            // in a tail group a query may have no valid token yet (m_new still -inf): nothing to rescale
            float alpha = (tail && m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(m_old - m_new);
            st.l[qt] *= alpha;
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) {
                st.o[dt][qt][0] *= alpha; st.o[dt][qt][1] *= alpha; st.o[dt][qt][2] *= alpha; st.o[dt][qt][3] *= alpha;
                ICARUS_IN_ACC(st.o[dt][qt]);
            }
        }
        const float m_ref = st.m[qt];
        float rs = 0.f;
        bf16x8 pb;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[e], scale_log2, -m_ref));
            if (tail && m_ref == -INFINITY) p = 0.f;
            rs += p;
            pb[e] = (__bf16)p;
        }
        st.l[qt] += rs;
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) st.o[dt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.v[dt], pb, st.o[dt][qt], 0, 0, 0);
    }
}

// A wave's walk over its share of the chunk: groups first, first + stride, ... with N query tiles, two register buffers, loads
// issued one group ahead; f0 holds group `first` (or is on its way) when the walk begins.  The first n_clean groups are valid for
// every query; the last ones of the wave, a partial last group among them, are multiplied with masks.  What the loop loads it also
// multiplies: loads that only repeat the last block would hold up the loads of the next piece.  (The loop's own loads are
// unconditional: with a load under a condition the compiler no longer knows how many younger loads are in flight when a buffer
// is consumed and waits for all of them, the prefetch included.)
template <int NT, int N, typename Frag, typename Load, typename Compute>
__device__ __forceinline__ void wave_walk(State<NT> &st, Frag &f0, int n_tok, int first, int stride, Load load, Compute compute) {
    const int n_grp = (n_tok + kGrp - 1) / kGrp;
    Frag f1;
    int grp = first;
#pragma nounroll
    for (; grp + 2 * stride < n_grp; grp += 2 * stride) {
        load(f1, grp + stride);
        compute(std::false_type(), f0, kGrp);
        load(f0, grp + 2 * stride);
        compute(std::false_type(), f1, kGrp);
    }
    if (grp + stride < n_grp) {
        load(f1, grp + stride);
        compute(std::false_type(), f0, kGrp);
        f0 = f1;
        grp += stride;
    }
    if (grp < n_grp) compute(std::true_type(), f0, n_tok - grp * kGrp);
}

// ---- FP8 (E4M3) cache: 1-byte codes, value = code * scale (one scale for K, one for V) ----------------
// The codes are exact in bf16, so they go through the same bf16 MFMAs after a register conversion; the
// scales are folded into the softmax scale (K) and the final normalisation (V).  Loads stay 16 bytes
// per lane for K: a lane's 16 codes are 16 consecutive d of one token, i.e. the lane's operand
// elements of TWO k-steps, so the contraction index is laid out differently from the bf16 path
//   k-step 2s + h, lane quarter q  <->  d = 64 s + 16 q + 8 h .. + 7
// and the Q fragments are staged in the same order (a dot product does not care).  V^T rows hold 16
// tokens in 16 bytes; a lane needs the 8 of its quarter: 8-byte loads, 16 rows x 16 bytes of a block
// fully used by each wave-wide load.
struct KVRaw8 {
    uint4 k[2][2];  // k[t][s]: tile t, d slab s (64 codes per row, 16 per lane)
    uint2 v[kDT];   // v[dt]: 8 tokens of row d = 16 dt + l%16
};

__device__ __forceinline__ void load_group8(KVRaw8 &f, const uint8_t *__restrict__ pool, int blk0, int blk1, int c, int Hkv,
                                            int lane) {
    const int m = lane & 15, q = lane >> 4;
    const size_t head_stride = (size_t)2 * kBk * kD;  // bytes
    const uint8_t *kb = pool + ((size_t)((m >> 3) ? blk1 : blk0) * Hkv + c) * head_stride;
    const int tok0 = 8 * ((m >> 2) & 1) + (m & 3);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) f.k[t][sl] = *(const uint4 *)(kb + (size_t)(tok0 + 4 * t) * kD + 64 * sl + 16 * q);
    const uint8_t *vb = pool + ((size_t)((q >> 1) ? blk1 : blk0) * Hkv + c) * head_stride + (size_t)kBk * kD;
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt) f.v[dt] = *(const uint2 *)(vb + (size_t)(16 * dt + m) * kBk + 8 * (q & 1));
}

// 8 FP8 codes (two dwords) -> 8 bf16, exactly.
__device__ __forceinline__ bf16x8 cvt8(uint32_t lo, uint32_t hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    uint4 r;
    r.x = __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, false));
    r.y = __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, true));
    r.z = __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, false));
    r.w = __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, true));
    return __builtin_bit_cast(bf16x8, r);
}

// compute_group for raw FP8 fragments: the scores of all N tiles first (K codes are converted one
// k-step at a time and die at once), then the softmax of every tile, then PV with V^T codes converted
// one d tile at a time.  scale_log2 includes the K scale; the V scale is applied when the piece ends.
template <int NT, int N, bool tail>
__device__ __forceinline__ void compute_group8(State<NT> &st, const KVRaw8 &f, const bf16x8 (&qr)[NT][kKS], const bf16x8 *__restrict__ qlds, int left,
                                               const int (&stag)[NT], float scale_log2, int lane) {
    const int q = lane >> 4;
    const int tbase = 16 * (q >> 1) + 8 * (q & 1);
    f32x4 s0[N], s1[N];
#pragma unroll
    for (int qt = 0; qt < N; ++qt) {
        s0[qt] = f32x4{0.f, 0.f, 0.f, 0.f}; s1[qt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) ICARUS_IN_ACC(st.o[dt][qt]);
    }
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) {
        const uint4 r0 = f.k[0][ks >> 1], r1 = f.k[1][ks >> 1];
        const bf16x8 a0 = (ks & 1) ? cvt8(r0.z, r0.w) : cvt8(r0.x, r0.y);
        const bf16x8 a1 = (ks & 1) ? cvt8(r1.z, r1.w) : cvt8(r1.x, r1.y);
#pragma unroll
        for (int qt = 0; qt < N; ++qt) {
            const bf16x8 qv = kQInRegs<NT> ? qr[qt][ks] : qlds[(qt * kKS + ks) * 64 + lane];
            s0[qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, qv, s0[qt], 0, 0, 0);
            s1[qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, qv, s1[qt], 0, 0, 0);
        }
    }
    bf16x8 pb[N];
#pragma unroll
    for (int qt = 0; qt < N; ++qt) {
        float sv[8];  // raw scores, see compute_group
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sv[i] = s0[qt][i];
            sv[4 + i] = s1[qt][i];
        }
        if (tail) {
            const int lim = left - stag[qt];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (tbase + e >= lim) sv[e] = -INFINITY;  // also replaces whatever stale codes produced
        }
        float mx = sv[0];
#pragma unroll
        for (int e = 1; e < 8; ++e) mx = fmaxf(mx, sv[e]);
        mx *= scale_log2;
        if (__any(mx > st.m[qt] + kSlack)) {  // see compute_group: lazy softmax reference
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float m_old = st.m[qt];
            const float m_new = fmaxf(m_old, mx);
            st.m[qt] = m_new;
            float alpha = (tail && m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(m_old - m_new);
            st.l[qt] *= alpha;
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) {
                st.o[dt][qt][0] *= alpha; st.o[dt][qt][1] *= alpha; st.o[dt][qt][2] *= alpha; st.o[dt][qt][3] *= alpha;
                ICARUS_IN_ACC(st.o[dt][qt]);
            }
        }
        const float m_ref = st.m[qt];
        float rs = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[e], scale_log2, -m_ref));
            if (tail && m_ref == -INFINITY) p = 0.f;
            rs += p;
            pb[qt][e] = (__bf16)p;
        }
        st.l[qt] += rs;
    }
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt) {
        bf16x8 av = cvt8(f.v[dt].x, f.v[dt].y);
        if (tail) {  // stale codes past the end may decode to anything, NaN included
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (tbase + e >= left) av[e] = (__bf16)0.f;
        }
#pragma unroll
        for (int qt = 0; qt < N; ++qt) st.o[dt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, pb[qt], st.o[dt][qt], 0, 0, 0);
    }
}

// The walk used when the query tiles are split over wave pairs (more than 3 tiles), for an FP8 cache (a bf16
// cache takes shared_walk_dma below).  Every group must reach two waves (one per tile set) but should come
// from HBM once and stay a distinct load in flight, so loading and computing are decoupled: in each round of
// four groups wave w loads the raw codes of group 4r + w into registers, expands them to bf16 MFMA fragments
// (k-step order of KVRaw8) as it publishes them to an LDS ring in lane order, and after one barrier computes
// the two groups of its parity (half) for its own tiles from the ring.  The loads of the next round are in
// flight while a round is computed.  ring: [2][4][16][64] x 16 B.
template <int NT, int N>
__device__ __forceinline__ void shared_walk8(State<NT> &st, const uint8_t *__restrict__ pool8, const int *__restrict__ blds,
                                             int n_blk, int n_tok, int n_clean, const int (&stag)[NT], int w, int half, int c,
                                             int Hkv, bf16x8 *__restrict__ ring, const bf16x8 (&qr)[NT][kKS], const bf16x8 *__restrict__ qlds,
                                             float scale_log2, int lane) {
    const int n_grp = (n_tok + kGrp - 1) / kGrp;                       // groups, the masked ones included
    const int n_round = (n_grp + 3) / 4;                               // the same for every wave
    auto blk_of = [&](int grp, int which) {
        return __builtin_amdgcn_readfirstlane(blds[min(grp * 2 + which, n_blk - 1)]);
    };
    KVRaw8 f8;
    auto load = [&](int grp) { load_group8(f8, pool8, blk_of(grp, 0), blk_of(grp, 1), c, Hkv, lane); };
    if (w < n_grp) load(w);
#pragma nounroll
    for (int r = 0; r < n_round; ++r) {
        bf16x8 *stage = ring + (size_t)(r & 1) * 4 * 16 * 64;
        const int mine = 4 * r + w;
        if (mine < n_grp) {
            bf16x8 *dst = stage + (size_t)w * 16 * 64 + lane;
#pragma unroll
            for (int i = 0; i < 2 * kKS; ++i) {
                const uint4 rk = f8.k[i / kKS][(i % kKS) >> 1];
                dst[i * 64] = (i & 1) ? cvt8(rk.z, rk.w) : cvt8(rk.x, rk.y);
            }
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) dst[(2 * kKS + dt) * 64] = cvt8(f8.v[dt].x, f8.v[dt].y);
        }
        if (mine + 4 < n_grp) load(mine + 4);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int gi = half + 2 * u, grp = 4 * r + gi;
            if (grp < n_grp) {
                const bf16x8 *src = stage + (size_t)gi * 16 * 64 + lane;
                KVFrag gfr;
#pragma unroll
                for (int i = 0; i < 2 * kKS; ++i) gfr.k[i / kKS][i % kKS] = src[i * 64];
#pragma unroll
                for (int dt = 0; dt < kDT; ++dt) gfr.v[dt] = src[(2 * kKS + dt) * 64];
                if (grp >= n_clean)
                    compute_group<NT, N, true>(st, gfr, qr, qlds, n_tok - grp * kGrp, stag, scale_log2, lane);
                else
                    compute_group<NT, N, false>(st, gfr, qr, qlds, kGrp, stag, scale_log2, lane);
            }
        }
    }
    __syncthreads();  // the ring may be reused now
}

// 16-byte LDS-direct load: lane i copies 16 bytes from its own global address to LDS byte lds_base + 16 i
// (lds_base wave-uniform, passed in m0); the load counts in vmcnt until the data is in LDS.
__device__ __forceinline__ void dma16(const void *g, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(g) : "memory");
}

// The shared walk of a bf16 cache with the ring filled by LDS-direct loads.  A wave's 16-byte loads of a
// group ARE its MFMA fragments in lane order, so they can land in the ring as they are: no register buffer,
// and what is in flight is bounded by LDS, not by VGPRs.  The ring (the same 128 KB) is cut into four
// stages of two groups; in round r wave w loads half (w & 1: K or V^T fragments) of group 2r + w/2, three
// rounds ahead -- 96 KB in flight per CU against 64 KB with one group per wave in registers, which is what
// the five-tile walk was short of (a round waited for the load issued one round earlier).  Each wave issues
// exactly 8 loads per round (a group past the end is clamped to the last one and never read), so the
// number of younger loads at a wait is known: vmcnt(16) leaves the two younger rounds in flight.  One
// barrier per round: after it every wave's loads of round r are in LDS and every wave has finished round
// r-1, whose stage takes the loads of round r+3.
template <int NT, int N>
__device__ __forceinline__ void shared_walk_dma(State<NT> &st, const bf16_t *__restrict__ pool, const int *__restrict__ blds,
                                                int n_blk, int n_tok, int n_clean, const int (&stag)[NT], int w, int half, int c,
                                                int Hkv, bf16x8 *__restrict__ ring, const bf16x8 (&qr)[NT][kKS], const bf16x8 *__restrict__ qlds,
                                                float scale_log2, int lane) {
    constexpr int kStages = 4, kStageFrags = 2 * 16;  // fragments (1 KiB each) per stage
    static_assert(kRingBytes == (size_t)kStages * kStageFrags * 1024, "ring size");
    const int n_grp = (n_tok + kGrp - 1) / kGrp;
    const int n_round = (n_grp + 1) / 2;
    const int part = w & 1, gl = w >> 1;
    const int m = lane & 15, q = lane >> 4;
    const size_t head_stride = (size_t)2 * kBk * kD;
    const uint32_t ring0 = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)ring;
    auto issue = [&](int r) {
        const int grp = min(2 * r + gl, n_grp - 1);
        const int blk0 = __builtin_amdgcn_readfirstlane(blds[min(grp * 2, n_blk - 1)]);
        const int blk1 = __builtin_amdgcn_readfirstlane(blds[min(grp * 2 + 1, n_blk - 1)]);
        const uint32_t dst = __builtin_amdgcn_readfirstlane(ring0 + ((r & (kStages - 1)) * kStageFrags + gl * 16 + part * 8) * 1024);
        if (part == 0) {  // K fragments k[t][ks]: block m/8, token 8((m/4)%2) + 4t + m%4, d = 32ks + 8q
            const bf16_t *kb = pool + ((size_t)((m >> 3) ? blk1 : blk0) * Hkv + c) * head_stride +
                               (size_t)(8 * ((m >> 2) & 1) + (m & 3)) * kD + 8 * q;
#pragma unroll
            for (int i = 0; i < 2 * kKS; ++i) dma16(kb + (size_t)(4 * (i / kKS)) * kD + 32 * (i % kKS), dst + i * 1024);
        } else {  // V^T fragments v[dt]: block q/2, d = 16dt + m, tokens 8(q%2) .. +7
            const bf16_t *vb = pool + ((size_t)((q >> 1) ? blk1 : blk0) * Hkv + c) * head_stride + (size_t)kBk * kD +
                               (size_t)m * kBk + 8 * (q & 1);
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) dma16(vb + (size_t)(16 * dt) * kBk, dst + dt * 1024);
        }
    };
#pragma unroll
    for (int r = 0; r < kStages - 1; ++r)
        if (r < n_round) issue(r);
#pragma nounroll
    for (int r = 0; r < n_round; ++r) {
        const int younger = min(n_round, r + kStages - 1) - (r + 1);  // rounds this wave has issued after round r
        if (younger >= 2) __builtin_amdgcn_s_waitcnt(0x0f70 | 0x4000);  // vmcnt(16)
        else if (younger == 1) __builtin_amdgcn_s_waitcnt(0x0f70 | 8);  // vmcnt(8)
        else __builtin_amdgcn_s_waitcnt(0x0f70);                        // vmcnt(0)
        __syncthreads();
        if (r + kStages - 1 < n_round) issue(r + kStages - 1);
        const int grp = 2 * r + half;
        if (grp < n_grp) {
            const bf16x8 *src = ring + ((size_t)(r & (kStages - 1)) * kStageFrags + half * 16) * 64 + lane;
            KVFrag gfr;
#pragma unroll
            for (int i = 0; i < 2 * kKS; ++i) gfr.k[i / kKS][i % kKS] = src[i * 64];
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) gfr.v[dt] = src[(2 * kKS + dt) * 64];
            if (grp >= n_clean)
                compute_group<NT, N, true>(st, gfr, qr, qlds, n_tok - grp * kGrp, stag, scale_log2, lane);
            else
                compute_group<NT, N, false>(st, gfr, qr, qlds, kGrp, stag, scale_log2, lane);
        }
    }
    __syncthreads();  // the ring may be reused now
}

// LDS image of a state: o as [dt][qt][i][lane], then m[qt][lane], l[qt][lane].
template <int NT>
__device__ __forceinline__ void merge_from_lds(State<NT> &st, const float *__restrict__ lds, int lane) {
    const float *lo = lds;
    const float *lm = lds + kDT * NT * 4 * 64;
    const float *ll = lm + NT * 64;
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        float m2 = lm[qt * 64 + lane], l2 = ll[qt * 64 + lane];
        float mn = fmaxf(st.m[qt], m2);
        float a1 = st.m[qt] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(st.m[qt] - mn);
        float a2 = m2 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m2 - mn);
        st.m[qt] = mn;
        st.l[qt] = st.l[qt] * a1 + l2 * a2;
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) st.o[dt][qt][i] = st.o[dt][qt][i] * a1 + lo[((dt * NT + qt) * 4 + i) * 64 + lane] * a2;
    }
}
template <int NT>
__device__ __forceinline__ void store_to_lds(const State<NT> &st, float *__restrict__ lds, int lane) {
    float *lo = lds;
    float *lm = lds + kDT * NT * 4 * 64;
    float *ll = lm + NT * 64;
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        lm[qt * 64 + lane] = st.m[qt];
        ll[qt * 64 + lane] = st.l[qt];
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) lo[((dt * NT + qt) * 4 + i) * 64 + lane] = st.o[dt][qt][i];
    }
}

// The four waves' states of a piece, each over its own groups, put together: every wave leaves its state in LDS (image_store) and, after a
// barrier, each takes a quarter of the head dimension (image_finish): d tiles 2w, 2w + 1 of all queries.
template <int NT>
struct Image {
    static constexpr int kO = kDT * NT * 64, kBytes = kO * 16 + NT * 64 * 8;  // f32x4 [dt][qt][lane], float2 (max, sum) [qt][lane]
};
template <int NT>
__device__ __forceinline__ void image_store(const State<NT> &st, char *__restrict__ img, int lane) {
    f32x4 *o = (f32x4 *)img;
    float2 *ml = (float2 *)(img + Image<NT>::kO * 16);
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        ml[qt * 64 + lane] = make_float2(st.m[qt], st.l[qt]);
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) o[(dt * NT + qt) * 64 + lane] = st.o[dt][qt];
    }
}
template <int NT, typename ReadDone>
__device__ __forceinline__ void image_finish(const char *__restrict__ imgs, int w, int G, int g, int row0, int c, int Hq, int Hkv, int direct, int slot,
                                             int g_max, float v_scale, bf16_t *__restrict__ out, float *__restrict__ part_o,
                                             float *__restrict__ part_ml, int lane, ReadDone read_done) {
    const int m = lane & 15, q = lane >> 4;
    f32x4 o[NT][2];
    float mn[NT], l[NT];
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        float2 ml[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) ml[k] = ((const float2 *)(imgs + k * Image<NT>::kBytes + Image<NT>::kO * 16))[qt * 64 + lane];
        mn[qt] = fmaxf(fmaxf(ml[0].x, ml[1].x), fmaxf(ml[2].x, ml[3].x));
        l[qt] = 0.f;
#pragma unroll
        for (int h = 0; h < 2; ++h) o[qt][h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float a = ml[k].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[k].x - mn[qt]);  // a wave without groups
            l[qt] += a * ml[k].y;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 v = ((const f32x4 *)(imgs + k * Image<NT>::kBytes))[((2 * w + h) * NT + qt) * 64 + lane];
#pragma unroll
                for (int i = 0; i < 4; ++i) o[qt][h][i] += a * v[i];
            }
        }
    }
    read_done();
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        l[qt] += __shfl_xor(l[qt], 16, 64);
        l[qt] += __shfl_xor(l[qt], 32, 64);
        const int j = 16 * qt + m;
        if (j >= G) continue;
        if (direct) {
            const float inv = v_scale / l[qt];
            bf16_t *op = out + ((size_t)(row0 + j / g) * Hq + c * g + j % g) * kD + 32 * w + 4 * q;
#pragma unroll
            for (int h = 0; h < 2; ++h)
                *(uint2 *)(op + 16 * h) = make_uint2(pack_bf16(o[qt][h][0] * inv, o[qt][h][1] * inv), pack_bf16(o[qt][h][2] * inv, o[qt][h][3] * inv));
        } else {
            const size_t pj = ((size_t)slot * Hkv + c) * g_max + j;
#pragma unroll
            for (int h = 0; h < 2; ++h) *(f32x4 *)(part_o + pj * kD + 32 * w + 16 * h + 4 * q) = o[qt][h] * v_scale;
            if (w == 0 && q == 0) *(float2 *)(part_ml + pj * 2) = make_float2(mn[qt], l[qt]);
        }
    }
}

// Write tiles [0, n) of st as the call's query tiles qt0 .. qt0+n-1: the final output when the
// sequence has a single chunk, else this chunk's partial result.
template <int NT>
__device__ __forceinline__ void finish(State<NT> &st, int qt0, int n, int G, int g, int row0, int c, int Hq, int Hkv,
                                       int direct, int slot, int g_max, bf16_t *__restrict__ out,
                                       float *__restrict__ part_o, float *__restrict__ part_ml, int lane) {
    const int m = lane & 15, q = lane >> 4;
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        float l = st.l[qt];
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        int j = 16 * (qt0 + qt) + m;
        if (qt >= n || j >= G) continue;
        if (direct) {
            float inv = 1.f / l;
            bf16_t *op = out + ((size_t)(row0 + j / g) * Hq + c * g + j % g) * kD;
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) {
                uint2 pk;
                pk.x = pack_bf16(st.o[dt][qt][0] * inv, st.o[dt][qt][1] * inv);
                pk.y = pack_bf16(st.o[dt][qt][2] * inv, st.o[dt][qt][3] * inv);
                *(uint2 *)(op + 16 * dt + 4 * q) = pk;
            }
        } else {
            size_t pj = ((size_t)slot * Hkv + c) * g_max + j;
            float *po = part_o + pj * kD;
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) *(f32x4 *)(po + 16 * dt + 4 * q) = st.o[dt][qt];
            if (q == 0) {
                part_ml[pj * 2] = st.m[qt];
                part_ml[pj * 2 + 1] = l;
            }
        }
    }
}

// 4-byte LDS-direct load, as dma16
__device__ __forceinline__ void dma4(const void *g, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_base), "v"(g) : "memory");
}
__device__ uint4 g_zero_query;  // source of Q fragments past a sequence's last query

// A piece as its workgroups read it (AttnPlan::pieces).
struct Piece {
    int row0, rows, bt_row, begin, n_tok, slot;
    bool direct, last;  // last: of its share
    __device__ __forceinline__ Piece(const int32_t *p)
        : row0(p[0] & 0xffff), rows(p[0] >> 16), bt_row(p[1]), begin(p[2]), n_tok(p[3] & kPieceTokens), slot(p[4]), direct(p[3] & kPieceDirect), last(p[3] & kPieceLast) {}
};

// Up to three query tiles: every wave holds all of them and takes every fourth group of the piece.  KV8: the pool holds FP8 codes
// (scale_log2 then includes the K scale, v_scale multiplies the output).
//
// A workgroup walks the pieces of its share one after the other, and between two of them nothing of it would be under way: the next piece's
// numbers, its Q and block ids, its first keys and values each wait for the one before.  So the Q and ids of the next piece are requested (LDS-direct,
// into the other of two buffers) before this one is walked, and its first groups as soon as the waves' states are in LDS: the merge
// runs under them.  A merge of two halvings through single floats, and each piece from nothing, took, us before / now: 16 sequences of
// 500-8192 tokens, 72 k in all 60.3 / 57.0 (5.2 TB/s), one of 4096 14.5 / 12.0, 32 of 1024-8192 114 / 112, 64 of 1024-16384 418 / 416.5: long walks
// are held by what HBM gives (5.6 TB/s of permuted blocks, where plain reads get 6.1).  Two workgroups of one query tile to a CU: no gain (112.6).
template <int NT, bool KV8>
__global__ void __launch_bounds__(256) k_attn_decode(const bf16_t *__restrict__ qg, const void *__restrict__ pool_v, const int32_t *__restrict__ bt,
                                                     int max_blocks, AttnPlan pl, bf16_t *__restrict__ out, float *__restrict__ part_o,
                                                     float *__restrict__ part_ml, int Hq, int Hkv, float scale_log2, float v_scale) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    // LDS: the waves' states | two buffers of Q fragments [qt][ks][lane] | two of block ids
    constexpr int kQBytes = NT * kKS * 1024, kQAt = 4 * Image<NT>::kBytes, kIdsAt = kQAt + 2 * kQBytes;
    static_assert(kQAt % 1024 == 0 || Image<NT>::kBytes % 512 == 0, "16-byte aligned");
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)smem;
    const int ids_bytes = ((pl.chunk + kBk - 1) / kBk * 4 + 255) & ~255;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = Hq / Hkv, m = lane & 15, q = lane >> 4;
    // the Hkv workgroups of a share (one per kv-head, on different XCDs) walk the same blocks at about the same time
    const int share = blockIdx.x / Hkv, c = blockIdx.x % Hkv;
    Piece p(pl.pieces + 5 * share);
    int next = pl.share_next[share];
    // query j = 16qt + m  ->  row row0 + j / g, head c*g + j % g; wave w brings k-step w: d = 32 w + 8 q (bf16 cache),
    // d = 64 (w / 2) + 16 q + 8 (w % 2) (FP8 cache, see KVRaw8)
    auto stage = [&](const Piece &p, int buf) {
        const int d0 = KV8 ? 64 * (w >> 1) + 16 * q + 8 * (w & 1) : 8 * q + 32 * w;
#pragma unroll
        for (int qt = 0; qt < NT; ++qt) {
            const int j = 16 * qt + m;
            const bf16_t *qp = qg + ((size_t)(p.row0 + j / g) * Hq + c * g + j % g) * kD + d0;
            dma16(j < p.rows * g ? (const void *)qp : (const void *)&g_zero_query, lds0 + kQAt + buf * kQBytes + (qt * kKS + w) * 1024);
        }
        const int32_t *ids = bt + (size_t)p.bt_row * max_blocks + p.begin / kBk;
        const int n_blk = (p.n_tok + kBk - 1) / kBk;
        for (int i = 64 * w; i < n_blk; i += 256) dma4(ids + min(i + lane, n_blk - 1), lds0 + kIdsAt + buf * ids_bytes + i * 4);
    };
    typedef typename std::conditional<KV8, KVRaw8, KVFrag>::type Frag;
    auto load = [&](Frag &f, const Piece &p, int buf, int grp) {
        const int *ids = (const int *)(smem + kIdsAt + buf * ids_bytes);
        const int n_blk = (p.n_tok + kBk - 1) / kBk;
        const int b0 = __builtin_amdgcn_readfirstlane(ids[min(2 * grp, n_blk - 1)]), b1 = __builtin_amdgcn_readfirstlane(ids[min(2 * grp + 1, n_blk - 1)]);
        if constexpr (KV8) load_group8(f, (const uint8_t *)pool_v, b0, b1, c, Hkv, lane);
        else load_group(f, (const bf16_t *)pool_v, b0, b1, c, Hkv, lane);
    };
    // this wave's loads into LDS have landed and its LDS accesses are done; then those of all waves
    auto meet = [] { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    stage(p, 0);
    meet();
    Frag f0;
    load(f0, p, 0, w);
    for (int buf = 0;; buf ^= 1) {
        const Piece nx(pl.pieces + 5 * (p.last ? share : next));
        const bf16x8 *qlds = (const bf16x8 *)(smem + kQAt + buf * kQBytes);
        // the wave's Q fragments, see kQInRegs
        bf16x8 qr[NT][kKS];
        if constexpr (kQInRegs<NT>) {
#pragma unroll
            for (int qt = 0; qt < NT; ++qt)
#pragma unroll
                for (int ks = 0; ks < kKS; ++ks) qr[qt][ks] = qlds[(qt * kKS + ks) * 64 + lane];
        }
        if (!p.last) stage(nx, buf ^ 1);
        State<NT> st;
        int stag[NT];  // every stacked query of a decode step sits at the same position
#pragma unroll
        for (int qt = 0; qt < NT; ++qt) {
            st.m[qt] = -INFINITY;
            st.l[qt] = 0.f;
            stag[qt] = 0;
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) st.o[dt][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        // the launch is sized for the largest stacked group of the call; a sequence with fewer
        // streams multiplies only the query tiles it has
        auto walk = [&](auto tiles) {
            constexpr int N = decltype(tiles)::value;
            auto compute = [&](auto kind, Frag &f, int left) {
                constexpr bool tail = decltype(kind)::value;
                if constexpr (KV8) compute_group8<NT, N, tail>(st, f, qr, qlds, left, stag, scale_log2, lane);
                else compute_group<NT, N, tail>(st, f, qr, qlds, left, stag, scale_log2, lane);
            };
            wave_walk<NT, N>(st, f0, p.n_tok, w, 4, [&](Frag &f, int grp) { load(f, p, buf, grp); }, compute);
        };
        const int n_act = (p.rows * g + 15) >> 4;
        if (NT >= 3 && n_act >= 3) walk(std::integral_constant<int, NT>());
        else if (NT >= 2 && n_act == 2) walk(std::integral_constant<int, (NT >= 2 ? 2 : 1)>());
        else walk(std::integral_constant<int, 1>());
        image_store<NT>(st, smem + w * Image<NT>::kBytes, lane);
        meet();
        if (!p.last) load(f0, nx, buf ^ 1, w);
        image_finish<NT>(smem, w, p.rows * g, g, p.row0, c, Hq, Hkv, p.direct, p.slot, pl.g_max, v_scale, out, part_o, part_ml, lane,
                         [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); });  // the states' LDS is free again
        if (p.last) break;
        p = nx;
        next = next + 1;
    }
}

// Four and five query tiles: NA tiles of waves 0,1, NB of waves 2,3.
template <int NA, int NB, bool KV8>
__global__ void __launch_bounds__(256) k_attn_decode_pairs(const bf16_t *__restrict__ qg, const void *__restrict__ pool_v,
                                                     const int32_t *__restrict__ bt, int max_blocks, AttnPlan pl,
                                                     bf16_t *__restrict__ out, float *__restrict__ part_o,
                                                     float *__restrict__ part_ml, int Hq, int Hkv, float scale_log2,
                                                     float v_scale) {
    const bf16_t *pool = (const bf16_t *)pool_v;
    constexpr int NQT = NA + NB;
    constexpr int kImg = kDT * NA * 4 * 64 + 2 * NA * 64;  // floats per wave image of the merge
    extern __shared__ float lds[];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int g = Hq / Hkv;
    const int m = lane & 15, q = lane >> 4;
  // the pieces of this workgroup's share, one after the other; the Hkv workgroups of a share (one per
  // kv-head, on different XCDs) walk the same blocks at about the same time
  const int share = blockIdx.x / Hkv, c = blockIdx.x % Hkv;
  for (int item = share, next = pl.share_next[share];; item = next++) {
    const Piece p(pl.pieces + 5 * item);
    const int tok_begin = p.begin, n_tok = p.n_tok;
    const int row0 = p.row0;
    const int G = p.rows * g;
    const int32_t *btr = bt + (size_t)p.bt_row * max_blocks;

    // Q fragments (B operands) go to LDS once, as [qt][ks][lane]; wave w stages k-step w.
    // query j = 16qt + m  ->  row row0 + j / g, head c*g + j % g; rows past G are zero.
    // LDS: [merge images | KV ring] [Q fragments] [block ids]; the merge images reuse the ring.
    static_assert(kRingBytes >= (size_t)2 * kImg * sizeof(float), "merge images must fit the ring");
    bf16x8 *qlds = (bf16x8 *)((char *)lds + kRingBytes);
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) {
        int j = 16 * qt + m;
        // k-step w of this lane: d = 32 w + 8 q (bf16 cache), d = 64 (w / 2) + 16 q + 8 (w % 2) (FP8 cache, see KVRaw8)
        const int d0 = KV8 ? 64 * (w >> 1) + 16 * q + 8 * (w & 1) : 8 * q + 32 * w;
        const bf16_t *qp = qg + ((size_t)(row0 + j / g) * Hq + c * g + j % g) * kD + d0;
        qlds[(qt * kKS + w) * 64 + lane] = j < G ? *(const bf16x8 *)qp : zero8();
    }
    // The chunk's block ids go to LDS too: a lookup in the loop is then an LDS read, not a global
    // load whose wait would also drain the KV loads in flight.
    int *blds = (int *)(qlds + NQT * kKS * 64);
    const int n_blk = (n_tok + kBk - 1) / kBk;
    for (int i = threadIdx.x; i < n_blk; i += 256) blds[i] = btr[tok_begin / kBk + i];
    __syncthreads();
    // the wave's own Q fragments, see kQInRegs (waves 2, 3 of a launch with NB tiles hold tiles NA .. NA + NB - 1)
    bf16x8 qr[NA][kKS];
    if constexpr (kQInRegs<NA>) {
        const bool second = w >> 1;
        const bf16x8 *qsrc = qlds + (second ? NA * kKS * 64 : 0) + lane;
        const int nq = second ? NB : NA;
#pragma unroll
        for (int qt = 0; qt < NA; ++qt)
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) qr[qt][ks] = qt < nq ? qsrc[(qt * kKS + ks) * 64] : zero8();
    }

    State<NA> st;
#pragma unroll
    for (int qt = 0; qt < NA; ++qt) {
        st.m[qt] = -INFINITY;
        st.l[qt] = 0.f;
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) st.o[dt][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int direct = p.direct, slot = p.slot;
    // every stacked query of a decode step sits at the same position: all whole groups need no mask
    const int n_clean = n_tok / kGrp;
    int stag[NA];
#pragma unroll
    for (int qt = 0; qt < NA; ++qt) stag[qt] = 0;

    const int role = w >> 1, half = w & 1;  // role: which query tiles; half: which groups
    bf16x8 *ring = (bf16x8 *)lds;
    if constexpr (KV8) {  // codes are expanded on the way into the ring: through registers
        const uint8_t *pool8 = (const uint8_t *)pool_v;
        if (role == 0)
            shared_walk8<NA, NA>(st, pool8, blds, n_blk, n_tok, n_clean, stag, w, half, c, Hkv, ring, qr, qlds, scale_log2, lane);
        else
            shared_walk8<NA, NB>(st, pool8, blds, n_blk, n_tok, n_clean, stag, w, half, c, Hkv, ring, qr, qlds,
                                 scale_log2, lane);
    } else if (role == 0) {
        shared_walk_dma<NA, NA>(st, pool, blds, n_blk, n_tok, n_clean, stag, w, half, c, Hkv, ring, qr, qlds, scale_log2, lane);
    } else {
        shared_walk_dma<NA, NB>(st, pool, blds, n_blk, n_tok, n_clean, stag, w, half, c, Hkv, ring, qr, qlds,
                                scale_log2, lane);
    }
    if constexpr (KV8) {
#pragma unroll
        for (int qt = 0; qt < NA; ++qt)
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) {
                st.o[dt][qt][0] *= v_scale; st.o[dt][qt][1] *= v_scale; st.o[dt][qt][2] *= v_scale; st.o[dt][qt][3] *= v_scale;
            }
    }
    // each pair merges its two halves through its own LDS image
    if (half == 1) store_to_lds<NA>(st, lds + role * kImg, lane);
    __syncthreads();
    if (half == 0) {
        merge_from_lds<NA>(st, lds + role * kImg, lane);
        finish<NA>(st, role ? NA : 0, role ? NB : NA, G, g, row0, c, Hq, Hkv, direct, slot, pl.g_max, out, part_o, part_ml, lane);
    }
    if (p.last) break;
    __syncthreads();  // LDS (Q fragments, block ids, merge images) is reused by the next piece
  }
}

constexpr int kPrefillWaves = 4, kPrefillNT = 4;  // 4 waves x 4 tiles x 16 = 256 stacked queries per workgroup
constexpr int kRoundGroups = 4;                   // 32-token groups of a round of the prefill walk

template <int V> struct Int { static constexpr int value = V; };
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

// The walk of one prefill wave over a piece, its four query tiles as two pairs.  The arithmetic of a tile, in its order and its
// precision, is that of compute_group_lds: the same bits from both kernels.
//
// A wave is alone on its SIMD and issues in order, so it has to put its own vector instructions beneath its own MFMAs: an
// MFMA takes the pipe 16 cycles and the issue slot 4.  Group g is four steps of 16 MFMAs, each with independent work of
// the other pair between them, in the order they are written here (a scheduling barrier behind every MFMA):
//     1  S^T of pair 0                  exponentials of pair 1 of group g - 1
//     2  P V of pair 1 of group g - 1   their sum; V^T fragments of g into the registers this leaves; the check of pair 0's scores
//     3  S^T of pair 1                  exponentials of pair 0
//     4  P V of pair 0                  their sum; K fragments of g + 1; the check of pair 1's scores
// The check: the softmax reference is lazy (see compute_group), it moves only when a score exceeds it by more than kSlack.
// 32 chunks of 512 rows over 8192 tokens, 32 query heads: 2.34 ms with eight waves of two tiles, 2.21 here (1.03 PFLOP/s).  The
// vector instructions bound it: beside an MFMA one is free (8.8 ns), each further one costs 1.3-1.7 ns.  The scale rounded into q,
// scores that start from minus the reference in the accumulators and denominators by an MFMA over the rounded probabilities took
// 32 multiply-adds and 32 additions out of a group, 1.95 ms; but sums of probabilities in 16 bits are fewer bits than the callers had.
//
// The ring has two stages of one round (four groups) each; the four waves bring a quarter of each group (K rows or V^T rows)
// by LDS-direct loads, and read every group as MFMA fragments in lane order.  A stage is filled while the other one is read: the
// loads for round r + 1 are issued beside steps 2 and 4 of the first two groups of round r.  A stage's last reads precede
// the one barrier of a round, which sits before the first reads of the next round.  Past the end of the piece the loads repeat its last block.
// ring: [2][4][16][64] x 16 B.
struct PrefillWalk {
    State<kPrefillNT> &st;
    bf16x8 (&qr)[kPrefillNT][kKS];
    const int (&stag)[kPrefillNT];
    const float scale;
    const int lane;
    float neg[kPrefillNT];    // minus the reference (State::m); 0 while there is none
    float limit[kPrefillNT];  // the largest scaled score that leaves the reference alone
    f32x4 sc[kPrefillNT][2];  // scores of the two 16-token halves of a group, then their exponentials
    float sum[kPrefillNT];    // of a group's exponentials
    bf16x8 pb[kPrefillNT];    // probabilities
    bf16x8 kf[2 * kKS], vf[kDT];
    float top[2];             // of a check: the largest scaled score of each tile of the pair

    __device__ __forceinline__ PrefillWalk(State<kPrefillNT> &s, bf16x8 (&q)[kPrefillNT][kKS], const int (&g)[kPrefillNT], float f, int l)
        : st(s), qr(q), stag(g), scale(f), lane(l) {
#pragma unroll
        for (int t = 0; t < kPrefillNT; ++t) {
            neg[t] = 0.f;
            limit[t] = -INFINITY;
        }
        none_pending();
    }
    // a pair 1 of no group: probabilities of zero
    __device__ __forceinline__ void none_pending() {
#pragma unroll
        for (int t = 2; t < kPrefillNT; ++t) sc[t][0] = sc[t][1] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) vf[dt] = zero8();
    }
    // MFMA m of 16 of the scores of pair P.  In assembly: the compiler gives every MFMA of a kernel that may use the accumulation
    // registers its result in them, and the scores would be copied out for the arithmetic.  What reads a result is at least
    // four MFMAs (64 cycles) behind it.
    template <int P>
    __device__ __forceinline__ void score(int m) {
        const int ks = m >> 2, t = 2 * P + ((m >> 1) & 1), hf = m & 1;
        if (ks == 0) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(sc[t][hf]) : "v"(kf[4 * hf]), "a"(qr[t][0]));
        else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(sc[t][hf]) : "v"(kf[4 * hf + ks]), "a"(qr[t][ks]));
    }
    // MFMA m of 16 of P V of pair P
    template <int P>
    __device__ __forceinline__ void pv(int m) {
        const int dt = m >> 1, t = 2 * P + (m & 1);
        st.o[dt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], pb[t], st.o[dt][t], 0, 0, 0);
    }
    // element i of the 16 of pair P
    template <int P> __device__ __forceinline__ float at(int i) const { return sc[2 * P + (i >> 3)][(i >> 2) & 1][i & 3]; }
    // exponential i of the 16 of pair P, beside the exponent of the next one and the rounding of those before it (i = 16: the last
    // two); exponent(0) goes before
    template <int P>
    __device__ __forceinline__ void exponent(int i) {
        const int t = 2 * P + (i >> 3);
        sc[t][(i >> 2) & 1][i & 3] = __builtin_fmaf(at<P>(i), scale, neg[t]);
    }
    template <int P>
    __device__ __forceinline__ void exp_one(int i) {
        if (i < 16) {
            const int t = 2 * P + (i >> 3);
            sc[t][(i >> 2) & 1][i & 3] = __builtin_amdgcn_exp2f(at<P>(i));
        }
        if (i + 1 < 16) exponent<P>(i + 1);
        if (i == 0) return;
        const int t = 2 * P + ((i - 1) >> 3), e = (i - 1) & 7;
        if (!(e & 1)) return;
        uint32_t two = pack_bf16(at<P>(i - 2), at<P>(i - 1));
        asm volatile("" : "+v"(two));  // here, not all of them ahead of the next step's MFMAs
        u32x4 w = __builtin_bit_cast(u32x4, pb[t]);
        w[e >> 1] = two;
        pb[t] = __builtin_bit_cast(bf16x8, w);
    }
    // addition i of the 16 of pair P to the denominators: float32, of the unrounded exponentials
    template <int P>
    __device__ __forceinline__ void add_one(int i) {
        const int t = 2 * P + (i >> 3);
        sum[t] = i & 7 ? sum[t] + at<P>(i) : at<P>(i);
        asm volatile("" : "+v"(sum[t]));
        if ((i & 7) == 7) st.l[t] += sum[t];
    }
    // part i of kCheckParts of pair P's check (v_max3 by hand: for fmaxf the compiler first turns every score into itself, in case it
    // were a signalling NaN)
    static constexpr int kCheckParts = 10;
    template <int P>
    __device__ __forceinline__ void check_part(int i) {
        float &x = top[i / 5];
        const int e = 8 * (i / 5), k = i % 5;
        if (k == 0) asm("v_max3_f32 %0, %1, %2, %3" : "=v"(x) : "v"(at<P>(e)), "v"(at<P>(e + 1)), "v"(at<P>(e + 2)));
        else if (k < 3) asm("v_max3_f32 %0, %0, %1, %2" : "+v"(x) : "v"(at<P>(e + 2 * k + 1)), "v"(at<P>(e + 2 * k + 2)));
        else if (k == 3) asm("v_max_f32 %0, %0, %1" : "+v"(x) : "v"(at<P>(e + 7)));
        else x *= scale;
    }
    // After the check of pair P: the reference of a tile of which a score exceeds its limit is moved up to their maximum.
    template <int P>
    __device__ __forceinline__ void move_reference() {
        if (__builtin_expect(!__any(top[0] > limit[2 * P] || top[1] > limit[2 * P + 1]), 1)) return;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int t = 2 * P + i;
            if (!__any(top[i] > limit[t])) continue;
            float mx = fmaxf(top[i], __shfl_xor(top[i], 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float m_old = st.m[t], m_new = fmaxf(m_old, mx);
            const bool none = m_new == -INFINITY;  // the query has had no valid token yet: nothing to rescale
            const float alpha = none ? 1.f : __builtin_amdgcn_exp2f(m_old - m_new);
            st.m[t] = m_new;
            neg[t] = none ? 0.f : -m_new;
            limit[t] = m_new + kSlack;
            st.l[t] *= alpha;
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) {
                st.o[dt][t][0] *= alpha; st.o[dt][t][1] *= alpha; st.o[dt][t][2] *= alpha; st.o[dt][t][3] *= alpha;
                ICARUS_IN_ACC(st.o[dt][t]);
            }
        }
    }
    // scores of the tokens that a query does not attend to
    template <int P>
    __device__ __forceinline__ void mask(int left) {
        const int q = lane >> 4, tbase = 16 * (q >> 1) + 8 * (q & 1);
#pragma unroll
        for (int t = 2 * P; t < 2 * P + 2; ++t)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (tbase + e >= left - stag[t]) sc[t][e >> 2][e & 3] = -INFINITY;
    }
    // One group.  src: its fragments; next: those of the group after it, in the next round (LAST: read after before_next()) or
    // in this one.  between: runs beside steps 2 and 4, part i of 8.  MASKED: one of the last groups, `left` tokens of the sequence
    // remain from its first on for its last row; else every query attends to all of it.
    template <bool LAST, bool MASKED, typename Between, typename BeforeNext>
    __device__ __forceinline__ void group(const bf16x8 *__restrict__ src, const bf16x8 *__restrict__ next, int left, Between between, BeforeNext before_next) {
#pragma unroll
        for (int t = 0; t < kPrefillNT; ++t) {
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) ICARUS_IN_ACC(st.o[dt][t]);
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) ICARUS_IN_ACC(qr[t][ks]);
            asm volatile("" : "+v"(sc[t][0]), "+v"(sc[t][1]), "+v"(neg[t]));
        }
        exponent<1>(0);
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            score<0>(m);
            exp_one<1>(m);
            __builtin_amdgcn_sched_barrier(0);
        }
        exp_one<1>(16);
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            pv<1>(m);
            add_one<1>(m);
            if (m & 1) vf[m >> 1] = src[(2 * kKS + (m >> 1)) * 64];
            if (MASKED && m == 4) mask<0>(left);
            if (m >= 4 && m - 4 < kCheckParts) check_part<0>(m - 4);
            if (m & 2) between(2 * (m >> 3) + (m >> 2) % 2, m & 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        move_reference<0>();
        if (MASKED && left < kGrp) {  // stale cache bytes past the end may hold anything: zero those V columns
            const int q = lane >> 4, tbase = 16 * (q >> 1) + 8 * (q & 1);
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (tbase + e >= left) vf[dt][e] = (__bf16)0.f;
        }
        exponent<0>(0);
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            score<1>(m);
            exp_one<0>(m);
            __builtin_amdgcn_sched_barrier(0);
        }
        exp_one<0>(16);
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            if (LAST && m == 8) before_next();
            pv<0>(m);
            add_one<0>(m);
            if (MASKED && m == 4) mask<1>(left);
            if (m >= 4 && m - 4 < kCheckParts) check_part<1>(m - 4);
            if (LAST ? m >= 8 : m < 8) kf[k_order(m & 7)] = next[k_order(m & 7) * 64];
            if (m >= 8) between(4 + (m - 8) / 2, m & 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        move_reference<1>();
    }
    __device__ __forceinline__ void read_k(const bf16x8 *__restrict__ src) {
#pragma unroll
        for (int i = 0; i < 2 * kKS; ++i) kf[k_order(i)] = src[k_order(i) * 64];
    }
    // K fragment i in the order in which step 1 needs them
    static constexpr int k_order(int i) { return i & 1 ? kKS + (i >> 1) : i >> 1; }
    template <int P>
    __device__ __forceinline__ void finish_pair() {
        exponent<P>(0);
#pragma unroll
        for (int i = 0; i <= 16; ++i) exp_one<P>(i);
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            pv<P>(m);
            add_one<P>(m);
        }
    }
};

// Causal attention of a prefill chunk.  A workgroup owns one kv-head of one group of T consecutive
// chunk tokens (T * g <= 256 stacked queries; token t attends to kv_len - (T-1-t) positions) and
// walks the sequence's cache, or one piece of it, once for all of them; wave w holds query tiles
// [4 w, 4 w + 4).  Bound by what a CU issues, so what counts is that every CU has a walk: with
// whole walks only, 14 groups x 8 kv-heads of a round of agent turns (60-400 rows over 600-8192 cached
// tokens each) take 211 us on 112 CUs, cut into pieces 119 us with the merge; 512 rows over 32000 tokens
// (16 groups) 827 us and 483 us.
__global__ void __launch_bounds__(64 * kPrefillWaves) k_attn_prefill(const bf16_t *__restrict__ qg, const bf16_t *__restrict__ pool,
                                                                     const int32_t *__restrict__ bt, int max_blocks, AttnPlan pl,
                                                                     bf16_t *__restrict__ out, float *__restrict__ part_o,
                                                                     float *__restrict__ part_ml, int Hq, int Hkv, float scale_log2) {
    constexpr int NT = kPrefillNT;
    extern __shared__ float lds[];
    const int item = blockIdx.x / Hkv, c = blockIdx.x % Hkv;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int s = pl.item_seq[item];
    const bool parts = pl.item_begin != nullptr;  // else every piece is a whole walk
    const int begin = parts ? pl.item_begin[item] : 0, left = pl.seq_kvlen[s] - begin, n_tok = parts ? pl.item_len[item] : left;
    const int row0 = pl.seq_row0[s], T = pl.seq_rows[s];
    const int g = Hq / Hkv, G = T * g;
    const int m = lane & 15, q = lane >> 4;
    const int32_t *btr = bt + (size_t)pl.seq_bt[s] * max_blocks + begin / kBk;
    // LDS: [KV ring, two stages of 64 KB] [block ids]; the wave's Q fragments (B operands) stay in registers
    bf16x8 *ring = (bf16x8 *)lds;
    const uint32_t ring0 = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)lds;
    int *blds = (int *)(ring + 2 * kRoundGroups * 16 * 64);
    const int n_blk = (n_tok + kBk - 1) / kBk;
    for (int i = threadIdx.x; i < n_blk; i += 64 * kPrefillWaves) blds[i] = btr[i];
    bf16x8 qr[NT][kKS];
    State<NT> st;
    int stag[NT];
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        const int j = 16 * (w * NT + qt) + m;
        const bf16_t *qp = qg + ((size_t)(row0 + j / g) * Hq + c * g + j % g) * kD;
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) qr[qt][ks] = j < G ? *(const bf16x8 *)(qp + 32 * ks + 8 * q) : zero8();
        st.m[qt] = -INFINITY;
        st.l[qt] = 0.f;
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) st.o[dt][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
        stag[qt] = T - 1 - min(j / g, T - 1);
    }
    // every load so far has landed: the walk's waits then count its own prefetch loads only (left to its own
    // bookkeeping the compiler waits for the Q fragments inside the loop, and with them for the prefetch)
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __syncthreads();

    // This wave's quarter of every group: w = 0, 1 the K rows of tile w, w = 2, 3 the V^T rows of four d tiles; four fragments.
    const bool kside = w < 2;
    const int sel = kside ? m >> 3 : q >> 1;  // which of the group's two blocks this lane reads
    const int at = kside ? (8 * ((m >> 2) & 1) + (m & 3) + 4 * w) * kD + 8 * q : kBk * kD + (64 * (w - 2) + m) * kBk + 8 * (q & 1);
    constexpr size_t head_stride = (size_t)2 * kBk * kD;
    auto id_of = [&](int grp) { return blds[min(2 * grp + sel, n_blk - 1)]; };
    // The fragments go straight to LDS: those of round r + 1 are requested in the first two groups of round r.
    int ids[kRoundGroups];
    auto request = [&](auto GI, int i, int stage) {  // part i of 4
        constexpr int gi = decltype(GI)::value;
        dma16(pool + ((size_t)ids[gi] * Hkv + c) * head_stride + at + i * (kside ? 32 : 16 * kBk),
              ring0 + (uint32_t)((stage * kRoundGroups + gi) * 16 + 4 * w + i) * 1024);
    };
    constexpr Int<0> I0; constexpr Int<1> I1; constexpr Int<2> I2; constexpr Int<3> I3;
    auto each = [&](auto &&f) { f(I0); f(I1); f(I2); f(I3); };
    auto read_ids = [&](int r) {
#pragma unroll
        for (int gi = 0; gi < kRoundGroups; ++gi) ids[gi] = id_of(kRoundGroups * r + gi);
    };
    auto meet = [&] {  // what this wave brought has landed in LDS, and so has what the others brought
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
        __syncthreads();
    };

    const int n_grp = (n_tok + kGrp - 1) / kGrp;                          // groups, the masked ones included
    const int n_round = (n_grp + kRoundGroups - 1) / kRoundGroups;        // the same for every wave
    const int n_clean = min(n_grp, max(0, left - (T - 1)) / kGrp);         // groups valid for every query (further ones may be in later pieces)
    const bool busy = 16 * w * NT < G;                                    // a wave without queries only helps to load
    PrefillWalk walk(st, qr, stag, scale_log2, lane);
    read_ids(0);
    each([&](auto GI) {
        if (GI.value >= n_grp) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) request(GI, i, 0);
    });
    read_ids(1);
    meet();
    if (busy && n_clean > 0) walk.read_k(ring + lane);
#pragma nounroll
    for (int r = 0; r < n_round; ++r) {
        const int here = r & 1;
        const bf16x8 *stage = ring + (size_t)here * kRoundGroups * 16 * 64 + lane;
        const bf16x8 *other = ring + (size_t)(here ^ 1) * kRoundGroups * 16 * 64 + lane;
        const int n_here = min(kRoundGroups, n_grp - kRoundGroups * r), n_plain = busy ? max(0, min(n_here, n_clean - kRoundGroups * r)) : 0;
        bool met = false;  // the barrier of this round is behind us
        each([&](auto GI) {
            constexpr int gi = decltype(GI)::value;
            auto between = [&](int i, int sub) {  // parts 0-3 beside step 2, 4-7 beside step 4
                if (sub) return;
                if constexpr (gi < 2) {
                    if (i < 4) request(Int<2 * gi>(), i, here ^ 1);
                    else request(Int<2 * gi + 1>(), i - 4, here ^ 1);
                } else if (gi == 2 && i == 3) {
                    read_ids(r + 2);
                }
            };
            if (gi < n_plain) {
                walk.template group<gi + 1 == kRoundGroups, false>(stage + gi * 16 * 64, gi + 1 < kRoundGroups ? stage + (gi + 1) * 16 * 64 : other, 0,
                                                                   between, meet);
                if (gi + 1 == kRoundGroups) met = true;
            } else {
                if (r + 1 < n_round) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) between(i, 0);
                }
            }
        });
        if (busy) {
            if (n_plain > 0 && kRoundGroups * r + n_plain == n_clean) walk.finish_pair<1>();  // no group of this loop follows that would
            if (n_plain < n_here) {  // the masked groups, which bring nothing
                walk.read_k(stage + n_plain * 16 * 64);
                walk.none_pending();
#pragma nounroll
                for (int gi = n_plain; gi < n_here; ++gi)
                    walk.group<false, true>(stage + gi * 16 * 64, stage + min(gi + 1, kRoundGroups - 1) * 16 * 64, left - (kRoundGroups * r + gi) * kGrp,
                                            [](int, int) {}, [] {});
                walk.finish_pair<1>();
                walk.none_pending();
            }
        }
        if (!met) meet();
    }
    finish<NT>(st, w * NT, NT, G, g, row0, c, Hq, Hkv, parts ? pl.item_direct[item] : 1, parts ? pl.item_part[item] : 0, pl.g_max, out, part_o,
               part_ml, lane);
}

// The same attention in eight waves of two query tiles, one phase after the other, two waves a SIMD: the kernel for the
// FP8 cache, whose codes pass through registers that k_attn_prefill does not have, and see attn_prefill_pipelined.
constexpr int kShortWaves = 8, kShortNT = 2;
static_assert(kShortWaves * kShortNT == kPrefillWaves * kPrefillNT, "the plan's groups fit both");

// compute_group for a group that sits in LDS as fragments (src[i * 64]: K fragments i = 0..7, then
// V^T fragments) with the wave's Q fragments in registers (qr[qt][ks]).  A wave issues in order and a
// fragment read takes a few hundred cycles to come back, so the reads are batched ahead of the MFMAs
// that need them instead of sitting between them: the eight K fragments at the top, the eight V^T
// fragments as soon as the S^T MFMAs are issued (into the registers the K fragments leave), so that
// they travel while the softmax arithmetic runs and the P V MFMAs follow each other without a wait.
template <int NT, bool tail>
__device__ __forceinline__ void compute_group_lds(State<NT> &st, const bf16x8 *__restrict__ src, const bf16x8 (&qr)[NT][kKS],
                                                  int left, const int (&stag)[NT], float scale_log2, int lane) {
    const int q = lane >> 4;
    const int tbase = 16 * (q >> 1) + 8 * (q & 1);
    float sv[NT][8];
    __builtin_amdgcn_s_setprio(1);  // matrix-core sections run at raised priority, see prefill_walk_short
    {
        f32x4 s0[NT], s1[NT];
#pragma unroll
        for (int qt = 0; qt < NT; ++qt) { s0[qt] = f32x4{0.f, 0.f, 0.f, 0.f}; s1[qt] = f32x4{0.f, 0.f, 0.f, 0.f}; }
        bf16x8 kf[2 * kKS];
#pragma unroll
        for (int i = 0; i < 2 * kKS; ++i) kf[i] = src[i * 64];
        __builtin_amdgcn_sched_barrier(0);  // all reads first
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {
#pragma unroll
            for (int qt = 0; qt < NT; ++qt) {
                s0[qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], qr[qt][ks], s0[qt], 0, 0, 0);
                s1[qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kKS + ks], qr[qt][ks], s1[qt], 0, 0, 0);
            }
        }
#pragma unroll
        for (int qt = 0; qt < NT; ++qt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {  // raw scores, see compute_group
                sv[qt][i] = s0[qt][i];
                sv[qt][4 + i] = s1[qt][i];
            }
    }
    __builtin_amdgcn_s_setprio(0);
    bf16x8 vf[kDT];
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt) vf[dt] = src[(2 * kKS + dt) * 64];
    __builtin_amdgcn_sched_barrier(0);  // the reads stay ahead of the arithmetic
    bf16x8 pb[NT];
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        if (tail) {
            const int lim = left - stag[qt];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (tbase + e >= lim) sv[qt][e] = -INFINITY;
        }
        float mx = sv[qt][0];
#pragma unroll
        for (int e = 1; e < 8; ++e) mx = fmaxf(mx, sv[qt][e]);
        mx *= scale_log2;
        if (__any(mx > st.m[qt] + kSlack)) {  // see compute_group: lazy softmax reference
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float m_old = st.m[qt];
            const float m_new = fmaxf(m_old, mx);
            st.m[qt] = m_new;
            float alpha = (tail && m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(m_old - m_new);
            st.l[qt] *= alpha;
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) {
                st.o[dt][qt][0] *= alpha; st.o[dt][qt][1] *= alpha; st.o[dt][qt][2] *= alpha; st.o[dt][qt][3] *= alpha;
            }
        }
        const float m_ref = st.m[qt];
        float rs = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[qt][e], scale_log2, -m_ref));
            if (tail && m_ref == -INFINITY) p = 0.f;
            rs += p;
            pb[qt][e] = (__bf16)p;
        }
        st.l[qt] += rs;
    }
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt) {
        if (tail) {  // stale cache bytes past the end may hold anything: zero those V columns
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (tbase + e >= left) vf[dt][e] = (__bf16)0.f;
        }
#pragma unroll
        for (int qt = 0; qt < NT; ++qt) st.o[dt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], pb[qt], st.o[dt][qt], 0, 0, 0);
    }
    __builtin_amdgcn_s_setprio(0);
}

// Half of a group's loads: part 0 = the 8 K fragments, part 1 = the 8 V^T fragments, in the order
// they take in a KVFrag (k[t][ks] as 4t + ks, then v[dt]).
__device__ __forceinline__ void load_half(bf16x8 (&h)[8], int part, const bf16_t *__restrict__ pool, int blk0, int blk1, int c,
                                          int Hkv, int lane) {
    const int m = lane & 15, q = lane >> 4;
    const size_t head_stride = (size_t)2 * kBk * kD;
    if (part == 0) {
        const bf16_t *kb = pool + ((size_t)((m >> 3) ? blk1 : blk0) * Hkv + c) * head_stride;
        const int tok0 = 8 * ((m >> 2) & 1) + (m & 3);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) h[t * kKS + ks] = *(const bf16x8 *)(kb + (size_t)(tok0 + 4 * t) * kD + 32 * ks + 8 * q);
    } else {
        const bf16_t *vb = pool + ((size_t)((q >> 1) ? blk1 : blk0) * Hkv + c) * head_stride + (size_t)kBk * kD;
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) h[dt] = *(const bf16x8 *)(vb + (size_t)(16 * dt + m) * kBk + 8 * (q & 1));
    }
}
static_assert(2 * kKS == 8 && kDT == 8, "a half group is 8 fragments");

// The same half group from an FP8 cache: raw codes, r[i] = the 8 codes that become fragment i
// (K: i = 4 t + k-step, in the k-step order of KVRaw8; V^T: i = d tile).
__device__ __forceinline__ void load_half8(uint2 (&r)[8], int part, const uint8_t *__restrict__ pool, int blk0, int blk1, int c,
                                           int Hkv, int lane) {
    const int m = lane & 15, q = lane >> 4;
    const size_t head_stride = (size_t)2 * kBk * kD;
    if (part == 0) {
        const uint8_t *kb = pool + ((size_t)((m >> 3) ? blk1 : blk0) * Hkv + c) * head_stride;
        const int tok0 = 8 * ((m >> 2) & 1) + (m & 3);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int sl = 0; sl < 2; ++sl) {
                const uint4 v = *(const uint4 *)(kb + (size_t)(tok0 + 4 * t) * kD + 64 * sl + 16 * q);
                r[4 * t + 2 * sl] = uint2{v.x, v.y};
                r[4 * t + 2 * sl + 1] = uint2{v.z, v.w};
            }
    } else {
        const uint8_t *vb = pool + ((size_t)((q >> 1) ? blk1 : blk0) * Hkv + c) * head_stride + (size_t)kBk * kD;
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) r[dt] = *(const uint2 *)(vb + (size_t)(16 * dt + m) * kBk + 8 * (q & 1));
    }
}

// Short prefill walk: the eight waves hold different query tiles and every wave needs every group, so a
// group is loaded once -- in round r wave w loads half (w & 1: K or V^T) of group 4r + w/2 into
// registers, one round ahead -- published to an LDS ring as MFMA fragments in lane order, and read
// from there by all eight.  The ring has two stages of one round each: a wave publishes round r into
// stage r % 2, whose last readers (round r - 2) all passed the barrier of round r - 1, so one barrier
// per round is enough and the waves may drift up to a round apart (the matrix-core work of one then
// overlaps the softmax arithmetic of the other on the same SIMD).  ring: [2][4][16][64] x 16 B.
template <int NT, bool KV8>
__device__ __forceinline__ void prefill_walk_short(State<NT> &st, const void *__restrict__ pool_v, const int *__restrict__ blds,
                                             int n_blk, int n_tok, int left, int n_clean, const int (&stag)[NT], bool busy, int w, int c,
                                             int Hkv, bf16x8 *__restrict__ ring, const bf16x8 (&qr)[NT][kKS], float scale_log2, int lane) {
    // left: tokens of the sequence from this piece's first on (n_tok or more); busy: this wave holds queries
    const int n_grp = (n_tok + kGrp - 1) / kGrp;  // groups, the masked ones included
    const int n_round = (n_grp + 3) / 4;          // the same for every wave
    const int part = w & 1, gl = w >> 1;
    auto blk_of = [&](int grp, int which) {
        return __builtin_amdgcn_readfirstlane(blds[min(grp * 2 + which, n_blk - 1)]);
    };
    bf16x8 h[8];
    uint2 h8[8];
    auto load = [&](int grp) {
        if constexpr (KV8) load_half8(h8, part, (const uint8_t *)pool_v, blk_of(grp, 0), blk_of(grp, 1), c, Hkv, lane);
        else load_half(h, part, (const bf16_t *)pool_v, blk_of(grp, 0), blk_of(grp, 1), c, Hkv, lane);
    };
    if (gl < n_grp) load(gl);
#pragma nounroll
    for (int r = 0; r < n_round; ++r) {
        bf16x8 *stage = ring + (size_t)(r & 1) * 4 * 16 * 64;
        const int mine = 4 * r + gl;
        if (mine < n_grp) {
            bf16x8 *dst = stage + ((size_t)gl * 16 + part * 8) * 64 + lane;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if constexpr (KV8) dst[i * 64] = cvt8(h8[i].x, h8[i].y);  // codes are exact in bf16
                else dst[i * 64] = h[i];
            }
        }
        if (mine + 4 < n_grp) load(mine + 4);
        __syncthreads();
        if (!busy) continue;  // a wave of a partly filled group only helps to load
        // the round's unmasked groups, then its masked ones: two loops of one code path each (with both paths
        // in one loop body the accumulators are copied between the registers the two paths leave them in)
        const int n_here = min(4, n_grp - 4 * r), n_plain = max(0, min(n_here, n_clean - 4 * r));
#pragma nounroll
        for (int gi = 0; gi < n_plain; ++gi)
            compute_group_lds<NT, false>(st, stage + (size_t)gi * 16 * 64 + lane, qr, kGrp, stag, scale_log2, lane);
#pragma nounroll
        for (int gi = n_plain; gi < n_here; ++gi)
            compute_group_lds<NT, true>(st, stage + (size_t)gi * 16 * 64 + lane, qr, left - (4 * r + gi) * kGrp, stag, scale_log2, lane);
    }
}

template <bool KV8>
__global__ void __launch_bounds__(64 * kShortWaves) k_attn_prefill_short(const bf16_t *__restrict__ qg, const void *__restrict__ pool,
                                                                     const int32_t *__restrict__ bt, int max_blocks, AttnPlan pl,
                                                                     bf16_t *__restrict__ out, float *__restrict__ part_o,
                                                                     float *__restrict__ part_ml, int Hq, int Hkv, float scale_log2, float v_scale) {
    constexpr int NT = kShortNT;
    extern __shared__ float lds[];
    const int item = blockIdx.x / Hkv, c = blockIdx.x % Hkv;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int s = pl.item_seq[item];
    const bool parts = pl.item_begin != nullptr;  // else every piece is a whole walk
    const int begin = parts ? pl.item_begin[item] : 0, left = pl.seq_kvlen[s] - begin, n_tok = parts ? pl.item_len[item] : left;
    const int row0 = pl.seq_row0[s], T = pl.seq_rows[s];
    const int g = Hq / Hkv, G = T * g;
    const int m = lane & 15, q = lane >> 4;
    const int32_t *btr = bt + (size_t)pl.seq_bt[s] * max_blocks + begin / kBk;
    // LDS: [KV ring, two stages of 64 KB] [block ids]; the wave's Q fragments (B operands) stay in registers
    bf16x8 *ring = (bf16x8 *)lds;
    bf16x8 qr[NT][kKS];
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        int j = 16 * (w * NT + qt) + m;
        const bf16_t *qp = qg + ((size_t)(row0 + j / g) * Hq + c * g + j % g) * kD;
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {  // FP8 cache: the k-step order of KVRaw8
            const int d0 = KV8 ? 64 * (ks >> 1) + 16 * q + 8 * (ks & 1) : 32 * ks + 8 * q;
            qr[qt][ks] = j < G ? *(const bf16x8 *)(qp + d0) : zero8();
        }
    }
    int *blds = (int *)(ring + 2 * 4 * 16 * 64);
    const int n_blk = (n_tok + kBk - 1) / kBk;
    for (int i = threadIdx.x; i < n_blk; i += 64 * kShortWaves) blds[i] = btr[i];
    // every load so far has landed: the walk's waits then count its own prefetch loads only (left to its own
    // bookkeeping the compiler waits for the Q fragments inside the loop, and with them for the prefetch)
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __syncthreads();

    State<NT> st;
    int stag[NT];
#pragma unroll
    for (int qt = 0; qt < NT; ++qt) {
        st.m[qt] = -INFINITY;
        st.l[qt] = 0.f;
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) st.o[dt][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
        stag[qt] = T - 1 - min((16 * (w * NT + qt) + m) / g, T - 1);
    }
    const int n_clean = max(0, left - (T - 1)) / kGrp;  // groups valid for every query (further ones may be in later pieces)
    const bool busy = __builtin_amdgcn_readfirstlane(16 * w * NT) < G;
    prefill_walk_short<NT, KV8>(st, pool, blds, n_blk, n_tok, left, n_clean, stag, busy, w, c, Hkv, ring, qr, scale_log2, lane);
    if constexpr (KV8) {
#pragma unroll
        for (int qt = 0; qt < NT; ++qt)
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt) {
                st.o[dt][qt][0] *= v_scale; st.o[dt][qt][1] *= v_scale; st.o[dt][qt][2] *= v_scale; st.o[dt][qt][3] *= v_scale;
            }
    }
    finish<NT>(st, w * NT, NT, G, g, row0, c, Hq, Hkv, parts ? pl.item_direct[item] : 1, parts ? pl.item_part[item] : 0, pl.g_max, out, part_o,
               part_ml, lane);
}

// Combine the partial results of sequences that were split into several pieces.  32 threads per (row, query head),
// four output elements each; four pieces' loads in flight (a piece past the last repeats it with weight zero).
// row_pseq: plan sequence of each of the R rows; null: a grid row per plan sequence, R rows of it at most.
__global__ void __launch_bounds__(256) k_attn_merge(const float *__restrict__ part_o, const float *__restrict__ part_ml,
                                                    AttnPlan pl, const int32_t *__restrict__ row_pseq,
                                                    bf16_t *__restrict__ out, int R, int Hq, int Hkv) {
    const int idx = blockIdx.x * 8 + (threadIdx.x >> 5), d = (threadIdx.x & 31) * 4;
    if (idx >= (row_pseq ? R : pl.seq_rows[blockIdx.y]) * Hq) return;
    const int h = idx % Hq, row = idx / Hq + (row_pseq ? 0 : pl.seq_row0[blockIdx.y]);
    const int s = row_pseq ? row_pseq[row] : blockIdx.y;
    const int g = Hq / Hkv, c = h / g;
    const int np = pl.seq_nparts[s];
    if (np <= 1) return;  // written directly by the attention kernel
    const size_t pj0 = ((size_t)pl.seq_part0[s] * Hkv + c) * pl.g_max + (row - pl.seq_row0[s]) * g + h % g;
    const size_t pstep = (size_t)Hkv * pl.g_max;  // between consecutive pieces
    float M = -INFINITY;
    for (int p = 0; p < np; p += 4) {
        float m4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) m4[u] = part_ml[(pj0 + min(p + u, np - 1) * pstep) * 2];
#pragma unroll
        for (int u = 0; u < 4; ++u) M = fmaxf(M, m4[u]);
    }
    float num[4] = {0.f, 0.f, 0.f, 0.f}, den = 0.f;
    for (int p = 0; p < np; p += 4) {
        float2 ml[4];
        f32x4 o[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t pj = pj0 + min(p + u, np - 1) * pstep;
            ml[u] = *(const float2 *)(part_ml + pj * 2);
            o[u] = *(const f32x4 *)(part_o + pj * kD + d);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // in piece order
            const float wgt = p + u < np ? __builtin_amdgcn_exp2f(ml[u].x - M) : 0.f;
            den += wgt * ml[u].y;
#pragma unroll
            for (int i = 0; i < 4; ++i) num[i] += wgt * o[u][i];
        }
    }
    uint2 pk;
    pk.x = pack_bf16(num[0] / den, num[1] / den);
    pk.y = pack_bf16(num[2] / den, num[3] / den);
    *(uint2 *)(out + ((size_t)row * Hq + h) * kD + d) = pk;
}

template <int NA, int NB, bool KV8 = false>
hipError_t launch_one(const void *q, const void *pool, const int32_t *bt, int max_blocks, const AttnPlan &pl, void *out,
                      float *part_o, float *part_ml, int Hq, int Hkv, float scale_log2, float v_scale, hipStream_t st) {
    // block ids of pieces of up to kAttnMaxChunk tokens
    constexpr int kIds = (kAttnMaxChunk / kBk) * 4;
    constexpr size_t shm = NB ? kRingBytes + (size_t)(NA + NB) * kKS * 1024 + kIds : 4 * (size_t)Image<NA>::kBytes + 2 * ((size_t)NA * kKS * 1024 + kIds);
    const auto kernel = [] {
        if constexpr (NB > 0) return k_attn_decode_pairs<NA, NB, KV8>;
        else return k_attn_decode<NA, KV8>;
    }();
    static bool attr_set = false;  // per instantiation
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(kernel, dim3(pl.n_wgs * Hkv), dim3(256), shm, st, (const bf16_t *)q, pool, bt, max_blocks, pl,
                       (bf16_t *)out, part_o, part_ml, Hq, Hkv, scale_log2, v_scale);
    return hipGetLastError();
}

}  // namespace

bool attn_decode_mfma_supported(const Dims &dm, int g_max) {
    return dm.bf16 && dm.D == kD && dm.Bk == kBk && g_max >= 1 && g_max <= 80;
}

// Tokens one prefill workgroup can walk: its block ids take what the KV ring leaves of the CU's 160 KB of LDS.  (The
// ring already limits a CU to one workgroup, so the ids cost no occupancy; bounded by the 16384 tokens of a decode
// piece, a 512-row chunk over a 32000-token prefix fell to the vector kernel and took 860 ms instead of 1.67 ms.)
constexpr size_t kPrefillRing = (size_t)2 * 4 * 16 * 64 * 16, kLdsBytes = (size_t)160 << 10;
constexpr int kPrefillMaxCtx = (int)((kLdsBytes - kPrefillRing) / 4) * kBk;
int attn_prefill_max_ctx() { return kPrefillMaxCtx; }
int attn_prefill_round() { return kRoundGroups * kGrp; }

int attn_prefill_group_queries() { return kPrefillWaves * kPrefillNT * 16; }  // stacked queries one prefill workgroup holds

// In pieces of up to some length a wave's first and last groups, which nothing hides, count for more than what the pipeline of
// k_attn_prefill hides of the others; and a token group that is not full leaves whole waves of it idle, of four tiles each, where
// eight waves are idle in twos.  Eight waves / four, us, whole walks and cut ones, by the longest piece: groups full to 97 % and more, 1088
// tokens 49.8 / 51.0, 1408 63.0 / 61.9, 1792 78.2 / 75.7, 2750 101 / 96, 8250 277 / 252, 14064 486 / 441; less full (400 rows in groups
// of 64 or 32), 1400 51.0 / 53.7, 2900 90.3 / 93.0, 3900 115.8 / 116.6, 5400 168 / 164, 14400 415 / 402.
bool attn_prefill_pipelined(int longest, int64_t queries, int64_t groups) {
    return longest > (100 * queries >= 97 * groups * attn_prefill_group_queries() ? 1280 : 5120);
}

bool attn_prefill_mfma_supported(const Dims &dm, int g_max) {
    return dm.bf16 && dm.D == kD && dm.Bk == kBk && g_max >= 1 && g_max <= attn_prefill_group_queries();
}

hipError_t launch_attn_prefill_mfma(const Dims &dm, const void *q, const void *pool, const int32_t *bt, int max_blocks,
                                    const AttnPlan &pl, void *out, float *part_o, float *part_ml, hipStream_t st) {
    if (pl.n_items <= 0) return hipSuccess;
    if (!pl.causal || pl.chunk > kPrefillMaxCtx) return hipErrorInvalidValue;
    const size_t shm = kPrefillRing + (size_t)((pl.chunk + kBk - 1) / kBk) * 4;  // two ring stages + the block ids
    const dim3 grid(pl.n_items * dm.Hkv);
    const float scale_log2 = kLog2e / sqrtf((float)dm.D) * (dm.kv8 ? dm.k_scale : 1.f);
    auto allow_lds = [](auto kernel, bool &set) {
        if (set) return hipSuccess;
        const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
        set = e == hipSuccess;
        return e;
    };
    if (!dm.kv8 && pl.pipelined) {
        static bool set = false;
        const hipError_t e = allow_lds(k_attn_prefill, set);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_attn_prefill, grid, dim3(64 * kPrefillWaves), shm, st, (const bf16_t *)q, (const bf16_t *)pool, bt, max_blocks, pl,
                           (bf16_t *)out, part_o, part_ml, dm.Hq, dm.Hkv, scale_log2);
        return hipGetLastError();
    }
    auto launch = [&](auto kernel, bool &set) {
        const hipError_t e = allow_lds(kernel, set);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, grid, dim3(64 * kShortWaves), shm, st, (const bf16_t *)q, pool, bt, max_blocks, pl, (bf16_t *)out, part_o,
                           part_ml, dm.Hq, dm.Hkv, scale_log2, dm.kv8 ? dm.v_scale : 1.f);
        return hipGetLastError();
    };
    static bool set_bf16 = false, set_fp8 = false;
    return dm.kv8 ? launch(k_attn_prefill_short<true>, set_fp8) : launch(k_attn_prefill_short<false>, set_bf16);
}

hipError_t launch_attn_decode_mfma(const Dims &dm, const void *q, const void *pool, const int32_t *bt, int max_blocks,
                                   const AttnPlan &pl, void *out, float *part_o, float *part_ml, hipStream_t st) {
    if (pl.n_items <= 0) return hipSuccess;
    if (pl.causal || pl.chunk > kAttnMaxChunk || pl.n_wgs <= 0) return hipErrorInvalidValue;
    float scale_log2 = kLog2e / sqrtf((float)dm.D);
    int nqt = (pl.g_max + 15) / 16;
    if (dm.kv8) {  // FP8 codes: the K scale joins the softmax scale, the V scale the output
        scale_log2 *= dm.k_scale;
        switch (nqt) {
        case 1: return launch_one<1, 0, true>(q, pool, bt, max_blocks, pl, out, part_o, part_ml, dm.Hq, dm.Hkv, scale_log2, dm.v_scale, st);
        case 2: return launch_one<2, 0, true>(q, pool, bt, max_blocks, pl, out, part_o, part_ml, dm.Hq, dm.Hkv, scale_log2, dm.v_scale, st);
        case 3: return launch_one<3, 0, true>(q, pool, bt, max_blocks, pl, out, part_o, part_ml, dm.Hq, dm.Hkv, scale_log2, dm.v_scale, st);
        case 4: return launch_one<2, 2, true>(q, pool, bt, max_blocks, pl, out, part_o, part_ml, dm.Hq, dm.Hkv, scale_log2, dm.v_scale, st);
        case 5: return launch_one<3, 2, true>(q, pool, bt, max_blocks, pl, out, part_o, part_ml, dm.Hq, dm.Hkv, scale_log2, dm.v_scale, st);
        default: return hipErrorInvalidValue;
        }
    }
    switch (nqt) {
    case 1: return launch_one<1, 0>(q, pool, bt, max_blocks, pl, out, part_o, part_ml, dm.Hq, dm.Hkv, scale_log2, 1.f, st);
    case 2: return launch_one<2, 0>(q, pool, bt, max_blocks, pl, out, part_o, part_ml, dm.Hq, dm.Hkv, scale_log2, 1.f, st);
    case 3: return launch_one<3, 0>(q, pool, bt, max_blocks, pl, out, part_o, part_ml, dm.Hq, dm.Hkv, scale_log2, 1.f, st);
    case 4: return launch_one<2, 2>(q, pool, bt, max_blocks, pl, out, part_o, part_ml, dm.Hq, dm.Hkv, scale_log2, 1.f, st);
    case 5: return launch_one<3, 2>(q, pool, bt, max_blocks, pl, out, part_o, part_ml, dm.Hq, dm.Hkv, scale_log2, 1.f, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_attn_merge(const Dims &dm, const float *part_o, const float *part_ml, const AttnPlan &pl,
                             const int32_t *row_pseq, void *out, int R, int n_seq, hipStream_t st) {
    if (R <= 0 || n_seq <= 0) return hipSuccess;
    const dim3 grid((R * dm.Hq + 7) / 8, row_pseq ? 1 : n_seq);
    hipLaunchKernelGGL(k_attn_merge, grid, dim3(256), 0, st, part_o, part_ml, pl, row_pseq, (bf16_t *)out, R, dm.Hq, dm.Hkv);
    return hipGetLastError();
}

}  // namespace icarus
