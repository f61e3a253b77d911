// Chunk preparation: everything about a chunk that does not depend on the
// state entering it.  One workgroup (4 waves) per (chunk, head, sequence).
//
// For chunk rows r, s = 0..63 (rows past the chunk's end are zero-padded,
// which makes them inert: zero key, zero value, zero beta, zero gate):
//   G_r   = sum_{s<=r} g_s                      (chunk-local, fp32)
//   Gp_r  = G_{r-1} (literal rule; G_{-1} = 0) or G_r (decayed rule)
//   A     = strictly lower part of beta_r exp(Gp_r - G_s) (k_r . k_s)
//   X     = (I + A)^{-1}                       (unit lower triangular, fp32)
//   W     = X diag(beta exp(Gp)) K             (stored negated, A-operand order;
//                                               computed as W^T tiles, whose
//                                               accumulator layout is that order)
//   U~    = X diag(beta) V                     (fp32, C-layout)
//   K~^T  = (diag(exp(G_63 - G)) K)^T          (A-operand order, chunk rows permuted)
//   P     = (Q K^T) exp(G_r - G_s) on s <= r   (for the output; B operand of P^T
//                                               per token tile, chunk rows permuted)
//   Q     = the queries as the B operand of Q^T per token tile (dk permuted)
// so that, for the state S_0 entering the chunk, U = U~ - W S_0 holds the
// per-row corrections u_r = beta_r (v_r - pred_r) and the state leaving the
// chunk is exp(G_63) S_0 + K~^T U.  (Derivation: unroll the recurrence
// inside the chunk; the prediction of row r sees S_0 decayed by exp(Gp_r)
// plus the rank-one writes of earlier rows decayed by exp(Gp_r - G_s).)
//
// K is staged row-major only; operands that contract over chunk rows are read
// one element per lane.
// Exponentials of gate differences use exp2 on log2(e)-scaled cumulative
// gates; every exponent is a difference formed before exponentiation.
#pragma once
#include "la_common.h"

namespace la {

struct PrepArgs {
    const void *q, *k, *v;
    const float *g, *beta;
    const int32_t *cu;
    int32_t n_heads, C, cps, variant;
    Workspace ws;
    UnitMap map;           // the block's unit (see unit_of_block)
};

constexpr float kLog2e = 1.4426950408889634f;

// Cross-lane moves (DPP): CTRL selects the source lane, ROWS enables rows of
// 16 lanes; lanes without a source, and disabled rows, read 0.
template <int CTRL, int ROWS = 0xF>
__device__ inline float dpp_f(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROWS, 0xF, true));
}

// Inclusive prefix sum over the wave's 64 lanes: shifts within each row of
// 16 lanes, then each row's carry from the rows before it (row broadcasts).
__device__ inline float wave_inclusive_sum(float x) {
    x += dpp_f<0x111>(x);          // row_shr:1
    x += dpp_f<0x112>(x);          // row_shr:2
    x += dpp_f<0x114>(x);          // row_shr:4
    x += dpp_f<0x118>(x);          // row_shr:8
    x += dpp_f<0x142, 0xA>(x);     // row_bcast:15 into rows 1 and 3
    x += dpp_f<0x143, 0xC>(x);     // row_bcast:31 into rows 2 and 3
    return x;
}

// One column-oriented step of the diagonal-block substitution: lane s of
// each row holds the final x[s] of its columns; broadcast it along the row
// (row_newbcast:s) and subtract L[r][s] x[s] (L is zero at and above the
// diagonal, so rows r <= s are left unchanged).
template <int S>
__device__ inline void subst_step(float (&x)[4], const float (&L)[16]) {
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] -= L[S] * dpp_f<0x150 + S>(x[c]);
}

template <int S = 0>
__device__ inline void subst_all(float (&x)[4], const float (&L)[16]) {
    if constexpr (S < 16) {
        subst_step<S>(x, L);
        subst_all<S + 1>(x, L);
    }
}

// NMT: 16-row tiles of a chunk that can hold tokens (chunks have at most
// min(C, 64) rows; the rows past them are inert and are left out).
template <int DK, int NMT> struct alignas(16) PrepSmem {
    static constexpr int R = 16 * NMT;
    float ks[R][DK + 4];                       // K, row-major (the pad keeps 16-byte alignment)
    float am[R][kChunk + 4];                   // A (strictly lower)
    float xm[R][kChunk + 4];                   // X = (I + A)^{-1}
    float ysc[4][16][17];                      // per-wave 16x16 scratch
    float G2[kChunk], Gp2[kChunk], bs[kChunk]; // log2e-scaled gates, beta
    float dW[kChunk], dK[kChunk];              // beta exp(Gp), exp(G_63 - G)
};

// 16x16x16 fp32 product of two LDS blocks with fp32 MFMA, accumulated in c.
__device__ inline f32x4 mm16_f32(const float *A, int lda, const float *B, int ldb, f32x4 c,
                                 int lane) {
    const int r = lane & 15, g = lane >> 4;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(A[r * lda + 4 * ks + g], B[(4 * ks + g) * ldb + r],
                                                 c, 0, 0, 0);
    return c;
}

// Transposed reads of a row-major LDS tile.
template <typename T> struct RowTile;

template <> struct RowTile<__bf16> {
    typedef short i16x4 __attribute__((ext_vector_type(4)));
    // LDS transpose read: in each 16-lane group, source lane s reads 4
    // elements of row `row(s)` at column n0 + 4 (s % 4); with row(s) chosen
    // as base + s / 4, lane i of the group receives column n0 + i of rows
    // base .. base + 3.
    __device__ static inline i16x4 tr4(const __bf16 *tile, int ld, int row, int n0, int lane) {
        const int s = lane & 15;
        const __bf16 *p = tile + row * ld + n0 + 4 * (s & 3);
        return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)p);
    }
};

// fp32 MFMA issues one 16x16x4 product per 32 cycles, so what bounds a unit is
// its count of products and the LDS reads that feed them.  Wave w computes row
// tile w of A and row tile NMT - 1 - w of P (16-byte reads of K's rows, in the
// order the state's accumulators contract dk) and, of W^T, U~ and K~^T, the column
// tiles w, w + 4, ... of every row tile: X's fragments are then read once, V
// goes from memory straight to the lanes that use it, and the products over X's
// zero triangle are left out.  Without V the LDS holds two workgroups per CU
// (74 KB at dk = 128).  Three prompts of 1,791, 640 and 257 tokens (8 heads,
// dk = dv = 128): 24.7 us against 36.9 with V staged and a row tile per wave
// throughout; 256 tokens with C = 16 (1 head, dk = dv = 64): 3.8 against 11.6 us.
template <int DK, int DV, int NMT> __global__ __launch_bounds__(256, 2) void gdr_prep_kernel(PrepArgs a) {
    typedef float T;
    using M = MT<T>;
    using Sm = PrepSmem<DK, NMT>;
    constexpr int VEC = 4, R = Sm::R, LDA = kChunk + 4;
    constexpr int NW = DK / 64, NV = DV / 64;   // column tiles of W^T (K~^T) and of U~ per wave
    __shared__ Sm sm;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g16 = lane >> 4, c16 = lane & 15;
    int64_t j;
    int seq, h;
    if (!unit_of_block(a.map, a.cu, &seq, &h, &j)) return;
    const int H = a.n_heads;
    const int64_t cu0 = a.cu[seq];
    const int len = a.cu[seq + 1] - a.cu[seq];
    if (j >= n_chunks32(len, a.C, a.cps)) return;
    int lo, hi;
    chunk_range32((int)j, len, a.C, a.cps, &lo, &hi);
    const int n = hi - lo;
    const int64_t t0 = cu0 + lo;
    const int64_t sh = (slot_base_dev(cu0, seq, a.C, a.cps) + j) * H + h;   // slot-head index

    const T *kin = (const T *)a.k;
    const T *vin = (const T *)a.v;

    // ---- 1. every global load first; rows past the chunk's end read the last
    // valid row and are zeroed afterwards.
    // This lane's queries: token row 16 mp + lane % 16 at dk perm_row(f, g)
    // for f < DK/4 (g = lane / 16), runs of 4.  That is exactly this lane's
    // part of the B operand of Q^T for token tile mp in the order the
    // state's accumulator layout contracts dk, so it is stored as is for the
    // output, and the P product below contracts dk in the same order.
    const int mp = NMT - 1 - wave;              // this wave's row tile of P
    T qf[DK / 4];
    if (mp >= 0) {
        const int r = 16 * mp + c16, rr = r < n ? r : n - 1;
        const T *qrow = (const T *)a.q + ((t0 + rr) * H + h) * DK + 4 * g16;
#pragma unroll
        for (int p4 = 0; p4 < DK / 16; ++p4) *(uint4 *)&qf[4 * p4] = *(const uint4 *)(qrow + 16 * p4);
    }
    // V as the B operand of U~: rows 4 ks + g, one column per lane
    T vb[NV][4 * NMT];
    {
        constexpr int KIT = R * DK / VEC / 256;
        static_assert(KIT * 256 * VEC == R * DK, "tiling");
        uint4 kr[KIT];
#pragma unroll
        for (int it = 0; it < KIT; ++it) {
            const int vi = tid + 256 * it, r = vi / (DK / VEC), c = (vi % (DK / VEC)) * VEC;
            const int rr = r < n ? r : n - 1;
            kr[it] = *(const uint4 *)(kin + ((t0 + rr) * H + h) * DK + c);
        }
        float gv = 0.f, bv = 0.f;
        if (tid < kChunk) {
            const int rr = tid < n ? tid : n - 1;
            gv = a.g[(t0 + rr) * H + h];
            bv = a.beta[(t0 + rr) * H + h];
        }
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int ks = 0; ks < 4 * NMT; ++ks) {
                const int r = 4 * ks + g16, rr = r < n ? r : n - 1;
                vb[i][ks] = vin[((t0 + rr) * H + h) * DV + 16 * (wave + 4 * i) + c16];
            }
        for (int e = tid; e < R * LDA; e += 256) (&sm.xm[0][0])[e] = 0.f;
#pragma unroll
        for (int it = 0; it < KIT; ++it) {
            const int vi = tid + 256 * it, r = vi / (DK / VEC), c = (vi % (DK / VEC)) * VEC;
            if (r >= n) kr[it] = make_uint4(0, 0, 0, 0);
            *(uint4 *)&sm.ks[r][c] = kr[it];
        }
        // ---- 2. chunk-local gate prefix sum (wave 0) --------------------------
        if (wave == 0) {
            const float b = tid < n ? bv : 0.f;
            const float x = wave_inclusive_sum(tid < n ? gv : 0.f);
            const float prev = dpp_f<0x138>(x);   // wave_shr:1: lane - 1's sum, 0 on lane 0
            const float gp = (a.variant == 0) ? prev : x;
            const float g63 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
            sm.G2[lane] = x * kLog2e;
            sm.Gp2[lane] = gp * kLog2e;
            sm.bs[lane] = b;
            sm.dW[lane] = b * __builtin_amdgcn_exp2f(gp * kLog2e);
            sm.dK[lane] = __builtin_amdgcn_exp2f((g63 - x) * kLog2e);
            a.ws.g[sh * kChunk + 4 * (lane & 15) + (lane >> 4)] = x;   // G layout: row 16 m + c at 4 c + m
        }
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int ks = 0; ks < 4 * NMT; ++ks)
                if (4 * ks + g16 >= n) vb[i][ks] = 0.f;
    }
    __syncthreads();

    // ---- 3. A = strictly-lower beta_r exp(Gp_r - G_s) K K^T, row tile `wave`, and
    // P = (Q K^T) exp(G_r - G_s) on s <= r, row tile mp: a row tile has as many
    // tiles as its number + 1, so every wave computes NMT + 1 of them.  P is
    // computed as the tiles K Q^T: the result tile (s tile nt, token tile mp) holds
    // P[16 mp + c16][16 nt + 4 g + i] in lane (g, c16), which is element 4 nt + i of
    // that lane's P^T operand, so it is stored straight from the accumulator.
    // Tiles above the diagonal are neither written nor read.
    if (wave < NMT) {
        const int mt = wave;
        auto row = [&](int t, T (&f)[DK / 4]) {
#pragma unroll
            for (int p4 = 0; p4 < DK / 16; ++p4)
                *(uint4 *)&f[4 * p4] = *(const uint4 *)&sm.ks[16 * t + c16][16 * p4 + 4 * g16];
        };
        T kb[DK / 4];
        {
            T ka[DK / 4];
            row(mt, ka);
            const float4 brow = *(const float4 *)&sm.bs[16 * mt + 4 * g16];
            const float4 gprow = *(const float4 *)&sm.Gp2[16 * mt + 4 * g16];
            const float bv[4] = {brow.x, brow.y, brow.z, brow.w};
            const float gv[4] = {gprow.x, gprow.y, gprow.z, gprow.w};
            for (int nt = 0; nt <= mt; ++nt) {   // wave-uniform
                row(nt, kb);
                f32x4 acc = zero4();
#pragma unroll
                for (int f = 0; f < DK / 4; ++f) acc = M::mma(ka[f], kb[f], acc);
                const float gcol = sm.G2[16 * nt + c16];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = 16 * mt + 4 * g16 + i, s = 16 * nt + c16;
                    const float e = __builtin_amdgcn_exp2f(gv[i] - gcol);
                    sm.am[r][s] = (s < r) ? bv[i] * e * acc[i] : 0.f;
                }
            }
        }
        const float gr = sm.G2[16 * mp + c16];
        T *pout = (T *)a.ws.p + sh * WsLayout<T, DK, DV>::p_elems;
        for (int nt = 0; nt <= mp; ++nt) {
            row(nt, kb);
            f32x4 pc = zero4();
#pragma unroll
            for (int f = 0; f < DK / 4; ++f) pc = M::mma(kb[f], qf[f], pc);
            const float4 gs = *(const float4 *)&sm.G2[16 * nt + 4 * g16];
            const float gsv[4] = {gs.x, gs.y, gs.z, gs.w};
            T vals[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool in = 16 * nt + 4 * g16 + i <= 16 * mp + c16;
                vals[i] = in ? pc[i] * __builtin_amdgcn_exp2f(gr - gsv[i]) : 0.f;
            }
            *(uint4 *)(pout + ((size_t)(mp * 4 + nt) * 64 + lane) * VEC) = *(const uint4 *)vals;
        }
        constexpr int NQ = DK / 4 / VEC;
        T *qout = (T *)a.ws.qf + sh * WsLayout<T, DK, DV>::qf_elems;
#pragma unroll
        for (int v = 0; v < NQ; ++v)
            *(uint4 *)(qout + ((size_t)(mp * NQ + v) * 64 + lane) * VEC) = *(const uint4 *)&qf[v * VEC];
    }
    __syncthreads();

    // ---- 4. X = (I + A)^{-1}: diagonal 16-blocks by substitution ---------------
    // Wave w inverts block w with all 64 lanes: lane (q, r), q = lane / 16,
    // r = lane % 16, holds row r of columns 4q .. 4q + 3 of the block's
    // inverse.  Each x[r] receives the updates L[r][s] x[s] in the order
    // s = 0, 1, ..., as forward substitution does.
    if (wave < NMT) {
        const int base = 16 * wave, q = lane >> 4, r = lane & 15;
        float L[16];
#pragma unroll
        for (int s4 = 0; s4 < 16; s4 += 4) {
            const float4 v = *(const float4 *)&sm.am[base + r][base + s4];
            L[s4] = v.x;
            L[s4 + 1] = v.y;
            L[s4 + 2] = v.z;
            L[s4 + 3] = v.w;
        }
        float x[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = (r == 4 * q + c) ? 1.f : 0.f;
        subst_all(x, L);
        *(float4 *)&sm.xm[base + r][base + 4 * q] = make_float4(x[0], x[1], x[2], x[3]);
    }
    __syncthreads();
    // off-diagonal blocks by bands: X_ij = -X_ii sum_{k=j}^{i-1} A_ik X_kj
    for (int d = 1; d < NMT; ++d) {
        const int bi = d + wave, bj = wave;
        const bool active = bi < NMT;
        if (active) {
            f32x4 y = zero4();
            for (int bk = bj; bk < bi; ++bk)
                y = mm16_f32(&sm.am[16 * bi][16 * bk], LDA, &sm.xm[16 * bk][16 * bj], LDA, y, lane);
#pragma unroll
            for (int i = 0; i < 4; ++i) sm.ysc[wave][4 * g16 + i][c16] = y[i];
        }
        // ysc[wave] is written and read by this wave alone: its LDS accesses
        // execute in order, so only the compiler needs holding back here
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (active) {
            f32x4 xij = mm16_f32(&sm.xm[16 * bi][16 * bi], LDA, &sm.ysc[wave][0][0], 17, zero4(), lane);
#pragma unroll
            for (int i = 0; i < 4; ++i) sm.xm[16 * bi + 4 * g16 + i][16 * bj + c16] = -xij[i];
        }
        __syncthreads();
    }

    // ---- 5. W, U~ = X diag(beta) V and the K~^T fragments, column tiles wave,
    // wave + 4, ...: X's fragments of every row tile (k-steps up to its diagonal)
    {
        T x1[NMT][4 * NMT], x2[NMT][4 * NMT];   // X diag(beta exp(Gp)), X diag(beta)
#pragma unroll
        for (int ks = 0; ks < 4 * NMT; ++ks) {
            const int s = 4 * ks + g16;
            const float w1 = sm.dW[s], w2 = sm.bs[s];
#pragma unroll
            for (int mt = 0; mt < NMT; ++mt)
                if (ks < 4 * (mt + 1)) {
                    const float x = sm.xm[16 * mt + c16][s];
                    x1[mt][ks] = x * w1;
                    x2[mt][ks] = x * w2;
                }
        }
        // W^T tile (dk tile nt, row tile mt) = K^T (X diag(dW))^T: per lane the
        // element of K read as a B operand of K is the A operand of K^T, and x1
        // (A operand of X diag(dW)) is the B operand of its transpose.  The
        // accumulator then holds W[16 mt + c16][16 nt + 4 g + i], element
        // 4 nt + i of this lane's -W fragment in the scan's permuted dk
        // order, so -W is stored straight from registers.
        T *wout = (T *)a.ws.w + sh * WsLayout<T, DK, DV>::w_elems;
        T *kout = (T *)a.ws.kt + sh * WsLayout<T, DK, DV>::kt_elems;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const int nt = wave + 4 * i;
            T kf[4 * NMT];
#pragma unroll
            for (int ks = 0; ks < 4 * NMT; ++ks) kf[ks] = sm.ks[4 * ks + g16][16 * nt + c16];
            f32x4 acc[NMT];
#pragma unroll
            for (int ks = 0; ks < 4 * NMT; ++ks)
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt)
                    if (ks < 4 * (mt + 1)) acc[mt] = M::mma(kf[ks], x1[mt][ks], ks == 0 ? zero4() : acc[mt]);
#pragma unroll
            for (int mt = 0; mt < NMT; ++mt)
                *(float4 *)(wout + ((size_t)(mt * (DK / 16) + nt) * 64 + lane) * VEC) =
                    make_float4(-acc[mt][0], -acc[mt][1], -acc[mt][2], -acc[mt][3]);
            // K~^T: the lane holds chunk rows perm_row(f, g) of dk row 16 nt + c16
#pragma unroll
            for (int q = 0; q < NMT; ++q) {
                const float4 d = *(const float4 *)&sm.dK[16 * q + 4 * g16];
                const int r = 16 * q + 4 * g16, c = 16 * nt + c16;
                *(float4 *)(kout + ((size_t)(nt * 4 + q) * 64 + lane) * VEC) =
                    make_float4(sm.ks[r][c] * d.x, sm.ks[r + 1][c] * d.y, sm.ks[r + 2][c] * d.z, sm.ks[r + 3][c] * d.w);
            }
        }
        T *ut = (T *)a.ws.ut + sh * WsLayout<T, DK, DV>::ut_elems;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int nt = wave + 4 * i;
            f32x4 acc[NMT];
#pragma unroll
            for (int ks = 0; ks < 4 * NMT; ++ks)
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt)
                    if (ks < 4 * (mt + 1)) acc[mt] = M::mma(x2[mt][ks], vb[i][ks], ks == 0 ? zero4() : acc[mt]);
#pragma unroll
            for (int mt = 0; mt < NMT; ++mt)
                *(float4 *)(ut + ((size_t)(nt * 4 + mt) * 64 + lane) * 4) =
                    make_float4(acc[mt][0], acc[mt][1], acc[mt][2], acc[mt][3]);
        }
    }
}

}  // namespace la
