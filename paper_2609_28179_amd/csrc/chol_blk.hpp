// chol_blk.hpp -- device routines of the blocked MFMA Cholesky family
// (orders 17..64, one problem per wavefront); used by the batched kernels
// (chol_blk.hip) and the ragged solver (ragged.hip).
//
// POTRF / POSV / POTRS / TRSV of one problem of order 17..64 per wavefront,
// blocked in 16 x 16 tiles, with every block product on the matrix cores
// (v_mfma_f32_16x16x4_f32).  From order 25 on, and in every solve with several
// right-hand sides, a diagonal block enters the products as its explicit
// inverse.  Against substitution that leaves the error of X as it is up to
// condition 1e4 (0.6 to 0.9 times as large at conditions of a few, 1.15 at 1e6) but a
// residual 1.2 to 2.5 times as large at 1e4, 0.02 of n u |A| |X|; the factor's own error
// grows too (kBlkSubstMaxN), so that orders up to 24 factor by substitution.
//
// Right-looking block Cholesky (the factorization of Sec. III-B, in blocks):
// for each block column k, factor the diagonal block A_kk = L_kk L_kk^T, form
// the panel L_ik = A_ik L_kk^{-T} for i > k, and update the trailing blocks
// A_ij -= L_ik L_jk^T for k < j <= i.  The unblocked row-per-lane kernel
// issues one v_fmac per lane for every (step, trailing column), two thirds of
// which fall on the upper part; here the trailing update is a dense
// 16 x 16 x 16 contraction per lower block.
//
// Register layout ("T layout"): block (i, j) of the lower triangle sits in
// four VGPRs per lane; lane (q, r) = (lane / 16, lane % 16) holds
// A[16 i + r][16 j + 4 q + c], c = 0..3 -- one 16-byte piece of a row, so
// loads and stores are row-major vectors.  Read as an MFMA accumulator
// (lane (q, r) holds D[4 q + c][r]) the same registers hold the block's
// transpose.  With M in T layout as the A operand and X in accumulator
// layout as the B operand, four v_mfma_f32_16x16x4_f32 (k = 4 q + c in step c)
// give D = M X + C in accumulator layout, and each product of the algorithm
// has that form with no data movement:
//   panel     L_ik^T  = L_kk^{-1} A_ik^T            M = L_kk^{-1}
//   update    A_ij^T -= L_jk L_ik^T                 M = -L_jk
//   forward   Y_k = L_kk^{-1} (B_k - sum_j L_kj Y_j)  M = L_kk^{-1}, -L_kj
// The backward substitution needs L_ik^T and L_kk^{-T} as M; those come from
// a transpose through LDS.  A diagonal block is factored in T layout by panels
// of four columns, and is inverted, from its rows read back from LDS (each
// 16-lane row of the wavefront receives all 16), by forward substitution
// against the identity, which yields L_kk^{-1} in T layout.
//
// Rows past n are identity rows (unit pivots that leave the real rows alone;
// L = I there for the solves) and columns past n are zero.
#pragma once

#include "device_common.hpp"
#include "glass_internal.hpp"
#include "chol_device.hpp"

namespace glass {

constexpr int kXS = kBlkXS;
static_assert(16 * blk_row_stride(4) <= kBlkRegionFloats && 4 * 16 * kXS <= kBlkRegionFloats, "LDS region");
static_assert(16 * kXS <= kBlkSolve1Floats, "LDS region of the one-column solves");
static_assert(16 * kXS <= 16 * blk_row_stride(2), "exchange block inside the staging area");

constexpr int BI(int i, int j) { return i * (i + 1) / 2 + j; }

GLASS_DEV f4_t zero4() { return f4_t{0.f, 0.f, 0.f, 0.f}; }
GLASS_DEV f4_t neg4(const f4_t& v) { return f4_t{-v[0], -v[1], -v[2], -v[3]}; }

// D = M X + C for 16 x 16 blocks: M in T layout, X and C in accumulator layout.
GLASS_DEV f4_t mma(const f4_t& m, const f4_t& x, f4_t c) {
#pragma unroll
    for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f32_16x16x4f32(m[s], x[s], c, 0, 0, 0);
    return c;
}

// The lower blocks of the problem at Ag in T layout.  FULL: n == 16 NBLK;
// otherwise 16 (NBLK - 1) < n < 16 NBLK, so that only the last block row and
// column are cut: the blocks above it load at compile-time positions, rows
// past n load nothing, and the pieces of the last diagonal block past column
// n hold entries right of the diagonal, which are cleared anyway.  The one
// piece that would run past the problem (row n - 1, over the last column) is
// loaded as the problem's last 16 bytes and moved down.  The strict upper
// part of a diagonal block is cleared.  Every load is issued before any is
// read.
template <int NBLK, bool FULL>
GLASS_DEV void blk_load(f4_t (&T)[NBLK * (NBLK + 1) / 2], const float* Ag, int n, int q, int r) {
    const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(Ag, (uint32_t)(n * n) * 4u);
    constexpr int LB = NBLK - 1;
    const int lane_off = (r * n + 4 * q) * 4;
    const int R = 16 * LB + r, C = 16 * LB + 4 * q;  // of the last diagonal block
    const bool tail = !FULL && R == n - 1 && C + 4 > n;
#pragma unroll
    for (int i = 0; i < NBLK; ++i) {
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            int off = lane_off, soff = (16 * i * n + 16 * j) * 4;
            if (!FULL && i == LB) {
                if (R >= n) off = kOob;
                if (j == LB) {
                    off = (R >= n || C > R) ? kOob : tail ? (n * n - 4) * 4 : (R * n + C) * 4;
                    soff = 0;
                }
            }
            T[BI(i, j)] = __builtin_bit_cast(f4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, off, soff, 0));
        }
    }
    if (!FULL) {
        f4_t v = T[BI(LB, LB)];
        const int over = C + 4 - n;  // entries of the piece past column n
        const f4_t d = over == 1   ? f4_t{v[1], v[2], v[3], 0.f}
                       : over == 2 ? f4_t{v[2], v[3], 0.f, 0.f}
                                   : f4_t{v[3], 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x = tail ? d[e] : v[e];
            v[e] = R < n ? x : (4 * q + e == r) ? 1.f : 0.f;
        }
        T[BI(LB, LB)] = v;
    }
#pragma unroll
    for (int i = 0; i < NBLK; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) T[BI(i, i)][e] = (4 * q + e <= r) ? T[BI(i, i)][e] : 0.f;
}

// Diagonal block (T layout) to row-per-lane form with its diagonal entries
// cleared: lane (q, r) receives row r (every 16-lane row of the wavefront a
// full copy).  Returns the lane's diagonal entry.
GLASS_DEV float diag_rows(const f4_t& t, float (&a)[16], float* xs, int q, int r) {
    *reinterpret_cast<f4_t*>(xs + r * kXS + 4 * q) = t;
    wave_sync();
    const float d = xs[r * kXS + r];
    xs[r * kXS + r] = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const f4_t v = *reinterpret_cast<const f4_t*>(xs + r * kXS + 4 * u);
#pragma unroll
        for (int e = 0; e < 4; ++e) a[4 * u + e] = v[e];
    }
    wave_sync();
    return d;
}

// acc += bcast_K(acc) * m, the broadcast of lane K of the 16-lane row folded
// into the v_fmac.  Consecutive calls on one register are three instructions
// apart (four accumulators in turn), above the two wait states a DPP read of a
// just-written VGPR needs.
template <int K>
GLASS_DEV void fmac_self_bcast(float& acc, float m) {
    asm volatile("v_fmac_f32_dpp %0, %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf"
                 : "+v"(acc)
                 : "v"(m), "n"(K));
}

template <int K, int END>
struct InvStep {
    static GLASS_DEV void run(float (&u)[4], const float (&m)[16]) {
#pragma unroll
        for (int c = 0; c < 4; ++c) fmac_self_bcast<K>(u[c], m[K]);
        InvStep<K + 1, END>::run(u, m);
    }
};
template <int END>
struct InvStep<END, END> {
    static GLASS_DEV void run(float (&)[4], const float (&)[16]) {}
};

// Rows of diagonal block k that belong to the problem, rows past them being
// the identity: pivot steps on those would find unit pivots and zero
// coefficients, so the last block of an order that is no multiple of 16 runs
// its first 4, 8, 12 or 16 steps.  With the staged rows of blk_one serving the
// inverse (16 registers fewer): POSV n = 22 x 65,536 107 -> 91 us, n = 36, 3 columns x
// 16,384 63 -> 60, ragged solve of 50,000 systems 144 -> 133.
template <int NBLK, bool FULL>
GLASS_DEV int blk_live(int n, int k) {
    return FULL || k + 1 < NBLK ? 16 : n - 16 * (NBLK - 1);
}

// Panel S (columns 4 S .. 4 S + 3) of a diagonal block in T layout, held by the
// 16 lanes of row S: each column is scaled by 1 / sqrt of its pivot and taken
// off the later columns of the panel.  inv: 1 / sqrt of the first pivot; it and
// the block's registers were written by instructions of the compiler's own, so
// that nothing the asm writes can still be an operand of a product in flight.
// The DPP row mask keeps the other rows' registers; rows above the panel's
// diagonal hold values that are cleared after the last panel.  This is the
// serial chain of the factorization, so the wait states (one before a
// transcendental result or a lane read of a VALU result, two before a DPP read
// or a use of a scalar written by the VALU) are filled with the other columns'
// updates where there are any.
template <int S>
GLASS_DEV void panel_cols(f4_t& t, float inv, float& myinv) {
    constexpr int J = 4 * S;
    constexpr unsigned long long m = seg_mask<16>() << J;
    float d;
    asm volatile(
        "s_nop 0\n\t"
        "v_mul_f32_dpp %0, %0, %5 quad_perm:[0,1,2,3] row_mask:%11 bank_mask:0xf\n\t"
        "v_cndmask_b32_e64 %4, %4, %5, %7\n\ts_nop 0\n\t"
        "v_fmac_f32_dpp %1, %0, -%0 row_newbcast:%13 row_mask:%11 bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %0, -%0 row_newbcast:%14 row_mask:%11 bank_mask:0xf\n\t"
        "v_readlane_b32 %6, %1, %16\n\t"
        "v_fmac_f32_dpp %3, %0, -%0 row_newbcast:%15 row_mask:%11 bank_mask:0xf\n\t"
        "s_nop 0\n\tv_rsq_f32_e32 %5, %6\n\ts_nop 0\n\t"
        "v_mul_f32_dpp %1, %1, %5 quad_perm:[0,1,2,3] row_mask:%11 bank_mask:0xf\n\t"
        "v_cndmask_b32_e64 %4, %4, %5, %8\n\ts_nop 0\n\t"
        "v_fmac_f32_dpp %2, %1, -%1 row_newbcast:%14 row_mask:%11 bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %1, -%1 row_newbcast:%15 row_mask:%11 bank_mask:0xf\n\t"
        "v_readlane_b32 %6, %2, %17\n\t"
        "s_nop 1\n\tv_rsq_f32_e32 %5, %6\n\ts_nop 0\n\t"
        "v_mul_f32_dpp %2, %2, %5 quad_perm:[0,1,2,3] row_mask:%11 bank_mask:0xf\n\t"
        "v_cndmask_b32_e64 %4, %4, %5, %9\n\ts_nop 0\n\t"
        "v_fmac_f32_dpp %3, %2, -%2 row_newbcast:%15 row_mask:%11 bank_mask:0xf\n\t"
        "s_nop 0\n\tv_readlane_b32 %6, %3, %18\n\t"
        "s_nop 1\n\tv_rsq_f32_e32 %5, %6\n\ts_nop 0\n\t"
        "v_mul_f32_dpp %3, %3, %5 quad_perm:[0,1,2,3] row_mask:%11 bank_mask:0xf\n\t"
        "v_cndmask_b32_e64 %4, %4, %5, %10"
        : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(myinv), "+v"(inv), "=&s"(d)
        : "s"(m), "s"(m << 1), "s"(m << 2), "s"(m << 3), "n"(1 << S), "n"(0), "n"(J + 1), "n"(J + 2), "n"(J + 3),
          "n"(16 * S + J + 1), "n"(16 * S + J + 2), "n"(16 * S + J + 3));
}

// Panel S of the block as an MFMA operand of depth 4: lane (q, r) receives
// register q of lane (S, r), which is P[r][q] as the first operand and
// P^T[q][r] as the second.  Two wait states between a VALU write and the swap
// or MFMA that reads it.
template <int S>
GLASS_DEV float panel_operand(const f4_t& t) {
    float u0 = t[0], u1 = t[1], u2 = t[2], u3 = t[3];
    asm volatile(
        "s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\tv_permlane16_swap_b32 %2, %3\n\ts_nop 1\n\t"
        ".if %4\n\tv_permlane32_swap_b32 %1, %3\n\t.else\n\tv_permlane32_swap_b32 %0, %2\n\t.endif\n\ts_nop 1"
        : "+v"(u0), "+v"(u1), "+v"(u2), "+v"(u3)
        : "n"(S & 1));
    return S == 0 ? u0 : S == 1 ? u1 : u2;
}

// Panels S .. of a diagonal block: four columns, then their product P P^T off
// the columns to the right, one v_mfma_f32_16x16x4_f32.  The finished columns
// are kept by a select and not by zero rows of P, so that a failed pivot's NaN
// leaves the columns left of it as they are.
template <int S>
GLASS_DEV void panel_steps(f4_t& t, float& myinv, int q, int live) {
    panel_cols<S>(t, rsq(readlane(t[0], 20 * S)), myinv);
    if constexpr (S < 3) {
        if (live > 4 * (S + 1)) {
            const float p = panel_operand<S>(t);
            const f4_t d = __builtin_amdgcn_mfma_f32_16x16x4f32(-p, p, t, 0, 0, 0);
#pragma unroll
            for (int c = 0; c < 4; ++c) t[c] = q > S ? d[c] : t[c];
            panel_steps<S + 1>(t, myinv, q, live);
        }
    }
}

// Cholesky of a diagonal block in T layout, in place (strict upper part
// cleared); rows from `live` (1 .. 16, wave-uniform) on are the identity.  In
// row-per-lane form, all four 16-lane rows with a copy, the 120 updates of the
// trailing columns were the largest part of the factorization's VALU work
// (without them POSV n = 22 x 65,536 took 76 of 96 us, n = 30 x 16,384 31 of
// 37); by panels of four columns they are 24, and three matrix-core products.
// Row form against panels: POTRF n = 20 x 65,536 74 -> 65.5 us, POSV n = 22 x
// 65,536 96 -> 88, n = 30 x 16,384 38.5 -> 36, n = 36 with 3 columns x 16,384
// 59.7 -> 57, n = 48 x 256 (the chain alone) 7.6 -> 7.0, ragged solve of
// 50,000 systems with its plan 155 -> 143; POTRF n = 32 x 65,536, at its
// bytes, 94 -> 95.
GLASS_DEV void diag_factor(f4_t& t, int& f, float& myinv, int q, int r, int live) {
    panel_steps<0>(t, myinv, q, live);
    f = first_nonfinite<16>(myinv);
#pragma unroll
    for (int c = 0; c < 4; ++c) t[c] = 4 * q + c <= r ? t[c] : 0.f;
}

// panel_cols with the same columns of the block u below the diagonal one (rows
// in the same lanes, T layout): each is scaled by its pivot's 1 / sqrt and
// taken off u's later columns against the diagonal block's rows.  Most of
// u's instructions stand where panel_cols waits.
template <int S>
GLASS_DEV void panel_cols_rows(f4_t& t, f4_t& u, float inv, float& myinv) {
    constexpr int J = 4 * S;
    constexpr unsigned long long m = seg_mask<16>() << J;
    float d;
    asm volatile(
        "s_nop 0\n\t"
        "v_mul_f32_dpp %0, %0, %9 quad_perm:[0,1,2,3] row_mask:%15 bank_mask:0xf\n\t"
        "v_mul_f32_dpp %4, %4, %9 quad_perm:[0,1,2,3] row_mask:%15 bank_mask:0xf\n\t"
        "v_cndmask_b32_e64 %8, %8, %9, %11\n\t"
        "v_fmac_f32_dpp %1, %0, -%0 row_newbcast:%16 row_mask:%15 bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %5, %0, -%4 row_newbcast:%16 row_mask:%15 bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %0, -%0 row_newbcast:%17 row_mask:%15 bank_mask:0xf\n\t"
        "v_readlane_b32 %10, %1, %19\n\t"
        "v_fmac_f32_dpp %6, %0, -%4 row_newbcast:%17 row_mask:%15 bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %0, -%0 row_newbcast:%18 row_mask:%15 bank_mask:0xf\n\t"
        "v_rsq_f32_e32 %9, %10\n\t"
        "v_fmac_f32_dpp %7, %0, -%4 row_newbcast:%18 row_mask:%15 bank_mask:0xf\n\t"
        "v_mul_f32_dpp %1, %1, %9 quad_perm:[0,1,2,3] row_mask:%15 bank_mask:0xf\n\t"
        "v_mul_f32_dpp %5, %5, %9 quad_perm:[0,1,2,3] row_mask:%15 bank_mask:0xf\n\t"
        "v_cndmask_b32_e64 %8, %8, %9, %12\n\t"
        "v_fmac_f32_dpp %2, %1, -%1 row_newbcast:%17 row_mask:%15 bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %6, %1, -%5 row_newbcast:%17 row_mask:%15 bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %1, -%1 row_newbcast:%18 row_mask:%15 bank_mask:0xf\n\t"
        "v_readlane_b32 %10, %2, %20\n\t"
        "v_fmac_f32_dpp %7, %1, -%5 row_newbcast:%18 row_mask:%15 bank_mask:0xf\n\t"
        "s_nop 0\n\tv_rsq_f32_e32 %9, %10\n\ts_nop 0\n\t"
        "v_mul_f32_dpp %2, %2, %9 quad_perm:[0,1,2,3] row_mask:%15 bank_mask:0xf\n\t"
        "v_mul_f32_dpp %6, %6, %9 quad_perm:[0,1,2,3] row_mask:%15 bank_mask:0xf\n\t"
        "v_cndmask_b32_e64 %8, %8, %9, %13\n\t"
        "v_fmac_f32_dpp %3, %2, -%2 row_newbcast:%18 row_mask:%15 bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %7, %2, -%6 row_newbcast:%18 row_mask:%15 bank_mask:0xf\n\t"
        "v_readlane_b32 %10, %3, %21\n\t"
        "s_nop 1\n\tv_rsq_f32_e32 %9, %10\n\ts_nop 0\n\t"
        "v_mul_f32_dpp %3, %3, %9 quad_perm:[0,1,2,3] row_mask:%15 bank_mask:0xf\n\t"
        "v_mul_f32_dpp %7, %7, %9 quad_perm:[0,1,2,3] row_mask:%15 bank_mask:0xf\n\t"
        "v_cndmask_b32_e64 %8, %8, %9, %14"
        : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(u[0]), "+v"(u[1]), "+v"(u[2]), "+v"(u[3]), "+v"(myinv),
          "+v"(inv), "=&s"(d)
        : "s"(m), "s"(m << 1), "s"(m << 2), "s"(m << 3), "n"(1 << S), "n"(J + 1), "n"(J + 2), "n"(J + 3),
          "n"(16 * S + J + 1), "n"(16 * S + J + 2), "n"(16 * S + J + 3));
}

// panel_operand of t and of u.
template <int S>
GLASS_DEV void panel_operands(const f4_t& t, const f4_t& u, float& p, float& pu) {
    float t0 = t[0], t1 = t[1], t2 = t[2], t3 = t[3], u0 = u[0], u1 = u[1], u2 = u[2], u3 = u[3];
    asm volatile(
        "s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\tv_permlane16_swap_b32 %2, %3\n\t"
        "v_permlane16_swap_b32 %4, %5\n\tv_permlane16_swap_b32 %6, %7\n\t"
        ".if %8\n\tv_permlane32_swap_b32 %1, %3\n\ts_nop 0\n\tv_permlane32_swap_b32 %5, %7\n\t"
        ".else\n\tv_permlane32_swap_b32 %0, %2\n\ts_nop 0\n\tv_permlane32_swap_b32 %4, %6\n\t.endif\n\ts_nop 1"
        : "+v"(t0), "+v"(t1), "+v"(t2), "+v"(t3), "+v"(u0), "+v"(u1), "+v"(u2), "+v"(u3)
        : "n"(S & 1));
    p = S == 0 ? t0 : S == 1 ? t1 : t2;
    pu = S == 0 ? u0 : S == 1 ? u1 : u2;
}

template <int S>
GLASS_DEV void panel_steps_rows(f4_t& t, f4_t& u, float& myinv, int q) {
    panel_cols_rows<S>(t, u, rsq(readlane(t[0], 20 * S)), myinv);
    if constexpr (S < 3) {
        float p, pu;
        panel_operands<S>(t, u, p, pu);
        const f4_t d = __builtin_amdgcn_mfma_f32_16x16x4f32(-p, p, t, 0, 0, 0);
        const f4_t e = __builtin_amdgcn_mfma_f32_16x16x4f32(-p, pu, u, 0, 0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            t[c] = q > S ? d[c] : t[c];
            u[c] = q > S ? e[c] : u[c];
        }
        panel_steps_rows<S + 1>(t, u, myinv, q);
    }
}

// diag_factor of a whole diagonal block t and, column by column with it, the
// block u below it: u <- u t^{-T}, by substitution and not by t's inverse.
// With the inverse, POSV n = 22 took 10.0 us against 10.5 at 4096 problems (27.8
// and 28.0 at 16,384, POTRF alike throughout), and its factor was off by 1.3 to
// 1.6 times as much at condition 1e4, 1.7 to 2.2 times at 1e6.
GLASS_DEV void diag_factor_rows(f4_t& t, f4_t& u, int& f, float& myinv, int q, int r) {
    panel_steps_rows<0>(t, u, myinv, q);
    f = first_nonfinite<16>(myinv);
#pragma unroll
    for (int c = 0; c < 4; ++c) t[c] = 4 * q + c <= r ? t[c] : 0.f;
}

// X = L^{-1} of a 16 x 16 lower diagonal block, in T layout: lane (q, r)
// returns row r, columns 4 q .. 4 q + 3.  Forward substitution against the
// identity with the lane's own coefficients m_K = -L_rK / L_rr (zero in lane
// K and above the diagonal) and myinv = 1 / L_rr reads
// X_r = e_r / L_rr + sum_{K<r} m_K X_K, so the rows are finished in order
// K = 0..15 and each step is one v_fmac per column with lane K's row
// broadcast.  Rows from `live` on are the identity.
GLASS_DEV f4_t tri_inverse_l(const float (&m)[16], float myinv, int q, int r, int live = 16) {
    float u[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) u[c] = (4 * q + c == r) ? myinv : 0.f;
    asm volatile("s_nop 1" : "+v"(u[0]), "+v"(u[1]), "+v"(u[2]), "+v"(u[3]));
    InvStep<0, 4>::run(u, m);
    if (live > 4) {
        InvStep<4, 8>::run(u, m);
        if (live > 8) {
            InvStep<8, 12>::run(u, m);
            if (live > 12) InvStep<12, 16>::run(u, m);
        }
    }
    return f4_t{u[0], u[1], u[2], u[3]};
}

// Row r of a factored diagonal block that is in LDS at xs (row stride S), with
// its diagonal entry cleared; the entry itself is put back if KEEP.
template <int S, bool KEEP>
GLASS_DEV void staged_rows_zero_diag(float (&az)[16], float* xs, int r) {
    float* d = xs + r * S + r;
    const float keep = KEEP ? *d : 0.f;
    *d = 0.f;
    wave_sync();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const f4_t v = *reinterpret_cast<const f4_t*>(xs + r * S + 4 * u);
#pragma unroll
        for (int e = 0; e < 4; ++e) az[4 * u + e] = v[e];
    }
    wave_sync();
    if (KEEP) {
        *d = keep;
        wave_sync();
    }
}

// The same for a block whose rows are in registers (every 16-lane row a copy):
// the lanes of row 0 write them to LDS first.
template <int S>
GLASS_DEV void rows_zero_diag(const float (&a)[16], float (&az)[16], float* xs, int q, int r) {
    if (q == 0) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            *reinterpret_cast<f4_t*>(xs + r * S + 4 * u) = f4_t{a[4 * u], a[4 * u + 1], a[4 * u + 2], a[4 * u + 3]};
    }
    wave_sync();
    staged_rows_zero_diag<S, false>(az, xs, r);
}

// Rows 16 k .. of a row-major n x n matrix from the staged block row at xs
// (row stride blk_row_stride): a block row is contiguous in memory, so it
// leaves as 16-byte pieces whatever the order and alignment (a piece that
// spans two rows is gathered by element), one per lane and round in NBLK
// rounds.  The last piece of an odd-sized last block row moves back over its
// neighbour and writes the same values.  The row of an element comes from
// (g + 1/2) * (1 / n) in FP32: g < 1024 and n <= 64 keep its error below
// 2e-5, against a distance of 1 / (2 n) >= 1/128 from the next integer.
// With element-wise 4-byte stores (an integer division each) and loads and
// right-hand-side accesses under lane conditions, the cut instances issued
// nearly twice the instructions of the whole-tile ones (POSV n = 64, several
// columns: 4511 against 2521 static, now about 2900).  At 16,384 problems: adjoint
// n = 36, 3 columns 58.3 -> 48.3 us, n = 25 23.7 -> 19.1, POSV n = 36, 3 columns 67 -> 63
// (there the diagonal blocks' VALU work is the bound), ragged solve of
// 50,000 systems 153 -> 146.
template <int NBLK, bool FULL>
GLASS_DEV void block_row_store(float* Mg, int k, int n, const float* xs, int lane) {
    constexpr int RS = blk_row_stride(NBLK);
    float* dst = Mg + (size_t)16 * k * n;
    if (FULL) {
        constexpr int N4 = 4 * NBLK;  // 16-byte pieces per row
#pragma unroll
        for (int g = lane; g < 16 * N4; g += 64) {
            const int rr = g / N4, c4 = g % N4;
            reinterpret_cast<f4_t*>(dst)[g] = *reinterpret_cast<const f4_t*>(xs + rr * RS + 4 * c4);
        }
        return;
    }
    const bool last = k == NBLK - 1;
    const int len = (last ? n - 16 * k : 16) * n;
    const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(dst, (uint32_t)len * 4u);
    asm volatile("" : "+v"(lane));  // the piece addresses are formed anew for each block row, not kept in registers between them
    const float rn = recip((float)n);
    const bool whole = (n & 3) == 0;
#pragma unroll
    for (int u = 0; u < NBLK; ++u) {
        const int g = 4 * (lane + 64 * u), at = min(g, len - 4);
        const int rr = (int)(((float)at + 0.5f) * rn), cc = at - rr * n;
        const float* src = xs + rr * RS + cc;
        f4_t v;
        if (whole) {
            v = *reinterpret_cast<const f4_t*>(src);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = src[cc + e >= n ? e + RS - n : e];
        }
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned, v), rs,
                                               g < len ? at * 4 : kOob, 0, 0);
    }
}

// Block row k of L (rows 16 k .. 16 k + 15) staged in LDS for block_row_store:
// the finished blocks up to the diagonal and +0 to the right.
template <int NBLK>
GLASS_DEV void stage_block_row(const f4_t (&T)[NBLK * (NBLK + 1) / 2], int k, float* xs, int q, int r) {
    constexpr int kRS = blk_row_stride(NBLK);
#pragma unroll
    for (int j = 0; j < NBLK; ++j)
        *reinterpret_cast<f4_t*>(xs + r * kRS + 16 * j + 4 * q) = j <= k ? T[BI(k, j)] : zero4();
    wave_sync();
}

// Transposes of up to four blocks through LDS (exchange areas of 16 x kXS):
// a block in T layout comes back in T layout of its transpose.
template <int NB>
GLASS_DEV void transpose_blocks(f4_t (&v)[4], float* xs, int q, int r) {
#pragma unroll
    for (int b = 0; b < NB; ++b) *reinterpret_cast<f4_t*>(xs + b * 16 * kXS + r * kXS + 4 * q) = v[b];
    wave_sync();
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) v[b][c] = xs[b * 16 * kXS + (4 * q + c) * kXS + r];
    wave_sync();
}

// The first nb (a constant once unrolled) of up to NB blocks.
template <int NB>
GLASS_DEV void transpose_first(f4_t (&v)[4], int nb, float* xs, int q, int r) {
    if (nb == NB) {
        transpose_blocks<NB>(v, xs, q, r);
    } else {
        if constexpr (NB > 1) transpose_first<NB - 1>(v, nb, xs, q, r);
    }
}

// Columns cb .. cb + 15 of the row-major [n][nr] right-hand sides, in
// accumulator layout per block row (lane (q, r), element e: row 16 k + 4 q + e,
// column cb + r): buffer accesses at a per-lane offset plus a scalar row
// offset, out of range for columns past nr; the last block row carries its
// whole offset per lane, so that rows past n fall out of range too.
template <int NBLK, bool FULL>
struct RhsOffsets {
    int lane, nr;
    GLASS_DEV RhsOffsets(int nr_, int cb, int q, int r)
        : lane(cb + r < nr_ ? (4 * q * nr_ + cb + r) * 4 : kOob), nr(nr_) {}
    GLASS_DEV int v(int k, int e) const { return !FULL && k == NBLK - 1 ? lane + (16 * k + e) * nr * 4 : lane; }
    GLASS_DEV int s(int k, int e) const { return !FULL && k == NBLK - 1 ? 0 : (16 * k + e) * nr * 4; }
};

template <int NBLK, bool FULL>
GLASS_DEV void rhs_load(f4_t (&Y)[NBLK], const float* Bg, int n, int nr, int cb, int q, int r) {
    const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(Bg, (uint32_t)(n * nr) * 4u);
    const RhsOffsets<NBLK, FULL> o(nr, cb, q, r);
#pragma unroll
    for (int k = 0; k < NBLK; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            Y[k][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, o.v(k, e), o.s(k, e), 0));
}

template <int NBLK, bool FULL>
GLASS_DEV void rhs_store(const f4_t (&Y)[NBLK], float* Bg, int n, int nr, int cb, int q, int r) {
    const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(Bg, (uint32_t)(n * nr) * 4u);
    const RhsOffsets<NBLK, FULL> o(nr, cb, q, r);
#pragma unroll
    for (int k = 0; k < NBLK; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(Y[k][e]), rs, o.v(k, e), o.s(k, e), 0);
}

template <int NBLK, int K>
struct BwdBlk {
    // X_K = L_KK^{-T} (Y_K - sum_{i>K} L_iK^T X_i); nT holds -L blocks.
    static GLASS_DEV void run(const f4_t (&nT)[NBLK * (NBLK + 1) / 2], const f4_t (&linv)[NBLK], f4_t (&Y)[NBLK],
                              float* xs, int q, int r) {
        constexpr int NI = NBLK - 1 - K;
        f4_t v[4];
#pragma unroll
        for (int i = 0; i < NI; ++i) v[i] = nT[BI(K + 1 + i, K)];
        v[NI] = linv[K];
        transpose_blocks<NI + 1>(v, xs, q, r);
        f4_t s = Y[K];
#pragma unroll
        for (int i = 0; i < NI; ++i) s = mma(v[i], Y[K + 1 + i], s);
        Y[K] = mma(v[NI], s, zero4());
        BwdBlk<NBLK, K - 1>::run(nT, linv, Y, xs, q, r);
    }
};
template <int NBLK>
struct BwdBlk<NBLK, -1> {
    static GLASS_DEV void run(const f4_t (&)[NBLK * (NBLK + 1) / 2], const f4_t (&)[NBLK], f4_t (&)[NBLK], float*,
                              int, int) {}
};

// ------------------------------------------------- up to four columns at a time
// A 16 x 16 x 16 product holds the matrix cores 128 cycles however few columns
// X has.  With at most four, the sixteen 4 x 4 x 1 products of one
// v_mfma_f32_4x4x1 do the work of a 16 x 16 x 4 in a quarter of the time: block
// (q, i) multiplies rows 4 i .. 4 i + 3 and column 4 q + c of M by row 4 q + c
// of X, so that M's T layout (register c of lane (q, 4 i + a) is
// M[4 i + a][4 q + c]) is its operand as it stands, and what is left is a sum
// over the four lane rows q.  Two forms of a 16 x 4 block of columns:
//   piece form    lane (q, 4 i + j): V[4 i + q][j], one register (loads,
//                 stores and what sum_pieces leaves)
//   operand form  lane (q, 4 i + j), register c: V[4 q + c][j], for every i

GLASS_DEV f4_t mma4(const f4_t& m, const f4_t& x, f4_t c) {
#pragma unroll
    for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f32_4x4x1f32(m[s], x[s], c, 0, 0, 0);
    return c;
}

// Sum over the lane rows of products with register e, lane (q, 4 i + j)
// holding row 4 i + e, column j: row e of the lanes receives register e's sum,
// the piece form.  The leading wait covers the product's last write.
GLASS_DEV float sum_pieces(f4_t d) {
    float d0 = d[0], d1 = d[1], d2 = d[2], d3 = d[3];
    asm volatile(
        "s_nop 7\n\tv_permlane32_swap_b32 %0, %2\n\tv_permlane32_swap_b32 %1, %3\n\t"
        "v_add_f32 %0, %0, %2\n\tv_add_f32 %1, %1, %3\n\ts_nop 1\n\t"
        "v_permlane16_swap_b32 %0, %1\n\tv_add_f32 %0, %0, %1"
        : "+v"(d0), "+v"(d1), "+v"(d2), "+v"(d3));
    return d0;
}

// Piece form to operand form through 64 floats of LDS.
GLASS_DEV f4_t piece_operand(float v, float* xs, int q, int r) {
    xs[16 * (r & 3) + 4 * (r >> 2) + q] = v;
    wave_sync();
    const f4_t o = *reinterpret_cast<const f4_t*>(xs + 16 * (r & 3) + 4 * q);
    wave_sync();
    return o;
}

// The row-major [n][nr] right-hand sides, nr <= 4, in piece form (zero past n
// and nr): byte offset of block row k.
GLASS_DEV int piece_offset(int nr, int k, int q, int r) {
    return (r & 3) < nr ? ((16 * k + 4 * (r >> 2) + q) * nr + (r & 3)) * 4 : kOob;
}

// L y = b, then L^T x = y, x stored and returned in piece form; nT: L in T layout with its off-diagonal blocks negated.
template <int NBLK>
GLASS_DEV void blk_solve4(const f4_t (&nT)[NBLK * (NBLK + 1) / 2], const f4_t (&linv)[NBLK], float (&y)[NBLK],
                          const float* Bi, float* Bg, int n, int nr, float* xs, int q, int r) {
    const __amdgpu_buffer_rsrc_t ri = buffer_rsrc(Bi, (uint32_t)(n * nr) * 4u);
    const __amdgpu_buffer_rsrc_t ro = buffer_rsrc(Bg, (uint32_t)(n * nr) * 4u);
#pragma unroll
    for (int k = 0; k < NBLK; ++k) y[k] = buf_load1(ri, piece_offset(nr, k, q, r), 0);
    f4_t o[NBLK];
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
        f4_t acc = zero4();
#pragma unroll
        for (int j = 0; j < k; ++j) acc = mma4(nT[BI(k, j)], o[j], acc);
        if (k) y[k] += sum_pieces(acc);
        y[k] = sum_pieces(mma4(linv[k], piece_operand(y[k], xs, q, r), zero4()));
        if (k + 1 < NBLK) o[k] = piece_operand(y[k], xs, q, r);
    }
#pragma unroll
    for (int k = NBLK - 1; k >= 0; --k) {
        const int ni = NBLK - 1 - k;
        f4_t v[4] = {zero4(), zero4(), zero4(), zero4()};
#pragma unroll
        for (int i = 0; i < ni; ++i) v[i] = nT[BI(k + 1 + i, k)];
        v[ni] = linv[k];
        transpose_first<NBLK>(v, ni + 1, xs, q, r);
        f4_t acc = zero4();
#pragma unroll
        for (int i = 0; i < ni; ++i) acc = mma4(v[i], o[k + 1 + i], acc);
        if (ni) y[k] += sum_pieces(acc);
        y[k] = sum_pieces(mma4(v[ni], piece_operand(y[k], xs, q, r), zero4()));
        if (k) o[k] = piece_operand(y[k], xs, q, r);
    }
#pragma unroll
    for (int k = 0; k < NBLK; ++k)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y[k]), ro, piece_offset(nr, k, q, r), 0, 0);
}

// --------------------------------------------- one right-hand side, no inverses
// A single right-hand side (TRSV; POTRS with nrhs = 1) gains nothing from the
// matrix cores: an MFMA product spends 15 of its 16 columns on padding, and
// the 16 x 16 diagonal-block inverses cost more VALU than the substitution
// itself.  This path keeps L in T layout and runs everything on VALU:
//   R form: a 16-vector of block row k with lane (q, r) holding v[r] in
//           every one of the four 16-lane rows q;
//   diagonal block: plain substitution on its rows (forward) or columns
//           (backward) in row-per-lane form, one DPP step per unknown on
//           s = b_r / L_rr: s += bcast_K(s) * m_K with m_K = -L_rK / L_rr
//           (forward) or -L_Kr / L_rr (backward), the lane's own entries
//           times its own -1 / L_rr (the diagonal entry is cleared on the
//           way through LDS, so m_K is zero in lane K with no select);
//   off-diagonal blocks: a lane's four T-layout entries times the matching
//           four unknowns, summed across the four rows q (two permlane
//           swaps) for L_kj x_j, or across the 16 lanes of a row (four DPP
//           steps) for L_ik^T x_i.
// Pending products are accumulated as soon as a block of x is known
// (right-looking), so only one partial sum per later block stays live.

// acc += bcast_K(acc) * m with the two wait states the DPP read of a
// just-written acc needs.
template <int K>
GLASS_DEV void fmac_self_bcast_w(float& acc, float m) {
    asm volatile("s_nop 1\n\tv_fmac_f32_dpp %0, %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf"
                 : "+v"(acc)
                 : "v"(m), "n"(K));
}

template <int K, int END>  // steps K, K + 1 .. END - 1, or K, K - 1 .. END + 1
struct DiagSub {
    static GLASS_DEV void run(float& s, const float (&m)[16]) {
        fmac_self_bcast_w<K>(s, m[K]);
        DiagSub<K + (K < END ? 1 : -1), END>::run(s, m);
    }
};
template <int END>
struct DiagSub<END, END> {
    static GLASS_DEV void run(float&, const float (&)[16]) {}
};

// Forward (unknowns 0 .. 15) and backward (15 .. 0) substitution; rows from
// `live` on are the identity, whose steps add nothing.
GLASS_DEV void diag_fwd(float& s, const float (&m)[16], int live) {
    DiagSub<0, 4>::run(s, m);
    if (live > 4) {
        DiagSub<4, 8>::run(s, m);
        if (live > 8) {
            DiagSub<8, 12>::run(s, m);
            if (live > 12) DiagSub<12, 16>::run(s, m);
        }
    }
}
GLASS_DEV void diag_bwd(float& s, const float (&m)[16], int live) {
    if (live > 4) {
        if (live > 8) {
            if (live > 12) DiagSub<15, 11>::run(s, m);
            DiagSub<11, 7>::run(s, m);
        }
        DiagSub<7, 3>::run(s, m);
    }
    DiagSub<3, -1>::run(s, m);
}

// The same on unscaled coefficients (row r of L forward, column r backward, the
// diagonal entry cleared), for a right-hand side with an infinity or a NaN: in
// step K unknown K is s_K / L_KK, kept in lane K of y, and its products leave
// s.  The lanes whose unknown is already final meet zero coefficients, whose
// product with such an entry is no zero: it lands in their s, and y keeps
// every unknown that does not depend on it.  The select fills one of the two
// wait states between the product and its DPP read.
template <int K>
GLASS_DEV void keep_and_fmac(float& s, float& y, float t, float a) {
    asm volatile("v_cndmask_b32_e64 %1, %1, %2, %4\n\ts_nop 0\n\t"
                 "v_fmac_f32_dpp %0, %2, -%3 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
                 : "+v"(s), "+v"(y)
                 : "v"(t), "v"(a), "s"(seg_mask<16>() << K), "n"(K));
}

template <int K, int END>  // steps K, K + 1 .. END - 1, or K, K - 1 .. END + 1
struct DiagKeep {
    static GLASS_DEV void run(float& s, float& y, const float (&a)[16], float myinv) {
        keep_and_fmac<K>(s, y, s * myinv, a[K]);
        DiagKeep<K + (K < END ? 1 : -1), END>::run(s, y, a, myinv);
    }
};
template <int END>
struct DiagKeep<END, END> {
    static GLASS_DEV void run(float&, float&, const float (&)[16], float) {}
};

GLASS_DEV float diag_keep_fwd(float s, const float (&a)[16], float myinv, int live) {
    float y = 0.f;
    DiagKeep<0, 4>::run(s, y, a, myinv);
    if (live > 4) {
        DiagKeep<4, 8>::run(s, y, a, myinv);
        if (live > 8) {
            DiagKeep<8, 12>::run(s, y, a, myinv);
            if (live > 12) DiagKeep<12, 16>::run(s, y, a, myinv);
        }
    }
    return y;
}
GLASS_DEV float diag_keep_bwd(float s, const float (&a)[16], float myinv, int live) {
    float y = 0.f;
    if (live > 4) {
        if (live > 8) {
            if (live > 12) DiagKeep<15, 11>::run(s, y, a, myinv);
            DiagKeep<11, 7>::run(s, y, a, myinv);
        }
        DiagKeep<7, 3>::run(s, y, a, myinv);
    }
    DiagKeep<3, -1>::run(s, y, a, myinv);
    return y;
}

// v summed over the four 16-lane rows (lanes r, r + 16, r + 32, r + 48), in
// every lane: each v_permlane*_swap exchanges half of v with half of a copy,
// and the VALU write of the copy gets its two wait states before the swap.
GLASS_DEV float sum_rows4(float v) {
    float t;
    asm volatile(
        "v_mov_b32 %1, %0\n"
        "s_nop 1\n"
        "v_permlane32_swap_b32 %0, %1\n"
        "v_add_f32 %0, %0, %1\n"
        "v_mov_b32 %1, %0\n"
        "s_nop 1\n"
        "v_permlane16_swap_b32 %0, %1\n"
        "v_add_f32 %0, %0, %1\n"
        : "+v"(v), "=&v"(t));
    return v;
}

// Each of z[0..3] summed over the 16 lanes of its row, in every lane of the
// row (quad swaps, then the half-row and row mirrors).  The four registers
// take turns, so every DPP read is three instructions after the write of its
// source; the leading s_nop covers the caller's last writes.
GLASS_DEV void sum_row16(float (&z)[4]) {
    asm volatile(
        "s_nop 1\n"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %2, %2, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %3, %3, %3 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %2, %2, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %3, %3, %3 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %2, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %3, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %1, %1, %1 row_mirror row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %2, %2, %2 row_mirror row_mask:0xf bank_mask:0xf\n"
        "v_add_f32_dpp %3, %3, %3 row_mirror row_mask:0xf bank_mask:0xf\n"
        : "+v"(z[0]), "+v"(z[1]), "+v"(z[2]), "+v"(z[3]));
}

// xc[c] = v[4 q + c] of an R-form v (lane (q, 4 q + c) holds it).
GLASS_DEV void r_to_c(float v, float (&xc)[4], int q) {
    const int vi = __float_as_int(v);
#pragma unroll
    for (int c = 0; c < 4; ++c) xc[c] = __int_as_float(__builtin_amdgcn_ds_bpermute((20 * q + c) * 4, vi));
}

// R form of w with w[4 q + c] = z[c] in every lane of row q: lane (q', r')
// takes z[r' % 4] from lane r' % 4 of row r' / 4.
GLASS_DEV float c_to_r(const float (&z)[4], int r) {
    const int c = r & 3;
    const float w = c == 0 ? z[0] : c == 1 ? z[1] : c == 2 ? z[2] : z[3];
    return __int_as_float(__builtin_amdgcn_ds_bpermute((16 * (r >> 2) + c) * 4, __float_as_int(w)));
}

// Diagonal block k of L (T layout) transposed through LDS: lane (q, r)
// receives column r (col[j] = L_kk[j][r]) with its diagonal entry cleared;
// returns L_kk[r][r].
GLASS_DEV float diag_cols(const f4_t& t, float (&col)[16], float* xs, int q, int r) {
#pragma unroll
    for (int c = 0; c < 4; ++c) xs[(4 * q + c) * kXS + r] = t[c];
    wave_sync();
    const float d = xs[r * kXS + r];
    xs[r * kXS + r] = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const f4_t v = *reinterpret_cast<const f4_t*>(xs + r * kXS + 4 * u);
#pragma unroll
        for (int e = 0; e < 4; ++e) col[4 * u + e] = v[e];
    }
    wave_sync();
    return d;
}

// The pieces of the single-column solve; x[k] is block k of the vector in R
// form (lane (q, r) holds element 16 k + r in every row q).
template <int NBLK, bool FULL>
GLASS_DEV void blk_x_load(float (&x)[NBLK], const float* bg, int n, int r) {
    const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(bg, (uint32_t)n * 4u);
#pragma unroll
    for (int k = 0; k < NBLK; ++k)
        x[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (16 * k + r) * 4, 0, 0));
}

template <int NBLK, bool FULL>
GLASS_DEV void blk_x_store(const float (&x)[NBLK], float* bg, int n, int q, int r) {
    const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(bg, (uint32_t)n * 4u);
#pragma unroll
    for (int k = 0; k < NBLK; ++k)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x[k]), rs, q == 0 ? (16 * k + r) * 4 : kOob, 0, 0);
}

// Forward step k: block k of y from its pending sum p[k] by the diagonal
// block's lane-local coefficients m_K = -L_rK / L_rr and 1 / L_rr (the
// right-hand side is scaled by it first; KEEP: m_K = L_rK, diag_keep_fwd), then
// its contributions L_ik y_k to the pending sums of the later blocks
// (right-looking, p[i] split over the rows q).
template <int NBLK, bool KEEP>
GLASS_DEV void blk_fwd_step(const f4_t (&T)[NBLK * (NBLK + 1) / 2], int k, const float (&m)[16], float myinv,
                            float (&x)[NBLK], float (&p)[NBLK], int q, int live) {
    float s = k > 0 ? x[k] - sum_rows4(p[k]) : x[k];
    if (KEEP) {
        x[k] = diag_keep_fwd(s, m, myinv, live);
    } else {
        s *= myinv;
        diag_fwd(s, m, live);
        x[k] = s;
    }
    if (k + 1 < NBLK) {
        float xc[4];
        r_to_c(x[k], xc, q);
#pragma unroll
        for (int i = k + 1; i < NBLK; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) p[i] = fmaf(T[BI(i, k)][c], xc[c], p[i]);
    }
}

// L^T x = y, bottom block first (left-looking over the columns: z[j] collects
// sum_i L_ij^T x_i split over the lanes of a row).
template <int NBLK, bool FULL, bool KEEP>
GLASS_DEV void blk_bwd1(const f4_t (&T)[NBLK * (NBLK + 1) / 2], float (&x)[NBLK], float* xs, int n, int q, int r) {
    float z[NBLK][4];
#pragma unroll
    for (int k = 0; k < NBLK; ++k)
#pragma unroll
        for (int c = 0; c < 4; ++c) z[k][c] = 0.f;
#pragma unroll
    for (int k = NBLK - 1; k >= 0; --k) {
        float s = x[k];
        if (k + 1 < NBLK) {
            sum_row16(z[k]);
            s -= c_to_r(z[k], r);
        }
        float col[16];
        const float myinv = recip(diag_cols(T[BI(k, k)], col, xs, q, r)), nmy = -myinv;
        if (KEEP) {
            x[k] = diag_keep_bwd(s, col, myinv, blk_live<NBLK, FULL>(n, k));
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j) col[j] *= nmy;  // -L_jr / L_rr
            s *= myinv;
            diag_bwd(s, col, blk_live<NBLK, FULL>(n, k));
            x[k] = s;
        }
#pragma unroll
        for (int j = 0; j < k; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) z[j][c] = fmaf(T[BI(k, j)][c], x[k], z[j][c]);
    }
}

// The backward pass of op 4 (POSV, one right-hand side), L^T x = y with y in
// R form in x, on what the factorization leaves behind:
//   last block K: the rows of L_KK are still staged in LDS (xs, row stride
//       blk_row_stride(NBLK)) with the diagonal entry cleared, so lane r
//       reads column r and scales it by its own -1 / L_rr, the coefficients
//       of blk_bwd1: x_r = s_r / L_rr + sum_{j>r} (-L_jr / L_rr) x_j, one
//       DPP step per unknown;
//   blocks k < K: L_kk^{-1} is in LDS at lt (T layout, 16 x kXS floats per
//       block), so lane (q, r) reads its column r, rows 4 q .. 4 q + 3, and
//       x_k = L_kk^{-T} s is four FMAs on s in C form (the form the sum of
//       the pending products L_ik^T x_i already has) and one sum over the
//       four rows q -- no substitution chain.  SUB: block 0 by substitution on
//       its columns, as the last block (there is no inverse of it).
template <int NBLK, bool FULL, bool SUB>
GLASS_DEV void blk_bwd1_posv(const f4_t (&T)[NBLK * (NBLK + 1) / 2], float (&x)[NBLK], float myinv_last,
                             const float* lt, float* xs, int n, int q, int r) {
    constexpr int K = NBLK - 1;
    constexpr int RS = blk_row_stride(NBLK);
    float z[NBLK][4];
#pragma unroll
    for (int k = 0; k < NBLK; ++k)
#pragma unroll
        for (int c = 0; c < 4; ++c) z[k][c] = 0.f;
    {
        const float* colr = xs + 16 * K + r;  // column r of the staged L_KK
        const float nmy = -myinv_last;
        float mt[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) mt[j] = colr[j * RS] * nmy;
        float s = x[K] * myinv_last;
        diag_bwd(s, mt, blk_live<NBLK, FULL>(n, K));
        x[K] = s;
#pragma unroll
        for (int j = 0; j < K; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) z[j][c] = fmaf(T[BI(K, j)][c], x[K], z[j][c]);
    }
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
        sum_row16(z[k]);
        if (SUB) {
            float col[16];
            const float myinv = recip(diag_cols(T[BI(k, k)], col, xs, q, r)), nmy = -myinv;
#pragma unroll
            for (int j = 0; j < 16; ++j) col[j] *= nmy;
            x[k] = (x[k] - c_to_r(z[k], r)) * myinv;
            diag_bwd(x[k], col, 16);
            continue;  // block 0, the last to be solved
        }
        float yc[4];
        r_to_c(x[k], yc, q);
        float part = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) part = fmaf(lt[k * 16 * kXS + (4 * q + c) * kXS + r], yc[c] - z[k][c], part);
        x[k] = sum_rows4(part);
#pragma unroll
        for (int j = 0; j < k; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) z[j][c] = fmaf(T[BI(k, j)][c], x[k], z[j][c]);
    }
}

// L x = b (FWD) and / or L^T x = b (BWD) for one right-hand side in x; T: L in T
// layout (diagonal blocks with a zero strict upper part, identity rows past n).
// KEEP: see diag_keep_fwd.
template <int NBLK, bool FULL, bool FWD, bool BWD, bool KEEP>
GLASS_DEV void blk_solve1(const f4_t (&T)[NBLK * (NBLK + 1) / 2], float (&x)[NBLK], int n, float* xs, int q, int r) {
    if (FWD) {
        float p[NBLK];  // pending sum_j L_kj x_j of block row k, split over the rows q
#pragma unroll
        for (int k = 0; k < NBLK; ++k) p[k] = 0.f;
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            float a[16];
            const float myinv = recip(diag_rows(T[BI(k, k)], a, xs, q, r)), nmy = -myinv;
            if (!KEEP) {
#pragma unroll
                for (int j = 0; j < 16; ++j) a[j] *= nmy;  // -L_rj / L_rr
            }
            blk_fwd_step<NBLK, KEEP>(T, k, a, myinv, x, p, q, blk_live<NBLK, FULL>(n, k));
        }
    }
    if (BWD) blk_bwd1<NBLK, FULL, KEEP>(T, x, xs, n, q, r);
}

// One problem: factor (POTRF, POSV) or take L as given (POTRS), then solve.
// op: 0 POTRF, 1 POSV, 2 POTRS, 5 and 6 these two with 2..4 right-hand sides
// (blk_solve4), 4 POSV with one right-hand side (the factorization of op 1
// with VALU substitutions on the factor in registers: each forward step runs
// inside its factorization step with the block inverse's coefficients, the
// backward pass of blk_bwd1_posv after it on the inverses the panels used; no
// inverse of the last diagonal block and no block transposes).  Every op forms
// the diagonal blocks' inverses with tri_inverse_l on lane-local coefficients:
// after a factorization from the rows of the staged block row with their
// diagonal cleared, for the solves from rows read without it.  Ai is A (L for
// the solves), Bi the problem's [n][nrhs] right-hand sides; L goes to Ag and
// the solution to Bg, which are Ai and Bi themselves for a call in place.  SUB
// (orders up to kBlkSubstMaxN): the panel under the first diagonal block is
// factored with it (diag_factor_rows) instead of by its inverse.  xs: the wavefront's LDS, kBlkRegionFloats (op 4: blk_posv1_floats(NBLK)).
// Returns info (0 for the solves); a failed factorization leaves B untouched
// (out of place: copies it).
template <int NBLK, int OP, bool FULL, bool SUB>
GLASS_DEV int blk_one(const float* Ai, float* Ag, const float* Bi, float* Bg, int n, int nrhs, float* xs, int lane) {
    constexpr int NT = NBLK * (NBLK + 1) / 2;
    constexpr bool FACTOR = OP != 2 && OP != 6, THIN = OP >= 5;
    constexpr bool MFMA_SOLVE = OP != 0 && OP != 4;
    static_assert(!SUB || (NBLK == 2 && !FULL), "orders 17 .. 24");
    const int q = lane >> 4, r = lane & 15;
    f4_t T[NT];
    // op 4: the right-hand side, loaded with A, and the forward substitution's
    // pending sums; step k of the substitution runs inside factorization step k
    float x1[NBLK], p1[NBLK], myinv_last = 1.f;
    float* lt = xs + 16 * blk_row_stride(NBLK);  // op 4: L_kk^{-1} of the blocks k < NBLK - 1
    if (OP == 4 && FULL) blk_x_load<NBLK, FULL>(x1, Bi, n, r);
    blk_load<NBLK, FULL>(T, Ai, n, q, r);
    if (OP == 4) {
        if (!FULL) blk_x_load<NBLK, FULL>(x1, Bi, n, r);
#pragma unroll
        for (int k = 0; k < NBLK; ++k) p1[k] = 0.f;
    }
    f4_t linv[NBLK];
    int inf = 0;
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
        // Block row k is final once its diagonal block is factored, and is
        // staged in LDS at once (its rows then serve the inverse, and no longer
        // need registers).  On three or four tiles per side it is stored while
        // the matrix cores run the panel products (3 % on POTRF / POSV n = 64 x
        // 4096, whose waves are bound by this chain); on two tiles, memory-bound
        // at large batches, and for the last block it goes out first.
        const bool early = NBLK < 3 || k + 1 == NBLK;
        const int live = blk_live<NBLK, FULL>(n, k);
        constexpr int RS = blk_row_stride(NBLK);
        float m[16], myinv = 1.f;
        if (FACTOR) {
            int f = 0;
            if (SUB && k == 0)
                diag_factor_rows(T[0], T[BI(1, 0)], f, myinv, q, r);
            else
                diag_factor(T[BI(k, k)], f, myinv, q, r, live);
            if (inf == 0 && f != 0) inf = 16 * k + f;
            stage_block_row<NBLK>(T, k, xs, q, r);
            if (early) {
                block_row_store<NBLK, FULL>(Ag, k, n, xs, lane);
                wave_sync();
            }
        } else {
            myinv = recip(diag_rows(T[BI(k, k)], m, xs, q, r));
        }
        // The coefficients -L_rj / L_rr of the block's substitutions (its
        // inverse; op 4's forward step): the rows with their diagonal entry
        // cleared, from the staged block row after a factorization, as they
        // come for the solves.
        const bool need_inv = MFMA_SOLVE || (!SUB && k + 1 < NBLK);
        if (need_inv || OP == 4) {
            if (FACTOR) {
                if (early)
                    staged_rows_zero_diag<RS, false>(m, xs + 16 * k, r);
                else
                    staged_rows_zero_diag<RS, true>(m, xs + 16 * k, r);
            }
            const float nmy = -myinv;
#pragma unroll
            for (int j = 0; j < 16; ++j) m[j] *= nmy;
        }
        if (need_inv) {
            linv[k] = tri_inverse_l(m, myinv, q, r, live);
            if (OP == 4) *reinterpret_cast<f4_t*>(lt + k * 16 * kXS + r * kXS + 4 * q) = linv[k];
        }
        if (OP == 4 && k + 1 == NBLK) myinv_last = myinv;
        if (FACTOR) {
#pragma unroll
            for (int i = k + 1; i < NBLK; ++i)
                if (!SUB) T[BI(i, k)] = mma(linv[k], T[BI(i, k)], zero4());
            if (!early) {
                block_row_store<NBLK, FULL>(Ag, k, n, xs, lane);
                wave_sync();
            }
#pragma unroll
            for (int j = k + 1; j < NBLK; ++j) {
                const f4_t nq = neg4(T[BI(j, k)]);
#pragma unroll
                for (int i = j; i < NBLK; ++i) T[BI(i, j)] = mma(nq, T[BI(i, k)], T[BI(i, j)]);
            }
            // op 4: forward step k (needs this step's panel L_ik), on VALU
            // while the matrix cores run the trailing products
            if (OP == 4) blk_fwd_step<NBLK, false>(T, k, m, myinv, x1, p1, q, live);
        }
    }
    if (FACTOR && OP != 0 && inf != 0 && Bi != Bg) {  // a failed factorization passes B through
        for (int g = lane; g < n * nrhs; g += 64) Bg[g] = Bi[g];
    }
    if (OP == 4) {
        if (inf == 0) {
            blk_bwd1_posv<NBLK, FULL, SUB>(T, x1, myinv_last, lt, xs, n, q, r);
            blk_x_store<NBLK, FULL>(x1, Bg, n, q, r);
        }
        return inf;
    }
    if (OP == 0 || inf != 0) return inf;
    // off-diagonal blocks of L, negated: the forward pass subtracts L_kj Y_j
#pragma unroll
    for (int k = 1; k < NBLK; ++k)
#pragma unroll
        for (int j = 0; j < k; ++j) T[BI(k, j)] = neg4(T[BI(k, j)]);
    if (THIN) {
        float y[NBLK];
        blk_solve4<NBLK>(T, linv, y, Bi, Bg, n, nrhs, xs, q, r);
        return 0;
    }
    for (int cb = 0; cb < nrhs; cb += 16) {
        f4_t Y[NBLK];
        rhs_load<NBLK, FULL>(Y, Bi, n, nrhs, cb, q, r);
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            f4_t s = Y[k];
#pragma unroll
            for (int j = 0; j < k; ++j) s = mma(T[BI(k, j)], Y[j], s);
            Y[k] = mma(linv[k], s, zero4());
        }
        BwdBlk<NBLK, NBLK - 1>::run(T, linv, Y, xs, q, r);
        rhs_store<NBLK, FULL>(Y, Bg, n, nrhs, cb, q, r);
    }
    return 0;
}

}  // namespace glass
