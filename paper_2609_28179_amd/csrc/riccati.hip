// riccati.hip -- fused LQR feedback gain K = (R + B^T P B)^{-1} B^T P A
// (Sec. III-B names it as a fused composition of GEMM and solve primitives;
// Sec. IV-E measures fused against a chain of separate launches).
//
// Every intermediate stays on chip.  At wave scope (one wavefront per
// problem, P problems per workgroup) riccati_mfma; at sub-wave scope
// riccati_seg; at thread scope riccati_thread.
//
// riccati_thread (thread scope, nx <= 8, nu <= 4): one problem per lane.  A
// lane loads its own P, B, R and A (every load issued before any is used),
// forms PB = P B, the lower triangle of S = R + B^T PB and the columns of
// T = PB^T A in VGPRs, factors S with the thread-scope Cholesky and solves
// S k = t for each column of T; its problem's K goes out in one run of stores.
//
// riccati_seg (sub-wave scope, nx <= 16, nu <= 8): four problems per
// wavefront, one per 16-lane row; lane i of a row holds row i of P, B and R
// and column i of A.  PB's row i takes B's rows as DPP row broadcasts;
// S = R + B^T PB sums each lane's outer product B_i PB_i^T over the row with
// four DPP exchanges; S is factored with the segment Cholesky (lane a holds
// row a of L); column i of T = PB^T A takes PB's rows as broadcasts, and
// lane i solves L L^T k = t for its own column of K with L's entries as
// broadcasts.  Every cross-lane move stays inside a 16-lane row.  The operands
// come by buffer loads at one per-lane offset per operand and a scalar row
// offset, and S's rows are picked from the sums by one select per entry; with
// 64-bit addresses and selects per element (12 x 4: 322 VALU instructions per
// wavefront, 180 now) 65,536 problems took (12, 4) 20.7 us against 17.2 (its
// bytes take 18.4 at the rate of a copy), (16, 4) 31.5 against 29.9, (16, 8) 50.6 against
// 39.8 (38.3), (14, 7) 42.7 against 41.2 (29.3).
//
// riccati_mfma (every size): every product on the matrix cores, operands read
// once by branch-free buffer loads (device_common.hpp), in the blocked layouts
// of chol_blk.hpp (nx padded to 16-row blocks; nu <= 16 is one block).  With B_k in accumulator layout (lane (q, r) holds B[16k+4q+c][r])
// the products chain without data movement:
//   PB_i = sum_k P_ik B_k                 P_ik loaded row-wise (T layout)
//   S    = R + sum_i B_i^T PB_i           B_i's registers are the T layout of B_i^T
//   T_j  = sum_i PB_i^T A_ij              PB_i's registers are the T layout of PB_i^T
//                                         (B^T P = (P B)^T: P is symmetric)
//   K_j  = L^{-T} L^{-1} T_j              S = L L^T factored as a diagonal block
// S's padded diagonal (orders nu..15) is the identity, so the solve runs on a
// full 16 x 16 block while the factorization and the inverse stop after nu
// rounded up to 4, 8 or 16 pivots (the rest would find unit pivots and zero
// coefficients).
#include <type_traits>

#include "device_common.hpp"
#include "glass_internal.hpp"
#include "chol_device.hpp"
#include "chol_blk.hpp"
#include "riccati.hpp"

namespace glass {
namespace {

// NUB: nu rounded up to 4, 8 or 16.  S is the identity past nu, so its
// factorization and inverse run NUB pivot steps instead of 16.  All of P and
// the first block column of A are in flight before the chain that factors
// S.  With guarded element-wise loads at the point of use, 16,384 problems took
// (20, 3) 28.4 us against 22.3 now, (27, 6) 35.6 against 27.6, (41, 9) 104
// against 62.5, (48, 16) 97.6 against 84.7, and (32, 8) at 65,536 144.5 against
// 131.9.  With T = ceil(nx / 16) tiles of states the products are T^2 (P B), T (S) and
// T (T + 2) (T_j and its two solves) blocks of 16 x 16 x 16, four matrix
// instructions each: 14 blocks at two tiles, a third of them padding, about 12 us of
// matrix-core time at (27, 6) x 16,384.  The rest is the serial part between: S
// through LDS into row form, its factorization and its inverse.
template <int NXB, int NUB>
__global__ void __launch_bounds__(512) riccati_mfma(int nx, int nu, int batch, const float* __restrict__ A,
                                                    const float* __restrict__ B, const float* __restrict__ P,
                                                    const float* __restrict__ R, float* __restrict__ K,
                                                    int32_t* __restrict__ info) {
    extern __shared__ float lds[];
    const int w = wave_index(), lane = threadIdx.x & 63, q = lane >> 4, r = lane & 15;
    const long long p = (long long)blockIdx.x * (blockDim.x >> 6) + w;
    if (p >= batch) return;
    float* xs = lds + (size_t)w * kRiccatiRegionFloats;
    const float* Ap = A + p * nx * nx;
    const float* Bp = B + p * nx * nu;
    const float* Pp = P + p * nx * nx;
    const float* Rp = R + p * nu * nu;
    const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(Ap, (uint32_t)(nx * nx) * 4u);
    const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(Bp, (uint32_t)(nx * nu) * 4u);
    const __amdgpu_buffer_rsrc_t rp = buffer_rsrc(Pp, (uint32_t)(nx * nx) * 4u);
    const __amdgpu_buffer_rsrc_t rr = buffer_rsrc(Rp, (uint32_t)(nu * nu) * 4u);
    f4_t Bb[NXB], Pf[NXB][NXB], Rf[1];
    tile_col_elems<NXB>(Bb, rb, nu, nx, r, q);
#pragma unroll
    for (int i = 0; i < NXB; ++i) tile_row_pieces<NXB>(Pf[i], rp, nx, nx, 16 * i + r, q);
    tile_col_elems<1>(Rf, rr, nu, nu, r, q);
    f4_t PB[NXB];
#pragma unroll
    for (int i = 0; i < NXB; ++i) {
        f4_t acc = zero4();
#pragma unroll
        for (int k = 0; k < NXB; ++k) acc = mma(Pf[i][k], Bb[k], acc);
        PB[i] = acc;
    }
    // the first block column of A, in flight behind the factorization of S
    f4_t Af[2][NXB];
    tile_col_elems<NXB>(Af[0], ra, nx, nx, r, q);
    // S = R + B^T P B in accumulator layout, its padded rows and columns set to
    // the identity after the products (an infinity in P B times a padded zero of
    // B is no zero)
    f4_t S = Rf[0];
#pragma unroll
    for (int i = 0; i < NXB; ++i) S = mma(Bb[i], PB[i], S);
#pragma unroll
    for (int e = 0; e < 4; ++e) S[e] = 4 * q + e < nu && r < nu ? S[e] : 4 * q + e == r ? 1.f : 0.f;
    // rows of S to the lanes: lane (q, r) holds row r of S after the exchange
#pragma unroll
    for (int e = 0; e < 4; ++e) xs[(4 * q + e) * kXS + r] = S[e];
    wave_sync();
    float a[16];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const f4_t v = *reinterpret_cast<const f4_t*>(xs + r * kXS + 4 * u);
#pragma unroll
        for (int e = 0; e < 4; ++e) a[4 * u + e] = v[e];
    }
    wave_sync();
    int f = 0;
    float myinv = 1.f;
    {
        float as[NUB];  // the first NUB columns; rows from NUB on are identity rows
#pragma unroll
        for (int c = 0; c < NUB; ++c) as[c] = a[c];
        SegStep<16, NUB, 0>::run(as, f, myinv);
#pragma unroll
        for (int c = 0; c < 16; ++c) a[c] = c < NUB ? (c <= r ? as[c] : 0.f) : (c == r ? 1.f : 0.f);
    }
    if (info && lane == 0) info[p] = f;
    if (f != 0) return;  // K is not written for an indefinite S
    float m[16];  // the rows again, diagonal entry cleared, scaled by -1 / L_rr
    rows_zero_diag<kXS>(a, m, xs, q, r);
#pragma unroll
    for (int j = 0; j < 16; ++j) m[j] *= -myinv;
    const f4_t linv = tri_inverse_l(m, myinv, q, r, NUB);  // L^{-1} in T layout
    f4_t lt[4];
    lt[0] = linv;
    transpose_blocks<1>(lt, xs, q, r);  // lt[0]: L^{-T} in T layout
    const __amdgpu_buffer_rsrc_t rk = buffer_rsrc(K + p * nu * nx, (uint32_t)(nu * nx) * 4u);
#pragma unroll
    for (int j = 0; j < NXB; ++j) {
        if (j + 1 < NXB) tile_col_elems<NXB>(Af[(j + 1) & 1], ra, nx, nx, 16 * (j + 1) + r, q);
        f4_t t = zero4();
#pragma unroll
        for (int i = 0; i < NXB; ++i) t = mma(PB[i], Af[j & 1][i], t);
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = 4 * q + e < nu ? t[e] : 0.f;  // the padded rows, likewise
        const f4_t kj = mma(lt[0], mma(linv, t, zero4()), zero4());  // L^{-T} (L^{-1} T_j)
        const int col = 16 * j + r;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(kj[e]), rk,
                                                  4 * q + e < nu && col < nx ? ((4 * q + e) * nx + col) * 4 : kOob, 0, 0);
    }
}

// L consecutive floats of one lane's problem at p, in accesses as wide as the
// problem's size allows when `wide` (the batch's base pointer is 16-byte
// aligned, so problem p starts at a multiple of L floats from it).
template <int L>
GLASS_DEV void lane_load(float (&v)[L], const float* __restrict__ p, bool wide) {
    constexpr int AL = L % 4 == 0 ? 4 : L % 2 == 0 ? 2 : 1;
    if (AL == 4 && wide) {
#pragma unroll
        for (int t = 0; t < L / 4; ++t) {
            const f4_t x = *reinterpret_cast<const f4_t*>(p + 4 * t);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * t + e] = x[e];
        }
    } else if (AL == 2 && wide) {
#pragma unroll
        for (int t = 0; t < L / 2; ++t) {
            const float2 x = *reinterpret_cast<const float2*>(p + 2 * t);
            v[2 * t] = x.x;
            v[2 * t + 1] = x.y;
        }
    } else {
#pragma unroll
        for (int t = 0; t < L; ++t) v[t] = p[t];
    }
}

template <int L>
GLASS_DEV void lane_store(float* __restrict__ p, const float (&v)[L], bool wide) {
    constexpr int AL = L % 4 == 0 ? 4 : L % 2 == 0 ? 2 : 1;
    if (AL == 4 && wide) {
#pragma unroll
        for (int t = 0; t < L / 4; ++t) *reinterpret_cast<f4_t*>(p + 4 * t) = f4_t{v[4 * t], v[4 * t + 1], v[4 * t + 2], v[4 * t + 3]};
    } else if (AL == 2 && wide) {
#pragma unroll
        for (int t = 0; t < L / 2; ++t) *reinterpret_cast<float2*>(p + 2 * t) = make_float2(v[2 * t], v[2 * t + 1]);
    } else {
#pragma unroll
        for (int t = 0; t < L; ++t) p[t] = v[t];
    }
}

template <int NX, int NU>
__global__ void __launch_bounds__(512) riccati_thread(int batch, const float* __restrict__ A,
                                                      const float* __restrict__ B, const float* __restrict__ P,
                                                      const float* __restrict__ R, float* __restrict__ K,
                                                      int32_t* __restrict__ info, bool wide) {
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= batch) return;
    float pm[NX * NX], b[NX * NU], r[NU * NU], a[NX * NX];
    lane_load<NX * NX>(pm, P + p * (NX * NX), wide);
    lane_load<NX * NU>(b, B + p * (NX * NU), wide);
    lane_load<NU * NU>(r, R + p * (NU * NU), wide);
    lane_load<NX * NX>(a, A + p * (NX * NX), wide);
    float pb[NX * NU];  // P B
#pragma unroll
    for (int i = 0; i < NX; ++i)
#pragma unroll
        for (int j = 0; j < NU; ++j) {
            float s = 0.f;
#pragma unroll
            for (int k = 0; k < NX; ++k) s = fmaf(pm[i * NX + k], b[k * NU + j], s);
            pb[i * NU + j] = s;
        }
    float sl[NU * (NU + 1) / 2];  // lower triangle of S = R + B^T (P B)
#pragma unroll
    for (int i = 0; i < NU; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            float s = r[i * NU + j];
#pragma unroll
            for (int k = 0; k < NX; ++k) s = fmaf(b[k * NU + i], pb[k * NU + j], s);
            sl[TI(i, j)] = s;
        }
    float dinv[NU];
    const int inf = tri_potrf<NU>(sl, dinv);
    if (info) info[p] = inf;
    if (inf != 0) return;
    float kk[NU * NX];
#pragma unroll
    for (int c = 0; c < NX; ++c) {
        float y[NU];  // column c of T = (P B)^T A = B^T P A (P symmetric)
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            float s = 0.f;
#pragma unroll
            for (int k = 0; k < NX; ++k) s = fmaf(pb[k * NU + i], a[k * NX + c], s);
            y[i] = s;
        }
        tri_fwd<NU>(sl, dinv, y);
        tri_bwd<NU>(sl, dinv, y);
#pragma unroll
        for (int i = 0; i < NU; ++i) kk[i * NX + c] = y[i];
    }
    lane_store<NU * NX>(K + p * (NU * NX), kk, wide);
}

template <int CTRL>
GLASS_DEV float row_dpp(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, false));
}
// lane K of the 16-lane row (row_newbcast)
template <int K>
GLASS_DEV float row_bcast(float v) {
    return row_dpp<0x150 + K>(v);
}
// the sum over the 16 lanes of a row, the same value in each: pairs, quads
// (quad_perm [1,0,3,2] and [2,3,0,1]), then half rows and rows (row_half_mirror,
// row_mirror); each step adds two equal-order operands, so every lane agrees
GLASS_DEV float row_sum16(float v) {
    v += row_dpp<0xB1>(v);
    v += row_dpp<0x4E>(v);
    v += row_dpp<0x141>(v);
    v += row_dpp<0x140>(v);
    return v;
}

template <int I, int N, class F>
GLASS_DEV void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

template <int NXB, int NUB>
__global__ void __launch_bounds__(512) riccati_seg(int nx, int nu, int batch, const float* __restrict__ A,
                                                   const float* __restrict__ B, const float* __restrict__ P,
                                                   const float* __restrict__ R, float* __restrict__ K,
                                                   int32_t* __restrict__ info) {
    const int lane = threadIdx.x & 63, s = lane >> 4, i = lane & 15;
    const long long p0 = ((long long)blockIdx.x * (blockDim.x >> 6) + wave_index()) * 4;
    if (p0 >= batch) return;
    const long long ps = p0 + s;
    const bool act = ps < batch;
    const bool row = i < nx;
    // The wavefront's problems are adjacent, so one descriptor per operand
    // covers them; a lane past its matrix or the batch gets an offset out of
    // its range and reads 0.  nx > NXB - 4 from 12 states up, so that only the
    // last rows of P and A need a test there.
    const int np = (int)min(4ll, batch - p0);
    const __amdgpu_buffer_rsrc_t rp = buffer_rsrc(P + p0 * nx * nx, (uint32_t)(np * nx * nx) * 4u);
    const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(A + p0 * nx * nx, (uint32_t)(np * nx * nx) * 4u);
    const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(B + p0 * nx * nu, (uint32_t)(np * nx * nu) * 4u);
    const __amdgpu_buffer_rsrc_t rr = buffer_rsrc(R + p0 * nu * nu, (uint32_t)(np * nu * nu) * 4u);
    const int off = row ? (s * nx * nx + i) * 4 : kOob;
    const int offb = row ? (s * nx + i) * nu * 4 : kOob, offr = i < nu ? (s * nu + i) * nu * 4 : kOob;
    float prow[NXB], acol[NXB], brow[NUB], rrow[NUB];
    if (nu == NUB) {  // whole 16-byte pieces
#pragma unroll
        for (int j = 0; j < NUB; j += 4) {
            const f4_t bv = buf_load4(rb, offb, 4 * j);
#pragma unroll
            for (int e = 0; e < 4; ++e) brow[j + e] = bv[e];
        }
#pragma unroll
        for (int j = 0; j < NUB; j += 4) {
            const f4_t rv = buf_load4(rr, offr, 4 * j);
#pragma unroll
            for (int e = 0; e < 4; ++e) rrow[j + e] = rv[e];
        }
    } else {
#pragma unroll
        for (int j = 0; j < NUB; ++j) {
            brow[j] = buf_load1(rb, j < nu ? offb : kOob, 4 * j);
            rrow[j] = buf_load1(rr, j < nu ? offr : kOob, 4 * j);
        }
    }
#pragma unroll
    for (int k = 0; k < NXB; ++k)  // P symmetric: row i read as column i (consecutive lanes, consecutive floats)
        prow[k] = buf_load1(rp, (NXB > 8 && k < NXB - 3) || k < nx ? off : kOob, k * nx * 4);
#pragma unroll
    for (int k = 0; k < NXB; ++k)
        acol[k] = buf_load1(ra, (NXB > 8 && k < NXB - 3) || k < nx ? off : kOob, k * nx * 4);
    // row i of P B; the broadcasts are folded into the FMAs (one DPP op each,
    // so no broadcast value is held), after the wait states their sources need
    float pb[NUB];
#pragma unroll
    for (int j = 0; j < NUB; ++j) {
        pb[j] = 0.f;
        asm volatile("s_nop 1" : "+v"(brow[j]));
    }
    static_for<0, NXB>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
#pragma unroll
        for (int j = 0; j < NUB; ++j) fmac_bcast<k>(pb[j], brow[j], prow[k]);
    });
    // S = R + B^T P B: lane i contributes B_i PB_i^T; row i of S to lane i
    // (identity rows from nu to NUB, zero rows past NUB)
    float srow[NUB];
#pragma unroll
    for (int c = 0; c < NUB; ++c) srow[c] = 0.f;
#pragma unroll
    for (int a = 0; a < NUB; ++a)
#pragma unroll
        for (int c = 0; c <= a; ++c) {
            const float v = row_sum16(brow[a] * pb[c]);
            srow[c] = i == a ? v : srow[c];
            if (c != a) srow[a] = i == c ? v : srow[a];
        }
#pragma unroll
    for (int c = 0; c < NUB; ++c) srow[c] += rrow[c];
    if (nu != NUB) {  // wave-uniform; set, as an infinity in P B times a padded zero of B is no zero
#pragma unroll
        for (int c = 0; c < NUB; ++c) srow[c] = i < nu && c < nu ? srow[c] : i == c ? 1.f : 0.f;
    }
    int f = 0;
    float myinv = 1.f;
    SegStep<16, NUB, 0>::run(srow, f, myinv);
    if (act && i == 0 && info) info[ps] = f;
    if (f != 0) return;  // the row's problem is indefinite (or past the batch): K is not written
    // column i of T = (P B)^T A
    float t[NUB];
#pragma unroll
    for (int a = 0; a < NUB; ++a) {
        t[a] = 0.f;
        asm volatile("s_nop 1" : "+v"(pb[a]));
    }
    static_for<0, NXB>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
#pragma unroll
        for (int a = 0; a < NUB; ++a) fmac_bcast<k>(t[a], pb[a], acol[k]);
    });
    if (nu != NUB) {
#pragma unroll
        for (int a = 0; a < NUB; ++a) t[a] = a < nu ? t[a] : 0.f;  // the padded rows of T, likewise
    }
    // L's strictly lower entries and 1 / L_aa as broadcasts, then L L^T k = t
    float lo[NUB][NUB], inv[NUB];
    static_for<0, NUB>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        inv[a] = row_bcast<a>(myinv);
#pragma unroll
        for (int b = 0; b < a; ++b) lo[a][b] = row_bcast<a>(srow[b]);
    });
#pragma unroll
    for (int a = 0; a < NUB; ++a) {
        float v = t[a];
#pragma unroll
        for (int b = 0; b < a; ++b) v = fmaf(-lo[a][b], t[b], v);
        t[a] = v * inv[a];
    }
#pragma unroll
    for (int a = NUB - 1; a >= 0; --a) {
        float v = t[a];
#pragma unroll
        for (int b = a + 1; b < NUB; ++b) v = fmaf(-lo[b][a], t[b], v);
        t[a] = v * inv[a];
    }
    if (act && row) {
        float* Kp = K + ps * nu * nx + i;
#pragma unroll
        for (int a = 0; a < NUB; ++a)
            if (a < nu) Kp[a * nx] = t[a];
    }
}

}  // namespace

static_assert(kRiccatiRegionFloats == 16 * kXS, "one exchange block");

int launch_riccati(int nx, int nu, int batch, int pack, const float* A, const float* B, const float* P,
                   const float* R, float* K, int32_t* info, void* stream) {
    (void)hipGetLastError();  // a stale error of an earlier runtime call is not ours
    hipStream_t st = (hipStream_t)stream;
    dim3 grid((unsigned)((batch + pack - 1) / pack)), block(64 * pack);
    const size_t lds = sizeof(float) * (size_t)kRiccatiRegionFloats * pack;
    const int nub = nu <= 4 ? 4 : nu <= 8 ? 8 : 16;
    switch ((nx + 15) / 16 * 100 + nub) {
#define RM(NXB, NUB)                                                                                            \
    case NXB * 100 + NUB:                                                                                       \
        hipLaunchKernelGGL((riccati_mfma<NXB, NUB>), grid, block, lds, st, nx, nu, batch, A, B, P, R, K, info); \
        break;
#define RM_NX(NXB) RM(NXB, 4) RM(NXB, 8) RM(NXB, 16)
        RM_NX(1) RM_NX(2) RM_NX(3) RM_NX(4)
#undef RM_NX
#undef RM
    default: return (int)hipErrorInvalidValue;
    }
    return (int)hipGetLastError();
}

int launch_riccati_seg(int nx, int nu, int batch, int pack, const float* A, const float* B, const float* P,
                       const float* R, float* K, int32_t* info, void* stream) {
    (void)hipGetLastError();  // a stale error of an earlier runtime call is not ours
    hipStream_t st = (hipStream_t)stream;
    const int per_wg = 4 * pack;
    dim3 grid((unsigned)((batch + per_wg - 1) / per_wg)), block(64 * pack);
    // states rounded up to 8, 12 or 16 (rows of P, B and A loaded and multiplied), inputs to 4 or 8
    const int nxb = nx <= 8 ? 8 : nx <= 12 ? 12 : 16, nub = nu <= 4 ? 4 : 8;
#define RS(NXB, NUB)                                                                                       \
    if (nxb == NXB && nub == NUB) {                                                                        \
        hipLaunchKernelGGL((riccati_seg<NXB, NUB>), grid, block, 0, st, nx, nu, batch, A, B, P, R, K, info); \
        return (int)hipGetLastError();                                                                     \
    }
    RS(8, 4) RS(8, 8) RS(12, 4) RS(12, 8) RS(16, 4) RS(16, 8)
#undef RS
    return (int)hipErrorInvalidValue;
}

int launch_riccati_thread(int nx, int nu, int batch, int pack, const float* A, const float* B, const float* P,
                          const float* R, float* K, int32_t* info, void* stream) {
    (void)hipGetLastError();  // a stale error of an earlier runtime call is not ours
    hipStream_t st = (hipStream_t)stream;
    const int threads = 64 * pack;
    dim3 grid((unsigned)((batch + threads - 1) / threads)), block(threads);
    auto al16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
    const bool wide = al16(A) && al16(B) && al16(P) && al16(R) && al16(K);
#define RT(NX, NU)                                                                                          \
    if (nx == NX && nu == NU) {                                                                             \
        hipLaunchKernelGGL((riccati_thread<NX, NU>), grid, block, 0, st, batch, A, B, P, R, K, info, wide); \
        return (int)hipGetLastError();                                                                      \
    }
#define RT_NX(NX) RT(NX, 1) RT(NX, 2) RT(NX, 3) RT(NX, 4)
    RT_NX(1) RT_NX(2) RT_NX(3) RT_NX(4) RT_NX(5) RT_NX(6) RT_NX(7) RT_NX(8)
#undef RT_NX
#undef RT
    return (int)hipErrorInvalidValue;
}

}  // namespace glass
