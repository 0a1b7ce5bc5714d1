// chol_blk.hip -- batched wave-scope kernels of POTRF / POSV / POTRS / TRSV
// for orders 17..64 on the blocked routines of chol_blk.hpp (one problem per
// wavefront; 2, 3 or 4 tiles of 16 per side): the MFMA kernel for the
// factorizations and multi-column solves, the VALU substitution for one
// right-hand side.
#include "chol_blk.hpp"

namespace glass {
namespace {

// op: 0 POTRF, 1 POSV, 2 POTRS (five right-hand sides or more), 4 POSV with one, 5
// POSV and 6 POTRS with two to four (POTRS with one and TRSV: chol_blk_solve1).
// SUB: orders up to kBlkSubstMaxN.
template <int NBLK, int OP, bool FULL, bool SUB>
__global__ void __launch_bounds__(512) chol_blk(int n, int nrhs, int batch, const float* Ai, float* A,
                                                const float* Bi, float* B, int32_t* __restrict__ info) {
    extern __shared__ float lds[];
    // POTRF on whole 16 x 16 tiles above order 32 (n = 48, 64) is write-bound
    // and runs 1.5-3 % faster at 4 waves per SIMD than at the 5-7 its
    // registers allow (at n = 40 the extra waves pay instead): reserving VGPRs
    // up to v103 makes the allocation 104 registers, which caps the occupancy.
    if (OP == 0 && FULL && NBLK >= 3) asm volatile("" ::: "v103");
    // POSV with one right-hand side likewise: n = 64 x 65,536 368 us at four
    // waves, 371 at five; n = 41 x 16,384 56.5 at six, 58.2 at eight.
    if (OP == 4 && FULL && NBLK == 4) asm volatile("" ::: "v103");
    if (OP == 4 && !FULL && NBLK == 3) asm volatile("" ::: "v79");
    const int w = wave_index(), lane = threadIdx.x & 63;
    const long long p = (long long)blockIdx.x * (blockDim.x >> 6) + w;
    if (p >= batch) return;
    const int nr = OP == 4 ? 1 : nrhs;
    constexpr int region = OP == 4 ? blk_posv1_floats(NBLK) : kBlkRegionFloats;
    const int inf = blk_one<NBLK, OP, FULL, SUB>(Ai + p * n * n, A + p * n * n, OP == 0 ? nullptr : Bi + p * n * nr,
                                            OP == 0 ? nullptr : B + p * n * nr, n, nrhs,
                                            lds + (size_t)w * region, lane);
    if (OP != 2 && OP != 6 && info && lane == 0) info[p] = inf;
}

// One right-hand side (TRSV; POTRS with nrhs = 1) on VALU, no inverses:
// FWD solves L y = b, BWD L^T x = y.  L is read, B[batch][n] overwritten.
template <int NBLK, bool FULL, bool FWD, bool BWD>
__global__ void __launch_bounds__(512) chol_blk_solve1(int n, int batch, const float* __restrict__ L,
                                                       float* __restrict__ B) {
    extern __shared__ float lds[];
    const int w = wave_index(), lane = threadIdx.x & 63;
    const long long p = (long long)blockIdx.x * (blockDim.x >> 6) + w;
    if (p >= batch) return;
    const int q = lane >> 4, r = lane & 15;
    f4_t T[NBLK * (NBLK + 1) / 2];
    float x[NBLK];
    // On whole tiles b is loaded ahead of L (the first diagonal step waits for
    // it: TRSV transposed n = 64 x 256 3.22 us against 3.42), on cut tiles behind
    // it (n = 33 x 16 2.52 us against 2.70).  Computing the two addresses here makes
    // the schedule mask the last diagonal block behind the first substitution step
    // instead of waiting for every tile ahead of it (POTRS n = 53 x 1024 6.46 us
    // against 6.82).
    if (FULL) blk_x_load<NBLK, FULL>(x, B + p * n, n, r);
    blk_load<NBLK, FULL>(T, L + p * n * n, n, q, r);
    float* bg = B + p * n;
    float* xs = lds + (size_t)w * kBlkSolve1Floats;
    if (!FULL) blk_x_load<NBLK, FULL>(x, bg, n, r);
    blk_solve1<NBLK, FULL, FWD, BWD, false>(T, x, n, xs, q, r);
    // One direction leaves the unknowns before a non-finite entry of b finite: such
    // a problem is solved again, from its operands, by the form that keeps them
    // (in every problem it took TRSV n = 22 x 65,536 from 27 us to 31).
    if (FWD != BWD) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < NBLK; ++k) s += fabsf(x[k]);
        if (__builtin_expect(__ballot(!(s < INFINITY)) != 0, 0)) {
            blk_load<NBLK, FULL>(T, L + p * n * n, n, q, r);
            blk_x_load<NBLK, FULL>(x, bg, n, r);
            blk_solve1<NBLK, FULL, FWD, BWD, true>(T, x, n, xs, q, r);
        }
    }
    blk_x_store<NBLK, FULL>(x, bg, n, q, r);
}

}  // namespace

int launch_chol_blk(const Shape& sh, const Geometry& g, int batch, const float* Ai, float* A, const float* Bi, float* B,
                    int32_t* info, void* stream) {
    (void)hipGetLastError();  // a stale error of an earlier runtime call is not ours
    hipStream_t st = (hipStream_t)stream;
    const int n = sh.n;
    if (n < kBlkMinN || n > kMaxN) return (int)hipErrorInvalidValue;
    const int nblk = n <= 32 ? 2 : n <= 48 ? 3 : 4;
    const bool full =
        n == 16 * nblk && ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(Ai)) & 15) == 0;
    const int op = sh.op == GLASS_OP_POTRF ? 0
                   : sh.op == GLASS_OP_POSV ? (sh.nrhs == 1 ? 4 : sh.nrhs <= 4 ? 5 : 1)
                   : sh.op == GLASS_OP_POTRS ? (sh.nrhs == 1 ? 3 : sh.nrhs <= 4 ? 6 : 2)
                                             : 3;
    dim3 grid((unsigned)g.grid), block(g.threads);
    if (op == 3) {
        const int mode = sh.op == GLASS_OP_POTRS ? 3 : sh.trans == 0 ? 1 : 2;  // 1: L y = b, 2: L^T x = b, 3: both
#define ONE(NBLK, FULL, MODE)                                                                                   \
    if (nblk == NBLK && full == FULL && mode == MODE) {                                                         \
        hipLaunchKernelGGL((chol_blk_solve1<NBLK, FULL, (MODE & 1) != 0, (MODE & 2) != 0>), grid, block,          \
                           g.lds_bytes, st, n, batch, A, B);                                                    \
        return (int)hipGetLastError();                                                                          \
    }
#define ONE_MODES(NBLK, FULL) ONE(NBLK, FULL, 1) ONE(NBLK, FULL, 2) ONE(NBLK, FULL, 3)
        ONE_MODES(2, false) ONE_MODES(2, true) ONE_MODES(3, false) ONE_MODES(3, true) ONE_MODES(4, false)
        ONE_MODES(4, true)
#undef ONE_MODES
#undef ONE
        return (int)hipErrorInvalidValue;
    }
#define BLK(NBLK, OP, FULL, SUB)                                                                               \
    if (nblk == NBLK && op == OP && full == FULL && sub == SUB) {                                              \
        hipLaunchKernelGGL((chol_blk<NBLK, OP, FULL, SUB>), grid, block, g.lds_bytes, st, n, sh.nrhs, batch, Ai, A, \
                           Bi, B, info);                                                                       \
        return (int)hipGetLastError();                                                                         \
    }
#define BLK_OPS(NBLK, FULL, SUB)                                                                               \
    BLK(NBLK, 0, FULL, SUB) BLK(NBLK, 1, FULL, SUB) BLK(NBLK, 2, FULL, SUB) BLK(NBLK, 4, FULL, SUB)            \
    BLK(NBLK, 5, FULL, SUB) BLK(NBLK, 6, FULL, SUB)
    const bool sub = n <= kBlkSubstMaxN;
    BLK_OPS(2, false, true) BLK_OPS(2, false, false) BLK_OPS(2, true, false) BLK_OPS(3, false, false)
    BLK_OPS(3, true, false) BLK_OPS(4, false, false) BLK_OPS(4, true, false)
#undef BLK_OPS
#undef BLK
    return (int)hipErrorInvalidValue;
}

}  // namespace glass
