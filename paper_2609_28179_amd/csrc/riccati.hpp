// riccati.hpp -- launch interface of the thread- and sub-wave-scope forms of
// the fused LQR gain (riccati.hip) and its default placement; the wave-scope
// form is declared with the other launchers in glass_internal.hpp.
#pragma once
#include "glass_internal.hpp"

namespace glass {

// Thread scope: one problem per lane with every operand and intermediate in
// VGPRs, at compile-time orders up to these.
constexpr int kRiccatiThreadMaxNx = 8;
constexpr int kRiccatiThreadMaxNu = 4;

inline bool riccati_thread_ok(int nx, int nu) {
    return nx >= 1 && nu >= 1 && nx <= kRiccatiThreadMaxNx && nu <= kRiccatiThreadMaxNu;
}

// Sub-wave scope: four problems per wavefront, one per 16-lane row.
constexpr int kRiccatiSegMaxNx = 16;
constexpr int kRiccatiSegMaxNu = 8;

inline bool riccati_seg_ok(int nx, int nu) {
    return nx >= 1 && nu >= 1 && nx <= kRiccatiSegMaxNx && nu <= kRiccatiSegMaxNu;
}

// pack wavefronts (4 * pack problems) per workgroup; the caller has checked
// riccati_seg_ok.
int launch_riccati_seg(int nx, int nu, int batch, int pack, const float* A, const float* B, const float* P,
                       const float* R, float* K, int32_t* info, void* stream);

// 64 * pack lanes per workgroup; the caller has checked riccati_thread_ok.
int launch_riccati_thread(int nx, int nu, int batch, int pack, const float* A, const float* B, const float* P,
                          const float* R, float* K, int32_t* info, void* stream);

// Scope and pack without a forced placement.  Thread scope wherever it runs
// (faster at every batch from 16 to 65,536 at (1, 1), (4, 2), (6, 3), (8, 1)
// and (8, 4)).  Otherwise sub-wave scope from the batch where four problems a
// wavefront still fill the chip and its longer chain per wavefront is hidden,
// measured against wave scope: up to nu = 4 from 4096 problems ((12, 4): 4.8
// against 5.4 us at 4096, 20.6 against 38.4 at 65,536, 4.4 against 4.0 at
// 2048); past it from 8192 up to nx = 8 ((8, 8): 11.9 against 19.2 at 16,384),
// from 16,384 up to nx = 12 ((12, 7): 13.1 against 13.9, 34.0 against 42.4 at
// 65,536) and from 32,768 up to nx = 14 ((14, 7): 41.9 against 46.2 at 65,536,
// 14.8 against 14.5 at 16,384); at (16, 8) wave scope stays ahead (46.1
// against 50.7 at 65,536).  Four wavefronts per workgroup from 2048 problems
// (wave scope, (27, 6) x 16,384: 25.7 against 27.6), one below (they spread
// over more compute units).
inline void riccati_default(int nx, int nu, int batch, int* scope, int* pack) {
    *pack = 1;
    if (riccati_thread_ok(nx, nu)) {
        *scope = GLASS_SCOPE_THREAD;
        return;
    }
    const int from = nu <= 4 ? 4096 : nx <= 8 ? 8192 : nx <= 12 ? 16384 : nx <= 14 ? 32768 : 0x7fffffff;
    *scope = riccati_seg_ok(nx, nu) && batch >= from ? GLASS_SCOPE_SUBWAVE : GLASS_SCOPE_WAVE;
    if (batch >= 2048) *pack = 4;
}

}  // namespace glass
