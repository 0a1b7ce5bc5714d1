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
// and (8, 4)).  Otherwise sub-wave scope, against wave scope measured: up to
// nu = 4 at every batch ((12, 4): 3.1 against 3.3 us at 512, 3.9 against 5.3
// at 4096, 17.2 against 37.7 at 65,536); past it, where its chain per
// wavefront is the longer one, from the batch that hides it, 4096 up to nx =
// 12 ((8, 8): 4.9 against 5.6, and 4.5 against 3.6 at 1024; (12, 8): 5.8
// against 5.7) and 8192 above ((14, 7): 8.5 against 8.8, and 6.4 against 6.1
// at 4096; (16, 8): 8.8 against 8.8, 39.8 against 45.5 at 65,536).  Four
// wavefronts per workgroup from 2048 problems (wave scope, (27, 6) x 16,384:
// 25.7 against 27.6), one below (they spread over more compute units).
inline void riccati_default(int nx, int nu, int batch, int* scope, int* pack) {
    *pack = 1;
    if (riccati_thread_ok(nx, nu)) {
        *scope = GLASS_SCOPE_THREAD;
        return;
    }
    const int from = nu <= 4 ? 1 : nx <= 12 ? 4096 : 8192;
    *scope = riccati_seg_ok(nx, nu) && batch >= from ? GLASS_SCOPE_SUBWAVE : GLASS_SCOPE_WAVE;
    if (batch >= 2048) *pack = 4;
}

}  // namespace glass
