// Interface between pcmm.hip and pcmm_resident.hip: the MFMA kernel for contractions whose digits fit LDS.
// Host-side declarations only.
#ifndef PCMM_RESIDENT_HPP
#define PCMM_RESIDENT_HPP

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pcmm_host.hpp"

namespace pcmm_resident {

// What one launch needs.  Wp is the plan's packed weights in the layout pack_w_kernel writes; the residues are read as they are,
// their digits never go through memory.
struct Args {
    const int8_t *Wp;                     // [S][nkb][MB][64][16]
    const uint64_t *A;                    // [L][K][Ncols]
    uint64_t *C;                          // [L][M][Ncols]
    const pcmm_host::LimbConst *lc;       // [L]
    int64_t M, K, Ncols;
    int64_t MB;                           // 16-row blocks in Wp
    int nkb;                              // k-steps of 64 in Wp
    int L;
};

// Enqueues the kernel on `st`.  hipErrorInvalidValue if there is no kernel for these parameters.
hipError_t launch(const Args &a, const pcmm_host::ResidentTile &tile, int D, int S, int epi, hipStream_t st);

}  // namespace pcmm_resident

#endif  // PCMM_RESIDENT_HPP
