// The pointwise kernel for wide layers (k loop outermost over a workgroup tile of pixels x output
// channels; prom_pw_gemm.hip), selected by pw_prepare (prom_pw.hip).
#pragma once
#include "prom_pw_stream.h"

namespace prom {

// A workgroup's tile: tm pixels x tn output channels.
struct GemmTile {
    int tm, tn, threads;
    size_t lds;
    PwKernelFn fn;
};

// pt: 16-pixel tiles per wavefront (2, 4 or 8); nw: wavefronts, 64 output channels each (2 or 4).
GemmTile pw_gemm_tile(int pt, int nw, bool prelu);

}  // namespace prom
