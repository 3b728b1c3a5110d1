// The pointwise kernel for wide layers (k loop outermost over a workgroup tile of pixels x output
// channels; prom_pw_gemm.hip), selected by pw_prepare (prom_pw.hip).
#pragma once
#include "prom_pw_stream.h"

namespace prom {

// A workgroup's tile: tm pixels x tn output channels; wgs: workgroups resident per compute unit.
struct GemmTile {
    int tm, tn, wgs;
    size_t lds;
    PwKernelFn fn;
};

// pt: 16-pixel tiles per wavefront (2, 4 or 8).
GemmTile pw_gemm_tile(int pt, bool prelu);

}  // namespace prom
