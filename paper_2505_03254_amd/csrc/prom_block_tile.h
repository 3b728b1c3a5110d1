// The block kernel whose wavefronts own pixel tiles (prom_block_tile.hip): arguments, planning and launch, used by
// prom_block_ex (prom_block.hip).
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace prom {

struct TileArgs {
    const int8_t *x;
    int8_t *y;
    const uint32_t *we;  // packed expand weights [chid][cin]
    const int8_t *wd;    // depthwise weights [3][3][chid]
    const uint32_t *wp;  // packed project weights [cout][chid]
    const int32_t *be, *me, *se;  // expand bias / mult / shift [chid]
    const int32_t *bd, *md, *sd;  // depthwise [chid]
    const int32_t *bp, *mp, *sp;  // project [cout]
    const int32_t *ne, *nd, *np;  // PReLU negative-side multipliers of the three layers, or nullptr
    int N, H, W, Ho, Wo, cin, chid, cout, stride;
    int add_res;
    int lo_e, hi_e, lo_d, hi_d, lo_p, hi_p;
    int n_tiles, per_img, cols_n;   // tiles in all, of an image, of a row of tiles
    unsigned magic_img, magic_col;  // division by per_img, by cols_n
    int magic_s;         // division by S
    int S, T;            // wavefronts that share a tile's hidden channels; tiles of a workgroup at a time
    int NQ;              // pairs of 16-channel planes of the hidden tensor
    int KWe, KWp;        // packed words per expand / project weight row
    int t1_bytes;        // a wavefront's plane
    int off_fp, off_pe, off_dw, off_slot, off_t1;  // LDS byte offsets
    int inst;            // which kernel
    double us;           // the planner's estimate
};

// A caller's choice, 0 for the planner's: variant 1, 2, ..., wavefronts that share a tile, tiles of a workgroup.
struct TileChoice { int variant, split, tiles; };
// Tile, split and LDS layout for the shape in `a`; false if the kernel does not take it.
bool plan_tile(TileArgs &a, bool prelu, size_t &lds, int &grid, const TileChoice &only = {});
// Launch; PROM_OK or PROM_EHIP.
int launch_tile(const TileArgs &a, size_t lds, int grid, void *stream);

}  // namespace prom
