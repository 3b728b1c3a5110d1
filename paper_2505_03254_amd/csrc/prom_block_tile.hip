// Inverted-residual block (paper Section 2 and Figure 4: ternary pointwise expansion -> int8 depthwise
// 3x3 -> ternary pointwise projection, + skip) as ONE kernel in which every wavefront works for itself on a
// tile of output pixels, for blocks with few channels on large maps.
//
// Such blocks are bound by the requantisation of the expanded tensor (14 clocks of a SIMD per output and
// wavefront, twice per hidden element, plus the halo), 13 us for 56x56x144 at batch 128 in tiles of 8 rows (10
// without the halo), as long as nothing else stands in the way: three launches take the expanded tensor through HBM twice each way (68 us),
// the kernel with whole planes in LDS fills a CU with one workgroup whose phases follow each other (70 us).
// Here nothing but the weights is shared:
//   - the workgroup decodes the weights of the whole block into LDS once and stays resident, walking over
//     tiles (S = 1), so that prologue and weights are paid once per CU;
//   - a wavefront keeps the input of its tile in registers as MFMA operands (a row of 16 input columns is one
//     16-pixel tile, straight from the NHWC rows, 14 (7 at stride 2) output columns wide) and walks over the
//     hidden channels in planes of 16: expansion (1 MFMA per row), requantisation, 256 bytes a row into the
//     wavefront's own plane of 1 to 4.6 KB; depthwise filter on the matrix cores (one-hot operands, tap rows in
//     the k dimension), requantisation; and the outputs of two planes ARE the B operand of a projection MFMA
//     (v_mfma_i32_16x16x32_i8) -- the projection accumulates in registers.  No barrier, no second pass
//     through LDS; LDS operations of one wavefront complete in order.
//   - stride 1: the four lane groups of an operand hold four input rows, so one read serves two output rows
//     (against tap groups (0,0) (0,1) (0,2) (1,0) ...: half the reads); one lane address and constant offsets
//     for all of a plane's accesses (per-pixel address registers for arbitrary tile shapes were built first:
//     2 to 4 us more per round in address arithmetic, spills, bank conflicts where rows end inside a tile);
//   - small problems: S wavefronts share a tile's planes and add their partial projections in LDS.
// In the loop the kernel is at its instruction count: 3 wavefronts per SIMD with 10 tiles (4 rows) take 870
// clocks per plane each, 2 with 18 tiles (8 rows) 1600, where the sum of the instructions' issue times is 870
// and 1440.  Around it a tile costs 0.9 us and 0.21 per 16 pixels and 16 output channels (projection's
// requantisation, skip and store: 4.3 us with 8 rows, of which 0.4 are issue), launch and prologue 4 us: the 36 us of
// 56x56 24-144-24 at batch 128 are two rounds of 11.5 us in the loop and 4.3 behind it.
// Variants of 8, 6, 4 and 2 rows trade halo rows and per-plane work against registers (2, 2, 3 and 4 wavefronts per
// SIMD); plan_tile prices them.  With 8 rows the 256 registers do not quite do: the plain kernel of stride 1 spills 3
// (16 bytes of scratch a lane), that of stride 2 with PReLU 1; written once, read once per tile, not in the loop.
// Measured (replayed from graphs, us; three launches or the plane-resident kernel before): batch 128,
// 112x112 16-96-24 stride 2 91 -> 45.4, 56x56 24-144-24 67.3 -> 34.8, 24-144-32 stride 2 42.2 -> 20.9, 28x28
// 32-192-32 22.1 -> 17.9, 32-192-64 stride 2 16.3 -> 13.1; batch 8, the first two 12.5 -> 9.6 and 10.3 -> 9.1.
// All shifts >= 2 and windows [0, 127], which every time above is for; the first at batch 128 on another machine 43.4, with
// one shift of 1 45.8, of 0 53.3, with PReLU 56.4, and one shift of 1 72.1 (the plane-resident kernel 86 in all of these);
// in the network's chain, whose expansion has shifts of 1 and whose tensors come from memory, up to 53.
#include "prom_pw_stream.h"
#include "prom_launch.h"
#include "prom_block_tile.h"

#include <mutex>
#include <vector>

namespace prom {

#ifdef PROM_TIMELINE
// Developer build: wavefronts of the first 256 workgroups record the 100 MHz clock and their own cycles.
__device__ unsigned long long g_tl_stamps[256 * 16 * 16];
#define TL_STAMP(i) do { if (lane == 0 && blockIdx.x < 256) { unsigned long long *s_ = g_tl_stamps + (blockIdx.x * 16 + wave) * 16; s_[i] = wall_clock64(); s_[8 + (i)] = clock64(); } } while (0)
#else
#define TL_STAMP(i) do { } while (0)
#endif

template <int V> struct TlConst { static constexpr int value = V; };

// The four codes of channels 4*d .. 4*d+3 of a packed word as int8.
__device__ __forceinline__ int decode_quarter(uint32_t word, int d)
{
    const uint32_t sel = ((word >> (2 * d)) & 0x03030303u) << 1;
    return (int)__builtin_amdgcn_perm(0x00FF0000u, 0x00010000u, sel);
}

// LDS by byte offset (the kernel has no other LDS than the dynamic array, which starts at 0): an address that is kept in
// a register is then used as it is, with the constant part of an access in its offset field.
typedef __attribute__((address_space(3))) v4i lds_v4i;
typedef __attribute__((address_space(3))) v2i lds_v2i;
typedef __attribute__((address_space(3))) uint32_t lds_u32;
__device__ __forceinline__ v4i lds_read16(int at) { return *(const lds_v4i *)(uintptr_t)(uint32_t)at; }
__device__ __forceinline__ v2i lds_read8(int at) { return *(const lds_v2i *)(uintptr_t)(uint32_t)at; }
__device__ __forceinline__ v2i lds_read8_a4(int at)  // at a multiple of 4
{
    const lds_u32 *p = (const lds_u32 *)(uintptr_t)(uint32_t)at;
    return v2i{(int)p[0], (int)p[1]};
}
__device__ __forceinline__ void lds_write4(int at, uint32_t v) { *(lds_u32 *)(uintptr_t)(uint32_t)at = v; }

// STRIDE; TR: output rows of a tile; COT: 16-channel tiles of the output; NW: most wavefronts of a workgroup (sets the
// registers).
template <int STRIDE, int TR, int COT, bool PRELU, int NW>
__global__ __launch_bounds__(64 * NW, NW / 4) void block_tile_kernel(const TileArgs a)
{
    constexpr int TC = STRIDE == 1 ? 14 : 7;                // output columns of a tile
    constexpr int NT1 = (TR - 1) * STRIDE + 3;              // its input rows, 16 columns each: tiles of the expansion
    constexpr int NT2 = STRIDE == 1 ? TR : TR / 2;          // tiles of the output: a row, or two rows of 8 columns
    constexpr int ROW = 256;                                // LDS bytes of a row of a plane: 16 cells of 16 channels
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    TL_STAMP(0);
    const int W = a.W, H = a.H, Wo = a.Wo, Ho = a.Ho;
    const int cin = a.cin, cout = a.cout, chid = a.chid;
    const int NP = chid >> 4, NQ = a.NQ, S = a.S, T = a.T;
    const int tg = S == 1 ? wave : (wave * a.magic_s) >> 16, kg = wave - tg * S;

    constexpr int FE = COT * 256;                                  // LDS: the projection's parameters, then the weights
    v4i *pp = reinterpret_cast<v4i *>(lds);                        // [16 COT] projection parameters
    v4i *fe = reinterpret_cast<v4i *>(lds + FE);                   // [2 NQ][64] decoded expansion weights
    v2i *fp = reinterpret_cast<v2i *>(lds + a.off_fp);             // [NQ][COT][64] decoded projection weights
    v4i *pe = reinterpret_cast<v4i *>(lds + a.off_pe);             // [2][32 NQ] parameters of the expansion, of the depthwise layer
    uint32_t *dwt = reinterpret_cast<uint32_t *>(lds + a.off_dw);  // [32 NQ][5]: 0, the three rows of taps (3 bytes each), 0
    int *slot = reinterpret_cast<int *>(lds + a.off_slot);         // [16] what each wavefront found out about its shifts

    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(a.x), 0, a.N * H * W * cin, kBufFlags);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(a.y, 0, a.N * Ho * Wo * cout, kBufFlags);

    // ---- a tile: where it lies, its input into registers -------------------------------------------------
    // Row i of the input under the tile's taps is expansion tile i, lane j its column j.  LDS: 16 cells a row; for
    // stride 2 the even columns first, then the odd ones, so that every tap of neighbouring outputs reads neighbouring cells.
    const int t1o = a.off_t1 + wave * a.t1_bytes;                  // this wavefront's plane
    const int t1w = t1o + 4 * g + 16 * (STRIDE == 1 ? j : (j & 1) * 8 + (j >> 1));
    // the filter's operand: tap row g of pixel j (stride 1: of a pair of output rows, g - 1 for the second of them)
    const int t1r = t1o + (STRIDE == 1 ? g * ROW + 16 * j : ((j >> 3) * 2 + g) * ROW + 16 * (j & 7));
    struct Where { int img, oy0, ox0; } at;
    uint32_t byte_mask = ~0u;  // 0x7f7f7f7f where the requantisation leaves the top bits to the border's mask
    v4i xr[NT1];
    uint32_t inside[NT1];  // byte mask of row i, column j: zero outside the image (the filter's border)
    auto setup = [&](const int tile) __attribute__((always_inline)) {
        at.img = a.per_img == 1 ? tile : __umulhi((unsigned)tile, a.magic_img);
        const int q = tile - at.img * a.per_img;
        const int tr = a.cols_n == 1 ? q : __umulhi((unsigned)q, a.magic_col);
        at.oy0 = tr * TR;
        at.ox0 = (q - tr * a.cols_n) * TC;
        const int iy0 = at.oy0 * STRIDE - 1, ix = at.ox0 * STRIDE - 1 + j;
        const bool colok = ix >= 0 && ix < W;
        const uint32_t colmask = colok ? byte_mask : 0u;
        const unsigned xcol = colok ? (unsigned)ix * (unsigned)cin + 16u * g : (unsigned)kOobOffset;
#pragma unroll
        for (int i = 0; i < NT1; ++i) {
            const int iy = iy0 + i;
            const bool rowok = iy >= 0 && iy < H;
            // (rows outside are loaded from inside and masked)
            const int xrow = ((at.img * H + (rowok ? iy : 0)) * W) * cin;
            xr[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)xcol, xrow, 0);
            inside[i] = rowok ? colmask : 0u;
        }
    };
    // (the tiles of a round that is not full are spread over all workgroups)
    const int step = gridDim.x * T;
    int tile = tg * gridDim.x + blockIdx.x;
    int form, form_p;
    // ---- weights and parameters into LDS.  Every global load of the prologue leaves before the first value is used.
    {
        constexpr int U = 2;
        const int KWe = a.KWe, KWp = a.KWp;
        const int ne = 2 * NQ * 64, npj = NQ * COT * 64, npar = 32 * NQ;
        auto rsrc = [&](const void *p, const int n) __attribute__((always_inline)) {
            return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, n, kBufFlags);
        };
        const __amdgpu_buffer_rsrc_t rwe = rsrc(a.we, chid * KWe * 4), rwp = rsrc(a.wp, cout * KWp * 4), rwd = rsrc(a.wd, 9 * chid);
        const int nb = chid * 4;
        // channels beyond the layer's read zero
        const __amdgpu_buffer_rsrc_t rbe = rsrc(a.be, nb), rme = rsrc(a.me, nb), rse = rsrc(a.se, nb), rne = rsrc(a.ne ? a.ne : a.me, nb);
        const __amdgpu_buffer_rsrc_t rbd = rsrc(a.bd, nb), rmd = rsrc(a.md, nb), rsd = rsrc(a.sd, nb), rnd = rsrc(a.nd ? a.nd : a.md, nb);
        struct Par { v4i e, d; };
        auto ld = [&](const __amdgpu_buffer_rsrc_t r, const int i) __attribute__((always_inline)) {
            return (int)__builtin_amdgcn_raw_buffer_load_b32(r, i * 4, 0, 0);
        };
        auto load_par = [&](const int c) __attribute__((always_inline)) {
            Par p;
            p.e = v4i{ld(rbe, c), ld(rme, c), PRELU ? ld(rne, c) : 0, ld(rse, c)};
            p.d = v4i{ld(rbd, c), ld(rmd, c), PRELU ? ld(rnd, c) : 0, ld(rsd, c)};
            return p;
        };
        auto load_e = [&](const int e) __attribute__((always_inline)) {
            const int kw = (e >> 4) & 3;
            const int w = __umul24(16 * (e >> 6) + (e & 15), KWe) + kw;
            return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rwe, kw < KWe ? w * 4 : kOobOffset, 0, 0);
        };
        // row m of output tile ct is channel 4 COT (m / 4) + 4 ct + m % 4: a lane's outputs are 4 COT consecutive channels
        auto load_p = [&](const int e, uint32_t(&w)[2]) __attribute__((always_inline)) {
            const int m = e & 15, qc = e >> 6;
            const int q = qc / COT, ct = qc - q * COT;
            const int ch = 4 * COT * (m >> 2) + 4 * ct + (m & 3);
            const int o = (__umul24(ch, KWp) + 2 * q) * 4;
            w[0] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rwp, o, 0, 0);
            w[1] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rwp, 2 * q + 1 < KWp ? o + 4 : kOobOffset, 0, 0);
        };
        // k byte 8 kq + 4 i + r is hidden channel 16 (2 q + i) + 4 kq + r: what a lane of the depthwise filter's outputs holds
        auto store_p = [&](const int e, const uint32_t(&w)[2]) __attribute__((always_inline)) {
            const int kq = (e >> 4) & 3;
            fp[e] = v2i{decode_quarter(w[0], kq), decode_quarter(w[1], kq)};
        };
        auto load_d = [&](const int c4, uint32_t(&t)[9]) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 9; ++k) t[k] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rwd, c4 * 4, k * chid, 0);
        };
        auto store_d = [&](const int c4, const uint32_t(&t)[9]) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                uint32_t *dst = dwt + (4 * c4 + r) * 5;
                dst[0] = 0u;
                dst[4] = 0u;
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const uint32_t lo = __builtin_amdgcn_perm(t[3 * dy + 1], t[3 * dy], 0x0c0c0000u | ((4 + r) << 8) | r);
                    dst[1 + dy] = __builtin_amdgcn_perm(t[3 * dy + 2], lo, 0x0c000100u | ((4 + r) << 16));
                }
            }
        };
        const Par par = load_par(tid);
        const int co = min(tid, cout - 1);
        const int pb = a.bp[co], pm = a.mp[co], ps = a.sp[co], pn = a.np ? a.np[co] : 0;
        uint32_t we[U], wp[U][2], wd[9];
#pragma unroll
        for (int u = 0; u < U; ++u) we[u] = load_e(tid + u * nthr);
#pragma unroll
        for (int u = 0; u < U; ++u) load_p(tid + u * nthr, wp[u]);
        load_d(tid, wd);
        if (tile < a.n_tiles) setup(tile);
        // ---- which forms of the requantisation the layers' shifts allow: each wavefront looks at the ones it holds
        int smin = 31;
#pragma clang loop unroll(disable)
        for (int c = tid; c < chid; c += nthr) {
            const bool own = c == tid;
            smin = min(smin, own ? min(par.e[3], par.d[3]) : min(a.se[c], a.sd[c]));
        }
        {
            const int f = (__builtin_amdgcn_ballot_w64(smin < 1) != 0 ? 1 : 0) | (__builtin_amdgcn_ballot_w64(smin < 2) != 0 ? 2 : 0) |
                          (__builtin_amdgcn_ballot_w64(tid < cout && ps < 1) != 0 ? 4 : 0);
            if (lane == 0) slot[wave] = f;
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);  // LDS only: the weights are still on their way
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int f = slot[min(lane, (nthr >> 6) - 1)];
        const bool ge1 = __builtin_amdgcn_ballot_w64(f & 1) == 0, ge2 = __builtin_amdgcn_ballot_w64(f & 2) == 0;
        const int form_e = pair_form_of(PRELU, ge1, ge2, a.lo_e, a.hi_e), form_d = pair_form_of(PRELU, ge1, ge2, a.lo_d, a.hi_d);
        // (One choice for both layers and all channels.  A pair of forms, with kPairLow for shifts of 1 and kPairRelu for the
        // depthwise layer behind them, was built: 112x112 16-96-24 at batch 128 45.8 -> 44.7 us with a shift of 1 and 72.1 ->
        // 69.1 with PReLU, but 43.4 -> 44.2 and 56.4 -> 57.6 without; over 44 blocks 2.5 % slower with shifts >= 2, 3.7 %
        // with PReLU and 0.9 % with a shift of 1 -- more registers spill, and the prologue is 0.2 us longer.)
        if (PRELU) form = form_e == form_d ? form_e : kPairPreluAny;
        else form = form_e == kPairRelu && form_d == kPairRelu ? kPairRelu : ge1 ? kPairClamp : kPairAny;
        form_p = a.np ? kPairPreluAny : __builtin_amdgcn_ballot_w64(f & 4) == 0 && a.lo_p == -128 && a.hi_p == 127 ? kPairFull : kPairAny;
        // parameters with the shifts as the forms take them
        const int less = pair_shift_less(form);
        auto store_par = [&](const int c, const Par &p) __attribute__((always_inline)) {
            v4i e = requant_params(p.e[0], p.e[1], p.e[2], p.e[3], PRELU), d = requant_params(p.d[0], p.d[1], p.d[2], p.d[3], PRELU);
            e[3] -= less;
            d[3] -= less;
            pe[c] = c < chid ? e : v4i{0, 0, 0, 0};
            pe[npar + c] = c < chid ? d : v4i{0, 0, 0, 0};
        };
        if (tid < npar) store_par(tid, par);
        if (tid < 16 * COT) {
            v4i r = tid < cout ? requant_params(pb, pm, pn, ps, a.np != nullptr) : v4i{0, 0, 0, 1};
            if (form_p == kPairFull) r[3] -= pair_shift_less(kPairFull);
            pp[tid] = r;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (tid + u * nthr < ne) fe[tid + u * nthr] = decode_word(we[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (tid + u * nthr < npj) store_p(tid + u * nthr, wp[u]);
        if (tid < 8 * NQ) store_d(tid, wd);
        // what is left of wider blocks, four loads in flight
        constexpr int V = 4;
#pragma clang loop unroll(disable)
        for (int e0 = tid + U * nthr; e0 < ne; e0 += V * nthr) {
            uint32_t w[V];
#pragma unroll
            for (int u = 0; u < V; ++u) w[u] = load_e(e0 + u * nthr);
#pragma unroll
            for (int u = 0; u < V; ++u)
                if (e0 + u * nthr < ne) fe[e0 + u * nthr] = decode_word(w[u]);
        }
#pragma clang loop unroll(disable)
        for (int e0 = tid + U * nthr; e0 < npj; e0 += V * nthr) {
            uint32_t w[V][2];
#pragma unroll
            for (int u = 0; u < V; ++u) load_p(e0 + u * nthr, w[u]);
#pragma unroll
            for (int u = 0; u < V; ++u)
                if (e0 + u * nthr < npj) store_p(e0 + u * nthr, w[u]);
        }
#pragma clang loop unroll(disable)
        for (int c = tid + nthr; c < 8 * NQ; c += nthr) {
            load_d(c, wd);
            store_d(c, wd);
        }
#pragma clang loop unroll(disable)
        for (int c = tid + nthr; c < npar; c += nthr) store_par(c, load_par(c));
    }
    if (form == kPairRelu) {
        byte_mask = 0x7f7f7f7fu;
#pragma unroll
        for (int i = 0; i < NT1; ++i) inside[i] &= byte_mask;
    }
    __syncthreads();
    TL_STAMP(1);
#ifdef PROM_TIMELINE
    int nround = 0;
#endif
    const int lo_e = in_vgpr(a.lo_e), hi_e = in_vgpr(a.hi_e);
    const int lo_d = in_vgpr(a.lo_d), hi_d = in_vgpr(a.hi_d);
    const v4i zero4 = {0, 0, 0, 0};

    // one-hot operands: byte dx of a channel's row of taps at byte j of the lane's 16
    uint32_t sel[3], mask[4];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) sel[dx] = 0x0c0c0c0cu ^ ((uint32_t)(0x0c ^ dx) << (8 * (j & 3)));
#pragma unroll
    for (int k = 0; k < 4; ++k) mask[k] = (uint32_t)in_vgpr((j >> 2) == k ? -1 : 0);  // (as a value: a condition would cost a v_cndmask_b32 per use)

    while (true) {
        const bool live = tile < a.n_tiles;
        if (!live && S == 1) break;
        v4i acc[COT][NT2];
#pragma unroll
        for (int ct = 0; ct < COT; ++ct)
#pragma unroll
            for (int t = 0; t < NT2; ++t) acc[ct][t] = zero4;

        constexpr int NB = STRIDE == 1 ? NT2 / 2 : NT2;
        auto planes = [&](auto fm) __attribute__((always_inline)) {
            constexpr int FORM = decltype(fm)::value;
            // this wavefront's pairs of planes; LDS addresses of the pair's weights and parameters
            int at_e = FE + kg * 2048 + lane * 16;
            int at_p = a.off_fp + kg * (COT * 512) + lane * 8;
            int at_par = a.off_pe + kg * 512 + g * 64;
            int at_w = a.off_dw + kg * 640 + j * 20 + g * 4;
            for (int q = kg; q < NQ; q += S) {
                // (opaque, or the compiler counts them from the far end, and offsets below zero cannot be folded)
                asm("" : "+v"(at_e), "+v"(at_p), "+v"(at_par), "+v"(at_w));
                int bq[NT2][2];
#pragma unroll
                for (int i2 = 0; i2 < 2; ++i2) {
                    if (i2 == 1 && 2 * q + 1 >= NP) {  // half a pair: against zero weights
#pragma unroll
                        for (int t = 0; t < NT2; ++t) bq[t][1] = 0;
                        break;
                    }
                    // expansion of the plane
                    {
                        v4i par[4], d[NT1];
                        const v4i A = lds_read16(at_e + i2 * 1024);
#pragma unroll
                        for (int r = 0; r < 4; ++r) par[r] = lds_read16(at_par + i2 * 256 + r * 16);
                        const v4i cinit = PRELU ? v4i{par[0][0], par[1][0], par[2][0], par[3][0]} : zero4;
#pragma unroll
                        for (int i = 0; i < NT1; ++i) d[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, xr[i], cinit, 0, 0, 0);
#pragma unroll
                        for (int i = 0; i < NT1; i += 2) {
                            uint32_t q0, q1;
                            const int i1 = i + 1 < NT1 ? i + 1 : i;
                            requant_pair4<FORM, true, false>(d[i], d[i1], par, lo_e, hi_e, q0, q1);
                            lds_write4(t1w + i * ROW, q0 & inside[i]);
                            if (i1 != i) lds_write4(t1w + i1 * ROW, q1 & inside[i1]);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    // its depthwise filter
                    {
                        v4i B[NB][3];
#pragma unroll
                        for (int u = 0; u < NB; ++u) {
                            // two output rows of 14 columns need four rows of the plane, two of 7 columns five
                            const int at = t1r + u * (STRIDE == 1 ? 2 : 4) * ROW;
                            B[u][0] = lds_read16(at);
                            B[u][1] = lds_read16(at + (STRIDE == 1 ? 16 : 128));
                            B[u][2] = lds_read16(at + (STRIDE == 1 ? 32 : 16));
                        }
                        const v2i tap = lds_read8_a4(at_w + i2 * 320);
                        const uint32_t tlo = (uint32_t)tap[0], thi = (uint32_t)tap[1];
                        v4i Ae[3], Ao[3], par[4], d[NT2];
#pragma unroll
                        for (int r = 0; r < 4; ++r) par[r] = lds_read16(at_par + 512 * NQ + i2 * 256 + r * 16);
#pragma unroll
                        for (int dx = 0; dx < 3; ++dx) {
                            const uint32_t ve = __builtin_amdgcn_perm(thi, thi, sel[dx]);
                            const uint32_t vo = __builtin_amdgcn_perm(tlo, tlo, sel[dx]);
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                Ae[dx][k] = (int)(ve & mask[k]);
                                if (STRIDE == 1) Ao[dx][k] = (int)(vo & mask[k]);
                            }
                        }
                        const v4i cinit = PRELU ? v4i{par[0][0], par[1][0], par[2][0], par[3][0]} : zero4;
#pragma unroll
                        for (int t = 0; t < NT2; ++t) d[t] = cinit;
#pragma unroll
                        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                            for (int u = 0; u < NB; ++u) {
                                if constexpr (STRIDE == 1) {
                                    d[2 * u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(Ae[dx], B[u][dx], d[2 * u], 0, 0, 0);
                                    d[2 * u + 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(Ao[dx], B[u][dx], d[2 * u + 1], 0, 0, 0);
                                } else {
                                    d[u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(Ae[dx], B[u][dx], d[u], 0, 0, 0);
                                }
                            }
#pragma unroll
                        for (int t = 0; t < NT2; t += 2) {
                            uint32_t q0, q1;
                            requant_pair4<FORM, true>(d[t], d[t + 1], par, lo_d, hi_d, q0, q1);
                            bq[t][i2] = (int)q0;
                            bq[t + 1][i2] = (int)q1;
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                // the two planes' part of the projection
#pragma unroll
                for (int ct = 0; ct < COT; ++ct) {
                    const v2i A = lds_read8(at_p + ct * 512);
#pragma unroll
                    for (int t = 0; t < NT2; ++t)
                        acc[ct][t] = __builtin_amdgcn_mfma_i32_16x16x32_i8(__builtin_bit_cast(long, A), __builtin_bit_cast(long, v2i{bq[t][0], bq[t][1]}), acc[ct][t], 0, 0, 0);
                }
                at_e += S * 2048;
                at_p += S * (COT * 512);
                at_par += S * 512;
                at_w += S * 640;
            }
        };
        if (live) {
            if constexpr (PRELU) {
                if (form == kPairPreluFull) planes(TlConst<kPairPreluFull>{});
                else planes(TlConst<kPairPreluAny>{});
            } else {
                if (form == kPairRelu) planes(TlConst<kPairRelu>{});
                else if (form == kPairClamp) planes(TlConst<kPairClamp>{});
                else planes(TlConst<kPairAny>{});
            }
        }
#ifdef PROM_TIMELINE
        if (nround == 0) TL_STAMP(2);
#endif
        const Where now = at;
        const int next = tile + step;
        if (S == 1 && next < a.n_tiles) setup(next);

        // ---- the projection's requantisation, the skip, the store: output tiles t and t + 1 --------------
        const int rows_left = Ho - now.oy0, cols_left = Wo - now.ox0;
        const int yrow = Wo * cout;
        const int ybase = ((now.img * Ho + now.oy0) * Wo + now.ox0) * cout;
        const bool whole = cout % (4 * COT) == 0;  // all or none of a lane's channels exist
        const int ox = STRIDE == 1 ? j : j & 7;
        const int oyj = STRIDE == 1 ? 0 : j >> 3;  // stride 2: the second row of a tile sits in lanes 8 to 15
        const unsigned ocol = ox < TC && ox < cols_left && 4 * COT * g < cout
                                  ? (unsigned)(ox * cout + oyj * yrow + 4 * COT * g) : (unsigned)kOobOffset;
        auto finish = [&](const int t, const int t1, const v4i(&d0)[COT], const v4i(&d1)[COT]) __attribute__((always_inline)) {
            unsigned off[2];
            int row[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int oy = (k ? t1 : t) * (STRIDE == 1 ? 1 : 2);
                row[k] = oy < rows_left ? ybase + oy * yrow : 0;
                off[k] = oy + oyj < rows_left ? ocol : (unsigned)kOobOffset;
            }
            uint32_t out[2][COT];
            auto requant = [&](auto fm) __attribute__((always_inline)) {
                const int lo_p = in_vgpr(a.lo_p), hi_p = in_vgpr(a.hi_p);
#pragma unroll
                for (int ct = 0; ct < COT; ++ct) {
                    v4i par[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) par[r] = pp[4 * COT * g + 4 * ct + r];
                    requant_pair4<decltype(fm)::value>(d0[ct], d1[ct], par, lo_p, hi_p, out[0][ct], out[1][ct]);
                }
            };
            uint32_t res[2][COT];
            if (a.add_res) {
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int ct = 0; ct < COT; ++ct)
                        res[k][ct] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rx, (int)off[k] + 4 * ct, row[k], 0);
            }
            if (form_p == kPairPreluAny) requant(TlConst<kPairPreluAny>{});
            else if (form_p == kPairFull) requant(TlConst<kPairFull>{});
            else requant(TlConst<kPairAny>{});
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if (a.add_res) {
#pragma unroll
                    for (int ct = 0; ct < COT; ++ct) out[k][ct] = add_sat_i8x4(out[k][ct], res[k][ct]);
                }
                if (whole && COT == 2) {
                    __builtin_amdgcn_raw_buffer_store_b64(v2i{(int)out[k][0], (int)out[k][1]}, ry, (int)off[k], row[k], 0);
                } else {
#pragma unroll
                    for (int ct = 0; ct < COT; ++ct)
                        __builtin_amdgcn_raw_buffer_store_b32((int)out[k][ct], ry, 4 * COT * g + 4 * ct < cout ? (int)off[k] + 4 * ct : kOobOffset, row[k], 0);
                }
            }
        };
        if (S == 1) {
#pragma unroll
            for (int t = 0; t < NT2; t += 2) {
                v4i d0[COT], d1[COT];
#pragma unroll
                for (int ct = 0; ct < COT; ++ct) {
                    d0[ct] = acc[ct][t];
                    d1[ct] = acc[ct][t + 1];
                }
                finish(t, t + 1, d0, d1);
            }
        } else {
            // the partial sums of the wavefronts of a tile meet in LDS; each finishes its share of the pairs
            // (in place of the weights: with S > 1 a workgroup has one round)
            v4i *red = reinterpret_cast<v4i *>(lds + FE);
            __syncthreads();
#pragma unroll
            for (int t = 0; t < NT2; ++t)
#pragma unroll
                for (int ct = 0; ct < COT; ++ct) red[((wave * NT2 + t) * COT + ct) * 64 + lane] = acc[ct][t];
            __syncthreads();
            if (live) {
                for (int t = 2 * kg; t < NT2; t += 2 * S) {
                    v4i d0[COT], d1[COT];
#pragma unroll
                    for (int ct = 0; ct < COT; ++ct) d0[ct] = d1[ct] = zero4;
                    for (int s = 0; s < S; ++s) {
                        const v4i *r0 = red + (((tg * S + s) * NT2 + t) * COT) * 64 + lane;
#pragma unroll
                        for (int ct = 0; ct < COT; ++ct) {
                            d0[ct] += r0[ct * 64];
                            d1[ct] += r0[(COT + ct) * 64];
                        }
                    }
                    finish(t, t + 1, d0, d1);
                }
            }
            break;
        }
#ifdef PROM_TIMELINE
        if (nround++ == 0) TL_STAMP(3);
#endif
        tile = next;
    }
    TL_STAMP(4);
}

using TileFn = void (*)(const TileArgs);
struct TileInst { int stride, tr, cot, nw; TileFn plain, prelu; };
#define TL(S, R, C, NW) {S, R, C, NW, &block_tile_kernel<S, R, C, false, NW>, &block_tile_kernel<S, R, C, true, NW>}
static const TileInst kTileInst[] = {
    TL(1, 8, 2, 8), TL(1, 6, 2, 8), TL(1, 4, 2, 12), TL(1, 2, 2, 16), TL(1, 6, 4, 8), TL(1, 4, 4, 8), TL(1, 2, 4, 12),
    TL(2, 8, 2, 8), TL(2, 4, 2, 12), TL(2, 4, 4, 8),
};
#undef TL

// Tile height, split of the hidden channels and workgroup for the shape in `a` (N, H, W, Ho, Wo, cin, chid, cout, stride
// set; prelu: a layer of the first two has negative-side multipliers); of those `only` leaves, if it is given.
//
// Every kernel, S and T is priced in microseconds.  A plane of a wavefront's tile takes the longer of its own chain
// (lat) and, with k wavefronts on a SIMD, k times the instructions it issues (thr); both grow with the 16-pixel tiles
// of the expansion and the filter.  Constants: least squares over 62771 plans of 1029 blocks (batch 1 to 256, maps of
// 11 to 115, up to 64 channels in and out, with and without PReLU), error 10 %; the plan it picks is 1.7 % behind the
// best one on average, 15 % at most.  Those blocks have few hidden channels: over 620 blocks with up to 512 the error grew
// to 36 % where the weights are many.  What a workgroup reads before it begins is the same for every plan, so it does not
// change the pick; it is added at the end (0.28 us for 4096 weights) and takes the error over these from 10 to 5.6 %.
bool plan_tile(TileArgs &a, bool prelu, size_t &lds, int &grid, const TileChoice &only)
{
    const int s = a.stride;
    if (a.cin % 4 != 0 || a.chid % 16 != 0 || a.cout % 4 != 0) return false;
    if ((long long)a.N * a.H * a.W * a.cin >= (long long)kOobOffset - 4096) return false;
    if ((long long)a.N * a.Ho * a.Wo * a.cout >= (long long)kOobOffset) return false;
    a.NQ = (a.chid / 16 + 1) / 2;
    a.KWe = (a.cin + 15) / 16;
    a.KWp = a.chid / 16;
    const int TC = s == 1 ? 14 : 7;
    a.cols_n = (a.Wo + TC - 1) / TC;
    const double slow = prelu ? 1.62 : 1.0;
    const int np = a.chid / 16;
    double best = 0;
    size_t best_lds = 0;
    int best_wgs = 0;
    for (int i = 0; i < (int)(sizeof(kTileInst) / sizeof(kTileInst[0])); ++i) {
        const TileInst &I = kTileInst[i];
        if (I.stride != s || a.cin > 64 || a.cout > 16 * I.cot || (only.variant && i + 1 != only.variant)) continue;
        const int TR = I.tr, nt1 = (TR - 1) * s + 3, nt2 = s == 1 ? TR : TR / 2;
        const long long per_img = (long long)((a.Ho + TR - 1) / TR) * a.cols_n, tiles = per_img * a.N;
        // (tile / per_img is a multiplication, right for tiles * per_img < 2^32)
        if (tiles > (1 << 28) || tiles * per_img >= (1LL << 32)) continue;
        // the plane: the rows under a tap (stride 2: one more, which the fourth lane group reads), and the cells that
        // lanes without an output column read behind the last one
        const int t1_bytes = (nt1 + (s == 1 ? 0 : 1)) * 256 + 32;
        const int off_fp = I.cot * 256 + 2 * a.NQ * 1024;
        const int off_pe = off_fp + a.NQ * I.cot * 512;
        const int off_dw = off_pe + a.NQ * 1024;
        const int off_slot = off_dw + a.NQ * 640;
        const int off_t1 = off_slot + 64;
        const double lat = (0.102 + 0.0315 * (nt1 + nt2)) * slow, thr = (0.067 + 0.0317 * (nt1 + nt2)) * slow;
        const int fin = nt2 * I.cot;
        for (int S : {1, 2, 3, 4, 6}) {
            if (S > a.NQ || S > I.nw || (only.split && S != only.split)) continue;
            const int npw = S == 1 ? np : 2 * ((a.NQ + S - 1) / S);  // planes of a wavefront
            for (int T = I.nw / S; T >= 1; --T) {
                if (only.tiles && T != only.tiles) continue;
                int bytes = off_t1 + S * T * t1_bytes;
                const int red = I.cot * 256 + S * T * fin * 1024;  // partial sums, in place of the weights
                if (S > 1 && bytes < red) bytes = red;
                if (bytes > 160 * 1024) continue;
                const int thr_wg = 64 * S * T;
                int percu = I.nw / (S * T);
                if (percu > 160 * 1024 / bytes) percu = 160 * 1024 / bytes;
                const long long wgs = (tiles + T - 1) / T;
                if (S > 1 && wgs * thr_wg >= (1LL << 32)) continue;  // (a launch has fewer threads than that)
                // rounds of the prologue's loads, and its entries per thread
                const int ne = 2 * a.NQ * 64, npj = a.NQ * I.cot * 64;
                const int extra = (ne > 2 * thr_wg ? (ne - 2 * thr_wg + 4 * thr_wg - 1) / (4 * thr_wg) : 0) +
                                  (npj > 2 * thr_wg ? (npj - 2 * thr_wg + 4 * thr_wg - 1) / (4 * thr_wg) : 0);
                const double ent = (double)(ne + npj) / thr_wg, pro = 1.76 + 0.39 * extra;
                auto loaded = [](double w) { return w > 1.0 ? w : 1.0; };
                auto planes = [&](long long k) { return npw * (lat > k * thr ? lat : k * thr); };
                double us = 2.33;
                if (S == 1) {  // one resident set of workgroups, whose wavefronts walk over the tiles
                    const long long g = wgs < 256 * percu ? wgs : 256 * percu, per = (g + 255) / 256;
                    us += pro + 0.026 * ent * loaded(per * T / 4.0);
                    auto round = [&](long long t) {
                        const long long k = (per * t + 3) / 4;
                        const double e = 0.93 + 0.21 * fin, f = 0.012 * k * fin;
                        return planes(k) + (e > f ? e : f);
                    };
                    const long long full = tiles / (g * T), left = tiles - full * g * T;
                    us += full * round(T);
                    if (left) us += round((left + g - 1) / g);
                } else {  // a workgroup has one round
                    auto round = [&](long long m) {
                        const long long per = (m + 255) / 256, k = (per * S * T + 3) / 4;
                        const double e = 0.93 + 0.21 * fin / S, f = 0.012 * k * fin / S;
                        return pro + 0.026 * ent * loaded(per * S * T / 4.0) + planes(k) + (e > f ? e : f) + 0.05 * fin * k;
                    };
                    const long long cap = 256 * percu, full = wgs / cap;
                    us += full * round(cap);
                    if (wgs % cap) us += round(wgs % cap);
                }
                if (best != 0 && us >= best) continue;
                best = us;
                best_lds = (size_t)bytes;
                best_wgs = (int)(S == 1 && wgs > 256 * percu ? 256 * percu : wgs);
                a.inst = i; a.S = S; a.T = T;
                a.per_img = (int)per_img;
                a.n_tiles = (int)tiles;
                a.t1_bytes = t1_bytes;
                a.off_fp = off_fp; a.off_pe = off_pe; a.off_dw = off_dw; a.off_slot = off_slot; a.off_t1 = off_t1;
            }
        }
    }
    if (best == 0) return false;
    a.us = best + 0.284 / 4096 * a.chid * (a.cin + a.cout) - 0.477;
    a.magic_img = (unsigned)(((1ull << 32) + a.per_img - 1) / a.per_img);
    a.magic_col = (unsigned)(((1ull << 32) + a.cols_n - 1) / a.cols_n);
    a.magic_s = 65536 / a.S + 1;
    lds = best_lds;
    grid = best_wgs;
    return true;
}

int launch_tile(const TileArgs &a, size_t lds, int grid, void *stream)
{
    const bool prelu = a.ne != nullptr || a.nd != nullptr;
    const TileFn fn = prelu ? kTileInst[a.inst].prelu : kTileInst[a.inst].plain;
    static std::mutex mu;
    static std::vector<TileFn> attr_done;
    {
        std::lock_guard<std::mutex> lock(mu);
        bool done = false;
        for (TileFn f : attr_done) done |= f == fn;
        if (!done) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (e != hipSuccess && lds > 64 * 1024) {
                last_hip_error() = e;
                (void)hipGetLastError();
                return PROM_EHIP;
            }
            attr_done.push_back(fn);
        }
    }
    clear_hip_error();
    TileArgs args = a;
    void *kargs[] = {&args};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(fn), dim3(grid), dim3(64 * a.S * a.T), kargs, lds,
                                         static_cast<hipStream_t>(stream));
    if (e != hipSuccess) {
        last_hip_error() = e;
        (void)hipGetLastError();
        return PROM_EHIP;
    }
    return check_launch();
}

}  // namespace prom

#ifdef PROM_TIMELINE
extern "C" int prom_debug_tl_stamps(unsigned long long *host)
{
    if (hipDeviceSynchronize() != hipSuccess) return PROM_EHIP;
    return hipMemcpyFromSymbol(host, HIP_SYMBOL(prom::g_tl_stamps), sizeof(unsigned long long) * 256 * 256) == hipSuccess ? PROM_OK : PROM_EHIP;
}
#endif
