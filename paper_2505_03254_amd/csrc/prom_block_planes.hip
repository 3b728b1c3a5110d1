// Inverted-residual block (paper Section 2 and Figure 4: ternary pointwise expansion -> int8
// depthwise 3x3 -> ternary pointwise projection, + skip) as ONE kernel with the expanded tensor
// of a band of rows resident in LDS as 16-channel planes.
//
// The chunk-interleaved fused kernel of prom_block.hip keeps every weight of the block decoded in
// LDS and walks the hidden channels in barrier-separated chunks; beyond 192 hidden channels its
// weights no longer fit.  This kernel turns the ownership round so that NO weight matrix passes
// through LDS and the workgroup meets at two or three barriers in all:
//   phase 0  the band's input rows, the per-channel parameters of the expansion and the depthwise
//            layer and the depthwise weights go to LDS; the borders of the planes are zeroed;
//   phase 1  expansion.  A wavefront owns 16-channel planes of the hidden tensor (plane p, p + 8,
//            ...): it fetches the 16 x cin packed ternary codes of its plane straight from global
//            memory into registers (one dword per lane and k step, the next plane's one plane
//            ahead), decodes them once, and runs every 16-pixel tile of the band through
//            v_mfma_i32_16x16x64_i8 with the pixels as the B operand (a 16-byte LDS read), the
//            requantised outputs go to the plane [row][col + 1][16 channels] with a zero border;
//   phase 2  depthwise 3x3 of the same planes on the matrix cores (k = 4 taps x 16 channels; the A
//            operand holds the lane's one weight per tap group), by the same owner, so that a
//            plane needs no barrier between its expansion and its filter; the requantised outputs
//            go to the compact plane [pixel][16 channels];
//   phase 3  projection.  A wavefront owns an output-channel tile (and a group of up to 4 pixel
//            tiles), fetches and decodes that tile's rows of packed codes itself and reads the B
//            operands (pixel, 16 hidden channels) from the planes; epilogue, skip (the block input
//            is still in LDS), store.
// With at least as many planes as wavefronts a plane's depthwise output overwrites the slot of a
// plane its owner has already consumed (plane p -> slot p, its expansion sits in slot p + 8), so
// the hidden tensor takes (planes + 8) slots in all; with fewer planes the pixel tiles of a plane
// are spread over wavefronts, there is a barrier between phases 1 and 2 and the depthwise output
// has a region of its own.
//
// On few images the kernel is bound by the instructions around the tiles -- 16 wavefronts make one cost 16 clocks --, so:
// the parameters of the first two layers are made once per channel and kept in LDS where it has room (PARL; each unit
// made its own, 60 instructions, 16 lanes the same), index tables and copies divide by multiplication, and the
// prologue's loops of one or two rounds are not unrolled (up to 1.5 us).  Measured at batch 8, replayed from a graph, before and
// after: 7x7 160-960-160 15.5 -> 13.5 us, 14x14 64-384-64 8.5 -> 7.8, with PReLU 16.8 -> 14.6 and 9.8 -> 8.5; batch 128
// 18.9 -> 17.1 and 13.4 -> 12.7; 28x28 32-192-64 stride 2 16.6 -> 14.5.
#include "prom_pw_stream.h"
#include "prom_launch.h"
#include "prom_block_planes.h"

#include <cstdlib>
#include <mutex>
#include <vector>

namespace prom {

// Wavefronts per workgroup: 8, 12 or 16 (the planner takes the count that divides the planes best).

#ifdef PROM_TIMELINE
// Developer build: workgroups 0 .. 255 record the 100 MHz clock at the phase boundaries.
__device__ unsigned long long g_pl_stamps[256 * 8];
#define PL_STAMP(i) do { if (threadIdx.x == 0 && blockIdx.x < 256) g_pl_stamps[blockIdx.x * 8 + (i)] = wall_clock64(); } while (0)
#else
#define PL_STAMP(i) do { } while (0)
#endif

// Epilogue forms (requant_pair4) and tile counts as types.
template <int MODE> struct PlMode { static constexpr int value = MODE; };

// n / d by multiplication with ceil(2^32 / d): right for n * d < 2^32.  A divisor of 1 has none.
static inline uint32_t div_magic(int d) { return d > 1 ? (uint32_t)(((1ull << 32) + d - 1) / d) : 0u; }
// mul24: a product of numbers below 2^24.  (A full 32-bit product with a sum becomes v_mad_u64_u32, whose addend is a
// register pair; its unused upper half may be where a load in flight will land, and the prologue then waits 1 us for it.)
__device__ __forceinline__ int mul24(int x, int y) { return (int)__umul24((unsigned)x, (unsigned)y); }
__device__ __forceinline__ int fast_div(int n, uint32_t magic) { return magic == 0 ? n : (int)__umulhi((uint32_t)n, magic); }

// Bias, multiplier(s) and shift of a lane's four channels (16*plane + 4*g + 0..3) as loaded.
struct PlRawPar { v4i b, m, n, s; };

// KSE: 64-wide k steps of the expansion (cin <= 64*KSE).  PRELU: the expansion and depthwise
// epilogues take the PReLU form (a layer of the two without negative-side multipliers runs it with
// mult_neg = mult, which is the plain form).
// PARL: the parameters of the first two layers are made once per channel and kept in LDS (where it has room); otherwise
// each unit of work makes its own, 16 lanes the same.  (A template parameter: a choice at run time puts the prologue's
// loads under a branch, which costs a wait for those in flight, 1 us.)
template <int KSE, bool PRELU, int NW, bool PARL>
__global__ __launch_bounds__(64 * NW, 1) void block_planes_kernel(const PlanesArgs a)
{
    constexpr int kPlWaves = NW, kPlThreads = 64 * NW;
    extern __shared__ __align__(16) unsigned char lds[];
    PL_STAMP(0);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int W = a.W, Wo = a.Wo, W2 = W + 2, s = a.stride;
    const int cin = a.cin, chid = a.chid, cout = a.cout, cinp = a.cinp;
    const int NP = a.NP;

    const int img = blockIdx.x / a.bands;
    const int band = blockIdx.x - img * a.bands;
    const int ro0 = band * a.R;                                // first output row of the band
    const int rows_out = min(a.R, a.Ho - ro0);
    const int ri0 = ro0 * s - 1;                               // first input row under a tap (may be -1)
    const int ri_last = ri0 + (rows_out - 1) * s + 2;          // last one (may be H)
    const int rlo = max(ri0, 0), rhi = min(ri_last, a.H - 1);  // the rows that exist
    const int rv0 = rlo - ri0;                                 // plane row of the first existing input row
    const int nvr = rhi - rlo + 1;
    const int rib = ri_last - ri0 + 1;                         // plane rows in use
    const int np1 = nvr * W;                                   // pixels to expand
    const int np2 = rows_out * Wo;                             // output pixels of the band
    const int nt1 = (np1 + 15) >> 4, nt2 = (np2 + 15) >> 4;

    int8_t *xs = reinterpret_cast<int8_t *>(lds);
    uint16_t *o1 = reinterpret_cast<uint16_t *>(lds + a.off_o1);  // pixel of phase 1 -> 16-byte cell of its plane
    uint16_t *o2 = reinterpret_cast<uint16_t *>(lds + a.off_o2);  // output pixel -> cell of its tap (0, 0)
    v4i *pp = reinterpret_cast<v4i *>(lds + a.off_pp);            // [16*COT] projection parameters
    int8_t *wdl = reinterpret_cast<int8_t *>(lds + a.off_wd);     // [9][chid] depthwise weights
    uint32_t *w3l = reinterpret_cast<uint32_t *>(lds + a.off_w3); // [16*COT][S3] packed projection codes
    unsigned char *t1 = lds + a.off_t1;
    unsigned char *t2 = lds + a.off_t2;
    const int slot1 = a.slot1, slot2 = a.slot2;

    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(a.x), 0, a.N * a.H * W * cin, kBufFlags);

    const int KWe = a.KWe, KWp = a.KWp, S3 = a.S3;
    const int G1 = a.G1, G2 = a.G2, G3 = a.G3;
    const int units1 = NP * G1, units2 = NP * G2;
    const bool prelu_p = a.np != nullptr;

    // ---- phase 0: every global load of the prologue leaves first, the index tables and the zero
    // cells are made while they fly, then the loaded values go to LDS -------------------------------
    // the band's existing input rows: one contiguous run of the NHWC tensor, 8-byte pieces
    constexpr int NX = 4;
    const int xtotal = np1 * cin;  // multiple of 8
    const int xbase = ((img * a.H + rlo) * W) * cin;
    v2i xv[NX];
#pragma unroll
    for (int q = 0; q < NX; ++q) {
        const int o = (tid + q * kPlThreads) * 8;
        xv[q] = __builtin_amdgcn_raw_buffer_load_b64(rx, o < xtotal ? xbase + o : kOobOffset, 0, 0);
    }
    // the packed codes and the parameters of this wavefront's first plane
    auto load_w1 = [&](int u, uint32_t(&w)[KSE]) __attribute__((always_inline)) {
        const int pl = G1 == 1 ? u : u / G1;
        const uint32_t *row = a.we + (long long)(16 * pl + j) * KWe;
#pragma unroll
        for (int ks = 0; ks < KSE; ++ks) {
            const int kw = 4 * ks + g;
            const bool ok = kw < KWe;
            const uint32_t v = row[ok ? kw : 0];
            w[ks] = ok ? v : 0u;
        }
    };
    auto load_par = [&](const int32_t *B, const int32_t *M, const int32_t *Nn, const int32_t *S, int pl,
                        PlRawPar &r) __attribute__((always_inline)) {
        const int c = 16 * pl + 4 * g;
        r.b = *reinterpret_cast<const v4i *>(B + c);
        r.m = *reinterpret_cast<const v4i *>(M + c);
        r.s = *reinterpret_cast<const v4i *>(S + c);
        if (PRELU) r.n = *reinterpret_cast<const v4i *>((Nn ? Nn : M) + c);
    };
    auto make_par = [&](const PlRawPar &r, v4i(&par)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) par[i] = requant_params(r.b[i], r.m[i], r.n[i], r.s[i], PRELU);
    };
    uint32_t w1n[KSE];
    PlRawPar rawe, rawd;
    v4i *parl = reinterpret_cast<v4i *>(lds + a.off_par);  // [2][chid] parameters of the expansion, of the depthwise layer
    load_w1(min(wave, units1 - 1), w1n);
    int qe[4], qd[4];  // a channel of the two layers
    auto load_q = [&](const unsigned c) __attribute__((always_inline)) {
        // (one of two pointers, not a load under a condition: that waits for every load in flight)
        const int32_t *ne = PRELU && a.ne ? a.ne : a.me, *nd = PRELU && a.nd ? a.nd : a.md;
        qe[0] = a.be[c]; qe[1] = a.me[c]; qe[2] = ne[c]; qe[3] = a.se[c];
        qd[0] = a.bd[c]; qd[1] = a.md[c]; qd[2] = nd[c]; qd[3] = a.sd[c];
    };
    if constexpr (!PARL) {
        const int u = min(wave, units1 - 1), u2 = min(wave, units2 - 1);
        load_par(a.be, a.me, a.ne, a.se, G1 == 1 ? u : u / G1, rawe);
        load_par(a.bd, a.md, a.nd, a.sd, G2 == 1 ? u2 : u2 / G2, rawd);
    } else {
        load_q(min(tid, chid - 1));
    }
    // the projection's parameters: one channel per thread
    int pbp, pmp, pnp, psp;
    {
        const int c = min(tid, cout - 1);
        pbp = a.bp[c]; pmp = a.mp[c]; psp = a.sp[c];
        pnp = prelu_p ? a.np[c] : 0;
    }
    // depthwise weights, dword pieces
    constexpr int NWD = 5;
    const uint32_t *wd4 = reinterpret_cast<const uint32_t *>(a.wd);
    const int nwd = (9 * chid) >> 2;
    uint32_t wdv[NWD];
#pragma unroll
    for (int q = 0; q < NWD; ++q) wdv[q] = wd4[min(tid + q * kPlThreads, nwd - 1)];
    asm volatile("" ::: "memory");

    {
        // (loops of one or two rounds: unrolled by the compiler they cost the prologue 4 KB of code and up to 1.5 us)
        // (pixels beyond the band land in a spare cell behind the plane's rows)
#pragma clang loop unroll(disable) vectorize(disable)
        for (int p = tid; p < nt1 * 16; p += kPlThreads) {
            const int row = fast_div(p, a.by_w), col = p - mul24(row, W);
            o1[p] = (uint16_t)(p < np1 ? mul24(rv0 + row, W2) + col + 1 : a.RI * W2);
        }
#pragma clang loop unroll(disable) vectorize(disable)
        for (int p = tid; p < nt2 * 16; p += kPlThreads) {
            const int pc = min(p, np2 - 1);
            const int oy = fast_div(pc, a.by_wo), ox = pc - mul24(oy, Wo);
            o2[p] = (uint16_t)(mul24(oy * s, W2) + ox * s);
        }
        // zero cells of the expansion planes: the two border columns of every row in use and the
        // rows outside the image
        const int ninv = rib - nvr;
        const int per = 2 * rib + ninv * W;
        const v4i zero4 = {0, 0, 0, 0};
#pragma clang loop unroll(disable) vectorize(disable)
        for (int e = tid; e < per; e += kPlThreads) {
            int cell;
            if (e < 2 * rib) {
                cell = mul24(e >> 1, W2) + ((e & 1) ? W + 1 : 0);
            } else {
                const int q = e - 2 * rib;
                const int ir = fast_div(q, a.by_w), col = q - mul24(ir, W);
                // invalid rows: those before rv0, then those from rv0 + nvr on
                const int row = ir < rv0 ? ir : ir + nvr;
                cell = mul24(row, W2) + col + 1;
            }
            unsigned char *dst = t1 + cell * 16;
            for (int pl = 0; pl < NP; ++pl) *reinterpret_cast<v4i *>(dst + pl * slot1) = zero4;
        }
    }
    {
        const int pieces = cin >> 3;
#pragma unroll
        for (int q = 0; q < NX; ++q) {
            const int pc = tid + q * kPlThreads;
            if (pc * 8 < xtotal) {
                const int px = fast_div(pc, a.by_xp);
                *reinterpret_cast<v2i *>(xs + mul24(px, cinp) + 8 * (pc - mul24(px, pieces))) = xv[q];
            }
        }
#pragma clang loop unroll(disable) vectorize(disable)
        for (int o = (tid + NX * kPlThreads) * 8; o < xtotal; o += kPlThreads * 8) {
            const v2i v = __builtin_amdgcn_raw_buffer_load_b64(rx, xbase + o, 0, 0);
            const int pc = o >> 3;
            const int px = fast_div(pc, a.by_xp);
            *reinterpret_cast<v2i *>(xs + mul24(px, cinp) + 8 * (pc - mul24(px, pieces))) = v;
        }
        if constexpr (PARL) {
#pragma clang loop unroll(disable) vectorize(disable)
            for (int c = tid; c < chid; c += kPlThreads) {
                if (c != tid) load_q(c);
                parl[c] = requant_params(qe[0], qe[1], qe[2], qe[3], PRELU);
                parl[chid + c] = requant_params(qd[0], qd[1], qd[2], qd[3], PRELU);
            }
        }
        if (tid < 16 * a.COT) pp[tid] = tid < cout ? requant_params(pbp, pmp, pnp, psp, prelu_p) : v4i{0, 0, 0, 1};
#pragma unroll
        for (int q = 0; q < NWD; ++q) {
            const int i = tid + q * kPlThreads;
            if (i < nwd) reinterpret_cast<uint32_t *>(wdl)[i] = wdv[q];
        }
#pragma clang loop unroll(disable) vectorize(disable)
        for (int i = tid + NWD * kPlThreads; i < nwd; i += kPlThreads) reinterpret_cast<uint32_t *>(wdl)[i] = wd4[i];
    }
    __syncthreads();
    PL_STAMP(1);

    const int lo_e = in_vgpr(a.lo_e), hi_e = in_vgpr(a.hi_e);
    const int lo_d = in_vgpr(a.lo_d), hi_d = in_vgpr(a.hi_d);
    const v4i zero4 = {0, 0, 0, 0};

    // ---- phase 1: expansion of the owned planes -----------------------------------------------------
    {
        const int tpg = G1 == 1 ? nt1 : (nt1 + G1 - 1) / G1;
        for (int u = wave; u < units1; u += kPlWaves) {
            v4i A[KSE];
#pragma unroll
            for (int ks = 0; ks < KSE; ++ks) A[ks] = decode_word(w1n[ks]);
            const int pl = G1 == 1 ? u : u / G1;
            const int grp = u - pl * G1;
            v4i par[4];
            if constexpr (!PARL) {
                make_par(rawe, par);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) par[r] = parl[16 * pl + 4 * g + r];
            }
            {   // the next unit's codes and parameters fly during this one
                const int un = min(u + kPlWaves, units1 - 1);
                load_w1(un, w1n);
                if constexpr (!PARL) load_par(a.be, a.me, a.ne, a.se, G1 == 1 ? un : un / G1, rawe);
            }
            unsigned char *t1p = t1 + pl * slot1 + 4 * g;
            const int pt0 = grp * tpg, pt1 = min((grp + 1) * tpg, nt1);
            // (PReLU: the biases are what the accumulators start from)
            const v4i cinit = PRELU ? v4i{par[0][0], par[1][0], par[2][0], par[3][0]} : zero4;
            // NTL pixel tiles at once: independent chains for the matrix cores and the epilogue
            auto tiles = [&](auto mode, auto ntl, int pt) __attribute__((always_inline)) {
                constexpr int FORM = decltype(mode)::value;
                constexpr int NTL = decltype(ntl)::value;
                v4i d[NTL];
                int cell[NTL], p[NTL];
#pragma unroll
                for (int i = 0; i < NTL; ++i) {
                    p[i] = (pt + i) * 16 + j;
                    const int8_t *xp = xs + __umul24(p[i], cinp) + 16 * g;
                    cell[i] = o1[p[i]];
                    d[i] = cinit;
#pragma unroll
                    for (int ks = 0; ks < KSE; ++ks)
                        d[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[ks], *reinterpret_cast<const v4i *>(xp + 64 * ks), d[i], 0, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < NTL; i += 2) {  // two pixel tiles at a time; a tile alone is its own partner
                    uint32_t q0, q1;
                    requant_pair4<FORM, true>(d[i], d[i + (NTL > 1)], par, lo_e, hi_e, q0, q1);
                    *reinterpret_cast<uint32_t *>(t1p + cell[i] * 16) = q0;
                    if constexpr (NTL > 1) *reinterpret_cast<uint32_t *>(t1p + cell[i + 1] * 16) = q1;
                }
            };
            auto run = [&](auto mode) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < 4; ++r) par[r][3] -= pair_shift_less(decltype(mode)::value);
                int pt = pt0;
                for (; pt + 4 <= pt1; pt += 4) tiles(mode, PlMode<4>{}, pt);
                if (pt + 2 <= pt1) {
                    tiles(mode, PlMode<2>{}, pt);
                    pt += 2;
                }
                if (pt < pt1) tiles(mode, PlMode<1>{}, pt);
            };
            const int form = pair_form<PRELU>(min_shift(par), a.lo_e, a.hi_e);
            if constexpr (PRELU) {
                if (form == kPairPreluFull) run(PlMode<kPairPreluFull>{});
                else run(PlMode<kPairPreluAny>{});
            } else {
                if (form == kPairRelu) run(PlMode<kPairRelu>{});
                else if (form == kPairFull || form == kPairLow) run(PlMode<kPairLow>{});
                else if (form == kPairClamp) run(PlMode<kPairClamp>{});
                else run(PlMode<kPairAny>{});
            }
        }
    }
    PL_STAMP(2);
    if (G1 != 1 || G2 != 1) __syncthreads();

    // The projection's packed codes go to LDS while phase 2 runs: loads now, stores behind the loop.
    // Wide rows (whole 16-byte pieces): the matrix is one flat run of pieces.
    // (NW3 pieces per thread cover 960 x 320 whatever the wavefronts; more pieces would only hold registers
    // through phase 2, and with 16 wavefronts spill)
    constexpr int NW3 = (80 + NW - 1) / NW;
    const bool w3wide = (KWp & 3) == 0 && (reinterpret_cast<uintptr_t>(a.wp) & 15) == 0;
    const int kq3 = KWp >> 2;
    const int n3 = w3wide ? cout * kq3 : cout * KWp;  // pieces: 16 bytes or one word
    v4i w3v[NW3];
    if (w3wide) {
#pragma unroll
        for (int q = 0; q < NW3; ++q)
            w3v[q] = *reinterpret_cast<const v4i *>(a.wp + 4 * (long long)min(tid + q * kPlThreads, n3 - 1));
    } else {
#pragma unroll
        for (int q = 0; q < NW3; ++q) w3v[q][0] = (int)a.wp[min(tid + q * kPlThreads, n3 - 1)];
    }
    asm volatile("" ::: "memory");  // (the loads leave here; where registers are short they would sink below the filter)

    // ---- phase 2: depthwise 3x3 of the owned planes on the matrix cores ------------------------------
    {
        const int li = lane & 15;
        int toff[3];  // byte offset of the lane's tap in each tap group (tap 8 again where there is none)
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int tap = min(4 * q + g, 8);
            toff[q] = ((tap / 3) * W2 + tap % 3) * 16;
        }
        const int tpg = G2 == 1 ? nt2 : (nt2 + G2 - 1) / G2;
        for (int u = wave; u < units2; u += kPlWaves) {
            const int pl = G2 == 1 ? u : u / G2;
            const int grp = u - pl * G2;
            // A operands: for tap group q the weight of channel 16*pl + li under tap 4q + g at byte li
            // of the lane's 16, zero elsewhere
            v4i adw[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int tap = 4 * q + g;
                const uint32_t wb = tap < 9 ? (uint32_t)(uint8_t)wdl[mul24(tap, chid) + 16 * pl + li] : 0u;
                const uint32_t val = wb << (8 * (li & 3));
                adw[q] = v4i{(li >> 2) == 0 ? (int)val : 0, (li >> 2) == 1 ? (int)val : 0,
                             (li >> 2) == 2 ? (int)val : 0, (li >> 2) == 3 ? (int)val : 0};
            }
            v4i par[4];
            if constexpr (PARL) {
#pragma unroll
                for (int r = 0; r < 4; ++r) par[r] = parl[chid + 16 * pl + 4 * g + r];
            } else {
                make_par(rawd, par);
                const int un = min(u + kPlWaves, units2 - 1);
                load_par(a.bd, a.md, a.nd, a.sd, G2 == 1 ? un : un / G2, rawd);
            }
            const v4i cinit = PRELU ? v4i{par[0][0], par[1][0], par[2][0], par[3][0]} : zero4;
            const unsigned char *t1p = t1 + pl * slot1;
            unsigned char *t2p = t2 + pl * slot2 + 4 * g;
            const int pt0 = grp * tpg, pt1 = min((grp + 1) * tpg, nt2);
            auto tiles = [&](auto mode, auto ntl, int pt) __attribute__((always_inline)) {
                constexpr int FORM = decltype(mode)::value;
                constexpr int NTL = decltype(ntl)::value;
                v4i d[NTL];
#pragma unroll
                for (int i = 0; i < NTL; ++i) {
                    const unsigned char *src = t1p + o2[(pt + i) * 16 + j] * 16;
                    d[i] = cinit;
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        d[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(adw[q], *reinterpret_cast<const v4i *>(src + toff[q]), d[i], 0, 0, 0);
                }
                // (the reads of every tile are complete before the first write: with one owner per
                // plane the output may land in a slot this wavefront has consumed, never in its own)
#pragma unroll
                for (int i = 0; i < NTL; i += 2) {  // two pixel tiles at a time; a tile alone is its own partner
                    uint32_t q0, q1;
                    requant_pair4<FORM, true>(d[i], d[i + (NTL > 1)], par, lo_d, hi_d, q0, q1);
                    *reinterpret_cast<uint32_t *>(t2p + ((pt + i) * 16 + j) * 16) = q0;
                    if constexpr (NTL > 1) *reinterpret_cast<uint32_t *>(t2p + ((pt + i + 1) * 16 + j) * 16) = q1;
                }
            };
            auto run = [&](auto mode) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < 4; ++r) par[r][3] -= pair_shift_less(decltype(mode)::value);
                int pt = pt0;
                for (; pt + 4 <= pt1; pt += 4) tiles(mode, PlMode<4>{}, pt);
                if (pt + 2 <= pt1) {
                    tiles(mode, PlMode<2>{}, pt);
                    pt += 2;
                }
                if (pt < pt1) tiles(mode, PlMode<1>{}, pt);
            };
            const int form = pair_form<PRELU>(min_shift(par), a.lo_d, a.hi_d);
            if constexpr (PRELU) {
                if (form == kPairPreluFull) run(PlMode<kPairPreluFull>{});
                else run(PlMode<kPairPreluAny>{});
            } else {
                if (form == kPairRelu) run(PlMode<kPairRelu>{});
                else if (form == kPairFull || form == kPairLow) run(PlMode<kPairLow>{});
                else if (form == kPairClamp) run(PlMode<kPairClamp>{});
                else run(PlMode<kPairAny>{});
            }
        }
    }
    // the projection's codes: rows of S3 words in LDS
    if (w3wide) {
#pragma unroll
        for (int q = 0; q < NW3; ++q) {
            const int i = tid + q * kPlThreads;
            if (i < n3) {
                const int row = fast_div(i, a.by_kq);
                *reinterpret_cast<v4i *>(w3l + mul24(row, S3) + 4 * (i - mul24(row, kq3))) = w3v[q];
            }
        }
#pragma clang loop unroll(disable) vectorize(disable)
        for (int i = tid + NW3 * kPlThreads; i < n3; i += kPlThreads) {
            const int row = fast_div(i, a.by_kq);
            *reinterpret_cast<v4i *>(w3l + mul24(row, S3) + 4 * (i - mul24(row, kq3))) = *reinterpret_cast<const v4i *>(a.wp + 4 * (long long)i);
        }
    } else {
#pragma unroll
        for (int q = 0; q < NW3; ++q) {
            const int i = tid + q * kPlThreads;
            if (i < n3) {
                const int row = fast_div(i, a.by_kq);
                w3l[mul24(row, S3) + (i - mul24(row, KWp))] = (uint32_t)w3v[q][0];
            }
        }
#pragma clang loop unroll(disable) vectorize(disable)
        for (int i = tid + NW3 * kPlThreads; i < n3; i += kPlThreads) {
            const int row = fast_div(i, a.by_kq);
            w3l[mul24(row, S3) + (i - mul24(row, KWp))] = a.wp[i];
        }
        // words between the row's end and the next multiple of four are read as codes: zero
#pragma clang loop unroll(disable) vectorize(disable)
        for (int r = tid; r < cout; r += kPlThreads)
            for (int w = KWp; w < ((KWp + 3) & ~3); ++w) w3l[r * S3 + w] = 0u;
    }
    PL_STAMP(3);
    __syncthreads();
    PL_STAMP(4);

    // ---- phase 3: projection ---------------------------------------------------------------------------
    // The k dimension is walked in groups of 16 packed words (256 hidden channels): k step 4*gi + e
    // of lane group kg covers plane 16*gi + 4*kg + e, so that a lane's codes of four k steps are one
    // 16-byte LDS read.
    {
        const int lo_p = in_vgpr(a.lo_p), hi_p = in_vgpr(a.hi_p);
        const __amdgpu_buffer_rsrc_t ry =
            __builtin_amdgcn_make_buffer_rsrc(a.y, 0, a.N * a.Ho * Wo * cout, kBufFlags);
        const int obase = (img * a.Ho + ro0) * Wo;  // first output pixel of the band
        const int TPG3 = a.TPG3;
        const int units3 = a.COT * G3;
        const int R4 = (KWp + 3) & ~3;
        const int ng3 = (KWp + 15) >> 4;
        // TPG pixel tiles of one output-channel tile per unit (tiles beyond the band are computed on
        // whatever the planes hold there and never stored: no branch in the k loop)
        auto unit = [&](auto tpg, int ct, int pt0) __attribute__((always_inline)) {
            constexpr int TPG = decltype(tpg)::value;
            v4i acc[TPG];
#pragma unroll
            for (int i = 0; i < TPG; ++i) acc[i] = zero4;
            const unsigned char *bq = t2 + (pt0 * 16 + j) * 16;
            const uint32_t *wrow = w3l + mul24(16 * ct + j, S3);
            // One k step ahead: the B operands of the next step and the codes of the next group are
            // on their way while this step's codes are decoded and its MFMAs issue.  Steps past the
            // last plane read the last plane against zero codes (the rows are zero-padded to R4 and
            // groups past R4 take zeros), the reads past the last step go nowhere.
            auto load_b = [&](v4i(&B)[TPG], int plane) __attribute__((always_inline)) {
                const unsigned char *bp = bq + mul24(min(plane, NP - 1), slot2);
#pragma unroll
                for (int i = 0; i < TPG; ++i) B[i] = *reinterpret_cast<const v4i *>(bp + i * 256);
            };
            auto load_w = [&](int wo) __attribute__((always_inline)) {
                v4i wv = *reinterpret_cast<const v4i *>(wrow + min(wo, R4 - 4));
                if (wo >= R4) wv = zero4;
                return wv;
            };
            v4i Bn[TPG];
            load_b(Bn, 4 * g);
            v4i wn = load_w(4 * g);
            for (int gi = 0; gi < ng3; ++gi) {
                const int wo = 16 * gi + 4 * g;
                const v4i wv = wn;
                wn = load_w(wo + 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v4i Bc[TPG];
#pragma unroll
                    for (int i = 0; i < TPG; ++i) Bc[i] = Bn[i];
                    load_b(Bn, e < 3 ? wo + e + 1 : wo + 16);
                    const v4i A = decode_word((uint32_t)wv[e]);
#pragma unroll
                    for (int i = 0; i < TPG; ++i)
                        acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, Bc[i], acc[i], 0, 0, 0);
                }
            }
            const int c = 16 * ct + 4 * g;
            const bool cok = c < cout;
            v4i pr[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) pr[r] = pp[c + r];
            // two pixel tiles at a time (a tile alone is its own partner; tiles beyond the band are not stored)
            auto finish = [&](auto form) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < 4; ++r) pr[r][3] -= pair_shift_less(decltype(form)::value);
#pragma unroll
                for (int i = 0; i < TPG; i += 2) {
                    uint32_t q[2];
                    requant_pair4<decltype(form)::value>(acc[i], acc[i + (TPG > 1)], pr, lo_p, hi_p, q[0], q[1]);
#pragma unroll
                    for (int k = 0; k < (TPG > 1 ? 2 : 1); ++k) {
                        const int p = (pt0 + i + k) * 16 + j;
                        if (a.add_res) {
                            // stride 1 and cin == cout: the block input at the same pixel, still in LDS
                            const uint32_t res = *reinterpret_cast<const uint32_t *>(
                                xs + mul24((1 - rv0) * W + min(p, np2 - 1), cinp) + (cok ? c : 0));
                            q[k] = add_sat_i8x4(q[k], res);
                        }
                        __builtin_amdgcn_raw_buffer_store_b32((int)q[k], ry, cok && p < np2 ? (obase + p) * cout + c : kOobOffset, 0, 0);
                    }
                }
            };
            if (prelu_p) {
                finish(PlMode<kPairPreluAny>{});
            } else if constexpr (TPG == 1) {
                finish(PlMode<kPairAny>{});  // (one tile does not pay for the test)
            } else {
                const int form = pair_form<false>(min_shift(pr), a.lo_p, a.hi_p);
                if (form == kPairFull) finish(PlMode<kPairFull>{});
                else finish(PlMode<kPairAny>{});
            }
        };
        for (int u = wave; u < units3; u += kPlWaves) {
            const int ct = G3 == 1 ? u : u / G3;
            const int pt0 = (u - ct * G3) * TPG3;
            if (pt0 >= nt2) continue;
            if (TPG3 == 8) unit(PlMode<8>{}, ct, pt0);
            else if (TPG3 == 4) unit(PlMode<4>{}, ct, pt0);
            else if (TPG3 == 2) unit(PlMode<2>{}, ct, pt0);
            else unit(PlMode<1>{}, ct, pt0);
        }
    }
    PL_STAMP(6);
    __builtin_amdgcn_s_waitcnt(0);
    PL_STAMP(7);
}

using PlanesFn = void (*)(const PlanesArgs);

static inline int align16i(int v) { return (v + 15) & ~15; }

// Plans the kernel for the shape in `a` (N, H, W, Ho, Wo, cin, chid, cout, stride set): band height,
// unit split of the three phases, LDS layout.  False if the shape does not fit.
bool plan_planes(PlanesArgs &a, size_t &lds, int &grid, int &kse)
{
    const int cin = a.cin, chid = a.chid, cout = a.cout, s = a.stride;
    if (cin % 8 != 0 || chid % 16 != 0 || cout % 4 != 0 || cin > 192) return false;
    if ((long long)a.N * a.H * a.W * cin >= (long long)kOobOffset) return false;
    if ((long long)a.N * a.Ho * a.Wo * cout >= (long long)kOobOffset) return false;
    if (a.W > 4096) return false;
    kse = (cin + 63) / 64;
    const int NP = chid / 16, COT = (cout + 15) / 16;
    const int KS3 = (chid + 63) / 64;
    const int KWp = chid / 16;
    int cinp = align16i(cin);
    if (((cinp >> 4) & 1) == 0) cinp += 16;  // odd number of 16-byte pieces per pixel: no bank conflicts
    const int W2 = a.W + 2;
    const int kLdsMax = 160 * 1024;
    int only_nw = 0;
#ifdef PROM_TIMELINE
    if (const char *env = getenv("PROM_PLANES_NW")) only_nw = atoi(env);
#endif

    // Candidates: wavefronts per workgroup (more of them keep the vector ALU busier while others
    // wait on LDS and the matrix cores; the planes must divide among them), the padding of the
    // projection's code rows in LDS (against bank conflicts; dropped where LDS is short), the band
    // height.  The estimate counts wavefront instructions: a SIMD issues one every `cpi` cycles.
    struct Pick { int nw, pad, R, G, G3, TPG3; double cost; } best = {0, 0, 0, 0, 0, 0, 0};
    for (int nw : {8, 12, 16}) {
        if (only_nw && nw != only_nw) continue;
        if (cout > 64 * nw) continue;
        const double cpi = nw == 8 ? 4.9 : nw == 12 ? 4.45 : 3.95;  // measured: phases 1 and 2 of 14x14x384
        // few planes: spread the pixel tiles of a plane over wavefronts (about 3 units per wavefront)
        const int G = NP >= nw ? 1 : (3 * nw + NP - 1) / NP;
        for (int pad : {4, 0}) {
            const int s3 = ((KWp + 3) & ~3) + pad;
            for (int R = 1; R <= a.Ho; ++R) {
                const int RI = (R - 1) * s + 3;
                const long long np1 = (long long)RI * a.W, np2 = (long long)R * a.Wo;
                if (np1 > 8192 || (long long)RI * W2 >= 65535) break;
                const int nt1 = (int)((np1 + 15) / 16), nt2 = (int)((np2 + 15) / 16);
                const int plane1 = (RI * W2 + 1) * 16, plane2 = nt2 * 256;
                long long bytes = align16i(nt1 * 16 * cinp + 64 * kse + 64);  // xs
                bytes += align16i(nt1 * 32) + align16i(nt2 * 32);             // o1, o2
                bytes += COT * 256;                                           // pp
                bytes += 16LL * COT * s3 * 4;                                 // w3l
                bytes += align16i(9 * chid);                                  // wdl
                if (G == 1) bytes += (long long)(NP + nw) * (plane1 > plane2 ? plane1 : plane2);
                else bytes += (long long)NP * (plane1 + plane2);
                if (bytes + 2048 > kLdsMax) break;
                // phase 3: 1, 2, 4 or 8 pixel tiles of one output-channel tile per unit
                int g3 = 1, tpg3 = 1;
                double c3 = 0;
                for (int t = 1; t <= 8; t *= 2) {
                    const int gg = (nt2 + t - 1) / t;
                    const long long rounds = ((long long)COT * gg + nw - 1) / nw;
                    const double c = (double)rounds * (KS3 * (20.0 + 3.0 * t) + 40.0 * t + 40.0);
                    if (t == 1 || c < c3) {
                        c3 = c;
                        g3 = gg;
                        tpg3 = t;
                    }
                }
                // phases 1 and 2: the SIMDs share the units' instructions (a wavefront that is done
                // leaves its SIMD to the others, so uneven plane counts cost little); spread planes
                // pay a barrier
                const double per1 = 60.0 + ((nt1 + G - 1) / G) * (38.0 + 3.0 * kse);
                const double per2 = 80.0 + ((nt2 + G - 1) / G) * 42.0;
                const double units = (double)NP * G;
                double work = cpi * units * (per1 + per2) / 4.0 + (nw / 4) * cpi * c3;
                if (G > 1) work *= 1.15;
                const int bands = (a.Ho + R - 1) / R;
                const long long rounds = ((long long)a.N * bands + 255) / 256;
                // fixed part: launch, the prologue's memory round trip, barriers, the drain
                const double cost = (double)rounds * (12000.0 + work);
                if (best.nw == 0 || cost < best.cost) best = {nw, pad, R, G, g3, tpg3, cost};
            }
        }
    }
    if (best.nw == 0) return false;
    const int R = best.R, G = best.G, nw = best.nw;
    a.NW = nw;
    a.cost = best.cost;
    a.R = R;
    a.RI = (R - 1) * s + 3;
    a.bands = (a.Ho + R - 1) / R;
    a.NP = NP;
    a.COT = COT;
    a.KWe = (cin + 15) / 16;
    a.KWp = KWp;
    a.KS3 = KS3;
    a.cinp = cinp;
    a.by_w = div_magic(a.W);
    a.by_wo = div_magic(a.Wo);
    a.by_xp = div_magic(cin >> 3);
    a.G1 = a.G2 = G;
    a.G3 = best.G3;
    a.TPG3 = best.TPG3;
    const int np1 = a.RI * a.W, np2 = R * a.Wo;
    const int nt1 = (np1 + 15) / 16, nt2 = (np2 + 15) / 16;
    const int plane1 = (a.RI * W2 + 1) * 16, plane2 = nt2 * 256;
    int off = align16i(nt1 * 16 * cinp + 64 * kse + 64);
    a.off_o1 = off; off += align16i(nt1 * 32);
    a.off_o2 = off; off += align16i(nt2 * 32);
    a.off_pp = off; off += COT * 256;
    a.S3 = ((KWp + 3) & ~3) + best.pad;
    a.off_w3 = off; off += 16 * COT * a.S3 * 4;
    a.off_wd = off; off += align16i(9 * chid);
    if (G == 1) {
        const int slot = plane1 > plane2 ? plane1 : plane2;
        a.slot1 = a.slot2 = slot;
        a.off_t2 = off;
        a.off_t1 = off + nw * slot;
        off += (NP + nw) * slot;
    } else {
        a.slot1 = plane1;
        a.slot2 = plane2;
        a.off_t1 = off; off += NP * plane1;
        a.off_t2 = off; off += NP * plane2;
    }
    a.off_par = 0;
    if (off + 2 * chid * 16 + 2048 <= kLdsMax) {
        a.off_par = off;
        off += 2 * chid * 16;
    }
    off += 2048;  // phase 3 reads up to 8 pixel tiles from a unit's first one, whatever the band holds
    lds = (size_t)off;
    const long long gsz = (long long)a.N * a.bands;
    if (gsz > (1LL << 30)) return false;
    grid = (int)gsz;
    return true;
}

template <int NW, bool PARL> static PlanesFn planes_fn_nw(int kse, bool prelu)
{
    switch (kse) {
    case 1: return prelu ? &block_planes_kernel<1, true, NW, PARL> : &block_planes_kernel<1, false, NW, PARL>;
    case 2: return prelu ? &block_planes_kernel<2, true, NW, PARL> : &block_planes_kernel<2, false, NW, PARL>;
    default: return prelu ? &block_planes_kernel<3, true, NW, PARL> : &block_planes_kernel<3, false, NW, PARL>;
    }
}
template <bool PARL> static PlanesFn planes_fn(int kse, bool prelu, int nw)
{
    return nw == 16   ? planes_fn_nw<16, PARL>(kse, prelu)
           : nw == 12 ? planes_fn_nw<12, PARL>(kse, prelu)
                      : planes_fn_nw<8, PARL>(kse, prelu);
}

int launch_planes(const PlanesArgs &a, size_t lds, int grid, int kse, void *stream)
{
    const bool prelu = a.ne != nullptr || a.nd != nullptr;
    const PlanesFn fn = a.off_par ? planes_fn<true>(kse, prelu, a.NW) : planes_fn<false>(kse, prelu, a.NW);
    static std::mutex mu;
    static std::vector<PlanesFn> attr_done;
    {
        std::lock_guard<std::mutex> lock(mu);
        bool done = false;
        for (PlanesFn f : attr_done) done |= f == fn;
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
    PlanesArgs args = a;
    args.by_kq = div_magic((a.KWp & 3) == 0 && ((uintptr_t)a.wp & 15) == 0 ? a.KWp >> 2 : a.KWp);  // (w3wide in the kernel)
    void *kargs[] = {&args};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(fn), dim3(grid), dim3(64 * a.NW), kargs, lds,
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
extern "C" double prom_debug_planes_cost(int n, int h, int w, int cin, int chid, int cout, int stride)
{
    prom::PlanesArgs a = {};
    a.N = n; a.H = h; a.W = w; a.Ho = (h - 1) / stride + 1; a.Wo = (w - 1) / stride + 1;
    a.cin = cin; a.chid = chid; a.cout = cout; a.stride = stride;
    size_t lds = 0; int grid = 0, kse = 0;
    return prom::plan_planes(a, lds, grid, kse) ? a.cost : -1.0;
}
extern "C" int prom_debug_pl_stamps(unsigned long long *host)
{
    if (hipDeviceSynchronize() != hipSuccess) return PROM_EHIP;
    return hipMemcpyFromSymbol(host, HIP_SYMBOL(prom::g_pl_stamps), sizeof(unsigned long long) * 256 * 8) == hipSuccess ? PROM_OK : PROM_EHIP;
}
#endif
