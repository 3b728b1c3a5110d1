// Ternary pointwise convolution with the k loop outermost over a workgroup tile of pixels x output channels:
// wide layers (hundreds to thousands of input AND output channels: the 1x1 layers of ResNeXt and RegNet,
// paper Section 5) and, launched alone, the expansion layers of MobileNetV2.
//
// The streaming kernel (prom_pw_stream.h) keeps the decoded weights of a chunk of output channels
// for ALL input channels in LDS and streams the pixels past them once per chunk: every MFMA reads a
// weight fragment from LDS (256 B per cycle and CU at the matrix cores' rate, twice what LDS gives), the
// activations pass the texture addresser once per chunk, and a workgroup decodes up to 64 KB of
// fragments before its first MFMA.  Here
//   - a wavefront owns PT x 4 accumulator tiles: 16*PT pixels x 64 output channels of the workgroup's
//     16*PT x 128 or 256.  It decodes the packed codes of its own 64 channels in registers, 48 instructions per
//     k step against 4*PT MFMAs of 16 cycles, so no decoded weight passes through LDS;
//   - everything comes from global memory in lane order: four neighbouring lanes read one 64-byte run.  The
//     texture addresser takes 24 to 30 cycles for such an instruction of 1 KB, and 65 for one in operand
//     order (16 rows, neighbouring lanes in different lines), however few bytes its lanes load: a first
//     version that fetched its codes as one dword per lane in operand order took 33 us (4 pixel tiles) and
//     57 us (2) for 512 -> 1024 at 12544 and 25088 pixels, where this one takes 14.7 and 25.9;
//   - the packed codes of four k steps (64 bytes per channel) go through 4 KB of LDS of the wavefront's own
//     into operand order; no barrier, LDS operations of a wavefront keep their order;
//   - the activations of a k step (64 bytes per pixel) are fetched by all threads D k steps ahead in
//     registers and put into one of two LDS slabs, from which every wavefront reads its B operands: 1 KB
//     per 4 MFMAs, half of what LDS delivers.  The 16-byte pieces of a pixel are exchanged by the pixel's
//     index, so that neither the writes nor the operand reads meet bank conflicts.  One barrier per k step,
//     on LDS traffic only;
//   - workgroups that share a pixel tile are neighbours in the XCD-aware order;
//   - the epilogue requantises two pixels at a time (requant_pair4), assembles the tile in LDS and writes
//     whole rows in 16-byte pieces; the skip connection is read and added in the same pieces.
//
// What bounds it: the chain of a k step in a wavefront (barrier, first operand reads, 128 to 512 cycles of
// MFMAs with the decode between them, barrier: 0.27, 0.30 and 0.43 us with 2, 4 and 8 pixel tiles) and the 4 us
// around the k loop, which 2 to 4 workgroups per CU overlap: 14x14 1024 -> 1024 at batch 128 runs at 1.5 Pop/s
// (35 us; 58 with the streaming kernel, 53 with the kernel this one replaced, which fetched its pixels in
// operand order and passed its decoded weights through LDS).  Without the decode (wrong results) the layers
// take 4 to 7 % less, without the requantisation 10 %.
#include "prom_pw_gemm.h"

namespace prom {

// Workgroup barrier that orders LDS traffic only.  __syncthreads() carries a release fence over
// every address space, which makes the compiler wait for ALL outstanding global loads -- here the
// pixels and codes requested for the k steps ahead.  The wavefront's LDS writes are complete when
// lgkmcnt reaches 0 (LDS operations of a wavefront finish in order).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// A wavefront's packed codes of four k steps in LDS: [k step][64 channels][16 bytes], the k steps
// 32 bytes further apart than they need (bank conflicts of the writes).
constexpr int kGemmCodeStep = 64 * 16 + 32;
constexpr int kGemmCodes = 4 * kGemmCodeStep;

template <int PT, int NW> struct GemmGeom {
    static constexpr int NT = 64 * NW;            // threads
    static constexpr int TM = 16 * PT;            // pixels of a workgroup's tile
    static constexpr int TN = 64 * NW;            // output channels of it, 64 per wavefront
    static constexpr int NQ = (TM * 4 + NT - 1) / NT;  // 16-byte pieces of activations per thread and k step
    static constexpr int SLAB = NQ * NT * 16;     // bytes of one k step's activations, rounded up to whole pieces per thread
    static constexpr int PITCH = TN + 16;         // bytes between pixels of the assembled tile
    static constexpr int BODY = 2 * SLAB > TM * PITCH ? 2 * SLAB : TM * PITCH;
    static constexpr size_t LDS = (size_t)TN * 16 + NW * kGemmCodes + BODY;
    // k steps of activations requested ahead, as many as the registers hold
    static constexpr int D = PT == 8 ? (NW == 2 ? 1 : 2) : PT == 4 && NW < 4 ? 2 : 4;
    static constexpr int NP = (TM * TN / 16 + NT - 1) / NT;  // 16-byte pieces of the output tile per thread
};

// a.n_chunks = column tiles of TN channels, a.wg_per_chunk = row tiles of TM pixels; requires
// K % 16 == 0, Nc % 16 == 0 and 16-byte aligned x, y, residual.
template <int PT, int NW, bool PRELU>
__global__ __launch_bounds__(64 * NW, PT == 8 ? 2 : PT == 4 ? 3 : 4) void pw_gemm_kernel(const PwArgs a)
{
    using G = GemmGeom<PT, NW>;
    constexpr int D = G::D, NQ = G::NQ;
    extern __shared__ __align__(16) unsigned char lds[];
    v4i *lpar = reinterpret_cast<v4i *>(lds);  // [TN]
    unsigned char *body = lds + G::TN * 16 + NW * kGemmCodes;  // two slabs of activations, then the assembled tile

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;

    const int lid = logical_block_id();
    const int ntile = lid % a.n_chunks;
    const int mtile = lid / a.n_chunks;
    if (mtile >= a.wg_per_chunk) return;
    const int n0 = ntile * G::TN;
    const int m0 = mtile * G::TM;
    const int K = a.K, Nc = a.Nc, KW = a.KW, KS = a.KS;

    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(a.x), 0, a.M * K, kBufFlags);
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.wq), 0, Nc * KW * 4, kBufFlags);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(a.y, 0, a.M * Nc, kBufFlags);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int8_t *>(a.residual ? a.residual : a.y), 0, a.M * Nc, kBufFlags);

    // Activations: piece idx = tid + NT*q of a slab is 16-byte slot idx & 3 of pixel idx >> 2 and holds
    // piece slot ^ ((pixel >> 1) & 3) of the pixel's 64 bytes.
    // (the piece is the same in all of a thread's pixels; xlast: the k steps in which it exists)
    const int xpiece = (tid & 3) ^ ((tid >> 3) & 3);
    const int xlast = (K - 16 * xpiece + 63) >> 6;
    unsigned xoff[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int idx = tid + G::NT * q;
        const int px = idx >> 2;
        const long long o = (long long)(m0 + px) * K + 16 * xpiece;
        xoff[q] = px < G::TM && o < (long long)kOobOffset ? (unsigned)o : (unsigned)kOobOffset;
    }
    // Codes of a group of four k steps: 64 bytes per channel.  Instruction r of a load: channel
    // 16*r + (lane >> 2) of the wavefront's 64, 16-byte piece (= k step of the group) lane & 3; channels
    // past the layer lie past the matrix and read zero, k steps past the row go out of range.
    const int wpiece = lane & 3;
    const unsigned woff = (unsigned)((n0 + 64 * wave + (lane >> 2)) * KW + 4 * wpiece) * 4u;
    const unsigned wstep = 64u * (unsigned)KW;  // 16 rows
    unsigned char *codes = lds + G::TN * 16 + wave * kGemmCodes;
    unsigned char *wput = codes + wpiece * kGemmCodeStep + (lane >> 2) * 16;
    const unsigned char *wget = codes + j * 16 + g * 4;

    // (requests past the last k step go out of range and move nothing; pieces past the end of a row are zeros,
    // so that the codes beside them, the next row's, count for nothing)
    auto load_x = [&](int ks, v4i(&v)[NQ]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            v[q] = __builtin_amdgcn_raw_buffer_load_b128(
                rx, ks < xlast ? (int)min(xoff[q] + 64u * (unsigned)ks, (unsigned)kOobOffset) : kOobOffset, 0, 0);
    };
    auto load_w = [&](int ks, v4i(&v)[4]) __attribute__((always_inline)) {  // ks: first step of the group
        const unsigned ko = ks + wpiece < KS ? 16u * (unsigned)ks : (unsigned)kOobOffset;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            v[r] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)min(woff + r * wstep + ko, (unsigned)kOobOffset), 0, 0);
    };
    auto put_w = [&](const v4i(&v)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) *reinterpret_cast<v4i *>(wput + 256 * r) = v[r];
    };
    auto get_w = [&](int d, uint32_t(&v)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = *reinterpret_cast<const uint32_t *>(wget + d * kGemmCodeStep + 256 * t);
    };
    auto put_x = [&](int slab, const v4i(&v)[NQ]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) *reinterpret_cast<v4i *>(body + slab * G::SLAB + (tid + G::NT * q) * 16) = v[q];
    };

    // Ring: slot (s % D) holds step s's activations until they are put into LDS one step early.
    v4i xr[D][NQ], wr[4];
    load_w(0, wr);
#pragma unroll
    for (int d = 0; d < D; ++d) load_x(d, xr[d]);
    int pb = 0, pm = 0, pn = 0, ps = 31;
    if (tid < G::TN) {
        const int c = min(n0 + tid, Nc - 1);
        pb = a.bias[c];
        pm = a.mult[c];
        ps = a.shift[c];
        if (PRELU) pn = a.mult_neg[c];
    }

    v4i acc[PT][4];
#pragma unroll
    for (int i = 0; i < PT; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[i][t] = v4i{0, 0, 0, 0};

    uint32_t wc[4];
    put_w(wr);
    load_w(4, wr);
    get_w(0, wc);
    put_x(0, xr[0]);
    load_x(D, xr[0]);
    if (tid < G::TN) lpar[tid] = requant_params(pb, pm, pn, ps, PRELU);
    lds_barrier();

    // One k step; d = ks % 4.  The words of the next step are read one step early; the codes of the next
    // group replace this group's once its last words have been requested (LDS operations of a wavefront
    // keep their order, and no other wavefront reads them).
    const unsigned char *bsrc = body + (j * 4 + (g ^ ((j >> 1) & 3))) * 16;
    auto step = [&](auto dtag, int ks) __attribute__((always_inline)) {
        constexpr int d = decltype(dtag)::value;
        v4i B[PT];
#pragma unroll
        for (int i = 0; i < PT; ++i) B[i] = *reinterpret_cast<const v4i *>(bsrc + (d & 1) * G::SLAB + i * 1024);
        if constexpr (d == 3) {
            put_w(wr);
            load_w(ks + 5, wr);
        }
        uint32_t wnext[4];
        get_w((d + 1) & 3, wnext);
        put_x((d + 1) & 1, xr[(d + 1) % D]);
        load_x(ks + 1 + D, xr[(d + 1) % D]);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const v4i A = decode_word(wc[t]);
#pragma unroll
            for (int i = 0; i < PT; ++i) acc[i][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, B[i], acc[i][t], 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) wc[t] = wnext[t];
        lds_barrier();
    };
    // straight-line code for four steps (a branch inside makes the compiler wait for the newest load
    // instead of the one it needs); the last KS % 4 steps one by one
    int ks0 = 0;
    for (; ks0 + 4 <= KS; ks0 += 4) {
        step(std::integral_constant<int, 0>{}, ks0);
        step(std::integral_constant<int, 1>{}, ks0 + 1);
        step(std::integral_constant<int, 2>{}, ks0 + 2);
        step(std::integral_constant<int, 3>{}, ks0 + 3);
    }
    if (ks0 < KS) {
        step(std::integral_constant<int, 0>{}, ks0);
        if (ks0 + 1 < KS) {
            step(std::integral_constant<int, 1>{}, ks0 + 1);
            if (ks0 + 2 < KS) step(std::integral_constant<int, 2>{}, ks0 + 2);
        }
    }

    // ---- epilogue ------------------------------------------------------------------------------------
    const int lo = in_vgpr(a.lo), hi = in_vgpr(a.hi);
    // output piece q of this thread: 16 bytes of channels 16*(idx % (TN/16)) of pixel idx / (TN/16)
    constexpr int PPR = G::TN / 16;
    int yoff[G::NP];
    v4i res[G::NP];
#pragma unroll
    for (int q = 0; q < G::NP; ++q) {
        const int idx = tid + G::NT * q;
        const int px = idx / PPR, c = n0 + 16 * (idx % PPR);
        const long long o = (long long)(m0 + px) * Nc + c;
        yoff[q] = c < Nc && o < (long long)kOobOffset ? (int)o : kOobOffset;
    }
    if (a.residual) {
#pragma unroll
        for (int q = 0; q < G::NP; ++q) res[q] = __builtin_amdgcn_raw_buffer_load_b128(rr, yoff[q], 0, 0);
    }
    unsigned char *sp = body + j * G::PITCH + 64 * wave + 4 * g;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        v4i par[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) par[r] = lpar[64 * wave + 16 * t + 4 * g + r];
        auto tile = [&](auto form) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 4; ++r) par[r][3] -= pair_shift_less(decltype(form)::value);
#pragma unroll
            for (int i = 0; i < PT; i += 2) {
                uint32_t o0, o1;
                requant_pair4<decltype(form)::value>(acc[i][t], acc[i + 1][t], par, lo, hi, o0, o1);
                *reinterpret_cast<uint32_t *>(sp + 16 * i * G::PITCH + 16 * t) = o0;
                *reinterpret_cast<uint32_t *>(sp + 16 * (i + 1) * G::PITCH + 16 * t) = o1;
            }
        };
        const int form = pair_form<PRELU>(min_shift(par), a.lo, a.hi);
        if constexpr (PRELU) {
            if (form == kPairPreluFull) tile(std::integral_constant<int, kPairPreluFull>{});
            else tile(std::integral_constant<int, kPairPreluAny>{});
        } else {
            if (form == kPairRelu) tile(std::integral_constant<int, kPairRelu>{});
            else if (form == kPairFull) tile(std::integral_constant<int, kPairFull>{});
            else if (form == kPairLow) tile(std::integral_constant<int, kPairLow>{});
            else tile(std::integral_constant<int, kPairAny>{});
        }
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < G::NP; ++q) {
        const int idx = tid + G::NT * q;
        v4i v = *reinterpret_cast<const v4i *>(body + (idx / PPR) * G::PITCH + 16 * (idx % PPR));
        if (a.residual) {
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = (int)add_sat_i8x4((uint32_t)v[r], (uint32_t)res[q][r]);
        }
        store_b128_guarded(v, ry, yoff[q]);
    }
}

template <int PT, int NW> static GemmTile gemm_tile(bool prelu)
{
    using G = GemmGeom<PT, NW>;
    return {G::TM, G::TN, G::NT, G::LDS, prelu ? &pw_gemm_kernel<PT, NW, true> : &pw_gemm_kernel<PT, NW, false>};
}
GemmTile pw_gemm_tile(int pt, int nw, bool prelu)
{
    if (nw == 4) return pt == 8 ? gemm_tile<8, 4>(prelu) : pt == 4 ? gemm_tile<4, 4>(prelu) : gemm_tile<2, 4>(prelu);
    return pt == 8 ? gemm_tile<8, 2>(prelu) : pt == 4 ? gemm_tile<4, 2>(prelu) : gemm_tile<2, 2>(prelu);
}

}  // namespace prom
