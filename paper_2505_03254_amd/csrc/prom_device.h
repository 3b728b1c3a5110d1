// Device helpers shared by the HIP kernels: exact requantisation and byte packing.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace prom {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
// 4-byte-aligned views for global accesses whose address is only dword aligned
typedef int v4i_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef int v2i_a4 __attribute__((ext_vector_type(2), aligned(4)));

// min(max(v, lo), hi); becomes one v_med3_i32 when lo and hi sit in vector registers or are
// inline constants (the instruction can read at most one scalar register).
__device__ __forceinline__ int clamp_i32(int v, int lo, int hi) { return min(max(v, lo), hi); }

// Median of three = clamp of v to [lo, hi] when lo <= hi.  Written as the instruction because
// the compiler cannot prove lo <= hi and would emit a max and a min.
__device__ __forceinline__ int med3_i32(int v, int lo, int hi)
{
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "v"(lo), "v"(hi));
    return r;
}

// Moves a wave-uniform value into a vector register and hides its origin from the optimiser,
// so that two such bounds can feed one v_med3_i32.
__device__ __forceinline__ int in_vgpr(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// ---- integer requantisation ------------------------------------------------------------------

// The four per-channel values the epilogue keeps in registers.
__device__ __forceinline__ v4i requant_params(int bias, int mult, int mult_neg, int shift, bool prelu)
{
    if (prelu) return v4i{bias, mult, mult_neg, shift};
    const long long C = (long long)bias * mult + (1LL << (30 + shift));
    return v4i{(int)(uint32_t)C, (int)(C >> 32), mult, shift};
}

// t = acc*mult + C; q = t >> (31 + shift); clamp to [lo, hi].  pr = (C lo, C hi, mult, s) with
// s = shift-1 when !GENERAL (the caller guarantees shift >= 1) and s = shift when GENERAL.
template <bool GENERAL>
__device__ __forceinline__ int requant_i64(int accv, const v4i &pr, int lo, int hi)
{
    const long long C = (long long)(((unsigned long long)(uint32_t)pr[1] << 32) | (uint32_t)pr[0]);
    const long long t = (long long)accv * (long long)pr[2] + C;
    int q;
    if constexpr (GENERAL)
        q = (int)(t >> 31) >> pr[3];
    else
        q = (int)(t >> 32) >> pr[3];
    return med3_i32(q, lo, hi);
}

// PReLU form: pr = (bias, mult, mult_neg, shift); the multiplier follows the sign of
// s = acc + bias, then q = floor((s*m + 2^(30+shift)) / 2^(31+shift)), clamp.  Computed as
// floor((floor(s*m / 2^shift) + 2^30) / 2^31), which is the same number (2^30 is an integer and
// nested floors of divisions by positive integers collapse) and needs no per-channel rounding
// constant: such constants are loop invariants the compiler would keep in registers, two more
// per channel.
__device__ __forceinline__ int requant_prelu_s(int s, int mult, int mult_neg, int shift, int lo, int hi)
{
    const int m = s < 0 ? mult_neg : mult;
    const long long u = ((long long)s * (long long)m) >> shift;
    const int q = (int)((u + (1LL << 30)) >> 31);
    return med3_i32(q, lo, hi);
}
__device__ __forceinline__ int requant_prelu_i64(int accv, const v4i &pr, int lo, int hi)
{
    return requant_prelu_s(accv + pr[0], pr[1], pr[2], pr[3], lo, hi);
}

// The definition itself for one value, with s = acc + bias already formed and the multiplier already
// chosen (PReLU: by the sign of s): q = floor((s*m + 2^(30+shift)) / 2^(31+shift)), clamp.  An
// arithmetic right shift of a 64-bit integer is a floor division; |s*m| < 2^62 and the rounding
// constant is at most 2^61.  Used by the one-thread-per-output kernels.
__device__ __forceinline__ int requant_s_i64(int s, int m, int shift, int lo, int hi)
{
    const long long t = (long long)s * (long long)m + (1LL << (30 + shift));
    return clamp_i32((int)(t >> (31 + shift)), lo, hi);
}

// Epilogue forms: 0 = every shift of the wavefront's channels >= 1 (pr.w holds shift-1),
// 1 = any shift, 2 = PReLU.
template <int MODE>
__device__ __forceinline__ int requant_mode(int accv, const v4i &pr, int lo, int hi)
{
    if constexpr (MODE == 2)
        return requant_prelu_i64(accv, pr, lo, hi);
    else
        return requant_i64<MODE == 1>(accv, pr, lo, hi);
}

// 16-byte buffer store, offset in the vector operand, with its data registers protected in the
// source.  On gfx950 a buffer store of more than 8 bytes picked up, now and then, the NEW contents
// of its data registers when the instruction right behind it overwrote them (seen with a scalar
// offset register, the one form for which the compiler inserts no wait state).  The empty
// statement behind the store reads the four data registers, so no instruction that overwrites them
// can be scheduled before it, and its two wait states are what the store needs -- whatever form of
// offset a later compiler picks.
__device__ __forceinline__ void store_b128_guarded(const v4i v, __amdgpu_buffer_rsrc_t rsrc, int voffset)
{
    __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, voffset, 0, 0);
    asm volatile("s_nop 1" : : "v"(v));
}

// Low bytes of four ints -> one dword (a in bits 0..7).
__device__ __forceinline__ uint32_t pack4_low_bytes(int a, int b, int c, int d)
{
    const uint32_t ab = __builtin_amdgcn_perm((uint32_t)b, (uint32_t)a, 0x0c0c0400u);
    const uint32_t cd = __builtin_amdgcn_perm((uint32_t)d, (uint32_t)c, 0x0c0c0400u);
    return __builtin_amdgcn_perm(cd, ab, 0x05040100u);
}

// Sign-extended byte i (0..3) of a dword.
__device__ __forceinline__ int sbyte(uint32_t v, int i)
{
    return (int)(v << (24 - 8 * i)) >> 24;
}

// ---- requantisation of two pixels at a time ----------------------------------------------------------
// v_ashr_pk_u8_i32 / v_ashr_pk_i8_i32 (gfx950) shift two dwords by one amount, saturate both to 8 bits
// and pack them.  With two pixels of the same channel in the pair, four instructions replace the eight
// shifts and the eight clamps of 2 x 4 outputs, and the bytes are put in order by four v_perm_b32 instead
// of six: 12.7 (window [0, 127]) and 11.8 ([-128, 127]) cycles per output and SIMD against 16.9 for
// requant_mode<0> with pack4_low_bytes, measured on independent outputs in registers.
//
// Forms (template argument of requant_pair4):
//   kPairRelu   window [0, 127], every shift >= 2: the pair instruction saturates floor(2v) to [0, 255];
//               clamp(floor(v), 0, 127) is half of that, rounded down -- one shift and one mask per dword
//   kPairFull   window [-128, 127], every shift >= 1
//   kPairLow    either of the two windows, every shift >= 1 (one maximum per output more)
//   kPairClamp  any window, every shift >= 1: one shift and one clamp per output (requant_i64<false>)
//   kPairAny    any window, any shift (requant_i64<true>)
//   kPairPreluFull  PReLU layer (par = (bias, mult, mult_neg, shift)), window [-128, 127], every shift >= 2
//   kPairPreluAny   PReLU layer, any window, any shift
constexpr int kPairRelu = 0, kPairFull = 1, kPairAny = 2, kPairPreluFull = 3, kPairPreluAny = 4, kPairLow = 5, kPairClamp = 6;

// What a form's shifts are reduced by in the parameters handed to requant_pair4.
__host__ __device__ constexpr int pair_shift_less(int form) { return form == kPairRelu || form == kPairPreluFull ? 2 : form == kPairFull || form == kPairLow || form == kPairClamp ? 1 : 0; }

// a0, a1: the accumulators of two pixels, four channels each; par: the channels' parameters as
// requant_params made them, the shifts reduced by pair_shift_less(FORM); out0, out1: the packed outputs.
// BIASED: the bias of a PReLU layer is in the accumulators already.  MASKED = false: with kPairRelu the top bit of
// every byte is left undefined, for a caller that masks the outputs anyway.
template <int FORM, bool BIASED = false, bool MASKED = true>
__device__ __forceinline__ void requant_pair4(const v4i &a0, const v4i &a1, const v4i (&par)[4], int lo, int hi,
                                              uint32_t &out0, uint32_t &out1)
{
    if constexpr (FORM == kPairAny || FORM == kPairClamp || FORM == kPairPreluAny) {
        int v[4], w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if constexpr (FORM != kPairPreluAny) {
                v[r] = requant_i64<FORM == kPairAny>(a0[r], par[r], lo, hi);
                w[r] = requant_i64<FORM == kPairAny>(a1[r], par[r], lo, hi);
            } else {
                const int b = BIASED ? 0 : par[r][0];
                v[r] = requant_prelu_s(a0[r] + b, par[r][1], par[r][2], par[r][3], lo, hi);
                w[r] = requant_prelu_s(a1[r] + b, par[r][1], par[r][2], par[r][3], lo, hi);
            }
        }
        out0 = pack4_low_bytes(v[0], v[1], v[2], v[3]);
        out1 = pack4_low_bytes(w[0], w[1], w[2], w[3]);
        return;
    } else {
        uint32_t h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int t0, t1;
            if constexpr (FORM == kPairPreluFull) {
                const int b = BIASED ? 0 : par[r][0];
                const int s0 = a0[r] + b, s1 = a1[r] + b;
                // (a bit select by the sign: the compiler turns a ternary between two elements of one vector
                // into a chain of compares and selects, and this too if it sees where the mask comes from)
                int n0 = s0 >> 31, n1 = s1 >> 31;
                asm("" : "+v"(n0));
                asm("" : "+v"(n1));
                const int m0 = (n0 & par[r][2]) | (~n0 & par[r][1]), m1 = (n1 & par[r][2]) | (~n1 & par[r][1]);
                // floor((s*m + 2^(30+shift)) / 2^32): the rounding term is a whole multiple of 2^32
                t0 = __mulhi(s0, m0) + (1 << par[r][3]);
                t1 = __mulhi(s1, m1) + (1 << par[r][3]);
            } else {
                const long long C = (long long)(((unsigned long long)(uint32_t)par[r][1] << 32) | (uint32_t)par[r][0]);
                t0 = (int)(((long long)a0[r] * par[r][2] + C) >> 32);
                t1 = (int)(((long long)a1[r] * par[r][2] + C) >> 32);
            }
            if constexpr (FORM == kPairLow) {  // the high halves at least 0, or at least INT_MIN
                const int low = (int)((unsigned)lo << 24);
                t0 = max(t0, low);
                t1 = max(t1, low);
            }
            // (the instruction, not the builtin: the builtin's 16-bit result costs a mask)
            const int sh = FORM == kPairPreluFull ? par[r][3] + 1 : par[r][3];
            if constexpr (FORM == kPairRelu)
                asm("v_ashr_pk_u8_i32 %0, %1, %2, %3" : "=v"(h[r]) : "v"(t0), "v"(t1), "v"(sh));
            else
                asm("v_ashr_pk_i8_i32 %0, %1, %2, %3" : "=v"(h[r]) : "v"(t0), "v"(t1), "v"(sh));
        }
        const uint32_t ab = __builtin_amdgcn_perm(h[1], h[0], 0x05010400u);  // (p0 c0, p0 c1, p1 c0, p1 c1)
        const uint32_t cd = __builtin_amdgcn_perm(h[3], h[2], 0x05010400u);
        out0 = __builtin_amdgcn_perm(cd, ab, 0x05040100u);
        out1 = __builtin_amdgcn_perm(cd, ab, 0x07060302u);
        if constexpr (FORM == kPairRelu) {
            out0 >>= 1;
            out1 >>= 1;
            if constexpr (MASKED) {
                out0 &= 0x7f7f7f7fu;
                out1 &= 0x7f7f7f7fu;
            }
        }
    }
}

// The form for a window and channels whose shifts are all >= 1 (ge1), all >= 2 (ge2).  Every window has a form
// without the 64-bit shift of kPairAny as long as no shift is 0: windows other than the first two through
// kPairAny cost the depthwise kernel 4 to 11 % and the blocks with planes in LDS 2 to 5 %.
__host__ __device__ constexpr int pair_form_of(bool prelu, bool ge1, bool ge2, int lo, int hi)
{
    const bool full = lo == -128 && hi == 127, relu = lo == 0 && hi == 127;
    if (prelu) return full && ge2 ? kPairPreluFull : kPairPreluAny;
    if (!ge1) return kPairAny;
    return full ? kPairFull : relu ? (ge2 ? kPairRelu : kPairLow) : kPairClamp;
}

// The form a wavefront can take for the channels of its lanes; wave-uniform.
// s: the smallest shift of the lane's channels.
template <bool PRELU>
__device__ __forceinline__ int pair_form(int s, int lo, int hi)
{
    // (shifts are looked at only where they decide: ahead of the window, the test takes the PReLU kernel of the
    // grouped convolutions from 242 registers to 256 and 180 bytes of scratch, RegNetX-400MF from 99 to 113 us)
    if constexpr (PRELU) return lo == -128 && hi == 127 && __builtin_amdgcn_ballot_w64(s < 2) == 0 ? kPairPreluFull : kPairPreluAny;
    const bool ge2 = __builtin_amdgcn_ballot_w64(s < 2) == 0;
    return pair_form_of(false, __builtin_amdgcn_ballot_w64(s < 1) == 0, ge2, lo, hi);
}

__device__ __forceinline__ int min_shift(const v4i (&par)[4])
{
    return min(min(par[0][3], par[1][3]), min(par[2][3], par[3][3]));
}

// Saturating sum of two dwords of four int8 each: the odd bytes as the high halves of 16-bit lanes, the
// even ones shifted there; the byte below a summand never carries because the other summand's is zero.
__device__ __forceinline__ uint32_t add_sat_i8x4(uint32_t a, uint32_t b)
{
    typedef short s16x2 __attribute__((ext_vector_type(2)));
    const uint32_t odd = __builtin_bit_cast(uint32_t, __builtin_elementwise_add_sat(
        __builtin_bit_cast(s16x2, a), __builtin_bit_cast(s16x2, b & 0xff00ff00u)));
    const uint32_t even = __builtin_bit_cast(uint32_t, __builtin_elementwise_add_sat(
        __builtin_bit_cast(s16x2, a << 8), __builtin_bit_cast(s16x2, (b << 8) & 0xff00ff00u)));
    return __builtin_amdgcn_perm(odd, even, 0x07030501u);
}

}  // namespace prom
