// Fused Bicoptor 2.0 DReLU (Alg. 7) and UBL ReLU (Alg. 8) kernel.
//
// One thread owns one element and plays P0, P1 and P2 for it, in the order
// of Alg. 7:
//   P0/P1  flip     both shares negated when the seed_01 bit t is set
//          windows  l_x + 1 windows trc(x, k_lo + i, l - l_x - k_lo - i)
//          sums     adjacent sums v_i = u_i + u_{i+1} - 1 (P0 adds the -1)
//          switch   modulo switch to Z_p (Alg. 6)
//          shuffle  slot s takes position sigma(s) of a seed_01 Fisher-Yates
//                   shuffle run in the thread's slice of LDS
//          mask     multiply by r_s in Z_p^*, reshare by +-z_s
//   P2     test     reconstruct every slot, D' = [some slot is 0]
//          reply    reshare D' with rho from seed_02 (DReLU)
//   P0/P1  unflip   t + (1 - 2t) [D']
// ReLU replaces the reply and the unflip by the Beaver product of Alg. 8
// with the triple generated from seed_02 / seed_12 and the unflipped input
// shares.
//
// The l_x + 1 window values never leave VGPRs.  Kernels are instantiated
// per window count N = l_x + 1, so every loop over windows is unrolled.  The
// shuffle is applied by computing, for slot s, the window of the position
// sigma(s) read back from LDS: the message in slot s is v_{sigma(s)} r_s + z_s,
// exactly the array that the shuffle and mask produce.  With a capture
// pointer the same code also stores both parties' round-1 messages.
#pragma once

#include <type_traits>

#include "bc_device.h"
#include "internal.h"

namespace bc {

struct DreluKArgs {
    const void* x0;
    const void* x1;
    void* y0;
    void* y1;
    void* cap;
    uint64_t n;
    uint64_t ncap;        // elements of the whole call (the capture's P1 half starts at ncap * N)
    uint64_t elem_base;
    uint64_t ring_mask;   // 2^l - 1
    uint64_t in_mask;     // 2^l_in - 1 of the input ring (l_in = l + k_in)
    uint32_t k_lo, k_in;  // k_in > 0: Alg. 5 truncation of the inputs by k_in bits first
    Stream s01, s02, s12;
};

// The share already shifted down by k_lo (pos <= l_x), shifted down by pos:
// bits [0, l_x] are the window, bits above it are left for the caller to
// mask.  With 64-bit shares: when bits [0, 2 l_x] fit in 32 bits a 32-bit
// shift of the low word, else (windows of at most 32 bits) one
// v_alignbit_b32 of the two halves does the variable shift.
template <typename T, int N, typename FT>
__device__ __forceinline__ FT window_low(T a, uint32_t pos) {
    if constexpr (sizeof(T) == 8 && 2 * N - 1 <= 32)     // bits [0, 2 l_x] fit in the low word
        return (FT)((uint32_t)a >> pos);
    else if constexpr (sizeof(T) == 8 && N <= 32)
        return (FT)__builtin_amdgcn_alignbit((uint32_t)(a >> 32), (uint32_t)a, pos);
    else
        return (FT)(a >> pos);
}

// a * b + c in Z_p with b and c given shifted left by SH bits (SH = 0: the
// plain values; see MaskDraws).
template <int SH, typename F>
__device__ __forceinline__ typename F::T field_mul_add(const F& f, typename F::T a, typename F::T b, typename F::T c) {
    if constexpr (SH == 0)
        return f.mul_add(a, b, c);
    else if constexpr (SH < 8)
        return f.mul_add(a, b >> SH, c >> SH);        // N > 24: the fields fold from plain values
    else
        return f.template mul_add_sh<SH>(a, b, c);
}

// P1's reshare addend p - z, kept shifted by SH like z, from a z <= p whose
// low SH bits may carry stray bits (stream_draws): they are masked first.
template <int SH, typename F>
__device__ __forceinline__ typename F::T reshare_neg(const F& f, typename F::T z) {
    using FT = typename F::T;
    constexpr FT KEEP = (FT)~(((FT)1 << SH) - 1);
    return (FT)((f.p << SH) - (FT)(z & KEEP));
}

// v_min3_u32 written out: the compiler would otherwise re-associate P2's
// running minimum into a tree over all slots, which defers every slot's
// end and keeps all of them live at once.
__device__ __forceinline__ uint32_t min3_in_order(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t d;
    asm("v_min3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// The adjacent sums of one window position (sigma of a slot), before the
// modulo switch (Alg. 7, Alg. 6):
//   P0   v_0 = (u_i + u_{i+1} - 2) mod 2^l_x; its switched value, v mod p of
//        v = u_i + u_{i+1} - 1 with 0 standing as 2^l_x, is s_0 = v_0 + 1
//   P1   v_1 = (cut_i + cut_{i+1} - 1) mod 2^l_x; its switched value
//        -(cut_i + cut_{i+1}) mod 2^l_x + p - 2^l_x is p - (v_1 + 1)
// a is P0's share or P1's negated share, flipped and shifted down by k_lo.
// With W = a >> pos, u_i + u_{i+1} = W + floor(W / 2) = floor(3 W / 2) in
// bits [0, l_x), and for pos = l_x (u_{l_x+1} := 0) floor(2 W / 2): so
// v = (times W - 2 minus) >> 1 mod 2^l_x with times = 3, or 2 for pos = l_x, which
// the shuffle keeps beside the position.  Bits of W above the window only
// reach bits above the sum.  Three operations a party: the shift, one
// multiply-add, one bit-field extract.
template <typename T, int N, int MINUS>
__device__ __forceinline__ uint32_t window_sum(T a, uint32_t pos, uint32_t times) {
    constexpr int LX = N - 1;
    if constexpr (N <= 24)                                   // W's low 24 bits hold the window and u_{i+1}
        return __builtin_amdgcn_ubfe(mad24<-2 * MINUS>(window_low<T, N, uint32_t>(a, pos), times), 1, LX);
    else if constexpr (N <= 32)
        return __builtin_amdgcn_ubfe(
            (uint32_t)mad_u64_u32(window_low<T, N, uint32_t>(a, pos), times, 0ull - 2 * MINUS), 1, LX);
    else {                                                   // 32-bit windows of a 64-bit share
        const uint64_t W = a >> pos;
        return (uint32_t)W + ((uint32_t)(W >> 1) & (2u - times)) - MINUS;
    }
}
template <typename T, int N>
__device__ __forceinline__ void window_sums(T a0, T nb1, uint32_t pos, uint32_t times, uint32_t& v0, uint32_t& v1) {
    v0 = window_sum<T, N, 2>(a0, pos, times);
    v1 = window_sum<T, N, 1>(nb1, pos, times);
}
template <typename T, int N>
__device__ __forceinline__ void window_sums(T a0, T nb1, uint32_t pos, uint32_t& v0, uint32_t& v1) {
    window_sums<T, N>(a0, nb1, pos, 3u - (pos + 1) / N, v0, v1);    // 2 at pos = l_x = N - 1
}

// Both parties' round-1 messages of one slot in [0, p), from its sums and its
// plain mask r and reshare z: w0 = s_0 r + z, w1 = s_1 r - z.
template <typename F>
__device__ __forceinline__ void slot_messages(uint32_t v0, uint32_t v1, typename F::T r, typename F::T z, const F& f,
                                              typename F::T& w0, typename F::T& w1) {
    using FT = typename F::T;
    w0 = f.mul_add((FT)v0 + 1, r, z);
    w1 = f.mul_add((FT)(f.p - 1) - (FT)v1, r, (FT)(f.p - z));
}

// P2's test of one slot where nothing captures the messages.  P1 keeps its
// message negated, as it keeps its negated share: s_1 r - z is
// -((v_1 + 1) r + z) mod p.  So both parties form m = v r + c with
// c = r + z, unreduced (a value congruent to the message, or to its
// negation), and P2 reconstructs by subtraction: the slot is zero exactly
// when p divides D = m0 - m1.  mark() is at most LIMIT for these slots and
// above it for all others; P2 keeps the minimum.  No division or reduction
// is needed for that: with p' = p^-1 mod 2^32, k = D p' mod 2^32 (as a signed
// number) is the only candidate for the quotient, so
//  * p < 2^16 (N <= 16): |D| < 2^31 and a quotient has |k| <= K = 2^l_x - 1.  No
//    other D in that range has k in [-K, K] (|k| p < 2^31), so the test is
//    D p' + K mod 2^32 <= 2 K, one multiply-add.
//  * p < 2^31: r and z are kept shifted left by SH, and D with them;
//    |D| < 2^62 and a quotient is below 2^31 in magnitude (l_x + SH <= 31).
//    D - k p has a zero low word, so p divides D exactly when its high word
//    is zero.
//  * p in (2^31, 2^32): the same, as (D + (2^32 - p) k) = k 2^32.
//  * p = 2^33 - 9: 2^33 = 9 mod p, so twice a message v r + c,
//    r = r_1 2^32 + r_0, is 9 (hi(v r_0) + v r_1) + 2 lo(v r_0) + 2 c, below
//    2^38; a quotient of the two's difference U is at most 32 in magnitude, so
//    k is taken from its low 8 bits and U + 9 k = k 2^33 decides.
//  * any other prime above 2^32: the messages in [0, p), compared.
// The products are opaque to the compiler (asm), which would otherwise
// subtract the shares before masking them.
// These kernels are bound by VALU issue, about 4.1 cycles an instruction
// whatever its kind, so the instruction count decides.  With the reduced
// messages and their compares replaced by this test, the packed windows, the
// grouped shuffle digits and window_sum (886 -> 725 instructions an element
// at N = 19, 647 -> 463 for the N = 8 ReLU): DReLU at N = 19 and 2^24
// elements 0.360 -> 0.298 ms (0.285-0.288 at 691 instructions, with the scalar
// Philox rounds and zero_high), ReLU at N = 8 0.255 -> 0.209 ms; DReLU at
// N = 32 and 2^23 0.378 -> 0.277 ms, at N = 33 and 2^22 0.422 -> 0.231 ms.
template <int N, typename F, int SH>
struct SlotTest {
    using FT = typename F::T;
    static constexpr bool SMALL = N <= 16;
    static constexpr uint32_t K = SMALL ? (1u << (N - 1)) - 1 : 0;
    static constexpr uint32_t LIMIT = 2 * K;

    uint64_t zero_high;
    __device__ __forceinline__ SlotTest() {
        if constexpr (!SMALL && N <= 31) asm("v_mov_b64 %0, 0" : "=v"(zero_high));
    }
    static __device__ __forceinline__ uint32_t mark_small(uint32_t m0, uint32_t m1, const F& f) {
        return (uint32_t)mad_u64_u32(m0 - m1, f.pinv32(), K);
    }
    // Both sums in one word, v_0 in the low half and v_1 in the high half.
    static __device__ __forceinline__ uint32_t mark_pair(uint32_t pair, uint32_t r, uint32_t z, const F& f) {
        const uint32_t c = r + z;
        return mark_small(mad_half<false>(pair, r, c), mad_half<true>(pair, r, c), f);
    }
    __device__ __forceinline__ uint32_t mark(uint32_t v0, uint32_t v1, FT r, FT z, const F& f) {
        if constexpr (SMALL) {
            const uint32_t c = r + z;
            return mark_small(mad_half<false>(v0, r, c), mad_half<false>(v1, r, c), f);
        } else if constexpr (N <= 32) {
            uint64_t c;
            if constexpr (N <= 31) {
                // r + z through a register pair whose high word stays zero from
                // slot to slot, which the compiler would set again for each
                // (N = 19: 708 -> 691 instructions); at N = 32 z is a stream
                // word that would have to be moved there
                zero_high = (zero_high & 0xFFFFFFFF00000000ull) | z;
                c = mad_u64_u32(r, 1u, zero_high);
            } else {
                c = add_wide(r, z);
            }
            const uint64_t D = mad_u64_u32(v0, r, c) - mad_u64_u32(v1, r, c);
            const uint32_t k = (uint32_t)D * f.pinv32();
            if constexpr (N <= 31)
                return (uint32_t)((uint64_t)((int64_t)(int32_t)k * (int32_t)(0u - f.p) + (int64_t)D) >> 32);
            else
                return (uint32_t)((uint64_t)((int64_t)(int32_t)k * (int32_t)(0u - f.p) + (int64_t)D) >> 32) ^ k;
        } else if constexpr (F::kDefault) {
            const uint32_t r0 = (uint32_t)r, r1 = 0u - (uint32_t)(r >> 32);
            const uint64_t c2 = (r + z) << 1;
            const uint64_t U = message2(v0, r0, r1, c2) - message2(v1, r0, r1, c2);
            int32_t k = (int32_t)((uint32_t)U * f.pinv32() << 24) >> 24;
            asm("" : "+v"(k));       // a plain 32-bit factor: one v_mad_i64_i32
            const uint64_t e = (uint64_t)((int64_t)k * 9 + (int64_t)U);
            return (uint32_t)e | ((uint32_t)(e >> 32) ^ (uint32_t)(2 * k));
        } else {
            const FT w0 = f.mul_add((FT)v0 + 1, r, z), w1 = f.mul_add((FT)v1 + 1, r, z);
            return (uint32_t)(w0 ^ w1) | (uint32_t)((w0 ^ w1) >> 32);
        }
    }
    // N = 33: twice the message v r + c, with r1 = -(r >> 32) as a mask.
    static __device__ __forceinline__ uint64_t message2(uint32_t v, uint32_t r0, uint32_t r1, uint64_t c2) {
        const uint64_t x = mad_u64_u32(v, r0, 0);
        return mad_u64_u32((uint32_t)x, 2u, mad_u64_u32(v & r1, 9u, mad_u64_u32((uint32_t)(x >> 32), 9u, c2)));
    }
};

// The minimum of a slot loop's marks in slot order, two slots to one
// three-operand minimum (j compile-time after unrolling).
template <int N>
struct LeastMark {
    uint32_t least = 0xFFFFFFFFu, last = 0;
    __device__ __forceinline__ void take(int j, uint32_t mark) {
        if (j % 2 == 0 && j < N - 1)
            last = mark;
        else
            least = min3_in_order(least, j % 2 == 0 ? mark : last, mark);
    }
};

// ------------------------------------------------------- windows as pairs
//
// For N <= 16 (p < 2^16) both parties' values of one window position fit in
// one 32-bit word, P0's v_0 in the low half and P1's v_1 in the high half,
// and the shuffle moves these words themselves, as the message array it
// permutes.  Position i is then computed when i is known at compile time:
// windows are constant shifts of both shares at once (v_pk_lshrrev_b16 on a
// word that packs 16 bits of each), u_{l_x+1} = 0 needs no flag, and the slot
// loop reads one word per slot.
typedef uint16_t half2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ half2 as_half2(uint32_t w) { return __builtin_bit_cast(half2, w); }
__device__ __forceinline__ uint32_t as_word(half2 h) { return __builtin_bit_cast(uint32_t, h); }

template <int N>
constexpr bool kPairs = N <= 16;

template <typename T, int N>
struct PairWindows {
    static constexpr int LX = N - 1;
    static constexpr int PER = 17 - LX;                       // positions in one packed word
    static constexpr uint32_t WIN2 = ((1u << LX) - 1) * 0x10001u;
    T a, b;                                                   // the flipped shares, shifted down by k_lo
    half2 minus;                                              // (-2, -1), the parties' constants
    half2 next;                                               // position k of the coming value()

    __device__ __forceinline__ PairWindows(T a0k, T nb1k, uint32_t c) : a(a0k), b(nb1k), minus(as_half2(c)) {
        next = window(0);
    }
    // Bits [k, k + l_x) of both shares, with other bits above; even positions
    // carry the parties' constants (every adjacent sum takes exactly one).
    __device__ __forceinline__ half2 window(int k) const {
        const int off = k / PER * PER;
        const half2 w = as_half2(__builtin_amdgcn_perm((uint32_t)(b >> off), (uint32_t)(a >> off), 0x05040100u));
        const half2 m = w >> (half2)(uint16_t)(k - off);
        return k % 2 == 0 ? m + minus : m;
    }
    // (v_0, v_1) of position k; called for k = 0, 1, ..., l_x in this order.
    __device__ __forceinline__ uint32_t value(int k) {
        half2 sum = next;
        if (k < LX) {
            next = window(k + 1);
            sum += next;
        } else if (k % 2 != 0) {
            sum += minus;                                     // u_{l_x+1} = 0
        }
        return as_word(sum) & WIN2;
    }
};

// All ones when t = 1, else zero, in the share width.
template <typename T>
__device__ __forceinline__ T spread(uint32_t t) {
    const uint32_t w = 0u - t;
    if constexpr (sizeof(T) == 8)
        return join64(w, w);
    else
        return w;
}

// m ? a : b for m all ones or zero, as bit selects (v_bfi_b32).  A select on
// a condition compiles to runs of v_cndmask_b32 on VCC, which issue at 22
// cycles each on gfx950 when they follow each other.
template <typename T>
__device__ __forceinline__ T select_bits(T m, T a, T b) {
    return (m & a) | (~m & b);
}

// (-1)^t v mod 2^l for v < 2^l (Alg. 7's flip): (v ^ -t) + t.
template <typename T>
__device__ __forceinline__ T flip_by(T v, uint32_t t, T mask) {
    return (T)((v ^ spread<T>(t)) + (T)t) & mask;
}

// The shares a DReLU/ReLU works on, from the loaded ones: with k_in > 0 the
// loaded shares are of Z_{2^(l + k_in)} (in_mask) and each party first
// truncates its own by k_in bits (Alg. 5); with k_in = 0 and in_mask = mask
// the same expressions are the plain shares.  P0 holds in0 = cut(x0, k_in);
// P1 holds -n1 with n1 = cut(-x1, k_in), and n1, its negated share, is what it
// cuts the windows from (Alg. 7).
template <typename T>
__device__ __forceinline__ void input_shares(T x0, T x1, T mask, T in_mask, uint32_t k_in, T& in0, T& n1) {
    if (k_in == 0) {                                  // the plain shares (in_mask = mask): a uniform branch
        in0 = x0 & mask;
        n1 = (T)((T)0 - x1) & mask;
    } else {
        in0 = (T)((x0 & in_mask) >> k_in) & mask;
        n1 = (T)((((T)0 - x1) & in_mask) >> k_in) & mask;
    }
}

// DReLU's end (Alg. 7): P2's fresh sharing (rho, D' - rho), then the unflip:
// y0 = t + (1 - 2t) rho, y1 = (1 - 2t)(D' - rho), select-free with tm = -t
// (all ones when t = 1): (v ^ tm) - tm = (1 - 2t) v.  Each step keeps the low
// l bits a function of the low l bits, so rho may carry bits above l and one
// mask at the end reduces mod 2^l.
template <typename T>
__device__ __forceinline__ void drelu_finish(T dp, T rho, uint32_t t, T mask, T& y0, T& y1) {
    const T tm = spread<T>(t);
    y0 = (T)((rho ^ tm) + (T)(2 * t)) & mask;          // t = 1: ~rho + 2 = 1 - rho
    y1 = (T)(((T)(dp - rho) ^ tm) + (T)t) & mask;
}

// Alg. 8's preprocessing draws of element g: [a]_0, [b]_0, [c]_0 from
// seed_02 (blocks 0 and 1 of TAG_BEAVER), [a]_1, [b]_1 from seed_12 (block 0);
// P2 forms [c]_1 = (a0 + a1)(b0 + b1) - c0 from them.
template <typename T>
__device__ __forceinline__ void beaver_shares(const Stream& s02, const Stream& s12, Index g, T mask, T& ba0, T& bb0,
                                              T& bc0, T& ba1, T& bb1) {
    const StreamAt r02 = s02.at(g);
    const Words4 w0 = r02.block(TAG_BEAVER, 0);
    const Words4 w1 = r02.block(TAG_BEAVER, 1);
    const Words4 w2 = s12.block(g, TAG_BEAVER, 0);
    ba0 = (T)join64(w0.w0, w0.w1) & mask;
    bb0 = (T)join64(w0.w2, w0.w3) & mask;
    bc0 = (T)join64(w1.w0, w1.w1) & mask;
    ba1 = (T)join64(w2.w0, w2.w1) & mask;
    bb1 = (T)join64(w2.w2, w2.w3) & mask;
}

// Alg. 8 after the zero test: e = D' - b, d = x - a and the product, with
// the triple ([a]_j, [b]_j, [c]_j) and the unflipped inputs.
template <typename T>
__device__ __forceinline__ void relu_finish(T dp, T in0, T in1, T ba0, T bb0, T bc0, T ba1, T bb1, T bc1, uint32_t t,
                                            T mask, T& y0, T& y1) {
    const T ee = (T)(dp - (T)(bb0 + bb1)) & mask;                 // P2: e = D' - b
    const T dd = (T)((in0 - ba0) + (in1 - ba1)) & mask;           // P0, P1: d = x - a
    const T m0 = (T)(dd * ee + dd * bb0 + ee * ba0 + bc0) & mask; // de + d[b] + e[a] + [c]
    const T m1 = (T)(dd * bb1 + ee * ba1 + bc1) & mask;
    const T tm = spread<T>(t);
    y0 = select_bits<T>(tm, (T)(in0 - m0) & mask, m0);              // t[x] + (1 - 2t)[x D']
    y1 = select_bits<T>(tm, (T)(in1 - m1) & mask, m1);
}

// The flip bit t and the shuffle of one element, both from seed_01 (Alg. 7).
// N digits: t (radix 2), then j_i in [0, i] (radix i + 1) for i = 1..N-1, the
// choices of an inside-out Fisher-Yates shuffle: A[0] = 0, and for each i,
// A[i] = A[j_i], A[j_i] = i; slot s takes window position A[s].  The digits
// are cut from 64-bit chunks F of the TAG_SHUFFLE stream (chunk c: words
// 2 (c % 2) and 2 (c % 2) + 1 of block c / 2, low word first); a chunk takes
// digits in order while the product of their radices stays <= 2^32, and a
// digit of radix m is the part of F m above 2^64, F m mod 2^64 the next F.
//
// The kernels cut the digits of a chunk group by group: with M the product of
// a group's radices, X = floor(F M / 2^64) holds its digits (mixed radix,
// first digit most significant) and F M mod 2^64 is the next F.  With
// C = ceil(2^32 / M), f = X C is X / M as a 32-bit fraction, too large by less
// than 1 / M when (M - 1) (C M - 2^32) < 2^32, so the digits of f are those of
// X: digit of radix m = the high word of f m, the low word the next f.  That
// is one multiply a digit after four operations a group, where cutting each
// digit from the 64-bit F takes two multiplies and a move: N = 19 runs its 19
// digits in 4 groups.
template <int N>
struct ShufflePlan {
    int chunk[N];          // the chunk of digit k
    bool group[N];         // digit k is the first of a group
    uint32_t prod[N];      // the product of the radices of the group that starts at k
    static constexpr uint64_t radix(int k) { return k == 0 ? 2 : (uint64_t)k + 1; }
    static constexpr uint64_t scale(uint64_t m) { return ((1ull << 32) + m - 1) / m; }
    static constexpr bool fits(uint64_t m) {
        return m < (1ull << 32) && (m - 1) * scale(m) < (1ull << 32) && (m - 1) * (scale(m) * m - (1ull << 32)) < (1ull << 32);
    }
    constexpr ShufflePlan() : chunk(), group(), prod() {
        uint64_t prod_c = 1, prod_g = 1;
        int c = 0, g = 0;
        for (int k = 0; k < N; ++k) {
            const uint64_t m = radix(k);
            const bool next = prod_c * m > (1ull << 32);
            if (next) {
                ++c;
                prod_c = 1;
            }
            if (k == 0 || next || !fits(prod_g * m)) {
                g = k;
                prod_g = 1;
            }
            prod_c *= m;
            prod_g *= m;
            chunk[k] = c;
            group[k] = g == k;
            prod[g] = (uint32_t)prod_g;
        }
    }
};

// Runs the shuffle in this thread's slice of a per-block LDS array (blocks of
// at most 256 threads: every kernel is launched with __launch_bounds__(256))
// and returns the slice.  Entry A[k] is E bytes at byte k ROW of the slice,
// ROW = 256 E, so entry k of the 256 threads is one contiguous row and the
// address of a drawn index j is one multiply-add.  With E = 4 the 64 lanes of
// a wave touch 64 different banks whatever their k; E = 4 while 8 blocks of N
// rows fit the compute unit's 160 KiB of LDS (N <= 20), else E = 2.  Byte 0
// of an entry is the window position; its top byte is the slot's factor of
// the window sum (window_sum): 2 for the slot that received the top position
// l_x (u_{l_x+1} is 0; the last swap puts it at slot j_{N-1}, and nothing
// moves it after) and 3 for every other slot (ShuffledPositions).  The slice
// stays valid until the thread's next call.
template <int N>
struct ShuffleSlice {
    static constexpr int E = N <= 20 ? 4 : 2;               // bytes per entry
    static constexpr int ROW = 256 * E;
    using U = typename std::conditional<E == 4, uint32_t, uint16_t>::type;
    static constexpr U entry(int k) { return (U)((U)(k == N - 1 ? 2 : 3) << (8 * (E - 1)) | (U)k); }
};

// The digits of the plan in order: t, then j_1, j_2, ... (k compile-time after
// unrolling).
template <int N>
struct ShuffleDigits {
    const StreamAt& r01;
    Words4 w = {0, 0, 0, 0};
    uint32_t lo = 0, hi = 0;     // the chunk's F
    uint32_t f = 0;              // the group's fraction

    __device__ __forceinline__ explicit ShuffleDigits(const StreamAt& r) : r01(r) {}
    __device__ __forceinline__ uint32_t digit(int k) {
        constexpr ShufflePlan<N> plan{};
        const int c = plan.chunk[k];
        if (k == 0 || plan.chunk[k > 0 ? k - 1 : 0] != c) {
            if (c % 2 == 0) w = r01.block(TAG_SHUFFLE, (uint32_t)(c / 2));
            lo = c % 2 ? w.w2 : w.w0;
            hi = c % 2 ? w.w3 : w.w1;
        }
        if (plan.group[k]) {
            const uint32_t M = plan.prod[k];
            const uint64_t pl = (uint64_t)lo * M;
            const uint64_t ph = (uint64_t)hi * M + (uint32_t)(pl >> 32);
            lo = (uint32_t)pl;
            hi = (uint32_t)ph;
            f = (uint32_t)(ph >> 32) * (uint32_t)ShufflePlan<N>::scale(M);
        }
        const uint32_t m = (uint32_t)ShufflePlan<N>::radix(k);
        const uint64_t p = (m & (m - 1)) == 0 ? mul_wide_s(f, m) : (uint64_t)f * m;
        f = (uint32_t)p;
        uint32_t d = (uint32_t)(p >> 32);                     // t, or j_k <= k
        // d as a register of its own: the entry's address is then one
        // shift-add, where the compiler would otherwise cut d * ROW out
        // of the 64-bit product with an alignbit and a mask
        if (k > 0) asm("" : "+v"(d));
        return d;
    }
};

// This block's LDS array of shuffle entries: one per (N, U), whoever runs the
// shuffle.
template <int N, typename U>
__device__ __forceinline__ U* shuffle_lds() {
    __shared__ U lds[N * 256];
    return lds;
}

// The shuffle proper (digits j_1, ... still to come) over entries of type U,
// entry(k) being the one of position k.  work(k) runs between the read and
// the writes of swap k: independent work placed there covers the read's
// latency where few waves share a SIMD.
template <int N, typename U, typename Entry, typename Work>
__device__ __forceinline__ uint8_t* shuffle_run(ShuffleDigits<N>& digits, Entry&& entry, Work&& work) {
    constexpr int ROW = 256 * (int)sizeof(U);
    uint8_t* A = reinterpret_cast<uint8_t*>(shuffle_lds<N, U>() + threadIdx.x);
    *reinterpret_cast<U*>(A) = entry(0);                      // A[0] = 0
#pragma unroll
    for (int k = 1; k < N; ++k) {
        U* aj = reinterpret_cast<U*>(A + digits.digit(k) * ROW);
        const U old = *aj;
        work(k);
        *reinterpret_cast<U*>(A + k * ROW) = old;             // A[k] = A[j_k]
        *aj = entry(k);                                       // A[j_k] = k
    }
    return A;
}
template <int N, typename U, typename Entry>
__device__ __forceinline__ uint8_t* shuffle_run(ShuffleDigits<N>& digits, Entry&& entry) {
    return shuffle_run<N, U>(digits, entry, [](int) {});
}

// A filled slice of window positions.  The factors are read through a
// pointer of their own: with 2-byte entries the compiler would otherwise read
// both bytes at once and take them apart again on the VALU.
template <int N>
struct ShuffledPositions {
    typedef const __attribute__((address_space(3))) uint8_t LdsByte;
    LdsByte* entries;
    LdsByte* factors;
    __device__ __forceinline__ explicit ShuffledPositions(const uint8_t* A)
        : entries((LdsByte*)A), factors((LdsByte*)A + (ShuffleSlice<N>::E - 1)) {
        if constexpr (ShuffleSlice<N>::E == 2) asm("" : "+v"(factors));
    }
    // Window position of slot s, and its factor of the window sum: 3, or 2 for
    // position l_x.
    __device__ __forceinline__ uint32_t pos(uint32_t s) const { return entries[s * ShuffleSlice<N>::ROW]; }
    __device__ __forceinline__ uint32_t times(uint32_t s) const { return factors[s * ShuffleSlice<N>::ROW]; }
};

// The shuffle of the window positions, after t was taken from the digits.
template <int N, typename Work>
__device__ __forceinline__ ShuffledPositions<N> shuffle_fill(ShuffleDigits<N>& digits, Work&& work) {
    using S = ShuffleSlice<N>;
    using U = typename S::U;
    return ShuffledPositions<N>(shuffle_run<N, U>(digits, [](int k) { return S::entry(k); }, work));
}
template <int N>
__device__ __forceinline__ ShuffledPositions<N> shuffle_fill(ShuffleDigits<N>& digits) {
    return shuffle_fill<N>(digits, [](int) {});
}

// The shuffle as words: byte q of perm[k] is the position of slot 4k + q
// (bytes past N zero).
template <int N>
__device__ __forceinline__ uint32_t shuffle_perm(const StreamAt& r01, uint32_t (&perm)[(N + 3) / 4]) {
    ShuffleDigits<N> digits(r01);
    const uint32_t t = digits.digit(0);
    const ShuffledPositions<N> A = shuffle_fill<N>(digits);
#pragma unroll
    for (int k = 0; k < (N + 3) / 4; ++k) {
        uint32_t v = 0;
#pragma unroll
        for (int q = 0; q < 4 && 4 * k + q < N; ++q) v |= A.pos((uint32_t)(4 * k + q)) << (8 * q);
        perm[k] = v;
    }
    return t;
}

// Layout of the masks r in Z_p^* and reshares z in Z_p of Alg. 7 in the
// seed_01 stream TAG_MASK, per window count N and field:
//  * the default prime at N >= 17 (STREAM): value v = 2s (r of slot s) or
//    2s + 1 (z of slot s) is the N-bit field at bits [N v, N v + N) of the
//    stream, whose bit i is bit i % 32 of word i / 32, word w being word
//    w % 4 of block w / 4; r = min(max(R, 1), p - 1), z = Z mod p.  Up to
//    N = 31 the kernels keep both shifted left by SH = 32 - N: a field is then
//    one v_alignbit_b32 of two stream words, whether it straddles them or
//    not, and P2's test needs no shift back.
//  * otherwise, p < 2^32: two slots to a block, words (0, 1) and (2, 3), by
//    32-bit multiply-shift; p > 2^32: one slot per block, 64-bit words.
template <int N, typename F>
struct MaskDraws {
    static constexpr bool WIDE = std::is_same<typename F::T, uint64_t>::value;
    static constexpr bool STREAM = F::kDefault && N >= 17;
    static constexpr int SPB = WIDE ? 1 : 2;                                            // slots per block otherwise
    static constexpr int NB = STREAM ? (2 * N * N + 127) / 128 : (N + SPB - 1) / SPB;   // blocks per element
    static constexpr int SH = STREAM && N <= 31 ? 32 - N : 0;                           // shift of the kept r and z
};

// r and z in the kept representation from the raw fields R, Z (STREAM,
// already shifted left by SH).  z is left as the field, a value below 2^N
// congruent to Z mod p (reduced_z finishes it where a message is stored).
template <int N, typename F>
__device__ __forceinline__ void stream_draws(typename F::T R, typename F::T Z, typename F::T& r,
                                             typename F::T& z) {
    using FT = typename F::T;
    z = Z;
    if constexpr (MaskDraws<N, F>::WIDE) {
        // r = min(max(R, 1), p - 1) for p = 2^33 - 9, word by word: with bit 32
        // set the low word is at most 2^32 - 10, without it at least 1
        const uint32_t r1 = (uint32_t)(R >> 32);
        const uint32_t low = min((uint32_t)R, ~((0u - r1) & 9u));
        r = join64(max(low, r1 ^ 1u), r1);
    } else {
        // clamp into Z_p^* (one v_med3); the low SH bits of r are cleared, so
        // that a product r s has zero low SH bits.  z keeps whatever bits Z
        // carries below SH: an addend's low SH bits stay below bit SH of
        // a r + z and cancel in P2's difference, and a subtraction from z masks
        // them first (reshare_neg).
        constexpr int SH = MaskDraws<N, F>::SH;
        constexpr FT KEEP = (FT)~(((FT)1 << SH) - 1);
        r = min(max((FT)(R & KEEP), (FT)((FT)1 << SH)), (FT)((FT)(F::p - 1) << SH));
    }
}

// A kept z (shifted by SH) as Z mod p, still shifted (a Mersenne Z = p may
// stay: it stands for 0 and is a valid addend).
template <int N, typename F>
__device__ __forceinline__ typename F::T reduced_z(const F& f, typename F::T z) {
    using FT = typename F::T;
    using D = MaskDraws<N, F>;
    if constexpr (D::STREAM) {
        if constexpr (F::p != (FT)((1ull << N) - 1)) return min(z, (FT)(z - ((FT)F::p << D::SH)));
    }
    return z;
}

// Slot H's r and z of mask block w without STREAM (H < SPB, compile-time).
template <int N, typename F, int H>
__device__ __forceinline__ void block_draws(const Words4& w, const F& f, typename F::T& r, typename F::T& z) {
    if constexpr (MaskDraws<N, F>::WIDE) {
        r = 1 + __umul64hi(join64(w.w0, w.w1), f.p - 1);
        z = __umul64hi(join64(w.w2, w.w3), f.p);
    } else {
        r = draw_r(H ? w.w2 : w.w0, f.p);
        z = draw_z(H ? w.w3 : w.w1, f.p);
    }
}

// The masks of one element slot after slot (j compile-time after unrolling):
// with STREAM the block holding a field's last bit is fetched when the
// previous field ended in an earlier block, and that block's last word kept
// for a field that straddles the two (a field spans at most two words);
// otherwise block j / SPB is fetched at its first slot.  Every decision
// depends on j alone, so it folds away once the slot loop is unrolled.
template <int N, typename F>
struct MaskReader {
    using FT = typename F::T;
    using D = MaskDraws<N, F>;
    Words4 cur = {0, 0, 0, 0};
    uint32_t prev = 0;     // the last word of the block before cur

    // Word w of the stream, with block b current (w >= 4 b - 1).
    __device__ __forceinline__ uint32_t word(int w, int b) const {
        const int q = w - 4 * b;
        return q < 0 ? prev : q == 0 ? cur.w0 : q == 1 ? cur.w1 : q == 2 ? cur.w2 : cur.w3;
    }
    // The raw field of value v (shifted left by SH; with SH > 0 the low SH
    // bits are left as they come, see stream_draws).
    __device__ __forceinline__ FT field(const StreamAt& r01, int v, bool first) {
        const int o = N * v;
        const int b = (o + N - 1) / 128;                    // the block of the field's last bit
        if (first && o / 128 != b) cur = r01.block(TAG_MASK, (uint32_t)b - 1);   // a field that straddles two blocks
        if (first || o == 0 || (o - 1) / 128 != b) {        // the previous field ended in an earlier block
            prev = cur.w3;
            cur = r01.block(TAG_MASK, (uint32_t)b);
        }
        if constexpr (D::SH > 0) {
            const int lo = o + N - 32;              // the field is the top of the word [lo, lo + 32)
            if (lo < 0) return word(0, b) << D::SH;
            const int k = lo / 32, s = lo % 32;
            if (s == 0) return word(k, b);
            return __builtin_amdgcn_alignbit(word(k + 1, b), word(k, b), s);
        } else if constexpr (D::WIDE) {
            const int k = o / 32, s = o % 32;       // 33 bits: always two words
            return join64(__builtin_amdgcn_alignbit(word(k + 1, b), word(k, b), s), (word(k + 1, b) >> s) & 1u);
        } else {
            const int k = o / 32, s = o % 32;
            constexpr uint32_t M = N >= 32 ? ~0u : (1u << N) - 1;
            if (s + N <= 32) return (word(k, b) >> s) & M;
            return __builtin_amdgcn_alignbit(word(k + 1, b), word(k, b), s) & M;
        }
    }
    // Slot j's draws; `first` for the first slot read when that is not slot 0.
    __device__ __forceinline__ void slot(const StreamAt& r01, int j, const F& f, FT& r, FT& z, bool first = false) {
        if constexpr (D::STREAM) {
            const FT R = field(r01, 2 * j, first);
            const FT Z = field(r01, 2 * j + 1, false);
            stream_draws<N, F>(R, Z, r, z);
        } else {
            constexpr int SPB = D::SPB;
            if (first || j % SPB == 0) cur = r01.block(TAG_MASK, (uint32_t)(j / SPB));
            if (j % SPB == 0)
                block_draws<N, F, 0>(cur, f, r, z);
            else
                block_draws<N, F, (SPB > 1 ? 1 : 0)>(cur, f, r, z);
        }
    }
};

// Plain canonical values of kept draws (captured messages, the record of the
// precomputed mode).
template <int N, typename F>
__device__ __forceinline__ void plain_draws(const F& f, typename F::T& r, typename F::T& z) {
    using D = MaskDraws<N, F>;
    if constexpr (D::STREAM) {
        using FT = typename F::T;
        r >>= D::SH;
        z >>= D::SH;
        z = min(z, (FT)(z - f.p));
    }
}

// Alg. 7 from the flip through P2's zero test for one element: the 2-of-2
// input (in0, -n1) of Z_{2^l} (n1: P1's negated share, see input_shares),
// randomness of global index g.  Returns D'
// (1 when some slot reconstructs to 0) and the flip bit t.  With CAP the
// round-1 messages go to cap[e * N + slot] (P0) and cap[(ncap + e) * N +
// slot] (P1).
template <typename T, int N, typename F, bool CAP>
__device__ __forceinline__ T drelu_round1(T in0, T n1, Index g, T mask, uint32_t k_lo, const Stream& s01,
                                          typename F::T* cap, uint64_t ncap, uint64_t e, const F& f,
                                          uint32_t& t_out) {
    using FT = typename F::T;
    constexpr bool WIDE = std::is_same<FT, uint64_t>::value;
    static_assert(WIDE == (N == 33), "64-bit field elements exactly when l_x = 32");

    const StreamAt r01 = s01.at(g);
    using Test = SlotTest<N, F, MaskDraws<N, F>::SH>;
    Test test;
    LeastMark<N> p2;
    MaskReader<N, F> masks;
    ShuffleDigits<N> digits(r01);
    const uint32_t t = digits.digit(0);
    t_out = t;

    // Flip: [x] := (-1)^t [x]  (both parties); P1 cuts its negated share
    // -(-1)^t [x]_1 = (-1)^t n1.  Then the common low cut of every window.
    const T a0k = flip_by(in0, t, mask) >> k_lo, nb1k = flip_by(n1, t, mask) >> k_lo;

    if constexpr (kPairs<N> && !CAP) {
        PairWindows<T, N> win(a0k, nb1k, in_vgpr(0xFFFFFFFEu));
        const uint8_t* A = shuffle_run<N, uint32_t>(digits, [&](int k) { return win.value(k); });
#pragma unroll
        for (int j = 0; j < N; ++j) {
            FT r, z;
            masks.slot(r01, j, f, r, z);
            p2.take(j, Test::mark_pair(*reinterpret_cast<const uint32_t*>(A + j * 1024), r, z, f));
        }
    } else {
        const ShuffledPositions<N> A = shuffle_fill<N>(digits);
#pragma unroll
        for (int j = 0; j < N; ++j) {
            FT r, z;
            masks.slot(r01, j, f, r, z);
            uint32_t v0, v1;
            window_sums<T, N>(a0k, nb1k, A.pos(j), A.times(j), v0, v1);
            if constexpr (CAP) {
                FT w0, w1;
                plain_draws<N, F>(f, r, z);
                slot_messages<F>(v0, v1, r, z, f, w0, w1);
                cap[e * N + j] = w0;
                cap[(ncap + e) * N + j] = w1;
                const FT w = addmod(w0, w1, f);                // P2 reconstructs and tests
                p2.take(j, w == 0 ? 0u : 0xFFFFFFFFu);
            } else {
                p2.take(j, test.mark(v0, v1, r, z, f));
            }
        }
    }
    return p2.least <= Test::LIMIT ? 1 : 0;                // D' = [some slot is 0]
}

// One element, all three parties.  N = l_x + 1 windows, fixed at compile
// time: every loop over windows and slots is unrolled and all window masks
// are constants.  From the loaded shares x0, x1 to the output shares y0,
// y1; the randomness belongs to global index g, and e is the element's
// index in the call (for the capture).  With CAP, the round-1 messages are captured
// (drelu_round1).  With k_in > 0 the inputs are shares of Z_{2^(l + k_in)}
// (in_mask) and are first truncated by k_in bits into Z_{2^l} (Alg. 5); with
// k_in = 0 and in_mask = mask the same expressions are the plain load.
template <typename T, int N, typename F, bool RELU, bool CAP>
__device__ __forceinline__ void drelu_element_of(T x0, T x1, T& y0, T& y1, typename F::T* cap, uint64_t ncap,
                                                 uint64_t e, Index g, T mask, T in_mask, uint32_t k_in,
                                                 uint32_t k_lo, const Stream& s01, const Stream& s02,
                                                 const Stream& s12, const F& f) {
    T in0, n1;
    input_shares<T>(x0, x1, mask, in_mask, k_in, in0, n1);

    uint32_t t;
    const T dp = drelu_round1<T, N, F, CAP>(in0, n1, g, mask, k_lo, s01, cap, ncap, e, f, t);

    if constexpr (!RELU) {
        const Words4 w = s02.block(g, TAG_RESP, 0);               // rho from seed_02
        drelu_finish<T>(dp, (T)join64(w.w0, w.w1), t, mask, y0, y1);
    } else {
        const T in1 = (T)((T)0 - n1) & mask;
        // Alg. 8 preprocessing; P2 forms [c]_1 = (a0 + a1)(b0 + b1) - c0.
        T ba0, bb0, bc0, ba1, bb1;
        beaver_shares<T>(s02, s12, g, mask, ba0, bb0, bc0, ba1, bb1);
        const T bc1 = (T)((T)(ba0 + ba1) * (T)(bb0 + bb1) - bc0) & mask;
        relu_finish<T>(dp, in0, in1, ba0, bb0, bc0, ba1, bb1, bc1, t, mask, y0, y1);
    }
}

// drelu_element_of from X0[e], X1[e] to Y0[e], Y1[e].
template <typename T, int N, typename F, bool RELU, bool CAP>
__device__ __forceinline__ void drelu_element(const T* __restrict__ X0, const T* __restrict__ X1, T* Y0, T* Y1,
                                              typename F::T* cap, uint64_t ncap, uint64_t e, Index g, T mask,
                                              T in_mask, uint32_t k_in, uint32_t k_lo, const Stream& s01,
                                              const Stream& s02, const Stream& s12, const F& f) {
    T y0, y1;
    drelu_element_of<T, N, F, RELU, CAP>(ld_nt(&X0[e]), ld_nt(&X1[e]), y0, y1, cap, ncap, e, g, mask, in_mask, k_in,
                                         k_lo, s01, s02, s12, f);
    st_nt(&Y0[e], y0);
    st_nt(&Y1[e], y1);
}

// Element i of the buffer r (a raw buffer of 4- or 8-byte elements), loaded
// nontemporal; an element past the buffer's end reads as 0 without a memory
// access (the buffer's range check).
template <typename T>
__device__ __forceinline__ T load_buf(__amdgpu_buffer_rsrc_t r, uint32_t i) {
    constexpr int kNontemporal = 2;
    if constexpr (sizeof(T) == 8) {
        const auto w = __builtin_amdgcn_raw_buffer_load_b64(r, i * 8u, 0, kNontemporal);
        return (T)w[0] | ((T)w[1] << 32);
    } else {
        return (T)__builtin_amdgcn_raw_buffer_load_b32(r, i * 4u, 0, kNontemporal);
    }
}

// A raw buffer over n elements of T at p (word 3: the gfx9 data format of
// raw, unswizzled buffers).
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const T* p, uint32_t n) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), (short)0, (int)(n * (uint32_t)sizeof(T)), 0x00020000);
}

// The loop of one k_drelu launch (see k_drelu), with the ring mask given.
template <typename T, int N, typename F, bool RELU, bool CAP>
__device__ __forceinline__ void drelu_launch_loop(const DreluKArgs& A, const F& f, T mask) {
    const T* X0 = static_cast<const T*>(A.x0);
    const T* X1 = static_cast<const T*>(A.x1);
    T* Y0 = static_cast<T*>(A.y0);
    T* Y1 = static_cast<T*>(A.y1);
    typename F::T* cap = static_cast<typename F::T*>(A.cap);
    const uint32_t n = (uint32_t)A.n;
    const uint32_t stride = gridDim.x * blockDim.x;
    uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const __amdgpu_buffer_rsrc_t B0 = buffer_of(X0, n), B1 = buffer_of(X1, n);
    T x0 = load_at(X0, e), x1 = load_at(X1, e);
    // Wait for the first shares before the loop: its head then waits on no
    // memory operation (later entries have only the last stores outstanding).
    asm volatile("" : "+v"(x0), "+v"(x1));
    for (;;) {
        const uint32_t en = e + stride;
        const T x0n = load_buf<T>(B0, en), x1n = load_buf<T>(B1, en);   // past the last: 0, no access
        T y0, y1;
        drelu_element_of<T, N, F, RELU, CAP>(x0, x1, y0, y1, cap, A.ncap, e, Index::of(A.elem_base, e), mask,
                                             (T)A.in_mask,
                                             A.k_in, A.k_lo, A.s01, A.s02, A.s12, f);
        store_at(Y0, e, y0);
        store_at(Y1, e, y1);
        if (en >= n) break;
        e = en;
        x0 = x0n;
        x1 = x1n;
    }
}

// One launch: grid-stride over its n <= kLaunchElems elements of one share
// pair.  Each thread loads its next element's shares before computing the
// current one, so the loads have a whole element's work to land: with other
// traffic on the memory system (the truncation beside it), a load at the top
// of each element stalled the kernel.
template <typename T, int N, typename F, bool RELU, bool CAP>
__global__ BC_KERNEL_ATTRS void k_drelu(DreluKArgs A, F f_arg) {
    const F f = f_arg.vgpr();
    // A full-width ring (l = 64 in 64-bit storage, l = 32 in 32-bit) makes
    // every reduction mod 2^l a no-op: that loop runs with the mask as a
    // constant, so the compiler drops the masking instructions.
    if constexpr (!CAP) {
        if ((T)A.ring_mask == (T)~(T)0) {
            drelu_launch_loop<T, N, F, RELU, CAP>(A, f, (T)~(T)0);
            return;
        }
    }
    drelu_launch_loop<T, N, F, RELU, CAP>(A, f, in_vgpr((T)A.ring_mask));
}

// Small calls: G waves of a block share 64 elements, so a call of n elements
// still runs n G threads.  Role r of the G takes a fixed range of slots
// (compile-time, so its mask fields and blocks are constants as in the
// one-wave kernel), draws the masks of those slots only, runs the whole
// shuffle in its own LDS slices, and hands its P2 minimum to role 0 through
// LDS; role 0 also draws the reply (DReLU) or the triple (ReLU), finishes and
// writes, and takes fewer slots for it.  The mask draws are placed between the
// shuffle's LDS reads and writes, whose latency nothing else covers at one or
// two waves on a SIMD.  Results are those of drelu_element: same draws, same
// slots, same messages.
// Splitting the slots over waves keeps every field offset a constant, where
// lanes of one wave with different slots read their fields from LDS at computed
// addresses (1,650 instructions an element and lane at N = 33 with two lanes,
// against 1,286 here): DReLU at 65,536 elements, N = 33 9.8 -> 8.5 us, N = 19
// 5.1 -> 4.5 us with two; 16,384 elements with four 6.4 -> 5.7 and 3.9 -> 3.7.
template <int N, int FINISH, int G>
struct WaveSlots {
    // VALU instructions, roughly: a slot with its share of the mask blocks (and
    // FINISH, role 0's draws and finish)
    static constexpr int SLOT = N <= 16 ? 24 : N <= 32 ? 19 + N / 2 : 58;
    static constexpr int first_count() {
        const int c = ((N * SLOT + FINISH) / G - FINISH + SLOT / 2) / SLOT;
        return c < 0 ? 0 : c;
    }
    // The first slot of role r (r = G: N).
    static constexpr int begin(int r) { return r == 0 ? 0 : first_count() + (N - first_count()) * (r - 1) / (G - 1); }
};

// Role ROLE's part of the element (in0, -n1): P2's minimum over its slots, and
// the flip bit t.
template <typename T, int N, typename F, int FINISH, int G, int ROLE>
__device__ __forceinline__ uint32_t wave_slots(T in0, T n1, Index g, T mask, uint32_t k_lo, const Stream& s01, const F& f,
                                               uint32_t& t) {
    using FT = typename F::T;
    using W = WaveSlots<N, FINISH, G>;
    using Test = SlotTest<N, F, MaskDraws<N, F>::SH>;
    constexpr int J0 = W::begin(ROLE), C = W::begin(ROLE + 1) - J0;
    const StreamAt r01 = s01.at(g);
    ShuffleDigits<N> digits(r01);
    t = digits.digit(0);
    uint32_t least = 0xFFFFFFFFu;
    if constexpr (C > 0) {
        const T a0k = flip_by(in0, t, mask) >> k_lo, nb1k = flip_by(n1, t, mask) >> k_lo;   // as in drelu_round1
        MaskReader<N, F> masks;
        FT r[C], z[C];
        int drawn = 0;
        const auto draw_until = [&](int count) {             // compile-time counts, once unrolled
#pragma unroll
            for (int i = 0; i < C; ++i)
                if (i >= drawn && i < count) masks.slot(r01, J0 + i, f, r[i], z[i], i == 0 && J0 > 0);
            drawn = drawn > count ? drawn : count;
        };
        const auto work = [&](int k) { draw_until((k * C + N - 2) / (N - 1)); };
        if constexpr (kPairs<N>) {
            PairWindows<T, N> win(a0k, nb1k, in_vgpr(0xFFFFFFFEu));
            const uint8_t* A = shuffle_run<N, uint32_t>(digits, [&](int k) { return win.value(k); }, work);
#pragma unroll
            for (int i = 0; i < C; ++i)
                least = min(least, Test::mark_pair(*reinterpret_cast<const uint32_t*>(A + (J0 + i) * 1024), r[i], z[i], f));
        } else {
            const ShuffledPositions<N> A = shuffle_fill<N>(digits, work);
            Test test;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                uint32_t v0, v1;
                window_sums<T, N>(a0k, nb1k, A.pos(J0 + i), A.times(J0 + i), v0, v1);
                least = min(least, test.mark(v0, v1, r[i], z[i], f));
            }
        }
    }
    return least;
}

template <typename T, int N, typename F, int FINISH, int G, int ROLE>
__device__ __forceinline__ uint32_t wave_role(uint32_t role, T in0, T n1, Index g, T mask, uint32_t k_lo, const Stream& s01,
                                              const F& f, uint32_t& t) {
    if constexpr (ROLE == G - 1) {
        return wave_slots<T, N, F, FINISH, G, ROLE>(in0, n1, g, mask, k_lo, s01, f, t);
    } else {
        if (role == ROLE) return wave_slots<T, N, F, FINISH, G, ROLE>(in0, n1, g, mask, k_lo, s01, f, t);
        return wave_role<T, N, F, FINISH, G, ROLE + 1>(role, in0, n1, g, mask, k_lo, s01, f, t);
    }
}

// Blocks of 256 threads take 256 / G elements at a time: wave w serves
// elements 64 (w / G) .. + 63 of them in role w % G.  The loop bound is the
// block's, so every wave reaches both barriers the same number of times; a
// lane past the last element works on that element and writes nothing.
template <typename T, int N, typename F, bool RELU, int G>
__global__ BC_KERNEL_ATTRS void k_drelu_waves(DreluKArgs A, F f_arg) {
    static_assert(G == 2 || G == 4, "G: waves of a 256-thread block that share elements");
    constexpr uint32_t EPB = 256 / G;
    __shared__ uint32_t least_of[256];
    const F f = f_arg.vgpr();
    const T* X0 = static_cast<const T*>(A.x0);
    const T* X1 = static_cast<const T*>(A.x1);
    T* Y0 = static_cast<T*>(A.y0);
    T* Y1 = static_cast<T*>(A.y1);
    const T mask = in_vgpr((T)A.ring_mask);
    const uint32_t n = (uint32_t)A.n;                        // at most kLaunchElems
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), role = wave % G;
    for (uint32_t b = blockIdx.x * EPB; b < n; b += gridDim.x * EPB) {
        const uint32_t want = b + (wave / G) * 64 + (threadIdx.x & 63u);
        const uint32_t e = want < n ? want : n - 1;
        const Index g = Index::of(A.elem_base, e);
        T in0, n1;
        input_shares<T>(load_at(X0, e), load_at(X1, e), mask, (T)A.in_mask, A.k_in, in0, n1);
        uint32_t t;
        uint32_t least = wave_role<T, N, F, (RELU ? 165 : 45), G, 0>(role, in0, n1, g, mask, A.k_lo, A.s01, f, t);
        if (role != 0) least_of[threadIdx.x] = least;
        T ba0 = 0, bb0 = 0, bc0 = 0, ba1 = 0, bb1 = 0, rho = 0;
        if (role == 0) {                                     // role 0's draws, before it waits
            if constexpr (RELU) {
                beaver_shares<T>(A.s02, A.s12, g, mask, ba0, bb0, bc0, ba1, bb1);
            } else {
                const Words4 w = A.s02.block(g, TAG_RESP, 0);
                rho = (T)join64(w.w0, w.w1);
            }
        }
        __syncthreads();
        if (role == 0) {
#pragma unroll
            for (int r = 1; r < G; ++r) least = min(least, least_of[threadIdx.x + 64 * r]);
            const T dp = least <= SlotTest<N, F, MaskDraws<N, F>::SH>::LIMIT ? 1 : 0;
            T y0, y1;
            if constexpr (RELU) {
                const T in1 = (T)((T)0 - n1) & mask;
                const T bc1 = (T)((T)(ba0 + ba1) * (T)(bb0 + bb1) - bc0) & mask;
                relu_finish<T>(dp, in0, in1, ba0, bb0, bc0, ba1, bb1, bc1, t, mask, y0, y1);
            } else {
                drelu_finish<T>(dp, rho, t, mask, y0, y1);
            }
            if (want < n) {
                store_at(Y0, e, y0);
                store_at(Y1, e, y1);
            }
        }
        __syncthreads();                                     // role 0 has read before the next elements' minima
    }
}

// Host helpers: field parameters for each prime size.
inline FieldSmall make_field_small(uint64_t p) { return FieldSmall{(uint32_t)p, 1.0f / (float)p, inverse32((uint32_t)p)}; }
inline Field24 make_field24(uint64_t p) { return Field24{(uint32_t)p, (double)p, 1.0 / (double)p, inverse32((uint32_t)p)}; }
inline Field32 make_field32(uint64_t p) { return Field32{(uint32_t)p, UINT64_MAX / p, inverse32((uint32_t)p)}; }
inline Field64 make_field64(uint64_t p) { return Field64{p, (double)p, 1.0 / (double)p}; }

inline DreluKArgs make_kargs(const DreluLaunch& L) {
    DreluKArgs A;
    A.x0 = L.x0;
    A.x1 = L.x1;
    A.y0 = L.y0;
    A.y1 = L.y1;
    A.cap = L.cap;
    A.n = L.n;
    A.ncap = L.n;
    A.elem_base = L.elem_base;
    A.ring_mask = L.ell >= 64 ? ~0ull : ((1ull << L.ell) - 1);
    A.in_mask = L.ell + L.k_in >= 64 ? ~0ull : ((1ull << (L.ell + L.k_in)) - 1);
    A.k_lo = L.k_lo;
    A.k_in = L.k_in;
    A.s01 = Stream{L.s01.k0, L.s01.k1, L.s01.n0, L.s01.n1};
    A.s02 = Stream{L.s02.k0, L.s02.k1, L.s02.n0, L.s02.n1};
    A.s12 = Stream{L.s12.k0, L.s12.k1, L.s12.n0, L.s12.n1};
    return A;
}

// Calls launch(begin, end) for the consecutive ranges of n elements of at most
// kLaunchElems that share the high word of their global index, and returns the
// first launch error.
template <typename Fn>
hipError_t by_index_range(uint64_t elem_base, uint64_t n, Fn&& launch) {
    for (uint64_t begin = 0, end; begin < n; begin = end) {
        end = index_end(elem_base, begin, n);
        if (end - begin > kLaunchElems) end = begin + kLaunchElems;
        launch(begin, end);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

template <typename T, int N, typename F, bool RELU>
hipError_t launch_field(const DreluLaunch& L, const F& f, hipStream_t st) {
    const DreluKArgs A = make_kargs(L);
    // consecutive ranges of at most kLaunchElems elements that share the high
    // word of their global index
    for (uint64_t off = 0, end; off < L.n; off = end) {
        end = index_end(L.elem_base, off, L.n);
        if (end - off > kLaunchElems) end = off + kLaunchElems;
        DreluKArgs R = A;
        R.n = end - off;
        R.x0 = static_cast<const T*>(A.x0) + off;
        R.x1 = static_cast<const T*>(A.x1) + off;
        R.y0 = static_cast<T*>(A.y0) + off;
        R.y1 = static_cast<T*>(A.y1) + off;
        R.elem_base = A.elem_base + off;
        if (L.cap) R.cap = static_cast<typename F::T*>(A.cap) + off * N;
        if (L.group == 4)
            hipLaunchKernelGGL((k_drelu_waves<T, N, F, RELU, 4>), dim3(L.grid), dim3(L.block), 0, st, R, f);
        else if (L.group == 2)
            hipLaunchKernelGGL((k_drelu_waves<T, N, F, RELU, 2>), dim3(L.grid), dim3(L.block), 0, st, R, f);
        else if (L.cap)
            hipLaunchKernelGGL((k_drelu<T, N, F, RELU, true>), dim3(L.grid), dim3(L.block), 0, st, R, f);
        else
            hipLaunchKernelGGL((k_drelu<T, N, F, RELU, false>), dim3(L.grid), dim3(L.block), 0, st, R, f);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

constexpr bool mersenne_exponent(int k) { return k == 13 || k == 17 || k == 19; }   // 2^k - 1 prime, 12 < k <= 24

// Calls fn(field) with the Z_p arithmetic for N = l_x + 1 (p has N bits):
// for the default primes the Mersenne fold (2^13 - 1, 2^17 - 1, 2^19 - 1)
// or the pseudo-Mersenne folds (every other default prime up to 2^33); for
// any other prime fp32-quotient 24-bit products (p < 2^12), an fp64
// quotient (p < 2^24), Barrett (p < 2^32), or the 128-bit product with an
// fp64 quotient (l_x = 32).
template <int N, typename Fn>
hipError_t with_field(uint64_t p, Fn&& fn) {
    if constexpr (N <= 12) {
        if (p == (1ull << N) - kPrimeDelta[N]) return fn(FieldPM<N, kPrimeDelta[N]>{});
        return fn(make_field_small(p));
    } else if constexpr (N <= 32) {
        if constexpr (mersenne_exponent(N)) {
            if (p == (1ull << N) - 1) return fn(FieldMersenne<N>{});
        } else {
            if (p == (1ull << N) - kPrimeDelta[N]) return fn(FieldPM<N, kPrimeDelta[N]>{});
        }
        if constexpr (N <= 24)
            return fn(make_field24(p));
        else
            return fn(make_field32(p));
    } else {
        if (p == (1ull << 33) - kPrimeDelta[33]) return fn(FieldPM33{});
        return fn(make_field64(p));
    }
}

// The field type follows from N = l_x + 1 (p has N bits), and from p itself
// when p is a Mersenne prime.
template <typename T, int N, bool RELU>
hipError_t launch_exact(const DreluLaunch& L, hipStream_t st) {
    return with_field<N>(L.p, [&](auto f) { return launch_field<T, N, decltype(f), RELU>(L, f, st); });
}

template <typename T, bool RELU, int NLO, int NHI>
hipError_t launch_range(const DreluLaunch& L, hipStream_t st) {
    if constexpr (NLO > NHI) {
        return hipErrorInvalidValue;
    } else {
        if (L.npos == (uint32_t)NLO) return launch_exact<T, NLO, RELU>(L, st);
        return launch_range<T, RELU, NLO + 1, NHI>(L, st);
    }
}

}  // namespace bc
