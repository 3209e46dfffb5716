// The DReLU (Alg. 7) with the parties apart: each party's part as its own
// kernel, the round-1 messages bit-packed as they would cross a link.
//
//   k_send<P>   P0 or P1 alone, from its own share: flip, windows, adjacent
//               sums, modulo switch, shuffle, mask and reshare (the same
//               draws and slot arithmetic as the fused kernel), then the N
//               slot values of N bits each packed into ceil(N^2 / 32) words:
//               bit b of slot s is bit s N + b of the element's string, word
//               k holds bits 32k .. 32k + 31, stored word-major (msg[k n + i])
//               so that every word plane is one coalesced stream.
//   k_reply     P2: unpacks both messages, reconstructs every slot, D' = [some
//               slot is 0], and writes its reply shares (rho, D' - rho).
//   k_finish<P> P0 or P1 unflips its reply share with t.
// Every step before P2 uses one share only, so k_send reads one array.  Sends
// are bound by VALU issue up to N = 19 (591 instructions, P1 609, 264 of them Philox,
// 1,000,003 elements: 21 us) and by the message's writes above; the reply (202
// instructions) and the finish by memory: N = 19, 16.6 us, 6.7 TB/s out of the
// memory-side cache (21.6 us with nontemporal loads in block order).
#pragma once

#include "drelu_kernel.h"

namespace bc {

struct SplitKArgs {
    const void* in0;      // send: the party's share; reply: P0's message; finish: the reply share
    const void* in1;      // reply: P1's message
    void* out0;           // send: the message; reply: P0's reply share; finish: the output share
    void* out1;           // reply: P1's reply share
    uint64_t n, begin, end;   // this launch: elements [begin, end) of the call's n
    uint64_t elem_base, ring_mask;
    uint32_t k_lo;
    Stream s01, s02;
};

// One party's message for one slot in [0, p) (the P0 or P1 half of the fused
// kernel's slot).  ak: the party's flipped share (P1: its negation) shifted
// down by k_lo; r and z in the kept representation of MaskDraws (shifted
// left by SH).
template <typename T, int N, typename F, int PARTY, int SH = MaskDraws<N, F>::SH>
__device__ __forceinline__ typename F::T party_message(T ak, uint32_t pos, uint32_t times, typename F::T r,
                                                       typename F::T z, const F& f) {
    using FT = typename F::T;
    z = reduced_z<N, F>(f, z);
    if constexpr (PARTY == 0)                                            // s_0 = v_0 + 1
        return field_mul_add<SH>(f, (FT)window_sum<T, N, 2>(ak, pos, times) + 1, r, z);
    else                                                                 // s_1 = p - (v_1 + 1)
        return field_mul_add<SH>(f, (FT)((f.p - 1) - window_sum<T, N, 1>(ak, pos, times)), r, reshare_neg<SH>(f, z));
}

template <int N>
struct Packing {
    static constexpr int W = (N * N + 31) / 32;
};

// OR an N-bit value into the element's words at bit offset j N (j constant
// after unrolling, so every index and shift is too).
template <int N>
__device__ __forceinline__ void pack_slot(uint32_t (&w)[Packing<N>::W], int j, uint64_t v) {
    const int off = j * N, wi = off >> 5, sh = off & 31;
    w[wi] |= (uint32_t)(v << sh);
    if (sh + N > 32 && wi + 1 < Packing<N>::W) w[wi + 1] |= (uint32_t)(v >> (32 - sh));
}

template <int N>
__device__ __forceinline__ uint64_t unpack_slot(const uint32_t (&w)[Packing<N>::W], int j) {
    const int off = j * N, wi = off >> 5, sh = off & 31;
    uint64_t v = (uint64_t)w[wi] >> sh;
    if (sh + N > 32 && wi + 1 < Packing<N>::W) v |= (uint64_t)w[wi + 1] << (32 - sh);
    return v & ((1ull << N) - 1);
}

template <typename T, int N, typename F, int PARTY, bool NT>
__global__ BC_KERNEL_ATTRS void k_send(SplitKArgs A, F f_arg) {
    using FT = typename F::T;
    constexpr int W = Packing<N>::W;
    const F f = f_arg.vgpr();
    const T* X = static_cast<const T*>(A.in0);
    uint32_t* M = static_cast<uint32_t*>(A.out0);
    const T mask = in_vgpr((T)A.ring_mask);
    const WalkRange R = walk_range<!NT>((uint32_t)(A.end - A.begin));
    // a 64-bit element: with a 32-bit offset from scalar bases the compiler
    // keeps a pointer for every word plane (N = 32: 98 registers for 79)
    for (uint64_t e = A.begin + R.begin; e < A.begin + R.end; e += R.stride) {
        const Index g = Index::of(A.elem_base + A.begin, e - A.begin);
        const T x = X[e] & mask;
        const StreamAt r01 = A.s01.at(g);
        ShuffleDigits<N> digits(r01);
        const uint32_t t = digits.digit(0);
        const ShuffledPositions<N> sig = shuffle_fill<N>(digits);
        // the flipped share (-1)^t x; P1 cuts its negation (-1)^(t+1) x
        const T ak = flip_by(x, PARTY == 0 ? t : t ^ 1u, mask) >> A.k_lo;
        uint32_t words[W];
#pragma unroll
        for (int k = 0; k < W; ++k) words[k] = 0;
        MaskReader<N, F> masks;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            FT r, z;
            masks.slot(r01, j, f, r, z);
            pack_slot<N>(words, j, (uint64_t)party_message<T, N, F, PARTY>(ak, sig.pos(j), sig.times(j), r, z, f));
        }
#pragma unroll
        for (int k = 0; k < W; ++k) st_plane<NT>(&M[(uint64_t)k * A.n + e], words[k]);
    }
}

template <typename T, int N, typename F, bool NT>
__global__ BC_KERNEL_ATTRS void k_reply(SplitKArgs A, F f_arg) {
    using FT = typename F::T;
    constexpr int W = Packing<N>::W;
    const F f = f_arg.vgpr();
    const uint32_t* M0 = static_cast<const uint32_t*>(A.in0);
    const uint32_t* M1 = static_cast<const uint32_t*>(A.in1);
    T* D0 = static_cast<T*>(A.out0);
    T* D1 = static_cast<T*>(A.out1);
    const T mask = in_vgpr((T)A.ring_mask);
    const WalkRange R = walk_range<!NT>((uint32_t)(A.end - A.begin));
    for (uint64_t e = A.begin + R.begin; e < A.begin + R.end; e += R.stride) {
        uint32_t w0[W], w1[W];
#pragma unroll
        for (int k = 0; k < W; ++k) {
            w0[k] = ld_plane<NT>(&M0[(uint64_t)k * A.n + e]);
            w1[k] = ld_plane<NT>(&M1[(uint64_t)k * A.n + e]);
        }
        FT least = f.p;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const FT v = addmod((FT)unpack_slot<N>(w0, j), (FT)unpack_slot<N>(w1, j), f);
            least = v < least ? v : least;
        }
        const T dp = least == 0 ? 1 : 0;                              // D'
        const Words4 w = A.s02.block(Index::of(A.elem_base + A.begin, e - A.begin), TAG_RESP, 0);    // rho from seed_02
        const T rho = (T)join64(w.w0, w.w1) & mask;
        st_nt(&D0[e], rho);
        st_nt(&D1[e], (T)((T)(dp - rho) & mask));
    }
}

template <typename T, int PARTY>
__global__ __launch_bounds__(256) void k_finish(SplitKArgs A) {
    const T* D = static_cast<const T*>(A.in0);
    T* Y = static_cast<T*>(A.out0);
    const T mask = (T)A.ring_mask;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t e = A.begin + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < A.end; e += stride) {
        // t is the shuffle's first digit (radix 2) of chunk 0: the top bit of its high word
        const uint32_t t = A.s01.block(Index::of(A.elem_base + A.begin, e - A.begin), TAG_SHUFFLE, 0).w1 >> 31;
        const T d = D[e] & mask;
        if constexpr (PARTY == 0)
            Y[e] = (T)((d ^ ((T)0 - (T)t)) + (T)(2 * t)) & mask;      // t + (1 - 2t) d
        else
            Y[e] = flip_by(d, t, mask);                              // (1 - 2t) d
    }
}

inline SplitKArgs make_split_kargs(const SplitLaunch& L) {
    SplitKArgs A;
    A.in0 = L.in0;
    A.in1 = L.in1;
    A.out0 = L.out0;
    A.out1 = L.out1;
    A.n = L.n;
    A.elem_base = L.elem_base;
    A.ring_mask = L.ell >= 64 ? ~0ull : ((1ull << L.ell) - 1);
    A.k_lo = L.k_lo;
    A.s01 = Stream{L.s01.k0, L.s01.k1, L.s01.n0, L.s01.n1};
    A.s02 = Stream{L.s02.k0, L.s02.k1, L.s02.n0, L.s02.n1};
    return A;
}

template <typename T, int N, typename F, bool NT>
hipError_t launch_send(const SplitLaunch& L, SplitKArgs A, const F& f, hipStream_t st) {
    return by_index_range(L.elem_base, L.n, [&](uint64_t begin, uint64_t end) {
        A.begin = begin;
        A.end = end;
        if (L.party == 0)
            hipLaunchKernelGGL((k_send<T, N, F, 0, NT>), dim3(walk_grid(!NT, L.grid)), dim3(256), 0, st, A, f);
        else
            hipLaunchKernelGGL((k_send<T, N, F, 1, NT>), dim3(walk_grid(!NT, L.grid)), dim3(256), 0, st, A, f);
    });
}

template <typename T, int N, typename F, bool NT>
hipError_t launch_reply(const SplitLaunch& L, SplitKArgs A, const F& f, hipStream_t st) {
    return by_index_range(L.elem_base, L.n, [&](uint64_t begin, uint64_t end) {
        A.begin = begin;
        A.end = end;
        hipLaunchKernelGGL((k_reply<T, N, F, NT>), dim3(walk_grid(!NT, L.grid)), dim3(256), 0, st, A, f);
    });
}

template <typename T, int N>
hipError_t launch_split_exact(const SplitLaunch& L, hipStream_t st) {
    constexpr uint64_t bytes = 8 * Packing<N>::W;          // of both messages an element
    const SplitKArgs A = make_split_kargs(L);
    return with_field<N>(L.p, [&](auto f) {
        using F = decltype(f);
        if (L.kind == SplitLaunch::SEND)
            return planes_around_l2(A.out0, L.n, bytes, true) ? launch_send<T, N, F, true>(L, A, f, st)
                                                              : launch_send<T, N, F, false>(L, A, f, st);
        return planes_cached(A.in0, L.n, bytes, true) ? launch_reply<T, N, F, false>(L, A, f, st)
                                                      : launch_reply<T, N, F, true>(L, A, f, st);
    });
}

template <typename T, int NLO, int NHI>
hipError_t launch_split_range(const SplitLaunch& L, hipStream_t st) {
    if constexpr (NLO > NHI) {
        return hipErrorInvalidValue;
    } else {
        if (L.npos == (uint32_t)NLO) return launch_split_exact<T, NLO>(L, st);
        return launch_split_range<T, NLO + 1, NHI>(L, st);
    }
}

}  // namespace bc
