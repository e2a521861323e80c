// Device code shared by the table-driven kernels (flat.hip, flat_batch.hip).
#pragma once

#include "accum.h"
#include "flat.h"

namespace {

constexpr int kChunk = 8;  // table entries of a state in flight together

struct Entries {
    uint32_t e[kChunk];
};

// The first CM entries (CM <= kChunk) of state s, which is in bounds.
template <int CM>
__device__ __forceinline__ void load_entries(Entries &r, const uint32_t *__restrict__ pred, uint32_t N, uint32_t s)
{
#pragma unroll
    for (int i = 0; i < CM; ++i) r.e[i] = (pred + (size_t)i * N)[s];
}

// Entries c0 .. c0 + kChunk - 1 of state s, those from cmax on padded.
__device__ __forceinline__ void load_chunk(Entries &r, const uint32_t *__restrict__ pred, uint32_t N, uint32_t cmax,
                                           uint32_t c0, uint32_t s, uint32_t pad)
{
#pragma unroll
    for (int i = 0; i < kChunk; ++i) {
        r.e[i] = pad;
        if (c0 + i < cmax) r.e[i] = (pred + (size_t)(c0 + i) * N)[s];
    }
}

// acc += the first CM terms; all loads are issued before the sums.  X holds
// layer k - 1: in LDS with a zero after its last state, which padded entries
// name (GLOBAL = false), or in memory, where they are taken as zero here.
// Padded entries name mode m, whose coefficient is zero.
template <typename T, int COMP, int CM, bool GLOBAL>
__device__ __forceinline__ void add_terms(Acc<T, COMP> &acc, const Entries &en, const typename Cx<T>::type *X,
                                          uint32_t Nprev, const typename Cx<T>::type *u)
{
    using C = typename Cx<T>::type;
    C v[CM], uj[CM];
    // byte offset of a rank: one 24-bit multiply, which ignores the mode byte
    // (the size is hidden from the optimiser, which would make it a mask and a shift)
    uint32_t esz = (uint32_t)sizeof(C);
    if (!GLOBAL) asm volatile("" : "+v"(esz));
#pragma unroll
    for (int i = 0; i < CM; ++i) {
        if (GLOBAL) v[i] = X[min(en.e[i] & SLOS_PRED_MASK, Nprev - 1u)];
        else v[i] = *(const C *)((const char *)X + __umul24(en.e[i], esz));
        uj[i] = u[en.e[i] >> 24];
    }
#pragma unroll
    for (int i = 0; i < CM; ++i) {
        if (GLOBAL && (en.e[i] & SLOS_PRED_MASK) >= Nprev) v[i] = C{0, 0};
        acc.mac(uj[i], v[i]);
    }
}

// acc += the terms past the first kChunk of state s (more than kChunk occupied modes)
template <typename T, int COMP, bool GLOBAL>
__device__ __forceinline__ void add_chunks(Acc<T, COMP> &acc, const uint32_t *__restrict__ pred, uint32_t N, uint32_t cmax,
                                           uint32_t s, const typename Cx<T>::type *X, uint32_t Nprev,
                                           const typename Cx<T>::type *u, int m)
{
    for (uint32_t c0 = kChunk; c0 < cmax; c0 += kChunk) {
        Entries en;
        load_chunk(en, pred, N, cmax, c0, s, SLOS_FLAT_PAD(m, Nprev));
        add_terms<T, COMP, kChunk, GLOBAL>(acc, en, X, Nprev, u);
    }
}

// The sum of state s; CM = min(cmax, kChunk), its first CM entries loaded.
template <typename T, int COMP, int CM, bool GLOBAL>
__device__ __forceinline__ Acc<T, COMP> state_sum(const Entries &first, const uint32_t *__restrict__ pred, uint32_t N,
                                                  uint32_t cmax, uint32_t s, const typename Cx<T>::type *X,
                                                  uint32_t Nprev, const typename Cx<T>::type *u, int m, float sigma)
{
    Acc<T, COMP> acc;
    acc.zero();
    acc.start(sigma);
    add_terms<T, COMP, CM, GLOBAL>(acc, first, X, Nprev, u);
    if constexpr (CM == kChunk) add_chunks<T, COMP, GLOBAL>(acc, pred, N, cmax, s, X, Nprev, u, m);
    return acc;
}

// f(CM as an integral constant), CM = min(cmax, kChunk)
template <int CM> struct Terms {
    static constexpr int value = CM;
};
template <typename F>
__device__ __forceinline__ void with_terms(uint32_t cmax, F &&f)
{
    switch (cmax) {
    case 1: f(Terms<1>{}); break;
    case 2: f(Terms<2>{}); break;
    case 3: f(Terms<3>{}); break;
    case 4: f(Terms<4>{}); break;
    case 5: f(Terms<5>{}); break;
    case 6: f(Terms<6>{}); break;
    case 7: f(Terms<7>{}); break;
    default: f(Terms<kChunk>{}); break;
    }
}

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Store one output of the pass's layer: A_k as it is, or (last layer) a(S) or
// P(S) with the FP64 normalisation f; returns P(S) for the sum.  Nothing in the
// launch reads it again: past the L2, it leaves that to the tables (a c64 batch of
// 4096 with 200 MB of outputs: 218 us through the L2, 168 past it).
template <typename T, int MODE, int COMP>
__device__ __forceinline__ double store_last(const Acc<T, COMP> &acc, double f, void *Y, uint32_t s)
{
    const double ar = acc.re() * f, ai = acc.im() * f;
    const double pr = prob(ar, ai);
    typedef T V __attribute__((ext_vector_type(2)));
    if (MODE == SLOS_MODE_AMPL) __builtin_nontemporal_store(V{(T)ar, (T)ai}, (V *)Y + s);
    else __builtin_nontemporal_store((T)pr, (T *)Y + s);
    return pr;
}

} // namespace
