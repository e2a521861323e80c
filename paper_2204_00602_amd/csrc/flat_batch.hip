// HIP kernel (gfx950): a batch of uneven table-driven instances in one launch.
//
// The instances of a training loop are small (hundreds to tens of thousands of
// outputs), so a layer's time is its chain of dependent accesses and, in the
// larger ones, instruction issue.  A workgroup (one per CU, sixteen waves) runs an
// instance from the vacuum to its amplitudes with the layers in its LDS: table
// entries are coalesced loads that depend on nothing, issued a state ahead, and
// the predecessors are LDS reads; one barrier per layer.  Layers too large for
// the LDS go through a scratch pair that stays in the L2.  The last layer of an
// instance that would outlast the rest of the batch is cut into parts: each
// part's workgroup computes the layers below for itself.  Instances too small
// for sixteen waves run on single waves, each in its own part of the LDS,
// without barriers.  The host deals both kinds out largest first to the least
// loaded workgroup or wave, so no workgroup waits for another.  Instances of
// one mode count share its tables (see flat.hip).
//
// 4096 instances of m 6..14, n 2..7 (25.3 M outputs): c64 168 us, c128 319; the
// tiled kernel takes 480 and 677, the outputs alone 43 and 86 at the rate of a
// copy.  16 of m 6..14: c128 58 us against 376, 64 in c64 42 against 282.  What
// bounds it is instruction issue (65 M vector instructions, 106 us on 1024 SIMDs),
// lane moves for 71 spilled scalar registers among them, and, in c128, the blocks of
// layers that no longer fit the LDS (36 vector registers spill there).
// Sixteen waves hide the gathers' latency; eight with twice the registers: 195 us
// instead of 152 for 256 of (14, 7).
#include <algorithm>

#include "flat_dev.h"

namespace {

// Where a layer's predecessors are read from.
enum Source {
    kLds,     // the whole layer in LDS, a zero after its last state
    kBlock,   // states [base, base + size) of it in LDS, a zero after them; a state's only
              // predecessor below base is A[s - shift] (see run_instance)
    kMemory,  // memory
};
template <typename T> struct SourceArgs {
    const typename Cx<T>::type *X;   // in LDS
    const typename Cx<T>::type *A;   // in memory
    uint32_t base, size, shift;
};

// The states first, first + step, .. < end of one layer; `cur` holds the entries
// of the first (of a clamped one where there is none).  put(sum, state) stores.
template <typename T, int CM, Source SRC, typename F>
__device__ __forceinline__ void layer_states(Entries &cur, const uint32_t *__restrict__ pred, uint32_t N, uint32_t cmax,
                                             const SourceArgs<T> &x, uint32_t Nprev, const typename Cx<T>::type *u, int m,
                                             uint32_t first, uint32_t end, uint32_t step, F &&put)
{
    using C = typename Cx<T>::type;
    auto sum = [&](const Entries &en, uint32_t s) {
        if constexpr (SRC == kBlock) {
            Acc<T, SLOS_COMP_NONE> acc;
            acc.zero();
            C below{0, 0};
            if (x.base) below = x.A[s - x.shift];
            auto add = [&](const Entries &ec) {
#pragma unroll
                for (int i = 0; i < CM; ++i) {
                    const uint32_t r = (ec.e[i] & SLOS_PRED_MASK) - x.base;
                    C v = x.X[min(r, x.size)];  // below the base wraps to the zero after the block
                    if ((int32_t)r < 0) v = below;
                    acc.mac(u[ec.e[i] >> 24], v);
                }
            };
            add(en);
            if constexpr (CM == kChunk) {
                for (uint32_t c0 = kChunk; c0 < cmax; c0 += kChunk) {
                    Entries ec;
                    load_chunk(ec, pred, N, cmax, c0, s, SLOS_FLAT_PAD(m, Nprev));
                    add(ec);
                }
            }
            return acc;
        } else {
            return state_sum<T, SLOS_COMP_NONE, CM, SRC == kMemory>(en, pred, N, cmax, s, SRC == kMemory ? x.A : x.X, Nprev,
                                                                    u, m, 0.f);
        }
    };
    for (uint32_t s = first; s < end; s += step) {
        Entries nxt;
        load_entries<CM>(nxt, pred, N, min(s + step, N - 1u));
        put(sum(cur, s), s);
        cur = nxt;
    }
}

// One instance on a workgroup (WAVE = false: tid of SLOS_FB_THREADS, barriers)
// or a wave (tid = lane).  lds: the layers, U's columns at its end.
template <typename T, bool WAVE>
__device__ __forceinline__ void run_instance(const FlatBatchParams &p, uint32_t item, typename Cx<T>::type *lds,
                                             uint32_t elems, typename Cx<T>::type *scr, double *wsum, int tid)
{
    using C = typename Cx<T>::type;
    constexpr int TH = WAVE ? 64 : SLOS_FB_THREADS;
    auto sync = [] {
        if constexpr (WAVE) {
            // a wave's LDS instructions run in order; the fences keep the compiler to it
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
            __syncthreads();
        }
    };
    // a workgroup's item is an instance or one of the parts of its last layer
    const uint32_t ii = WAVE ? item : p.items[item].inst;
    const uint32_t part = WAVE ? 0u : p.items[item].part, parts = WAVE ? 1u : p.items[item].parts;
    const FlatInst &I = p.inst[ii];
    const FlatModes &M = p.modes[I.modes];
    const int m = (int)M.m, n = (int)I.n;
    const C *__restrict__ Um = (const C *)p.U + I.U_off;
    C *out = (C *)p.out + I.out_off;
    double psum = 0.0;
    if (n == 0) {
        // no photons: the single output is the vacuum, amplitude 1
        if (tid == 0) {
            out[0] = C{(T)1, (T)0};
            psum = 1.0;
        }
    } else {
        // U's columns, each followed by the zero that padded entries name
        const int mu = m + 1;
        C *ucol = lds + elems - (uint32_t)(n * mu);
        for (int i = tid; i < n * mu; i += TH) {
            const int j = i % mu;
            C v{0, 0};
            if (j < m) v = Um[(size_t)j * m + I.col[i / mu]];
            ucol[i] = v;
        }
        // layers 0..kl are in LDS: the even ones at ev, the odd ones at od
        const uint32_t room = elems - (uint32_t)(n * mu);
        int kl = 0;
        while (kl + 1 < n && M.N[kl] + M.N[kl + 1] + 2u <= room) ++kl;
        const uint32_t even = kl & 1 ? (kl > 0 ? M.N[kl - 1] : 1u) : M.N[kl];
        C *ev = lds, *od = lds + even + 1u;
        if (tid == 0) {
            ev[0] = C{(T)1, (T)0};
            ev[1] = C{0, 0};
        }
        // states [first, end) of layer k that this workgroup computes
        const uint32_t per = (M.N[n] + parts - 1u) / parts;
        auto first_of = [&](int k) -> uint32_t { return k < n ? 0u : part * per; };
        Entries cur;
        auto fetch_first = [&](int k) {
            const uint32_t N = M.N[k];
            load_chunk(cur, p.pred + M.off[k], N, (uint32_t)min(m, k), 0u, min(first_of(k) + tid, N - 1u), 0u);
        };
        fetch_first(1);
        sync();
        for (int k = 1; k <= n; ++k) {
            const uint32_t N = M.N[k], Nprev = M.N[k - 1], cmax = (uint32_t)min(m, k);
            const uint32_t *pred = p.pred + M.off[k];
            const C *u = ucol + (k - 1) * mu;
            const bool last = k == n;
            const uint32_t s0 = first_of(k) + tid, s1 = last ? min((part + 1u) * per, N) : N;
            const double *scale = p.scale + M.scale_off[k];
            C *Yg = scr + (uint64_t)(k & 1) * p.scratch_stride;  // beyond the LDS
            C *Yl = k & 1 ? od : ev;
            const double nt = I.norm_t;
            // where a sum goes: amplitudes, the next layer in LDS or in memory
            auto amplitude = [&](const Acc<T, SLOS_COMP_NONE> &acc, uint32_t s) {
                psum += store_last<T, SLOS_MODE_AMPL, SLOS_COMP_NONE>(acc, scale[s] * nt, out, s);
            };
            auto to_lds = [&](const Acc<T, SLOS_COMP_NONE> &acc, uint32_t s) { Yl[s] = acc.value(); };
            auto to_memory = [&](const Acc<T, SLOS_COMP_NONE> &acc, uint32_t s) { Yg[s] = acc.value(); };
            if (k - 1 <= kl) {
                const SourceArgs<T> x{k & 1 ? ev : od, nullptr, 0u, 0u, 0u};
                with_terms(cmax, [&](auto t) {
                    constexpr int CM = decltype(t)::value;
                    if (last) layer_states<T, CM, kLds>(cur, pred, N, cmax, x, Nprev, u, m, s0, s1, TH, amplitude);
                    else if (WAVE || k <= kl) layer_states<T, CM, kLds>(cur, pred, N, cmax, x, Nprev, u, m, s0, s1, TH, to_lds);
                    else layer_states<T, CM, kLds>(cur, pred, N, cmax, x, Nprev, u, m, s0, s1, TH, to_memory);
                });
            } else if constexpr (!WAVE) {
                // A_{k-1} is in memory.  In colex order the outputs with top photon
                // d come one d after the other; without that photon output s of
                // them is state s - (their first), and without another photon it
                // is a state whose top photon is d: a contiguous block.  So the
                // blocks go through LDS one after the other (the first d's
                // together, as a prefix), each element once.
                const C *A = scr + (uint64_t)((k - 1) & 1) * p.scratch_stride;
                auto Bn = [&](int a, int c) -> uint32_t { return a < c ? 0u : (uint32_t)p.binom[(size_t)a * p.bstride + c]; };
                int d = -1;  // top photons 0..d are the prefix
                while (d + 1 < m && Bn(d + 1 + k - 1, k - 1) + 1u <= room) ++d;
                for (int first_d = -1; d < m;) {
                    const uint32_t base = first_d < 0 ? 0u : Bn(d + k - 2, k - 1), end = Bn(d + k - 1, k - 1);
                    const uint32_t out0 = first_d < 0 ? 0u : Bn(d + k - 1, k), out1 = Bn(d + k, k);
                    const bool fits = end - base + 1u <= room;
                    const uint32_t lo = max(out0, last ? part * per : 0u), hi = min(out1, s1);
                    if (lo < hi) {
                        const SourceArgs<T> x{lds, A, base, end - base, out0};
                        if (fits) {
                            const uint32_t size = end - base;
                            for (uint32_t i0 = tid; i0 < size; i0 += 8u * TH) {  // eight loads in flight
                                C v[8];
#pragma unroll
                                for (int i = 0; i < 8; ++i) v[i] = A[base + min(i0 + (uint32_t)(i * TH), size - 1u)];
#pragma unroll
                                for (int i = 0; i < 8; ++i)
                                    if (i0 + (uint32_t)(i * TH) < size) lds[i0 + (uint32_t)(i * TH)] = v[i];
                            }
                            if (tid == 0) lds[end - base] = C{0, 0};
                        }
                        const uint32_t f = lo + tid;
                        load_chunk(cur, pred, N, cmax, 0u, min(f, N - 1u), 0u);
                        sync();
                        with_terms(cmax, [&](auto t) {
                            constexpr int CM = decltype(t)::value;
                            auto states = [&](auto &&put) {
                                if (end == Nprev && base == 0u)
                                    layer_states<T, CM, kLds>(cur, pred, N, cmax, x, Nprev, u, m, f, hi, TH, put);
                                else if (fits) layer_states<T, CM, kBlock>(cur, pred, N, cmax, x, Nprev, u, m, f, hi, TH, put);
                                else layer_states<T, CM, kMemory>(cur, pred, N, cmax, x, Nprev, u, m, f, hi, TH, put);
                            };
                            if (last) states(amplitude);
                            else states(to_memory);
                        });
                        sync();  // the block is free
                    }
                    first_d = 0;
                    ++d;
                }
            }
            if (!last) {
                if (k <= kl && tid == 0) Yl[N] = C{0, 0};
                fetch_first(k + 1);
            }
            sync();  // layer k is complete; after the last one the LDS is free
        }
    }
    // sum P: over the wave, then over the waves in order
    psum = wave_sum(psum);
    if constexpr (WAVE) {
        if (tid == 0 && p.sum_p) p.sum_p[ii] = psum;
    } else {
        if ((tid & 63) == 0) wsum[tid >> 6] = psum;
        __syncthreads();
        if (tid == 0 && p.sum_p) {
            for (int w = 1; w < SLOS_FB_WAVES; ++w) psum += wsum[w];
            if (parts == 1) {
                p.sum_p[ii] = psum;
            } else {
                // The part that ends last adds the parts' sums in order (the
                // partials and the count as in finish_sum of flat.hip).
                const FlatItem &it = p.items[item];
                double *partials = p.partials + it.slot;
                uint32_t *count = p.counts + it.count;
                __hip_atomic_store(&partials[part], psum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_s_waitcnt(0);
                if (__hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 1u) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                    double s = 0.0;
                    for (uint32_t q = 0; q < parts; ++q)
                        s += __hip_atomic_load(&partials[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    p.sum_p[ii] = s;
                    __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
    }
}

template <typename T>
__global__ __launch_bounds__(SLOS_FB_THREADS) void flat_batch_kernel(FlatBatchParams p)
{
    using C = typename Cx<T>::type;
    extern __shared__ __align__(16) unsigned char dyn[];
    __shared__ double wsum[2][SLOS_FB_WAVES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    C *scr = (C *)p.scratch + (uint64_t)p.wg_scr[blockIdx.x] * 2u * p.scratch_stride;
    const uint32_t e1 = p.wg_start[blockIdx.x + 1];
    for (uint32_t e = p.wg_start[blockIdx.x]; e < e1; ++e)
        run_instance<T, false>(p, p.wg_list[e], (C *)dyn, p.lds_elems, scr, wsum[e & 1], tid);
    __syncthreads();
    const uint32_t slot = blockIdx.x * (uint32_t)SLOS_FB_WAVES + (uint32_t)wv;
    const uint32_t v1 = p.wv_start[slot + 1];
    for (uint32_t e = p.wv_start[slot]; e < v1; ++e)
        run_instance<T, true>(p, p.wv_list[e], (C *)dyn + (uint32_t)wv * p.wave_elems, p.wave_elems, nullptr, nullptr, lane);
}

template <typename T>
hipError_t launch(const FlatBatchParams &p, int grid, hipStream_t s)
{
    static bool attr_set = false;  // per instantiation; first call per process
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)flat_batch_kernel<T>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)SLOS_LDS_DYNAMIC_MAX);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const size_t lds = (size_t)std::max(p.lds_elems, p.wave_elems * SLOS_FB_WAVES) * sizeof(typename Cx<T>::type);
    hipLaunchKernelGGL(flat_batch_kernel<T>, dim3(grid), dim3(SLOS_FB_THREADS), lds, s, p);
    return hipGetLastError();
}

} // namespace

int slos_launch_flat_batch(const FlatBatchParams &p, int c64, int grid, void *stream)
{
    return (int)(c64 ? launch<float>(p, grid, (hipStream_t)stream) : launch<double>(p, grid, (hipStream_t)stream));
}
