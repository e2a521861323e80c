// HIP kernels (gfx950): amplitudes of selected outputs only.
//
// The layer recurrence of Section 3.2.3 restricted to one target S: only the
// states t <= S (componentwise) can reach S, so for each target the kernel runs
//     A[0] = 1,  A[t] = sum_{j : t_j > 0} U[j, i_|t|] A[t - e_j]
// over that sub-lattice and returns a(S) = A[S] sqrt(prod s_j!) / sqrt(prod t_i!)
// (Eq. eqperm).  The sub-lattice has R = prod_j (s_j + 1) states, 2^n for an
// output without bunching, instead of the C(m+n-1, n) states of the full
// distribution: the way to a few outputs of a space too large to enumerate.
//
// States are numbered in mixed radix over the occupied modes of S (digit q =
// occupation of the q-th occupied mode, radix s_q + 1), so t - e_j is the index
// minus a stride.  Targets with the same multiset of occupations share one table
// (built on the host): the states listed layer by layer, each with the mask of its
// non-zero digits, read from global memory (it stays in cache).  A target has A,
// and U's columns with the strides, in LDS and fills A layer by layer.  Each state's
// terms are summed in a fixed order (digits ascending), so results are reproducible.
//
// What bounds it is the chain of a state's terms and the wait between layers, with
// most layers smaller than a workgroup.  So a target has one, two, four or eight of
// a workgroup's waves, by the LDS it needs, and every target of the workgroup is at
// the same layer: 10,000 targets of 24 modes and 12 photons (65 M terms) 80 us,
// 50 of them instruction issue; a workgroup of four waves per target, with strides
// and columns read from memory, 187.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "slos_ext.h"

namespace {

template <typename T> struct Cs;
template <> struct Cs<float> { using type = float2; };
template <> struct Cs<double> { using type = double2; };

// One digit's entry of a column: U[mode_q, i_k] and the digit's stride in bytes of A.
template <typename T> struct Entry;
template <> struct alignas(16) Entry<float> { float x, y; uint32_t stride; };
template <> struct alignas(16) Entry<double> { double x, y; uint32_t stride; };
static_assert(sizeof(Entry<float>) == SLOS_SELECT_ENTRY(true) && sizeof(Entry<double>) == SLOS_SELECT_ENTRY(false),
              "the host sizes LDS by these");

template <typename T>
__global__ __launch_bounds__(SLOS_SELECT_THREADS) void select_kernel(SelectParams p)
{
    using C = typename Cs<T>::type;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ Entry<T> one[SLOS_SELECT_MAX_OCC];  // a column at a time, for a target that leaves no room for all
    const C *Um = (const C *)p.U;
    const int m = p.m, n = p.n, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    for (int64_t bi = blockIdx.x; bi < p.blocks[SLOS_SELECT_CLASSES]; bi += gridDim.x) {
        int j = 0;
        while (bi >= p.blocks[j + 1]) ++j;
        const int c = SLOS_SELECT_CLASSES - 1 - j;      // 2^c waves to a target
        const int group = wv >> c, per = SLOS_SELECT_THREADS / 64 >> c;
        const int tid = threadIdx.x & ((64 << c) - 1), nt = 64 << c;
        const int64_t ti = p.start[j] + (bi - p.blocks[j]) * per + group;
        const bool live = ti < p.start[j + 1];          // the last workgroup of a class can have idle waves
        auto sync = [&] {
            if (c == 0) {
                // a wave's LDS instructions run in order; the fences keep the compiler to it
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            } else {
                __syncthreads();
            }
        };
        // A lane holds an entry of the target's and the pattern's arrays: a layer's
        // bounds and a column's rows are then lane reads, not loads that depend on loads.
        const uint64_t item = p.order[live ? ti : p.start[j]];
        const int64_t target = (int64_t)(item >> SLOS_SELECT_PATTERN_BITS);
        const int lane = threadIdx.x & 63;
        const int my_row = lane < n ? (int)p.rows[target * n + lane] * m : 0;
        const SelectPattern &pt = p.patterns[item & ((1u << SLOS_SELECT_PATTERN_BITS) - 1u)];
        const int nocc = (int)pt.nocc;
        const uint32_t my_stride = pt.stride[lane & 31] * (uint32_t)sizeof(C), my_start = pt.lstart[min(lane, n + 1)];
        const uint32_t R = pt.R;
        const uint16_t *__restrict__ state = p.state + pt.off;
        const uint32_t *__restrict__ mask = p.mask + pt.off;
        auto lstart = [&](int k) { return (uint32_t)__builtin_amdgcn_readlane((int)my_start, k); };
        unsigned char *mine = lds + (size_t)group * (p.lds / per);
        const bool all = (uint64_t)R * sizeof(C) + (uint64_t)n * nocc * sizeof(Entry<T>) <= p.lds / per;
        Entry<T> *cols = all ? (Entry<T> *)mine : one;
        C *A = (C *)(all ? mine + (size_t)n * nocc * sizeof(Entry<T>) : mine);
        auto fill = [&](Entry<T> *to, int k, int row, uint32_t stride) {  // column k (0..) of a digit
            const C u = Um[(size_t)row + p.cols[k]];
            to->x = u.x;
            to->y = u.y;
            to->stride = stride;
        };
        if (all) {
            const int sh = nocc <= 16 ? 4 : 5, q = tid & ((1 << sh) - 1);  // sixteen or 32 lanes to a column
            const int row = __shfl(my_row, q, 64);
            const uint32_t stride = __shfl(my_stride, q, 64);
            if (q < nocc)
                for (int k = tid >> sh; k < n; k += nt >> sh) fill(cols + k * nocc + q, k, row, stride);
        }
        if (tid == 0) A[0] = C{(T)1, (T)0};
        // the next layer's first state of this thread, loaded before the wait
        uint32_t x = 0, mk = 0;
        auto fetch = [&](uint32_t i, uint32_t end) {
            if (i < end) {
                x = state[i];
                mk = mask[i];
            }
        };
        fetch(lstart(1) + tid, n > 0 ? lstart(2) : 0u);
        for (int k = 1; k <= n; ++k) {
            sync();  // layer k - 1 complete
            const Entry<T> *uk = one;
            if (all) {
                uk = cols + (k - 1) * nocc;
            } else {
                if (tid < nocc) fill(one + tid, k - 1, my_row, my_stride);
                sync();
            }
            const uint32_t end = live ? lstart(k + 1) : 0u;
            for (uint32_t i = lstart(k) + tid; i < end; i += nt) {
                const uint32_t xs = x, ms = mk;
                fetch(i + nt, end);
                T ar = 0, ai = 0;
                uint32_t w = ms;
                auto terms = [&](auto count) {  // the next non-zero digits, ascending, their reads in flight together
                    constexpr int N = decltype(count)::value;
                    Entry<T> u[N];
                    C v[N];
#pragma unroll
                    for (int e = 0; e < N; ++e) {
                        u[e] = uk[__builtin_ctz(w)];
                        w &= w - 1u;
                    }
#pragma unroll
                    for (int e = 0; e < N; ++e) v[e] = *(const C *)((const char *)A + (xs * (uint32_t)sizeof(C) - u[e].stride));
#pragma unroll
                    for (int e = 0; e < N; ++e) {
                        ar = fma(u[e].x, v[e].x, ar);
                        ar = fma(-u[e].y, v[e].y, ar);
                        ai = fma(u[e].x, v[e].y, ai);
                        ai = fma(u[e].y, v[e].x, ai);
                    }
                };
                const int d = __builtin_popcount(ms);
                if (d & 1) terms(std::integral_constant<int, 1>{});
                if (d & 2) terms(std::integral_constant<int, 2>{});
                while (w) terms(std::integral_constant<int, 4>{});
                A[xs] = C{ar, ai};
            }
            if (k < n) fetch(lstart(k + 1) + tid, lstart(k + 2));
        }
        sync();
        if (tid == 0 && live) {
            const C a = A[R - 1];
            ((C *)p.out)[target] = C{(T)((double)a.x * pt.fac), (T)((double)a.y * pt.fac)};
        }
        __syncthreads();  // the LDS is reused by the next turn
    }
}

} // namespace

int slos_launch_select(const SelectParams &p, int c64, void *stream)
{
    const int grid = (int)std::min<int64_t>(p.blocks[SLOS_SELECT_CLASSES], 1 << 20);
    hipStream_t s = (hipStream_t)stream;
    const void *f = c64 ? (const void *)select_kernel<float> : (const void *)select_kernel<double>;
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SLOS_LDS_DYNAMIC_MAX);
    if (e != hipSuccess) return (int)e;
    if (c64)
        hipLaunchKernelGGL(select_kernel<float>, dim3(grid), dim3(SLOS_SELECT_THREADS), p.lds, s, p);
    else
        hipLaunchKernelGGL(select_kernel<double>, dim3(grid), dim3(SLOS_SELECT_THREADS), p.lds, s, p);
    return (int)hipGetLastError();
}
