// HIP kernels (gfx950) of the small layers: the recurrence
//     A_k[t] = sum_{j : t_j > 0} U[j, i_k] * A_{k-1}[t - e_j]
// (arXiv 2204.00602, Section 3.2.3) driven by a table of predecessor ranks.
//
// A layer of up to a million states is far too small to be bound by memory: its
// time is the launch and the chain of dependent loads of one work unit.  The
// tiled kernel (layer.hip) has a long chain (ticket, descriptor, staged block,
// inner table, sum), which pays for itself only on layers that stream from HBM.
// Here a thread owns one output: its table entries are one coalesced load each,
// all in flight together, then its predecessors, then the sum.
//   head_kernel   layers 1..h+1 in one launch: every workgroup computes layers
//                 1..h whole in its own LDS, and its own share of layer h+1
//   flat_kernel   one further layer per launch
// Tables are built on the device when the plan is made (table_kernel): entry c
// of state s of layer k is (mode << 24) | rank of the state without one photon
// of that mode, in the tiled kernel's order of summation, stored term-major (pred[c * N_k + s]) and
// padded with entries that stand for a zero coefficient and a zero state.
#include <algorithm>

#include "flat_dev.h"

namespace {

// The sum of the workgroups' FP64 partials, formed by the workgroup that ends
// last: each publishes its partial and counts itself in, and the one that finds
// itself the last adds all of them in a fixed order, so the sum does not depend
// on which that was.  *count is zero before the launch and again after it.
// `mine` is valid in thread 0.  Saves the launch of a separate reduction (m=12,
// n=6: 10.7 against 12.0 us a pass); with thousands of workgroups the counter
// would be the bottleneck (2,873 of them: 92 us against 13 + 6 for the
// reduction), so only the first launch, of at most 512, ends this way.
//
// Only the partials cross between workgroups.  They are written and read with
// agent-scope atomic accesses, which go through to the memory that all XCDs
// share, and the wait between the store and the count makes the one complete
// before the other is issued.  (A release at agent scope would also write back
// every line of outputs in the XCD's L2: 2 to 3 us more at 64 instances.)
__device__ __forceinline__ void finish_sum(double mine, double *partials, uint32_t *count, double *sum_p)
{
    __shared__ double ws[16];
    __shared__ bool last;
    const uint32_t n = gridDim.x;
    if (threadIdx.x == 0) {
        __hip_atomic_store(&partials[blockIdx.x], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);  // the partial is where every XCD reads it
        last = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1u;
    }
    __syncthreads();
    if (!last) return;  // the same for the whole workgroup
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    double s = 0.0;
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x)
        s += __hip_atomic_load(&partials[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) s += ws[w];
        *sum_p = s;
        __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Layers 1..h+1 of an instance (blockIdx.y), one launch.  Every workgroup
// computes layers 1..h for itself: the two LDS buffers hold layer k-1 and layer
// k, a barrier separates layers, and nothing is exchanged between workgroups;
// then each takes its share of layer h+1.  The repeated work costs less than
// the launches it saves: at m=12, n=6 the whole pass of one instance (layers of
// 12 to 12,376 states and the sum of P) is this one launch, 10.9 us against
// 36.1 for nine tiled launches (c64); m=6, n=3 takes 8.4 against 22.6, the
// host's share of a call.  Bound by instruction issue and LDS reads of the
// repeated layers.  The entries of a thread's next state are loaded before the
// current one is summed, and those of the next layer before the barrier, and
// the number of terms is a constant of the inner loop: with a test per term
// instead, each term's LDS read waited for the one before (18.8 us).
template <typename T, int MODE, int COMP>
__global__ __launch_bounds__(1024) void head_kernel(HeadParams p)
{
    using C = typename Cx<T>::type;
    extern __shared__ __align__(16) unsigned char dyn[];
    __shared__ float l1s[SLOS_MAX_PHOTONS + 1];       // sum_j |Re U[j, i_k]| + |Im U[j, i_k]|
    __shared__ uint32_t vmx[SLOS_MAX_PHOTONS + 1];    // max |Re| + |Im| over layer k, float bits
    __shared__ double wsum[16];
    const int tid = threadIdx.x, TH = blockDim.x, lane = tid & 63, wv = tid >> 6, W = TH >> 6;
    const int m = p.m, h = p.h;
    C *buf0 = (C *)dyn, *buf1 = buf0 + p.cap[0], *ucol = buf1 + p.cap[1];
    const uint64_t b = blockIdx.y;
    const C *__restrict__ Um = (const C *)((const char *)p.U + b * p.u_stride);

    // columns of U, each followed by the zero that padded entries name
    for (int i = tid; i < (h + 1) * (m + 1); i += TH) {
        const int j = i % (m + 1);
        C v{0, 0};
        if (j < m) v = Um[(size_t)j * m + p.col[i / (m + 1) + 1]];
        ucol[i] = v;
    }
    if (tid == 0) {
        buf0[0] = C{(T)1, (T)0};
        buf0[1] = C{0, 0};
    }
    if (tid <= SLOS_MAX_PHOTONS) vmx[tid] = tid == 0 ? __float_as_uint(1.0f) : 0u;
    for (uint32_t i = blockIdx.x * (uint32_t)TH + tid; i < p.nzero; i += gridDim.x * (uint32_t)TH)
        p.zero[b * p.zero_stride + i] = 0u;

    // first state of this thread in layer k, and its entries (clamped: in bounds)
    auto first = [&](int k) -> uint32_t { return k <= h ? (uint32_t)tid : blockIdx.x * (uint32_t)TH + tid; };
    Entries cur;
    auto fetch_first = [&](int k) {
        const uint32_t N = p.N[k];
        load_chunk(cur, p.pred + p.off[k], N, (uint32_t)min(m, k), 0u, min(first(k), N - 1u), 0u);
    };
    fetch_first(1);
    __syncthreads();
    if constexpr (COMP == SLOS_COMP_BIASED) {
        for (int k = 1 + wv; k <= h + 1; k += W) {
            float l1 = 0.f;
            for (int j = lane; j < m; j += 64) {
                const C u = ucol[(k - 1) * (m + 1) + j];
                l1 += (float)(fabs(u.x) + fabs(u.y));
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) l1 += __shfl_xor(l1, o, 64);
            if (lane == 0) l1s[k] = l1;
        }
        __syncthreads();
    }
    auto sigma_of = [&](int k) -> float {
        if constexpr (COMP == SLOS_COMP_BIASED) return bias_for(l1s[k] * __uint_as_float(vmx[k - 1]) * 1.001f);
        return 0.f;
    };

    C *keep = (C *)p.keep;
    for (int k = 1; k <= h; ++k) {
        const C *X = k & 1 ? buf0 : buf1;
        C *Yl = k & 1 ? buf1 : buf0;
        const C *u = ucol + (k - 1) * (m + 1);
        const uint32_t N = p.N[k], Nprev = p.N[k - 1], cmax = (uint32_t)min(m, k);
        const uint32_t *pred = p.pred + p.off[k];
        C *kept = keep && blockIdx.x == 0 ? (C *)((char *)keep + b * p.keep_stride + p.keep_off[k]) : nullptr;
        const float sigma = sigma_of(k);
        float omax = 0.f;
        auto layer = [&](auto comp, auto terms) {
            constexpr int CP = decltype(comp)::value, CM = decltype(terms)::value;
            for (uint32_t s = tid; s < N; s += TH) {
                Entries nxt;
                load_entries<CM>(nxt, pred, N, min(s + TH, N - 1u));
                const C a = state_sum<T, CP, CM, false>(cur, pred, N, cmax, s, X, Nprev, u, m, sigma).value();
                Yl[s] = a;
                if (kept) kept[s] = a;
                if (COMP == SLOS_COMP_BIASED) omax = fmaxf(omax, (float)(fabs(a.x) + fabs(a.y)));
                cur = nxt;
            }
        };
        if (COMP != SLOS_COMP_NONE && k >= p.comp_from) with_terms(cmax, [&](auto t) { layer(Terms<COMP>{}, t); });
        else with_terms(cmax, [&](auto t) { layer(Terms<SLOS_COMP_NONE>{}, t); });
        if (tid == 0) Yl[N] = C{0, 0};
        fetch_first(k + 1);
        if constexpr (COMP == SLOS_COMP_BIASED) {
            omax = wave_max(omax);  // every lane of a wave is here
            if (lane == 0) atomicMax(&vmx[k], __float_as_uint(omax));
        }
        __syncthreads();
    }

    // this workgroup's share of layer h + 1
    const int k = h + 1;
    const C *X = k & 1 ? buf0 : buf1;
    const C *u = ucol + h * (m + 1);
    const uint32_t N = p.N[k], Nprev = p.N[h], cmax = (uint32_t)min(m, k), step = gridDim.x * (uint32_t)TH;
    const uint32_t *pred = p.pred + p.off[k];
    void *Y = (char *)p.Y + b * p.y_stride;
    const float sigma = sigma_of(k);
    float omax = 0.f;
    double psum = 0.0;
    auto share = [&](auto comp, auto terms) {
        constexpr int CP = decltype(comp)::value, CM = decltype(terms)::value;
        for (uint32_t s = first(k); s < N; s += step) {
            Entries nxt;
            load_entries<CM>(nxt, pred, N, min(s + step, N - 1u));
            const double f = MODE == SLOS_MODE_MID ? 1.0 : p.scale[s];
            const Acc<T, CP> acc = state_sum<T, CP, CM, false>(cur, pred, N, cmax, s, X, Nprev, u, m, sigma);
            if (MODE == SLOS_MODE_MID) {
                const C a = acc.value();
                ((C *)Y)[s] = a;
                omax = fmaxf(omax, (float)(fabs(a.x) + fabs(a.y)));
            } else {
                psum += store_last<T, MODE, CP>(acc, f, Y, s);
            }
            cur = nxt;
        }
    };
    if (COMP != SLOS_COMP_NONE && k >= p.comp_from) with_terms(cmax, [&](auto t) { share(Terms<COMP>{}, t); });
    else with_terms(cmax, [&](auto t) { share(Terms<SLOS_COMP_NONE>{}, t); });
    if (MODE == SLOS_MODE_MID) {
        if (p.vm) {
            omax = wave_max(omax);
            if (lane == 0) wsum[wv] = (double)omax;
            __syncthreads();
            if (tid == 0) {
                for (int w = 1; w < W; ++w) omax = fmaxf(omax, (float)wsum[w]);
                p.vm[b * p.vm_stride + blockIdx.x] = omax;
            }
        }
    } else {
        // one FP64 partial per workgroup: over lanes, then over waves in order
        psum = wave_sum(psum);
        if (lane == 0) wsum[wv] = psum;
        __syncthreads();
        if (tid == 0)
            for (int w = 1; w < W; ++w) psum += wsum[w];
        if (p.count) {
            finish_sum(psum, p.partials + b * p.partials_stride, p.count + b * p.count_stride, p.sum_p + b);
        } else if (tid == 0) {
            if (gridDim.x > 1) p.partials[b * p.partials_stride + blockIdx.x] = psum;
            else if (p.sum_p) p.sum_p[b] = psum;
        }
    }
}

// One layer, one output per thread, U's column in LDS.  Two dependent memory
// reads per output and no barrier after the first; bound by that latency up to
// a few hundred thousand states, then by the table's bytes (4 per term, from
// the L2 or the memory-side cache) and the predecessors' lines.  735,471 states
// take 12.6 us (c64) where the tiled layer took 27.8.
template <typename T, int MODE, int COMP, int CM>
__global__ __launch_bounds__(SLOS_FLAT_THREADS) void flat_kernel(FlatParams p)
{
    using C = typename Cx<T>::type;
    constexpr int kWaves = SLOS_FLAT_THREADS / 64;
    __shared__ C u[256];
    __shared__ float wl1[kWaves], wvm[kWaves];
    __shared__ double wsum[kWaves];
    const uint64_t b = blockIdx.y;
    const C *__restrict__ X = (const C *)((const char *)p.X + b * p.x_stride);
    const C *__restrict__ Um = (const C *)((const char *)p.U + b * p.u_stride);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const uint32_t s = blockIdx.x * (uint32_t)SLOS_FLAT_THREADS + tid;
    const uint32_t sc = min(s, p.N - 1u);
    Entries en;
    load_entries<CM>(en, p.pred, p.N, sc);
    double f = 1.0;
    if (MODE != SLOS_MODE_MID) f = p.scale[sc];
    C uj{0, 0};
    if (tid < p.m) uj = Um[(size_t)tid * p.m + p.col];
    u[tid] = uj;
    if constexpr (COMP == SLOS_COMP_BIASED) {
        float l1 = (float)(fabs(uj.x) + fabs(uj.y));
        float vm = p.vmax_in ? 0.f : 1.f;
        if (p.vmax_in)
            for (uint32_t i = tid; i < p.nvmax; i += SLOS_FLAT_THREADS)
                vm = fmaxf(vm, __uint_as_float(p.vmax_in[b * p.vin_stride + i]));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) l1 += __shfl_xor(l1, o, 64);
        vm = wave_max(vm);
        if (lane == 0) {
            wl1[wv] = l1;
            wvm[wv] = vm;
        }
    }
    __syncthreads();
    float sigma = 0.f;
    if constexpr (COMP == SLOS_COMP_BIASED) {
        float l1 = wl1[0], vm = wvm[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
            l1 += wl1[w];
            vm = fmaxf(vm, wvm[w]);
        }
        sigma = bias_for(l1 * vm * 1.001f);
    }
    const Acc<T, COMP> acc = state_sum<T, COMP, CM, true>(en, p.pred, p.N, p.cmax, sc, X, p.Nprev, u, p.m, sigma);
    void *Y = (char *)p.Y + b * p.y_stride;
    if (MODE == SLOS_MODE_MID) {
        const C a = acc.value();
        if (s < p.N) ((C *)Y)[s] = a;
        if (p.vmax_out) {
            float omax = s < p.N ? (float)(fabs(a.x) + fabs(a.y)) : 0.f;
            omax = wave_max(omax);
            __syncthreads();
            if (lane == 0) wvm[wv] = omax;
            __syncthreads();
            if (tid == 0) {
#pragma unroll
                for (int w = 1; w < kWaves; ++w) omax = fmaxf(omax, wvm[w]);
                // spread over slots: thousands of workgroups on one would queue up
                atomicMax(p.vmax_out + b * p.vout_stride + blockIdx.x % SLOS_FLAT_VMAX, __float_as_uint(omax));
            }
        }
    } else {
        double pr = 0.0;
        if (s < p.N) pr = store_last<T, MODE, COMP>(acc, f, Y, s);
        pr = wave_sum(pr);
        if (lane == 0) wsum[wv] = pr;
        __syncthreads();
        if (tid == 0) {
#pragma unroll
            for (int w = 1; w < kWaves; ++w) pr += wsum[w];
            p.partials[b * p.partials_stride + blockIdx.x] = pr;
        }
    }
}

// Photon modes d[0] <= .. <= d[k-1] of colex rank s of k photons in m modes
// (rank = sum_r C(d_r + r - 1, r) over positions r = 1..k).
__device__ __forceinline__ void unrank_photons(const FlatTables &p, int k, uint64_t s, uint8_t *d)
{
    int c = p.m + k - 1;  // exclusive upper bound of c_k = d_k + k - 1
    for (int r = k; r >= 1; --r) {
        int cc = c - 1;
        while (cc >= r && p.binom[(size_t)cc * p.bstride + r] > s) --cc;
        if (cc < r) cc = r - 1;
        else s -= p.binom[(size_t)cc * p.bstride + r];
        d[r - 1] = (uint8_t)(cc - r + 1);
        c = cc;
    }
}

// Predecessor (and successor) tables: blockIdx.y < kf is layer blockIdx.y + 1's
// predecessor table (and its normalisation where scale_on asks for it), the others the
// successor tables of layers 1..kb.
__global__ __launch_bounds__(256) void table_kernel(FlatTables p)
{
    const bool succ = (int)blockIdx.y >= p.kf;
    const int k = (succ ? (int)blockIdx.y - p.kf : (int)blockIdx.y) + 1;
    const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    auto B = [&](int a, int b) -> uint64_t { return a < b ? 0 : p.binom[(size_t)a * p.bstride + b]; };
    uint8_t d[SLOS_MAX_PHOTONS + 1];
    if (!succ) {
        const uint32_t N = p.N[k];
        if (s >= N) return;
        unrank_photons(p, k, s, d);
        // the tiled kernel's leaf of this state (plan.cpp, gen_leaves): modes
        // q.. are its high ones.  Its order of summation, high modes descending
        // and then low ones ascending, is kept, so both give the same bits.
        int q = p.m, K = k;
        while (K > 0 && q > 1 && B(q + K - 1, K) > p.leaf_cap[k]) {
            --q;
            while (K > 0 && (int)d[K - 1] == q) --K;
        }
        uint64_t up = 0, here = 0;  // photons above: one position down; below: in place
        for (int r = 2; r <= k; ++r) up += B(d[r - 1] + r - 2, r - 1);
        int nh = 0;                 // occupied high modes
        for (int r = K + 1; r <= k; ++r) nh += r == k || d[r] != d[r - 1];
        uint32_t *out = p.pred + p.off[k] + s;
        const int cmax = min(p.m, k);
        int hi = nh, lo = nh;
        for (int r = 1; r <= k; ++r) {
            // the last photon of each mode is the one taken away
            if (r == k || d[r] != d[r - 1]) {
                const int c = r > K ? --hi : lo++;
                out[(size_t)c * N] = (uint32_t)d[r - 1] << 24 | (uint32_t)(here + up);
            }
            here += B(d[r - 1] + r - 1, r);
            if (r < k) up -= B(d[r] + r - 1, r);
        }
        for (int c = lo; c < cmax; ++c) out[(size_t)c * N] = SLOS_FLAT_PAD(p.m, p.N[k - 1]);
        if (p.scale_on >> k & 1u) {
            // sqrt(prod s_j!) / sqrt(prod t_i!), in the tiled kernel's two factors
            double fh = 1.0, fl = 1.0;
            int run = 0;
            for (int r = k; r > K; --r) {
                run = r < k && d[r - 1] == d[r] ? run + 1 : 1;
                fh *= (double)run;
            }
            for (int r = 1; r <= K; ++r) {
                run = r > 1 && d[r - 1] == d[r - 2] ? run + 1 : 1;
                fl *= (double)run;
            }
            p.scale[p.scale_off[k] + s] = (sqrt(fh) * p.norm_t) * sqrt(fl);
        }
        return;
    }
    const uint32_t N = p.N[k - 1], row = slos_succ_row(N, k <= p.kt);
    if (s >= row) return;
    uint32_t *out = p.succ + p.succ_off[k] + s;
    if (k <= p.kt) out[(size_t)p.m * row] = p.N[k];
    if (s == N) {
        for (int j = 0; j < p.m; ++j) out[(size_t)j * row] = p.N[k];
        return;
    }
    unrank_photons(p, k - 1, s, d);
    uint64_t here = 0, up = 0;  // photons above the new one: one position up
    for (int r = 1; r < k; ++r) up += B(d[r - 1] + r, r + 1);
    int q = 0;                  // photons in modes <= j
    for (int j = 0; j < p.m; ++j) {
        while (q < k - 1 && d[q] <= j) {
            here += B(d[q] + q, q + 1);
            up -= B(d[q] + q + 1, q + 2);
            ++q;
        }
        out[(size_t)j * row] = (uint32_t)(here + B(j + q, q + 1) + up);
    }
}

template <typename T, int MODE, int COMP>
hipError_t launch_head(const FlatLaunch &l, hipStream_t s)
{
    static bool attr_set = false;  // per instantiation; first call per process
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)head_kernel<T, MODE, COMP>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)SLOS_LDS_DYNAMIC_MAX);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const HeadParams &p = *l.head;
    const size_t lds = ((size_t)p.cap[0] + p.cap[1] + (size_t)(p.h + 1) * (p.m + 1)) * sizeof(typename Cx<T>::type);
    hipLaunchKernelGGL((head_kernel<T, MODE, COMP>), dim3(l.grid, l.batch), dim3(l.threads), lds, s, p);
    return hipGetLastError();
}

template <typename T, int MODE, int COMP, int CM>
hipError_t launch_cm(const FlatLaunch &l, hipStream_t s)
{
    hipLaunchKernelGGL((flat_kernel<T, MODE, COMP, CM>),
                       dim3((l.flat->N + SLOS_FLAT_THREADS - 1) / SLOS_FLAT_THREADS, l.batch), dim3(SLOS_FLAT_THREADS), 0,
                       s, *l.flat);
    return hipGetLastError();
}

template <typename T, int MODE, int COMP>
hipError_t launch_mode(const FlatLaunch &l, hipStream_t s)
{
    if (l.head) return launch_head<T, MODE, COMP>(l, s);
    switch (l.flat->cmax) {
    case 1: return launch_cm<T, MODE, COMP, 1>(l, s);
    case 2: return launch_cm<T, MODE, COMP, 2>(l, s);
    case 3: return launch_cm<T, MODE, COMP, 3>(l, s);
    case 4: return launch_cm<T, MODE, COMP, 4>(l, s);
    case 5: return launch_cm<T, MODE, COMP, 5>(l, s);
    case 6: return launch_cm<T, MODE, COMP, 6>(l, s);
    case 7: return launch_cm<T, MODE, COMP, 7>(l, s);
    default: return launch_cm<T, MODE, COMP, kChunk>(l, s);
    }
}

template <typename T, int COMP>
hipError_t launch_comp(const FlatLaunch &l, hipStream_t s)
{
    switch (l.mode) {
    case SLOS_MODE_AMPL: return launch_mode<T, SLOS_MODE_AMPL, COMP>(l, s);
    case SLOS_MODE_PROB: return launch_mode<T, SLOS_MODE_PROB, COMP>(l, s);
    default: return launch_mode<T, SLOS_MODE_MID, COMP>(l, s);
    }
}

} // namespace

int slos_launch_flat(const FlatLaunch &l, void *stream)
{
    hipStream_t s = (hipStream_t)stream;
    if (l.tables) {
        const FlatTables &t = *l.tables;
        uint32_t most = 1;  // N_k, and one more in a tail layer's successor table
        for (int k = 1; k <= t.kf; ++k) most = std::max(most, t.N[k] + 1u);
        hipLaunchKernelGGL(table_kernel, dim3((most + 255) / 256, t.kf + t.kb), dim3(256), 0, s, t);
        return (int)hipGetLastError();
    }
    if (!l.c64) return (int)launch_comp<double, SLOS_COMP_NONE>(l, s);
    switch (l.compensated) {
    case SLOS_COMP_BIASED: return (int)launch_comp<float, SLOS_COMP_BIASED>(l, s);
    case SLOS_COMP_TWOSUM: return (int)launch_comp<float, SLOS_COMP_TWOSUM>(l, s);
    case SLOS_COMP_F64: return (int)launch_comp<float, SLOS_COMP_F64>(l, s);
    default: return (int)launch_comp<float, SLOS_COMP_NONE>(l, s);
    }
}
