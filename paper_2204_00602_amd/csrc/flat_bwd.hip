// HIP kernels (gfx950): the adjoint of the table-driven layers (flat.hip).
//
// With g = dL/d conj(.), the reverse of layer k is, over the states y of layer
// k - 1,
//     g_{k-1}[y] = sum_j conj(U[j, i_k]) g_k[y + e_j]        (every mode j)
//     G_U[j, i_k] += sum_y g_k[y + e_j] conj(A_{k-1}[y]),
// the rank of y + e_j read from the layer's successor table.  Both sums take
// the same loads.  A thread owns a state and visits the modes four at a time;
// the gradient products stay in registers and go through a wave reduction that
// gives each quarter of the wave one of the four modes, so no term touches LDS
// except to read g.  FP64 sums, every order fixed, no atomics.
//   bwd_flat_kernel   one layer per launch, partials per workgroup
//   tail_kernel       layers t..1 of an instance in the LDS of one workgroup,
//                     then the partials of the layers above and G_U
#include <algorithm>

#include "accum.h"
#include "flat.h"

namespace {

// v of lane l and w of its partner, added after the lanes' halves (rows) have
// been exchanged: of v the lower (even) ones stay, of w the upper (odd) ones.
// HALVES: lanes 0-31 end with v[l] + v[l + 32], lanes 32-63 with w[l - 32] +
// w[l]; else the same within each pair of 16-lane rows.
template <bool HALVES>
__device__ __forceinline__ double swap_add(double v, double w)
{
    const uint64_t a = (uint64_t)__double_as_longlong(v), b = (uint64_t)__double_as_longlong(w);
    auto swap = [](uint32_t x, uint32_t y) {
        if constexpr (HALVES) return __builtin_amdgcn_permlane32_swap(x, y, false, false);
        else return __builtin_amdgcn_permlane16_swap(x, y, false, false);
    };
    const auto lo = swap((uint32_t)a, (uint32_t)b), hi = swap((uint32_t)(a >> 32), (uint32_t)(b >> 32));
    return __longlong_as_double((long long)((uint64_t)lo[0] | (uint64_t)hi[0] << 32)) +
           __longlong_as_double((long long)((uint64_t)lo[1] | (uint64_t)hi[1] << 32));
}
// v of the lane ROT places on in the 16-lane row
template <int ROT>
__device__ __forceinline__ double row_rotate(double v)
{
    const uint64_t a = (uint64_t)__double_as_longlong(v);
    constexpr int ctrl = 0x120 + ROT;  // row_ror
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)a, ctrl, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(a >> 32), ctrl, 0xF, 0xF, true);
    return __longlong_as_double((long long)((uint64_t)lo | (uint64_t)hi << 32));
}
__device__ __forceinline__ double row_sum(double v)
{
    v += row_rotate<8>(v);
    v += row_rotate<4>(v);
    v += row_rotate<2>(v);
    v += row_rotate<1>(v);
    return v;
}
// sums over the four lanes of a quad, and over the lanes of one place in each quad
template <int CTRL>
__device__ __forceinline__ double quad_perm(double v)
{
    const uint64_t a = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)a, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(a >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)((uint64_t)lo | (uint64_t)hi << 32));
}
__device__ __forceinline__ double quad_sum(double v)
{
    v += quad_perm<0xB1>(v);  // lanes 1 0 3 2
    v += quad_perm<0x4E>(v);  // lanes 2 3 0 1
    return v;
}
__device__ __forceinline__ double lanes4_sum(double v)
{
    v += row_rotate<8>(v);
    v += row_rotate<4>(v);
    v = swap_add<false>(v, v);
    return swap_add<true>(v, v);
}
// Sums of p[0..3] over the wave: every lane of row q = lane / 16 ends with the
// sum of p[q].  Two exchange steps keep half of the modes each, then a row sum:
// register moves only (with LDS permutes the tail's reductions alone took
// several microseconds).
__device__ __forceinline__ double2 quarter_sums(const double2 p[4])
{
    const double2 a{swap_add<true>(p[0].x, p[2].x), swap_add<true>(p[0].y, p[2].y)};
    const double2 b{swap_add<true>(p[1].x, p[3].x), swap_add<true>(p[1].y, p[3].y)};
    return double2{row_sum(swap_add<false>(a.x, b.x)), row_sum(swap_add<false>(a.y, b.y))};
}

__device__ __forceinline__ double2 wide(const float2 v) { return double2{(double)v.x, (double)v.y}; }
__device__ __forceinline__ double2 wide(const double2 v) { return v; }

// g += u s, p += s conj(a)
__device__ __forceinline__ void grad_terms(double2 &g, double2 &p, const double2 u, const double2 s, const double2 a)
{
    cmac(g, u, s);
    p.x = fma_(s.x, a.x, p.x);
    p.x = fma_(s.y, a.y, p.x);
    p.y = fma_(s.y, a.x, p.y);
    p.y = fma_(-s.x, a.y, p.y);
}

// Bound by latency (two dependent reads per four modes) up to a few hundred
// thousand states, then by the successor table's bytes.  m=16, n=8 in c128:
// layer 8 (170,544 states) 12.4 us, layers 7..5 4.5 to 7 us each, where the
// unit kernel (gradient products read and written in LDS per term) took 28,
// 25, 22 and 19, after a 15 us seed launch that SEED folds in.
//
// Reverse layer of the states of one workgroup: PT consecutive blocks of
// SLOS_BWD_THREADS states, one of each per thread.  SEED: gk holds dL/da, and g_n = c_S
// dL/da is formed (and rounded to the plan's type) where it is read.
template <typename T, int PT, bool SEED>
__global__ __launch_bounds__(SLOS_BWD_THREADS) void bwd_flat_kernel(FlatBwdParams p)
{
    using C = typename Cx<T>::type;
    constexpr int kWaves = SLOS_BWD_THREADS / 64;
    extern __shared__ __align__(16) unsigned char dyn[];
    double2 *u = (double2 *)dyn;           // conj(U[j, i_k]), zero from m to the next multiple of four
    const int m = p.m, m4 = (m + 3) & ~3;
    double2 *wpart = u + m4;               // [waves][m4]
    const uint64_t b = blockIdx.y;
    const C *__restrict__ gk = (const C *)((const char *)p.gk + b * p.gk_stride);
    C *__restrict__ gkm1 = (C *)((char *)p.gkm1 + b * p.gkm1_stride);
    const C *__restrict__ A = (const C *)((const char *)p.Akm1 + b * p.a_stride);
    const C *__restrict__ Um = (const C *)((const char *)p.U + b * p.u_stride);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (int j = tid; j < m4; j += SLOS_BWD_THREADS) {
        double2 v{0.0, 0.0};
        if (j < m) {
            v = wide(Um[(size_t)j * m + p.col]);
            v.y = -v.y;
        }
        u[j] = v;
    }
    uint32_t y[PT];
    double2 a[PT], g[PT];
    const uint32_t N = p.N, y0 = blockIdx.x * (uint32_t)(PT * SLOS_BWD_THREADS) + tid;
    const bool whole = (blockIdx.x + 1u) * (uint64_t)(PT * SLOS_BWD_THREADS) <= N;  // no state past the end here
#pragma unroll
    for (int r = 0; r < PT; ++r) {
        const uint32_t yr = y0 + (uint32_t)r * SLOS_BWD_THREADS;
        y[r] = min(yr, N - 1u);
        // a state past the end contributes nothing to the gradient
        a[r] = yr < N ? wide(A[y[r]]) : double2{0.0, 0.0};
        g[r] = double2{0.0, 0.0};
    }
    __syncthreads();
    uint32_t e[PT][4];
    auto fetch = [&](int j0) {
#pragma unroll
        for (int r = 0; r < PT; ++r)
#pragma unroll
            for (int d = 0; d < 4; ++d) e[r][d] = p.succ[(size_t)min(j0 + d, m - 1) * N + y[r]];
    };
    fetch(0);
    for (int j0 = 0; j0 < m; j0 += 4) {
        double2 s[PT][4], pj[4];
#pragma unroll
        for (int r = 0; r < PT; ++r)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                s[r][d] = wide(gk[e[r][d]]);
                if (SEED) {
                    const double f = p.scale[e[r][d]];
                    s[r][d] = double2{(double)(T)(f * s[r][d].x), (double)(T)(f * s[r][d].y)};
                }
            }
        if (j0 + 4 < m) fetch(j0 + 4);
        // no term of a state past the end or of a mode past the last: an infinite g
        // would not vanish against their zeros
        if (!whole || j0 + 4 > m) {
#pragma unroll
            for (int r = 0; r < PT; ++r)
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    if (y0 + (uint32_t)r * SLOS_BWD_THREADS >= N || j0 + d >= m) s[r][d] = double2{0.0, 0.0};
        }
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            pj[d] = double2{0.0, 0.0};
            const double2 uj = u[j0 + d];
#pragma unroll
            for (int r = 0; r < PT; ++r) grad_terms(g[r], pj[d], uj, s[r][d], a[r]);
        }
        const double2 q = quarter_sums(pj);
        if ((lane & 15) == 0) wpart[wv * m4 + j0 + (lane >> 4)] = q;
    }
#pragma unroll
    for (int r = 0; r < PT; ++r)
        if (y0 + (uint32_t)r * SLOS_BWD_THREADS < N) gkm1[y[r]] = C{(T)g[r].x, (T)g[r].y};
    __syncthreads();
    double2 *out = (double2 *)((char *)p.partials + b * p.partials_stride) + (size_t)blockIdx.x * m;
    for (int j = tid; j < m; j += SLOS_BWD_THREADS) {
        double2 v = wpart[j];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
            v.x += wpart[w * m4 + j].x;
            v.y += wpart[w * m4 + j].y;
        }
        out[j] = v;
    }
}

template <int NM> struct Modes {
    static constexpr int value = NM;
};

// Bound by instruction issue in the layers of thousands of states and by the
// chain of one state's terms and the reductions in the others: m=12, n=6 (c64,
// 64 instances) 29 us for the loss, six layers and G_U, of which layer 6 takes
// 9.8 and layers 3..1 1.4 each; the launches it replaces took 109 us.
//
// Layers t..1 of instance blockIdx.x in one workgroup: g_k and g_{k-1} in LDS,
// one barrier between layers.  A thread keeps the gradient sums of
// SLOS_BWD_TAIL_MODES modes over all its states of a layer; further modes take
// another turn over the states.  The wave reductions come once per layer (and
// turn); the waves' sums stay apart in LDS and are added at the end, all layers
// together.  A layer's first loads (A and successor ranks, which depend on
// nothing computed here) are issued before the barrier that precedes it.  TH = 64
// only for t = n: the partials of layers above t are added by groups of m threads.
template <typename T, int TH>
__global__ __launch_bounds__(TH) __attribute__((amdgpu_waves_per_eu(4))) void tail_kernel(TailParams p)
{
    using C = typename Cx<T>::type;
    constexpr int GM = SLOS_BWD_TAIL_MODES;
    extern __shared__ __align__(16) unsigned char dyn[];
    __shared__ double sh[256];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int m = p.m, n = p.n, t = p.t, ms = m + 16;
    double2 *u = (double2 *)dyn;                 // [t][ms]: conj(U[j, i_k]), zero from m on
    double2 *cs = u + t * ms;                    // [n + 1][m]: column sums of layer k
    double2 *wpart = cs + (n + 1) * m;           // [wave_rows][m]: wave sums, layer k from row wrow[k]
    C *buf0 = (C *)(wpart + p.wave_rows * m), *buf1 = buf0 + p.cap[0];
    const uint64_t b = blockIdx.x;
    const C *__restrict__ Um = (const C *)((const char *)p.U + b * p.u_stride);

    // A and the successor ranks of state y: NM modes jb, jb + step, ..  The rank of
    // a mode past the last or of a state past the end is that of the zero behind
    // g_k, whatever the layer's values are (the tables have a row and a column for
    // them: forming that index here cost 43 spilled registers and 16 us).
    struct First {
        double2 a;
        uint32_t e[GM];
    };
    auto load = [&](First &f, int k, int jb, uint32_t y, auto modes, int step) {
        const uint32_t N = p.N[k - 1];
        const uint32_t *__restrict__ succ = p.succ + p.succ_off[k];
        y = min(y, N);
        f.a = wide(((const C *)((const char *)p.keep + b * p.keep_stride + p.keep_off[k - 1]))[min(y, N - 1u)]);
#pragma unroll
        for (int d = 0; d < decltype(modes)::value; ++d) {
            f.e[d] = 0;
            if (jb / 4 * 4 + step * (step == 1 ? d & ~3 : d) < m) f.e[d] = (succ + (size_t)min(jb + d * step, m) * (N + 1u))[y];
        }
    };
    auto small = [&](int k) { return p.N[k - 1] <= (uint32_t)TH; };  // four lanes a state
    First cur;
    auto load_first = [&](int k) {
        if (small(k)) load(cur, k, lane & 3, (uint32_t)tid >> 2, Modes<4>{}, 4);
        else load(cur, k, 0, (uint32_t)tid, Modes<GM>{}, 1);
    };
    load_first(t);
    for (int i = tid; i < t * ms; i += TH) {
        const int j = i % ms;
        double2 v{0.0, 0.0};
        if (j < m) {
            v = wide(Um[(size_t)j * m + p.col[i / ms + 1]]);
            v.y = -v.y;
        }
        u[i] = v;
    }

    // g_t
    C *top = t & 1 ? buf1 : buf0;
    const uint32_t Nt = p.N[t];
    if (p.a) {
        // the loss L = sum_s (|a(r_s)|^2 - P_s)^2 on the targets: zeros, then
        // g_n = c_S 4 (|a|^2 - P) a, each value formed as the loss and the seed
        // kernels form it one after the other, and the loss in the same order
        const C *a = (const C *)p.a + b * p.a_stride;
        const double *pt = p.p_target + b * (uint64_t)p.count;
        for (uint32_t s = tid; s <= Nt; s += TH) top[s] = C{0, 0};
        __syncthreads();
        for (int q = tid; q < 256; q += TH) {
            double s = 0.0;
            for (int64_t i = q; i < p.count; i += 256) {
                const int64_t r = p.ranks[i];
                if (r < 0 || (uint64_t)r >= Nt) continue;  // outside the output set: ignored
                const C v = a[r];
                const double P = (double)v.x * (double)v.x + (double)v.y * (double)v.y;
                const double d = P - pt[i];
                s += d * d;
                const T f = (T)(4.0 * d);
                const C ga{f * v.x, f * v.y};
                const double c = p.target_scale[i];
                top[r] = C{(T)(c * (double)ga.x), (T)(c * (double)ga.y)};
            }
            sh[q] = s;
        }
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            for (int q = tid; q < w; q += TH) sh[q] += sh[q + w];
            __syncthreads();
        }
        if (tid == 0 && p.loss) p.loss[b] = sh[0];
    } else {
        const C *g = (const C *)((const char *)p.gt + b * p.gt_stride);
        for (uint32_t s = tid; s < Nt; s += TH) {
            C v = g[s];
            if (p.scale) {
                const double f = p.scale[s];
                v = C{(T)(f * (double)v.x), (T)(f * (double)v.y)};
            }
            top[s] = v;
        }
        if (tid == 0) top[Nt] = C{0, 0};
    }
    __syncthreads();

    int wrow = 0;
    for (int k = t; k >= 1; --k) {
        const C *gk = k & 1 ? buf1 : buf0;
        C *gd = k & 1 ? buf0 : buf1;
        const uint32_t N = p.N[k - 1];
        const double2 *uk = u + (k - 1) * ms;
        const int busy = slos_tail_waves(N, TH);
        if (tid == 0) gd[N] = C{0, 0};
        if (small(k)) {
            // Four lanes a state, lane q of them modes q, q + 4, ..: the chain of
            // a layer with few states is a quarter as long.
            const int q = lane & 3;
            for (int jb = 0; jb < m; jb += 16) {
                double2 acc[4];
#pragma unroll
                for (int d = 0; d < 4; ++d) acc[d] = double2{0.0, 0.0};
                for (uint32_t y0 = 0; y0 < N; y0 += TH / 4) {
                    const uint32_t y = y0 + ((uint32_t)tid >> 2);
                    if (y0 + ((uint32_t)wv << 4) >= N) break;  // no state of this wave
                    First nxt;
                    load(nxt, k, jb + q, y + TH / 4, Modes<4>{}, 4);
                    const bool on = y < N;
                    const double2 a = on ? cur.a : double2{0.0, 0.0};
                    double2 g{0.0, 0.0};
#pragma unroll
                    for (int d = 0; d < 4; ++d)
                        if (jb + 4 * d < m) grad_terms(g, acc[d], uk[jb + 4 * d + q], wide(gk[cur.e[d]]), a);
                    if (jb == 0) {
                        for (int j = 16 + q; j < m; j += 4)
                            cmac(g, uk[j], wide(gk[(p.succ + p.succ_off[k] + (size_t)j * (N + 1u))[min(y, N)]]));
                        g.x = quad_sum(g.x);
                        g.y = quad_sum(g.y);
                        if (on && q == 0) gd[y] = C{(T)g.x, (T)g.y};
                    }
                    cur = nxt;
                }
                if (jb + 16 < m) load(cur, k, jb + 16 + q, (uint32_t)tid >> 2, Modes<4>{}, 4);
                else if (k > 1) load_first(k - 1);
                if (wv < busy) {
#pragma unroll
                    for (int d = 0; d < 4; ++d)
                        if (jb + 4 * d < m) {
                            const double2 v{lanes4_sum(acc[d].x), lanes4_sum(acc[d].y)};
                            const int j = jb + 4 * d + q;
                            if (lane < 4 && j < m) wpart[(wrow + wv) * m + j] = v;
                        }
                }
            }
        } else {
            for (int jb = 0; jb < m; jb += GM) {
                double2 acc[GM];
#pragma unroll
                for (int d = 0; d < GM; ++d) acc[d] = double2{0.0, 0.0};
                for (uint32_t y = tid; y < N; y += TH) {
                    if (y >= (uint32_t)TH) load(cur, k, jb, y, Modes<GM>{}, 1);
                    double2 g{0.0, 0.0};
#pragma unroll
                    for (int d = 0; d < GM; ++d)
                        if (jb + (d & ~3) < m) grad_terms(g, acc[d], uk[jb + d], wide(gk[cur.e[d]]), cur.a);
                    if (jb == 0) {
                        // modes beyond the first turn's, for g_{k-1} alone
                        for (int j = GM; j < m; ++j)
                            cmac(g, uk[j], wide(gk[(p.succ + p.succ_off[k] + (size_t)j * (N + 1u))[y]]));
                        gd[y] = C{(T)g.x, (T)g.y};
                    }
                }
                if (jb + GM < m) load(cur, k, jb + GM, (uint32_t)tid, Modes<GM>{}, 1);
                else if (k > 1) load_first(k - 1);
#pragma unroll
                for (int d = 0; d < GM; d += 4)
                    if (jb + d < m) {
                        const double2 q = quarter_sums(acc + d);
                        const int j = jb + d + (lane >> 4);
                        if ((lane & 15) == 0 && j < m) wpart[(wrow + wv) * m + j] = q;
                    }
            }
        }
        wrow += busy;
        __syncthreads();  // g_{k-1} and the wave sums are complete
    }
    // column sums: layers t..1 over their waves, in order
    for (int i = tid; i < t * m; i += TH) {
        const int k = t - i / m, j = i % m;
        int row = 0;
        for (int q = t; q > k; --q) row += slos_tail_waves(p.N[q - 1], TH);
        const int end = row + slos_tail_waves(p.N[k - 1], TH);
        double2 v{0.0, 0.0};
        for (; row < end; ++row) {
            v.x += wpart[row * m + j].x;
            v.y += wpart[row * m + j].y;
        }
        cs[k * m + j] = v;
    }
    // The layers above t, four at a time: G groups of m threads, group q adds
    // rows q, q + G, .. of each layer's partials (neighbouring threads read
    // neighbouring values), then one thread per layer and mode adds the groups.
    const double2 *part = (const double2 *)((const char *)p.partials + b * p.partials_stride);
    double2 *red = (double2 *)buf0;  // the g buffers are free: room for 4 TH values (see slos_tail_lds)
    const int G = TH / m, q = tid / m, j = tid % m;
    for (int k0 = t + 1; k0 <= n; k0 += 4) {
        if (q < G) {
            double2 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = double2{0.0, 0.0};
                if (k0 + i > n) continue;
                const double2 *pk = part + p.part_off[k0 + i] + j;
                const uint32_t rows = p.rows[k0 + i];
#pragma unroll 4
                for (uint32_t r = (uint32_t)q; r < rows; r += (uint32_t)G) {
                    const double2 w = pk[(size_t)r * m];
                    v[i].x += w.x;
                    v[i].y += w.y;
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) red[i * G * m + q * m + j] = v[i];
        }
        __syncthreads();
        for (int i = tid; i < 4 * m; i += TH) {
            const int k = k0 + i / m, jj = i % m;
            if (k > n) continue;
            const double2 *rk = red + (i / m) * G * m + jj;
            double2 v{0.0, 0.0};
#pragma unroll 8
            for (int g = 0; g < G; ++g) {
                v.x += rk[g * m].x;
                v.y += rk[g * m].y;
            }
            cs[k * m + jj] = v;
        }
        __syncthreads();
    }
    __syncthreads();
    // G_U[j, i] = sum over the layers of column i, in order
    C *GU = (C *)((char *)p.GU + b * p.gu_stride);
    for (int e = tid; e < m * m; e += TH) {
        const int j = e / m, i = e % m;
        double2 v{0.0, 0.0};
        for (int k = 1; k <= n; ++k)
            if (p.col[k] == i) {
                v.x += cs[k * m + j].x;
                v.y += cs[k * m + j].y;
            }
        GU[e] = C{(T)v.x, (T)v.y};
    }
}

template <typename T, int PT>
void launch_layer(const FlatBwdParams &p, int batch, hipStream_t s)
{
    const int m4 = (p.m + 3) & ~3;
    const size_t lds = (size_t)m4 * (1 + SLOS_BWD_THREADS / 64) * sizeof(double2);
    const dim3 g(slos_bwd_rows(p.N, PT), batch);
    if (p.scale) hipLaunchKernelGGL((bwd_flat_kernel<T, PT, true>), g, dim3(SLOS_BWD_THREADS), lds, s, p);
    else hipLaunchKernelGGL((bwd_flat_kernel<T, PT, false>), g, dim3(SLOS_BWD_THREADS), lds, s, p);
}

template <typename T, int TH>
hipError_t launch_tail(const TailParams &p, int batch, hipStream_t s)
{
    static bool attr_set = false;  // per instantiation; first call per process
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)tail_kernel<T, TH>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)SLOS_LDS_DYNAMIC_MAX);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const size_t lds =
        (size_t)slos_tail_lds(p.cap[0], p.cap[1], p.m, p.n, p.t, p.wave_rows, TH, sizeof(typename Cx<T>::type));
    hipLaunchKernelGGL((tail_kernel<T, TH>), dim3(batch), dim3(TH), lds, s, p);
    return hipGetLastError();
}

template <typename T>
hipError_t launch(const FlatBwdLaunch &l, int batch, hipStream_t s)
{
    if (l.tail) {
        switch (l.tail->threads) {
        case 64: return launch_tail<T, 64>(*l.tail, batch, s);
        case 256: return launch_tail<T, 256>(*l.tail, batch, s);
        default: return launch_tail<T, SLOS_BWD_TAIL_THREADS>(*l.tail, batch, s);
        }
    }
    if (l.per_thread == 1) launch_layer<T, 1>(*l.layer, batch, s);
    else if (l.per_thread == 2) launch_layer<T, 2>(*l.layer, batch, s);
    else launch_layer<T, 4>(*l.layer, batch, s);
    return hipGetLastError();
}

} // namespace

int slos_launch_flat_bwd(const FlatBwdLaunch &l, int c64, int batch, void *stream)
{
    return (int)(c64 ? launch<float>(l, batch, (hipStream_t)stream) : launch<double>(l, batch, (hipStream_t)stream));
}
