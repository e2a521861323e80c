// HIP kernels (gfx950): weak simulation from the strong one.
//
// The sampler the paper builds on its strong back-ends (Section 3.2) draws
// outputs S with probability P(S).  From the full distribution in colex order
// this is an inverse-CDF lookup: for a uniform r in [0, 1) the sample is the
// first S whose cumulative probability exceeds r * sum P.  The same prefix sums
// give the partial certificate of Eq. eqpk: P(K), the probability that modes
// K..m-1 are empty, is the sum over the first C(K+n-1, n) states (those states
// form a colex prefix).
//
// Layout: P is cut into blocks of SLOS_CDF_BLOCK states.  cdf_block_kernel sums
// each block in FP64 (one wave per block, fixed order) and keeps the sums of its
// 16 chunks of 64 states (cs = sp + nsup + 1); runs of SLOS_CDF_BLOCK block sums
// are summed again (sp = bp + nb + 1), and cdf_scan_kernel turns the block sums
// into the exclusive prefix bp[0..nb] (bp[nb] = sum P), every step in a fixed
// order, so the table is reproducible, and copies every 16^l-th prefix into a
// 16-ary search tree (after cs).  A sample finds its block in the tree, its chunk
// from the block's 16 chunk sums (one line), and then its state with a scan of
// that chunk's 64 probabilities: about 1 KB per sample.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "slos_ext.h"

namespace {

constexpr int kChunks = SLOS_CDF_BLOCK / 64;

typedef float cdf_f4 __attribute__((ext_vector_type(4)));
typedef double cdf_d2 __attribute__((ext_vector_type(2)));

// Block b is read in SLOS_CDF_BLOCK / 256 steps of 256 consecutive states: in
// step i lane l holds states 256 i + 4 l .. 256 i + 4 l + 3 (one 16-byte load
// for fp32, two for fp64), so each load of the wave covers one contiguous KiB
// (fp32).  part[i] = the lane's sum of its four states of step i.
constexpr int kSteps = SLOS_CDF_BLOCK / 256;

template <typename T>
__device__ __forceinline__ void lane_parts(const T *__restrict__ P, int64_t M, int64_t b, int lane, bool full,
                                           double *part)
{
    const int64_t base = b * SLOS_CDF_BLOCK + 4 * (int64_t)lane;
    if (full) {
        if constexpr (sizeof(T) == 4) {
            cdf_f4 v[kSteps];
#pragma unroll
            for (int i = 0; i < kSteps; ++i) v[i] = __builtin_nontemporal_load((const cdf_f4 *)(P + base + 256 * i));
#pragma unroll
            for (int i = 0; i < kSteps; ++i)
                part[i] = ((double)v[i].x + (double)v[i].y) + ((double)v[i].z + (double)v[i].w);
        } else {
            cdf_d2 v[2 * kSteps];
#pragma unroll
            for (int i = 0; i < kSteps; ++i) {
                v[2 * i] = __builtin_nontemporal_load((const cdf_d2 *)(P + base + 256 * i));
                v[2 * i + 1] = __builtin_nontemporal_load((const cdf_d2 *)(P + base + 256 * i) + 1);
            }
#pragma unroll
            for (int i = 0; i < kSteps; ++i)
                part[i] = (v[2 * i].x + v[2 * i].y) + (v[2 * i + 1].x + v[2 * i + 1].y);
        }
    } else {
        for (int i = 0; i < kSteps; ++i) {
            double s = 0.0;
            for (int e = 0; e < 4; ++e) {
                const int64_t x = base + 256 * i + e;
                if (x < M) s += (double)P[x];
            }
            part[i] = s;
        }
    }
}

// block sum bp[b] and the block's 16 chunk sums from the lanes' parts: chunk
// 4 i + g (64 states) is step i of lanes 16 g .. 16 g + 15
__device__ __forceinline__ void block_finish(const double *part, int64_t b, int lane, double *__restrict__ bp,
                                             double *__restrict__ cs)
{
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
        double c = part[i];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) c += __shfl_xor(c, o, 64);
        if ((lane & 15) == 0) cs[b * kChunks + 4 * i + (lane >> 4)] = c;
        s += part[i];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) bp[b] = s;
}

// One wave per pair of blocks (b, b + nw) per step: both blocks' loads are in
// flight together.
template <typename T>
__global__ __launch_bounds__(256) void cdf_block_kernel(const T *__restrict__ P, int64_t M, int64_t nb,
                                                        double *__restrict__ bp, double *__restrict__ cs)
{
    static_assert(SLOS_CDF_BLOCK == 1024, "16 chunks of 64 states in 4 steps of 256");
    const int lane = threadIdx.x & 63;
    const int64_t gw = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
    const int64_t nfull = M / SLOS_CDF_BLOCK;  // blocks without a tail
    for (int64_t b0 = gw; b0 < nb; b0 += 2 * nw) {
        const int64_t b1 = b0 + nw;
        double p0[kSteps], p1[kSteps];
        lane_parts(P, M, b0, lane, b0 < nfull, p0);
        if (b1 < nb) lane_parts(P, M, b1, lane, b1 < nfull, p1);
        block_finish(p0, b0, lane, bp, cs);
        if (b1 < nb) block_finish(p1, b1, lane, bp, cs);
    }
}

// Sum of each run of SLOS_CDF_BLOCK consecutive entries of v[0..nv): one wave per
// run, its sixteen loads in flight together.
__global__ __launch_bounds__(64) void cdf_super_kernel(const double *__restrict__ v, int64_t nv, int64_t nsup,
                                                       double *__restrict__ out)
{
    const int lane = threadIdx.x;
    for (int64_t b = blockIdx.x; b < nsup; b += gridDim.x) {
        double x[kChunks];
#pragma unroll
        for (int i = 0; i < kChunks; ++i) x[i] = v[min(b * SLOS_CDF_BLOCK + i * 64 + lane, nv - 1)];
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < kChunks; ++i) s += b * SLOS_CDF_BLOCK + i * 64 + lane < nv ? x[i] : 0.0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (lane == 0) out[b] = s;
    }
}

// Block sums -> exclusive prefix, its total bp[nb] and the search tree over it.
// A workgroup takes one run of SLOS_CDF_BLOCK block sums: it adds up the sums sp
// of the runs before it (1024 parts, then their serial prefix, the same order in
// every workgroup), and each of its waves scans a chunk of 64 block sums (wave
// scan in a fixed order) and adds the prefix of the run's chunks, serially, to
// it.  Every 16^l-th prefix goes to level l of the tree.  What bounds it is the
// serial prefix and the latency of a few loads: for 126,000 blocks (123 runs) this
// and the launch above take 9.4 us; as four launches (run sums, their scan on
// one workgroup, prefix, tree) 33.
__global__ __launch_bounds__(1024) void cdf_scan_kernel(double *__restrict__ bp, int64_t nb,
                                                        const double *__restrict__ sp, int64_t nsup,
                                                        double *__restrict__ tree, CdfTree t)
{
    __shared__ double part[1024];
    __shared__ double chunk[kChunks];
    __shared__ double start;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t per = (nsup + 1023) / 1024;
    const int nparts = (int)((nsup + per - 1) / per);
    for (int64_t b = blockIdx.x; b < nsup; b += gridDim.x) {
        const int64_t x = b * SLOS_CDF_BLOCK + tid;
        const double v = x < nb ? bp[x] : 0.0;
        double s = 0.0;
        for (int64_t i = min(tid * per, nsup); i < min((tid + 1) * per, nsup); ++i) s += sp[i];
        part[tid] = s;
        double c = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double u = __shfl_up(c, o, 64);
            if (lane >= o) c += u;
        }
        if (lane == 63) chunk[wv] = c;
        __syncthreads();
        if (tid == 0) {
            // prefix of the part that run b is in, then of the runs in it; the
            // last run goes on to the total
            const int pb = (int)(b / per);
            double run = 0.0;
            auto add_parts = [&](int i, int end) {
                for (; i + 16 <= end; i += 16) {  // sixteen reads in flight before their chain of additions
                    double y[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) y[e] = part[i + e];
#pragma unroll
                    for (int e = 0; e < 16; ++e) run += y[e];
                }
                for (; i < end; ++i) run += part[i];
            };
            add_parts(0, pb);
            double r = run;
            for (int64_t i = pb * per; i < b; ++i) r += sp[i];
            start = r;
            if (b == nsup - 1) {
                add_parts(pb, nparts);
                bp[nb] = run;
            }
        }
        __syncthreads();
        double run = start;
        for (int i = 0; i < wv; ++i) run += chunk[i];
        if (x < nb) {
            const double y = run + (c - v);
            bp[x] = y;
            int64_t i = x;
            for (int l = 1; l < t.nlev && (i & 15) == 0; ++l) {
                i >>= 4;
                tree[t.off[l] + i] = y;
            }
        }
        __syncthreads();  // part, chunk and start are free
    }
}

// pk[K-1] = sum of P over the first ends[K-1] states, K = 1..m; one wave per K.
template <typename T>
__global__ __launch_bounds__(256) void marginal_kernel(const T *__restrict__ P, const double *__restrict__ bp,
                                                       const int64_t *__restrict__ ends, int m,
                                                       double *__restrict__ pk)
{
    const int lane = threadIdx.x & 63;
    const int K = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (K >= m) return;
    const int64_t e = ends[K];
    const int64_t b = e / SLOS_CDF_BLOCK;
    T v[kChunks];  // the block's states below e: sixteen loads in flight
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
        const int64_t x = b * SLOS_CDF_BLOCK + i * 64 + lane;
        v[i] = x < e ? P[x] : (T)0;
    }
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kChunks; ++i) s += (double)v[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) pk[K] = bp[b] + s;
}

// States x .. x + 3, zeros from M on.  P needs no more than its elements'
// alignment.
typedef float cdf_f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef double cdf_d2u __attribute__((ext_vector_type(2), aligned(8)));
template <typename T> __device__ __forceinline__ void load_states(T *v, const T *__restrict__ P, int64_t x, int64_t M)
{
    if (x + 4 <= M) {
        if constexpr (sizeof(T) == 4) {
            const cdf_f4u y = *(const cdf_f4u *)(P + x);
            v[0] = y.x, v[1] = y.y, v[2] = y.z, v[3] = y.w;
        } else {
            const cdf_d2u y = *(const cdf_d2u *)(P + x);
            const cdf_d2u z = *((const cdf_d2u *)(P + x) + 1);
            v[0] = y.x, v[1] = y.y, v[2] = z.x, v[3] = z.y;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = x + e < M ? P[x + e] : (T)0;
    }
}

// The group's sixteen lanes: inclusive prefix of c, each partial sum from the
// lane o below (o = 1, 2, 4, 8); the lanes without one add nothing.
template <int CTRL> __device__ __forceinline__ double row_shr(double x)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double group_prefix(double c)
{
    c += row_shr<0x111>(c);
    c += row_shr<0x112>(c);
    c += row_shr<0x114>(c);
    c += row_shr<0x118>(c);
    return c;
}

// ranks[s] = first state whose cumulative P exceeds r[s] * total.  The finest
// level of the tree that fits the LDS is searched there by one lane per sample;
// from it down, sixteen lanes serve a sample, four samples to an instruction and
// kFlight of these in flight: what bounds a sample is its chain of dependent loads
// (tree lines, chunk sums, states), and what bounds many of them is their random
// lines (two of states, two of sums: 131 us for 1,048,576 samples of 129 M
// states, 4 TB/s; with sixteen lanes on every level and one sample each 222).
// States are read through the caches: 93 us at 490,314 states in c128, 122 past
// them, and the same at 129 M.
constexpr int kFlight = 4;

template <typename T>
__global__ __launch_bounds__(256) void sample_kernel(const T *__restrict__ P, int64_t M, const double *__restrict__ bp,
                                                      int64_t nb, const double *__restrict__ r, int64_t count,
                                                      int64_t *__restrict__ ranks, CdfTree tr, int top, int per_wave)
{
    extern __shared__ double tab[];  // level `top`
    const int64_t nsup = (nb + SLOS_CDF_BLOCK - 1) / SLOS_CDF_BLOCK;
    const double *__restrict__ sp = bp + nb + 1;  // run sums, nsup + 1 places
    const double *__restrict__ cs = sp + nsup + 1;  // chunk sums, kChunks per block
    const double *__restrict__ tree = cs + kChunks * nb;
    const int lane = threadIdx.x & 63, g = lane >> 4, l16 = lane & 15;
    const int64_t gw = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
    const double total = bp[nb];
    const uint32_t ntop = (uint32_t)tr.n[top];
    {
        const double *src = top == 0 ? bp : tree + tr.off[top];
        for (uint32_t i = threadIdx.x; i < ntop; i += blockDim.x) tab[i] = src[i];
    }
    __syncthreads();
    uint32_t half = 1;
    while (half * 2 < ntop) half *= 2;
    // the group's 16 bits of a wave ballot
    auto gbits = [&](bool pred) -> uint32_t { return (uint32_t)((__ballot(pred) >> (16 * g)) & 0xFFFFu); };
    for (int64_t w0 = gw * per_wave; w0 < count; w0 += nw * per_wave) {
        // lane: one sample.  The largest entry <= t: the tables are non-decreasing
        // and start at 0 <= t.
        const int64_t own = w0 + (lane & (per_wave - 1));
        const double t_own = r[min(own, count - 1)] * total;
        uint32_t at = 0;
        for (uint32_t h = half; h > 0; h >>= 1)
            if (at + h < ntop && tab[at + h] <= t_own) at += h;
        for (int q = 0; q < per_wave && w0 + q < count; q += 4 * kFlight) {
            // group: kFlight samples.  Down the tree: at each level the largest
            // entry <= t among the 16 children of the choice above
            double t[kFlight], b0[kFlight], c_own[kFlight];
            uint32_t lo[kFlight];
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {
                t[u] = __shfl(t_own, q + 4 * u + g, 64);
                lo[u] = (uint32_t)__shfl((int)at, q + 4 * u + g, 64);
                if (top == 0) b0[u] = tab[lo[u]];
            }
            for (int l = top - 1; l >= 0; --l) {
                const double *lev = l == 0 ? bp : tree + tr.off[l];
                const int64_t n = tr.n[l];
                double y[kFlight];
#pragma unroll
                for (int u = 0; u < kFlight; ++u) y[u] = lev[min((int64_t)lo[u] * 16 + l16, n - 1)];
#pragma unroll
                for (int u = 0; u < kFlight; ++u) {
                    const uint32_t bal = gbits((int64_t)lo[u] * 16 + l16 < n && y[u] <= t[u]);
                    const int i = bal ? 31 - __builtin_clz(bal) : 0;
                    lo[u] = lo[u] * 16 + (uint32_t)i;
                    if (l == 0) b0[u] = __shfl(y[u], i, 16);
                }
            }
            // the block's chunk sums (one line): the first chunk whose running sum
            // exceeds t, else the last chunk of non-zero probability
#pragma unroll
            for (int u = 0; u < kFlight; ++u) c_own[u] = cs[(int64_t)lo[u] * kChunks + l16];
            double run[kFlight];
            int ci[kFlight];
            T p[kFlight][4];  // the chunk's states, four per lane
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {
                const double c_inc = group_prefix(c_own[u]);
                const uint32_t c_cross = gbits(b0[u] + c_inc > t[u] && c_own[u] > 0.0);
                const uint32_t c_pos = gbits(c_own[u] > 0.0);
                ci[u] = c_cross ? __builtin_ctz(c_cross) : (c_pos ? 31 - __builtin_clz(c_pos) : 0);
                run[u] = b0[u] + __shfl(c_inc - c_own[u], ci[u], 16);
                const int64_t x0 = (int64_t)lo[u] * SLOS_CDF_BLOCK + (int64_t)ci[u] * 64 + 4 * l16;
                load_states(p[u], P, x0, M);
            }
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {
                // the states of the chunks from ci on (rounding between the chunk
                // sums and this scan can move the crossing on to a later chunk)
                const int64_t base = (int64_t)lo[u] * SLOS_CDF_BLOCK;
                int64_t found = -1, last_pos = -1;
                int c = ci[u];
                for (int it = 0; it < kChunks; ++it) {
                    const bool open = found < 0 && c < kChunks;
                    if (!__ballot(open)) break;
                    if (it > 0) load_states(p[u], P, open ? base + (int64_t)c * 64 + 4 * l16 : M, M);
                    double v[4], in[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = (double)p[u][e];
                    in[0] = v[0];
#pragma unroll
                    for (int e = 1; e < 4; ++e) in[e] = in[e - 1] + v[e];
                    const double lsum = group_prefix(in[3]);  // of the lanes' sums
                    const double excl = lsum - in[3];
                    int first_e = -1, last_e = -1;
#pragma unroll
                    for (int e = 3; e >= 0; --e) {
                        if (v[e] > 0.0 && run[u] + excl + in[e] > t[u]) first_e = e;
                        if (last_e < 0 && v[e] > 0.0) last_e = e;
                    }
                    const uint32_t cross = gbits(open && first_e >= 0);
                    const uint32_t pos = gbits(open && last_e >= 0);
                    if (open) {
                        if (cross) {
                            const int src = __builtin_ctz(cross);
                            found = base + (int64_t)c * 64 + 4 * src + __shfl(first_e, src, 16);
                        }
                        if (pos) {
                            const int src = 31 - __builtin_clz(pos);
                            last_pos = base + (int64_t)c * 64 + 4 * src + __shfl(last_e, src, 16);
                        }
                        run[u] += __shfl(lsum, 15, 16);  // shuffles stay within the group, all of whose lanes are here
                        ++c;
                    }
                }
                // rounding can leave the crossing past the block's recomputed sum:
                // take the block's last state of non-zero probability
                if (found < 0) found = last_pos >= 0 ? last_pos : min(base, M - 1);
                const int64_t sidx = w0 + q + 4 * u + g;
                if (l16 == 0 && sidx < count) ranks[sidx] = found;
            }
        }
    }
}

} // namespace

int slos_launch_cdf(const void *P, int c64, int64_t M, double *bp, void *stream)
{
    const int64_t nb = (M + SLOS_CDF_BLOCK - 1) / SLOS_CDF_BLOCK;
    const int64_t nsup = (nb + SLOS_CDF_BLOCK - 1) / SLOS_CDF_BLOCK;
    double *sp = bp + nb + 1;    // nsup + 1 run prefixes after the table
    double *cs = sp + nsup + 1;  // then 16 chunk sums per block
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((nb + 3) / 4, 8192));
    const int gsup = (int)std::max<int64_t>(1, std::min<int64_t>(nsup, 8192));
    hipStream_t s = (hipStream_t)stream;
    if (c64)
        hipLaunchKernelGGL(cdf_block_kernel<float>, dim3(grid), dim3(256), 0, s, (const float *)P, M, nb, bp, cs);
    else
        hipLaunchKernelGGL(cdf_block_kernel<double>, dim3(grid), dim3(256), 0, s, (const double *)P, M, nb, bp, cs);
    hipLaunchKernelGGL(cdf_super_kernel, dim3(gsup), dim3(64), 0, s, (const double *)bp, nb, nsup, sp);
    hipLaunchKernelGGL(cdf_scan_kernel, dim3(gsup), dim3(1024), 0, s, bp, nb, (const double *)sp, nsup, cs + kChunks * nb,
                       cdf_tree_layout(nb));
    return (int)hipGetLastError();
}

int slos_launch_marginals(const void *P, int c64, const double *bp, const int64_t *ends, int m, double *pk,
                          void *stream)
{
    const int grid = (m + 3) / 4;
    hipStream_t s = (hipStream_t)stream;
    if (c64)
        hipLaunchKernelGGL(marginal_kernel<float>, dim3(grid), dim3(256), 0, s, (const float *)P, bp, ends, m, pk);
    else
        hipLaunchKernelGGL(marginal_kernel<double>, dim3(grid), dim3(256), 0, s, (const double *)P, bp, ends, m, pk);
    return (int)hipGetLastError();
}

int slos_launch_sample(const void *P, int c64, int64_t M, const double *bp, const double *r, int64_t count,
                       int64_t *ranks, void *stream)
{
    const int64_t nb = (M + SLOS_CDF_BLOCK - 1) / SLOS_CDF_BLOCK;
    const CdfTree tr = cdf_tree_layout(nb);
    // A lane for every sample's search where there are enough of them for the
    // chip's 8192 waves, else sixteen samples to a wave, which spreads their chains
    // of loads over the chip (65,536 samples of 20 modes, 10 photons in c128 with
    // the table: 53 us, 72 at 64 to a wave; 1,048,576 of 22 and 11: 241 and 228).
    // A level of at most 1024 entries (8 KB) in the LDS: one of 8192 for large
    // workgroups is no faster (225 us against 228, 123 against 122 at 16 and 8).
    const int threads = 256, group = threads / 64, per_wave = count >= 64 * 8192 ? 64 : 16;
    int top = 0;
    while (tr.n[top] > 1024) ++top;  // the last level has at most 16 entries
    const size_t lds = (size_t)tr.n[top] * sizeof(double);
    const int64_t waves = (count + per_wave - 1) / per_wave;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((waves + group - 1) / group, 2048));
    hipStream_t s = (hipStream_t)stream;
    if (c64)
        hipLaunchKernelGGL(sample_kernel<float>, dim3(grid), dim3(threads), lds, s, (const float *)P, M, bp, nb, r, count,
                           ranks, tr, top, per_wave);
    else
        hipLaunchKernelGGL(sample_kernel<double>, dim3(grid), dim3(threads), lds, s, (const double *)P, M, bp, nb, r,
                           count, ranks, tr, top, per_wave);
    return (int)hipGetLastError();
}
