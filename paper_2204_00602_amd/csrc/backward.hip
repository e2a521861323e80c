// HIP kernels (gfx950) for differentiation: the adjoint of the SLOS layer
// recurrence and the rectangular MZI mesh (phases -> U and its reverse sweep).
//
// Forward layer (arXiv 2204.00602, Section 3.2.3 recurrence):
//     A_k[t] = sum_j U[j, i_k] A_{k-1}[t - e_j].
// With g = dL/d conj(.) (the PyTorch convention for a real loss L), the
// reverse of one layer is
//     g_{k-1}[t'] = sum_j conj(U[j, i_k]) g_k[t' + e_j]          (every mode j)
//     G_U[j, i_k] += sum_{t'} g_k[t' + e_j] conj(A_{k-1}[t'])
// and the last-layer normalisation a = c_S A_n[S] (c_S real) seeds
//     g_n[S] = c_S g_a[S].
// Work unit: the low block of one forward leaf of layer k (these blocks
// partition A_{k-1}); one wave per unit, every output written by one lane, no
// atomics.  Gradient partials are kept per (unit, mode) and summed in a fixed
// order.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "flat.h"
#include "slos_internal.h"

namespace {

template <typename T> struct Cb;
template <> struct Cb<float> { using type = float2; };
template <> struct Cb<double> { using type = double2; };

// ---- seed: g_n = c_S * g_a over the last layer's leaves --------------------
// One wave per leaf.  (Eight waves per leaf, one row of 64 states each, measured
// slower at m=12 n=6 with 64 instances: 10.5 against 8.9 us.)
template <typename T>
__global__ __launch_bounds__(256) void seed_kernel(const LeafDescHead *__restrict__ heads, uint64_t nleaves,
                                                   uint32_t stride_bytes, const double *__restrict__ lowfac,
                                                   const typename Cb<T>::type *__restrict__ ga,
                                                   typename Cb<T>::type *__restrict__ gn, uint64_t ga_stride,
                                                   uint64_t gn_stride)
{
    using C = typename Cb<T>::type;
    // instance blockIdx.y: element offsets
    ga += blockIdx.y * ga_stride;
    gn += blockIdx.y * gn_stride;
    const int lane = threadIdx.x & 63;
    const uint64_t gw = (uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const uint64_t nw = (uint64_t)gridDim.x * (blockDim.x >> 6);
    for (uint64_t li = gw; li < nleaves; li += nw) {
        const LeafDescHead h = *(const LeafDescHead *)((const char *)heads + li * stride_bytes);
        for (uint32_t x = lane; x < h.size; x += 64) {
            const double f = h.fac_hi * lowfac[h.fac_off + x];
            const C v = ga[h.out_base + x];
            gn[h.out_base + x] = C{(T)(f * (double)v.x), (T)(f * (double)v.y)};
        }
    }
}

// ---- one reverse layer --------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(64) void bwd_layer_kernel(BwdParams p)
{
    using C = typename Cb<T>::type;
    __shared__ C uc[256];                  // conj(U[j, i_k])
    extern __shared__ double2 part[];      // [jn][64] gradient partials of this wave
    if (blockIdx.y) {
        // instance blockIdx.y of a batch of unitaries through one plan
        const uint64_t b = blockIdx.y;
        p.gk = (const char *)p.gk + b * p.gk_stride;
        p.gkm1 = (char *)p.gkm1 + b * p.gkm1_stride;
        p.Akm1 = (const char *)p.Akm1 + b * p.a_stride;
        p.U = (const char *)p.U + b * p.u_stride;
        p.partials = (char *)p.partials + b * p.partials_stride;
    }
    const C *__restrict__ gk = (const C *)p.gk;
    C *__restrict__ gkm1 = (C *)p.gkm1;
    const C *__restrict__ A = (const C *)p.Akm1;
    const C *__restrict__ Um = (const C *)p.U;
    const int lane = threadIdx.x;
    for (int j = lane; j < 256; j += 64) {
        C v{0, 0};
        if (j < p.m) {
            v = Um[(size_t)j * p.m + p.col];
            v.y = -v.y;
        }
        uc[j] = v;
    }
    __syncthreads();

    for (uint64_t u = blockIdx.x; u < p.nunits; u += gridDim.x) {
        const BwdUnit U = p.units[u];
        for (int j = 0; j < p.jn; ++j) part[j * 64 + lane] = double2{0.0, 0.0};
        const uint32_t *__restrict__ succ = p.succ + U.succ_off;
        const uint64_t *__restrict__ hb = p.hbase + U.hbase_off;
        const uint32_t yend = U.low_size - U.y0 < p.chunk ? U.low_size : U.y0 + p.chunk;
        for (uint32_t y0 = U.y0; y0 < yend; y0 += 64) {
            const uint32_t y = y0 + lane;
            const bool ok = y < yend;
            const uint32_t yc = ok ? y : yend - 1u;
            const C a = A[U.low_base + yc];
            const double ar = (double)a.x, ai = (double)a.y;
            double accr = 0.0, acci = 0.0;
            // the pass that forms g_{k-1} visits every mode, the others only
            // their block of partials
            const int jlo = p.write_g ? 0 : p.jb;
            const int jhi = p.write_g ? p.m : p.jb + p.jn;
            // four successor modes per step, their loads issued first (modes in
            // ascending order within and across steps, so the sums keep one order)
            for (int j0 = jlo; j0 < jhi; j0 += 4) {
                C sv[4];
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const int j = j0 + d < jhi ? j0 + d : j0;
                    // successor t' + e_j: inside the forward leaf for a low mode,
                    // the aligned block of the high part + e_j otherwise
                    const uint64_t pos = j < (int)U.q ? U.out_base + succ[(size_t)j * U.low_size + yc]
                                                      : hb[j - (int)U.q] + yc;
                    sv[d] = gk[pos];
                }
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const int j = j0 + d;
                    if (j >= jhi) break;
                    const double sr = (double)sv[d].x, si = (double)sv[d].y;
                    const double ur = (double)uc[j].x, ui = (double)uc[j].y;
                    accr += ur * sr - ui * si;
                    acci += ur * si + ui * sr;
                    const int jj = j - p.jb;
                    if (ok && jj >= 0 && jj < p.jn) {
                        // s * conj(a)
                        double2 &pj = part[jj * 64 + lane];
                        pj.x += sr * ar + si * ai;
                        pj.y += si * ar - sr * ai;
                    }
                }
            }
            if (ok && p.write_g) gkm1[U.low_base + y] = C{(T)accr, (T)acci};
        }
        // reduce this unit's partials over lanes in a fixed tree
        __syncthreads();
        for (int j = 0; j < p.jn; ++j) {
            double2 v = part[j * 64 + lane];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                v.x += __shfl_xor(v.x, off, 64);
                v.y += __shfl_xor(v.y, off, 64);
            }
            if (lane == 0) ((double2 *)p.partials)[u * (uint64_t)p.m + p.jb + j] = v;
        }
        __syncthreads();
    }
}

// One launch after all reverse layers: for every layer k, colsum_k[j] = sum over
// the layer's units u of partials_k[u][j], formed by one wave in a fixed order
// (per lane over u = lane, lane + 64, ..., then a butterfly over the 64 lanes;
// wave w takes layers w, w + 4, ...), then G_U[j, i] = sum over layers k with
// i_k = i of colsum_k[j], in order of k.
template <typename T>
__global__ __launch_bounds__(256) void colsum_gradu_kernel(const double2 *__restrict__ partials, ColsumLayers L,
                                                            const int32_t *__restrict__ photons, int n, int m,
                                                            typename Cb<T>::type *__restrict__ GU,
                                                            uint64_t partials_stride, uint64_t gu_stride)
{
    using C = typename Cb<T>::type;
    __shared__ double2 cs[SLOS_MAX_PHOTONS];
    partials += blockIdx.y * partials_stride;  // instance blockIdx.y (element strides)
    GU += blockIdx.y * gu_stride;
    const int j = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int W = blockDim.x >> 6;
    for (int k = threadIdx.x >> 6; k < n; k += W) {
        const double2 *pk = partials + L.off[k];
        double2 s{0.0, 0.0};
        for (uint64_t u = (uint64_t)lane; u < L.nunits[k]; u += 64) {
            const double2 v = pk[u * (uint64_t)m + j];
            s.x += v.x;
            s.y += v.y;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            s.x += __shfl_xor(s.x, off, 64);
            s.y += __shfl_xor(s.y, off, 64);
        }
        if (lane == 0) cs[k] = s;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += blockDim.x) {
        double gr = 0.0, gi = 0.0;
        for (int k = 0; k < n; ++k)
            if (photons[k] == i) {
                gr += cs[k].x;
                gi += cs[k].y;
            }
        GU[(size_t)j * m + i] = C{(T)gr, (T)gi};
    }
}

// The squared-error loss on target outputs of a batch and its gradient with
// respect to the amplitudes.  One workgroup per instance b:
//   L_b = sum_t (|a_b(r_t)|^2 - P_t[b, t])^2 in FP64 (fixed-order sum), and
//   grad_a[b] = 4 (|a_b(r_t)|^2 - P_t[b, t]) a_b(r_t) at r_t, 0 elsewhere
// (the PyTorch-convention gradient d L / d Re a + i d L / d Im a).  The zeros are
// stored and complete before any target value is written to the same row.
template <typename T>
__global__ __launch_bounds__(256) void sq_loss_kernel(const typename Cb<T>::type *__restrict__ a, uint64_t M,
                                                       const int64_t *__restrict__ ranks, int64_t count,
                                                       const double *__restrict__ p_target,
                                                       typename Cb<T>::type *__restrict__ grad_a,
                                                       double *__restrict__ loss)
{
    using C = typename Cb<T>::type;
    __shared__ double sh[256];
    const uint64_t b = blockIdx.x;
    a += b * M;
    grad_a += b * M;
    p_target += b * (uint64_t)count;
    for (uint64_t r = threadIdx.x; r < M; r += 256) grad_a[r] = C{(T)0, (T)0};
    __builtin_amdgcn_s_waitcnt(0);  // this wave's zeros have reached memory
    __syncthreads();
    double s = 0.0;
    for (int64_t t = threadIdx.x; t < count; t += 256) {
        const int64_t r = ranks[t];
        if (r < 0 || (uint64_t)r >= M) continue;  // outside the output set: ignored
        const C v = a[r];
        const double P = (double)v.x * (double)v.x + (double)v.y * (double)v.y;
        const double d = P - p_target[t];
        s += d * d;
        const T f = (T)(4.0 * d);
        grad_a[r] = C{f * v.x, f * v.y};
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0 && loss) loss[b] = sh[0];
}

// The same loss with the seed of the adjoint fused in: g_n[b] = c_S grad_a[b]
// at the targets (c_S = scale[t], the normalisation a(S) = c_S A_n[S]) and 0
// elsewhere, written straight into the last layer's gradient buffer (row b at
// b * gn_stride).  Workgroup (x, b) owns states [x * SLOS_SEED_SLICE, ...) of
// row b: it zeroes them, then writes the targets among them; workgroup 0 of
// the row also forms the loss over all targets.  The values are formed
// exactly as the loss kernel and the seed kernel form them one after the
// other, and the loss in the same order, so the results are the same.
#define SLOS_SEED_SLICE 2048u
template <typename T>
__global__ __launch_bounds__(256) void sq_loss_seed_kernel(const typename Cb<T>::type *__restrict__ a, uint64_t M,
                                                            const int64_t *__restrict__ ranks,
                                                            const double *__restrict__ scale, int64_t count,
                                                            const double *__restrict__ p_target,
                                                            typename Cb<T>::type *__restrict__ gn,
                                                            uint64_t gn_stride, double *__restrict__ loss)
{
    using C = typename Cb<T>::type;
    __shared__ double sh[256];
    const uint64_t b = blockIdx.y;
    a += b * M;
    gn += b * gn_stride;
    p_target += b * (uint64_t)count;
    const uint64_t lo = (uint64_t)blockIdx.x * SLOS_SEED_SLICE;
    const uint64_t hi = lo + SLOS_SEED_SLICE < M ? lo + SLOS_SEED_SLICE : M;
    for (uint64_t r = lo + threadIdx.x; r < hi; r += 256) gn[r] = C{(T)0, (T)0};
    __builtin_amdgcn_s_waitcnt(0);  // this wave's zeros have reached memory
    __syncthreads();
    double s = 0.0;
    for (int64_t t = threadIdx.x; t < count; t += 256) {
        const int64_t r = ranks[t];
        if (r < 0 || (uint64_t)r >= M) continue;  // outside the output set: ignored
        const bool mine = (uint64_t)r >= lo && (uint64_t)r < hi;
        if (!mine && blockIdx.x != 0) continue;
        const C v = a[r];
        const double P = (double)v.x * (double)v.x + (double)v.y * (double)v.y;
        const double d = P - p_target[t];
        s += d * d;
        if (mine) {
            const T f = (T)(4.0 * d);
            const C ga{f * v.x, f * v.y};
            const double c = scale[t];
            gn[r] = C{(T)(c * (double)ga.x), (T)(c * (double)ga.y)};
        }
    }
    if (blockIdx.x != 0) return;
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0 && loss) loss[b] = sh[0];
}

// ---- rectangular MZI mesh --------------------------------------------------------
// MZI(a, b) = PS_1(b) BS PS_0(a) BS with BS = [[c, i s], [i s, c]] at theta = pi/2
// (Eq. eq:bs): the composition BS, PS(phi_a) on mode 0, BS, PS(phi_b) on mode 1.
// Column c holds MZIs on (p, p+1), p = c mod 2, c mod 2 + 2, ..., p + 1 < m, in
// this order; U = T_last ... T_first.
struct Cd {
    double x, y;
};
__device__ __forceinline__ Cd cmul(Cd a, Cd b) { return Cd{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ __forceinline__ Cd cadd(Cd a, Cd b) { return Cd{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ Cd cconj(Cd a) { return Cd{a.x, -a.y}; }

// MZI block B = diag(1, e^{ib}) M, M = BS PS_0(a) BS = 1/2 [[e^{ia} - 1, i (e^{ia} + 1)],
// [i (e^{ia} + 1), 1 - e^{ia}]], row-major in v[0..3], with e^{ib} in v[4].
struct MziBlock {
    Cd v[5];
};
__device__ __forceinline__ MziBlock mzi_block(Cd ea, Cd eb)
{
    MziBlock b;
    b.v[0] = Cd{0.5 * (ea.x - 1.0), 0.5 * ea.y};
    b.v[1] = Cd{-0.5 * ea.y, 0.5 * (ea.x + 1.0)};
    b.v[2] = cmul(eb, b.v[1]);
    b.v[3] = cmul(eb, Cd{0.5 * (1.0 - ea.x), -0.5 * ea.y});
    b.v[4] = eb;
    return b;
}

__device__ __forceinline__ Cd cexp_i(double a)
{
    double s, c;
    sincos(a, &s, &c);
    return Cd{c, s};
}

// The MZI blocks of one phase set, prepared by all threads before the sweep as
// far as LDS reaches: whole blocks, else the phase factors e^{i phi}, else
// nothing (sincos on the sweep's chain).
enum MeshStage { kMeshNone = 0, kMeshFactors = 1, kMeshBlocks = 2 };
template <int STAGE> struct MeshBlocks {
    const double *ph;
    Cd *lds;
    __device__ void prepare(int nmzi, int tid, int nt)
    {
        if constexpr (STAGE == kMeshBlocks) {
            for (int k = tid; k < nmzi; k += nt)
                ((MziBlock *)lds)[k] = mzi_block(cexp_i(ph[2 * k]), cexp_i(ph[2 * k + 1]));
        } else if constexpr (STAGE == kMeshFactors) {
            for (int i = tid; i < 2 * nmzi; i += nt) lds[i] = cexp_i(ph[i]);
        }
    }
    __device__ __forceinline__ MziBlock block(int k) const
    {
        if constexpr (STAGE == kMeshBlocks) return ((const MziBlock *)lds)[k];
        else if constexpr (STAGE == kMeshFactors) return mzi_block(lds[2 * k], lds[2 * k + 1]);
        else return mzi_block(cexp_i(ph[2 * k]), cexp_i(ph[2 * k + 1]));
    }
};

// One workgroup per phase set (m <= 64).  Matrix columns are independent, so
// each wave takes cw of them through the whole mesh by itself, in its own part
// of LDS: no barrier inside the sweep.  The MZIs of one mesh column act on
// disjoint row pairs, so the wave applies (and differentiates) a whole mesh
// column per step: lane l serves MZI i = l / gc on its wave's matrix columns
// l % gc, l % gc + gc, .., with gc = 64 / (most MZIs in a column) rounded down
// to a power of two (8 at m = 12).
struct MeshLanes {
    int gc, waves, cw;
};
__host__ __device__ inline MeshLanes mesh_lanes(int m, int max_waves)
{
    const int most = m / 2 > 0 ? m / 2 : 1;
    MeshLanes l{1, 1, m};
    while (l.gc * 2 * most <= 64) l.gc *= 2;
    l.waves = (m + l.gc - 1) / l.gc;
    if (l.waves > max_waves) l.waves = max_waves;
    l.cw = (m + l.waves - 1) / l.waves;
    return l;
}

// Every lane's LDS accesses of a step are done before the next step's: a wave
// runs its LDS instructions in order, the fence keeps the compiler to it.
__device__ __forceinline__ void wave_step()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// X <- T X, one mesh column
__device__ __forceinline__ void mesh_apply(Cd *X, const MziBlock &B, int p0, int cw, int nc, int g, int gc)
{
    for (int c = g; c < nc; c += gc) {
        const Cd x0 = X[p0 * cw + c], x1 = X[(p0 + 1) * cw + c];
        X[p0 * cw + c] = cadd(cmul(B.v[0], x0), cmul(B.v[1], x1));
        X[(p0 + 1) * cw + c] = cadd(cmul(B.v[2], x0), cmul(B.v[3], x1));
    }
}

// The whole mesh on this wave's columns of X.  A prepared block is read while the
// step before still computes; one that is formed here is formed in its own step.
template <int STAGE>
__device__ __forceinline__ void mesh_forward_sweep(Cd *X, const MeshBlocks<STAGE> &mb, int m, int nmzi, int i, int cw,
                                                   int nc, int g, int gc)
{
    int k0 = 0;
    MziBlock B;
    if constexpr (STAGE == kMeshBlocks) B = mb.block(min(i, nmzi - 1));
    for (int col = 0; col < m; ++col) {
        const int cnt = (m - col % 2) / 2;
        MziBlock nb;
        if constexpr (STAGE == kMeshBlocks) nb = mb.block(min(k0 + cnt + i, nmzi - 1));
        if (i < cnt) {
            if constexpr (STAGE != kMeshBlocks) B = mb.block(k0 + i);
            mesh_apply(X, B, col % 2 + 2 * i, cw, nc, g, gc);
        }
        k0 += cnt;
        if constexpr (STAGE == kMeshBlocks) B = nb;
        wave_step();
    }
}

template <typename T, int STAGE>
__global__ __launch_bounds__(1024) void mesh_forward_kernel(int m, int nmzi, const double *__restrict__ phases,
                                                            typename Cb<T>::type *__restrict__ Uout, MeshLanes ml)
{
    using C = typename Cb<T>::type;
    extern __shared__ Cd Ush[];  // per wave m x cw, then the prepared blocks
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    MeshBlocks<STAGE> mb{phases + (size_t)b * 2 * nmzi, Ush + ml.waves * m * ml.cw};
    mb.prepare(nmzi, tid, blockDim.x);
    const int gc = ml.gc, cw = ml.cw, i = lane / gc, g = lane % gc;
    const int c0 = wv * cw, nc = min(cw, m - c0);  // this wave's matrix columns (none if nc <= 0)
    Cd *X = Ush + wv * m * cw;
    for (int e = lane; e < m * cw; e += 64) X[e] = Cd{e / cw == c0 + e % cw ? 1.0 : 0.0, 0.0};
    __syncthreads();
    mesh_forward_sweep(X, mb, m, nmzi, i, cw, nc, g, gc);
    for (int e = lane; e < m * cw; e += 64) {
        const int r = e / cw, c = e % cw;
        if (c < nc) Uout[((size_t)b * m + r) * m + c0 + c] = C{(T)X[e].x, (T)X[e].y};
    }
}

// Reverse sweep: with U = L_k T_k R_k, P = L_k^H G_U and Q = L_k^H U = T_k R_k,
//   dL/dphi = Re sum conj(P) o (dT_k T_k^H Q),
// then P <- T_k^H P and Q <- T_k^H Q move to the previous column (the MZIs of a
// column commute, so they share P and Q).  On the MZI's rows, with BS unitary,
//   dT/da T^H = 1/2 [[i, e^{-ib}], [-e^{ib}, i]],   dT/db T^H = diag(0, i),
// so a matrix column (p0, p1), (q0, q1) contributes
//   a: 1/2 [-Im(p0* q0 + p1* q1) + Re(e^{-ib} p0* q1 - e^{ib} p1* q0)],  b: -Im(p1* q1).
// Each MZI's sum is over its gc lanes, then over the waves, in a fixed order:
// after the sweep, from one term per lane in LDS where they fit (lane_sums), so
// that no cross-lane move is on the sweep's chain.
// m=12, 64 phase sets: bound by the chain of 2 m steps of LDS reads, complex
// products and LDS writes; with one wave on all matrix columns, a barrier per
// step, and the 2x2 derivative products formed in full it took 20 us.
template <typename T, int STAGE>
__global__ __launch_bounds__(1024) void mesh_backward_kernel(int m, int nmzi, const double *__restrict__ phases,
                                                             const typename Cb<T>::type *__restrict__ GU,
                                                             double *__restrict__ gphases, MeshLanes ml, int lane_sums)
{
    extern __shared__ Cd sh[];  // per wave P and Q (m x cw each), the prepared blocks, the waves' sums
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int gc = ml.gc, cw = ml.cw, W = ml.waves, i = lane / gc, g = lane % gc;
    Cd *blocks = sh + 2 * W * m * cw;
    MeshBlocks<STAGE> mb{phases + (size_t)b * 2 * nmzi, blocks};
    double *part = (double *)(blocks + (STAGE == kMeshBlocks ? 5 * nmzi : STAGE == kMeshFactors ? 2 * nmzi : 0));
    mb.prepare(nmzi, tid, blockDim.x);
    const int c0 = wv * cw, nc = min(cw, m - c0);
    Cd *P = sh + wv * 2 * m * cw, *Q = P + m * cw;
    // Q = U (rebuilt here), P = G_U
    for (int e = lane; e < m * cw; e += 64) {
        const int r = e / cw, c = e % cw;
        Q[e] = Cd{r == c0 + c ? 1.0 : 0.0, 0.0};
        Cd v{0.0, 0.0};
        if (c < nc) {
            const auto u = GU[((size_t)b * m + r) * m + c0 + c];
            v = Cd{(double)u.x, (double)u.y};
        }
        P[e] = v;
    }
    __syncthreads();
    mesh_forward_sweep(Q, mb, m, nmzi, i, cw, nc, g, gc);
    int k0 = nmzi;
    MziBlock B;
    if constexpr (STAGE == kMeshBlocks) B = mb.block(min(nmzi - (m - (m - 1) % 2) / 2 + i, nmzi - 1));
    double *out = gphases + (size_t)b * 2 * nmzi;
    // columns in reverse
    for (int col = m - 1; col >= 0; --col) {
        const int cnt = (m - col % 2) / 2;
        k0 -= cnt;
        double va = 0.0, vb = 0.0;
        MziBlock nb;
        if constexpr (STAGE == kMeshBlocks) nb = mb.block(max(k0 - (m - (col + 1) % 2) / 2 + i, 0) % nmzi);
        if (i < cnt) {
            if constexpr (STAGE != kMeshBlocks) B = mb.block(k0 + i);
            const int p0 = col % 2 + 2 * i;
            const Cd eb = B.v[4], h0 = cconj(B.v[0]), h1 = cconj(B.v[1]), h2 = cconj(B.v[2]), h3 = cconj(B.v[3]);
            for (int c = g; c < nc; c += gc) {
                const Cd q0 = Q[p0 * cw + c], q1 = Q[(p0 + 1) * cw + c];
                const Cd x0 = P[p0 * cw + c], x1 = P[(p0 + 1) * cw + c];
                const double i0 = x0.x * q0.y - x0.y * q0.x, i1 = x1.x * q1.y - x1.y * q1.x;
                const double re = (x0.x * q1.x + x0.y * q1.y) - (x1.x * q0.x + x1.y * q0.y);
                const double im = (x0.x * q1.y - x0.y * q1.x) + (x1.x * q0.y - x1.y * q0.x);
                va += 0.5 * ((eb.x * re + eb.y * im) - (i0 + i1));
                vb -= i1;
                // P <- T^H P, Q <- T^H Q on rows p0, p0+1
                Q[p0 * cw + c] = cadd(cmul(h0, q0), cmul(h2, q1));
                Q[(p0 + 1) * cw + c] = cadd(cmul(h1, q0), cmul(h3, q1));
                P[p0 * cw + c] = cadd(cmul(h0, x0), cmul(h2, x1));
                P[(p0 + 1) * cw + c] = cadd(cmul(h1, x0), cmul(h3, x1));
            }
        }
        if (lane_sums) {
            // one term per lane, added after the sweep
            if (i < cnt) ((double2 *)part)[(size_t)(wv * gc + g) * nmzi + k0 + i] = double2{va, vb};
        } else {
            // sum over the gc lanes of each MZI (aligned groups of a power of two)
            for (int o = gc / 2; o > 0; o >>= 1) {
                va += __shfl_xor(va, o, 64);
                vb += __shfl_xor(vb, o, 64);
            }
            if (i < cnt && g == 0) {
                double *to = W > 1 ? part + (size_t)wv * 2 * nmzi : out;
                to[2 * (k0 + i)] = va;
                to[2 * (k0 + i) + 1] = vb;
            }
        }
        if constexpr (STAGE == kMeshBlocks) B = nb;
        wave_step();
    }
    const int rows = lane_sums ? W * gc : W;
    if (rows > 1) {
        __syncthreads();
        for (int e = tid; e < 2 * nmzi; e += blockDim.x) {
            double s = part[e];
            for (int w = 1; w < rows; ++w) s += part[(size_t)w * 2 * nmzi + e];
            out[e] = s;
        }
    }
}

} // namespace

int slos_launch_seed(const void *heads, uint64_t nleaves, uint32_t stride, const double *lowfac, const void *ga,
                     void *gn, int c64, void *stream, int batch, uint64_t ga_stride, uint64_t gn_stride)
{
    const int grid = (int)(nleaves < 1024 ? (nleaves + 3) / 4 : 256);
    const dim3 g(grid > 0 ? grid : 1, batch > 1 ? batch : 1);
    if (c64)
        hipLaunchKernelGGL(seed_kernel<float>, g, dim3(256), 0, (hipStream_t)stream, (const LeafDescHead *)heads,
                           nleaves, stride, lowfac, (const float2 *)ga, (float2 *)gn, ga_stride, gn_stride);
    else
        hipLaunchKernelGGL(seed_kernel<double>, g, dim3(256), 0, (hipStream_t)stream, (const LeafDescHead *)heads,
                           nleaves, stride, lowfac, (const double2 *)ga, (double2 *)gn, ga_stride, gn_stride);
    return (int)hipGetLastError();
}

// raise the dynamic-LDS limit of a kernel once per process
template <typename K>
static hipError_t allow_lds(K kernel, bool &done)
{
    if (done) return hipSuccess;
    hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)SLOS_LDS_DYNAMIC_MAX);
    if (e == hipSuccess) done = true;
    return e;
}

int slos_launch_bwd_layer(const BwdParams &p, int c64, int grid, void *stream, int batch)
{
    if (p.flat) return slos_launch_flat_bwd(*p.flat, c64, batch, stream);
    static bool a32 = false, a64 = false;
    hipError_t e = c64 ? allow_lds(bwd_layer_kernel<float>, a32) : allow_lds(bwd_layer_kernel<double>, a64);
    if (e != hipSuccess) return (int)e;
    const size_t lds = (size_t)p.jn * 64 * sizeof(double2);
    const dim3 g(grid, batch > 1 ? batch : 1);
    if (c64)
        hipLaunchKernelGGL(bwd_layer_kernel<float>, g, dim3(64), lds, (hipStream_t)stream, p);
    else
        hipLaunchKernelGGL(bwd_layer_kernel<double>, g, dim3(64), lds, (hipStream_t)stream, p);
    return (int)hipGetLastError();
}

int slos_launch_colsum_gradu(const void *partials, const ColsumLayers &L, const int32_t *photons, int n, int m,
                             void *GU, int c64, void *stream, int batch, uint64_t partials_stride, uint64_t gu_stride)
{
    const dim3 g(m, batch > 1 ? batch : 1);
    if (c64)
        hipLaunchKernelGGL(colsum_gradu_kernel<float>, g, dim3(256), 0, (hipStream_t)stream, (const double2 *)partials,
                           L, photons, n, m, (float2 *)GU, partials_stride, gu_stride);
    else
        hipLaunchKernelGGL(colsum_gradu_kernel<double>, g, dim3(256), 0, (hipStream_t)stream,
                           (const double2 *)partials, L, photons, n, m, (double2 *)GU, partials_stride, gu_stride);
    return (int)hipGetLastError();
}

int slos_launch_sq_loss_seed(const void *a, uint64_t M, const int64_t *ranks, const double *scale, int64_t count,
                             const double *p_target, void *gn, uint64_t gn_stride, double *loss, int batch, int c64,
                             void *stream)
{
    const dim3 g((unsigned)((M + SLOS_SEED_SLICE - 1) / SLOS_SEED_SLICE), (unsigned)batch);
    if (c64)
        hipLaunchKernelGGL(sq_loss_seed_kernel<float>, g, dim3(256), 0, (hipStream_t)stream, (const float2 *)a, M,
                           ranks, scale, count, p_target, (float2 *)gn, gn_stride, loss);
    else
        hipLaunchKernelGGL(sq_loss_seed_kernel<double>, g, dim3(256), 0, (hipStream_t)stream, (const double2 *)a, M,
                           ranks, scale, count, p_target, (double2 *)gn, gn_stride, loss);
    return (int)hipGetLastError();
}

int slos_launch_sq_loss(const void *a, uint64_t M, const int64_t *ranks, int64_t count, const double *p_target,
                        void *grad_a, double *loss, int batch, int c64, void *stream)
{
    if (c64)
        hipLaunchKernelGGL(sq_loss_kernel<float>, dim3(batch), dim3(256), 0, (hipStream_t)stream, (const float2 *)a, M,
                           ranks, count, p_target, (float2 *)grad_a, loss);
    else
        hipLaunchKernelGGL(sq_loss_kernel<double>, dim3(batch), dim3(256), 0, (hipStream_t)stream,
                           (const double2 *)a, M, ranks, count, p_target, (double2 *)grad_a, loss);
    return (int)hipGetLastError();
}

// What the mesh kernels keep in LDS: the waves' matrices (mats of m x cw), the
// blocks or factors prepared ahead, and the waves' sums; fewer waves, then less
// prepared, where that does not fit.
//
// That is the shape for the shortest chain.  Many sets are bound by issue and by how
// many of them LDS holds instead: they get factors alone, no term per lane, and few
// waves (each with most of its lanes at work).  Forward from 1024 sets on (four to a
// compute unit) and up to 40 modes (48: 445 us for 2048, 798 so); the adjoint where
// the sets are more than LDS holds at a time and that is fewer than 16 to a unit.
// 16,384 sets, us forward and adjoint in the shape for few and so: m=12 71 and 219, 52
// and 162; m=16 100 and 426, 80 and 240; m=24 556 and 2032, 360 and 1177; m=32
// 1128 and 3975, 951 and 2983.  m=8, whose adjoint LDS holds 20 times: 67, 76 so.
struct MeshShape {
    MeshLanes ml;
    int stage;
    int lane_sums;
    size_t lds;
};
static MeshShape mesh_shape(int m, int nmzi, int mats, bool sums, int batch)
{
    MeshShape s{};
    bool many = !sums && m <= 40 && batch >= 1024;
    if (sums) {
        // the mesh adjoint with a term per lane, all blocks prepared
        s.ml = mesh_lanes(m, 16);
        if (s.ml.gc > s.ml.cw) s.ml.gc = s.ml.cw;  // idle lanes add nothing: no terms for them
        s.stage = kMeshBlocks;
        s.lane_sums = s.ml.waves * s.ml.gc > 1;
        s.lds = ((size_t)mats * s.ml.waves * m * s.ml.cw + 5 * (size_t)nmzi) * sizeof(Cd) +
                (size_t)s.ml.waves * s.ml.gc * nmzi * 2 * sizeof(double);
        const size_t fit = SLOS_LDS_DYNAMIC_MAX / s.lds;
        many = fit < 16 && (size_t)batch > 256 * fit;
        if (s.lane_sums && fit > 0 && !many) return s;
        s.lane_sums = 0;
    }
    const int most = many ? m <= 18 ? 1 : m < 24 ? 2 : 4 : 16;
    for (int waves = most; waves >= 1; waves /= 2) {
        s.ml = mesh_lanes(m, waves);
        const size_t mat = (size_t)mats * s.ml.waves * m * s.ml.cw * sizeof(Cd);
        const size_t part = sums && s.ml.waves > 1 ? (size_t)s.ml.waves * 2 * nmzi * sizeof(double) : 0;
        for (s.stage = many ? kMeshFactors : kMeshBlocks; s.stage >= kMeshNone; --s.stage) {
            const int per = s.stage == kMeshBlocks ? 5 : s.stage == kMeshFactors ? 2 : 0;
            s.lds = mat + part + (size_t)per * nmzi * sizeof(Cd);
            // sincos on the chain only where one wave's matrices leave no room
            if (s.lds <= SLOS_LDS_DYNAMIC_MAX && (s.stage > kMeshNone || waves == 1)) return s;
        }
    }
    s.stage = kMeshNone;
    return s;
}

template <typename T, int STAGE>
static hipError_t mesh_forward(const MeshShape &sh, int m, int batch, const double *phases, void *U, hipStream_t s)
{
    static bool done = false;
    hipError_t e = allow_lds(mesh_forward_kernel<T, STAGE>, done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((mesh_forward_kernel<T, STAGE>), dim3(batch), dim3(64 * sh.ml.waves), sh.lds, s, m, m * (m - 1) / 2,
                       phases, (typename Cb<T>::type *)U, sh.ml);
    return hipGetLastError();
}
template <typename T, int STAGE>
static hipError_t mesh_backward(const MeshShape &sh, int m, int batch, const double *phases, const void *GU, double *gphases,
                                hipStream_t s)
{
    static bool done = false;
    hipError_t e = allow_lds(mesh_backward_kernel<T, STAGE>, done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((mesh_backward_kernel<T, STAGE>), dim3(batch), dim3(64 * sh.ml.waves), sh.lds, s, m, m * (m - 1) / 2,
                       phases, (const typename Cb<T>::type *)GU, gphases, sh.ml, sh.lane_sums);
    return hipGetLastError();
}

// f(STAGE as an integral constant)
template <typename F> static hipError_t with_stage(int stage, F &&f)
{
    if (stage == kMeshBlocks) return f(std::integral_constant<int, kMeshBlocks>{});
    if (stage == kMeshFactors) return f(std::integral_constant<int, kMeshFactors>{});
    return f(std::integral_constant<int, kMeshNone>{});
}

int slos_launch_mesh_forward(int m, int batch, const double *phases, void *U, int c64, void *stream)
{
    const MeshShape sh = mesh_shape(m, m * (m - 1) / 2, 1, false, batch);
    const hipStream_t s = (hipStream_t)stream;
    return (int)with_stage(sh.stage, [&](auto st) {
        constexpr int ST = decltype(st)::value;
        return c64 ? mesh_forward<float, ST>(sh, m, batch, phases, U, s) : mesh_forward<double, ST>(sh, m, batch, phases, U, s);
    });
}

int slos_launch_mesh_backward(int m, int batch, const double *phases, const void *GU, double *gphases, int c64,
                              void *stream)
{
    const MeshShape sh = mesh_shape(m, m * (m - 1) / 2, 2, true, batch);
    const hipStream_t s = (hipStream_t)stream;
    return (int)with_stage(sh.stage, [&](auto st) {
        constexpr int ST = decltype(st)::value;
        return c64 ? mesh_backward<float, ST>(sh, m, batch, phases, GU, gphases, s)
                   : mesh_backward<double, ST>(sh, m, batch, phases, GU, gphases, s);
    });
}
