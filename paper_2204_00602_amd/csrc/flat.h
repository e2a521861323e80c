// Table-driven layers (flat.hip): the layers small enough that each state's
// predecessor ranks are kept as a table.  Not part of the public ABI.
#pragma once

#include "slos_internal.h"

#if defined(__HIPCC__)
#define SLOS_HD __host__ __device__
#else
#define SLOS_HD
#endif

// Table entries are (mode << 24) | rank.  A padded entry names mode m, whose
// coefficient is held at zero, and the state after the last of layer k - 1,
// taken as zero: it adds nothing, whatever the layer's values are.
#define SLOS_FLAT_PAD(m, Nprev) ((uint32_t)(m) << 24 | (uint32_t)(Nprev))
// Layers of at most this many states are table-driven.  Measured on one layer
// (microseconds, tiled against table-driven): 657,800 states 27 against 11
// (c64), 1,081,575 31 against 15 (c64) and 37 against 18 (c128), 2,220,075 38
// against 24 and 53 against 31, 3,124,550 55 against 42 and 78 against 53;
// 4,686,825 66 against 70 (c64; c128 99 against 84, but its table alone is
// 170 MB), 6,906,900 83 against 100.  The line holds for several instances as for
// one (whole calls, c64, 8 and 64 instances of 3,124,550 states in the last layer:
// 686 against 397 and 5143 against 2976).  Also keeps every rank within 24 bits.
#define SLOS_FLAT_MAX_STATES 3200000u
// Entries of a plan's successor tables: 512 MiB, as the tables of a batch (by the
// line above its predecessor tables have at most 410 MiB).
#define SLOS_FLAT_MAX_SUCC (uint64_t(1) << 27)
// Largest layer that every workgroup of the first launch computes for itself,
// and the LDS its two layers may take.  One instance: m=13, n=6 (6,188 states
// in layer 5) 12.1 us a pass with that layer in the first launch, 15.6 without;
// ten instances at m=15, n=6 (11,628 states) 24.9 us with, 16.0 without, the
// workgroups then outnumbering the CUs.
#define SLOS_HEAD_MAX_STATES 12288u
#define SLOS_HEAD_MAX_STATES_MANY 6144u
#define SLOS_HEAD_LDS_MAX (144u * 1024u)
// Workgroups of that launch: one output of its last layer per thread for one
// instance; several instances share 256 in all, one per CU (64 instances at
// m=12, n=6: 13.6 us, against 20.4 with 512 and 63 with 1024).
#define SLOS_HEAD_MAX_GROUPS 512
#define SLOS_HEAD_MAX_GROUPS_MANY 256
#define SLOS_FLAT_THREADS 256
#define SLOS_FLAT_VMAX 256u             // slots of a table-driven layer's recorded maximum

// Layers 1..h+1 in one launch: 1..h in LDS by every workgroup, h+1 to Y.
struct HeadParams {
    const void *U;
    void *Y;                     // layer h + 1
    void *keep;                  // kept layers 1..h are stored here too, or NULL
    const uint32_t *pred;
    const double *scale;         // normalisation of every output when h + 1 is the last layer
    double *partials;            // one FP64 partial of sum P per workgroup
    double *sum_p;               // the sum itself, by one workgroup or with `count`; or NULL
    uint32_t *count;             // zero: the last workgroup to end sums the partials; or NULL
    uint32_t *zero;              // words the later launches of the pass need cleared
    float *vm;                   // per workgroup: max |Re| + |Im| over its part of layer h + 1, or NULL
    uint64_t u_stride, y_stride, keep_stride;             // bytes per instance (blockIdx.y)
    uint64_t partials_stride, zero_stride, vm_stride, count_stride;  // elements per instance
    uint64_t keep_off[SLOS_MAX_PHOTONS + 1];              // bytes
    uint64_t off[SLOS_MAX_PHOTONS + 1];                   // layer k's table, in entries
    uint32_t N[SLOS_MAX_PHOTONS + 1];
    uint32_t cap[2];             // elements of the even and the odd LDS buffer (a zero follows each layer)
    uint32_t nzero;
    int m, h;
    int comp_from;               // first compensated layer
    uint8_t col[SLOS_MAX_PHOTONS + 1];
};

// One layer, one output per thread.
struct FlatParams {
    const void *X;
    void *Y;
    const void *U;
    const uint32_t *pred;        // this layer's table, term-major
    const double *scale;
    double *partials;            // one FP64 partial of sum P per workgroup
    const uint32_t *vmax_in;     // float bits of the maxima whose largest bounds |Re| + |Im| over X
    uint32_t *vmax_out;          // SLOS_FLAT_VMAX cleared slots for this layer's maximum, or NULL
    uint64_t x_stride, y_stride, u_stride;     // bytes per instance (blockIdx.y)
    uint64_t partials_stride, vin_stride, vout_stride;
    uint32_t nvmax;
    uint32_t N, Nprev, cmax;
    int m, col;
};

// Device-side construction of the tables of layers 1..kf.
struct FlatTables {
    const uint64_t *binom;       // binom[a * bstride + b] = C(a, b)
    int bstride;
    int m, kf;
    uint32_t *pred;
    uint64_t off[SLOS_MAX_PHOTONS + 1];
    uint32_t N[SLOS_MAX_PHOTONS + 1];
    uint32_t leaf_cap[SLOS_MAX_PHOTONS + 1];  // the tiled kernel's leaf size of each layer
    double *scale;               // normalisation of the states of the layers in scale_on (bit k), at scale_off[k]
    uint64_t scale_off[SLOS_MAX_PHOTONS + 1];
    uint64_t scale_on;
    double norm_t;
    uint32_t *succ;              // mode-major: succ[succ_off[k] + j * slos_succ_row + y] = rank of y + e_j
    int kb, kt;                  // layers with a successor table: 1..kb; 1..kt are the tail launch's
    uint64_t succ_off[SLOS_MAX_PHOTONS + 1];
};

// Successor tables: N entries to a mode, N the states of layer k - 1.  In the tail
// launch's layers a column for the states past the end and a row for the modes past
// the last, which hold N_k, the index of the zero behind g_k.
SLOS_HD static inline uint32_t slos_succ_row(uint32_t N, bool tail) { return N + (tail ? 1u : 0u); }
static inline uint64_t slos_succ_entries(uint64_t N, int m, bool tail) { return tail ? (N + 1) * (m + 1) : N * m; }

struct FlatLaunch {
    const HeadParams *head;      // exactly one of the three is set
    const FlatParams *flat;
    const FlatTables *tables;
    int c64, mode, compensated;
    int batch;
    int grid;                    // head: workgroups per instance
    int threads;                 // head: workgroup size
};
int slos_launch_flat(const FlatLaunch &l, void *stream);

// ---- batches of table-driven instances (flat_batch.hip) --------------------------

#define SLOS_FB_THREADS 1024
#define SLOS_FB_GRID 256          // workgroups: one per CU
#define SLOS_FB_WAVES (SLOS_FB_THREADS / 64)
#define SLOS_FB_MAX_ENTRIES (uint64_t(1) << 27)  // 512 MiB of tables
#define SLOS_FB_MAX_PARTS 16
// Cycles of a compute unit that the host deals instances out by, per state and
// entry of its table unless said otherwise, c64 / c128.  Fitted to 256 equal
// instances of 12 types from (8, 6) to (14, 7) on workgroups, and to 4096 of
// (6, 3) .. (10, 4) on waves.
#define SLOS_FB_WG_CYCLES(c64) ((c64) ? 0.234 : 0.4)      // workgroup, layer read from LDS
#define SLOS_FB_BLOCK_CYCLES(c64) ((c64) ? 0.5 : 0.9)     // workgroup, layer staged in blocks
#define SLOS_FB_LAYER_CYCLES(c64) ((c64) ? 2850.0 : 4500.0)  // workgroup, per layer
#define SLOS_FB_WAVE_CYCLES(c64) ((c64) ? 4.66 : 8.0)     // wave among sixteen busy ones
#define SLOS_FB_WAVE_LAYER_CYCLES(c64) ((c64) ? 1700.0 : 2500.0)

// The tables of one mode count.
struct FlatModes {
    uint64_t off[SLOS_BATCH_MAX_N + 1];        // layer k's predecessor table, in entries
    uint64_t scale_off[SLOS_BATCH_MAX_N + 1];  // sqrt(prod s_j!) of its states, where some instance ends there
    uint32_t N[SLOS_BATCH_MAX_N + 1];
    uint32_t m;
};
struct FlatInst {
    uint64_t U_off, out_off;      // elements
    double norm_t;                // 1 / sqrt(prod t_i!)
    uint32_t modes;               // index of its FlatModes
    uint32_t n;
    uint8_t col[SLOS_BATCH_MAX_N];
};
// What a workgroup runs: an instance, or part `part` of `parts` of its last
// layer (with the layers below); the parts' sums of P go to partials[slot ..].
struct FlatItem {
    uint32_t inst, part, parts, slot, count;
};
struct FlatBatchParams {
    const void *U;
    void *out;
    double *sum_p;                // per instance, or NULL
    const FlatInst *inst;
    const FlatModes *modes;
    const uint32_t *pred;
    const double *scale;
    const FlatItem *items;
    double *partials;
    uint32_t *counts;                     // zero between launches
    const uint32_t *wg_start, *wg_list;   // items that a workgroup runs with all its waves, first
    const uint32_t *wv_start, *wv_list;   // then each wave its own
    void *scratch;                // per workgroup two layers of scratch_stride elements, for layers beyond the LDS
    const uint32_t *wg_scr;       // per workgroup: its place in the scratch
    uint64_t scratch_stride;
    const uint64_t *binom;        // binom[a * bstride + b] = C(a, b)
    int bstride;
    uint32_t lds_elems;           // elements of LDS for the layers and U's columns
    uint32_t wave_elems;          // the same of one wave
};
int slos_launch_flat_batch(const FlatBatchParams &p, int c64, int grid, void *stream);

// ---- adjoint of the table-driven layers (flat_bwd.hip) -------------------------

#define SLOS_BWD_LDS_MAX (149u * 1024u)
#define SLOS_BWD_THREADS 512     // of a reverse layer
// Threads of a tail workgroup.  With more instances than compute units
// (SLOS_BWD_TAIL_MANY) small ones leave most of 1024 threads idle while no second
// workgroup fits beside them (128 registers a thread), so those whose LDS lets four
// workgroups share a unit get 256 threads, and those whose layers below the last
// have at most 64 states 64.  Microseconds of slos_backward_many in c64 with 1024, 256 and
// 64 threads, and of the unit kernels: m=6, n=3, 4096 instances 109, 34, 14 and
// 66, 65,535 of them 1780, 487, 166 and 756; m=3, n=2, 65,535: 1264, 349, 108
// and 311; m=10, n=5, 4096: 261, 102 and 332 (256 the most that fits).  One
// instance: m=10, n=5 16.9 with 1024, 17.6 with 256; m=64, n=2 21.5 and 24.9.
#define SLOS_BWD_TAIL_THREADS 1024
#define SLOS_BWD_TAIL_MANY 256
#define SLOS_BWD_TAIL_LDS_256 (40u * 1024u)
#define SLOS_BWD_TAIL_LDS_64 (10u * 1024u)
// Modes whose gradient sums a thread of the tail keeps in registers: the most that
// the 128 registers of four waves a SIMD hold (8: none spilled, 12: 2 to 12, 16: 39 to 49).
#define SLOS_BWD_TAIL_MODES 12

// One reverse layer: g_{k-1} and, per workgroup, the gradient partials of every mode.
struct FlatBwdParams {
    const void *gk;              // g_k, or dL/da with `scale` (then g_n = scale * dL/da)
    const double *scale;
    void *gkm1;
    const void *Akm1;
    const void *U;
    const uint32_t *succ;        // mode-major, N entries per mode
    void *partials;              // double2 [workgroups][m]
    uint64_t gk_stride, gkm1_stride, a_stride, u_stride, partials_stride;  // bytes per instance (blockIdx.y)
    uint32_t N;                  // states of layer k - 1
    int m, col;
};

// Reverse layers t..1 and the assembly of G_U, one workgroup per instance.
struct TailParams {
    const void *gt;              // g_t, or dL/da with `scale`; unused with a loss
    const double *scale;
    const void *keep;            // kept layers
    const void *U;
    void *GU;
    const uint32_t *succ;
    const void *partials;        // of the layers above t: double2 [rows[k]][m] at part_off[k]
    // squared-error loss on target outputs as the source of g_n (t = n), or a = NULL
    const void *a;
    const int64_t *ranks;
    const double *target_scale;
    const double *p_target;
    double *loss;
    int64_t count;
    uint64_t gt_stride, keep_stride, u_stride, gu_stride, partials_stride;  // bytes per instance (blockIdx.x)
    uint64_t a_stride;           // elements
    uint64_t keep_off[SLOS_MAX_PHOTONS + 1];   // bytes
    uint64_t succ_off[SLOS_MAX_PHOTONS + 1];   // entries
    uint64_t part_off[SLOS_MAX_PHOTONS + 1];   // double2
    uint32_t rows[SLOS_MAX_PHOTONS + 1];
    uint32_t N[SLOS_MAX_PHOTONS + 1];
    uint32_t cap[2];             // elements of the even and the odd LDS buffer (a zero follows each layer)
    int m, n, t;
    int threads;                 // of a workgroup: SLOS_BWD_TAIL_THREADS, 256 or 64 (t = n)
    int wave_rows;               // sum of slos_tail_waves over its layers
    uint8_t col[SLOS_MAX_PHOTONS + 1];
};

struct FlatBwdLaunch {
    const FlatBwdParams *layer;  // exactly one is set
    const TailParams *tail;
    int per_thread;              // layer: states per thread (1, 2 or 4)
};
int slos_launch_flat_bwd(const FlatBwdLaunch &l, int c64, int batch, void *stream);

// states of a workgroup of one reverse layer, and LDS bytes of the tail
static inline uint32_t slos_bwd_rows(uint64_t N, int per_thread)
{
    return (uint32_t)((N + (uint64_t)per_thread * SLOS_BWD_THREADS - 1) / ((uint64_t)per_thread * SLOS_BWD_THREADS));
}
// the g buffers hold four layers' partial sums per thread at the end
static inline uint64_t slos_tail_lds(uint64_t cap0, uint64_t cap1, int m, int n, int t, int wave_rows, int threads, uint64_t es)
{
    const uint64_t g = (cap0 + cap1) * es, red = t < n ? 4u * (uint64_t)threads * 16u : 0u;
    return (g > red ? g : red) + 16u * ((uint64_t)t * (m + 16) + (uint64_t)(n + 1 + wave_rows) * m);
}
// waves of the tail (of `threads` threads) that have a state of a layer of N states: four
// lanes a state up to as many states as threads, else one
SLOS_HD static inline int slos_tail_waves(uint32_t N, uint32_t threads)
{
    const uint32_t w = N <= threads ? (N + 15u) / 16u : threads / 64u;
    return (int)(w < threads / 64u ? w : threads / 64u);
}
