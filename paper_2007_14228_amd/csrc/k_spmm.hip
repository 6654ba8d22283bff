// Sparse products on the shared P1 CSR pattern.
//
//  k_spmm_pair   : Y1 = A1 X and Y2 = A2 X in one pass (H X and B X, the
//                  "function evaluation" of Algorithm PCAL).  The values of the
//                  two matrices are interleaved per nonzero, so one 16-byte
//                  (f64) or 8-byte (f32) load feeds both products; with one
//                  output the caller selects which of the pair is used.
//  k_spmm_shift  : Q[:,l] = (L/2 - lam_l B) D[:,l] (operator of the paper's
//                  preconditioner T_l, eq. precondition-T); for a step of its
//                  CG with the per-column dot products <D_l, Q_l> and <Q_l, J Q_l>.
//  k_cg_iter     : one Hartree CG iteration (one vector, FP64), and
//  k_spmv_dot    : q = A d and <d, q> for that of scattered numberings.
//
// Work mapping (wave64).  A row is owned by a group of LPR = 2^lpr_log2 lanes;
// each lane covers V consecutive columns (one vector load of an X row slice)
// and CH column chunks when p > LPR*V.  A row's p values are contiguous, so a
// group reads one contiguous X row per nonzero (p = 128 in f64: 1 KB per
// neighbour per wave).
//
// Latency: the neighbours of a row are independent, so the group first loads
// up to LPR (column, weight) pairs with one coalesced access, then broadcasts
// them lane to lane and issues U neighbour loads back to back before any
// arithmetic.  Control flow around the broadcasts is uniform across the wave
// (loop bounds use the wave's longest row; rows past n just have no entries).
#include <algorithm>

#include "common.hpp"
#include "cg_report.hpp"
#include "cg_step.hpp"

// Tuning: neighbour loads in flight per wave for one-column-chunk rows, and
// whether streamed data (CSR entries read once, outputs written once) use
// non-temporal accesses so that they do not evict reused X rows from L2.
#ifndef OFKS_SPMM_U
#define OFKS_SPMM_U 16
#endif
#ifndef OFKS_SPMM_NT
#define OFKS_SPMM_NT 1
#endif

namespace ofks {

template <typename T> __device__ __forceinline__ T stream_load(const T *p) {
#if OFKS_SPMM_NT
    return __builtin_nontemporal_load(p);
#else
    return *p;
#endif
}

template <typename T, int V>
__device__ __forceinline__ void stream_store_vec(T *__restrict__ p, const T (&in)[V]) {
#if OFKS_SPMM_NT
#pragma unroll
    for (int i = 0; i < V; ++i) __builtin_nontemporal_store(in[i], p + i);
#else
    store_vec<T, V>(p, in);
#endif
}

// What the shifted product forms from q = (A1 - lam_c A2) d on the active
// columns (zero elsewhere): SHIFT writes q; SHIFT_CG writes q and sums <d, q> and
// <q, J q> over the rows of a block (part[block][0..p), [p..2p)), J the inverse
// of the operator's diagonal (lhd - lam_c bd); SHIFT_DOT, the last step of a CG,
// only sums <d, q>.
enum { DUAL = 0, SHIFT = 1, SHIFT_CG = 2, SHIFT_DOT = 3 };

template <typename T> struct pair_t;
template <> struct pair_t<double> { using type = double2; };
template <> struct pair_t<float> { using type = float2; };

__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
    return v;
}

// a1[ch][v] = sum_e w(e).x X[col e][c], a2 likewise with w(e).y, for the row
// owned by this lane group (cnt entries starting at e0; cnt = 0: no row).
// All 64 lanes of the wave must call this together.
template <typename T, int V, int CH, int U>
__device__ __forceinline__ void gather_row(int64_t e0, int cnt, int lpr_log2, int p,
                                           const int32_t *__restrict__ col,
                                           const typename pair_t<T>::type *__restrict__ w,
                                           const T *__restrict__ X, T (&a1)[CH][V], T (&a2)[CH][V]) {
    using P2 = typename pair_t<T>::type;
    const int lpr = 1 << lpr_log2;
    const int glane = threadIdx.x & (lpr - 1);
    const int lane_in_wave = threadIdx.x & 63;
    const int cmax = wave_max(cnt);
#pragma unroll
    for (int ch = 0; ch < CH; ++ch)
#pragma unroll
        for (int v = 0; v < V; ++v) { a1[ch][v] = T(0); a2[ch][v] = T(0); }
    for (int base = 0; base < cmax; base += lpr) {
        int mycol = 0;
        T mwx = T(0), mwy = T(0);
        if (base + glane < cnt) {
            mycol = col[e0 + base + glane];
            const P2 ww = w[e0 + base + glane];
            mwx = ww.x;
            mwy = ww.y;
        }
        const int kend = min(lpr, cmax - base);   // uniform across the wave
        for (int k0 = 0; k0 < kend; k0 += U) {
            int jj[U];
            T wx[U], wy[U];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int src = (lane_in_wave & ~(lpr - 1)) + ((k0 + u) & (lpr - 1));
                jj[u] = __shfl(mycol, src, 64);
                wx[u] = __shfl(mwx, src, 64);
                wy[u] = __shfl(mwy, src, 64);
                ok[u] = (k0 + u < kend) && (base + k0 + u < cnt);
            }
            T xb[U][CH][V];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int ch = 0; ch < CH; ++ch) {
                    const int c0 = (glane + ch * lpr) * V;
                    if (ok[u] && c0 < p) {
                        load_vec<T, V>(X + (int64_t)jj[u] * p + c0, xb[u][ch]);
                    } else {
#pragma unroll
                        for (int v = 0; v < V; ++v) xb[u][ch][v] = T(0);
                    }
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int ch = 0; ch < CH; ++ch)
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        a1[ch][v] = fma(wx[u], xb[u][ch][v], a1[ch][v]);
                        a2[ch][v] = fma(wy[u], xb[u][ch][v], a2[ch][v]);
                    }
        }
    }
}

// One element of the shifted product: returns what MODE writes and adds to the
// dots.  Selects, so that nothing of an inactive column (whose d may be
// anything) reaches the sums.
template <int MODE, typename T>
__device__ __forceinline__ T shift_value(bool on, T a1, T a2, T lm, T ld, T bdv, T d, double &dq, double &qw) {
    const T q = on ? fma(-lm, a2, a1) : T(0);
    if (MODE == SHIFT) return q;
    dq = on ? fma((double)d, (double)q, dq) : dq;
    if (MODE == SHIFT_DOT) return q;
    const T w = on ? q / (ld - lm * bdv) : T(0);
    qw = on ? fma((double)q, (double)w, qw) : qw;
    return q;
}

// Workgroups are dispatched to the 8 XCDs round-robin (block b on XCD b % 8).
// The logical block index gives each XCD a contiguous range of rows, so the
// neighbour rows a row reads were mostly fetched into the same XCD's L2.
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t nb_padded) {
    return (b % 8) * (nb_padded / 8) + b / 8;
}

template <typename T, int V, int CH, int U, int NOUT>
__global__ __launch_bounds__(256) void k_spmm_pair(int64_t n, int p, int lpr_log2,
                                                  const int64_t *__restrict__ rp,
                                                  const int32_t *__restrict__ col,
                                                  const typename pair_t<T>::type *__restrict__ ab,
                                                  const T *__restrict__ X, T *__restrict__ Y1,
                                                  T *__restrict__ Y2, int sel) {
    const int lpr = 1 << lpr_log2;
    const int64_t lb = xcd_block(blockIdx.x, gridDim.x);
    const int64_t row = (lb * blockDim.x + threadIdx.x) >> lpr_log2;
    const int glane = threadIdx.x & (lpr - 1);
    int64_t e0 = 0;
    int cnt = 0;
    if (row < n) {
        e0 = rp[row];
        cnt = (int)(rp[row + 1] - e0);
    }
    T a1[CH][V], a2[CH][V];
    gather_row<T, V, CH, U>(e0, cnt, lpr_log2, p, col, ab, X, a1, a2);
    if (row >= n) return;
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
        const int c0 = (glane + ch * lpr) * V;
        if (c0 >= p) continue;
        if (NOUT == 2) {
            store_vec<T, V>(Y1 + row * p + c0, a1[ch]);
            store_vec<T, V>(Y2 + row * p + c0, a2[ch]);
        } else {
            store_vec<T, V>(Y1 + row * p + c0, sel ? a2[ch] : a1[ch]);
        }
    }
}

// Persistent grid: each wave owns a fixed sequence of row groups, so every
// block's share and summation order are fixed by the launch shape and the
// per-block partial dot products are reproducible.
template <typename T, int V, int CH, int U, int MODE>
__global__ __launch_bounds__(256) void k_spmm_shift(int64_t n, int p, int lpr_log2,
                                                   const int64_t *__restrict__ rp,
                                                   const int32_t *__restrict__ col,
                                                   const typename pair_t<T>::type *__restrict__ lb,
                                                   const T *__restrict__ lam,
                                                   const uint8_t *__restrict__ active,
                                                   const double *__restrict__ lhd, const double *__restrict__ bd,
                                                   const T *__restrict__ D, T *__restrict__ Q,
                                                   double *__restrict__ part) {
    extern __shared__ double red[];  // [groups][p]
    const int lpr = 1 << lpr_log2;
    const int groups = blockDim.x >> lpr_log2;
    const int g = threadIdx.x >> lpr_log2;
    const int glane = threadIdx.x & (lpr - 1);
    const int gpw = 64 >> lpr_log2;   // row groups per wave
    double dot[2][CH][V];
    T lm[CH][V];
    bool on[CH][V];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch)
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int c = (glane + ch * lpr) * V + v;
            dot[0][ch][v] = dot[1][ch][v] = 0.0;
            lm[ch][v] = c < p ? lam[c] : T(0);
            on[ch][v] = c < p ? active[c] != 0 : false;
        }
    // XCD x = blockIdx % 8 sweeps the row slab [x S, (x+1) S); its blocks take
    // consecutive row groups of the slab in rounds.  rb is the first row of
    // this wave in a round and is uniform across the wave.
    const int64_t bpx = gridDim.x / 8;
    const int64_t slab = ((n + 7) / 8 + groups - 1) / groups * groups;
    const int64_t s0 = (blockIdx.x % 8) * slab;
    const int64_t s1 = min(n, s0 + slab);
    const int64_t stride = bpx * groups;
    for (int64_t rb = s0 + (int64_t)(blockIdx.x / 8) * groups + (g & ~(gpw - 1)); rb < s1; rb += stride) {
        const int64_t row = rb + (g & (gpw - 1));
        int64_t e0 = 0;
        int cnt = 0;
        if (row < s1) {
            e0 = rp[row];
            cnt = (int)(rp[row + 1] - e0);
        }
        T a1[CH][V], a2[CH][V];
        gather_row<T, V, CH, U>(e0, cnt, lpr_log2, p, col, lb, D, a1, a2);
        if (row < s1) {
            const T ld = MODE == SHIFT_CG ? (T)lhd[row] : T(0), bdv = MODE == SHIFT_CG ? (T)bd[row] : T(0);
#pragma unroll
            for (int ch = 0; ch < CH; ++ch) {
                const int c0 = (glane + ch * lpr) * V;
                if (c0 >= p) continue;
                T q[V], dv[V];
                if (MODE != SHIFT) load_vec<T, V>(D + row * p + c0, dv);
#pragma unroll
                for (int v = 0; v < V; ++v)
                    q[v] = shift_value<MODE, T>(on[ch][v], a1[ch][v], a2[ch][v], lm[ch][v], ld, bdv, dv[v],
                                                dot[0][ch][v], dot[1][ch][v]);
                if (MODE != SHIFT_DOT) store_vec<T, V>(Q + row * p + c0, q);
            }
        }
    }
    // block reduction over row groups, fixed order
    if (MODE == SHIFT) return;
#pragma unroll
    for (int d = 0; d < (MODE == SHIFT_CG ? 2 : 1); ++d) {
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
            const int c0 = (glane + ch * lpr) * V;
            if (c0 < p) {
#pragma unroll
                for (int v = 0; v < V; ++v) red[g * p + c0 + v] = dot[d][ch][v];
            }
        }
        __syncthreads();
        for (int c = threadIdx.x; c < p; c += blockDim.x) {
            double s = 0.0;
            for (int k = 0; k < groups; ++k) s += red[k * p + c];
            part[((int64_t)blockIdx.x * 2 + d) * p + c] = s;
        }
        __syncthreads();
    }
}

// One wave per row (used when a row's p values need all 64 lanes).  The row
// index is wave-uniform, so the row bounds, column indices and weights are
// scalar loads, and all U neighbour loads of a row go out as one batch before
// the arithmetic.
//
// Locality: with a locality-preserving node numbering the neighbours of a
// row have nearby numbers, so the rows in flight on one XCD must be a narrow
// window of consecutive rows for their neighbour rows to stay in that XCD's
// L2.  Rows go to XCDs in contiguous slabs (block b runs on XCD b % 8).
//  DUAL (Y1 = A1 X, Y2 = A2 X, or A2 X into Y1 when sel = 1): one row per
//    wave, blocks in slab order, so the dispatcher sweeps each slab forward.
//  SHIFT, SHIFT_CG, SHIFT_DOT (shifted operator, per-block partial dots):
//    persistent; the launcher sizes the grid to the blocks that can be
//    resident at once, and round r of block j takes rows base + 4 (r B + j),
//    so each round sweeps a window of 4 B consecutive rows per XCD.
template <typename T, int V, int CH, int U, int MODE>
__global__ __launch_bounds__(256) void k_spmm_wave(int64_t n, int p, const int64_t *__restrict__ rp,
                                                  const int32_t *__restrict__ col,
                                                  const typename pair_t<T>::type *__restrict__ w,
                                                  const T *__restrict__ X, T *__restrict__ Y1,
                                                  T *__restrict__ Y2, int sel, const T *__restrict__ lam,
                                                  const uint8_t *__restrict__ active,
                                                  const double *__restrict__ lhd, const double *__restrict__ bd,
                                                  double *__restrict__ part) {
    __shared__ double red[4][64 * V * CH];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t row, s1, stride;
    if (MODE == DUAL) {
        row = xcd_block(blockIdx.x, gridDim.x) * 4 + wave;
        s1 = n;
        stride = n;   // one row
    } else {
        const int64_t bpx = gridDim.x / 8;
        const int64_t slab = ((n + 7) / 8 + 3) / 4 * 4;
        const int64_t s0 = (blockIdx.x % 8) * slab;
        s1 = min(n, s0 + slab);
        row = s0 + (int64_t)(blockIdx.x / 8) * 4 + wave;
        stride = bpx * 4;
    }
    double dot[2][CH][V];
    T lm[CH][V];
    bool on[CH][V];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch)
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int c = (lane + ch * 64) * V + v;
            dot[0][ch][v] = dot[1][ch][v] = 0.0;
            if (MODE != DUAL) {
                lm[ch][v] = c < p ? lam[c] : T(0);
                on[ch][v] = c < p ? active[c] != 0 : false;
            }
        }
    for (; row < s1; row += stride) {
        const int64_t e0 = rp[row], e1 = rp[row + 1];
        T a1[CH][V], a2[CH][V];
#pragma unroll
        for (int ch = 0; ch < CH; ++ch)
#pragma unroll
            for (int v = 0; v < V; ++v) { a1[ch][v] = T(0); a2[ch][v] = T(0); }
        for (int64_t e = e0; e < e1; e += U) {
            const int m = (int)min((int64_t)U, e1 - e);
            int jj[U];
            T wx[U], wy[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u < m) {
                    jj[u] = stream_load(col + e + u);
                    wx[u] = stream_load(&w[e + u].x);
                    wy[u] = stream_load(&w[e + u].y);
                } else {
                    jj[u] = 0;
                    wx[u] = T(0);
                    wy[u] = T(0);
                }
            }
            T xb[U][CH][V];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int ch = 0; ch < CH; ++ch) {
                    const int c0 = (lane + ch * 64) * V;
                    if (u < m && c0 < p) {
                        load_vec<T, V>(X + (int64_t)jj[u] * p + c0, xb[u][ch]);
                    } else {
#pragma unroll
                        for (int v = 0; v < V; ++v) xb[u][ch][v] = T(0);
                    }
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int ch = 0; ch < CH; ++ch)
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        a1[ch][v] = fma(wx[u], xb[u][ch][v], a1[ch][v]);
                        a2[ch][v] = fma(wy[u], xb[u][ch][v], a2[ch][v]);
                    }
        }
        const T ld = MODE == SHIFT_CG ? (T)lhd[row] : T(0), bdv = MODE == SHIFT_CG ? (T)bd[row] : T(0);
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
            const int c0 = (lane + ch * 64) * V;
            if (c0 >= p) continue;
            if (MODE == DUAL) {
                if (Y2) {
                    stream_store_vec<T, V>(Y1 + row * p + c0, a1[ch]);
                    stream_store_vec<T, V>(Y2 + row * p + c0, a2[ch]);
                } else {
                    stream_store_vec<T, V>(Y1 + row * p + c0, sel ? a2[ch] : a1[ch]);
                }
            } else {
                T q[V], dv[V];
                if (MODE != SHIFT) load_vec<T, V>(X + row * p + c0, dv);
#pragma unroll
                for (int v = 0; v < V; ++v)
                    q[v] = shift_value<MODE, T>(on[ch][v], a1[ch][v], a2[ch][v], lm[ch][v], ld, bdv, dv[v],
                                                dot[0][ch][v], dot[1][ch][v]);
                if (MODE != SHIFT_DOT) stream_store_vec<T, V>(Y1 + row * p + c0, q);
            }
        }
    }
    if (MODE == SHIFT_CG || MODE == SHIFT_DOT) {
#pragma unroll
        for (int d = 0; d < (MODE == SHIFT_CG ? 2 : 1); ++d) {
#pragma unroll
            for (int ch = 0; ch < CH; ++ch)
#pragma unroll
                for (int v = 0; v < V; ++v) red[wave][(lane + ch * 64) * V + v] = dot[d][ch][v];
            __syncthreads();
            for (int c = threadIdx.x; c < p; c += blockDim.x)
                part[((int64_t)blockIdx.x * 2 + d) * p + c] = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
            __syncthreads();
        }
    }
}

// blocks of the non-persistent mode (one row per wave), whole XCD slabs
int64_t spmm_wave_blocks(int64_t n) { return ((n + 3) / 4 + 7) / 8 * 8; }

// Persistent grid of the shifted mode: the blocks that fit on the device at
// once (occupancy of this kernel instance), a multiple of 8 and at most cap.
template <typename K> int resident_grid(K kernel, int cap) {
    static int cached = 0;
    if (cached == 0) {
        int dev = 0, cus = 0, per = 0;
        (void)hipGetDevice(&dev);
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, 256, 0);
        int g = cus * (per > 0 ? per : 1);
        g = g / 8 * 8;
        cached = g < 8 ? 8 : g;
    }
    return cached < cap ? cached : cap;
}

// ---------------------------------------------------------------------------
// LDS-halo SpMM.  Plan block b owns the consecutive rows [row0[b], row0[b+1])
// (at most HALO_RMAX, each with at most 64 entries) and their halo: the
// distinct columns of those rows together with the rows themselves in
// ascending order, at most HALO_MAX rows of X, listed at halo[b HALO_STRIDE
// ...] (padded to the stride with the last one).  info[b] packs the halo's
// size, the number of rows and the halo slot of the first row (the rows sit at
// consecutive slots).  brp[b HALO_BRP + k] is the CSR row pointer of row
// row0[b] + k, for k = 0 .. HALO_RMAX (padded with row0[b+1]'s, so rows past
// the block have no entries).  lcol[e] is the halo slot of CSR entry e.
// Every per-block address depends on b alone, so the metadata loads issue
// together.
//
// One workgroup per plan block (and column range of cw, a whole number of
// slices: where the plan has too few blocks to fill the device, the slices are
// spread over workgroups); consecutive plan blocks run on one XCD, in
// dispatch order, so neighbouring blocks' halos meet in that XCD's L2.  For
// each 256-byte slice of the columns the workgroup stages its halo rows of X
// in LDS with direct global-to-LDS loads (no registers).  A wave then forms
// four rows at once, sixteen lanes a row and 16 bytes a lane.  A row's
// entries sit one per lane of its sixteen lanes, loaded once for all slices,
// and are handed round by DPP row broadcasts on the vector units: the LDS
// serves nothing but X.  (With one row per wave and the entries broadcast
// through LDS, the broadcasts took 2.5 times the LDS cycles of X and set the
// time.)  Entries past a row's end point to a slot of zeros, since a zero
// weight on a neighbour's row would turn its infinities into NaN.  ROUNDS (1,
// or 2 where some row has more than sixteen entries) times sixteen entries of
// a row are held in registers; later ones are loaded as they come.
//  DUAL: Y1 = A1 X and Y2 = A2 X (or, Y2 = NULL, A1 X or A2 X by sel).
//  SHIFT, SHIFT_CG, SHIFT_DOT: the shifted product into Y1, dots per plan block.
// SEGB: bytes per staging lane, 16 where the rows of X are 16-byte aligned,
// else 4.  Columns at or past p in a ragged last slice stage in-bounds data of
// the row's first segment; no output reads them.
//
// Measured (n = 1e6, p = 128, FP64; before: 16-row blocks of 76 halo rows in
// 512-byte slices, entries broadcast through LDS): shifted product 877 -> 615
// us, dual product 945 -> 745 us; n = 5.1e5, p = 128, FP32: 286 -> 192 and 297
// -> 189 us.  The shifted product moves 2.7 GB (1.24 times what it must) at
// 4.4 TB/s, the dual product 3.8 GB at 5.0 TB/s (a copy: 4.8), so memory
// bounds it.  Block shapes tried, FP64 shifted product in us with the call
// around it: (halo rows, rows, waves per SIMD) (200, 64, 3) 741, (120, 32, 4) 788,
// (148, 48, 4) 835, (240, 64, 2) 818, (76, 16, 6) 851; (192, 64, 3), which leaves
// the LDS room for the partials, against (200, 64, 3) later 656 and 657; workgroups that
// walk several blocks with the next one's loads in flight drift apart, and
// the widened window misses L2 (794, 2.4 to 3.4 GB fetched instead of 1.7).
// ---------------------------------------------------------------------------
// Tunables: halo rows (LDS = (HALO_MAX + 1) x 256 B and the dot partials,
// three workgroups a CU) and rows per block.
#ifndef OFKS_HALO_MAX
#define OFKS_HALO_MAX 192
#endif
#ifndef OFKS_HALO_RMAX
#define OFKS_HALO_RMAX 64
#endif
#ifndef OFKS_HALO_WPE
#define OFKS_HALO_WPE 3
#endif
constexpr int HALO_MAX = OFKS_HALO_MAX, HALO_RMAX = OFKS_HALO_RMAX, HALO_WAVES = 4, HALO_EMAX = 64;
constexpr int HALO_SETS = HALO_RMAX / (4 * HALO_WAVES);   // row sets (four rows each) per wave
constexpr int HALO_SST = 4 * HALO_WAVES;   // halo slots filled by one 16-byte load of every wave
constexpr int HALO_STRIDE = (HALO_MAX + HALO_SST - 1) / HALO_SST * HALO_SST;
constexpr int HALO_BRP = HALO_RMAX + 1;    // per-block row pointer stride
static_assert(HALO_WAVES == 4, "four partials per column");
static_assert(HALO_RMAX % (4 * HALO_WAVES) == 0, "whole row sets per wave");
static_assert(HALO_MAX % 4 == 0, "a wave fills four slots at a time");
static_assert(HALO_MAX < 256 && HALO_RMAX < 256, "info fields");

template <typename T> __device__ __forceinline__ void stream_store16(T *p, const T (&in)[16 / sizeof(T)]) {
    typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
    vec v;
#pragma unroll
    for (int i = 0; i < 16 / (int)sizeof(T); ++i) v[i] = in[i];
    __builtin_nontemporal_store(v, (vec *)p);
}

// lane K of each 16 lanes, to all of them
template <int K> __device__ __forceinline__ int row_bcast(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x150 + K, 0xf, 0xf, true);
}
template <int K> __device__ __forceinline__ float row_bcast(float v) {
    return __builtin_amdgcn_update_dpp(0.0f, v, 0x150 + K, 0xf, 0xf, true);
}
template <int K> __device__ __forceinline__ double row_bcast(double v) {
    return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + K, 0xf, 0xf, true);
}

// sum over the wave's four rows of sixteen lanes, to all of them: (r0 + r1)
// + (r2 + r3) on the vector units (a lane exchange through LDS costs its cycles)
__device__ __forceinline__ double rows_sum(double v) {
    // swap(x, x): the odd rows of the first and the even rows of the second
    // change places, so the two hold each row pair's even and odd row twice
    const auto a = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = __hiloint2double(b[0], a[0]) + __hiloint2double(b[1], a[1]);
    const auto c = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto d = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double(d[0], c[0]) + __hiloint2double(d[1], c[1]);
}

// entries K .. K + 3 of the sixteen: all LDS reads, then the FMAs in entry order
template <int K, typename T>
__device__ __forceinline__ void halo_four(const char *__restrict__ xs, int off, T wx, T wy, T (&a1)[16 / sizeof(T)],
                                          T (&a2)[16 / sizeof(T)]) {
    constexpr int VW = 16 / (int)sizeof(T);
    T x[4][VW];
    const int o[4] = {row_bcast<K>(off), row_bcast<K + 1>(off), row_bcast<K + 2>(off), row_bcast<K + 3>(off)};
#pragma unroll
    for (int u = 0; u < 4; ++u) load_vec<T, VW>((const T *)(xs + o[u]), x[u]);
    const T w1[4] = {row_bcast<K>(wx), row_bcast<K + 1>(wx), row_bcast<K + 2>(wx), row_bcast<K + 3>(wx)};
    const T w2[4] = {row_bcast<K>(wy), row_bcast<K + 1>(wy), row_bcast<K + 2>(wy), row_bcast<K + 3>(wy)};
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < VW; ++v) {
            a1[v] = fma(w1[u], x[u][v], a1[v]);
            a2[v] = fma(w2[u], x[u][v], a2[v]);
        }
}
// a round of sixteen entries, of which the first cnt are some row's (cnt the same in the whole wave)
template <typename T>
__device__ __forceinline__ void halo_round(const char *__restrict__ xs, int cnt, int off, T wx, T wy,
                                           T (&a1)[16 / sizeof(T)], T (&a2)[16 / sizeof(T)]) {
    halo_four<0, T>(xs, off, wx, wy, a1, a2);
    if (cnt > 4) halo_four<4, T>(xs, off, wx, wy, a1, a2);
    if (cnt > 8) halo_four<8, T>(xs, off, wx, wy, a1, a2);
    if (cnt > 12) halo_four<12, T>(xs, off, wx, wy, a1, a2);
}

template <typename T, int MODE, int SEGB, int ROUNDS>
__global__ __launch_bounds__(64 * HALO_WAVES) __attribute__((amdgpu_waves_per_eu(OFKS_HALO_WPE, OFKS_HALO_WPE))) void
k_spmm_halo(int64_t nb, int p, int cw, const int64_t *__restrict__ row0, const int32_t *__restrict__ info,
            const int32_t *__restrict__ halo, const int64_t *__restrict__ brp, const uint16_t *__restrict__ lcol,
            const typename pair_t<T>::type *__restrict__ w, const T *__restrict__ X, T *__restrict__ Y1,
            T *__restrict__ Y2, int sel, const T *__restrict__ lam, const uint8_t *__restrict__ active,
            const double *__restrict__ lhd, const double *__restrict__ bd, double *__restrict__ part) {
    using P2 = typename pair_t<T>::type;
    constexpr int CP = 256 / sizeof(T);   // columns per slice: 32 (f64) or 64 (f32)
    constexpr int VW = 16 / sizeof(T);    // columns per lane
    constexpr int NSLOT = HALO_STRIDE / HALO_SST;   // slots a thread stages, in 16-byte pieces
    static_assert(HALO_STRIDE / HALO_WAVES <= 64, "a wave's slots fit its lanes");
    __shared__ __align__(16) char Xs[(HALO_MAX + 1) * 256];
    constexpr int NDOT = MODE == SHIFT_CG ? 2 : MODE == SHIFT_DOT ? 1 : 0;
    __shared__ double red[NDOT ? NDOT * HALO_WAVES * CP : 1];
    const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t b = xcd_block(blockIdx.x, gridDim.x);
    const int cb = blockIdx.y * cw, ce = min(p, cb + cw);   // this workgroup's columns
    if (b >= nb) {   // padding block of the XCD mapping: a zero partial row
        for (int d = 0; d < NDOT; ++d)
            for (int c = cb + threadIdx.x; c < ce; c += blockDim.x) part[(2 * b + d) * p + c] = 0.0;
        return;
    }
    // this thread's halo rows (SEGB 4: lane u holds the wave's u-th slot's),
    // then the rows' entry ranges, all in flight together
    int hrow[NSLOT];
    const int32_t *hp = halo + b * HALO_STRIDE;
    if (SEGB == 16) {
#pragma unroll
        for (int u = 0; u < NSLOT; ++u) hrow[u] = hp[HALO_SST * u + 4 * wave + g];
    } else {
        hrow[0] = hp[min(HALO_WAVES * lane + wave, HALO_STRIDE - 1)];
    }
    __builtin_amdgcn_sched_barrier(0);
    // set i of this lane's wave: row 16 wave + 4 i + g of the block
    const int64_t *bp = brp + b * HALO_BRP + 4 * HALO_SETS * wave + g;
    int64_t e0[HALO_SETS];
    int len[HALO_SETS];
#pragma unroll
    for (int i = 0; i < HALO_SETS; ++i) {
        e0[i] = bp[4 * i];
        len[i] = (int)(bp[4 * i + 1] - e0[i]);
    }
    const int inf = info[b];
    const int64_t r0 = row0[b];
    const int hn = inf & 255, nrows = (inf >> 8) & 255, rb = (inf >> 16) & 255;
    // the rows' diagonals of L/2 and B: lane i of each sixteen holds set i's
    static_assert(HALO_SETS == 4, "the broadcasts below");
    T ldl = T(0), bdl = T(0);
    if (MODE == SHIFT_CG) {
        const int64_t r = r0 + min(4 * HALO_SETS * wave + 4 * (li & 3) + g, nrows - 1);
        ldl = (T)lhd[r];
        bdl = (T)bd[r];
    }
    if (threadIdx.x < 16) {
        const T z[VW] = {};
        store_vec<T, VW>((T *)(Xs + HALO_MAX * 256 + 16 * threadIdx.x), z);
    }
    auto stage = [&](int c0) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        if (SEGB == 16) {
#pragma unroll
            for (int u = 0; u < NSLOT; ++u) asm volatile("" : "+v"(hrow[u]));   // no addresses kept from slice to slice
            const int c = c0 + VW * li;
            const T *base = X + (c < p ? c : 0);
#pragma unroll
            for (int u = 0; u < NSLOT; ++u) {
                const int s0 = HALO_SST * u + 4 * wave;
                if (s0 < hn)
                    __builtin_amdgcn_global_load_lds((const void *)(base + (int64_t)hrow[u] * p),
                                                     (__attribute__((address_space(3))) void *)(Xs + s0 * 256), 16, 0, 0);
            }
        } else {
            constexpr int DW = sizeof(T) / 4;   // dwords per column
            const int c = c0 + lane / DW;
            const uint32_t *base = (const uint32_t *)(X + (c < p ? c : 0)) + lane % DW;
            for (int s0 = wave, u = 0; s0 < hn; s0 += HALO_WAVES, ++u)
                __builtin_amdgcn_global_load_lds(
                    (const void *)(base + (int64_t)__builtin_amdgcn_readlane(hrow[0], u) * p * DW),
                    (__attribute__((address_space(3))) void *)(Xs + s0 * 256), 4, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    stage(cb);
    // the first ROUNDS rounds of sixteen entries of each row, in registers:
    // LDS offset and weights of this lane's entry (past the row's end: entry
    // 0, which exists, for the load, the slot of zeros and weights of zero)
    auto entry = [&](int64_t e0, int len, int base, int &off, T &wx, T &wy) __attribute__((always_inline)) {
        const bool in = base + li < len;
        const int64_t e = in ? e0 + base + li : 0;
        const P2 ww = w[e];
        const int lc = lcol[e];
        off = (in ? lc : HALO_MAX) * 256;
        wx = in ? ww.x : T(0);
        wy = in ? ww.y : T(0);
    };
    int off[ROUNDS][HALO_SETS], m[HALO_SETS];
    T wx[ROUNDS][HALO_SETS], wy[ROUNDS][HALO_SETS];
#pragma unroll
    for (int i = 0; i < HALO_SETS; ++i) {
        m[i] = max(max(__builtin_amdgcn_readlane(len[i], 0), __builtin_amdgcn_readlane(len[i], 16)),
                   max(__builtin_amdgcn_readlane(len[i], 32), __builtin_amdgcn_readlane(len[i], 48)));
        entry(e0[i], len[i], 0, off[0][i], wx[0][i], wy[0][i]);
        if (ROUNDS == 2) entry(e0[i], len[i], 16, off[ROUNDS - 1][i], wx[ROUNDS - 1][i], wy[ROUNDS - 1][i]);
    }
    for (int c0 = cb; c0 < ce; c0 += CP) {
        const int c = c0 + VW * li;   // this lane's columns
        T lm[VW];
        bool on[VW];
        double dot[2][VW];
#pragma unroll
        for (int v = 0; v < VW; ++v) {
            lm[v] = (MODE != DUAL && c + v < p) ? lam[c + v] : T(0);
            on[v] = (MODE != DUAL && c + v < p) ? active[c + v] != 0 : false;
            dot[0][v] = dot[1][v] = 0.0;
        }
        __builtin_amdgcn_s_waitcnt(0);   // this thread's loads
        __builtin_amdgcn_s_barrier();    // every wave's: the slice is in LDS
        __builtin_amdgcn_sched_barrier(0);
        const char *xs = Xs + 16 * li;
#pragma unroll
        for (int i = 0; i < HALO_SETS; ++i) {
            const int k = 4 * HALO_SETS * wave + 4 * i + g;
            T a1[VW], a2[VW];
#pragma unroll
            for (int v = 0; v < VW; ++v) a1[v] = a2[v] = T(0);
            halo_round<T>(xs, m[i], off[0][i], wx[0][i], wy[0][i], a1, a2);
            if (ROUNDS == 2 && m[i] > 16)
                halo_round<T>(xs, m[i] - 16, off[ROUNDS - 1][i], wx[ROUNDS - 1][i], wy[ROUNDS - 1][i], a1, a2);
            for (int base = 16 * ROUNDS; base < m[i]; base += 16) {
                int oo;
                T x1, x2;
                const int64_t ee = bp[4 * i];
                entry(ee, (int)(bp[4 * i + 1] - ee), base, oo, x1, x2);
                halo_round<T>(xs, m[i] - base, oo, x1, x2, a1, a2);
            }
            if (MODE != DUAL) {
                T dv[VW];   // D's own row, staged with the halo (rows past the block: zeros, and q = 0)
                const T ld = i == 0 ? row_bcast<0>(ldl) : i == 1 ? row_bcast<1>(ldl) : i == 2 ? row_bcast<2>(ldl) : row_bcast<3>(ldl);
                const T bdv = i == 0 ? row_bcast<0>(bdl) : i == 1 ? row_bcast<1>(bdl) : i == 2 ? row_bcast<2>(bdl) : row_bcast<3>(bdl);
                if (NDOT) load_vec<T, VW>((const T *)(xs + (k < nrows ? rb + k : HALO_MAX) * 256), dv);
#pragma unroll
                for (int v = 0; v < VW; ++v)
                    a1[v] = shift_value<MODE, T>(on[v], a1[v], a2[v], lm[v], ld, bdv, dv[v], dot[0][v], dot[1][v]);
            }
            if (MODE != SHIFT_DOT && k < nrows && c < p) {
                T *y = Y1 + (r0 + k) * p + c;
                T *y2 = Y2 + (r0 + k) * p + c;
                if (SEGB == 16) {   // p is a multiple of VW: a piece lies wholly inside or past p
                    if (MODE == DUAL && !Y2 && sel) {
                        stream_store16(y, a2);
                    } else {
                        stream_store16(y, a1);
                        if (MODE == DUAL && Y2) stream_store16(y2, a2);
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < VW; ++v) {
                        if (c + v >= p) continue;
                        if (MODE == DUAL && !Y2 && sel) {
                            y[v] = a2[v];
                        } else {
                            y[v] = a1[v];
                            if (MODE == DUAL && Y2) y2[v] = a2[v];
                        }
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);   // one set's LDS reads in flight at a time (registers)
        }
#pragma unroll
        for (int d = 0; d < NDOT; ++d)
#pragma unroll
            for (int v = 0; v < VW; ++v) {   // over the wave's four rows in flight, then one LDS slot per wave
                const double sum = rows_sum(dot[d][v]);
                if (g == 0) red[(d * HALO_WAVES + wave) * CP + VW * li + v] = sum;
            }
        __builtin_amdgcn_s_waitcnt(0xc07f);   // LDS done (lgkmcnt 0); vector memory untouched
        __builtin_amdgcn_s_barrier();         // the slice is consumed and the partials written
        __builtin_amdgcn_sched_barrier(0);
        if (c0 + CP < ce) stage(c0 + CP);
        if (NDOT && (int)threadIdx.x < NDOT * CP) {
            const int d = threadIdx.x / CP, cl = threadIdx.x % CP;
            const double *rd = red + d * HALO_WAVES * CP + cl;
            if (c0 + cl < p) part[(2 * b + d) * p + c0 + cl] = ((rd[0] + rd[CP]) + rd[2 * CP]) + rd[3 * CP];
        }
    }
}

// SpMV with the dot <d, A d> fused (Hartree CG); persistent grid, 16 lanes
// per row (P1 rows hold about 15 entries): each lane takes every 16th entry
// of the row with coalesced loads, the 16 partial sums are combined by
// shuffles in a fixed order, and the group's first lane writes q_i and
// accumulates d_i q_i.  Per-block partial written to part[block].
__global__ __launch_bounds__(256) void k_spmv_dot(int64_t n, const int64_t *__restrict__ rp,
                                                 const int32_t *__restrict__ col,
                                                 const double *__restrict__ a,
                                                 const double *__restrict__ d,
                                                 double *__restrict__ q,
                                                 double *__restrict__ part) {
    __shared__ double red[256];
    const int sub = threadIdx.x & 15;
    double s = 0.0;
    const int64_t rows_per_pass = (int64_t)gridDim.x * (blockDim.x / 16);
    for (int64_t i = (int64_t)blockIdx.x * (blockDim.x / 16) + (threadIdx.x >> 4); i - (threadIdx.x >> 4) < n;
         i += rows_per_pass) {
        double acc = 0.0;
        if (i < n) {
            const int64_t e1 = rp[i + 1];
            for (int64_t e = rp[i] + sub; e < e1; e += 16) acc = fma(a[e], d[col[e]], acc);
        }
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 16);
        if (sub == 0 && i < n) {
            q[i] = acc;
            s = fma(d[i], acc, s);
        }
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// ---------------------------------------------------------------------------
// One Hartree CG iteration in one kernel (one vector, FP64): the Jacobi-CG of
// Chronopoulos and Gear, J. Comput. Appl. Math. 25 (1989), whose two dots come
// from one product.  A row's state is u = M^-1 r, v = M^-1 A u, t = M^-1 A p
// and p, 32 bytes together, M = diag dg.  With gamma = <r, u> and delta = <A
// u, u> of the previous launch's partials,
//   beta = gamma / gamma_old, alpha = gamma / (delta - beta gamma / alpha_old),
//   t' = v + beta t, p' = u + beta p, x += alpha p', u' = u - alpha t',
//   w = A u', v' = M^-1 w, partials of <r', u'>, <w, u'> and <r', r'>.
// The product needs u' of the neighbours, which each workgroup forms itself
// from their old states: the launch boundary between two iterations is the only
// synchronisation.  Every workgroup sums all partials in one fixed order.  in
// and out, pin and pout and the scalars' two slots alternate, so nothing is
// overwritten that another workgroup still reads.  first: alpha = beta = 0 (v
// = M^-1 A u of a new u), and the next launch takes beta = 0.  check: the
// launch stops, and those after it do, once <r', r'> of the last one is within
// sc[3]; report (host memory) gets that sum with whether no iteration went before
// (cg_report_word), and the bound, so the host can queue iterations ahead of
// knowing.
//
// With the halo plan (which a mesh's matrices always have: its rows hold at
// most 64 entries) a state is read once per 64-row block (two to three times
// in all) instead of once per entry, the columns are two-byte slots, and a
// row's product reads LDS.  A team of 256 threads works on a plan block, a halo
// slot a thread and sixteen lanes a row, with the next block's loads in flight.
//
// Bound by latency where a workgroup has one block or two (the launch, the
// block's metadata, its states, the partials) and by memory on top of that.  An
// iteration in a captured ten, us, here against product, update and direction
// kernels: 5.1e4 rows 9.7 and 16.7, 6.4e4 9.8 and 17.2, 2.05e5 (60 MB) 17.7 and
// 27.1.  Plan blocks a workgroup at once, 2, 3, 4: 8.2, 9.7, 9.0; 9.7, 9.8, 11.3;
// 17.9, 17.7, 17.9.  One block a workgroup of 256 threads was 1.1 us slower at the
// small end (768 workgroups; more of them pay for the partials that each must sum).
// ---------------------------------------------------------------------------
#ifndef OFKS_CG_BLOCKS
#define OFKS_CG_BLOCKS 256   // a multiple of 8, at most 256 (a partial a thread of a team)
#endif
#ifndef OFKS_CG_TEAMS
#define OFKS_CG_TEAMS 3      // plan blocks a workgroup works on at once (2 to 4 fit; 4 spills)
#endif
struct CgIter {
    int first, check, parity, np;
    const double *dg;
    const double2 *in;
    double2 *out;
    double *x, *sc;
    const double *pin;
    double *pout, *report;
};

// v + the v of the lane N further on in each sixteen
template <int N> __device__ __forceinline__ double row_ror_add(double v) {
    return v + __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + N, 0xf, 0xf, true),
                                __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + N, 0xf, 0xf, true));
}
// sum over each sixteen lanes, to all of them
__device__ __forceinline__ double row_sum(double v) {
    return row_ror_add<1>(row_ror_add<2>(row_ror_add<4>(row_ror_add<8>(v))));
}

// what a thread loads ahead for a plan block
template <int ROUNDS, bool LONG> struct CgBlock {
    int h, rb;
    bool own;
    int64_t e0[LONG ? HALO_SETS : 1];
    int len[LONG ? HALO_SETS : 1];
    double2 s0, s1;
    double x, dg, a[HALO_SETS][ROUNDS];
    int sl[HALO_SETS][ROUNDS];
};

template <int ROUNDS, bool LONG>
__global__ __launch_bounds__(256 * OFKS_CG_TEAMS) void k_cg_iter(
    int64_t nb, const int32_t *__restrict__ info, const int32_t *__restrict__ halo, const int64_t *__restrict__ brp,
    const uint16_t *__restrict__ lcol, const double *__restrict__ a, CgIter c) {
    static_assert(HALO_MAX <= 256 && HALO_RMAX == 64 && HALO_WAVES == 4, "one slot a thread of a team");
    constexpr int W = 4 * OFKS_CG_TEAMS;
    __shared__ double us_[OFKS_CG_TEAMS][256], ws_[OFKS_CG_TEAMS][HALO_RMAX], red[3][W];
    const int team = threadIdx.x >> 8, tid = threadIdx.x & 255, li = tid & 15, g = tid >> 4;
    double *us = us_[team], *ws = ws_[team];
    const int lane = threadIdx.x & 63;
    // this lane's share of array j of the partials (np <= 256), summed over the wave
    auto partials = [&](int j, double (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = c.pin[j * c.np + min(lane + 64 * u, c.np - 1)];
    };
    auto partials_sum = [&](double (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (lane + 64 * u >= c.np) v[u] = 0.0;
        return rows_sum(row_sum((v[0] + v[1]) + (v[2] + v[3])));
    };
    if (c.check) {
        double v[4];
        partials(2, v);
        const double rr = partials_sum(v), tol2 = c.sc[3];
        const bool stop = !(rr > tol2);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            c.sc[0] = stop ? 1.0 : 0.0;
            // (no iteration yet: a first launch leaves gamma 0)
            __hip_atomic_store(c.report + 1, tol2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(c.report, cg_report_word(rr, c.sc[4 + 2 * c.parity] == 0.0), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
        }
        if (stop) return;
    } else if (!c.first && c.sc[0] != 0.0) {
        return;
    }
    // XCD x takes the plan blocks from x per on, OFKS_CG_TEAMS at a time and workgroup
    const int64_t per = (nb + 7) / 8, base = (blockIdx.x % 8) * per, end = min(base + per, nb);
    const int64_t step = (int64_t)(gridDim.x / 8) * OFKS_CG_TEAMS;
    const int64_t k0 = base + (int64_t)(blockIdx.x / 8) * OFKS_CG_TEAMS;   // the turn's first plan block
    // metadata of block k (past the end: the last one, whose loads go unused)
    int mh, mi;
    int64_t me[HALO_SETS];
    int ml[HALO_SETS];
    auto meta = [&](int64_t k) __attribute__((always_inline)) {
        k = min(k, nb - 1);
        mh = halo[k * HALO_STRIDE + min(tid, HALO_STRIDE - 1)];
        mi = info[k];
        const int64_t *bp = brp + k * HALO_BRP + g;   // this lane's rows: 16 i + g
#pragma unroll
        for (int i = 0; i < HALO_SETS; ++i) {
            me[i] = bp[16 * i];
            ml[i] = (int)(bp[16 * i + 1] - me[i]);
        }
    };
    auto data = [&](CgBlock<ROUNDS, LONG> &B, bool valid) __attribute__((always_inline)) {
        B.h = mh;
        B.rb = (mi >> 16) & 255;
        B.own = valid && tid >= B.rb && tid < B.rb + ((mi >> 8) & 255);
        B.s0 = c.in[2 * (int64_t)mh];
        B.s1 = c.in[2 * (int64_t)mh + 1];
        B.dg = 1.0;
        B.x = 0.0;
        if (B.own) {
            B.x = c.x[B.h];
            B.dg = c.dg[B.h];
        }
#pragma unroll
        for (int i = 0; i < HALO_SETS; ++i) {
            if (LONG) {
                B.e0[i] = me[i];
                B.len[i] = ml[i];
            }
#pragma unroll
            for (int u = 0; u < ROUNDS; ++u) {
                const bool on = 16 * u + li < ml[i];
                const int64_t e = on ? me[i] + 16 * u + li : 0;   // entry 0 exists
                B.a[i][u] = a[e];
                B.sl[i][u] = lcol[e];
                if (!on) {
                    B.a[i][u] = 0.0;
                    B.sl[i][u] = B.rb;
                }
            }
        }
    };
    double ga = 0.0, de = 0.0, rr = 0.0, alpha = 0.0, beta = 0.0;
    if (k0 < end) {
        meta(k0 + team);
        // every wave sums the partials itself: no barrier, and the first block's loads in flight
        double pg[4], pd[4];
        partials(0, pg);
        partials(1, pd);
        const double go = c.sc[4 + 2 * c.parity], ao = c.sc[5 + 2 * c.parity];
        CgBlock<ROUNDS, LONG> A, B;
        data(A, k0 + team < end);
        meta(k0 + team + step);
        if (!c.first) {
            const double gs = partials_sum(pg), ds = partials_sum(pd);
            beta = go > 0.0 ? gs / go : 0.0;
            const double den = ao > 0.0 ? ds - beta * gs / ao : ds;
            alpha = den > 0.0 ? gs / den : 0.0;
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                c.sc[4 + 2 * (c.parity ^ 1)] = gs;
                c.sc[5 + 2 * (c.parity ^ 1)] = alpha;
            }
        } else if (blockIdx.x == 0 && threadIdx.x == 0) {
            c.sc[4 + 2 * (c.parity ^ 1)] = 0.0;
            c.sc[5 + 2 * (c.parity ^ 1)] = 0.0;
        }
        auto work = [&](CgBlock<ROUNDS, LONG> &B) __attribute__((always_inline)) {
            const double t = fma(beta, B.s1.x, B.s0.y), un = fma(-alpha, t, B.s0.x);
            us[tid] = un;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < HALO_SETS; ++i) {
                double acc = 0.0;
#pragma unroll
                for (int u = 0; u < ROUNDS; ++u) acc = fma(B.a[i][u], us[B.sl[i][u]], acc);
                if (LONG)
                    for (int q = 16 * ROUNDS + li; q < B.len[i]; q += 16)
                        acc = fma(a[B.e0[i] + q], us[lcol[B.e0[i] + q]], acc);
                acc = row_sum(acc);
                if (li == 0) ws[16 * i + g] = acc;
            }
            __syncthreads();
            if (B.own) {
                const double w = ws[tid - B.rb], r = B.dg * un, p = fma(beta, B.s1.y, B.s0.x);
                if (!c.first) c.x[B.h] = fma(alpha, p, B.x);
                c.out[2 * (int64_t)B.h] = make_double2(un, w / B.dg);
                c.out[2 * (int64_t)B.h + 1] = make_double2(t, p);
                ga = fma(r, un, ga);
                de = fma(w, un, de);
                rr = fma(r, r, rr);
            }
        };
        // two sets of registers in turn: a block's loads are in flight while the one before is worked on
        for (int64_t k = k0;; k += 2 * step) {
            if (k + step < end) {
                data(B, k + step + team < end);
                meta(k + 2 * step + team);
            }
            work(A);
            if (k + step >= end) break;
            if (k + 2 * step < end) {
                data(A, k + 2 * step + team < end);
                meta(k + 3 * step + team);
            }
            work(B);
            if (k + 2 * step >= end) break;
        }
    }
    const double s[3] = {rows_sum(row_sum(ga)), rows_sum(row_sum(de)), rows_sum(row_sum(rr))};
    if ((threadIdx.x & 63) == 0)
        for (int j = 0; j < 3; ++j) red[j][threadIdx.x >> 6] = s[j];
    __syncthreads();
    if (threadIdx.x < 3) {
        double v = 0.0;
        for (int j = 0; j < W; ++j) v += red[threadIdx.x][j];
        c.pout[threadIdx.x * c.np + blockIdx.x] = v;
    }
}

// ---------------------------------------------------------------------------
// The inner CG of small blocks (FP64), one kernel an iteration, for every column c
// of its own: T_c = L/2 - lambda_c B, M_c = diag T_c.  The two-term recurrences in
// d, r and q = T d; a launch sums the previous one's partials of <d, q>, <q, M^-1
// q> and <r, M^-1 r>, takes alpha and the predicted beta from them (cg_coef), forms
//   r' = r - alpha q, d' = M^-1 r' + beta d   on the plan block's halo rows,
//   x += alpha d, q' = T d' and the new partials   on its own rows.
// A step of the three-kernel form is three launches of 3 to 6 us whatever the
// size; this one is bound by the same latencies, once.
//
// x is carried in twice the digits (its low part in a block of its own).  Error
// of ten steps on graded meshes (80-bit sums): 0.83 times that of the two-term
// recurrence; with M^-1 T p from a recurrence of its own (one product for both
// dots, as in k_cg_iter) it was 1.68 times, up to 5.4.
//
// A workgroup takes a plan block and CGB_COLS columns, a thread one column of
// one row and of three halo rows; what does not depend on alpha and beta (the
// states, sixteen entries of the row) is loaded while they are summed.  d, r, q
// (in) and d2, r2, q2 (out) change places from launch to launch, as do pin and
// pout (rows of 3 p a plan block).  first: q of d alone.  last: x alone.
// ---------------------------------------------------------------------------
constexpr int CGB_COLS = 4, CGB_AHEAD = 16;
struct CgBlockArgs {
    int first, last, start, p;   // start: the first iteration (x from zero)
    const double *lhd, *bd, *lam;
    const uint8_t *active;
    const double *d, *r, *q;
    double *d2, *r2, *q2, *x, *xl;
    const double *pin;
    double *pout;
};

// sums of three values over the workgroup's 64 rows of threads, to all of them
__device__ __forceinline__ void cgb_sum(double (&red)[3][16], double (&v)[3]) {
    // lanes of one column are four apart: on the vector units within a wave, then over the four waves
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, c = threadIdx.x & (CGB_COLS - 1);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        v[k] = row_ror_add<4>(row_ror_add<8>(v[k]));
        v[k] = rows_sum(v[k]);
        if (l < CGB_COLS) red[k][CGB_COLS * w + l] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k)
        v[k] = (red[k][c] + red[k][CGB_COLS + c]) + (red[k][2 * CGB_COLS + c] + red[k][3 * CGB_COLS + c]);
}

__global__ __launch_bounds__(256) void k_cgb_iter(int64_t nb, const int64_t *__restrict__ row0,
                                                 const int32_t *__restrict__ info, const int32_t *__restrict__ halo,
                                                 const int64_t *__restrict__ brp, const uint16_t *__restrict__ lcol,
                                                 const double2 *__restrict__ lb, CgBlockArgs c) {
    constexpr int G = 256 / CGB_COLS, NS = (HALO_MAX + G - 1) / G;   // thread rows, halo rows a thread
    static_assert(G == HALO_RMAX, "a matrix row a thread");
    static_assert(CGB_COLS * 4 == 16, "cgb_sum");
    __shared__ double ds[NS * G * CGB_COLS], red[2][3][16];
    const int tid = threadIdx.x, cl = tid & (CGB_COLS - 1), g = tid / CGB_COLS;
    const int64_t b = blockIdx.x;
    const int col = (int)blockIdx.y * CGB_COLS + cl;
    const bool in = col < c.p, on = in && c.active[in ? col : 0] != 0;
    const double lm = c.lam[in ? col : 0];
    int hr[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) hr[i] = halo[b * HALO_STRIDE + min(g + i * G, HALO_STRIDE - 1)];
    const int inf = info[b], nr = (inf >> 8) & 255, rb = (inf >> 16) & 255;
    const int64_t row = row0[b] + min(g, nr - 1), e0 = brp[b * HALO_BRP + g];
    const int len = (int)(brp[b * HALO_BRP + g + 1] - e0);   // 0 past the block's rows
    // partials of <d, q>, <q, M^-1 q>, <r, M^-1 r>: the first 64 plan blocks' now
    double sum[3] = {0.0, 0.0, 0.0};
    if (!c.first && in && g < nb)
#pragma unroll
        for (int u = 0; u < 3; ++u) sum[u] = c.pin[(3 * (int64_t)g + u) * c.p + col];
    double2 w[CGB_AHEAD];
    int lc[CGB_AHEAD];
    if (!c.last)
#pragma unroll
        for (int j = 0; j < CGB_AHEAD; ++j) {
            const int64_t e = j < len ? e0 + j : 0;   // entry 0 exists
            w[j] = lb[e];
            lc[j] = lcol[e];
        }
    double d[NS], r[NS], q[NS], iv[NS], x[NS], xl[NS];   // (iv: M^-1)
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int s = g + i * G;
        const bool own = on && s >= rb && s < rb + nr;
        const int64_t e = (int64_t)hr[i] * c.p + (in ? col : 0);
        d[i] = on ? c.d[e] : 0.0;
        r[i] = on && !c.last ? c.r[e] : 0.0;
        q[i] = on && !c.first && !c.last ? c.q[e] : 0.0;
        iv[i] = c.last ? 1.0 : 1.0 / (c.lhd[hr[i]] - lm * c.bd[hr[i]]);
        x[i] = own && !c.first && !c.start ? c.x[e] : 0.0;
        xl[i] = own && !c.first && !c.start ? c.xl[e] : 0.0;
    }
    const double ivr = c.last ? 1.0 : 1.0 / (c.lhd[row] - lm * c.bd[row]);
    CgCoef<double> k{0.0, 0.0, 0.0};
    if (!c.first) {
        if (in)
            for (int64_t b2 = g + G; b2 < nb; b2 += G)
#pragma unroll
                for (int u = 0; u < 3; ++u) sum[u] += c.pin[(3 * b2 + u) * c.p + col];
        cgb_sum(red[0], sum);
        k = cg_coef<double>(sum[0], sum[1], sum[2], 0.0);
        sum[2] = 0.0;
    }
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        const int s = g + i * G;
        const bool own = on && s >= rb && s < rb + nr;
        const int64_t e = (int64_t)hr[i] * c.p + col;
        const double rn = fma(-k.alpha, q[i], r[i]), z = rn * iv[i];   // (first: alpha = 0)
        const double dn = c.first ? d[i] : fma(k.beta, d[i], z);
        if (own) {
            sum[2] = fma(rn, z, sum[2]);
            if (!c.first) {
                double lo = xl[i];
                c.x[e] = cg_carry(x[i], lo, k.alpha, d[i], c.last);
                if (!c.last) {
                    c.xl[e] = lo;
                    c.d2[e] = dn;
                    c.r2[e] = rn;
                }
            }
        }
        ds[s * CGB_COLS + cl] = on ? dn : 0.0;
    }
    if (c.last) return;
    __syncthreads();
    sum[0] = sum[1] = 0.0;
    if (on && g < nr) {
        double a1 = 0.0, a2 = 0.0;
#pragma unroll
        for (int j = 0; j < CGB_AHEAD; ++j)
            if (j < len) {
                const double dn = ds[lc[j] * CGB_COLS + cl];
                a1 = fma(w[j].x, dn, a1);
                a2 = fma(w[j].y, dn, a2);
            }
        for (int j = CGB_AHEAD; j < len; ++j) {
            const double2 wj = lb[e0 + j];
            const double dn = ds[(int)lcol[e0 + j] * CGB_COLS + cl];
            a1 = fma(wj.x, dn, a1);
            a2 = fma(wj.y, dn, a2);
        }
        const double qn = fma(-lm, a2, a1);
        c.q2[row * c.p + col] = qn;
        sum[0] = ds[(rb + g) * CGB_COLS + cl] * qn;
        sum[1] = qn * (qn * ivr);
    }
    cgb_sum(red[1], sum);
    if (g == 0 && in)
#pragma unroll
        for (int u = 0; u < 3; ++u) c.pout[(3 * b + u) * c.p + col] = sum[u];
}

// Workgroups of a launch.
int64_t cgb_blocks(int64_t nb, int p) { return nb * ((p + CGB_COLS - 1) / CGB_COLS); }
// doubles of the blocks and partials that a width p takes beside the caller's blocks
size_t cgb_doubles(int64_t n, int64_t nb, int p) { return (size_t)(4 * n + 6 * nb) * p; }

// m iterations on D (M^-1 R; R the residual at x = 0) into X's active columns.
// D, R, Q: n p values each, overwritten; extra: cgb_doubles.
hipError_t launch_cgb(hipStream_t s, int m, int64_t n, int64_t nb, int p, const int64_t *row0, const int32_t *info,
                      const int32_t *halo, const int64_t *brp, const uint16_t *lcol, const void *lb, const double *lhd,
                      const double *bd, const double *lam, const uint8_t *active, double *D, double *R, double *Q,
                      double *X, double *extra) {
    if (m <= 0) return hipErrorInvalidValue;
    const int64_t np = n * p;
    const dim3 grid((unsigned)nb, (unsigned)((p + CGB_COLS - 1) / CGB_COLS));
    double *st[2][3] = {{D, R, Q}, {extra, extra + np, extra + 2 * np}};
    double *part = extra + 4 * np, *pt[2] = {part, part + 3 * nb * p};
    CgBlockArgs c{1, 0, 0, p, lhd, bd, lam, active, D, R, nullptr, nullptr, nullptr, Q, X, extra + 3 * np, pt[1], pt[0]};
    hipLaunchKernelGGL(k_cgb_iter, grid, dim3(256), 0, s, nb, row0, info, halo, brp, lcol, (const double2 *)lb, c);
    c.first = 0;
    for (int j = 0; j < m; ++j) {
        c.start = j == 0;
        c.last = j + 1 == m;
        c.d = st[j & 1][0];
        c.r = st[j & 1][1];
        c.q = st[j & 1][2];
        c.d2 = st[(j & 1) ^ 1][0];
        c.r2 = st[(j & 1) ^ 1][1];
        c.q2 = st[(j & 1) ^ 1][2];
        c.pin = pt[j & 1];
        c.pout = pt[(j & 1) ^ 1];
        hipLaunchKernelGGL(k_cgb_iter, grid, dim3(256), 0, s, nb, row0, info, halo, brp, lcol, (const double2 *)lb, c);
    }
    return hipGetLastError();
}

// The grid, and with it the number of partials: a multiple of 8, at most
// OFKS_CG_BLOCKS, with the plan's blocks spread evenly.
int cg_iter_blocks(int64_t nb) {
    const int64_t per = ((nb + 7) / 8 + OFKS_CG_TEAMS - 1) / OFKS_CG_TEAMS, most = OFKS_CG_BLOCKS / 8;
    const int64_t rounds = (per + most - 1) / most;
    return (int)(8 * ((per + rounds - 1) / rounds));
}
int cg_iter_blocks_max() { return OFKS_CG_BLOCKS; }

// out[g][c] = sum of rows [g G, (g + 1) G) of an nb x p partial matrix, in row
// order; threads run over columns, so every read is coalesced.
__global__ __launch_bounds__(256) void k_part_rows(int64_t nb, int p, int G, const double *__restrict__ in,
                                                  double *__restrict__ out) {
    const int64_t g = blockIdx.x;
    const int64_t b0 = g * G, b1 = min(nb, b0 + G);
    for (int c = threadIdx.x; c < p; c += blockDim.x) {
        double sum = 0.0;
#pragma unroll 8
        for (int64_t b = b0; b < b1; ++b) sum += in[b * p + c];
        out[g * p + c] = sum;
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

static inline int ilog2_ceil(int x) {
    int l = 0;
    while ((1 << l) < x) ++l;
    return l;
}

template <typename T> static inline int pick_v(int p) {
    if (sizeof(T) == 8) return (p % 2 == 0) ? 2 : 1;
    return (p % 4 == 0) ? 4 : ((p % 2 == 0) ? 2 : 1);
}

// lanes per row: enough lanes to cover p with V-wide accesses, at most 64
static inline int lpr_log2_for(int p, int v) {
    int l = ilog2_ceil((p + v - 1) / v);
    return l > 6 ? 6 : l;
}

// Dispatch over (V, CH); U (neighbour loads in flight) shrinks as CH grows to
// bound registers.
#define OFKS_VCH_DISPATCH(LAUNCH)                                 \
    do {                                                          \
        if (v == 1 && ch <= 1) { LAUNCH(1, 1, 8); break; }        \
        if (v == 1 && ch <= 2) { LAUNCH(1, 2, 8); break; }        \
        if (v == 1 && ch <= 4) { LAUNCH(1, 4, 4); break; }        \
        if (v == 1 && ch <= 8) { LAUNCH(1, 8, 2); break; }        \
        if (v == 2 && ch <= 1) { LAUNCH(2, 1, 8); break; }        \
        if (v == 2 && ch <= 2) { LAUNCH(2, 2, 4); break; }        \
        if (v == 2 && ch <= 4) { LAUNCH(2, 4, 2); break; }        \
        if (v == 2 && ch <= 8) { LAUNCH(2, 8, 1); break; }        \
        if constexpr (sizeof(T) == 4) {                           \
            if (v == 4 && ch <= 1) { LAUNCH(4, 1, 8); break; }    \
            if (v == 4 && ch <= 2) { LAUNCH(4, 2, 4); break; }    \
            if (v == 4 && ch <= 4) { LAUNCH(4, 4, 2); break; }    \
        }                                                         \
        return hipErrorInvalidValue;                              \
    } while (0)

template <typename T>
hipError_t launch_spmm_pair(hipStream_t s, int64_t n, int p, const int64_t *rp, const int32_t *col,
                            const void *ab, const T *X, T *Y1, T *Y2, int sel) {
    using P2 = typename pair_t<T>::type;
    const int v = pick_v<T>(p);
    const int l2 = lpr_log2_for(p, v);
    const int ch = (p + (v << l2) - 1) / (v << l2);
    const P2 *w = (const P2 *)ab;
    if (l2 == 6) {
        const unsigned grid = (unsigned)spmm_wave_blocks(n);
#define OFKS_WAVE0(VV, CC)                                                                                   \
    hipLaunchKernelGGL((k_spmm_wave<T, VV, CC, (CC >= 8 ? 2 : OFKS_SPMM_U / CC), 0>), dim3(grid), dim3(256), 0, s, n, p, rp, col, w, X, Y1, Y2, \
                       sel, (const T *)nullptr, (const uint8_t *)nullptr, (const double *)nullptr, (const double *)nullptr, (double *)nullptr)
        if (v == 1 && ch == 1) OFKS_WAVE0(1, 1);
        else if (v == 1 && ch <= 2) OFKS_WAVE0(1, 2);
        else if (v == 2 && ch == 1) OFKS_WAVE0(2, 1);
        else if (v == 2 && ch <= 2) OFKS_WAVE0(2, 2);
        else if (v == 2 && ch <= 4) OFKS_WAVE0(2, 4);
        else if (v == 2 && ch <= 8) OFKS_WAVE0(2, 8);
        else if constexpr (sizeof(T) == 4) {
            if (v == 4 && ch == 1) OFKS_WAVE0(4, 1);
            else if (v == 4 && ch <= 2) OFKS_WAVE0(4, 2);
            else if (v == 4 && ch <= 4) OFKS_WAVE0(4, 4);
            else return hipErrorInvalidValue;
        } else return hipErrorInvalidValue;
#undef OFKS_WAVE0
        return hipGetLastError();
    }
    const int64_t threads = n << l2;
    const int bs = 256;
    const unsigned grid = (unsigned)((((threads + bs - 1) / bs) + 7) / 8 * 8);   // multiple of the XCD count
    const bool two = Y2 != nullptr;
#define OFKS_PAIR(VV, CC, UU)                                                                                 \
    if (two) hipLaunchKernelGGL((k_spmm_pair<T, VV, CC, UU, 2>), dim3(grid), dim3(bs), 0, s, n, p, l2, rp, col, w, X, Y1, Y2, sel); \
    else hipLaunchKernelGGL((k_spmm_pair<T, VV, CC, UU, 1>), dim3(grid), dim3(bs), 0, s, n, p, l2, rp, col, w, X, Y1, Y2, sel)
    OFKS_VCH_DISPATCH(OFKS_PAIR);
#undef OFKS_PAIR
    return hipGetLastError();
}

// Shifted product by row gather in `mode`.  Launches at most `grid` blocks (the
// caller's partial buffer holds 2 p values for each) and reports the number
// used in *blocks_used.
template <int MODE, typename T>
static hipError_t launch_spmm_shift_mode(hipStream_t s, int grid, int64_t n, int p, const int64_t *rp, const int32_t *col,
                                         const void *lb, const T *lam, const uint8_t *active, const double *lhd,
                                         const double *bd, const T *D, T *Q, double *part, int *blocks_used) {
    using P2 = typename pair_t<T>::type;
    if (grid % 8 != 0 || grid < 8) return hipErrorInvalidValue;   // whole XCD slabs
    const int v = pick_v<T>(p);
    const int l2 = lpr_log2_for(p, v);
    const int ch = (p + (v << l2) - 1) / (v << l2);
    const int bs = 256;
    // no more blocks than there are rounds of row groups
    const int64_t rounds = ((n + (bs >> l2) - 1) / (bs >> l2) + 7) / 8 * 8;
    if (grid > rounds) grid = (int)rounds;
    *blocks_used = grid;
    const size_t shm = (size_t)(bs >> l2) * p * sizeof(double);
    const P2 *w = (const P2 *)lb;
    if (l2 == 6) {
#define OFKS_WAVE1(VV, CC)                                                                                   \
    do {                                                                                                     \
        auto kfn = k_spmm_wave<T, VV, CC, (CC >= 8 ? 2 : OFKS_SPMM_U / CC), MODE>;                            \
        const int wgrid = resident_grid(kfn, grid);                                                          \
        *blocks_used = wgrid;                                                                                \
        hipLaunchKernelGGL(kfn, dim3(wgrid), dim3(256), 0, s, n, p, rp, col, w, D, Q, (T *)nullptr, 0, lam,   \
                           active, lhd, bd, part);                                                           \
    } while (0)
        if (v == 1 && ch == 1) OFKS_WAVE1(1, 1);
        else if (v == 1 && ch <= 2) OFKS_WAVE1(1, 2);
        else if (v == 2 && ch == 1) OFKS_WAVE1(2, 1);
        else if (v == 2 && ch <= 2) OFKS_WAVE1(2, 2);
        else if (v == 2 && ch <= 4) OFKS_WAVE1(2, 4);
        else if (v == 2 && ch <= 8) OFKS_WAVE1(2, 8);
        else if constexpr (sizeof(T) == 4) {
            if (v == 4 && ch == 1) OFKS_WAVE1(4, 1);
            else if (v == 4 && ch <= 2) OFKS_WAVE1(4, 2);
            else if (v == 4 && ch <= 4) OFKS_WAVE1(4, 4);
            else return hipErrorInvalidValue;
        } else return hipErrorInvalidValue;
#undef OFKS_WAVE1
        return hipGetLastError();
    }
#define OFKS_SHIFT(VV, CC, UU)                                                                                        \
    hipLaunchKernelGGL((k_spmm_shift<T, VV, CC, UU, MODE>), dim3(grid), dim3(bs), shm, s, n, p, l2, rp, col, w, lam,  \
                       active, lhd, bd, D, Q, part)
    OFKS_VCH_DISPATCH(OFKS_SHIFT);
#undef OFKS_SHIFT
    return hipGetLastError();
}

template <typename T>
hipError_t launch_spmm_shift(hipStream_t s, int mode, int grid, int64_t n, int p, const int64_t *rp, const int32_t *col,
                             const void *lb, const T *lam, const uint8_t *active, const double *lhd, const double *bd,
                             const T *D, T *Q, double *part, int *blocks_used) {
    if (mode == SHIFT)
        return launch_spmm_shift_mode<SHIFT, T>(s, grid, n, p, rp, col, lb, lam, active, lhd, bd, D, Q, part, blocks_used);
    if (mode == SHIFT_CG)
        return launch_spmm_shift_mode<SHIFT_CG, T>(s, grid, n, p, rp, col, lb, lam, active, lhd, bd, D, Q, part, blocks_used);
    return launch_spmm_shift_mode<SHIFT_DOT, T>(s, grid, n, p, rp, col, lb, lam, active, lhd, bd, D, Q, part, blocks_used);
}

// in, out: four doubles a row; pin, pout: 3 np doubles, np from cg_iter_blocks
hipError_t launch_cg_iter(hipStream_t s, int np, int first, int check, int parity, int64_t nb, int maxlen, const int32_t *info,
                          const int32_t *halo, const int64_t *brp, const uint16_t *lcol, const double *a,
                          const double *dg, const double *in, double *out, double *x, double *sc, const double *pin,
                          double *pout, double *report) {
    const CgIter c{first, check, parity, np, dg, (const double2 *)in, (double2 *)out, x, sc, pin, pout, report};
    const dim3 block(256 * OFKS_CG_TEAMS);
    if (maxlen <= 16)
        hipLaunchKernelGGL((k_cg_iter<1, false>), dim3(np), block, 0, s, nb, info, halo, brp, lcol, a, c);
    else if (maxlen <= 32)
        hipLaunchKernelGGL((k_cg_iter<2, false>), dim3(np), block, 0, s, nb, info, halo, brp, lcol, a, c);
    else hipLaunchKernelGGL((k_cg_iter<2, true>), dim3(np), block, 0, s, nb, info, halo, brp, lcol, a, c);
    return hipGetLastError();
}

hipError_t launch_spmv_dot(hipStream_t s, int grid, int64_t n, const int64_t *rp, const int32_t *col,
                           const double *a, const double *d, double *q, double *part) {
    hipLaunchKernelGGL(k_spmv_dot, dim3(grid), dim3(256), 0, s, n, rp, col, a, d, q, part);
    return hipGetLastError();
}

// Halo-SpMM launch: nb blocks of the plan (grid padded to whole XCD slabs).
// SHIFT_CG and SHIFT_DOT leave *rows_out rows of 2 p partial dots at the start
// of part: sums over groups of HALO_G plan blocks (formed from the per-block
// rows that follow them), or the blocks' own rows up to OFKS_HALO_DIRECT of them
// (ten inner CG iterations, us, own rows against grouped: n = 2.4e4 (381 blocks),
// p = 64 350 and 380; 4.3e4 (670), p = 16 284 and 303; 6.4e4 (1000), p = 11 376
// and 396; 1.2e5 (1838), p = 16 497 and 499; 2.1e5 (3209), p = 16 733 and 710).
// part_capacity in doubles.
#ifndef OFKS_HALO_DIRECT
#define OFKS_HALO_DIRECT 1536
#endif
constexpr int HALO_G = 64, HALO_DIRECT = OFKS_HALO_DIRECT;
static int64_t halo_grid(int64_t nb) { return (nb + 7) / 8 * 8; }

size_t spmm_halo_part_doubles(int64_t nb, int p) {
    const int64_t nbp = halo_grid(nb);
    return (size_t)((nbp + HALO_G - 1) / HALO_G + nbp) * 2 * p;
}

template <typename T>
hipError_t launch_spmm_halo(hipStream_t s, int mode, int64_t nb, int maxlen, int p, const int64_t *row0, const int32_t *info,
                            const int32_t *halo, const int64_t *brp, const uint16_t *lcol, const void *wv, const T *X,
                            T *Y1, T *Y2, int sel, const T *lam, const uint8_t *active, const double *lhd,
                            const double *bd, double *part, size_t part_capacity, int *rows_out) {
    using P2 = typename pair_t<T>::type;
    const P2 *w = (const P2 *)wv;
    const int64_t nbp = halo_grid(nb), ng = nbp <= HALO_DIRECT ? 0 : (nbp + HALO_G - 1) / HALO_G;
    if (nbp <= 0 || nbp > 0x7fffffff) return hipErrorInvalidValue;
    // rows of X, Y1 and Y2 16-byte aligned: 16-byte pieces
    const bool vec = p % (16 / (int)sizeof(T)) == 0 &&
                     (reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Y1) | reinterpret_cast<uintptr_t>(Y2)) % 16 == 0;
    const bool dots = mode == SHIFT_CG || mode == SHIFT_DOT;
    if (dots && (size_t)(ng + nbp) * 2 * p > part_capacity) return hipErrorInvalidValue;
    double *bpart = part + ng * 2 * p;
    // slices per workgroup: all of them once the plan's blocks fill the device
    // (three workgroups on each of 256 CUs), fewer below that
    const int cp = 256 / (int)sizeof(T), ns = (p + cp - 1) / cp;
    const int gy = (int)std::min<int64_t>(ns, (767 + nbp) / nbp), cw = (ns + gy - 1) / gy * cp;
    const dim3 grid((unsigned)nbp, (unsigned)((p + cw - 1) / cw));
#define OFKS_HALO_LAUNCH(M_, S_, R_)                                                                                  \
    hipLaunchKernelGGL((k_spmm_halo<T, M_, S_, R_>), grid, dim3(64 * HALO_WAVES), 0, s, nb, p, cw, row0, info, halo, brp, \
                       lcol, w, X, Y1, Y2, sel, lam, active, lhd, bd, bpart)
#define OFKS_HALO(M_)                                    \
    do {                                                 \
        if (vec && maxlen > 16) OFKS_HALO_LAUNCH(M_, 16, 2); \
        else if (vec) OFKS_HALO_LAUNCH(M_, 16, 1);       \
        else if (maxlen > 16) OFKS_HALO_LAUNCH(M_, 4, 2); \
        else OFKS_HALO_LAUNCH(M_, 4, 1);                 \
    } while (0)
    if (mode == DUAL) OFKS_HALO(DUAL);
    else if (mode == SHIFT) OFKS_HALO(SHIFT);
    else if (mode == SHIFT_CG) OFKS_HALO(SHIFT_CG);
    else OFKS_HALO(SHIFT_DOT);
#undef OFKS_HALO
#undef OFKS_HALO_LAUNCH
    if (dots) {
        // (SHIFT_DOT leaves the second half of each row unset: its sums are not read)
        if (ng) hipLaunchKernelGGL(k_part_rows, dim3((unsigned)ng), dim3(256), 0, s, nbp, 2 * p, HALO_G, bpart, part);
        *rows_out = (int)(ng ? ng : nbp);
    }
    return hipGetLastError();
}

template hipError_t launch_spmm_halo<double>(hipStream_t, int, int64_t, int, int, const int64_t *, const int32_t *,
                                             const int32_t *, const int64_t *, const uint16_t *, const void *,
                                             const double *, double *, double *, int, const double *,
                                             const uint8_t *, const double *, const double *, double *, size_t, int *);
template hipError_t launch_spmm_halo<float>(hipStream_t, int, int64_t, int, int, const int64_t *, const int32_t *,
                                            const int32_t *, const int64_t *, const uint16_t *, const void *,
                                            const float *, float *, float *, int, const float *, const uint8_t *,
                                            const double *, const double *, double *, size_t, int *);
int halo_max_rows() { return HALO_MAX; }
int halo_max_block_rows() { return HALO_RMAX; }
int halo_max_row_entries() { return HALO_EMAX; }
int halo_pad_stride() { return HALO_STRIDE; }
int halo_row_ptr_stride() { return HALO_BRP; }

template hipError_t launch_spmm_pair<double>(hipStream_t, int64_t, int, const int64_t *, const int32_t *,
                                             const void *, const double *, double *, double *, int);
template hipError_t launch_spmm_pair<float>(hipStream_t, int64_t, int, const int64_t *, const int32_t *,
                                            const void *, const float *, float *, float *, int);
template hipError_t launch_spmm_shift<double>(hipStream_t, int, int, int64_t, int, const int64_t *, const int32_t *,
                                              const void *, const double *, const uint8_t *, const double *,
                                              const double *, const double *, double *, double *, int *);
template hipError_t launch_spmm_shift<float>(hipStream_t, int, int, int64_t, int, const int64_t *, const int32_t *,
                                             const void *, const float *, const uint8_t *, const double *,
                                             const double *, const float *, float *, double *, int *);

}  // namespace ofks
