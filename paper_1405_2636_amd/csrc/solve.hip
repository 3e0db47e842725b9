// Triangular solves with the supernodal factor, FP64 residual and the
// refinement helpers (the solve phase of A x = b; the paper states the
// problem, the sweeps are the standard supernodal ones).
//
// Forward sweep, column blocks in ascending dependency levels:
//   z_k = L_kk^{-1} y_k                   (diagonal rows split over workgroups)
//   y[rows of k] -= L_k,off z_k           (64-row chunks, FP64 atomics)
// Backward sweep, levels descending:
//   t_k  = L_k,off^T x[rows of k]         (64- or 256-row chunks)
//   x_k  = L_kk^{-T} (z_k - t_k)
// Both use the inverse of each diagonal block kept by the factorization.
// On the narrow levels two consecutive pieces p, q of a split supernode are
// one block of the sweeps: the diagonal steps use the pair's inverse
// (pair_inv, formed after each factorization), so p's rows facing q are left
// out of its off-diagonal steps.  Every launch reads its work from a list of
// self-contained items (DiagItem, OffItem) built once per analysis.
// Several right-hand sides are handled in blocks of up to 8 per pass over
// the panels (each loaded entry serves the whole block); with 4 or 8 the
// off-diagonal steps are matrix-core products (fwd_off_mm, bwd_off_mm).
// Column blocks of width <= 32 with at most 128 panel rows take both halves
// of a step in one kernel per level, a wave or 16 lanes per block
// (fwd_small, bwd_small).
// Every sweep step writes a different vector than it reads (y -> z -> x), so
// a diagonal block can be spread over several workgroups.  Every dot product
// is split over 4, 16 or 32 lanes (interleaved inner indices) and combined by
// shuffles: that many times fewer dependent load rounds per thread than a
// one-lane loop.  The sweeps stream the panels once each: they are bound by
// HBM bandwidth and, on the narrow top levels, by load latency.
// The factor is read in its storage type T (double, or float in the FP32
// refinement mode); vectors and arithmetic are FP64 in both cases.
// L U (unit L and U in the square diagonal blocks, L below them, U^T in a
// second panel array of the same layout, kept inverses L_kk^{-1} and
// U_kk^{-T}): the forward sweep reads L and L_kk^{-1}, the backward sweep the
// U^T panels and U_kk^{-T} (x_k = U_kk^{-1} (z_k - t_k), t_k = U_k,off x[rows])
// in the places of L and L_kk^{-1}.
// L D L^T (unit L, d_j on the panel diagonal, kept inverse Y = D^{-1} L^{-1}):
// the same steps give w_k = Y_kk y_k = D_k^{-1} z_k in z, so the forward rows
// below take D_k w_k, and the backward step x_k = L_kk^{-T} (w_k - t_k) is
// Y_kk^T applied to D_k (w_k - t_k); the scaling by d is applied where z_k
// and z_k - t_k are staged.
#include "device.hpp"

namespace spx {

constexpr int kChunk = 64;     // off-diagonal rows per chunk of the level lists

// sum over the LANES consecutive lanes of a group (LANES = 4, 16 or 32)
template <int LANES>
__device__ __forceinline__ double group_sum(double v)
{
#pragma unroll
    for (int o = 1; o < LANES; o <<= 1) v += __shfl_xor(v, o);
    return v;
}

// Every sweep kernel handles the right-hand sides in blocks of NR (1, 4 or
// 8; chosen from nrhs at launch): the panel and inverse entries a thread
// loads serve all NR columns of the block, so a panel is read once per
// block of right-hand sides instead of once per right-hand side.  The
// kernels take one block per grid row (a loop
// over the blocks kept the loop-invariant addresses of the hoisted loads
// live: 150-210 registers per lane instead of 85-135, and half the
// resident waves).
// (staged vectors: element c of right-hand side j at [c * NR + j]; a masked
// term is formed as 0 * value, so clamped indices stay inside the staged
// entries: a value read from unwritten LDS may be NaN)

// cnt values, s[idx] = fin(i, load(idx)), idx = threadIdx.x + 256 i: all N loads
// of a thread before the first use (j = idx % NR is the same for all of them)
template <int N, class F, class G>
__device__ __forceinline__ void stage(double* s, int cnt, F load, G fin)
{
    const int tid = threadIdx.x;
    double v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        v[i] = 0.0;
        if (256 * i < cnt) v[i] = load(min(tid + 256 * i, cnt - 1));
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (tid + 256 * i < cnt) s[tid + 256 * i] = fin(i, v[i]);
}

// ---- forward, diagonal block: z_k = D y_k, D = L_kk^{-1} (lower, w x w,
// column-major).  LANES lanes per row, one workgroup per item: the rows
// r0 .. r0 + 256/LANES - 1 of one block; lane q of a row takes the
// columns p = q, q+LANES, ..., sixteen loads at a time (p > row clamped and
// multiplied by zero).  Narrow levels (few blocks) use 16 lanes, or 32 when
// they hold a pair of pieces (a 512-wide inverse): fewer dependent load
// rounds; wide levels 4 (the items of a level are cut to match).  ys:
// kMaxPairWidth * NR
template <class T, int LANES, int NR>
__device__ __forceinline__ void fwd_diag_step(const SweepArgs& a, const DiagItem& it, int rb, double* ys)
{
    const int f = it.f, w = it.w, r0 = it.r0;
    const T* D = static_cast<const T*>(a.dinv) + it.dofs;
    const int tid = threadIdx.x, q = tid % LANES, row = min(r0 + tid / LANES, w - 1);
    const int nv = min(NR, a.nrhs - rb);
    T d[16];   // the first sixteen loads are issued before the staging barrier
#pragma unroll
    for (int u = 0; u < 16; ++u) d[u] = D[(uint32_t)(row + min(q + LANES * u, row) * w)];
    stage<2 * NR>(ys, w * NR, [&](int idx) {
        return a.y[(int64_t)(rb + min(idx % NR, nv - 1)) * a.n + f + idx / NR];
    }, [&](int, double v) { return tid % NR < nv ? v : 0.0; });
    __syncthreads();
    double v[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) v[j] = 0.0;
    for (int pb = 0; pb <= row; pb += 16 * LANES) {
        if (pb != 0) {
#pragma unroll
            for (int u = 0; u < 16; ++u) d[u] = D[(uint32_t)(row + min(pb + q + LANES * u, row) * w)];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int p = pb + q + LANES * u;
            const double dv = p <= row ? (double)d[u] : 0.0;
            const double* yp = ys + min(p, w - 1) * NR;
#pragma unroll
            for (int j = 0; j < NR; ++j) v[j] += dv * yp[j];
        }
    }
#pragma unroll
    for (int j = 0; j < NR; ++j) v[j] = group_sum<LANES>(v[j]);
    if (r0 + tid / LANES < w && q == 0)
        for (int j = 0; j < nv; ++j) a.z[(int64_t)(rb + j) * a.n + f + row] = v[j];
}
template <class T, int LANES, int NR>
__global__ void __launch_bounds__(256) fwd_diag(SweepArgs a, const DiagItem* items)
{
    __shared__ double ys[kMaxPairWidth * NR];
    fwd_diag_step<T, LANES, NR>(a, items[blockIdx.x], blockIdx.y * NR, ys);
}

// ---- forward, off-diagonal rows, one right-hand side: y[g(r)] -= sum_c
// L[r, c] z_k[c].  One workgroup per item: up to 64 panel rows from row0 by
// the columns c0..c1-1 (levels with few row chunks split each chunk's columns
// over several items so that the launch fills the chip; their partial sums
// meet in the atomics).  Lane = row (each load covers 64 consecutive rows of
// one column), wave v = quarter v of the columns, issued 16 at a time, the
// first sixteen before the staging barrier; the four partial sums meet in
// LDS.
template <class T>
__global__ void __launch_bounds__(256) fwd_off(SweepArgs a, const OffItem* items)
{
    __shared__ double zk[256], part[4 * 64];
    const OffItem it = items[blockIdx.x];
    const int f = it.f, c0 = it.cnr & 511, c1 = (it.cnr >> 9) & 511, nr = it.cnr >> 18;
    const int64_t ld = it.ld;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = min(lane, nr - 1);
    const int gi = a.rowg[it.gofs + r];   // global row of the lane's panel row (read ahead of the products)
    const int qw = (c1 - c0 + 3) >> 2, cb = c0 + wave * qw, ce = min(c1, cb + qw);
    const T* Lr = static_cast<const T*>(a.panels) + it.pofs + r;
    const T* Pd = static_cast<const T*>(a.panels) + (it.pofs - it.row0);   // d_c at c * (ld + 1) (L D L^T)
    T l[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) l[u] = Lr[(int64_t)min(cb + u, c1 - 1) * ld];
    const int cz = min(c0 + tid, c1 - 1);
    const double dz = a.ldlt ? (double)Pd[cz * (ld + 1)] : 1.0;
    const double z = a.z[f + cz];
    if (c0 + tid < c1) zk[tid] = z * dz;
    __syncthreads();
    double v = 0.0;
    for (int c = cb; c < ce; c += 16) {
        if (c != cb) {
#pragma unroll
            for (int u = 0; u < 16; ++u) l[u] = Lr[(int64_t)min(c + u, ce - 1) * ld];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) v += (c + u < ce ? (double)l[u] : 0.0) * zk[min(c + u, ce - 1) - c0];
    }
    part[wave * 64 + lane] = v;
    __syncthreads();
    if (wave == 0 && lane < nr)
        unsafeAtomicAdd(a.y + gi, -((part[lane] + part[64 + lane]) + (part[128 + lane] + part[192 + lane])));
}

// ---- backward, off-diagonal rows, one right-hand side: tacc[f + c] +=
// sum_r L[r, c] x[g(r)].  One workgroup per item: up to 16 LANES panel rows
// from row0 by the columns c0 .. c1 - 1, 256 / LANES columns at a time; LANES
// lanes per column, lane q takes the rows q, q + LANES, ... with all sixteen
// loads in flight (the first block's before the staging barrier).  LANES = 4:
// 64-row items, the forward kernel's (wide levels: many blocks, few rows
// each); LANES = 16: 256-row items of 16 columns (narrow levels; their blocks
// have thousands of rows: a column of tacc then takes one atomic add per 256
// rows instead of per 64, and each load instruction covers 16 consecutive
// rows of four columns instead of four rows of sixteen).
template <class T, int LANES>
__global__ void __launch_bounds__(256) bwd_off(SweepArgs a, const OffItem* items)
{
    __shared__ double xr[16 * LANES];
    const OffItem it = items[blockIdx.x];
    constexpr int COLS = 256 / LANES;
    const int f = it.f, c0 = it.cnr & 511, c1 = (it.cnr >> 9) & 511, nr = it.cnr >> 18;
    const int64_t ld = it.ld;
    const int tid = threadIdx.x, q = tid % LANES, cl = tid / LANES;
    const T* L = static_cast<const T*>(a.panels_b) + it.pofs;
    // global row of the thread's staged entry, loaded ahead of the panel: the
    // gather then waits for it only, not for the panel loads issued after it
    const int gv = a.rowg[it.gofs + min(tid, nr - 1)];
    T l[16];
    {
        const T* Lc = L + (int64_t)min(c0 + cl, c1 - 1) * ld;
#pragma unroll
        for (int u = 0; u < 16; ++u) l[u] = Lc[min(q + LANES * u, nr - 1)];
    }
    if (tid < nr) xr[tid] = a.x[gv];
    __syncthreads();
    for (int cb = c0; cb < c1; cb += COLS) {
        const int c = min(cb + cl, c1 - 1);
        if (cb != c0) {
            const T* Lc = L + (int64_t)c * ld;
#pragma unroll
            for (int u = 0; u < 16; ++u) l[u] = Lc[min(q + LANES * u, nr - 1)];
        }
        double v = 0.0;
#pragma unroll
        for (int u = 0; u < 16; ++u) v += (q + LANES * u < nr ? (double)l[u] : 0.0) * xr[min(q + LANES * u, nr - 1)];
        v = group_sum<LANES>(v);
        if (cb + cl < c1 && q == 0) unsafeAtomicAdd(a.tacc + f + c, v);
    }
}

// ---- off-diagonal steps for blocks of NR = 4 or 8 right-hand sides, on
// the matrix cores (v_mfma_f64_16x16x4f64: operand A lane l holds
// A[l%16][l/16], operand B lane l holds B[l/16][l%16], result slot v of
// lane l holds D[4v + l/16][l%16]); FP32 panels are converted, so the
// arithmetic stays FP64.  With several right-hand sides the scalar kernels
// spend a product and an LDS read per loaded entry and right-hand side:
// they were bound by that, not by the panel bytes.
typedef double sw_d4 __attribute__((ext_vector_type(4)));

// forward: y[g(r)] -= (L z)[r] over the item's 64 rows and columns c0..c1.
// Wave v takes a quarter of the columns, all four 16-row tiles (A = panel
// rows, B = the staged z, right-hand sides past NR zero), the first sixteen
// columns before the staging barrier; the four waves' partial sums meet in
// LDS.
template <class T, int NR>
__global__ void __launch_bounds__(256) fwd_off_mm(SweepArgs a, const OffItem* items)
{
    __shared__ double zk[256 * NR], part[4 * 64 * NR];
    const OffItem it = items[blockIdx.x];
    const int rb = blockIdx.y * NR;
    const int f = it.f, c0 = it.cnr & 511, c1 = (it.cnr >> 9) & 511, nr = it.cnr >> 18;
    const int64_t ld = it.ld;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
    const int nv = min(NR, a.nrhs - rb);
    const int qw = (((c1 - c0 + 3) >> 2) + 3) & ~3;   // a wave's columns, a multiple of 4
    const int cb = c0 + wave * qw, ce = min(c1, cb + qw);
    const T* L = static_cast<const T*>(a.panels) + it.pofs;
    const T* Pd = static_cast<const T*>(a.panels) + (it.pofs - it.row0);   // d_c at c * (ld + 1) (L D L^T)
    constexpr int NG = NR / 4;   // rows of y per thread
    int gr[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) gr[i] = a.rowg[it.gofs + min((tid + 256 * i) / NR, nr - 1)];
    // (columns past ce read a clamped column and meet B = 0; rows past nr
    // read a clamped row whose results are not stored)
    T al[4][4];
    auto load = [&](int k0) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                al[t][s] = L[min(16 * t + li, nr - 1) + (int64_t)min(k0 + 4 * s + lk, c1 - 1) * ld];
    };
    load(cb);
    const int n0 = (c1 - c0) * NR;
    double dz[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i)
        dz[i] = a.ldlt && 256 * i < n0 ? (double)Pd[min(c0 + (tid + 256 * i) / NR, c1 - 1) * (ld + 1)] : 1.0;
    stage<NR>(zk, n0, [&](int idx) {
        return a.z[(int64_t)(rb + min(idx % NR, nv - 1)) * a.n + f + c0 + idx / NR];
    }, [&](int i, double v) { return tid % NR < nv ? v * dz[i] : 0.0; });
    __syncthreads();
    sw_d4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = sw_d4{0, 0, 0, 0};
    for (int k0 = cb; k0 < ce; k0 += 16) {
        if (k0 != cb) load(k0);
        double bz[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int c = k0 + 4 * s + lk;
            bz[s] = (c < ce && li < NR) ? zk[(min(c, ce - 1) - c0) * NR + li] : 0.0;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)al[t][s], bz[s], acc[t], 0, 0, 0);
    }
    if (li < NR)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[(wave * 64 + 16 * t + 4 * v + lk) * NR + li] = acc[t][v];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        const int idx = tid + 256 * i, r = idx / NR, j = idx % NR;
        if (r < nr && j < nv) {
            const double sum = (part[r * NR + j] + part[(64 + r) * NR + j]) +
                               (part[(128 + r) * NR + j] + part[(192 + r) * NR + j]);
            unsafeAtomicAdd(a.y + (int64_t)(rb + j) * a.n + gr[i], -sum);
        }
    }
}

// backward: tacc[f + c] += (L^T x)[c] over the item's rows.  A = the staged
// x (right-hand side by row, rows past nr zero), B = 16 panel columns; wave
// v takes the column tiles c0 + 16 v, c0 + 16 (v + 4), ...
template <class T, int NR>
__global__ void __launch_bounds__(256) bwd_off_mm(SweepArgs a, const OffItem* items)
{
    __shared__ double xr[kChunk * NR];
    const OffItem it = items[blockIdx.x];
    const int rb = blockIdx.y * NR;
    const int f = it.f, c0 = it.cnr & 511, c1 = (it.cnr >> 9) & 511, nr = it.cnr >> 18;
    const int64_t ld = it.ld;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
    const int nv = min(NR, a.nrhs - rb);
    const T* L = static_cast<const T*>(a.panels_b) + it.pofs;
    constexpr int NG = kChunk * NR / 256;
    int gr[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) gr[i] = a.rowg[it.gofs + min((tid + 256 * i) / NR, nr - 1)];
    T bl[16];
    auto load = [&](int cb) {
        const T* Lc = L + (int64_t)min(cb + li, c1 - 1) * ld;
#pragma unroll
        for (int s = 0; s < 16; ++s) bl[s] = Lc[min(4 * s + lk, nr - 1)];
    };
    load(c0 + 16 * wave);
    double xg[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) xg[i] = a.x[(int64_t)(rb + min((tid + 256 * i) % NR, nv - 1)) * a.n + gr[i]];
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        const int idx = tid + 256 * i;
        xr[idx] = idx / NR < nr && idx % NR < nv ? xg[i] : 0.0;
    }
    __syncthreads();
    double ax[16];   // A[rhs = li][row = 4 s + lk]
#pragma unroll
    for (int s = 0; s < 16; ++s) ax[s] = li < NR ? xr[(4 * s + lk) * NR + li] : 0.0;
    for (int cb = c0 + 16 * wave; cb < c1; cb += 64) {
        if (cb != c0 + 16 * wave) load(cb);
        sw_d4 acc = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < 16; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ax[s], (double)bl[s], acc, 0, 0, 0);
        if (cb + li < c1)
#pragma unroll
            for (int v = 0; v < NR / 4; ++v)
                if (4 * v + lk < nv) unsafeAtomicAdd(a.tacc + (int64_t)(rb + 4 * v + lk) * a.n + f + cb + li, acc[v]);
    }
}

// ---- backward, diagonal block: x_k = D^T (z_k - t_k); LANES lanes per
// column c of D, lane q takes the rows p = c+q, c+q+LANES, ... (p >= w
// clamped and multiplied by zero); the forward kernel's items, columns
// r0 .. r0 + 256/LANES - 1.  zs: kMaxPairWidth * NR
template <class T, int LANES, int NR>
__device__ __forceinline__ void bwd_diag_step(const SweepArgs& a, const DiagItem& it, int rb, double* zs)
{
    const int f = it.f, w = it.w, c0 = it.r0;
    const T* D = static_cast<const T*>(a.dinv_b) + it.dofs;
    const int tid = threadIdx.x, q = tid % LANES, col = min(c0 + tid / LANES, w - 1);
    const T* Pd = static_cast<const T*>(a.panels) + it.pofs;    // L D L^T: d_c, c < w1, at c * (ld + 1)
    const T* Pd2 = static_cast<const T*>(a.panels) + it.pofs2;  // and c >= w1 at (c - w1) * (ld2 + 1)
    const int64_t ld = it.ld, ld2 = it.ld2;
    const int w1 = it.w1;
    const int nv = min(NR, a.nrhs - rb);
    T d[16];   // the first sixteen loads are issued before the staging barrier
#pragma unroll
    for (int u = 0; u < 16; ++u) d[u] = D[(uint32_t)(col * w + min(col + q + LANES * u, w - 1))];
    double zr[2 * NR], dz[2 * NR];   // z and d of the thread's staged entries
#pragma unroll
    for (int i = 0; i < 2 * NR; ++i) {
        zr[i] = 0.0;
        dz[i] = 1.0;
        if (256 * i < w * NR) {
            const int idx = tid + 256 * i, c = min(idx / NR, w - 1);
            zr[i] = a.z[(int64_t)(rb + min(idx % NR, nv - 1)) * a.n + f + c];
            if (a.ldlt) dz[i] = (double)(c < w1 ? Pd[c * (ld + 1)] : Pd2[(c - w1) * (ld2 + 1)]);
        }
    }
    stage<2 * NR>(zs, w * NR, [&](int idx) {
        return a.tacc[(int64_t)(rb + min(idx % NR, nv - 1)) * a.n + f + idx / NR];
    }, [&](int i, double v) { return tid % NR < nv ? (zr[i] - v) * dz[i] : 0.0; });
    __syncthreads();
    double v[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) v[j] = 0.0;
    for (int pb = col; pb < w; pb += 16 * LANES) {
        if (pb != col) {
#pragma unroll
            for (int u = 0; u < 16; ++u) d[u] = D[(uint32_t)(col * w + min(pb + q + LANES * u, w - 1))];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int p = pb + q + LANES * u;
            const double dv = p < w ? (double)d[u] : 0.0;
            const double* zp = zs + min(p, w - 1) * NR;
#pragma unroll
            for (int j = 0; j < NR; ++j) v[j] += dv * zp[j];
        }
    }
#pragma unroll
    for (int j = 0; j < NR; ++j) v[j] = group_sum<LANES>(v[j]);
    if (c0 + tid / LANES < w && q == 0)
        for (int j = 0; j < nv; ++j) a.x[(int64_t)(rb + j) * a.n + f + col] = v[j];
}
template <class T, int LANES, int NR>
__global__ void __launch_bounds__(256) bwd_diag(SweepArgs a, const DiagItem* items)
{
    __shared__ double zs[kMaxPairWidth * NR];
    bwd_diag_step<T, LANES, NR>(a, items[blockIdx.x], blockIdx.y * NR, zs);
}

// ---- small blocks (width <= 32, at most 128 panel rows), both halves of a
// sweep step in one kernel per level.  Two sizes in one launch: tiny blocks
// (width <= 8, at most 32 rows), 16 lanes each, 16 per workgroup (the bottom
// levels of small systems hold tens of thousands of blocks a few columns
// wide), and the others, a wave each, 4 per workgroup; one block of right-hand
// sides per grid row.  What bounds them is latency: a level is a few
// microseconds, and its launches follow each other.  So every block has a
// record with all of its offsets, and its inverse, its panel (the whole of a
// tiny one, the first columns of a larger one), its row numbers and its part
// of the vector are requested in one go after it: two round trips to memory
// instead of one per four or eight columns.  256 grids of side 16 to 96, one
// right-hand side, 18 levels: 344 -> 212 us forward, 324 -> 179 backward (16
// lanes for every block, four or eight columns per round trip); 48^3 with 13
// right-hand sides, 3 levels: 358 -> 48 and 506 -> 58 us (the blocks of
// right-hand sides were a loop of two at a time inside the kernels).
// Lanes without a block leave at once: a chain has one block per level, and
// the other lanes repeating its loads made a level of it 2.8 us instead of
// 2.2 (band of 3 in natural order, 1558 levels, one right-hand side 8.78 ->
// 6.91 ms, two 12.28 -> 9.85).
constexpr int kSG = 16;                    // lanes per tiny block
constexpr int kSGroups = 256 / kSG;        // tiny blocks per workgroup

// forward, tiny block: z_k = D y_k, then y[g(r)] -= L[r, :] z_k
template <class T, int NR>
__device__ __forceinline__ void fwd_tiny(const SweepArgs& a, const SmallItem& it, int rb)
{
    const int l = threadIdx.x % kSG, w = it.w(), ld = it.ld(), f = it.f;
    const T* D = static_cast<const T*>(a.dinv) + it.dofs;
    const T* L = static_cast<const T*>(a.panels) + it.pofs;
    const int nv = min(NR, a.nrhs - rb);
    const int lw = min(l, w - 1);
    T d[8], lv[2][8];
    int g[2];
    double y[NR];
    // (indices past the triangle or the panel are clamped, their terms
    // multiplied by zero or not stored)
#pragma unroll
    for (int p = 0; p < 8; ++p) d[p] = D[lw + min(p, lw) * w];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int c = 0; c < 8; ++c) lv[i][c] = L[min(w + l + kSG * i, ld - 1) + min(c, w - 1) * ld];
#pragma unroll
    for (int i = 0; i < 2; ++i) g[i] = ld > w ? a.rowg[it.gofs + min(l + kSG * i, ld - w - 1)] : 0;
    const double s = a.ldlt ? (double)L[lw * (ld + 1)] : 1.0;
#pragma unroll
    for (int j = 0; j < NR; ++j) y[j] = a.y[(int64_t)(rb + min(j, nv - 1)) * a.n + f + lw];
    double z[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        z[j] = 0.0;
#pragma unroll
        for (int p = 0; p < 8; ++p) z[j] += (p <= lw ? (double)d[p] : 0.0) * __shfl(y[j], p, kSG);
        if (l < w && j < nv) a.z[(int64_t)(rb + j) * a.n + f + l] = z[j];
        z[j] *= s;
        double v[2] = {0.0, 0.0};
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const double zc = c < w ? __shfl(z[j], c, kSG) : 0.0;
#pragma unroll
            for (int i = 0; i < 2; ++i) v[i] += (double)lv[i][c] * zc;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (w + l + kSG * i < ld && j < nv) unsafeAtomicAdd(a.y + (int64_t)(rb + j) * a.n + g[i], -v[i]);
    }
}

// forward, a wave: lane = row and half of the columns of D, then lane = row
// below (two of them)
template <class T, int NR>
__device__ __forceinline__ void fwd_wave(const SweepArgs& a, const SmallItem& it, int rb, double* ys,
                                         double* zs)
{
    const int lane = threadIdx.x & 63, w = it.w(), ld = it.ld(), f = it.f, R = ld - w;
    const T* D = static_cast<const T*>(a.dinv) + it.dofs;
    const T* L = static_cast<const T*>(a.panels) + it.pofs;
    const int nv = min(NR, a.nrhs - rb);
    const int r = lane & 31, half = lane >> 5, rw = min(r, w - 1);
    T d[16], lv[2][8];
    int g[2];
#pragma unroll
    for (int i = 0; i < 16; ++i) d[i] = D[rw + min(2 * i + half, rw) * w];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int c = 0; c < 8; ++c) lv[i][c] = L[min(w + lane + 64 * i, ld - 1) + min(c, w - 1) * ld];
#pragma unroll
    for (int i = 0; i < 2; ++i) g[i] = R > 0 ? a.rowg[it.gofs + min(lane + 64 * i, R - 1)] : 0;
    const double s = a.ldlt ? (double)L[rw * (ld + 1)] : 1.0;
    {
        constexpr int NY = (32 * NR + 63) / 64;
        double yv[NY];
#pragma unroll
        for (int i = 0; i < NY; ++i) {
            const int idx = lane + 64 * i;
            yv[i] = a.y[(int64_t)(rb + min(idx % NR, nv - 1)) * a.n + f + min(idx / NR, w - 1)];
        }
#pragma unroll
        for (int i = 0; i < NY; ++i) {
            const int idx = lane + 64 * i;
            if (idx < 32 * NR) ys[idx] = idx / NR < w && idx % NR < nv ? yv[i] : 0.0;
        }
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);   // (LDS operations of a wave complete in order)
    double z[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) z[j] = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const double dv = 2 * i + half <= rw ? (double)d[i] : 0.0;
#pragma unroll
        for (int j = 0; j < NR; ++j) z[j] += dv * ys[(2 * i + half) * NR + j];
    }
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        z[j] += __shfl_xor(z[j], 32);
        if (half == 0) zs[r * NR + j] = r < w ? z[j] * s : 0.0;
        if (half == 0 && r < w && j < nv) a.z[(int64_t)(rb + j) * a.n + f + r] = z[j];
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    if (R <= 0) return;
    double v[2][NR];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NR; ++j) v[i][j] = 0.0;
#pragma unroll 1
    for (int c0 = 0; c0 < w; c0 += 8) {
        T ln[2][8];   // the next eight columns, on their way
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int c = 0; c < 8; ++c) ln[i][c] = L[min(w + lane + 64 * i, ld - 1) + min(c0 + 8 + c, w - 1) * ld];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const double* zc = zs + (c0 + c) * NR;   // (zero past w)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < NR; ++j) v[i][j] += (double)lv[i][c] * zc[j];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int c = 0; c < 8; ++c) lv[i][c] = ln[i][c];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (lane + 64 * i < R)
            for (int j = 0; j < nv; ++j) unsafeAtomicAdd(a.y + (int64_t)(rb + j) * a.n + g[i], -v[i][j]);
}

// workgroup b of a level's small blocks: ceil(ntiny / 16) of tiny ones, then
// ceil((count - ntiny) / 4) of the others.  sm: 4 * 2 * 32 * NR
template <class T, int NR>
__device__ __forceinline__ void fwd_small_step(const SweepArgs& a, const SmallItem* items, int count, int ntiny, int b,
                                               int rb, double* sm)
{
    const int nt = (ntiny + kSGroups - 1) / kSGroups, tid = threadIdx.x;
    if (b < nt) {
        const int idx = b * kSGroups + tid / kSG;
        if (idx >= ntiny) return;
        const SmallItem it = items[idx];
        fwd_tiny<T, NR>(a, it, rb);
    } else {
        const int wave = tid >> 6, idx = ntiny + (b - nt) * 4 + wave;
        if (idx >= count) return;
        const SmallItem it = items[idx];
        fwd_wave<T, NR>(a, it, rb, sm + wave * 64 * NR, sm + wave * 64 * NR + 32 * NR);
    }
}
template <class T, int NR>
__global__ void __launch_bounds__(256) fwd_small(SweepArgs a, const SmallItem* items, int count, int ntiny)
{
    __shared__ double sm[4 * 64 * NR];
    fwd_small_step<T, NR>(a, items, count, ntiny, blockIdx.x, blockIdx.y * NR, sm);
}

// backward, tiny block: t = L_off^T x[g(rows below)], x_k = D^T (z_k - t)
template <class T, int NR>
__device__ __forceinline__ void bwd_tiny(const SweepArgs& a, const SmallItem& it, int rb)
{
    const int l = threadIdx.x % kSG, w = it.w(), ld = it.ld(), f = it.f;
    const T* D = static_cast<const T*>(a.dinv_b) + it.dofs;
    const T* L = static_cast<const T*>(a.panels_b) + it.pofs;
    const int nv = min(NR, a.nrhs - rb);
    // after the sums below lane l holds column (l >> 1) & 7; lane c of the
    // first eight takes column c of D^T
    const int cs = (l >> 1) & 7, cw = min(cs, w - 1), lw = min(l, w - 1);
    int g[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) g[i] = ld > w ? a.rowg[it.gofs + min(l + kSG * i, ld - w - 1)] : 0;
    T d[8], lv[2][8];
#pragma unroll
    for (int p = 0; p < 8; ++p) d[p] = D[min(max(p, lw), w - 1) + lw * w];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int c = 0; c < 8; ++c) lv[i][c] = L[min(w + l + kSG * i, ld - 1) + min(c, w - 1) * ld];
    const double s = a.ldlt ? (double)L[cw * (ld + 1)] : 1.0;
    double zc[NR], x[2][NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) zc[j] = a.z[(int64_t)(rb + min(j, nv - 1)) * a.n + f + cw];
#pragma unroll
    for (int j = 0; j < NR; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i) x[i][j] = a.x[(int64_t)(rb + min(j, nv - 1)) * a.n + g[i]];
#pragma unroll
    for (int j = 0; j < NR; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i) x[i][j] = w + l + kSG * i < ld ? x[i][j] : 0.0;
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        double t[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) t[c] = (double)lv[0][c] * x[0][j] + (double)lv[1][c] * x[1][j];
        // sums over the 16 lanes, half of the columns handed over per step
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double keep = l & 8 ? t[c + 4] : t[c], give = l & 8 ? t[c] : t[c + 4];
            t[c] = keep + __shfl_xor(give, 8);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const double keep = l & 4 ? t[c + 2] : t[c], give = l & 4 ? t[c] : t[c + 2];
            t[c] = keep + __shfl_xor(give, 4);
        }
        const double keep = l & 2 ? t[1] : t[0], give = l & 2 ? t[0] : t[1];
        t[0] = keep + __shfl_xor(give, 2);
        t[0] += __shfl_xor(t[0], 1);
        const double u = (zc[j] - t[0]) * s;   // column cs
        double v = 0.0;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            const double up = __shfl(u, 2 * p, kSG);
            v += (p >= l && p < w ? (double)d[p] : 0.0) * (p < w ? up : 0.0);
        }
        if (l < w && j < nv) a.x[(int64_t)(rb + j) * a.n + f + l] = v;
    }
}

// backward, a wave: lane = column and half of the rows below, then of the
// rows of D
template <class T, int NR>
__device__ __forceinline__ void bwd_wave(const SweepArgs& a, const SmallItem& it, int rb, double* xs,
                                         double* us)
{
    const int lane = threadIdx.x & 63, w = it.w(), ld = it.ld(), f = it.f, R = ld - w;
    const T* D = static_cast<const T*>(a.dinv_b) + it.dofs;
    const T* L = static_cast<const T*>(a.panels_b) + it.pofs;
    const int nv = min(NR, a.nrhs - rb);
    const int c = lane & 31, half = lane >> 5, cw = min(c, w - 1);
    int g[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) g[i] = R > 0 ? a.rowg[it.gofs + min(lane + 64 * i, R - 1)] : 0;
    T d[16], lv[8];
    const int Rh = (R + 1) / 2, rs = half * Rh, re = min(R, rs + Rh);   // this half's rows below
    const T* Lc = L + (int64_t)cw * ld + w;
#pragma unroll
    for (int u = 0; u < 8; ++u) lv[u] = Lc[min(rs + u, ld - w - 1)];
#pragma unroll
    for (int i = 0; i < 16; ++i) d[i] = D[min(max(2 * i + half, cw), w - 1) + cw * w];
    const double s = a.ldlt ? (double)L[cw * (ld + 1)] : 1.0;
    double zc[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) zc[j] = a.z[(int64_t)(rb + min(j, nv - 1)) * a.n + f + cw];
    {
        double xv[2][NR];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NR; ++j) xv[i][j] = a.x[(int64_t)(rb + min(j, nv - 1)) * a.n + g[i]];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NR; ++j) xs[(lane + 64 * i) * NR + j] = lane + 64 * i < R && j < nv ? xv[i][j] : 0.0;
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);   // (LDS operations of a wave complete in order)
    double t[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) t[j] = 0.0;
#pragma unroll 1
    for (int r0 = rs; r0 < re; r0 += 8) {
        T ln[8];   // the next eight rows, on their way
#pragma unroll
        for (int u = 0; u < 8; ++u) ln[u] = Lc[min(r0 + 8 + u, ld - w - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const double lu = r0 + u < re ? (double)lv[u] : 0.0;
            const double* xp = xs + min(r0 + u, 127) * NR;
#pragma unroll
            for (int j = 0; j < NR; ++j) t[j] += lu * xp[j];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) lv[u] = ln[u];
    }
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        t[j] += __shfl_xor(t[j], 32);
        if (half == 0) us[c * NR + j] = c < w ? (zc[j] - t[j]) * s : 0.0;
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    double v[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) v[j] = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int p = 2 * i + half;
        const double dv = p >= c && p < w ? (double)d[i] : 0.0;
#pragma unroll
        for (int j = 0; j < NR; ++j) v[j] += dv * us[p * NR + j];
    }
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        v[j] += __shfl_xor(v[j], 32);
        if (half == 0 && c < w && j < nv) a.x[(int64_t)(rb + j) * a.n + f + c] = v[j];
    }
}

// sm: 4 * 160 * NR
template <class T, int NR>
__device__ __forceinline__ void bwd_small_step(const SweepArgs& a, const SmallItem* items, int count, int ntiny, int b,
                                               int rb, double* sm)
{
    const int nt = (ntiny + kSGroups - 1) / kSGroups, tid = threadIdx.x;
    if (b < nt) {
        const int idx = b * kSGroups + tid / kSG;
        if (idx >= ntiny) return;
        const SmallItem it = items[idx];
        bwd_tiny<T, NR>(a, it, rb);
    } else {
        const int wave = tid >> 6, idx = ntiny + (b - nt) * 4 + wave;
        if (idx >= count) return;
        const SmallItem it = items[idx];
        bwd_wave<T, NR>(a, it, rb, sm + wave * 160 * NR, sm + wave * 160 * NR + 128 * NR);
    }
}
template <class T, int NR>
__global__ void __launch_bounds__(256) bwd_small(SweepArgs a, const SmallItem* items, int count, int ntiny)
{
    __shared__ double sm[4 * 160 * NR];
    bwd_small_step<T, NR>(a, items, count, ntiny, blockIdx.x, blockIdx.y * NR, sm);
}

// ---- both kinds of a level in one launch, one right-hand side: nd diagonal
// items, then the small blocks (a launch of the graph takes about 4.5 us
// however little it does; with 4 or 8 right-hand sides the small blocks need
// 256 registers, which would halve the diagonal items' waves: two launches)
template <class T, int LANES>
__global__ void __launch_bounds__(256) fwd_level(SweepArgs a, const DiagItem* ditems, int nd, const SmallItem* items,
                                                 int count, int ntiny)
{
    __shared__ double sm[kMaxPairWidth];
    const int b = blockIdx.x;
    if (b < nd) fwd_diag_step<T, LANES, 1>(a, ditems[b], 0, sm);
    else fwd_small_step<T, 1>(a, items, count, ntiny, b - nd, 0, sm);
}
template <class T, int LANES>
__global__ void __launch_bounds__(256) bwd_level(SweepArgs a, const DiagItem* ditems, int nd, const SmallItem* items,
                                                 int count, int ntiny)
{
    __shared__ double sm[4 * 160];
    const int b = blockIdx.x;
    if (b < nd) bwd_diag_step<T, LANES, 1>(a, ditems[b], 0, sm);
    else bwd_small_step<T, 1>(a, items, count, ntiny, b - nd, 0, sm);
}

// ---- vector kernels
// y = the permuted right-hand sides, t = 0 (the backward partial sums)
__global__ void permute_in(double* y, double* t, const double* b, int64_t ldb, const int32_t* perm, int32_t n,
                           int32_t nrhs)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t p = perm[i];
        for (int32_t c = blockIdx.y; c < nrhs; c += gridDim.y) {
            y[(int64_t)c * n + i] = b[c * ldb + p];
            t[(int64_t)c * n + i] = 0.0;
        }
    }
}

// the solution in the user's order; the statistics of the residual that
// follows cleared
__global__ void permute_out(double* x, int64_t ldx, const double* y, const int32_t* perm, int32_t n, int32_t nrhs,
                            unsigned long long* stats)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 5) stats[threadIdx.x * kStatStride] = 0ull;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t p = perm[i];
        for (int32_t c = blockIdx.y; c < nrhs; c += gridDim.y) x[c * ldx + p] = y[(int64_t)c * n + i];
    }
}

__global__ void axpy_kernel(double* x, const double* d, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        x[i] += d[i];
}

// order-preserving bits of a non-negative double (NaN is treated as +inf)
__device__ __forceinline__ unsigned long long key_of(double v)
{
    if (v != v) v = __builtin_inf();
    return (unsigned long long)__double_as_longlong(v);
}

__device__ __forceinline__ unsigned long long block_max(unsigned long long v)
{
    __shared__ unsigned long long sm[4];
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(v, off);
        v = o > v ? o : v;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) sm[wave] = v;
    __syncthreads();
    unsigned long long r = sm[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) r = sm[i] > r ? sm[i] : r;
    __syncthreads();
    return r;
}

// r = b - A x and componentwise / normwise error statistics, in FP64.
// A is read through the symmetric row pattern (rptr, rcol) with its values rv
// in the same order (the input's lower triangle mirrored, gathered once per
// factorization by gather_kernel so that the residual reads them in order).
// stats[0] = max_i |r_i| / (|A||x| + |b|)_i   (0/0 = 0, p/0 = inf)
// stats[1] = max |r_i|, stats[2] = max |x_i|, stats[3] = max |b_i|, stats[4] = max_i sum_j |a_ij|
// (stats[q] at word q * kStatStride: every block adds its maxima by atomics,
// one cache line per statistic)
// A thread takes a row and NR right-hand sides at a time (grid rows): its
// entries are read once for all of them, kRU entries and their x at a time
// (bound by the round trips to memory; four entries at a time took dense rows
// of 1500 and four right-hand sides 761 us, longer than a thread per row and
// right-hand side, 684; eight: solve 867 -> 684 us).
template <int NR>
__global__ void __launch_bounds__(256) residual_kernel(const int64_t* rptr, const int32_t* rcol, const double* rv,
                                                       const double* x, const double* b,
                                                       int64_t ldb, double* r, int32_t n, int32_t nrhs,
                                                       unsigned long long* stats)
{
    constexpr int kRU = 8;
    unsigned long long m0 = 0, m1 = 0, m2 = 0, m3 = 0, m4 = 0;
    auto up = [](unsigned long long& m, double v) {
        const unsigned long long k = key_of(v);
        m = k > m ? k : m;
    };
    for (int c0 = blockIdx.y * NR; c0 < nrhs; c0 += gridDim.y * NR) {
        const int nv = min(NR, nrhs - c0);
        const double* xc = x + (int64_t)c0 * n;
        for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
            double acc[NR], den[NR], arow = 0.0;
#pragma unroll
            for (int j = 0; j < NR; ++j) {
                const double bi = b[(c0 + min(j, nv - 1)) * ldb + i];
                acc[j] = bi;
                den[j] = fabs(bi);
                up(m3, fabs(bi));
            }
            const int64_t qe = rptr[i + 1];
            for (int64_t q = rptr[i]; q < qe; q += kRU) {
                double av[kRU], xv[kRU][NR];
                int32_t col[kRU];
#pragma unroll
                for (int u = 0; u < kRU; ++u) {
                    av[u] = rv[min(q + u, qe - 1)];
                    col[u] = rcol[min(q + u, qe - 1)];
                }
#pragma unroll
                for (int u = 0; u < kRU; ++u)
#pragma unroll
                    for (int j = 0; j < NR; ++j) xv[u][j] = xc[(int64_t)min(j, nv - 1) * n + col[u]];
#pragma unroll
                for (int u = 0; u < kRU; ++u)
                    if (q + u < qe) {
#pragma unroll
                        for (int j = 0; j < NR; ++j) {
                            acc[j] -= av[u] * xv[u][j];
                            den[j] += fabs(av[u]) * fabs(xv[u][j]);
                        }
                        arow += fabs(av[u]);
                    }
            }
#pragma unroll
            for (int j = 0; j < NR; ++j) {
                if (j < nv) r[(int64_t)(c0 + j) * n + i] = acc[j];
                const double ar = fabs(acc[j]);
                up(m0, ar == 0.0 ? 0.0 : (den[j] == 0.0 ? __builtin_inf() : ar / den[j]));
                up(m1, ar);
                up(m2, fabs(xc[(int64_t)min(j, nv - 1) * n + i]));
            }
            up(m4, arow);
        }
    }
    m0 = block_max(m0);
    m1 = block_max(m1);
    m2 = block_max(m2);
    m3 = block_max(m3);
    m4 = block_max(m4);
    if (threadIdx.x == 0) {
        atomicMax(stats + 0 * kStatStride, m0);
        atomicMax(stats + 1 * kStatStride, m1);
        atomicMax(stats + 2 * kStatStride, m2);
        atomicMax(stats + 3 * kStatStride, m3);
        atomicMax(stats + 4 * kStatStride, m4);
    }
}

// ---- rv[q] = vals[idx[q]]
__global__ void gather_kernel(double* rv, const double* vals, const int64_t* idx, int64_t m)
{
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < m; q += (int64_t)gridDim.x * blockDim.x)
        rv[q] = vals[idx[q]];
}

// ---- value gradient of x = A^{-1} b (adjoint): for a stored entry p = (i, j),
// grad[p] = -sum_k (db[i,k] x[j,k] + db[j,k] x[i,k]) if i > j, -sum_k db[i,k] x[i,k]
// if i == j, and 0 for entries above the diagonal (erow[p] < 0: not read by
// the factorization)
__global__ void values_grad_kernel(const int32_t* erow, const int32_t* ecol, int64_t nnz, const double* x,
                                   const double* db, int64_t ld, int32_t nrhs, double* grad)
{
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < nnz; p += (int64_t)gridDim.x * blockDim.x) {
        const int32_t i = erow[p], j = ecol[p];
        double g = 0.0;
        if (i >= 0) {
            for (int32_t k = 0; k < nrhs; ++k) {
                const double* xk = x + (int64_t)k * ld;
                const double* dk = db + (int64_t)k * ld;
                g -= i == j ? dk[i] * xk[i] : dk[i] * xk[j] + dk[j] * xk[i];
            }
        }
        grad[p] = g;
    }
}

// ---- inverses of paired pieces (built after the factorization): the pair's
// inverse [[D_p, 0], [X, D_q]], X = -D_q (L_qp D_p), on the matrix cores
// (16x16x4 products; operand A lane l holds A[l%16][l/16], operand B lane l
// holds B[l/16][l%16], result slot v of lane l holds D[row(v, l/16)][l%16]).
// Workgroup (pair, jb): for jb < ceil(w_p/16) the columns j0 = 16 jb ..
// j0 + 15 of p: D_p's columns staged in LDS (zero above the diagonal) and
// copied, T = L_qp D_p[:, cols] (inner indices from j0: D_p is lower
// triangular) into LDS, then X[:, cols] = -D_q T (inner indices up to each
// row tile's end: D_q is lower triangular); for the remaining jb the columns
// of q: zeros above, D_q below.  L D L^T (kept inverses Y = D^{-1} L^{-1},
// unit L): X = -Y_q L_qp D_p Y_p, the staged rows of Y_p scaled by p's
// pivots.  Each wave takes the 16-row tiles
// wave, wave + 4, ...; the loads of sixteen inner steps go out together.
template <class T>
struct PairMM;
template <>
struct PairMM<double> {
    typedef double acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc mfma(double a, double b, acc c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int v, int lk) { return 4 * v + lk; }
};
template <>
struct PairMM<float> {
    typedef float acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc mfma(float a, float b, acc c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int v, int lk) { return 4 * lk + v; }
};

constexpr int kPairLd = 17;   // LDS leading dimension of the staged 16-column blocks

template <class T>
__global__ void __launch_bounds__(256) pair_inv(const T* panels, T* dinv, const PairItem* items, int ldlt)
{
    typedef typename PairMM<T>::acc acc;
    __shared__ T dps[256 * kPairLd];   // D_p[kk][n]
    __shared__ T ts[256 * kPairLd];    // T[kk][n]
    const PairItem it = items[blockIdx.x];
    const int wp = it.wp, wq = it.wq, W = wp + wq;
    const int nbp = (wp + 15) / 16, nbq = (wq + 15) / 16;
    const int jb = blockIdx.y;
    if (jb >= nbp + nbq) return;
    T* P = dinv + it.out;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
    if (jb >= nbp) {
        const int j0 = 16 * (jb - nbp);
        const T* Dq = dinv + it.dq;
        for (int idx = tid; idx < 16 * W; idx += 256) {
            const int j = j0 + idx / W, r = idx % W;
            if (j < wq) P[(int64_t)(wp + j) * W + r] = (r >= wp + j) ? Dq[(int64_t)j * wq + (r - wp)] : T(0);
        }
        return;
    }
    const int j0 = 16 * jb;
    const T* Dp = dinv + it.dp;
    const T* Pp = panels + (it.lofs - wp);   // p's panel: L D L^T pivot d_r at r * (ldp + 1)
    for (int idx = tid; idx < 16 * wp; idx += 256) {
        const int c = idx / wp, r = idx % wp, j = j0 + c;
        const T v = (j < wp && r >= j) ? Dp[(int64_t)j * wp + r] : T(0);
        dps[r * kPairLd + c] = ldlt ? v * Pp[(int64_t)r * (it.ldp + 1)] : v;
        if (j < wp) P[(int64_t)j * W + r] = v;
    }
    __syncthreads();
    const int ntile = (wq + 15) / 16;
    const T* Lq = panels + it.lofs;   // L_qp[i][kk] at Lq[i + kk * ldp]
    const int64_t ldp = it.ldp;
    for (int t = wave; t < ntile; t += 4) {
        acc c = {0, 0, 0, 0};
        const int i = min(16 * t + li, wq - 1);
        for (int kk0 = j0; kk0 < wp; kk0 += 64) {
            T av[16], bv[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int kk = kk0 + 4 * u + lk;
                av[u] = Lq[i + (int64_t)min(kk, wp - 1) * ldp];
                bv[u] = kk < wp ? dps[kk * kPairLd + li] : T(0);
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) c = PairMM<T>::mfma(av[u], bv[u], c);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) ts[(16 * t + PairMM<T>::row(v, lk)) * kPairLd + li] = c[v];
    }
    __syncthreads();
    const T* Dq = dinv + it.dq;   // D_q[i][kk] at Dq[i + kk * wq]
    for (int t = wave; t < ntile; t += 4) {
        acc c = {0, 0, 0, 0};
        const int irow = 16 * t + li, i = min(irow, wq - 1);
        const int kend = min(16 * t + 16, wq);
        for (int kk0 = 0; kk0 < kend; kk0 += 64) {
            T av[16], bv[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int kk = kk0 + 4 * u + lk;
                const T d = Dq[i + (int64_t)min(kk, wq - 1) * wq];
                av[u] = kk <= irow ? d : T(0);
                bv[u] = kk < kend ? ts[kk * kPairLd + li] : T(0);
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) c = PairMM<T>::mfma(av[u], bv[u], c);
        }
        if (j0 + li < wp)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * t + PairMM<T>::row(v, lk);
                if (r < wq) P[(int64_t)(j0 + li) * W + wp + r] = -c[v];
            }
    }
}

// ---- host launchers
static int grid_for(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 8192)); }

// right-hand sides per pass over a panel: 1, 4 or 8
static int nr_block(int nrhs) { return nrhs <= 1 ? 1 : (nrhs <= 4 ? 4 : 8); }

#define SPX_NR_DISPATCH(NRV, CALL) \
    do {                           \
        if ((NRV) == 1) { constexpr int NR = 1; CALL; } \
        else if ((NRV) == 4) { constexpr int NR = 4; CALL; } \
        else { constexpr int NR = 8; CALL; } \
    } while (0)

hipError_t launch_fwd_off(const SweepArgs& a, const OffItem* items, int count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    if (a.nrhs > 1) {   // blocks of 4 or 8 right-hand sides: the matrix-core form
        const dim3 grid(count, (a.nrhs + (a.nrhs <= 4 ? 3 : 7)) / (a.nrhs <= 4 ? 4 : 8));
        if (a.nrhs <= 4) {
            if (a.f32) fwd_off_mm<float, 4><<<grid, 256, 0, s>>>(a, items);
            else fwd_off_mm<double, 4><<<grid, 256, 0, s>>>(a, items);
        } else {
            if (a.f32) fwd_off_mm<float, 8><<<grid, 256, 0, s>>>(a, items);
            else fwd_off_mm<double, 8><<<grid, 256, 0, s>>>(a, items);
        }
        return hipGetLastError();
    }
    if (a.f32) fwd_off<float><<<count, 256, 0, s>>>(a, items);
    else fwd_off<double><<<count, 256, 0, s>>>(a, items);
    return hipGetLastError();
}
hipError_t launch_bwd_off(const SweepArgs& a, const OffItem* items, int count, bool tall, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    if (a.nrhs > 1) {   // blocks of 4 or 8 right-hand sides (64-row items): the matrix-core form
        const dim3 grid(count, (a.nrhs + (a.nrhs <= 4 ? 3 : 7)) / (a.nrhs <= 4 ? 4 : 8));
        if (a.nrhs <= 4) {
            if (a.f32) bwd_off_mm<float, 4><<<grid, 256, 0, s>>>(a, items);
            else bwd_off_mm<double, 4><<<grid, 256, 0, s>>>(a, items);
        } else {
            if (a.f32) bwd_off_mm<float, 8><<<grid, 256, 0, s>>>(a, items);
            else bwd_off_mm<double, 8><<<grid, 256, 0, s>>>(a, items);
        }
        return hipGetLastError();
    }
    if (tall) {
        if (a.f32) bwd_off<float, 16><<<count, 256, 0, s>>>(a, items);
        else bwd_off<double, 16><<<count, 256, 0, s>>>(a, items);
    } else {
        if (a.f32) bwd_off<float, 4><<<count, 256, 0, s>>>(a, items);
        else bwd_off<double, 4><<<count, 256, 0, s>>>(a, items);
    }
    return hipGetLastError();
}
// the diagonal items and the small blocks of a level
hipError_t launch_fwd_level(const SweepArgs& a, const DiagItem* ditems, int nd, int lanes, const SmallItem* items,
                            int count, int ntiny, hipStream_t s)
{
    const int ns = (ntiny + kSGroups - 1) / kSGroups + (count - ntiny + 3) / 4;
    const int nrv = nr_block(a.nrhs), rows = (a.nrhs + nrv - 1) / nrv;
    if (nd > 0 && ns > 0 && nrv == 1) {
#define SPX_LEVEL(L) (a.f32 ? fwd_level<float, L><<<nd + ns, 256, 0, s>>>(a, ditems, nd, items, count, ntiny) \
                            : fwd_level<double, L><<<nd + ns, 256, 0, s>>>(a, ditems, nd, items, count, ntiny))
        if (lanes == 32) SPX_LEVEL(32);
        else if (lanes == 16) SPX_LEVEL(16);
        else SPX_LEVEL(4);
#undef SPX_LEVEL
        return hipGetLastError();
    }
    if (nd > 0) {
#define SPX_DIAG(L) SPX_NR_DISPATCH(nrv, (a.f32 ? fwd_diag<float, L, NR><<<dim3(nd, rows), 256, 0, s>>>(a, ditems) \
                                                 : fwd_diag<double, L, NR><<<dim3(nd, rows), 256, 0, s>>>(a, ditems)))
        if (lanes == 32) SPX_DIAG(32);
        else if (lanes == 16) SPX_DIAG(16);
        else SPX_DIAG(4);
#undef SPX_DIAG
    }
    if (ns > 0)
        SPX_NR_DISPATCH(nrv, (a.f32 ? fwd_small<float, NR><<<dim3(ns, rows), 256, 0, s>>>(a, items, count, ntiny)
                                    : fwd_small<double, NR><<<dim3(ns, rows), 256, 0, s>>>(a, items, count, ntiny)));
    return hipGetLastError();
}
hipError_t launch_bwd_level(const SweepArgs& a, const DiagItem* ditems, int nd, int lanes, const SmallItem* items,
                            int count, int ntiny, hipStream_t s)
{
    const int ns = (ntiny + kSGroups - 1) / kSGroups + (count - ntiny + 3) / 4;
    const int nrv = nr_block(a.nrhs), rows = (a.nrhs + nrv - 1) / nrv;
    if (nd > 0 && ns > 0 && nrv == 1) {
#define SPX_LEVEL(L) (a.f32 ? bwd_level<float, L><<<nd + ns, 256, 0, s>>>(a, ditems, nd, items, count, ntiny) \
                            : bwd_level<double, L><<<nd + ns, 256, 0, s>>>(a, ditems, nd, items, count, ntiny))
        if (lanes == 32) SPX_LEVEL(32);
        else if (lanes == 16) SPX_LEVEL(16);
        else SPX_LEVEL(4);
#undef SPX_LEVEL
        return hipGetLastError();
    }
    if (nd > 0) {
#define SPX_DIAG(L) SPX_NR_DISPATCH(nrv, (a.f32 ? bwd_diag<float, L, NR><<<dim3(nd, rows), 256, 0, s>>>(a, ditems) \
                                                 : bwd_diag<double, L, NR><<<dim3(nd, rows), 256, 0, s>>>(a, ditems)))
        if (lanes == 32) SPX_DIAG(32);
        else if (lanes == 16) SPX_DIAG(16);
        else SPX_DIAG(4);
#undef SPX_DIAG
    }
    if (ns > 0)
        SPX_NR_DISPATCH(nrv, (a.f32 ? bwd_small<float, NR><<<dim3(ns, rows), 256, 0, s>>>(a, items, count, ntiny)
                                    : bwd_small<double, NR><<<dim3(ns, rows), 256, 0, s>>>(a, items, count, ntiny)));
    return hipGetLastError();
}
hipError_t launch_pair_inv(const void* panels, void* dinv, bool f32, bool ldlt, const PairItem* items, int count,
                          int maxnb, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    const dim3 grid(count, maxnb);
    if (f32)
        pair_inv<float><<<grid, 256, 0, s>>>(static_cast<const float*>(panels), static_cast<float*>(dinv), items,
                                             ldlt ? 1 : 0);
    else
        pair_inv<double><<<grid, 256, 0, s>>>(static_cast<const double*>(panels), static_cast<double*>(dinv), items,
                                              ldlt ? 1 : 0);
    return hipGetLastError();
}
hipError_t launch_permute_in(double* y, double* t, const double* b, int64_t ldb, const int32_t* perm, int32_t n,
                             int32_t nrhs, hipStream_t s)
{
    permute_in<<<dim3(grid_for(n), std::min(nrhs, 64)), 256, 0, s>>>(y, t, b, ldb, perm, n, nrhs);
    return hipGetLastError();
}
hipError_t launch_permute_out(double* x, int64_t ldx, const double* y, const int32_t* perm, int32_t n, int32_t nrhs,
                              unsigned long long* stats, hipStream_t s)
{
    permute_out<<<dim3(grid_for(n), std::min(nrhs, 64)), 256, 0, s>>>(x, ldx, y, perm, n, nrhs, stats);
    return hipGetLastError();
}
hipError_t launch_axpy(double* x, const double* d, int64_t n, hipStream_t s)
{
    axpy_kernel<<<grid_for(n), 256, 0, s>>>(x, d, n);
    return hipGetLastError();
}
hipError_t launch_residual(const int64_t* rptr, const int32_t* rcol, const double* rv, const double* x,
                           const double* b, int64_t ldb, double* r, int32_t n, int32_t nrhs,
                           unsigned long long* stats, hipStream_t s)
{
    const int nr = nrhs <= 1 ? 1 : 4;
    const int rows = std::min((nrhs + nr - 1) / nr, 64);
    const int blocks = (int)std::min<int64_t>(std::max(64, kResidualBlocks / rows), std::max<int64_t>(1, ((int64_t)n + 255) / 256));
    if (nr == 1) residual_kernel<1><<<dim3(blocks, rows), 256, 0, s>>>(rptr, rcol, rv, x, b, ldb, r, n, nrhs, stats);
    else residual_kernel<4><<<dim3(blocks, rows), 256, 0, s>>>(rptr, rcol, rv, x, b, ldb, r, n, nrhs, stats);
    return hipGetLastError();
}

}  // namespace spx

namespace spx {
hipError_t launch_gather(double* rv, const double* vals, const int64_t* idx, int64_t m, hipStream_t s)
{
    if (m <= 0) return hipSuccess;
    gather_kernel<<<grid_for(m), 256, 0, s>>>(rv, vals, idx, m);
    return hipGetLastError();
}
hipError_t launch_values_grad(const int32_t* erow, const int32_t* ecol, int64_t nnz, const double* x, const double* db,
                              int64_t ld, int32_t nrhs, double* grad, hipStream_t s)
{
    if (nnz <= 0) return hipSuccess;
    values_grad_kernel<<<grid_for(nnz), 256, 0, s>>>(erow, ecol, nnz, x, db, ld, nrhs, grad);
    return hipGetLastError();
}
}  // namespace spx
