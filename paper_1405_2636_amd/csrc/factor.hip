// Numerical supernodal LL^T factorization on one MI355X (gfx950).
//
// The method is the paper's (Section III): for every column block k, (1)
// Cholesky of its diagonal block, (2) triangular solve of its off-diagonal
// rows, (3) right-looking updates C_j -= L_k[rows] L_k[facing j]^T scattered
// into every facing column block j (the sparse GEMM of Section V-B, computed
// directly into the gapped destination panel, without a temporary buffer).
// As in the runtime versions of the paper the 1D task is split: one task
// factors a panel, the updates become separate tasks.  Here they are further
// tiled, and all of them are scheduled by one persistent kernel that pulls
// work items from device-side ready queues:
//   FACT(k)          Cholesky of the diagonal block and its inverse L_kk^{-1}
//   TRSM(k, rows)    64, 128 or 256 off-diagonal rows of panel k times
//                    L_kk^{-T}; chain blocks: 16 rows by block substitution
//   INV(k)           the rest of L_kk^{-1} of a chain block, beside the chain
//   UPDATE(k,j,r,c)  a 256x64 (or 128x128; 64x64 on levels with little work)
//                    tile of the outer product of panel k, subtracted into
//                    panel j with atomics; for a group of pieces of a split
//                    supernode, the sum of their products
//   SMALL(k)         a narrow column block (width <= 32, <= 128 rows): all
//                    three steps and every update tile of the block at once
//   TINY(k, ...)     the same for a group of blocks of width <= 16 with at most
//                    64 rows, a wave each
// Dependencies are counters: FACT(j) becomes ready when every UPDATE tile
// into j is done, the TRSM tiles of k when FACT(k) is done, the UPDATE tiles
// of k when its last TRSM tile is done.  FACT, TRSM and the updates into the
// first facing block go to a high-priority queue that workers poll first.
// Products run on the matrix cores: v_mfma_f64_16x16x4f64 for the FP64
// factor, v_mfma_f32_16x16x4f32 for the FP32 factor of the refinement mode
// (whose 32x32 diagonal tiles are still factored and inverted in FP64), and
// split-BF16 products (v_mfma_f32_16x16x16_bf16) in the split mode.
#include "device.hpp"

#include <type_traits>

namespace spx {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

#define AGENT __HIP_MEMORY_SCOPE_AGENT

// Pointers into device (global) memory.  The panels reach the tasks as
// generic pointers; typing them as global lets the compiler use global
// stores and atomics (scalar base, 32-bit lane offset) instead of flat ones.
template <class T>
struct Glob {
    typedef __attribute__((address_space(1))) T type;
};
template <class T>
__device__ __forceinline__ typename Glob<T>::type* glob(T* p)
{
    return (typename Glob<T>::type*)p;
}
// A generic pointer known to point into LDS, as an LDS pointer (never null:
// the cast then needs no null test)
template <class T>
__device__ __forceinline__ __attribute__((address_space(3))) T* lds(T* p)
{
    if (p == nullptr) __builtin_unreachable();
    return (__attribute__((address_space(3))) T*)p;
}

// The 16x16x4 matrix-core product of one element type.  Operand A lane l
// holds A[l%16][l/16], operand B lane l holds B[l/16][l%16]; the four result
// slots of lane l hold column l%16 of D, at the rows drow(v, l/16).
template <class T>
struct MM;
template <>
struct MM<double> {
    typedef d4 acc;
    static __device__ __forceinline__ acc mfma(double a, double b, acc c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int drow(int v, int lk) { return 4 * v + lk; }
};
template <>
struct MM<float> {
    typedef f4 acc;
    static __device__ __forceinline__ acc mfma(float a, float b, acc c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int drow(int v, int lk) { return 4 * lk + v; }
};

__device__ __forceinline__ double readlane_d(double v, int lane)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// A global operand read through a buffer resource covering one array (a panel
// or an inverse): element (i, p) (i = row or column index of the product, p =
// inner index) is at byte off + i*si + p*sk.  Reads past the end of the array
// return zero (buffer range check), so tiles need no bounds masks: rows or
// columns beyond a tile only feed results that are not stored, and the inner
// ranges either end at the array's end or meet zeros (upper triangle of an
// inverse).
struct GOp {
    __amdgpu_buffer_rsrc_t rs;
    int off, si, sk;
};

// Values the whole wave shares, moved to scalar registers (buffer resources
// must be uniform; the compiler cannot prove it for values read from memory).
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <class T>
__device__ __forceinline__ const T* uni(const T* p)
{
    const uint64_t u = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return reinterpret_cast<const T*>(((uint64_t)hi << 32) | lo);
}

template <class T>
__device__ __forceinline__ GOp make_gop(const T* base, int64_t count, int64_t off, int64_t si, int64_t sk)
{
    constexpr int e = (int)sizeof(T);
    GOp g;
    g.rs = __builtin_amdgcn_make_buffer_rsrc((void*)uni(base), (short)0, uni((int)(count * e)), 0x00020000);
    g.off = uni((int)(off * e));
    g.si = uni((int)(si * e));
    g.sk = uni((int)(sk * e));
    return g;
}

template <class T>
__device__ __forceinline__ T gload(const GOp& g, int voff);
template <>
__device__ __forceinline__ double gload<double>(const GOp& g, int voff)
{
    const u32x2 b = __builtin_amdgcn_raw_buffer_load_b64(g.rs, voff, 0, 0);
    return __builtin_bit_cast(double, b);
}
template <>
__device__ __forceinline__ float gload<float>(const GOp& g, int voff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(g.rs, voff, 0, 0));
}

// Byte offset of a masked-off buffer load: past the end of any array here,
// so the load returns zero (the value is discarded by a select anyway).
constexpr int kOffNone = 0x7f000000;

// Store at byte offset voff (per lane, range-checked) + soff (wave-uniform,
// not) of g's array; a voff outside the array drops the store.
__device__ __forceinline__ void gstore_s(const GOp& g, int voff, int soff, double v)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), g.rs, voff, soff, 0);
}
__device__ __forceinline__ void gstore_s(const GOp& g, int voff, int soff, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), g.rs, voff, soff, 0);
}

// One wave accumulates a 64 x (16*NB) tile: acc += X Y^T, X(r, p) r < 64,
// Y(c, p) c < 16*NB, p < K (K rounded up to 4 reads zeros or is exact).  The
// whole tile is always computed (no per-block predicates); rows and columns
// beyond the caller's bounds produce results that are not stored.
// Y feeds operand A and X operand B (lane layout in MM), so
//   acc[bi][bj][v] = C(16*bj + l%16, 16*bi + drow(v, l/16))
// and the 16 lanes of a result slot cover 16 consecutive rows of C.  Rows of
// X and of Y are consecutive in memory (si of both is the element size).
// The inner dimension advances 4 at a time through a ring of NBUF operand
// buffers, each loaded again as soon as its products are issued: NBUF - 1
// steps are in flight (a step is 16 products of 64 cycles in FP64, 32 in
// FP32).  Four buffers in FP64 and eight in FP32 fill the 256 registers of a
// wave at two workgroups per CU beside the accumulators; six and sixteen
// spill.  Update tiles alone with an inner dimension of 2048: 62 TFLOP/s in
// FP64 and 122 in FP32, 52 and 102 with two and three buffers of 8 inner
// indices whose 16 offsets were formed anew per chunk (100^3 scheduler
// kernel 89.9 -> 86.4 ms).  A load between every two products instead of a
// step's loads in one go: 53 and 126.
// The offset of a step is added to one vector register per operand, the
// 16-row blocks of a step are immediate offsets of it: both are range-checked.
template <int NB, class T, int RB = 4>
__device__ __forceinline__ void wave_gemm(typename MM<T>::acc (&acc)[NB][RB], const GOp& X, const GOp& Y, int K)
{
    constexpr int e = (int)sizeof(T);
    constexpr int NBUF = sizeof(T) == 8 ? 4 : 8;
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lk = lane >> 4;
    const int steps = (K + 3) >> 2;
    if (steps <= 0) return;
    int xo = X.off + li * e + lk * X.sk, yo = Y.off + li * e + lk * Y.sk;
    const int dx = 4 * X.sk, dy = 4 * Y.sk;
    T xs[NBUF][RB], ys[NBUF][NB];
    // (scheduling barriers keep every group of loads behind the products
    // whose buffer it fills and ahead of the next ones; left alone, the
    // compiler sinks the loads next to their uses and waits for them)
    auto load = [&](int q) {
#pragma unroll
        for (int b = 0; b < RB; ++b) xs[q][b] = gload<T>(X, xo + 16 * e * b);
#pragma unroll
        for (int b = 0; b < NB; ++b) ys[q][b] = gload<T>(Y, yo + 16 * e * b);
        xo += dx;
        yo += dy;
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mma = [&](int q) {
#pragma unroll
        for (int bi = 0; bi < NB; ++bi)
#pragma unroll
            for (int bj = 0; bj < RB; ++bj) acc[bi][bj] = MM<T>::mfma(ys[q][bi], xs[q][bj], acc[bi][bj]);
        __builtin_amdgcn_sched_barrier(0);
    };
    // (steps past the last one read zeros past the array, or entries that are not used)
#pragma unroll
    for (int q = 0; q < NBUF - 1; ++q) load(q);
    int st = 0;
    for (; st + NBUF <= steps; st += NBUF) {
#pragma unroll
        for (int q = 0; q < NBUF; ++q) {
            load((q + NBUF - 1) % NBUF);
            mma(q);
        }
    }
#pragma unroll
    for (int q = 0; q < NBUF - 1; ++q)
        if (st + q < steps) mma(q);
}

// L D L^T update products: acc += X (Y D)^T, the facing operand Y scaled by
// d_p (element p of Dg at p * Dg.sk: the diagonal of the source panel) just
// before the products, so its loads stay in flight with the others; two
// register buffers of 8 inner indices in both precisions (a separate
// function: the extra operand registers would change the allocation of the
// plain product, and a third FP32 buffer spills).
template <int NB, class T, int RB = 4>
__device__ __forceinline__ void wave_gemm_d(typename MM<T>::acc (&acc)[NB][RB], const GOp& X, const GOp& Y, int K,
                                          const GOp& Dg)
{
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lk = lane >> 4;
    const int nchunks = (K + 7) >> 3;
    if (nchunks <= 0) return;
    int xo[2][RB], yo[2][NB];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
        for (int b = 0; b < RB; ++b) xo[u][b] = X.off + (16 * b + li) * X.si + (4 * u + lk) * X.sk;
#pragma unroll
        for (int b = 0; b < NB; ++b) yo[u][b] = Y.off + (16 * b + li) * Y.si + (4 * u + lk) * Y.sk;
    }
    const int dx = 8 * X.sk, dy = 8 * Y.sk;
    T xa[2][RB], ya[2][NB], da[2], xb[2][RB], yb[2][NB], db[2];
    // (scheduling barriers keep every group of loads ahead of the products
    // it is meant to overlap; left alone, the compiler sinks the FP32 loads
    // next to their uses and waits for them)
    auto load = [&](T (&xs)[2][RB], T (&ys)[2][NB], T (&ds)[2], int ch) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int b = 0; b < RB; ++b) xs[u][b] = gload<T>(X, xo[u][b] + ch * dx);
#pragma unroll
            for (int b = 0; b < NB; ++b) ys[u][b] = gload<T>(Y, yo[u][b] + ch * dy);
            ds[u] = gload<T>(Dg, Dg.off + (8 * ch + 4 * u + lk) * Dg.sk);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mma = [&](const T (&xs)[2][RB], const T (&ys)[2][NB], const T (&ds)[2]) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int bi = 0; bi < NB; ++bi) {
                const T yv = ys[u][bi] * ds[u];
#pragma unroll
                for (int bj = 0; bj < RB; ++bj) acc[bi][bj] = MM<T>::mfma(yv, xs[u][bj], acc[bi][bj]);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    // (reads past the last chunk repeat it and are not used)
    const int last = nchunks - 1;
    load(xa, ya, da, 0);
    int ch = 0;
    for (; ch + 2 <= nchunks; ch += 2) {
        load(xb, yb, db, ch + 1);
        mma(xa, ya, da);
        load(xa, ya, da, min(ch + 2, last));
        mma(xb, yb, db);
    }
    if (ch < nchunks) mma(xa, ya, da);
}

// Split-BF16 products (FP32 panels): each FP32 operand x is split into
// hi = bf16(x) (round to nearest) and lo = bf16(x - hi); the product is
// hi*hi + hi*lo + lo*hi on the BF16 matrix cores with FP32 accumulation
// (lo*lo is dropped: relative error about 2^-16 per product).  The inner
// dimension advances 16 at a time; lane (l%16, l/16) loads its FP32 operands
// at inner indices 4s + l/16 (s < 4), the order of the FP32 products, and
// packs them as the 4 BF16 values the 16x16x16 instruction takes from it at
// 4*(l/16) + s: the same permutation of the inner index for both operands,
// so the sum is unchanged.  Two raw buffers: the next 16 in flight while the
// current 16 are split and multiplied (with 32 per step, the 16x16x32 form,
// the buffers and accumulators exceed the registers and spill).
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void split_bf16(const float (&v)[4], s16x4& hi, s16x4& lo)
{
    bf16x4 h, l;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const __bf16 t = (__bf16)v[j];
        h[j] = t;
        l[j] = (__bf16)(v[j] - (float)t);
    }
    hi = __builtin_bit_cast(s16x4, h);
    lo = __builtin_bit_cast(s16x4, l);
}

template <int NB, int RB = 4>
__device__ __forceinline__ void wave_gemm_split(f4 (&acc)[NB][RB], const GOp& X, const GOp& Y, int K)
{
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lk = lane >> 4;
    const int nchunks = (K + 15) >> 4;
    if (nchunks <= 0) return;
    int xo[RB], yo[NB];
#pragma unroll
    for (int b = 0; b < RB; ++b) xo[b] = X.off + (16 * b + li) * X.si + lk * X.sk;
#pragma unroll
    for (int b = 0; b < NB; ++b) yo[b] = Y.off + (16 * b + li) * Y.si + lk * Y.sk;
    const int dx = 4 * X.sk, dy = 4 * Y.sk;
    float xa[RB][4], ya[NB][4], xb[RB][4], yb[NB][4];
    auto load = [&](float (&xs)[RB][4], float (&ys)[NB][4], int ch) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int b = 0; b < RB; ++b) xs[b][s] = gload<float>(X, xo[b] + (4 * ch + s) * dx);
#pragma unroll
            for (int b = 0; b < NB; ++b) ys[b][s] = gload<float>(Y, yo[b] + (4 * ch + s) * dy);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mma = [&](const float (&xs)[RB][4], const float (&ys)[NB][4]) {
        s16x4 xh[RB], xl[RB];
#pragma unroll
        for (int b = 0; b < RB; ++b) split_bf16(xs[b], xh[b], xl[b]);
#pragma unroll
        for (int bi = 0; bi < NB; ++bi) {
            s16x4 yh, yl;
            split_bf16(ys[bi], yh, yl);
#pragma unroll
            for (int bj = 0; bj < RB; ++bj) {
                acc[bi][bj] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(yh, xh[bj], acc[bi][bj], 0, 0, 0);
                acc[bi][bj] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(yh, xl[bj], acc[bi][bj], 0, 0, 0);
                acc[bi][bj] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(yl, xh[bj], acc[bi][bj], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // (reads past the last chunk repeat it and are not used)
    const int last = nchunks - 1;
    load(xa, ya, 0);
    int ch = 0;
    for (; ch + 2 <= nchunks; ch += 2) {
        load(xb, yb, ch + 1);
        mma(xa, ya);
        load(xa, ya, min(ch + 2, last));
        mma(xb, yb);
    }
    if (ch < nchunks) mma(xa, ya);
}

// Split-BF16 L D L^T update products: the facing operand scaled by d_p in
// FP32 before it is split (as in wave_gemm_d).
template <int NB, int RB = 4>
__device__ __forceinline__ void wave_gemm_split_d(f4 (&acc)[NB][RB], const GOp& X, const GOp& Y, int K, const GOp& Dg)
{
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lk = lane >> 4;
    const int nchunks = (K + 15) >> 4;
    if (nchunks <= 0) return;
    int xo[RB], yo[NB];
#pragma unroll
    for (int b = 0; b < RB; ++b) xo[b] = X.off + (16 * b + li) * X.si + lk * X.sk;
#pragma unroll
    for (int b = 0; b < NB; ++b) yo[b] = Y.off + (16 * b + li) * Y.si + lk * Y.sk;
    const int dx = 4 * X.sk, dy = 4 * Y.sk;
    float xa[RB][4], ya[NB][4], da[4], xb[RB][4], yb[NB][4], db[4];
    auto load = [&](float (&xs)[RB][4], float (&ys)[NB][4], float (&ds)[4], int ch) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int b = 0; b < RB; ++b) xs[b][s] = gload<float>(X, xo[b] + (4 * ch + s) * dx);
#pragma unroll
            for (int b = 0; b < NB; ++b) ys[b][s] = gload<float>(Y, yo[b] + (4 * ch + s) * dy);
            // inner index 16 ch + 4 s + l/16
            ds[s] = gload<float>(Dg, Dg.off + (16 * ch + 4 * s + lk) * Dg.sk);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mma = [&](const float (&xs)[RB][4], const float (&ys)[NB][4], const float (&ds)[4]) {
        s16x4 xh[RB], xl[RB];
#pragma unroll
        for (int b = 0; b < RB; ++b) split_bf16(xs[b], xh[b], xl[b]);
#pragma unroll
        for (int bi = 0; bi < NB; ++bi) {
            s16x4 yh, yl;
            float yv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) yv[q] = ys[bi][q] * ds[q];
            split_bf16(yv, yh, yl);
#pragma unroll
            for (int bj = 0; bj < RB; ++bj) {
                acc[bi][bj] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(yh, xh[bj], acc[bi][bj], 0, 0, 0);
                acc[bi][bj] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(yh, xl[bj], acc[bi][bj], 0, 0, 0);
                acc[bi][bj] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(yl, xh[bj], acc[bi][bj], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // (reads past the last chunk repeat it and are not used)
    const int last = nchunks - 1;
    load(xa, ya, da, 0);
    int ch = 0;
    for (; ch + 2 <= nchunks; ch += 2) {
        load(xb, yb, db, ch + 1);
        mma(xa, ya, da);
        load(xa, ya, da, min(ch + 2, last));
        mma(xb, yb, db);
    }
    if (ch < nchunks) mma(xa, ya, da);
}

// acc += X Y^T over K inner indices: FP64 or FP32 products, or (FP32 panels
// with the split option) split-BF16 products; DS: acc += X (Y D)^T with the
// d_p read through Dg
template <int NB, class T, int RB = 4, bool DS = false>
__device__ __forceinline__ void tile_gemm(typename MM<T>::acc (&acc)[NB][RB], const GOp& X, const GOp& Y, int K, bool split,
                                          const GOp& Dg)
{
    if constexpr (sizeof(T) == 4) {
        if (split) {
            if constexpr (DS) wave_gemm_split_d<NB, RB>(acc, X, Y, K, Dg);
            else wave_gemm_split<NB, RB>(acc, X, Y, K);
            return;
        }
    }
    if constexpr (DS) wave_gemm_d<NB, T, RB>(acc, X, Y, K, Dg);
    else wave_gemm<NB, T, RB>(acc, X, Y, K);
}
template <int NB, class T, int RB = 4>
__device__ __forceinline__ void tile_gemm(typename MM<T>::acc (&acc)[NB][RB], const GOp& X, const GOp& Y, int K, bool split)
{
    tile_gemm<NB, T, RB, false>(acc, X, Y, K, split, X);
}

template <int NB, class A, int RB>
__device__ __forceinline__ void zero_acc(A (&acc)[NB][RB])
{
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < RB; ++j) acc[i][j] = A{0, 0, 0, 0};
}

// epi(r, c, value) over a wave's accumulator, r < mv, c < nv
template <class T, int NB, int RB, class Epi>
__device__ __forceinline__ void wave_store(const typename MM<T>::acc (&acc)[NB][RB], int mv, int nv, Epi epi)
{
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int bj = 0; bj < RB; ++bj)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * bj + li, c = 16 * bi + MM<T>::drow(v, lk);
                if (r < mv && c < nv) epi(r, c, acc[bi][bj][v]);
            }
}

// Geometry of a panel, from the second half of an item's descriptor
struct Geo {
    int f, w, ld;         // first column, width, panel stride
    int64_t poff, doff;   // panel and kept inverse
};
__device__ __forceinline__ int64_t words64(int lo, int hi) { return (int64_t)(uint32_t)lo | ((int64_t)hi << 32); }

// (L D L^T) the pivots of the diagonal block in work: one array for FACT and
// INV items, which never run at once in a workgroup (an array each left LDS
// for one workgroup per CU instead of two)
template <bool LDL>
__device__ __forceinline__ double* ldl_pivots()
{
    __shared__ double dd[LDL ? 256 : 1];
    return dd;
}

// ---------------------------------------------------------------- FACT(k)
// The static pivoting threshold eps * max |a_ij| (0: off) sits in LDS after
// the 64-entry broadcast buffer bc and the 32-entry pivot buffer of the
// fused small items, written once by each worker at its start: a global
// load at the start of every tile factorization would wait for memory
// (each item begins with a cache invalidation) on the elimination chain.
constexpr int kThrSlot = 3 * kNB;   // offset from bc

// acc[i] += m * (lane i's value of b within each row of 16 lanes), i = I0 ..
// I0 + N - 1: FP64 multiply-adds that take one operand from a fixed lane
// (DPP row_newbcast; 4.5 cycles each in a row of their own, where a readlane
// pair and a multiply-add took 23 and a broadcast read of LDS 10 plus the
// multiply-add).  b comes from LDS, not from a vector instruction; the
// s_nop keeps the distance a DPP read needs even if a register copy
// precedes it.
template <int I0, int N, int NV>
__device__ __forceinline__ void fmac_rows(double (&acc)[NV], int at, double b, double m)
{
#define SPX_FM(q, k) "v_fmac_f64_dpp %" #q ", %[b], %[m] row_newbcast:%[" #k "] row_mask:0xf bank_mask:0xf\n"
    if constexpr (N >= 4) {
        asm("s_nop 1\n" SPX_FM(0, k0) SPX_FM(1, k1) SPX_FM(2, k2) SPX_FM(3, k3)
            : "+v"(acc[at]), "+v"(acc[at + 1]), "+v"(acc[at + 2]), "+v"(acc[at + 3])
            : [b] "v"(b), [m] "v"(m), [k0] "n"(I0), [k1] "n"(I0 + 1), [k2] "n"(I0 + 2), [k3] "n"(I0 + 3));
        fmac_rows<I0 + 4, N - 4>(acc, at + 4, b, m);
    } else if constexpr (N >= 1) {
        asm("s_nop 1\n" SPX_FM(0, k0) : "+v"(acc[at]) : [b] "v"(b), [m] "v"(m), [k0] "n"(I0));
        fmac_rows<I0 + 1, N - 1>(acc, at + 1, b, m);
    }
#undef SPX_FM
}

// Cholesky factor and inverse of one 32x32 diagonal tile, in FP64, by one
// wave.  Lt (column-major, ld 33) holds the lower triangle of the tile; rows
// and columns >= jb hold the identity.  Lane r < 32 keeps row r of the tile,
// lane 32 + q keeps column q of X = L^{-1}, starting from the unit vector
// e_q.  One right-looking pass over the columns c serves both halves: the
// pivot l_cc is broadcast by readlane, column c is scaled by 1/l_cc (the
// pivot itself becomes sqrt of it), its entries l_ic go through LDS (bc) into
// every row of 16 lanes, and every lane updates v[i] -= v[c] * l_ic for
// i > c (fmac_rows).  For a row of the tile that is the Cholesky update of
// its remaining columns; for a column of X it is the forward substitution
// step x_iq -= l_ic x_cq after x_cq was divided by l_cc.  A pivot that is not
// > 0 records its column with atomicMin (NaN propagates).  Result in
// registers: v[c] of lane r < 32 is l_rc for r >= c (undefined above the
// diagonal), of lane 32 + q it is x_cq (zero for q > c), columns 0 .. jb - 1;
// NC (8, 16 or 32, >= jb) bounds them.
//
// What bounds it is the chain from one pivot to the next (readlane,
// multiply-add, readlane, estimate, one third-order step, scaling) and the
// issue of the multiply-adds: about 145 cycles a column and 8.4 a
// multiply-add (8, 16, 24 and 32 columns of the pass take 2980, 5500, 7470
// and 8750).  The next column is updated by a readlane of l_{c+1,c}, so that
// its pivot does not wait for the LDS round trip of the others, and the
// updates of the columns after it are put, four at a time, into the gaps of
// the next column's chain (column() below is in the order of issue, held by
// scheduling barriers: the compiler puts them behind the chain).  A tile alone
// on the chip, its loads from LDS and the inverse's stores included, takes
// 10,000 cycles, 4.2 us (L D L^T 10,430), the first time 11,200; 12,000 with
// the updates behind the chain; a form that read l_ic from LDS for every
// update and branched around each load of Lt took 38,400.
//
// LDL = true: the L D L^T form of the same pass (unit L): the pivot d is
// not square-rooted (a breakdown is a zero or non-finite d), a row keeps the
// unscaled value t of column c for its update (a_ri -= t l_ic) and ends as
// t / d (1 on the diagonal; the pivots go to dg[0..]); on the identity rows
// the same steps give Y = D^{-1} L^{-1}.  Static pivoting: a pivot with |d|
// below the threshold is replaced by +-threshold (a select beside the
// reciprocal) and counted.
template <int NC, bool LDL>
struct TileChol {
    double v[NC];
    double inv, d, y, thr;     // 1/l_cc (1/d) of the current column; the pivot d in work and its estimate
    double b0, b1, m;          // the last column's entries (rows 0..15, 16..31 in every row of lanes), minus its factor
    int lane, jb;
    uint32_t bad, rep;         // columns with a failed (replaced) pivot
    __attribute__((address_space(3))) double *bc, *dg;

    // d and the hardware estimate y of 1/sqrt(d) (1/d) of column C
    template <int C>
    __device__ __forceinline__ void estimate()
    {
        if constexpr (LDL) {
            const bool small = C < jb && fabs(d) < thr;
            d = small ? (d < 0.0 ? -thr : thr) : d;
            rep |= small ? 1u << C : 0u;
            y = __builtin_amdgcn_rcp(d);
        } else {
            y = __builtin_amdgcn_rsq(d);
        }
    }
    template <int C>
    __device__ __forceinline__ void check()
    {
        if constexpr (LDL) {
            bad |= !(d != 0.0 && d - d == 0.0) ? 1u << C : 0u;
            dg[C] = d;
        } else {
            bad |= !(d > 0.0) ? 1u << C : 0u;
        }
    }
    // the last column's updates of v[A .. B - 1]
    template <int A, int B0>
    __device__ __forceinline__ void update()
    {
        constexpr int B = B0 < NC ? B0 : NC;
        constexpr int lo = A < 16 ? (B < 16 ? B : 16) : A;
        if constexpr (A < lo) fmac_rows<A, lo - A>(v, A, b0, m);
        if constexpr (lo < B && B > 16) fmac_rows<lo - 16, B - lo>(v, lo, b1, m);
        __builtin_amdgcn_sched_barrier(0);
    }
    // column C; v[C] is final but for its scaling, the last column's updates
    // of the columns C + 1 .. are still to be made
    template <int C>
    __device__ __forceinline__ void column()
    {
        const double t = v[C], x = t * inv;   // lane C: l_cc = d / sqrt(d) (L D L^T: 1)
        if constexpr (C + 1 >= NC) {
            v[C] = x;
            return;
        } else {
            if constexpr (C + 2 < NC) bc[lane] = x;
            const double mc = LDL ? -t : -x;   // minus the factor of this column's updates
            const double l1 = readlane_d(x, C + 1);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (C > 0) update<C + 1, C + 5>();
            v[C] = x;
            v[C + 1] = __builtin_fma(mc, l1, v[C + 1]);
            __builtin_amdgcn_sched_barrier(0);
            double n0 = 0.0, n1 = 0.0;
            if constexpr (C + 2 < NC) {   // LDS operations of one wave complete in order: the reads see column C
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                if constexpr (C + 2 < 16) n0 = bc[lane & 15];
                if constexpr (NC > 16) n1 = bc[16 + (lane & 15)];
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (C > 0) update<C + 5, C + 7>();
            d = readlane_d(v[C + 1], C + 1);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (C > 0) update<C + 7, C + 11>();
            estimate<C + 1>();
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (C > 0) update<C + 11, C + 15>();
            if constexpr (LDL) {
                const double e = __builtin_fma(-d, y, 1.0);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (C > 0) update<C + 15, C + 19>();
                const double q = __builtin_fma(e, e, e);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (C > 0) update<C + 19, C + 23>();
                inv = __builtin_fma(y, q, y);
            } else {
                const double g = d * y;
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (C > 0) update<C + 15, C + 17>();
                const double e = __builtin_fma(-g, y, 1.0);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (C > 0) update<C + 17, C + 21>();
                const double q = e * y, p = __builtin_fma(e, 0.375, 0.5);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (C > 0) update<C + 21, C + 23>();
                inv = __builtin_fma(q, p, y);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (C > 0) update<C + 23, NC>();
            check<C + 1>();
            b0 = n0;
            b1 = n1;
            m = mc;
            if constexpr ((C & 7) == 7) {
                if (jb <= C + 1) return;
            }
            column<C + 1>();
        }
    }
    // rows of the tile from LDS (column-major, ld 33), columns of the identity
    __device__ __forceinline__ void load(const double* Lt_g)
    {
        auto Lt = lds(Lt_g);
        const int ln = threadIdx.x & 63, r = ln & 31;
#pragma unroll
        for (int c = 0; c < NC; ++c) v[c] = Lt[r + c * 33];
        // (all loads issued before the selects: a conditional load is a branch each)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            asm volatile("" : "+v"(v[c]));
            v[c] = ln >= 32 ? (c == r ? 1.0 : 0.0) : v[c];
        }
    }
    // factors what is in v; bc: 64 entries, dg: NC entries (L D L^T) of LDS
    __device__ __forceinline__ void run(double* bc_g, double* dg_g, double thr_, int jb_, int col0, int32_t* status)
    {
        static_assert(NC == 8 || NC == 16 || NC == 32, "tile width");
        bc = lds(bc_g);
        dg = lds(dg_g);
        jb = jb_;
        bad = rep = 0;
        thr = thr_;
        lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));   // (keeps the columns' lane masks from being formed ahead and held)
        d = readlane_d(v[0], 0);
        estimate<0>();
        if constexpr (LDL) {
            const double e = __builtin_fma(-d, y, 1.0);
            inv = __builtin_fma(y, __builtin_fma(e, e, e), y);
        } else {
            const double e = __builtin_fma(-(d * y), y, 1.0);
            inv = __builtin_fma(e * y, __builtin_fma(e, 0.375, 0.5), y);
        }
        check<0>();
        column<0>();
        const uint32_t in = jb >= 32 ? ~0u : (1u << jb) - 1;
        if (lane == 0 && (bad & in)) atomicMin(status, col0 + __builtin_ctz(bad & in));
        if (LDL && lane == 0 && rep) atomicAdd(status + kStReplaced, __builtin_popcount(rep));
    }
    // the inverse times s to an LDS tile: X(c, q) at tile[c + 33 q]
    __device__ __forceinline__ void put_inverse(double* tile_g, double s)
    {
        auto o = lds(tile_g) + 33 * (lane & 31);
        if (lane >= 32) {
#pragma unroll
            for (int c = 0; c < NC; ++c) o[c] = s * v[c];
        }
    }
    // put(r, c, l_rc) for every row and column (L D L^T: d on the diagonal)
    template <class Put>
    __device__ __forceinline__ void put_rows(Put put)
    {
        if (lane < 32) {
            const double dr = LDL ? dg[lane < NC ? lane : 0] : 0.0;
#pragma unroll
            for (int c = 0; c < NC; ++c) put(lane, c, LDL && c == lane ? dr : v[c]);
        }
    }
};

// L U factorization without pivoting (the static pivoting of Section III:
// the elimination order is the analysis' order) of one 32x32 diagonal tile
// and the two inverses the panel solves use, in FP64, by one wave.  Lt
// (column-major, ld 33) holds the whole tile; rows and columns >= jb hold
// the identity.  The tile is kept twice: lane r < 32 holds row r, lane
// 32 + q holds column q (v); a second set of registers (z) holds column r of
// X = L^{-1} in lane r and column q of Y = U^{-T} in lane 32 + q, starting
// from unit vectors.  Step c: the pivot u_cc is broadcast by readlane; the
// row lanes scale their entry of column c to l_rc = a_rc / u_cc, the column
// lanes hold u_cq; both sets go to LDS (bc), and every lane updates
//   row lane r     v_q -= l_rc u_cq,     column lane q  v_p -= u_cq l_pc,
//   X lane         z_i -= l_ic z_c,      Y lane         z_i -= u_ci z_c (after z_c /= u_cc)
// for the indices past c (fmac_rows: the operand in l or u from a fixed lane
// of each row of 16).  Rows and columns up to c go on being updated; nothing
// reads them.  Out: out(c, lane, x, z) with x = l_rc (rows r > c) or u_cq
// (columns q >= c) and z = X(c, r) or Y(c, q), columns 0 .. jb - 1 rounded up
// to a multiple of 8.  Static pivoting and breakdown as in L D L^T.
// Bound: the multiply-adds (992) beside the chain of pivots (the next one
// formed by readlanes): FACT of 32 columns takes 31,200 cycles, 18,400 in
// L L^T, whose pass has 496.  The form
// before it (two passes, a broadcast LDS read per multiply-add, the code
// unrolled with a branch for each replaced pivot's retry) is part of the
// 490 us of a 256-wide FACT below.
template <class Out>
struct TileLu {
    double v[kNB], z[kNB];
    double inv, d, y, thr;
    int lane, jb, fail, nrep;
    __attribute__((address_space(3))) double* bc;
    Out out;

    __device__ __forceinline__ void estimate(int c, double x)
    {
        d = readlane_d(x, c);
        const bool rep = c < jb && fabs(d) < thr;
        d = rep ? (d < 0.0 ? -thr : thr) : d;
        nrep += rep ? 1 : 0;
        fail = (c < jb && !(d != 0.0 && d - d == 0.0) && fail == 32) ? c : fail;
        y = __builtin_amdgcn_rcp(d);
    }
    __device__ __forceinline__ void finish()
    {
        const double e = __builtin_fma(-d, y, 1.0);
        inv = __builtin_fma(y, __builtin_fma(e, e, e), y);
    }
    template <int C>
    __device__ __forceinline__ void columns()
    {
        const bool upper = lane >= 32;
        const double t = v[C];
        const double x0 = t * inv;
        double x = upper ? t : x0;
        const double zc = upper ? z[C] * inv : z[C];
        const double m = -x, mz = -zc;
        // (a replaced pivot: u_cc itself)
        if (lane == 32 + C) x = d;
        if constexpr (C + 1 < kNB) {
            bc[lane] = x;
            const double e = __builtin_fma(-x0, readlane_d(t, 33 + C), v[C + 1]);   // row lane C+1: the next pivot
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            // LDS operations of one wave complete in order: the reads see column C
            const int o = lane & 15, ow = (upper ? 0 : 32) + o, oz = (upper ? 32 : 0) + o;
            double w0 = 0.0, u0 = 0.0;
            if constexpr (C + 1 < 16) { w0 = bc[ow]; u0 = bc[oz]; }
            const double w1 = bc[ow + 16], u1 = bc[oz + 16];
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            estimate(C + 1, e);
            out(C, lane, x, zc);
            finish();
            if constexpr (C + 1 < 16) {
                fmac_rows<C + 1, 15 - C>(v, C + 1, w0, m);
                fmac_rows<C + 1, 15 - C>(z, C + 1, u0, mz);
            }
            constexpr int i = C + 1 > 16 ? C + 1 : 16;
            fmac_rows<i - 16, kNB - i>(v, i, w1, m);
            fmac_rows<i - 16, kNB - i>(z, i, u1, mz);
            if constexpr ((C & 7) == 7) {
                if (jb <= C + 1) return;
            }
            columns<C + 1>();
        } else {
            out(C, lane, x, zc);
        }
    }
};

template <class Out>
__device__ __forceinline__ void tile_lu_inv(double* Lt_g, double* bc_g, int jb, int col0, int32_t* status, Out out)
{
    auto Lt = lds(Lt_g);
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));   // (keeps the lane masks of the columns from being formed ahead and held)
    const int r = lane & 31;
    TileLu<Out> tc{{}, {}, 0.0, 0.0, 0.0, readlane_d(lds(bc_g)[kThrSlot], 0), lane, jb, 32, 0, lds(bc_g), out};
    const int base = lane >= 32 ? 33 * r : r, step = lane >= 32 ? 1 : 33;
#pragma unroll
    for (int c = 0; c < kNB; ++c) tc.v[c] = Lt[base + c * step];
#pragma unroll
    for (int c = 0; c < kNB; ++c) tc.z[c] = c == r ? 1.0 : 0.0;
    tc.estimate(0, tc.v[0]);
    tc.finish();
    tc.template columns<0>();
    if (lane == 0 && tc.fail < jb) atomicMin(status, col0 + tc.fail);
    if (lane == 0 && tc.nrep > 0) atomicAdd(status + kStReplaced, tc.nrep);
}

constexpr int kTSz = kNB * 33;                 // a 32x32 tile in LDS, column-major, ld 33
constexpr int kTiles = 256 / kNB;              // tiles of the widest block: the LDS buffer of every item but FACT's own

// A 32x32 block held by one wave, in the form of the matrix cores' results:
// b[h][q][v] of lane l holds M(16 q + l%16, 16 h + drow(v, l/16)).  As the
// inner index of a product may be taken in any order, provided both operands
// take the same one, this is also the form of an operand whose inner index
// is its column: results feed the next product without a pass through LDS.
template <class T>
struct Blk {
    typename MM<T>::acc b[2][2];
};

template <class T>
__device__ __forceinline__ void blk_zero(Blk<T>& m)
{
    zero_acc(m.b);
}

// rows row0.. of half h (16 columns) of the block at column col0 of g's
// array.  The whole offset is in the vector offset: the range check, which
// makes rows and columns past the array read as zero, does not see a scalar
// offset.
template <class T>
__device__ __forceinline__ void blk_load_half(T (&m)[2][4], const GOp& g, int row0, int col0, int h)
{
    const int lane = threadIdx.x & 63;
    const int vo = (lane & 15) * g.si + MM<T>::drow(0, lane >> 4) * g.sk;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            m[q][v] = gload<T>(g, vo + uni(g.off + (row0 + 16 * q) * g.si + (col0 + 16 * h + MM<T>::drow(v, 0)) * g.sk));
}

template <class T>
__device__ __forceinline__ void blk_load(Blk<T>& m, const GOp& g, int row0, int col0)
{
    T x[2][2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) blk_load_half<T>(x[h], g, row0, col0, h);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) m.b[h][q][v] = x[h][q][v];
}

// C += X Y^T of two blocks; LOW: the blocks of C on and below the diagonal
// only; YTRI: Y is lower triangular (its upper right quarter is zero)
template <class T, bool LOW, bool YTRI>
__device__ __forceinline__ void blk_mul(Blk<T>& C, const Blk<T>& X, const Blk<T>& Y)
{
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (LOW && h == 1 && q == 0) continue;
                    if (YTRI && h == 0 && p == 1) continue;
                    C.b[h][q] = MM<T>::mfma(Y.b[p][h][v], X.b[p][q][v], C.b[h][q]);
                }
}

// C += X Y with the result and Y transposed in the lanes (b[h][q][v] of lane
// l: row 16 h + drow(v, l/16), column 16 q + l%16); XTRI: X is lower triangular
template <class T, bool XTRI>
__device__ __forceinline__ void blk_mul_t(Blk<T>& C, const Blk<T>& X, const Blk<T>& Y)
{
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (XTRI && h == 0 && p == 1) continue;
                    C.b[h][q] = MM<T>::mfma(X.b[p][h][v], Y.b[p][q][v], C.b[h][q]);
                }
}

template <class T>
__device__ __forceinline__ void blk_sub(Blk<T>& m, const Blk<T>& o)
{
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 2; ++q) m.b[h][q] -= o.b[h][q];
}

template <class T>
__device__ __forceinline__ void blk_neg(Blk<T>& m)
{
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 2; ++q) m.b[h][q] = -m.b[h][q];
}

// the block to memory, rows < mv: M(r, c) at out[r sr + c sc]
template <class T, class P>
__device__ __forceinline__ void blk_store(const Blk<T>& m, P out, int64_t sr, int64_t sc, int mv)
{
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (16 * q + li < mv) out[(16 * q + li) * sr + (16 * h + MM<T>::drow(v, lk)) * sc] = m.b[h][q][v];
}

// a tile in LDS (column-major, ld 33) as a block, M(c, p) = tile[c + 33 p]
template <class T>
__device__ __forceinline__ void blk_from_lds(Blk<T>& m, const double* tile_g)
{
    auto tile = lds(tile_g);
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) m.b[h][q][v] = (T)tile[16 * q + li + 33 * (16 * h + MM<T>::drow(v, lk))];
}

// the block's columns times d[0..31] (LDS, FP64)
template <class T>
__device__ __forceinline__ void blk_scale(Blk<T>& m, const double* d_g)
{
    auto d = lds(d_g);
    const int lk = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const T dv = (T)d[16 * h + MM<T>::drow(v, lk)];
#pragma unroll
            for (int q = 0; q < 2; ++q) m.b[h][q][v] *= dv;
        }
}

// C += X Y^T over nblk 32-wide inner blocks: X(r, p) at row xr, inner index
// xp + p of gx (row = the array's row index), Y(c, p) likewise; SWAP: the
// result transposed in the lanes, C.b[h][q][v] = C(16 h + drow(v, l/16),
// 16 q + l%16), the operand form of a block whose inner index is its row.
// d: X's columns scaled by d[p] (LDS, indexed from inner index 0).  The
// next half block (16 inner indices) is in flight while the current one is
// multiplied.
template <class T, bool SWAP, bool DS>
__device__ __forceinline__ void blk_gemm(Blk<T>& C, const GOp& gx, int xr, int xp, const GOp& gy, int yr, int yp, int nblk,
                                         const double* d_g)
{
    if (nblk <= 0) return;
    const int lk = (threadIdx.x & 63) >> 4;
    T xa[2][4], ya[2][4], xb[2][4], yb[2][4];
    auto load = [&](T (&x)[2][4], T (&y)[2][4], int ch) {
        blk_load_half<T>(x, gx, xr, xp + 16 * ch, 0);
        blk_load_half<T>(y, gy, yr, yp + 16 * ch, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mma = [&](T (&x)[2][4], T (&y)[2][4], int ch) {
        if constexpr (DS) {
            auto d = lds(d_g);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const T dv = (T)d[16 * ch + MM<T>::drow(v, lk)];
#pragma unroll
                for (int q = 0; q < 2; ++q) x[q][v] *= dv;
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    C.b[h][q] = SWAP ? MM<T>::mfma(x[h][v], y[q][v], C.b[h][q]) : MM<T>::mfma(y[h][v], x[q][v], C.b[h][q]);
        __builtin_amdgcn_sched_barrier(0);
    };
    load(xa, ya, 0);
    for (int ch = 0; ch < 2 * nblk; ch += 2) {
        load(xb, yb, ch + 1);
        mma(xa, ya, ch);
        load(xa, ya, min(ch + 2, 2 * nblk - 1));   // (the last one repeats and is not used)
        mma(xb, yb, ch + 1);
    }
}

// Progress words of the row blocks of a diagonal block, in LDS: a wave waits
// until another one has published what it reads.  Every wait ends: row
// block i waits for row blocks < i only, and row block 0 for none.
__device__ __forceinline__ void wait_for(const int* flag_g, int value)
{
    auto flag = lds(flag_g);
    while (__hip_atomic_load(flag, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < value) __builtin_amdgcn_s_sleep(1);
}
// (all lanes store the same value; release: the wave's stores are visible
// to the workgroup first)
__device__ __forceinline__ void publish(int* flag_g, int value)
{
    __hip_atomic_store(lds(flag_g), value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// the same for data in LDS alone (stores to memory may still be on their way)
__device__ __forceinline__ void publish_lds(int* flag_g, int value)
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __hip_atomic_store(lds(flag_g), value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Block column c of the inverse D of a lower triangular w x w block L (its
// blocks below the diagonal at gL), below the tile D_cc:
//   D_Jc = -D_JJ sum_{c<=K<J} L_JK D_Kc,   J = c+1 .. nb-1,
// by one wave.  Every product is formed transposed in the lanes, so that its
// result is the operand of the next one; the last D_Kc stays in registers,
// the earlier ones are read back (the wave's own stores).  DS: L_JK d_K in
// place of L_JK (d in LDS).  LDSD: -D_JJ from LDS (tiles); otherwise D_JJ
// from memory.
template <class T, bool DS, bool LDSD>
__device__ __forceinline__ void inv_column(const GOp& gL, const GOp& gD, T* D, int w, int nb, int c, int* s_x, int* s_d,
                                           const double* tiles, const double* dd)
{
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    GOp gDt = gD;   // D^T(i, p) = D(p, i)
    gDt.si = gD.sk;
    gDt.sk = gD.si;
    Blk<T> N;   // -D_Kc of the last step, as an operand over its rows
    wait_for(&s_x[c], c + 1);   // D_cc in memory (and its tile in LDS)
    if constexpr (LDSD) {
        auto tile = lds(tiles + c * kTSz);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int v = 0; v < 4; ++v) N.b[h][q][v] = (T)tile[16 * h + MM<T>::drow(v, lk) + 33 * (16 * q + li)];
    } else {
        blk_load<T>(N, gDt, kNB * c, kNB * c);
        blk_neg<T>(N);
    }
    for (int J = c + 1; J < nb; ++J) {
        wait_for(&s_x[J], LDSD ? J : J + 1);
        Blk<T> C, L;
        blk_zero<T>(C);
        // minus the sum: K < J - 1 from memory, then K = J - 1
        blk_gemm<T, true, DS>(C, gL, kNB * J, kNB * c, gDt, kNB * c, kNB * c, J - 1 - c, dd + kNB * c);
        blk_load<T>(L, gL, kNB * J, kNB * (J - 1));
        if (DS) blk_scale<T>(L, dd + kNB * (J - 1));
        blk_neg<T>(C);
        blk_mul_t<T, false>(C, L, N);
        const int jb = min(kNB, w - kNB * J);
        if (jb < kNB) {   // rows of L past w are the panel's next rows: not to meet the zeros of D_JJ (0 x inf)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (16 * h + MM<T>::drow(v, lk) >= jb) C.b[h][q][v] = T(0);
        }
        // N = -D_Jc = (-D_JJ) (minus the sum)
        Blk<T> Dj;
        if constexpr (LDSD) {
            wait_for(s_d, J + 1);
            blk_from_lds<T>(Dj, tiles + J * kTSz);
        } else {
            blk_load<T>(Dj, gD, kNB * J, kNB * J);
            blk_neg<T>(Dj);
        }
        blk_zero<T>(N);
        blk_mul_t<T, true>(N, Dj, C);
        auto oD = glob(D + kNB * J + (int64_t)kNB * c * w);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = 16 * h + MM<T>::drow(v, lk);
                    if (r < jb) oD[r + (int64_t)(16 * q + li) * w] = -N.b[h][q][v];
                }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);   // (the wave's later loads of D_Jc follow its stores)
    }
}

// Cholesky factorization of the w x w diagonal block (w <= 256) of panel k
// and the inverse D = L_kk^{-1}, by one workgroup.  The block is cut into
// row blocks of 32; wave v owns the row blocks v and v + 4.  Row block i is
// a forward substitution against the finished row blocks above it,
//   L_iJ = (A_iJ - sum_{K<J} L_iK L_JK^T) D_JJ^T,   J = 0 .. i-1,
// then its diagonal tile A_ii - sum_K L_iK L_iK^T is factored and inverted
// (TileChol).  Nothing is updated in memory: a block is read once,
// collected on the matrix cores and written once.  The waves run as a
// pipeline without barriers: row block i takes L_J* as soon as row block J
// has published it (s_x) and D_JJ as soon as tile J is factored (s_d), so a
// step of the chain is one tile factorization, one 32x32 product with D_JJ
// and one with L_i,i-1; the long sums over K are formed ahead of it by waves
// that wait for D_JJ.  -D_JJ stays in LDS for the whole item, L_iJ in
// registers between the product that makes it and the ones that use it.
// The rest of the inverse follows by block columns,
//   D_Jc = -D_JJ sum_{c<=K<J} L_JK D_Kc,
// dealt to the waves as they run out of row blocks (the longest columns to
// the wave that is free first); a chain block leaves it to its INV item
// (full false).  Bound: the chain of 32-column tile factorizations.
// The right-looking form before it (trailing blocks read, updated and
// written in memory at every 32-column step, two barriers per step) took
// 294 us at w = 256 in FP64 and 252 us without the inverse's off-diagonal
// blocks, in a kernel of its own on an idle MI355X; this one 109 and 71 us
// (FP32 233 and 206 us before, 89 and 57 us now); the eight tiles are 34 of
// the 71 us.  A further row block of 32 costs 17,000 cycles up to 128 columns
// and 25,500 beyond, where a wave owns two.  With a wave's second row
// block begun after its first was finished it took 123 and 83 us: the sums
// of the last row blocks came late.
//
// LDL = true: L D L^T of the diagonal block (unit L with D on its diagonal,
// and Y = D^{-1} L^{-1} as the stored inverse, so that the panel solve and
// the rows below stay one product A_rows Y^T): the same with d between the
// factors of every product of two L's, and -Y_JJ in place of -D_JJ.
template <class T, bool LDL = false>
__device__ __noinline__ void task_fact(const SchedArgs& a, Geo g, bool full, double* Lt, double* tiles)
{
    const int f = uni(g.f), w = uni(g.w);
    const int64_t ld = g.ld;
    T* A = static_cast<T*>(a.panels) + g.poff;
    T* D = static_cast<T*>(a.dinv) + g.doff;
    const GOp gA = make_gop(A, ld * w, 0, 1, ld);           // A(i, p) at i + p*ld
    const GOp gD = make_gop(D, (int64_t)w * w, 0, 1, w);    // D(i, p) at i + p*w
    const int tid = threadIdx.x, wave = uni(tid >> 6), lane = tid & 63, li = lane & 15, lk = lane >> 4;
    double* bc = Lt + kNB * 33;
    __shared__ int s_x[8], s_d;      // blocks of row block i published (i + 1: D_ii too); tiles factored
    double* dd = ldl_pivots<LDL>();
    const int nb = (w + kNB - 1) / kNB;
    if (tid < 8) s_x[tid] = 0;
    if (tid == 8) s_d = 0;
    __syncthreads();
    // block J of row block i into the panel, and into the sum S of its tile.
    // (Entries past w are read from the rows below or as zeros and only
    // reach rows and columns past w; the sums are collected from zero and
    // subtracted once: fewer roundings than from A downwards.)
    auto step = [&](int i, int J, Blk<T>& S) {
        const int i0 = kNB * i;
        Blk<T> B, C, X;
        blk_load<T>(B, gA, i0, kNB * J);
        blk_zero<T>(C);
        if (J > 0) {
            wait_for(&s_x[J], J - 1);
            blk_gemm<T, false, LDL>(C, gA, i0, 0, gA, kNB * J, 0, J - 1, dd);
            wait_for(&s_x[J], J);
            blk_gemm<T, false, LDL>(C, gA, i0, kNB * (J - 1), gA, kNB * J, kNB * (J - 1), 1, dd + kNB * (J - 1));
        }
        blk_sub<T>(C, B);
        wait_for(&s_d, J + 1);
        blk_from_lds<T>(B, tiles + J * kTSz);
        blk_zero<T>(X);
        blk_mul<T, false, true>(X, C, B);   // (sum - A) (-D)^T
        blk_store<T>(X, glob(A + i0 + (int64_t)kNB * J * ld), 1, ld, min(kNB, w - i0));
        if (LDL) {
            Blk<T> Xd = X;
            blk_scale<T>(Xd, dd + kNB * J);
            blk_mul<T, true, false>(S, Xd, X);
        } else {
            blk_mul<T, true, false>(S, X, X);
        }
        publish(&s_x[i], J + 1);
    };
    // tile i: A_ii - S factored and inverted
    auto tile = [&](int i, const Blk<T>& S, const Blk<T>& B) {
        const int i0 = kNB * i, jb = min(kNB, w - i0);
        // identity padded, to LDS; row block i-1 is done with Lt (s_d)
        {
            auto L = lds(Lt);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int r = 16 * q + li, c = 16 * h + MM<T>::drow(v, lk);
                        L[r + 33 * c] = (r < jb && c < jb) ? (double)(B.b[h][q][v] - S.b[h][q][v]) : (r == c ? 1.0 : 0.0);
                    }
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
        }
        TileChol<kNB, LDL> tc;
        tc.load(Lt);
        tc.run(bc, LDL ? dd + i0 : bc, LDL ? readlane_d(lds(bc)[kThrSlot], 0) : 0.0, jb, f + i0, a.status);
        tc.put_inverse(tiles + i * kTSz, -1.0);
        publish_lds(&s_d, i + 1);
        // (masked entries go past the arrays, where the stores are dropped)
        const int vL = uni(gA.off + i0 * (gA.si + gA.sk)), vD = uni(gD.off + i0 * (gD.si + gD.sk));
        tc.put_rows([&](int r, int c, double x) { gstore_s(gA, r >= c && r < jb ? r * gA.si : kOffNone, uni(vL + c * gA.sk), (T)x); });
        auto Di = lds(tiles + i * kTSz);
        const int r = lane & 31;
#pragma unroll
        for (int cb = 0; cb < kNB; cb += 2) {
            const int c = cb + (lane >> 5);
            gstore_s(gD, r >= c && r < jb ? r * gD.si + c * gD.sk : kOffNone, vD, (T)-Di[r + 33 * c]);
        }
        publish(&s_x[i], i + 1);
    };
    // a wave's row blocks v and v + 4 go on side by side: block J of both as
    // soon as tile J is there, the first row block's, which is nearer in the
    // chain, ahead
    const int i1 = wave, i2 = wave + kThreads / 64;
    Blk<T> S1, S2, B;
    blk_zero<T>(S1);
    blk_zero<T>(S2);
    if (i1 < nb) {
        for (int J = 0; J + 1 < i1; ++J) {
            step(i1, J, S1);
            if (i2 < nb) step(i2, J, S2);
        }
        blk_load<T>(B, gA, kNB * i1, kNB * i1);   // (requested ahead of the last wait)
        if (i1 > 0) step(i1, i1 - 1, S1);
        tile(i1, S1, B);
    }
    if (i2 < nb) {
        for (int J = max(0, i1 - 1); J + 1 < i2; ++J) step(i2, J, S2);
        blk_load<T>(B, gA, kNB * i2, kNB * i2);
        step(i2, i2 - 1, S2);
        tile(i2, S2, B);
    }
    if (!full) return;
    // block columns of the inverse: wave v takes column v (first the columns
    // 0 .. 3 with the most blocks; wave 0 runs out of row blocks first), then
    // the short columns 4 .. 6 go to the waves 3, 2, 1
    for (int t = 0; t < 2; ++t) {
        const int c = t == 0 ? wave : 7 - wave;
        if (c + 1 < nb) inv_column<T, LDL, true>(gA, gD, D, w, nb, c, s_x, &s_d, tiles, dd);
    }
}

// ---------------------------------------------------------------- FACT(k), L U
// L U factorization of the w x w diagonal block (w <= 256) of panel k, in
// place in the L panel (unit L below the diagonal, U on and above), with the
// inverses X = L_kk^{-1} (L inverse array) and Y = U_kk^{-T} (U inverse
// array), both lower triangular, by one workgroup: the row-block pipeline of
// task_fact with two sides.  Row block i holds its rows of L and its rows of
// U^T, Z_iJ = U_Ji^T:
//   L_iJ = (A_iJ - sum_{K<J} L_iK Z_JK^T) Y_JJ^T
//   Z_iJ = (A_Ji^T - sum_{K<J} Z_iK L_JK^T) X_JJ^T,   J = 0 .. i-1,
// then the tile A_ii - sum_K L_iK Z_iK^T is factored and inverted
// (tile_lu_inv), and after the row blocks the block columns of both
// inverses follow (inv_column with L, and with U^T).  -X_JJ and -Y_JJ of the
// last four tiles are kept in LDS; earlier ones are read back from memory:
// row block J+4 overwrites tile J's after row block J+3 is factored, so only
// the row blocks up to J+3 take it from LDS.  At w = 256 in FP64 the
// right-looking form before it took 490 us in a kernel of its own (FP32
// 410), this one 246 to 257 us (216 to 224), and 147 to 157 (116 to 120)
// without the inverses' off-diagonal blocks, as on the chain; with a panel
// stride that is a multiple of 64, 291 and 167 (247, 129).
template <class T>
__device__ __noinline__ void task_fact_lu(const SchedArgs& a, Geo g, bool full, double* Lt, double* tiles)
{
    const int f = uni(g.f), w = uni(g.w);
    const int64_t ld = g.ld;
    T* A = static_cast<T*>(a.panels) + g.poff;
    T* X = static_cast<T*>(a.dinv) + g.doff;
    T* Y = X + a.uinv;
    const GOp gA = make_gop(A, ld * w, 0, 1, ld);    // A(i, p) at i + p*ld
    const GOp gAt = make_gop(A, ld * w, 0, ld, 1);   // A^T
    const GOp gX = make_gop(X, (int64_t)w * w, 0, 1, w), gY = make_gop(Y, (int64_t)w * w, 0, 1, w);
    const int tid = threadIdx.x, wave = uni(tid >> 6), lane = tid & 63, li = lane & 15, lk = lane >> 4;
    double* bc = Lt + kNB * 33;
    __shared__ int s_x[8], s_d;   // blocks of row block i published (i + 1: its inverse tiles too); tiles factored
    const int nb = (w + kNB - 1) / kNB;
    if (tid < 8) s_x[tid] = 0;
    if (tid == 8) s_d = 0;
    __syncthreads();
    auto step = [&](int i, int J, Blk<T>& S) {
        const int i0 = kNB * i, jb = min(kNB, w - i0);
        Blk<T> CL, CU, Q;
        blk_zero<T>(CL);
        blk_zero<T>(CU);
        if (J > 0) {
            wait_for(&s_x[J], J - 1);
            blk_gemm<T, false, false>(CL, gA, i0, 0, gAt, kNB * J, 0, J - 1, nullptr);
            blk_gemm<T, false, false>(CU, gAt, i0, 0, gA, kNB * J, 0, J - 1, nullptr);
            wait_for(&s_x[J], J);
            blk_gemm<T, false, false>(CL, gA, i0, kNB * (J - 1), gAt, kNB * J, kNB * (J - 1), 1, nullptr);
            blk_gemm<T, false, false>(CU, gAt, i0, kNB * (J - 1), gA, kNB * J, kNB * (J - 1), 1, nullptr);
        }
        blk_load<T>(Q, gA, i0, kNB * J);
        blk_sub<T>(CL, Q);
        blk_load<T>(Q, gAt, i0, kNB * J);
        blk_sub<T>(CU, Q);
        Blk<T> XL, XU;
        blk_zero<T>(XL);
        blk_zero<T>(XU);
        if (J + 3 >= i) {
            wait_for(&s_d, J + 1);
            blk_from_lds<T>(Q, tiles + (2 * (J & 3) + 1) * kTSz);
            blk_mul<T, false, true>(XL, CL, Q);
            blk_from_lds<T>(Q, tiles + 2 * (J & 3) * kTSz);
            blk_mul<T, false, true>(XU, CU, Q);
        } else {
            wait_for(&s_x[J], J + 1);
            blk_load<T>(Q, gY, kNB * J, kNB * J);
            blk_neg<T>(Q);
            blk_mul<T, false, true>(XL, CL, Q);
            blk_load<T>(Q, gX, kNB * J, kNB * J);
            blk_neg<T>(Q);
            blk_mul<T, false, true>(XU, CU, Q);
        }
        blk_store<T>(XL, glob(A + i0 + (int64_t)kNB * J * ld), 1, ld, jb);
        blk_store<T>(XU, glob(A + kNB * J + (int64_t)i0 * ld), ld, 1, jb);
        blk_mul<T, false, false>(S, XL, XU);
        publish(&s_x[i], J + 1);
    };
    auto tile = [&](int i, const Blk<T>& S) {
        const int i0 = kNB * i, jb = min(kNB, w - i0);
        // identity padded, to LDS; row block i-1 is done with Lt (s_d)
        {
            Blk<T> B;
            blk_load<T>(B, gA, i0, i0);
            auto L = lds(Lt);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int r = 16 * q + li, c = 16 * h + MM<T>::drow(v, lk);
                        L[r + 33 * c] = (r < jb && c < jb) ? (double)(B.b[h][q][v] - S.b[h][q][v]) : (r == c ? 1.0 : 0.0);
                    }
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
        }
        auto Ti = lds(tiles + 2 * (i & 3) * kTSz);   // -X_ii, then -Y_ii
        const int vL = uni(gA.off + i0 * gA.si + i0 * gA.sk), vD = uni(i0 * (gX.si + gX.sk));
        auto out = [&](int c, int ln, double x, double z) {
            // (masked entries go past the array, where the store is dropped)
            const int r = ln & 31;
            const int vo = ln >= 32 ? (r >= c && r < jb && c < jb ? c * gA.si + r * gA.sk : kOffNone)
                                    : (r > c && r < jb && c < jb ? r * gA.si + c * gA.sk : kOffNone);
            gstore_s(gA, vo, vL, (T)x);
            Ti[(ln >= 32 ? kTSz : 0) + 33 * r + c] = -z;
        };
        tile_lu_inv(Lt, bc, jb, f + i0, a.status, out);
        publish_lds(&s_d, i + 1);
        const int r = lane & 31;
#pragma unroll
        for (int cb = 0; cb < kNB; cb += 2) {
            const int c = cb + (lane >> 5), vo = r >= c && r < jb ? r * gX.si + c * gX.sk : kOffNone;
            gstore_s(gX, vo, vD, (T)-Ti[r + 33 * c]);
            gstore_s(gY, vo, vD, (T)-Ti[kTSz + r + 33 * c]);
        }
        publish(&s_x[i], i + 1);
    };
    // (the two row blocks of a wave side by side, as in task_fact)
    const int i1 = wave, i2 = wave + kThreads / 64;
    Blk<T> S1, S2;
    blk_zero<T>(S1);
    blk_zero<T>(S2);
    if (i1 < nb) {
        for (int J = 0; J + 1 < i1; ++J) {
            step(i1, J, S1);
            if (i2 < nb) step(i2, J, S2);
        }
        if (i1 > 0) step(i1, i1 - 1, S1);
        tile(i1, S1);
    }
    if (i2 < nb) {
        for (int J = max(0, i1 - 1); J < i2; ++J) step(i2, J, S2);
        tile(i2, S2);
    }
    if (!full) return;   // (left to the INV item)
    // block columns 0 .. nb - 2 of both inverses, dealt as in task_fact
    for (int t = 0; t < 4; ++t) {
        const int c = (t & 2) == 0 ? wave : 7 - wave;
        if (c + 1 >= nb) continue;
        if ((t & 1) == 0) inv_column<T, false, false>(gA, gX, X, w, nb, c, s_x, &s_d, tiles, nullptr);
        else inv_column<T, false, false>(gAt, gY, Y, w, nb, c, s_x, &s_d, tiles, nullptr);
    }
}

// ---------------------------------------------------------------- INV(k)
// The off-diagonal tiles of the kept inverse after a FACT that stored the
// factor and the diagonal tiles D_JJ only (blocks of elimination chains: the
// inverse is then built beside the chain instead of inside FACT): the block
// columns of inv_column, two per wave; L U: of both inverses.
template <class T, bool LDL, bool LU>
__device__ __noinline__ void task_inv(const SchedArgs& a, Geo g)
{
    const int w = uni(g.w);
    const int64_t ld = g.ld;
    const T* A = static_cast<const T*>(a.panels) + g.poff;
    T* D = static_cast<T*>(a.dinv) + g.doff;
    const GOp gA = make_gop(A, ld * w, 0, 1, ld);
    const int tid = threadIdx.x, wave = uni(tid >> 6), nb = (w + kNB - 1) / kNB;
    __shared__ int s_x[8], s_d;
    double* dd = ldl_pivots<LDL>();
    if (tid < 8) s_x[tid] = 9;   // everything is there
    if (tid == 8) s_d = 9;
    if (LDL && tid < w) dd[tid] = (double)A[tid * (ld + 1)];
    __syncthreads();
    for (int t = 0; t < 2; ++t) {
        const int c = t == 0 ? wave : 7 - wave;
        if (c + 1 >= nb) continue;
        inv_column<T, LDL, false>(gA, make_gop(D, (int64_t)w * w, 0, 1, w), D, w, nb, c, s_x, &s_d, nullptr, dd);
        if constexpr (LU) {
            T* Y = D + a.uinv;
            inv_column<T, false, false>(make_gop(A, ld * w, 0, ld, 1), make_gop(Y, (int64_t)w * w, 0, 1, w), Y, w, nb, c, s_x, &s_d,
                                        nullptr, nullptr);
        }
    }
}

// ---------------------------------------------------------------- TRSM(k, rows)
// Rows [row0, row0+nrows) (nrows <= 64 * (4 / ceil(w / 64))) of panel k below its diagonal block
// are replaced by B L_kk^{-T} = B D^T.  Wave v computes the 64 output columns
// starting at 64v; the inner range stops at the diagonal of the lower
// triangular D.  poff / doff select the panel array and the inverse (L U:
// the L rows take U_kk^{-T}, giving A_off U_kk^{-1}; the U^T rows take
// L_kk^{-1}, giving A_up^T L_kk^{-T}).
// RB: 16-row blocks per wave tile (4: 64-row wave tiles; 1: the thin items
// of elimination chains, a quarter of the work per wave).
template <class T, int RB = 4>
__device__ __noinline__ void task_trsm(const SchedArgs& a, Geo g, int row0, int nrows, int64_t poff = 0,
                                       int64_t doff = 0)
{
    const int w = g.w;
    const int64_t ld = g.ld;
    T* P = static_cast<T*>(a.panels) + poff + g.poff;
    auto B = glob(P + row0);
    const T* D = static_cast<const T*>(a.dinv) + doff + g.doff;
    const int wave = threadIdx.x >> 6;
    typename MM<T>::acc acc[4][RB];
    zero_acc(acc);
    // (16 RB) x 64 wave tiles: ncb column blocks of the output, and 4/ncb
    // blocks of 16 RB rows (a chunk has 16 RB * (4/ncb) rows), so narrow
    // panels keep all four waves busy
    constexpr int TR = 16 * RB;
    const int ncb = (w + 63) >> 6, nrb = 4 / ncb;
    const int cb = wave % ncb, rb = wave / ncb;
    const int c0 = 64 * cb, r0 = TR * rb;
    const int nv = min(64, w - c0);
    const bool on = rb < nrb && nv > 0 && r0 < nrows;
    if (on)
        tile_gemm<4, T, RB>(acc, make_gop(P, ld * w, row0 + r0, 1, ld), make_gop(D, (int64_t)w * w, c0, 1, w),
                            min(w, c0 + 64), a.split != 0);
    __syncthreads();   // every wave has read all of B before any result is written
    if (on)
        wave_store<T>(acc, min(TR, nrows - r0), nv,
                      [&](int r, int c, T v) { B[(r0 + r) + (int64_t)(c0 + c) * ld] = v; });
}

// Rows [row0, row0+nrows) (nrows <= 16) of a chain block's panel below its
// diagonal block, by block forward substitution with the diagonal tiles of
// the inverse only (the rest of the inverse is formed beside the chain, by
// the INV item):
//   X_J = (B_J - sum_{K<J} X_K L_JK^T) D_JJ^T,   J = 0 .. nb-1   (X = B L_kk^{-T}),
// by the four waves together: wave v owns the column blocks v and v + 4.  A
// finished X_K goes to LDS as it lies in the lanes (results have the form of
// operands, see Blk) and every wave adds its product to the sums of its own
// later blocks while the owner of the next one goes on; L_JK for the next
// K is on its way meanwhile.  L D L^T: X_K D_K is what goes to LDS (Y_JJ in
// place of D_JJ); L U: the L rows take U_kk^T and Y_JJ (uside 0), the U^T
// rows L_kk and X_JJ (uside 1).
// A chain link waits for these items, so they are cut for latency: 28
// products of 16x16x4 per step of the substitution.  One wave per 16 rows
// with all of its blocks (576 products in a row at 256 columns) took 36 us
// on the chain, this form 20 to 24 us.
template <class T, bool LDL, bool LU>
__device__ __noinline__ void task_trsm_chain(const SchedArgs& a, Geo g, int row0, int nrows, int uside, double* tiles)
{
    typedef typename MM<T>::acc acc_t;
    const int w = uni(g.w);
    const int64_t ld = g.ld;
    const T* A = static_cast<const T*>(a.panels) + g.poff;
    T* P = static_cast<T*>(a.panels) + g.poff + (LU && uside ? a.upanel : 0);
    const T* D = static_cast<const T*>(a.dinv) + g.doff + (LU && !uside ? a.uinv : 0);
    const int tid = threadIdx.x, wave = uni(tid >> 6), lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int nb = (w + kNB - 1) / kNB;
    const GOp gP = make_gop(P, ld * w, row0, 1, ld);
    const GOp gA = make_gop(A, ld * w, 0, 1, ld);
    const GOp gL = LU && !uside ? make_gop(A, ld * w, 0, ld, 1) : gA;   // (c, p) of L_kk or U_kk^T
    const GOp gD = make_gop(D, (int64_t)w * w, 0, 1, w);
    T* xs = reinterpret_cast<T*>(tiles);   // X_K: entry s of lane l at (8 K + s) * 64 + l
    __shared__ int s_t[8];                 // X_K is in LDS
    if (tid < 8) s_t[tid] = 0;
    __syncthreads();
    // rows 0..15 of a block row, columns col0.. of g: m[p][v] = M(li, 16 p + drow(v, lk))
    auto load = [&](T (&m)[2][4], const GOp& g, int r0, int col0) {
        const int vo = li * g.si + MM<T>::drow(0, lk) * g.sk;
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v) m[p][v] = gload<T>(g, vo + uni(g.off + r0 * g.si + (col0 + 16 * p + MM<T>::drow(v, 0)) * g.sk));
    };
    // (everything in flight at once fits the registers: the tile of D and the
    // pivots of one own block at a time, L_JK of the next K into the
    // registers of the last)
    T B[2][2][4], L[2][2][2][4], Dj[2][2][4], d[2][4];   // [own block][column tile][p][v]
    acc_t S[2][2];
    auto load_own = [&](int J) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            load(Dj[h], gD, kNB * J + 16 * h, kNB * J);
#pragma unroll
            for (int v = 0; v < 4 && LDL; ++v)
                d[h][v] = gload<T>(gA, (kNB * J + 16 * h + MM<T>::drow(v, lk)) * (gA.si + gA.sk));
        }
    };
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        load(B[o], gP, 0, kNB * (wave + 4 * o));   // (blocks past w read zeros and are not used)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            load(L[o][h], gL, kNB * (wave + 4 * o) + 16 * h, 0);
            S[o][h] = acc_t{0, 0, 0, 0};
        }
    }
    load_own(wave);
    for (int K = 0; K < nb; ++K) {
        if ((K & 3) == wave) {
            // X_K = (B_K - S) D_KK^T; columns past w count zero
            T x[2][4];
            const int jb = w - kNB * K;
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const T r = K < 4 ? B[0][p][v] - S[0][p][v] : B[1][p][v] - S[1][p][v];
                    x[p][v] = 16 * p + MM<T>::drow(v, lk) < jb ? r : T(0);
                }
            acc_t X[2] = {acc_t{0, 0, 0, 0}, acc_t{0, 0, 0, 0}};
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int h = p; h < 2; ++h) X[h] = MM<T>::mfma(Dj[h][p][v], x[p][v], X[h]);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int v = 0; v < 4; ++v) lds(xs)[(8 * K + 4 * h + v) * 64 + lane] = LDL ? X[h][v] * d[h][v] : X[h][v];
            publish_lds(&s_t[K], 1);
            auto out = glob(P);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int c = 16 * h + MM<T>::drow(v, lk);
                    if (li < nrows && c < jb) out[(row0 + li) + (int64_t)(kNB * K + c) * ld] = X[h][v];
                }
            if (K < 4) load_own(wave + 4);
        }
        if (K + 1 >= nb || K >= wave + 4) continue;   // no own block after K
        wait_for(&s_t[K], 1);
        T x[2][4];
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v) x[p][v] = lds(xs)[(8 * K + 4 * p + v) * 64 + lane];
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            if (o == 0 && K >= wave) continue;
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int h = 0; h < 2; ++h) S[o][h] = MM<T>::mfma(L[o][h][p][v], x[p][v], S[o][h]);
#pragma unroll
            for (int h = 0; h < 2; ++h) load(L[o][h], gL, kNB * (wave + 4 * o) + 16 * h, kNB * (K + 1));
        }
    }
}

// ---------------------------------------------------------------- UPDATE
// W = L_k[row0 : row0+mrows] * L_k[col0 : col0+ncols]^T (inner dimension =
// width of k), C_j[rmap(row), rmap(col)] -= W on the lower triangle of j.
// rmap (precomputed from the symbolic structure) gives, for every panel row
// of k from the first block facing j on, its row inside panel j; for facing
// rows that is also the column of j.  Two tile shapes: ncols <= 64 and
// mrows <= 256 (the four waves cover 64 rows each), or 64 < ncols <= 128 and
// mrows <= 128 (the waves form a 2x2 grid of 64x64 wave tiles).  A merged
// item (np > 1, kind bits 8..) sums the products of the np consecutive
// pieces k-np+1 .. k of a split supernode (piece p's rows are k's rows
// shifted by fcol[k] - fcol[p]) before its one scatter.  LDL: each
// piece's product is L_p[rows] D_p L_p[cols]^T, D_p on the diagonal of panel p.
// LU: the tile covers the whole square of the facing rows (no triangle);
// W_L = L_k[rows] U^T_k[cols]^T goes to j's L panel (its square diagonal
// block included), and, for rows below j's diagonal block, W_U =
// U^T_k[rows] L_k[cols]^T to j's U^T panel.
// RB = 1: a thin tile (levels with little work), at most 64 x 64, each wave
// 16 rows of it (a quarter of the work of a 64-row wave tile).
template <class T, bool LDL = false, bool LU = false, int RB = 4>
__device__ __noinline__ void task_update(const SchedArgs& a, const int4 d0, const int4 d1, const int4 d2, const int4 d3,
                                         int* rpos_g, int* cpos_g)
{
    // the row and column maps are LDS arrays of the calling kernel: stated,
    // so that their accesses are LDS operations without a generic-address
    // test (whether the compiler derives it depends on the set of callers)
    auto rpos = lds(rpos_g);
    auto cpos = lds(cpos_g);
    const DevPlan& pl = a.pl;
    const int k = d0.y, j = d0.z, row0 = d0.w, np = ((d0.x >> 8) & 15) + 1;
    const int mrows = d1.x, col0 = d1.y, ncols = d1.z, mbase = d1.w;
    const int64_t ldj = d2.y;
    auto Cg = glob(static_cast<T*>(a.panels) + words64(d2.z, d2.w));
    const int tid = threadIdx.x, wave = tid >> 6;
    if (tid < mrows) rpos[tid] = a.rmap[mbase + row0 + tid];
    if (tid < ncols) cpos[tid] = a.rmap[mbase + col0 + tid];
    __syncthreads();
    const bool square = RB == 4 && ncols > 64;
    const int r0 = square ? 64 * (wave & 1) : 16 * RB * wave;
    const int c0 = square ? 64 * (wave >> 1) : 0;
    const int mv = min(16 * RB, mrows - r0), nv = min(64, ncols - c0);
    if (mv > 0 && nv > 0) {
        // half 0: W = X Y^T with X the rows and Y the facing rows of the L
        // panels (L U: Y from the U^T panels); half 1 (L U, rows below j's
        // diagonal block only): X from the U^T panels, Y from the L panels
        const int wj = LU ? pl.lcol[j] - pl.fcol[j] + 1 : 0;
        const int nhalf = (LU && rpos[r0 + mv - 1] >= wj) ? 2 : 1;
        for (int half = 0; half < nhalf; ++half) {
            typename MM<T>::acc acc[4][RB];
            zero_acc(acc);
            const int64_t xo = (LU && half == 1) ? a.upanel : 0, yo = (LU && half == 0) ? a.upanel : 0;
            // piece p = k first (its geometry is in the descriptor); a piece
            // before it has as many more panel rows as it has columns, and
            // its panel ends where the next one begins
            int w = d3.x, sh = 0;
            int64_t ld = d3.y, po = words64(d3.z, d3.w);
            for (int p = k;; --p) {
                int wn = 0;   // width of the next piece, on its way meanwhile
                if (p > k - np + 1) wn = pl.lcol[p - 1] - pl.fcol[p - 1] + 1;
                const T* A = static_cast<const T*>(a.panels) + po;
                if constexpr (LDL)
                    tile_gemm<4, T, RB, true>(acc, make_gop(A, ld * w, row0 + r0 + sh, 1, ld),
                                              make_gop(A, ld * w, col0 + c0 + sh, 1, ld), w, a.split != 0,
                                              make_gop(A, ld * w, 0, 0, ld + 1));
                else
                    tile_gemm<4, T, RB>(acc, make_gop(A + xo, ld * w, row0 + r0 + sh, 1, ld),
                                        make_gop(A + yo, ld * w, col0 + c0 + sh, 1, ld), w, a.split != 0);
                if (p == k - np + 1) break;
                sh += wn;
                ld += wn;
                po -= ld * wn;
                w = wn;
            }
            if constexpr (LU) {
                auto Cu = Cg + (half == 1 ? a.upanel : 0);
                wave_store<T>(acc, mv, nv, [&](int r, int c, T v) {
                    const int tr = rpos[r0 + r], tc = cpos[c0 + c];
                    if (half == 0 || tr >= wj) __hip_atomic_fetch_add(Cu + (int64_t)tc * ldj + tr, -v, __ATOMIC_RELAXED, AGENT);
                });
            } else {
                wave_store<T>(acc, mv, nv, [&](int r, int c, T v) {
                    const int tr = rpos[r0 + r], tc = cpos[c0 + c];
                    if (tr >= tc) __hip_atomic_fetch_add(Cg + (int64_t)tc * ldj + tr, -v, __ATOMIC_RELAXED, AGENT);
                });
            }
        }
    }
}

// ---------------------------------------------------------------- queues
__device__ __forceinline__ void push_items(const SchedArgs& a, bool hp, int base, int first, int count)
{
    int32_t* q = hp ? a.hp_queue : a.queue;
    const int cap = hp ? a.hp_total : a.total_normal;
    for (int i = threadIdx.x; i < count; i += kThreads) {
        if (base + i < cap)
            __hip_atomic_store(&q[base + i], first + i, __ATOMIC_RELAXED, AGENT);
        else
            __hip_atomic_store(&a.status[kStAbort], 2, __ATOMIC_RELAXED, AGENT);   // more pushes than slots
    }
}

// Deterministic mode: queue the items of pair p (one thread).
__device__ __forceinline__ void push_pair(const SchedArgs& a, int p)
{
    const int4 q = a.pairs[p];
    const bool hp = q.w != 0;
    int32_t* qu = hp ? a.hp_queue : a.queue;
    const int cap = hp ? a.hp_total : a.total_normal;
    const int base = __hip_atomic_fetch_add(hp ? a.hp_tail : a.qtail, q.y, __ATOMIC_RELAXED, AGENT);
    for (int i = 0; i < q.y; ++i) {
        if (base + i < cap)
            __hip_atomic_store(&qu[base + i], q.x + i, __ATOMIC_RELAXED, AGENT);
        else
            __hip_atomic_store(&a.status[kStAbort], 2, __ATOMIC_RELAXED, AGENT);
    }
}

// Deterministic mode: the pairs of source k lose their panel dependency
// (all threads of the workgroup; out of line, so that the scheduler loop
// does not keep its registers).
__device__ __noinline__ void release_pairs(const SchedArgs& a, int k)
{
    for (int p = a.kpair[k] + threadIdx.x; p < a.kpair[k + 1]; p += kThreads)
        if (__hip_atomic_fetch_add(&a.pdep[p], -1, __ATOMIC_RELAXED, AGENT) == 1) push_pair(a, p);
}

// Count down one update tile of a target (j: the item that factors it); queue
// that item when it was the last one (any lane).
__device__ __forceinline__ void finish_update(const SchedArgs& a, int j)
{
    if (__hip_atomic_fetch_add(&a.fact_dep[j], -1, __ATOMIC_RELAXED, AGENT) != 1) return;
    const bool hp = a.hp_item[j] != 0;
    const int slot = __hip_atomic_fetch_add(hp ? a.hp_tail : a.qtail, 1, __ATOMIC_RELAXED, AGENT);
    if (slot < (hp ? a.hp_total : a.total_normal))
        __hip_atomic_store(&(hp ? a.hp_queue : a.queue)[slot], j, __ATOMIC_RELAXED, AGENT);
    else
        __hip_atomic_store(&a.status[kStAbort], 2, __ATOMIC_RELAXED, AGENT);
}

// ---------------------------------------------------------------- fused small block
// A column block of width w <= 32 with at most 128 panel rows as one item:
// the panel is read into LDS once; the diagonal block is factored and
// inverted (TileChol); the rows below become A_off D^T; every update
// tile of the block (fused-tile table) is formed from the LDS copy and
// scattered with the atomics of the update items; then the item counts its
// targets down.  Blocks at the bottom of the elimination
// tree of small systems are a few columns wide: as separate factor, solve
// and update items each paid several queue round trips and chains of
// dependent metadata loads for a few hundred flops.  Products accumulate in
// FP64 from the stored (type T) values.  LDL: the tile is factored as
// L D L^T (static pivoting as in FACT), the rows below become A_off Y^T with
// Y = D^{-1} L^{-1}, and the update products take d_t (FP64, from the
// factored tile) between the two rows.
constexpr int kSLd = kSmallRows + 1;   // leading dimension of the LDS panel copy
static_assert(kSLd * kNB * sizeof(float) + (kSmallMap + 8 * kSmallMaxUpd) * sizeof(int) +
                      kSmallMaxUpd * sizeof(int64_t) <= (kTiles - 1) * kTSz * sizeof(double),
              "small-block tables exceed the LDS row buffer");
static_assert((kSLd * kNB * sizeof(float) + (kSmallMap + 8 * kSmallMaxUpd) * sizeof(int)) % 8 == 0,
              "misaligned small-block offset table");
static_assert(kSmallRows * kNB % kThreads == 0, "rows below per thread");

template <class T, bool LDL = false>
__device__ __noinline__ void task_small(const SchedArgs& a, Geo g, const int4 d1, double* Lt, double* Dt, T* Pb)
{
    const int tfirst = d1.x, nupd = d1.y, mstart = d1.z, mlen = d1.w;
    const int f = g.f, w = g.w, ld = g.ld;
    const int R = ld - w;   // rows below the diagonal block
    T* A = static_cast<T*>(a.panels) + g.poff;
    T* D = static_cast<T*>(a.dinv) + g.doff;
    T* S = Pb;                                                // S[r + c*kSLd] for panel rows r >= w
    int* smap = reinterpret_cast<int*>(S + kSLd * kNB);       // row-map entries mstart ..
    int* dtab = smap + kSmallMap;                             // per tile: j, row0, mrows, col0, ncols, map base, ldj
    int64_t* dpo = reinterpret_cast<int64_t*>(dtab + 8 * kSmallMaxUpd);   // panel offset of the target
    double* bc = Lt + kNB * 33;
    const int tid = threadIdx.x, wave = tid >> 6;
    for (int idx = tid; idx < kNB * kNB; idx += kThreads) {
        const int r = idx & 31, c = idx >> 5;
        Lt[r + c * 33] = (r < w && c < w) ? (c <= r ? (double)A[r + (int64_t)c * ld] : 0.0) : (r == c ? 1.0 : 0.0);
    }
    for (int idx = tid; idx < R * w; idx += kThreads) {
        const int i = idx % R, c = idx / R;
        S[(w + i) + c * kSLd] = A[(w + i) + (int64_t)c * ld];
    }
    for (int idx = tid; idx < mlen; idx += kThreads) smap[idx] = a.rmap[mstart + idx];
    if (tid < nupd) {
        const int4* ft = a.ftab + 3 * (int64_t)(tfirst + tid);
        const int4 u0 = ft[0], u1 = ft[1], u2 = ft[2];
        int* e = dtab + 8 * tid;
        e[0] = u0.x;
        e[1] = u0.y;
        e[2] = u0.z;
        e[3] = u0.w;
        e[4] = u1.x;
        e[5] = u1.y - mstart;
        e[6] = u1.z;
        dpo[tid] = words64(u2.x, u2.y);
    }
    __syncthreads();
    if (wave == 0) {
        auto tile = [&](auto nc) {
            TileChol<decltype(nc)::value, LDL> tc;
            tc.load(Lt);
            tc.run(bc, bc + 64, LDL ? readlane_d(lds(bc)[kThrSlot], 0) : 0.0, w, f, a.status);
            tc.put_inverse(Dt, 1.0);
            tc.put_rows([&](int r, int c, double x) { lds(Lt)[r + 33 * c] = x; });
        };
        if (w <= 8) tile(std::integral_constant<int, 8>());
        else if (w <= 16) tile(std::integral_constant<int, 16>());
        else tile(std::integral_constant<int, 32>());
    }
    __syncthreads();
    for (int idx = tid; idx < kNB * kNB; idx += kThreads) {
        const int r = idx & 31, c = idx >> 5;
        if (r < w && c <= r) {
            A[r + (int64_t)c * ld] = (T)Lt[r + c * 33];
            D[r + (int64_t)c * w] = (T)Dt[r + c * 33];
        }
    }
    // rows below: P = A_off D^T, D lower triangular
    constexpr int kPer = kSmallRows * kNB / kThreads;
    double p[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int idx = tid + q * kThreads;
        double acc = 0.0;
        if (idx < R * w) {
            const int i = idx % R, c = idx / R;
            for (int t = 0; t <= c; ++t) acc += (double)S[(w + i) + t * kSLd] * (double)(T)Dt[c + t * 33];
        }
        p[q] = acc;
    }
    __syncthreads();   // every product has read its row of S
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int idx = tid + q * kThreads;
        if (idx < R * w) {
            const int i = idx % R, c = idx / R;
            const T v = (T)p[q];
            S[(w + i) + c * kSLd] = v;
            A[(w + i) + (int64_t)c * ld] = v;
        }
    }
    __syncthreads();
    // update tiles: C_j[rmap(r), rmap(c)] -= P_r . P_c (L D L^T: P_r D P_c) on
    // the lower triangle of j
    double* dg = bc + 64;   // (L D L^T) the pivots d_t
    if (LDL && tid < w) dg[tid] = Lt[tid * 34];
    __syncthreads();
    for (int u = 0; u < nupd; ++u) {
        const int* e = dtab + 8 * u;
        const int row0 = e[1], mrows = e[2], col0 = e[3], ncols = e[4], mb = e[5], ldj = e[6];
        auto Cg = glob(static_cast<T*>(a.panels) + dpo[u]);
        for (int idx = tid; idx < mrows * ncols; idx += kThreads) {
            const int r = row0 + idx % mrows, c = col0 + idx / mrows;
            const int tr = smap[mb + r], tc = smap[mb + c];
            if (tr >= tc) {
                double acc = 0.0;
                if constexpr (LDL) {
                    for (int t = 0; t < w; ++t) acc += (double)S[r + t * kSLd] * dg[t] * (double)S[c + t * kSLd];
                } else {
                    for (int t = 0; t < w; ++t) acc += (double)S[r + t * kSLd] * (double)S[c + t * kSLd];
                }
                __hip_atomic_fetch_add(Cg + (int64_t)tc * ldj + tr, (T)(-acc), __ATOMIC_RELAXED, AGENT);
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();   // every atomic of the item has completed
    if (tid < nupd) finish_update(a, dtab[8 * tid]);
}

// ---------------------------------------------------------------- tiny blocks
// Column blocks of at most 16 columns and 64 panel rows, a wave each, up to
// kTinyGroup blocks of one dependency level per item (no block of a level
// depends on another one).  At the bottom of a 2-D problem or of a batch
// nearly all blocks are a few columns wide; as an item of a whole workgroup
// each of them cost about ten round trips to memory and four barriers for a
// few hundred flops.  Here the round trips of a claim, of the record, of the
// operands and of the counters are shared by the group, and the whole panel
// goes through the tile factorization: its rows below the block are more
// rows of the tile (l_rc = (a_rc - sum) / l_cc, stepped with the block's own
// columns), so that L comes out in one pass; rows past 32 (TALL) become
// A_off D^T, row by lane, from the inverse in LDS.  The update tiles are
// formed from LDS, row by lane (up to 32 rows: two columns at a time), and
// scattered by atomics.
// LDS per wave: rows of L (stride NC + 2), the row map, the target of every
// facing row, the tiles, the broadcast buffer, the inverse.
// 701x503, where half the time of the small blocks went into blocks of 33 to
// 64 panel rows as items of a workgroup: 2.20 -> 1.90 ms; 256 grids of side 16
// to 96: 1.60 -> 1.49.
constexpr int kTinyLds = 2112;   // doubles per wave
static_assert(kTinyRows * (kTinyW + 2) + kTinyMap / 2 + 2 * kTinyRows + 4 * kTinyTiles + 64 + kTinyW + kTinyW * kTinyW <= kTinyLds,
              "LDS of a tiny block");
static_assert(kTinyTiles <= 64 && kTinyRows <= 64, "a lane each");
static_assert((kThreads / 64) * kTinyLds <= kTiles * kTSz, "LDS of a group of tiny blocks");

// TALL: more than 32 panel rows, 8 tiles or 256 row-map entries
template <class T, int NC, bool LDL, bool TALL>
__device__ __forceinline__ void tiny_block(const SchedArgs& a, const int4 q0, const int4 q1, int tfirst, double thr, double* ws)
{
    constexpr int LS = NC + 2, NM = TALL ? kTinyMap / 64 : 4;
    const int f = uni(q0.x), w = uni(q0.y) & 255, ld = (uni(q0.y) >> 8) & 255, nupd = uni(q0.y) >> 16, mstart = uni(q0.z),
              mlen = uni(q0.w);
    T* A = static_cast<T*>(a.panels) + words64(uni(q1.x), uni(q1.y));
    T* D = static_cast<T*>(a.dinv) + words64(uni(q1.z), uni(q1.w));
    const int lane = threadIdx.x & 63, r = lane & 31;
    auto S = lds(ws);
    auto smap = reinterpret_cast<__attribute__((address_space(3))) int*>(S + kTinyRows * (kTinyW + 2));
    auto tab = smap + kTinyMap;             // facing row r: map base, stride and panel offset of its target
    auto dt = tab + 4 * kTinyRows;          // tile u: gate, first and last + 1 facing row, map base, stride, offset
    double* bc = ws + kTinyRows * (kTinyW + 2) + (kTinyMap + 4 * kTinyRows + 8 * kTinyTiles) / 2;
    auto M = lds(bc + 64 + kTinyW);         // TALL: the inverse, row by row
    const GOp gA = make_gop(A, (int64_t)ld * w, 0, 1, ld);
    T av[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) av[c] = gload<T>(gA, c < w && r < ld ? r * gA.si + c * gA.sk : kOffNone);
    T bv[TALL ? NC : 1];   // row 32 + r
    if constexpr (TALL)
#pragma unroll
        for (int c = 0; c < NC; ++c) bv[c] = gload<T>(gA, c < w && r + 32 < ld ? (r + 32) * gA.si + c * gA.sk : kOffNone);
    int mv[NM];
#pragma unroll
    for (int q = 0; q < NM; ++q) mv[q] = a.rmap[mlen > 0 ? mstart + min(lane + 64 * q, mlen - 1) : 0];
    int4 u0 = {0, 0, 0, 0}, u1 = u0, u2 = u0;
    if (lane < nupd) {
        const int4* ft = a.ftab + 3 * (int64_t)(tfirst + lane);
        u0 = ft[0];
        u1 = ft[1];
        u2 = ft[2];
    }
    TileChol<NC, LDL> tc;
#pragma unroll
    for (int c = 0; c < NC; ++c) tc.v[c] = lane >= 32 || c >= w ? (c == r ? 1.0 : 0.0) : (double)av[c];
    tc.run(bc, bc + 64, thr, w, f, a.status);
    // L and the inverse to memory; the rows of L, as stored, to LDS
    const double dr = LDL ? lds(bc)[64 + min(lane, NC - 1)] : 0.0;
    auto oA = glob(A), oD = glob(D);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (c < w) {
            if (lane < 32) {
                if (r >= c && r < ld) oA[r + c * ld] = (T)(LDL && r == c ? dr : tc.v[c]);
            } else if (r <= c) {
                oD[c + r * w] = (T)tc.v[c];
            }
        }
    }
    if (lane < 32) {
#pragma unroll
        for (int c = 0; c < NC; ++c) S[r * LS + c] = c < w ? (double)(T)tc.v[c] : 0.0;
    }
    if constexpr (TALL) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (lane >= 32 && r < NC) M[c * NC + r] = r <= c && c < w ? tc.v[c] : 0.0;
        __atomic_signal_fence(__ATOMIC_SEQ_CST);   // (LDS operations of a wave complete in order)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            double x = 0.0;
#pragma unroll
            for (int t = 0; t <= c; ++t) x += (double)bv[t] * M[c * NC + t];
            if (lane < 32) {
                if (c < w && r + 32 < ld) oA[r + 32 + c * ld] = (T)x;
                S[(r + 32) * LS + c] = (double)(T)x;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < NM; ++q) smap[lane + 64 * q] = mv[q];
    if (lane < nupd) {
        auto e = dt + 8 * lane;
        e[0] = u0.w;               // first facing row
        e[1] = u0.w + u1.x;        // and past the last
        e[2] = u1.y - mstart;
        e[3] = u1.z;
        e[4] = u2.x;
        e[5] = u2.y;
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);   // (LDS operations of a wave complete in order)
    for (int u = 0; u < nupd; ++u) {
        const int b = dt[8 * u], e = dt[8 * u + 1];
        if (lane < kTinyRows && lane >= b && lane < e) {
#pragma unroll
            for (int i = 0; i < 4; ++i) tab[4 * lane + i] = dt[8 * u + 2 + i];
        }
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    // C_j[rmap(r), rmap(c)] -= L_r . L_c (L D L^T: L_r D L_c), r >= c; up to 32
    // rows: the halves of the wave take the facing rows c alternately
    constexpr int half = TALL ? 1 : 2;
    const int ro = TALL ? lane : r;
    double own[NC];
#pragma unroll
    for (int t = 0; t < NC; ++t) {
        const double s = S[min(ro, ld - 1) * LS + t];
        own[t] = !LDL ? s : t < w ? s * lds(bc)[64 + t] : 0.0;   // (pivots past w are undefined)
    }
    if (nupd > 0)
        for (int c = w + (TALL ? 0 : lane >> 5); c < ld; c += half) {
            double acc = 0.0;
#pragma unroll
            for (int t = 0; t < NC; ++t) acc += own[t] * S[c * LS + t];
            const int mb = tab[4 * c], ldj = tab[4 * c + 1];
            auto Cg = glob(static_cast<T*>(a.panels) + words64(tab[4 * c + 2], tab[4 * c + 3]));
            if (ro >= c && ro < ld)
                __hip_atomic_fetch_add(Cg + (int64_t)smap[mb + c] * ldj + smap[mb + ro], (T)(-acc), __ATOMIC_RELAXED, AGENT);
        }
    __builtin_amdgcn_s_waitcnt(0);   // the block's atomics have completed
    if (lane < nupd) finish_update(a, u0.x);
}

template <class T, bool LDL>
__device__ __noinline__ void task_tiny(const SchedArgs& a, int first, int count, double thr, double* tiles)
{
    const int wave = uni((int)threadIdx.x >> 6);
    for (int q = wave; q < count; q += kThreads / 64) {
        const int4* t = a.tiny + 3 * (int64_t)(first + q);
        const int4 q0 = t[0], q1 = t[1];
        const int tf = uni(t[2].x);
        const int w = uni(q0.y) & 255, ld = (uni(q0.y) >> 8) & 255, nupd = uni(q0.y) >> 16;
        double* ws = tiles + wave * kTinyLds;
        if (ld > 32 || nupd > 8 || uni(q0.w) > 256) {
            if (w <= 8) tiny_block<T, 8, LDL, true>(a, q0, q1, tf, thr, ws);
            else tiny_block<T, 16, LDL, true>(a, q0, q1, tf, thr, ws);
        } else if (w <= 8) {
            tiny_block<T, 8, LDL, false>(a, q0, q1, tf, thr, ws);
        } else {
            tiny_block<T, 16, LDL, false>(a, q0, q1, tf, thr, ws);
        }
    }
}

// ---------------------------------------------------------------- scheduler
// LDL: the L D L^T factor.  LU: the L U factor (two panel arrays; no fused
// small items).
template <class T, bool LDL = false, bool LU = false>
__global__ void __launch_bounds__(kThreads, 2) sched_kernel(SchedArgs a)
{
    __shared__ double Lt[kNB * 33 + 3 * kNB + 1];   // tile, bc, small-item pivots, pivot threshold
    // the tiles of a diagonal block; as elements of T, rows of a block or
    // tile and the small-block tables, followed by one tile
    __shared__ __align__(16) double tiles[kTiles * kTSz];
    T* Pb = reinterpret_cast<T*>(tiles);
    double* Dt = tiles + (kTiles - 1) * kTSz;
    __shared__ int rpos[256], cpos[128];
    __shared__ int s_item;
    __shared__ int s_push[6];   // {hp first, hp count, hp base, normal first, normal count, normal base}
    __shared__ int s_rel;       // deterministic mode: source whose update pairs lose one dependency
    __shared__ int64_t s_t0, s_t1;
    const int tid = threadIdx.x;
    // Tickets of the two FIFO queues held by this worker and not yet served
    // (thread 0).  A ticket below the queue's total is always served: its item
    // is pushed eventually.  A high-priority ticket is taken only when the
    // next slot is already published, so that an idle worker picks up a
    // released critical item at once; a worker holding one serves whichever
    // of its two items is published first.
    // Items served by this worker are counted in a register and added to the
    // done count once, at exit.
    int my_slot = -1, hp_slot = -1, ndone = 0;
    if (tid == 0) {
        s_rel = -1;
        double thr = 0.0;   // (read after the first barrier of the loop)
        if ((LDL || LU) && a.pivot_eps > 0.0)
            thr = a.pivot_eps * __longlong_as_double(*reinterpret_cast<const long long*>(a.status + kStAmax));
        Lt[kNB * 33 + kThrSlot] = thr;
    }
    for (;;) {
        if (tid == 0) {
            int item = -1;
            s_t0 = wall_clock64();
            const int64_t t0 = s_t0;
            for (int spin = 0;; ++spin) {
                if ((spin & 15) == 0 && __hip_atomic_load(&a.status[kStAbort], __ATOMIC_RELAXED, AGENT) != 0) {
                    item = -1;
                    break;
                }
                if (hp_slot < 0) {
                    const int h = __hip_atomic_load(a.hp_head, __ATOMIC_RELAXED, AGENT);
                    if (h < a.hp_total && __hip_atomic_load(&a.hp_queue[h], __ATOMIC_RELAXED, AGENT) >= 0) {
                        const int t = __hip_atomic_fetch_add(a.hp_head, 1, __ATOMIC_RELAXED, AGENT);
                        hp_slot = t < a.hp_total ? t : -1;
                    }
                }
                if (hp_slot >= 0) {
                    item = __hip_atomic_load(&a.hp_queue[hp_slot], __ATOMIC_RELAXED, AGENT);
                    if (item >= 0) { hp_slot = -1; break; }
                }
                if (my_slot < 0) my_slot = __hip_atomic_fetch_add(a.qhead, 1, __ATOMIC_RELAXED, AGENT);
                if (my_slot < a.total_normal) {
                    item = __hip_atomic_load(&a.queue[my_slot], __ATOMIC_RELAXED, AGENT);
                    if (item >= 0) { my_slot = -1; break; }
                } else if (hp_slot < 0 && __hip_atomic_load(a.hp_head, __ATOMIC_RELAXED, AGENT) >= a.hp_total) {
                    item = -1;   // no ticket left to serve in either queue
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
                if (wall_clock64() - t0 > a.timeout_ticks) {
                    __hip_atomic_store(&a.status[kStAbort], 1, __ATOMIC_RELAXED, AGENT);
                    item = -1;
                    break;
                }
            }
            if (item < 0) __hip_atomic_fetch_add(&a.status[kStDone], ndone, __ATOMIC_RELAXED, AGENT);
            s_item = item;
            s_t1 = wall_clock64();
        }
        __syncthreads();
        const int item = s_item;
        if (item < 0) break;
        if (tid < 64) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        __syncthreads();
        const int4 d0 = a.desc[4 * (int64_t)item], d1 = a.desc[4 * (int64_t)item + 1];
        const int4 d2 = a.desc[4 * (int64_t)item + 2], d3 = a.desc[4 * (int64_t)item + 3];
        const Geo g{d0.z, d2.x, d2.y, words64(d2.z, d2.w), words64(d3.x, d3.y)};   // (not of an update)
        const int kind = d0.x & 0xff;   // (bits 8..11 of an update: pieces merged - 1; bit 12: thin item)
        const bool thin = (d0.x & kThinItem) != 0;
        if (kind == kFact) {
            __builtin_amdgcn_s_setprio(3);
            if constexpr (LU) task_fact_lu<T>(a, g, d1.z < 0, Lt, tiles);
            else task_fact<T, LDL>(a, g, d1.z < 0, Lt, tiles);
            __builtin_amdgcn_s_setprio(0);
        } else if (kind == kTrsm) {
            __builtin_amdgcn_s_setprio(2);
            if (d0.x & kSubstItem) {
                task_trsm_chain<T, LDL, LU>(a, g, d0.z, d0.w, (d0.x & kUSideItem) != 0, tiles);
            } else if constexpr (LU) {
                if (thin) {
                    task_trsm<T, 1>(a, g, d0.z, d0.w, 0, a.uinv);
                    task_trsm<T, 1>(a, g, d0.z, d0.w, a.upanel, 0);
                } else {
                    task_trsm<T>(a, g, d0.z, d0.w, 0, a.uinv);
                    task_trsm<T>(a, g, d0.z, d0.w, a.upanel, 0);
                }
            } else {
                if (thin) {
                    task_trsm<T, 1>(a, g, d0.z, d0.w);
                } else {
                    task_trsm<T>(a, g, d0.z, d0.w);
                }
            }
            __builtin_amdgcn_s_setprio(0);
        } else if (kind == kUpdate) {
            if (thin) task_update<T, LDL, LU, 1>(a, d0, d1, d2, d3, rpos, cpos);
            else task_update<T, LDL, LU>(a, d0, d1, d2, d3, rpos, cpos);
        } else if (kind == kInv) {
            __builtin_amdgcn_s_setprio(2);
            task_inv<T, LDL, LU>(a, g);
            __builtin_amdgcn_s_setprio(0);
        } else if constexpr (!LU) {
            if (kind == kTiny) task_tiny<T, LDL>(a, d0.z, d0.w, LDL ? Lt[kNB * 33 + kThrSlot] : 0.0, tiles);
            else task_small<T, LDL>(a, g, d1, Lt, Dt, Pb);
        }
        // every wave's stores and atomics have completed before the barrier
        // (FACT and TRSM items ran at raised wave priority: they are on the
        // elimination chain and share their CU with update tiles)
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid < 64 && (kind == kFact || kind == kTrsm || kind == kInv)) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        if (tid == 0) {
            int hf = 0, hc = 0, nf = 0, nc = 0;
            if (kind == kFact) {
                // the panel solves; a chain block (high priority) also its
                // INV item, in the normal queue
                if (d1.w) {
                    hf = d1.x;
                    hc = d1.y;
                    if (d1.z >= 0) { nf = d1.z; nc = 1; }
                } else {
                    nf = d1.x;
                    nc = d1.y;
                }
            } else if (kind == kTrsm) {
                if (__hip_atomic_fetch_add(&a.trsm_left[d0.y], -1, __ATOMIC_RELAXED, AGENT) == 1) {
                    if (a.npair > 0) {
                        s_rel = d0.y;   // its pairs, below
                    } else {
                        hf = d1.x;
                        hc = d1.y;
                        nf = hf + hc;
                        nc = d1.z - hc;
                    }
                }
            } else if (kind == kUpdate) {
                if (__hip_atomic_fetch_add(&a.fact_dep[d2.x], -1, __ATOMIC_RELAXED, AGENT) == 1) {
                    if (a.hp_item[d2.x]) { hf = d2.x; hc = 1; }
                    else { nf = d2.x; nc = 1; }
                }
                if (a.npair > 0) {
                    // the pair's last item releases the next pair into the
                    // same target (which then cannot have released the target)
                    const int p = a.upair[item - a.ubase];
                    if (__hip_atomic_fetch_add(&a.pleft[p], -1, __ATOMIC_RELAXED, AGENT) == 1) {
                        const int4 q = a.pairs[p];
                        if (q.z >= 0 && __hip_atomic_fetch_add(&a.pdep[q.z], -1, __ATOMIC_RELAXED, AGENT) == 1) {
                            const int4 r = a.pairs[q.z];
                            if (r.w) { hf = r.x; hc = r.y; }
                            else { nf = r.x; nc = r.y; }
                        }
                    }
                }
            }
            s_push[0] = hf;
            s_push[1] = hc;
            s_push[2] = hc > 0 ? __hip_atomic_fetch_add(a.hp_tail, hc, __ATOMIC_RELAXED, AGENT) : 0;
            s_push[3] = nf;
            s_push[4] = nc;
            s_push[5] = nc > 0 ? __hip_atomic_fetch_add(a.qtail, nc, __ATOMIC_RELAXED, AGENT) : 0;
            ++ndone;
            if (a.trace) {
                int64_t* t = a.trace + 4 * (int64_t)item;
                t[0] = s_t0;
                t[1] = s_t1;
                t[2] = wall_clock64();
                t[3] = (int64_t)__builtin_amdgcn_s_getreg((31 << 11) | 4);   // HW_ID: wave/simd/cu/se
            }
        }
        __syncthreads();
        if (s_push[1] > 0) push_items(a, true, s_push[2], s_push[0], s_push[1]);
        if (s_push[4] > 0) push_items(a, false, s_push[5], s_push[3], s_push[4]);
        if (s_rel >= 0) release_pairs(a, s_rel);   // deterministic mode
        __syncthreads();
        if (tid == 0) s_rel = -1;
    }
}

// ---------------------------------------------------------------- update microbenchmark
// The update tiles of one synthetic (source, target) pair, as a plain grid:
// block b runs tile b % ntiles ({row0, mrows, col0, ncols}) of source 0 into
// target 1 through the same task_update as the scheduler (row map base
// mbase).  Several calls of the grid, or one grid of several calls, measure
// the update kernel alone (the paper's update-kernel study).
template <class T, bool LDL>
__global__ void __launch_bounds__(kThreads, 2) update_bench_kernel(SchedArgs a, const int4* tiles, int ntiles, int mbase,
                                                                  int4 tgt, int4 src)
{
    __shared__ int rpos[256], cpos[128];
    const int4 t = tiles[blockIdx.x % ntiles];
    task_update<T, LDL, false>(a, int4{kUpdate, 0, 1, t.x}, int4{t.y, t.z, t.w, mbase}, tgt, src, rpos, cpos);
}

hipError_t launch_update_bench(const SchedArgs& a, bool f32, bool ldl, const int4* tiles, int ntiles, int mbase,
                               int4 tgt, int4 src, int copies, hipStream_t s)
{
    const int grid = ntiles * copies;
    if (f32 && ldl) update_bench_kernel<float, true><<<grid, kThreads, 0, s>>>(a, tiles, ntiles, mbase, tgt, src);
    else if (f32) update_bench_kernel<float, false><<<grid, kThreads, 0, s>>>(a, tiles, ntiles, mbase, tgt, src);
    else if (ldl) update_bench_kernel<double, true><<<grid, kThreads, 0, s>>>(a, tiles, ntiles, mbase, tgt, src);
    else update_bench_kernel<double, false><<<grid, kThreads, 0, s>>>(a, tiles, ntiles, mbase, tgt, src);
    return hipGetLastError();
}

// ---------------------------------------------------------------- set-up kernels
template <class T>
__global__ void fill_kernel(T* p, int64_t n, T v)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// panels[amap[p]] = values[p] (rounded to the panel type) for entries read
// by the factorization
template <class T>
__global__ void assemble_kernel(T* panels, const int64_t* amap, const double* values, int64_t nnz)
{
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < nnz; p += (int64_t)gridDim.x * blockDim.x) {
        const int64_t d = amap[p];
        if (d >= 0) panels[d] = (T)values[p];
    }
}

// max |values[p]| over the entries the factorization reads (amap[p] >= 0),
// into two status words as the bits of a non-negative double (ordered like
// the doubles; a NaN value counts as larger than every number)
__global__ void absmax_kernel(const int64_t* amap, const double* values, int64_t nnz, int32_t* status)
{
    unsigned long long m = 0;
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < nnz; p += (int64_t)gridDim.x * blockDim.x)
        if (amap[p] >= 0) {
            const unsigned long long b = (unsigned long long)__double_as_longlong(fabs(values[p]));
            m = b > m ? b : m;
        }
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(m, off);
        m = o > m ? o : m;
    }
    if ((threadIdx.x & 63) == 0 && m) atomicMax(reinterpret_cast<unsigned long long*>(status + kStAmax), m);
}

__global__ void zero_amax_kernel(int32_t* status)
{
    if (threadIdx.x < 2) status[kStAmax + threadIdx.x] = 0;
}

hipError_t launch_absmax(const int64_t* amap, const double* values, int64_t nnz, int32_t* status, hipStream_t s)
{
    zero_amax_kernel<<<1, 64, 0, s>>>(status);
    if (nnz > 0) {
        const int blocks = (int)std::min<int64_t>((nnz + 255) / 256, 2048);
        absmax_kernel<<<blocks, 256, 0, s>>>(amap, values, nnz, status);
    }
    return hipGetLastError();
}

// queues and counters of one factorization: the ready FACT items are the
// first entries of their queues (ready[0..nready_hp) high priority, the rest
// normal)
__global__ void sched_init(SchedArgs a, const int32_t* ready, int32_t nready, int32_t nready_hp,
                           const int32_t* fact_dep0, int32_t ncblk)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int32_t nready_n = nready - nready_hp;
    for (int64_t i = t; i < a.total_normal; i += stride) a.queue[i] = i < nready_n ? ready[nready_hp + i] : -1;
    for (int64_t i = t; i < a.hp_total; i += stride) a.hp_queue[i] = i < nready_hp ? ready[i] : -1;
    for (int64_t i = t; i < ncblk; i += stride) {
        a.fact_dep[i] = fact_dep0[i];
        a.trsm_left[i] = a.trsm_count[i];
    }
    for (int64_t i = t; i < a.npair; i += stride) {
        a.pdep[i] = a.pdep0[i];
        a.pleft[i] = a.pairs[i].y;
    }
    if (t == 0) {
        *a.qhead = 0;
        *a.qtail = nready_n;
        *a.hp_head = 0;
        *a.hp_tail = nready_hp;
        a.status[kStFail] = 0x7fffffff;
        a.status[kStAbort] = 0;
        a.status[kStDone] = 0;
        a.status[kStReplaced] = 0;
    }
}

// ---------------------------------------------------------------- host launchers
hipError_t launch_fill_f64(double* p, int64_t n, double v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
    fill_kernel<double><<<blocks, 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, int64_t n, float v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
    fill_kernel<float><<<blocks, 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}

hipError_t launch_assemble(void* panels, bool f32, const int64_t* amap, const double* values, int64_t nnz,
                           hipStream_t s)
{
    if (nnz <= 0) return hipSuccess;
    const int blocks = (int)std::min<int64_t>((nnz + 255) / 256, 8192);
    if (f32) assemble_kernel<float><<<blocks, 256, 0, s>>>(static_cast<float*>(panels), amap, values, nnz);
    else assemble_kernel<double><<<blocks, 256, 0, s>>>(static_cast<double*>(panels), amap, values, nnz);
    return hipGetLastError();
}

// FP32 panels widened to FP64 (export of the refinement-mode factor)
__global__ void widen_kernel(double* dst, const float* src, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = (double)src[i];
}

// dst[j] = panels[off[j]] widened to FP64 (the diagonal of every panel, one
// entry per column, for the log-determinant)
template <class T>
__global__ void gather_diag_kernel(double* dst, const T* panels, const int64_t* off, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = (double)panels[off[i]];
}

hipError_t launch_gather_diag(double* dst, const void* panels, bool f32, const int64_t* off, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
    if (f32) gather_diag_kernel<float><<<blocks, 256, 0, s>>>(dst, static_cast<const float*>(panels), off, n);
    else gather_diag_kernel<double><<<blocks, 256, 0, s>>>(dst, static_cast<const double*>(panels), off, n);
    return hipGetLastError();
}

hipError_t launch_widen(double* dst, const float* src, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
    widen_kernel<<<blocks, 256, 0, s>>>(dst, src, n);
    return hipGetLastError();
}

hipError_t launch_sched_init(const SchedArgs& a, const int32_t* ready, int32_t nready, int32_t nready_hp,
                             const int32_t* fact_dep0, int32_t ncblk, hipStream_t s)
{
    const int64_t n = std::max<int64_t>(std::max<int64_t>(a.total_normal, a.hp_total), std::max(ncblk, a.npair));
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096));
    sched_init<<<blocks, 256, 0, s>>>(a, ready, nready, nready_hp, fact_dep0, ncblk);
    return hipGetLastError();
}

int sched_blocks_per_cu(bool f32, bool ldlt, bool lu)
{
    int nb = 0;
    hipError_t e;
    if (lu)
        e = f32 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, sched_kernel<float, false, true>, kThreads, 0)
                : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, sched_kernel<double, false, true>, kThreads, 0);
    else if (f32 && ldlt)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, sched_kernel<float, true>, kThreads, 0);
    else if (f32)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, sched_kernel<float>, kThreads, 0);
    else if (ldlt)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, sched_kernel<double, true>, kThreads, 0);
    else
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, sched_kernel<double>, kThreads, 0);
    if (e != hipSuccess) return 1;
    return nb > 0 ? nb : 1;
}

hipError_t launch_sched(const SchedArgs& a, bool f32, bool lu, int grid, hipStream_t s)
{
    if (lu && f32) sched_kernel<float, false, true><<<grid, kThreads, 0, s>>>(a);
    else if (lu) sched_kernel<double, false, true><<<grid, kThreads, 0, s>>>(a);
    else if (f32 && a.ldlt) sched_kernel<float, true><<<grid, kThreads, 0, s>>>(a);
    else if (f32) sched_kernel<float><<<grid, kThreads, 0, s>>>(a);
    else if (a.ldlt) sched_kernel<double, true><<<grid, kThreads, 0, s>>>(a);
    else sched_kernel<double><<<grid, kThreads, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace spx
