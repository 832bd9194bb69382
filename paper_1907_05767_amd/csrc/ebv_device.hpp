/*
 * Device building blocks for the EbV LU kernels (gfx950, wave64).
 *
 * Elimination (Eq. 6-a, 6-c) is blocked in 64 x 64 tiles.  A diagonal tile is
 * factored in LDS in four 16-column strips (tile_lu64): every wave runs the 16
 * pivot steps of a strip's diagonal block in registers, the pivot row
 * broadcast within 16-lane rows by DPP, and carries a share of the U rows
 * beside it, the L columns below it and the identity along; the rank-16
 * update of the rest runs on the matrix cores.  The inverses of the tile's
 * two triangular factors follow by block recursion on the matrix cores
 * (tile_inv_off), so that every triangular solve against a diagonal tile --
 * the U blocks right of it, the L blocks below it, the blocks of a
 * substitution -- becomes a 64 x 64 product.  The rank-64 trailing update,
 * where the flops are, runs on the FP64 (or FP32) matrix cores.
 *
 * The EbV equal-work pairing (join the longest unit of work with the
 * shortest) is applied where parallel units receive unequal work: whole
 * systems of a ragged batch are taken largest-with-smallest (ebv_pairing.h).
 */
#ifndef EBV_DEVICE_HPP
#define EBV_DEVICE_HPP

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ebv_pairing.h"

namespace ebv {

constexpr int TB = 64;     /* tile edge */
constexpr int NT = 256;    /* threads per workgroup */
constexpr int LDT = TB + 1;/* LDS row pitch of a staged tile (odd: spreads banks) */

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

template <typename T> struct vec4;
template <> struct vec4<double> { typedef d4 type; };
template <> struct vec4<float> { typedef f4 type; };

/* 16x16x4 matrix-core step: D = A(16x4) * B(4x16) + C.
 * Lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]; element r of the
 * result is D[acc_row<T>(l / 16, r)][l % 16].  The two precisions place the
 * rows differently (measured on gfx950): the double form interleaves them,
 * row l/16 + 4r; the float form keeps them contiguous, row 4*(l/16) + r. */
__device__ __forceinline__ d4 mfma16(double a, double b, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma16(float a, float b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
template <typename T> __device__ __forceinline__ constexpr int acc_row(int lk, int r);
template <> __device__ __forceinline__ constexpr int acc_row<double>(int lk, int r) { return lk + 4 * r; }
template <> __device__ __forceinline__ constexpr int acc_row<float>(int lk, int r) { return 4 * lk + r; }

/* Reciprocal: hardware estimate refined by Newton steps (each squares the
 * relative error), within an ulp or two of 1/x; exact zeros give inf. */
__device__ __forceinline__ double recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = __builtin_fma(-x, r, 1.0);
    r = __builtin_fma(r, e, r);
    e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, e, r);
}
__device__ __forceinline__ float recip(float x)
{
    float r = __builtin_amdgcn_rcpf(x);
    const float e = __builtin_fmaf(-x, r, 1.0f);
    return __builtin_fmaf(r, e, r);
}

/* Index of the calling wave in its workgroup, as a wave-uniform (scalar)
 * value, so that branches on it are uniform branches. */
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

/* Wave-wide broadcast of lane `lane`'s value (lane uniform). */
__device__ __forceinline__ double bcast(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ float bcast(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

/* ---------------------------------------------- compiler controls --- */

/* Returns p unchanged, opaquely: address arithmetic based on the result
 * cannot be hoisted above this point (out of an enclosing loop), which keeps
 * the many LDS addresses of a fully unrolled tile routine from staying live
 * across the whole loop; emits no instruction. */
template <typename T> __device__ __forceinline__ T *launder(T *p)
{
    int off = 0;
    asm volatile("" : "+v"(off));
    return p + off;
}
template <typename T> __device__ __forceinline__ const T *launder(const T *p)
{
    int off = 0;
    asm volatile("" : "+v"(off));
    return p + off;
}
__device__ __forceinline__ int launder(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

/* -------------------------------------------------------- LDS layouts --- */

/* Scratch shared by the tile routines of one workgroup. */
template <typename T> struct TileSmem {
    T t0[TB * LDT];   /* diagonal tile / staged operand / operator tile */
    T t1[TB * LDT];   /* inverses of the factors / B operand / staged solved block */
    T rinv[TB];       /* reciprocals of the pivots of t0 */
    int ticket;
    int zflag;        /* zero-pivot report shared by the workgroup */
    int avail;        /* blocks known solved (multi-workgroup solves) */
};

/*
 * Element-wise pass over a 64 x 64 tile by the workgroup: thread t handles
 * column t % 64 and rows t / 64 + 4i, i = 0..15, and issues all 16 of its
 * loads before any of its stores, so that the memory latency is paid once
 * rather than once per element.  ld(r, c) returns element (r, c); st(r, c, v)
 * stores it.
 */
template <typename T, typename LD, typename ST> __device__ __forceinline__ void tile_xfer(LD &&ld, ST &&st)
{
    static_assert(NT == 4 * TB, "one column per lane, four rows per pass");
    const int c = launder((int)threadIdx.x & 63), r0 = launder((int)threadIdx.x >> 6);
    T v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
        v[i] = ld(r0 + 4 * i, c);
#pragma unroll
    for (int i = 0; i < 16; ++i)
        st(r0 + 4 * i, c, v[i]);
}

/* Store the nr x nc corner of an LDS tile (pitch LDT) to G (pitch ldg). */
template <typename T>
__device__ __forceinline__ void lds_store_tile(const T *S, T *__restrict__ G, int64_t ldg, int nr, int nc)
{
    tile_xfer<T>([&](int r, int c) { return S[r * LDT + c]; },
                 [&](int r, int c, T v) {
                     if (r < nr && c < nc)
                         G[(int64_t)r * ldg + c] = v;
                 });
}

/* ------------------------------------------------------------ staging --- */

/* Copy an nr x nc corner of the 64x64 tile at G into LDS (pitch LDT), zero
 * elsewhere; TRANS stores element (r, c) at S[c*LDT + r]. */
template <typename T, bool TRANS>
__device__ __forceinline__ void stage64(T *S, const T *__restrict__ G, int64_t ldg, int nr, int nc)
{
    tile_xfer<T>([&](int r, int c) { return (r < nr && c < nc) ? G[(int64_t)r * ldg + c] : T(0); },
                 [&](int r, int c, T v) {
                     if (TRANS)
                         S[c * LDT + r] = v;
                     else
                         S[r * LDT + c] = v;
                 });
}

/* Address map of a tile in memory: element (r, c) of an nr x nc tile. */
template <typename T> struct DenseC {
    T *C;
    int64_t ldc;
    int nr, nc;
    __device__ __forceinline__ T *operator()(int r, int c) const
    {
        return (r < nr && c < nc) ? C + (int64_t)r * ldc + c : nullptr;
    }
};

/* --------------------------------------------- blocked tile factor --- */


/* Accumulator of one 16x16 matrix-core block: element r of lane l is
 * (acc_row<T>(l / 16, r), l % 16). */
template <typename T>
__device__ __forceinline__ void acc_load(typename vec4<T>::type &acc, const T *C, int ldc)
{
    const int l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        acc[r] = C[acc_row<T>(lk, r) * ldc + lr];
}
template <typename T>
__device__ __forceinline__ void acc_store(const typename vec4<T>::type &acc, T *C, int ldc)
{
    const int l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        C[acc_row<T>(lk, r) * ldc + lr] = acc[r];
}

/* One wave: acc += A(16 x K) * B(K x 16) with fa(r, k) = A[r][k] and
 * fb(k, c) = B[k][c].  Inside each group of four, lane group lk contributes
 * k index acc_row<T>(lk, ks): the order in which an accumulator holds its
 * rows, so an accumulator can serve directly as the B operand of the next
 * product (see wave_mma16_acc). */
template <typename T, int K, typename FA, typename FB>
__device__ __forceinline__ void wave_mma16(typename vec4<T>::type &acc, FA &&fa, FB &&fb)
{
    const int l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += 16)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int k = k0 + acc_row<T>(lk, ks);
            acc = mfma16(fa(lr, k), fb(k, lr), acc);
        }
}
/* One wave: acc += A(16 x 16) * Bacc with the B operand an accumulator. */
template <typename T, typename FA>
__device__ __forceinline__ void wave_mma16_acc(typename vec4<T>::type &acc, FA &&fa,
                                               const typename vec4<T>::type &b)
{
    const int l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
        acc = mfma16(fa(lr, acc_row<T>(lk, ks)), b[ks], acc);
}

/* ------------------------------------------- 16 x 16 blocks in lanes --- */

/* The same 16 values in each of the four 16-lane rows of a wave can be
 * broadcast within the row by the data path of the instruction that uses
 * them (DPP row_newbcast), FP64 included, so an elimination step over
 * registers costs one fused multiply-add per element: no LDS round trip and
 * no readlane. */
template <int K, typename T> __device__ __forceinline__ T row_bcast(T v)
{
    return __builtin_amdgcn_update_dpp(v, v, 0x150 + K, 0xf, 0xf, true);
}

/* One elimination step over a lane's registers: with the row held by lane K
 * of each 16-lane row as the pivot row, a[j] -= f a[j](lane K) for j > K and
 * x[j] -= f x[j](lane K) for all j.  The compiler does not fold the broadcast
 * into the FP64 multiply-add, so the block is written out (a mov and a
 * multiply-add per element instead took 1.5x the issue slots).  A DPP read
 * needs two wait states after a vector write of the register, which the
 * compiler does not count across inline assembly: the s_nop covers the
 * writes before the block, and a[K + 1], the only register the next step's
 * broadcast reads, is written first, at least eight instructions before the
 * block's end. */
#define EBV_ROW_FMA(N, C, J)                                                                                           \
    ".if " C "\n\tv_fmac_" N "_dpp %" J ", %" J ", -%[f] row_newbcast:%c[k] row_mask:0xf bank_mask:0xf\n\t.endif\n\t"
#define EBV_ROW_A(N, OP)                                                                                               \
    EBV_ROW_FMA(N, "%c[k] + 1 " OP " 1", "1") EBV_ROW_FMA(N, "%c[k] + 1 " OP " 2", "2")                                \
    EBV_ROW_FMA(N, "%c[k] + 1 " OP " 3", "3") EBV_ROW_FMA(N, "%c[k] + 1 " OP " 4", "4")                                \
    EBV_ROW_FMA(N, "%c[k] + 1 " OP " 5", "5") EBV_ROW_FMA(N, "%c[k] + 1 " OP " 6", "6")                                \
    EBV_ROW_FMA(N, "%c[k] + 1 " OP " 7", "7") EBV_ROW_FMA(N, "%c[k] + 1 " OP " 8", "8")                                \
    EBV_ROW_FMA(N, "%c[k] + 1 " OP " 9", "9") EBV_ROW_FMA(N, "%c[k] + 1 " OP " 10", "10")                              \
    EBV_ROW_FMA(N, "%c[k] + 1 " OP " 11", "11") EBV_ROW_FMA(N, "%c[k] + 1 " OP " 12", "12")                            \
    EBV_ROW_FMA(N, "%c[k] + 1 " OP " 13", "13") EBV_ROW_FMA(N, "%c[k] + 1 " OP " 14", "14")                            \
    EBV_ROW_FMA(N, "%c[k] + 1 " OP " 15", "15")
#define EBV_ROW_STEP(N)                                                                                                \
    "s_nop 1\n\t" EBV_ROW_A(N, "==")                                                                                   \
    EBV_ROW_FMA(N, "1", "16") EBV_ROW_FMA(N, "1", "17") EBV_ROW_FMA(N, "1", "18") EBV_ROW_FMA(N, "1", "19")            \
    EBV_ROW_FMA(N, "1", "20") EBV_ROW_FMA(N, "1", "21") EBV_ROW_FMA(N, "1", "22") EBV_ROW_FMA(N, "1", "23")            \
    EBV_ROW_A(N, "<")
#define EBV_ROW_ARGS(a, x)                                                                                             \
    "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]), "+v"(a[8]),        \
        "+v"(a[9]), "+v"(a[10]), "+v"(a[11]), "+v"(a[12]), "+v"(a[13]), "+v"(a[14]), "+v"(a[15]), "+v"(x[0]),          \
        "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7])
template <int K> __device__ __forceinline__ void row_step(double (&a)[16], double (&x)[8], double f)
{
    asm(EBV_ROW_STEP("f64") : EBV_ROW_ARGS(a, x) : [f] "v"(f), [k] "i"(K));
}
template <int K> __device__ __forceinline__ void row_step(float (&a)[16], float (&x)[8], float f)
{
    asm(EBV_ROW_STEP("f32") : EBV_ROW_ARGS(a, x) : [f] "v"(f), [k] "i"(K));
}

/* The step over eight carried values alone (the matrix kept elsewhere). */
#define EBV_ROW_STEP8(N)                                                                                               \
    "s_nop 1\n\t" EBV_ROW_FMA(N, "1", "0") EBV_ROW_FMA(N, "1", "1") EBV_ROW_FMA(N, "1", "2") EBV_ROW_FMA(N, "1", "3")    \
    EBV_ROW_FMA(N, "1", "4") EBV_ROW_FMA(N, "1", "5") EBV_ROW_FMA(N, "1", "6") EBV_ROW_FMA(N, "1", "7")
#define EBV_ROW_ARGS8(x)                                                                                               \
    "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7])
template <int K> __device__ __forceinline__ void row_step8(double (&x)[8], double f)
{
    asm(EBV_ROW_STEP8("f64") : EBV_ROW_ARGS8(x) : [f] "v"(f), [k] "i"(K));
}
template <int K> __device__ __forceinline__ void row_step8(float (&x)[8], float f)
{
    asm(EBV_ROW_STEP8("f32") : EBV_ROW_ARGS8(x) : [f] "v"(f), [k] "i"(K));
}

constexpr int DBP = 17; /* pitch of the four diagonal blocks packed by themselves */

/* Compile-time loop: f(integral_constant<int, I>) for I = 0 .. N - 1. */
template <int I, int N, typename F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        static_for<I + 1, N>(f);
    }
}

struct NoStripHook {
    __device__ __forceinline__ void operator()(int, int) const {}
};

/*
 * Doolittle LU (Eq. 6-a, 6-c) of the 64 x 64 tile S in LDS (pitch LDT), in
 * place, in four 16-column strips.  Per strip all four waves eliminate the
 * strip's 16 x 16 diagonal block redundantly, lane i % 16 holding row i of it
 * in registers (waves 0, 2) or row i of its transpose (waves 1, 3), and carry
 * eight further columns per 16-lane row through the elimination:
 *   waves 0, 2: the U rows right of the block (L11^{-1} A12) and L11^{-1}
 *               (the identity carried along),
 *   waves 1, 3: the L columns below it, as the columns of (U11^T) X = A21^T,
 *               and U11^{-1}.
 * So a strip's L, U and both inverses of its diagonal block are ready after
 * one 16-step chain; the rank-16 update of the rest runs on the matrix cores.
 * What bounds it is the chain: per step a broadcast pivot, its reciprocal and
 * about 16 fused multiply-adds.
 *
 * P receives the inverses of the four diagonal blocks as tile_inv16 packs them
 * (L^{-1} strictly lower, U^{-1} upper): element (r, c) of block p at
 * P[(16p + r) LDT + 16p + c], or with PACKED, where nothing else goes there,
 * at P[(16p + r) DBP + c]; rinv (if not null) 1/U_kk.
 * Rows and columns past nvalid must hold the identity, which is kept.
 * Returns 0 or k+1 for the first exactly-zero pivot k < nvalid (the same in
 * every thread).  strip(p, 0) is called by every thread once strip p of S, its
 * blocks in P and rinv are final and visible, ahead of the update of the rest
 * (which does not touch them): a caller uses or publishes the strip there.
 * strip(p, 1), p < 3, follows inside the next strip's chain, where a caller
 * that published can wait for its stores without holding anybody up.
 *
 * Measured alone, one 64 x 64 tile in LDS, cycles: FP64 18.6k, FP32 15.6k,
 * inverses of the diagonal blocks included; of an FP64 strip's 4.6k the chain
 * takes 2.5k, its LDS reads and writes 1.3k and the update 0.7k (two blocks
 * each).  A form with the chain on one wave, two pivots at a time over LDS
 * broadcasts, and the inverses after it took 46k (FP32 47k).
 */
template <typename T, bool PACKED = false, typename Strip = NoStripHook>
__device__ __forceinline__ int tile_lu64(T *S, T *P, T *rinv, int nvalid, int *zflag, Strip &&strip = Strip())
{
    typedef typename vec4<T>::type V;
    constexpr int PP = PACKED ? DBP : LDT; /* pitch of P */
    S = launder(S);
    P = launder(P);
    const int t = threadIdx.x, w = wave_id(), l = launder(t & 63), i = l & 15, g = l >> 4;
    const bool lside = w & 1; /* transposed: L below the block */
    const int half = w >> 1, q = 4 * half + g; /* this lane's chunk of eight carried columns */
    const int ks = lside ? (q < 6 ? LDT : PP) : 1; /* LDS step from one carried column (row) to the next */
    if (t == 0)
        *zflag = 0;
#pragma unroll 1
    for (int p = 0; p < 4; ++p) {
        const int c0 = 16 * p;
        T *D = S + c0 * LDT + c0;
        /* chunks 0 .. 5 - 2p hold the tile's columns (rows) past the block, 6
         * and 7 the identity; of those the part its factor's triangle keeps
         * goes to P (lim of the lane's eight), the rest to the pad column */
        const int e0 = q < 6 ? 16 + 8 * q : 8 * (q - 6);
        const bool tile = q < 6 - 2 * p;
        T *E = q < 6 ? D + (lside ? e0 * LDT + i : i * LDT + e0)
                     : P + c0 * PP + (PACKED ? 0 : c0) + (lside ? e0 * PP + i : i * PP + e0);
        const int lim = q < 6 ? (tile ? 8 : 0) : i - e0 + (lside ? 1 : 0);
        T *pad = P + l * PP + (PACKED ? 16 : TB);
        T a[16], x[8], rv = T(0);
#pragma unroll
        for (int j = 0; j < 16; ++j)
            a[j] = lside ? D[j * LDT + i] : D[i * LDT + j];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const T v = *(tile ? E + j * ks : pad);
            x[j] = tile ? v : (q >= 6 && i == e0 + j ? T(1) : T(0));
        }
        static_for<0, 16>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            const T r = recip(row_bcast<k>(a[k]));
            const T m = a[k] * r;
            rv = i == k ? r : rv;
            a[k] = i > k ? m : a[k]; /* the multiplier (L) in place */
            row_step<k>(a, x, i > k ? m : T(0));
            if constexpr (k == 7)
                if (p > 0)
                    strip(p - 1, 1);
        });
        if (lside)
#pragma unroll
            for (int j = 0; j < 8; ++j)
                x[j] *= rv;
        __syncthreads(); /* every wave has read the strip */
#pragma unroll
        for (int j = 0; j < 8; ++j)
            *(j < lim ? E + j * ks : pad) = x[j];
        if (!lside && g == 0) { /* the block itself, half of its columns each; the reciprocals */
#pragma unroll
            for (int j = 0; j < 8; ++j)
                D[i * LDT + 8 * half + j] = half ? a[8 + j] : a[j];
            if (half == 0 && rinv)
                rinv[c0 + i] = rv;
        }
        __syncthreads();
        /* a zero pivot leaves no finite reciprocal */
        if (w == 0 && __any(!(__builtin_fabs((double)rv) <= 1.7976931348623157e308))) {
            const unsigned long long z = __ballot(l < 16 && c0 + i < nvalid && D[i * (LDT + 1)] == T(0));
            if (l == 0 && z && *zflag == 0)
                *zflag = c0 + __ffsll((long long)z);
        }
        strip(p, 0);
        /* rank-16 update of the rest, nb2 x nb2 blocks dealt to the waves, two
         * of a wave's at a time (their products do not depend on each other) */
        const int nb2 = 3 - p, nblk = nb2 * nb2;
        const int inv = nb2 == 3 ? 11 : (nb2 == 2 ? 16 : 32); /* b / nb2 = b inv >> 5 for b < 9 */
        for (int b = w; b < nblk; b += 8) {
            const int b1 = b + 4 < nblk ? b + 4 : b;
            const int i0 = 16 + 16 * ((b * inv) >> 5), j0 = 16 + 16 * (b - nb2 * ((b * inv) >> 5));
            const int i1 = 16 + 16 * ((b1 * inv) >> 5), j1 = 16 + 16 * (b1 - nb2 * ((b1 * inv) >> 5));
            T a0[4], a1[4], b0[4], bb[4];
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4) {
                const int k = acc_row<T>(g, k4);
                a0[k4] = -D[(i0 + i) * LDT + k];
                b0[k4] = D[k * LDT + j0 + i];
            }
            V u, v;
            acc_load<T>(u, D + i0 * LDT + j0, LDT);
            if (b1 != b) {
#pragma unroll
                for (int k4 = 0; k4 < 4; ++k4) {
                    const int k = acc_row<T>(g, k4);
                    a1[k4] = -D[(i1 + i) * LDT + k];
                    bb[k4] = D[k * LDT + j1 + i];
                }
                acc_load<T>(v, D + i1 * LDT + j1, LDT);
#pragma unroll
                for (int k4 = 0; k4 < 4; ++k4) {
                    u = mfma16(a0[k4], b0[k4], u);
                    v = mfma16(a1[k4], bb[k4], v);
                }
                acc_store<T>(v, D + i1 * LDT + j1, LDT);
            } else {
#pragma unroll
                for (int k4 = 0; k4 < 4; ++k4)
                    u = mfma16(a0[k4], b0[k4], u);
            }
            acc_store<T>(u, D + i0 * LDT + j0, LDT);
        }
        __syncthreads();
    }
    return *zflag;
}

/* The 16 x 16 diagonal blocks of the inverses of the factors of a tile that
 * is factored already (S, with 1/U_kk in rinv), packed in P (LDS, pitch LDT)
 * as tile_lu64 packs them: the 16-lane rows of a wave take one block each,
 * lane i its row (waves 0, 2: L) or its column (waves 1, 3: U transposed),
 * and carry eight columns of the identity through the substitution.  The
 * off-diagonal blocks of P are left untouched. */
template <typename T>
__device__ __forceinline__ void tile_diag_inv16(const T *S, const T *rinv, T *P)
{
    S = launder(S);
    P = launder(P);
    rinv = launder(rinv);
    const int w = wave_id(), l = launder((int)threadIdx.x & 63), i = l & 15, g = l >> 4;
    const bool lside = w & 1;
    const int e0 = 8 * (w >> 1);
    const T *D = S + 16 * g * (LDT + 1);
    const T rv = rinv[16 * g + i];
    T a[16], x[8];
#pragma unroll
    for (int j = 0; j < 16; ++j)
        a[j] = lside ? D[j * LDT + i] : D[i * LDT + j];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        x[j] = i == e0 + j ? T(1) : T(0);
    static_for<0, 16>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        const T rk = row_bcast<k>(rv);
        const T m = lside ? a[k] * rk : a[k];
        row_step8<k>(x, i > k ? m : T(0));
    });
    T *E = P + 16 * g * (LDT + 1) + (lside ? e0 * LDT + i : i * LDT + e0);
    const int lim = i - e0 + (lside ? 1 : 0), ks = lside ? LDT : 1;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (j < lim)
            E[j * ks] = lside ? x[j] * rv : x[j];
    __syncthreads();
}

/*
 * Inverses of the factors of a factored tile S from the inverses of their
 * 16 x 16 diagonal blocks: P (LDS, pitch LDT) holds those and receives L^{-1}
 * in its strict lower part (its unit diagonal implied) and U^{-1} in its
 * upper part.  The off-diagonal blocks follow one block diagonal at a time on
 * the matrix cores, from L X = I and U Y = I:
 *   X_ij = -X_ii sum_{k=j}^{i-1} L_ik X_kj   (i > j)
 *   Y_ij = -Y_ii sum_{k=i+1}^{j} U_ik Y_kj   (i < j).
 */
template <typename T> __device__ __forceinline__ void tile_inv_off(const T *S, T *P)
{
    typedef typename vec4<T>::type V;
    S = launder(S);
    P = launder(P);
    const int w = wave_id();
    /* diagonal blocks of the inverses, with the other factor's part masked
     * (loads unconditional, selects after: no divergent branches) */
    auto xdiag = [&](int bi, int r, int k) -> T {
        const T v = P[(16 * bi + r) * LDT + 16 * bi + k];
        return r > k ? v : (r == k ? T(1) : T(0));
    };
    auto ydiag = [&](int bi, int r, int k) -> T {
        const T v = P[(16 * bi + r) * LDT + 16 * bi + k];
        return r <= k ? v : T(0);
    };
#pragma unroll 1
    for (int d = 1; d < 4; ++d) {
        const int ntask = 2 * (4 - d);
        for (int task = w; task < ntask; task += 4) {
            const bool lower = task < 4 - d;
            const int a = lower ? task : task - (4 - d);
            V tacc = {0, 0, 0, 0};
            V x = {0, 0, 0, 0};
            if (lower) {
                const int i = a + d, j = a; /* T = sum_{k=j}^{i-1} L_ik X_kj */
                wave_mma16<T, 16>(
                    tacc, [&](int r, int k) { return S[(16 * i + r) * LDT + 16 * j + k]; },
                    [&](int k, int cc) { return xdiag(j, k, cc); });
                for (int kb = j + 1; kb < i; ++kb)
                    wave_mma16<T, 16>(
                        tacc, [&](int r, int k) { return S[(16 * i + r) * LDT + 16 * kb + k]; },
                        [&](int k, int cc) { return P[(16 * kb + k) * LDT + 16 * j + cc]; });
                wave_mma16_acc<T>(x, [&](int r, int k) { return -xdiag(i, r, k); }, tacc);
                acc_store<T>(x, P + 16 * i * LDT + 16 * j, LDT);
            } else {
                const int i = a, j = a + d; /* T = sum_{k=i+1}^{j} U_ik Y_kj */
                for (int kb = i + 1; kb < j; ++kb)
                    wave_mma16<T, 16>(
                        tacc, [&](int r, int k) { return S[(16 * i + r) * LDT + 16 * kb + k]; },
                        [&](int k, int cc) { return P[(16 * kb + k) * LDT + 16 * j + cc]; });
                wave_mma16<T, 16>(
                    tacc, [&](int r, int k) { return S[(16 * i + r) * LDT + 16 * j + k]; },
                    [&](int k, int cc) { return ydiag(j, k, cc); });
                wave_mma16_acc<T>(x, [&](int r, int k) { return -ydiag(i, r, k); }, tacc);
                acc_store<T>(x, P + 16 * i * LDT + 16 * j, LDT);
            }
        }
        __syncthreads();
    }
}

/* Both inverses of a tile that is factored already (see above). */
template <typename T> __device__ __forceinline__ void tile_inv16(const T *S, const T *rinv, T *P)
{
    tile_diag_inv16(S, rinv, P);
    tile_inv_off(S, P);
}

/*
 * 64 x 64 products on the matrix cores, in pieces: the workgroup's
 * accumulators (wave w holds the 32 x 32 quadrant (w / 2, w % 2) as 2 x 2
 * blocks of 16 x 16) are loaded from C, take acc (+|-)= A * B with
 * fa(r, k) = A[r][k] and fb(k, c) = B[k][c] read from LDS (inner size K),
 * and are stored.  `cref(r, c)` gives the address of C's element (r, c) or
 * nullptr outside the tile's valid part (read as zero, not written).
 */
template <typename T> struct Acc64 {
    typename vec4<T>::type v[2][2];
};
template <typename T, typename CRef> __device__ __forceinline__ void acc64_load(Acc64<T> &acc, const CRef &cref)
{
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const T *p = cref(wm + 16 * bi + acc_row<T>(lk, r), wn + 16 * bj + lr);
                acc.v[bi][bj][r] = p ? *p : T(0);
            }
}
template <typename T> __device__ __forceinline__ void acc64_zero(Acc64<T> &acc)
{
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc.v[bi][bj][r] = T(0);
}
template <typename T, typename CRef> __device__ __forceinline__ void acc64_store(const Acc64<T> &acc, const CRef &cref)
{
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                T *p = cref(wm + 16 * bi + acc_row<T>(lk, r), wn + 16 * bj + lr);
                if (p)
                    *p = acc.v[bi][bj][r];
            }
}
template <typename T, bool NEG, int K = TB, typename FA, typename FB>
__device__ __forceinline__ void acc64_mma(Acc64<T> &acc, FA &&fa, FB &&fb)
{
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
#pragma unroll 8
    for (int k = 0; k < K; k += 4) {
        T a[2], b[2];
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
            a[bi] = NEG ? -fa(wm + 16 * bi + lr, k + lk) : fa(wm + 16 * bi + lr, k + lk);
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
            b[bj] = fb(k + lk, wn + 16 * bj + lr);
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int bj = 0; bj < 2; ++bj)
                acc.v[bi][bj] = mfma16(a[bi], b[bj], acc.v[bi][bj]);
    }
}

/* C = A * B (SET) or C -= A * B for one 64 x 64 tile (see above). */
template <typename T, bool SET, int K = TB, typename CRef, typename FA, typename FB>
__device__ __forceinline__ void wg_gemm64f(const CRef &cref, FA &&fa, FB &&fb)
{
    Acc64<T> acc;
    if (SET)
        acc64_zero(acc);
    else
        acc64_load(acc, cref);
    acc64_mma<T, !SET, K>(acc, fa, fb);
    acc64_store(acc, cref);
}

/* C addressing of a full 64 x 64 LDS tile (pitch LDT). */
template <typename T> struct LdsTile {
    T *S;
    __device__ __forceinline__ T *operator()(int r, int c) const { return S + r * LDT + c; }
};

/* Operand readers for the inverse pack P (LDS, pitch LDT) of tile_inv16. */
template <typename T> struct InvL { /* L^{-1}: strict lower of P, unit diagonal */
    const T *P;
    __device__ __forceinline__ T operator()(int r, int k) const
    {
        const T v = P[r * LDT + k];
        return r > k ? v : (r == k ? T(1) : T(0));
    }
};
template <typename T> struct InvU { /* U^{-1}: upper part of P */
    const T *P;
    __device__ __forceinline__ T operator()(int k, int c) const
    {
        const T v = P[k * LDT + c];
        return k <= c ? v : T(0);
    }
};

/* U^{-1} as a left operand: element (r, k) of the upper part of P. */
template <typename T> struct InvUFull {
    const T *P;
    __device__ __forceinline__ T operator()(int r, int k) const
    {
        const T v = P[r * LDT + k];
        return r <= k ? v : T(0);
    }
};

/* Load the nr x nc corner of the 64x64 tile at G into LDS S (pitch LDT), the
 * rest the identity (the padding a partial diagonal tile is factored with). */
template <typename T>
__device__ __forceinline__ void stage_tile_identity(T *S, const T *__restrict__ G, int64_t ldg, int nr, int nc)
{
    tile_xfer<T>([&](int r, int c) { return (r < nr && c < nc) ? G[(int64_t)r * ldg + c] : (r == c ? T(1) : T(0)); },
                 [&](int r, int c, T v) { S[r * LDT + c] = v; });
}

/*
 * Product of a BM x K and a K x BN block of a matrix in memory (K a multiple
 * of 16) into the accumulators of four waves, each a 16 MB x 16 NB part of the
 * BM x BN tile: acc += A B, or with NEG acc -= A B, the rank-K update of Eq.
 * 6-c.  K runs in 16-deep chunks through double-buffered LDS: the loads of the
 * next AHEAD (1 or 2) chunks are in flight while the current one feeds the
 * matrix cores -- two where a workgroup may have its compute unit to itself
 * and a chunk's products (0.4 us) do not cover a load, one where three
 * workgroups do that for each other.
 * Both operands are read row by row in 16-byte vectors (at any alignment of
 * the leading dimension), with nothing but two pointer increments per chunk
 * between them and no branch, so that the waits count single loads.  A lies in
 * LDS by rows, pitch 16 + one vector, so that a lane reads two (four) inner
 * indices of its row at once and lane group lk supplies the indices 2 lk, 2 lk
 * + 1 (4 lk ..) of each eight (sixteen); B by rows, the pitch spreading those
 * indices' rows over the banks.
 * EDGE 1: only nr rows of A and nc columns of B exist; past them the last one
 * is read instead, and what that gives is the caller's to drop.  EDGE 2: K may
 * also be any positive number (A's elements past it count as zero).  tail() is called
 * before the last chunk's products: loads issued there are covered by them.
 * No barrier follows the last reads of `lds`.
 *
 * Measured alone on 3840 x 1280 with K = 192 (600 tiles of 128 x 64, 1200 of
 * 64 x 64): 31 TFLOP/s in FP64 with a bounds check per element, scalar LDS
 * traffic and 128-row tiles, 39 as written here, 48 with 64-row tiles and
 * three workgroups per compute unit, which leave less of the chip idle at the
 * end; in FP32, 128 x 64 on 15360 x 4096 with K = 256, 54 -> 104.
 */
template <typename T, int MB, int NB, int BK_ = 16> struct TileGemm {
    static constexpr int BM = 32 * MB, BN = 32 * NB, BK = BK_;
    static constexpr int W = 16 / sizeof(T); /* elements of a 16-byte vector */
    static constexpr int PA = BK + W, PB = BN + (sizeof(T) == 8 ? 8 : 4);
    static constexpr size_t LDS = sizeof(T) * 2 * (BM * PA + BK * PB);
};

template <typename T, int MB, int NB, bool NEG, int EDGE, int AHEAD, int BK_ = 16, typename Tail>
__device__ __forceinline__ void tile_gemm(typename vec4<T>::type (&acc)[MB][NB], const T *A, int64_t lda, int nr,
                                          const T *B, int64_t ldb, int nc, int K, char *lds, Tail &&tail)
{
    typedef TileGemm<T, MB, NB, BK_> G;
    constexpr int BM = G::BM, BN = G::BN, BK = G::BK, W = G::W, PA = G::PA, PB = G::PB;
    constexpr int EA = BM * BK / NT, EB = BK * BN / NT; /* elements per thread and chunk */
    constexpr int WB = W < EB ? W : EB;
    typedef T VW __attribute__((ext_vector_type(W)));
    typedef T VB __attribute__((ext_vector_type(WB)));
    T *sA = reinterpret_cast<T *>(lds), *sB = sA + 2 * BM * PA;
    const int t = launder((int)threadIdx.x), w = wave_id(), l = t & 63, lr = l & 15, lk = l >> 4;
    const int wm = (w >> 1) * 16 * MB, wn = (w & 1) * 16 * NB;
    /* this thread's share of a chunk: A row ar, columns ak.., B row bk, columns bc.. */
    const int ar = t / (BK / EA), ak = (t % (BK / EA)) * EA;
    const int bk = t / (BN / EB), bc = (t % (BN / EB)) * EB;
    const T *pa = A + (int64_t)(EDGE ? min(ar, nr - 1) : ar) * lda + (EDGE == 2 ? 0 : ak);
    const T *pb = B + (EDGE == 2 ? 0 : (int64_t)bk * ldb) + (EDGE ? 0 : bc);
    int ob[EB]; /* columns of B past the last one: it again */
#pragma unroll
    for (int e = 0; e < EB; ++e)
        ob[e] = EDGE ? min(bc + e, nc - 1) : e;
    const int nch = EDGE == 2 ? (K + BK - 1) / BK : K / BK;
    struct Chunk {
        T a[EA], b[EB];
    };
    int fetched = 0; /* chunks requested; past the last one it again, from the cache */
    const int64_t bstep = (int64_t)BK * ldb;
    auto fetch = [&](Chunk &x) __attribute__((always_inline)) {
        if (EDGE == 2) {
            const int kc = min(fetched, nch - 1) * BK;
            const T *row = pb + (int64_t)min(kc + bk, K - 1) * ldb;
#pragma unroll
            for (int e = 0; e < EA; ++e) {
                const T v = pa[min(kc + ak + e, K - 1)];
                x.a[e] = kc + ak + e < K ? v : T(0);
            }
#pragma unroll
            for (int e = 0; e < EB; ++e)
                x.b[e] = row[ob[e]];
            ++fetched;
            return;
        }
#pragma unroll
        for (int e = 0; e < EA; ++e)
            x.a[e] = pa[e];
#pragma unroll
        for (int e = 0; e < EB; ++e)
            x.b[e] = pb[ob[e]];
        ++fetched;
        const bool more = AHEAD == 1 || fetched < nch;
        pa += more ? BK : 0;
        pb += more ? bstep : 0;
    };
    auto park = [&](const Chunk &x, int buf) __attribute__((always_inline)) {
        T *da = sA + buf * BM * PA + ar * PA + ak, *db = sB + buf * BK * PB + bk * PB + bc;
#pragma unroll
        for (int e = 0; e < EA; e += W)
            *reinterpret_cast<VW *>(da + e) = *reinterpret_cast<const VW *>(x.a + e);
#pragma unroll
        for (int e = 0; e < EB; e += WB)
            *reinterpret_cast<VB *>(db + e) = *reinterpret_cast<const VB *>(x.b + e);
    };
    const T *ua = sA + (wm + lr) * PA + W * lk, *ub = sB + W * lk * PB + wn + lr;
    auto multiply = [&](int buf) __attribute__((always_inline)) {
        const T *xa = ua + buf * BM * PA, *xb = ub + buf * BK * PB;
#pragma unroll
        for (int h = 0; h < BK; h += 4 * W) {
            VW av[MB];
            T bv[NB][W];
#pragma unroll
            for (int bi = 0; bi < MB; ++bi)
                av[bi] = *reinterpret_cast<const VW *>(xa + 16 * bi * PA + h);
#pragma unroll
            for (int bj = 0; bj < NB; ++bj)
#pragma unroll
                for (int k = 0; k < W; ++k)
                    bv[bj][k] = xb[(h + k) * PB + 16 * bj];
#pragma unroll
            for (int k = 0; k < W; ++k)
#pragma unroll
                for (int bi = 0; bi < MB; ++bi)
#pragma unroll
                    for (int bj = 0; bj < NB; ++bj)
                        acc[bi][bj] = mfma16(NEG ? -av[bi][k] : av[bi][k], bv[bj][k], acc[bi][bj]);
        }
    };
    Chunk x[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
        fetch(x[u]);
    park(x[0], 0);
    __syncthreads();
    int c = 0;
    if (AHEAD == 1) {
#pragma unroll 1
        for (; c + 1 < nch; ++c) {
            fetch(x[0]);
            multiply(c & 1);
            park(x[0], (c & 1) ^ 1);
            __syncthreads();
        }
    } else {
        static_assert(AHEAD == 1 || AHEAD % 2 == 0, "the buffers alternate within a round");
#pragma unroll 1
        for (; c + AHEAD < nch; c += AHEAD)
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                fetch(x[u]);
                multiply(u & 1);
                park(x[(u + 1) % AHEAD], (u & 1) ^ 1);
                __syncthreads();
            }
#pragma unroll
        for (int u = 0; u + 1 < AHEAD; ++u)
            if (c + u + 1 < nch) {
                multiply(u & 1);
                park(x[u + 1], (u & 1) ^ 1);
                __syncthreads();
            }
    }
    tail();
    multiply((nch - 1) & 1);
}

/* Chunks in flight of a product whose workgroup may be alone on its compute
 * unit (FP32: measured 3 % slower with two). */
template <typename T> constexpr int kAhead = sizeof(T) == 8 ? 2 : 1;

/* A (32 MB) x (32 NB) tile's accumulators, as tile_gemm deals it to the waves:
 * f(bi, bj, r, i, j) for each element, (i, j) its place in the tile. */
template <typename T, int NB, int MB = 2, typename F> __device__ __forceinline__ void for_tile(F &&f)
{
    const int w = wave_id(), l = launder((int)threadIdx.x) & 63, lr = l & 15, lk = l >> 4;
    const int wm = (w >> 1) * 16 * MB + acc_row<T>(lk, 0), wn = (w & 1) * 16 * NB + lr;
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
        for (int bj = 0; bj < NB; ++bj)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                f(bi, bj, r, wm + 16 * bi + acc_row<T>(0, r), wn + 16 * bj);
}

/* acc -= A B for such a tile, whole or at the edge; KEDGE: K need not be a
 * multiple of 16. */
template <typename T, int NB, bool KEDGE = false>
__device__ __forceinline__ void tile_minus(typename vec4<T>::type (&acc)[2][NB], const T *A, int64_t lda, int nr,
                                           const T *B, int64_t ldb, int nc, int K, char *lds)
{
    auto none = []() {};
    if (K == 0)
        return;
    if (nr == TB && nc == 32 * NB && (!KEDGE || K % 16 == 0))
        tile_gemm<T, 2, NB, true, 0, kAhead<T>>(acc, A, lda, nr, B, ldb, nc, K, lds, none);
    else
        tile_gemm<T, 2, NB, true, KEDGE ? 2 : 1, kAhead<T>>(acc, A, lda, nr, B, ldb, nc, K, lds, none);
}

/* The tile's pending update: acc = C - A B (nr rows, nc columns of it exist;
 * the rest of the accumulators is the caller's to drop). */
template <typename T, int NB, bool KEDGE = false>
__device__ __forceinline__ void tile_pending(typename vec4<T>::type (&acc)[2][NB], const T *C, int64_t ldc, const T *A,
                                             int64_t lda, int nr, const T *B, int64_t ldb, int nc, int K, char *lds)
{
    for_tile<T, NB>([&](int bi, int bj, int r, int i, int j) {
        acc[bi][bj][r] = C[(int64_t)min(i, nr - 1) * ldc + min(j, nc - 1)];
    });
    tile_minus<T, NB, KEDGE>(acc, A, lda, nr, B, ldb, nc, K, lds);
}

template <typename T, int NB>
__device__ __forceinline__ void tile_store(const typename vec4<T>::type (&acc)[2][NB], T *C, int64_t ldc, int nr, int nc)
{
    for_tile<T, NB>([&](int bi, int bj, int r, int i, int j) {
        if (i < nr && j < nc)
            C[(int64_t)i * ldc + j] = acc[bi][bj][r];
    });
}

/* The tile to LDS (pitch LDT): the nr x nc elements that exist, the rest zero
 * or the identity. */
template <typename T, int NB>
__device__ __forceinline__ void tile_to_lds(const typename vec4<T>::type (&acc)[2][NB], T *S, int nr, int nc,
                                            bool identity)
{
    for_tile<T, NB>([&](int bi, int bj, int r, int i, int j) {
        S[i * LDT + j] = (i < nr && j < nc) ? acc[bi][bj][r] : (identity && i == j ? T(1) : T(0));
    });
}

/* Workgroups per compute unit of the kernels around wg_crout: what LDS (70 KB
 * in FP64, 46 KB in FP32) admits; FP32's third one took the mixed-precision
 * batch of 4096 systems from 6.6 to 6.4 ms (smaller ragged batches run two). */
template <typename T> constexpr int kCroutPerCu = sizeof(T) == 8 ? 2 : 3;

template <typename T> struct CroutSmem {
    static constexpr int BK = sizeof(T) == 8 ? 8 : 16; /* chunk depth: two workgroups' buffers fit a compute unit */
    static constexpr size_t PAIR = TileGemm<T, 4, 2, BK>::LDS > TileGemm<T, 2, 4, BK>::LDS
                                       ? TileGemm<T, 4, 2, BK>::LDS
                                       : TileGemm<T, 2, 4, BK>::LDS,
                            GEMM = PAIR > TileGemm<T, 2, 2>::LDS ? PAIR : TileGemm<T, 2, 2>::LDS;
    union alignas(16) {
        T t0[TB * LDT];  /* diagonal tile / updated tile */
        char gemm[GEMM]; /* operand buffers of the streamed products */
    };
    T t1[TB * LDT]; /* inverses of the diagonal tile's factors */
    int ticket;
    int zflag; /* zero-pivot report shared by the workgroup */
};

/* G = L_jj^{-1} X (LEFT) or X U_jj^{-1} for the 64 x 64 tile X in t0 and the
 * pack of inverses in t1, the nr x nc elements that exist stored.  Of the
 * triangle's four 16-wide block rows (columns) a wave takes the shortest and
 * the longest or the two between, five inner blocks either way instead of
 * eight: 40 products of 64 cycles a wave instead of 64. */
template <typename T, bool LEFT>
__device__ __forceinline__ void tri_product(T *G, int64_t ldg, int nr, int nc, const T *t0, const T *t1)
{
    typedef typename vec4<T>::type V;
    const int w = wave_id(), l = launder((int)threadIdx.x) & 63, lr = l & 15, lk = l >> 4;
    const int tri = LEFT ? w >> 1 : w & 1, oth = (LEFT ? w & 1 : w >> 1) * 32;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int tb = b == 0 ? 3 - tri : tri; /* this wave's block of the triangle */
        V x[2] = {V{0, 0, 0, 0}, V{0, 0, 0, 0}};
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q <= tb)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const int k = 16 * q + 4 * ks + lk, i = 16 * tb + lr;
                    const T p = LEFT ? t1[i * LDT + k] : t1[k * LDT + i];
                    const T f = LEFT ? (i > k ? p : (i == k ? T(1) : T(0))) : (k <= i ? p : T(0));
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const int o = oth + 16 * c + lr;
                        if (LEFT)
                            x[c] = mfma16(f, t0[k * LDT + o], x[c]);
                        else
                            x[c] = mfma16(t0[o * LDT + k], f, x[c]);
                    }
                }
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = (LEFT ? 16 * tb : oth + 16 * c) + acc_row<T>(lk, r), j = (LEFT ? oth + 16 * c : 16 * tb) + lr;
                if (i < nr && j < nc)
                    G[(int64_t)i * ldg + j] = x[c][r];
            }
    }
}

/* One piece of a Crout step: G (32 MB x 32 NB: a 64 x 64 tile, two side by side
 * or one below the other, or half of one) receives its pending updates A B, K
 * deep, and is multiplied by the diagonal tile's inverse (t1), LEFT: U or Y
 * tiles, L_jj^{-1} G, else L tiles, G U_jj^{-1}. */
template <typename T, int MB, int NB, bool LEFT>
__device__ __forceinline__ void crout_piece(T *G, int64_t ldg, int nr, int nc, const T *A, int64_t lda, const T *B,
                                            int64_t ldb, int K, CroutSmem<T> &sm)
{
    typedef typename vec4<T>::type V;
    constexpr int BK = CroutSmem<T>::BK, AHEAD = sizeof(T) == 8 ? 4 : 2;
    V acc[MB][NB];
    for_tile<T, NB, MB>([&](int bi, int bj, int r, int i, int j) {
        acc[bi][bj][r] = G[(int64_t)min(i, nr - 1) * ldg + min(j, nc - 1)];
    });
    auto none = []() {};
    if (K > 0) {
        if (nr == 32 * MB && nc == 32 * NB)
            tile_gemm<T, MB, NB, true, 0, AHEAD, BK>(acc, A, lda, nr, B, ldb, nc, K, sm.gemm, none);
        else
            tile_gemm<T, MB, NB, true, 1, AHEAD, BK>(acc, A, lda, nr, B, ldb, nc, K, sm.gemm, none);
    }
#pragma unroll
    for (int h = 0; h < (MB * NB > 4 ? 2 : 1); ++h) {
        const int i0 = MB > 2 ? TB * h : 0, j0 = NB > 2 ? TB * h : 0; /* tile h of the piece */
        __syncthreads();
        for_tile<T, NB, MB>([&](int bi, int bj, int r, int i, int j) {
            if (MB * NB <= 4 || (MB > 2 ? i >> 6 : j >> 6) == h)
                sm.t0[(i - i0) * LDT + j - j0] = (i < nr && j < nc) ? acc[bi][bj][r] : T(0);
        });
        __syncthreads();
        tri_product<T, LEFT>(G + (int64_t)i0 * ldg + j0, ldg, min(TB, nr - i0), min(NB == 1 ? 32 : TB, nc - j0), sm.t0,
                             sm.t1);
    }
    __syncthreads();
}

/*
 * Blocked Doolittle LU of one n x n system by one workgroup in Crout order
 * (Eq. 6-c's updates applied lazily): at block step j the diagonal tile and
 * the tiles of block row j and block column j receive, in one streamed
 * product each, every update of the steps before (K = 64 j), then
 *   - the diagonal tile is factored in LDS (tile_lu64, Eq. 6-a) and its
 *     factors inverted (tile_inv_off),
 *   - block row j becomes U:   U_jc = L_jj^{-1} A_jc,
 *   - block column j becomes L: L_rj = A_rj U_jj^{-1},
 * all products on the matrix cores, the streamed ones through tile_gemm with
 * two tiles that share an operand at a time (it is read once for both) and
 * four chunks in flight (two in FP32), since with two workgroups on a compute
 * unit a chunk's products do not cover a load from HBM.  Every tile is read
 * and written once for its whole update.  With right-hand sides (B != NULL, n x nrhs, pitch
 * ldb) the forward substitution L Y = B (Eq. 1) rides along as extra columns
 * of block row j: Y_j = L_jj^{-1} (B_j - L_j,0:j Y_0:j).  Returns the first
 * zero pivot (1-based) or 0; the factor overwrites A, Y overwrites B.
 *
 * Where the time goes (FP64; copies of the kernel with one part left out), 4096
 * systems of n = 16..512 | 512 of n = 1024, of 4.63 | 9.29 ms: streamed
 * products 1.6 | 6.2, products with the inverses 0.9 | 1.3, diagonal tiles 0.6
 * | 0.7, right-hand sides 0.35 | 0.45, backward substitution 0.45 | 0.35.
 * With operands streamed to registers without LDS, full 64-deep inverse
 * products and 64-wide right-hand sides the two took 5.6 | 10.9 ms.
 */
template <typename T>
__device__ __forceinline__ int wg_crout(T *__restrict__ A, int64_t lda, int n, T *__restrict__ B, int64_t ldb, int nrhs,
                                     CroutSmem<T> &sm)
{
    const int nt = (n + TB - 1) / TB;
    int zero_at = 0;
    for (int j = 0; j < nt; ++j) {
        const int k0 = j * TB, kw = min(TB, n - k0);
        const T *Lrow = A + (int64_t)k0 * lda; /* L_j,0:j (rows k0.., columns 0..k0) */
        const T *Ucol = A + k0;                /* U_0:j,j (rows 0..k0, columns k0..) */
        /* diagonal tile: all pending updates, then into LDS with the
         * identity past the system's end */
        {
            typename vec4<T>::type acc[2][2];
            T *Akk = A + (int64_t)k0 * lda + k0;
            tile_pending<T, 2>(acc, Akk, lda, Lrow, lda, kw, Ucol, lda, kw, k0, sm.gemm);
            __syncthreads();
            tile_to_lds<T, 2>(acc, sm.t0, kw, kw, true);
            __syncthreads();
            const int z = tile_lu64(sm.t0, sm.t1, (T *)nullptr, kw, &sm.zflag);
            if (z && !zero_at)
                zero_at = k0 + z;
            lds_store_tile(sm.t0, Akk, lda, kw, kw);
            if (j + 1 == nt && !B)
                break;
            tile_inv_off(sm.t0, sm.t1);
        }
        /* block row j right of the diagonal (U), two tiles at a time where two
         * remain (the left operand read once), then the right-hand sides (Y) */
        for (int c0 = k0 + TB; c0 < n;) {
            T *G = A + (int64_t)k0 * lda + c0;
            if (c0 + TB < n)
                crout_piece<T, 2, 4, true>(G, lda, kw, min(2 * TB, n - c0), Lrow, lda, A + c0, lda, k0, sm);
            else
                crout_piece<T, 2, 2, true>(G, lda, kw, n - c0, Lrow, lda, A + c0, lda, k0, sm);
            c0 += 2 * TB;
        }
        if (B)
            for (int c0 = 0; c0 < nrhs; c0 += 32)
                crout_piece<T, 2, 1, true>(B + (int64_t)k0 * ldb + c0, ldb, kw, min(32, nrhs - c0), Lrow, lda, B + c0, ldb,
                                           k0, sm);
        /* block column j below the diagonal (L), two tiles at a time where
         * two remain (the right operand read once) */
        for (int r0 = k0 + TB; r0 < n; r0 += 2 * TB) {
            T *G = A + (int64_t)r0 * lda + k0;
            if (r0 + TB < n)
                crout_piece<T, 4, 2, false>(G, lda, min(2 * TB, n - r0), kw, A + (int64_t)r0 * lda, lda, Ucol, lda, k0, sm);
            else
                crout_piece<T, 2, 2, false>(G, lda, n - r0, kw, A + (int64_t)r0 * lda, lda, Ucol, lda, k0, sm);
        }
    }
    __syncthreads();
    return zero_at;
}

/* ------------------------------------------------- triangular solves --- */

enum TriMode { TRI_L = 0, TRI_U = 1, TRI_UT = 2, TRI_LT = 3 };

/* Which triangle of the packed factor a mode reads, and whether it is read
 * transposed:  TRI_L  L (unit lower)   -> forward
 *              TRI_U  U (upper)        -> backward
 *              TRI_UT U^T (lower)      -> forward
 *              TRI_LT L^T (unit upper) -> backward */
__host__ __device__ constexpr bool tri_forward(int mode) { return mode == TRI_L || mode == TRI_UT; }
__host__ __device__ constexpr bool tri_trans(int mode) { return mode == TRI_UT || mode == TRI_LT; }
__host__ __device__ constexpr bool tri_unit(int mode) { return mode == TRI_L || mode == TRI_LT; }

/* Stages block (bi, bj) of the operator op(T) of `MODE` from the packed dense
 * factor into S (element (r, c) at S[r*LDT + c]), zero outside the matrix. */
template <typename T, int MODE> struct DenseOp {
    const T *LU;
    int64_t lda;
    int n;
    __device__ __forceinline__ void operator()(T *S, int bi, int bj) const
    {
        const int r0 = bi * TB, c0 = bj * TB;
        const int nr = min(TB, n - r0), nc = min(TB, n - c0);
        if (tri_trans(MODE)) /* op(r, c) = LU[c0 + c][r0 + r] */
            stage64<T, true>(S, LU + (int64_t)c0 * lda + r0, lda, nc, nr);
        else
            stage64<T, false>(S, LU + (int64_t)r0 * lda + c0, lda, nr, nc);
    }
    /* Row rr, columns 16q..16q+15 of operator block (bi, bj), zero outside. */
    __device__ __forceinline__ void seg(int bi, int bj, int rr, int q, T (&m)[16]) const
    {
        const int r = bi * TB + rr, c0 = bj * TB + 16 * q;
#pragma unroll
        for (int cc = 0; cc < 16; ++cc) {
            const int c = c0 + cc;
            const bool ok = r < n && c < n;
            m[cc] = ok ? (tri_trans(MODE) ? LU[(int64_t)c * lda + r] : LU[(int64_t)r * lda + c]) : T(0);
        }
    }
};


/*
 * Exchange between the workgroups of a multi-workgroup solve.  Blocks are
 * solved in a fixed order and each workgroup, after storing its block,
 * raises a shared counter `solved` to (its position + 1); a workgroup that
 * needs the block at position d waits for solved > d.  The solved values
 * are stored and loaded with device-coherent (agent-scope) atomic
 * operations, which go to the point of coherence instead of the caches of
 * one XCD, so neither side needs cache write-back or invalidation: a
 * producer that signals through a counter first waits for its own stores to
 * complete (s_waitcnt).
 */
template <typename T> __device__ __forceinline__ T load_coherent(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T> __device__ __forceinline__ void store_coherent(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

/* Bookkeeping of every bounded wait, called once per spin: true when the
 * waiter must stop waiting -- after `limit` spins (it then ORs 1 into the
 * status word) or as soon as any waiter of the call has given up (the status
 * word is re-read every 64 spins).  One lost producer therefore ends all the
 * waits of a call within a few hundred spins each instead of a full budget
 * per wait, and the launches drain. */
__device__ __forceinline__ bool wait_give_up(int *status, long spins, long limit)
{
    if (spins > limit) {
        atomicOr(status, 1);
        __threadfence();
        return true;
    }
    return (spins & 63) == 63 && load_coherent(status) != 0;
}

/* Wait until *solved > d (thread 0 polls, at most `limit` spins; the value
 * seen is kept in *avail so later positions below it need no poll); every
 * thread returns after the workgroup barrier. */
__device__ __forceinline__ void wait_solved(const int *solved, int d, int *avail, int *status, long limit)
{
    if (threadIdx.x == 0 && *avail <= d) {
        int a = *avail;
        long spins = 0;
        while ((a = __hip_atomic_load(solved, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) <= d) {
            __builtin_amdgcn_s_sleep(1);
            if (wait_give_up(status, ++spins, limit)) {
                a = d + 1;
                break;
            }
        }
        *avail = a;
    }
    __syncthreads();
}

/* Marker of a value not yet produced in an exchange buffer: a signaling
 * NaN, which no arithmetic result can be (operations return quiet NaNs), so
 * a value read as anything else is final. */
__device__ __forceinline__ bool is_unsolved_mark(double x) { return __double_as_longlong(x) == 0x7FF40000DEADBEEFll; }
__device__ __forceinline__ bool is_unsolved_mark(float x) { return __float_as_int(x) == 0x7FA0BEEF; }
constexpr unsigned long long kUnsolvedMark64 = 0x7FF40000DEADBEEFull;
constexpr unsigned int kUnsolvedMark32 = 0x7FA0BEEFu;

/*
 * Solve one 64-row block `blk` of op(T) Y = B (Eq. 1's forward or backward
 * substitution, blocked): accumulate the contributions of the blocks solved
 * before it (at most `maxdep` of them, the earliest solved first), then solve
 * with the diagonal block.  NR <= 8 columns of B are handled (nrhs_here of
 * them valid), all by the calling workgroup.  `op(S, bi, bj)` stages
 * operator blocks.
 *
 * Thread t handles row rr = t / 4; for the off-diagonal products its quarter
 * q = t % 4 covers 16 of the 64 columns and the four partial sums are joined
 * with wavefront shuffles.
 */
template <typename T, int MODE, int NR, typename Op>
__device__ void solve_block(const Op &op, int n, T *__restrict__ B, int64_t ldb, int nrhs_here, int blk,
                            int maxdep, TileSmem<T> &sm)
{
    constexpr bool FWD = tri_forward(MODE);
    const int nb = (n + TB - 1) / TB;
    const int r0 = blk * TB, nr = min(TB, n - r0);
    const int t = threadIdx.x, rr = t >> 2, q = t & 3;
    T acc[NR];
#pragma unroll
    for (int c = 0; c < NR; ++c)
        acc[c] = T(0);
    const int ndep = min(maxdep, FWD ? blk : nb - 1 - blk);
    T *Y = sm.t1;
    T mc[16], mn[16];
    /* this block's own right-hand side, loaded before any wait (no other
     * workgroup writes these rows) */
    T rhs[NR];
#pragma unroll
    for (int c = 0; c < NR; ++c)
        rhs[c] = (q == 0 && rr < nr && c < nrhs_here) ? B[(int64_t)(r0 + rr) * ldb + c] : T(0);
    if (ndep > 0)
        op.seg(blk, FWD ? blk - ndep : blk + ndep, rr, q, mc);
    for (int d = 0; d < ndep; ++d) {
        const int j = FWD ? blk - ndep + d : blk + ndep - d;
        const int jw = min(TB, n - j * TB);
        if (d + 1 < ndep)
            op.seg(blk, FWD ? j + 1 : j - 1, rr, q, mn);
        for (int idx = t; idx < TB * NR; idx += NT) {
            const int r = idx / NR, c = idx % NR;
            Y[r * NR + c] = (r < jw && c < nrhs_here) ? B[(int64_t)(j * TB + r) * ldb + c] : T(0);
        }
        __syncthreads();
#pragma unroll
        for (int cc = 0; cc < 16; ++cc) {
            const int col = 16 * q + cc;
#pragma unroll
            for (int c = 0; c < NR; ++c)
                acc[c] = __builtin_fma(mc[cc], Y[col * NR + c], acc[c]);
        }
        __syncthreads();
#pragma unroll
        for (int cc = 0; cc < 16; ++cc)
            mc[cc] = mn[cc];
    }
#pragma unroll
    for (int c = 0; c < NR; ++c) {
        acc[c] += __shfl_xor(acc[c], 1);
        acc[c] += __shfl_xor(acc[c], 2);
    }
    /* right-hand side of the diagonal block, row-major in LDS */
    if (q == 0)
#pragma unroll
        for (int c = 0; c < NR; ++c)
            Y[rr * NR + c] = rhs[c] - acc[c];
    op(sm.t0, blk, blk);
    __syncthreads();
    /* diagonal block: wave w sweeps it for the right-hand sides w, w + NW, ...,
     * lane r holding row r; the finished row's values are broadcast with
     * readlane, so no barrier is needed */
    constexpr int NW = NR < 4 ? NR : 4, CPW = NR / NW;
    const int w = wave_id();
    if (w < NW) {
        const T *M = sm.t0;
        const int r = t & 63;
        T y[CPW];
#pragma unroll
        for (int j = 0; j < CPW; ++j)
            y[j] = Y[r * NR + w + NW * j];
        const T rin = (!tri_unit(MODE) && r < nr) ? recip(M[r * LDT + r]) : T(1);
        for (int s = 0; s < nr; ++s) {
            const int m = FWD ? s : nr - 1 - s;
            const bool after = FWD ? (r > m) : (r < m);
            const T cf = after ? M[r * LDT + m] : T(0);
#pragma unroll
            for (int j = 0; j < CPW; ++j) {
                if (!tri_unit(MODE))
                    y[j] = (r == m) ? y[j] * rin : y[j];
                const T ym = bcast(y[j], m);
                y[j] = __builtin_fma(-cf, ym, y[j]);
            }
        }
        if (r < nr)
#pragma unroll
            for (int j = 0; j < CPW; ++j)
                if (w + NW * j < nrhs_here)
                    B[(int64_t)(r0 + r) * ldb + w + NW * j] = y[j];
    }
    __syncthreads();
}

/*
 * A wave's pass over rows of a row-major matrix M (pitch ld), four rows at a
 * time: items are (group g of four rows starting at row0(g), 256-column block
 * of [c0, c1)); lane l loads rows row0(g) + u, columns cb + 64 m + l (u, m <
 * 4; indices clamped to nrows - 1 and c1 - 1, so every load is valid and the
 * consumer masks) one item ahead of the item it consumes, so that a load's
 * latency overlaps the previous item instead of stalling each one.
 * consume(g, cb, v) receives an item's values, finish(g) follows a group's
 * last column block.  Nothing happens when c1 <= c0 or ngroups <= 0.
 */
template <typename T, typename RowOf, typename Consume, typename Finish>
__device__ __forceinline__ void wave_rows4_stream(const T *__restrict__ M, int64_t ld, int ngroups, RowOf &&row0,
                                                  int nrows, int c0, int c1, Consume &&consume, Finish &&finish)
{
    const int l = threadIdx.x & 63;
    const int ncb = c1 > c0 ? (c1 - c0 + 255) >> 8 : 0;
    const int total = ngroups > 0 ? ngroups * ncb : 0;
    if (total == 0)
        return;
    auto load = [&](int it, T (&v)[4][4]) {
        const int g = it / ncb, cb = c0 + ((it - g * ncb) << 8), r = row0(g);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const T *rp = M + (int64_t)min(r + u, nrows - 1) * ld;
#pragma unroll
            for (int m = 0; m < 4; ++m)
                v[u][m] = rp[min(cb + 64 * m + l, c1 - 1)];
        }
    };
    auto step = [&](int it, const T (&v)[4][4]) {
        const int g = it / ncb, cbi = it - g * ncb;
        consume(g, c0 + (cbi << 8), v);
        if (cbi == ncb - 1)
            finish(g);
    };
    T va[4][4], vb[4][4];
    load(0, va);
#pragma unroll 1
    for (int it = 0; it < total; it += 2) {
        load(min(it + 1, total - 1), vb); /* unconditional: no branch around the loads */
        step(it, va);
        if (it + 1 >= total)
            break;
        load(min(it + 2, total - 1), va);
        step(it + 1, vb);
    }
}

/*
 * Triangular solve of op(T) x = b with ONE right-hand side by one workgroup,
 * x held in LDS (xs, in place, n elements): MODE TRI_L (L unit lower,
 * forward substitution), TRI_U (U upper, backward), or their transposes
 * TRI_UT (U^T, forward) and TRI_LT (L^T, backward), Eq. 1.  Block by block
 * (64 rows of op(T)), in solve order:
 *   1. the block row's product with the part of x already solved, read
 *      straight from the factor with coalesced loads, while the 64 x 64
 *      diagonal block is fetched into registers for LDS (tri, pitch LDT):
 *      L and U by rows (a GEMV: wave w takes rows 16w .. 16w+15 of the
 *      block, four at a time, its lanes the columns, all of a group's loads
 *      issued before its sums, reduced with wavefront shuffles); U^T and L^T
 *      by the columns of T (lane l the column, wave w every fourth solved
 *      row, 16 rows' loads in flight ahead of their sums, the four waves'
 *      sums added through LDS);
 *   2. the diagonal triangle by wave 0 (lane r holds row r; each finished
 *      value is broadcast with readlane, no barrier).
 * The vector never leaves LDS.  Ends with a barrier.
 */
template <typename T, int MODE>
__device__ __forceinline__ void wg_trsv1(const T *__restrict__ LU, int64_t lda, int n, T *xs, T *tri)
{
    constexpr bool FWD = tri_forward(MODE), UNIT = tri_unit(MODE), TRANS = tri_trans(MODE);
    const int nb = (n + TB - 1) / TB;
    const int t = threadIdx.x, w = wave_id(), l = t & 63;
    for (int step = 0; step < nb; ++step) {
        const int blk = FWD ? step : nb - 1 - step;
        const int r0 = blk * TB, rw = min(TB, n - r0);
        const int c0 = FWD ? 0 : r0 + rw, c1 = FWD ? r0 : n; /* solved columns of op(T) */
        /* diagonal block: loads issued now, parked in LDS after the product */
        T dv[16];
        {
            /* unconditional loads (clamped), masked when parked */
            const int c = min(l, rw - 1);
#pragma unroll
            for (int i = 0; i < 16; ++i)
                dv[i] = LU[(int64_t)(r0 + min(w + 4 * i, rw - 1)) * lda + r0 + c];
        }
        if (!TRANS) {
            /* GEMV of the block row with the solved part, 4 rows at a time,
             * loads one item ahead */
            T sum[4] = {T(0), T(0), T(0), T(0)};
            wave_rows4_stream<T>(
                LU + (int64_t)r0 * lda, lda, 4, [&](int g) { return 16 * w + 4 * g; }, rw, c0, c1,
                [&](int, int cb, const T(&v)[4][4]) {
                    T xv[4];
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const int c = cb + 64 * m + l;
                        xv[m] = c < c1 ? xs[c] : T(0);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int m = 0; m < 4; ++m)
                            sum[u] = __builtin_fma(v[u][m], xv[m], sum[u]);
                },
                [&](int g) {
                    const int rbase = 16 * w + 4 * g;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
#pragma unroll
                        for (int o = 32; o > 0; o >>= 1)
                            sum[u] += __shfl_xor(sum[u], o);
                        if (l == 0 && rbase + u < rw)
                            xs[r0 + rbase + u] -= sum[u];
                        sum[u] = T(0);
                    }
                });
        } else if (c1 > c0) {
            /* sum over the solved rows k of T of T[k][r0 + l] x[k]: wave w
             * the rows c0 + w + 4j, RB of them per item, one item's loads in
             * flight while the previous one is summed (addresses clamped,
             * rows past c1 masked at use) */
            constexpr int RB = 16;
            const int nit = (c1 - c0 + 4 * RB - 1) / (4 * RB);
            const T *col = LU + r0 + min(l, rw - 1);
            T acc = T(0);
            auto load = [&](int it, T(&v)[RB]) {
#pragma unroll
                for (int u = 0; u < RB; ++u)
                    v[u] = col[(int64_t)min(c0 + 4 * (it * RB + u) + w, n - 1) * lda];
            };
            auto use = [&](int it, const T(&v)[RB]) {
#pragma unroll
                for (int u = 0; u < RB; ++u) {
                    const int k = c0 + 4 * (it * RB + u) + w;
                    const T a = __builtin_fma(v[u], xs[min(k, n - 1)], acc);
                    acc = k < c1 ? a : acc;
                }
            };
            T va[RB], vb[RB];
            load(0, va);
#pragma unroll 1
            for (int it = 0; it < nit; it += 2) {
                load(min(it + 1, nit - 1), vb); /* unconditional: no branch around the loads */
                use(it, va);
                if (it + 1 >= nit)
                    break;
                load(min(it + 2, nit - 1), va);
                use(it + 1, vb);
            }
            tri[w * LDT + l] = acc;
            __syncthreads();
            if (w == 0 && l < rw)
                xs[r0 + l] -= (tri[l] + tri[LDT + l]) + (tri[2 * LDT + l] + tri[3 * LDT + l]);
            __syncthreads(); /* tri is rewritten below */
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = w + 4 * i;
            const T v = (r < rw && l < rw) ? dv[i] : T(0);
            if (TRANS)
                tri[l * LDT + r] = v; /* op(T) = T^T: element (l, r) */
            else
                tri[r * LDT + l] = v;
        }
        __syncthreads();
        /* the triangle: wave 0, lane r holds row r */
        if (w == 0) {
            const int r = l;
            T y = r < rw ? xs[r0 + r] : T(0);
            const T rin = (!UNIT && r < rw) ? recip(tri[r * LDT + r]) : T(1);
            if (rw == TB) {
                /* a full block: unrolled in chunks of 16 steps, each chunk's
                 * coefficients read before its chain starts */
#pragma unroll
                for (int s0 = 0; s0 < TB; s0 += 16) {
                    T cf[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int m = FWD ? s0 + i : TB - 1 - s0 - i;
                        const T c = tri[r * LDT + m];
                        cf[i] = (FWD ? (r > m) : (r < m)) ? c : T(0);
                    }
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int m = FWD ? s0 + i : TB - 1 - s0 - i;
                        if (!UNIT)
                            y = (r == m) ? y * rin : y;
                        y = __builtin_fma(-cf[i], bcast(y, m), y);
                    }
                }
            } else {
                for (int s = 0; s < rw; ++s) {
                    const int m = FWD ? s : rw - 1 - s;
                    const bool after = FWD ? (r > m) : (r < m);
                    const T cf = after ? tri[r * LDT + m] : T(0);
                    if (!UNIT)
                        y = (r == m) ? y * rin : y;
                    const T ym = bcast(y, m);
                    y = __builtin_fma(-cf, ym, y);
                }
            }
            if (r < rw)
                xs[r0 + r] = y;
        }
        __syncthreads();
    }
}

/* Whole triangular solve of op(T) by one workgroup, block after block. */
template <typename T, int MODE, int NR>
__device__ void wg_solve(const T *LU, int64_t lda, int n, T *B, int64_t ldb, int nrhs_here, TileSmem<T> &sm)
{
    const int nb = (n + TB - 1) / TB;
    const DenseOp<T, MODE> op{LU, lda, n};
    for (int s = 0; s < nb; ++s) {
        const int blk = tri_forward(MODE) ? s : nb - 1 - s;
        solve_block<T, MODE, NR>(op, n, B, ldb, nrhs_here, blk, nb, sm);
    }
}

} /* namespace ebv */

#endif /* EBV_DEVICE_HPP */
