/*
 * HIP kernels and their launchers for libebv (gfx950).
 *
 * Dense single system (Eq. 6-a/6-c applied 64 steps at a time):
 *   k_flow    the whole factor in one launch (the default schedule): a
 *             workgroup per 64 x 64 tile, which receives its products as
 *             their operands are finished and is factored or solved at the
 *             end; k_sky_factor is the same on a skyline's tiles;
 *   k_step    one launch per 64-wide block step (very large FP32 systems, or
 *             by tuning): the diagonal tile's update and factor, the panel
 *             tiles solved against it strip by strip, and the update of the
 *             trailing region's column classes that are due, as
 *             ticket-ordered work items;
 *   k_diag, k_panel, k_update: the schedule without look-ahead (one launch
 *             per phase), kept as a tuning choice.
 * Triangular solves (Eq. 1): k_trsv, three workgroups per 64-row block (two
 *   helpers that take two thirds of the older blocks' contributions, and the
 *   block's own); workgroups take tickets in solve order, invert their
 *   diagonal block while the earlier blocks are solved, and wait for the
 *   blocks they depend on through marked exchange rows and a solved-blocks
 *   counter (no grid barrier).
 * Batches: one workgroup per system (k_lu_batch, k_solve_batch, and the
 *   persistent k_batched for ragged sizes, which takes systems from a queue
 *   in the EbV largest-with-smallest order).
 * Band, adjoint and mixed-precision helpers follow.
 */
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "ebv_device.hpp"
#include "ebv_internal.hpp"

namespace ebv {

/* ------------------------------------------------------------ utility --- */

__global__ void k_fill_i32(int *p, int64_t count, int value)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

hipError_t fill_i32(int *p, int64_t count, int value, hipStream_t st)
{
    if (count <= 0)
        return hipSuccess;
    int grid = (int)std::min<int64_t>((count + 255) / 256, 1024);
    hipLaunchKernelGGL(k_fill_i32, dim3(grid), dim3(256), 0, st, p, count, value);
    return hipGetLastError();
}

__global__ void k_fold_status(const int *status, int32_t *info)
{
    if (threadIdx.x == 0) {
        const int v = *status;
        if (v)
            *info = -v;
    }
}

hipError_t fold_status(const int *status, int32_t *info, hipStream_t st)
{
    if (!info)
        return hipSuccess;
    hipLaunchKernelGGL(k_fold_status, dim3(1), dim3(64), 0, st, status, info);
    return hipGetLastError();
}

/* ------------------------------------------------------- dense factor --- */

/* LDS of the workgroup that factors a diagonal tile: the tile, the packed
 * inverses of its factors, the pivot reciprocals. */
template <typename T> struct DiagSmem {
    T S[TB * LDT];
    T P[TB * LDT];
    T rinv[TB];
    int zflag;
    int avail;
};

/*
 * Diagonal tile of a block step: factor the 64x64 tile at (d0, d0), already
 * staged in sm.S with identity padding (tile_lu64), store it in place, and
 * store the packed inverses of its factors (tile_inv_off) to Pg (64 x 64,
 * pitch TB) for the panel solves of the next launch (for the last tile only
 * when inv_last: right-hand sides ride along).  Run by the single
 * workgroup of k_diag (the first step) and by the extra workgroup of
 * k_update (every later step).
 */
template <typename T>
__device__ __forceinline__ void diag_tile(T *__restrict__ A, int64_t lda, int n, int d0, int32_t *info,
                                          T *__restrict__ Pg, DiagSmem<T> &sm, bool inv_last)
{
    const int dw = min(TB, n - d0);
    T *Add = A + (int64_t)d0 * lda + d0;
    const int z = tile_lu64(sm.S, sm.P, sm.rinv, dw, &sm.zflag);
    lds_store_tile(sm.S, Add, lda, dw, dw);
    if (threadIdx.x == 0 && info && z && *info == 0)
        *info = d0 + z;
    if (d0 + dw >= n && !inv_last)
        return; /* last tile: no panel follows */
    tile_inv_off(sm.S, sm.P);
    tile_xfer<T>([&](int r, int c) { return sm.P[r * LDT + c]; }, [&](int r, int c, T v) { Pg[r * TB + c] = v; });
}

template <typename T>
__global__ __launch_bounds__(NT) void k_diag(T *__restrict__ A, int64_t lda, int n, int d0, int32_t *info,
                                             T *__restrict__ Pg, int inv_last)
{
    __shared__ DiagSmem<T> sm;
    const int dw = min(TB, n - d0);
    stage_tile_identity(sm.S, A + (int64_t)d0 * lda + d0, lda, dw, dw);
    __syncthreads();
    diag_tile(A, lda, n, d0, info, Pg, sm, inv_last != 0);
}

/*
 * Panel solves of one block step, as products with the inverses of the
 * diagonal tile's factors (Pg, packed by tile_inv16): a U block right of the
 * diagonal tile, U_kj = L_kk^{-1} A_kj, or an L block below it,
 * L_ik = A_ik U_kk^{-1}; one 64x64 block per workgroup, on the matrix cores.
 * With right-hand sides B (nrhs columns) the last workgroups also take the
 * forward-substitution step of Eq. 1 for block row k, Y_k = L_kk^{-1} B_k,
 * 64 columns each: B is carried as extra columns of the elimination.
 */
template <typename T>
__global__ __launch_bounds__(NT) void k_panel(T *__restrict__ A, int64_t lda, int n, int k0,
                                              const T *__restrict__ Pg, T *__restrict__ B, int64_t ldb, int nrhs)
{
    __shared__ T sP[TB * LDT], sX[TB * LDT];
    const int kw = min(TB, n - k0);
    const int nrem = (n - k0 - kw + TB - 1) / TB;
    const int t = blockIdx.x;
    tile_xfer<T>([&](int r, int c) { return Pg[r * TB + c]; }, [&](int r, int c, T v) { sP[r * LDT + c] = v; });
    if (t < nrem) {
        const int j0 = k0 + kw + t * TB, jw = min(TB, n - j0);
        T *G = A + (int64_t)k0 * lda + j0;
        stage64<T, false>(sX, G, lda, kw, jw);
        __syncthreads();
        wg_gemm64f<T, true>(DenseC<T>{G, lda, kw, jw}, InvL<T>{sP},
                            [&](int k, int c) { return sX[k * LDT + c]; });
    } else if (t < 2 * nrem) {
        const int i0 = k0 + kw + (t - nrem) * TB, iw = min(TB, n - i0);
        T *G = A + (int64_t)i0 * lda + k0;
        stage64<T, false>(sX, G, lda, iw, kw);
        __syncthreads();
        wg_gemm64f<T, true>(DenseC<T>{G, lda, iw, kw}, [&](int r, int k) { return sX[r * LDT + k]; },
                            InvU<T>{sP});
    } else {
        const int c0 = (t - 2 * nrem) * TB, cw = min(TB, nrhs - c0);
        T *G = B + (int64_t)k0 * ldb + c0;
        stage64<T, false>(sX, G, ldb, kw, cw);
        __syncthreads();
        wg_gemm64f<T, true>(DenseC<T>{G, ldb, kw, cw}, InvL<T>{sP},
                            [&](int k, int c) { return sX[k * LDT + c]; });
    }
}

/* Trailing update A22 -= L21 U12 of the tile at (r0, c0) by the kw columns
 * from k0: the product first, the tile's own elements loaded under its last
 * chunk.  The top-left skip x skip corner is not stored (it belongs to
 * another workgroup). */
template <typename T, int MB, int NB, int EDGE>
__device__ __forceinline__ void update_tile_part(T *__restrict__ A, int64_t lda, int nr, int nc, int k0, int kw, int r0,
                                                 int c0, int skip, char *lds)
{
    typedef typename vec4<T>::type V;
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const int wm = (w >> 1) * 16 * MB + acc_row<T>(lk, 0), wn = (w & 1) * 16 * NB + lr;
    T *C = A + (int64_t)r0 * lda + c0;
    auto row = [&](int bi, int r) { return wm + 16 * bi + acc_row<T>(0, r); };
    V acc[MB][NB], cv[MB][NB];
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
        for (int bj = 0; bj < NB; ++bj)
            acc[bi][bj] = V{0, 0, 0, 0};
    tile_gemm<T, MB, NB, false, EDGE, 1>(acc, A + (int64_t)r0 * lda + k0, lda, nr, A + (int64_t)k0 * lda + c0, lda, nc, kw,
                                      lds, [&]() __attribute__((always_inline)) {
#pragma unroll
                                          for (int bi = 0; bi < MB; ++bi)
#pragma unroll
                                              for (int bj = 0; bj < NB; ++bj)
#pragma unroll
                                                  for (int r = 0; r < 4; ++r) {
                                                      const int i = row(bi, r), j = wn + 16 * bj;
                                                      cv[bi][bj][r] = EDGE ? C[(int64_t)min(i, nr - 1) * lda + min(j, nc - 1)]
                                                                           : C[(int64_t)i * lda + j];
                                                  }
                                      });
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
        for (int bj = 0; bj < NB; ++bj)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = row(bi, r), j = wn + 16 * bj;
                if ((!EDGE || (i < nr && j < nc)) && !(i < skip && j < skip))
                    C[(int64_t)i * lda + j] = cv[bi][bj][r] - acc[bi][bj][r];
            }
}

template <typename T, int MB, int NB>
__device__ __forceinline__ void update_tile(T *__restrict__ A, int64_t lda, int n, int k0, int kw, int r0, int c0,
                                            int skip, char *lds)
{
    typedef TileGemm<T, MB, NB> G;
    const int nr = min(G::BM, n - r0), nc = min(G::BN, n - c0);
    if (nr == G::BM && nc == G::BN)
        update_tile_part<T, MB, NB, 0>(A, lda, nr, nc, k0, kw, r0, c0, skip, lds);
    else
        update_tile_part<T, MB, NB, 1>(A, lda, nr, nc, k0, kw, r0, c0, skip, lds);
}

/* Tile index -> position: tiles are dealt to the 8 XCDs in contiguous runs
 * (workgroups are dispatched round-robin over XCDs), so neighbouring tiles
 * share an XCD's L2. */
__device__ __forceinline__ int xcd_tile(int b, int ntiles)
{
    const int xcd = b & 7, per = ntiles >> 3, rem = ntiles & 7;
    return xcd * per + min(xcd, rem) + (b >> 3);
}

/*
 * One block step of the launch-per-phase factor: the trailing update of the
 * region right of and below the panel at k0 in tiles, plus one extra workgroup
 * that updates, factors and inverts the next diagonal tile (the tile
 * workgroup covering that corner does not store it), plus (with right-hand
 * sides) workgroups for B_i -= L_ik Y_k.
 */
template <typename T, int MB, int NB>
__global__ __launch_bounds__(NT, 2) void k_update(T *__restrict__ A, int64_t lda, int n, int k0, int kw,
                                                  int32_t *info, T *__restrict__ Pg, T *__restrict__ B,
                                                  int64_t ldb, int nrhs)
{
    typedef TileGemm<T, MB, NB> G;
    constexpr size_t GEMM_LDS = std::max(G::LDS, TileGemm<T, 2, 2>::LDS);
    __shared__ __attribute__((aligned(16))) char lds_raw[std::max(GEMM_LDS, sizeof(DiagSmem<T>))];

    const int i0 = k0 + kw, m = n - i0;
    const int tiles_n = (m + G::BN - 1) / G::BN;
    const int ntiles = ((m + G::BM - 1) / G::BM) * tiles_n;
    const int b = blockIdx.x;
    const int dw = min(TB, m); /* next diagonal tile: rows/cols i0..i0+dw */
    if (b == ntiles) {
        /* the extra workgroup: the next diagonal tile updated in registers,
         * then factored in place in LDS */
        DiagSmem<T> &sm = *reinterpret_cast<DiagSmem<T> *>(lds_raw);
        Acc64<T> acc;
        tile_pending<T, 2>(acc.v, A + (int64_t)i0 * lda + i0, lda, A + (int64_t)i0 * lda + k0, lda, dw,
                     A + (int64_t)k0 * lda + i0, lda, dw, kw, lds_raw);
        __syncthreads();
        tile_to_lds<T, 2>(acc.v, sm.S, dw, dw, true);
        __syncthreads();
        diag_tile(A, lda, n, i0, info, Pg, sm, B != nullptr);
        return;
    }
    if (b > ntiles) {
        /* right-hand-side workgroups: B_i -= L_ik Y_k for one 64-row block
         * below the panel and one 64-column chunk of B */
        const int nbc = (nrhs + TB - 1) / TB, q = b - ntiles - 1;
        const int r0 = i0 + (q / nbc) * TB, c0 = (q % nbc) * TB;
        const int nr = min(TB, n - r0), nc = min(TB, nrhs - c0);
        T *C = B + (int64_t)r0 * ldb + c0;
        Acc64<T> acc;
        tile_pending<T, 2>(acc.v, C, ldb, A + (int64_t)r0 * lda + k0, lda, nr, B + (int64_t)k0 * ldb + c0, ldb, nc, kw,
                           lds_raw);
        tile_store<T, 2>(acc.v, C, ldb, nr, nc);
        return;
    }
    const int tile = xcd_tile(b, ntiles);
    const int r0 = i0 + (tile / tiles_n) * G::BM, c0 = i0 + (tile % tiles_n) * G::BN;
    update_tile<T, MB, NB>(A, lda, n, k0, kw, r0, c0, (r0 == i0 && c0 == i0) ? dw : 0, lds_raw);
}

/* Strip q of a tile being factored (tile_lu64: S the tile, P its diagonal
 * blocks' inverses, pitch PP), sent to the workgroups that solve against it: by all
 * threads, the inverses of the diagonal block to Pg (64 x 64, pitch 64), the
 * L part below it and the U part right of it to the tile D (pitch ldd) with
 * device-coherent stores, the block itself (read by nobody else) plainly.
 * Nothing past the tile's n valid rows and columns is stored to D. */
template <int PP, typename T>
__device__ __forceinline__ void publish_strip(const T *S, const T *P, int q, T *Pg, T *D, int64_t ldd, int n)
{
    const int t = launder((int)threadIdx.x), r = t >> 4, c = t & 15, b0 = 16 * q;
    store_coherent(Pg + (b0 + r) * TB + b0 + c, P[(b0 + r) * PP + (PP == LDT ? b0 : 0) + c]);
    if (b0 + r < n && b0 + c < n)
        D[(int64_t)(b0 + r) * ldd + b0 + c] = S[(b0 + r) * LDT + b0 + c];
    for (int a = b0 + 16 + r; a < TB; a += 16) {
        if (a < n && b0 + c < n)
            store_coherent(D + (int64_t)a * ldd + b0 + c, S[a * LDT + b0 + c]);
        if (b0 + r < n && a - r + c < n)
            store_coherent(D + (int64_t)(b0 + r) * ldd + a - r + c, S[(b0 + r) * LDT + a - r + c]);
    }
}

/* Counts a published strip, one per wave, once the wave's stores have landed. */
__device__ __forceinline__ void count_strip(int *flag)
{
    __builtin_amdgcn_s_waitcnt(0);
    if ((threadIdx.x & 63) == 0)
        __hip_atomic_fetch_add(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

/*
 * One block step of the look-ahead factor: launch s factors diagonal tile s
 * (rows/columns d0 = 64 s ...) and forms panel s, while it brings the
 * region right of and below tile s up to date.  Block column J belongs to
 * class J mod G; the steps not yet applied to class c are the last pend(c)
 * steps before s (pend(c) = byte c of pendp), and each tile applies all of
 * its column's pending steps at once (K = 64 pend(c)).  The region's tiles
 * are updated for class upd only (upd >= 0) or for every class (upd < 0);
 * B rows below block row s receive step s - 1 in every launch.
 * Work items are taken in ticket order (word 0 of the step's control words
 * w = ctl + 3 + 2 s):
 *   ticket 0     the diagonal tile: its pending update, then the factor
 *                (tile_lu64); the pack the panel items solve against (the
 *                factored tile, its 16 x 16 diagonal blocks replaced by the
 *                inverses of their factors) is published a 16-column strip
 *                at a time as it is factored, each wave adding one to w[1]
 *                once its stores have landed (4 per strip), checked inside
 *                the next strip's chain so that the factorization never
 *                waits for the stores;
 *   then         the first wave of BM x 64 region tiles (first_wave of
 *                them): tiles right of and below the panel, in the updated
 *                classes, update only;
 *   then         the panel tiles of step s -- U_sj = L_ss^{-1} A_sj and
 *                L_is = A_is U_ss^{-1} -- and Y_s = L_ss^{-1} B_s: each
 *                applies its own pending update first, then runs the block
 *                substitution against the pack, step p as soon as strip p
 *                is out (w[1] >= 4 (p + 1));
 *   last         the other region tiles, and (with B) B_i -= L_{i,s-1}
 *                Y_{s-1} below block row s.
 * The panel tiles start as soon as the first wave of region tiles frees
 * slots, not behind all of them.  The item they wait for (ticket 0) is
 * running before any of them starts and waits for nothing, so the wait
 * always ends (it is also bounded, reporting into ctl[0]).  The pack and
 * the flag are exchanged with device-coherent operations (store_coherent /
 * load_coherent, wait_solved).
 */
template <typename T> struct StepSmem {
    T S[TB * LDT]; /* the diagonal or panel tile */
    T P[TB * DBP]; /* its diagonal blocks' inverses, or a strip of the pack */
};
constexpr int kStepPerCu = 3; /* workgroups per compute unit that k_step's LDS and registers admit */

template <typename T, int MB>
__global__ __launch_bounds__(NT, kStepPerCu) void k_step(T *__restrict__ A, int64_t lda, int n, int s, int G, int upd,
                                                         int pendp, int first_wave, int32_t *info, T *__restrict__ Pg,
                                                         T *__restrict__ B, int64_t ldb, int nrhs, int *ctl, long wlim)
{
    constexpr int BM = TileGemm<T, MB, 2>::BM;
    static_assert(TileGemm<T, MB, 2>::BN == TB, "one block column per update tile (one class)");
    __shared__ __attribute__((aligned(16))) char
        lds_raw[std::max(std::max(TileGemm<T, MB, 2>::LDS, TileGemm<T, 2, 2>::LDS), sizeof(StepSmem<T>))];
    static_assert(kStepPerCu * (sizeof(lds_raw) + 256) <= 160 * 1024, "workgroups per compute unit");
    __shared__ int s_ticket, s_avail, s_zero;
    StepSmem<T> &sm = *reinterpret_cast<StepSmem<T> *>(lds_raw);

    const int d0 = s * TB, dw = min(TB, n - d0);
    /* pending rank of block column J (a multiple of 64) */
    auto kw_of = [&](int J) { return TB * ((pendp >> (8 * (J % G))) & 255); };
    const int kwB = s > 0 ? TB : 0;                /* B rows: one step behind */
    const int e0 = d0 + dw, m2 = n - e0;            /* region past the diagonal tile */
    const int nr2 = (m2 + TB - 1) / TB;             /* its block columns (and rows) */
    const int J0 = s + 1;                           /* its first block column */
    const int jfirst = upd < 0 ? 0 : ((upd - J0 % G) % G + G) % G; /* first updated column, from J0 */
    const int jstep = upd < 0 ? 1 : G;
    const int ncu = upd == -2 || jfirst >= nr2 ? 0 : (nr2 - jfirst + jstep - 1) / jstep;
    const int nrt = (m2 + BM - 1) / BM;
    const int nt2 = nrt * ncu;
    const int nbc = B ? (nrhs + TB - 1) / TB : 0;
    const int nb2 = kwB > 0 ? nr2 * nbc : 0;
    const int npan = 2 * nr2 + nbc; /* panel tiles of step s */
    int *status = ctl, *wstep = ctl + kCtlHead + 2 * s, *flag = wstep + 1;

    if (threadIdx.x == 0) {
        s_ticket = atomicAdd(wstep, 1);
        s_avail = 0;
    }
    __syncthreads();
    int q = __builtin_amdgcn_readfirstlane(s_ticket);
    if (q >= 1 + nt2 + nb2 + npan) { /* counter not reset: refuse */
        if (threadIdx.x == 0)
            atomicOr(status, 2);
        return;
    }

    /* after the diagonal tile: the first wave of region tiles (first_wave of
     * them), then the panel tiles, then the other region tiles and the B
     * rows: the panel tiles start as soon as the first region tiles finish
     * instead of after all of them */
    const int n1 = min(nt2, first_wave);
    enum { U_TILE, L_TILE, RHS_TILE, RHS_ROWS, DIAGONAL } kind;
    int r0, c0, nr, nc, kw;
    T *C;
    int64_t ldc = lda;
    if (q == 0) {
        kind = DIAGONAL;
        r0 = c0 = d0;
        nr = nc = dw;
        kw = kw_of(s);
        /* the launch's longest chain: ahead of its compute unit's other waves */
        __builtin_amdgcn_s_setprio(3);
    } else if (q - 1 >= n1 && q - 1 < n1 + npan) { /* a panel tile of step s */
        const int p = q - 1 - n1;
        if (p < nr2) {
            kind = U_TILE;
            r0 = d0, c0 = e0 + p * TB;
            nr = dw, nc = min(TB, n - c0);
            kw = kw_of(J0 + p);
        } else if (p < 2 * nr2) {
            kind = L_TILE;
            r0 = e0 + (p - nr2) * TB, c0 = d0;
            nr = min(TB, n - r0), nc = dw;
            kw = kw_of(s);
        } else {
            kind = RHS_TILE;
            r0 = d0, c0 = (p - 2 * nr2) * TB;
            nr = dw, nc = min(TB, nrhs - c0);
            kw = kwB;
        }
    } else {
        q = q - 1 < n1 ? q - 1 : q - 1 - npan;
        if (q < nt2) { /* trailing tile of an updated class, update only */
            const int tile = xcd_tile(q, nt2);
            const int jc = jfirst + jstep * (tile % ncu);
            const int kwj = kw_of(J0 + jc);
            update_tile<T, MB, 2>(A, lda, n, d0 - kwj, kwj, e0 + (tile / ncu) * BM, e0 + jc * TB, 0, lds_raw);
            return;
        }
        /* B_i -= L_{i,s-1} Y_{s-1} for a 64-row block below block row s */
        q -= nt2;
        kind = RHS_ROWS;
        r0 = e0 + (q / nbc) * TB, c0 = (q % nbc) * TB;
        nr = min(TB, n - r0), nc = min(TB, nrhs - c0);
        kw = kwB;
    }
    /* the tile's own pending update: C -= L_{r0,pending} (U_{pending,c0} or
     * Y_{pending}) */
    const T *Bop = A;
    if (kind == RHS_TILE || kind == RHS_ROWS) {
        Bop = B;
        ldc = ldb;
    }
    C = const_cast<T *>(Bop) + (int64_t)r0 * ldc + c0;
    const int k0 = d0 - kw;
    Acc64<T> acc;
    tile_pending<T, 2>(acc.v, C, ldc, A + (int64_t)r0 * lda + k0, lda, nr, Bop + (int64_t)k0 * ldc + c0, ldc, nc, kw,
                       lds_raw);
    if (kind == RHS_ROWS) {
        tile_store<T, 2>(acc.v, C, ldc, nr, nc);
        return;
    }
    __syncthreads(); /* the product's last operand reads */
    tile_to_lds<T, 2>(acc.v, sm.S, nr, nc, kind == DIAGONAL);
    __syncthreads();
    if (kind == DIAGONAL) {
        const bool pub = nr2 > 0 || nbc > 0;
        /* what the panel items read, published a strip at a time as it is
         * factored (publish_strip); the waves' stores of strip q are counted
         * in the flag a little later, the last strip's at the end */
        const int z = tile_lu64<T, true>(sm.S, sm.P, (T *)nullptr, dw, &s_zero,
                                         [&](int p, int stage) __attribute__((always_inline)) {
                                             if (!pub)
                                                 return;
                                             if (stage == 0)
                                                 publish_strip<DBP>(sm.S, sm.P, p, Pg, C, lda, dw);
                                             else
                                                 count_strip(flag);
                                         });
        if (threadIdx.x == 0 && info && z && *info == 0)
            *info = d0 + z;
        if (pub)
            count_strip(flag);
        else
            lds_store_tile(sm.S, C, lda, dw, dw);
        return;
    }
    /* the solve against the factored diagonal tile, block step p as soon as
     * strip p of its pack is published (its flag counts 4 per strip): each
     * wave keeps its 16-wide slab of the tile in accumulators (transposed for
     * the L tiles, X = A U^{-1} solved as U^T X^T = A^T) and runs step p with
     * the strip staged in P, by rows of the lower operator (for the L tiles
     * U^T: its columns): the diagonal block times the inverse of the strip's
     * diagonal block, then its contribution removed from the blocks after it,
     * each product taking the finished block as its B operand */
    typedef typename vec4<T>::type V;
    const bool right = kind == L_TILE;
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const T *Add = A + (int64_t)d0 * lda + d0;
    V a[4];
#pragma unroll
    for (int q2 = 0; q2 < 4; ++q2)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            a[q2][r] = right ? sm.S[(16 * w + lr) * LDT + 16 * q2 + acc_row<T>(lk, r)]
                             : sm.S[(16 * q2 + acc_row<T>(lk, r)) * LDT + 16 * w + lr];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        wait_solved(flag, 4 * p + 3, &s_avail, status, wlim);
        /* strip p: rows 16p.. of columns 16p..16p+15 (lower), or columns
         * 16p.. of rows 16p..16p+15 (right); diagonal block from Pg, zero
         * past the matrix end */
        const int len = 64 - 16 * p;
        T v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int idx = threadIdx.x + NT * i;
            const int r = right ? 16 * p + idx / len : 16 * p + (idx >> 4);
            const int c = right ? 16 * p + idx % len : 16 * p + (idx & 15);
            v[i] = idx >= len * 16 ? T(0)
                   : (r >> 4) == (c >> 4) ? load_coherent(Pg + r * TB + c)
                   : (r < dw && c < dw)   ? load_coherent(Add + (int64_t)r * lda + c)
                                          : T(0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int idx = threadIdx.x + NT * i;
            if (idx < len * 16)
                sm.P[right ? (16 * p + idx % len) * DBP + idx / len : (16 * p + (idx >> 4)) * DBP + (idx & 15)] = v[i];
        }
        __syncthreads();
        V x = {0, 0, 0, 0};
        wave_mma16_acc<T>(
            x,
            [&](int r, int k) {
                const T u = sm.P[(16 * p + r) * DBP + k];
                return r > k ? u : (r == k ? (right ? u : T(1)) : T(0));
            },
            a[p]);
        a[p] = x;
#pragma unroll
        for (int q2 = p + 1; q2 < 4; ++q2)
            wave_mma16_acc<T>(a[q2], [&](int r, int k) { return -sm.P[(16 * q2 + r) * DBP + k]; }, a[p]);
    }
    __syncthreads();
#pragma unroll
    for (int q2 = 0; q2 < 4; ++q2)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (right)
                sm.S[(16 * w + lr) * LDT + 16 * q2 + acc_row<T>(lk, r)] = a[q2][r];
            else
                sm.S[(16 * q2 + acc_row<T>(lk, r)) * LDT + 16 * w + lr] = a[q2][r];
        }
    __syncthreads();
    lds_store_tile(sm.S, C, ldc, nr, nc);
}

/* ----------------------------------------- update-kernel measurement --- */

/* When enabled on a handle, dense_factor brackets every block-step launch
 * with a pair of events (created up front) and records the launch's
 * algorithmic flop count, so that the caller can report the kernel's live
 * average duration and achieved rate. */
int profile_update_enable(UpdateProfile &p, int max_launches)
{
    for (hipEvent_t e : p.ev)
        (void)hipEventDestroy(e);
    p.ev.clear();
    p.flops.clear();
    p.used = 0;
    if (max_launches <= 0)
        return 0;
    p.ev.resize(2 * (size_t)max_launches);
    p.flops.resize((size_t)max_launches);
    for (hipEvent_t &e : p.ev)
        if (hipEventCreate(&e) != hipSuccess)
            return 1;
    return 0;
}

int profile_update_read(UpdateProfile &p, double *ms_total, int64_t *launches, double *flops_total)
{
    double ms = 0.0, fl = 0.0;
    for (int i = 0; i < p.used; ++i) {
        if (hipEventSynchronize(p.ev[2 * i + 1]) != hipSuccess)
            return 1;
        float t = 0.f;
        if (hipEventElapsedTime(&t, p.ev[2 * i], p.ev[2 * i + 1]) != hipSuccess)
            return 1;
        ms += t;
        fl += p.flops[i];
    }
    *ms_total = ms;
    *launches = p.used;
    *flops_total = fl;
    p.used = 0;
    return 0;
}

static bool profile_slot(UpdateProfile *p, hipStream_t st, double flops, int &slot)
{
    if (!p || p->used >= (int)p->flops.size())
        return false;
    slot = p->used++;
    p->flops[slot] = flops;
    (void)hipEventRecord(p->ev[2 * slot], st);
    return true;
}

/* Rows of an update tile: 64 in FP64, where the matrix cores are busy enough
 * with them and more tiles fill the last wave of workgroups (48 against 39
 * TFLOP/s, tile_gemm); 128 in FP32 while the region is larger than
 * small_update_below, half the operand traffic per product (104 against 99
 * TFLOP/s at 15360 x 4096, K = 256). */
template <typename T> constexpr int kTallBlocks = sizeof(T) == 8 ? 2 : 4;
template <typename T> static int update_rows(const DenseTuning &tun, int m)
{
    return m > tun.small_update_below ? 32 * kTallBlocks<T> : 64;
}

/* Launch-per-phase factor: k_diag, then per block step k_panel + k_update. */
template <typename T>
static hipError_t factor_phases(T *A, int64_t lda, int n, int32_t *info, T *Pg, const DenseTuning &tun,
                                UpdateProfile *pr, hipStream_t st, T *B, int64_t ldb, int nrhs)
{
    const int nbc = B ? (nrhs + TB - 1) / TB : 0;
    hipError_t e = hipSuccess;
    hipLaunchKernelGGL(k_diag<T>, dim3(1), dim3(NT), 0, st, A, lda, n, 0, info, Pg, B ? 1 : 0);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    for (int k0 = 0; k0 < n; k0 += TB) {
        const int kw = min(TB, n - k0);
        const int nrem = (n - k0 - kw + TB - 1) / TB;
        if (nrem == 0 && !B)
            break;
        hipLaunchKernelGGL(k_panel<T>, dim3(2 * nrem + nbc), dim3(NT), 0, st, A, lda, n, k0, Pg, B, ldb, nrhs);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        if (nrem == 0)
            break;
        const int m = n - k0 - kw;
        const int nbr = (m + TB - 1) / TB;
        int pslot = -1;
        const bool prof = profile_slot(pr, st, 2.0 * (double)m * (double)m * (double)kw, pslot);
        const int bm = update_rows<T>(tun, m);
        const int nt = ((m + bm - 1) / bm) * ((m + 63) / 64);
        if (bm == 128)
            hipLaunchKernelGGL((k_update<T, kTallBlocks<T>, 2>), dim3(nt + 1 + nbr * nbc), dim3(NT), 0, st, A, lda, n,
                               k0, kw, info, Pg, B, ldb, nrhs);
        else
            hipLaunchKernelGGL((k_update<T, 2, 2>), dim3(nt + 1 + nbr * nbc), dim3(NT), 0, st, A, lda, n, k0, kw, info,
                               Pg, B, ldb, nrhs);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        if (prof)
            (void)hipEventRecord(pr->ev[2 * pslot + 1], st);
    }
    return e;
}

/* Look-ahead factor: one k_step launch per diagonal tile.  While the region
 * past the current panel is large (> tun.defer_above), the block columns are
 * split into G = tun.defer_group classes (J mod G) and launch s updates the
 * region's tiles of class (s + 1) mod G only, with K = 64 G: every tile is
 * read and written once per G steps, every launch carries about the same
 * update work beside the diagonal tile's critical path, and the class of
 * the next diagonal tile is always the one just updated (so the diagonal
 * tile and the L panel apply a single step).  Smaller regions are updated in
 * full in every launch.  applied[c] counts the steps applied to class c. */
template <typename T>
static hipError_t factor_lookahead(T *A, int64_t lda, int n, int32_t *info, T *Pg, int *ctl,
                                   const DenseTuning &tun, UpdateProfile *pr, hipStream_t st, T *B, int64_t ldb,
                                   int nrhs)
{
    const int nb = (n + TB - 1) / TB;
    const int nbc = B ? (nrhs + TB - 1) / TB : 0;
    const int G = max(1, min(4, sizeof(T) == 4 ? tun.defer_group_f32 : tun.defer_group));
    hipError_t e = hipSuccess;
    /* workgroups resident at once, less the diagonal
     * tile's: the size of the first wave of region tiles */
    int dev = 0, cus = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess ||
        (e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess)
        return e;
    const int first_wave = max(1, kStepPerCu * cus - 1);
    const long wlim = tun.wait_limit > 0 ? (long)tun.wait_limit : 1L << 24;
    int applied[4] = {0, 0, 0, 0};
    for (int s = 0; s < nb; ++s) {
        const int d0 = s * TB, e0 = min(n, d0 + TB), m2 = n - e0;
        const int nr2 = (m2 + TB - 1) / TB, J0 = s + 1;
        int pend[4], pendp = 0;
        for (int c = 0; c < 4; ++c) {
            pend[c] = c < G ? s - applied[c] : 0;
            pendp |= pend[c] << (8 * c);
        }
        /* updated classes: none in the first launch, one while split, else all */
        const int upd = s == 0 ? -2 : (G > 1 && m2 > tun.defer_above && s + 1 < nb) ? (s + 1) % G : -1;
        const int bm = update_rows<T>(tun, m2);
        const int jfirst = upd < 0 ? 0 : ((upd - J0 % G) % G + G) % G, jstep = upd < 0 ? 1 : G;
        const int ncu = upd == -2 || jfirst >= nr2 ? 0 : (nr2 - jfirst + jstep - 1) / jstep;
        const int nt2 = ((m2 + bm - 1) / bm) * ncu;
        const int nb2 = s > 0 ? nr2 * nbc : 0;
        const int grid = 1 + nt2 + nb2 + 2 * nr2 + nbc;
        /* algorithmic update flops of the launch: the diagonal tile, the
         * panel tiles and the updated region tiles, 2 rows cols K each */
        const double dw = n - d0 < TB ? n - d0 : TB;
        double fl = 2.0 * dw * dw * TB * pend[s % G];
        for (int j = 0; j < nr2; ++j) {
            const int J = J0 + j;
            const double cols = min(TB, n - (e0 + j * TB));
            const double kwj = (double)TB * pend[J % G];
            fl += 2.0 * dw * cols * kwj;                                    /* U tile (s, J) */
            fl += 2.0 * cols * dw * TB * pend[s % G];                       /* L tile (J, s) */
            if (upd == -1 || (upd >= 0 && J % G == upd))
                fl += 2.0 * m2 * cols * kwj;                                /* region column J */
        }
        int pslot = -1;
        const bool prof = s > 0 && profile_slot(pr, st, fl, pslot);
        if (bm == 128)
            hipLaunchKernelGGL((k_step<T, kTallBlocks<T>>), dim3(grid), dim3(NT), 0, st, A, lda, n, s, G, upd, pendp,
                               first_wave, info, Pg, B, ldb, nrhs, ctl, wlim);
        else
            hipLaunchKernelGGL((k_step<T, 2>), dim3(grid), dim3(NT), 0, st, A, lda, n, s, G, upd, pendp, first_wave,
                               info, Pg, B, ldb, nrhs, ctl, wlim);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        if (prof)
            (void)hipEventRecord(pr->ev[2 * pslot + 1], st);
        if (upd == -1)
            for (int c = 0; c < G; ++c)
                applied[c] = s;
        else if (upd >= 0)
            applied[upd] = s;
    }
    return e;
}

/* ------------------------------------------------- factor as a dataflow --- */

/*
 * Blocked LU with the tiles as the units, one workgroup each, that wait for
 * the tiles they need instead of for a launch: tile (I, K) keeps its elements
 * in accumulators while it receives the products L_Ik U_kK (Eq. 6-c), k
 * ascending, as their operands appear, and then
 *   - K = I: is factored (tile_lu64, Eq. 6-a) and published a strip at a time;
 *   - K < I (I < K): is solved against the diagonal tile of block K (I), step p
 *     as soon as strip p is out.
 * The chain of the elimination is diagonal tile -> the two tiles below and
 * right of it -> next diagonal tile.  Those two are published 16 columns (rows)
 * at a time, as they are solved, and the next diagonal tile subtracts each
 * rank-16 product when it appears, its operands read straight to registers:
 * after the last strip one such product is left.
 *
 * Workgroups take their tiles from a ticket in the order of steps J: the
 * diagonal tile, then the tiles (I, J) below, then (J, K) right of it.  A tile
 * needs only tiles with smaller tickets, which run or have run, so that every
 * wait ends (they are bounded all the same, into the status word).
 *
 * What bounds it is the chain, 16 us a block: 9 us for the diagonal tile (FP32
 * 8), 2 us on each of the two hops until a flag is seen, 1 us until what it
 * announces is loaded, and the last products; from n = 8192 (dense) the update
 * work, 50 TFLOP/s of the 72 that a large FP64 product reaches.  Against one
 * launch per block step: dense FP64 n = 4096 2031 -> 1207 us (use_flow has
 * more); skyline, n = 16384 with half-widths up to 1024, 5.6 -> 4.07 ms; full
 * profile of n = 16384, 161 -> 68 ms.  Tried and slower: the diagonal's
 * workgroup solving both neighbours itself (25.6 us a block, its coherent stores
 * hold up every later wait), strips handed over one at a time.
 *
 * F describes the matrix: tile(I, K), pitch ld(K), rows(I) of block I that
 * exist, first(I, K) the first k with a product; the flags lflag(I), uflag(K)
 * count 16 per finished tile of block row I's L part (block column K's U part),
 * 4 per strip, which finish in order, lcount(I, J), ucount(K, J) being the
 * tiles before (I, J), (J, K).  dflag(J) counts 4 per published strip of the
 * diagonal tile, pack(J) holds the inverses of its diagonal blocks (64 x 16),
 * and guard(J), called by the publishing waves, returns when pack(J) is free.
 * Finished tiles are written through (store_coherent) and read coherently or
 * after an acquire; a waiting workgroup polls with one thread.
 */
template <typename T> struct FlowSmem {
    union alignas(16) {
        StepSmem<T> tile;
        char gemm[TileGemm<T, 2, 2>::LDS];
    };
    int seen[3]; /* flag values seen: L, U, strips */
    int ticket, zero;
};

/* The publishing waves of a diagonal tile's workgroup: two more than the four
 * that factor the tile, so that neither the stores nor the wait for them lie
 * on the chain of its strips (they took 2 of the 11 us of a tile).  Called by
 * those waves while the others are in tile_lu64, whose barriers they share,
 * three a strip: strip read, strip final, rest updated.  S, P: the tile and its
 * diagonal blocks' inverses (pitch DBP); they go to D (n x n of it exist) and to
 * the pack Pg; flag counts 4 per strip. */
constexpr int kPubWaves = 2, NTP = NT + 64 * kPubWaves;
constexpr int kFlowWaves = 3; /* waves per SIMD: two workgroups per compute unit */
template <typename T>
__device__ __forceinline__ void publish_strips(const T *S, const T *P, T *Pg, T *D, int64_t ldd, int n, int *flag)
{
    constexpr int R = 4 * kPubWaves; /* rows of 16 lanes */
    const int t = (int)threadIdx.x - NT, r0 = t >> 4, c = t & 15;
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
        const int b0 = 16 * q;
        __syncthreads();
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16 / R; ++i) {
            const int r = r0 + R * i;
            store_coherent(Pg + (b0 + r) * 16 + c, P[(b0 + r) * DBP + c]);
            if (b0 + r < n && b0 + c < n)
                store_coherent(D + (int64_t)(b0 + r) * ldd + b0 + c, S[(b0 + r) * LDT + b0 + c]);
#pragma unroll 3
            for (int a = b0 + 16; a < TB; a += 16) {
                if (a + r < n && b0 + c < n)
                    store_coherent(D + (int64_t)(a + r) * ldd + b0 + c, S[(a + r) * LDT + b0 + c]);
                if (b0 + r < n && a + c < n)
                    store_coherent(D + (int64_t)(b0 + r) * ldd + a + c, S[(b0 + r) * LDT + a + c]);
            }
        }
        __syncthreads();
        __builtin_amdgcn_s_waitcnt(0);
        if ((t & 63) == 0)
            __hip_atomic_fetch_add(flag, 4 / kPubWaves, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

/* Returns (all threads) once *pa >= na and *pb >= nb (pb may be null); off the
 * chain a workgroup polls less often. */
__device__ __forceinline__ void flow_wait(const int *pa, int na, int *sa, const int *pb, int nb, int *sb, int *status,
                                          long limit, bool chain)
{
    if (threadIdx.x == 0 && (*sa < na || (pb && *sb < nb))) {
        long spins = 0;
        int va = *sa, vb = pb ? *sb : nb;
        for (;;) {
            if (va < na)
                va = load_coherent(pa);
            if (vb < nb)
                vb = load_coherent(pb);
            if (va >= na && vb >= nb)
                break;
            if (chain)
                __builtin_amdgcn_s_sleep(1);
            else
                __builtin_amdgcn_s_sleep(16);
            if (wait_give_up(status, ++spins, limit)) {
                va = max(va, na);
                vb = max(vb, nb);
                break;
            }
        }
        *sa = va;
        if (pb)
            *sb = vb;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
}

/* Adds c per wave to a flag, once the wave's stores have landed. */
__device__ __forceinline__ void flow_count(int *flag, int c)
{
    __builtin_amdgcn_s_waitcnt(0);
    if ((threadIdx.x & 63) == 0)
        __hip_atomic_fetch_add(flag, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

/* End of the run of products from k on whose operands have been seen: more
 * than one where the tiles of a row lie side by side (F::joined; no flag counts
 * less than 16 per tile then). */
template <typename T, typename F> __device__ __forceinline__ int flow_run(int k, int k1, const FlowSmem<T> &sm)
{
    return F::joined ? min(k1, __builtin_amdgcn_readfirstlane(min(sm.seen[0], sm.seen[1])) / 16) : k + 1;
}

/* acc = C - sum of the products of tile (I, K), k < k1. */
template <typename T, typename F>
__device__ __forceinline__ void flow_products(typename vec4<T>::type (&acc)[2][2], const F &f, int I, int K, int k1,
                                              bool chain, FlowSmem<T> &sm)
{
    const int nr = f.rows(I), nc = f.rows(K);
    const T *C = f.tile(I, K);
    for_tile<T, 2>([&](int bi, int bj, int r, int i, int j) {
        acc[bi][bj][r] = C[(int64_t)min(i, nr - 1) * f.ld(K) + min(j, nc - 1)];
    });
    for (int k = f.first(I, K); k < k1;) {
        flow_wait(f.lflag(I), 16 * (f.lcount(I, k) + 1), sm.seen, f.uflag(K), 16 * (f.ucount(K, k) + 1), sm.seen + 1,
                  f.status(), f.limit, chain);
        const int kn = flow_run<T, F>(k, k1, sm);
        tile_minus<T, 2>(acc, f.tile(I, k), f.ld(k), nr, f.tile(k, K), f.ld(K), nc, TB * (kn - k), sm.gemm);
        k = kn;
    }
    __syncthreads(); /* the products' last operand reads */
}

/* Strip p of the factored diagonal tile D to LDS, by rows of the lower
 * operator, pitch DBP: rows 16p.. of columns 16p..16p+15 (L), or RIGHT the
 * columns 16p.. of rows 16p..16p+15 (U^T); its diagonal block from the pack,
 * zero past its n rows and columns. */
template <typename T, bool RIGHT>
__device__ __forceinline__ void flow_strip(T *dst, int p, const T *Pg, const T *D, int64_t ld, int n)
{
    const int len = TB - 16 * p;
    T v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int idx = threadIdx.x + NT * i;
        const int r = RIGHT ? 16 * p + idx / len : 16 * p + (idx >> 4);
        const int c = RIGHT ? 16 * p + idx % len : 16 * p + (idx & 15);
        v[i] = idx >= len * 16          ? T(0)
               : (r >> 4) == (c >> 4)   ? load_coherent(Pg + r * 16 + (c & 15))
               : (r < n && c < n)       ? load_coherent(D + (int64_t)r * ld + c)
                                        : T(0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int idx = threadIdx.x + NT * i;
        if (idx < len * 16)
            dst[RIGHT ? (16 * p + idx % len) * DBP + idx / len : (16 * p + (idx >> 4)) * DBP + (idx & 15)] = v[i];
    }
}

/* Block step p of a wave's 16-wide slab (transposed for an L tile, X = A
 * U^{-1} solved as U^T X^T = A^T) against a staged strip. */
template <typename T, bool RIGHT>
__device__ __forceinline__ void flow_solve(typename vec4<T>::type (&a)[4], const T *strip, int p)
{
    typename vec4<T>::type x = {0, 0, 0, 0};
    wave_mma16_acc<T>(
        x,
        [&](int r, int k) {
            const T u = strip[(16 * p + r) * DBP + k];
            return r > k ? u : (r == k ? (RIGHT ? u : T(1)) : T(0));
        },
        a[p]);
    a[p] = x;
#pragma unroll
    for (int q = p + 1; q < 4; ++q)
        wave_mma16_acc<T>(a[q], [&](int r, int k) { return -strip[(16 * q + r) * DBP + k]; }, a[p]);
}

/* Tile (I, J) below (RIGHT) or (J, I) right of the diagonal tile J. */
template <typename T, bool RIGHT, typename F>
__device__ __forceinline__ void flow_panel(const F &f, int J, int I, FlowSmem<T> &sm)
{
    typedef typename vec4<T>::type V;
    const int r0 = RIGHT ? I : J, c0 = RIGHT ? J : I, nr = f.rows(r0), nc = f.rows(c0);
    T *S = sm.tile.S, *G = f.tile(r0, c0);
    const bool next = f.next(J, I); /* the next diagonal tile waits for it */
    const bool chain = I <= J + 2;  /* or the next but one */
    V acc[2][2];
    flow_products<T>(acc, f, r0, c0, J, chain, sm);
    tile_to_lds<T, 2>(acc, S, nr, nc, false);
    __syncthreads();
    int *flag = RIGHT ? f.lflag(I) : f.uflag(I), *seen = sm.seen + (RIGHT ? 0 : 1);
    const int before = 16 * (RIGHT ? f.lcount(I, J) : f.ucount(I, J)); /* a row's (column's) tiles count in order */
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const bool ok = 16 * w + lr < (RIGHT ? nr : nc);
    V a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            a[q][r] = RIGHT ? S[(16 * w + lr) * LDT + 16 * q + acc_row<T>(lk, r)]
                            : S[(16 * q + acc_row<T>(lk, r)) * LDT + 16 * w + lr];
    if (next)
        flow_wait(flag, before, seen, nullptr, 0, nullptr, f.status(), f.limit, chain);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        flow_wait(f.dflag(J), 4 * p + 4, sm.seen + 2, nullptr, 0, nullptr, f.status(), f.limit, chain);
        flow_strip<T, RIGHT>(sm.tile.P, p, f.pack(J), f.tile(J, J), f.ld(J), f.valid(J));
        if (next && p > 0) /* the strip before; its stores landed with this one's loads */
            flow_count(flag, 1);
        __syncthreads();
        flow_solve<T, RIGHT>(a, sm.tile.P, p);
        if (next) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = 16 * p + acc_row<T>(lk, r), o = 16 * w + lr;
                if (ok)
                    store_coherent(G + (RIGHT ? (int64_t)o * f.ld(J) + k : (int64_t)k * f.ld(I) + o), a[p][r]);
            }
        }
    }
    if (next) {
        flow_count(flag, 1);
        return;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            S[RIGHT ? (16 * w + lr) * LDT + 16 * q + acc_row<T>(lk, r)
                    : (16 * q + acc_row<T>(lk, r)) * LDT + 16 * w + lr] = a[q][r];
    __syncthreads();
    tile_xfer<T>([&](int r, int c) { return S[r * LDT + c]; },
                 [&](int r, int c, T v) {
                     if (r < nr && c < nc)
                         store_coherent(G + (int64_t)r * f.ld(c0) + c, v);
                 });
    flow_wait(flag, before, seen, nullptr, 0, nullptr, f.status(), f.limit, chain);
    flow_count(flag, 4);
}

/* Diagonal tile J. */
template <typename T, typename F>
__device__ __forceinline__ void flow_diagonal(const F &f, int J, int32_t *info, FlowSmem<T> &sm)
{
    typedef typename vec4<T>::type V;
    const int nr = f.rows(J), valid = f.valid(J), w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const bool last = J > 0 && f.has_l(J, J - 1) && f.has_u(J - 1, J); /* a product with block J - 1 */
    T *S = sm.tile.S, *D = f.tile(J, J);
    constexpr bool chain = true;
    const bool pub = f.publish(J);
    if (w >= NT / 64) { /* the publishing waves: past the barriers of the others up to tile_lu64 */
        if (!pub)
            return;
        for (int k = f.first(J, J); k < J - 1;) { /* flow_products */
            __syncthreads();
            const int kn = flow_run<T, F>(k, J - 1, sm);
            for (int b = TB / 16 * (kn - k); b > 0; --b)
                __syncthreads();
            k = kn;
        }
        for (int b = last ? 5 : 2; b > 0; --b)
            __syncthreads();
        f.guard(J);
        publish_strips(S, sm.tile.P, f.pack(J), D, f.ld(J), valid, f.dflag(J));
        return;
    }
    V acc[2][2];
    flow_products<T>(acc, f, J, J, J - 1, chain, sm);
    tile_to_lds<T, 2>(acc, S, valid, valid, true);
    __syncthreads();
    if (last) {
        const T *TL = f.tile(J, J - 1), *TU = f.tile(J - 1, J);
        const int fl = 16 * f.lcount(J, J - 1), fu = 16 * f.ucount(J, J - 1);
        V d[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                d[c][r] = S[(16 * w + acc_row<T>(lk, r)) * LDT + 16 * c + lr];
        /* rows and columns past the matrix end: the last one again, dropped below */
        const int64_t row = (int64_t)min(16 * w + lr, nr - 1) * f.ld(J - 1);
        /* two strips at a time: a wait and the loads cost more than a strip's
         * products */
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            flow_wait(f.lflag(J), fl + 8 * h + 8, sm.seen, f.uflag(J), fu + 8 * h + 8, sm.seen + 1, f.status(), f.limit,
                      chain);
            T a[8], b[4][8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = 32 * h + 16 * (e >> 2) + acc_row<T>(lk, e & 3);
                a[e] = load_coherent(TL + row + k);
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    b[c][e] = load_coherent(TU + (int64_t)k * f.ld(J) + min(16 * c + lr, nr - 1));
            }
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    d[c] = mfma16(-a[e], b[c][e], d[c]);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * w + acc_row<T>(lk, r), j = 16 * c + lr;
                if (i < valid && j < valid)
                    S[i * LDT + j] = d[c][r];
            }
        __syncthreads();
    }
    const int z = tile_lu64<T, true>(S, sm.tile.P, (T *)nullptr, valid, &sm.zero);
    if (!pub)
        lds_store_tile(S, D, f.ld(J), valid, valid);
    if (threadIdx.x == 0 && info && z) { /* the smallest over the diagonal tiles */
        const int at = J * TB + z;
        int was = 0;
        while (!__hip_atomic_compare_exchange_strong(info, &was, at, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT) &&
               (was == 0 || was > at))
            ;
    }
}

/* The dense matrix as a dataflow, right-hand sides (if any) as block columns
 * nb .. of U: Y_J = L_JJ^{-1} (B_J - sum L_Jk Y_k).  ctl: the status word, then
 * from word 3 the ticket, the strip flags, the flags of the right-hand sides'
 * columns; behind the control words the flags of the block rows and columns, a
 * cache line each, then the packs of the last two (three) diagonal tiles.  A pack is
 * free again when every tile of its step is finished. */
constexpr int kFlowLine = 32; /* ints of a cache line */
template <typename T, bool WIDE> struct DenseFlow { /* WIDE: tickets in the order of pairs of steps */
    T *A, *B;
    int64_t lda, ldb;
    int n, nb, nrhs, nbc, line; /* line: ints from one flag to the next */
    static constexpr int npacks = WIDE ? 3 : 2;
    int *ctl, *flags;
    T *packs;
    long limit;
    static constexpr bool joined = true;
    __device__ __forceinline__ T *tile(int I, int K) const
    {
        return K < nb ? A + (int64_t)I * TB * lda + K * TB : B + (int64_t)I * TB * ldb + (K - nb) * TB;
    }
    __device__ __forceinline__ int64_t ld(int K) const { return K < nb ? lda : ldb; }
    __device__ __forceinline__ int rows(int I) const { return min(TB, I < nb ? n - I * TB : nrhs - (I - nb) * TB); }
    __device__ __forceinline__ int valid(int I) const { return rows(I); }
    __device__ __forceinline__ int first(int, int) const { return 0; }
    __device__ __forceinline__ bool has_l(int, int) const { return true; }
    __device__ __forceinline__ bool has_u(int, int) const { return true; }
    __device__ __forceinline__ int lcount(int, int J) const { return J; }
    __device__ __forceinline__ int ucount(int, int J) const { return J; }
    __device__ __forceinline__ bool next(int J, int I) const { return I == J + 1 && I < nb; }
    __device__ __forceinline__ bool publish(int J) const { return J + 1 < nb || nbc > 0; }
    __device__ __forceinline__ int *status() const { return ctl; }
    __device__ __forceinline__ int *ticket() const { return ctl + 3; }
    __device__ __forceinline__ int *dflag(int J) const { return ctl + 4 + J; }
    __device__ __forceinline__ int *lflag(int I) const { return flags + line * I; }
    __device__ __forceinline__ int *uflag(int K) const
    {
        return K < nb ? flags + line * (nb + K) : ctl + 4 + K;
    }
    __device__ __forceinline__ T *pack(int J) const { return packs + (J % npacks) * TB * 16; }
    /* tiles of step J, or WIDE of the steps J, J + 1 */
    __device__ __forceinline__ int tiles(int J) const
    {
        const bool pair = WIDE && J + 1 < nb;
        return (pair ? 2 : 1) * (2 * (nb - 1 - J) + nbc) + (pair ? 0 : 1);
    }
    __device__ __forceinline__ void guard(int J) const
    {
        const int done = J - npacks, rows = nb - 1 - done; /* block rows below and columns right of that tile */
        for (int e = (int)threadIdx.x - NT; done >= 0 && e < 2 * rows + nbc; e += NTP - NT) {
            const int *flag = e < rows ? lflag(done + 1 + e) : uflag(done + 1 + e - rows);
            long spins = 0;
            while (load_coherent(flag) < 16 * (done + 1)) {
                __builtin_amdgcn_s_sleep(1);
                if (wait_give_up(status(), ++spins, limit))
                    break;
            }
        }
    }
};
template <typename T, bool WIDE>
__global__ __launch_bounds__(NTP, kFlowWaves) void k_flow(DenseFlow<T, WIDE> f, int32_t *info)
{
    __shared__ FlowSmem<T> sm;
    if (threadIdx.x == 0) {
        sm.ticket = atomicAdd(f.ticket(), 1);
        sm.seen[0] = sm.seen[1] = sm.seen[2] = 0;
    }
    __syncthreads();
    int q = __builtin_amdgcn_readfirstlane(sm.ticket), J = 0;
    for (; J < f.nb && q >= f.tiles(J); J += WIDE ? 2 : 1)
        q -= f.tiles(J);
    if (J >= f.nb) { /* counter not reset: refuse */
        if (threadIdx.x == 0)
            atomicOr(f.status(), 2);
        return;
    }
    /* I: the tile's other block row or column.  One step: the diagonal tile,
     * the tiles below and right of it in turn, the right-hand sides.  Two: their
     * corner in the order of the chain, then the rows below and the columns
     * right of it eight at a time, so that the two tiles of a row (column) are
     * eight tickets apart, which puts them on one XCD as workgroups are dealt
     * out, where they read the same operand from one L2; then the right-hand
     * sides. */
    int I = J;
    bool lower = false;
    const bool pair = WIDE && J + 1 < f.nb;
    const int R = pair ? f.nb - 2 - J : f.nb - 1 - J;
    if (!pair) {
        lower = q > 0 && q <= 2 * R && (q & 1);
        I = q == 0 ? J : (q <= 2 * R ? J + 1 + (q - 1) / 2 : f.nb + q - 1 - 2 * R);
    } else if (q < 4) {
        I = q == 0 ? J : J + 1;
        lower = q == 1;
        J += q == 3;
    } else if (q < 4 + 4 * R) {
        const int g = (q - 4) / 32, p = (q - 4) % 32, c8 = min(8, R - 8 * g), h = p / c8;
        I = J + 2 + 8 * g + p % c8;
        lower = (h & 1) == 0;
        J += h >> 1;
    } else {
        q -= 4 + 4 * R;
        I = f.nb + q % f.nbc;
        J += q / f.nbc;
    }
    if (I == J) {
        __builtin_amdgcn_s_setprio(3); /* the chain, ahead of its compute unit's other waves */
        flow_diagonal<T>(f, J, info, sm);
        return;
    }
    if (threadIdx.x >= NT)
        return;
    if (I == J + 1)
        __builtin_amdgcn_s_setprio(2);
    if (lower)
        flow_panel<T, true>(f, J, I, sm);
    else
        flow_panel<T, false>(f, J, I, sm);
}

/* Beyond this the tickets go by pairs of steps: what bounds the factor then is
 * the operands' way past L2 (6 TB/s).  One step | two, ms: FP64 n = 4096 1.20 |
 * 1.21, 6000 2.95 | 3.06, 8192 7.26 | 7.20, 16384 57.3 | 54.9; FP32 4096 1.26 |
 * 1.28, 6000 2.24 | 2.23, 8192 4.54 | 4.28, 16384 32.3 | 30.0 (the mixed-
 * precision solve of that size 38.9 | 36.6). */
constexpr int kFlowWide = 7168;

/* Ints from one flag of a block row or column to the next: a cache line, or
 * less where there are more than the room in front of the packs (of the
 * 64 x 64 elements that a block step's pack takes) holds. */
template <typename T> static int flow_line(int n)
{
    const int nb = (n + TB - 1) / TB, npacks = n > kFlowWide ? 3 : 2;
    const size_t room = (factor_pg_bytes(sizeof(T)) - npacks * TB * 16 * sizeof(T)) / sizeof(int);
    int line = kFlowLine;
    while (line > 1 && (size_t)2 * nb * line > room)
        line /= 2;
    return (size_t)2 * nb * line <= room ? line : 0;
}

/* Whether the factor runs as one dataflow launch.  FP64 | FP32, us, dataflow
 * against block steps: n = 256 69 against 75 | 66, 66; 1024 270, 298 | 247, 261;
 * 4096 1207, 2031 | 1253, 1483; 8192 7328, 9625 | 4470, 6662; 16384 54.9, 61.8
 * ms | 30.0, 36.2; 24576 193, 201 | 107, 108; 32768 449, 469 | 251, 236: the
 * block steps' taller FP32 tiles win once there is nothing but update work.
 * Deferral that is asked for at every size (defer_above 0) and the other factor
 * variants stay launches. */
constexpr int kFlowF32 = 28672;
template <typename T> static bool use_flow(int n, int nrhs, const DenseTuning &tun)
{
    const int nb = (n + TB - 1) / TB, nbc = (nrhs + TB - 1) / TB;
    return (sizeof(T) == 8 || n <= kFlowF32) && tun.lookahead && tun.defer_above > 0 && flow_line<T>(n) > 0 &&
           (size_t)(4 + nb + nbc) * sizeof(int) <= factor_ctl_bytes(n);
}
/* Words of the workspace to clear before a factor: the control words and, right
 * behind them, the dataflow's flags. */
template <typename T> static int factor_words(int n)
{
    const int nb = (n + TB - 1) / TB;
    return (int)(factor_ctl_bytes(n) / sizeof(int)) + 2 * nb * flow_line<T>(n);
}
template <bool WIDE, typename T>
static hipError_t factor_flow(T *A, int64_t lda, int n, int32_t *info, void *ws, const DenseTuning &tun,
                              UpdateProfile *pr, hipStream_t st, T *B, int64_t ldb, int nrhs)
{
    char *p = static_cast<char *>(ws) + factor_ctl_bytes(n);
    DenseFlow<T, WIDE> f;
    f.A = A, f.B = B, f.lda = lda, f.ldb = ldb, f.n = n, f.nb = (n + TB - 1) / TB;
    f.nrhs = B ? nrhs : 0, f.nbc = (f.nrhs + TB - 1) / TB;
    f.ctl = static_cast<int *>(ws), f.flags = reinterpret_cast<int *>(p);
    f.line = flow_line<T>(n);
    f.packs = reinterpret_cast<T *>(p + factor_pg_bytes(sizeof(T))) - f.npacks * TB * 16;
    f.limit = tun.wait_limit > 0 ? (long)tun.wait_limit : 1L << 24;
    double fl = 0.0; /* update flops: step k takes 2 * 64 for each element of the region past its panel */
    for (int e0 = TB; e0 < n; e0 += TB)
        fl += 2.0 * TB * (double)(n - e0) * (double)(n - e0);
    int pslot = -1;
    const bool prof = profile_slot(pr, st, fl, pslot);
    hipLaunchKernelGGL((k_flow<T, WIDE>), dim3(f.nb * (f.nb + f.nbc)), dim3(NTP), 0, st, f, info);
    const hipError_t e = hipGetLastError();
    if (prof)
        (void)hipEventRecord(pr->ev[2 * pslot + 1], st);
    return e;
}

template <typename T>
hipError_t dense_factor(T *A, int64_t lda, int n, int32_t *info, void *ws, const DenseTuning &tun,
                        UpdateProfile *pr, hipStream_t st, T *B, int64_t ldb, int nrhs, bool prefilled)
{
    if (nrhs <= 0)
        B = nullptr;
    if (info && !prefilled) {
        hipError_t e = fill_i32(info, 1, 0, st);
        if (e != hipSuccess)
            return e;
    }
    int *ctl = static_cast<int *>(ws);
    T *Pg = reinterpret_cast<T *>(static_cast<char *>(ws) + factor_ctl_bytes(n));
    if (!prefilled) { /* status word and the block steps' counters */
        hipError_t e = fill_i32(ctl, factor_words<T>(n), 0, st);
        if (e != hipSuccess)
            return e;
    }
    if (use_flow<T>(n, B ? nrhs : 0, tun))
        return n > kFlowWide ? factor_flow<true>(A, lda, n, info, ws, tun, pr, st, B, ldb, nrhs)
                             : factor_flow<false>(A, lda, n, info, ws, tun, pr, st, B, ldb, nrhs);
    if (tun.lookahead)
        return factor_lookahead(A, lda, n, info, Pg, ctl, tun, pr, st, B, ldb, nrhs);
    return factor_phases(A, lda, n, info, Pg, tun, pr, st, B, ldb, nrhs);
}

/* Start of a solve (or a factor + solve): control words and info cleared and
 * the substitution's exchange rows marked unsolved, in one launch. */
template <typename T>
__global__ void k_solve_init(int *ctl, int nctl, int32_t *info, T *xb, int64_t nxb)
{
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = i0; i < nctl; i += step)
        ctl[i] = 0;
    if (info && i0 == 0)
        *info = 0;
    if (sizeof(T) == 8) {
        unsigned long long *x = reinterpret_cast<unsigned long long *>(xb);
        for (int64_t i = i0; i < nxb; i += step)
            x[i] = kUnsolvedMark64;
    } else {
        unsigned int *x = reinterpret_cast<unsigned int *>(xb);
        for (int64_t i = i0; i < nxb; i += step)
            x[i] = kUnsolvedMark32;
    }
}

template <typename T>
static hipError_t solve_init(int *ctl, int nctl, int32_t *info, T *xb, int64_t nxb, hipStream_t st)
{
    const int grid = (int)std::min<int64_t>((nxb + 255) / 256 + 1, 1024);
    hipLaunchKernelGGL((k_solve_init<T>), dim3(grid), dim3(256), 0, st, ctl, nctl, info, xb, nxb);
    return hipGetLastError();
}

template <typename T>
hipError_t factor_solve(T *A, int64_t lda, int n, int32_t *info, void *ws, int chunks, const DenseTuning &tun,
                        UpdateProfile *pr, hipStream_t st, T *B, int64_t ldb, int nrhs)
{
    const int nb = (n + TB - 1) / TB;
    int *ctl = static_cast<int *>(ws);
    T *xb = reinterpret_cast<T *>(static_cast<char *>(ws) + factor_ws_bytes(sizeof(T), n));
    /* the exchange rows are marked here when one chunk at a time uses them */
    const bool mark = nrhs > 0 && (chunks == 1 || nrhs <= 16);
    const int64_t nxb = mark ? (int64_t)(kTrsvHelpers + 1) * nb * TB * 16 : 0;
    hipError_t e = solve_init<T>(ctl, factor_words<T>(n), info, xb, nxb, st);
    if (e == hipSuccess)
        e = dense_factor<T>(A, lda, n, info, ws, tun, pr, st, B, ldb, nrhs, true);
    if (e != hipSuccess)
        return e;
    /* the backward substitution reports the status word into info at its
     * end; without right-hand sides a separate launch does */
    if (nrhs > 0)
        return dense_trsv<T>(TRI_U, A, lda, n, B, ldb, nrhs, ctl, xb, chunks, nullptr, info, st,
                             mark ? TrsvStart::ready : TrsvStart::running, tun.wait_limit);
    return fold_status(ctl, info, st);
}

/* ------------------------------------------------- triangular solves --- */

/*
 * Multi-workgroup triangular solve op(T) Y = B (Eq. 1, blocked): per
 * 64-row block, kTrsvHelpers helper workgroups and the block's own, tickets
 * taken in solve order (a block's helpers before it).  The block's own
 * workgroup does everything that does not need the block solved just
 * before it first:
 *   - the inverse of its diagonal operator block D (tile_inv16 on the
 *     factored diagonal tile) and W_j = D^{-1} M_j for the two blocks solved
 *     just before it;
 *   - the contributions of all earlier blocks, as they appear:
 *     r = b - sum_j M_j y_j (the older ones shared with its helpers, whose
 *     partial sums follow the exchange rows, marked like them), and
 *     z = D^{-1} r;
 * so that each of the two last blocks costs one product in registers as it
 * arrives: y = z - W_{j1} y_{j1} - W_{j2} y_{j2} (the two products in an
 * accumulator of their own, so neither waits for z).  The 16 columns of the
 * matrix-core products are 16 right-hand sides; further ones go in chunks of
 * 16, up to kTrsvChunks of them side by side in one launch, each a chain of
 * its own (the launch is bound by the chain's latency, 2.2 us a block, not by
 * the compute units: 47 blocks and 40 right-hand sides, forward and backward,
 * 656 us in three launches each, one after the other).  Wave w owns rows
 * 16w..16w+15 of the block.
 * Solved blocks are exchanged through XB (n rounded up to 64 rows, pitch 16,
 * filled with the unsolved mark before the launch): a workgroup stores its
 * block there with coherent stores and, without waiting for them, raises
 * the solved-blocks counter.  The workgroups of the next three blocks poll
 * a block's values directly (re-reading until none is the mark), so each of
 * those dependencies costs one round trip; every other reader first waits
 * for the counter to pass the block and reads it through the caches, so the
 * lines being polled see three readers rather than every later workgroup.
 * Solutions also go to B.
 */
template <typename T, int MODE>
__global__ __launch_bounds__(NT) void k_trsv(const T *__restrict__ LU, int64_t lda, int n, T *__restrict__ B,
                                             int64_t ldb, int nrhs, int nch, int *wsi, T *__restrict__ XB,
                                             const int *skip, int32_t *info, long wlim)
{
    typedef typename vec4<T>::type V;
    if (skip && *skip)
        return;
    __shared__ TileSmem<T> sm;
    __shared__ T wls[2][16][NT]; /* -W of the last two blocks, A-operand order per thread */
    int *status = wsi, *ctr = wsi + 1;
    if (threadIdx.x == 0) {
        sm.ticket = atomicAdd(ctr, 1);
        sm.avail = 0;
    }
    __syncthreads();
    const int nb = (n + TB - 1) / TB;
    if (sm.ticket >= (kTrsvHelpers + 1) * nb * nch) { /* counter not reset: refuse rather than index out of range */
        if (threadIdx.x == 0)
            atomicOr(status, 2);
        return;
    }
    constexpr bool FWD = tri_forward(MODE), TR = tri_trans(MODE), UNITL = (MODE == TRI_L || MODE == TRI_LT);
    /* kTrsvHelpers helpers, then the block's own workgroup, per position:
     * a workgroup only ever waits for lower tickets */
    const int item = sm.ticket / (kTrsvHelpers + 1), role = sm.ticket % (kTrsvHelpers + 1);
    const int pos = item / nch, ch = item - pos * nch;
    const bool helper = role < kTrsvHelpers;
    /* this chunk's columns, exchange rows and counter */
    const int nrhs_here = min(16, nrhs - 16 * ch);
    int *solved = wsi + 2 + ch;
    B += 16 * ch;
    XB += (int64_t)ch * (kTrsvHelpers + 1) * nb * TB * 16;
    const int blk = FWD ? pos : nb - 1 - pos;
    const int ndep = pos; /* blocks solved before this one */
    const int t = threadIdx.x, w = wave_id(), l = t & 63, lr = l & 15, lk = l >> 4;
    const int r0 = blk * TB, nr = min(TB, n - r0);
    auto dep_blk = [&](int d) { return FWD ? d : nb - 1 - d; };
    /* element (r, k) of operator block (blk, bj): op(T)[r0 + r][bj*64 + k];
     * the address is clamped and the value selected, so the loads of a tile
     * are issued without branches (the compiler then waits for exactly the
     * loads a use needs) */
    auto opel = [&](int bj, int r, int k) -> T {
        const int gr = r0 + r, gk = bj * TB + k;
        const int cr = min(gr, n - 1), ck = min(gk, n - 1);
        const T v = TR ? LU[(int64_t)ck * lda + cr] : LU[(int64_t)cr * lda + ck];
        return ((gr < n) & (gk < n)) ? v : T(0);
    };
    /* this lane's 16 elements of operator block (blk, bj) as the A operand,
     * loaded raw from clamped addresses; a_op applies the bounds where the
     * values are used, so nothing waits for these loads before then */
    auto load_a = [&](int bj, T(&a)[16]) {
        const int cr = min(r0 + 16 * w + lr, n - 1);
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) {
            const int ck = min(bj * TB + 4 * ks + lk, n - 1);
            a[ks] = TR ? LU[(int64_t)ck * lda + cr] : LU[(int64_t)cr * lda + ck];
        }
    };
    auto a_op = [&](int bj, int ks, T a) {
        return ((r0 + 16 * w + lr < n) & (bj * TB + 4 * ks + lk < n)) ? a : T(0);
    };
    /* solved block bj (all 64 rows, as the B operand); every row and column
     * of an exchange block is written by its producer (zeros past n and past
     * the right-hand sides), so the loads need no bounds */
    auto fetch_y = [&](int bj, T(&y)[16]) {
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
            y[ks] = load_coherent(XB + (int64_t)(bj * TB + 4 * ks + lk) * 16 + lr);
    };
    /* the same through the caches, for a block the counter has passed: the
     * XCD's L2 fetches it once for all its readers instead of every wave of
     * every later workgroup going to the point of coherence.  A cached line
     * can only hold final values or the mark (each element is written once
     * per launch), and a mark sends the reader to load_y's coherent reads. */
    auto fetch_y_cached = [&](int bj, T(&y)[16]) {
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
            y[ks] = XB[(int64_t)(bj * TB + 4 * ks + lk) * 16 + lr];
    };
    auto has_mark = [&](const T(&y)[16]) {
        bool miss = false;
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
            miss = miss || is_unsolved_mark(y[ks]);
        return miss;
    };
    /* re-read block bj while any value this wave needs still holds the mark */
    auto load_y = [&](int bj, T(&y)[16]) {
        for (long spins = 0;; ++spins) {
            fetch_y(bj, y);
            if (!__any(has_mark(y)))
                break;
            if (wait_give_up(status, spins, wlim))
                break;
            __builtin_amdgcn_s_sleep(1);
        }
    };

    /* Contributions of the blocks solved before, all but the last three:
     * dependency d goes to role d mod (kTrsvHelpers + 1), so that a block's
     * older dependencies are taken by kTrsvHelpers helper workgroups and its
     * own workgroup together.  One pass per dependency: its values are
     * requested first, then the operator block of this role's next one, so
     * the operator loads overlap the wait for the values; the two operator
     * register sets (and two accumulators) alternate between passes, so no
     * copy makes a pass wait for the loads it has just issued.  The loads are
     * issued unconditionally (indices clamped) so that the waits count only
     * the loads each use needs. */
    constexpr int STRIDE = kTrsvHelpers + 1;
    const int K = ndep - 2;  /* blocks before the last two */
    const int KP = K - 1;    /* ... of which those taken in passes; block K-1 is polled */
    V acc = {0, 0, 0, 0}, acc2 = {0, 0, 0, 0};
    auto pass = [&](int d, const T(&cur)[16], T(&nxt)[16], V &ac) __attribute__((always_inline)) {
        /* read once the counter has passed the block (the values are then
         * normally there: re-read below if not) */
        wait_solved(solved, d, &sm.avail, status, wlim);
        T y[16];
        fetch_y_cached(dep_blk(d), y);
        __builtin_amdgcn_sched_barrier(0);
        load_a(dep_blk(min(d + STRIDE, KP - 1)), nxt);
        __builtin_amdgcn_sched_barrier(0);
        if (__any(has_mark(y)))
            load_y(dep_blk(d), y);
        const int bd = dep_blk(d);
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
            ac = mfma16(a_op(bd, ks, cur[ks]), y[ks], ac);
    };
    auto passes = [&]() __attribute__((always_inline)) {
        if (role < KP) {
            T a0[16], a1[16];
            load_a(dep_blk(role), a0);
            for (int d = role; d < KP; d += 2 * STRIDE) {
                pass(d, a0, a1, acc);
                if (d + STRIDE < KP)
                    pass(d + STRIDE, a1, a0, acc2);
            }
        }
    };
    /* the helpers' partial sums follow the exchange rows, in accumulator
     * layout (thread t's four values at 4t), marked like them */
    T *PB = XB + (int64_t)nb * TB * 16;
    if (helper) {
        passes();
        T *pp = PB + ((int64_t)pos * kTrsvHelpers + role) * (TB * 16) + 4 * t;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            store_coherent(pp + r, acc[r] + acc2[r]);
        return;
    }

    /* own right-hand side, in accumulator layout (rows 16w + acc_row, column lr) */
    V rhs;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * w + acc_row<T>(lk, r);
        rhs[r] = (row < nr && lr < nrhs_here) ? B[(int64_t)(r0 + row) * ldb + lr] : T(0);
    }

    /* inverse of the diagonal operator block, from the factored tile; it
     * stays in sm.t1 and is read into registers where it is used */
    stage_tile_identity(sm.t0, LU + (int64_t)r0 * lda + r0, lda, nr, nr);
    __syncthreads();
    if (t < TB)
        sm.rinv[t] = recip(sm.t0[t * (LDT + 1)]);
    __syncthreads();
    tile_inv16(sm.t0, sm.rinv, sm.t1);
    auto load_dinv = [&](T(&dA)[16]) { /* op(D)^{-1}[16w + lr][4ks + lk] */
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) {
            const int r = 16 * w + lr, k = 4 * ks + lk;
            const int i = TR ? k : r, j = TR ? r : k; /* element (i, j) of L^{-1} or U^{-1} */
            const T v = sm.t1[i * LDT + j];
            dA[ks] = UNITL ? (i > j ? v : (i == j ? T(1) : T(0))) : (i <= j ? v : T(0));
        }
    };

    /* -W_j = -D^{-1} M_j for the two blocks solved last (M_j: their operator
     * blocks), needed only after the last waits but independent of every
     * solution: formed now and kept in LDS in this thread's A-operand order */
    auto form_w = [&](int bj, const T(&dA)[16], int slot) {
        tile_xfer<T>([&](int r, int c) { return opel(bj, r, c); }, [&](int r, int c, T v) { sm.t0[r * LDT + c] = v; });
        __syncthreads();
        V wacc[4];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            wacc[cb] = V{0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < 16; ++ks)
                wacc[cb] = mfma16(dA[ks], sm.t0[(4 * ks + lk) * LDT + 16 * cb + lr], wacc[cb]);
        }
        __syncthreads();
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                sm.t0[(16 * w + acc_row<T>(lk, r)) * LDT + 16 * cb + lr] = wacc[cb][r];
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
            wls[slot][ks][t] = -sm.t0[(16 * w + lr) * LDT + 4 * ks + lk];
        __syncthreads();
    };
    {
        T dA[16];
        load_dinv(dA);
        if (ndep >= 1)
            form_w(dep_blk(ndep - 1), dA, 0);
        if (ndep >= 2)
            form_w(dep_blk(ndep - 2), dA, 1);
    }

    if (K > 0) {
        T al[16]; /* operator block of block K-1, loaded first */
        load_a(dep_blk(K - 1), al);
        passes();
        /* block K-1 (three before this one) is polled directly: at the front
         * of the chain it is what z waits for */
        T y[16];
        load_y(dep_blk(K - 1), y);
        const int bl = dep_blk(K - 1);
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
            acc = mfma16(a_op(bl, ks, al[ks]), y[ks], acc);
        /* the helpers' partial sums, re-read until none is the mark */
#pragma unroll
        for (int h = 0; h < kTrsvHelpers; ++h) {
            const T *pp = PB + ((int64_t)pos * kTrsvHelpers + h) * (TB * 16) + 4 * t;
            T pv[4];
            for (long spins = 0;; ++spins) {
                bool miss = false;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    pv[r] = load_coherent(pp + r);
                    miss = miss || is_unsolved_mark(pv[r]);
                }
                if (!__any(miss))
                    break;
                if (wait_give_up(status, spins, wlim))
                    break;
                __builtin_amdgcn_s_sleep(1);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc[r] += pv[r];
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
        acc[r] += acc2[r];

    /* x = D^{-1} (b - acc), through LDS (rows of r come from all four waves),
     * then - W_j y_j for the two blocks solved last, each a product in
     * registers as its values arrive */
    T *Rl = sm.t0; /* 64 x 16, pitch 17 */
#pragma unroll
    for (int r = 0; r < 4; ++r)
        Rl[(16 * w + acc_row<T>(lk, r)) * 17 + lr] = rhs[r] - acc[r];
    __syncthreads();
    V x = {0, 0, 0, 0};
    {
        T dA[16];
        load_dinv(dA);
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
            x = mfma16(dA[ks], Rl[(4 * ks + lk) * 17 + lr], x);
    }
    /* the last two blocks, polled directly, into their own accumulator so
     * that neither waits for z */
    V xw = {0, 0, 0, 0};
    if (ndep >= 2) {
        T wa[16], y[16];
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
            wa[ks] = wls[1][ks][t];
        load_y(dep_blk(ndep - 2), y);
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
            xw = mfma16(wa[ks], y[ks], xw);
    }
    if (ndep >= 1) {
        T wa[16], y[16];
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
            wa[ks] = wls[0][ks][t];
        load_y(dep_blk(ndep - 1), y);
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
            xw = mfma16(wa[ks], y[ks], xw);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
        x[r] += xw[r];
    /* all 64 rows and 16 columns of the exchange block are written (zeros
     * outside the system), the solution rows also to B */
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * w + acc_row<T>(lk, r);
        const bool ok = row < nr && lr < nrhs_here;
        store_coherent(XB + (int64_t)(r0 + row) * 16 + lr, ok ? x[r] : T(0));
        if (ok)
            B[(int64_t)(r0 + row) * ldb + lr] = x[r];
    }
    /* the hint for the readers of later blocks (they check the values); a
     * maximum, since without a wait for the stores above the updates of
     * consecutive blocks may land out of order */
    __syncthreads();
    if (t == 0)
        __hip_atomic_fetch_max(solved, pos + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    /* the last block's workgroup ends after every wait of the launch has
     * ended (each block waited for the one before it and for its helpers),
     * so a give-up anywhere is in the status word by now: report it */
    if (info && pos == nb - 1 && t == 0) {
        __threadfence();
        const int st = load_coherent(status);
        if (st)
            *info = -st;
    }
}

template <typename T, int MODE>
static hipError_t trsv_mode(const T *LU, int64_t lda, int n, T *B, int64_t ldb, int nrhs, int *wsi, T *xb, int chunks,
                            const int *skip, int32_t *info, hipStream_t st, TrsvStart start, long wlim)
{
    const int nb = (n + TB - 1) / TB;
    const int64_t nx = (int64_t)(kTrsvHelpers + 1) * nb * TB * 16;
    hipError_t e = hipSuccess;
    for (int c0 = 0; c0 < nrhs; c0 += 16 * chunks) {
        const int nc = min(16 * chunks, nrhs - c0), nch = (nc + 15) / 16;
        if (c0 > 0 || start != TrsvStart::ready) { /* counters cleared, exchange rows marked */
            const bool all = c0 == 0 && start == TrsvStart::fresh;
            if ((e = solve_init<T>(wsi + (all ? 0 : 1), (all ? 2 : 1) + nch, all ? info : nullptr, xb, nch * nx, st)) !=
                hipSuccess)
                return e;
        }
        hipLaunchKernelGGL((k_trsv<T, MODE>), dim3((kTrsvHelpers + 1) * nb * nch), dim3(NT), 0, st, LU, lda, n, B + c0,
                           ldb, nc, nch, wsi, xb, skip, info, wlim);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    return e;
}

template <typename T>
hipError_t dense_trsv(int mode, const T *LU, int64_t lda, int n, T *B, int64_t ldb, int nrhs, int *wsi, T *xb,
                      int chunks, const int *skip, int32_t *info, hipStream_t st, TrsvStart start, long long wait_limit)
{
    const long wl = wait_limit > 0 ? (long)wait_limit : 1L << 22;
    switch (mode) {
    case TRI_L: return trsv_mode<T, TRI_L>(LU, lda, n, B, ldb, nrhs, wsi, xb, chunks, skip, info, st, start, wl);
    case TRI_U: return trsv_mode<T, TRI_U>(LU, lda, n, B, ldb, nrhs, wsi, xb, chunks, skip, info, st, start, wl);
    case TRI_UT: return trsv_mode<T, TRI_UT>(LU, lda, n, B, ldb, nrhs, wsi, xb, chunks, skip, info, st, start, wl);
    default: return trsv_mode<T, TRI_LT>(LU, lda, n, B, ldb, nrhs, wsi, xb, chunks, skip, info, st, start, wl);
    }
}

/* ---------------------------------------------------- uniform batches --- */

template <typename T>
__global__ __launch_bounds__(NT, kCroutPerCu<T>) void k_lu_batch(T *__restrict__ A, int64_t lda, int n, int64_t strideA,
                                                    int32_t *info)
{
    __shared__ CroutSmem<T> sm;
    T *Ab = A + (int64_t)blockIdx.x * strideA;
    const int z = wg_crout<T>(Ab, lda, n, nullptr, 0, 0, sm);
    if (threadIdx.x == 0 && info)
        info[blockIdx.x] = z;
}

template <typename T, int M1, int M2, int NR>
__global__ __launch_bounds__(NT, 2) void k_solve_batch(const T *__restrict__ LU, int64_t lda, int n, int64_t strideLU,
                                                       T *__restrict__ B, int64_t ldb, int64_t strideB, int nrhs_here)
{
    __shared__ TileSmem<T> sm;
    const T *L = LU + (int64_t)blockIdx.x * strideLU;
    T *Bb = B + (int64_t)blockIdx.x * strideB;
    wg_solve<T, M1, NR>(L, lda, n, Bb, ldb, nrhs_here, sm);
    wg_solve<T, M2, NR>(L, lda, n, Bb, ldb, nrhs_here, sm);
}

/* One right-hand side per system (n <= 64 LDT): both substitutions with the
 * vector in LDS, the factor read once with coalesced loads (wg_trsv1). */
template <typename T, int M1, int M2>
__global__ __launch_bounds__(NT, 2) void k_solve_batch1(const T *__restrict__ LU, int64_t lda, int n, int64_t strideLU,
                                                        T *__restrict__ B, int64_t ldb, int64_t strideB)
{
    __shared__ TileSmem<T> sm;
    const T *L = LU + (int64_t)blockIdx.x * strideLU;
    T *Bb = B + (int64_t)blockIdx.x * strideB;
    for (int i = threadIdx.x; i < n; i += NT)
        sm.t1[i] = Bb[(int64_t)i * ldb];
    __syncthreads();
    wg_trsv1<T, M1>(L, lda, n, sm.t1, sm.t0);
    wg_trsv1<T, M2>(L, lda, n, sm.t1, sm.t0);
    for (int i = threadIdx.x; i < n; i += NT)
        Bb[(int64_t)i * ldb] = sm.t1[i];
}

template <typename T>
hipError_t batch_factor(T *A, int64_t lda, int n, int64_t batch, int64_t strideA, int32_t *info, hipStream_t st)
{
    for (int64_t b0 = 0; b0 < batch; b0 += 65535) {
        const int nb = (int)std::min<int64_t>(65535, batch - b0);
        hipLaunchKernelGGL(k_lu_batch<T>, dim3(nb), dim3(NT), 0, st, A + b0 * strideA, lda, n, strideA,
                           info ? info + b0 : nullptr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

template <typename T, int M1, int M2>
static hipError_t batch_solve_modes(const T *LU, int64_t lda, int n, int64_t strideLU, T *B, int64_t ldb,
                                    int64_t strideB, int nrhs, int64_t batch, hipStream_t st)
{
    for (int64_t b0 = 0; b0 < batch; b0 += 65535) {
        const int nb = (int)std::min<int64_t>(65535, batch - b0);
        for (int c0 = 0; c0 < nrhs; c0 += 8) {
            const int nh = min(8, nrhs - c0);
            const T *L = LU + b0 * strideLU;
            T *Bb = B + b0 * strideB + c0;
            if (nh == 1 && n <= TB * LDT)
                hipLaunchKernelGGL((k_solve_batch1<T, M1, M2>), dim3(nb), dim3(NT), 0, st, L, lda, n, strideLU, Bb, ldb,
                                   strideB);
            else if (nh == 1)
                hipLaunchKernelGGL((k_solve_batch<T, M1, M2, 1>), dim3(nb), dim3(NT), 0, st, L, lda, n, strideLU, Bb, ldb, strideB, nh);
            else if (nh <= 4)
                hipLaunchKernelGGL((k_solve_batch<T, M1, M2, 4>), dim3(nb), dim3(NT), 0, st, L, lda, n, strideLU, Bb, ldb, strideB, nh);
            else
                hipLaunchKernelGGL((k_solve_batch<T, M1, M2, 8>), dim3(nb), dim3(NT), 0, st, L, lda, n, strideLU, Bb, ldb, strideB, nh);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess)
                return e;
        }
    }
    return hipSuccess;
}

template <typename T>
hipError_t batch_solve(bool adjoint, const T *LU, int64_t lda, int n, int64_t strideLU, T *B, int64_t ldb,
                       int64_t strideB, int nrhs, int64_t batch, hipStream_t st)
{
    if (adjoint)
        return batch_solve_modes<T, TRI_UT, TRI_LT>(LU, lda, n, strideLU, B, ldb, strideB, nrhs, batch, st);
    return batch_solve_modes<T, TRI_L, TRI_U>(LU, lda, n, strideLU, B, ldb, strideB, nrhs, batch, st);
}

/* ----------------------------------------------------- ragged batches --- */

/* Persistent factor + solve of a ragged batch: each workgroup repeatedly
 * takes the next system from the queue (in `order`, the EbV schedule), and
 * factors and solves it alone.  Every workgroup leaves the loop once the
 * queue is exhausted.  TWO workgroups to a compute unit, or as many as
 * kCroutPerCu. */
template <typename T, bool TWO>
__global__ __launch_bounds__(NT, TWO ? 2 : kCroutPerCu<T>) void k_batched(int count, const int *__restrict__ ns, const int64_t *__restrict__ offA,
                                                   T *__restrict__ A, const int64_t *__restrict__ offB, T *__restrict__ B,
                                                   const int *__restrict__ order, int32_t *info, int *queue)
{
    __shared__ union { CroutSmem<T> c; TileSmem<T> s; } smu;
    CroutSmem<T> &sm = smu.c;
    for (;;) {
        if (threadIdx.x == 0)
            sm.ticket = atomicAdd(queue, 1);
        __syncthreads();
        /* uniform across the workgroup: the system's addresses stay scalar */
        const int idx = __builtin_amdgcn_readfirstlane(sm.ticket);
        __syncthreads();
        if (idx >= count)
            break;
        const int s = order ? order[idx] : idx;
        const int n = ns[s];
        if (n <= 0 || (int64_t)n * n * (int64_t)sizeof(T) >= kWgMaxSystemBytes) {
            /* empty, or beyond what one workgroup addresses: reported, untouched */
            if (threadIdx.x == 0 && info)
                info[s] = n <= 0 ? 0 : -3;
            continue;
        }
        T *As = A + offA[s];
        T *Bs = B ? B + offB[s] : nullptr;
        /* factor with the forward substitution riding along, then the
         * backward substitution */
        const int z = wg_crout<T>(As, n, n, Bs, 1, 1, sm);
        if (threadIdx.x == 0 && info)
            info[s] = z;
        if (Bs) {
            if (n <= TB * LDT) {
                /* the vector in LDS (sm.t1), the diagonal blocks staged in sm.t0 */
                for (int i = threadIdx.x; i < n; i += NT)
                    sm.t1[i] = Bs[i];
                __syncthreads();
                wg_trsv1<T, TRI_U>(As, n, n, sm.t1, sm.t0);
                for (int i = threadIdx.x; i < n; i += NT)
                    Bs[i] = sm.t1[i];
            } else {
                wg_solve<T, TRI_U, 1>(As, n, n, Bs, 1, 1, smu.s);
            }
        }
    }
}

/* Largest system whose refinement keeps its float vector in LDS (t1). */
constexpr int kMixLdsN = TB * LDT;
/* ... and, three workgroups to a compute unit, x in double beside it, in what the
 * products' buffers leave of LDS past the diagonal blocks' place. */
constexpr int kMixXdN = (CroutSmem<float>::GEMM - sizeof(float) * TB * LDT) / sizeof(double);
static_assert(kMixXdN == 1568, "both sides of it are tested");

/* Workgroup-wide maximum (result valid in every thread). */
__device__ double wg_max(double v, double *red)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        v = fmax(v, __shfl_xor(v, o));
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    __syncthreads();
    return v;
}

/* Ragged batch, mixed precision: per system a float copy is factored and the
 * float solve is refined in double (residual r = b - A x over the double A,
 * update x += solve_float(r)).  The stop test bounds the forward error: with
 * the system's dominance margin m = min_i (|a_ii| - sum_{j != i} |a_ij|) > 0,
 * ||x - x*||_inf <= ||r||_inf / m, and the loop ends once
 * ||r||_inf <= tol m ||x||_inf (never for m = 0: iters reports -1).
 *
 * TWO workgroups to a compute unit have LDS for x and the registers the
 * refinement wants; three spill 53 of them. */
template <bool TWO>
__global__ __launch_bounds__(NT, TWO ? 2 : kCroutPerCu<float>) void k_batched_mixed(int count, const int *__restrict__ ns, const int64_t *__restrict__ offA,
                                                         const double *__restrict__ A, const int64_t *__restrict__ offB,
                                                         double *__restrict__ B, const int *__restrict__ order,
                                                         int32_t *info, int *queue, float *__restrict__ W,
                                                         float *__restrict__ R32, double *__restrict__ X,
                                                         int max_iter, double tol, int32_t *iters)
{
    __shared__ union { CroutSmem<float> c; TileSmem<float> s; } smu;
    CroutSmem<float> &sm = smu.c;
    __shared__ double red[4], xlds[TWO ? kMixLdsN : 1];
    const int t = threadIdx.x, w = wave_id(), l = t & 63;
    for (;;) {
        if (t == 0)
            sm.ticket = atomicAdd(queue, 1);
        __syncthreads();
        const int idx = __builtin_amdgcn_readfirstlane(sm.ticket);
        __syncthreads();
        if (idx >= count)
            break;
        const int s = order ? order[idx] : idx;
        const int n = ns[s];
        if (n <= 0 || (int64_t)n * n * (int64_t)sizeof(double) >= kWgMaxSystemBytes) {
            /* empty, or beyond what one workgroup addresses: reported, untouched */
            if (t == 0) {
                if (info)
                    info[s] = n <= 0 ? 0 : -3;
                if (iters)
                    iters[s] = n <= 0 ? 0 : -1;
            }
            continue;
        }
        const double *As = A + offA[s];
        double *bs = B + offB[s];
        float *Ws = W + offA[s];
        float *rs = R32 + offB[s];
        double *xs = X + offB[s];
        /* x in double: in LDS of its own, or past the diagonal blocks' place in t0
         * while it fits there, else in memory */
        double *xd = TWO ? xlds : n <= kMixXdN ? reinterpret_cast<double *>(sm.gemm + sizeof(sm.t0)) : xs;
        /* float copy and dominance margin: wave w takes rows 4w .. 4w+3,
         * 4w+16 .., four rows at a time, its lanes the columns (all of a
         * group's loads issued before its sums) */
        double mrow = __longlong_as_double(0x7FF0000000000000ll);
        const int ngr = 4 * w < n ? (n - 4 * w + 15) / 16 : 0; /* this wave's groups of rows */
        auto grow = [&](int g) { return 4 * w + 16 * g; };
        {
            double off[4] = {0.0, 0.0, 0.0, 0.0}, dg[4] = {0.0, 0.0, 0.0, 0.0};
            wave_rows4_stream<double>(
                As, n, ngr, grow, n, 0, n,
                [&](int g, int cb, const double(&v)[4][4]) {
                    const int i0 = grow(g);
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int m = 0; m < 4; ++m) {
                            const int c = cb + 64 * m + l;
                            if (c < n && i0 + u < n) {
                                Ws[(int64_t)(i0 + u) * n + c] = (float)v[u][m];
                                if (c == i0 + u)
                                    dg[u] = fabs(v[u][m]);
                                else
                                    off[u] += fabs(v[u][m]);
                            }
                        }
                },
                [&](int g) {
                    const int i0 = grow(g);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
#pragma unroll
                        for (int o = 32; o > 0; o >>= 1) {
                            off[u] += __shfl_xor(off[u], o);
                            dg[u] += __shfl_xor(dg[u], o);
                        }
                        if (i0 + u < n)
                            mrow = fmin(mrow, fmax(dg[u] - off[u], 0.0));
                        off[u] = dg[u] = 0.0;
                    }
                });
        }
        const double margin = -wg_max(-mrow, red);
        for (int i = t; i < n; i += NT)
            rs[i] = (float)bs[i];
        __syncthreads();
        /* float factor with the first forward substitution riding along */
        const int z = wg_crout<float>(Ws, n, n, rs, 1, 1, sm);
        if (t == 0 && info)
            info[s] = z;
        int used = -1;
        if (n <= kMixLdsN) {
            /* vectors in LDS: the float correction (sm.t1) and x in double */
            float *xf = sm.t1;
            for (int i = t; i < n; i += NT)
                xf[i] = rs[i];
            __syncthreads();
            wg_trsv1<float, TRI_U>(Ws, n, n, xf, sm.t0);
            double xmax = 0.0;
            for (int i = t; i < n; i += NT) {
                xd[i] = (double)xf[i];
                xmax = fmax(xmax, fabs(xd[i]));
            }
            xmax = wg_max(xmax, red);
            for (int it = 0;; ++it) {
                /* r = b - A x in double (four rows per wave at a time), kept
                 * in float as the next correction's right-hand side */
                double rmax = 0.0;
                {
                    double sum[4] = {0.0, 0.0, 0.0, 0.0};
                    wave_rows4_stream<double>(
                        As, n, ngr, grow, n, 0, n,
                        [&](int, int cb, const double(&v)[4][4]) {
                            double xv[4];
#pragma unroll
                            for (int m = 0; m < 4; ++m) {
                                const int c = cb + 64 * m + l;
                                xv[m] = c < n ? xd[c] : 0.0;
                            }
#pragma unroll
                            for (int u = 0; u < 4; ++u)
#pragma unroll
                                for (int m = 0; m < 4; ++m)
                                    sum[u] = __builtin_fma(v[u][m], xv[m], sum[u]);
                        },
                        [&](int g) {
                            const int i0 = grow(g);
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
#pragma unroll
                                for (int o = 32; o > 0; o >>= 1)
                                    sum[u] += __shfl_xor(sum[u], o);
                                if (i0 + u < n) {
                                    const double r = bs[i0 + u] - sum[u];
                                    rmax = fmax(rmax, fabs(r));
                                    if (l == 0)
                                        xf[i0 + u] = (float)r;
                                }
                                sum[u] = 0.0;
                            }
                        });
                }
                rmax = wg_max(rmax, red);
                if (rmax == 0.0 || rmax <= tol * margin * xmax) {
                    used = it;
                    break;
                }
                if (it == max_iter)
                    break;
                /* d = solve_float(r), x += d */
                wg_trsv1<float, TRI_L>(Ws, n, n, xf, sm.t0);
                wg_trsv1<float, TRI_U>(Ws, n, n, xf, sm.t0);
                xmax = 0.0;
                for (int i = t; i < n; i += NT) {
                    xd[i] += (double)xf[i];
                    xmax = fmax(xmax, fabs(xd[i]));
                }
                xmax = wg_max(xmax, red);
            }
            __syncthreads();
            for (int i = t; i < n; i += NT)
                bs[i] = xd[i];
        } else {
            for (int it = 0; it <= max_iter; ++it) {
                if (it > 0)
                    wg_solve<float, TRI_L, 1>(Ws, n, n, rs, 1, 1, smu.s);
                wg_solve<float, TRI_U, 1>(Ws, n, n, rs, 1, 1, smu.s);
                double xmax = 0.0;
                for (int i = t; i < n; i += NT) {
                    const double x = (it == 0) ? (double)rs[i] : xs[i] + (double)rs[i];
                    xs[i] = x;
                    xmax = fmax(xmax, fabs(x));
                }
                xmax = wg_max(xmax, red);
                __syncthreads();
                /* r = b - A x: wave w takes rows w, w+4, ...; lanes split the row */
                double rmax = 0.0;
                for (int i = w; i < n; i += 4) {
                    double sacc = 0.0;
                    for (int j = l; j < n; j += 64)
                        sacc += As[(int64_t)i * n + j] * xs[j];
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1)
                        sacc += __shfl_xor(sacc, o);
                    const double r = bs[i] - sacc;
                    if (l == 0)
                        rs[i] = (float)r;
                    rmax = fmax(rmax, fabs(r));
                }
                rmax = wg_max(rmax, red);
                if (rmax == 0.0 || rmax <= tol * margin * xmax) {
                    used = it;
                    break;
                }
            }
            __syncthreads();
            for (int i = t; i < n; i += NT)
                bs[i] = xs[i];
        }
        if (t == 0 && iters)
            iters[s] = used;
        __syncthreads();
    }
}

template <typename T>
hipError_t batched_run(int count, const int *ns, const int64_t *offA, T *A, const int64_t *offB, T *B,
                       const int *order, int32_t *info, int *queue, int grid, bool two, hipStream_t st)
{
    hipError_t e = fill_i32(queue, 1, 0, st);
    if (e != hipSuccess)
        return e;
    auto run = two || kCroutPerCu<T> == 2 ? k_batched<T, true> : k_batched<T, kCroutPerCu<T> == 2>;
    hipLaunchKernelGGL(run, dim3(grid), dim3(NT), 0, st, count, ns, offA, A, offB, B, order, info, queue);
    return hipGetLastError();
}

hipError_t batched_mixed_run(int count, const int *ns, const int64_t *offA, const double *A, const int64_t *offB,
                             double *B, const int *order, int32_t *info, int *queue, float *W, float *R32,
                             double *X, int max_iter, double tol, int32_t *iters, int grid, bool two, hipStream_t st)
{
    hipError_t e = fill_i32(queue, 1, 0, st);
    if (e != hipSuccess)
        return e;
    auto run = two ? k_batched_mixed<true> : k_batched_mixed<false>;
    hipLaunchKernelGGL(run, dim3(grid), dim3(NT), 0, st, count, ns, offA, A, offB, B, order, info, queue, W, R32, X,
                       max_iter, tol, iters);
    return hipGetLastError();
}

/* ---------------------------------------------------------------- band --- */

/*
 * Tile (rb, cb) of a band matrix in row-wise band storage (a_ij at
 * AB[i*ldab + j - i + kl] for -kl <= j - i <= ku): element (r, c) is
 * a_{64rb+r, 64cb+c}, held in slot c - r + d0 of storage row 64rb + r with
 * d0 = 64 (cb - rb) + kl.  It exists when that slot lies in 0..kl+ku and its
 * row and column are inside the matrix.  Loads are unconditional (`raw`: the
 * tile's first slot stands in for an element that does not exist, and the
 * user masks with `in`), so that a run of them stays in flight together
 * instead of each waiting behind a branch.
 */
struct BandTile {
    double *base; /* storage row 64 rb */
    int64_t ldab;
    int d0, w, nr, nc;
    __device__ __forceinline__ BandTile(double *AB, int64_t ldab_, int n, int kl, int ku, int rb, int cb)
        : base(AB + (int64_t)rb * TB * ldab_), ldab(ldab_), d0(TB * (cb - rb) + kl), w(kl + ku), nr(n - TB * rb),
          nc(n - TB * cb)
    {
    }
    __device__ __forceinline__ bool in(int r, int c) const
    {
        return (unsigned)(c - r + d0) <= (unsigned)w && r < nr && c < nc;
    }
    __device__ __forceinline__ double *addr(int r, int c) const { return base + (int64_t)r * ldab + (c - r + d0); }
    __device__ __forceinline__ double raw(int r, int c) const { return *(in(r, c) ? addr(r, c) : base); }
    /* accumulator address map (acc64_store): nullptr where no element */
    __device__ __forceinline__ double *operator()(int r, int c) const { return in(r, c) ? addr(r, c) : nullptr; }
};

/*
 * Strip p of the band step's off-diagonal tiles, once strip p of the diagonal
 * tile S (its diagonal blocks' inverses in P) is final: u holds the columns
 * 16w.. of the tile right of S, lt the rows 16wl.. of the tile below it
 * transposed, 16 x 16 blocks down the slab.  Block p of each is finished with
 * the strip's inverse and its contribution removed from the blocks after it,
 * the finished block being the products' B operand.  Blocks p < w of u and
 * p < wl of lt are zero (kl, ku <= 64) and stay so.
 */
__device__ __forceinline__ void band_strip(const double *S, const double *P, int p, int w, int wl,
                                           vec4<double>::type (&u)[4], vec4<double>::type (&lt)[4])
{
    typedef vec4<double>::type V;
    const int c0 = 16 * p;
    auto slab = [&](V(&x)[4], auto &&diag, auto &&off) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if (b == p) {
                V f = {0, 0, 0, 0};
                wave_mma16_acc<double>(f, diag, x[b]);
                x[b] = f;
#pragma unroll
                for (int a = b + 1; a < 4; ++a)
                    wave_mma16_acc<double>(x[a], [&](int r, int k) { return -off(16 * a + r, k); }, x[b]);
            }
    };
    if (p >= w)
        slab(u,
             [&](int r, int k) {
                 const double v = P[(c0 + r) * LDT + c0 + k];
                 return r > k ? v : (r == k ? 1.0 : 0.0);
             },
             [&](int r, int k) { return S[r * LDT + c0 + k]; });
    if (p >= wl)
        slab(lt,
             [&](int r, int k) {
                 const double v = P[(c0 + k) * LDT + c0 + r];
                 return k <= r ? v : 0.0;
             },
             [&](int r, int k) { return S[(c0 + k) * LDT + r]; });
}

/*
 * One lane's column c (or row r) of a BandTile, its rows (columns) counted
 * from the lane's first one, o: which of them exist and where they are, so
 * that an access at a compile-time offset costs one compare and one 64-bit
 * addition of a scalar instead of the tile's general form (whose address
 * arithmetic took a third of a band step's cycles).
 */
struct BandLine {
    double *p0, *any;
    int64_t step;
    int lo;
    unsigned len;
    __device__ __forceinline__ bool in(int x) const { return (unsigned)(x - lo) <= len; }
    __device__ __forceinline__ double *at(int x) const { return p0 + x * step; }
    __device__ __forceinline__ double raw(int x) const { return *(in(x) ? at(x) : any); }
};
__device__ __forceinline__ BandLine band_line(double *p0, double *any, int64_t step, int lo, int hi, int o)
{
    return {p0 + o * step, any, step, hi < lo ? 1 << 30 : lo - o, hi < lo ? 0u : (unsigned)(hi - lo)};
}
__device__ __forceinline__ BandLine band_col(const BandTile &t, int c, int o)
{
    return band_line(t.base + (c + t.d0), t.base, t.ldab - 1, max(0, c + t.d0 - t.w),
                     c < t.nc ? min(t.nr - 1, c + t.d0) : -1, o);
}
__device__ __forceinline__ BandLine band_row(const BandTile &t, int r, int o)
{
    return band_line(t.base + ((int64_t)r * t.ldab - r + t.d0), t.base, 1, max(0, r - t.d0),
                     r < t.nr ? min(t.nc - 1, r - t.d0 + t.w) : -1, o);
}

/* LDS of the band factor: the running diagonal tile, the inverses of its
 * diagonal blocks, and the tile below it for the product with the one to its
 * right. */
struct BandSmem {
    double s[TB * LDT];
    double p[TB * LDT];
    double l[TB * LDT];
    double rinv[TB];
    int zflag;
};

/* One workgroup's share of a band factorization: block rows first .. end - 1,
 * started at block row begin <= first (those before first are computed and
 * dropped).  With pk the tiles are read from there (k_band_pack), else from
 * the band itself; s0 is the first diagonal tile where it is known (64 x 64,
 * else A's); sstart and send receive the diagonal tiles that the factor of
 * block rows first and end starts from (each if not null). */
struct BandRange {
    int begin, first, end;
    const double *pk, *s0;
    double *sstart, *send;
};

/* Tiles per block row in k_band_pack's storage: the diagonal one, the one
 * right of it and the one below it, as a lane of band_range holds them: the
 * 16 values of lane l of wave w in pairs at ((8w + h) 64 + l) 2. */
constexpr int kBandPackTiles = 3;
typedef double d2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void band_pack_load(const double *P, vec4<double>::type (&v)[4])
{
    const d2 *q = reinterpret_cast<const d2 *>(P) + wave_id() * 512 + (threadIdx.x & 63);
#pragma unroll
    for (int h = 0; h < 8; ++h) {
        const d2 x = q[64 * h];
        v[h >> 1][2 * (h & 1)] = x[0];
        v[h >> 1][2 * (h & 1) + 1] = x[1];
    }
}
__device__ __forceinline__ void band_pack_store(double *P, const vec4<double>::type (&v)[4])
{
    d2 *q = reinterpret_cast<d2 *>(P) + wave_id() * 512 + (threadIdx.x & 63);
#pragma unroll
    for (int h = 0; h < 8; ++h)
        q[64 * h] = d2{v[h >> 1][2 * (h & 1)], v[h >> 1][2 * (h & 1) + 1]};
}

/*
 * Band Doolittle LU by one workgroup (see BandRange).  With kl, ku <= 64 the
 * matrix is block tridiagonal in 64 x 64 tiles and, without pivoting, so are
 * its factors: block step k factors the diagonal tile S_k (Eq. 6-a), turns
 * the tile to its right into U_{k,k+1} = L_kk^{-1} A_{k,k+1} and the one below
 * it into L_{k+1,k} = A_{k+1,k} U_kk^{-1}, and takes the next diagonal tile
 * S_{k+1} = A_{k+1,k+1} - L_{k+1,k} U_{k,k+1} (Eq. 6-c) on the matrix cores.
 * The two off-diagonal tiles stay in accumulators, wave w the columns 16w..
 * of U and the rows 16(3 - w).. of L (transposed: U^T L^T = A^T; the lower
 * triangle of the former and the upper of the latter make that an equal
 * share), and are solved strip by strip inside the diagonal tile's
 * factorization (tile_lu64's hook).  Their loads are issued at the top of the
 * step and first used after a strip.  Entries outside the band stay exactly
 * zero and are never stored.  The step is bound by its chain, the tile
 * factorization (18.6k of 40k cycles): 16.8 us from packed tiles, 20.6 us from
 * the band itself (address arithmetic and scattered loads), 26 us before the
 * off-diagonal tiles moved into accumulators.
 */
template <bool PACKED>
__device__ __forceinline__ int band_range(double *AB, int64_t ldab, int n, int kl, int ku, const BandRange &R,
                                          BandSmem &sm)
{
    typedef vec4<double>::type V;
    const int nt = (n + TB - 1) / TB;
    const int w = wave_id(), lane = launder((int)threadIdx.x & 63), lr = lane & 15, lk = lane >> 4;
    const int wl = 3 - w; /* this wave's row slab of L */
    auto tile = [&](int rb, int cb) { return BandTile(AB, ldab, n, kl, ku, rb, cb); };
    auto packed = [&](int kb, int i) { return R.pk + ((int64_t)kb * kBandPackTiles + i) * TB * TB; };
    auto arow = [&](int a, int r) { return 16 * a + acc_row<double>(lk, r); }; /* = lk + 16 a + 4 r */
    int zero_at = 0;
    if (R.s0) {
        tile_xfer<double>([&](int r, int c) { return R.s0[r * TB + c]; },
                          [&](int r, int c, double v) { sm.s[r * LDT + c] = v; });
    } else if (PACKED) {
        V d[4];
        band_pack_load(packed(R.begin, 0), d);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                sm.s[arow(a, r) * LDT + 16 * w + lr] = d[a][r];
    } else {
        const BandTile t0 = tile(R.begin, R.begin);
        tile_xfer<double>(
            [&](int r, int cc) {
                const double v = t0.raw(r, cc);
                return t0.in(r, cc) ? v : (r == cc ? 1.0 : 0.0); /* the identity past the end */
            },
            [&](int r, int cc, double v) { sm.s[r * LDT + cc] = v; });
    }
    __syncthreads();
    auto save_tile = [&](double *G) {
        tile_xfer<double>([&](int r, int c) { return sm.s[r * LDT + c]; },
                          [&](int r, int c, double v) { G[r * TB + c] = v; });
    };
#pragma unroll 1
    for (int kb = R.begin; kb < R.end; ++kb) {
        const bool last = kb + 1 == nt, own = kb >= R.first;
        if (kb == R.first && R.sstart)
            save_tile(R.sstart);
        /* U and the next diagonal tile by columns 16w.., L by rows 16wl..
         * (transposed); from the band unmasked, the mask applied where they
         * are first used */
        const BandLine cu = band_col(tile(kb, kb + 1), 16 * w + lr, lk);
        const BandLine cn = band_col(tile(kb + 1, kb + 1), 16 * w + lr, lk);
        const BandLine rl = band_row(tile(kb + 1, kb), 16 * wl + lr, lk);
        V u[4], lt[4], nx[4];
        if (!last) {
            if (PACKED) {
                band_pack_load(packed(kb, 1), u);
                band_pack_load(packed(kb, 2), lt);
                band_pack_load(packed(kb + 1, 0), nx);
            } else {
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        u[a][r] = cu.raw(16 * a + 4 * r);
                        lt[a][r] = rl.raw(16 * a + 4 * r);
                        nx[a][r] = cn.raw(16 * a + 4 * r);
                    }
            }
        }
        const int z = tile_lu64(sm.s, sm.p, sm.rinv, min(TB, n - kb * TB), &sm.zflag,
                                [&](int p, int stage) __attribute__((always_inline)) {
                                    if (last || stage != 0)
                                        return;
                                    if (!PACKED && p == 0)
#pragma unroll
                                        for (int a = 0; a < 4; ++a)
#pragma unroll
                                            for (int r = 0; r < 4; ++r) {
                                                u[a][r] = cu.in(16 * a + 4 * r) ? u[a][r] : 0.0;
                                                lt[a][r] = rl.in(16 * a + 4 * r) ? lt[a][r] : 0.0;
                                            }
                                    band_strip(sm.s, sm.p, p, w, wl, u, lt);
                                });
        if (own) {
            if (z && !zero_at)
                zero_at = kb * TB + z;
            const BandLine cd = band_col(tile(kb, kb), lane, w);
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (cd.in(4 * i))
                    *cd.at(4 * i) = sm.s[(w + 4 * i) * LDT + lane];
        }
        if (last)
            break;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                sm.l[(16 * wl + lr) * LDT + arow(a, r)] = lt[a][r];
                if (!PACKED)
                    nx[a][r] = cn.in(16 * a + 4 * r) ? nx[a][r] : (arow(a, r) == 16 * w + lr ? 1.0 : 0.0);
            }
        __syncthreads();
        /* L_{k+1,k} (upper) times U_{k,k+1} (lower): inner blocks from
         * max(a, w) */
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q >= w)
#pragma unroll
                for (int a = 0; a <= q; ++a)
                    wave_mma16_acc<double>(nx[a], [&](int r, int k) { return -sm.l[(16 * a + r) * LDT + 16 * q + k]; },
                                           u[q]);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                sm.s[arow(a, r) * LDT + 16 * w + lr] = nx[a][r];
        if (own) {
            const BandLine cl = band_col(tile(kb + 1, kb), lane, w);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if (cu.in(4 * i))
                    *cu.at(4 * i) = u[i >> 2][i & 3];
                if (cl.in(4 * i))
                    *cl.at(4 * i) = sm.l[(w + 4 * i) * LDT + lane];
            }
        }
        __syncthreads();
    }
    if (R.send && R.end < nt)
        save_tile(R.send);
    __syncthreads();
    return zero_at;
}

/* The whole chain by one workgroup: short bands, and callers without the
 * workspace of the segmented form. */
__global__ __launch_bounds__(NT) void k_band_factor(double *AB, int64_t ldab, int n, int kl, int ku, int32_t *info)
{
    __shared__ BandSmem sm;
    const BandRange R{0, 0, (n + TB - 1) / TB, nullptr, nullptr, nullptr, nullptr};
    const int z = band_range<false>(AB, ldab, n, kl, ku, R, sm);
    if (threadIdx.x == 0 && info)
        *info = z;
}

/*
 * The band factor in segments.  The only thing block row k hands to the next
 * is the diagonal tile S_{k+1}, and what S_k was fades quadratically fast: a change
 * D of S_k arrives in S_{k+1} as B S^{-1} D S^{-1} C with B, C the off-diagonal
 * tiles.  So the block rows are split into segments, one workgroup each, and a
 * segment starts kBandWarm block rows early from A's own tile.  How far that fades
 * depends on the values: with 64 + 1 + 64 diagonals of random sign a factor of
 * about 3e-4 (row sum 0.5) to 1e-3 (0.9) per block row, and six rows pass with at
 * most half of what the check allows; off-diagonals of one sign need 9 (0.5) to 24
 * (0.9), a five-point grid 25 and more.  Nothing rests on it: the tile a
 * segment started from is compared with the one its predecessor ended with
 * (k_band_check), element by element against the terms it was formed from, and
 * segments that do not agree are factored again from the true tile, in order
 * (k_band_fix) -- for a matrix that forgets slowly all of them.
 *
 * Segments are four block rows long (longer once that makes more than 256,
 * one per compute unit): at n = 16384 the chain is 10 steps instead of 256.
 * Below 16 block rows the serial chain is as fast (10 steps, and four more
 * launches).  Before that the band is copied as tiles (k_band_pack: the
 * segments' early rows are written by their neighbours, and the chain then
 * loads whole vectors without masks).  n = 16384, 64 + 1 + 64: 0.20 ms (pack 9 us,
 * segments 171, check 11, fix 5) where the starts agree, 5.0 ms where every segment
 * is repaired (one-signed bands, grids), 5.2 ms for the serial chain.
 */
constexpr int kBandWarm = 6;

__device__ __forceinline__ BandRange band_segment(const BandWs &ws, int nt, int m, int j, bool again)
{
    BandRange R;
    R.first = j * m;
    R.end = min(nt, R.first + m);
    R.begin = again ? R.first : max(0, R.first - kBandWarm);
    R.pk = ws.pk;
    R.s0 = again ? ws.send + (int64_t)(j - 1) * TB * TB : nullptr;
    R.sstart = again ? nullptr : ws.sstart + (int64_t)j * TB * TB;
    R.send = ws.send + (int64_t)j * TB * TB;
    return R;
}

__global__ __launch_bounds__(NT) void k_band_pack(double *AB, int64_t ldab, int n, int kl, int ku, double *P)
{
    typedef vec4<double>::type V;
    const int kb = blockIdx.x, nt = (n + TB - 1) / TB;
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4, wl = 3 - w;
    auto tile = [&](int rb, int cb) { return BandTile(AB, ldab, n, kl, ku, rb, cb); };
    const bool last = kb + 1 == nt; /* nothing right of or below the last tile */
    const BandLine cd = band_col(tile(kb, kb), 16 * w + lr, lk);
    const BandLine cu = last ? cd : band_col(tile(kb, kb + 1), 16 * w + lr, lk);
    const BandLine rl = last ? cd : band_row(tile(kb + 1, kb), 16 * wl + lr, lk);
    V d[4], u[4], lt[4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int x = 16 * a + 4 * r;
            d[a][r] = cd.raw(x);
            u[a][r] = cu.raw(x);
            lt[a][r] = rl.raw(x);
        }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int x = 16 * a + 4 * r;
            d[a][r] = cd.in(x) ? d[a][r] : (lk + x == 16 * w + lr ? 1.0 : 0.0); /* the identity past the end */
            u[a][r] = !last && cu.in(x) ? u[a][r] : 0.0;
            lt[a][r] = !last && rl.in(x) ? lt[a][r] : 0.0;
        }
    double *G = P + (int64_t)kb * kBandPackTiles * TB * TB;
    band_pack_store(G, d);
    band_pack_store(G + TB * TB, u);
    band_pack_store(G + 2 * TB * TB, lt);
}

__global__ __launch_bounds__(NT) void k_band_segments(double *AB, int64_t ldab, int n, int kl, int ku, BandWs ws,
                                                      int m)
{
    __shared__ BandSmem sm;
    const int j = blockIdx.x;
    const int z = band_range<true>(AB, ldab, n, kl, ku, band_segment(ws, (n + TB - 1) / TB, m, j, false), sm);
    if (threadIdx.x == 0) {
        ws.zero[j] = z;
        ws.flags[j] = 0;
    }
}

/* What is known of a segment: its start differs from its predecessor's end; by
 * more than rounding; a pivot of it is tiny. */
enum { kBandInexact = 1, kBandOff = 2, kBandTiny = 4 };

/* Whether the diagonal tile t that segment j started from is the one s that its
 * predecessor ended with: each element to 2^-51 of the terms it was formed from,
 * |A| + |L| |U| of the factor's tiles left of and above it, which is what the
 * product's own rounding is measured by.  A row's largest element is no measure:
 * where a row meets columns of two scales, an element of the small scale would
 * pass with none of its digits right.  Returns kBand* flags, the same in every
 * thread; not a number, and a sum that overflows, never agree. */
__device__ __forceinline__ int band_seam(double *AB, int64_t ldab, int n, int kl, int ku, const BandWs &ws, int m,
                                         int j, double *sl, double *su)
{
    typedef vec4<double>::type V;
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4, kb = j * m;
    const BandTile tl(AB, ldab, n, kl, ku, kb, kb - 1), tu(AB, ldab, n, kl, ku, kb - 1, kb);
    auto stage = [&](const BandTile &x, double *D) {
        tile_xfer<double>(
            [&](int r, int c) {
                const double v = x.raw(r, c);
                return x.in(r, c) ? fabs(v) : 0.0;
            },
            [&](int r, int c, double v) { D[r * LDT + c] = v; });
    };
    stage(tl, sl);
    stage(tu, su);
    const double *S = ws.send + (int64_t)(j - 1) * TB * TB, *T = ws.sstart + (int64_t)j * TB * TB;
    V s[4], t[4], bound[4];
    band_pack_load(ws.pk + (int64_t)kb * kBandPackTiles * TB * TB, bound);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = (16 * a + acc_row<double>(lk, r)) * TB + 16 * w + lr;
            s[a][r] = S[e];
            t[a][r] = T[e];
            bound[a][r] = fabs(bound[a][r]);
        }
    __syncthreads();
    bool same = true, exact = true;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        wave_mma16<double, TB>(
            bound[a], [&](int r, int k) { return sl[(16 * a + r) * LDT + k]; },
            [&](int k, int c) { return su[k * LDT + 16 * w + c]; });
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool eq = s[a][r] == t[a][r];
            exact = exact && eq;
            same = same && (eq || (fabs(s[a][r] - t[a][r]) <= 0x1p-51 * bound[a][r] &&
                                   bound[a][r] <= 0x1.fffffffffffffp1023));
        }
    }
    same = __syncthreads_and(same);
    return __syncthreads_and(exact) ? 0 : (same ? kBandInexact : kBandInexact | kBandOff);
}

/* Whether a pivot of block rows b0 .. b1 - 1 is tiny against the terms it was
 * formed from, sum_k |l_ik u_ki| (four threads a pivot), or not a number: it, or
 * one near it, may then be zero but for a start's last bits.  The same in every
 * thread. */
__device__ __forceinline__ bool band_tiny_pivot(const double *AB, int64_t ldab, int n, int kl, int ku, int b0, int b1)
{
    const int q = threadIdx.x & 3, depth = min(kl, ku);
    bool tiny = false;
    for (int b = b0; b < b1; ++b) {
        const int i = b * TB + (threadIdx.x >> 2);
        const double *row = AB + (int64_t)min(i, n - 1) * ldab + kl;
        double sum = 0.0;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int d = 1 + q + 4 * e;
            const bool in = i < n && d <= min(depth, i);
            const double x = *(in ? row - d : row), y = *(in ? row - d * ldab + d : row);
            sum += in ? fabs(x * y) : 0.0;
        }
        sum += __shfl_xor(sum, 1);
        sum += __shfl_xor(sum, 2);
        tiny = tiny || (i < n && !(fabs(*row) > 0x1p-40 * sum));
    }
    return __syncthreads_or(tiny);
}

/* The seams, a workgroup each, and the block rows past the first segment, whose
 * start is exact. */
__global__ __launch_bounds__(NT) void k_band_check(double *AB, int64_t ldab, int n, int kl, int ku, BandWs ws, int m,
                                                   int nseg)
{
    __shared__ double sl[TB * LDT], su[TB * LDT];
    const bool seam = (int)blockIdx.x < nseg - 1;
    const int j = seam ? blockIdx.x + 1 : 0, b = m + (int)blockIdx.x - (nseg - 1);
    const int f = seam ? band_seam(AB, ldab, n, kl, ku, ws, m, j, sl, su)
                       : (band_tiny_pivot(AB, ldab, n, kl, ku, b, b + 1) ? kBandTiny : 0);
    if (threadIdx.x == 0 && f)
        atomicOr(ws.flags + (seam ? j : b / m), f);
}

/* Segments that started wrong are factored again in order.  A kept segment may
 * differ from the chain's in its last bits, which a pivot formed by cancellation
 * shows whole: the chain's exact zero is then a rounding error there.  Where a
 * pivot is tiny, all segments from the first inexact start on are therefore
 * factored again, and the answer is the chain's. */
__global__ __launch_bounds__(NT) void k_band_fix(double *AB, int64_t ldab, int n, int kl, int ku, BandWs ws, int m,
                                                 int nseg, int32_t *info)
{
    __shared__ BandSmem sm;
    __shared__ int first_zero;
    const int nt = (n + TB - 1) / TB;
    bool off = false, tiny = false;
    for (int j = 1 + threadIdx.x; j < nseg; j += NT) {
        off = off || (ws.flags[j] & kBandOff);
        tiny = tiny || (ws.flags[j] & kBandTiny);
    }
    bool strict = __syncthreads_or(tiny);
    for (bool more = __syncthreads_or(off) || strict; more;) {
        bool redone = false, kept = false; /* segment j - 1 was factored again; an inexact start was kept */
        more = false;
        for (int j = 1; j < nseg; ++j) {
            const int f = strict   ? (redone || (ws.flags[j] & kBandInexact) ? kBandOff : 0)
                          : redone ? band_seam(AB, ldab, n, kl, ku, ws, m, j, sm.l, sm.s)
                                   : ws.flags[j];
            redone = f & kBandOff;
            if (!redone) {
                kept = kept || (f & kBandInexact);
                continue;
            }
            const BandRange R = band_segment(ws, nt, m, j, true);
            const int z = band_range<true>(AB, ldab, n, kl, ku, R, sm);
            if (threadIdx.x == 0)
                ws.zero[j] = z;
            if (kept)
                more = band_tiny_pivot(AB, ldab, n, kl, ku, R.first, R.end) || more;
        }
        strict = true; /* once more if a pivot of the new ones is tiny */
    }
    if (threadIdx.x == 0)
        first_zero = 0x7fffffff;
    __syncthreads();
    for (int j = threadIdx.x; j < nseg; j += NT)
        if (ws.zero[j])
            atomicMin(&first_zero, ws.zero[j]);
    __syncthreads();
    if (threadIdx.x == 0 && info)
        *info = first_zero == 0x7fffffff ? 0 : first_zero;
}

/*
 * Operands of the band substitutions (Eq. 1), one workgroup per 64-row block
 * b, kBandSolveTiles 64 x 64 tiles at P + b * 4 * 4096:
 *   0  the inverses of the diagonal tile's factors, packed (tile_inv16),
 *   1  M_b = L_bb^{-1} L_{b,b-1}: forward,  y_b = L_bb^{-1} b_b - M_b y_{b-1},
 *   2  N_b = U_bb^{-1} U_{b,b+1}: backward, x_b = U_bb^{-1} y_b - N_b x_{b+1},
 *   3  room for the segmented sweeps (BandSweep).
 * M and N lie as the matrix cores' left operand (band_pack_load's order: lane
 * (lr, lk) of wave w holds row 16w + lr, columns 16a + acc_row(lk, r)), zero
 * where the band or the matrix has no element.  With the product of the two
 * triangular operators taken here, in parallel, the chain has one 64 x 64
 * product per block instead of two.
 */
constexpr int kBandSolveTiles = 4;

__global__ __launch_bounds__(NT) void k_band_packs(const double *AB, int64_t ldab, int n, int kl, int ku,
                                                   double *__restrict__ P)
{
    typedef vec4<double>::type V;
    __shared__ TileSmem<double> sm;
    const int b = blockIdx.x, nt = (n + TB - 1) / TB;
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    double *AB_ = const_cast<double *>(AB);
    const BandTile t(AB_, ldab, n, kl, ku, b, b);
    tile_xfer<double>(
        [&](int r, int c) {
            const double v = t.raw(r, c);
            return t.in(r, c) ? v : (r == c ? 1.0 : 0.0);
        },
        [&](int r, int c, double v) { sm.t0[r * LDT + c] = v; });
    __syncthreads();
    if (threadIdx.x < TB)
        sm.rinv[threadIdx.x] = recip(sm.t0[threadIdx.x * LDT + threadIdx.x]);
    __syncthreads();
    tile_inv16(sm.t0, sm.rinv, sm.t1);
    double *Pb = P + (int64_t)b * kBandSolveTiles * TB * TB;
    tile_xfer<double>([&](int r, int c) { return sm.t1[r * LDT + c]; },
                      [&](int r, int c, double v) { Pb[r * TB + c] = v; });
    for (int side = 0; side < 2; ++side) {
        const int o = side ? b + 1 : b - 1;
        if (o < 0 || o >= nt)
            continue; /* outside the matrix: never read */
        const BandTile to(AB_, ldab, n, kl, ku, b, o);
        __syncthreads();
        tile_xfer<double>(
            [&](int r, int c) {
                const double v = to.raw(r, c);
                return to.in(r, c) ? v : 0.0;
            },
            [&](int r, int c, double v) { sm.t0[r * LDT + c] = v; });
        __syncthreads();
        Acc64<double> acc;
        acc64_zero(acc);
        auto off = [&](int k, int c) { return sm.t0[k * LDT + c]; };
        if (side)
            acc64_mma<double, false>(acc, InvUFull<double>{sm.t1}, off);
        else
            acc64_mma<double, false>(acc, InvL<double>{sm.t1}, off);
        __syncthreads();
        acc64_store(acc, LdsTile<double>{sm.t0});
        __syncthreads();
        V v[4];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                v[a][r] = sm.t0[(16 * w + lr) * LDT + 16 * a + acc_row<double>(lk, r)];
        band_pack_store(Pb + (1 + side) * TB * TB, v);
    }
}

/*
 * The band substitutions of up to 16 right-hand sides (one chunk of B's
 * columns).  The blocks are taken in positions, 0 the first one solved.  With
 * m < nt block rows the positions are split into segments as the factor's
 * are: a segment starts kBandSweepWarm positions early from zero, which the
 * products M_b (N_b) fade below the last bit where they are small enough (0.05 in
 * norm for random signs at row sum 0.5; one-signed bands of that sum take 18
 * positions, a five-point grid 22); its start is compared with its predecessor's
 * end, component by component (k_band_sweep_check), and it is swept again from
 * there if they disagree (k_band_sweep_fix).  Its
 * own operands are then formed ahead (k_band_z): z_b = L_bb^{-1} b_b, held in
 * tile 3 of the block, whose rest holds the segment's ends and flags.
 * n = 16384, 8 right-hand sides: 40 us a direction and 22 us for the operands,
 * 0.79 ms in all where every segment is swept again, against 1.42 ms for two
 * chains of 256 with two products a block.
 */
struct BandSweep {
    int n;
    double *P, *B;
    int64_t ldb;
    int nrhs, m; /* columns from B on; positions per segment */
};
constexpr int kBandSweepWarm = 16;
constexpr int kBandSweepChunks = 2; /* chunks of right-hand sides side by side (tile 3 has room for two) */

/* A 64 x 16 block of right-hand sides as its waves' accumulators: lane l of
 * wave w holds four values, in pairs at (128 h + 64 w + ...): pair h of them
 * at ((4h + w) 64 + l) 2. */
__device__ __forceinline__ void band_y_store(double *Y, const d4 &y)
{
    d2 *q = reinterpret_cast<d2 *>(Y) + 64 * wave_id() + (threadIdx.x & 63);
    q[0] = d2{y[0], y[1]};
    q[256] = d2{y[2], y[3]};
}
__device__ __forceinline__ d4 band_y_load(const double *Y, int w)
{
    const d2 *q = reinterpret_cast<const d2 *>(Y) + 64 * w + (threadIdx.x & 63);
    const d2 a = q[0], b = q[256];
    return d4{a[0], a[1], b[0], b[1]};
}

/* Places in tile 3: of block b (in solve order position pos) the formed
 * z_b, and of a segment the state it started from and ended with and, in its
 * third position, whether its successor's start agreed. */
__device__ __forceinline__ double *band_room(const BandSweep &a, int b)
{
    return a.P + ((int64_t)b * kBandSolveTiles + 3) * TB * TB;
}
template <bool FWD> __device__ __forceinline__ int band_blk(const BandSweep &a, int pos)
{
    return FWD ? pos : (a.n + TB - 1) / TB - 1 - pos;
}
template <bool FWD> __device__ __forceinline__ double *band_start(const BandSweep &a, int j, int ch)
{
    return band_room(a, band_blk<FWD>(a, j * a.m)) + (2 + ch) * TB * 16;
}
template <bool FWD> __device__ __forceinline__ double *band_end(const BandSweep &a, int j, int ch)
{
    return band_room(a, band_blk<FWD>(a, j * a.m + 1)) + (2 + ch) * TB * 16;
}
template <bool FWD> __device__ __forceinline__ int *band_ok(const BandSweep &a, int j, int ch)
{
    return reinterpret_cast<int *>(band_room(a, band_blk<FWD>(a, j * a.m + 2)) + (2 + ch) * TB * 16);
}

/* z_b = L_bb^{-1} b_b (FWD) or U_bb^{-1} y_b: the left operand, rows 16w + lr
 * of the pack, columns 16q + 4 lk + ks, and the right one from B, columns
 * past the last read as zero. */
struct BandZ {
    double p[16], y[16];
};
__device__ __forceinline__ void band_z_load(const BandSweep &a, int b, int c0, BandZ &o)
{
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const double *Pr = a.P + (int64_t)b * kBandSolveTiles * TB * TB + (16 * w + lr) * TB + 4 * lk;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            o.p[4 * q + ks] = Pr[16 * q + ks];
            const int row = b * TB + 16 * q + 4 * lk + ks;
            o.y[4 * q + ks] = a.B[(int64_t)min(row, a.n - 1) * a.ldb + min(c0 + lr, a.nrhs - 1)];
        }
}
template <bool FWD> __device__ __forceinline__ d4 band_z_product(const BandSweep &a, int b, int c0, const BandZ &o)
{
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4, r = 16 * w + lr;
    d4 z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int k = 16 * q + 4 * lk + ks;
            const double p = o.p[4 * q + ks];
            const double f = FWD ? (r > k ? p : (r == k ? 1.0 : 0.0)) : (r <= k ? p : 0.0);
            z = mfma16(f, (b * TB + k < a.n && c0 + lr < a.nrhs) ? o.y[4 * q + ks] : 0.0, z);
        }
    return z;
}

template <bool FWD> __global__ __launch_bounds__(NT) void k_band_z(BandSweep a)
{
    const int b = blockIdx.x, ch = blockIdx.y;
    BandZ o;
    band_z_load(a, b, 16 * ch, o);
    band_y_store(band_room(a, b) + ch * TB * 16, band_z_product<FWD>(a, b, 16 * ch, o));
}

/* y -= M_b y_prev, y_prev (all four waves') in LDS. */
__device__ __forceinline__ void band_sweep_product(d4 &y, const vec4<double>::type (&M)[4], const double *prev)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const d4 x = band_y_load(prev, q);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            y = mfma16(-M[q][ks], x[ks], y);
    }
}
__device__ __forceinline__ void band_sweep_put(const BandSweep &a, int b, int c0, const d4 &y)
{
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = b * TB + 16 * w + acc_row<double>(lk, r);
        if (row < a.n && c0 + lr < a.nrhs)
            a.B[(int64_t)row * a.ldb + c0 + lr] = y[r];
    }
}

/* Positions begin .. end - 1 of one segment, those from first on written to B;
 * from y0 (the state before begin) or from zero.  One product per position;
 * its operands are loaded two positions ahead in a ring of three register
 * sets.  The state before first goes to start, the last to end_. */
template <bool FWD>
__device__ __forceinline__ void band_sweep_segment(const BandSweep &a, int ch, int begin, int first, int end,
                                                   const double *y0, double *start, double *end_, double (*ybuf)[TB * 16])
{
    struct Ops {
        vec4<double>::type M[4];
        d4 z;
    };
    auto load = [&](int pos, Ops &o) {
        const int b = band_blk<FWD>(a, min(pos, end - 1));
        band_pack_load(a.P + ((int64_t)b * kBandSolveTiles + (FWD ? 1 : 2)) * TB * TB, o.M);
        o.z = band_y_load(band_room(a, b) + ch * TB * 16, wave_id());
    };
    if (y0) {
        band_y_store(ybuf[0], band_y_load(y0, wave_id()));
        __syncthreads();
    }
    int cur = 0;
    auto step = [&](int pos, const Ops &o) __attribute__((always_inline)) {
        d4 y = o.z;
        if (pos > begin || y0)
            band_sweep_product(y, o.M, ybuf[cur]);
        cur ^= 1;
        band_y_store(ybuf[cur], y);
        if (pos >= first)
            band_sweep_put(a, band_blk<FWD>(a, pos), 16 * ch, y);
        if (start && pos == first - 1)
            band_y_store(start, y);
        if (end_ && pos == end - 1)
            band_y_store(end_, y);
        __syncthreads();
    };
    Ops o0, o1, o2;
    load(begin, o0);
    load(begin + 1, o1);
    for (int pos = begin; pos < end; pos += 3) {
        load(pos + 2, o2);
        step(pos, o0);
        if (pos + 1 >= end)
            break;
        load(pos + 3, o0);
        step(pos + 1, o1);
        if (pos + 2 >= end)
            break;
        load(pos + 4, o1);
        step(pos + 2, o2);
    }
}

template <bool FWD> __global__ __launch_bounds__(NT) void k_band_sweep_segments(BandSweep a)
{
    __shared__ double ybuf[2][TB * 16];
    const int j = blockIdx.x, ch = blockIdx.y, nt = (a.n + TB - 1) / TB;
    const int first = j * a.m, end = min(nt, first + a.m);
    band_sweep_segment<FWD>(a, ch, max(0, first - kBandSweepWarm), first, end, nullptr,
                            j > 0 ? band_start<FWD>(a, j, ch) : nullptr, end < nt ? band_end<FWD>(a, j, ch) : nullptr,
                            ybuf);
}

/* Whether the state t that segment j + 1 started from is its predecessor's end
 * s: each component to 2^-51 of the terms it was formed from, |z| + |M| |y_prev|
 * at the predecessor's last position (y_prev stands in B), which is what that
 * product's own rounding is measured by.  The largest value of the block is no
 * measure: y scales with the rows of L (the columns of U), and in a block of two
 * scales a small component's error would pass and reach the next block whole.
 * The same in every thread; not a number, and a sum that overflows, never agree. */
template <bool FWD> __device__ __forceinline__ bool band_same_state(const BandSweep &a, int j, int ch)
{
    typedef vec4<double>::type V;
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const int pos = (j + 1) * a.m - 1, b = band_blk<FWD>(a, pos), prev = band_blk<FWD>(a, pos - 1);
    const d4 s = band_y_load(band_end<FWD>(a, j, ch), w), t = band_y_load(band_start<FWD>(a, j + 1, ch), w);
    d4 bound = band_y_load(band_room(a, b) + ch * TB * 16, w);
    V M[4];
    band_pack_load(a.P + ((int64_t)b * kBandSolveTiles + (FWD ? 1 : 2)) * TB * TB, M);
    const int c = 16 * ch + lr;
    double y[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = prev * TB + 16 * (i >> 2) + acc_row<double>(lk, i & 3);
        const double v = a.B[(int64_t)min(row, a.n - 1) * a.ldb + min(c, a.nrhs - 1)];
        y[i] = row < a.n && c < a.nrhs ? fabs(v) : 0.0;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
        bound[r] = fabs(bound[r]);
#pragma unroll
    for (int i = 0; i < 16; ++i)
        bound = mfma16(fabs(M[i >> 2][i & 3]), y[i], bound);
    bool same = true;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        same = same && (s[r] == t[r] || (fabs(s[r] - t[r]) <= 0x1p-51 * bound[r] && bound[r] <= 0x1.fffffffffffffp1023));
    return __syncthreads_and(same);
}

template <bool FWD> __global__ __launch_bounds__(NT) void k_band_sweep_check(BandSweep a)
{
    const int j = blockIdx.x, ch = blockIdx.y;
    const bool ok = band_same_state<FWD>(a, j, ch);
    if (threadIdx.x == 0)
        *band_ok<FWD>(a, j, ch) = ok;
}

template <bool FWD> __global__ __launch_bounds__(NT) void k_band_sweep_fix(BandSweep a, int nseg)
{
    __shared__ double ybuf[2][TB * 16];
    const int ch = blockIdx.x, nt = (a.n + TB - 1) / TB;
    bool mine = true;
    for (int j = threadIdx.x; j < nseg - 1; j += NT)
        mine = mine && *band_ok<FWD>(a, j, ch);
    if (__syncthreads_and(mine))
        return;
    bool redone = false; /* segment j was swept again */
    for (int j = 0; j < nseg - 1; ++j) {
        const bool ok = redone ? band_same_state<FWD>(a, j, ch) : *band_ok<FWD>(a, j, ch) != 0;
        redone = !ok;
        if (ok)
            continue;
        const int first = (j + 1) * a.m, end = min(nt, first + a.m);
        band_sweep_segment<FWD>(a, ch, first, first, end, band_end<FWD>(a, j, ch), nullptr,
                                end < nt ? band_end<FWD>(a, j + 1, ch) : nullptr, ybuf);
    }
}

/* Both substitutions of a short band by one workgroup per chunk, the diagonal
 * products taken in the chain: one launch, operands loaded a block ahead. */
template <bool FWD> __device__ __forceinline__ void band_sweep_whole(const BandSweep &a, int ch, double (*ybuf)[TB * 16])
{
    const int nt = (a.n + TB - 1) / TB;
    struct Ops {
        vec4<double>::type M[4];
        BandZ z;
    };
    auto load = [&](int pos, Ops &o) {
        const int b = band_blk<FWD>(a, min(pos, nt - 1));
        band_pack_load(a.P + ((int64_t)b * kBandSolveTiles + (FWD ? 1 : 2)) * TB * TB, o.M);
        band_z_load(a, b, 16 * ch, o.z);
    };
    int cur = 0;
    auto step = [&](int pos, const Ops &o) __attribute__((always_inline)) {
        const int b = band_blk<FWD>(a, pos);
        d4 y = band_z_product<FWD>(a, b, 16 * ch, o.z);
        if (pos > 0)
            band_sweep_product(y, o.M, ybuf[cur]);
        cur ^= 1;
        band_y_store(ybuf[cur], y);
        band_sweep_put(a, b, 16 * ch, y);
        __syncthreads();
    };
    Ops o0, o1;
    load(0, o0);
    for (int pos = 0; pos < nt; pos += 2) {
        load(pos + 1, o1);
        step(pos, o0);
        if (pos + 1 >= nt)
            break;
        load(pos + 2, o0);
        step(pos + 1, o1);
    }
}
__global__ __launch_bounds__(NT) void k_band_sweep(BandSweep a)
{
    __shared__ double ybuf[2][TB * 16];
    band_sweep_whole<true>(a, blockIdx.x, ybuf);
    band_sweep_whole<false>(a, blockIdx.x, ybuf);
}

/* Block rows per segment of a band of nt of them: short segments make the
 * chain short, and 256 of them fill the compute units. */
static int band_segment_rows(int nt, int least) { return std::max(least, (nt + 255) / 256); }

BandWs band_ws(void *ws, int64_t n, size_t &bytes)
{
    const int nt = (int)((n + TB - 1) / TB), m = band_segment_rows(nt, 4), nseg = (nt + m - 1) / m;
    BandWs b{};
    bytes = 0;
    if (nt < 16)
        return b;
    const size_t tiles = (2 * sizeof(int) * (size_t)nseg + 255) / 256 * 256, tile = sizeof(double) * TB * TB;
    const size_t pk = tiles + 2 * (size_t)nseg * tile;
    bytes = pk + (size_t)nt * kBandPackTiles * tile;
    if (ws) {
        char *p = static_cast<char *>(ws);
        b.zero = reinterpret_cast<int *>(p);
        b.flags = b.zero + nseg;
        b.sstart = reinterpret_cast<double *>(p + tiles);
        b.send = reinterpret_cast<double *>(p + tiles + (size_t)nseg * tile);
        b.pk = reinterpret_cast<double *>(p + pk);
    }
    return b;
}

hipError_t band_factor(double *AB, int64_t ldab, int n, int kl, int ku, int32_t *info, void *ws, hipStream_t st)
{
    size_t bytes = 0;
    const BandWs b = band_ws(ws, n, bytes);
    if (!ws || bytes == 0) {
        hipLaunchKernelGGL(k_band_factor, dim3(1), dim3(NT), 0, st, AB, ldab, n, kl, ku, info);
        return hipGetLastError();
    }
    const int nt = (n + TB - 1) / TB, m = band_segment_rows(nt, 4), nseg = (nt + m - 1) / m;
    hipLaunchKernelGGL(k_band_pack, dim3(nt), dim3(NT), 0, st, AB, ldab, n, kl, ku, b.pk);
    hipLaunchKernelGGL(k_band_segments, dim3(nseg), dim3(NT), 0, st, AB, ldab, n, kl, ku, b, m);
    hipLaunchKernelGGL(k_band_check, dim3(nseg - 1 + nt - m), dim3(NT), 0, st, AB, ldab, n, kl, ku, b, m, nseg);
    hipLaunchKernelGGL(k_band_fix, dim3(1), dim3(NT), 0, st, AB, ldab, n, kl, ku, b, m, nseg, info);
    return hipGetLastError();
}

template <bool FWD> static void band_sweep_launch(const BandSweep &a, int nt, int nch, hipStream_t st)
{
    const int nseg = (nt + a.m - 1) / a.m;
    hipLaunchKernelGGL((k_band_z<FWD>), dim3(nt, nch), dim3(NT), 0, st, a);
    hipLaunchKernelGGL((k_band_sweep_segments<FWD>), dim3(nseg, nch), dim3(NT), 0, st, a);
    hipLaunchKernelGGL((k_band_sweep_check<FWD>), dim3(nseg - 1, nch), dim3(NT), 0, st, a);
    hipLaunchKernelGGL((k_band_sweep_fix<FWD>), dim3(nch), dim3(NT), 0, st, a, nseg);
}

hipError_t band_solve(const double *AB, int64_t ldab, int n, int kl, int ku, double *B, int64_t ldb, int nrhs,
                      double *P, hipStream_t st)
{
    const int nt = (n + TB - 1) / TB;
    hipLaunchKernelGGL(k_band_packs, dim3(nt), dim3(NT), 0, st, AB, ldab, n, kl, ku, P);
    hipError_t e = hipGetLastError();
    /* segments from 48 block rows on: their 24 positions and four launches a
     * direction against a chain of nt in one launch for both */
    const bool seg = nt >= 48;
    const int step = 16 * (seg ? kBandSweepChunks : 65535);
    for (int c0 = 0; c0 < nrhs && e == hipSuccess; c0 += step) {
        const int nc = min(step, nrhs - c0), nch = (nc + 15) / 16;
        const BandSweep a{n, P, B + c0, ldb, nc, band_segment_rows(nt, 8)};
        if (seg) {
            band_sweep_launch<true>(a, nt, nch, st);
            band_sweep_launch<false>(a, nt, nch, st);
        } else {
            hipLaunchKernelGGL(k_band_sweep, dim3(nch), dim3(NT), 0, st, a);
        }
        e = hipGetLastError();
    }
    return e;
}

/* ---------------------------------------------------- explicit inverse --- */

/* Inverse packs of every 64 x 64 diagonal tile of a factored system (one
 * workgroup per tile, all independent): tile_inv16 of the factored tile,
 * stored 64 x 64 (pitch 64) at P + b * 4096 -- the inverse of its unit lower
 * factor in the strict lower part, the inverse of its upper factor in the
 * upper part. */
template <typename T>
__global__ __launch_bounds__(NT) void k_diag_packs(const T *__restrict__ LU, int64_t lda, int n, T *__restrict__ P)
{
    __shared__ TileSmem<T> sm;
    const int b = blockIdx.x, k0 = b * TB, kw = min(TB, n - k0);
    stage_tile_identity(sm.t0, LU + (int64_t)k0 * lda + k0, lda, kw, kw);
    __syncthreads();
    if (threadIdx.x < TB)
        sm.rinv[threadIdx.x] = recip(sm.t0[threadIdx.x * LDT + threadIdx.x]);
    __syncthreads();
    tile_inv16(sm.t0, sm.rinv, sm.t1);
    T *Pb = P + (int64_t)b * TB * TB;
    tile_xfer<T>([&](int r, int c) { return sm.t1[r * LDT + c]; }, [&](int r, int c, T v) { Pb[r * TB + c] = v; });
}

/*
 * Explicit inverse X = A^{-1} = U^{-1} L^{-1} from the factors (Eq. 4-c: the
 * elementary upper factors times the elementary lower factors), as two
 * right-looking blocked triangular solves on the identity, one launch per
 * 64-wide block step, one workgroup per 64 x 64 tile of the result.  A tile
 * takes the terms of G steps at a time, so that it is read and written once per
 * G steps and its product is G times as deep:
 *   forward, W = L^{-1} (block lower triangular): launch k takes the rows r =
 *     k+1, k+1+G, ... and subtracts L_rs W_sc of the steps s = k-G+1 .. k
 *     (those >= c: W_sc is zero before; a tile first touched here starts from
 *     zero); row k + 1 then has its last term and is multiplied by
 *     L_{k+1,k+1}^{-1} at once; one more workgroup writes the diagonal tile
 *     W_{k+1,k+1} = L_{k+1,k+1}^{-1};
 *   backward, X = U^{-1} W (dense): launch k takes the rows r = k-1, k-1-G,
 *     ... and subtracts U_rs X_sc of the steps s = k .. k+G-1 (fewer at the
 *     first launches); the tiles above W's diagonal start from zero at their
 *     first update; row k - 1 has then received every term and is multiplied
 *     by U_{k-1,k-1}^{-1}.
 * W is kept in X's storage and overwritten in place.  The inverses of the
 * diagonal tiles come from their packs (k_diag_packs), read as the products'
 * left operand straight from memory.
 * What bounds it is the product's rate and, where a launch has fewer tiles
 * than the chip holds, one tile's own length.  n = 4096, forward | backward
 * launches on average: one step a tile, operands streamed without LDS, 26 | 58
 * us, two steps backward 26 | 54, tile_gemm and four steps 17 | 29.
 *
 * G: a launch of a few tiles lasts as long as one tile, whose product one step
 * keeps short; a launch that fills the chip gains by the tiles' reads and writes
 * saved.  One | two | four steps, us, FP64 n = 1000 324 | 357 | 438, 2000 841 | 814
 * | 934, 3000 1864 | 1669 | 1766, 4000 3331 | 2981 | 2860; FP32 1000 312 | 366 |
 * 472, 2000 709 | 792 | 996, 4000 2281 | 2164 | 2393, 6000 5918 | 5135 | 5443, 7000
 * (two | four) 7700 | 7650, 8000 9590 | 9140.
 */
constexpr int kInvOne = 2048;                                       /* largest n for one step, */
template <typename T> constexpr int kInvTwo = sizeof(T) == 8 ? 3072 : 6144; /* for two */

template <typename T, bool FWD, int NB, int G>
__global__ __launch_bounds__(NT, 3) void k_inv_step(const T *__restrict__ LU, int64_t lda, int n,
                                                    const T *__restrict__ P, T *__restrict__ X, int64_t ldx, int k)
{
    typedef typename vec4<T>::type V;
    constexpr int H = 2 / NB; /* H workgroups per 64 x 64 tile */
    __shared__ __attribute__((aligned(16))) char lds_raw[std::max(TileGemm<T, 2, NB>::LDS, sizeof(T) * TB * LDT)];
    T *S = reinterpret_cast<T *>(lds_raw);
    const int nt = (n + TB - 1) / TB, b = blockIdx.x / H, h0 = blockIdx.x % H * 32;
    int r, c, s0, K; /* the tile, the first step of its terms and their inner length */
    bool fresh;
    if (FWD) {
        const int cols = k + 1, nupd = (nt - 1 - k + G - 1) / G * cols;
        if (b >= nupd) { /* W_{k+1,k+1} = L_{k+1,k+1}^{-1} */
            const int d0 = (k + 1) * TB, nd = min(TB, n - d0);
            const T *Pr = P + (int64_t)(k + 1) * TB * TB;
            T *C = X + (int64_t)d0 * ldx + d0;
            tile_xfer<T>(
                [&](int rr, int cc) {
                    const T v = Pr[rr * TB + cc];
                    return rr > cc ? v : (rr == cc ? T(1) : T(0));
                },
                [&](int rr, int cc, T v) {
                    if (rr < nd && cc < nd && (H == 1 || cc >> 5 == h0 >> 5))
                        C[(int64_t)rr * ldx + cc] = v;
                });
            return;
        }
        r = k + 1 + G * (b / cols);
        c = b % cols;
        s0 = max(c, k + 1 - G);
        K = (k + 1 - s0) * TB;
        fresh = c > k - G;
    } else if (k == nt) { /* the last block row: no terms */
        r = nt - 1;
        c = b;
        s0 = K = 0;
        fresh = false;
    } else {
        r = k - 1 - G * (b / nt);
        c = b % nt;
        s0 = k;
        K = min(G * TB, n - k * TB);
        fresh = r < c && k + G >= nt;
    }
    const int nr = min(TB, n - r * TB), nc = min(32 * NB, n - c * TB - h0);
    if (nc <= 0)
        return;
    T *C = X + (int64_t)r * TB * ldx + (int64_t)c * TB + h0;
    const T *Ap = LU + (int64_t)r * TB * lda + (int64_t)s0 * TB, *Bp = X + (int64_t)s0 * TB * ldx + (int64_t)c * TB + h0;
    V acc[2][NB];
    if (fresh) {
        for_tile<T, NB>([&](int bi, int bj, int rr, int, int) { acc[bi][bj][rr] = T(0); });
        tile_minus<T, NB, true>(acc, Ap, lda, nr, Bp, ldx, nc, K, lds_raw);
    } else {
        tile_pending<T, NB, true>(acc, C, ldx, Ap, lda, nr, Bp, ldx, nc, K, lds_raw);
    }
    if (r != (FWD ? k + 1 : k - 1)) {
        tile_store<T, NB>(acc, C, ldx, nr, nc);
        return;
    }
    /* the row is complete: times its diagonal tile's inverse, the triangle's
     * zero half of inner indices left out */
    __syncthreads();
    tile_to_lds<T, NB>(acc, S, nr, nc, false);
    const T *Pr = P + (int64_t)r * TB * TB;
    const int w = wave_id(), l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const int wm = (w >> 1) * 32, wn = (w & 1) * 16 * NB;
    V x[2][NB];
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < NB; ++bj)
            x[bi][bj] = V{0, 0, 0, 0};
    __syncthreads();
#pragma unroll 1
    for (int kc = FWD ? 0 : wm; kc < (FWD ? wm + 32 : TB); kc += 32) {
        T a[2][8];
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
                a[bi][ks] = Pr[(wm + 16 * bi + lr) * TB + kc + 4 * ks + lk];
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const int kk = kc + 4 * ks + lk;
#pragma unroll
            for (int bi = 0; bi < 2; ++bi) {
                const int rr = wm + 16 * bi + lr;
                const T av = FWD ? (rr > kk ? a[bi][ks] : (rr == kk ? T(1) : T(0))) : (rr <= kk ? a[bi][ks] : T(0));
#pragma unroll
                for (int bj = 0; bj < NB; ++bj)
                    x[bi][bj] = mfma16(av, S[kk * LDT + wn + 16 * bj + lr], x[bi][bj]);
            }
        }
    }
    tile_store<T, NB>(x, C, ldx, nr, nc);
}

template <typename T, bool FWD, int G>
static hipError_t inv_step(int tiles, const T *LU, int64_t lda, int n, const T *P, T *X, int64_t ldx, int k,
                           hipStream_t st)
{
    /* up to 384 tiles: halves of 32 columns, which fill the chip's 768 places
     * once and finish in half the time; more: whole tiles, half the operand
     * traffic (n = 4096: 264 tiles 21 -> 18 us, 1024 tiles 43 us) */
    if (tiles <= 384)
        hipLaunchKernelGGL((k_inv_step<T, FWD, 1, G>), dim3(2 * tiles), dim3(NT), 0, st, LU, lda, n, P, X, ldx, k);
    else
        hipLaunchKernelGGL((k_inv_step<T, FWD, 2, G>), dim3(tiles), dim3(NT), 0, st, LU, lda, n, P, X, ldx, k);
    return hipGetLastError();
}

template <typename T, int G>
static hipError_t inv_steps(const T *LU, int64_t lda, int n, T *X, int64_t ldx, const T *P, hipStream_t st)
{
    const int nt = (n + TB - 1) / TB;
    hipError_t e = hipSuccess;
    for (int k = -1; k + 1 < nt && e == hipSuccess; ++k) /* rows k+1, k+1+G, ... and the diagonal tile */
        e = inv_step<T, true, G>((nt - 1 - k + G - 1) / G * (k + 1) + 1, LU, lda, n, P, X, ldx, k, st);
    for (int k = nt; k > 0 && e == hipSuccess; --k) /* rows k-1, k-1-G, ... */
        e = inv_step<T, false, G>(k == nt ? nt : (k + G - 1) / G * nt, LU, lda, n, P, X, ldx, k, st);
    return e;
}

template <typename T>
hipError_t lu_inverse(const T *LU, int64_t lda, int n, T *X, int64_t ldx, T *P, hipStream_t st)
{
    const int nt = (n + TB - 1) / TB;
    hipLaunchKernelGGL(k_diag_packs<T>, dim3(nt), dim3(NT), 0, st, LU, lda, n, P);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess)
        e = n <= kInvOne      ? inv_steps<T, 1>(LU, lda, n, X, ldx, P, st)
            : n <= kInvTwo<T> ? inv_steps<T, 2>(LU, lda, n, X, ldx, P, st)
                              : inv_steps<T, 4>(LU, lda, n, X, ldx, P, st);
    return e;
}

/* ------------------------------------------------------- skyline (profile) --- */

/* Tile (I, J) of the block envelope (nullptr outside it). */
__device__ __forceinline__ double *sky_tile(const SkyPlan &pl, double *tiles, int I, int J)
{
    if (J <= I)
        return J >= pl.F(I) ? tiles + (int64_t)(pl.LTo(I) + J - pl.F(I)) * TB * TB : nullptr;
    return I >= pl.G(J) ? tiles + (int64_t)(pl.LTo(pl.nt) + pl.UTo(J) + I - pl.G(J)) * TB * TB : nullptr;
}

/* Pack (or unpack) the skyline arrays and the envelope tiles: workgroup b < nt
 * takes the lower tiles of block row b (lanes over columns: a row of L is
 * contiguous), b >= nt the upper tiles of block column b - nt (lanes over
 * rows: a column of U is contiguous).  Elements outside the element envelope
 * or past n are zero in the tiles and never written back. */
__global__ __launch_bounds__(NT) void k_sky_pack(SkyPlan pl, const int32_t *__restrict__ f,
                                                 const int64_t *__restrict__ rp, double *__restrict__ AL,
                                                 const int32_t *__restrict__ g, const int64_t *__restrict__ cp,
                                                 double *__restrict__ AU, double *__restrict__ tiles, int unpack)
{
    const int b = blockIdx.x, n = pl.n, lane = threadIdx.x & 63, r4 = threadIdx.x >> 6;
    const bool lower = b < pl.nt;
    const int I0 = lower ? b : pl.G(b - pl.nt), I1 = lower ? b : b - pl.nt - 1;
    const int J0 = lower ? pl.F(b) : b - pl.nt, J1 = lower ? b : b - pl.nt;
    for (int I = I0; I <= I1; ++I)
        for (int J = J0; J <= J1; ++J) {
            double *T = sky_tile(pl, tiles, I, J);
            for (int k = r4; k < TB; k += 4) {
                /* lower tiles: row r = k, column c = lane; upper: column c = k, row r = lane */
                const int r = lower ? k : lane, c = lower ? lane : k;
                const int i = I * TB + r, j = J * TB + c;
                double *p = nullptr;
                if (i < n && j < n) {
                    if (j < i)
                        p = j >= f[i] ? AL + rp[i] + (j - f[i]) : nullptr;
                    else
                        p = i >= g[j] ? AU + cp[j] + (i - g[j]) : nullptr;
                }
                if (unpack) {
                    if (p)
                        *p = T[r * TB + c];
                } else {
                    T[r * TB + c] = p ? *p : 0.0;
                }
            }
        }
}

/* The cnt-th of the indices x >= from, x < nt, with X(x) <= lim, or -1. */
template <typename X> __device__ __forceinline__ int sky_nth(X &&first, int from, int nt, int lim, int cnt)
{
    /* 64 entries per round, one per lane (a scan entry by entry waits for each
     * load), the hit picked from the wave's ballot; every wave gets the same */
    const int lane = threadIdx.x & 63;
    for (int base = from; base < nt; base += 64) {
        const int x = base + lane;
        const int v = first(min(x, nt - 1));
        const unsigned long long m = __ballot(x < nt && v <= lim);
        const int c = __popcll(m);
        if (cnt < c) {
            unsigned long long mm = m;
            for (int i = 0; i < cnt; ++i)
                mm &= mm - 1;
            return base + __ffsll((long long)mm) - 1;
        }
        cnt -= c;
    }
    return -1;
}

/* Skyline LU on the envelope tiles as a dataflow (above), restricted to the
 * envelope, which the elimination keeps: if L_Ik and U_kK exist, so does tile
 * (I, K).  Tiles outside stay zero and are never touched.  ctl: the status word
 * and the ticket.  A block's flags lie behind its diagonal blocks' inverses,
 * each in a cache line of its own: side by side in the
 * control words the polls for all of them met in a few lines (18.2 -> 21.7 us a
 * block). */
struct SkyOrder {
    int32_t first[kSkyMaxBlocks + 1]; /* first ticket of each step */
};
struct SkyFlow {
    const SkyPlan &pl;
    double *tiles, *P;
    int *ctl;
    long limit;
    __device__ __forceinline__ double *tile(int I, int J) const { return sky_tile(pl, tiles, I, J); }
    static constexpr bool joined = false;
    __device__ __forceinline__ static constexpr int ld(int) { return TB; }
    __device__ __forceinline__ static bool next(int J, int I) { return I == J + 1; }
    __device__ __forceinline__ static void guard(int) {}
    __device__ __forceinline__ int rows(int) const { return TB; } /* zero-padded */
    __device__ __forceinline__ int valid(int I) const { return min(TB, pl.n - I * TB); }
    __device__ __forceinline__ int first(int I, int K) const { return max(pl.F(I), pl.G(K)); }
    __device__ __forceinline__ bool has_l(int I, int J) const { return pl.F(I) <= J; }
    __device__ __forceinline__ bool has_u(int J, int K) const { return pl.G(K) <= J; }
    __device__ __forceinline__ int lcount(int I, int J) const { return J - pl.F(I); }
    __device__ __forceinline__ int ucount(int K, int J) const { return J - pl.G(K); }
    __device__ __forceinline__ bool publish(int J) const { return order_n > 1; }
    __device__ __forceinline__ int *status() const { return ctl; }
    __device__ __forceinline__ int *lflag(int I) const { return reinterpret_cast<int *>(pack(I) + TB * 16 + 16); }
    __device__ __forceinline__ int *uflag(int K) const { return reinterpret_cast<int *>(pack(K) + TB * 16 + 32); }
    __device__ __forceinline__ double *pack(int J) const { return P + (int64_t)J * TB * TB; }
    __device__ __forceinline__ int *dflag(int J) const { return reinterpret_cast<int *>(pack(J) + TB * 16); }
    int order_n; /* tiles of this workgroup's step */
};
__global__ __launch_bounds__(NT) void k_sky_clear(SkyPlan pl, double *P, int *ctl, int32_t *info)
{
    for (int i = threadIdx.x; i < kCtlHead + 2 * pl.nt; i += NT)
        ctl[i] = 0;
    for (int b = threadIdx.x; b < pl.nt; b += NT) {
        double *flags = P + (int64_t)b * TB * TB + TB * 16;
        flags[0] = flags[16] = flags[32] = 0.0;
    }
    if (threadIdx.x == 0 && info)
        *info = 0;
}
__global__ __launch_bounds__(NTP, 2) void k_sky_factor(SkyPlan pl, SkyOrder ord, double *tiles, double *P,
                                                               int *ctl, int32_t *info, long wlim)
{
    __shared__ FlowSmem<double> sm;
    if (threadIdx.x == 0) {
        sm.ticket = atomicAdd(ctl + 1, 1);
        sm.seen[0] = sm.seen[1] = sm.seen[2] = 0;
    }
    __syncthreads();
    const int nt = pl.nt, q0 = __builtin_amdgcn_readfirstlane(sm.ticket);
    if (q0 >= ord.first[nt]) { /* counter not reset: refuse */
        if (threadIdx.x == 0)
            atomicOr(ctl, 2);
        return;
    }
    int J = 0; /* the step: the last with first[J] <= q0 */
    for (int step = kSkyMaxBlocks / 2; step; step >>= 1)
        if (J + step < nt && ord.first[J + step] <= q0)
            J += step;
    const int q = q0 - ord.first[J];
    const SkyFlow f{pl, tiles, P, ctl, wlim, ord.first[J + 1] - ord.first[J]};
    if (q == 0) {
        __builtin_amdgcn_s_setprio(3); /* the chain, ahead of its compute unit's other waves */
        flow_diagonal<double>(f, J, info, sm);
        return;
    }
    if (threadIdx.x >= NT)
        return;
    int I = sky_nth([&](int x) { return pl.F(x); }, J + 1, nt, J, q - 1);
    if (I >= 0) {
        if (I == J + 1)
            __builtin_amdgcn_s_setprio(2);
        flow_panel<double, true>(f, J, I, sm);
        return;
    }
    int nl = 0;
    for (int base = J + 1; base < nt; base += 64) {
        const int x = base + (threadIdx.x & 63);
        nl += __popcll(__ballot(x < nt && pl.F(min(x, nt - 1)) <= J));
    }
    I = sky_nth([&](int x) { return pl.G(x); }, J + 1, nt, J, q - 1 - nl);
    if (I < 0)
        return;
    if (I == J + 1)
        __builtin_amdgcn_s_setprio(2);
    flow_panel<double, false>(f, J, I, sm);
}

hipError_t skyline_factor(const SkyPlan &pl, double *tiles, double *P, int *ctl, int32_t *info, long wlim,
                          hipStream_t st)
{
    SkyOrder ord;
    ord.first[0] = 0;
    for (int J = 0; J < pl.nt; ++J) {
        int c = 1;
        for (int I = J + 1; I < pl.nt; ++I)
            c += (pl.F(I) <= J) + (pl.G(I) <= J);
        ord.first[J + 1] = ord.first[J] + c;
    }
    hipLaunchKernelGGL(k_sky_clear, dim3(1), dim3(NT), 0, st, pl, P, ctl, info);
    hipLaunchKernelGGL(k_sky_factor, dim3(ord.first[pl.nt]), dim3(NTP), 0, st, pl, ord, tiles, P, ctl, info, wlim);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && info)
        e = fold_status(ctl, info, st);
    return e;
}

/* Inverse packs of the skyline factor's diagonal tiles, one workgroup per
 * tile (all independent): P + b * 4096 (pitch 64) receives L_bb^{-1} in its
 * strict lower part (unit diagonal implied) and U_bb^{-1} in its upper part;
 * a partial last tile is padded with the identity.  The diagonal tile is not
 * needed any more then (a solve packs its own copy of the factors): its
 * storage becomes the block's exchange rows of k_sky_trsv, marked unsolved
 * here for the first chunk of right-hand sides, and the control words are
 * cleared. */
__device__ __forceinline__ void sky_mark(double *T)
{
    unsigned long long *x = reinterpret_cast<unsigned long long *>(T);
    for (int i = threadIdx.x; i < TB * TB; i += NT)
        x[i] = kUnsolvedMark64;
}
__device__ __forceinline__ void sky_ctl_clear(int *ctl, bool all)
{
    if (blockIdx.x == 0 && threadIdx.x < kSkyCtl && (all || threadIdx.x > 0))
        ctl[threadIdx.x] = 0;
}
__global__ __launch_bounds__(NT) void k_sky_packs(SkyPlan pl, double *__restrict__ tiles, double *__restrict__ P,
                                                  int *ctl)
{
    __shared__ TileSmem<double> sm;
    const int b = blockIdx.x, kb = min(TB, pl.n - b * TB);
    double *D = sky_tile(pl, tiles, b, b);
    stage_tile_identity(sm.t0, D, TB, kb, kb);
    __syncthreads();
    sky_mark(D);
    sky_ctl_clear(ctl, true);
    if (threadIdx.x < TB)
        sm.rinv[threadIdx.x] = recip(sm.t0[threadIdx.x * LDT + threadIdx.x]);
    __syncthreads();
    tile_inv16(sm.t0, sm.rinv, sm.t1);
    double *Pb = P + (int64_t)b * TB * TB;
    tile_xfer<double>([&](int r, int c) { return sm.t1[r * LDT + c]; },
                      [&](int r, int c, double v) { Pb[r * TB + c] = v; });
}
/* The same marks and words for a further chunk. */
__global__ __launch_bounds__(NT) void k_sky_marks(SkyPlan pl, double *__restrict__ tiles, int *ctl)
{
    sky_mark(sky_tile(pl, tiles, blockIdx.x, blockIdx.x));
    sky_ctl_clear(ctl, false);
}

/*
 * Skyline substitution (Eq. 1) of up to 16 right-hand sides in one launch,
 * FWD: L Y = B (block order 0, 1, ...), else U X = Y (block order nt-1, ...),
 * chained like the dense one (k_trsv): workgroups take tickets in solve order,
 * per block one helper and the block's own; solved blocks and the helpers'
 * partial sums travel through marked exchange rows.  A block depends on the
 * envelope tiles of its own row: forward J = F .. blk-1, backward the J > blk
 * whose columns reach it, oldest first.  All but the last three are shared
 * with the helper and read through the caches once the solved-blocks counter
 * has passed them; the last three are polled, and the last two, as D^{-1} M_j
 * formed while waiting, cost one product in registers each as they arrive:
 *   y = D^{-1} (b - sum_j M_j y_j) - W_1 y_1 - W_2 y_2.
 * Operand tiles are read as the matrix cores' left operand, four contiguous
 * inner indices a lane.  What bounds it is the chain of blocks: 560 us a
 * direction at n = 16384, 2.2 us a block; one launch per block and direction,
 * its updates spread over as many workgroups as the block column has tiles,
 * took 2.9 ms (11.3 us a block).
 */
template <bool FWD>
__global__ __launch_bounds__(NT) void k_sky_trsv(SkyPlan pl, double *__restrict__ tiles, const double *__restrict__ P,
                                                 double *__restrict__ B, int64_t ldb, int nrhs_here, int *ctl, long wlim)
{
    constexpr int ROLES = 2; /* the helper, then the block's own */
    __shared__ TileSmem<double> sm;
    __shared__ double wls[2][16][NT]; /* -W of the last two blocks, operand order per thread */
    __shared__ int16_t dl[kSkyMaxBlocks];
    int *status = ctl, *ctr = ctl + (FWD ? 1 : 3), *solved = ctr + 1;
    const int n = pl.n, nt = pl.nt;
    if (threadIdx.x == 0) {
        sm.ticket = atomicAdd(ctr, 1);
        sm.avail = 0;
    }
    __syncthreads();
    if (sm.ticket >= ROLES * nt) { /* counter not reset: refuse rather than index out of range */
        if (threadIdx.x == 0)
            atomicOr(status, 2);
        return;
    }
    const int pos = __builtin_amdgcn_readfirstlane(sm.ticket / ROLES), role = sm.ticket % ROLES;
    const int blk = FWD ? pos : nt - 1 - pos;
    const int t = threadIdx.x, w = wave_id(), l = t & 63, lr = l & 15, lk = l >> 4;
    const int r0 = blk * TB, nr = min(TB, n - r0);
    /* dependencies, oldest first */
    int nd = 0;
    if (FWD) {
        nd = blk - pl.F(blk);
        for (int d = t; d < nd; d += NT)
            dl[d] = (int16_t)(pl.F(blk) + d);
    } else {
        for (int base = blk + 1 + (nt - blk - 2) / 64 * 64; base > blk; base -= 64) {
            const int J = base + l;
            const bool dep = J < nt && pl.G(min(J, nt - 1)) <= blk;
            const unsigned long long m = __ballot(dep);
            if (w == 0 && dep)
                dl[nd + __popcll(m & ~((2ull << l) - 1))] = (int16_t)J;
            nd += __popcll(m);
        }
    }
    __syncthreads();
    auto dep_blk = [&](int d) { return __builtin_amdgcn_readfirstlane((int)dl[d]); };
    auto dep_pos = [&](int bj) { return FWD ? bj : nt - 1 - bj; };
    /* exchange rows of block b (64 x 16), then the helper's partial sums */
    auto rows = [&](int b) { return sky_tile(pl, tiles, b, b) + (FWD ? 0 : 2 * TB * 16); };
    auto load_a = [&](int bj, double(&a)[16]) {
        const double *T = sky_tile(pl, tiles, blk, bj) + (16 * w + lr) * TB + 4 * lk;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const d4 v = *reinterpret_cast<const d4 *>(T + 16 * q);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                a[4 * q + ks] = v[ks];
        }
    };
    auto row_of = [&](int i) { return 16 * (i >> 2) + 4 * lk + (i & 3); }; /* inner index of operand value i */
    auto fetch_y = [&](int bj, double(&y)[16]) {
        const double *X = rows(bj);
#pragma unroll
        for (int i = 0; i < 16; ++i)
            y[i] = load_coherent(X + row_of(i) * 16 + lr);
    };
    auto fetch_y_cached = [&](int bj, double(&y)[16]) {
        const double *X = rows(bj);
#pragma unroll
        for (int i = 0; i < 16; ++i)
            y[i] = X[row_of(i) * 16 + lr];
    };
    auto has_mark = [&](const double(&y)[16]) {
        bool miss = false;
#pragma unroll
        for (int i = 0; i < 16; ++i)
            miss = miss || is_unsolved_mark(y[i]);
        return miss;
    };
    auto load_y = [&](int bj, double(&y)[16]) {
        for (long spins = 0;; ++spins) {
            fetch_y(bj, y);
            if (!__any(has_mark(y)))
                break;
            if (wait_give_up(status, spins, wlim))
                break;
            __builtin_amdgcn_s_sleep(1);
        }
    };
    const int K = nd - 2;  /* dependencies before the last two */
    const int KP = K - 1;  /* ... of which those taken in passes; the next one is polled */
    d4 acc = {0, 0, 0, 0}, acc2 = {0, 0, 0, 0};
    auto pass = [&](int d, const double(&cur)[16], double(&nxt)[16], d4 &ac) __attribute__((always_inline)) {
        const int bd = dep_blk(d);
        wait_solved(solved, dep_pos(bd), &sm.avail, status, wlim);
        double y[16];
        fetch_y_cached(bd, y);
        __builtin_amdgcn_sched_barrier(0);
        load_a(dep_blk(min(d + ROLES, KP - 1)), nxt);
        __builtin_amdgcn_sched_barrier(0);
        if (__any(has_mark(y)))
            load_y(bd, y);
#pragma unroll
        for (int i = 0; i < 16; ++i)
            ac = mfma16(cur[i], y[i], ac);
    };
    auto passes = [&]() __attribute__((always_inline)) {
        if (role < KP) {
            double a0[16], a1[16];
            load_a(dep_blk(role), a0);
            for (int d = role; d < KP; d += 2 * ROLES) {
                pass(d, a0, a1, acc);
                if (d + ROLES < KP)
                    pass(d + ROLES, a1, a0, acc2);
            }
        }
    };
    double *PB = rows(blk) + TB * 16 + 4 * t; /* the helper's sums, accumulator layout */
    if (role == 0) {
        if (KP <= 0)
            return; /* nothing to share: the block's own does not wait for it */
        passes();
#pragma unroll
        for (int r = 0; r < 4; ++r)
            store_coherent(PB + r, acc[r] + acc2[r]);
        return;
    }
    d4 rhs;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * w + acc_row<double>(lk, r);
        rhs[r] = (row < nr && lr < nrhs_here) ? B[(int64_t)(r0 + row) * ldb + lr] : 0.0;
    }
    /* the diagonal tile's inverse, operand order */
    double dA[16];
    {
        const double *Pb = P + (int64_t)blk * TB * TB + (16 * w + lr) * TB;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = 16 * w + lr, k = row_of(i);
            const double v = Pb[k];
            dA[i] = FWD ? (r > k ? v : (r == k ? 1.0 : 0.0)) : (r <= k ? v : 0.0);
        }
    }
    auto form_w = [&](int bj, int slot) {
        const double *T = sky_tile(pl, tiles, blk, bj);
        tile_xfer<double>([&](int r, int c) { return T[r * TB + c]; },
                          [&](int r, int c, double v) { sm.t0[r * LDT + c] = v; });
        __syncthreads();
        d4 wacc[4];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            wacc[cb] = d4{0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < 16; ++i)
                wacc[cb] = mfma16(dA[i], sm.t0[row_of(i) * LDT + 16 * cb + lr], wacc[cb]);
        }
        __syncthreads();
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                sm.t0[(16 * w + acc_row<double>(lk, r)) * LDT + 16 * cb + lr] = wacc[cb][r];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16; ++i)
            wls[slot][i][t] = -sm.t0[(16 * w + lr) * LDT + row_of(i)];
        __syncthreads();
    };
    if (nd >= 1)
        form_w(dep_blk(nd - 1), 0);
    if (nd >= 2)
        form_w(dep_blk(nd - 2), 1);
    if (K > 0) {
        double al[16], y[16];
        load_a(dep_blk(K - 1), al);
        passes();
        load_y(dep_blk(K - 1), y);
#pragma unroll
        for (int i = 0; i < 16; ++i)
            acc = mfma16(al[i], y[i], acc);
        if (KP > 0) { /* the helper's sums, re-read until none is the mark */
            double pv[4];
            for (long spins = 0;; ++spins) {
                bool miss = false;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    pv[r] = load_coherent(PB + r);
                    miss = miss || is_unsolved_mark(pv[r]);
                }
                if (!__any(miss))
                    break;
                if (wait_give_up(status, spins, wlim))
                    break;
                __builtin_amdgcn_s_sleep(1);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc[r] += pv[r];
        }
    }
    /* z = D^{-1} (b - acc) through LDS, then the last two blocks, polled, into
     * their own accumulator so that neither waits for z */
    double *Rl = sm.t0; /* 64 x 16, pitch 17 */
#pragma unroll
    for (int r = 0; r < 4; ++r)
        Rl[(16 * w + acc_row<double>(lk, r)) * 17 + lr] = rhs[r] - (acc[r] + acc2[r]);
    __syncthreads();
    d4 x = {0, 0, 0, 0}, xw = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 16; ++i)
        x = mfma16(dA[i], Rl[row_of(i) * 17 + lr], x);
#pragma unroll
    for (int slot = 1; slot >= 0; --slot)
        if (nd >= slot + 1) {
            double wa[16], y[16];
#pragma unroll
            for (int i = 0; i < 16; ++i)
                wa[i] = wls[slot][i][t];
            load_y(dep_blk(nd - 1 - slot), y);
#pragma unroll
            for (int i = 0; i < 16; ++i)
                xw = mfma16(wa[i], y[i], xw);
        }
    /* all 64 rows and 16 columns of the exchange block are written (zeros
     * outside the system), the solution rows also to B */
    double *X = rows(blk);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * w + acc_row<double>(lk, r);
        const bool ok = row < nr && lr < nrhs_here;
        const double v = x[r] + xw[r];
        store_coherent(X + row * 16 + lr, ok ? v : 0.0);
        if (ok)
            B[(int64_t)(r0 + row) * ldb + lr] = v;
    }
    __syncthreads();
    if (t == 0)
        __hip_atomic_fetch_max(solved, pos + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

hipError_t skyline_pack(const SkyPlan &pl, const int32_t *f, const int64_t *rp, double *AL, const int32_t *g,
                        const int64_t *cp, double *AU, double *tiles, bool unpack, hipStream_t st)
{
    hipLaunchKernelGGL(k_sky_pack, dim3(2 * pl.nt), dim3(NT), 0, st, pl, f, rp, AL, g, cp, AU, tiles, unpack ? 1 : 0);
    return hipGetLastError();
}

hipError_t skyline_solve(const SkyPlan &pl, double *tiles, double *P, int *ctl, double *B, int64_t ldb, int nrhs,
                         long wlim, hipStream_t st)
{
    hipLaunchKernelGGL(k_sky_packs, dim3(pl.nt), dim3(NT), 0, st, pl, tiles, P, ctl);
    hipError_t e = hipGetLastError();
    for (int c0 = 0; c0 < nrhs && e == hipSuccess; c0 += 16) {
        const int nh = min(16, nrhs - c0);
        if (c0 > 0)
            hipLaunchKernelGGL(k_sky_marks, dim3(pl.nt), dim3(NT), 0, st, pl, tiles, ctl);
        hipLaunchKernelGGL(k_sky_trsv<true>, dim3(2 * pl.nt), dim3(NT), 0, st, pl, tiles, P, B + c0, ldb, nh, ctl, wlim);
        hipLaunchKernelGGL(k_sky_trsv<false>, dim3(2 * pl.nt), dim3(NT), 0, st, pl, tiles, P, B + c0, ldb, nh, ctl, wlim);
        e = hipGetLastError();
    }
    return e;
}

/* ------------------------------------------------------------- adjoint --- */

/* Abar = -Bbar X^T for each system: coalesced row-major writes of the n x n
 * result; with one right-hand side each thread keeps its columns of x in
 * registers, otherwise the n x nrhs factors are read through the cache. */
template <typename T>
__global__ __launch_bounds__(NT) void k_outer_neg(int n, int nrhs, const T *__restrict__ Bb, int64_t ldb, int64_t strideB,
                                                  const T *__restrict__ X, int64_t ldx, int64_t strideX, T *__restrict__ Abar,
                                                  int64_t ldabar, int64_t strideAbar)
{
    const int sys = blockIdx.y;
    const T *bb = Bb + (int64_t)sys * strideB;
    const T *x = X + (int64_t)sys * strideX;
    T *ab = Abar + (int64_t)sys * strideAbar;
    if (nrhs == 1) {
        /* x in registers, 4 * NT columns at a time, for all the rows of the
         * workgroup: x is read once per workgroup rather than once per row
         * (the stream of writes evicts it from L2) */
        for (int j0 = 0; j0 < n; j0 += 4 * NT) {
            T xv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                xv[u] = x[(int64_t)min(j0 + u * NT + (int)threadIdx.x, n - 1) * ldx];
            for (int i = blockIdx.x; i < n; i += gridDim.x) {
                const T bi = bb[(int64_t)i * ldb];
                T *row = ab + (int64_t)i * ldabar;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = j0 + u * NT + threadIdx.x;
                    if (j < n)
                        row[j] = -(bi * xv[u]);
                }
            }
        }
        return;
    }
    for (int i = blockIdx.x; i < n; i += gridDim.x)
        for (int j = threadIdx.x; j < n; j += NT) {
            T s = T(0);
            for (int c = 0; c < nrhs; ++c)
                s += bb[(int64_t)i * ldb + c] * x[(int64_t)j * ldx + c];
            ab[(int64_t)i * ldabar + j] = -s;
        }
}

template <typename T>
hipError_t outer_neg(int n, int nrhs, const T *Bb, int64_t ldb, int64_t strideB, const T *X, int64_t ldx,
                     int64_t strideX, T *Abar, int64_t ldabar, int64_t strideAbar, int64_t batch, hipStream_t st)
{
    for (int64_t b0 = 0; b0 < batch; b0 += 65535) {
        const int nb = (int)std::min<int64_t>(65535, batch - b0);
        const int gx = (int)std::min<int64_t>(n, std::max<int64_t>(1, 4096 / nb));
        hipLaunchKernelGGL(k_outer_neg<T>, dim3(gx, nb), dim3(NT), 0, st, n, nrhs, Bb + b0 * strideB, ldb, strideB,
                           X + b0 * strideX, ldx, strideX, Abar + b0 * strideAbar, ldabar, strideAbar);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

/* ----------------------------------------------------- mixed precision --- */

template <typename TI, typename TO>
__global__ void k_convert(int rows, int cols, const TI *__restrict__ S, int64_t lds, TO *__restrict__ D, int64_t ldd,
                          const int *skip)
{
    if (skip && *skip)
        return;
    const int64_t total = (int64_t)rows * cols;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e / cols, j = e % cols;
        D[i * ldd + j] = (TO)S[i * lds + j];
    }
}

template <typename TI, typename TO>
hipError_t convert(int rows, int cols, const TI *S, int64_t lds, TO *D, int64_t ldd, const int *skip, hipStream_t st)
{
    const int64_t total = (int64_t)rows * cols;
    if (total <= 0)
        return hipSuccess;
    const int grid = (int)std::min<int64_t>((total + 255) / 256, 8192);
    hipLaunchKernelGGL((k_convert<TI, TO>), dim3(grid), dim3(256), 0, st, rows, cols, S, lds, D, ldd, skip);
    return hipGetLastError();
}

/* The larger of two magnitudes, a NaN above all (as their bits compare). */
__device__ __forceinline__ double max_nan(double a, double b)
{
    return (unsigned long long)__double_as_longlong(a) < (unsigned long long)__double_as_longlong(b) ? b : a;
}

/* float(A) and the dominance margin, one wave per row: lanes split the row,
 * convert it and sum |a_ij| off the diagonal; the row's margin
 * |a_ii| - sum, clamped at 0, goes into *mbits by atomic minimum. */
__global__ __launch_bounds__(NT) void k_convert_margin(int n, const double *__restrict__ A, int64_t lda,
                                                       float *__restrict__ D, int64_t ldd, unsigned long long *mbits)
{
    const int l = threadIdx.x & 63;
    const int w = blockIdx.x * (NT / 64) + wave_id(), nw = gridDim.x * (NT / 64);
    double mloc = __longlong_as_double(0x7FF0000000000000ll);
    for (int i = w; i < n; i += nw) {
        const double *a = A + (int64_t)i * lda;
        float *d = D + (int64_t)i * ldd;
        double off = 0.0, dg = 0.0;
        for (int j = l; j < n; j += 64) {
            const double v = a[j];
            d[j] = (float)v;
            if (j == i)
                dg = fabs(v);
            else
                off += fabs(v);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            off += __shfl_xor(off, o);
            dg += __shfl_xor(dg, o);
        }
        mloc = fmin(mloc, fmax(dg - off, 0.0));
    }
    if (l == 0)
        atomicMin(mbits, (unsigned long long)__double_as_longlong(mloc));
}

/* R = float(B - A X) for NR <= 8 columns, the right-hand sides of the next
 * correction; max |r_ic| (in double) into bits[c].  RR rows per workgroup, a
 * thread every 256th column of them, so that X is read once per RR rows: one
 * row per workgroup read four times as many bytes of X, from L2, as of A
 * (n = 16384, 4 columns: 1.46 ms; A alone at the copy's rate 0.45 ms).  Two
 * columns' loads are issued before either is used. */
template <int NR, int RR>
__global__ __launch_bounds__(NT) void k_residual(int n, int nrhs, const double *__restrict__ A, int64_t lda,
                                                 const double *__restrict__ B, int64_t ldb, const double *__restrict__ X,
                                                 int64_t ldx, float *__restrict__ R, int64_t ldr,
                                                 unsigned long long *bits, const int *skip)
{
    if (skip && *skip)
        return;
    __shared__ double red[4][RR][NR];
    const int t = threadIdx.x, i0 = blockIdx.x * RR;
    double acc[RR][NR];
#pragma unroll
    for (int u = 0; u < RR; ++u)
#pragma unroll
        for (int c = 0; c < NR; ++c)
            acc[u][c] = 0.0;
    /* rows past the last one read it again */
    const double *ai[RR];
#pragma unroll
    for (int u = 0; u < RR; ++u)
        ai[u] = A + (int64_t)min(i0 + u, n - 1) * lda;
    auto load = [&](int j, double(&a)[RR], double(&x)[NR]) __attribute__((always_inline)) {
        const int jc = min(j, n - 1);
#pragma unroll
        for (int u = 0; u < RR; ++u)
            a[u] = ai[u][jc];
#pragma unroll
        for (int c = 0; c < NR; ++c)
            x[c] = X[(int64_t)jc * ldx + min(c, nrhs - 1)];
    };
    auto add = [&](int j, const double(&a)[RR], const double(&x)[NR]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < RR; ++u) {
            const double v = j < n ? a[u] : 0.0;
#pragma unroll
            for (int c = 0; c < NR; ++c)
                acc[u][c] = __builtin_fma(v, x[c], acc[u][c]);
        }
    };
    for (int j = t; j < n; j += 2 * NT) {
        double a0[RR], a1[RR], x0[NR], x1[NR];
        load(j, a0, x0);
        load(j + NT, a1, x1);
        add(j, a0, x0);
        add(j + NT, a1, x1);
    }
#pragma unroll
    for (int u = 0; u < RR; ++u)
#pragma unroll
        for (int c = 0; c < NR; ++c) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1)
                acc[u][c] += __shfl_xor(acc[u][c], o);
            if ((t & 63) == 0)
                red[t >> 6][u][c] = acc[u][c];
        }
    __syncthreads();
    if (t < NR && t < nrhs) {
        double m = 0.0;
        for (int u = 0; u < RR && i0 + u < n; ++u) {
            const double r = B[(int64_t)(i0 + u) * ldb + t] - ((red[0][u][t] + red[1][u][t]) + (red[2][u][t] + red[3][u][t]));
            R[(int64_t)(i0 + u) * ldr + t] = (float)r;
            m = max_nan(m, fabs(r));
        }
        atomicMax(bits + t, (unsigned long long)__double_as_longlong(m));
    }
}

/* Stopping test after refinement step `it` (single thread).  With margin
 * m = min_i (|a_ii| - sum_{j != i} |a_ij|) > 0 the inverse is bounded,
 * ||A^{-1}||_inf <= 1/m, so the forward error of column c is at most
 * ||r_c||_inf / m; relative to the solution, ||r_c|| / (m ||x_c||). */
__device__ __forceinline__ void mixed_test(int nrhs, unsigned long long *rbits, unsigned long long *xbits,
                                           const unsigned long long *mbits, double tol, int it, int32_t *iters,
                                           double *ferr, int *conv)
{
    const double m = __longlong_as_double((long long)*mbits);
    bool all = true;
    for (int c = 0; c < nrhs; ++c) {
        const double r = __longlong_as_double((long long)rbits[c]);
        const double x = __longlong_as_double((long long)xbits[c]);
        const double den = m * x;
        const double bound = r == 0.0 ? 0.0 : (den > 0.0 ? r / den : __longlong_as_double(0x7FF0000000000000ll));
        if (ferr)
            ferr[c] = bound;
        if (bound <= tol) {
            if (iters && iters[c] < 0)
                iters[c] = it;
        } else {
            all = false;
        }
        rbits[c] = 0ull;
        xbits[c] = 0ull;
    }
    if (all)
        *conv = 1;
}

/* The test, and (nctl > 0) the start of the next correction's forward
 * substitution: its counters cleared and its exchange rows marked, in the one
 * launch.  Workgroups that do not see the test's outcome yet mark rows that
 * nobody reads. */
__global__ void k_check(int nrhs, unsigned long long *rbits, unsigned long long *xbits,
                        const unsigned long long *mbits, double tol, int it, int32_t *iters, double *ferr, int *conv,
                        int *ctl, int nctl, unsigned int *xb, int64_t nxb)
{
    if (*conv)
        return;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = i0; i < nctl; i += step)
        ctl[i] = 0;
    for (int64_t i = i0; i < nxb; i += step)
        xb[i] = kUnsolvedMark32;
    if (i0 == 0)
        mixed_test(nrhs, rbits, xbits, mbits, tol, it, iters, ferr, conv);
}

/* Start of a mixed-precision solve: status, control words, info, the stopping
 * test's state and the first forward substitution's exchange rows. */
__global__ void k_mixed_init(int *ctl, int nctl, int32_t *info, int *conv, unsigned long long *mbits,
                             unsigned long long *rbits, unsigned long long *xbits, int32_t *iters, int nrhs,
                             unsigned int *xb, int64_t nxb)
{
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = i0; i < nctl; i += step)
        ctl[i] = 0;
    for (int64_t i = i0; i < nxb; i += step)
        xb[i] = kUnsolvedMark32;
    for (int64_t c = i0; c < nrhs; c += step) {
        rbits[c] = xbits[c] = 0ull;
        if (iters)
            iters[c] = -1;
    }
    if (i0 == 0) {
        *conv = 0;
        *mbits = 0x7FF0000000000000ull; /* +inf */
        if (info)
            *info = 0;
    }
}

/* X (+)= D for the mixed-precision update; max |x_ic| of the result into
 * xbits[c], one atomic per wave and column (one per element, all to the same
 * words, took 180 us for 65536 of them). */
__global__ void k_xupdate(int n, int nrhs, double *__restrict__ X, int64_t ldx, const float *__restrict__ D,
                          int64_t ldd, int first, unsigned long long *xbits, const int *skip)
{
    if (skip && *skip)
        return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int c = 0; c < nrhs; ++c) {
        double m = 0.0;
        if (i < n) {
            const double d = (double)D[i * ldd + c];
            const double x = first ? d : X[i * ldx + c] + d;
            X[i * ldx + c] = x;
            m = fabs(x);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
            m = max_nan(m, __shfl_xor(m, o));
        if ((threadIdx.x & 63) == 0)
            atomicMax(xbits + c, (unsigned long long)__double_as_longlong(m));
    }
}

hipError_t convert_margin(int n, const double *A, int64_t lda, float *D, int64_t ldd, unsigned long long *mbits,
                          hipStream_t st)
{
    const int grid = std::max(1, std::min((n + 3) / 4, 4096));
    hipLaunchKernelGGL(k_convert_margin, dim3(grid), dim3(NT), 0, st, n, A, lda, D, ldd, mbits);
    return hipGetLastError();
}

template <int NR, int RR>
static void residual_launch(int n, int nh, const double *A, int64_t lda, const double *B, int64_t ldb, const double *X,
                            int64_t ldx, float *R, int64_t ldr, unsigned long long *bits, const int *skip, hipStream_t st)
{
    hipLaunchKernelGGL((k_residual<NR, RR>), dim3((n + RR - 1) / RR), dim3(NT), 0, st, n, nh, A, lda, B, ldb, X, ldx, R,
                       ldr, bits, skip);
}
hipError_t mixed_residual(int n, int nrhs, const double *A, int64_t lda, const double *B, int64_t ldb, const double *X,
                          int64_t ldx, float *R, int64_t ldr, unsigned long long *bits, const int *skip, hipStream_t st)
{
    hipError_t e = hipSuccess;
    for (int c0 = 0; c0 < nrhs && e == hipSuccess; c0 += 8) {
        const int nh = min(8, nrhs - c0);
        auto run = nh == 1 ? residual_launch<1, 8> : nh <= 4 ? residual_launch<4, 8> : residual_launch<8, 4>;
        run(n, nh, A, lda, B + c0, ldb, X + c0, ldx, R + c0, ldr, bits + c0, skip, st);
        e = hipGetLastError();
    }
    return e;
}

static int mark_grid(int64_t nxb) { return (int)std::min<int64_t>((nxb + 255) / 256 + 1, 1024); }
/* Exchange rows of `chunks` chunks, and the control words ahead of them. */
static int64_t mixed_marks(int n, int chunks) { return (int64_t)chunks * (kTrsvHelpers + 1) * ((n + TB - 1) / TB) * TB * 16; }

hipError_t mixed_init(int n, int nrhs, int *ctl, int32_t *info, int *conv, unsigned long long *mbits,
                      unsigned long long *rbits, unsigned long long *xbits, int32_t *iters, float *xb, hipStream_t st)
{
    const int64_t nxb = mixed_marks(n, 1);
    hipLaunchKernelGGL(k_mixed_init, dim3(mark_grid(nxb)), dim3(256), 0, st, ctl, factor_words<float>(n), info, conv,
                       mbits, rbits, xbits, iters, nrhs, reinterpret_cast<unsigned int *>(xb), nxb);
    return hipGetLastError();
}

hipError_t mixed_check(int n, int nrhs, unsigned long long *rbits, unsigned long long *xbits,
                       const unsigned long long *mbits, double tol, int it, int32_t *iters, double *ferr, int *conv,
                       int *ctl, float *xb, int chunks, bool last, hipStream_t st)
{
    const int nch = last ? 0 : min(chunks, (nrhs + 15) / 16);
    const int64_t nxb = mixed_marks(n, nch);
    hipLaunchKernelGGL(k_check, dim3(mark_grid(nxb)), dim3(256), 0, st, nrhs, rbits, xbits, mbits, tol, it, iters, ferr,
                       conv, ctl + 1, last ? 0 : 1 + nch, reinterpret_cast<unsigned int *>(xb), nxb);
    return hipGetLastError();
}

hipError_t mixed_xupdate(int n, int nrhs, double *X, int64_t ldx, const float *D, int64_t ldd, int first,
                         unsigned long long *xbits, const int *skip, hipStream_t st)
{
    hipLaunchKernelGGL(k_xupdate, dim3((n + 255) / 256), dim3(256), 0, st, n, nrhs, X, ldx, D, ldd, first, xbits, skip);
    return hipGetLastError();
}

/* ------------------------------------------------ explicit instances --- */

template hipError_t dense_factor<double>(double *, int64_t, int, int32_t *, void *, const DenseTuning &, UpdateProfile *,
                                        hipStream_t, double *, int64_t, int, bool);
template hipError_t dense_factor<float>(float *, int64_t, int, int32_t *, void *, const DenseTuning &, UpdateProfile *,
                                       hipStream_t, float *, int64_t, int, bool);
template hipError_t factor_solve<double>(double *, int64_t, int, int32_t *, void *, int, const DenseTuning &, UpdateProfile *,
                                         hipStream_t, double *, int64_t, int);
template hipError_t factor_solve<float>(float *, int64_t, int, int32_t *, void *, int, const DenseTuning &, UpdateProfile *,
                                        hipStream_t, float *, int64_t, int);
template hipError_t dense_trsv<double>(int, const double *, int64_t, int, double *, int64_t, int, int *, double *, int,
                                       const int *, int32_t *, hipStream_t, TrsvStart, long long);
template hipError_t dense_trsv<float>(int, const float *, int64_t, int, float *, int64_t, int, int *, float *, int,
                                      const int *, int32_t *, hipStream_t, TrsvStart, long long);
template hipError_t batch_factor<double>(double *, int64_t, int, int64_t, int64_t, int32_t *, hipStream_t);
template hipError_t batch_factor<float>(float *, int64_t, int, int64_t, int64_t, int32_t *, hipStream_t);
template hipError_t batch_solve<double>(bool, const double *, int64_t, int, int64_t, double *, int64_t, int64_t, int, int64_t, hipStream_t);
template hipError_t batch_solve<float>(bool, const float *, int64_t, int, int64_t, float *, int64_t, int64_t, int, int64_t, hipStream_t);
template hipError_t batched_run<double>(int, const int *, const int64_t *, double *, const int64_t *, double *, const int *, int32_t *, int *, int, bool, hipStream_t);
template hipError_t batched_run<float>(int, const int *, const int64_t *, float *, const int64_t *, float *, const int *, int32_t *, int *, int, bool, hipStream_t);
template hipError_t lu_inverse<double>(const double *, int64_t, int, double *, int64_t, double *, hipStream_t);
template hipError_t lu_inverse<float>(const float *, int64_t, int, float *, int64_t, float *, hipStream_t);
template hipError_t outer_neg<double>(int, int, const double *, int64_t, int64_t, const double *, int64_t, int64_t, double *, int64_t, int64_t, int64_t, hipStream_t);
template hipError_t outer_neg<float>(int, int, const float *, int64_t, int64_t, const float *, int64_t, int64_t, float *, int64_t, int64_t, int64_t, hipStream_t);
template hipError_t convert<double, float>(int, int, const double *, int64_t, float *, int64_t, const int *, hipStream_t);

} /* namespace ebv */
