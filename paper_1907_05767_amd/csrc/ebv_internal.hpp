/* Launchers shared between the kernels (ebv_kernels.hip) and the C ABI (ebv_api.cpp). */
#ifndef EBV_INTERNAL_HPP
#define EBV_INTERNAL_HPP

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include <vector>

namespace ebv {

/* Event brackets around the block-step launches of the single-system
 * factor (owned by a library handle): created up front, one pair per launch
 * up to their number, with each launch's algorithmic flop count. */
struct UpdateProfile {
    std::vector<hipEvent_t> ev;
    std::vector<double> flops;
    int used = 0;
};
int profile_update_enable(UpdateProfile &p, int max_launches);
int profile_update_read(UpdateProfile &p, double *ms_total, int64_t *launches, double *flops_total);

struct DenseTuning {
    int small_update_below; /* trailing size at or below which 64-row update tiles are used */
    int lookahead;          /* 1: one launch (k_flow), or one per block step (k_step); 0: panel + update launches */
    int defer_group;        /* block steps: column classes G; a class is updated every G-th step (1..4) */
    int defer_above;        /* ... while the region past the panel is larger than this */
    long long wait_limit;   /* spins before a bounded wait gives up (0: the defaults) */
    int defer_group_f32;    /* defer_group of the FP32 factor (1..4) */
};

/* Control words at the head of every multi-workgroup workspace: the status
 * word (bounded waits that give up OR 1 into it, a launch that finds its
 * ticket counter not reset ORs 2), then the triangular solve's ticket and
 * solved-blocks counters. */
constexpr int kCtlHead = 3;

/* Systems factored by a single workgroup (uniform and ragged batches) are
 * addressed with 32-bit byte offsets: n * lda * sizeof(element) must stay
 * below this. */
constexpr int64_t kWgMaxSystemBytes = int64_t(1) << 31;

/* Workspace of the single-system factor: first the control words -- the
 * kCtlHead words above, then per block step s the words kCtlHead + 2s
 * (ticket counter) and kCtlHead + 1 + 2s (the diagonal tile's ready flag)
 * -- then the factored diagonal tile's pack for the panel solves (64 x 64
 * elements).  The one-launch factor uses the same bytes for its own words,
 * flags and packs (DenseFlow). */
constexpr size_t factor_ctl_bytes(int64_t n)
{
    const int64_t nb = (n + 63) / 64;
    return (sizeof(int) * (size_t)(kCtlHead + 2 * nb) + 255) / 256 * 256;
}
constexpr size_t factor_pg_bytes(size_t elem) { return (64 * 64 * elem + 255) / 256 * 256; }
constexpr size_t factor_ws_bytes(size_t elem, int64_t n) { return factor_ctl_bytes(n) + factor_pg_bytes(elem); }

/* Exchange buffer of the multi-workgroup triangular solve: the solved rows
 * (n rounded up to 64, 16 columns), then the partial sums of the helper
 * workgroups (kTrsvHelpers per 64-row block, 64 x 16 each). */
constexpr int kTrsvHelpers = 2;
constexpr size_t trsv_xb_bytes(size_t elem, int64_t n)
{
    const int64_t nb = (n + 63) / 64;
    return ((size_t)(kTrsvHelpers + 1) * nb * 64 * 16 * elem + 255) / 256 * 256;
}
/* Chunks of 16 right-hand sides solved side by side: what a workspace is sized
 * for (four chains of n = 4096 and three workgroups a block put 768 workgroups
 * on 256 compute units; more would only queue). */
constexpr int kTrsvChunks = 4;
constexpr int trsv_chunks(int64_t nrhs)
{
    return nrhs <= 16 ? 1 : (int)((nrhs + 15) / 16 < kTrsvChunks ? (nrhs + 15) / 16 : kTrsvChunks);
}

/* Explicit inverse from the factors: P receives the inverse packs of the
 * diagonal tiles (ceil(n/64) * 64 * 64 elements), X (n x n, pitch ldx) the
 * inverse. */
template <typename T>
hipError_t lu_inverse(const T *LU, int64_t lda, int n, T *X, int64_t ldx, T *P, hipStream_t st);

/* Block envelope of a skyline (profile) system, at 64 x 64 tile granularity:
 * block row I holds its lower tiles J = F(I) .. I (the diagonal tile last),
 * block column J its upper tiles I = G(J) .. J-1, packed 64 x 64 (pitch 64)
 * at tile indices LTo(I) + (J - F(I)) and LTo(nt) + UTo(J) + (I - G(J)) of
 * the tile array.  Passed to the kernels by value, two values to a word: byte
 * and half-word arrays are read through vector memory, and the compiler has
 * split the address of a word beside them into a base and an offset that are
 * not multiples of four, which scalar loads round down one by one. */
constexpr int kSkyMaxBlocks = 256; /* n <= 16384; tile indices fit 16 bits */
struct SkyPlan {
    int n, nt;
    uint32_t fg[kSkyMaxBlocks], to[kSkyMaxBlocks + 1];
    __host__ __device__ int F(int b) const { return (int)(fg[b] & 0xFFFF); }
    __host__ __device__ int G(int b) const { return (int)(fg[b] >> 16); }
    __host__ __device__ int LTo(int b) const { return (int)(to[b] & 0xFFFF); }
    __host__ __device__ int UTo(int b) const { return (int)(to[b] >> 16); }
};
/* Pack the skyline arrays into the tiles (unpack = false) or the tiles back
 * into them (only entries inside the envelope are written). */
hipError_t skyline_pack(const SkyPlan &pl, const int32_t *f, const int64_t *rp, double *AL, const int32_t *g,
                        const int64_t *cp, double *AU, double *tiles, bool unpack, hipStream_t st);
/* P: 64 x 64 doubles per block (inverses of the diagonal blocks, flags); ctl:
 * kCtlHead ints (all cleared here); wlim: spins before a bounded wait gives up
 * (its status then lands in info as -status). */
hipError_t skyline_factor(const SkyPlan &pl, double *tiles, double *P, int *ctl, int32_t *info, long wlim,
                          hipStream_t st);
/* tiles: the packed factors, their diagonal tiles overwritten; P: an inverse
 * pack per diagonal tile (nt of them); ctl: kSkyCtl ints (status, then a ticket
 * and a solved-blocks counter per direction; cleared here); wlim: spins before
 * a bounded wait gives up (the results then hold not-a-numbers). */
constexpr int kSkyCtl = 5;
hipError_t skyline_solve(const SkyPlan &pl, double *tiles, double *P, int *ctl, double *B, int64_t ldb, int nrhs,
                         long wlim, hipStream_t st);

hipError_t fill_i32(int *p, int64_t count, int value, hipStream_t st);
/* info = -status when the workspace's status word is nonzero (one thread). */
hipError_t fold_status(const int *status, int32_t *info, hipStream_t st);

/* Single-system factor; prefilled: info, the control words and the flags
 * behind them were cleared by the caller on the same stream. */
template <typename T>
hipError_t dense_factor(T *A, int64_t lda, int n, int32_t *info, void *ws, const DenseTuning &tun, UpdateProfile *prof,
                        hipStream_t st, T *B = nullptr, int64_t ldb = 0, int nrhs = 0, bool prefilled = false);
/* Factor + backward substitution on a workspace of factor_ws_bytes followed
 * by `chunks` (>= 1) times trsv_xb_bytes (B riding along in the factor). */
template <typename T>
hipError_t factor_solve(T *A, int64_t lda, int n, int32_t *info, void *ws, int chunks, const DenseTuning &tun,
                        UpdateProfile *prof, hipStream_t st, T *B, int64_t ldb, int nrhs);
/* Multi-workgroup triangular solve: wsi = status, ticket counter, a solved
 * counter per chunk of 16 right-hand sides; xb = `chunks` (>= 1) exchange
 * buffers of trsv_xb_bytes(sizeof(T), n), as many chunks run side by side;
 * info (or NULL): receives -status at the end of each launch when the status
 * word is nonzero.  start: what the first launch finds -- fresh: nothing
 * (status, info and counters are cleared, xb marked), running: the status of
 * earlier launches, which is kept, ready: also its chunks' counters cleared
 * and their rows marked. */
enum class TrsvStart { fresh, running, ready };
template <typename T>
hipError_t dense_trsv(int mode, const T *LU, int64_t lda, int n, T *B, int64_t ldb, int nrhs, int *wsi, T *xb,
                      int chunks, const int *skip, int32_t *info, hipStream_t st, TrsvStart start,
                      long long wait_limit = 0);
template <typename T>
hipError_t batch_factor(T *A, int64_t lda, int n, int64_t batch, int64_t strideA, int32_t *info, hipStream_t st);
template <typename T>
hipError_t batch_solve(bool adjoint, const T *LU, int64_t lda, int n, int64_t strideLU, T *B, int64_t ldb,
                       int64_t strideB, int nrhs, int64_t batch, hipStream_t st);
/* Ragged batches; two: two workgroups to a compute unit (FP64's always), else
 * three. */
template <typename T>
hipError_t batched_run(int count, const int *ns, const int64_t *offA, T *A, const int64_t *offB, T *B,
                       const int *order, int32_t *info, int *queue, int grid, bool two, hipStream_t st);
hipError_t batched_mixed_run(int count, const int *ns, const int64_t *offA, const double *A, const int64_t *offB,
                             double *B, const int *order, int32_t *info, int *queue, float *W, float *R32,
                             double *X, int max_iter, double tol, int32_t *iters, int grid, bool two, hipStream_t st);
/* Workspace of the segmented band factor (ws may be null: sizes only): per
 * segment its first zero pivot, what is known of its start and pivots, and the
 * diagonal tiles that it started from and ended with; then the band as tiles.  bytes =
 * 0 where the serial chain is used. */
struct BandWs {
    int *zero, *flags;
    double *sstart, *send, *pk;
};
BandWs band_ws(void *ws, int64_t n, size_t &bytes);
/* ws: band_ws(n) bytes or null (the serial chain). */
hipError_t band_factor(double *AB, int64_t ldab, int n, int kl, int ku, int32_t *info, void *ws, hipStream_t st);
hipError_t band_solve(const double *AB, int64_t ldab, int n, int kl, int ku, double *B, int64_t ldb, int nrhs,
                      double *P, hipStream_t st);
template <typename T>
hipError_t outer_neg(int n, int nrhs, const T *Bb, int64_t ldb, int64_t strideB, const T *X, int64_t ldx,
                     int64_t strideX, T *Abar, int64_t ldabar, int64_t strideAbar, int64_t batch, hipStream_t st);
template <typename TI, typename TO>
hipError_t convert(int rows, int cols, const TI *S, int64_t lds, TO *D, int64_t ldd, const int *skip, hipStream_t st);
/* Mixed precision.  convert_margin: D = float(A) (n x n) and the strict
 * diagonal-dominance margin min_i (|a_ii| - sum_{j != i} |a_ij|), clamped at
 * 0, into *mbits as the bits of a non-negative double (atomic minimum; the
 * word starts at the bits of +inf).  Non-negative doubles order like their
 * bit patterns, which every *bits word below relies on. */
hipError_t convert_margin(int n, const double *A, int64_t lda, float *D, int64_t ldd, unsigned long long *mbits,
                          hipStream_t st);
/* One launch ahead of everything: status, info and the factor's control words
 * cleared, the words below set up, iters (or NULL) to -1, and the exchange rows
 * of the first forward substitution (one chunk) marked. */
hipError_t mixed_init(int n, int nrhs, int *ctl, int32_t *info, int *conv, unsigned long long *mbits,
                      unsigned long long *rbits, unsigned long long *xbits, int32_t *iters, float *xb, hipStream_t st);
/* R = float(B - A X), the next correction's right-hand sides, and
 * max_i |r_ic| into rbits[c]. */
hipError_t mixed_residual(int n, int nrhs, const double *A, int64_t lda, const double *B, int64_t ldb, const double *X,
                          int64_t ldx, float *R, int64_t ldr, unsigned long long *rbits, const int *skip, hipStream_t st);
/* Stopping test after refinement step `it`: column c has converged when its
 * forward-error bound max_i|r_ic| / (margin * max_i|x_ic|) <= tol; every
 * column's bound goes to ferr[c].  Unless last, the launch also readies the
 * next forward substitution (TrsvStart::ready, up to `chunks` chunks). */
hipError_t mixed_check(int n, int nrhs, unsigned long long *rbits, unsigned long long *xbits,
                       const unsigned long long *mbits, double tol, int it, int32_t *iters, double *ferr, int *conv,
                       int *ctl, float *xb, int chunks, bool last, hipStream_t st);
/* X (+)= D, and max_i |x_ic| of the result into xbits[c]. */
hipError_t mixed_xupdate(int n, int nrhs, double *X, int64_t ldx, const float *D, int64_t ldd, int first,
                         unsigned long long *xbits, const int *skip, hipStream_t st);

} /* namespace ebv */

#endif
