// fb_lu.hip -- the LU function block (the paper's other offloaded block,
// section 5.1(b)): right-looking blocked LU factorization with partial
// pivoting of a row-major n x n binary64 matrix, in place.
//
// For each panel of LU_NB columns starting at column k:
//   lu_panel  factors rows k..n-1 of the panel column by column (pivot =
//             first row of largest magnitude, row exchange inside the panel,
//             scaling, rank-1 update of the panel's remaining columns); one
//             workgroup holds the whole panel in registers, four rows per
//             thread of 512, so n <= 2048, and exchanges rows by relabelling
//             them;
//   the update of the other columns: the panel's row exchanges, in order,
//             on every column outside the panel, U12 = L11^-1 A12 for the
//             columns right of it, A22 -= L21 U12.
// Two schedules of the same operations:
//   FB_LU_LOOKAHEAD = 1 (default): lu_panel for the first panel, then one
//             lu_step per panel k, whose workgroup 0 updates panel k+1's
//             columns and factors panel k+1 while the other workgroups
//             update the columns right of it (16-column strips) and apply
//             the exchanges left of panel k;
//   FB_LU_LOOKAHEAD = 0: three launches per panel, lu_panel, lu_swap_trsm
//             (exchanges and U12, one thread per column) and lu_gemm_mfma
//             (A22 on 64 x 64 tiles on the binary64 matrix cores; lu_gemm:
//             the same on the vector units, FB_LU_MFMA = 0).
// Every element receives its updates in increasing column order j, as in
// unblocked elimination, so both schedules and both update kernels give
// the same bits.
#include <hip/hip_runtime.h>

#include "fb_device.hpp"
#include "fb_lu.hpp"

namespace fb {

#ifndef FB_LU_PANEL_THREADS
#define FB_LU_PANEL_THREADS 512
#endif
constexpr int LU_PANEL_THREADS = FB_LU_PANEL_THREADS;
constexpr int LU_ROWS = (int)(LU_MAX_N / LU_PANEL_THREADS);   // rows of the panel per thread
static_assert(LU_ROWS * LU_PANEL_THREADS >= LU_MAX_N, "the panel kernel holds every row of a panel");

// ---- pivot search
//
// The pivot is the first row (smallest position) among those of largest
// magnitude.  Magnitudes are compared as the integers their binary64 bits
// are, high words first: the largest high word of a wavefront comes from four
// DPP maxima within its 16-lane rows (lanes l ^ 1, l ^ 2, 7 - l within 8,
// 15 - l within 16) and two row broadcasts, and the ballot of the rows that
// hold it names the candidate.  Only when several rows share it
// (a uniform branch) do the low words, and among equal magnitudes the
// positions, decide.  A NaN counts as larger than any number, so a column
// always has a pivot row.
template <int CTRL> __device__ __forceinline__ int dpp_i(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ int imax(int x, int y) { return x > y ? x : y; }
__device__ __forceinline__ int imin(int x, int y) { return x < y ? x : y; }
// all lanes of each group of 8 get the group's largest x
__device__ __forceinline__ int max8(int x)
{
    x = imax(x, dpp_i<0xB1>(x));    // quad_perm [1,0,3,2]: l ^ 1
    x = imax(x, dpp_i<0x4E>(x));    // quad_perm [2,3,0,1]: l ^ 2
    return imax(x, dpp_i<0x141>(x));   // row_half_mirror
}
// the largest x of the wavefront (x >= INT_MIN + 1), as a scalar
__device__ __forceinline__ int wave_max(int x)
{
    x = max8(x);
    x = imax(x, dpp_i<0x140>(x));   // row_mirror
    // rows 1 and 3 take row 0's and row 2's, then row 3 takes row 1's
    x = imax(x, __builtin_amdgcn_update_dpp((int)0x80000000, x, 0x142, 0xA, 0xF, false));   // row_bcast15
    x = imax(x, __builtin_amdgcn_update_dpp((int)0x80000000, x, 0x143, 0xC, 0xF, false));   // row_bcast31
    return __builtin_amdgcn_readlane(x, 63);
}
__device__ __forceinline__ int hi_word(double x) { return (int)(__double_as_longlong(x) >> 32); }
__device__ __forceinline__ int lo_word(double x) { return (int)__double_as_longlong(x); }
// a low word as an integer whose signed order is the word's unsigned order
__device__ __forceinline__ int lo_key(int lo) { return lo ^ (int)0x80000000; }
__device__ __forceinline__ double lane_d(double x, int l)
{
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)lo_word(x), l);
    const unsigned hi = __builtin_amdgcn_readlane((unsigned)hi_word(x), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// A wave's candidate for the pivot: the magnitude's words and the row's
// position; hi < 0 when the wave holds no row that can be the pivot.
struct __attribute__((aligned(16))) PanelCand {
    int hi, lo, row, pad;
};

// The factorization of one panel (columns k .. k+nb-1, rows k .. k+m-1)
// from registers: thread t holds rows in v[r][0 .. nb), each with its
// position in the panel in lab[r] (rows that are not in the panel carry a
// position >= m).  Rows never move between registers: exchanging rows j and
// p exchanges two positions, and at the end every row is stored at the
// position it carries.
//
// What bounds it: the chain of a column (pivot search, publication, barrier,
// quotients, update of the next column), and with several rows per thread
// the instructions of the two waves that share a SIMD.  So everything that is
// the same for a whole wave is kept in scalars: per register slot the lanes
// whose row has not been a pivot yet are a 64-bit mask (alive[r]) that the
// updates run under, with no select per element; the candidate is named by
// scalar bit scans; and after the column's single barrier each lane reads
// two elements of one of the W candidate rows, the winner among the W
// candidates is found the same way as within a wave, and the pivot row's
// elements are read out of the lanes as scalars, so the barrier is followed
// by one LDS round trip.  Measured against a search by compare-and-select on
// binary64 values with selects per element: 2048 x 2048 5.34 -> 4.87 ms,
// 333 x 333 572 -> 455 us (same bits).  The buffers alternate with the column's parity: a
// thread that reaches column j + 1's barrier has finished every read of
// column j - 1's buffers.
//
// R: the register slots that can hold rows of the panel (slot r holds
// physical rows t + LU_PANEL_THREADS r, so a panel of m rows needs
// ceil(m / LU_PANEL_THREADS) of them); the others are not compiled in, which
// shortens every column step of the short panels.
//
// FULL: nb == LU_NB (every panel but possibly the last), with no test per
// column.
constexpr int LU_W = LU_PANEL_THREADS / 64;   // waves of the panel's workgroup
struct PanelShared {
    PanelCand cand[2][LU_W];
    double crow[2][LU_W][LU_NB];
};

// A wave's 64 rows of one register slot between memory and the rows' threads,
// through the wave's part of the stage: 16 lanes move one row's 128 bytes, so
// an access covers 4 rows instead of the 64 of a row per lane (the first
// panel of 2048 rows 48.2 -> 36.5 us; 2048 x 2048 4.65 -> 4.59 ms; 333 x 333, one
// register slot, 424 -> 434 us, so its rows are stored by their threads).
constexpr int LU_STAGE_LD = LU_NB + 2;   // staged row stride in doubles: 16-byte aligned rows, spread banks
constexpr int LU_STAGE = LU_PANEL_THREADS * LU_STAGE_LD;
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// row `lane` of the wave (v, stored at row lab of the panel when lab < m)
__device__ __forceinline__ void store_rows(const double (&v)[LU_NB], int lab, double *__restrict__ a, int64_t lda,
                                           int64_t k, int m, int nb, double *stage)
{
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    double *st = stage + (threadIdx.x >> 6) * 64 * LU_STAGE_LD;
#pragma unroll
    for (int c = 0; c < LU_NB; c++) st[lane * LU_STAGE_LD + c] = v[c];
    *reinterpret_cast<int *>(&st[lane * LU_STAGE_LD + LU_NB]) = lab;
    wave_lds_order();
#pragma unroll
    for (int t = 0; t < 16; t++) {
        const int row = 4 * t + lk;
        const double x = st[row * LU_STAGE_LD + li];
        const int l = *reinterpret_cast<const int *>(&st[row * LU_STAGE_LD + LU_NB]);
        if (l < m && li < nb) a[(k + l) * lda + k + li] = x;
    }
    wave_lds_order();
}

template <bool FULL, int R>
__device__ __forceinline__ void panel_columns(double (&v)[LU_ROWS][LU_NB], int (&lab)[LU_ROWS],
                                              double *__restrict__ a, int64_t lda, int64_t k, int m, int nb,
                                              int32_t *__restrict__ ipiv, int32_t *__restrict__ info, PanelShared &sh,
                                              double *stage)
{
    constexpr int W = LU_W;
    static_assert(W == 8 && LU_NB == 16, "a wave reads the W candidate rows with one 16-byte access per lane");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (FULL) nb = LU_NB;
    // the first zero pivot and the pivot positions, kept in registers (a
    // global access per column would stall every column's barrier on memory
    // latency) and stored at the end; the first panel starts the record
    int32_t zero_at = k == 0 ? 0 : info[0];
    int piv_at[LU_NB];
    uint64_t alive[R];   // lanes whose row r may still be the pivot
#pragma unroll
    for (int r = 0; r < R; r++) alive[r] = __ballot(lab[r] < m);

    static_for<0, LU_NB>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if (FULL || j < nb) {   // uniform
            constexpr int h = j & 1;
            // ---- the wave's candidate: register slot cr, lane cl
            int hi[R], best = -1;
#pragma unroll
            for (int r = 0; r < R; r++) {
                hi[r] = __builtin_amdgcn_inverse_ballot_w64(alive[r]) ? (hi_word(v[r][j]) & 0x7fffffff) : -1;
                best = imax(best, hi[r]);
            }
            const int hm = wave_max(best);
            // lanes with a numerator too small for the reciprocal (below)
            uint64_t small = 0;
#pragma unroll
            for (int r = 0; r < R; r++) small |= __ballot((unsigned)hi[r] < (unsigned)(1023 - 600) << 20);
            uint64_t at[R];   // the candidate: one lane of one slot
            int count = 0;
#pragma unroll
            for (int r = 0; r < R; r++) {
                at[r] = __ballot(hi[r] == hm);
                count += __popcll(at[r]);
            }
            if (__builtin_expect(count != 1, 0)) {
                if (hm < 0) {   // no row left in this wave
#pragma unroll
                    for (int r = 0; r < R; r++) at[r] = 0;
                    if (lane == 0) sh.cand[h][wave].hi = -1;
                } else {   // the low words decide, then the positions
                    int lk = (int)0x80000000, lb = 0x7fffffff;
#pragma unroll
                    for (int r = 0; r < R; r++) lk = hi[r] == hm ? imax(lk, lo_key(lo_word(v[r][j]))) : lk;
                    const int lm = wave_max(lk);
#pragma unroll
                    for (int r = 0; r < R; r++)
                        lb = hi[r] == hm && lo_key(lo_word(v[r][j])) == lm ? imin(lb, lab[r]) : lb;
                    const int pm = -wave_max(-lb);
#pragma unroll
                    for (int r = 0; r < R; r++) at[r] &= __ballot(lab[r] == pm);   // positions are unique
                }
            }
            // ---- its holder publishes it and its row (columns j ..)
#pragma unroll
            for (int r = 0; r < R; r++) {
                if (__builtin_amdgcn_inverse_ballot_w64(at[r])) {
                    sh.cand[h][wave] = PanelCand{hi[r], lo_word(v[r][j]), lab[r], 0};
#pragma unroll
                    for (int c = j; c < LU_NB; c++) sh.crow[h][wave][c] = v[r][c];
                    asm volatile("" ::: "memory");   // keeps the slots apart (merged, they index v at run time)
                }
            }
            __syncthreads();
            // ---- the pivot: lane l reads candidate l mod W and two elements
            // of its row
            const PanelCand c8 = sh.cand[h][lane & (W - 1)];
            const double2 e = *reinterpret_cast<const double2 *>(&sh.crow[h][lane & (W - 1)][2 * (lane >> 3)]);
            const int ph = max8(c8.hi);
            uint64_t win = __ballot(c8.hi == ph) & 0xffull;
            if (__builtin_expect(__popcll(win) > 1, 0)) {
                const bool t = c8.hi == ph;
                const int lm = max8(t ? lo_key(c8.lo) : (int)0x80000000);
                const bool u = t && lo_key(c8.lo) == lm;
                const int pm = -max8(u ? -c8.row : -0x7fffffff);
                win = __ballot(u && c8.row == pm) & 0xffull;
            }
            const int pw = __ffsll((long long)win) - 1;
            const int p = __builtin_amdgcn_readlane(c8.row, pw);
            piv_at[j] = p;
            double pr[LU_NB];
#pragma unroll
            for (int c = j; c < LU_NB; c++) pr[c] = lane_d((c & 1) ? e.y : e.x, pw + 8 * (c >> 1));
            const double piv = pr[j];
            // ---- exchange the positions j and p; the pivot row is done
#pragma unroll
            for (int r = 0; r < R; r++) {
                const bool t = lab[r] == p;
                alive[r] &= ~__ballot(t);
                lab[r] = t ? j : (lab[r] == j ? p : lab[r]);
            }
            // ---- scale the column below the pivot.  The quotients are the
            // reciprocal's product corrected by one residual, as in Markstein,
            // "Computation of elementary functions on the IBM RISC System/6000
            // processor" (1990); the reciprocal is shared by the rows.  They are
            // what a division gives, bit for bit, while the quotient is normal
            // and the residual exact: with the pivot's exponent within 400 of 0
            // and every numerator of the wave at or above 2^-600 (and |v| <=
            // |piv|) the quotient is at least 2^-1000 and the residual a multiple
            // of 2^-1074.  Otherwise, and for zeros, whose sign the correction
            // would lose, the wave divides; a zero pivot scales nothing.  One
            // branch decides all three: a zero pivot's own branch ahead of it
            // cost 4 % (2048 x 2048 4.39 -> 4.58 ms, 333 x 333 417 -> 438 us).
            auto update = [&](double (&l)[R]) {
#pragma unroll
                for (int r = 0; r < R; r++) {
                    if (__builtin_amdgcn_inverse_ballot_w64(alive[r])) {
                        asm volatile("" : "+v"(l[r]));   // a masked region, not a select per element
                        v[r][j] = l[r];
#pragma unroll
                        for (int c = j + 1; c < LU_NB; c++) v[r][c] = fma(-l[r], pr[c], v[r][c]);
                    }
                }
            };
            const int ex = (hi_word(piv) >> 20) & 0x7ff;
            double l[R];
            if (__builtin_expect(((unsigned)(ex - (1023 - 399)) < 799u) & (small == 0), 1)) {   // uniform
                double rc = __builtin_amdgcn_rcp(piv);
                rc = fma(fma(-piv, rc, 1.0), rc, rc);
                rc = fma(fma(-piv, rc, 1.0), rc, rc);
                rc = fma(fma(-piv, rc, 1.0), rc, rc);
#pragma unroll
                for (int r = 0; r < R; r++) {
                    const double q = v[r][j] * rc;
                    l[r] = fma(fma(-piv, q, v[r][j]), rc, q);
                }
                update(l);
            } else if (piv != 0.0) {
#pragma unroll
                for (int r = 0; r < R; r++) l[r] = v[r][j] / piv;
                update(l);
            } else {
                zero_at = zero_at == 0 ? (int32_t)(k + j + 1) : zero_at;
            }
        }
    });

    if constexpr (R == 1) {   // too few rows for the lookups to matter: one LDS round trip less
        if (lab[0] < m) {
#pragma unroll
            for (int c = 0; c < LU_NB; c++)
                if (c < nb) a[(k + lab[0]) * lda + k + c] = v[0][c];
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; r++) store_rows(v[r], lab[r], a, lda, k, m, nb, stage);
    }
    if (tid == 0) {
#pragma unroll
        for (int j = 0; j < LU_NB; j++)
            if (j < nb) ipiv[k + j] = (int32_t)(k + piv_at[j]);
        info[0] = zero_at;
    }
}

// The first panel (and, with the lookahead off, every panel): rows k ..
// n-1 of columns k .. k+nb-1 loaded into registers, then factored.
template <bool FULL, int R>
__global__ void __launch_bounds__(LU_PANEL_THREADS)
    lu_panel(double *__restrict__ a, int64_t n, int64_t lda, int64_t k, int nb, int32_t *__restrict__ ipiv,
             int32_t *__restrict__ info)
{
    __shared__ PanelShared sh;
    const int tid = threadIdx.x;
    const int m = (int)(n - k);   // rows of the panel (<= LU_ROWS * LU_PANEL_THREADS, checked on the host)
    if (FULL) nb = LU_NB;
    __shared__ double stage[LU_STAGE];
    const int lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
    double *st = stage + wave * 64 * LU_STAGE_LD;
    double v[LU_ROWS][LU_NB];
    int lab[LU_ROWS];   // the row's position; rows past the panel keep positions >= m
    double g[R][16];    // every row's part in flight at once; past the end the last row and column again
#pragma unroll
    for (int r = 0; r < R; r++) {
#pragma unroll
        for (int t = 0; t < 16; t++) {
            const int i = LU_PANEL_THREADS * r + 64 * wave + 4 * t + lk;
            g[r][t] = a[(k + (i < m ? i : m - 1)) * lda + k + (li < nb ? li : nb - 1)];
        }
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
        lab[r] = tid + LU_PANEL_THREADS * r;
#pragma unroll
        for (int t = 0; t < 16; t++) st[(4 * t + lk) * LU_STAGE_LD + li] = g[r][t];
        wave_lds_order();
#pragma unroll
        for (int c = 0; c < LU_NB; c++) v[r][c] = st[lane * LU_STAGE_LD + c];
        wave_lds_order();
    }
    panel_columns<FULL, R>(v, lab, a, lda, k, m, nb, ipiv, info, sh, stage);
}

// The panel's swaps (rows k+j <-> ipiv[k+j], j = 0..nb-1 in order) on every
// column outside the panel, then U12 = L11^-1 A12 on the columns right of
// it.  The swaps are first composed into one permutation of the at most
// 2 nb rows they touch (each workgroup does it in LDS from ipiv), so that a
// column loads every touched row at once and stores each once, instead of
// nb dependent swaps.  One thread per column: row accesses are coalesced.
constexpr int LU_SWAP_THREADS = 64;
// the value of x in lane l (l uniform over the wave)
__device__ __forceinline__ int64_t lane_i64(int64_t x, int l)
{
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)(uint64_t)x, l);
    const unsigned hi = __builtin_amdgcn_readlane((unsigned)((uint64_t)x >> 32), l);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
// The panel's swaps composed by one wave into one permutation of the rows
// they touch: lane q < the returned count holds touched row d and the
// original row sr whose content moves there.  pv is ipiv[k + lane] for lanes
// < nb.  Lanes 0 .. nb-1 start with rows k .. k+nb-1; pivot rows below the
// block are appended as they first appear.  j and q are uniform, so every
// exchange is a scalar read of one lane.
__device__ __forceinline__ int compose_perm(int64_t pv, int64_t k, int nb, int lane, int64_t &d, int64_t &sr)
{
    d = lane < nb ? k + lane : -1;
    sr = d;
    int cnt = nb;
    for (int j = 0; j < nb; j++) {
        const int64_t pr = lane_i64(pv, j);
        int q;
        if (pr - k < nb) {
            q = (int)(pr - k);   // inside the block (pivot rows are >= k + j)
        } else {
            const unsigned long long hit = __ballot(lane >= nb && lane < cnt && d == pr);
            if (hit) {
                q = __ffsll((long long)hit) - 1;
            } else {
                q = cnt++;
                if (lane == q) d = sr = pr;
            }
        }
        const int64_t sj = lane_i64(sr, j), sq = lane_i64(sr, q);
        if (lane == j) sr = sq;
        if (lane == q) sr = sj;
    }
    return cnt;
}

__global__ void __launch_bounds__(LU_SWAP_THREADS)
    lu_swap_trsm(double *__restrict__ a, int64_t n, int64_t lda, int64_t k, int nb, const int32_t *__restrict__ ipiv)
{
    // The kernel is a chain of latencies (the pivots, the permutation, the
    // rows, the solve), so every step keeps its loads in flight together:
    // the pivots and L11 are requested at once, and the row addresses are
    // scalars read from the lanes that composed the permutation, with no LDS
    // round trip between them.
    static_assert(LU_SWAP_THREADS == 64 && 2 * LU_NB <= 64, "one wave composes the permutation");
    static_assert((LU_NB * LU_NB) % LU_SWAP_THREADS == 0, "L11 is loaded in whole rounds");
    constexpr int LR = LU_NB * LU_NB / LU_SWAP_THREADS;
    __shared__ double L[LU_NB][LU_NB + 1];
    const int lane = threadIdx.x;
    const int32_t pv32 = ipiv[k + (lane < nb ? lane : 0)];   // unconditional: no wait at a branch join
    double lv[LR];
#pragma unroll
    for (int t = 0; t < LR; t++) {
        const int idx = lane + LU_SWAP_THREADS * t, i = idx / LU_NB, j = idx % LU_NB;
        const int ic = i < nb ? i : 0, jc = j < nb ? j : 0;   // in bounds also for a short last panel
        lv[t] = a[(k + ic) * lda + k + jc];
    }
    const int64_t pv = lane < nb ? (int64_t)pv32 : 0;
    int64_t d, sr;
    const int cnt = compose_perm(pv, k, nb, lane, d, sr);
#pragma unroll
    for (int t = 0; t < LR; t++) {
        const int idx = lane + LU_SWAP_THREADS * t, i = idx / LU_NB, j = idx % LU_NB;
        L[i][j] = (i < nb && j < nb) ? lv[t] : 0.0;
    }
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * LU_SWAP_THREADS + lane;
    const bool live = c < n && !(c >= k && c < k + nb);   // the panel's own columns are done
    const int64_t cc = live ? c : (k + nb < n ? k + nb : 0);   // a column every lane may read
    double val[2 * LU_NB];
#pragma unroll
    for (int q = 0; q < 2 * LU_NB; q++) val[q] = q < cnt ? a[lane_i64(sr, q) * lda + cc] : 0.0;
    const bool right = c >= k + nb;
    if (right) {
        static_for<1, LU_NB>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
#pragma unroll
            for (int j = 0; j < i; j++) val[i] -= L[i][j] * val[j];
        });
    }
    if (live) {
#pragma unroll
        for (int q = 0; q < 2 * LU_NB; q++) {
            if (q < cnt) {
                const int64_t dq = lane_i64(d, q), sq = lane_i64(sr, q);
                if (dq != sq || (right && q < nb)) a[dq * lda + c] = val[q];
            }
        }
    }
}

// A22 -= L21 U12 on 64 x 64 tiles: rows and columns >= k + nb.
constexpr int LU_TILE = 64;
__global__ void __launch_bounds__(256)
    lu_gemm(double *__restrict__ a, int64_t n, int64_t lda, int64_t k, int nb)
{
    __shared__ double Ls[LU_TILE][LU_NB + 1];
    __shared__ double Us[LU_NB][LU_TILE + 4];
    const int64_t s = k + nb;   // first row and column of A22
    const int64_t r0 = s + (int64_t)blockIdx.y * LU_TILE, c0 = s + (int64_t)blockIdx.x * LU_TILE;
    const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
    for (int idx = tid; idx < LU_TILE * LU_NB; idx += 256) {
        const int i = idx / LU_NB, j = idx % LU_NB;
        Ls[i][j] = (r0 + i < n && j < nb) ? a[(r0 + i) * lda + k + j] : 0.0;
    }
    for (int idx = tid; idx < LU_NB * LU_TILE; idx += 256) {
        const int j = idx / LU_TILE, c = idx % LU_TILE;
        Us[j][c] = (c0 + c < n && j < nb) ? a[(k + j) * lda + c0 + c] : 0.0;
    }
    __syncthreads();
    double acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int64_t r = r0 + ty * 4 + i;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const int64_t cc = c0 + tx * 4 + c;
            acc[i][c] = (r < n && cc < n) ? a[r * lda + cc] : 0.0;
        }
    }
#pragma unroll
    for (int j = 0; j < LU_NB; j++) {
        if (j < nb) {
            double l[4], u[4];
#pragma unroll
            for (int i = 0; i < 4; i++) l[i] = Ls[ty * 4 + i][j];
#pragma unroll
            for (int c = 0; c < 4; c++) u[c] = Us[j][tx * 4 + c];
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int c = 0; c < 4; c++) acc[i][c] -= l[i] * u[c];
        }
    }
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int64_t r = r0 + ty * 4 + i;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const int64_t cc = c0 + tx * 4 + c;
            if (r < n && cc < n) a[r * lda + cc] = acc[i][c];
        }
    }
}

// The same update on the binary64 matrix cores (FB_LU_MFMA = 1):
// v_mfma_f64_16x16x4f64 computes D = A B + C for a 16 x 4 block A, a 4 x 16
// block B and a 16 x 16 block C; lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16] and holds D[4 r + l / 16][l % 16] in its register r < 4
// (rows interleaved over the four 16-lane groups; checked on the device with
// known operands).  Each wave of the 64 x 64 tile computes a 32 x 32
// quadrant as 2 x 2 such blocks over the panel's columns in steps of 4, with
// A = -L21 so that the accumulator starts from A22 and ends at A22 - L21 U12.
#ifndef FB_LU_MFMA
#define FB_LU_MFMA 1
#endif
typedef double lu_d4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(256)
    lu_gemm_mfma(double *__restrict__ a, int64_t n, int64_t lda, int64_t k, int nb)
{
    __shared__ double Ls[LU_TILE][LU_NB + 1];
    __shared__ double Us[LU_NB][LU_TILE + 4];
    const int64_t s = k + nb;   // first row and column of A22
    const int64_t r0 = s + (int64_t)blockIdx.y * LU_TILE, c0 = s + (int64_t)blockIdx.x * LU_TILE;
    const int tid = threadIdx.x;
    for (int idx = tid; idx < LU_TILE * LU_NB; idx += 256) {
        const int i = idx / LU_NB, j = idx % LU_NB;
        Ls[i][j] = (r0 + i < n && j < nb) ? -a[(r0 + i) * lda + k + j] : 0.0;
    }
    for (int idx = tid; idx < LU_NB * LU_TILE; idx += 256) {
        const int j = idx / LU_TILE, c = idx % LU_TILE;
        Us[j][c] = (c0 + c < n && j < nb) ? a[(k + j) * lda + c0 + c] : 0.0;
    }
    const int wave = tid >> 6, lane = tid & 63;
    const int qr = 32 * (wave >> 1), qc = 32 * (wave & 1);   // the wave's quadrant of the tile
    const int li = lane & 15, lk = lane >> 4;
    lu_d4 acc[2][2];
#pragma unroll
    for (int bi = 0; bi < 2; bi++) {
#pragma unroll
        for (int bj = 0; bj < 2; bj++) {
            const int64_t cc = c0 + qc + 16 * bj + li;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int64_t rr = r0 + qr + 16 * bi + 4 * r + lk;
                acc[bi][bj][r] = (rr < n && cc < n) ? a[rr * lda + cc] : 0.0;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int k4 = 0; k4 < LU_NB; k4 += 4) {
        if (k4 < nb) {   // uniform; columns nb .. k4 + 3 of the tiles are zero
            double av[2], bv[2];
#pragma unroll
            for (int bi = 0; bi < 2; bi++) av[bi] = Ls[qr + 16 * bi + li][k4 + lk];
#pragma unroll
            for (int bj = 0; bj < 2; bj++) bv[bj] = Us[k4 + lk][qc + 16 * bj + li];
#pragma unroll
            for (int bi = 0; bi < 2; bi++) {
#pragma unroll
                for (int bj = 0; bj < 2; bj++)
                    acc[bi][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[bi], bv[bj], acc[bi][bj], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int bi = 0; bi < 2; bi++) {
#pragma unroll
        for (int bj = 0; bj < 2; bj++) {
            const int64_t cc = c0 + qc + 16 * bj + li;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int64_t rr = r0 + qr + 16 * bi + 4 * r + lk;
                if (rr < n && cc < n) a[rr * lda + cc] = acc[bi][bj][r];
            }
        }
    }
}

// ---- one launch per panel: the previous panel's update and the next panel
//
// lu_step(k) runs after panel k (columns k .. k+nb-1) has been factored.  Its
// workgroups split the work by columns, each owning its columns in every
// row, so that the row exchanges can be applied in place with no other
// workgroup reading or writing those rows' elements:
//   workgroup 0     the next panel's columns s .. s+nb2-1 (s = k + nb): the
//                   exchanges, U12 = L11^-1 A12, A22 -= L21 U12, then the
//                   factorization of panel s from its registers (the
//                   lookahead: the next panel starts as soon as its own
//                   columns are up to date);
//   the next ones   the same update on 16-column strips right of it;
//   the last ones   the exchanges alone on the columns left of the panel,
//                   one column per thread.
// Every element receives the same operations in the same order as in
// lu_swap_trsm and lu_gemm, so the factors are bitwise those of the
// three-launch schedule.
struct StripShared {
    double L[LU_NB][LU_NB + 1];          // L11
    double U[LU_NB][LU_NB + 1];          // the strip's U12 block
    double slot[2 * LU_NB][LU_NB];       // the touched rows' contents, by composed index
    int64_t dst[2 * LU_NB], src[2 * LU_NB];
    int np;
    int16_t recv[LU_MAX_N];              // per row from k: the slot whose content it takes, or -1
    double stage[LU_STAGE];   // one register slot's rows on their way to their threads
};

// Columns [c0, c0 + w) of rows k .. n-1 after panel k.  KEEP: store only the
// U12 rows and leave the rows below them, updated, in v (thread t holds rows
// k + t + LU_PANEL_THREADS r in v[r][0 .. w)); otherwise store every row.
//
// Bound: the latency and the cache-line lookups of one CU's loads, since a
// strip is one workgroup's work.  So A22 -= L21 U12 runs on the binary64 matrix
// cores (as in lu_gemm_mfma: 16-row blocks, lane l holds rows 4 r + l / 16 of
// column l mod 16), whose operands load and store without passing through
// LDS: an access of A22 covers 4 whole rows and one of L21 16 rows' 32 bytes,
// where a row per lane covers 64 lines.  The rows that the exchanges touch (at
// most 2 LU_NB) are loaded apart, after the permutation is known: the first
// LU_NB of them are U12's right-hand sides, the others are updated by one
// thread per element and replace what the blocks computed in their place.
// Elements are updated in column order, so the factors are bitwise those of a
// row per lane on the vector units.  2048 x 2048 4.87 -> 4.65 ms, 333 x 333 452 ->
// 424 us.
template <bool KEEP, int R>
__device__ __forceinline__ void strip_update(double *__restrict__ a, int64_t n, int64_t lda, int64_t k, int nb,
                                             const int32_t *__restrict__ ipiv, int64_t c0, int w,
                                             double (&v)[LU_ROWS][LU_NB], StripShared &sh)
{
    static_assert(2 * LU_NB <= 64, "one wave composes the permutation");
    static_assert(2 * LU_NB * LU_NB == LU_PANEL_THREADS && LU_NB == 16, "one touched element per thread");
    constexpr int BLOCKS = 4;   // 16-row blocks of a wave's 64 rows of one register slot
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = (int)(n - k);
    const int li = lane & 15, lk = lane >> 4;
    const int q = tid >> 4, c = tid & 15;   // this thread's element of the touched rows
    const int cc = c < w ? c : w - 1;       // (columns past the strip read its last one and are not stored)
    const int lc = li < w ? li : w - 1;
    // ---- the pivots, L11, and the first rows' blocks: every load that does
    // not depend on the permutation.  Rows past the end read the last row
    // again and are not stored.  A strip is called with nb == LU_NB (a panel is
    // followed by columns only when it is whole).
    const int32_t pv32 = ipiv[k + (lane < nb ? lane : 0)];
    const double lv = a[(k + (q & 15)) * lda + k + c];   // threads 256.. read L11 again
    auto row_of = [&](int i) { return a + (k + (i < m ? i : m - 1)) * lda; };
    lu_d4 acc[BLOCKS];
    double la[BLOCKS][4];
    auto load_slot = [&](int r) {
#pragma unroll
        for (int b = 0; b < BLOCKS; b++) {
            const int i0 = LU_PANEL_THREADS * r + 64 * wave + 16 * b;
#pragma unroll
            for (int t = 0; t < 4; t++) acc[b][t] = row_of(i0 + 4 * t + lk)[c0 + lc];
            const double *lr = row_of(i0 + li) + k + lk;
#pragma unroll
            for (int t = 0; t < 4; t++) la[b][t] = lr[4 * t];
        }
    };
    load_slot(0);
    // ---- the permutation, composed by wave 0
    if constexpr (KEEP) {
        for (int i = tid; i < m; i += LU_PANEL_THREADS) sh.recv[i] = -1;
    }
    if (tid < LU_NB * LU_NB) sh.L[q][c] = lv;
    int64_t d = -1, sr = -1;
    int cnt = 0;
    if (wave == 0) {
        cnt = compose_perm(lane < nb ? (int64_t)pv32 : 0, k, nb, lane, d, sr);
        if (lane < cnt) {
            sh.dst[lane] = d;
            sh.src[lane] = sr;
        }
        if (lane == 0) sh.np = cnt;
    }
    __syncthreads();
    const int np = sh.np;
    const int64_t dq = q < np ? sh.dst[q] : k, sq = q < np ? sh.src[q] : k;
    double p = a[sq * lda + c0 + cc];
    double lrow[LU_NB];   // L21 of the touched row below U12
#pragma unroll
    for (int j = 0; j < LU_NB; j++) lrow[j] = q >= nb ? a[dq * lda + k + j] : 0.0;
    if constexpr (KEEP) {
        if (wave == 0 && lane >= nb && lane < cnt) sh.recv[d - k] = (int16_t)lane;
    }
    if (q < nb) sh.U[q][c] = p;
    asm volatile("" : "+v"(p));   // every touched row has arrived before a wave stores its blocks
    __syncthreads();
    // ---- U12 = L11^-1 A12, one thread per column
    if (tid < LU_NB) {
        double col[LU_NB];
#pragma unroll
        for (int i = 0; i < LU_NB; i++) col[i] = sh.U[i][tid];
        static_for<1, LU_NB>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
#pragma unroll
            for (int j = 0; j < i; j++) col[i] -= sh.L[i][j] * col[j];
        });
#pragma unroll
        for (int i = 0; i < LU_NB; i++) sh.U[i][tid] = col[i];
    }
    __syncthreads();
    // ---- the touched rows
    if (q < nb) {
        p = sh.U[q][c];
    } else {
#pragma unroll
        for (int j = 0; j < LU_NB; j++) p = fma(-lrow[j], sh.U[j][c], p);
        if constexpr (KEEP) sh.slot[q][c] = p;
    }
    // ---- A22 -= L21 U12
    double bu[4];
#pragma unroll
    for (int t = 0; t < 4; t++) bu[t] = sh.U[4 * t + lk][li];
    static_for<0, R>([&](auto rc) {
        constexpr int r = decltype(rc)::value;
#pragma unroll
        for (int b = 0; b < BLOCKS; b++) {
#pragma unroll
            for (int t = 0; t < 4; t++)
                acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(-la[b][t], bu[t], acc[b], 0, 0, 0);
        }
        if constexpr (KEEP) {
            // to the rows' threads, which are lanes of the same wave
            double *st = sh.stage + 64 * wave * LU_STAGE_LD;
#pragma unroll
            for (int b = 0; b < BLOCKS; b++) {
#pragma unroll
                for (int t = 0; t < 4; t++) st[(16 * b + 4 * t + lk) * LU_STAGE_LD + li] = acc[b][t];
            }
            if constexpr (r + 1 < R) load_slot(r + 1);
            wave_lds_order();
#pragma unroll
            for (int j = 0; j < LU_NB; j++) v[r][j] = st[lane * LU_STAGE_LD + j];
            wave_lds_order();
        } else {
#pragma unroll
            for (int b = 0; b < BLOCKS; b++) {
                const int i0 = LU_PANEL_THREADS * r + 64 * wave + 16 * b;
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    const int i = i0 + 4 * t + lk;
                    if (i >= nb && i < m && li < w) a[(k + i) * lda + c0 + li] = acc[b][t];
                }
            }
            if constexpr (r + 1 < R) load_slot(r + 1);
        }
    });
    // ---- the touched rows' own values over what the blocks put in their place
    if constexpr (KEEP) {
        __syncthreads();   // the slots are written
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int i = tid + LU_PANEL_THREADS * r;
            const int s = i < m ? sh.recv[i] : -1;
            if (s >= 0) {
#pragma unroll
                for (int j = 0; j < LU_NB; j++) v[r][j] = sh.slot[s][j];
            }
        }
        if (q < nb && c < w) a[(k + q) * lda + c0 + c] = p;
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the blocks' stores come first
        __syncthreads();
        if (q < np && c < w) a[dq * lda + c0 + c] = p;
    }
}

// The exchanges alone on columns [c0, min(c0 + LU_PANEL_THREADS, k)), one
// column per thread.
__device__ __forceinline__ void left_swaps(double *__restrict__ a, int64_t lda, int64_t k, int nb,
                                           const int32_t *__restrict__ ipiv, int64_t c0, StripShared &sh)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (wave == 0) {
        const int32_t pv32 = ipiv[k + (lane < nb ? lane : 0)];
        int64_t d, sr;
        const int cnt = compose_perm(lane < nb ? (int64_t)pv32 : 0, k, nb, lane, d, sr);
        if (lane < cnt) {
            sh.dst[lane] = d;
            sh.src[lane] = sr;
        }
        if (lane == 0) sh.np = cnt;
    }
    __syncthreads();
    const int64_t c = c0 + tid;
    if (c >= k) return;
    const int np = sh.np;
    double val[2 * LU_NB];
#pragma unroll
    for (int q = 0; q < 2 * LU_NB; q++) val[q] = q < np ? a[sh.src[q] * lda + c] : 0.0;
#pragma unroll
    for (int q = 0; q < 2 * LU_NB; q++)
        if (q < np && sh.dst[q] != sh.src[q]) a[sh.dst[q] * lda + c] = val[q];
}

#ifndef FB_LU_STRIP_DELAY
#define FB_LU_STRIP_DELAY 0   // pauses of 127 x 64 cycles per register slot before the strips start
#endif

// grid: nfirst (0 or 1: the next panel's workgroup), nstrips, then the
// left-column workgroups.  FULL_NEXT: the next panel is LU_NB wide.  R: the
// register slots that rows k .. n-1 need.
template <bool FULL_NEXT, int R>
__global__ void __launch_bounds__(LU_PANEL_THREADS)
    lu_step(double *__restrict__ a, int64_t n, int64_t lda, int64_t k, int nb, int32_t *__restrict__ ipiv,
            int32_t *__restrict__ info, int nfirst, int nstrips)
{
    __shared__ StripShared ss;
    __shared__ PanelShared ps;
    const int b = blockIdx.x;
    const int64_t s = k + nb;   // the first column right of panel k
    const int nb2 = (int)(n - s < LU_NB ? n - s : LU_NB);   // the next panel's width (when s < n)
    if (b < nfirst) {
        double v[LU_ROWS][LU_NB];
        strip_update<true, R>(a, n, lda, k, nb, ipiv, s, nb2, v, ss);
        // rows k + nb .. n-1 are the next panel's rows 0 .. n-s-1; the U12
        // rows above them are done
        const int m = (int)(n - k);
        int lab[LU_ROWS];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int i = threadIdx.x + LU_PANEL_THREADS * r;
            lab[r] = (i >= nb && i < m) ? i - nb : 0x3fffffff;
        }
        panel_columns<FULL_NEXT, R>(v, lab, a, lda, s, m - nb, nb2, ipiv, info, ps, ss.stage);
    } else if (b < nfirst + nstrips) {
        // the strips have the length of the next panel's factorization to
        // finish; they start after a pause, so that workgroup 0's own loads
        // do not queue behind theirs
        for (int t = 0; nfirst && t < FB_LU_STRIP_DELAY * R; t++) __builtin_amdgcn_s_sleep(127);
        const int64_t c0 = s + nb2 + (int64_t)LU_NB * (b - nfirst);
        const int w = (int)(n - c0 < LU_NB ? n - c0 : LU_NB);
        double v[LU_ROWS][LU_NB];
        strip_update<false, R>(a, n, lda, k, nb, ipiv, c0, w, v, ss);
    } else {
        for (int t = 0; nfirst && t < FB_LU_STRIP_DELAY * R; t++) __builtin_amdgcn_s_sleep(127);
        left_swaps(a, lda, k, nb, ipiv, (int64_t)LU_PANEL_THREADS * (b - nfirst - nstrips), ss);
    }
}

#ifndef FB_LU_LOOKAHEAD
#define FB_LU_LOOKAHEAD 1   // 0: three launches per panel (lu_panel, lu_swap_trsm, lu_gemm)
#endif

// R = ceil(m / LU_PANEL_THREADS) register slots for m rows
template <int R> struct LuKernels {
    static void panel(bool full, double *a, int64_t n, int64_t lda, int64_t k, int nb, int32_t *ipiv, int32_t *info,
                      hipStream_t st)
    {
        if (full)
            hipLaunchKernelGGL((lu_panel<true, R>), dim3(1), dim3(LU_PANEL_THREADS), 0, st, a, n, lda, k, nb, ipiv, info);
        else
            hipLaunchKernelGGL((lu_panel<false, R>), dim3(1), dim3(LU_PANEL_THREADS), 0, st, a, n, lda, k, nb, ipiv, info);
    }
    static void step(bool full_next, unsigned grid, double *a, int64_t n, int64_t lda, int64_t k, int nb,
                     int32_t *ipiv, int32_t *info, int nfirst, int nstrips, hipStream_t st)
    {
        if (full_next)
            hipLaunchKernelGGL((lu_step<true, R>), dim3(grid), dim3(LU_PANEL_THREADS), 0, st, a, n, lda, k, nb, ipiv,
                               info, nfirst, nstrips);
        else
            hipLaunchKernelGGL((lu_step<false, R>), dim3(grid), dim3(LU_PANEL_THREADS), 0, st, a, n, lda, k, nb, ipiv,
                               info, nfirst, nstrips);
    }
};
static_assert(LU_ROWS == 4, "the launches below instantiate 1 .. 4 register slots");
static void launch_panel(int64_t m, bool full, double *a, int64_t n, int64_t lda, int64_t k, int nb, int32_t *ipiv,
                         int32_t *info, hipStream_t st)
{
    switch ((m + LU_PANEL_THREADS - 1) / LU_PANEL_THREADS) {
    case 1: LuKernels<1>::panel(full, a, n, lda, k, nb, ipiv, info, st); break;
    case 2: LuKernels<2>::panel(full, a, n, lda, k, nb, ipiv, info, st); break;
    case 3: LuKernels<3>::panel(full, a, n, lda, k, nb, ipiv, info, st); break;
    default: LuKernels<4>::panel(full, a, n, lda, k, nb, ipiv, info, st); break;
    }
}
static void launch_step(int64_t m, bool full_next, unsigned grid, double *a, int64_t n, int64_t lda, int64_t k, int nb,
                        int32_t *ipiv, int32_t *info, int nfirst, int nstrips, hipStream_t st)
{
    switch ((m + LU_PANEL_THREADS - 1) / LU_PANEL_THREADS) {
    case 1: LuKernels<1>::step(full_next, grid, a, n, lda, k, nb, ipiv, info, nfirst, nstrips, st); break;
    case 2: LuKernels<2>::step(full_next, grid, a, n, lda, k, nb, ipiv, info, nfirst, nstrips, st); break;
    case 3: LuKernels<3>::step(full_next, grid, a, n, lda, k, nb, ipiv, info, nfirst, nstrips, st); break;
    default: LuKernels<4>::step(full_next, grid, a, n, lda, k, nb, ipiv, info, nfirst, nstrips, st); break;
    }
}

hipError_t launch_lu(double *a, int64_t n, int64_t lda, int32_t *ipiv, int32_t *info, hipStream_t st)
{
    hipError_t e = hipSuccess;
    if (FB_LU_LOOKAHEAD) {
        const int nb0 = (int)(n < LU_NB ? n : LU_NB);
        if (e == hipSuccess) {
            launch_panel(n, nb0 == LU_NB, a, n, lda, 0, nb0, ipiv, info, st);
            e = hipGetLastError();
        }
        for (int64_t k = 0; e == hipSuccess && k < n; k += LU_NB) {
            const int nb = (int)(n - k < LU_NB ? n - k : LU_NB);
            const int64_t s = k + nb;
            const int nfirst = s < n ? 1 : 0;
            const int64_t nb2 = s < n ? (n - s < LU_NB ? n - s : LU_NB) : 0;
            const int nstrips = s < n ? (int)((n - s - nb2 + LU_NB - 1) / LU_NB) : 0;
            const int nleft = (int)((k + LU_PANEL_THREADS - 1) / LU_PANEL_THREADS);
            const unsigned grid = (unsigned)(nfirst + nstrips + nleft);
            if (grid == 0) continue;
            launch_step(n - k, nb2 == LU_NB || nfirst == 0, grid, a, n, lda, k, nb, ipiv, info, nfirst, nstrips, st);
            e = hipGetLastError();
        }
        return e;
    }
    for (int64_t k = 0; e == hipSuccess && k < n; k += LU_NB) {
        const int nb = (int)(n - k < LU_NB ? n - k : LU_NB);
        launch_panel(n - k, nb == LU_NB, a, n, lda, k, nb, ipiv, info, st);
        if (n > nb)
            hipLaunchKernelGGL(lu_swap_trsm, dim3((unsigned)((n + LU_SWAP_THREADS - 1) / LU_SWAP_THREADS)),
                               dim3(LU_SWAP_THREADS), 0, st, a, n, lda, k, nb, ipiv);
        const int64_t rest = n - k - nb;
        if (rest > 0) {
            const unsigned t = (unsigned)((rest + LU_TILE - 1) / LU_TILE);
            if (FB_LU_MFMA) hipLaunchKernelGGL(lu_gemm_mfma, dim3(t, t), dim3(256), 0, st, a, n, lda, k, nb);
            else hipLaunchKernelGGL(lu_gemm, dim3(t, t), dim3(256), 0, st, a, n, lda, k, nb);
        }
        e = hipGetLastError();
    }
    return e;
}

}  // namespace fb
