// Kernel k-means++ seeding on the device (FP64).  The paper initialises with
// "the kernel version of k-means++" (Sections 1 and 4), which keeps every
// initial center a single feature vector, hence a convex combination of X.
//   pick 0 : floor(u_0 n)
//   pick r : the first row p whose running sum of D2 (row order) exceeds
//            u_r * sum_p D2(p),  D2(p) = min over chosen c of
//            K(p,p) - 2 K(p,c) + K(c,c);
//            sum = 0 -> floor(u_r n); no crossing (rounding) -> the last p
//            with D2(p) > 0.
// Each round is two launches (D2 update + block sums, selection), with the
// pick kept on the device, so seeding needs no host round trip.
//
// What bounds it: a round that evaluates every row reads all of X (512 MB for
// 1M x 128 or 4M x 32).  For the Gaussian and the Laplacian, K falls with an
// input-space metric (L2, L1), so most rows need no evaluation: with c(p) the
// nearest pick so far and e the metric, e(p, new) >= e(c(p), new) - e(p, c(p)),
// hence e(p, c(p)) <= e(c(p), new) / 2 leaves the row's minimum as it is.  The
// selection turns that into one threshold per earlier pick in units of D2
// (exact: see k_kpp_select), and a round reads 12 bytes per row (D2 and the
// rank of c(p)) plus the rows of X that may change.
#include "dev_common.h"
#include "kernels.h"

namespace mbkk {

constexpr int kKppBlock = 256;

// Partial kernel sums over the coordinates t = sub, sub + 16, ... of a row;
// the 16 lanes of a row then combine them and finish K (FP64).
template <int KIND>
__device__ __forceinline__ double kacc64(const float *__restrict__ a, const float *__restrict__ b, int d, int sub)
{
    double s = 0.0;
    for (int t = sub; t < d; t += 16) {
        const double x = (double)a[t], y = (double)b[t];
        if constexpr (KIND == MBKK_GAUSS) {
            const double v = x - y;
            s += v * v;
        } else if constexpr (KIND == MBKK_LAPLACE) {
            s += fabs(x - y);
        } else {
            s += x * y;
        }
    }
    for (int o = 8; o > 0; o >>= 1)
        s += __shfl_xor(s, o, 16);
    return s;
}

template <int KIND>
__device__ __forceinline__ double kfin64(double param, double s)
{
    if constexpr (KIND == MBKK_GAUSS || KIND == MBKK_LAPLACE)
        return exp(-s / param);
    else if constexpr (KIND == MBKK_LINEAR)
        return s;
    else
        return (s + param) * (s + param);
}

// Rank of the nearest pick so far (in the kself array, whose values are all 1
// for the kernels concerned): kNearNone before the first update, kNearBad for
// a row with a non-finite coordinate, whose K(p,p) is NaN: its D2 never
// changes, and as a pick it changes no row's D2.
constexpr int kNearNone = -1, kNearBad = -2;

// K(p,p) for every row, D2 = +inf.  16 lanes per row.
template <int KIND>
__global__ __launch_bounds__(256) void k_kpp_self(const float *__restrict__ X, int64_t n, int d, int64_t ld,
                                                   double param, double *__restrict__ kself,
                                                   double *__restrict__ D2)
{
    const int sub = threadIdx.x & 15;
    const int64_t p = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    if (p >= n)
        return;
    const float *x = X + p * ld;
    const double s = kacc64<KIND>(x, x, d, sub);
    if (sub == 0) {
        kself[p] = kfin64<KIND>(param, s);
        D2[p] = INFINITY;
    }
}

// The pruned kernels' start: no nearest pick yet, D2 = +inf.  ||x||^2 (from
// set_data) is finite only if every coordinate is; the few rows where it is
// not are looked at coordinate by coordinate, so X itself is not read
// (1M x 128: 155 us as K(p,p) over X, 5 us so).
__global__ __launch_bounds__(256) void k_kpp_start(const float *__restrict__ X, int64_t n, int d, int64_t ld,
                                                    const float *__restrict__ sqn, int32_t *__restrict__ near,
                                                    double *__restrict__ D2)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= n)
        return;
    int32_t v = kNearNone;
    if (!isfinite(sqn[p])) {
        for (int t = 0; t < d; ++t)
            if (!isfinite(X[p * ld + t]))
                v = kNearBad;
    }
    near[p] = v;
    D2[p] = INFINITY;
}

void launch_kpp_self(const Layout &L, const Buffers &B, int kind, double param, hipStream_t st)
{
    if (kind == MBKK_GAUSS || kind == MBKK_LAPLACE) {
        hipLaunchKernelGGL(k_kpp_start, dim3((unsigned)((L.n + 255) / 256)), dim3(256), 0, st, B.X, L.n, L.d, B.ld,
                           B.sqn, (int32_t *)B.kself, B.D2);
        return;
    }
    const dim3 grid((unsigned)((L.n + 15) / 16));
#define MBKK_KSELF(K) \
    hipLaunchKernelGGL(k_kpp_self<K>, grid, dim3(256), 0, st, B.X, L.n, L.d, B.ld, param, B.kself, B.D2)
    if (kind == MBKK_LINEAR)
        MBKK_KSELF(MBKK_LINEAR);
    else
        MBKK_KSELF(MBKK_POLY2);
#undef MBKK_KSELF
}

// Coordinate sums of the metric for R rows against the pick's row xc: LPR
// lanes per row, 16 bytes of a row per lane and load (V4: rows 16-byte
// aligned) or 4, the R rows' loads in flight together.  Every lane of the
// group returns the sums.
template <int KIND, int LPR, bool V4, int R>
__device__ __forceinline__ void kpp_sums(const float *const (&x)[R], const float *__restrict__ xc, int d, int sub,
                                         double (&s)[R])
{
    auto term = [](float a, float b) -> double {
        const double v = (double)a - (double)b;
        if constexpr (KIND == MBKK_GAUSS)
            return v * v;
        else
            return fabs(v);
    };
#pragma unroll
    for (int q = 0; q < R; ++q)
        s[q] = 0.0;
    const int d4 = V4 ? d & ~3 : 0;
    if constexpr (V4) {
        for (int t = 4 * sub; t < d4; t += 4 * LPR) {
            f32x4 a[R];
            const f32x4 c = *(const f32x4 *)(xc + t);
#pragma unroll
            for (int q = 0; q < R; ++q)
                a[q] = *(const f32x4 *)(x[q] + t);
#pragma unroll
            for (int q = 0; q < R; ++q)
                s[q] += (term(a[q][0], c[0]) + term(a[q][1], c[1])) + (term(a[q][2], c[2]) + term(a[q][3], c[3]));
        }
    }
    for (int t = d4 + sub; t < d; t += LPR) {
        const float c = xc[t];
#pragma unroll
        for (int q = 0; q < R; ++q)
            s[q] += term(x[q][t], c);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        s[q] += dpp_f64<0xb1>(s[q]);   // quad_perm [1,0,3,2]
        s[q] += dpp_f64<0x4e>(s[q]);   // quad_perm [2,3,0,1]
        s[q] += dpp_f64<0x141>(s[q]);  // row_half_mirror: 8 lanes
        if constexpr (LPR == 16)
            s[q] += dpp_f64<0x140>(s[q]);  // row_mirror: 16 lanes
    }
}

// D2 <- min(D2, 2 - 2 K(p,c)) with c = picks[r], Gaussian and Laplacian, and
// the sums over blocks of 256 rows.  A workgroup takes NQ blocks: a thread
// reads D2 and the nearest pick's rank of one row per block, the rows that
// the thresholds of the selection do not rule out are listed in LDS, groups of
// LPR lanes take their sums over X four rows at a time, and the rows' own
// threads finish them (one FP64 exp per listed row, full lanes).  Blocks
// whose D2 did not change keep their sum.
// Measured on one MI355X: 1M x 128, k = 100 (components of 10k rows): 218 us
// a round when every row was evaluated by 16 lanes with 4-byte loads.
template <int KIND, int LPR, bool V4, int NQ>
__global__ __launch_bounds__(256) void k_kpp_prune(const float *__restrict__ X, int64_t n, int d, int64_t ld,
                                                    double param, const int32_t *__restrict__ picks, int r,
                                                    const double *__restrict__ thr, int32_t *__restrict__ near,
                                                    double *__restrict__ D2, double *__restrict__ bsum)
{
    constexpr int R = 4, NG = 256 / LPR;
    __shared__ double sd[NQ * kKppBlock];
    __shared__ uint16_t list[NQ * kKppBlock];
    __shared__ int wcnt[NQ * 4];
    __shared__ double red[4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t p0 = (int64_t)blockIdx.x * (NQ * kKppBlock);
    const int64_t c = picks[r];
    double v[NQ];
    int nr[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int64_t p = p0 + q * kKppBlock + tid;
        v[q] = p < n ? D2[p] : 0.0;
        nr[q] = p < n ? near[p] : kNearBad;
    }
    if (near[c] == kNearBad && r > 0)
        return;  // block uniform: K(c,c) is NaN, no row changes (r = 0: the sums are still to be written)
    const bool cbad = near[c] == kNearBad;
    bool need[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        need[q] = !cbad && nr[q] != kNearBad && !(nr[q] >= 0 && v[q] <= thr[max(nr[q], 0)]);
        const uint64_t m = __ballot(need[q]);
        if (lane == 0)
            wcnt[q * 4 + w] = __popcll(m);
    }
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int i = 0; i < NQ * 4; ++i)
        total += wcnt[i];
    if (total == 0 && r > 0)
        return;  // block uniform
    {
        int base = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint64_t m = __ballot(need[q]);
            int at = base;
            for (int i = 0; i < w; ++i)
                at += wcnt[q * 4 + i];
            if (need[q])
                list[at + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)(q * kKppBlock + tid);
            base += wcnt[q * 4] + wcnt[q * 4 + 1] + wcnt[q * 4 + 2] + wcnt[q * 4 + 3];
        }
    }
    __syncthreads();
    const int sub = tid % LPR, grp = tid / LPR;
    const float *xc = X + c * ld;
    for (int i0 = grp; i0 < total; i0 += NG * R) {
        const float *x[R];
        int loc[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            loc[q] = list[min(i0 + q * NG, total - 1)];
            x[q] = X + (p0 + loc[q]) * ld;
        }
        double s[R];
        kpp_sums<KIND, LPR, V4, R>(x, xc, d, sub, s);
#pragma unroll
        for (int q = 0; q < R; ++q)
            if (sub == 0 && i0 + q * NG < total)
                sd[loc[q]] = s[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        bool ch = r == 0;
        if (need[q]) {
            const int64_t p = p0 + q * kKppBlock + tid;
            const double dd = (1.0 - 2.0 * kfin64<KIND>(param, sd[q * kKppBlock + tid])) + 1.0;
            if (dd < v[q]) {
                v[q] = dd;
                D2[p] = dd;
                near[p] = r;
                ch = true;
            }
        }
        if (__syncthreads_or(ch)) {
            const double t = wave_sum_f64(v[q]);
            if (lane == 0)
                red[w] = t;
            __syncthreads();
            const int64_t blk = (int64_t)blockIdx.x * NQ + q;
            if (tid == 0 && blk * kKppBlock < n)
                bsum[blk] = (red[0] + red[1]) + (red[2] + red[3]);
            __syncthreads();
        }
    }
}

// D2 <- min(D2, K(p,p) - 2K(p,c) + K(c,c)) with c = picks[r]; block sums over
// 256 consecutive rows (16 lanes per row, 16 rows at a time).  Linear and
// polynomial kernels.
template <int KIND>
__global__ __launch_bounds__(256) void k_kpp_update(const float *__restrict__ X, int64_t n, int d, int64_t ld,
                                                     double param, const int32_t *__restrict__ picks,
                                                     int r, const double *__restrict__ kself,
                                                     double *__restrict__ D2, double *__restrict__ bsum)
{
    __shared__ double red[kKppBlock];
    const int tid = threadIdx.x, sub = tid & 15, grp = tid >> 4;
    const int64_t c = picks[r];
    const float *xc = X + c * ld;
    const double kcc = kself[c];
    for (int it = 0; it < kKppBlock / 16; ++it) {
        const int local = it * 16 + grp;
        const int64_t p = (int64_t)blockIdx.x * kKppBlock + local;
        double s = 0.0;
        if (p < n)
            s = kacc64<KIND>(X + p * ld, xc, d, sub);
        if (sub == 0) {
            double v = 0.0;
            if (p < n) {
                const double dd = kself[p] - 2.0 * kfin64<KIND>(param, s) + kcc;
                v = fmin(D2[p], dd);
                D2[p] = v;
            }
            red[local] = v;
        }
    }
    __syncthreads();
    for (int h = kKppBlock / 2; h > 0; h >>= 1) {
        if (tid < h)
            red[tid] += red[tid + h];
        __syncthreads();
    }
    if (tid == 0)
        bsum[blockIdx.x] = red[0];
}

// Inclusive prefix sum of one double per lane.
__device__ __forceinline__ double wave_inclusive_f64(double v)
{
    const int lane = threadIdx.x & 63;
    for (int o = 1; o < 64; o <<= 1) {
        const double t = __shfl_up(v, o);
        if (lane >= o)
            v += t;
    }
    return v;
}

// Selection of pick r: the first row whose running sum of D2 exceeds u_r
// times the whole sum, searched over the thread's stretches of block sums, the
// blocks of the stretch that crosses, and the rows of that block, each level
// by a parallel scan.  (As one thread's running sums over 1024 stretches and
// 256 rows it took 32 us a round at 1M rows: a chain of LDS and memory
// latencies.)
//
// Every workgroup makes the same selection; workgroup 0 writes it, and with
// the pick known each takes its share of the thresholds of the next update
// (PRUNE): thr[r'] = D2 at half the distance of picks r' and r, lowered by
// 1e-9 of the distance and by 1e-14.  A row p with nearest pick r' and
// D2(p) <= thr[r'] has K(p, r') > K(half distance) + 4e-15, i.e. it lies
// nearer to r' than half the distance by more than the FP64 rounding of the
// sums and of exp (a few 1e-16), so that its computed D2 against pick r can't
// be the smaller one: the rows passed over keep exactly the D2 they had.
constexpr int kSelThreads = 1024;

template <int KIND, bool PRUNE>
__global__ __launch_bounds__(kSelThreads) void k_kpp_select(int64_t n, int64_t nblocks, const double *__restrict__ u,
                                                             int r, const double *__restrict__ D2,
                                                             const double *__restrict__ bsum,
                                                             int32_t *__restrict__ picks,
                                                             const float *__restrict__ X, int d, int64_t ld,
                                                             double param, double *__restrict__ thr)
{
    __shared__ double wtot[kSelThreads / 64];
    __shared__ int first;
    __shared__ double first_run;
    __shared__ int64_t found;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (r == 0) {
        if (tid == 0) {
            int64_t p = (int64_t)floor(u[0] * (double)n);
            picks[0] = (int32_t)(p >= n ? n - 1 : p);
        }
        return;
    }
    const int64_t per = (nblocks + kSelThreads - 1) / kSelThreads;
    const int64_t b0 = min(nblocks, tid * per), b1 = min(nblocks, b0 + per);
    double s = 0.0;
#pragma unroll 4
    for (int64_t q = b0; q < b1; ++q)
        s += bsum[q];
    const double inc = wave_inclusive_f64(s);
    if (lane == 63)
        wtot[w] = inc;
    if (tid == 0) {
        first = kSelThreads;
        found = -1;
    }
    __syncthreads();
    double below = 0.0, tot = 0.0;
    for (int q = 0; q < kSelThreads / 64; ++q) {
        if (q == w)
            below = tot;
        tot += wtot[q];
    }
    if (!(tot > 0.0)) {  // block uniform
        int64_t p = (int64_t)floor(u[r] * (double)n);
        if (tid == 0)
            found = p >= n ? n - 1 : p;
    } else {
        const double target = u[r] * tot;
        // (a stretch that weighs nothing holds no crossing, though its prefix, added
        // in another order, may come out above that of the stretch before it)
        if (s > 0.0 && below + inc > target)
            atomicMin(&first, tid);
        __syncthreads();
        const int f = first;
        if (tid == f)
            first_run = below + (inc - s);
        __syncthreads();
        if (w == 0 && f < kSelThreads) {
            // the blocks of stretch f, 64 at a time; rounding may leave the
            // crossing to none of them: then the last one that holds anything
            double run = first_run;
            const int64_t q0 = f * per, q1 = min(nblocks, q0 + per);
            int64_t hitb = -1, lastb = -1;
            double hitrun = run, lastrun = run;
            for (int64_t c0 = q0; c0 < q1 && hitb < 0; c0 += 64) {
                const double bv = c0 + lane < q1 ? bsum[c0 + lane] : 0.0;
                const double bi = wave_inclusive_f64(bv);
                const uint64_t cross = __ballot(bv > 0.0 && run + bi > target);
                const uint64_t some = __ballot(bv > 0.0);
                const int at = cross ? __ffsll((unsigned long long)cross) - 1
                                     : (some ? 63 - __clzll((long long)some) : -1);
                if (at >= 0) {
                    lastb = c0 + at;
                    lastrun = run + (__shfl(bi, at) - __shfl(bv, at));
                }
                if (cross) {
                    hitb = lastb;
                    hitrun = lastrun;
                }
                run += __shfl(bi, 63);
            }
            if (hitb < 0) {
                hitb = lastb;
                hitrun = lastrun;
            }
            if (hitb >= 0) {
                // the block's rows, four consecutive ones per lane; the block's
                // sum and the running sum can differ in the last bits: then
                // the block's last row with D2 > 0
                double v[4], a = 0.0;
                int pos = -1;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t p = hitb * kKppBlock + lane * 4 + i;
                    v[i] = p < n ? D2[p] : 0.0;
                    a += v[i];
                    pos = v[i] > 0.0 ? lane * 4 + i : pos;
                }
                double at = hitrun + (wave_inclusive_f64(a) - a);
                int hit = 1 << 20;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    at += v[i];
                    if (hit == 1 << 20 && at > target && v[i] > 0.0)
                        hit = lane * 4 + i;
                }
                const uint64_t hm = __ballot(hit != 1 << 20);
                const int last = wave_max(pos);
                const int h = hm ? __shfl(hit, __ffsll((unsigned long long)hm) - 1) : last;
                if (lane == 0 && h >= 0)
                    found = hitb * kKppBlock + h;
            }
        }
        __syncthreads();
        if (tid == 0 && found < 0) {
            int64_t p = -1;
            for (int64_t q = n - 1; q >= 0; --q)
                if (D2[q] > 0.0) {
                    p = q;
                    break;
                }
            found = p < 0 ? 0 : p;
        }
    }
    __syncthreads();
    const int64_t p = found;
    if (blockIdx.x == 0 && tid == 0)
        picks[r] = (int32_t)p;
    if constexpr (PRUNE) {
        const int sub = tid & 15;
        for (int q = blockIdx.x * (kSelThreads / 16) + (tid >> 4); q < r; q += gridDim.x * (kSelThreads / 16)) {
            const double e = kacc64<KIND>(X + (int64_t)picks[q] * ld, X + p * ld, d, sub);
            // half the distance: e is the squared distance (Gaussian) or the distance
            const double h = (KIND == MBKK_GAUSS ? 0.25 : 0.5) * (1.0 - 2e-9) * e;
            if (sub == 0)
                thr[q] = ((1.0 - 2.0 * exp(-h / param)) + 1.0) - 1e-14;
        }
    }
}

// Rows of X that a workgroup of the pruned update takes: 1024 from half a
// million rows on, where the scan of D2 and the ranks is most of a round and
// there are workgroups enough, else 256.
constexpr int64_t kKppWideRows = 1 << 19;

template <int KIND>
static void launch_kpp_prune(const Layout &L, const Buffers &B, int r, double param, hipStream_t st)
{
    const bool v4 = ((uintptr_t)B.X & 15) == 0 && B.ld % 4 == 0;
    const int nq = L.n >= kKppWideRows ? 4 : 1;
    const dim3 grid((unsigned)((L.n + nq * kKppBlock - 1) / (nq * kKppBlock)));
#define MBKK_KPRUNE(LPR, V4, NQ)                                                                                  \
    hipLaunchKernelGGL((k_kpp_prune<KIND, LPR, V4, NQ>), grid, dim3(256), 0, st, B.X, L.n, L.d, B.ld, param, B.picks, \
                       r, B.Nsig, (int32_t *)B.kself, B.D2, B.bsum)
    // 8 lanes cover a row of up to 32 coordinates with one 16-byte load each
    if (v4 && L.d <= 32) {
        if (nq == 4)
            MBKK_KPRUNE(8, true, 4);
        else
            MBKK_KPRUNE(8, true, 1);
    } else if (v4) {
        if (nq == 4)
            MBKK_KPRUNE(16, true, 4);
        else
            MBKK_KPRUNE(16, true, 1);
    } else {
        if (nq == 4)
            MBKK_KPRUNE(16, false, 4);
        else
            MBKK_KPRUNE(16, false, 1);
    }
#undef MBKK_KPRUNE
}

void launch_kpp_round(const Layout &L, const Buffers &B, int r, int kind, double param, hipStream_t st)
{
    // r == 0: select the first pick; r >= 1: update with pick r-1, then select pick r
    const int64_t nblocks = (L.n + kKppBlock - 1) / kKppBlock;
    if (r > 0) {
#define MBKK_KUPD(K)                                                                                     \
    hipLaunchKernelGGL(k_kpp_update<K>, dim3((unsigned)nblocks), dim3(kKppBlock), 0, st, B.X, L.n, L.d, B.ld, \
                       param, B.picks, r - 1, B.kself, B.D2, B.bsum)
        switch (kind) {
        case MBKK_GAUSS: launch_kpp_prune<MBKK_GAUSS>(L, B, r - 1, param, st); break;
        case MBKK_LAPLACE: launch_kpp_prune<MBKK_LAPLACE>(L, B, r - 1, param, st); break;
        case MBKK_LINEAR: MBKK_KUPD(MBKK_LINEAR); break;
        default: MBKK_KUPD(MBKK_POLY2); break;
        }
#undef MBKK_KUPD
    }
    // the thresholds' array is scratch here (mbkk_init_kmeanspp drops the self
    // norms at a bandwidth that it may hold)
    const bool prune = (kind == MBKK_GAUSS || kind == MBKK_LAPLACE) && r > 0 && r + 1 < L.k;
    const dim3 grid(prune ? (unsigned)((r + kSelThreads / 16 - 1) / (kSelThreads / 16)) : 1u);
#define MBKK_KSEL(K, PR)                                                                                          \
    hipLaunchKernelGGL((k_kpp_select<K, PR>), grid, dim3(kSelThreads), 0, st, L.n, nblocks, B.u, r, B.D2, B.bsum, \
                       B.picks, B.X, L.d, B.ld, param, B.Nsig)
    if (!prune)
        MBKK_KSEL(MBKK_GAUSS, false);
    else if (kind == MBKK_GAUSS)
        MBKK_KSEL(MBKK_GAUSS, true);
    else
        MBKK_KSEL(MBKK_LAPLACE, true);
#undef MBKK_KSEL
}

}  // namespace mbkk
