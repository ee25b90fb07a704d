// FP64 re-scoring of near ties (BF16 forms).  A row whose two best distances
// are closer than its bound gets the cross term of every candidate center
// (those whose approximate distance lies within the bound of the best)
// recomputed in FP64 from the FP32 coordinates: direct ||x - y||^2, FP64 exp,
// FP64 weights.  Its distances then carry only the error of N_j.
//
// What bounds it: a few rows of a launch are re-scored, so one row's chain of
// loads, and where a center has collapsed (a candidate of 10^4 entries) the
// FP64 rate of the compute units at work on it.  So a row of little work is
// done by the scoring workgroup that found it (kernels_score.hip), all 16 waves
// together (3 us a row), or a wave to each where it has many that can't be listed; a
// row of much work is listed for a later launch, the update's own where the small
// one runs (kernels_prep.hip), else k_rescore, and split over up to 16 of its
// workgroups.  (At most as many centers as the launch has threads per workgroup, 512
// in k_rescore: with more, a listed row is one workgroup's.)  That launch's chain is
// 20 us long, but it is the same for 1 and for 30 rows.  (In the scoring kernel with
// one wave per row and a lane per entry, a launch that re-scored any row took 35 us
// more, and up to 900 us with a collapsed center; 1M x 128, k = 100, b = 4096.)  An
// entry's row is read by 16 lanes (whole 256-byte stretches), and one exp serves 64
// entries.
#pragma once

#include "cross_layout.h"
#include "dev_common.h"

namespace mbkk {

constexpr int kRescoreChunk = 1024;   // centers whose candidates are listed at once
constexpr int kRescoreMaxWaves = 16;  // waves of a workgroup at most
constexpr int kRescoreWGs = 256;      // workgroups that share the listed rows
constexpr int kRescoreThreads = 512;  // threads of a k_rescore workgroup
constexpr int kRescoreMaxCand = 16;   // most candidates of a row that is split
constexpr int kRescoreMaxParts = 16;  // most workgroups per row
// Candidate entries up to which the scoring workgroup takes a row itself, its
// rows together: its 16 waves need about 12 us for that many, a chain of load
// latencies, against 10 to 25 us for the listed rows of the launch, however many.
constexpr int kRescoreOwnEntries = 2048;

__device__ __forceinline__ bool lex_less(double a, int la, double b, int lb)
{
    return a < b || (a == b && la < lb);
}

// A split row's candidates (in center order) and the smallest approximate
// distance of the other centers; n = 0: the row is finished.
struct RescoreRec {
    int n, pad;
    double outside;
    int cand[kRescoreMaxCand];
};

struct RescoreArgs {
    int k, dp, nb, RB, nranges, ldp;
    double kappa;
    const float *part;
    const float *bat32, *pool32;
    const int32_t *seg_off, *sup_row;
    const double *sup_w64, *N;
    // the listed rows (split: whether any may be), their thresholds, and ctr: rows
    // listed, workgroups done
    // (both 0 between the launches that use them)
    int32_t *list;
    double *delta;
    int32_t *ctr;
    // scratch of the split rows: sums [row, part][candidate] and records
    int split;  // 0: no room, no row is listed
    double *psum;
    RescoreRec *rec;
    // outputs: the library's arrays, the caller's and every distance (each may
    // be NULL), and the grouping ranks and counts (rank may be NULL)
    int32_t *labels, *labels_out;
    float *mind, *margin, *mind_out, *margin_out;
    double *Dout;
    int64_t ldD;
    int32_t *rank, *gcnt;
    unsigned long long *nresc;
};

// Stores that workgroups of other XCDs read in the same launch: agent scope,
// through the XCD's L2.  What workgroups hand over in a launch is ordered by
// these, by each wave's wait for its stores before its workgroup arrives at
// ctr[1], and by nothing else: no release or acquire.  So labels, mind and
// margin of listed rows, rec, psum and ctr[1] are accessed with store_agent,
// load_agent and atomics only, until the last workgroup to arrive has written
// the listed rows again (write_row) and may read them plainly; Dout and the
// caller's arrays are not read in the launch, and the list, its thresholds, the
// partials and the centers' arrays come from earlier launches.
template <typename T>
__device__ __forceinline__ void store_agent(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T load_agent(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One wave's FP64 sum of w K(x, y) over its share of the entries [s0, s1), one
// of `parts` waves: lane (grp, sub) owns entry c0 + 4 (parts sub + pt) + grp of
// each stretch of 64 parts entries.  The wave takes four entries' rows at a
// time, 16 lanes each, four such groups in flight, then one exp with every lane
// holding an entry of its own.  An entry's place in the sum counts from s0,
// so centers with equal entries get equal sums.
__device__ __forceinline__ double rescore_entries(const RescoreArgs &A, const f32x4 *__restrict__ x4, int s0, int s1,
                                                  int parts, int pt)
{
    const int lane = threadIdx.x & 63, grp = lane >> 4, sub = lane & 15;
    const int n4 = A.dp / 4;  // rows are zero past d up to the padded stride
    constexpr int EU = 4;     // entries per lane group in flight: the loop is a chain of load latencies
    double p = 0.0;
    for (int c0 = s0; c0 < s1; c0 += 64 * parts) {
        const int own = c0 + 4 * (parts * sub + pt) + grp;
        const double we = own < s1 ? A.sup_w64[own] : 0.0;
        const int re = own < s1 ? A.sup_row[own] : 0;
        double d2 = 0.0;
        const int left = s1 - c0 - 4 * pt;  // entries from the wave's first one on
        const int nit = min(16, left <= 0 ? 0 : (left + 4 * parts - 1) / (4 * parts));
        for (int it = 0; it < nit; it += EU) {  // wave uniform
            // (entry it + EU - 1 <= 15: past the range its lane owns no entry)
            const f32x4 *y4[EU];
            double e[EU];
#pragma unroll
            for (int q = 0; q < EU; ++q) {
                y4[q] = (const f32x4 *)(A.pool32 + (int64_t)__shfl(re, 16 * grp + it + q) * A.dp);
                e[q] = 0.0;
            }
#pragma nounroll
            for (int t = sub; t < n4; t += 16) {
                const f32x4 a = x4[t];
                f32x4 c[EU];
#pragma unroll
                for (int q = 0; q < EU; ++q)
                    c[q] = y4[q][t];
#pragma unroll
                for (int q = 0; q < EU; ++q)
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const double v = (double)a[u] - (double)c[q][u];
                        e[q] = fma(v, v, e[q]);
                    }
            }
#pragma unroll
            for (int q = 0; q < EU; ++q) {
                e[q] += dpp_f64<0xb1>(e[q]);   // quad_perm [1,0,3,2]
                e[q] += dpp_f64<0x4e>(e[q]);   // quad_perm [2,3,0,1]
                e[q] += dpp_f64<0x141>(e[q]);  // row_half_mirror
                e[q] += dpp_f64<0x140>(e[q]);  // row_mirror
                d2 = sub == it + q ? e[q] : d2;
            }
        }
        if (we != 0.0)
            p += we * exp(-d2 / A.kappa);
    }
    return wave_sum_f64(p);
}

// Smallest value of the 16 lanes of a DPP row.
__device__ __forceinline__ double row_min_f64(double v)
{
    v = fmin(v, dpp_f64<0xb1>(v));     // quad_perm [1,0,3,2]
    v = fmin(v, dpp_f64<0x4e>(v));     // quad_perm [2,3,0,1]
    v = fmin(v, dpp_f64<0x141>(v));    // row_half_mirror
    return fmin(v, dpp_f64<0x140>(v));  // row_mirror
}

// Smallest value over the workgroup (at most 16 waves), the same in every thread.
__device__ __forceinline__ double rescore_min(double v, double *lds)
{
    v = row_min_f64(v);
    v = fmin(v, __shfl_xor(v, 16));
    v = fmin(v, __shfl_xor(v, 32));
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
        lds[threadIdx.x >> 6] = v;
    __syncthreads();
    const int q = threadIdx.x & 15;
    return row_min_f64(lds[min(q, ((int)blockDim.x >> 6) - 1)]);
}

// The running (best, label, second) of a row.
struct RescoreBest {
    double b = INFINITY, s = INFINITY;
    int l = 0x7fffffff;
    __device__ __forceinline__ void take(double D, int j)
    {
        if (D < INFINITY && lex_less(D, j, b, l)) {
            s = b;
            b = D;
            l = j;
        } else if (D < s) {
            s = D;
        }
    }
};

__device__ __forceinline__ void rescore_result(const RescoreArgs &A, int row, const RescoreBest &B, double outside)
{
    store_agent(&A.labels[row], B.l < A.k ? B.l : 0);
    store_agent(&A.mind[row], (float)B.b);
    store_agent(&A.margin[row], (float)(fmin(B.s, outside) - B.b));
}

// LDS of a workgroup that re-scores rows.
struct RescoreLds {
    int *cand;     // [kRescoreChunk]
    double *sum;   // [kRescoreChunk]
    double *min;   // [kRescoreMaxWaves]
    int *cnt;      // [kRescoreMaxWaves]
};

// Whether `rows` rows like this one, of the nc candidates in S.cand, which may not
// be listed, are better taken a wave to each (rescore_row_wave) than one after
// another by the workgroup's waves, 2^lp to a candidate.  In microseconds, by the
// stretches of 64 entries of a candidate: a row costs the workgroup 3.5 and the
// longer of the latencies of its longest candidate's share and of its stretches'
// work; a wave takes 10, and for each stretch dp / 8, its rows being read by single
// lanes.  (10 to 17 rows of 16 stretches in one candidate of 3, 64 coordinates: 290
// us by the workgroup, 160 us by waves; 784 coordinates: 650 and 1540 us.  64 rows of
// 34 stretches in 8 candidates, 32 coordinates: 4.1 and 0.64 ms; 128 coordinates, 33 in
// 2: 2.7 and 2.3 ms.)
__device__ __forceinline__ bool rescore_by_waves(const RescoreArgs &A, const RescoreLds &S, int rows, int nc, int lp,
                                                 const int32_t *__restrict__ seg_off)
{
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    int sum = 0, top = 0;
    for (int i = lane; i < nc; i += 64) {
        const int n = (seg_off[S.cand[i] + 1] - seg_off[S.cand[i]] + 63) / 64;
        sum += n;
        top = max(top, n);
    }
#pragma nounroll
    for (int o = 32; o > 0; o >>= 1) {
        sum += __shfl_xor(sum, o);
        top = max(top, __shfl_xor(top, o));
    }
    const float d = (float)A.dp;
    const float row = 3.5f + fmaxf((float)((top + (1 << lp) - 1) >> lp) * (3.0f + 0.01f * d),
                                   (float)sum * (1.1f + 0.0015f * d));
    const float wave = 10.0f + (float)sum * fmaxf(4.0f, 0.125f * d) + 0.3f * (float)nc;
    return (float)rows * row > (float)((rows + nw - 1) / nw) * wave;
}

// Row `row`, by the whole workgroup.  SCORING: in the scoring workgroup; with
// nothing done, returns kRescoreList if the row is to be listed (more candidate
// entries than `room`, from which a row done is taken), and kRescoreWaves if it
// can't be and the `rows` rows from here on (1: not asked) are better taken a wave
// to each.  Else: listed row q, of which this workgroup takes one part (of 1 << pl;
// all of it in part 0 when pl = 0); returns kRescoreParts when the parts' sums are
// to be put together.  On kRescoreDone (part 0) thread 0 holds the result.
enum { kRescoreDone, kRescoreList, kRescoreWaves, kRescoreParts };
template <int LAYOUT, bool SCORING>
__device__ __forceinline__ int rescore_row(const RescoreArgs &A, const RescoreLds &S, int row, double delta,
                                            double best, int RB, const int32_t *__restrict__ seg_off,
                                            const double *__restrict__ Nv, int q, int pl, int part, int rows, int &room,
                                            RescoreBest &R, double &outside)
{
    const int lane = threadIdx.x & 63, nt = blockDim.x, nw = blockDim.x >> 6;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const f32x4 *x4 = (const f32x4 *)(A.bat32 + (int64_t)row * A.dp);
    auto approx = [&](int j) -> double {  // as the scoring pass had it
        return j < A.k ? 1.0 - 2.0 * cross_of<float, LAYOUT>(A.part, A.ldp, row, j, seg_off, RB) + Nv[j] : INFINITY;
    };
    outside = INFINITY;
    R = RescoreBest{};  // (wave 0's lanes)
    // passes over the centers; a listed row's best comes first, from passes of
    // its own unless there is only one (the code is rarely run, so that its
    // length counts too: it comes from memory)
    const int np = (A.k + nt - 1) / nt;
    int lanes = 64;  // of wave 0 that may hold a candidate's distance
    for (int ps = SCORING || np == 1 ? 0 : -np; ps < np; ++ps) {  // workgroup uniform; nt <= kRescoreChunk
        // the pass's candidates in center order
        const int jl = (ps < 0 ? ps + np : ps) * nt + threadIdx.x;
        const double Dap = approx(jl);
        if (!SCORING && (ps < 0 || np == 1))
            best = fmin(best, rescore_min(Dap, S.min));
        if (ps < 0)
            continue;
        const bool cand = jl < A.k && Dap <= best + delta;
        if (!cand)
            outside = fmin(outside, Dap);
        const uint64_t m = __ballot(cand);
        if (lane == 0)
            S.cnt[w] = __popcll(m);
        __syncthreads();
        int at = 0, nc = 0;
        for (int i = 0; i < nw; ++i) {
            at += i < w ? S.cnt[i] : 0;
            nc += S.cnt[i];
        }
        if (cand)
            S.cand[at + __popcll(m & ((1ull << lane) - 1ull))] = jl;
        __syncthreads();
        const bool split = !SCORING && pl > 0 && nc <= kRescoreMaxCand;  // (pl > 0: one pass)
        if (!SCORING && !split && part > 0)
            return kRescoreParts;
        // waves per candidate: all parts' (split), or all, a half, ... , one of
        // this workgroup's for 1, 2, 3-4, ... candidates
        int lp = 31 - __clz(nw);
        while (!split && lp > 0 && (nc << lp) > nw)
            --lp;
        if constexpr (SCORING) {
            if (A.split && nc <= kRescoreMaxCand) {
                int ne = 0;
                for (int i = 0; i < nc; ++i)
                    ne += seg_off[S.cand[i] + 1] - seg_off[S.cand[i]];
                if (ne > room)
                    return kRescoreList;
                room -= ne;
            } else if (rows > 1 && ps == 0 && rescore_by_waves(A, S, rows, nc, lp, seg_off)) {
                return kRescoreWaves;
            }
        }
        const int pt = split ? part * nw + w : w & ((1 << lp) - 1), waves = split ? nw << pl : 1 << lp;
        for (int ci = w >> lp; ci < nc; ci += nw >> lp) {  // wave uniform
            const int j = S.cand[ci];
            const double p = rescore_entries(A, x4, seg_off[j], seg_off[j + 1], waves, pt);
            if (lane == 0)
                S.sum[(ci << lp) + (w & ((1 << lp) - 1))] = p;
        }
        if (split) {
            __syncthreads();
            if ((int)threadIdx.x < nc) {
                double p = 0.0;
                for (int i = 0; i < nw; ++i)
                    p += S.sum[threadIdx.x * nw + i];
                store_agent(&A.psum[(int64_t)((q << pl) + part) * kRescoreMaxCand + threadIdx.x], p);
                if (part == 0)
                    store_agent(&A.rec[q].cand[threadIdx.x], S.cand[threadIdx.x]);
            }
            if (part == 0) {
                outside = rescore_min(outside, S.min);
                if (threadIdx.x == 0) {
                    store_agent(&A.rec[q].outside, outside);
                    store_agent(&A.rec[q].n, nc);
                }
            }
            __syncthreads();
            return kRescoreParts;
        }
        __syncthreads();
        lanes = np == 1 ? min(nc, 64) : 64;
        if (w == 0) {
            for (int ci = lane; ci < nc; ci += 64) {
                const int j = S.cand[ci];
                double p = 0.0;
                for (int i = 0; i < 1 << lp; ++i)
                    p += S.sum[(ci << lp) + i];
                const double D = 1.0 - 2.0 * p + Nv[j];
                if (A.Dout)
                    A.Dout[(int64_t)row * A.ldD + j] = D;  // replaces the approximate value
                R.take(D, j);
            }
        }
        __syncthreads();
    }
    outside = rescore_min(outside, S.min);
    if (w == 0) {
#pragma nounroll
        for (int o = 1; o < lanes; o <<= 1) {
            const double bq = __shfl_xor(R.b, o), sq = __shfl_xor(R.s, o);
            const int lq = __shfl_xor(R.l, o);
            if (lex_less(bq, lq, R.b, R.l)) {
                R.s = fmin(R.b, sq);
                R.b = bq;
                R.l = lq;
            } else {
                R.s = fmin(R.s, bq);
            }
        }
    }
    __syncthreads();
    return kRescoreDone;
}

// Row `row` by one wave, in the scoring workgroup: a lane per entry, so that 64
// rows' loads are in flight and nothing is added over the lanes but a center's
// sum.  A single row takes several times as long as by the whole workgroup, but 16
// of them are done at a time.  Returns false, with nothing done, if the row is to
// be listed; on true every lane holds the result.
template <int LAYOUT>
__device__ __forceinline__ bool rescore_row_wave(const RescoreArgs &A, int row, double delta, double best, int RB,
                                                 const int32_t *__restrict__ seg_off, const double *__restrict__ Nv,
                                                 RescoreBest &R, double &outside)
{
    const int lane = threadIdx.x & 63;
    const f32x4 *x4 = (const f32x4 *)(A.bat32 + (int64_t)row * A.dp);
    const int n4 = A.dp / 4;  // rows are zero past d up to the padded stride
    auto approx = [&](int j) -> double {  // as the scoring pass had it
        return j < A.k ? 1.0 - 2.0 * cross_of<float, LAYOUT>(A.part, A.ldp, row, j, seg_off, RB) + Nv[j] : INFINITY;
    };
    if (A.split) {
        int nc = 0, ne = 0;
        for (int j0 = 0; j0 < A.k; j0 += 64) {
            const int j = j0 + lane;
            const bool cand = j < A.k && approx(j) <= best + delta;
            nc += __popcll(__ballot(cand));
            ne += cand ? seg_off[j + 1] - seg_off[j] : 0;
        }
#pragma nounroll
        for (int o = 32; o > 0; o >>= 1)
            ne += __shfl_xor(ne, o);
        if (nc <= kRescoreMaxCand && ne > kRescoreOwnEntries)
            return false;
    }
    R = RescoreBest{};
    outside = INFINITY;
    for (int j0 = 0; j0 < A.k; j0 += 64) {
        const double Dap = approx(j0 + lane);
        const bool cand = j0 + lane < A.k && Dap <= best + delta;
        if (!cand)
            outside = fmin(outside, Dap);
        uint64_t m = __ballot(cand);
        while (m) {  // candidates in center order (wave uniform)
            const int j = j0 + __ffsll((unsigned long long)m) - 1;
            m &= m - 1;
            double p = 0.0;
            for (int s = seg_off[j] + lane; s < seg_off[j + 1]; s += 64) {
                const double w = A.sup_w64[s];
                if (w == 0.0)
                    continue;
                const f32x4 *y4 = (const f32x4 *)(A.pool32 + (int64_t)A.sup_row[s] * A.dp);
                double d2 = 0.0;
#pragma unroll 4
                for (int t = 0; t < n4; ++t) {
                    const f32x4 a = x4[t], c = y4[t];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const double v = (double)a[u] - (double)c[u];
                        d2 = fma(v, v, d2);
                    }
                }
                p += w * exp(-d2 / A.kappa);
            }
            const double D = 1.0 - 2.0 * wave_sum_f64(p) + Nv[j];
            if (A.Dout && lane == 0)
                A.Dout[(int64_t)row * A.ldD + j] = D;  // replaces the approximate value
            R.take(D, j);
        }
    }
#pragma nounroll
    for (int o = 32; o > 0; o >>= 1)
        outside = fmin(outside, __shfl_xor(outside, o));
    return true;
}

// A row's label, distance and margin, to the library's arrays and the caller's.
template <typename ARGS>
__device__ __forceinline__ void write_row(const ARGS &A, int row, int label, float mind, float margin)
{
    A.labels[row] = label;
    A.mind[row] = mind;
    A.margin[row] = margin;
    if (A.labels_out)
        A.labels_out[row] = label;
    if (A.mind_out)
        A.mind_out[row] = mind;
    if (A.margin_out)
        A.margin_out[row] = margin;
}

// Grouping ranks of one chunk of 64 rows by one wave: the rank of each row
// among the rows before it with its label, and the chunk's label counts.
__device__ __forceinline__ void rank_chunk(const RescoreArgs &A, int ch)
{
    const int lane = threadIdx.x & 63;
    int32_t *cnt = A.gcnt + (int64_t)ch * A.k;
    for (int j = lane; j < A.k; j += 64)
        cnt[j] = 0;
    __threadfence_block();  // the zeros before the counts
    const int nrow = min(64, A.nb - ch * 64);
    const int Ll = lane < nrow ? A.labels[ch * 64 + lane] : -1;
#pragma nounroll
    for (int r = 0; r < nrow; ++r) {  // wave uniform
        const int Lr = __builtin_amdgcn_readlane(Ll, r);
        const uint64_t m = __ballot(Ll == Lr);
        if (lane == 0) {
            const int rk = __popcll(m & ((1ull << r) - 1ull));
            const int c = __popcll(m);
            A.rank[ch * 64 + r] = rk;
            if (rk == c - 1)
                cnt[Lr] = c;
        }
    }
}

// Finishes the listed rows (nrows: ctr[0], loaded by the caller) with all
// workgroups of the launch.  Returns true in exactly one workgroup: in
// workgroup 0 at once when nothing is listed, else in the last one to arrive
// (every one with a row arrives, none waits for another), which then sees every
// row's final label, distance, rank and count.
template <int LAYOUT>
__device__ __forceinline__ bool rescore_listed(const RescoreArgs &A, int nrows)
{
    __shared__ int s_last;
    __shared__ int s_chunk[kMaxBatch / 64];
    __shared__ int s_cand[kRescoreChunk];
    __shared__ double s_sum[kRescoreChunk];
    __shared__ double s_min[kRescoreMaxWaves];
    __shared__ int s_cnt[kRescoreMaxWaves];
    if (nrows == 0)
        return blockIdx.x == 0;
    // (a row whose centers take the workgroup several passes is not split: its
    // parts would look for the candidates and return)
    int pl = 0;
    while (A.split && A.k <= (int)blockDim.x && (2 << pl) <= kRescoreMaxParts && (nrows << (pl + 1)) <= (int)gridDim.x)
        ++pl;
    // workgroups with no row don't arrive (their counts on one address take
    // their turns: 256 of them 5 us)
    const int nwg = min((int)gridDim.x, nrows << pl);
    if ((int)blockIdx.x >= nwg)
        return false;
    const RescoreLds S{s_cand, s_sum, s_min, s_cnt};
    const int RB = A.nranges > 0 ? bs_range_blocks(A.seg_off[A.k] / 32, A.nranges) : A.RB;
    for (int t = blockIdx.x; t < nrows << pl; t += gridDim.x) {  // workgroup uniform
        const int q = t >> pl, row = A.list[q];
        RescoreBest R;
        double outside;
        int room = 0;
        if (rescore_row<LAYOUT, false>(A, S, row, A.delta[q], INFINITY, RB, A.seg_off, A.N, q, pl,
                                       t & ((1 << pl) - 1), 1, room, R, outside) == kRescoreDone &&
            threadIdx.x == 0) {
            rescore_result(A, row, R, outside);
            if (pl > 0)
                store_agent(&A.rec[q].n, 0);
        }
    }
    // the wave's stores have reached the coherent level before its workgroup
    // arrives (they are agent-scope stores; a release fence here would write
    // the whole L2 back: with 4096 waves doing so it took 70 us)
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0)
        s_last = atomicAdd(&A.ctr[1], 1) == nwg - 1;
    for (int q = threadIdx.x; q < kMaxBatch / 64; q += blockDim.x)
        s_chunk[q] = 0;
    __syncthreads();
    if (!s_last)
        return false;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = blockDim.x >> 6;
    for (int q = w; q < nrows; q += nw) {  // wave uniform
        const int row = A.list[q];
        if (lane == 0)
            s_chunk[row / 64] = 1;
        const int nc = pl > 0 ? load_agent(&A.rec[q].n) : 0;
        if (nc == 0) {
            // finished by its workgroup: written again here, so that this
            // XCD's L2, which may hold the old values, has them too (an acquire
            // fence would empty it before the update's own loads)
            if (lane == 0) {
                const int l = load_agent(&A.labels[row]);
                const float m = load_agent(&A.mind[row]), g = load_agent(&A.margin[row]);
                write_row(A, row, l, m, g);
            }
            continue;
        }
        RescoreBest R;
        for (int ci = 0; ci < nc; ++ci) {
            const int j = load_agent(&A.rec[q].cand[ci]);
            const double v =
                lane < 1 << pl ? load_agent(&A.psum[(int64_t)((q << pl) + lane) * kRescoreMaxCand + ci]) : 0.0;
            const double D = 1.0 - 2.0 * wave_sum_f64(v) + A.N[j];
            if (A.Dout && lane == 0)
                A.Dout[(int64_t)row * A.ldD + j] = D;
            R.take(D, j);
        }
        if (lane == 0) {
            write_row(A, row, R.l < A.k ? R.l : 0, (float)R.b,
                      (float)(fmin(R.s, load_agent(&A.rec[q].outside)) - R.b));
        }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (A.rank) {
        const int nch = (A.nb + 63) / 64;
        for (int ch = w; ch < nch; ch += nw)
            if (s_chunk[ch])
                rank_chunk(A, ch);
    }
    if (threadIdx.x == 0) {
        atomicAdd(A.nresc, (unsigned long long)nrows);
        A.ctr[0] = A.ctr[1] = 0;
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    return true;
}

}  // namespace mbkk
