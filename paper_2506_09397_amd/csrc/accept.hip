// Vocab-parallel acceptance (greedy match or speculative sampling, Eq. 1 of Sec. 3.1).
//
// Four kinds of kernel, the second and third for large and for small batches only:
//   accept_row_stats   (.. _first and _part where a large batch's rows are scanned in parts)
//                      per row of logits (split over a few workgroups when the batch is small) the maximum, its
//                      lowest index, and sum exp((z - max)/tau).  Pure HBM scan: four float4 loads in flight per
//                      thread, wavefront reductions.
//   accept_over        a large batch is scanned in up to four launches that take the requests' rows from the front; between
//                      them this one makes the accept test of the rows so far: where one of them ended the prefix
//                      nothing reads what is behind it.
//   accept_sweep       a batch too small to fill the chip with one workgroup per request has its float64 sums over the
//                      drawn row made here, in two launches, instead of in accept_finish.
//   accept_finish      one workgroup per request.  Its first wavefront applies the accept test (or the
//                      argmax comparison) to all of the request's rows at once, one row per lane, and
//                      takes the first failure.  In sampling mode the workgroup then draws the request's
//                      one token by inverse CDF from the residual max(0, p - q) of the rejecting row (or
//                      from p of the bonus row), all in float64 and in a fixed order, so that the chosen
//                      token does not depend on anything beyond ~1e-15 of the total mass.  With draft
//                      distributions given as a few (token, probability) pairs per draft, the residual's
//                      mass per tile follows from the sums of p and one pass over the pairs.
#include "sled_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

struct RowStat {
    double s;   // sum of exp((z - m) / tau) over the segment
    float m;    // maximum over the segment
    int idx;    // lowest index attaining it
};

// how the rows of a request are cut into segments: rows before `cut` into n0, the others into n1; `stride` statistics lie between two rows
struct Split {
    int n0, n1, cut, stride;
    __host__ __device__ int of(int j) const { return j < cut ? n0 : n1; }
};

template <bool SAMPLE>
__device__ inline void stat_merge(float& m, int& idx, double& s, float m2, int i2, double s2, float inv_tau) {
    if (m2 > m || (m2 == m && i2 < idx)) {
        if (SAMPLE) s = (m == -INFINITY ? 0.0 : s * (double)expf((m - m2) * inv_tau)) + s2;
        m = m2;
        idx = i2;
    } else if (SAMPLE) {
        s += (m2 == -INFINITY ? 0.0 : s2 * (double)expf((m2 - m) * inv_tau));
    }
}

// statistics of a whole row from those of its segments, merged in ascending order
__device__ inline void row_stat(const RowStat* __restrict__ st, int n_split, float inv_tau, float& m, int& amax, double& S) {
    m = st[0].m;
    amax = st[0].idx;
    S = st[0].s;
    for (int sp0 = 1; sp0 < n_split; sp0 += 4) {   // four segments' statistics are requested together
        RowStat r[4];
#pragma unroll
        for (int u = 0; u < 4; u++) r[u] = st[min(sp0 + u, n_split - 1)];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            if (sp0 + u >= n_split || r[u].m == -INFINITY) continue;
            if (r[u].m > m) {  // strictly greater: equal maxima keep the lower index (earlier segment)
                S = S * exp(((double)m - (double)r[u].m) * (double)inv_tau) + r[u].s;
                m = r[u].m;
                amax = r[u].idx;
            } else {
                S += r[u].s * exp(((double)r[u].m - (double)m) * (double)inv_tau);
            }
        }
    }
}

// Where the draft distributions come from: dense rows q[sum k, V], or, per draft, `m` (token id, probability)
// pairs of a distribution that is zero elsewhere (ids distinct; an entry with probability 0 or an id outside
// the vocabulary is padding).
// With `rest` (sparse only): the pairs carry the probabilities as the drafter had them, not renormalised, and
// rest[draft] is the mass of everything not listed, taken to be spread evenly over the unlisted tokens.
struct QSrc {
    const float* dense;
    const int32_t* ids;
    const float* probs;
    const float* rest;
    int m;  // 0: dense
};

__device__ inline bool q_entry_real(int id, float pr, int V) { return id >= 0 && id < V && pr > 0.f; }

// probability of an unlisted token: the remainder mass over the number of unlisted tokens
__device__ inline double q_background(const QSrc& q, int qrow, int V, int n_real) {
    if (!q.rest || n_real >= V) return 0.0;
    return (double)q.rest[qrow] / (double)(V - n_real);
}

// Probability of token d (lane's own) in draft row qrow (lane's own), for the first n lanes; called by a whole wavefront.
// Pairs: as many lanes per row as the n rows leave (8 for up to eight drafts) search its list together, so that the look-up
// is a handful of independent loads instead of m dependent trips; of several equal ids the last one counts.
__device__ inline double q_lookup(const QSrc& q, int qrow, int V, int d, bool want, int n, int lane) {
    if (q.m == 0) return want ? (double)q.dense[(size_t)qrow * V + d] : 0.0;
    int per = 64;
    while (per > 1 && 64 / per < n) per >>= 1;   // lanes per row
    const int r = lane / per, sub = lane & (per - 1);
    const int d_r = __shfl(d, r), qrow_r = __shfl(qrow, r);
    const bool want_r = __shfl((int)want, r) != 0 && r < n;
    int best = -1, n_real = 0;
    float v = 0.f;
    if (want_r) {
        const int32_t* ids = q.ids + (size_t)qrow_r * q.m;
        const float* probs = q.probs + (size_t)qrow_r * q.m;
#pragma unroll 4
        for (int e = sub; e < q.m; e += per) {
            const int id = ids[e];
            const float pr = probs[e];
            if (!q_entry_real(id, pr, V)) continue;
            n_real++;
            if (id == d_r) {
                best = e;
                v = pr;
            }
        }
    }
    for (int off = 1; off < per; off <<= 1) {
        n_real += __shfl_xor(n_real, off);
        const int b2 = __shfl_xor(best, off);
        const float v2 = __shfl_xor(v, off);
        if (b2 > best) {
            best = b2;
            v = v2;
        }
    }
    // back from the searching lanes (r * per) to the lane that asked
    const int from = (lane * per) & 63;
    best = __shfl(best, from);
    v = __shfl(v, from);
    n_real = __shfl(n_real, from);
    if (!want) return 0.0;
    return best >= 0 ? (double)v : q_background(q, qrow, V, n_real);
}

struct __align__(16) KPack {
    uint8_t k[1024];
};

// rows before request i are its drafts and one more per request; every lane gets the drafts before it
__device__ inline int drafts_before(const KPack& kp, int i, int lane) {
    // lane l sums bytes 16 l .. 16 l + 15 below i: one load for all 1024
    const uint4 w = *reinterpret_cast<const uint4*>(kp.k + 16 * lane);
    const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
    int n = 0;
#pragma unroll
    for (int u = 0; u < 4; u++)
#pragma unroll
        for (int e = 0; e < 4; e++) n += 16 * lane + 4 * u + e < i ? (int)((ws[u] >> (8 * e)) & 0xffu) : 0;
    for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off);
    return n;
}

struct Judged {
    bool fail;    // the draft behind this lane's row is rejected ...
    bool close;   // ... or kept by so little that the decision needs the normaliser in float64
    float m;      // the row's maximum
    double zd, lhs;
};

// The accept test of up to 64 drafts of one request at once: lane l judges draft j0+l+1 against row j0+l, for the rows
// below jn (Eq. 1; in greedy mode equality with the row's argmax).
__device__ inline Judged judge_rows(int mode, int row0, int d0, int j0, int jn, int V, const Split& sp, float inv_tau, double it,
                                    const float* __restrict__ logits, const int32_t* __restrict__ tokens, const QSrc& draft_q,
                                    const float* __restrict__ u_acc, const RowStat* __restrict__ stats, int lane) {
    const int j = j0 + lane;
    const bool on = j < jn;
    Judged r{false, false, 0.f, 0.0, 0.0};
    const int d = on ? tokens[row0 + j + 1] : -1;
    const bool real = on && d >= 0 && d < V;
    if (mode == SLED_GREEDY) {
        if (on) {
            int amax;
            double S;
            row_stat(stats + (size_t)(row0 + j) * sp.stride, sp.of(j), inv_tau, r.m, amax, S);
            r.fail = d != amax;
        }
        return r;
    }
    const float zf = real ? logits[(size_t)(row0 + j) * V + d] : 0.f;
    const double qd = q_lookup(draft_q, d0 + j, V, d, real, min(64, jn - j0), lane);
    if (real) {
        int amax;
        double S;
        row_stat(stats + (size_t)(row0 + j) * sp.stride, sp.of(j), inv_tau, r.m, amax, S);
        r.zd = (double)zf;
        const double pd = exp((r.zd - (double)r.m) * it) / S;
        r.lhs = (double)u_acc[d0 + j] * qd;
        r.fail = !(r.lhs <= pd);
        // S carries the float32 round-off of the row scan (about 1e-7): a test this close is decided again
        r.close = fabs(r.lhs - pd) <= 1e-4 * pd;
    } else if (on) {
        r.fail = true;  // a draft outside the vocabulary has no target probability: rejected where it stands
    }
    return r;
}

// e^a in float32 for a <= 0, -inf or NaN, in fewer instructions than expf: a log2(e) = n + f with a whole n and |f| <= 1/2
// (Cody and Waite's reduction: n from a sum with 1.5 x 2^23, whose last bits then hold it; the remainder from fused products
// with log2(e) in two parts), the hardware exponential of f, and n added to the exponent's bits.  Below e^-87, where that would
// leave the normal numbers, 0.  Its relative error over [-85, 0] is 2.66e-8 rms, 8.8e-8 at most (expf: 2.62e-8 and 8.4e-8).
// It serves the acceptance alone, where nothing that it rounds reaches a result: the argmax compares logits, an accept test whose
// sides agree to four digits is decided in float64, and so is every draw.  (The scan of 16 segments per row is bound by the
// exponentials' instructions: with expf 256 requests take 222 us instead of 212, 16 requests 44.7 instead of 42.7.)
__device__ inline float expf_nonpos(float a) {
    constexpr float WHOLE = 12582912.f;
    const float t = fmaf(a, 1.44269502f, WHOLE);
    const float f = fmaf(a, 1.92596303e-8f, fmaf(a, 1.44269502f, WHOLE - t));
    const float e = __uint_as_float(__float_as_uint(__builtin_amdgcn_exp2f(f)) + (__float_as_uint(t) << 23));
    return a < -87.f ? 0.f : e;
}

// statistics of elements v0 .. v1-1 of a row, by the whole workgroup of 256; the sum of exponentials only with SAMPLE, and for a
// result of its own (SHOWN) by expf
// STREAM: the scan in parts reads its rows past the caches' replacement order.  Part of them may be in Infinity Cache, since the LM head has just
// written them, and is found there either way; what the scan reads does not push out the rest.  256 requests x 8 drafts x 128256 tokens (1.2 GB), us, in
// the ordinary order / past it: the same logits again 190 / 185, three sets in turn 204 / 197, rows just written 238 / 217; 128 requests 122 / 127,
// 136 / 135, 150 / 142.
template <bool SAMPLE, bool SHOWN, bool STREAM = false>
__device__ inline void scan_segment(const float* __restrict__ z, bool vec, int v0, int v1, float inv_tau, RowStat* __restrict__ dst) {
    auto e_to = [](float a) { return SHOWN ? expf(a) : expf_nonpos(a); };
    float m = -INFINITY;
    int idx = 0x7fffffff;
    double s = 0.0;

    // a chunk of values in ascending index order: its maximum first, then one rescale of the running sum, then
    // the chunk's terms (summed in float32, as accurate as the float32 exponentials themselves)
    auto take = [&](const float* x, auto n_c, auto index_of) {
        constexpr int n = decltype(n_c)::value;
        float cm = x[0];
        int ce = 0;
#pragma unroll
        for (int e = 1; e < n; e++) {
            const bool gt = x[e] > cm;
            cm = gt ? x[e] : cm;
            ce = gt ? e : ce;
        }
        if (cm > m) {
            if (SAMPLE) s *= (double)e_to((m - cm) * inv_tau);  // m = -inf: s is still 0
            m = cm;
            idx = index_of(ce);
        }
        if (SAMPLE) {
            float cs = 0.f;
#pragma unroll
            for (int e = 0; e < n; e++) cs += e_to((x[e] - m) * inv_tau);  // padding is -inf: adds 0
            s += (double)cs;
        }
    };

    if (vec) {
        // v0 is a multiple of 4 and rows are 16-byte aligned
        const float4* z4 = reinterpret_cast<const float4*>(z);
        const int e4 = v1 / 4;
        for (int v = v0 / 4 + threadIdx.x; v < e4; v += 256 * 4) {
            float4 q[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int vv = v + 256 * u;
                q[u] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
                if (vv < e4) {
                    if (STREAM) {
                        const float4_t y = __builtin_nontemporal_load(reinterpret_cast<const float4_t*>(z4 + vv));
                        q[u] = make_float4(y[0], y[1], y[2], y[3]);
                    } else {
                        q[u] = z4[vv];
                    }
                }
            }
            const float x[16] = {q[0].x, q[0].y, q[0].z, q[0].w, q[1].x, q[1].y, q[1].z, q[1].w,
                                 q[2].x, q[2].y, q[2].z, q[2].w, q[3].x, q[3].y, q[3].z, q[3].w};
            take(x, std::integral_constant<int, 16>{}, [&](int e) { return 4 * (v + 256 * (e >> 2)) + (e & 3); });
        }
    } else {
        for (int v = v0 + threadIdx.x; v < v1; v += 256) {
            const float x = z[v];
            take(&x, std::integral_constant<int, 1>{}, [&](int) { return v; });
        }
    }
    if (idx == 0x7fffffff) {  // this thread saw nothing
        m = -INFINITY;
        s = 0.0;
    }
    // over the wavefront, then across the 4 wavefronts through LDS: the maximum first, so that each sum is rescaled once
    auto rescaled = [&](double s2, float m2, float top) { return m2 == -INFINITY ? 0.0 : m2 == top ? s2 : s2 * (double)e_to((m2 - top) * inv_tau); };
    float top = m;
    for (int off = 32; off > 0; off >>= 1) top = fmaxf(top, __shfl_xor(top, off));
    int first = m == top ? idx : 0x7fffffff;   // of equal maxima the lowest index
    for (int off = 32; off > 0; off >>= 1) first = min(first, __shfl_xor(first, off));
    if (SAMPLE) {
        s = rescaled(s, m, top);
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    }
    __shared__ float sm[4];
    __shared__ int si[4];
    __shared__ double ss[4];
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sm[w] = top;
        si[w] = first;
        ss[w] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        RowStat r{0.0, fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3])), 0x7fffffff};
        for (int i = 0; i < 4; i++) {
            if (sm[i] == r.m) r.idx = min(r.idx, si[i]);
            if (SAMPLE) r.s += rescaled(ss[i], sm[i], r.m);
        }
        *dst = r;
    }
}

// Between two parts of the row scan: over[i] = 1 where one of request i's rows before jn, which the parts so far have scanned
// (or left out behind a rejection that this test sees first), ends the prefix for certain.  A close test, which the finish
// decides, ends nothing here.  One wavefront per request.
__global__ __launch_bounds__(64) void accept_over(int mode, KPack kp, int jn, int V, Split sp, float inv_tau, float temperature,
                                                  const float* __restrict__ logits, const int32_t* __restrict__ tokens, QSrc qsrc,
                                                  const float* __restrict__ u_acc, const RowStat* __restrict__ stats, int32_t* __restrict__ over) {
    const int i = blockIdx.x, lane = threadIdx.x;
    const int d0 = drafts_before(kp, i, lane);
    const Judged jd = judge_rows(mode, d0 + i, d0, 0, min(jn, (int)kp.k[i]), V, sp, inv_tau, 1.0 / (double)temperature, logits, tokens,
                                 qsrc, u_acc, stats, lane);
    const unsigned long long certain = __ballot(jd.fail && !jd.close);
    if (lane == 0) over[i] = certain != 0ull;
}

// blockIdx.x: the packed row
template <bool SAMPLE, bool SHOWN = false>
__global__ __launch_bounds__(256) void accept_row_stats(const float* __restrict__ logits, int V, int n_split, int seg,
                                                        float inv_tau, RowStat* __restrict__ stats) {
    const int split = blockIdx.y;
    const int v0 = split * seg;
    const int v1 = min(V, v0 + seg);
    const bool vec = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0;   // (seg is a multiple of 4)
    scan_segment<SAMPLE, SHOWN>(logits + (size_t)blockIdx.x * V, vec, v0, v1, inv_tau, stats + (size_t)blockIdx.x * n_split + split);
}

// The scan in parts.  The first: rows 0 .. of every request, blockIdx.x = request + B * row of the request.
template <bool SAMPLE>
__global__ __launch_bounds__(256) void accept_row_stats_first(const float* __restrict__ logits, int V, Split sp, float inv_tau, int B, KPack kp,
                                                              RowStat* __restrict__ stats) {
    const int split = blockIdx.y, seg = ((V + sp.n0 - 1) / sp.n0 + 3) & ~3;
    const bool vec = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0;
    // Workgroups go to the XCDs round robin, so with a batch of a multiple of eight all rows and segments of a request would
    // meet on one of them: turned by row and segment.
    const int j = blockIdx.x / B, i = (blockIdx.x - j * B + j + 3 * split) % B;
    if (j > kp.k[i]) return;
    const int row = drafts_before(kp, i, threadIdx.x & 63) + i + j;
    const int v0 = min(V, split * seg), v1 = min(V, v0 + seg);
    scan_segment<SAMPLE, false, true>(logits + (size_t)row * V, vec, v0, v1, inv_tau, stats + (size_t)row * sp.stride + split);
}

// The later parts: rows j0 .. j1-1 of the requests that no test so far has ended.  How many those are only the GPU
// knows, so a fixed number of workgroups deals them out by itself: every workgroup adds up the rows that are left (four requests to a
// thread) and takes items blockIdx.x, + gridDim.x, .. of (row, segment), the segment running slowest, so that neighbouring workgroups,
// which go to different XCDs, have different rows.  Few rows are left behind a cut, so they are cut finer than the first
// ones (Split): a workgroup's own time for a long segment is what such a launch takes.  256 requests x 8 drafts x 128256 tokens, 62 %
// accepted: rows 2, 3 take 23.5 us and rows 4 .. 8 23.7, 33.1 and 36.4 as launches of a workgroup for every row and segment there might be
// (their 170 and 190 rows are 15 and 17 us at a large copy's rate).
// (One workgroup for all of a request's rows of a part: 93 us for rows 4 .. 8.  Making the test in each workgroup instead of ahead of
// the launch: 59 us.)
template <bool SAMPLE>
__global__ __launch_bounds__(256) void accept_row_stats_part(const float* __restrict__ logits, int V, Split sp, float inv_tau, int B, int j0,
                                                             int j1, KPack kp, const int32_t* __restrict__ over, RowStat* __restrict__ stats) {
    __shared__ int sh_sum[2][4], sh_row;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const uint32_t ks = reinterpret_cast<const uint32_t*>(kp.k)[tid];
    int left[4], rows[4], mine = 0, mine_rows = 0;
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const int i = 4 * tid + e, k = (int)((ks >> (8 * e)) & 0xffu);
        const bool live = i < B && !over[i];
        rows[e] = i < B ? k + 1 : 0;
        left[e] = live ? max(0, min(j1, k + 1) - j0) : 0;
        mine += left[e];
        mine_rows += rows[e];
    }
    int before = mine, before_rows = mine_rows;   // running sums over the threads
    for (int off = 1; off < 64; off <<= 1) {
        const int a = __shfl_up(before, off), b = __shfl_up(before_rows, off);
        if (lane >= off) {
            before += a;
            before_rows += b;
        }
    }
    if (lane == 63) {
        sh_sum[0][wv] = before;
        sh_sum[1][wv] = before_rows;
    }
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int w = 0; w < 4; w++) {
        if (w < wv) {
            before += sh_sum[0][w];
            before_rows += sh_sum[1][w];
        }
        total += sh_sum[0][w];
    }
    before -= mine;
    before_rows -= mine_rows;
    const int n_split = sp.n1, seg = ((V + n_split - 1) / n_split + 3) & ~3;
    const bool vec = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0;
    for (int item = blockIdx.x; item < total * n_split; item += gridDim.x) {
        const int split = item / total, r = item - split * total;
        int a = before, row0 = before_rows;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            if (r >= a && r < a + left[e]) sh_row = row0 + j0 + (r - a);
            a += left[e];
            row0 += rows[e];
        }
        __syncthreads();
        const int row = sh_row;
        const int v0 = min(V, split * seg), v1 = min(V, v0 + seg);
        scan_segment<SAMPLE, false, true>(logits + (size_t)row * V, vec, v0, v1, inv_tau, stats + (size_t)row * sp.stride + split);
        __syncthreads();   // sh_row and the scan's own words have been read
    }
}

struct Decision {
    int a;       // accepted prefix length
    int row;     // packed row the output token comes from (row0 + a)
    int qrow;    // draft row whose q is subtracted there, or -1 (all accepted: bonus row)
    float m;     // that row's maximum
    int amax;    // and its argmax
};

// One wavefront decides one request: the first failing lane of judge_rows ends the accepted prefix.
__device__ inline Decision decide_request(int mode, int i, const KPack& kp, int V, const Split& sp, float inv_tau, double it,
                                          const float* __restrict__ logits, const int32_t* __restrict__ tokens,
                                          const QSrc& draft_q, const float* __restrict__ u_acc,
                                          const RowStat* __restrict__ stats, int lane) {
    const int d0 = drafts_before(kp, i, lane);   // drafts before this request
    const int row0 = d0 + i;                     // rows before it: one more per request
    const int k = kp.k[i];
    int a = k;
    for (int j0 = 0; j0 < k; j0 += 64) {
        const Judged jd = judge_rows(mode, row0, d0, j0, k, V, sp, inv_tau, it, logits, tokens, draft_q, u_acc, stats, lane);
        bool fail = jd.fail;
        // Rare: the two sides of Eq. 1 agree to four digits.  The whole wavefront then sums the row's normaliser in
        // float64, in a fixed order (lane-strided partial sums, then a butterfly), and the lane decides again.  Rows
        // behind the first certain rejection do not matter (and may not have been scanned).
        const unsigned long long certain = __ballot(jd.fail && !jd.close);
        unsigned long long todo = __ballot(jd.close);
        if (certain) todo &= (certain & (0ull - certain)) - 1ull;
        while (todo) {
            const int src = __ffsll((long long)todo) - 1;
            todo &= todo - 1;
            const float ms = __shfl(jd.m, src);
            const float* z = logits + (size_t)(row0 + j0 + src) * V;
            double part = 0.0;
            for (int v = lane; v < V; v += 64) part += exp(((double)z[v] - (double)ms) * it);
            for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
            if (lane == src) fail = !(jd.lhs <= exp((jd.zd - (double)jd.m) * it) / part);
        }
        const unsigned long long mask = __ballot(fail);
        if (mask) {
            a = j0 + __ffsll((long long)mask) - 1;
            break;
        }
    }
    Decision dc;
    dc.a = a;
    dc.row = row0 + a;
    dc.qrow = a < k ? d0 + a : -1;
    double S;
    row_stat(stats + (size_t)dc.row * sp.stride, sp.of(a), inv_tau, dc.m, dc.amax, S);
    return dc;
}

constexpr int SLED_SPARSE_Q_MAX = 1024;  // entries per draft of a sparse draft distribution
constexpr int WTILE = 1024;        // elements per wavefront tile: 16 consecutive ones per lane
constexpr int MAX_WTILES = 2048;   // covers vocabularies up to 2 097 152

// the row a request's token is drawn from, as the float64 sweeps see it
struct RowView {
    const float* z;
    const float* q;    // dense draft distribution of the rejected draft, or nullptr
    double m, it;
    int V;
    bool vec;          // rows of z and q are 16-byte aligned
};

// Sums over tiles t0, t0 + step, .. of exp((z - m)/tau) (proportional to p), or with `residual` of max(0, p - q), p = that *
// inv_S (qconst >= 0: against the same q everywhere -- the background of a sparse q with remainder mass); by one wavefront,
// into out[t].  Loads are whole KiB, and with AHEAD those of the next tile are under way while this one's exponentials are computed;
// the order of the additions within a tile is fixed (16 values of a lane, then a butterfly).
template <bool AHEAD>
__device__ inline void sweep_tiles(const RowView& r, bool residual, double inv_S, double qconst, int t0, int t_end, int step,
                                   double* out, int lane) {
    const bool use_q = residual && qconst < 0.0 && r.q;
    auto load = [&](const float* p, int t, float* x, float pad) {   // values 256 u + 4 lane + 0..3 of the tile (64 e + lane when unaligned)
        if (r.vec) {
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int v = t * WTILE + u * 256 + lane * 4;
                float4 y = make_float4(pad, pad, pad, pad);
                if (v < r.V) y = *reinterpret_cast<const float4*>(p + v);
                x[4 * u] = y.x;
                x[4 * u + 1] = y.y;
                x[4 * u + 2] = y.z;
                x[4 * u + 3] = y.w;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const int v = t * WTILE + e * 64 + lane;
                x[e] = v < r.V ? p[v] : pad;
            }
        }
    };
    float zx[16], qx[16], zn[16], qn[16];
    auto fetch = [&](int t) {
#pragma unroll
        for (int e = 0; e < 16; e++) qn[e] = 0.f;
        load(r.z, t, zn, -INFINITY);
        if (use_q) load(r.q, t, qn, 0.f);
    };
    if (AHEAD && t0 < t_end) fetch(t0);
    for (int t = t0; t < t_end; t += step) {
        if (!AHEAD) fetch(t);
#pragma unroll
        for (int e = 0; e < 16; e++) {
            zx[e] = zn[e];
            qx[e] = qn[e];
        }
        if (AHEAD && t + step < t_end) fetch(t + step);
        double acc = 0.0;
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const double ev = exp(((double)zx[e] - r.m) * r.it);  // exp(-inf) = 0 beyond the row
            if (residual) {
                const double d = ev * inv_S - (qconst >= 0.0 ? qconst : (double)qx[e]);
                acc += d > 0.0 ? d : 0.0;
            } else {
                acc += ev;
            }
        }
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
        if (lane == 0) out[t] = acc;
    }
}

// Total of the tile sums by one wavefront (per lane a run of tiles in ascending order, then a scan over the lanes); `incl`,
// `part`: the running sum behind this lane's run, and the run's own
__device__ inline double tile_total(const double* tile_sum, int n_tiles, int lane, double& incl, double& part) {
    const int per = (n_tiles + 63) / 64;
    const int t0 = lane * per, t1 = min(n_tiles, t0 + per);
    part = 0.0;
    for (int t = t0; t < t1; t++) part += tile_sum[t];
    incl = part;
    for (int off = 1; off < 64; off <<= 1) {
        const double o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    return __shfl(incl, 63);
}

// A batch too small to fill the chip with one workgroup per request: the sweeps run as launches of their own, gridDim.y
// workgroups per request, and leave their tile sums in the workspace (per request n_tiles of p, then n_tiles of the residual)
// for accept_finish.  SECOND: the residual's, which need the total of the first; same sums in the same order either way.
template <bool SECOND>
__global__ __launch_bounds__(512) void accept_sweep(KPack kp, int V, Split sp, float inv_tau, float temperature,
                                                    const float* __restrict__ logits, const int32_t* __restrict__ tokens, QSrc qsrc,
                                                    const float* __restrict__ u_acc, const RowStat* __restrict__ stats,
                                                    Decision* __restrict__ decisions, double* __restrict__ tile_sums) {
    __shared__ Decision sh_dc;
    __shared__ double sh_S;
    __shared__ int sh_real;
    const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int n_tiles = (V + WTILE - 1) / WTILE;
    double* sums = tile_sums + (size_t)i * 2 * n_tiles;
    if (tid == 64) sh_real = 0;
    const double it = 1.0 / (double)temperature;
    if (wv == 0) {
        if (SECOND) {
            double incl, part;
            const double S = tile_total(sums, n_tiles, lane, incl, part);
            if (lane == 0) {
                sh_S = S;
                sh_dc = decisions[i];
            }
        } else {
            const Decision dc = decide_request(SLED_SAMPLE, i, kp, V, sp, inv_tau, it, logits, tokens, qsrc, u_acc, stats, lane);
            if (lane == 0) {
                sh_dc = dc;
                if (blockIdx.y == 0) decisions[i] = dc;
            }
        }
    }
    __syncthreads();
    const Decision dc = sh_dc;
    const bool sparse = qsrc.m > 0;
    double qconst = -1.0;
    if (SECOND) {
        if (dc.qrow < 0) return;   // drawn from p
        if (sparse) {
            int n = 0;
            for (int e = tid; e < qsrc.m; e += blockDim.x)
                n += q_entry_real(qsrc.ids[(size_t)dc.qrow * qsrc.m + e], qsrc.probs[(size_t)dc.qrow * qsrc.m + e], V);
            if (n) atomicAdd(&sh_real, n);
            __syncthreads();
            qconst = q_background(qsrc, dc.qrow, V, sh_real);
            if (!(qconst > 0.0)) return;   // accept_finish has the background from the sums of p
        }
    }
    const bool vec = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0 && (reinterpret_cast<uintptr_t>(qsrc.dense) & 15) == 0;
    const RowView rv{logits + (size_t)dc.row * V, dc.qrow >= 0 && !sparse ? qsrc.dense + (size_t)dc.qrow * V : nullptr, (double)dc.m, it, V, vec};
    sweep_tiles<true>(rv, SECOND, SECOND ? 1.0 / sh_S : 1.0, qconst, blockIdx.y * (blockDim.x >> 6) + wv, n_tiles, gridDim.y * (blockDim.x >> 6),
                SECOND ? sums + n_tiles : sums, lane);
}

__global__ __launch_bounds__(1024) void accept_finish(int mode, KPack kp, int V, Split sp, float inv_tau, float temperature,
                                                      const float* __restrict__ logits, const int32_t* __restrict__ tokens,
                                                      QSrc qsrc, const float* __restrict__ u_acc,
                                                      const float* __restrict__ u_smp, const RowStat* __restrict__ stats,
                                                      int32_t* __restrict__ accept_len, int32_t* __restrict__ out_token,
                                                      const Decision* __restrict__ decisions, const double* __restrict__ tile_sums) {
    __shared__ double tile_sum[MAX_WTILES];
    __shared__ double sp_take[SLED_SPARSE_Q_MAX];   // sparse q: probability mass entry i removes from p
    __shared__ __align__(16) int sp_tile[SLED_SPARSE_Q_MAX];   //           and the tile it falls in (-1: padding)
    __shared__ double q_tile[WTILE];                //           q over the tile that holds the draw
    __shared__ Decision sh_dc;
    __shared__ int sh_tile;
    __shared__ double sh_base, sh_total;
    const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, n_wv = blockDim.x >> 6;
    if (wv == 0) {
        // float64 work divides by the temperature as given (a float32 number), exactly as a float64 reference does
        const Decision dc = decisions ? decisions[i]   // accept_sweep has decided
                                      : decide_request(mode, i, kp, V, sp, inv_tau, 1.0 / (double)temperature, logits, tokens, qsrc, u_acc, stats, lane);
        if (lane == 0) {
            sh_dc = dc;
            accept_len[i] = dc.a;
            if (mode == SLED_GREEDY) out_token[i] = dc.amax;
        }
    }
    if (mode == SLED_GREEDY) return;
    __syncthreads();
    const Decision dc = sh_dc;
    const float* z = logits + (size_t)dc.row * V;
    const bool sparse = qsrc.m > 0;
    const bool has_q = dc.qrow >= 0;
    const float* q = (has_q && !sparse) ? qsrc.dense + (size_t)dc.qrow * V : nullptr;
    const double m = (double)dc.m, it = 1.0 / (double)temperature;
    const int n_tiles = (V + WTILE - 1) / WTILE;  // at most MAX_WTILES: the host rejects larger vocabularies
    const bool vec = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0 &&
                     (reinterpret_cast<uintptr_t>(qsrc.dense) & 15) == 0;

    // 16 consecutive values of a row starting at v (0 beyond the end of the row when `pad0`, else -inf)
    auto load16 = [&](const float* p, int v, float* x, float pad) {
        if (vec) {
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int vv = v + 4 * u;
                float4 t = make_float4(pad, pad, pad, pad);
                if (vv < V) t = *reinterpret_cast<const float4*>(p + vv);
                x[4 * u] = t.x;
                x[4 * u + 1] = t.y;
                x[4 * u + 2] = t.z;
                x[4 * u + 3] = t.w;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 16; e++) x[e] = (v + e < V) ? p[v + e] : pad;
        }
    };
    // this lane's 16 weights of tile t: exp((z - m)/tau) (proportional to p), or max(0, p - q) with p = that / S
    // (with sparse q the residual is only ever needed inside the tile that holds the draw, whose q is in q_tile)
    auto weights = [&](int t, bool residual, double inv_S, double* w) {
        const int v = t * WTILE + lane * 16;
        float zx[16], qx[16];
        load16(z, v, zx, -INFINITY);
        if (residual && !sparse) load16(q, v, qx, 0.f);
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const double ev = exp(((double)zx[e] - m) * it);  // exp(-inf) = 0 beyond the row
            if (residual) {
                const double r = ev * inv_S - (sparse ? q_tile[lane * 16 + e] : (double)qx[e]);
                w[e] = r > 0.0 ? r : 0.0;
            } else {
                w[e] = ev;
            }
        }
    };
    const RowView rv{z, q, m, it, V, vec};
    // every wavefront sums whole tiles: no workgroup barrier per tile; or accept_sweep has summed them
    auto sweep = [&](bool residual, double inv_S, double qconst = -1.0) {
        if (tile_sums) {
            const double* src = tile_sums + ((size_t)i * 2 + (residual ? 1 : 0)) * n_tiles;
            for (int t = tid; t < n_tiles; t += blockDim.x) tile_sum[t] = src[t];
        } else {
            sweep_tiles<false>(rv, residual, inv_S, qconst, wv, n_tiles, n_wv, tile_sum, lane);
        }
        __syncthreads();
    };
    // wavefront 0: total of the tile sums (ascending), the tile in which the running sum first exceeds
    // u * total, and the running sum before that tile
    auto locate = [&](double u) {
        if (wv == 0) {
            const int per = (n_tiles + 63) / 64;
            const int t0 = lane * per, t1 = min(n_tiles, t0 + per);
            double incl, part;
            const double total = tile_total(tile_sum, n_tiles, lane, incl, part);
            const double target = u * total;
            const unsigned long long mask = __ballot(incl > target && t1 > t0);
            // round-off can leave no lane past the target: then the last tile holds the crossing
            const int owner = mask ? __ffsll((long long)mask) - 1 : (n_tiles - 1) / per;
            if (lane == owner) {
                double c = incl - part;
                int tt = t1 - 1;
                for (int t = t0; t < t1; t++) {
                    if (c + tile_sum[t] > target) {
                        tt = t;
                        break;
                    }
                    if (t < t1 - 1) c += tile_sum[t];
                }
                sh_tile = tt;
                sh_base = c;
                sh_total = total;
            }
        }
        __syncthreads();
    };

    const double u = (double)u_smp[i];
    double qbg = 0.0;   // sparse q with remainder mass: probability of a token that is not listed
    bool residual = false;
    double inv_S = 1.0;
    sweep(false, 1.0);  // tile sums of exp((z - m)/tau); their total is the normaliser S
    locate(u);
    if (has_q) {
        const double S = sh_total;
        __syncthreads();  // everybody has read the total before the tile sums are replaced
        if (!sparse) {
            sweep(true, 1.0 / S);
        } else {
            // sum over a tile of max(0, p - q) = background - sum over the entries in it of what listing them takes
            // away, where the background is the tile's residual against the probability c of an unlisted token.
            // Without remainder mass c = 0: the background is the sum of p, known from the first sweep, and an entry
            // takes min(p, q) -- one pass over the m entries instead of a second pass over the vocabulary.  With
            // remainder mass the background needs that second pass (against the constant c), and an entry takes
            // max(0, p - c) - max(0, p - q).
            const int32_t* ids = qsrc.ids + (size_t)dc.qrow * qsrc.m;
            const float* pr = qsrc.probs + (size_t)dc.qrow * qsrc.m;
            // (a workgroup has a thread for every entry a row can have)
            const int n_real = __syncthreads_count(tid < qsrc.m && q_entry_real(ids[tid < qsrc.m ? tid : 0], pr[tid < qsrc.m ? tid : 0], V));
            qbg = q_background(qsrc, dc.qrow, V, n_real);
            if (qbg > 0.0) {
                sweep(true, 1.0 / S, qbg);
            }
            if (tid >= qsrc.m && tid < ((qsrc.m + 3) & ~3)) sp_tile[tid] = -1;
            for (int e = tid; e < qsrc.m; e += blockDim.x) {
                const int id = ids[e];
                const double qv = (double)pr[e];
                const bool real = q_entry_real(id, pr[e], V);
                double take = 0.0;
                if (real) {
                    const double pv = exp(((double)z[id] - m) * it) * (1.0 / S);
                    const double with_c = pv > qbg ? pv - qbg : 0.0, with_q = pv > qv ? pv - qv : 0.0;
                    take = with_c - with_q;
                }
                sp_take[e] = take;
                sp_tile[e] = real ? id / WTILE : -1;
            }
            __syncthreads();
            for (int t = tid; t < n_tiles; t += blockDim.x) {
                double r = qbg > 0.0 ? tile_sum[t] : tile_sum[t] * (1.0 / S);
                for (int e = 0; e < qsrc.m; e += 4) {   // in entry order: the result does not depend on the thread layout
                    const int4 te = *reinterpret_cast<const int4*>(sp_tile + e);   // (the tail up to a multiple of 4 is padding)
                    if (te.x == t) r -= sp_take[e];
                    if (te.y == t) r -= sp_take[e + 1];
                    if (te.z == t) r -= sp_take[e + 2];
                    if (te.w == t) r -= sp_take[e + 3];
                }
                tile_sum[t] = r > 0.0 ? r : 0.0;
            }
            __syncthreads();
        }
        locate(u);
        if (sh_total > 0.0) {
            residual = true;
            inv_S = 1.0 / S;
        } else {
            // the residual has no mass (p <= q everywhere up to round-off): draw from p instead
            __syncthreads();
            sweep(false, 1.0);
            locate(u);
        }
    }
    if (residual && sparse) {
        // q over the tile of the draw, dense in LDS
        const int tt0 = sh_tile;
        for (int e = tid; e < WTILE; e += blockDim.x) q_tile[e] = qbg;
        __syncthreads();
        const int32_t* ids = qsrc.ids + (size_t)dc.qrow * qsrc.m;
        const float* pr = qsrc.probs + (size_t)dc.qrow * qsrc.m;
        for (int e = tid; e < qsrc.m; e += blockDim.x)
            if (sp_tile[e] == tt0) q_tile[ids[e] - tt0 * WTILE] = (double)pr[e];   // (ids are distinct within a row)
        __syncthreads();
    }
    if (wv != 0) return;
    // inside the tile: 16 weights per lane, an ordered scan over the lanes, then over the lane's own 16
    const int tt = sh_tile;
    const double target = u * sh_total;
    double w[16];
    weights(tt, residual, inv_S, w);
    double part = 0.0;
#pragma unroll
    for (int e = 0; e < 16; e++) part += w[e];
    double incl = part;
    for (int off = 1; off < 64; off <<= 1) {
        const double o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    const unsigned long long cross = __ballot(sh_base + incl > target);
    int found = -1;
    if (cross) {
        const int owner = __ffsll((long long)cross) - 1;
        if (lane == owner) {
            double c = sh_base + (incl - part);
            for (int e = 0; e < 16 && found < 0; e++) {
                if (c + w[e] > target) found = tt * WTILE + lane * 16 + e;
                else c += w[e];
            }
        }
        found = __shfl(found, owner);
    }
    if (found < 0) {
        // round-off between the two summation orders hid the crossing: the last index of the tile that carries
        // weight (of the row, if the tile carries none)
        int last = -1;
        for (int e = 15; e >= 0; e--)
            if (w[e] > 0.0) {
                last = tt * WTILE + lane * 16 + e;
                break;
            }
        for (int off = 32; off > 0; off >>= 1) last = max(last, __shfl_xor(last, off));
        found = last >= 0 ? last : dc.amax;
    }
    if (lane == 0) out_token[i] = found;
}

// confidence of every row: 1 / sum exp((z - max) / tau) is the probability of the most likely token
__global__ void row_confidence_finish(const RowStat* __restrict__ stats, int T, int n_split, float inv_tau,
                                      float* __restrict__ conf, int32_t* __restrict__ top) {
    const int row = blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= T) return;
    float m = -INFINITY;
    int idx = 0x7fffffff;
    double s = 0.0;
    for (int sp = 0; sp < n_split; sp++) {  // segments in ascending order of token id
        const RowStat r = stats[(size_t)row * n_split + sp];
        stat_merge<true>(m, idx, s, r.m, r.idx, r.s, inv_tau);
    }
    conf[row] = (float)(1.0 / s);
    if (top) top[row] = idx;
}

}  // namespace

size_t sled_accept_ws_bytes(int B, int T, int n_split) {
    (void)B;
    size_t stats = (size_t)T * n_split * sizeof(RowStat);
    return (stats + 255) & ~(size_t)255;
}

// Behind the statistics: accept_over's word on every request, then tile sums and decisions of the sweeps that run as launches of
// their own.  Each of the two is used where the workspace has room for it.  A workspace without is as good: the rows are then
// scanned in one launch, and the finish sweeps itself.
static size_t over_ws_bytes(int B) { return ((size_t)B * sizeof(int32_t) + 255) & ~(size_t)255; }
static size_t sweep_ws_bytes(int B, int vocab) { return (size_t)B * (sizeof(Decision) + 2 * (size_t)((vocab + WTILE - 1) / WTILE) * sizeof(double)); }
size_t sled_accept_ws_bytes_full(int B, int T, int vocab) { return sled_accept_ws_bytes(B, T, 16) + over_ws_bytes(B) + sweep_ws_bytes(B, vocab); }

int sled_accept_pick_split(int T, int vocab) {
    // enough workgroups (rows x segments) for several rounds over the chip, so that the last round is short
    int n = (8192 + T - 1) / T;
    if (n > 16) n = 16;
    if (n < 1) n = 1;
    while (n > 1 && vocab / n < 2048) n--;
    return n;
}

int sled_launch_accept(int mode, int B, int T, const int* k_host, int vocab, float temperature, const float* logits,
                       const int32_t* tokens, const float* draft_q, const int32_t* q_ids, const float* q_probs,
                       const float* q_rest, int q_m, const float* u_acc, const float* u_smp, int32_t* accept_len, int32_t* out_token, void* ws,
                       size_t ws_bytes, hipStream_t st) {
    if ((vocab + WTILE - 1) / WTILE > MAX_WTILES) SLED_FAIL(SLED_EINVAL, "accept: vocabulary %d too large", vocab);
    if (q_m < 0 || q_m > SLED_SPARSE_Q_MAX) SLED_FAIL(SLED_EINVAL, "accept: %d sparse entries per draft, at most %d", q_m, SLED_SPARSE_Q_MAX);
    KPack kp;
    for (int i = 0; i < B; i++) kp.k[i] = (uint8_t)k_host[i];
    QSrc qsrc{draft_q, q_ids, q_probs, q_m > 0 ? q_rest : nullptr, q_m};
    const float inv_tau = 1.0f / temperature;
    // The scan in parts.  A cut at row c saves the rows from c on of every request that ends before c and costs two launches and their
    // drain: made where the rows behind it are at least 64 MB x c (the longer the prefix, the fewer requests still get there).  Whole calls with
    // the first cut / without it, us, drafts 62 % accepted, by the MB behind row 2: 139 (64 requests x 2 to 8 drafts x 128256 tokens) 88 / 84,
    // 144 (40 x 8) 75 / 76, 158 (96 x 0 to 8) 100 / 101, 172 (48 x 8) 83 / 85, 230 (64 x 8) 96 / 104, 344 (96 x 8) 118 / 142, 919 (256 x 8)
    // 194 / 308; below the line 116 (56 x 2 to 8) 80 / 79.  With the second / without, by the MB behind row 4: 257 120 / 120, 298 125 / 126, 359 147 / 149,
    // 314 (200 x 4 to 8) 165 / 168.  20 requests of 16 drafts among 180 of one (154 MB behind row 2): 140 / 150.
    auto rows_from = [&](int c) {
        int64_t n = 0;
        for (int i = 0; i < B; i++) n += std::max(0, k_host[i] + 1 - c);
        return n;
    };
    int k_top = 0;
    for (int i = 0; i < B; i++) k_top = std::max(k_top, k_host[i]);
    const int n_tiles = (vocab + WTILE - 1) / WTILE;
    int cuts[4] = {0, 0, 0, 0}, n_part = 1;
    for (int c = 2; c <= 8 && c <= k_top; c *= 2)
        if (rows_from(c) * vocab * 4 >= (int64_t)64000000 * c) cuts[n_part++] = c;
    // Segments per row: about 2048 workgroups in the (first) launch.  More of them are shorter than their own start and
    // reduction: 276 rows in 16 segments took 45 us for 141 MB, in 7 27 us.
    auto segments = [&]() {
        const int64_t rows_first = n_part > 1 ? T - rows_from(cuts[1]) : T;
        return std::min(sled_accept_pick_split(T, vocab), (int)std::max<int64_t>(1, (2048 + rows_first / 2) / rows_first));
    };
    // Rows behind a cut are few and are cut finer, where the workspace holds as many statistics for all rows: eight segments (sixteen
    // scan no faster, and the next test, which adds up a row's segments, takes 6.9 instead of 5.4 us).  They come before room for the sweeps in
    // launches of their own (below) where the workspace has room for one of the two: 160 requests x 8 drafts x 32000 tokens in
    // the 256 KiB of sled_accept_static 68 us so, 74 with coarse segments and those sweeps; 150 requests 71 and 71, 100 x 16 drafts 66 and 65.
    int n_split = segments();
    const int n_fine = std::min(8, sled_accept_pick_split(1, vocab));
    Split sp{n_split, n_fine, cuts[1], std::max(n_split, n_fine)};
    if (n_part > 1 && ws_bytes < sled_accept_ws_bytes(B, T, sp.stride) + over_ws_bytes(B)) sp = Split{n_split, n_split, cuts[1], n_split};
    if (n_part > 1 && ws_bytes < sled_accept_ws_bytes(B, T, sp.stride) + over_ws_bytes(B)) n_part = 1;
    if (n_part == 1) {
        n_split = segments();
        sp = Split{n_split, n_split, 0, n_split};
    }
    RowStat* stats = reinterpret_cast<RowStat*>(ws);
    const size_t over_at = sled_accept_ws_bytes(B, T, sp.stride), sums_at = over_at + over_ws_bytes(B);
    int32_t* over = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + over_at);   // there when the scan comes in parts
    const bool sweep_room = ws_bytes >= sums_at + sweep_ws_bytes(B, vocab);
    if (n_part > 1) {
        const dim3 grid(B * cuts[1], n_split);
        if (mode == SLED_SAMPLE)
            hipLaunchKernelGGL(accept_row_stats_first<true>, grid, dim3(256), 0, st, logits, vocab, sp, inv_tau, B, kp, stats);
        else
            hipLaunchKernelGGL(accept_row_stats_first<false>, grid, dim3(256), 0, st, logits, vocab, sp, inv_tau, B, kp, stats);
        SLED_LAUNCH_CHECK();
    }
    for (int part = 1; part < n_part; part++) {
        const int j0 = cuts[part], j1 = part + 1 < n_part ? cuts[part + 1] : k_top + 1;
        hipLaunchKernelGGL(accept_over, dim3(B), dim3(64), 0, st, mode, kp, j0, vocab, sp, inv_tau, temperature, logits, tokens, qsrc, u_acc, stats, over);
        SLED_LAUNCH_CHECK();
        const int64_t items = (rows_from(j0) - (part + 1 < n_part ? rows_from(j1) : 0)) * sp.n1;
        const dim3 grid((unsigned)std::min<int64_t>(items, 2048));   // eight workgroups fill a CU
        if (mode == SLED_SAMPLE)
            hipLaunchKernelGGL(accept_row_stats_part<true>, grid, dim3(256), 0, st, logits, vocab, sp, inv_tau, B, j0, j1, kp, over, stats);
        else
            hipLaunchKernelGGL(accept_row_stats_part<false>, grid, dim3(256), 0, st, logits, vocab, sp, inv_tau, B, j0, j1, kp, over, stats);
        SLED_LAUNCH_CHECK();
    }
    if (n_part == 1) {
        const int seg = ((vocab + n_split - 1) / n_split + 3) & ~3;
        const dim3 grid(T, n_split);
        if (mode == SLED_SAMPLE)
            hipLaunchKernelGGL((accept_row_stats<true>), grid, dim3(256), 0, st, logits, vocab, n_split, seg, inv_tau, stats);
        else
            hipLaunchKernelGGL((accept_row_stats<false>), grid, dim3(256), 0, st, logits, vocab, n_split, seg, inv_tau, stats);
        SLED_LAUNCH_CHECK();
    }
    // The two float64 sweeps over a request's row are what the finish spends its time on: 93 us with one workgroup per request,
    // be they 48 or 256.  From 32 tiles (32768 tokens) on, they get launches of their own with two workgroups per CU: 48
    // requests 17 + 14 + 13 us.  Where most CUs have a request anyway that does not pay: whole calls of B requests x 8 drafts x
    // 128256 tokens, sweeps of their own / in the finish, dense q: 96 112 / 136 us, 128 132 / 150, 160 162 / 170, 192 193 / 182,
    // 256 221 / 209, 384 313 / 322; sparse: 160 201 / 206, 192 230 / 217, 256 261 / 248, 384 387 / 400.
    constexpr int SWEEP_MAX_B = 160;
    Decision* decisions = nullptr;
    double* tile_sums = nullptr;
    if (mode == SLED_SAMPLE && sweep_room && n_tiles >= 32 && B <= SWEEP_MAX_B) {
        tile_sums = reinterpret_cast<double*>(static_cast<char*>(ws) + sums_at);
        decisions = reinterpret_cast<Decision*>(tile_sums + (size_t)B * 2 * n_tiles);
        const dim3 grid(B, std::min((n_tiles + 7) / 8, std::max(2, 512 / B)));   // a workgroup has eight wavefronts, a tile each at a time
        hipLaunchKernelGGL(accept_sweep<false>, grid, dim3(512), 0, st, kp, vocab, sp, inv_tau, temperature, logits, tokens, qsrc, u_acc, stats,
                           decisions, tile_sums);
        SLED_LAUNCH_CHECK();
        hipLaunchKernelGGL(accept_sweep<true>, grid, dim3(512), 0, st, kp, vocab, sp, inv_tau, temperature, logits, tokens, qsrc, u_acc, stats,
                           decisions, tile_sums);
        SLED_LAUNCH_CHECK();
    }
    // greedy needs only the deciding wavefront
    hipLaunchKernelGGL(accept_finish, dim3(B), dim3(mode == SLED_SAMPLE ? 1024 : 64), 0, st, mode, kp, vocab, sp, inv_tau,
                       temperature, logits, tokens, qsrc, u_acc, u_smp, stats, accept_len, out_token, decisions, tile_sums);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

// ---------------------------------------------------------------------------------------------------------------
// sled_accept for callers that cannot allocate: the row statistics live in a fixed array of device memory that is
// part of the library's code object (one copy per GPU, held until the process ends) instead of a caller's workspace.
constexpr size_t SLED_STATIC_STATS = 16384;   // row-segment statistics: 256 KiB
static __device__ __align__(256) unsigned char scratch[SLED_STATIC_STATS * sizeof(RowStat)];

namespace {
constexpr int SLED_MAX_DEVICES = 64;
void* g_scratch_ptr[SLED_MAX_DEVICES];   // device address of `scratch` on each GPU (the array's name is no address on the host)

// the address of this GPU's copy of the array, looked up once per device with that device current
int static_scratch(void** out) {
    int dev = -1;
    SLED_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= SLED_MAX_DEVICES) SLED_FAIL(SLED_EINVAL, "sled_accept_static: device %d unsupported", dev);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        SLED_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) SLED_FAIL(SLED_EHIP, "sled_accept_static: no device address for the static scratch array");
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return SLED_OK;
}
}  // namespace

extern "C" int sled_accept_static(int mode, int B, const int* k, int vocab, float temperature, const float* logits,
                                  const int32_t* tokens, const float* draft_q, const float* u_acc, const float* u_smp,
                                  int32_t* accept_len, int32_t* out_token, void* stream) {
    if (!k || !logits || !tokens || !accept_len || !out_token) SLED_FAIL(SLED_EINVAL, "sled_accept_static: null argument");
    if (mode != SLED_GREEDY && mode != SLED_SAMPLE) SLED_FAIL(SLED_EINVAL, "sled_accept_static: unknown mode %d", mode);
    if (B < 1 || B > 1024) SLED_FAIL(SLED_EINVAL, "sled_accept_static: batch size %d outside [1, 1024]", B);
    if (vocab < 2 || vocab > 2000000) SLED_FAIL(SLED_EINVAL, "sled_accept_static: vocab %d unsupported", vocab);
    if (!(temperature > 0.f)) SLED_FAIL(SLED_EINVAL, "sled_accept_static: temperature must be positive");
    int T = 0, nd = 0;
    for (int i = 0; i < B; i++) {
        if (k[i] < 0 || k[i] > 255) SLED_FAIL(SLED_EINVAL, "sled_accept_static: k[%d] = %d outside [0, 255]", i, k[i]);
        T += k[i] + 1;
        nd += k[i];
    }
    if (mode == SLED_SAMPLE && (!u_smp || (nd > 0 && (!draft_q || !u_acc))))
        SLED_FAIL(SLED_EINVAL, "sled_accept_static: sampling needs draft_q, u_acc and u_smp");
    const size_t need = (size_t)T * sled_accept_pick_split(T, vocab);
    if (need > SLED_STATIC_STATS)
        SLED_FAIL(SLED_EINVAL, "sled_accept_static: %d rows in %d segments need %zu statistics, the static scratch holds %zu; use sled_accept",
                  T, sled_accept_pick_split(T, vocab), need, SLED_STATIC_STATS);
    void* ws = nullptr;
    int rc = static_scratch(&ws);
    if (rc != SLED_OK) return rc;
    // nothing in the array has to start at zero: the row scan writes every statistic that decides anything
    return sled_launch_accept(mode, B, T, k, vocab, temperature, logits, tokens, draft_q, nullptr, nullptr, nullptr, 0, u_acc,
                              u_smp, accept_len, out_token, ws, SLED_STATIC_STATS * sizeof(RowStat), static_cast<hipStream_t>(stream));
}

int sled_launch_row_confidence(int T, int vocab, float temperature, const float* logits, float* conf, int32_t* top, void* ws,
                               hipStream_t st) {
    const int n_split = sled_accept_pick_split(T, vocab);
    int seg = (vocab + n_split - 1) / n_split;
    seg = (seg + 3) & ~3;
    RowStat* stats = reinterpret_cast<RowStat*>(ws);
    const float inv_tau = 1.0f / temperature;
    hipLaunchKernelGGL((accept_row_stats<true, true>), dim3(T, n_split), dim3(256), 0, st, logits, vocab, n_split, seg, inv_tau, stats);
    SLED_LAUNCH_CHECK();
    hipLaunchKernelGGL(row_confidence_finish, dim3((T + 255) / 256), dim3(256), 0, st, stats, T, n_split, inv_tau, conf, top);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}
