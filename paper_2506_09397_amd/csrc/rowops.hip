// Row-wise operators of the verify step, one workgroup per packed row.  They sit between the
// projections and do everything that is not a contraction: embedding gather, reduction of the
// split-K partial sums (fixed order), residual add, RMSNorm, rotary embedding, the scatter of new
// K/V into the paged cache, SwiGLU for fp32 models, weight repacking at load time.
//
// Activations that feed a bf16 projection are written directly in MFMA operand order
// (frag_offset), so the projection kernels never transpose anything.  Weights are repacked once, at
// load time, into the k-step-major tile order of wfrag_offset.
#include "sled_internal.h"

#include <algorithm>

namespace {

// x + its value in the lane whose number differs in one bit, for the bits 5 .. 0 in turn: the sum over the wavefront in every lane.  Exchanges
// between register halves (bits 5, 4) and rotations within 16 lanes, which by then hold equal values in the lanes that a
// rotation and an exchange would tell apart; through LDS (shuffles) the six steps are as many round trips.
__device__ inline float wave_sum(float x) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x128, 0xf, 0xf, false));   // row_ror:8
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x124, 0xf, 0xf, false));   // row_ror:4
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x122, 0xf, 0xf, false));   // row_ror:2
    x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x121, 0xf, 0xf, false));   // row_ror:1
    return x;
}

// sum over the workgroup (blockDim.x a multiple of 64, at most 1024), once per kernel; every thread gets the result;
// the order of additions is fixed
__device__ inline float block_sum(float x, float* sh /*[16]*/) {
    x = wave_sum(x);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = x;
    __syncthreads();
    float t = 0.f;
    const int nw = blockDim.x >> 6;
    for (int i = 0; i < nw; i++) t += sh[i];
    return t;
}

// store 8 consecutive activations of row t starting at column c0; bf16 models keep an activation
// as a bf16 pair hi + lo in two planes of operand-ordered storage, `plane` elements apart
template <bool BF16>
__device__ inline void store_act8(void* X, size_t plane, int t, int c0, int K, const float* v) {
    if (BF16) {
        uint32_t wh[4], wl[4];
        for (int i = 0; i < 4; i++) {
            const bf16_t h0 = f32_to_bf16(v[2 * i]), h1 = f32_to_bf16(v[2 * i + 1]);
            const bf16_t l0 = f32_to_bf16(v[2 * i] - bf16_to_f32(h0)), l1 = f32_to_bf16(v[2 * i + 1] - bf16_to_f32(h1));
            wh[i] = (uint32_t)h0 | ((uint32_t)h1 << 16);
            wl[i] = (uint32_t)l0 | ((uint32_t)l1 << 16);
        }
        bf16_t* p = static_cast<bf16_t*>(X) + frag_offset(t, c0, K);
        *reinterpret_cast<uint4*>(p) = make_uint4(wh[0], wh[1], wh[2], wh[3]);
        *reinterpret_cast<uint4*>(p + plane) = make_uint4(wl[0], wl[1], wl[2], wl[3]);
    } else {
        float* p = static_cast<float*>(X) + (size_t)t * K + c0;
        *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
    }
}

// a + sum over the K slices s = 0 .. n_split-1 (ascending) of p[s * stride .. + 3].  The loads of up to eight slices
// are issued before the first is used: a row kernel is a chain of round trips to L2, not a stream, and a loop
// that adds slice after slice would pay one round trip per slice.
__device__ inline float4 add_slices4(float4 a, const float* __restrict__ p, size_t stride, int n_split) {
    for (int s0 = 0; s0 < n_split; s0 += 8) {
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; u++)
            v[u] = s0 + u < n_split ? *reinterpret_cast<const float4*>(p + (size_t)(s0 + u) * stride) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int u = 0; u < 8; u++) {
            a.x += v[u].x;
            a.y += v[u].y;
            a.z += v[u].z;
            a.w += v[u].w;
        }
    }
    return a;
}

// the same for two single values
__device__ inline void add_slices1x2(float& a, float& b, const float* __restrict__ pa, const float* __restrict__ pb, size_t stride,
                                     int n_split) {
    for (int s0 = 0; s0 < n_split; s0 += 8) {
        float v[8], w[8];
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const bool on = s0 + u < n_split;
            v[u] = on ? pa[(size_t)(s0 + u) * stride] : 0.f;
            w[u] = on ? pb[(size_t)(s0 + u) * stride] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; u++) {
            a += v[u];
            b += w[u];
        }
    }
}

// ... and for one
__device__ inline float add_slices1(float a, const float* __restrict__ p, size_t stride, int n_split) {
    for (int s0 = 0; s0 < n_split; s0 += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) v[u] = s0 + u < n_split ? p[(size_t)(s0 + u) * stride] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; u++) a += v[u];
    }
    return a;
}

// store 4 consecutive activations of row t starting at column c0 (a multiple of 4), as store_act8 does for 8
template <bool BF16>
__device__ inline void store_act4(void* X, size_t plane, int t, int c0, int K, const float4& v) {
    if (BF16) {
        const float f[4] = {v.x, v.y, v.z, v.w};
        uint32_t wh[2], wl[2];
        for (int i = 0; i < 2; i++) {
            const bf16_t h0 = f32_to_bf16(f[2 * i]), h1 = f32_to_bf16(f[2 * i + 1]);
            const bf16_t l0 = f32_to_bf16(f[2 * i] - bf16_to_f32(h0)), l1 = f32_to_bf16(f[2 * i + 1] - bf16_to_f32(h1));
            wh[i] = (uint32_t)h0 | ((uint32_t)h1 << 16);
            wl[i] = (uint32_t)l0 | ((uint32_t)l1 << 16);
        }
        bf16_t* p = static_cast<bf16_t*>(X) + frag_offset(t, c0, K);  // the 8 elements of a k-octet are contiguous
        *reinterpret_cast<uint2*>(p) = make_uint2(wh[0], wh[1]);
        *reinterpret_cast<uint2*>(p + plane) = make_uint2(wl[0], wl[1]);
    } else {
        *reinterpret_cast<float4*>(static_cast<float*>(X) + (size_t)t * K + c0) = v;
    }
}

// Workgroups go to the eight XCDs round robin, and each XCD has its own L2.  Where `group` neighbouring rows share the lines that a kernel
// writes (16 bytes of each: eight rows of an activation, sixteen tokens of a page), the group's workgroups are put on one XCD, so that
// its L2 gathers whole lines instead of eight of them writing pieces back.  The grid is rounded up to whole rounds of groups.
constexpr int XCDS = 8, ACT_LINE_ROWS = 8;
__device__ inline int row_of_block(int w, int group) {
    const int xcd = w % XCDS, local = w / XCDS;   // (group 1: row w)
    return (local / group * XCDS + xcd) * group + local % group;
}
inline int blocks_for_rows(int rows, int group) { return (rows + XCDS * group - 1) / (XCDS * group) * (XCDS * group); }

// h[t,:] += sum_s partial[s][t][:]  (s ascending);  X[t,:] = rmsnorm(h) * gain.  A thread owns 4 consecutive
// columns per trip over the row; rows of up to 8 * blockDim.x columns (two trips) stay in registers between the
// sum of squares and the scaling, longer rows are read back from h.
template <bool BF16>
__global__ __launch_bounds__(1024) void residual_norm_kernel(const float* __restrict__ partial, int n_split, int T_pad,
                                                            int d, float eps, const float* __restrict__ gain,
                                                            float* __restrict__ h, void* __restrict__ X, size_t plane, int T, int group) {
    __shared__ float sh[16];
    const int t = row_of_block(blockIdx.x, group);
    if (t >= T) return;
    const size_t stride = (size_t)T_pad * d;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    float ss = 0.f;
    if (d <= (int)blockDim.x * 8) {
        float4 a[2] = {zero, zero}, g[2] = {zero, zero};
#pragma unroll
        for (int trip = 0; trip < 2; trip++) {
            const int c = (trip * blockDim.x + threadIdx.x) * 4;
            if (c < d) {
                float* hp = h + (size_t)t * d + c;
                g[trip] = *reinterpret_cast<const float4*>(gain + c);
                a[trip] = add_slices4(*reinterpret_cast<const float4*>(hp), partial + (size_t)t * d + c, stride, n_split);
                *reinterpret_cast<float4*>(hp) = a[trip];
                ss += a[trip].x * a[trip].x + a[trip].y * a[trip].y + a[trip].z * a[trip].z + a[trip].w * a[trip].w;
            }
        }
        const float r = 1.0f / sqrtf(block_sum(ss, sh) / (float)d + eps);
#pragma unroll
        for (int trip = 0; trip < 2; trip++) {
            const int c = (trip * blockDim.x + threadIdx.x) * 4;
            if (c < d)
                store_act4<BF16>(X, plane, t, c, d,
                                 make_float4(a[trip].x * r * g[trip].x, a[trip].y * r * g[trip].y, a[trip].z * r * g[trip].z,
                                             a[trip].w * r * g[trip].w));
        }
        return;
    }
    for (int c = threadIdx.x * 4; c < d; c += blockDim.x * 4) {
        float* hp = h + (size_t)t * d + c;
        const float4 a = add_slices4(*reinterpret_cast<const float4*>(hp), partial + (size_t)t * d + c, stride, n_split);
        *reinterpret_cast<float4*>(hp) = a;
        ss += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
    }
    const float r = 1.0f / sqrtf(block_sum(ss, sh) / (float)d + eps);
    for (int c = threadIdx.x * 4; c < d; c += blockDim.x * 4) {
        const float4 a = *reinterpret_cast<const float4*>(h + (size_t)t * d + c);  // this thread's own stores
        const float4 g = *reinterpret_cast<const float4*>(gain + c);
        store_act4<BF16>(X, plane, t, c, d, make_float4(a.x * r * g.x, a.y * r * g.y, a.z * r * g.z, a.w * r * g.w));
    }
}

// Everything a step needs before its first projection, in one launch (four of them one after the other took 16 us, 5 of which are a launch's
// own time each; together they take as long as the longest, the rotary table's float64 functions):
//   rotary table   per packed row cos/sin of pos * theta^(-2i/D), evaluated in float64 and stored as float32, and where the row's K/V go
//                  (16 * page + slot) -- the chain of dependent lookups behind that is then paid once, not in every layer
//   work records   (bf16 models) per attention work item everything its workgroup needs to know before it can request its first
//                  page, gathered into one 48-byte record -- otherwise each of the step's attention launches starts with a chain of
//                  four dependent look-ups (item -> block -> request -> committed length); and the items' arrival counters, zero
//                  [0] block  [1] kv head  [2] first page  [3] pages  [4] L = context length of the block  [5] rows of the block
//                  [6] first packed row  [7] first entry of the block's page list  [8], [9] items of this (block, kv head): the
//                  first (the others follow Hkv places apart), how many
//   embedding      h[t,:] = E[token]; X[t,:] = rmsnorm(h) * gain
struct step_setup {
    const int32_t* len_dev;
    int half, Hkv;
    double theta;
    float2* cs;
    int32_t *kvslot, *plan, *arrive;
    int n_arrive;
    const int32_t* tokens;
    const void* E;
    int V, d;
    float eps;
    const float* gain;
    float* h;
    void* X;
    size_t plane;
    int rope_blocks, plan_blocks;
};
template <bool BF16>
__global__ __launch_bounds__(256) void step_setup_kernel(sled_step_meta meta, step_setup a) {
    __shared__ float sh[16];
    if ((int)blockIdx.x < a.rope_blocks) {   // a wavefront per row
        const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
        if (t >= meta.T) return;
        const int b = meta.row_req[t];
        const int pos = a.len_dev[meta.req_id[b]] + meta.pos0[b] + meta.row_j[t];
        if (lane == 0) a.kvslot[t] = meta.pages[meta.cu_pages[b] + (pos >> 4)] * 16 + (pos & 15);
        for (int i = lane; i < a.half; i += 64) {
            double inv = pow(a.theta, -(double)i / (double)a.half);
            double ang = (double)pos * inv;
            a.cs[(size_t)t * a.half + i] = make_float2((float)cos(ang), (float)sin(ang));
        }
        return;
    }
    if ((int)blockIdx.x < a.rope_blocks + a.plan_blocks) {
        const int w = (blockIdx.x - a.rope_blocks) * 256 + threadIdx.x;
        if (w < a.n_arrive) a.arrive[w] = 0;   // each layer leaves them at zero
        if (w >= meta.n_work) return;
        const int b = meta.work[4 * w + 0], g = meta.work[4 * w + 1];
        int32_t* r = a.plan + 12 * w;
        r[0] = b;
        r[1] = g;
        r[2] = meta.work[4 * w + 2];
        r[3] = meta.work[4 * w + 3];
        r[4] = a.len_dev[meta.req_id[b]] + meta.pos0[b];
        r[5] = meta.k[b] + 1;
        r[6] = meta.cu_rows[b];
        r[7] = meta.cu_pages[b];
        r[8] = meta.cu_work[2 * (b * a.Hkv + g)];
        r[9] = meta.cu_work[2 * (b * a.Hkv + g) + 1];
        r[10] = r[11] = 0;
        return;
    }
    const int t = blockIdx.x - a.rope_blocks - a.plan_blocks, d = a.d;
    int tok = a.tokens[t];
    tok = tok < 0 ? 0 : (tok >= a.V ? a.V - 1 : tok);
    float ss = 0.f;
    for (int c = threadIdx.x * 8; c < d; c += 256 * 8) {
        float v[8];
        if (BF16) {
            uint4 raw = *reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(a.E) + (size_t)tok * d + c);
            const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
            for (int i = 0; i < 4; i++) {
                v[2 * i] = bf16_to_f32((bf16_t)(w[i] & 0xffff));
                v[2 * i + 1] = bf16_to_f32((bf16_t)(w[i] >> 16));
            }
        } else {
            const float* p = static_cast<const float*>(a.E) + (size_t)tok * d + c;
            for (int i = 0; i < 8; i++) v[i] = p[i];
        }
        for (int i = 0; i < 8; i++) {
            a.h[(size_t)t * d + c + i] = v[i];
            ss += v[i] * v[i];
        }
    }
    const float tot = block_sum(ss, sh);
    const float r = 1.0f / sqrtf(tot / (float)d + a.eps);
    for (int c = threadIdx.x * 8; c < d; c += 256 * 8) {
        float v[8];
        for (int i = 0; i < 8; i++) v[i] = a.h[(size_t)t * d + c + i] * r * a.gain[c + i];
        store_act8<BF16>(a.X, a.plane, t, c, d, v);
    }
}

// Reduce the QKV partial sums of row t, rotate q and k, write q to Q[T, Hq, D] as a bf16 pair and k, v into the request's page slot for
// position L + j.  (Prompt slices; a verification step's attention does this itself.)  A thread takes four neighbouring rotary pairs of a
// q or k head, or four dims of a v head, so that all loads are 16 bytes and all stores but v's 8; sixteen rows, the tokens of a page, meet on
// one XCD.  1080 rows of the 8B shape (a wavefront per row and head, two bytes a store, rows spread over the XCDs before): 26.4 -> 13.8 us.
constexpr int QKV_ROWS = 16;
__global__ __launch_bounds__(256) void qkv_rope_store_bf16_kernel(const float* __restrict__ partial, int n_split, int T, int T_pad, int Hq, int Hkv,
                                                                  const float2* __restrict__ cs, const int32_t* __restrict__ kvslot,
                                                                  bf16_t* __restrict__ Q, size_t q_plane, bf16_t* __restrict__ k_pool,
                                                                  bf16_t* __restrict__ v_pool, int64_t n_pages, int layer, int blocks_per_row) {
    constexpr int D = 128, half = D / 2;
    const int w = blockIdx.x, xcd = w % XCDS, local = w / XCDS;
    const int t = row_of_block(local / blocks_per_row * XCDS + xcd, QKV_ROWS);
    if (t >= T) return;
    const int n_rot = (Hq + Hkv) * (half / 4), item = local % blocks_per_row * 256 + threadIdx.x;
    const int n_qkv = (Hq + 2 * Hkv) * D;
    const float* prow = partial + (size_t)t * n_qkv;
    const size_t stride = (size_t)T_pad * n_qkv;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    auto pair2 = [](float a, float b) { return (uint32_t)f32_to_bf16(a) | ((uint32_t)f32_to_bf16(b) << 16); };
    if (item < n_rot) {
        const int head = item / (half / 4), i = item % (half / 4) * 4;
        const float4 c01 = *reinterpret_cast<const float4*>(cs + (size_t)t * half + i), c23 = *reinterpret_cast<const float4*>(cs + (size_t)t * half + i + 2);
        const int ps = head < Hq ? 0 : kvslot[t];
        const float4 x1 = add_slices4(zero, prow + head * D + i, stride, n_split), x2 = add_slices4(zero, prow + head * D + i + half, stride, n_split);
        float y1[4], y2[4];
        rope_pair(x1.x, x2.x, c01.x, c01.y, y1[0], y2[0]);
        rope_pair(x1.y, x2.y, c01.z, c01.w, y1[1], y2[1]);
        rope_pair(x1.z, x2.z, c23.x, c23.y, y1[2], y2[2]);
        rope_pair(x1.w, x2.w, c23.z, c23.w, y1[3], y2[3]);
        const uint2 h1 = make_uint2(pair2(y1[0], y1[1]), pair2(y1[2], y1[3])), h2 = make_uint2(pair2(y2[0], y2[1]), pair2(y2[2], y2[3]));
        if (head < Hq) {   // q is kept as a bf16 pair, like every activation that is not cached
            auto low = [](float y) { return y - bf16_to_f32(f32_to_bf16(y)); };
            bf16_t* q = Q + ((size_t)t * Hq + head) * D + i;
            *reinterpret_cast<uint2*>(q) = h1;
            *reinterpret_cast<uint2*>(q + half) = h2;
            *reinterpret_cast<uint2*>(q + q_plane) = make_uint2(pair2(low(y1[0]), low(y1[1])), pair2(low(y1[2]), low(y1[3])));
            *reinterpret_cast<uint2*>(q + q_plane + half) = make_uint2(pair2(low(y2[0]), low(y2[1])), pair2(low(y2[2]), low(y2[3])));
        } else {           // four neighbouring dims share an 8-byte piece of the page's operand order
            bf16_t* kp = k_pool + (((size_t)layer * n_pages + (ps >> 4)) * Hkv + (head - Hq)) * (16 * D);
            *reinterpret_cast<uint2*>(kp + kpage_offset(ps & 15, i)) = h1;
            *reinterpret_cast<uint2*>(kp + kpage_offset(ps & 15, i + half)) = h2;
        }
    } else if (item < n_rot + Hkv * (D / 4)) {
        const int e = item - n_rot, g = e / (D / 4), dd = e % (D / 4) * 4;
        const int ps = kvslot[t];
        const float4 x = add_slices4(zero, prow + (Hq + Hkv + g) * D + dd, stride, n_split);
        bf16_t* vp = v_pool + (((size_t)layer * n_pages + (ps >> 4)) * Hkv + g) * (16 * D);
        vp[vpage_offset(ps & 15, dd)] = f32_to_bf16(x.x);
        vp[vpage_offset(ps & 15, dd + 1)] = f32_to_bf16(x.y);
        vp[vpage_offset(ps & 15, dd + 2)] = f32_to_bf16(x.z);
        vp[vpage_offset(ps & 15, dd + 3)] = f32_to_bf16(x.w);
    }
}

// The same for fp32 models, one head of row t (blockIdx = (t, head), heads ordered q, k, v) per workgroup.
__global__ __launch_bounds__(64) void qkv_rope_store_f32_kernel(const float* __restrict__ partial, int n_split, int T_pad, int Hq, int Hkv, int D,
                                                                const float2* __restrict__ cs, const int32_t* __restrict__ kvslot,
                                                                float* __restrict__ Q, float* __restrict__ k_pool, float* __restrict__ v_pool,
                                                                int64_t n_pages, int layer) {
    const int t = blockIdx.x, head = blockIdx.y;
    const int half = D >> 1;
    const int n_qkv = (Hq + 2 * Hkv) * D;
    const float* prow = partial + (size_t)t * n_qkv;
    const size_t stride = (size_t)T_pad * n_qkv;
    const int ps = kvslot[t];
    auto slot = [&](float* pool, int g) { return pool + (((size_t)layer * n_pages + (ps >> 4)) * Hkv + g) * (16 * D) + (size_t)(ps & 15) * D; };
    if (head < Hq + Hkv) {
        float* out = head < Hq ? Q + ((size_t)t * Hq + head) * D : slot(k_pool, head - Hq);
        for (int i = threadIdx.x; i < half; i += 64) {
            const int c1 = head * D + i, c2 = c1 + half;
            const float2 sc = cs[(size_t)t * half + i];
            float x1 = 0.f, x2 = 0.f;
            add_slices1x2(x1, x2, prow + c1, prow + c2, stride, n_split);
            rope_pair(x1, x2, sc.x, sc.y, out[i], out[i + half]);
        }
    } else {   // v head: no rotation
        const int g = head - Hq - Hkv;
        float* out = slot(v_pool, g);
        for (int dd = threadIdx.x; dd < D; dd += 64) out[dd] = add_slices1(0.f, prow + (Hq + Hkv) * D + g * D + dd, stride, n_split);
    }
}

// a[t, f] = silu(g) * u with (g, u) = sum over K slices of gu[s][t][2f], gu[s][t][2f+1]; used when the
// gate/up projection does not apply SwiGLU itself (fp32 models, or a gate/up projection split over K).
// One workgroup per row, 8 outputs per thread.
template <bool BF16>
__global__ __launch_bounds__(256) void swiglu_reduce_kernel(const float* __restrict__ gu, int n_split, int T_pad, int F,
                                                            void* __restrict__ A, size_t plane) {
    const int t = blockIdx.x;
    for (int f0 = (blockIdx.y * 256 + threadIdx.x) * 8; f0 < F; f0 += gridDim.y * 256 * 8) {
        float acc[16];
        const float* p = gu + (size_t)t * (2 * (size_t)F) + 2 * f0;
        for (int q = 0; q < 4; q++) {
            const float4 x = add_slices4(make_float4(0.f, 0.f, 0.f, 0.f), p + 4 * q, (size_t)T_pad * (2 * (size_t)F), n_split);
            acc[4 * q] = x.x;
            acc[4 * q + 1] = x.y;
            acc[4 * q + 2] = x.z;
            acc[4 * q + 3] = x.w;
        }
        float v[8];
        for (int i = 0; i < 8; i++) {
            const float g = acc[2 * i], u = acc[2 * i + 1];
            v[i] = g / (1.f + __expf(-g)) * u;
        }
        store_act8<BF16>(A, plane, t, f0, F, v);
    }
}

// ----- K/V taken over from elsewhere and handed on -------------------------------------------------------------------
// Both directions are pure data movement, so what counts is that every access is 16 bytes and every line is used once.
// One workgroup moves one page of one layer (16 tokens, all kv heads, K and V).  The K page order is a permutation of
// 16-byte chunks (8 dims of a token); four lanes per token give 64-byte pieces on the caller's side and whole KiB in the
// page.  A 16-byte chunk of a V page holds 4 tokens x 2 dims a tile of 16 apart: a thread takes 4 tokens x two runs of 8
// dims (eight 16-byte accesses), transposes them in registers, and has eight neighbouring chunks of the page.
// (Moving element by element, a workgroup per token, ran at 2.1 TB/s: 184 us for 1500 tokens of 32 layers, 197 MB read
// and written; by pages 90 us.)
struct chunk16 {
    bf16_t e[8];
};
// 16 bytes at p; `al`: p is known to be 16-byte aligned (a caller's buffer need not be)
__device__ inline chunk16 ld_chunk(const bf16_t* p, bool al) {
    if (al) return __builtin_bit_cast(chunk16, *reinterpret_cast<const uint4*>(p));
    chunk16 c;
#pragma unroll
    for (int i = 0; i < 8; i++) c.e[i] = p[i];
    return c;
}
__device__ inline void st_chunk(bf16_t* p, const chunk16& c, bool al) {
    if (al) {
        *reinterpret_cast<uint4*>(p) = __builtin_bit_cast(uint4, c);
        return;
    }
#pragma unroll
    for (int i = 0; i < 8; i++) p[i] = c.e[i];
}

// Between positions first .. first+n_tok-1 of a request (first = *len when len is given) and [n_layers, n_tok, Hkv, D] in the
// caller's buffers: INGEST into the pages, else out of them.  blockIdx.x counts the pages from the one that holds `first`, blockIdx.z the
// requests of the launch.
struct kv_pieces {
    sled_kv_piece p[SLED_KV_PIECES];
};
template <bool BF16, bool INGEST>
__global__ __launch_bounds__(256) void kv_move_kernel(kv_pieces pieces, int Hkv, int D, void* k_pool, void* v_pool, int64_t n_pages, bool staged) {
    extern __shared__ __attribute__((aligned(16))) uint4 stage[];
    const sled_kv_piece& pc = pieces.p[blockIdx.z];
    void *const k_buf = pc.k, *const v_buf = pc.v;
    const int32_t* const pages = pc.pages;
    const int first = pc.len ? *pc.len : pc.first, n_tok = pc.n_tok;
    const bool aligned = ((reinterpret_cast<uintptr_t>(k_buf) | reinterpret_cast<uintptr_t>(v_buf)) & 15) == 0;   // rows are multiples of 256 bytes
    const int layer = blockIdx.y, lp = (first >> 4) + blockIdx.x;
    // slots lo .. hi-1 of this page take part; slot s is token s - off of the caller's buffers
    const int off = first - lp * 16, lo = max(off, 0), hi = min(16, off + n_tok);
    if (lo >= hi) return;
    const size_t head_elems = (size_t)16 * D, page = ((size_t)layer * n_pages + pages[lp]) * Hkv * head_elems;
    const size_t row = (size_t)Hkv * D;   // elements of one token
    if (BF16) {
        bf16_t* kb = static_cast<bf16_t*>(k_buf) + (size_t)layer * n_tok * row;
        bf16_t* vb = static_cast<bf16_t*>(v_buf) + (size_t)layer * n_tok * row;
        bf16_t* kp = static_cast<bf16_t*>(k_pool) + page;
        bf16_t* vp = static_cast<bf16_t*>(v_pool) + page;
        // K: D is 128 (16 chunks per token and head); in page order chunk = (c / 4) * 64 + (c % 4) * 16 + slot
        // (four chunks in flight per thread: a loop of single ones waits for each before it stores it)
        for (int g0 = 0; g0 < Hkv; g0 += 4) {
            const int e = threadIdx.x, c4 = (e >> 6) & 3, slot = (e >> 2) & 15, c = c4 * 4 + (e & 3);
            if (slot < lo || slot >= hi) break;
            bf16_t* u = kb + (size_t)(slot - off) * row + g0 * 128 + c * 8;
            bf16_t* q = kp + (size_t)g0 * 2048 + (c4 * 64 + (e & 3) * 16 + slot) * 8;
            chunk16 t[4];
#pragma unroll
            for (int i = 0; i < 4; i++)
                if (g0 + i < Hkv) t[i] = INGEST ? ld_chunk(u + i * 128, aligned) : ld_chunk(q + i * 2048, true);
#pragma unroll
            for (int i = 0; i < 4; i++)
                if (g0 + i < Hkv) {
                    if (INGEST) st_chunk(q + i * 2048, t[i], true);
                    else st_chunk(u + i * 128, t[i], aligned);
                }
        }
        // V: thread = (head, 4 slots s4, pair of 16-dim tiles, half of their 16 dims).  The eight chunks that a thread makes of a whole page
        // are neighbours, so stored from here an instruction would put 16 bytes into each of 64 lines: they go through LDS instead (chunk
        // c at place c ^ (c / 8 % 8), which spreads the lanes over the banks both ways), if the host has found room for the page.
        // 1500 tokens of 32 layers: 101 -> 82 us (393 MB read and written); 100 tokens 11.1 -> 9.9.
        const bool through_lds = INGEST && staged && lo == 0 && hi == 16;
        for (int e = threadIdx.x; e < Hkv * 32; e += 256) {
            const int g = e >> 5, s4 = (e >> 3) & 3, dt2 = (e >> 1) & 3, h = e & 1;
            if (s4 * 4 + 4 <= lo || s4 * 4 >= hi) continue;
            bf16_t* u = vb + ((int64_t)s4 * 4 - off) * (int64_t)row + g * 128 + dt2 * 32 + h * 8;   // slot s4*4, first tile of the pair
            bf16_t* q = vp + (size_t)g * 2048 + (dt2 * 64 + s4 * 16 + h * 8) * 8;
            const bool whole = s4 * 4 >= lo && s4 * 4 + 4 <= hi;
            chunk16 a[4][2], t[8];
            if (INGEST) {
#pragma unroll
                for (int s = 0; s < 4; s++)
#pragma unroll
                    for (int x = 0; x < 2; x++)
                        if (s4 * 4 + s >= lo && s4 * 4 + s < hi) a[s][x] = ld_chunk(u + s * row + x * 16, aligned);
                if (whole) {
#pragma unroll
                    for (int j = 0; j < 8; j++) {
#pragma unroll
                        for (int i = 0; i < 8; i++) t[j].e[i] = a[i & 3][i >> 2].e[j];
                        const int c = e / 32 * 256 + dt2 * 64 + s4 * 16 + h * 8 + j;
                        if (through_lds) stage[c ^ ((c >> 3) & 7)] = __builtin_bit_cast(uint4, t[j]);
                        else st_chunk(q + j * 8, t[j], true);
                    }
                } else {   // the other slots belong to tokens that stay
#pragma unroll
                    for (int s = 0; s < 4; s++)
                        if (s4 * 4 + s >= lo && s4 * 4 + s < hi) {
#pragma unroll
                            for (int x = 0; x < 2; x++)
#pragma unroll
                                for (int j = 0; j < 8; j++) q[j * 8 + x * 4 + s] = a[s][x].e[j];
                        }
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; j++) t[j] = ld_chunk(q + j * 8, true);
#pragma unroll
                for (int s = 0; s < 4; s++)
                    if (s4 * 4 + s >= lo && s4 * 4 + s < hi) {
#pragma unroll
                        for (int x = 0; x < 2; x++) {
#pragma unroll
                            for (int j = 0; j < 8; j++) a[s][x].e[j] = t[j].e[x * 4 + s];
                            st_chunk(u + s * row + x * 16, a[s][x], aligned);
                        }
                    }
            }
        }
        if (through_lds) {
            __syncthreads();
            for (int c = threadIdx.x; c < Hkv * 256; c += 256) reinterpret_cast<uint4*>(vp)[c] = stage[c ^ ((c >> 3) & 7)];
        }
    } else {
        // fp32 models: [slot][dim] in the page, rows of one token and head alike on both sides
        float* kb = static_cast<float*>(k_buf) + (size_t)layer * n_tok * row;
        float* vb = static_cast<float*>(v_buf) + (size_t)layer * n_tok * row;
        float* kp = static_cast<float*>(k_pool) + page;
        float* vp = static_cast<float*>(v_pool) + page;
        // four chunks of 4 values per thread and trip, all requested before the first is stored (heads are multiples of 64 values)
        const int row4 = (int)row / 4, n4 = (hi - lo) * row4;
        auto ld4 = [&](const float* p, bool al) { return al ? *reinterpret_cast<const float4*>(p) : make_float4(p[0], p[1], p[2], p[3]); };
        auto st4 = [&](float* p, const float4& x, bool al) {
            if (al) {
                *reinterpret_cast<float4*>(p) = x;
                return;
            }
            p[0] = x.x;
            p[1] = x.y;
            p[2] = x.z;
            p[3] = x.w;
        };
        for (int e0 = threadIdx.x; e0 < n4; e0 += 4 * 256) {
            float4 a[4][2];
            size_t u[4], q[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int e = e0 + i * 256;
                if (e >= n4) continue;
                const int s = lo + e / row4, w = (e % row4) * 4, g = w / D, dd = w - g * D;
                u[i] = (size_t)(s - off) * row + w;
                q[i] = g * head_elems + (size_t)s * D + dd;
                a[i][0] = INGEST ? ld4(kb + u[i], aligned) : ld4(kp + q[i], true);
                a[i][1] = INGEST ? ld4(vb + u[i], aligned) : ld4(vp + q[i], true);
            }
#pragma unroll
            for (int i = 0; i < 4; i++) {
                if (e0 + i * 256 >= n4) continue;
                st4(INGEST ? kp + q[i] : kb + u[i], a[i][0], INGEST || aligned);
                st4(INGEST ? vp + q[i] : vb + u[i], a[i][1], INGEST || aligned);
            }
        }
    }
}

// row t of an activation buffer -> row 0 of another one
template <bool BF16>
__global__ __launch_bounds__(256) void copy_act_row_kernel(const void* __restrict__ X, size_t plane, int t, void* __restrict__ X1,
                                                           size_t plane1, int d) {
    for (int c = (blockIdx.x * 256 + threadIdx.x) * 8; c < d; c += gridDim.x * 256 * 8) {
        if (BF16) {
            const bf16_t* src = static_cast<const bf16_t*>(X) + frag_offset(t, c, d);
            bf16_t* dst = static_cast<bf16_t*>(X1) + frag_offset(0, c, d);
            *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
            *reinterpret_cast<uint4*>(dst + plane1) = *reinterpret_cast<const uint4*>(src + plane);
        } else {
            const float* src = static_cast<const float*>(X) + (size_t)t * d + c;
            float* dst = static_cast<float*>(X1) + c;
            *reinterpret_cast<float4*>(dst) = *reinterpret_cast<const float4*>(src);
            *reinterpret_cast<float4*>(dst + 4) = *reinterpret_cast<const float4*>(src + 4);
        }
    }
}

// committed lengths after an append (+ add[i]) or, with `accept`, a commit (+ accept[i] + 1); `fresh`: the request starts from zero whatever the slot held
__global__ void len_add_kernel(int32_t* __restrict__ len_dev, const int32_t* __restrict__ req_ids, const int32_t* __restrict__ add,
                               const int32_t* __restrict__ fresh, const int32_t* __restrict__ accept, int B) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= B) return;
    const int r = req_ids[i], from = fresh && fresh[i] ? 0 : len_dev[r];
    len_dev[r] = from + (accept ? accept[i] + 1 : add[i]);
}
// the lengths of requests that have just been opened, up to 128 in a launch
struct len_ids {
    int id[128];
};
__global__ void len_zero_kernel(int32_t* __restrict__ len_dev, len_ids ids, int n) {
    if ((int)threadIdx.x < n) len_dev[ids.id[threadIdx.x]] = 0;
}

// ----- weight repacking --------------------------------------------------------------------
// rows [0, rows) of src[rows, K] go to destination rows dst_row0 + r * dst_row_stride of a packed
// (bf16, operand order) or row-major (f32) matrix with K columns.
template <bool BF16>
__global__ void pack_rows_kernel(const void* __restrict__ src, void* __restrict__ dst, int rows, int K, int dst_row0,
                                 int dst_row_stride, int dst_row_tiles) {
    const size_t n8 = (size_t)rows * (K / 8);
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n8; e += (size_t)gridDim.x * blockDim.x) {
        const int r = (int)(e / (K / 8));
        const int c = (int)(e - (size_t)r * (K / 8)) * 8;
        const int dr = dst_row0 + r * dst_row_stride;
        if (BF16) {
            uint4 v = *reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(src) + (size_t)r * K + c);
            *reinterpret_cast<uint4*>(static_cast<bf16_t*>(dst) + wfrag_offset(dr, c, dst_row_tiles)) = v;
        } else {
            const float* s = static_cast<const float*>(src) + (size_t)r * K + c;
            float* d = static_cast<float*>(dst) + (size_t)dr * K + c;
            for (int i = 0; i < 8; i++) d[i] = s[i];
        }
    }
}

// rows of 8-bit weights (FP8 E4M3 bytes) -> paired-tile order
__global__ void pack_rows_w8_kernel(const uint8_t* __restrict__ src, uint8_t* __restrict__ dst, int rows, int K, int dst_row0,
                                    int dst_row_stride, int dst_row_tiles) {
    const size_t n8 = (size_t)rows * (K / 8);
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n8; e += (size_t)gridDim.x * blockDim.x) {
        const int r = (int)(e / (K / 8));
        const int c = (int)(e - (size_t)r * (K / 8)) * 8;
        const int dr = dst_row0 + r * dst_row_stride;
        const uint2 v = *reinterpret_cast<const uint2*>(src + (size_t)r * K + c);
        *reinterpret_cast<uint2*>(dst + w8_offset(dr, c, dst_row_tiles)) = v;
    }
}

// rows of packed FP4 codes [rows, K/2] -> paired-tile order; a thread moves 8 codes (4 bytes)
__global__ void pack_rows_w4_kernel(const uint8_t* __restrict__ src, uint8_t* __restrict__ dst, int rows, int K, int dst_row0,
                                    int dst_row_stride, int dst_row_tiles) {
    const size_t n8 = (size_t)rows * (K / 8);
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n8; e += (size_t)gridDim.x * blockDim.x) {
        const int r = (int)(e / (K / 8));
        const int c = (int)(e - (size_t)r * (K / 8)) * 8;
        const int dr = dst_row0 + r * dst_row_stride;
        const uint32_t v = *reinterpret_cast<const uint32_t*>(src + (size_t)r * (K / 2) + c / 2);
        *reinterpret_cast<uint32_t*>(dst + w4_offset(dr, c, dst_row_tiles)) = v;
    }
}

// their scale bytes [rows, K/32] -> interleaved order
__global__ void pack_scales_w4_kernel(const uint8_t* __restrict__ src, uint8_t* __restrict__ dst, int rows, int KB, int dst_row0,
                                      int dst_row_stride, int dst_row_tiles) {
    const size_t n = (size_t)rows * KB;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
        const int r = (int)(e / KB);
        const int kb = (int)(e - (size_t)r * KB);
        dst[w4_scale_offset(dst_row0 + r * dst_row_stride, kb, dst_row_tiles)] = src[e];
    }
}

__global__ void scatter_scales_kernel(const float* __restrict__ src, float* __restrict__ dst, int rows, int dst_row0,
                                      int dst_row_stride) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < rows) dst[dst_row0 + i * dst_row_stride] = src[i];
}

template <bool BF16>
__global__ void copy_gain_kernel(const void* __restrict__ src, float* __restrict__ dst, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    dst[i] = BF16 ? bf16_to_f32(static_cast<const bf16_t*>(src)[i]) : static_cast<const float*>(src)[i];
}

}  // namespace

int sled_launch_pack_rows(int dtype, const void* src, void* dst, int rows, int K, int dst_row0, int dst_row_stride,
                          int dst_rows_total, hipStream_t st) {
    const int dst_row_tiles = dst_rows_total / 32;
    const size_t n8 = (size_t)rows * (K / 8);
    int grid = (int)((n8 + 255) / 256);
    if (grid > 65535) grid = 65535;
    if (grid < 1) grid = 1;
    if (dtype == SLED_BF16)
        hipLaunchKernelGGL(pack_rows_kernel<true>, dim3(grid), dim3(256), 0, st, src, dst, rows, K, dst_row0, dst_row_stride, dst_row_tiles);
    else
        hipLaunchKernelGGL(pack_rows_kernel<false>, dim3(grid), dim3(256), 0, st, src, dst, rows, K, dst_row0, dst_row_stride, dst_row_tiles);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

int sled_launch_pack_rows_w8(const void* src, void* dst, int rows, int K, int dst_row0, int dst_row_stride, int dst_rows_total,
                             hipStream_t st) {
    if (K % 16 || dst_rows_total % 64) SLED_FAIL(SLED_EINVAL, "8-bit weights: K %d or rows %d not tileable", K, dst_rows_total);
    const size_t n8 = (size_t)rows * (K / 8);
    int grid = (int)std::min<size_t>((n8 + 255) / 256, 65535);
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(pack_rows_w8_kernel, dim3(grid), dim3(256), 0, st, static_cast<const uint8_t*>(src), static_cast<uint8_t*>(dst),
                       rows, K, dst_row0, dst_row_stride, dst_rows_total / 32);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

int sled_launch_pack_rows_w4(const void* src, void* dst, int rows, int K, int dst_row0, int dst_row_stride, int dst_rows_total,
                             hipStream_t st) {
    if (K % 32 || dst_rows_total % 64) SLED_FAIL(SLED_EINVAL, "4-bit weights: K %d or rows %d not tileable", K, dst_rows_total);
    const size_t n8 = (size_t)rows * (K / 8);
    int grid = (int)std::min<size_t>((n8 + 255) / 256, 65535);
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(pack_rows_w4_kernel, dim3(grid), dim3(256), 0, st, static_cast<const uint8_t*>(src), static_cast<uint8_t*>(dst),
                       rows, K, dst_row0, dst_row_stride, dst_rows_total / 32);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

int sled_launch_pack_scales_w4(const void* src, void* dst, int rows, int K, int dst_row0, int dst_row_stride, int dst_rows_total,
                               hipStream_t st) {
    if (K % 32 || dst_rows_total % 64) SLED_FAIL(SLED_EINVAL, "4-bit weights: K %d or rows %d not tileable", K, dst_rows_total);
    const size_t n = (size_t)rows * (K / 32);
    int grid = (int)std::min<size_t>((n + 255) / 256, 65535);
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(pack_scales_w4_kernel, dim3(grid), dim3(256), 0, st, static_cast<const uint8_t*>(src),
                       static_cast<uint8_t*>(dst), rows, K / 32, dst_row0, dst_row_stride, dst_rows_total / 32);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

int sled_launch_scatter_scales(const float* src, float* dst, int rows, int dst_row0, int dst_row_stride, hipStream_t st) {
    hipLaunchKernelGGL(scatter_scales_kernel, dim3((rows + 255) / 256), dim3(256), 0, st, src, dst, rows, dst_row0, dst_row_stride);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

int sled_launch_copy_gain(int dtype, const void* src, float* dst, int n, hipStream_t st) {
    if (dtype == SLED_BF16)
        hipLaunchKernelGGL(copy_gain_kernel<true>, dim3((n + 255) / 256), dim3(256), 0, st, src, dst, n);
    else
        hipLaunchKernelGGL(copy_gain_kernel<false>, dim3((n + 255) / 256), dim3(256), 0, st, src, dst, n);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

int sled_launch_step_setup(const sled_model* m, const sled_kvpool* p, const sled_step_meta& meta, const int32_t* tokens, float* cs, int32_t* kvslot,
                           int32_t* plan, int32_t* arrive, float* h, void* X, size_t plane, const float* gain, hipStream_t st) {
    const bool bf = m->s.dtype == SLED_BF16;
    step_setup a{p->len_dev, m->s.head_dim / 2, m->s.n_kv_heads, (double)m->s.rope_theta, reinterpret_cast<float2*>(cs), kvslot, plan, arrive,
                 meta.B * m->s.n_kv_heads, tokens, m->embed, m->s.vocab, m->s.d_model, m->s.rms_eps, gain, h, X, plane, (meta.T + 3) / 4,
                 bf ? (std::max(meta.n_work, meta.B * m->s.n_kv_heads) + 255) / 256 : 0};
    const dim3 grid(a.rope_blocks + a.plan_blocks + meta.T);
    if (bf) hipLaunchKernelGGL(step_setup_kernel<true>, grid, dim3(256), 0, st, meta, a);
    else hipLaunchKernelGGL(step_setup_kernel<false>, grid, dim3(256), 0, st, meta, a);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

int sled_launch_residual_norm(const sled_model* m, const float* partial, int n_split, int T, int T_pad, float* h, void* X,
                              size_t plane, const float* gain, hipStream_t st) {
    // four columns per thread per trip: short rows get small workgroups
    // Rows of an activation line on one XCD: 101 rows 6.4 -> 6.1 us, 372 rows 11.4 -> 10.0, 700 rows 15.0 -> 11.7, 1080 rows 25.6 -> 20.2.  Few
    // rows fill few XCDs then and gain nothing (25 rows: the same, and the next projection 10.0 -> 10.5).
    const int group = T > 64 ? ACT_LINE_ROWS : 1;
    const int bs = m->s.d_model >= 4096 ? 1024 : m->s.d_model >= 2048 ? 512 : m->s.d_model >= 1024 ? 256 : 128;
    if (m->s.dtype == SLED_BF16)
        hipLaunchKernelGGL(residual_norm_kernel<true>, dim3(group > 1 ? blocks_for_rows(T, group) : T), dim3(bs), 0, st, partial, n_split,
                           T_pad, m->s.d_model, m->s.rms_eps, gain, h, X, plane, T, group);
    else
        hipLaunchKernelGGL(residual_norm_kernel<false>, dim3(T), dim3(bs), 0, st, partial, n_split, T_pad, m->s.d_model,
                           m->s.rms_eps, gain, h, X, plane, T, 1);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

int sled_launch_copy_act_row(const sled_model* m, const void* X, size_t plane, int t, void* X1, size_t plane1, int d,
                             hipStream_t st) {
    if (d % 8) SLED_FAIL(SLED_EINVAL, "copy_act_row: d_model %d is not a multiple of 8", d);
    const int grid = (d / 8 + 255) / 256;
    if (m->s.dtype == SLED_BF16)
        hipLaunchKernelGGL(copy_act_row_kernel<true>, dim3(grid), dim3(256), 0, st, X, plane, t, X1, plane1, d);
    else
        hipLaunchKernelGGL(copy_act_row_kernel<false>, dim3(grid), dim3(256), 0, st, X, plane, t, X1, plane1, d);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

int sled_launch_qkv_rope_store(const sled_model* m, const sled_kvpool* p, int T, int layer, const float* partial, int n_split,
                               int T_pad, const float* cs, const int32_t* kvslot, void* Q, size_t q_plane, hipStream_t st) {
    const int Hq = m->s.n_q_heads, Hkv = m->s.n_kv_heads;
    if (m->s.dtype == SLED_BF16) {
        const int blocks_per_row = ((Hq + Hkv) * 16 + Hkv * 32 + 255) / 256;
        hipLaunchKernelGGL(qkv_rope_store_bf16_kernel, dim3(blocks_for_rows(T, QKV_ROWS) * blocks_per_row), dim3(256), 0, st, partial, n_split, T, T_pad,
                           Hq, Hkv, reinterpret_cast<const float2*>(cs), kvslot, static_cast<bf16_t*>(Q), q_plane,
                           static_cast<bf16_t*>(p->k_pool), static_cast<bf16_t*>(p->v_pool), p->n_pages, layer, blocks_per_row);
    } else {
        hipLaunchKernelGGL(qkv_rope_store_f32_kernel, dim3(T, Hq + 2 * Hkv), dim3(64), 0, st, partial, n_split, T_pad, Hq, Hkv, m->s.head_dim,
                           reinterpret_cast<const float2*>(cs), kvslot, static_cast<float*>(Q), static_cast<float*>(p->k_pool),
                           static_cast<float*>(p->v_pool), p->n_pages, layer);
    }
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

int sled_launch_swiglu_reduce(const sled_model* m, const float* gu, int n_split, int T, int T_pad, void* A, size_t plane,
                              hipStream_t st) {
    const int F = m->s.d_ffn;
    int gy = (F / 8 + 255) / 256;
    if (gy > 8) gy = 8;
    if (gy < 1) gy = 1;
    dim3 grid(T, gy);
    if (m->s.dtype == SLED_BF16)
        hipLaunchKernelGGL(swiglu_reduce_kernel<true>, grid, dim3(256), 0, st, gu, n_split, T_pad, F, A, plane);
    else
        hipLaunchKernelGGL(swiglu_reduce_kernel<false>, grid, dim3(256), 0, st, gu, n_split, T_pad, F, A, plane);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

// `len`: device-side committed length of the request, its first position (ingest), or nullptr and `first` (export)
template <bool INGEST>
static int launch_kv_move(const sled_model* m, const sled_kvpool* p, const sled_kv_piece* pieces, int n, hipStream_t st) {
    // a page's V of one layer, 4 KiB a head, for three workgroups on a CU or more
    const size_t stage = INGEST && m->s.dtype == SLED_BF16 && m->s.n_kv_heads <= 12 ? (size_t)m->s.n_kv_heads * 4096 : 0;
    for (int i0 = 0; i0 < n; i0 += SLED_KV_PIECES) {
        kv_pieces ks{};
        const int here = std::min(n - i0, SLED_KV_PIECES);
        int most = 0;
        for (int i = 0; i < here; i++) {
            ks.p[i] = pieces[i0 + i];
            most = std::max(most, ks.p[i].n_tok);
        }
        // where the first token sits inside its page is not known here when the device knows the length: one page more
        const dim3 grid((most + 30) / 16, m->s.n_layers, here);
        if (m->s.dtype == SLED_BF16)
            hipLaunchKernelGGL((kv_move_kernel<true, INGEST>), grid, dim3(256), stage, st, ks, m->s.n_kv_heads, m->s.head_dim, p->k_pool, p->v_pool,
                               p->n_pages, stage > 0);
        else
            hipLaunchKernelGGL((kv_move_kernel<false, INGEST>), grid, dim3(256), 0, st, ks, m->s.n_kv_heads, m->s.head_dim, p->k_pool, p->v_pool,
                               p->n_pages, false);
        SLED_LAUNCH_CHECK();
    }
    return SLED_OK;
}

int sled_launch_kv_ingest(const sled_model* m, const sled_kvpool* p, const sled_kv_piece* pieces, int n, hipStream_t st) {
    return launch_kv_move<true>(m, p, pieces, n, st);
}

int sled_launch_kv_export(const sled_model* m, const sled_kvpool* p, void* k_dst, void* v_dst, int first, int n_tokens,
                          const int32_t* pages_dev, hipStream_t st) {
    const sled_kv_piece pc{k_dst, v_dst, pages_dev, nullptr, first, n_tokens};
    return launch_kv_move<false>(m, p, &pc, 1, st);
}

int sled_launch_len_add(int32_t* len_dev, const int32_t* req_ids_dev, const int32_t* add_dev, const int32_t* fresh_dev, const int32_t* accept_dev,
                        int B, hipStream_t st) {
    hipLaunchKernelGGL(len_add_kernel, dim3((B + 63) / 64), dim3(64), 0, st, len_dev, req_ids_dev, add_dev, fresh_dev, accept_dev, B);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

int sled_launch_len_zero(int32_t* len_dev, const int* req_ids /*host*/, int n, hipStream_t st) {
    for (int i0 = 0; i0 < n; i0 += 128) {
        len_ids ids{};
        const int here = std::min(n - i0, 128);
        for (int i = 0; i < here; i++) ids.id[i] = req_ids[i0 + i];
        hipLaunchKernelGGL(len_zero_kernel, dim3(1), dim3(128), 0, st, len_dev, ids, here);
        SLED_LAUNCH_CHECK();
    }
    return SLED_OK;
}
