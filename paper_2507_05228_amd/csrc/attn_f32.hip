// fp32 partial attention (Algorithm 3) and its fused variant (running merge of Algorithm 4).
// One wavefront owns one (batch, head, packed query row[, kv shard]) and walks the key rows in
// chunks of 64: lane c scores key c (a = scale q.k + s), the row maximum and the sum of
// exponentials are 64-lane reductions, and u~ is accumulated with the lanes spread over the
// head dimension.  Plain fp32 FMA + expf, any head dimension and alignment; the usual case runs the MFMA kernel below.
#include "common.h"
#include "device_utils.h"

#define F32_MAX_D 256

template <bool FUSED>
__global__ __launch_bounds__(256) void attn_f32_kernel(
    const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v, int B, int H, int Hkv,
    int d, int N, int S, float scale, int causal, int64_t qs_b, int64_t qs_h, int64_t qs_n, int64_t ks_b,
    int64_t ks_h, int64_t ks_n, const int32_t *__restrict__ q_rowmap, const int32_t *__restrict__ kv_rowmap,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ pos_packed,
    const int32_t *__restrict__ pos_kv, float *__restrict__ m_out,
    float *__restrict__ e_out, float *__restrict__ u_out, int u_mode, float *__restrict__ o_out, int64_t o_ld,
    const int32_t *__restrict__ o_rowmap) {
    __shared__ float qs[4][F32_MAX_D];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = blockIdx.x * 4 + wave;
    const int h = blockIdx.y;
    const int b = FUSED ? blockIdx.z : blockIdx.z / S;
    const int kk = FUSED ? 0 : blockIdx.z % S;
    const bool live = r < N;                          // wave-uniform
    const int rr = live ? r : N - 1;
    const int g = h / (H / Hkv);
    const float *qrow = q + b * qs_b + h * qs_h + (int64_t)(q_rowmap ? q_rowmap[rr] : rr) * qs_n;
    for (int i = lane; i < d; i += 64) qs[wave][i] = qrow[i];
    __syncthreads();
    if (!live) return;
    const int pos_q = pos_packed[rr];
    const int c_begin = FUSED ? 0 : offsets[kk];
    const int c_end = FUSED ? N : offsets[kk + 1];
    const float *kb = k + b * ks_b + g * ks_h;
    const float *vb = v + b * ks_b + g * ks_h;

    float m = -INFINITY, e = 0.f;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int c0 = c_begin; c0 < c_end; c0 += 64) {
        const int c = c0 + lane;
        const bool valid = c < c_end;
        const int cc = valid ? c : c_end - 1;
        const int64_t krow = kv_rowmap ? kv_rowmap[cc] : cc;
        float s = -INFINITY;
        const bool seen = valid && (!causal || pos_kv[cc] <= pos_q);
        if (seen) {
            const float *kr = kb + krow * ks_n;
            float dot = 0.f;
            for (int i = 0; i < d; ++i) dot = fmaf(qs[wave][i], kr[i], dot);
            s = dot * scale;
        }
        if (!__any(seen)) continue;                   // (not read off the maximum: that leaves NaN scores out)
        const float cm = wave_max(s);
        const float m_new = fmaxf(m, cm);
        const float alpha = (m == -INFINITY) ? 0.f : expf(m - m_new);
        const float p = (s == -INFINITY) ? 0.f : expf(s - m_new);
        e = e * alpha + wave_sum(p);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] *= alpha;
        const int nc = min(64, c_end - c0);
        for (int t = 0; t < nc; ++t) {
            const float pt = __shfl(p, t, WAVE);
            if (pt == 0.f) continue;                  // wave-uniform
            const int64_t vrow = __shfl((int)krow, t, WAVE);
            const float *vr = vb + vrow * ks_n;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                int i = lane + 64 * j;
                if (i < d) acc[j] = fmaf(pt, vr[i], acc[j]);
            }
        }
        m = m_new;
    }
    if (FUSED) {
        const float inv = e > 0.f ? 1.0f / e : 0.f;
        float *op = o_out + ((int64_t)b * N + (o_rowmap ? o_rowmap[r] : r)) * o_ld + (int64_t)h * d;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int i = lane + 64 * j;
            if (i < d) op[i] = acc[j] * inv;
        }
    } else {
        const int64_t me = (((int64_t)b * H + h) * S + kk) * N + r;
        if (lane == 0) { m_out[me] = m; e_out[me] = e; }
        const float f = (u_mode == CASCADE_U_NORMALISED) ? (e > 0.f ? 1.0f / e : 0.f) : 1.0f;
        float *up = u_out + ((((int64_t)b * S + kk) * H + h) * N + r) * d;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int i = lane + 64 * j;
            if (i < d) up[i] = acc[j] * f;
        }
    }
}

// a + b rounded, and what the rounding left out (Knuth's two-sum)
__device__ __forceinline__ float two_sum(float a, float b, float &err) {
    const float s = a + b, bb = s - a;
    err = (a - (s - bb)) + (b - bb);
    return s;
}

// Main fp32 kernel (d % 4 == 0, 16-byte aligned rows): 16 query rows per workgroup, its NW wavefronts take every NW-th
// tile of 16 keys, both products on fp32 MFMA 16x16x4 (fp32 products and sums).  S^T = K Q^T leaves a lane 4 keys of one
// query, which are the B operand of O^T = V^T P^T as they stand (MFMA r takes key 4g + r from lane group g); the next
// tile's K and V are requested before the current one is multiplied; their running (m, e, O) states meet in LDS.
// Bound by the chain of tiles, hence 4 or 8 wavefronts on one query tile (128 tokens, 4 heads of 16: 47 us with one
// wavefront per row and a key per lane, 7 us here).  DB: blocks of 16 head dimensions.  ALONE (partials of short shards):
// every wavefront takes a query tile of its own through the whole shard, and nothing meets in LDS.  NW: wavefronts of a
// workgroup that share a query tile's keys.
template <int DB, bool FUSED, bool ALONE = false, int NW = 4>
__global__ __launch_bounds__(64 * NW) void attn_f32_mfma_kernel(
    const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v, int B, int H, int Hkv,
    int d, int N, int S, float scale, int causal, int64_t qs_b, int64_t qs_h, int64_t qs_n, int64_t ks_b,
    int64_t ks_h, int64_t ks_n, const int32_t *__restrict__ q_rowmap, const int32_t *__restrict__ kv_rowmap,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ pos_packed,
    const int32_t *__restrict__ pos_kv, float *__restrict__ m_out,
    float *__restrict__ e_out, float *__restrict__ u_out, int u_mode, float *__restrict__ o_out, int64_t o_ld,
    const int32_t *__restrict__ o_rowmap) {
    static_assert(!(FUSED && ALONE) && (!ALONE || NW == 4), "short shards: partials only");
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = (ALONE ? (int)blockIdx.x * 4 + wave : (int)blockIdx.x) * 16, h = blockIdx.y;
    if (ALONE && r0 >= N) return;                         // (no barrier in this instance)
    const int b = FUSED ? blockIdx.z : blockIdx.z / S, kk = FUSED ? 0 : blockIdx.z % S;
    const int gk = h / (H / Hkv);
    const int rq = min(r0 + l16, N - 1);
    const float *qrow = q + b * qs_b + h * qs_h + (int64_t)(q_rowmap ? q_rowmap[rq] : rq) * qs_n;
    const int pos_q = pos_packed[rq];
    const int c_begin = FUSED ? 0 : offsets[kk], c_end = FUSED ? N : offsets[kk + 1];
    const float *kb = k + b * ks_b + gk * ks_h, *vb = v + b * ks_b + gk * ks_h;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 qf[DB], O[DB], kf[2][DB], vf[2][DB];
    int pk[2][4];
#pragma unroll
    for (int x = 0; x < DB; ++x) {
        qf[x] = zero;
        O[x] = zero;
        if (16 * x + 4 * g < d) qf[x] = *(const f32x4 *)(qrow + 16 * x + 4 * g);
    }
    // tile at key c: K row c + lane%16, dims 4g.. of every block; V rows c + 4g + r, dim lane%16 of every block
    auto request = [&](int slot, int c) {
        const int ck = min(c + l16, c_end - 1);
        const float *kr = kb + (int64_t)(kv_rowmap ? kv_rowmap[ck] : ck) * ks_n;
#pragma unroll
        for (int x = 0; x < DB; ++x) {
            kf[slot][x] = zero;
            if (16 * x + 4 * g < d) kf[slot][x] = *(const f32x4 *)(kr + 16 * x + 4 * g);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int cv = min(c + 4 * g + r, c_end - 1);
            const float *vr = vb + (int64_t)(kv_rowmap ? kv_rowmap[cv] : cv) * ks_n;
            pk[slot][r] = pos_kv[cv];
#pragma unroll
            for (int x = 0; x < DB; ++x) vf[slot][x][r] = 16 * x + l16 < d ? vr[16 * x + l16] : 0.f;
        }
    };
    float m = -INFINITY, ml = 0.f, e = 0.f;               // of query lane%16; e still split over the lane groups
    auto tile = [&](int slot, int c) {
        // Four chains (shorter, and of smaller sums), added with their rounding errors kept: with logits in the hundreds
        // the last roundings of a score are what an error of 1e-5 in an exponential is made of.  A scaled score is
        // sc + rest, and the maximum that the exponentials refer to is m + ml likewise.
        f32x4 part[4] = {zero, zero, zero, zero}, sc, lo;
#pragma unroll
        for (int x = 0; x < DB; ++x)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                part[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[slot][x][j], qf[x][j], part[j], 0, 0, 0);
        f32x4 dot;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float e0, e1, e2;
            const float a = two_sum(part[0][r], part[1][r], e0), c2 = two_sum(part[2][r], part[3][r], e1);
            dot[r] = two_sum(a, c2, e2);
            lo[r] = (e0 + e1) + e2;
        }
        float cm = -INFINITY;
        bool any_seen = false;                            // (not read off the maximum: that leaves NaN scores out)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool seen = c + 4 * g + r < c_end && (!causal || pk[slot][r] <= pos_q);
            any_seen |= seen;
            sc[r] = seen ? dot[r] * scale : -INFINITY;
            lo[r] = fmaf(dot[r], scale, -sc[r]) + lo[r] * scale;
            cm = fmaxf(cm, sc[r]);
        }
        if (!__any(any_seen)) return;                     // no query of the tile sees a key of it
        cm = fmaxf(cm, __shfl_xor(cm, 16, WAVE));
        cm = fmaxf(cm, __shfl_xor(cm, 32, WAVE));
        float cl = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) cl = sc[r] == cm ? fmaxf(cl, lo[r]) : cl;
        cl = fmaxf(cl, __shfl_xor(cl, 16, WAVE));
        cl = fmaxf(cl, __shfl_xor(cl, 32, WAVE));
        const float m_new = fmaxf(m, cm);
        float ml_new = m == m_new ? ml : cl;
        if (m == cm) ml_new = fmaxf(ml, cl);
        const float alpha = m == -INFINITY ? 0.f : expf((m - m_new) + (ml - ml_new));
        f32x4 p;
        float sum = 0.f;
        bool odd = false;                                 // a value that 0 x does not make 0
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = sc[r] == -INFINITY ? 0.f : expf((sc[r] - m_new) + (lo[r] - ml_new));
            sum += p[r];
#pragma unroll
            for (int x = 0; x < DB; ++x) odd |= !(fabsf(vf[slot][x][r]) < INFINITY);
        }
        e = e * alpha + sum;
#pragma unroll
        for (int x = 0; x < DB; ++x) O[x] *= alpha;
        m = m_new;
        ml = ml_new;
        if (!__any(odd)) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int x = 0; x < DB; ++x) O[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[slot][x][r], p[r], O[x], 0, 0, 0);
        } else {                                          // keys a query does not see contribute nothing, whatever they hold
#pragma unroll
            for (int r = 0; r < 4; ++r)
                for (int gg = 0; gg < 4; ++gg) {
                    const float pt = __shfl(p[r], 16 * gg + l16, WAVE);
#pragma unroll
                    for (int x = 0; x < DB; ++x)
#pragma unroll
                        for (int y = 0; y < 4; ++y) {
                            const float vv = __shfl(vf[slot][x][r], 16 * gg + 4 * g + y, WAVE);
                            if (pt != 0.f) O[x][y] = fmaf(pt, vv, O[x][y]);
                        }
                }
        }
    };
    constexpr int STEP = ALONE ? 16 : 16 * NW;            // 16 keys x 1 or NW wavefronts
    int c = c_begin + (ALONE ? 0 : 16 * wave);
    if (c < c_end) {
        request(0, c);
        for (;;) {
            if (c + STEP < c_end) request(1, c + STEP);
            tile(0, c);
            c += STEP;
            if (c >= c_end) break;
            if (c + STEP < c_end) request(0, c + STEP);
            tile(1, c);
            c += STEP;
            if (c >= c_end) break;
        }
    }
    e += __shfl_xor(e, 16, WAVE);
    e += __shfl_xor(e, 32, WAVE);
    // Partials: m is stored as one float, and e and the unnormalised u refer to that one.
    auto refer_to_stored = [](float mh, float mlo, float &corr) {
        corr = 1.0f;
        if (!(fabsf(mh) < INFINITY)) return mh;
        float rest;
        const float m_st = two_sum(mh, mlo, rest);
        corr = expf(rest);
        return m_st;
    };
    if constexpr (ALONE) {
        float corr;
        const float m_st = refer_to_stored(m, ml, corr);
        const float f = u_mode == CASCADE_U_NORMALISED ? (e > 0.f ? 1.0f / e : 0.f) : corr;
        const int r = r0 + l16;
        if (r >= N) return;
        float *dst = u_out + ((((int64_t)b * S + kk) * H + h) * N + r) * d + 4 * g;
#pragma unroll
        for (int x = 0; x < DB; ++x)
            if (16 * x + 4 * g < d) *(f32x4 *)(dst + 16 * x) = O[x] * f;
        if (g == 0) {
            const int64_t me = (((int64_t)b * H + h) * S + kk) * N + r;
            m_out[me] = m_st;
            e_out[me] = e * corr;
        }
        return;
    }
    __shared__ float sm[NW][16], sl[NW][16], se[NW][16];
    __shared__ __attribute__((aligned(16))) float so[NW][256];
    if (g == 0) { sm[wave][l16] = m; sl[wave][l16] = ml; se[wave][l16] = e; }
    __syncthreads();
    // merge: thread -> query tid/16, dim tid%16 of every block
    const int qi = (tid >> 4) & 15, di = tid & 15, r = tid < 256 ? r0 + qi : N;   // (threads past the first 256 write nothing)
    float mm = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) mm = fmaxf(mm, sm[w][qi]);
    float f[NW], ee = 0.f, mml = -INFINITY;
    bool has[NW];                                          // the wavefront has seen a key (NaN scores: e is NaN, m may be -inf)
#pragma unroll
    for (int w = 0; w < NW; ++w) mml = sm[w][qi] == mm ? fmaxf(mml, sl[w][qi]) : mml;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        has[w] = se[w][qi] != 0.f;
        f[w] = has[w] ? expf((sm[w][qi] - mm) + (sl[w][qi] - mml)) : 0.f;
        ee += has[w] ? f[w] * se[w][qi] : 0.f;
    }
    float m_st = mm, corr = 1.0f;
    if (!FUSED) m_st = refer_to_stored(mm, mml, corr);
    const float norm = FUSED || u_mode == CASCADE_U_NORMALISED ? (ee > 0.f ? 1.0f / ee : 0.f) : corr;
    float *dst = FUSED ? o_out + ((int64_t)b * N + (r < N && o_rowmap ? o_rowmap[r] : r)) * o_ld + (int64_t)h * d
                       : u_out + ((((int64_t)b * S + kk) * H + h) * N + r) * d;
#pragma unroll
    for (int x = 0; x < DB; ++x) {
        if (x) __syncthreads();
        *(f32x4 *)&so[wave][l16 * 16 + 4 * g] = O[x];
        __syncthreads();
        float o = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) o += has[w] ? f[w] * so[w][tid & 255] : 0.f;
        if (r < N && 16 * x + di < d) dst[16 * x + di] = o * norm;
    }
    if (!FUSED && di == 0 && r < N) {
        const int64_t me = (((int64_t)b * H + h) * S + kk) * N + r;
        m_out[me] = m_st;
        e_out[me] = ee * corr;
    }
}

int32_t launch_attn_f32(const cascade_plan *p, const AttnArgs &a, hipStream_t s) {
    if (a.d > F32_MAX_D) return CASCADE_EUNSUPPORTED;
    const cascade_plan *kvp = kv_plan(p);             // key rows walk the key/value partition's packed order
    const int N = p->seq_len, S = kvp->n_shards;
    if (a.H > 65535 || (int64_t)a.B * S > 65535) return CASCADE_EUNSUPPORTED;
    dim3 grid((N + 3) / 4, a.H, a.fused ? a.B : a.B * S);
    const int causal = a.mask_kind == CASCADE_MASK_CAUSAL;
    // 16-byte pieces of q and k rows; 128 head dimensions hold their two tiles of K and V in registers
    const bool aligned = a.d % 4 == 0 && a.d <= 128 &&
                         (a.qs_b | a.qs_h | a.qs_n | a.ks_b | a.ks_h | a.ks_n) % 4 == 0 && ((uintptr_t)a.q | (uintptr_t)a.k) % 16 == 0;
    if (aligned) {
        dim3 mgrid((N + 15) / 16, a.H, a.fused ? a.B : a.B * S);
        // Partials of short shards, a query tile per wavefront: shards of one key tile leave three of the four wavefronts
        // idle, and launches that fill the CUs anyway (eight workgroups per CU and more) are done sooner without the
        // exchange, up to the 64 rows measured.  Plain-FMA kernel / tile per workgroup / per wavefront (us): 2 x 512
        // tokens, 12 heads of 64, 256 shards 2213 / 4786 / 1481, 64 shards 689 / 1163 / 299, 32 shards 493 / 591 / 159, 16
        // shards 410 / 316 / 125, 8 shards 368 / 176 / 110; 8 heads of 128, 64 shards 806 / 1114 / 293; 4 heads of 16,
        // 64 shards 197 / 105 / 60.
        const int64_t wgs = (int64_t)mgrid.x * mgrid.y * mgrid.z;
        const bool alone = !a.fused && (uintptr_t)a.u % 16 == 0 && (N <= 16 * (int64_t)S || (N <= 64 * (int64_t)S && wgs >= 2048));
        if (alone) mgrid.x = (N + 63) / 64;
        // Eight wavefronts per query tile where there are more key tiles than four, at most 256 workgroups, one to a CU, and up to 32
        // head dimensions: half the chain of tiles.  Layers of d head dimensions, 4 / 8 wavefronts (us, replayed from a graph): 4 heads of
        // 16, 128 tokens 24.9 / 22.9, 512 38.2 / 30.5, 1024 53.0 / 39.9; 12 of 16, 2 x 160 32.9 / 31.0; 4 heads of 32, 128 24.6 / 24.3,
        // 1024 51.6 / 43.7; 12 of 32, 128 32.2 / 32.3, 333 43.8 / 42.0.  Called one by one, the host enqueues the seven launches in 27
        // and bounds up to 128 tokens.  Wider heads have no registers for it (half as many as one wavefront per SIMD): 4 of 64, 128
        // 29.7 / 37.3, 1024 75.7 / 101.
        const bool eight = N > 64 && wgs <= 256;
#define ATTN_F32(DB, FUSED, ALONE, NW)                                                                                           \
    hipLaunchKernelGGL((attn_f32_mfma_kernel<DB, FUSED, ALONE, NW>), mgrid, dim3(64 * NW), 0, s, (const float *)a.q, (const float *)a.k,    \
                       (const float *)a.v, a.B, a.H, a.Hkv, a.d, N, S, a.scale, causal, a.qs_b, a.qs_h, a.qs_n, a.ks_b,      \
                       a.ks_h, a.ks_n, a.q_rowmap, a.kv_rowmap, kvp->offsets_d, p->pos_packed_d, kvp->pos_packed_d, a.m,     \
                       a.e, a.u, a.u_mode, (float *)a.o, a.o_ld, a.o_rowmap)
#define ATTN_F32_D(DB) do { if (a.fused && DB <= 2 && eight) ATTN_F32(DB, true, false, (DB <= 2 ? 8 : 4)); else if (a.fused) ATTN_F32(DB, true, false, 4); \
                            else if (alone) ATTN_F32(DB, false, true, 4); else ATTN_F32(DB, false, false, 4); } while (0)
        if (a.d <= 16) ATTN_F32_D(1);
        else if (a.d <= 32) ATTN_F32_D(2);
        else if (a.d <= 64) ATTN_F32_D(4);
        else ATTN_F32_D(8);
#undef ATTN_F32_D
#undef ATTN_F32
        CASCADE_HIP_TRY(hipGetLastError());
        return CASCADE_OK;
    }
    if (a.fused)
        hipLaunchKernelGGL(attn_f32_kernel<true>, grid, dim3(256), 0, s, (const float *)a.q, (const float *)a.k,
                           (const float *)a.v, a.B, a.H, a.Hkv, a.d, N, S, a.scale, causal, a.qs_b, a.qs_h, a.qs_n,
                           a.ks_b, a.ks_h, a.ks_n, a.q_rowmap, a.kv_rowmap, kvp->offsets_d, p->pos_packed_d, kvp->pos_packed_d,
                           a.m, a.e,
                           a.u, a.u_mode, (float *)a.o, a.o_ld, a.o_rowmap);
    else
        hipLaunchKernelGGL(attn_f32_kernel<false>, grid, dim3(256), 0, s, (const float *)a.q, (const float *)a.k,
                           (const float *)a.v, a.B, a.H, a.Hkv, a.d, N, S, a.scale, causal, a.qs_b, a.qs_h, a.qs_n,
                           a.ks_b, a.ks_h, a.ks_n, a.q_rowmap, a.kv_rowmap, kvp->offsets_d, p->pos_packed_d, kvp->pos_packed_d,
                           a.m, a.e,
                           a.u, a.u_mode, (float *)a.o, a.o_ld, a.o_rowmap);
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}
