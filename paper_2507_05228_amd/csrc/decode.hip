// Token-sharded KV-cache decode (Cost Optimizations appendix, "Caching"): the newest token's query
// row against the cached keys / values of every kv shard S_k, giving one partial (m, e, u~) per shard,
// which cascade_lse_merge then combines exactly as in the prefill path (the merge of Algorithm 4).
// Every cached key is at or before the new position, so there is no mask; only the shard lengths.
//
// Each cached K and V row is read once.  decode_attn_kernel takes every type, head dimension and number of query heads per
// kv head; decode_attn_mfma_kernel (below) the bf16 caches of 4 and 8 query heads per kv head.  WPS wavefronts share one (shard, kv head,
// sequence): 1 for small shards (four shards per workgroup, no LDS, no barrier), 4 for large ones and
// where a launch would be as long as the walk of one shard (more loads in flight per shard; the four
// running states are merged through LDS).  The REP query
// heads that share the kv head are processed together so the cache is read once for all of them.
// A row is spread over LPR = d / VEC lanes (16 bytes per lane), so one wavefront instruction reads
// 64 / LPR consecutive rows, fully coalesced, and the rows of the next two steps are requested before
// the arithmetic of the current one.  Scores are reduced over the LPR lanes with xor shuffles; each
// lane group keeps a running (m, e, u~) per head (the same online recurrence as the fused prefill
// kernel); the lane groups of a wavefront are merged with shuffles at the end.
#include <cmath>
#include <type_traits>
#include "common.h"
#include "device_utils.h"

#define LOG2E 1.4426950408889634f
#define LN2 0.6931471805599453f

struct DecodeParams {
    const void *q, *kc, *vc;
    const int32_t *shard_len;
    float *m, *e, *u;
    int32_t B, H, Hkv, S, cap, d;
    float scale, scale_log2;
    int32_t u_mode;
    int32_t per_head;        // 1: one query head per workgroup (kv head = head / rep)
    int32_t rep;
};

// Sum over the LPR lanes that hold one row (LPR a power of two, lane groups aligned).  Inside a 16-lane row
// the exchange is a data-parallel-primitive modifier on the add (no LDS traffic): lanes ^1 and ^2 by quad
// permutes, then the two mirrors (a sum does not care that they reverse instead of swapping halves); wider
// groups finish with cross-row shuffles.  Every lane of the group ends with the total.
template <int LPR>
__device__ __forceinline__ float group_sum(float s) {
    auto dpp_add = [](float v, auto ctrl_tag) {
        constexpr int ctrl = decltype(ctrl_tag)::value;
        return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, 0xf, 0xf, true));
    };
    if (LPR >= 2) s = dpp_add(s, std::integral_constant<int, 0xB1>());     // quad_perm [1,0,3,2]
    if (LPR >= 4) s = dpp_add(s, std::integral_constant<int, 0x4E>());     // quad_perm [2,3,0,1]
    if (LPR >= 8) s = dpp_add(s, std::integral_constant<int, 0x141>());    // row_half_mirror
    if (LPR >= 16) s = dpp_add(s, std::integral_constant<int, 0x140>());   // row_mirror
#pragma unroll
    for (int o = 16; o < LPR; o <<= 1) s += __shfl_xor(s, o, WAVE);
    return s;
}

// Four wavefronts per shard: their states (in LDS) merged and written.  Maxima times to_log2 are in log2 units, times
// to_m in those of m.
template <int REP>
__device__ __forceinline__ void write_merged_waves(const DecodeParams &p, const float (*red_me)[REP][2], const float *red_u,
                                                   int b, int head0, int k, int d, float to_log2, float to_m) {
    for (int id = threadIdx.x; id < REP * d; id += 256) {
        const int h = id / d, i = id - h * d;
        float n = -INFINITY;
#pragma unroll
        for (int w = 0; w < 4; ++w) n = fmaxf(n, red_me[w][h][0]);
        const float n_sub = n == -INFINITY ? 0.f : n;
        float wsum = 0.f, uu = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float c = __builtin_amdgcn_exp2f((red_me[w][h][0] - n_sub) * to_log2);
            wsum += c * red_me[w][h][1];
            uu += c * red_u[(w * REP + h) * d + i];
        }
        const int head = head0 + h;
        if (i == 0) {
            p.m[((int64_t)b * p.H + head) * p.S + k] = n * to_m;
            p.e[((int64_t)b * p.H + head) * p.S + k] = wsum;
        }
        const float f = p.u_mode == CASCADE_U_NORMALISED ? (wsum > 0.f ? 1.0f / wsum : 0.f) : 1.0f;
        p.u[(((int64_t)b * p.S + k) * p.H + head) * d + i] = uu * f;
    }
}

template <int REP, typename F>
__device__ __forceinline__ void for_heads(F f) {           // f(integral_constant) for heads 0 .. REP - 1
    f(std::integral_constant<int, REP - 1>());
    if constexpr (REP > 1) for_heads<REP - 1>(f);
}

// O = 32: lanes below 32 get a[l] + a[l + 32], the others b[l - 32] + b[l]; O = 16: the same within each half of 32 lanes.
template <int O>
__device__ __forceinline__ float swap_add(float a, float b) {
    const uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
    const u32x2 r = O == 32 ? __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(x, y, false, false))
                            : __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(x, y, false, false));
    return __builtin_bit_cast(float, (uint32_t)r.x) + __builtin_bit_cast(float, (uint32_t)r.y);
}

template <typename T, int REP, int LPR, int WPS>
__global__ __launch_bounds__(256) void decode_attn_kernel(DecodeParams p) {
    constexpr int VEC = 16 / sizeof(T);
    constexpr int RPW = 64 / LPR;                          // rows per wavefront instruction
    constexpr int AHEAD = WPS == 1 ? 2 : 1;                // row steps requested ahead of their use
    typedef T vecT __attribute__((ext_vector_type(VEC)));
    __shared__ float red_me[WPS == 1 ? 1 : 4][REP][2];
    extern __shared__ float red_u[];                       // [4][REP][d] when WPS == 4

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sub = lane % LPR, rgrp = lane / LPR;
    const int wsub = wave % WPS;                           // this wavefront's share of the shard's rows
    const int k = blockIdx.x * (4 / WPS) + wave / WPS, b = blockIdx.z;
    if (k >= p.S) return;                                  // uniform over the wavefronts that share a shard
    const int head0 = p.per_head ? blockIdx.y : blockIdx.y * REP;      // first query head handled here
    const int g = p.per_head ? blockIdx.y / p.rep : blockIdx.y;        // kv head
    const int d = p.d;
    const int len = min(p.shard_len[b * p.S + k], p.cap);

    float qf[REP][VEC];
#pragma unroll
    for (int h = 0; h < REP; ++h) {
        const vecT t = *(const vecT *)((const T *)p.q + ((int64_t)b * p.H + head0 + h) * d + sub * VEC);
#pragma unroll
        for (int i = 0; i < VEC; ++i) qf[h][i] = (float)t[i] * p.scale_log2;
    }
    float mrun[REP], erun[REP], acc[REP][VEC];
#pragma unroll
    for (int h = 0; h < REP; ++h) {
        mrun[h] = -INFINITY;
        erun[h] = 0.f;
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[h][i] = 0.f;
    }

    const int64_t base = (((int64_t)b * p.Hkv + g) * p.S + k) * p.cap;
    const T *kc = (const T *)p.kc + base * d + sub * VEC;
    const T *vc = (const T *)p.vc + base * d + sub * VEC;
    const int iters = (len + WPS * RPW - 1) / (WPS * RPW);  // uniform trip count: shuffles stay convergent
    vecT kbuf[AHEAD + 1], vbuf[AHEAD + 1];
    auto row_of = [&](int it) { return (it * WPS + wsub) * RPW + rgrp; };
    auto load_row = [&](int it, vecT &kv, vecT &vv) {
        const int r = row_of(it);
        const int rr = r < len ? r : 0;                    // row 0 exists whenever the loop runs
        kv = *(const vecT *)(kc + (int64_t)rr * d);
        vv = *(const vecT *)(vc + (int64_t)rr * d);
    };
#pragma unroll
    for (int a = 0; a < AHEAD; ++a)
        if (a < iters) load_row(a, kbuf[a], vbuf[a]);
    for (int it0 = 0; it0 < iters; it0 += AHEAD + 1) {
#pragma unroll
        for (int a = 0; a <= AHEAD; ++a) {                 // unrolled so the row buffers stay in registers
            const int it = it0 + a;
            if (it >= iters) break;
            if (it + AHEAD < iters) load_row(it + AHEAD, kbuf[(a + AHEAD) % (AHEAD + 1)], vbuf[(a + AHEAD) % (AHEAD + 1)]);
            const vecT kv = kbuf[a], vv = vbuf[a];
            const bool valid = row_of(it) < len;
#pragma unroll
            for (int h = 0; h < REP; ++h) {
                float s = 0.f;
#pragma unroll
                for (int i = 0; i < VEC; ++i) s = fmaf(qf[h][i], (float)kv[i], s);
                s = group_sum<LPR>(s);
                if (!valid) s = -INFINITY;
                const float m_new = fmaxf(mrun[h], s);
                const float m_sub = m_new == -INFINITY ? 0.f : m_new;
                const float alpha = __builtin_amdgcn_exp2f(mrun[h] - m_sub);
                const float pr = __builtin_amdgcn_exp2f(s - m_sub);
                mrun[h] = m_new;
                erun[h] = erun[h] * alpha + pr;
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[h][i] = acc[h][i] * alpha + pr * (float)vv[i];
            }
        }
    }
    // merge the RPW lane groups of the wavefront (lanes with equal `sub`)
#pragma unroll
    for (int h = 0; h < REP; ++h) {
#pragma unroll
        for (int o = LPR; o < 64; o <<= 1) {
            const float m_o = __shfl_xor(mrun[h], o, WAVE), e_o = __shfl_xor(erun[h], o, WAVE);
            const float m_new = fmaxf(mrun[h], m_o);
            const float m_sub = m_new == -INFINITY ? 0.f : m_new;
            const float a0 = __builtin_amdgcn_exp2f(mrun[h] - m_sub), a1 = __builtin_amdgcn_exp2f(m_o - m_sub);
            erun[h] = erun[h] * a0 + e_o * a1;
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[h][i] = acc[h][i] * a0 + __shfl_xor(acc[h][i], o, WAVE) * a1;
            mrun[h] = m_new;
        }
    }
    if (WPS == 1) {                                        // the wavefront owns the shard: write the partial
        if (lane < LPR) {
#pragma unroll
            for (int h = 0; h < REP; ++h) {
                const int head = head0 + h;
                if (lane == 0) {
                    p.m[((int64_t)b * p.H + head) * p.S + k] = mrun[h] * LN2;     // back to the units of a
                    p.e[((int64_t)b * p.H + head) * p.S + k] = erun[h];
                }
                const float f = p.u_mode == CASCADE_U_NORMALISED ? (erun[h] > 0.f ? 1.0f / erun[h] : 0.f) : 1.0f;
                float *up = p.u + (((int64_t)b * p.S + k) * p.H + head) * d + sub * VEC;
#pragma unroll
                for (int i = 0; i < VEC; ++i) up[i] = acc[h][i] * f;
            }
        }
        return;
    }
    // four wavefronts per shard: merge their states through LDS
    if (lane < LPR) {
#pragma unroll
        for (int h = 0; h < REP; ++h) {
            if (lane == 0) { red_me[wave][h][0] = mrun[h]; red_me[wave][h][1] = erun[h]; }
#pragma unroll
            for (int i = 0; i < VEC; ++i) red_u[(wave * REP + h) * d + sub * VEC + i] = acc[h][i];
        }
    }
    __syncthreads();
    write_merged_waves<REP>(p, red_me, red_u, b, head0, k, d, 1.f, LN2);
}

// bf16 caches whose kv heads serve REP = 4 or 8 query heads, D = 64 or 128.  The kernel above needs ~200 vector
// instructions per 2 KB of such a cache (each query head multiplies, reduces over 16 lanes, rescales), which held it at
// 5 TB/s.  Here a wavefront takes 16 cached rows at a time: their scores are D / 32 matrix instructions (rows x query
// heads; products of bf16 are exact, sums in fp32), whose accumulators hold, per lane, the four keys 4 g .. 4 g + 3 of
// lane group g = lane / 16 and query head lane % 4 (the heads fill the 16 columns four times over).  The lane group then
// loads those four value rows whole, 16 lanes to a row, and takes the probabilities in fp32 from its quad by
// data-parallel-primitive moves, so a running (m, e, u~) per lane group needs no exchange between lanes in the loop and
// the accumulators are rescaled once per 16 rows: ~75 vector instructions per 2 KB.  32 sequences of 64 shards of 128 rows,
// 32 / 8 heads of 128 (1.07 GB, cold): 246 -> 191 us (5.7 TB/s read, 0.17 written); 64 / 8 heads, 8 x 32 shards of 512:
// 185 -> 101; 4 x 16 shards of 128: 13.5 -> 9.4; heads of 64, 16 x 64 shards of 128: 62 -> 49.
template <int REP, int D, int WPS>
__global__ __launch_bounds__(256) void decode_attn_mfma_kernel(DecodeParams p) {
    constexpr int HG = REP / 4;                            // groups of four query heads
    constexpr int CH = D / 32;                             // reduction steps of a score
    constexpr int VPL = D / 16;                            // value elements per lane
    typedef bf16_t vvec __attribute__((ext_vector_type(VPL)));
    __shared__ float red_me[WPS == 1 ? 1 : 4][REP][2];
    extern __shared__ float red_u[];                       // [4][REP][D] when WPS == 4

    const int lane = threadIdx.x & 63, c16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wsub = wave % WPS;
    const int k = blockIdx.x * (4 / WPS) + wave / WPS, b = blockIdx.z;
    if (k >= p.S) return;                                  // uniform over the wavefronts that share a shard
    const int head0 = blockIdx.y * REP;
    const int len = max(0, min(p.shard_len[b * p.S + k], p.cap));

    bf16x8 qf[HG][CH];
#pragma unroll
    for (int hg = 0; hg < HG; ++hg)
#pragma unroll
        for (int c = 0; c < CH; ++c)
            qf[hg][c] = *(const bf16x8 *)((const bf16_t *)p.q + ((int64_t)b * p.H + head0 + hg * 4 + (lane & 3)) * D + c * 32 + g * 8);
    float mrun[HG], erun[HG], acc[REP][VPL];               // the maxima are those of the unscaled products
#pragma unroll
    for (int hg = 0; hg < HG; ++hg) { mrun[hg] = -INFINITY; erun[hg] = 0.f; }
#pragma unroll
    for (int h = 0; h < REP; ++h)
#pragma unroll
        for (int i = 0; i < VPL; ++i) acc[h][i] = 0.f;

    // rows behind the last are outside the descriptors: zeros, without a memory access
    const int64_t base = (((int64_t)b * p.Hkv + blockIdx.y) * p.S + k) * p.cap * D;
    const __amdgpu_buffer_rsrc_t kc = __builtin_amdgcn_make_buffer_rsrc((void *)((const bf16_t *)p.kc + base), 0, len * (D * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t vc = __builtin_amdgcn_make_buffer_rsrc((void *)((const bf16_t *)p.vc + base), 0, len * (D * 2), 0x00020000);
    const uint32_t k_off = c16 * (D * 2) + g * 16, v_off = 4 * g * (D * 2) + c16 * (VPL * 2);
    bf16x8 kb[2][CH];
    vvec vb[2][4];
    auto load = [&](int row0, bf16x8 (&kd)[CH], vvec (&vd)[4]) {      // 16 rows
        const uint32_t o = (uint32_t)row0 * (D * 2);
#pragma unroll
        for (int c = 0; c < CH; ++c)
            kd[c] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(kc, o + k_off + c * 64, 0, 0));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if constexpr (VPL == 8) vd[r] = __builtin_bit_cast(vvec, __builtin_amdgcn_raw_buffer_load_b128(vc, o + v_off + r * (D * 2), 0, 0));
            else vd[r] = __builtin_bit_cast(vvec, __builtin_amdgcn_raw_buffer_load_b64(vc, o + v_off + r * (D * 2), 0, 0));
        }
    };
    auto step = [&](int row0, const bf16x8 (&kd)[CH], const vvec (&vd)[4]) {
        float pr[HG][4], alpha[HG];
#pragma unroll
        for (int hg = 0; hg < HG; ++hg) {
            f32x4 s = {0.f, 0.f, 0.f, 0.f}, s1 = s;        // two sums: half the roundings in a row
#pragma unroll
            for (int c = 0; c < CH; c += 2) {
                s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kd[c], qf[hg][c], s, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kd[c + 1], qf[hg][c + 1], s1, 0, 0, 0);
            }
            s += s1;
            if (row0 + 16 > len) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (row0 + 4 * g + r >= len) s[r] = -INFINITY;
            }
            const float m_new = fmaxf(fmaxf(mrun[hg], fmaxf(s[0], s[1])), fmaxf(s[2], s[3]));
            const float m_sub = m_new == -INFINITY ? 0.f : m_new;
            alpha[hg] = __builtin_amdgcn_exp2f((mrun[hg] - m_sub) * p.scale_log2);
#pragma unroll
            for (int r = 0; r < 4; ++r) pr[hg][r] = __builtin_amdgcn_exp2f((s[r] - m_sub) * p.scale_log2);
            mrun[hg] = m_new;
            erun[hg] = erun[hg] * alpha[hg] + ((pr[hg][0] + pr[hg][1]) + (pr[hg][2] + pr[hg][3]));
        }
        auto head = [&](auto h_tag) {
            constexpr int h = decltype(h_tag)::value, quad = (h & 3) * 0x55;
            const float a = dpp_row_move<quad>(alpha[h / 4]);
#pragma unroll
            for (int i = 0; i < VPL; ++i) acc[h][i] *= a;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float pb = dpp_row_move<quad>(pr[h / 4][r]);
#pragma unroll
                for (int i = 0; i < VPL; ++i) acc[h][i] = fmaf(pb, (float)vd[r][i], acc[h][i]);
            }
        };
        for_heads<REP>(head);
    };
    constexpr int STEP = 16 * WPS;
    if (wsub * 16 < len) {
        // the request ahead is not conditional (behind the end it reads nothing): with a branch around it the
        // compiler cannot count the loads in flight and waits for all of them
        load(wsub * 16, kb[0], vb[0]);
        for (int row0 = wsub * 16;; row0 += 2 * STEP) {
            load(row0 + STEP, kb[1], vb[1]);
            step(row0, kb[0], vb[0]);
            if (row0 + STEP >= len) break;
            load(row0 + 2 * STEP, kb[0], vb[0]);
            step(row0 + STEP, kb[1], vb[1]);
            if (row0 + 2 * STEP >= len) break;
        }
    }

    // The four lane groups meet: their states on a common maximum, then the sums over groups by swapping register halves,
    // after which lane group h holds head h of each group of four.
    float total[HG][VPL], m_tot[HG], e_tot[HG];
#pragma unroll
    for (int hg = 0; hg < HG; ++hg) {
        float m = fmaxf(mrun[hg], __shfl_xor(mrun[hg], 16, WAVE));
        m = fmaxf(m, __shfl_xor(m, 32, WAVE));
        const float f = __builtin_amdgcn_exp2f((mrun[hg] - (m == -INFINITY ? 0.f : m)) * p.scale_log2);
        float e = erun[hg] * f;
        e += __shfl_xor(e, 16, WAVE);
        e += __shfl_xor(e, 32, WAVE);
        m_tot[hg] = m;
        e_tot[hg] = e;
        const float f0 = dpp_row_move<0x00>(f), f1 = dpp_row_move<0x55>(f), f2 = dpp_row_move<0xAA>(f), f3 = dpp_row_move<0xFF>(f);
#pragma unroll
        for (int i = 0; i < VPL; ++i) {
            const float x = swap_add<32>(acc[hg * 4][i] * f0, acc[hg * 4 + 2][i] * f2);
            const float y = swap_add<32>(acc[hg * 4 + 1][i] * f1, acc[hg * 4 + 3][i] * f3);
            total[hg][i] = swap_add<16>(x, y);
        }
    }
    if (WPS == 1) {                                        // the wavefront owns the shard: write the partial
#pragma unroll
        for (int hg = 0; hg < HG; ++hg) {
            if (lane < 4) {
                const int64_t at = ((int64_t)b * p.H + head0 + hg * 4 + lane) * p.S + k;
                p.m[at] = m_tot[hg] * p.scale;             // in the units of a
                p.e[at] = e_tot[hg];
            }
            const float e = __shfl(e_tot[hg], g, WAVE);    // lane g: head g
            const float f = p.u_mode == CASCADE_U_NORMALISED ? (e > 0.f ? 1.0f / e : 0.f) : 1.0f;
            float *up = p.u + (((int64_t)b * p.S + k) * p.H + head0 + hg * 4 + g) * D + c16 * VPL;
#pragma unroll
            for (int i = 0; i < VPL; ++i) up[i] = total[hg][i] * f;
        }
        return;
    }
#pragma unroll
    for (int hg = 0; hg < HG; ++hg) {
        if (lane < 4) { red_me[wave][hg * 4 + lane][0] = m_tot[hg]; red_me[wave][hg * 4 + lane][1] = e_tot[hg]; }
#pragma unroll
        for (int i = 0; i < VPL; ++i) red_u[(wave * REP + hg * 4 + g) * D + c16 * VPL + i] = total[hg][i];
    }
    __syncthreads();
    write_merged_waves<REP>(p, red_me, red_u, b, head0, k, D, p.scale_log2, p.scale);
}

template <typename T, int REP>
static int32_t launch_lpr(const DecodeParams &p, int y_dim, hipStream_t s) {
    constexpr int VEC = 16 / sizeof(T);
    const int lpr = p.d / VEC;
    // Shards of at least 256 rows get four wavefronts each (measured on MI355X: 5.1 against 3.8 TB/s at 512 rows).  From 96
    // rows on so do launches that cannot fill the SIMDs with a wavefront each (1024): they last as long as the walk of one
    // shard; and larger ones where that walk is long against the merge of the four states (REP heads of d floats, fewer
    // wavefronts resident for their registers), which `walk` weighs as the measurements fall.  Caches read cold (rotated
    // through 1.2 GB), with the merge of the shards, one wavefront / four (us): 32 / 8 heads of 128, 512 wavefronts of 96,
    // 128, 255 rows 26 / 22, 31 / 23, 56 / 27; 2048: 36 / 35, 43 / 40, 82 / 68; 4096: 52 / 59, 67 / 73, 137 / 126; 8192:
    // 98 / 113, 126 / 132, 253 / 230; 64 / 8 heads, 1024 wavefronts of 96, 255 rows 37 / 37, 79 / 64; 2048: 51 / 61,
    // 114 / 117; 8192: 171 / 213, 385 / 404; fp32, 32 / 8: 2048 of 96, 255 rows 53 / 47, 136 / 113; 6144: 136 / 120,
    // 360 / 304; 64 / 8 fp32, 8192: 220 / 238, 528 / 513; 12 / 12 heads of 64, 6144 wavefronts 35 / 33, 105 / 80.
    const int64_t waves = (int64_t)p.S * y_dim * p.B, walk = (int64_t)p.cap * lpr * (int)sizeof(T) * 4 / (REP * REP);
    const bool wide = p.cap >= 256 || (p.cap >= 96 && (waves <= 1024 || (waves <= 2048 && walk >= 1024) || (waves <= 8192 && walk >= 1920)));
    const dim3 grid(wide ? p.S : (p.S + 3) / 4, y_dim, p.B);
    const size_t lds = wide ? (size_t)4 * REP * p.d * sizeof(float) : 0;
    // the merge of the four wavefront states needs 4 * REP * d floats: up to 64 KiB at 8 query heads of 512,
    // above the default dynamic limit, so the limit is raised per kernel instance (once per device)
#define DECODE_LAUNCH(L)                                                                              \
    do {                                                                                              \
        if (wide) {                                                                                   \
            static std::atomic<uint64_t> lds_ready{0};                                                \
            CASCADE_HIP_TRY(ensure_dynamic_lds((const void *)decode_attn_kernel<T, REP, L, 4>, (int)lds, lds_ready)); \
            hipLaunchKernelGGL((decode_attn_kernel<T, REP, L, 4>), grid, dim3(256), lds, s, p);       \
        } else hipLaunchKernelGGL((decode_attn_kernel<T, REP, L, 1>), grid, dim3(256), 0, s, p);      \
    } while (0)
    switch (lpr) {
        case 1: DECODE_LAUNCH(1); break;
        case 2: DECODE_LAUNCH(2); break;
        case 4: DECODE_LAUNCH(4); break;
        case 8: DECODE_LAUNCH(8); break;
        case 16: DECODE_LAUNCH(16); break;
        case 32: DECODE_LAUNCH(32); break;
        case 64: DECODE_LAUNCH(64); break;
        default: return CASCADE_EUNSUPPORTED;
    }
#undef DECODE_LAUNCH
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}

template <int REP, int D>
static int32_t launch_mfma(const DecodeParams &p, hipStream_t s) {
    // Four wavefronts per shard where each has two steps of 16 rows or more (the merge of their states costs about one;
    // twice that for 8 query heads), and in launches of less than a wavefront per SIMD.  Cold caches, 8 kv heads, one
    // wavefront / four (us): 32 heads of 128, 4096 wavefronts of 64, 96, 112, 120 rows 27.6 / 31.9, 38.5 / 41.5, 45.1 /
    // 46.8, 48.2 / 47.7, 16384 of 128 213 / 191, 1024 of 512 49.8 / 47.3, 64 of 1000 44 / 15; 64 heads of 128, 2048
    // wavefronts of 160, 192, 256 rows 34.8 / 41.1, 40.4 / 43.5, 59.0 / 53.7; heads of 64 alike.
    const bool wide = p.cap >= (REP == 4 ? 120 : 224) || (p.cap > 16 && (int64_t)p.S * p.Hkv * p.B < 1024);
    const dim3 grid(wide ? p.S : (p.S + 3) / 4, p.Hkv, p.B);
    const size_t lds = wide ? (size_t)4 * REP * D * sizeof(float) : 0;
    if (wide) hipLaunchKernelGGL((decode_attn_mfma_kernel<REP, D, 4>), grid, dim3(256), lds, s, p);
    else hipLaunchKernelGGL((decode_attn_mfma_kernel<REP, D, 1>), grid, dim3(256), 0, s, p);
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}

template <typename T>
static int32_t launch_rep(DecodeParams p, hipStream_t s) {
    const int rep = p.H / p.Hkv;
    p.rep = rep;
    if (p.H > 65535 || p.B > 65535) return CASCADE_EUNSUPPORTED;
    if (rep == 1 || rep == 2 || rep == 4 || rep == 8) {
        p.per_head = 0;
        if (std::is_same<T, bf16_t>::value && rep >= 4 && (p.d == 64 || p.d == 128) && (int64_t)p.cap * p.d * 2 <= INT32_MAX) {
            if (rep == 4) return p.d == 64 ? launch_mfma<4, 64>(p, s) : launch_mfma<4, 128>(p, s);
            return p.d == 64 ? launch_mfma<8, 64>(p, s) : launch_mfma<8, 128>(p, s);
        }
        switch (rep) {
            case 1: return launch_lpr<T, 1>(p, p.Hkv, s);
            case 2: return launch_lpr<T, 2>(p, p.Hkv, s);
            case 4: return launch_lpr<T, 4>(p, p.Hkv, s);
            default: return launch_lpr<T, 8>(p, p.Hkv, s);
        }
    }
    p.per_head = 1;                                        // other group sizes: one query head per wavefront group
    return launch_lpr<T, 1>(p, p.H, s);
}

extern "C" int32_t cascade_decode_partial_attn(const cascade_attn_desc *d, int32_t batch, int32_t n_shards,
                                               int32_t shard_capacity, const int32_t *shard_len_dev, const void *q,
                                               const void *k_cache, const void *v_cache, float *m, float *e, float *u,
                                               void *stream) {
    if (!d || !shard_len_dev || !q || !k_cache || !v_cache || !m || !e || !u) return CASCADE_EINVAL;
    if (batch <= 0 || n_shards <= 0 || shard_capacity <= 0) return CASCADE_EINVAL;
    if (d->dtype != CASCADE_F32 && d->dtype != CASCADE_BF16) return CASCADE_EUNSUPPORTED;
    if (d->n_heads <= 0 || d->n_kv_heads <= 0 || d->head_dim <= 0 || !(d->scale > 0.f)) return CASCADE_EINVAL;
    if (d->n_heads % d->n_kv_heads) return CASCADE_ESHAPE;
    if (d->u_mode != CASCADE_U_NORMALISED && d->u_mode != CASCADE_U_UNNORMALISED) return CASCADE_EINVAL;
    const int vec = d->dtype == CASCADE_BF16 ? 8 : 4;
    const int lpr = d->head_dim / vec;
    if (d->head_dim % vec || lpr > 64 || (lpr & (lpr - 1))) return CASCADE_EUNSUPPORTED;   // d = vec * 2^j, at most 64 lanes per row
    if (((uintptr_t)q | (uintptr_t)k_cache | (uintptr_t)v_cache) % 16) return CASCADE_EUNSUPPORTED;
    DecodeParams p = {};
    p.q = q; p.kc = k_cache; p.vc = v_cache; p.shard_len = shard_len_dev; p.m = m; p.e = e; p.u = u;
    p.B = batch; p.H = d->n_heads; p.Hkv = d->n_kv_heads; p.S = n_shards; p.cap = shard_capacity; p.d = d->head_dim;
    p.scale = d->scale; p.scale_log2 = d->scale * LOG2E; p.u_mode = d->u_mode;
    hipStream_t s = (hipStream_t)stream;
    return d->dtype == CASCADE_BF16 ? launch_rep<bf16_t>(p, s) : launch_rep<float>(p, s);
}
