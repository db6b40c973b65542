// HBM-bound per-token kernels: normalisation with row gather (the optional normalisation step of the
// Pre-Pass subsection), rotary embedding at original token positions
// (the rotary step of Algorithm 2).  The gather into packed order is the row map of the norm's read; the
// scatter back is the row map of the last shard GEMM's store.
#include <climits>
#include <cmath>
#include "common.h"
#include "device_utils.h"
#include "rope.h"

// By-product of the pre-pass norm: the workgroup of row r writes that row's cos | sin table (the shard GEMM
// that follows rotates q and k with it in its epilogue).
struct RopeTableOut {
    float *table;
    const int32_t *pos;
    int32_t seq_len, head_dim;
    float theta;
};
// Second by-product: a few words cleared by the first workgroup (the flags of the split-reduction shard GEMMs that
// follow in the stream; a fill of its own would cost a launch, and a memset cannot be captured in a graph).
struct ZeroWords {
    uint32_t *words;
    int32_t n;
};
__device__ __forceinline__ void clear_words(const ZeroWords &z) {
    if (z.words && blockIdx.x == 0)
        for (int i = threadIdx.x; i < z.n; i += blockDim.x) z.words[i] = 0u;
}
__device__ __forceinline__ void write_rope_row(const RopeTableOut &t, int r, int first, int threads) {
    const int half = t.head_dim >> 1;
    const float pos = (float)t.pos[r % t.seq_len];
    for (int i = first; i < half; i += threads) {
        const RopeRev c = rope_rev(t.theta, i, t.head_dim);
        float cs, sn;
        rope_cos_sin(pos, c.hi, c.lo, cs, sn);
        t.table[(int64_t)r * t.head_dim + i] = cs;
        t.table[(int64_t)r * t.head_dim + half + i] = sn;
    }
}

// ---------------------------------------------------------------------------- norm
// One 256-thread block per row; the row is staged in LDS as fp32 (D * 4 bytes).
template <typename T>
__global__ __launch_bounds__(256) void norm_kernel(const T *__restrict__ x, const T *__restrict__ gain,
                                                   const T *__restrict__ bias, T *__restrict__ y, int D, int kind,
                                                   float eps, const int32_t *xmap, const int32_t *ymap, int seq_len,
                                                   RopeTableOut rope, ZeroWords zero) {
    extern __shared__ float row[];
    __shared__ float red[4];
    const int r = blockIdx.x;
    clear_words(zero);
    if (rope.table) write_rope_row(rope, r, threadIdx.x, 256);
    const T *xr = x + map_row(xmap, seq_len, r) * (int64_t)D;
    float s = 0.f;
    for (int i = threadIdx.x; i < D; i += 256) {
        float v = Elem<T>::load(xr + i);
        row[i] = v;
        s += v;
    }
    float mu = 0.f;
    if (kind == CASCADE_NORM_LAYERNORM) mu = block_sum_256(s, red) / D;
    float q = 0.f;
    for (int i = threadIdx.x; i < D; i += 256) {
        float c = row[i] - mu;
        q += c * c;
    }
    float var = block_sum_256(q, red) / D;
    float rstd = 1.0f / sqrtf(var + eps);
    T *yr = y + map_row(ymap, seq_len, r) * (int64_t)D;
    for (int i = threadIdx.x; i < D; i += 256) {
        float v = (row[i] - mu) * rstd * Elem<T>::load(gain + i);
        if (bias) v += Elem<T>::load(bias + i);
        Elem<T>::store(yr + i, v);
    }
}

// Sum over the ROW threads (a wavefront or the workgroup of 256) that share a row; every one gets it.  A wavefront's NS sums per
// lane are added as NS wavefronts of a workgroup would add theirs.
template <int ROW, int NS>
__device__ __forceinline__ float row_sum(const float (&v)[NS], float *scratch) {
    if constexpr (ROW == WAVE) {
        float sum = wave_sum(v[0]);
#pragma unroll
        for (int c = 1; c < NS; ++c) sum += wave_sum(v[c]);
        return sum;
    } else return block_sum_256(v[0], scratch);
}

// Vector variant: the row lives in registers (CH 16-byte pieces per thread), two passes over them.
// Requires D % VEC == 0 and D <= ROW * CH * VEC, VEC = 16 bytes / sizeof(T).  ROW threads per row: the workgroup of 256, or a
// wavefront, four rows to a workgroup, where that is two pieces per lane at most (bf16 up to 1024 columns, fp32 up to
// 512): a workgroup per such row leaves half of its threads and more without work, and its two sums meet at
// barriers.  Everything that is read is requested before the first sum.  4096 rows of 768 8.1 and 6.9 -> 5.6 and 5.5 us (the first
// gathers), a layer of them 152.6 -> 149.2, 6000 rows 191 -> 185; one generated token of four sequences 126.5 -> 123.7 (gain requested early).
// The sums of a wavefront's pieces are kept apart, so that a row has the same bits as from a workgroup of its own, here and
// behind a reduction in parts (splitk_finish_kernel).
template <typename T, int CH, int ROW>
__global__ __launch_bounds__(256) void norm_vec_kernel(const T *__restrict__ x, const T *__restrict__ gain,
                                                       const T *__restrict__ bias, T *__restrict__ y, int D, int kind,
                                                       float eps, const int32_t *xmap, const int32_t *ymap, int seq_len,
                                                       RopeTableOut rope, ZeroWords zero, int rows) {
    constexpr int VEC = 16 / sizeof(T);
    typedef T vecT __attribute__((ext_vector_type(VEC)));
    __shared__ float red[4];
    const int t = threadIdx.x % ROW;
    const int r = ROW == 256 ? (int)blockIdx.x : (int)blockIdx.x * (256 / ROW) + (int)(threadIdx.x / ROW);
    clear_words(zero);
    if (r >= rows) return;                                 // (whole wavefronts, which meet no barrier)
    if (rope.table) write_rope_row(rope, r, t, ROW);       // (behind the requests, 2048 rows of 4096 take 11.7 us for 10.1)
    const T *xr = x + map_row(xmap, seq_len, r) * (int64_t)D;
    T *yr = y + map_row(ymap, seq_len, r) * (int64_t)D;
    const int nvec = D / VEC;
    vecT in[CH], g[CH], bb[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int i = min(t + ROW * c, nvec - 1);
        in[c] = *(const vecT *)(xr + i * VEC);
        g[c] = *(const vecT *)(gain + i * VEC);
        if (bias) bb[c] = *(const vecT *)(bias + i * VEC);
    }
    constexpr int NS = ROW == WAVE ? CH : 1;
    float s[NS] = {};
#pragma unroll
    for (int c = 0; c < CH; ++c)
        if (t + ROW * c < nvec)
#pragma unroll
            for (int j = 0; j < VEC; ++j) s[c % NS] += (float)in[c][j];
    float mu = 0.f;
    if (kind == CASCADE_NORM_LAYERNORM) mu = row_sum<ROW>(s, red) / D;
    // (what is rounded between products and sums is written out, here and with the bias: the compiler's choice differed from
    // one instance to another and from column to column)
    float q[NS] = {};
#pragma unroll
    for (int c = 0; c < CH; ++c)
        if (t + ROW * c < nvec)
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                const float d0 = (float)in[c][j] - mu, d1 = j + 1 < VEC ? (float)in[c][j + 1] - mu : 0.f;
                float &sum = q[c % NS];
                if (c < NS && j == 0) sum = fmaf(d0, d0, d1 * d1);
                else if (c >= NS || j > 1) sum = fmaf(d0, d0, sum);
            }
    const float rstd = 1.0f / sqrtf(row_sum<ROW>(q, red) / D + eps);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int i = t + ROW * c;
        if (i < nvec) {
            vecT o;
            if (bias) {
#pragma unroll
                for (int j = 0; j < VEC; ++j) o[j] = (T)fmaf(((float)in[c][j] - mu) * rstd, (float)g[c][j], (float)bb[c][j]);
            } else {
#pragma unroll
                for (int j = 0; j < VEC; ++j) o[j] = (T)(((float)in[c][j] - mu) * rstd * (float)g[c][j]);
            }
            *(vecT *)(yr + i * VEC) = o;
        }
    }
}

template <typename T>
static int32_t launch_norm_t(const NormArgs &a, hipStream_t s) {
    constexpr int VEC = 16 / sizeof(T);
    const bool aligned = a.D % VEC == 0 && ((uintptr_t)a.x | (uintptr_t)a.y | (uintptr_t)a.gain | (uintptr_t)a.bias) % 16 == 0;
    const int nvec = a.D / VEC;
    const RopeTableOut rope = {a.rope_table, a.rope_pos, a.rope_seq_len, a.rope_head_dim, a.rope_theta};
    const ZeroWords zero = {a.zero_words, a.n_zero_words};
#define NORM_VEC(CH, ROW)                                                                                        \
    hipLaunchKernelGGL((norm_vec_kernel<T, CH, ROW>), dim3((a.rows + 256 / ROW - 1) / (256 / ROW)), dim3(256), 0, s, (const T *)a.x, \
                       (const T *)a.gain, (const T *)a.bias, (T *)a.y, a.D, a.kind, a.eps, a.xmap.map, a.ymap.map, \
                       a.xmap.map ? a.xmap.seq_len : a.ymap.seq_len, rope, zero, a.rows)
    if (aligned && nvec <= 64) NORM_VEC(1, 64);
    else if (aligned && nvec <= 128) NORM_VEC(2, 64);
    else if (aligned && nvec <= 256) NORM_VEC(1, 256);
    else if (aligned && nvec <= 512) NORM_VEC(2, 256);
    else if (aligned && nvec <= 1024) NORM_VEC(4, 256);
    else {
        size_t lds = (size_t)a.D * sizeof(float);
        if (lds > 64 * 1024) return CASCADE_EUNSUPPORTED;
        hipLaunchKernelGGL(norm_kernel<T>, dim3(a.rows), dim3(256), lds, s, (const T *)a.x, (const T *)a.gain,
                           (const T *)a.bias, (T *)a.y, a.D, a.kind, a.eps, a.xmap.map, a.ymap.map,
                           a.xmap.map ? a.xmap.seq_len : a.ymap.seq_len, rope, zero);
    }
#undef NORM_VEC
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}

int32_t launch_norm(const NormArgs &a, hipStream_t s) {
    if (a.rows == 0) return CASCADE_OK;
    return a.dtype == CASCADE_BF16 ? launch_norm_t<bf16_t>(a, s) : launch_norm_t<float>(a, s);
}

// ---------------------------------------------------------------------------- prefill k, v -> cache slabs
// One workgroup per (kv shard, kv head, sequence); 16-byte pieces, a row of d elements per d*sizeof(T)/16 lanes.
template <typename T>
__global__ __launch_bounds__(256) void kv_to_cache_kernel(KvCacheArgs a) {
    constexpr int VEC = 16 / sizeof(T);
    const int k = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
    const int r0 = a.offsets[k], n = a.offsets[k + 1] - r0;
    if (g == 0 && threadIdx.x == 0) a.shard_len[b * a.n_shards + k] = n;
    const int cpr = a.d / VEC;                              // pieces per row
    const T *act = (const T *)a.act + (int64_t)b * a.N * a.ld;
    T *kc = (T *)a.k_cache + (((int64_t)b * a.Hkv + g) * a.n_shards + k) * (int64_t)a.cap * a.d;
    T *vc = (T *)a.v_cache + (((int64_t)b * a.Hkv + g) * a.n_shards + k) * (int64_t)a.cap * a.d;
    typedef T vec_t __attribute__((ext_vector_type(VEC)));
    for (int id = threadIdx.x; id < n * cpr; id += 256) {
        const int i = id / cpr, c = id - i * cpr;
        const int row = a.row_of ? a.row_of[r0 + i] : r0 + i;
        const T *src = act + (int64_t)row * a.ld + g * a.d + c * VEC;
        *(vec_t *)(kc + (int64_t)i * a.d + c * VEC) = *(const vec_t *)(src + a.k_col0);
        *(vec_t *)(vc + (int64_t)i * a.d + c * VEC) = *(const vec_t *)(src + a.v_col0);
    }
}

int32_t launch_kv_to_cache(const KvCacheArgs &a, hipStream_t s) {
    const int vec = a.dtype == CASCADE_BF16 ? 8 : 4;
    if (a.d % vec || a.ld % vec || a.k_col0 % vec || a.v_col0 % vec ||
        ((uintptr_t)a.act | (uintptr_t)a.k_cache | (uintptr_t)a.v_cache) % 16)
        return CASCADE_EUNSUPPORTED;
    if (a.n_shards > 65535 * 32 || a.Hkv > 65535 || a.B > 65535) return CASCADE_EUNSUPPORTED;
    dim3 grid(a.n_shards, a.Hkv, a.B);
    if (a.dtype == CASCADE_BF16) hipLaunchKernelGGL(kv_to_cache_kernel<bf16_t>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(kv_to_cache_kernel<float>, grid, dim3(256), 0, s, a);
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}

// ---------------------------------------------------------------------------- end of a split reduction
// Row r of Y = sum of the fp32 planes [parts][rows][D] + bias + residual, rounded once; with a norm behind it, also
// that norm of the rounded row (the norm launch that would read it back).  One 256-thread block per row, CH 8-column
// pieces per thread, the planes added in ascending order.  Without a norm a row of more than 2048 columns is cut into a workgroup
// per 2048 of them (more workgroups than CUs, of less each: 8B layer of 333 rows 224.5 -> 222.7 us).  A wavefront per row of 768,
// as in norm_vec_kernel, was slower (3 x 389 rows in 2 and 4 parts 5.1 and 6.1 -> 6.3 and 6.9 us).  Bound by reading the planes (they come from the last-level
// cache: the launch in front wrote them).
struct FinishParams {
    const float *planes;
    int32_t parts, rows, D;
    const bf16_t *bias, *residual;
    bf16_t *y;
    const int32_t *ymap, *rmap;
    int32_t seq_len;
    int64_t ldy, ldres;
    const bf16_t *gain, *nbias;                            // gain == nullptr: no norm
    bf16_t *ny;
    const int32_t *nymap;
    int32_t kind;
    float eps;
    ZeroWords zero;
};

// PARTS: number of planes (0: any, four at a time): with it known all loads of a piece go out together.  Unrolled are the
// counts that outputs of 768 to 8192 columns come to; the others take the loop.
template <int CH, int PARTS>
__global__ __launch_bounds__(256) void splitk_finish_kernel(FinishParams p) {
    __shared__ float red[4];
    const int t = threadIdx.x + 256 * blockIdx.y, r = blockIdx.x, nvec = p.D >> 3;
    clear_words(p.zero);
    const size_t plane = (size_t)p.rows * p.D;
    const float *row = p.planes + (size_t)r * p.D;
    constexpr int NP = PARTS ? PARTS : 1;
    f32x4 a[CH][NP], b[CH][NP];
    if constexpr (PARTS > 0)
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int i = min(t + 256 * c, nvec - 1);
#pragma unroll
            for (int k = 0; k < PARTS; ++k) {
                a[c][k] = __builtin_nontemporal_load((const f32x4 *)(row + k * plane + 8 * i));
                b[c][k] = __builtin_nontemporal_load((const f32x4 *)(row + k * plane + 8 * i + 4));
            }
        }
    const bf16_t *res = p.residual ? p.residual + map_row(p.rmap, p.seq_len, r) * p.ldres : nullptr;
    bf16_t *y = p.y + map_row(p.ymap, p.seq_len, r) * p.ldy;
    float v[CH][8];
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int i = t + 256 * c;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[c][j] = 0.f;
        if (i >= nvec) continue;
        const bf16x4 z4 = {0, 0, 0, 0};
        bf16x4 r0 = z4, r1 = z4, b0 = z4, b1 = z4;
        if (res) { r0 = *(const bf16x4 *)(res + 8 * i); r1 = *(const bf16x4 *)(res + 8 * i + 4); }
        if (p.bias) { b0 = *(const bf16x4 *)(p.bias + 8 * i); b1 = *(const bf16x4 *)(p.bias + 8 * i + 4); }
        if constexpr (PARTS > 0) {
#pragma unroll
            for (int k = 0; k < PARTS; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) { v[c][j] += a[c][k][j]; v[c][4 + j] += b[c][k][j]; }
        } else {
#pragma unroll 4
            for (int k = 0; k < p.parts; ++k) {
                const f32x4 x0 = *(const f32x4 *)(row + k * plane + 8 * i), x1 = *(const f32x4 *)(row + k * plane + 8 * i + 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) { v[c][j] += x0[j]; v[c][4 + j] += x1[j]; }
            }
        }
        bf16x4 o0, o1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            o0[j] = (bf16_t)(v[c][j] + (float)b0[j] + (float)r0[j]);
            o1[j] = (bf16_t)(v[c][4 + j] + (float)b1[j] + (float)r1[j]);
            v[c][j] = (float)o0[j];                        // the norm is that of the stored row
            v[c][4 + j] = (float)o1[j];
            s += v[c][j] + v[c][4 + j];
        }
        *(bf16x4 *)(y + 8 * i) = o0;
        *(bf16x4 *)(y + 8 * i + 4) = o1;
    }
    if (!p.gain) return;
    float mu = 0.f;
    if (p.kind == CASCADE_NORM_LAYERNORM) mu = block_sum_256(s, red) / p.D;
    float q = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c)
        if (t + 256 * c < nvec)
#pragma unroll
            for (int j = 0; j < 8; ++j) { const float d0 = v[c][j] - mu; q += d0 * d0; }
    const float rstd = 1.0f / sqrtf(block_sum_256(q, red) / p.D + p.eps);
    bf16_t *ny = p.ny + map_row(p.nymap, p.seq_len, r) * (int64_t)p.D;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int i = t + 256 * c;
        if (i >= nvec) continue;
#pragma unroll
        for (int j = 0; j < 8; j += 4) {
            const bf16x4 g = *(const bf16x4 *)(p.gain + 8 * i + j);
            bf16x4 b = {0, 0, 0, 0}, o;
            if (p.nbias) b = *(const bf16x4 *)(p.nbias + 8 * i + j);
#pragma unroll
            for (int x = 0; x < 4; ++x) o[x] = (bf16_t)((v[c][j + x] - mu) * rstd * (float)g[x] + (float)b[x]);
            *(bf16x4 *)(ny + 8 * i + j) = o;
        }
    }
}

int32_t launch_splitk_finish(const GemmArgs &a, int parts, const NormArgs *norm, hipStream_t s) {
    FinishParams p = {};
    p.planes = a.planes; p.parts = parts; p.rows = a.M; p.D = a.N;
    p.bias = (a.epilogue & CASCADE_EPI_BIAS) ? (const bf16_t *)a.bias[0] : nullptr;
    p.residual = (a.epilogue & CASCADE_EPI_RESIDUAL) ? (const bf16_t *)a.residual : nullptr;
    p.y = (bf16_t *)a.Y; p.ymap = a.ymap.map; p.rmap = a.rmap.map;
    p.seq_len = a.ymap.map ? a.ymap.seq_len : a.rmap.map ? a.rmap.seq_len : 1;
    p.ldy = a.ldy; p.ldres = a.ldres;
    if (norm) {
        p.gain = (const bf16_t *)norm->gain; p.nbias = (const bf16_t *)norm->bias; p.ny = (bf16_t *)norm->y;
        p.nymap = norm->ymap.map; p.kind = norm->kind; p.eps = norm->eps;
        if (p.nymap) p.seq_len = norm->ymap.seq_len;
        p.zero = {norm->zero_words, norm->n_zero_words};
    }
    const int nvec = a.N / 8;
    const int pieces = norm ? 1 : (nvec + 255) / 256;      // workgroups per row
#define FINISH(CH, PARTS) hipLaunchKernelGGL((splitk_finish_kernel<CH, PARTS>), dim3(a.M, pieces), dim3(256), 0, s, p)
#define FINISH_PARTS(CH)                                                                                   \
    switch (parts) {                                                                                       \
        case 2: FINISH(CH, 2); break;                                                                      \
        case 3: FINISH(CH, 3); break;                                                                      \
        case 4: FINISH(CH, 4); break;                                                                      \
        case 5: FINISH(CH, 5); break;                                                                      \
        case 6: FINISH(CH, (CH > 2 ? 0 : 6)); break;                                                       \
        case 8: FINISH(CH, (CH > 2 ? 0 : 8)); break;                                                       \
        default: FINISH(CH, 0);                                                                            \
    }
    if (nvec <= 256 || pieces > 1) { FINISH_PARTS(1) }
    else if (nvec <= 512) { FINISH_PARTS(2) }
    else { FINISH_PARTS(4) }
#undef FINISH_PARTS
#undef FINISH
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}

// End of a split projection into heads: Y = sum of the planes + bias, the first rope_cols columns rotated, rounded once.  A
// thread owns 8 columns and the 8 half a head further on (8 rotation pairs; 16 neighbouring columns where nothing is rotated).
// Bound by one round trip to the planes, which the launch in front left in the last-level cache: all loads go out together
// (128 rows of 6144 columns in 5 parts: 5 us).
struct HeadsParams {
    const float *planes, *table;                           // table: cos | sin of every row, [rows][2 half]; nullptr: none
    const bf16_t *bias[3];
    int32_t seg_end[3];
    bf16_t *y;
    int64_t ldy;
    int32_t parts, rows, N, half, rope_cols, total;
};

template <int PARTS>
__global__ __launch_bounds__(256) void splitk_heads_kernel(HeadsParams p) {
    const int id = blockIdx.x * 256 + threadIdx.x;
    if (id >= p.total) return;
    const int upr = p.N >> 4, r = id / upr, u = id - r * upr;
    const int per = p.half >> 3, head = u / per, i0 = (u - head * per) * 8, c = head * 2 * p.half + i0;
    const size_t plane = (size_t)p.rows * p.N;
    const float *row = p.planes + (size_t)r * p.N + c;
    constexpr int NP = PARTS ? PARTS : 1;
    f32x4 a[4] = {}, x[NP][4];
    auto load = [&](f32x4 (&d)[4], int k) {
        const float *s = row + k * plane;
        d[0] = __builtin_nontemporal_load((const f32x4 *)s);
        d[1] = __builtin_nontemporal_load((const f32x4 *)(s + 4));
        d[2] = __builtin_nontemporal_load((const f32x4 *)(s + p.half));
        d[3] = __builtin_nontemporal_load((const f32x4 *)(s + p.half + 4));
    };
    if constexpr (PARTS > 0) {
#pragma unroll
        for (int k = 0; k < PARTS; ++k) load(x[k], k);
    }
    const bool rot = p.table && c < p.rope_cols;
    f32x4 t[4] = {};
    if (rot) {
        const float *tr = p.table + (size_t)r * 2 * p.half + i0;
        t[0] = *(const f32x4 *)tr; t[1] = *(const f32x4 *)(tr + 4);
        t[2] = *(const f32x4 *)(tr + p.half); t[3] = *(const f32x4 *)(tr + p.half + 4);
    }
    if constexpr (PARTS > 0) {
#pragma unroll
        for (int k = 0; k < PARTS; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) a[j] += x[k][j];
    } else {
#pragma unroll 4
        for (int k = 0; k < p.parts; ++k) {
            load(x[0], k);
#pragma unroll
            for (int j = 0; j < 4; ++j) a[j] += x[0][j];
        }
    }
    const int seg = c >= p.seg_end[1] ? 2 : c >= p.seg_end[0] ? 1 : 0;
    if (p.bias[seg]) {
        const bf16_t *b = p.bias[seg] + c - (seg ? p.seg_end[seg - 1] : 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bf16x4 v = *(const bf16x4 *)(b + (j & 1) * 4 + (j >> 1) * p.half);
            a[j] += f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
        }
    }
    if (rot) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const f32x4 lo = a[j] * t[j] - a[j + 2] * t[j + 2], hi = a[j + 2] * t[j] + a[j] * t[j + 2];
            a[j] = lo; a[j + 2] = hi;
        }
    }
    bf16_t *y = p.y + (int64_t)r * p.ldy + c;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        bf16x8 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) { o[i] = (bf16_t)a[2 * j][i]; o[4 + i] = (bf16_t)a[2 * j + 1][i]; }
        *(bf16x8 *)(y + j * p.half) = o;
    }
}

int32_t launch_splitk_heads(const GemmArgs &a, int parts, hipStream_t s) {
    HeadsParams p = {};
    p.planes = a.planes; p.table = a.rope_table; p.y = (bf16_t *)a.Y; p.ldy = a.ldy;
    for (int i = 0; i < 3; ++i) {
        p.bias[i] = (a.epilogue & CASCADE_EPI_BIAS) ? (const bf16_t *)a.bias[i] : nullptr;
        p.seg_end[i] = a.seg_end[i];
    }
    p.parts = parts; p.rows = a.M; p.N = a.N;
    p.half = a.rope_table ? a.rope_head_dim / 2 : 8;
    p.rope_cols = a.rope_table ? a.rope_cols : 0;
    const int64_t total = (int64_t)a.M * (a.N / 16);
    if (total > INT32_MAX - 256) return CASCADE_EUNSUPPORTED;
    p.total = (int32_t)total;
    const dim3 grid((unsigned)((total + 255) / 256));
    switch (parts) {
        case 2: hipLaunchKernelGGL(splitk_heads_kernel<2>, grid, dim3(256), 0, s, p); break;
        case 3: hipLaunchKernelGGL(splitk_heads_kernel<3>, grid, dim3(256), 0, s, p); break;
        case 4: hipLaunchKernelGGL(splitk_heads_kernel<4>, grid, dim3(256), 0, s, p); break;
        case 5: hipLaunchKernelGGL(splitk_heads_kernel<5>, grid, dim3(256), 0, s, p); break;
        case 6: hipLaunchKernelGGL(splitk_heads_kernel<6>, grid, dim3(256), 0, s, p); break;
        case 8: hipLaunchKernelGGL(splitk_heads_kernel<8>, grid, dim3(256), 0, s, p); break;
        default: hipLaunchKernelGGL(splitk_heads_kernel<0>, grid, dim3(256), 0, s, p);
    }
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}

// ---------------------------------------------------------------------------- greedy token
// Lowest index of the largest logit of a row (the CompNode holding the last token turns its logits
// into the next token).  One 1024-thread block per row; a thread walks ascending indices and keeps
// the first maximum it meets, the reductions prefer the lower index among equal values.  NaNs never
// win a comparison; a row of NaNs gives 0.
template <typename T>
__global__ __launch_bounds__(1024) void argmax_rows_kernel(const T *__restrict__ x, int64_t ld, int vocab,
                                                           int32_t *__restrict__ out) {
    __shared__ float sv[16];
    __shared__ int si[16];
    const T *row = x + (int64_t)blockIdx.x * ld;
    float best = -INFINITY;
    int idx = INT32_MAX;
    constexpr int VEC = 16 / sizeof(T);
    if (vocab % VEC == 0 && (((uintptr_t)x | (uintptr_t)(ld * sizeof(T))) % 16) == 0) {
        typedef T vec_t __attribute__((ext_vector_type(VEC)));     // 16-byte pieces, several in flight per thread
        const int nvec = vocab / VEC;
#pragma unroll 4
        for (int c = threadIdx.x; c < nvec; c += 1024) {
            const vec_t pv = *(const vec_t *)(row + (int64_t)c * VEC);
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                const float v = (float)pv[k];
                if (v > best) { best = v; idx = c * VEC + k; }      // ascending indices: the first maximum stays
            }
        }
    } else {
        for (int i = threadIdx.x; i < vocab; i += 1024) {
            const float v = Elem<T>::load(row + i);
            if (v > best) { best = v; idx = i; }
        }
    }
    auto take = [&](float ov, int oi) {
        if (ov > best || (ov == best && oi < idx)) { best = ov; idx = oi; }
    };
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) take(__shfl_xor(best, o, WAVE), __shfl_xor(idx, o, WAVE));
    if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = best; si[threadIdx.x >> 6] = idx; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) take(sv[w], si[w]);
        out[blockIdx.x] = idx == INT32_MAX ? 0 : idx;
    }
}

int32_t launch_argmax_rows(int32_t dtype, const void *x, int64_t ld, int32_t rows, int32_t vocab, int32_t *token_out,
                           hipStream_t s) {
    if (rows == 0) return CASCADE_OK;
    if (dtype == CASCADE_BF16)
        hipLaunchKernelGGL(argmax_rows_kernel<bf16_t>, dim3(rows), dim3(1024), 0, s, (const bf16_t *)x, ld, vocab, token_out);
    else
        hipLaunchKernelGGL(argmax_rows_kernel<float>, dim3(rows), dim3(1024), 0, s, (const float *)x, ld, vocab, token_out);
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}

// ---------------------------------------------------------------------------- rotary embedding
// Half-split pairing (i, i + d/2), angle = position * theta^(-2i/d); position = the token's own
// position (pos_packed[r mod N]), never the shard-local row number.  One thread per pair.
template <typename T, typename ANG>
__global__ __launch_bounds__(256) void rope_kernel(T *__restrict__ x, int64_t total_pairs, int n_rope_heads,
                                                   int head_dim, int64_t ld, float theta,
                                                   const int32_t *__restrict__ pos_packed, int seq_len) {
    const int half = head_dim >> 1;
    const int64_t pairs_per_row = (int64_t)n_rope_heads * half;
    for (int64_t id = blockIdx.x * 256ll + threadIdx.x; id < total_pairs; id += (int64_t)gridDim.x * 256) {
        int64_t r = id / pairs_per_row;
        int rem = (int)(id - r * pairs_per_row);
        int h = rem / half, i = rem - h * half;
        int pos = pos_packed[(int)(r % seq_len)];
        ANG inv_freq = (ANG)exp2((ANG)(-2.0 * i / head_dim) * (ANG)log2((ANG)theta));
        ANG ang = (ANG)pos * inv_freq;
        ANG sn = sin(ang), cs = cos(ang);
        T *p = x + r * ld + (int64_t)h * head_dim + i;
        ANG a = (ANG)Elem<T>::load(p), b = (ANG)Elem<T>::load(p + half);
        Elem<T>::store(p, (float)(a * cs - b * sn));
        Elem<T>::store(p + half, (float)(b * cs + a * sn));
    }
}

// Vector variant for bf16: one thread rotates 8 consecutive pairs (two 16-byte pieces half a head apart).
// rev[i] = theta^(-2i/d) / (2 pi) comes from the host in double precision, split into two floats.
#define ROPE_MAX_HALF 128
struct RopeFreq {
    float hi[ROPE_MAX_HALF], lo[ROPE_MAX_HALF];
};

__global__ __launch_bounds__(256) void rope_vec_kernel(bf16_t *__restrict__ x, int64_t total_units, int n_rope_heads,
                                                       int head_dim, int64_t ld, RopeFreq freq,
                                                       const int32_t *__restrict__ pos_packed, int seq_len) {
    const int half = head_dim >> 1;
    const int upr = n_rope_heads * (half / 8);                    // units per row
    for (int64_t id = blockIdx.x * 256ll + threadIdx.x; id < total_units; id += (int64_t)gridDim.x * 256) {
        const int64_t r = id / upr;
        const int rem = (int)(id - r * upr);
        const int h = rem / (half / 8), i0 = (rem % (half / 8)) * 8;
        const float pos = (float)pos_packed[(int)(r % seq_len)];  // exact: positions are below 2^24
        bf16_t *p = x + r * ld + (int64_t)h * head_dim + i0;
        const bf16x8 a = *(const bf16x8 *)p, b = *(const bf16x8 *)(p + half);
        bf16x8 oa, ob;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float cs, sn;
            rope_cos_sin(pos, freq.hi[i0 + j], freq.lo[i0 + j], cs, sn);
            const float fa = (float)a[j], fb = (float)b[j];
            oa[j] = (bf16_t)(fa * cs - fb * sn);
            ob[j] = (bf16_t)(fb * cs + fa * sn);
        }
        *(bf16x8 *)p = oa;
        *(bf16x8 *)(p + half) = ob;
    }
}

int32_t launch_rope(const RopeArgs &a, hipStream_t s) {
    int64_t total = (int64_t)a.rows * a.n_rope_heads * (a.head_dim / 2);
    if (total == 0) return CASCADE_OK;
    if (a.dtype == CASCADE_BF16 && (a.head_dim / 2) % 8 == 0 && a.head_dim / 2 <= ROPE_MAX_HALF && a.ld % 8 == 0 &&
        (uintptr_t)a.x % 16 == 0 && a.max_pos < (1 << 24)) {
        const int64_t units = total / 8;
        const int grid = (int)std::min<int64_t>((units + 255) / 256, 1 << 20);
        RopeFreq freq;
        for (int i = 0; i < a.head_dim / 2; ++i) {
            const double rev = pow((double)a.theta, -2.0 * i / a.head_dim) / 6.283185307179586476925;
            freq.hi[i] = (float)rev;
            freq.lo[i] = (float)(rev - (double)freq.hi[i]);
        }
        hipLaunchKernelGGL(rope_vec_kernel, dim3(grid), dim3(256), 0, s, (bf16_t *)a.x, units, a.n_rope_heads,
                           a.head_dim, a.ld, freq, a.pos_packed, a.seq_len);
        CASCADE_HIP_TRY(hipGetLastError());
        return CASCADE_OK;
    }
    int grid = (int)std::min<int64_t>((total + 255) / 256, 65536);
    if (a.dtype == CASCADE_BF16)
        hipLaunchKernelGGL((rope_kernel<bf16_t, float>), dim3(grid), dim3(256), 0, s, (bf16_t *)a.x, total,
                           a.n_rope_heads, a.head_dim, a.ld, a.theta, a.pos_packed, a.seq_len);
    else
        hipLaunchKernelGGL((rope_kernel<float, double>), dim3(grid), dim3(256), 0, s, (float *)a.x, total,
                           a.n_rope_heads, a.head_dim, a.ld, a.theta, a.pos_packed, a.seq_len);
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}
