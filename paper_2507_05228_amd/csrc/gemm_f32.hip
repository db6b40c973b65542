// fp32 shard GEMM: Y[rows] = epilogue(X[rows] W^T).  fp32 arithmetic throughout (no reduced-precision matrix path) so
// the result stays within 1e-5 of a float64 reference.  Two kernels: fp32 MFMA on small tiles for aligned operands,
// plain FMA for any K and alignment.
#include "common.h"
#include "device_utils.h"
#include "epilogue.h"

#define F32_BM 64
#define F32_BN 64
#define F32_BK 16

template <bool SWIGLU>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float *__restrict__ X, WeightSegs segs,
                                                       const float *__restrict__ Wup,
                                                       const float *__restrict__ residual, float *__restrict__ Y,
                                                       int M, int N, int K, int64_t ldx, int64_t ldy, int64_t ldres,
                                                       const int32_t *xmap, const int32_t *ymap,
                                                       const int32_t *rmap, int seq_len, int flags) {
    __shared__ float As[F32_BK][F32_BM + 1];
    __shared__ float Bs[F32_BK][F32_BN + 1];
    __shared__ float Us[SWIGLU ? F32_BK : 1][F32_BN + 1];
    const int t = threadIdx.x, tx = t & 15, ty = t >> 4;
    const int m0 = blockIdx.y * F32_BM, n0 = blockIdx.x * F32_BN;

    // each thread stages 4 elements of A and of B per k-tile: element id = t + 256 i -> (row, kk)
    const float *arow[4];
    const float *brow[4];
    const float *urow[4];
    int lrow[4], lk[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int id = t + 256 * i;
        lrow[i] = id >> 4;
        lk[i] = id & 15;
        int gm = m0 + lrow[i], gn = n0 + lrow[i];
        arow[i] = gm < M ? X + map_row(xmap, seq_len, gm) * ldx : nullptr;
        brow[i] = gn < N ? weight_row<float>(segs, gn, K) : nullptr;
        urow[i] = (SWIGLU && gn < N) ? Wup + (int64_t)gn * K : nullptr;
    }
    float acc[4][4] = {};
    float acc2[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += F32_BK) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int k = k0 + lk[i];
            As[lk[i]][lrow[i]] = (arow[i] && k < K) ? arow[i][k] : 0.f;
            Bs[lk[i]][lrow[i]] = (brow[i] && k < K) ? brow[i][k] : 0.f;
            if (SWIGLU) Us[lk[i]][lrow[i]] = (urow[i] && k < K) ? urow[i][k] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < F32_BK; ++kk) {
            float a[4], b[4], u[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[i] = As[kk][ty * 4 + i];
                b[i] = Bs[kk][tx * 4 + i];
                if (SWIGLU) u[i] = Us[kk][tx * 4 + i];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
                    if (SWIGLU) acc2[i][j] = fmaf(a[i], u[j], acc2[i][j]);
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int gm = m0 + ty * 4 + i;
        if (gm >= M) continue;
        int64_t yr = map_row(ymap, seq_len, gm);
        int64_t rr = (flags & CASCADE_EPI_RESIDUAL) ? map_row(rmap, seq_len, gm) : 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int gn = n0 + tx * 4 + j;
            if (gn >= N) continue;
            float v = acc[i][j];
            if (flags & CASCADE_EPI_BIAS) v += bias_at<float>(segs, gn);
            if (SWIGLU) v = silu_f(v) * acc2[i][j];
            else v = apply_act(v, flags);
            if (flags & CASCADE_EPI_RESIDUAL) v += residual[rr * ldres + gn];
            Y[yr * ldy + gn] = v;
        }
    }
}

// Main fp32 kernel (K % 4 == 0, 16-byte aligned rows): fp32 MFMA 16x16x4, whose products and sums are fp32.  The fp32
// configuration is latency-bound (a few dozen tiles, K of 64 to 256), so a workgroup takes one small tile, its 4
// wavefronts split K and load their operands straight into registers, all of a step's loads in flight at once, and the
// partial sums meet in LDS: no k-loop with two barriers and a memory round trip per 16 of K (128 x 64 x 256: 40 us with
// the kernel above, 5.4 us here).  A lane loads 4 consecutive k of a row; MFMA j of a step takes element j of every
// lane, the same k on both sides.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ f32x4 load_f32x4(rsrc_t r, uint32_t off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
#define OOB_OFF 0x80000000u

template <int TM, int TN, bool SWIGLU>
__global__ __launch_bounds__(256) void gemm_f32_mfma_kernel(const float *__restrict__ X, WeightSegs segs,
                                                            const float *__restrict__ Wup, const float *__restrict__ residual,
                                                            float *__restrict__ Y, int M, int N, int K, int64_t ldx, int64_t ldy,
                                                            int64_t ldres, const int32_t *xmap, const int32_t *ymap,
                                                            const int32_t *rmap, int seq_len, int flags, uint32_t x_bytes) {
    constexpr int NW = 4, TW = SWIGLU ? 2 * TN : TN, DEPTH = TM + TW <= 4 ? 2 : 1;   // steps of 16 k in flight
    __shared__ __attribute__((aligned(16))) float part[NW][TW][256];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = blockIdx.y * 16 * TM, n0 = blockIdx.x * 16 * TN;
    const rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(X), 0, x_bytes, 0x00020000);
    uint32_t x_off[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + 16 * i + l16;
        x_off[i] = m < M ? (uint32_t)(map_row(xmap, seq_len, m) * ldx * 4) + g * 16 : OOB_OFF;
    }
    const float *w[TW];                                   // this lane's weight rows (null: past the last column)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = n0 + 16 * j + l16;
        w[j] = n < N ? weight_row<float>(segs, n, K) + 4 * g : nullptr;
        if (SWIGLU) w[j + TN] = n < N ? Wup + (int64_t)n * K + 4 * g : nullptr;
    }
    f32x4 acc[TM][TW];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 xr[DEPTH][TM], wr[DEPTH][TW];
    auto request = [&](int slot, int k) {                 // k of the step; lanes past K read zeros
        const bool in = k + 4 * g < K;
#pragma unroll
        for (int i = 0; i < TM; ++i) xr[slot][i] = load_f32x4(rx, in && x_off[i] != OOB_OFF ? x_off[i] + 4u * k : OOB_OFF);
#pragma unroll
        for (int j = 0; j < TW; ++j) {
            wr[slot][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (in && w[j]) wr[slot][j] = *(const f32x4 *)(w[j] + k);
        }
    };
    constexpr int STEP = 16 * NW;
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) request(d, 16 * wave + STEP * d);
    for (int k = 16 * wave; k < K; k += STEP * DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TW; ++j)          // transposed: row 16i + lane%16, columns 4(lane/16) + r
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr[d][j][e], xr[d][i][e], acc[i][j], 0, 0, 0);
            request(d, k + STEP * (DEPTH + d));
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if (i) __syncthreads();                           // the sums of the row block before have been read
#pragma unroll
        for (int j = 0; j < TW; ++j) *(f32x4 *)&part[wave][j][l16 * 16 + g * 4] = acc[i][j];
        __syncthreads();
        const int m = m0 + 16 * i + (tid >> 4);
        if (m >= M) continue;
        const int64_t yr = map_row(ymap, seq_len, m);
        const int64_t rr = (flags & CASCADE_EPI_RESIDUAL) ? map_row(rmap, seq_len, m) : 0;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + 16 * j + (tid & 15);
            if (n >= N) continue;
            float v = (part[0][j][tid] + part[1][j][tid]) + (part[2][j][tid] + part[3][j][tid]);
            if (flags & CASCADE_EPI_BIAS) v += bias_at<float>(segs, n);
            if constexpr (SWIGLU) {
                const float up = (part[0][j + TN][tid] + part[1][j + TN][tid]) + (part[2][j + TN][tid] + part[3][j + TN][tid]);
                v = silu_f(v) * up;
            } else v = apply_act(v, flags);
            if (flags & CASCADE_EPI_RESIDUAL) v += residual[rr * ldres + n];
            Y[yr * ldy + n] = v;
        }
    }
}

template <int TM, int TN>
static int32_t launch_f32_mfma(const GemmArgs &a, const WeightSegs &segs, int seq, hipStream_t s) {
    const dim3 grid((a.N + 16 * TN - 1) / (16 * TN), (a.M + 16 * TM - 1) / (16 * TM));
    if (grid.y > 65535) return CASCADE_EUNSUPPORTED;
    auto kern = (a.epilogue & CASCADE_EPI_SWIGLU) ? gemm_f32_mfma_kernel<TM, TN, true> : gemm_f32_mfma_kernel<TM, TN, false>;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, (const float *)a.X, segs, (const float *)a.W_up, (const float *)a.residual,
                       (float *)a.Y, a.M, a.N, a.K, a.ldx, a.ldy, a.ldres, a.xmap.map, a.ymap.map, a.rmap.map, seq, a.epilogue,
                       (uint32_t)((int64_t)a.M * a.ldx * 4));
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}

int32_t launch_gemm_f32(const GemmArgs &a, hipStream_t s) {
    if (a.M == 0 || a.N == 0) return CASCADE_OK;
    WeightSegs segs;
    for (int i = 0; i < 3; ++i) { segs.w[i] = a.W[i]; segs.bias[i] = a.bias[i]; segs.end[i] = a.seg_end[i]; }
    dim3 grid((a.N + F32_BN - 1) / F32_BN, (a.M + F32_BM - 1) / F32_BM);
    if (grid.y > 65535) return CASCADE_EUNSUPPORTED;
    const int seq = a.xmap.map ? a.xmap.seq_len : a.ymap.map ? a.ymap.seq_len : a.rmap.seq_len;
    const uintptr_t align = (uintptr_t)a.X | (uintptr_t)a.W[0] | (uintptr_t)a.W[1] | (uintptr_t)a.W[2] | (uintptr_t)a.W_up;
    if (a.K % 4 == 0 && a.ldx % 4 == 0 && align % 16 == 0 && (int64_t)a.M * a.ldx * 4 < (int64_t)OOB_OFF &&
        (a.M + 15) / 16 <= 65535) {
        // 16 x 16 tiles while they number at most two per CU (latency counts), 32 x 32 beyond (operand bytes do)
        const int64_t tiles = (int64_t)((a.M + 15) / 16) * ((a.N + 15) / 16);
        return tiles <= 512 ? launch_f32_mfma<1, 1>(a, segs, seq, s) : launch_f32_mfma<2, 2>(a, segs, seq, s);
    }
    if (a.epilogue & CASCADE_EPI_SWIGLU)
        hipLaunchKernelGGL(gemm_f32_kernel<true>, grid, dim3(256), 0, s, (const float *)a.X, segs,
                           (const float *)a.W_up, (const float *)a.residual, (float *)a.Y, a.M, a.N, a.K, a.ldx,
                           a.ldy, a.ldres, a.xmap.map, a.ymap.map, a.rmap.map, seq, a.epilogue);
    else
        hipLaunchKernelGGL(gemm_f32_kernel<false>, grid, dim3(256), 0, s, (const float *)a.X, segs,
                           (const float *)a.W_up, (const float *)a.residual, (float *)a.Y, a.M, a.N, a.K, a.ldx,
                           a.ldy, a.ldres, a.xmap.map, a.ymap.map, a.rmap.map, seq, a.epilogue);
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}
