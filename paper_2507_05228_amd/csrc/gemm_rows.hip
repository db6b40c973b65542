// bf16 shard GEMM for few rows (a generated token's step, short prompts):
// Y[rows] = epilogue(X[rows] W^T) with at most 64 rows, fp32 accumulation, K % 64 == 0.
//
// What bounds it: every weight is used for a handful of rows, so the launch is as long as streaming W from HBM.
// Tiles of 128 or 256 rows give N / 128 workgroups that each walk all of K (16 to 128 workgroups for the layers
// of an 8B model: 1 to 1.4 TB/s; 4096 x 14336 for 4 rows 118 us, here 24).  Here a workgroup owns 16 or 32 output columns
// and its 8 wavefronts split the reduction: wavefront w takes the 128-byte pieces w, w + 8, ... of the weight rows, straight from memory into
// MFMA operand registers (each weight is read by exactly one wavefront, LDS would only add a stop), a ring of
// pieces ahead of their use.  X is re-read by every workgroup and comes from L2.  The 8 partial accumulators meet in
// LDS once at the end, are summed in a fixed order in fp32 and take the same epilogue as the other shard GEMMs.
#include <cmath>
#include <type_traits>
#include "common.h"
#include "device_utils.h"
#include "epilogue.h"
#include "rope.h"

#define OOB_OFF 0x80000000u

constexpr int ROWS_NW = 8;                                // wavefronts of a workgroup (parts of the reduction)

struct GemmRowsParams {
    const bf16_t *X;
    const bf16_t *W[3];
    const bf16_t *bias[3];
    int32_t seg_rows[3], seg_col0[3], seg_grp0[3];        // a segment's columns, first column, first workgroup
    const bf16_t *Wup;
    const bf16_t *residual;
    bf16_t *Y;
    int32_t M, K;
    int64_t ldx, ldy, ldres;
    const int32_t *xmap, *ymap, *rmap;
    int32_t seq_len, flags;
    uint32_t x_bytes, res_bytes;
    const float *rope_table;                              // cos | sin per row, see GemmArgs::rope_table
    int32_t rope_cols, rope_lh;
    const int32_t *rope_pos;                              // ROWS_ROPE_POS: positions of rows r % rope_seq_len
    int32_t rope_seq_len;
    double rope_log2_theta;
};

// ROWS_ROPE reads cos and sin from a table (a layer's norm kernel has written it); ROWS_ROPE_POS, where no kernel in front
// could, computes the one or two angles of a thread while the first weights are on their way.
enum { ROWS_PLAIN = 0, ROWS_SWIGLU = 1, ROWS_ROPE = 2, ROWS_ROPE_POS = 3 };

__device__ __forceinline__ bf16x8 load16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

// TM: 16-row blocks of X.  TN: 16-column blocks (two for SwiGLU: gate and up of the same columns; two for the
// rotary epilogue: the first halves of 16 rotation pairs and their partners).  D: steps in flight per wavefront.
template <int TM, int TN, int D, int MODE>
__global__ __launch_bounds__(ROWS_NW * 64) void gemm_rows_kernel(GemmRowsParams p) {
    static_assert(MODE == ROWS_PLAIN || TN % 2 == 0, "paired columns");
    static_assert(TN <= 2, "one block or one pair of blocks");
    constexpr bool ROT = MODE == ROWS_ROPE || MODE == ROWS_ROPE_POS;
    constexpr int RB = TM < 2 ? 1 : 2;                    // row blocks summed per pass of the reduction
    constexpr int NPASS = TM / RB, TNO = MODE == ROWS_PLAIN ? TN : TN / 2;
    constexpr int OUT = RB * TNO * 256, PER = (OUT + ROWS_NW * 64 - 1) / (ROWS_NW * 64);
    __shared__ __attribute__((aligned(16))) float part[ROWS_NW][RB][TN][256];

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = blockIdx.x;
    const int seg = grp >= p.seg_grp0[2] ? 2 : grp >= p.seg_grp0[1] ? 1 : 0;
    const int seg_rows = p.seg_rows[seg], K = p.K;
    int col[TN];                                          // first column (in the segment) of each block
    {
        const int q = grp - p.seg_grp0[seg];
        if constexpr (ROT) {                              // 16 pairs of one head
            const int pair0 = q * 16, half = 1 << p.rope_lh;
            col[0] = ((pair0 >> p.rope_lh) << (p.rope_lh + 1)) + (pair0 & (half - 1));
            col[1] = col[0] + half;
        } else
#pragma unroll
            for (int j = 0; j < TN; ++j) col[j] = (q * TNO + j % TNO) * 16;
    }
    const uint32_t w_bytes = (uint32_t)((int64_t)seg_rows * K * 2);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(p.X), 0, p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(p.W[seg]), 0, w_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(MODE == ROWS_SWIGLU ? p.Wup : p.W[seg]), 0, w_bytes, 0x00020000);
    uint32_t w_off[TN], x_off[TM];
#pragma unroll
    for (int j = 0; j < TN; ++j) w_off[j] = col[j] + l16 < seg_rows ? (uint32_t)((col[j] + l16) * (int64_t)K * 2) + g * 16 : OOB_OFF;
    {
        int32_t rows[TM], src[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) rows[i] = 16 * i + l16 < p.M ? 16 * i + l16 : -1;
        map_rows_near(p.xmap, p.seq_len, rows, 0, src);
#pragma unroll
        for (int i = 0; i < TM; ++i) x_off[i] = src[i] >= 0 ? (uint32_t)(src[i] * p.ldx * 2) + g * 16 : OOB_OFF;
    }

    // output o = tid (+ 512) of a pass: row block o / 256 / TNO, column block o / 256 % TNO; its rows are looked up
    // before the first weights are requested, so that no wait for a lookup drains the ring
    const bool has_res = p.flags & CASCADE_EPI_RESIDUAL;
    int32_t yrow[NPASS * PER], rrow[NPASS * PER];
    float pos[MODE == ROWS_ROPE_POS ? NPASS * PER : 1], cos_sin[MODE == ROWS_ROPE_POS ? NPASS * PER : 1][2];
    {
        int32_t rows[NPASS * PER];
#pragma unroll
        for (int ps = 0; ps < NPASS; ++ps)
#pragma unroll
            for (int x = 0; x < PER; ++x) {
                const int o = tid + x * ROWS_NW * 64, m = 16 * (ps * RB + (o >> 8) / TNO) + ((o >> 4) & 15);
                rows[ps * PER + x] = o < OUT && m < p.M && col[(o >> 8) % TNO] + (o & 15) < seg_rows ? m : -1;
            }
        if constexpr (MODE == ROWS_ROPE_POS) {
#pragma unroll
            for (int x = 0; x < NPASS * PER; ++x) pos[x] = (float)p.rope_pos[rows[x] < 0 ? 0 : rows[x] % p.rope_seq_len];
        }
        map_rows_near(p.ymap, p.seq_len, rows, 0, yrow);
        map_rows_near(has_res ? p.rmap : nullptr, p.seq_len, rows, 0, rrow);
    }

    // ring of pieces of 64 reduction elements (two MFMA steps); pieces past the end read as zeros.  The two halves of
    // a row's 128-byte line are requested back to back: the second one is served by the line the first one brings.
    bf16x8 wr[D][TN][2], xr[D][TM][2];
    const int n_pieces = K / 64;
    // The workgroups of an XCD (every eighth) start two pieces (256 bytes, the L2 channel interleave) apart and wrap
    // around: rows are a multiple of the 4 KB that the 16 channels cover apart, so workgroups in step would all ask
    // one channel for the same piece of X (8192 x 28672, 32 rows: 182 us in step, 160 us apart).
    const int rot = (int)(((uint32_t)grp >> 3) * 2u % (uint32_t)n_pieces);
    auto request = [&](int slot, int piece) {
        const int at = piece + rot - (piece + rot >= n_pieces ? n_pieces : 0);
        // an offset that is out of range already stays so: both marks added would wrap around to a valid one
        const uint32_t past = piece < n_pieces ? 0u : OOB_OFF, add = piece < n_pieces ? (uint32_t)at * 128 : 0u;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int s = 0; s < 2; ++s) wr[slot][j][s] = load16(MODE == ROWS_SWIGLU && j >= TNO ? ru : rw, (w_off[j] | past) + add + 64 * s);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int s = 0; s < 2; ++s) xr[slot][i][s] = load16(rx, (x_off[i] | past) + add + 64 * s);
    };
    f32x4 acc[TM][TN];                                    // transposed: row 16i + lane%16, columns 4(lane/16) + r
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < D; ++d) request(d, wave + ROWS_NW * d);
    if constexpr (MODE == ROWS_ROPE_POS) {
#pragma unroll
        for (int x = 0; x < PER; ++x) {                   // the same pair of columns in every pass
            const int c = col[((tid + x * ROWS_NW * 64) >> 8) % TNO] + (tid & 15);
            const RopeRev rev = rope_rev_log2(p.rope_log2_theta, c & ((1 << p.rope_lh) - 1), 2 << p.rope_lh);
#pragma unroll
            for (int ps = 0; ps < NPASS; ++ps)
                rope_cos_sin(pos[ps * PER + x], rev.hi, rev.lo, cos_sin[ps * PER + x][0], cos_sin[ps * PER + x][1]);
        }
    }

    // the residual values a thread adds at the end follow the first steps (no branch: zeros where there are none)
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(p.residual), 0,
                                                                        has_res ? p.res_bytes : 0, 0x00020000);
    uint16_t res[NPASS][PER];
#pragma unroll
    for (int ps = 0; ps < NPASS; ++ps)
#pragma unroll
        for (int x = 0; x < PER; ++x) {
            const int o = tid + x * ROWS_NW * 64, c = p.seg_col0[seg] + col[(o >> 8) % TNO] + (o & 15);
            const int32_t r = rrow[ps * PER + x];
            res[ps][x] = __builtin_amdgcn_raw_buffer_load_b16(rr, r >= 0 ? (uint32_t)((r * p.ldres + c) * 2) : OOB_OFF, 0, 0);
        }

    for (int piece = wave; piece < n_pieces; piece += ROWS_NW * D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[d][j][s], xr[d][i][s], acc[i][j], 0, 0, 0);
            request(d, piece + ROWS_NW * (D + d));
        }
    }

#pragma unroll
    for (int ps = 0; ps < NPASS; ++ps) {
        if (ps) __syncthreads();                          // the sums of the pass before have been read
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) *(f32x4 *)&part[wave][i][j][l16 * 16 + g * 4] = acc[ps * RB + i][j];
        __syncthreads();
#pragma unroll
        for (int x = 0; x < PER; ++x) {
            const int o = tid + x * ROWS_NW * 64, at = o & 255, i = (o >> 8) / TNO, j = (o >> 8) % TNO;
            if (yrow[ps * PER + x] < 0) continue;
            const int m = 16 * (ps * RB + i) + (at >> 4), c = col[j] + (at & 15);
            float v = 0.f, v2 = 0.f;
#pragma unroll
            for (int w = 0; w < ROWS_NW; ++w) {
                v += part[w][i][j][at];
                if (MODE != ROWS_PLAIN) v2 += part[w][i][j + TNO][at];
            }
            bf16_t *y = p.Y + (int64_t)yrow[ps * PER + x] * p.ldy + p.seg_col0[seg];
            const bf16_t *bias = (p.flags & CASCADE_EPI_BIAS) ? p.bias[seg] : nullptr;
            if constexpr (MODE == ROWS_SWIGLU) {
                v = v * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * v)) * v2;
            } else if constexpr (ROT) {
                if (bias) { v += (float)bias[c]; v2 += (float)bias[c + (1 << p.rope_lh)]; }
                if (p.seg_col0[seg] + c < p.rope_cols) {
                    const int half = 1 << p.rope_lh;
                    float cs, sn;
                    if constexpr (MODE == ROWS_ROPE_POS) {
                        cs = cos_sin[ps * PER + x][0];
                        sn = cos_sin[ps * PER + x][1];
                    } else {
                        const float *t = p.rope_table + (int64_t)m * (2 * half) + (c & (half - 1));
                        cs = t[0];
                        sn = t[half];
                    }
                    const float a = v;
                    v = a * cs - v2 * sn;
                    v2 = v2 * cs + a * sn;
                }
                y[c + (1 << p.rope_lh)] = (bf16_t)v2;
            } else {
                if (bias) v += (float)bias[c];
                v = apply_act_bf16(v, p.flags);
            }
            y[c] = (bf16_t)(has_res ? v + (float)__builtin_bit_cast(bf16_t, res[ps][x]) : v);
        }
    }
}

template <int TM, int TN, int D, int MODE>
static int32_t launch_rows(const GemmArgs &a, hipStream_t s) {
    GemmRowsParams p;
    constexpr int COLS = MODE == ROWS_SWIGLU ? 8 * TN : 16 * TN;      // of the output, per workgroup
    int col0 = 0;
    int64_t grp = 0;
    for (int i = 0; i < 3; ++i) {
        const int rows = std::max(0, a.seg_end[i] - col0);
        p.W[i] = (const bf16_t *)a.W[i];
        p.bias[i] = (const bf16_t *)a.bias[i];
        p.seg_rows[i] = rows;
        p.seg_col0[i] = col0;
        p.seg_grp0[i] = rows ? (int32_t)grp : INT32_MAX;
        grp += (rows + COLS - 1) / COLS;
        col0 = std::max(col0, a.seg_end[i]);
    }
    p.X = (const bf16_t *)a.X; p.Wup = (const bf16_t *)a.W_up; p.residual = (const bf16_t *)a.residual;
    p.Y = (bf16_t *)a.Y;
    p.M = a.M; p.K = a.K;
    p.ldx = a.ldx; p.ldy = a.ldy; p.ldres = a.ldres;
    p.xmap = a.xmap.map; p.ymap = a.ymap.map; p.rmap = a.rmap.map;
    p.seq_len = a.xmap.map ? a.xmap.seq_len : a.ymap.map ? a.ymap.seq_len : a.rmap.map ? a.rmap.seq_len : 1;
    p.flags = a.epilogue;
    p.x_bytes = (uint32_t)((int64_t)a.M * a.ldx * 2);
    p.res_bytes = (uint32_t)((int64_t)a.M * a.ldres * 2);
    p.rope_table = a.rope_table; p.rope_cols = a.rope_cols; p.rope_lh = 0;
    p.rope_pos = a.rope_pos; p.rope_seq_len = a.rope_seq_len;
    p.rope_log2_theta = MODE == ROWS_ROPE_POS ? std::log2((double)a.rope_theta) : 0.0;
    if (MODE == ROWS_ROPE || MODE == ROWS_ROPE_POS)
        while ((2 << p.rope_lh) < a.rope_head_dim) ++p.rope_lh;
    hipLaunchKernelGGL((gemm_rows_kernel<TM, TN, D, MODE>), dim3((unsigned)grp), dim3(ROWS_NW * 64), 0, s, p);
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}

// Column blocks per workgroup: two where that still gives the CUs a workgroup each, because X is re-read by every
// workgroup and arrives at ~18 bytes per clock and CU.  Blocks = N / 16 (gate and up counted apart).  Measured (us):
// 6144 x 4096 (384 blocks), 4 / 64 rows: one block 17.1 / 44.3, two 13.6 / 29.3; 8192 x 8192, 4 / 64 rows: 32 / 88 and
// 28 / 52.
static int64_t rows_blocks(const GemmArgs &a) {
    return (int64_t)((a.N + 15) / 16) * (a.epilogue & CASCADE_EPI_SWIGLU ? 2 : 1);
}
static int rows_blocks_per_workgroup(const GemmArgs &a) {
    return a.rope_table || a.rope_pos || (a.epilogue & CASCADE_EPI_SWIGLU) || rows_blocks(a) >= 2 * 192 ? 2 : 1;
}

template <int TM, int D1, int D2>
static int32_t launch_rows_tm(const GemmArgs &a, hipStream_t s) {
    if (a.rope_table) return launch_rows<TM, 2, D2, ROWS_ROPE>(a, s);
    if (a.rope_pos) return launch_rows<TM, 2, D2, ROWS_ROPE_POS>(a, s);
    if (a.epilogue & CASCADE_EPI_SWIGLU) return launch_rows<TM, 2, D2, ROWS_SWIGLU>(a, s);
    return rows_blocks_per_workgroup(a) == 2 ? launch_rows<TM, 2, D2, ROWS_PLAIN>(a, s) : launch_rows<TM, 1, D1, ROWS_PLAIN>(a, s);
}

// Whether the few-row kernel is the faster one.  Every round of workgroups (one per CU, of the 256 that the limits were
// measured on) re-reads X and waits for its first pieces, which the 128 x 128 tiles do once, so with the rounds the rows
// it can carry shrink and the reduction has to be longer.  Measured against those tiles, weights cold (us, tiles / rows).
// One round: 768 x 64, 1 row 4.9 / 4.0, 4096 x 4096, 16 rows 31 / 12, 8192 x 4096, 32 rows 33 / 21; above 32 rows from
// K = 768 (one block: 4096 x 512, 64 rows 7.5 / 8.2, x 768 10.4 / 9.2), 2048 (two: 8192 x 1024, 64 rows 12.0 / 13.1, x
// 4096 33 / 30) or 1024 (SwiGLU: 4096 x 512 8.3 / 10.3, x 1024 12.2 / 12.6 and 3 us ahead from the last-level cache).  Two rounds: 10240 x 2048, 16 rows 18.9 / 18.0, 24 rows 18.9 /
// 21.6, x 1024, 4 rows 11.5 / 12.7; SwiGLU 8192 x 4096, 16 rows 36 / 29, 32 rows 37 / 39.  More: 28672 x 4096, 4 rows
// 47 / 45, 16 rows 46 / 56; SwiGLU 28672 x 4096, 4 rows 87 / 77, 12 rows 87 / 93.  SwiGLU launches whose tiles number
// between one half and one to a CU stream the weights as fast in tiles, short of very long reductions: 8448 to 16384 x
// 4096, 4 rows 35 / 36, 39 / 37, 47 / 48, 44 / 48, 48 / 50; x 2048, 8 rows 21 / 23, 26 / 29; 11008 x 8192, 8 rows 75 / 70,
// 16384 x 8192, 8 rows 130 / 95.
static bool rows_faster(const GemmArgs &a) {
    const int per = rows_blocks_per_workgroup(a);
    const int64_t rounds = ((rows_blocks(a) + per - 1) / per + 255) / 256;
    const bool swiglu = a.epilogue & CASCADE_EPI_SWIGLU;
    if (rounds == 1) return a.M <= 32 || (a.M <= 64 && a.K >= (swiglu ? 1024 : per == 2 ? 2048 : 768));
    if (a.K < 2048) return false;
    if (rounds == 2) return a.M <= 16;
    const int64_t tiles = (a.N + 63) / 64;                // of a SwiGLU launch
    if (swiglu && tiles > 128 && tiles <= 256) return a.K >= 8192 && a.M <= 8;
    return a.M <= 4 && rounds <= 8;
}

bool gemm_rows_takes(const GemmArgs &a) {
    if (a.ascending_k || a.K % 64 || a.ldx % 8 || !rows_faster(a)) return false;
    if (((uintptr_t)a.X | (uintptr_t)a.W_up) % 16) return false;      // 16-byte operand loads
    if (a.rope_table && (a.rope_head_dim % 32 || (uintptr_t)a.rope_table % 4)) return false;   // 16 pairs stay in a head
    // columns of the output come as pairs half a head apart, 16 pairs of one head to a workgroup
    if (a.rope_pos && (a.rope_head_dim % 32 || (a.rope_head_dim & (a.rope_head_dim - 1)) || a.N % a.rope_head_dim)) return false;
    // A pair is two column blocks: where one to a workgroup is the better split, half of the workgroups each stream twice as much,
    // which from K = 2048 on costs more than the pass behind the GEMM.  One block and that pass / rotated here (us): 3072 x 4096,
    // 1, 16, 32, 64 rows 11.5 / 12.8, 14.2 / 15.8, 18.3 / 19.9, 26.2 / 28.8; x 2048 8.2 / 8.4, 10.1 / 9.7, 12.2 / 12.7, 17.4 /
    // 18.0; x 1536 8.2 / 7.8, 9.5 / 8.8, 11.1 / 10.1, 14.1 / 14.1; 1024 x 4096, 1 row 10.2 / 12.0.
    if (a.rope_pos && a.K > 1536 && rows_blocks(a) < 2 * 192) return false;
    if ((int64_t)a.M * std::max(a.ldx, a.ldres) * 2 >= (int64_t)OOB_OFF) return false;
    int col0 = 0;
    for (int i = 0; i < 3; ++i) {
        const int64_t rows = std::max(0, a.seg_end[i] - col0);
        if (rows && (uintptr_t)a.W[i] % 16) return false;
        if (rows * a.K * 2 >= (int64_t)OOB_OFF) return false;
        col0 = std::max(col0, a.seg_end[i]);
    }
    return a.seg_end[0] > 0;
}

int32_t launch_gemm_rows(const GemmArgs &a, hipStream_t s) {
    if (a.M <= 16) return launch_rows_tm<1, 5, 4>(a, s);
    if (a.M <= 32) return launch_rows_tm<2, 4, 3>(a, s);
    return launch_rows_tm<4, 3, 3>(a, s);
}
