// bf16 shard GEMM, main kernel: Y[rows] = epilogue(X[rows] W^T), fp32 accumulation, K % 64 == 0.
// (The token-as-batch linear layers: q/k/v projection of Algorithm 2, o projection that
// closes Algorithm 4, the MLP step that closes Algorithm 1.  Shards appear only as row maps.)
//
// Shape of the kernel (chosen from measurements on MI355X: 16x16x32 bf16 MFMA reaches ~98 % of the
// chip's matrix peak with two wavefronts per SIMD, ~89 % with one; LDS delivers ~235 B/clk/CU on
// conflict-free 16-byte reads):
//  * 8 wavefronts per workgroup (2 per SIMD, <= 256 registers each) or 4 (one per SIMD, up to 512
//    registers: 128-row wavefront tiles whose accumulators live in the accumulation registers; every
//    memory operation hand-placed between two MFMAs), 16x16x32 MFMA blocks.
//  * K walked in steps of 64.  Tiles go from HBM/L2 straight into LDS with buffer loads
//    that write LDS directly (no register staging, out-of-range rows read as zero), NST stages deep:
//    the loads of steps t+1 .. t+NST-1 are in flight while step t is multiplied.  The wait for "step
//    t has landed" is s_waitcnt vmcnt(loads of the younger steps), issued together with the
//    workgroup barrier as inline assembly: a compiler-generated barrier would wait for vmcnt(0) and
//    drain the pipeline.
//  * LDS rows are 64 bf16 without padding; the 16-byte chunk c of tile row r is stored at slot
//    c ^ ((r >> 1) & 7), which makes both the direct-to-LDS writes (1 KiB contiguous per wavefront instruction) and the MFMA operand reads
//    (16 rows x same chunk) bank-conflict free.
//  * Epilogue.  8 wavefronts, through LDS: each wavefront transposes 16 accumulator rows at a time so
//    that a lane ends up with 4 consecutive columns (and the 4 columns 64 further on): stores and
//    residual reads are 128-byte runs.
//    4 wavefronts: accumulators are computed transposed (a lane owns 4 consecutive columns already) from
//    weight rows in an order that makes them 8, and stored as they lie, 16 bytes per lane, without LDS.
//  * The machine is power-limited under this load (the clock falls from 2.4 to 1.7-2.0 GHz as the
//    matrix pipes fill up), so what counts is energy per flop as much as issue slots: fewer LDS bytes
//    and fewer instructions per MFMA, which is what the 4-wavefront schedule buys.
#include <cstdlib>
#include <type_traits>
#include "common.h"
#include "device_utils.h"
#include "epilogue.h"

#define MAX_BYTES 0x80000000u        // operands are smaller
#define OOB_OFF (MAX_BYTES + 4096)   // of a row outside: beyond any buffer, also one that starts FOUR_SHIFT bytes early

struct Gemm2Params {
    const bf16_t *X;
    const bf16_t *W[3];
    const bf16_t *bias[3];
    int32_t seg_rows[3], seg_col0[3], seg_tile0[3];
    const bf16_t *Wup;
    const bf16_t *residual;
    bf16_t *Y;
    int32_t M, K;
    int32_t tiles_m, tiles_n;
    int64_t ldx, ldy, ldres;
    const int32_t *xmap, *ymap, *rmap;
    int32_t seq_len, flags;
    uint32_t x_bytes;
    // rotary embedding in the epilogue (ROPE kernels): cos | sin of every packed row's angles, [M][head_dim] fp32;
    // output columns below rope_cols are rotated; rope_lh = log2(head_dim / 2)
    const float *rope_table;
    int32_t rope_cols, rope_lh;
    // split reduction: workgroups per tile; PARTS kernels: their fp32 planes [parts][M][columns]; PAIR kernels: the
    // first one's accumulators [tile][accumulator block][thread], and per tile a ticket word and a flag word
    float *planes;
    uint32_t *sk_sync;
    int32_t parts, planes_ld;
};
enum { SPLIT_NONE = 0, SPLIT_PAIR = 1, SPLIT_PARTS = 2 };
typedef __attribute__((address_space(3))) void lds_void;


// Instruction x of a wavefront's share of a tile, which lies at `lds`: 16 bytes per lane from a buffer straight into LDS,
// lane i at lds + 1024 x + 16 i.  The k offset is wavefront-uniform and goes into the scalar operand: no vector addition
// per load.  (A row outside carries OOB_OFF in voff; the range check covers the sum, which stays above the buffer's size.)
// FOUR: four of them share one LDS address (one write of m0) and differ in the instruction's offset, which the hardware
// adds on both sides: the buffer starts FOUR_SHIFT bytes early and voff is that much, less the instruction's offset, larger.
constexpr uint32_t FOUR_SHIFT = 3072;
template <bool FOUR>
__device__ __forceinline__ void load16_to_lds(__amdgpu_buffer_rsrc_t r, unsigned char *lds, int x, uint32_t voff, uint32_t soff) {
    lds_void *at = (lds_void *)(lds + (FOUR ? x & ~3 : x) * 1024);
    const int off = FOUR ? x & 3 : 0;
    if (off == 0) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, at, 16, voff, soff, 0, 0);
    else if (off == 1) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, at, 16, voff, soff, 1024, 0);
    else if (off == 2) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, at, 16, voff, soff, 2048, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(r, at, 16, voff, soff, 3072, 0);
}
template <bool FOUR>
__device__ __forceinline__ uint32_t load_off(uint32_t off, int x) { return FOUR ? off + FOUR_SHIFT - (x & 3) * 1024 : off; }
template <bool FOUR>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_buffer(const bf16_t *base, uint32_t bytes) {
    constexpr uint32_t early = FOUR ? FOUR_SHIFT : 0;
    return __builtin_amdgcn_make_buffer_rsrc((unsigned char *)const_cast<bf16_t *>(base) - early, 0, bytes + early, 0x00020000);
}

__device__ __forceinline__ float silu_fast(float x) {
    // x * 1/(1 + 2^(-x log2 e)); hardware reciprocal (1 ulp), output is rounded to bf16 anyway
    return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
}

// The residual values a lane adds in gemm_epilogue, all row blocks of its wavefront tile: [row block][row group
// of 4][4-column chunk].
template <int TM, int WTN>
struct ResidualAhead {
    static constexpr int NCH = (WTN + 63) / 64;
    bf16x4 r[TM][4][NCH];
    __device__ __forceinline__ void load(const Gemm2Params &p, int lane, int m0, int wm0, int wn0, int nloc0, int seg,
                                         int seg_rows) {
        const int m4 = (lane & 15) * 4, rsel = lane >> 4;
        const int wcol0 = nloc0 + wn0;
        const int gcol0 = p.seg_col0[seg];
        const int b0 = m0 / p.seq_len;                     // sequence of the tile's first row (uniform)
        int32_t rows[TM * 4], src[TM * 4];                 // every row's lookup goes out before the first residual load
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int gm = m0 + wm0 + 16 * i + 4 * t + rsel;
                rows[4 * i + t] = gm < p.M ? gm : m0;
            }
        map_rows_near(p.rmap, p.seq_len, rows, b0, src);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int gm = m0 + wm0 + 16 * i + 4 * t + rsel;
                const bf16_t *rrow = p.residual + (int64_t)src[4 * i + t] * p.ldres + gcol0;
#pragma unroll
                for (int cc = 0; cc < NCH; ++cc) {
                    const int c = wcol0 + 64 * cc + m4;
                    r[i][t][cc] = bf16x4{0, 0, 0, 0};
                    if (gm < p.M && c + 4 <= seg_rows && 64 * cc + m4 < WTN) r[i][t][cc] = *(const bf16x4 *)(rrow + c);
                }
            }
    }
};

// Epilogue of the 8-wavefront kernels.  acc[i][j][r] holds row 16i + 4(lane/16) + r, column
// 16j + lane%16 of the wavefront's WTM x WTN tile.  The caller guarantees (with a workgroup barrier)
// that every wavefront is done with the tile buffers: smem is reused as staging, one private region
// per wavefront, so inside the epilogue only wavefront-level ordering of LDS traffic is needed.
template <int TM, int TN, int WTN>
__device__ __forceinline__ void gemm_epilogue(const Gemm2Params &p, f32x4 (&acc)[TM][TN], unsigned char *smem,
                                              int wave, int lane, int m0, int wm0, int wn0, int nloc0, int seg,
                                              int seg_rows) {
    constexpr int STG_LD = WTN + 4;
    constexpr int NCH = (WTN + 63) / 64;                   // 4-column chunks per lane: columns 64 cc + m4
    const int flags = p.flags;
    float *stg = (float *)smem + wave * 16 * STG_LD;
    const int l16 = lane & 15, m4 = l16 * 4, rsel = lane >> 4;
    const int wcol0 = nloc0 + wn0;                         // first output column (in segment)
    const int gcol0 = p.seg_col0[seg];
    const int b0 = m0 / p.seq_len;                         // sequence of the tile's first row (uniform)
    const bf16_t *bias = (flags & CASCADE_EPI_BIAS) ? p.bias[seg] : nullptr;
    f32x4 bias_v[NCH];
#pragma unroll
    for (int cc = 0; cc < NCH; ++cc) {
        const int c = wcol0 + 64 * cc + m4;
        bias_v[cc] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (bias)
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (c + x < seg_rows) bias_v[cc][x] = (float)bias[c + x];
    }
    const bool act = flags & (CASCADE_EPI_GELU_ERF | CASCADE_EPI_GELU_TANH);
    // Residual of every row block requested up front: one memory latency for the whole epilogue instead of one per row block.
    static_assert(TM * 4 * NCH <= 32, "registers for the residual of all row blocks");
    ResidualAhead<TM, WTN> res;
    const bool has_res = flags & CASCADE_EPI_RESIDUAL;
    if (has_res) res.load(p, lane, m0, wm0, wn0, nloc0, seg, seg_rows);
    // Two copies of the unrolled loops, chosen once: without the (long) GELU code the plain one stays small
    // and contiguous in the instruction cache.
    auto blocks = [&](auto act_tag) {
    constexpr bool ACT = decltype(act_tag)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) stg[(4 * rsel + r) * STG_LD + 16 * j + l16] = acc[i][j][r];
        __builtin_amdgcn_wave_barrier();                   // LDS serves one wavefront's accesses in order
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int rl = 4 * t + rsel;
            const int gm = m0 + wm0 + 16 * i + rl;
            if (gm < p.M) {
                bf16_t *yrow = p.Y + map_row_near(p.ymap, p.seq_len, gm, b0) * p.ldy + gcol0;
                const bf16_t *rrow = has_res ? p.residual + map_row_near(p.rmap, p.seq_len, gm, b0) * p.ldres + gcol0 : nullptr;
#pragma unroll
                for (int cc = 0; cc < NCH; ++cc) {
                    const int c = wcol0 + 64 * cc + m4;
                    if (c >= seg_rows || 64 * cc + m4 >= WTN) continue;
                    f32x4 v = *(const f32x4 *)(stg + rl * STG_LD + 64 * cc + m4);
                    v += bias_v[cc];
                    if constexpr (ACT) {
#pragma unroll
                        for (int x = 0; x < 4; ++x) v[x] = apply_act_bf16(v[x], flags);
                    }
                    if (c + 4 <= seg_rows) {
                        if (has_res) {
                            const bf16x4 rv = res.r[i][t][cc];
#pragma unroll
                            for (int x = 0; x < 4; ++x) v[x] += (float)rv[x];
                        }
                        bf16x4 o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
                        *(bf16x4 *)(yrow + c) = o;
                    } else {
                        for (int x = 0; x < 4 && c + x < seg_rows; ++x)
                            yrow[c + x] = (bf16_t)(v[x] + (rrow ? (float)rrow[c + x] : 0.f));
                    }
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    };
    // A tile inside the matrix with no activation to apply takes a copy of the loop without the per-row and
    // per-chunk range checks and with the residual from the registers filled above: a fifth of the instructions.
    // The epilogue of a single-round launch runs once per workgroup, from a cold instruction cache, at about three
    // times the cycles per instruction of warm code, so its length in instructions is what it costs.
    auto blocks_inside = [&](auto res_tag) {
    constexpr bool RES = decltype(res_tag)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) stg[(4 * rsel + r) * STG_LD + 16 * j + l16] = acc[i][j][r];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int rl = 4 * t + rsel;
            const int gm = m0 + wm0 + 16 * i + rl;
            bf16_t *yrow = p.Y + map_row_near(p.ymap, p.seq_len, gm, b0) * p.ldy + gcol0 + wcol0 + m4;
#pragma unroll
            for (int cc = 0; cc < NCH; ++cc) {
                f32x4 v = *(const f32x4 *)(stg + rl * STG_LD + 64 * cc + m4);
                v += bias_v[cc];
                if constexpr (RES) {
                    const bf16x4 rv = res.r[i][t][cc];
#pragma unroll
                    for (int x = 0; x < 4; ++x) v[x] += (float)rv[x];
                }
                *(bf16x4 *)(yrow + 64 * cc) = bf16x4{(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    };
    const bool inside = m0 + wm0 + 16 * TM <= p.M && wcol0 + WTN <= seg_rows && WTN % 64 == 0;
    if (inside && !act && has_res) blocks_inside(std::true_type{});
    else if (inside && !act) blocks_inside(std::false_type{});
    else if (act) blocks(std::true_type{});
    else blocks(std::false_type{});
}

// Accumulator block of the one-wavefront kernels (held in accumulation registers by the tied MFMAs) -> vector
// registers, at the point of use.  Read through plain C++ the compiler copies all blocks across right behind
// the main loop, which a 256-accumulator tile has no registers for.
__device__ __forceinline__ f32x4 acc_load(const f32x4 &c) {
    float x0, x1, x2, x3;
    asm volatile("v_accvgpr_read_b32 %0, %4\n\tv_accvgpr_read_b32 %1, %5\n\tv_accvgpr_read_b32 %2, %6\n\t"
                 "v_accvgpr_read_b32 %3, %7"
                 : "=v"(x0), "=v"(x1), "=v"(x2), "=v"(x3)
                 : "a"(c[0]), "a"(c[1]), "a"(c[2]), "a"(c[3]));
    return f32x4{x0, x1, x2, x3};
}

// The kernel's argument read again from the argument segment (it is the only one), through a pointer the compiler does
// not know: what only the epilogue needs would otherwise be loaded ahead of the tile loop and kept in scalar registers
// that the loop does not have (spilled to lanes of vector registers, read back one lane at a time).
typedef const __attribute__((address_space(4))) Gemm2Params KernelArgs;
__device__ __forceinline__ KernelArgs &params_again() {
    KernelArgs *k = (KernelArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(k));
    return *k;
}

// Which output columns the blocks of a one-wavefront kernel's wavefront tile hold (TNO blocks of 16 output columns).
// Blocks 2t and 2t + 1 share 32 columns so that a lane's four columns of the first are followed by its four of the
// second: the rows of the weight tile are put into LDS in that order (a per-lane offset of the loads, free), and a lane
// stores 8 consecutive columns, 16 bytes, straight from its accumulators.  An odd last block keeps its columns in order.
template <int TNO>
__device__ constexpr int epi_col(int j, int g) {                 // first column of lane group g (lane / 16) in block j
    return (j | 1) < TNO ? 32 * (j >> 1) + 8 * g + 4 * (j & 1) : 16 * j + 4 * g;
}
template <int TNO>
__device__ __forceinline__ int epi_row_col(int row) {            // row of such a weight tile (of TNO * 16) -> column
    return (row >> 5) < TNO / 2 ? (row & ~31) + 8 * ((row >> 2) & 3) + 4 * ((row >> 4) & 1) + (row & 3) : row;
}
__device__ __forceinline__ bf16x4 to_bf16x4(const f32x4 &v) { return bf16x4{(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]}; }
__device__ __forceinline__ bf16x8 join8(const bf16x4 &a, const bf16x4 &b) { return bf16x8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]}; }

// Reads under a condition count as outstanding for the compiler when the condition has failed, and it would wait for
// all memory operations in every pass of the next tile's main loop (4096 x 768 x 3072 25 -> 34 us): the epilogues of
// edge tiles, which have such reads, wait here.
__device__ __forceinline__ void wait_conditional_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }   // vmcnt(0)

// Four rotation pairs.  Which product of a sum is rounded on its own is written out: left to the compiler it differed between
// the copies of the loop below, and a row's bits depended on whether its tile lies inside the matrix.
__device__ __forceinline__ void rotate4(f32x4 &a, f32x4 &b, const f32x4 &cs, const f32x4 &sn) {
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const float a0 = a[x];
        a[x] = fmaf(a0, cs[x], -(b[x] * sn[x]));
        b[x] = fmaf(a0, sn[x], b[x] * cs[x]);
    }
}

// ROPE: the wavefront tile holds WTN/2 rotation pairs (i, i + head_dim/2 of one head): block j the first
// halves, block j + TN/2 the second halves, same lane and slot, like gate and up of SwiGLU.  Pair p of a segment is
// column (p / half) head_dim + p % half and the column `half` further on, so 4 (8) consecutive pairs are 4 (8)
// consecutive columns as long as half is a multiple of 4 (8).  The rotation runs on the fp32 accumulators (one
// rounding to bf16), with cos and sin read from the table the pre-pass norm kernel wrote for every row.
template <int TM, int TN, int WTN>
__device__ __forceinline__ void gemm_epilogue_rope(KernelArgs &p, f32x4 (&acc)[TM][TN], int lane, int m0, int wm0,
                                                   int wn0, int pair0, int seg, int seg_rows) {
    static_assert(TN % 2 == 0, "pairs split the wavefront tile");
    constexpr int TNO = TN / 2;
    const int l16 = lane & 15, g = lane >> 4;
    const int wp0 = pair0 + (wn0 / WTN) * (WTN / 2);       // wavefront's first pair
    const int lh = p.rope_lh, half = 1 << lh, n_pairs = seg_rows >> 1;
    const int gcol0 = p.seg_col0[seg];
    const int b0 = m0 / p.seq_len;                         // sequence of the tile's first row (uniform)
    const bf16_t *bias = (p.flags & CASCADE_EPI_BIAS) ? p.bias[seg] : nullptr;
    int rows[TM], yrow[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int gm = m0 + wm0 + 16 * i + l16;
        rows[i] = gm < p.M ? gm : -1;
    }
    map_rows_near(p.ymap, p.seq_len, rows, b0, yrow);
    auto column = [&](int pp) { return ((pp >> lh) << (lh + 1)) + (pp & (half - 1)); };   // of a pair's first half
    // A wavefront tile inside the matrix, without bias, whose columns are all rotated (q, k) or all passed through (v)
    // takes a copy of the loop without the per-pair checks, with the cos | sin values requested three row blocks ahead
    // (2 x 16 bytes per pair block and row from the table in L2: one latency instead of one per row block).  The
    // code runs once per workgroup, from a cold instruction cache: its length in instructions is what it costs.
    auto inside_loop = [&](auto rot_tag) {
        constexpr bool ROT = decltype(rot_tag)::value;
        constexpr int AH = ROT ? (TNO > 4 ? 2 : 3) : 1;       // 8 registers per pair block and row block in flight
        f32x4 cs[AH][ROT ? TNO : 1], sn[AH][ROT ? TNO : 1];
        auto request = [&](int i) {
            if constexpr (ROT) {
                const float *trow = p.rope_table + (int64_t)(m0 + wm0 + 16 * i + l16) * (2 * half);
#pragma unroll
                for (int j = 0; j < TNO; ++j) {
                    const int ph = (wp0 + epi_col<TNO>(j, g)) & (half - 1);
                    cs[i % AH][j] = *(const f32x4 *)(trow + ph);
                    sn[i % AH][j] = *(const f32x4 *)(trow + half + ph);
                }
            }
        };
#pragma unroll
        for (int i = 0; i < AH - 1 && i < TM; ++i) request(i);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            bf16_t *y = p.Y + (int64_t)yrow[i] * p.ldy + gcol0;
            if (i + AH - 1 < TM) request(i + AH - 1);
            __builtin_amdgcn_sched_barrier(0);
            bf16x4 oa[TNO], ob[TNO];
#pragma unroll
            for (int j = 0; j < TNO; ++j) {
                f32x4 a = acc_load(acc[i][j]), b = acc_load(acc[i][j + TNO]);
                if constexpr (ROT) rotate4(a, b, cs[i % AH][j], sn[i % AH][j]);
                oa[j] = to_bf16x4(a);
                ob[j] = to_bf16x4(b);
            }
#pragma unroll
            for (int j = 0; j < TNO; j += 2) {
                bf16_t *yc = y + column(wp0 + epi_col<TNO>(j, g));
                if (j + 1 < TNO) {
                    *(bf16x8 *)yc = join8(oa[j], oa[j + 1 < TNO ? j + 1 : j]);
                    *(bf16x8 *)(yc + half) = join8(ob[j], ob[j + 1 < TNO ? j + 1 : j]);
                } else {
                    *(bf16x4 *)yc = oa[j];
                    *(bf16x4 *)(yc + half) = ob[j];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // columns of the wavefront tile: whole heads from the head of its first pair to the head of its last
    const int col_lo = gcol0 + ((wp0 >> lh) << (lh + 1)), col_hi = gcol0 + ((((wp0 + WTN / 2 - 1) >> lh) + 1) << (lh + 1));
    const bool wide = ((p.ldy | gcol0) % 8 == 0) && ((uintptr_t)p.Y % 16 == 0);
    const bool inside = m0 + wm0 + 16 * TM <= p.M && wp0 + WTN / 2 <= n_pairs && !bias && wide;
    if (inside && col_hi <= p.rope_cols) return inside_loop(std::true_type{});
    if (inside && col_lo >= p.rope_cols) return inside_loop(std::false_type{});
    f32x4 bias_a[TNO], bias_b[TNO];                        // of this lane's pairs, once
#pragma unroll
    for (int j = 0; j < TNO; ++j) {
        const int pp = wp0 + epi_col<TNO>(j, g);
        bias_a[j] = bias_b[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (bias && pp < n_pairs) {
            const bf16x4 a4 = *(const bf16x4 *)(bias + column(pp)), b4 = *(const bf16x4 *)(bias + column(pp) + half);
            bias_a[j] = f32x4{(float)a4[0], (float)a4[1], (float)a4[2], (float)a4[3]};
            bias_b[j] = f32x4{(float)b4[0], (float)b4[1], (float)b4[2], (float)b4[3]};
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const float *trow = p.rope_table + (int64_t)(rows[i] < 0 ? 0 : rows[i]) * (2 * half);
        bf16_t *y = p.Y + (int64_t)(rows[i] < 0 ? 0 : yrow[i]) * p.ldy + gcol0;
#pragma unroll
        for (int j = 0; j < TNO; ++j) {
            const int pp = wp0 + epi_col<TNO>(j, g), ph = pp & (half - 1);   // 4 consecutive pairs, one head
            const int col1 = column(pp);
            const bool ok = pp < n_pairs && rows[i] >= 0;  // n_pairs is a multiple of half, half of 8
            f32x4 a = acc_load(acc[i][j]) + bias_a[j], b = acc_load(acc[i][j + TNO]) + bias_b[j];
            if (ok && gcol0 + col1 < p.rope_cols) rotate4(a, b, *(const f32x4 *)(trow + ph), *(const f32x4 *)(trow + half + ph));
            if (ok) {
                *(bf16x4 *)(y + col1) = to_bf16x4(a);
                *(bf16x4 *)(y + col1 + half) = to_bf16x4(b);
            }
        }
    }
    wait_conditional_loads();
}

// Epilogue for accumulators computed transposed (W block as the first MFMA operand): acc[i][j][r]
// holds row 16i + lane%16, column epi_col(j, lane/16) + r of the wavefront's tile, so a lane owns four
// consecutive output columns per block and eight per pair of blocks.  Bias, activation, SwiGLU (block j = gate, block
// j + TN/2 = up: same lane, same slot) and the residual are applied in registers, before the one rounding to bf16, and
// stored from there: an instruction writes 16 rows x 64 bytes.  Through a tile in LDS (stores of whole rows, but twice the
// instructions and two barriers, where nothing overlaps them) the launches took longer: 4096 x 768 x 768 with bias and
// residual 11.5 -> 10.3 us, x 3072 24.8 -> 23.8, 4096 x 3072 x 768 with GELU 30.6 -> 28.7, SwiGLU 700 x 14336 x 4096 147 ->
// 143, 2048 x 14336 x 4096 346 -> 342, 8192 x 4096 x 4096 with residual 209 -> 207.
// PARTNER (split reduction, the workgroup that finishes the tile): the other workgroup's accumulators, stored at
// `part` as they lay in its registers, are added to this one's; they are valid once the word at
// `flag` reads `use`, which is waited for as late as possible, after the row lookups are on their way.
template <int NTHREADS, int TM, int TN, int WTN, bool SWIGLU, bool ACT_OK, bool PARTNER = false>
__device__ __forceinline__ void gemm_epilogue_direct(KernelArgs &p, f32x4 (&acc)[TM][TN], int tid, int m0, int wm0,
                                                     int wn0, int nloc0, int seg, int seg_rows, const f32x4 *part = nullptr,
                                                     uint32_t *flag = nullptr, uint32_t use = 0) {
    static_assert(!SWIGLU || TN % 2 == 0, "gate and up blocks pair up inside the wavefront tile");
    static_assert(!PARTNER || !SWIGLU, "the split reduction runs plain GEMMs");
    constexpr int TNO = SWIGLU ? TN / 2 : TN;              // output blocks of the wavefront tile
    constexpr int OW = SWIGLU ? WTN / 2 : WTN;
    const int flags = p.flags;
    const int lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int c0 = nloc0 + (wn0 / WTN) * OW;               // wavefront's first output column in the segment
    const bf16_t *bias = (!SWIGLU && (flags & CASCADE_EPI_BIAS)) ? p.bias[seg] : nullptr;
    const bool act = ACT_OK && (flags & (CASCADE_EPI_GELU_ERF | CASCADE_EPI_GELU_TANH));
    const int gcol0 = p.seg_col0[seg];
    const int b0 = m0 / p.seq_len;                         // sequence of the tile's first row (uniform)
    const bool has_res = flags & CASCADE_EPI_RESIDUAL;
    // 16-byte stores and residual reads need rows that start on 16-byte boundaries; otherwise 8-byte halves
    const bool wide = ((p.ldy | gcol0) % 8 == 0) && ((uintptr_t)p.Y % 16 == 0) &&
                      (!has_res || (p.ldres % 8 == 0 && (uintptr_t)p.residual % 16 == 0));
    // One wavefront per SIMD: the epilogue is as long as its instruction count, nothing overlaps it.  A wavefront tile
    // that lies inside the matrix takes a copy of the loop without any of the range checks, chosen once per tile; so
    // does the choice between residual and none.
    const bool interior = m0 + wm0 + 16 * TM <= p.M && c0 + OW <= seg_rows && wide;
    int rows[TM], yrow[TM];                                // this lane's rows and where they go
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int gm = m0 + wm0 + 16 * i + l16;
        rows[i] = gm < p.M ? gm : -1;
    }
    map_rows_near(p.ymap, p.seq_len, rows, b0, yrow);
    // BIAS, ACT: that code is present.  INTERIOR: no range checks.  RES: 0 no residual, 1 residual, 2 decided at run
    // time.  The residual of row block i + RES_AHEAD - 1 is requested before row block i is worked on
    // (the whole tile's residual costs about one memory latency, not one per row block;
    // with two sets the second workgroup of a split reduction spent 46 k cycles in this epilogue, half of them
    // waiting), and the compiler may not move anything across the row-block boundaries: left alone it hoists the
    // loads and the accumulator reads of all blocks to the top, which the 256-accumulator tile has no registers for.
    auto finish = [&](auto bias_tag, auto act_tag, auto interior_tag, auto res_tag) {
    constexpr bool BIAS = decltype(bias_tag)::value, ACT = decltype(act_tag)::value, INTERIOR = decltype(interior_tag)::value;
    constexpr int RES = decltype(res_tag)::value;
    const bool res = RES == 2 ? has_res : RES == 1;
    constexpr int AHEAD = PARTNER ? 3 : 5, RES_AHEAD = TM < AHEAD ? TM : AHEAD;
    bf16x4 rv[RES_AHEAD][TNO];
    int rrow[TM];                                          // where the residual's rows come from
    if (res) map_rows_near(p.rmap, p.seq_len, rows, b0, rrow);
    auto load_res = [&](int i, int buf) {
        const bf16_t *r = p.residual + (int64_t)(INTERIOR || rows[i] >= 0 ? rrow[i] : 0) * p.ldres + gcol0 + c0;
#pragma unroll
        for (int j = 0; j < TNO; ++j) {
            const int c = epi_col<TNO>(j, g);
            if (INTERIOR && (j | 1) < TNO) {               // a pair of blocks in one read
                if (j & 1) continue;
                const bf16x8 v = *(const bf16x8 *)(r + c);
                rv[buf][j] = bf16x4{v[0], v[1], v[2], v[3]};
                rv[buf][j + 1 < TNO ? j + 1 : j] = bf16x4{v[4], v[5], v[6], v[7]};
            } else if (INTERIOR) rv[buf][j] = *(const bf16x4 *)(r + c);
            else {
                rv[buf][j] = bf16x4{0, 0, 0, 0};
                if (rows[i] >= 0 && c0 + c < seg_rows) rv[buf][j] = *(const bf16x4 *)(r + c);
            }
        }
    };
    // the bias of this lane's columns, once (it does not depend on the row block)
    f32x4 bias_v[BIAS ? TNO : 1];
    if constexpr (BIAS) {
#pragma unroll
        for (int j = 0; j < TNO; ++j) {
            const int c = c0 + epi_col<TNO>(j, g);
            bias_v[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (bias && c < seg_rows) {
                const bf16x4 b4 = *(const bf16x4 *)(bias + c);
                bias_v[j] = f32x4{(float)b4[0], (float)b4[1], (float)b4[2], (float)b4[3]};
            }
        }
    }
    // the partner's accumulators, three row blocks ahead like the residual
    constexpr int P_AHEAD = PARTNER ? (TM < 3 ? TM : 3) : 1;
    f32x4 pvv[P_AHEAD][PARTNER ? TNO : 1];
    auto load_part = [&](int i) {
        if constexpr (PARTNER)
#pragma unroll
            for (int j = 0; j < TNO; ++j) pvv[i % P_AHEAD][j] = __builtin_nontemporal_load(part + (i * TN + j) * NTHREADS);
    };
    if constexpr (PARTNER)
#pragma unroll
        for (int i = 0; i < P_AHEAD - 1 && i < TM; ++i) load_part(i);
    if (res)
#pragma unroll
        for (int i = 0; i < RES_AHEAD - 1 && i < TM; ++i) load_res(i, i % RES_AHEAD);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if (PARTNER && i + P_AHEAD - 1 < TM) load_part(i + P_AHEAD - 1);
        if (res && i + RES_AHEAD - 1 < TM) load_res(i + RES_AHEAD - 1, (i + RES_AHEAD - 1) % RES_AHEAD);
        bf16_t *y = p.Y + (int64_t)(INTERIOR || rows[i] >= 0 ? yrow[i] : 0) * p.ldy + gcol0 + c0;
        __builtin_amdgcn_sched_barrier(0);
        bf16x4 before = {};
#pragma unroll
        for (int j = 0; j < TNO; ++j) {
            f32x4 v = acc_load(acc[i][j]);
            if constexpr (PARTNER) v += pvv[i % P_AHEAD][j];
            // the residual is added before the one rounding to bf16
            const bf16x4 r4 = res ? rv[i % RES_AHEAD][j] : bf16x4{0, 0, 0, 0};
            if constexpr (SWIGLU) {
                const f32x4 up = acc_load(acc[i][j + TNO]);
                // (one rounding for product and sum, written out so that every copy of this loop has it)
#pragma unroll
                for (int x = 0; x < 4; ++x) v[x] = res ? fmaf(silu_fast(v[x]), up[x], (float)r4[x]) : silu_fast(v[x]) * up[x];
            } else {
                if constexpr (BIAS) v += bias_v[j];
                if constexpr (ACT)
#pragma unroll
                    for (int x = 0; x < 4; ++x) v[x] = apply_act_bf16(v[x], flags);
                if (res)
#pragma unroll
                    for (int x = 0; x < 4; ++x) v[x] += (float)r4[x];
            }
            const bf16x4 o = to_bf16x4(v);
            const int c = epi_col<TNO>(j, g);
            if (INTERIOR && (j | 1) < TNO) {
                if (j & 1) *(bf16x8 *)(y + c - 4) = join8(before, o);
                before = o;
            } else if (INTERIOR || (rows[i] >= 0 && c0 + c < seg_rows)) *(bf16x4 *)(y + c) = o;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (RES == 2) wait_conditional_loads();
    };
    if constexpr (PARTNER) {
        // One wavefront polls and acquires (an acquire invalidates a whole L2); the workgroup barrier orders the
        // other wavefronts' loads behind it.  The partner holds its ticket already: it is running and waits for
        // nothing, so the wait ends (the spin count only guards against a partner that died).
        if (tid == 0) {
            int spins = 0;
            while (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != use && ++spins < (1 << 22))
                __builtin_amdgcn_s_sleep(8);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
    }
    const std::true_type yes;
    const std::false_type no;
    const std::integral_constant<int, 0> res_no;
    const std::integral_constant<int, 1> res_yes;
    const std::integral_constant<int, 2> res_rt;
    if constexpr (ACT_OK && !SWIGLU)
        if (act) {
            if (interior && !has_res) finish(yes, yes, yes, res_no);
            else finish(yes, yes, no, res_rt);
            return;
        }
    if constexpr (!SWIGLU && !PARTNER)
        if (bias && interior) {
            if (has_res) finish(yes, no, yes, res_yes);
            else finish(yes, no, yes, res_no);
            return;
        }
    if (!interior || bias) finish(std::bool_constant<!SWIGLU>{}, no, no, res_rt);
    else if (has_res) finish(no, no, yes, res_yes);
    else finish(no, no, yes, res_no);
}

// Tile number -> tile coordinates.  Row tiles run fastest inside groups of 8 rows of tiles, column tiles next, groups
// last: the 32 consecutive tiles an XCD works on at a time are then 8 row tiles x 4 column tiles (every activation
// tile shared by 4 workgroups through the XCD's L2, every weight tile by 8), however many rows of tiles the
// launch has; with up to 8 rows of tiles this is the plain row-fastest order.
__device__ __forceinline__ void tile_coords(int tile, int tiles_m, int tiles_n, int &tile_m, int &tile_n) {
    constexpr int GM = 8;                                  // 16 and 4 measured 1 % slower at 32 rows of tiles
    const int width = GM * tiles_n, group = tile / width, first_m = group * GM;
    const int gsz = min(tiles_m - first_m, GM), in_group = tile - group * width;
    tile_m = first_m + in_group % gsz;
    tile_n = in_group / gsz;
}

template <int N>
__device__ __forceinline__ void wait_loads_and_barrier() {
    // all but the N youngest vector-memory operations of this wavefront are complete and its LDS reads
    // have returned, then barrier
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// MFMA with the accumulator tied to the destination and held in the accumulation registers.  Used by
// the one-wavefront-per-SIMD schedule, where the 224-256 accumulator registers of a 128-row wavefront
// tile only fit there; written as assembly so that source and destination stay the same registers and
// so that the hand-placed operand reads and tile loads keep their place between the MFMAs (the
// compiler does not move memory operations across these statements).
__device__ __forceinline__ void mfma_tied(f32x4 &c, const bf16x8 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
// The compiler does not see those MFMAs: before anything else reads the accumulators, let the last
// ones leave the matrix pipeline.
__device__ __forceinline__ void mfma_drain() { asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory"); }

// The lane number from the execution mask, as assembly: the compiler can neither tell that it is threadIdx.x % 64
// nor merge two of these, so nothing is kept in a register between them.
__device__ __forceinline__ int lane_id_again() {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// Reduction split over two workgroups per tile (a launch whose tiles would fill half of the CUs).  Each computes
// one half of K into its accumulators.  Then it takes a ticket from the tile's counter: the holder of the even
// ticket (the first to finish) writes its accumulators to the tile's slot of the scratch as they lie in its
// registers, publishes them by setting the tile's flag to the use count of the slot (returned in `use`), and is
// done; the holder of the odd ticket returns true: it runs the epilogue, which waits for that flag and adds the
// stored accumulators to its own.  The workgroup that is waited for took its ticket earlier, so it is running, has its main loop
// behind it and waits for nothing itself: the wait ends whatever the order in which workgroups are placed on the
// CUs (the spin count only guards against a partner that died).  Ticket and flag count up over the launches that
// share the words (which run one after the other), so nothing has to be reset between them.
template <int TM, int TN, int NTHREADS>
__device__ __forceinline__ bool splitk_combine(const Gemm2Params &p, f32x4 (&acc)[TM][TN], int tile, int tid,
                                               unsigned char *smem, uint32_t &use_out) {
    uint32_t *sync = p.sk_sync + 2 * tile;
    f32x4 *part = (f32x4 *)p.planes + (size_t)tile * (TM * TN * NTHREADS) + tid;
    volatile uint32_t *sh = (volatile uint32_t *)smem;
    if (tid == 0) sh[0] = __hip_atomic_fetch_add(&sync[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const uint32_t ticket = sh[0];
    const uint32_t use = (ticket >> 1) + 1;
    use_out = use;
    // Cache maintenance across the XCDs' L2s is expensive (a release writes back, an acquire invalidates a whole
    // L2), so exactly one wavefront of each workgroup does it: the workgroup barrier orders the other wavefronts'
    // stores before thread 0's release and their loads after thread 0's acquire.
    if ((ticket & 1u) == 0u) {
        // stored straight from the accumulation registers (a vector-memory instruction takes them as data): this
        // runs once, on the path the other workgroup waits for, and 256 register moves less is a third of it
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                asm volatile("global_store_dwordx4 %0, %1, off" ::"v"(part + (i * TN + j) * NTHREADS), "a"(acc[i][j]) : "memory");
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the compiler does not count those stores
        __syncthreads();
        if (tid == 0) __hip_atomic_store(&sync[1], use, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        return false;
    }
    return true;
}

// Reduction split over p.parts workgroups per tile without an exchange between them: each leaves its fp32 sums in
// plane `part` of the scratch, [part][row][column], and splitk_finish_kernel adds the planes.  Straight from the
// accumulation registers, 16 rows x 64 bytes per instruction.
template <int TM, int TN>
__device__ __forceinline__ void store_partial(const Gemm2Params &p, f32x4 (&acc)[TM][TN], int lane, int row0, int col0, int part,
                                              bool inside, int seg) {
    const int n = p.seg_rows[seg], width = p.planes_ld, col = col0 + 4 * (lane >> 4);
    float *dst = p.planes + ((size_t)part * p.M + row0 + (lane & 15)) * width + p.seg_col0[seg] + col;
    auto store = [&](auto inside_tag) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const bool row_ok = decltype(inside_tag)::value || row0 + 16 * i + (lane & 15) < p.M;
#pragma unroll
            for (int j = 0; j < TN; ++j)
                if (row_ok && (decltype(inside_tag)::value || col + 16 * j < n))
                    asm volatile("global_store_dwordx4 %0, %1, off offset:%2" ::"v"(dst), "a"(acc[i][j]), "n"(64 * j) : "memory");
            dst += 16 * (size_t)width;
        }
    };
    if (inside) store(std::true_type{});
    else store(std::false_type{});
}

template <int BM, int BN, int WM, int WN, int BK, int NST, bool SWIGLU, bool ROPE = false, int SPLIT = SPLIT_NONE>
__global__ __launch_bounds__(WM *WN * 64) void gemm2_kernel(Gemm2Params p) {
    static_assert(!ROPE || (!SWIGLU && WM * WN == 4), "rotary epilogue: plain GEMM, one wavefront per SIMD");
    constexpr bool PAIR = SPLIT == SPLIT_PAIR, PARTS = SPLIT == SPLIT_PARTS, SPLITS = PAIR || PARTS;
    static_assert(!SPLITS || (!SWIGLU && !ROPE && WM * WN == 4), "split reduction: plain GEMM, one wavefront per SIMD");
    constexpr int NW = WM * WN;
    constexpr int WTM = BM / WM, WTN = BN / WN;
    constexpr int TM = WTM / 16, TN = WTN / 16;
    constexpr bool SOLO = NW == 4;                                 // one wavefront per SIMD, up to 512 registers
    constexpr int ROWB = BK * 2;                                   // bytes per tile row in LDS
    constexpr int RPI = 1024 / ROWB;                               // tile rows per direct-to-LDS instruction
    constexpr int CPR = ROWB / 16;                                 // 16-byte chunks per row
    constexpr int BNP = (BN + RPI * NW - 1) / (RPI * NW) * (RPI * NW);   // B rows held in LDS (BN rounded up)
    constexpr int A_INSTR = BM / RPI / NW, B_INSTR = BNP / RPI / NW;     // direct-to-LDS instructions per wavefront
    constexpr int LPT = A_INSTR + B_INSTR;                         // loads per tile per wavefront
    constexpr int A_BYTES = BM * ROWB, STAGE_BYTES = (BM + BNP) * ROWB;
    constexpr int STG_LD = WTN + 4;                                // widest epilogue staging row (floats)
    // One wavefront per SIMD and many blocks: the gaps between MFMAs hold one memory instruction and little else (see the
    // main loop), so loads share their LDS address by fours.
    constexpr bool WIDE = SOLO && TM * TN >= 32;
    static_assert(BK == 64, "rows of 128 bytes: two k-steps of an MFMA, and the swizzle below");
    static_assert(NST == 2 || (SOLO && NST == 3), "pipeline depth");
    static_assert(SOLO || !SWIGLU, "SwiGLU: one wavefront per SIMD");
    static_assert(BM % (RPI * NW) == 0, "tile rows must split over the wavefronts");
    static_assert(WTN % 16 == 0 && (SOLO || WTN <= 128) && BN % RPI == 0, "wavefront tile: whole MFMA blocks, at most 128 columns");
    static_assert(!SWIGLU || ((WTN / 2) % RPI == 0 && (WTN / 2) % 4 == 0),
                  "a load instruction / a store chunk must not straddle gate and up rows");
    static_assert(SOLO || NW * 16 * STG_LD * 4 <= NST * STAGE_BYTES, "epilogue staging must fit in the tile buffers");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave / WN) * WTM, wn0 = (wave % WN) * WTN;

    // workgroup -> tile: a contiguous run of the tile list per XCD (see tile_coords for the order of the list)
    // One wavefront per SIMD: the workgroup is persistent.  The launch has one workgroup per CU (a multiple of 8)
    // and workgroup w takes the tiles that workgroups w, w + gridDim.x, ... of a launch with one workgroup per
    // tile would take: nothing waits for a workgroup's last stores to be acknowledged, for its registers and LDS
    // to be handed on, or for a new workgroup to set itself up; the stores of a tile drain while the first
    // tile loads of the next are in flight.
    constexpr bool PERSISTENT = SOLO && !SPLITS;
    const int total = p.tiles_m * p.tiles_n * (SPLITS ? p.parts : 1);
    for (int pid = blockIdx.x;; pid += gridDim.x) {
    int tile;
    {
        const int xcd = pid & 7, idx = pid >> 3;
        const int base = total >> 3, rem = total & 7;
        tile = xcd * base + min(xcd, rem) + idx;
    }
    int tile_m, tile_n, part = 0;
    if constexpr (PAIR) {                                          // the two halves of a tile are neighbours, on one XCD
                                                                   // but where an XCD's run of the list starts or ends between them
        part = tile & 1;
        tile >>= 1;
    } else if constexpr (PARTS) {                                  // parts slowest: an XCD works on one or two of them
        part = tile / (p.tiles_m * p.tiles_n);                     // and reads that much less of the activations
        tile -= part * p.tiles_m * p.tiles_n;
    }
    tile_coords(tile, p.tiles_m, p.tiles_n, tile_m, tile_n);
    const int seg = tile_n >= p.seg_tile0[2] ? 2 : tile_n >= p.seg_tile0[1] ? 1 : 0;
    const int m0 = tile_m * BM;
    constexpr int BN_OUT = SWIGLU ? BN / 2 : BN;
    const int nloc0 = (tile_n - p.seg_tile0[seg]) * BN_OUT;
    const int seg_rows = p.seg_rows[seg];
    const int K = p.K;

    const __amdgpu_buffer_rsrc_t rx = tile_buffer<WIDE>(p.X, p.x_bytes);
    const uint32_t w_bytes = (uint32_t)((int64_t)seg_rows * K * 2);
    const __amdgpu_buffer_rsrc_t rw = tile_buffer<WIDE>(p.W[seg], w_bytes);
    const __amdgpu_buffer_rsrc_t ru = tile_buffer<WIDE>(SWIGLU ? p.Wup : p.W[seg], w_bytes);

    // ---- per-lane global offsets of the direct-to-LDS loads.  Instruction i of this wavefront fills
    // tile rows wave*(rows/NW) + RPI*i .. : lane -> row lane/CPR, LDS slot lane%CPR, which must hold the
    // logical chunk slot ^ swizzle(row).
    auto swz = [](int row) { return (row >> 1) & 7; };
    constexpr bool PAIRED = SOLO && !PARTS;                        // blocks hold the columns epi_col says
    constexpr int TNO = SWIGLU || ROPE ? TN / 2 : TN;              // blocks of gate, up, first or second halves
    uint32_t a_off[A_INSTR], b_off[B_INSTR];
#pragma unroll
    for (int i = 0; i < A_INSTR; ++i) {
        const int row = wave * (BM / NW) + RPI * i + lane / CPR;
        const int c = (lane % CPR) ^ swz(row);
        const int gm = m0 + row;
        a_off[i] = gm < p.M ? load_off<WIDE>((uint32_t)(map_row_near(p.xmap, p.seq_len, gm, m0 / p.seq_len) * p.ldx * 2) + c * 16, i) : OOB_OFF;
    }
#pragma unroll
    for (int i = 0; i < B_INSTR; ++i) {
        const int row = wave * (BNP / NW) + RPI * i + lane / CPR;
        const int c = (lane % CPR) ^ swz(row);
        int col;
        auto order = [](int r) { return PAIRED ? epi_row_col<TNO>(r) : r; };
        if (SWIGLU) col = nloc0 + (row / WTN) * (WTN / 2) + order(row % (WTN / 2));
        else if (ROPE) {                                           // tile row -> rotation pair and half of it
            const int rr = row % WTN, hs = rr / (WTN / 2);
            const int pp = (nloc0 >> 1) + (row / WTN) * (WTN / 2) + order(rr % (WTN / 2));
            const int lh = p.rope_lh;
            col = pp < (seg_rows >> 1) ? ((pp >> lh) << (lh + 1)) + (pp & ((1 << lh) - 1)) + (hs << lh) : seg_rows;
        } else col = nloc0 + row / WTN * WTN + order(row % WTN);
        b_off[i] = (row < BN && col < seg_rows) ? load_off<WIDE>((uint32_t)((int64_t)col * K * 2) + c * 16, i) : OOB_OFF;
    }

    // LDS layout.  8 wavefronts: NST stages of [A tile | B tile].  One wavefront per SIMD: three A stages
    // followed by two B stages (the A part of a refill is issued half a tile earlier than the B part, so the
    // vector-memory instructions are spread over both k-steps; that needs the third A stage).
    constexpr int B_BYTES = BNP * ROWB;
    constexpr int NSTA = NST + 1, NSTB = NST;
    auto a_stage = [&](int kt) { return SOLO ? (kt % NSTA) * A_BYTES : (kt % NST) * STAGE_BYTES; };   // LDS offsets
    auto b_stage = [&](int kt) { return SOLO ? NSTA * A_BYTES + (kt % NSTB) * B_BYTES : (kt % NST) * STAGE_BYTES + A_BYTES; };
    const int kt_first = SPLITS ? (int)((int64_t)part * (K / BK) / p.parts) : 0;
    const int KT = SPLITS ? (int)((int64_t)(part + 1) * (K / BK) / p.parts) - kt_first : K / BK;   // of this workgroup
    if constexpr (SPLITS) {                                        // (offsets of rows outside stay outside: K bytes < 2^31)
        const uint32_t koff = (uint32_t)kt_first * ROWB;
#pragma unroll
        for (int i = 0; i < A_INSTR; ++i) a_off[i] += koff;
#pragma unroll
        for (int i = 0; i < B_INSTR; ++i) b_off[i] += koff;
    }
    // instruction x of LPT of a k-tile: k offset in bytes, LDS offsets of its A and B stages
    auto issue_load = [&](uint32_t kb, int sa, int sb, int x) {    // (x known after unrolling)
        if (x < A_INSTR) load16_to_lds<WIDE>(rx, smem + sa + wave * (BM / NW) * ROWB, x, a_off[x], kb);
        else {
            const int i = x - A_INSTR, row0 = wave * (BNP / NW) + RPI * i;           // wavefront-uniform
            const bool up = SWIGLU && ((row0 % WTN) >= WTN / 2);
            if (up) load16_to_lds<WIDE>(ru, smem + sb + wave * (BNP / NW) * ROWB, i, b_off[i], kb);
            else load16_to_lds<WIDE>(rw, smem + sb + wave * (BNP / NW) * ROWB, i, b_off[i], kb);
        }
    };
    auto issue_loads = [&](int kt) {
#pragma unroll
        for (int x = 0; x < LPT; ++x) issue_load((uint32_t)kt * ROWB, a_stage(kt), b_stage(kt), x);
    };

    f32x4 acc[TM][TN];

    // operand fetch: lane -> tile row lane%16 of a 16-row block, chunk 4 ks + lane/16, swizzled
    const int frow = lane & 15, fch = lane >> 4, fsw = swz(lane & 15);
    const int a_lane = (wm0 + frow) * ROWB, b_lane = A_BYTES + (wn0 + frow) * ROWB;
    constexpr int NSETS = SOLO || 4 * TM * TN + 8 * (TM + TN) <= 216 ? 2 : 1;
    bf16x8 af[NSETS][TM], bfr[NSETS][TN];
    auto fetch_into = [&](int kt, auto set_tag, auto ks_tag) {   // operands of k-step ks of tile kt -> register set
        constexpr int set = decltype(set_tag)::value, ks = decltype(ks_tag)::value;
        const unsigned char *st = smem + (kt % NST) * STAGE_BYTES;
        const int coff = ((4 * ks + fch) ^ fsw) * 16;
#pragma unroll
        for (int i = 0; i < TM; ++i) af[set][i] = *(const bf16x8 *)(st + a_lane + i * 16 * ROWB + coff);
#pragma unroll
        for (int j = 0; j < TN; ++j) bfr[set][j] = *(const bf16x8 *)(st + b_lane + j * 16 * ROWB + coff);
    };
    auto mfmas = [&](auto ks_tag) {
        constexpr int ks = decltype(ks_tag)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[ks][i], bfr[ks][j], acc[i][j], 0, 0, 0);
    };
    // 8 wavefronts: tile kt has landed once no load is outstanding; the wavefront's own LDS reads have returned
    // (they were of the tile whose stage is refilled next); after the barrier every wavefront is done reading tile kt-1.
    auto tile_ready = [&](int kt) {
        wait_loads_and_barrier<0>();
        if (kt + 1 < KT) issue_loads(kt + 1);
    };
    const std::integral_constant<int, 0> k0;
    const std::integral_constant<int, 1> k1;
#pragma unroll
    for (int s = 0; s < NST - 1; ++s)
        if (s < KT) issue_loads(s);
    // One wavefront per SIMD: its A and B stages hold NST tiles besides the one being multiplied, so the NST-th
    // k-tile is requested right behind the others (requested only once the first had landed, its latency sat in
    // front of the first barrier of every output tile).
    if constexpr (SOLO)
        if (NST - 1 < KT) issue_loads(NST - 1);
    // (the accumulators are cleared while the first tile loads are in flight: up to 256 register writes)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    __builtin_amdgcn_sched_barrier(0);
    // Software pipeline over k-steps: the LDS reads of a k-step are in flight while the MFMAs of the
    // previous k-step run, also across the tile boundary (the second k-step of tile kt is multiplied
    // after the barrier that opens tile kt+1, from registers).  It needs two operand register sets;
    // the widest tile (256 columns: 128 accumulator + 96 operand registers) would spill with them and
    // keeps one k-step's reads directly ahead of its own MFMAs instead.
    constexpr bool PIPE = 4 * TM * TN + 8 * (TM + TN) <= 216;
    if constexpr (SOLO) {                                          // tile 0 has landed; the others may be on their way
        if (NST - 1 < KT) wait_loads_and_barrier<(NST - 1) * LPT>();
        else wait_loads_and_barrier<0>();
    } else tile_ready(0);
    if constexpr (SOLO) {
        // One wavefront per SIMD: nothing else covers this wavefront's waits, so every memory operation
        // is placed between two MFMAs of the k-step that runs meanwhile.  Tile kt, first k-step: its
        // MFMAs with the operand reads of the second k-step (the last of them early enough to have returned at
        // the barrier) and the A loads of tile kt+2 (into the A stage tile kt-1 left)
        // between them.  Barrier (tile kt+1 landed: everything but those A loads; everyone is done reading
        // tile kt).  Second k-step: its MFMAs with the B loads of tile kt+2 (into the B stage tile kt just
        // left) and the operand reads of tile kt+1's first k-step between them.
        // NST = P: the tile requested is kt + P.
        // Where they go: a 16-cycle MFMA leaves room to issue two instructions (a buffer load counts for both); what does not
        // fit in the gap behind it keeps the next one waiting.  So the operand reads and the A loads go evenly over three quarters
        // of a k-step's MFMAs, the B loads (whose tile is waited for half a tile earlier) over 3/8, where they share no gap
        // with reads in the widest tile; stage offsets are rotated from tile to tile instead of computed from the tile's
        // number, four loads share a write of m0, and there is one wait for the reads of a k-step.  Cycles per k-tile of 256 x
        // 256 x 64 (2048 of MFMA issue; a tile's start and end counted in): 2566 with a read per two MFMAs and a load per two at
        // the front of the k-step and vector additions for their offsets, 2436 spread.
        // 8192 x 4096 x 14336 with residual 672 us at first, spread 658, all 643; 8192 x 6144 x 4096 294 / 289 / 280; SwiGLU
        // 8192 x 14336 x 4096 1339 / 1306 / 1276, 2048 rows 358 / 347 / 337; 4096 x 768 x 3072 with bias and residual 25.9 / 24.7 / 23.4.
        // Reads over half to 7/8 and loads over 3/8 to 15/16 of the MFMAs are within 0.5 % of this.
        constexpr int NR = TM + TN, NM = TM * TN;
        constexpr int RSPAN = NM * 3 / 4 > NR ? NM * 3 / 4 : NR;
        constexpr int ASPAN = NM * 3 / 4 > A_INSTR ? NM * 3 / 4 : A_INSTR, BSPAN = NM * 3 / 8 > B_INSTR ? NM * 3 / 8 : B_INSTR;
        static_assert(RSPAN <= NM && ASPAN < NM && BSPAN < NM, "a k-step has room for its reads and loads");
        auto nth = [](int x, int n, int span) {                 // which of n operations over `span` MFMAs follows MFMA x (-1: none)
            const int r = (x * n + span - 1) / span;
            return x >= 0 && r < n && r * span / n == x ? r : -1;
        };
        auto read_at = [&](int x) { return nth(x, NR, RSPAN); };
        auto a_load_at = [&](int x) { return nth(x - 1, A_INSTR, ASPAN); };
        auto b_load_at = [&](int x) { return nth(x - 1, B_INSTR, BSPAN); };
        // LDS offsets of the stages, rotated from tile to tile: ast[0 .. NST] of the A parts of tiles kt .. kt + NST (the
        // last one's is the stage that tile kt - 1 has left), bst[0 .. NST - 1] of the B parts of kt .. kt + NST - 1.
        int ast[NSTA], bst[NSTB];
#pragma unroll
        for (int x = 0; x < NSTA; ++x) ast[x] = x * A_BYTES;
#pragma unroll
        for (int x = 0; x < NSTB; ++x) bst[x] = NSTA * A_BYTES + x * B_BYTES;
        auto rotate = [&]() {
            const int a0 = ast[0], b0 = bst[0];
#pragma unroll
            for (int x = 0; x + 1 < NSTA; ++x) ast[x] = ast[x + 1];
#pragma unroll
            for (int x = 0; x + 1 < NSTB; ++x) bst[x] = bst[x + 1];
            ast[NSTA - 1] = a0;
            bst[NSTB - 1] = b0;
        };
        const int a_ks[2] = {(wm0 + frow) * ROWB + (fch ^ fsw) * 16, (wm0 + frow) * ROWB + ((4 + fch) ^ fsw) * 16};
        const int b_ks[2] = {(wn0 + frow) * ROWB + (fch ^ fsw) * 16, (wn0 + frow) * ROWB + ((4 + fch) ^ fsw) * 16};
        auto fetch_one = [&](int sa, int sb, auto ks_tag, int r) {   // read r of a k-step: A block 0, the B blocks, the other A blocks
            constexpr int ks = decltype(ks_tag)::value;
            if (r == 0) af[ks][0] = *(const bf16x8 *)(smem + (sa + a_ks[ks]));
            else if (r <= TN) bfr[ks][r - 1] = *(const bf16x8 *)(smem + (sb + b_ks[ks]) + (r - 1) * 16 * ROWB);
            else af[ks][r - TN] = *(const bf16x8 *)(smem + (sa + a_ks[ks]) + (r - TN) * 16 * ROWB);
        };
        uint32_t kb = NST * ROWB;                              // k offset of tile kt + NST
        // Every read of a k-step has returned when the next one begins: said once, or the compiler waits in front of every
        // MFMA that is the first to use one.  (Few blocks: the last reads have not returned yet, and only theirs wait.)
        auto reads_done = [&]() { if (NM >= 32) __builtin_amdgcn_s_waitcnt(0xc07f); };   // lgkmcnt(0)
        auto phase = [&](auto ks_tag, auto &&between) {        // the MFMAs of one k-step; between(x) follows MFMA x
            constexpr int ks = decltype(ks_tag)::value;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    mfma_tied(acc[i][j], bfr[ks][j], af[ks][i]);     // transposed: lane = row, 4 columns
                    between(i * TN + j);
                }
        };
#pragma unroll
        for (int r = 0; r < NR; ++r) fetch_one(ast[0], bst[0], k0, r);
        int kt = 0;
        reads_done();
        auto k_tile = [&](auto younger_tag, auto load_tag) {   // one tile but the last; YOUNGER loads may be outstanding at its barrier
            constexpr int YOUNGER = decltype(younger_tag)::value;
            constexpr bool LOAD = decltype(load_tag)::value;
            phase(k0, [&](int x) {
                if (read_at(x) >= 0) fetch_one(ast[0], bst[0], k1, read_at(x));
                if (LOAD && a_load_at(x) >= 0) issue_load(kb, ast[NST], 0, a_load_at(x));
            });
            reads_done();
            wait_loads_and_barrier<YOUNGER>();
            phase(k1, [&](int x) {
                if (LOAD && b_load_at(x) >= 0) issue_load(kb, 0, bst[0], A_INSTR + b_load_at(x));
                if (read_at(x) >= 0) fetch_one(ast[1], bst[1], k0, read_at(x));
            });
            reads_done();
            rotate();
            kb += ROWB;
            ++kt;
        };
        const std::true_type load;
        const std::false_type no_load;
        while (kt + NST < KT) k_tile(std::integral_constant<int, (NST - 2) * LPT + A_INSTR>{}, load);   // tiles kt+1 .. kt+NST-1 are in flight or landed
        // the last tiles but one: nothing left to load, one tile fewer in flight at each
        if constexpr (NST == 3)
            if (KT - 2 - kt == 1) k_tile(std::integral_constant<int, LPT>{}, no_load);
        if (KT - 2 - kt == 0) k_tile(std::integral_constant<int, 0>{}, no_load);
        phase(k0, [&](int x) { if (read_at(x) >= 0) fetch_one(ast[0], bst[0], k1, read_at(x)); });
        reads_done();
        phase(k1, [&](int) {});
        mfma_drain();
    } else if constexpr (PIPE) {
        auto fetch = [&](int kt, auto ks_tag) { fetch_into(kt, ks_tag, ks_tag); };   // k-step ks -> register set ks
        fetch(0, k0);
        for (int kt = 0; kt + 1 < KT; ++kt) {              // straight-line body: the last tile is peeled
            fetch(kt, k1);
            __builtin_amdgcn_sched_barrier(0);             // reads stay ahead of the MFMAs they overlap with
            mfmas(k0);
            __builtin_amdgcn_sched_barrier(0);
            tile_ready(kt + 1);
            fetch(kt + 1, k0);
            __builtin_amdgcn_sched_barrier(0);
            mfmas(k1);
            __builtin_amdgcn_sched_barrier(0);
        }
        fetch(KT - 1, k1);
        __builtin_amdgcn_sched_barrier(0);
        mfmas(k0);
        mfmas(k1);
    } else {
        for (int kt = 0; kt < KT; ++kt) {
            if (kt > 0) tile_ready(kt);
            fetch_into(kt, k0, k0);
            mfmas(k0);
            fetch_into(kt, k0, k1);
            mfmas(k0);
        }
    }

    if constexpr (PARTS) {
        store_partial<TM, TN>(p, acc, lane, m0 + wm0, nloc0 + wn0, part, m0 + BM <= p.M && nloc0 + BN <= seg_rows, seg);
        return;
    }
    if constexpr (SOLO) {
        // The thread index computed again (the lane number from the execution mask, so that the compiler cannot
        // tell it is tid): otherwise everything the epilogue derives from it is computed once, ahead of the tile
        // loop, and kept in registers across the main loop, which has none to spare.
        int tid_e = wave * 64 + lane_id_again();
        KernelArgs &q = params_again();
        if constexpr (PAIR) {
            uint32_t use;
            __syncthreads();                               // everyone is done with the tile buffers (the ticket goes through LDS)
            if (!splitk_combine<TM, TN, NW * 64>(p, acc, tile, tid_e, smem, use)) return;
            tid_e = wave * 64 + lane_id_again();
            gemm_epilogue_direct<NW * 64, TM, TN, WTN, false, false, true>(
                q, acc, tid_e, m0, wm0, wn0, nloc0, seg, seg_rows,
                (const f32x4 *)p.planes + (size_t)tile * (TM * TN * NW * 64) + tid_e, p.sk_sync + 2 * tile + 1, use);
            return;
        }
        if constexpr (ROPE)
            gemm_epilogue_rope<TM, TN, WTN>(q, acc, tid_e & 63, m0, wm0, wn0, nloc0 >> 1, seg, seg_rows);
        else
            // tiles of up to 48 accumulator blocks take GELU launches: with more of them the compiler no longer
            // unrolls the (long) activation code and would index the accumulators through memory
            gemm_epilogue_direct<NW * 64, TM, TN, WTN, SWIGLU, TM * TN <= 48>(q, acc, tid_e, m0, wm0, wn0, nloc0, seg, seg_rows);
    } else {
        __syncthreads();                                   // everyone is done with the tile buffers
        gemm_epilogue<TM, TN, WTN>(p, acc, smem, wave, lane, m0, wm0, wn0, nloc0, seg, seg_rows);
    }
    if (!PERSISTENT || pid + (int)gridDim.x >= total) break;
    __syncthreads();                                       // everyone is done with the tile buffers: the next tile may load
    }
}

static int cu_count() {                                   // of the current device
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
        n = 256;
    return n;
}

template <int BM, int BN, int WM, int WN, int BK, int NST, bool SWIGLU, bool ROPE = false, int SPLIT = SPLIT_NONE>
static int32_t launch_cfg2(const GemmArgs &a, hipStream_t s, int parts = 1) {
    Gemm2Params p;
    p.planes = a.planes; p.sk_sync = a.sk_sync; p.parts = parts; p.planes_ld = a.N;
    p.rope_table = a.rope_table; p.rope_cols = a.rope_cols; p.rope_lh = 0;
    if (ROPE) {
        while ((2 << p.rope_lh) < a.rope_head_dim) ++p.rope_lh;
        if ((uintptr_t)a.rope_table % 16) return CASCADE_EINVAL;
    }
    constexpr int BN_OUT = SWIGLU ? BN / 2 : BN;
    int col0 = 0, tile0 = 0;
    for (int i = 0; i < 3; ++i) {
        int end = a.seg_end[i];
        int rows = std::max(0, end - col0);
        p.W[i] = (const bf16_t *)a.W[i];
        p.bias[i] = (const bf16_t *)a.bias[i];
        p.seg_rows[i] = rows;
        p.seg_col0[i] = col0;
        p.seg_tile0[i] = rows ? tile0 : INT32_MAX;
        tile0 += (rows + BN_OUT - 1) / BN_OUT;
        col0 = std::max(col0, end);
        if ((int64_t)rows * a.K * 2 >= (int64_t)MAX_BYTES) return CASCADE_EUNSUPPORTED;
    }
    if (p.seg_tile0[0] == INT32_MAX) return CASCADE_ESHAPE;
    p.X = (const bf16_t *)a.X; p.Wup = (const bf16_t *)a.W_up; p.residual = (const bf16_t *)a.residual;
    p.Y = (bf16_t *)a.Y;
    p.M = a.M; p.K = a.K;
    p.tiles_m = (a.M + BM - 1) / BM; p.tiles_n = tile0;
    p.ldx = a.ldx; p.ldy = a.ldy; p.ldres = a.ldres;
    p.xmap = a.xmap.map; p.ymap = a.ymap.map; p.rmap = a.rmap.map;
    p.seq_len = a.xmap.map ? a.xmap.seq_len : a.ymap.map ? a.ymap.seq_len : a.rmap.map ? a.rmap.seq_len : 1;
    p.flags = a.epilogue;
    int64_t xb = (int64_t)a.M * a.ldx * 2;
    if (xb >= (int64_t)MAX_BYTES) return CASCADE_EUNSUPPORTED;
    p.x_bytes = (uint32_t)xb;
    constexpr int LOAD_ROWS = 1024 / (BK * 2) * WM * WN;                  // B rows loaded per pass of all wavefronts
    constexpr int BNP = (BN + LOAD_ROWS - 1) / LOAD_ROWS * LOAD_ROWS;
    constexpr size_t lds_loop = (size_t)NST * (BM + BNP) * BK * 2;
    constexpr size_t lds_solo = (size_t)((NST + 1) * BM + NST * BNP) * BK * 2;   // one A stage more than B stages
    constexpr size_t lds = WM * WN == 4 ? lds_solo : lds_loop;
    static_assert(lds <= 160 * 1024, "tile buffers exceed the LDS of a CU");
    const void *kern = (const void *)gemm2_kernel<BM, BN, WM, WN, BK, NST, SWIGLU, ROPE, SPLIT>;
    static std::atomic<uint64_t> lds_ready{0};                 // one per instantiation of this launcher
    CASCADE_HIP_TRY(ensure_dynamic_lds(kern, (int)lds, lds_ready));
    int64_t total = (int64_t)p.tiles_m * p.tiles_n * parts;
    if (total > INT32_MAX) return CASCADE_EUNSUPPORTED;
    void *args[] = {&p};
    unsigned grid = (unsigned)total;
    if (SPLIT == SPLIT_NONE && WM * WN == 4) {     // persistent workgroups, 8 | grid
        const int64_t per_round = cu_count() / 8 * 8 * (lds <= 80 * 1024 ? 2 : 1);   // workgroups LDS has room for
        if (per_round >= 8 && total > per_round) grid = (unsigned)per_round;
    }
    CASCADE_HIP_TRY(hipLaunchKernel(kern, dim3(grid), dim3(WM * WN * 64), args, lds, s));
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}

static bool v2_eligible(const GemmArgs &a) {
    if (a.K % 64 != 0 || a.K < 64 || a.ldx % 8 != 0 || a.ldy % 4 != 0 || ((a.epilogue & CASCADE_EPI_RESIDUAL) && a.ldres % 4 != 0))
        return false;
    if (((uintptr_t)a.Y | (uintptr_t)a.residual | (uintptr_t)a.bias[0] | (uintptr_t)a.bias[1] | (uintptr_t)a.bias[2]) % 8)
        return false;                                                // 8-byte pieces of output, residual and bias
    for (int i = 0; i < 3; ++i)
        if (a.seg_end[i] % 4) return false;                         // 4-column store chunks stay inside a segment
    return true;
}

// Whether this launch (a.rope_head_dim and a.rope_cols set, a.rope_table not needed yet) can rotate its output
// in the epilogue: a plain projection (bias at most) whose segments hold whole heads of a power-of-two width.
bool gemm_bf16_rope_fusable(const GemmArgs &a) {
    if (a.dtype != CASCADE_BF16 || !v2_eligible(a)) return false;
    if (a.epilogue & ~CASCADE_EPI_BIAS) return false;
    const int hd = a.rope_head_dim;
    if (hd < 16 || hd > 256 || (hd & (hd - 1)) || a.rope_cols % hd) return false;
    int col0 = 0;
    for (int i = 0; i < 3; ++i) {
        const int rows = std::max(0, a.seg_end[i] - col0);
        if (rows % hd) return false;
        col0 = std::max(col0, a.seg_end[i]);
    }
    return true;
}

// Reduction split over several workgroups per tile: which tile, into how many parts; parts = 1: not split.
// It is for launches whose tiles leave CUs idle, or fill them only with tiles that are too small to feed (a CU draws
// ~50 bytes per ns from beyond its L2, so 128 x 128 tiles need 0.55 us per 64 of K whatever their depth); the price is a
// second launch and writing and reading 4 bytes per output and part.  Measured as one layer whole (us), with the main loop as
// it was before its loads and reads were spread (both sides have got 1 to 5 % faster since).
// 128 x 128 tiles wherever two parts or more fit on the CUs: eight k-tiles to a part where there are that many (GPT-2
// small, FFN down of 3072: 128 rows in 4, 8, 16 parts 66.2 / 65.0 / 66.6, 512 rows 81.4 / 83.4 / 87.3; o of 768: 64 rows in
// 2, 4 parts 54.8 / 54.2, 512 rows 82.4 / 83.5), two parts at least (four for up to 24 tiles) and eight
// at most; up to 64 rows, where the planes are small, three k-tiles and sixteen parts (40 rows 48.1 / 47.4).  Unsplit / split: 8B 100 rows 236 / 142; width 768, 2048 rows of K 768 122.4 / 119.5, of 3072 123 /
// 115; width 2048, 1024 rows of 5632 163 / 154; width 3072, 512 rows of 8192 195 / 176, of 3072 206 / 194.
// 256 x 256 tiles for long reductions where only two parts of the small ones would fit (K 14336, 333 rows in 2 parts of
// 128 / 8 of 256: 254 / 244, 512 rows 285 / 273; but K 4096 238 / 244, 266 / 273), and where not even those do: two parts,
// 1536 x 4096 (96 tiles) of K 8192 unsplit 462 / split 470, 11008 581 / 574, 2048 x 4096 (128) of 8256 595 / 603, 11008
// 666 / 668 and more above; three, 1536 x 3072 (72) of 4096 282 / 283, 6144 370 / 354, 11008 499 / 457, 1152 x 4096 (80) of
// 6144 343 / 337; four and five, 1024 x 4096 (64) of 8192 333 / 345, 8256 392 / 393, 11008 421 / 415, 1024 x 3072 (48) of 8256
// 336 / 325.  Up to 16 rows the few-row kernel is as fast (123 / 121).  Three parts and more take 192 x 256 tiles where those
// leave a CU 5 % less to multiply (up to a quarter less, and an eighth less to load): 8B 260 rows 217.9 / 213.4, 333 232.3 /
// 227.6, 560 317.5 / 311.1, 700 349.7 / 345.7; 70B 260 rows 626 / 604, 333 650 / 622, 700 1118 / 1112.
struct SplitChoice { int tile, parts; };
static int64_t parts128(int64_t M, int64_t N, int64_t K) {
    const int64_t kt = K / 64, t128 = ((M + 127) / 128) * ((N + 127) / 128);
    return std::min({(int64_t)cu_count() / t128, kt / 3, std::max<int64_t>(t128 <= 24 ? 4 : 2, kt / (M <= 64 ? 3 : 8)),
                     (int64_t)(M <= 64 ? 16 : 8)});
}
static SplitChoice choose_split(int64_t M, int64_t N, int64_t K) {
    if (M <= 16) return {0, 1};
    const int64_t p128 = parts128(M, N, K), p256 = std::min({cu_count() / (((M + 255) / 256) * ((N + 255) / 256)), K / 64 / 3, (int64_t)16});
    if (p128 >= 3 || (p128 == 2 && K <= 8192)) return {128, (int)p128};
    if (p256 >= 2 && K >= (p256 >= 8 ? 4096 : p256 >= 4 ? 8193 : p256 == 3 ? 6144 : 10240)) {
        const int64_t p192 = std::min({cu_count() / (((M + 191) / 192) * ((N + 255) / 256)), K / 64 / 3, (int64_t)16});
        if (p256 > 2 && p192 >= 2 && 192 * p256 * 20 <= 256 * p192 * 19) return {192, (int)p192};
        return {256, (int)p256};
    }
    return {0, 1};
}

// Two parts of 256 x 256 tiles hand over inside the kernel (SPLIT_PAIR) where a norm launch in front has cleared the flag
// words: it saves the planes' round trip (an 8B layer of 2048 rows 766 us, with planes 775).
static bool pair_shape(const SplitChoice &c, int64_t M, int64_t N) {
    return c.tile == 256 && c.parts == 2 && ((M + 255) / 256) * ((N + 255) / 256) <= GEMM_SPLIT_MAX_TILES;
}

// Bytes of GemmArgs::planes that a launch of this shape uses; 0: it does not split.
size_t gemm_bf16_split_bytes(int32_t M, int32_t N, int32_t K) {
    if (M <= 0 || N <= 0 || N % 8 || N > 8192 || K % 64) return 0;
    const SplitChoice c = choose_split(M, N, K);
    if (c.parts < 2) return 0;
    const size_t planes = (size_t)c.parts * M * N * 4;
    return pair_shape(c, M, N) ? std::max(planes, (size_t)((M + 255) / 256) * ((N + 255) / 256) * 256 * 256 * 4) : planes;
}
bool gemm_bf16_split_takes(const GemmArgs &a) {
    if (a.dtype != CASCADE_BF16 || !v2_eligible(a) || a.rope_table || (a.epilogue & ~(CASCADE_EPI_BIAS | CASCADE_EPI_RESIDUAL)))
        return false;
    if (a.seg_end[0] != a.N || a.seg_end[1] != a.N || a.seg_end[2] != a.N) return false;
    const size_t need = gemm_bf16_split_bytes(a.M, a.N, a.K);
    return need && a.planes && a.planes_bytes >= need && (uintptr_t)a.planes % 16 == 0;
}
int32_t launch_gemm_bf16_split(const GemmArgs &a, const NormArgs *norm, bool &norm_done, hipStream_t s) {
    const SplitChoice c = choose_split(a.M, a.N, a.K);
    norm_done = false;
    if (a.sk_sync && pair_shape(c, a.M, a.N)) return launch_cfg2<256, 256, 2, 2, 64, 2, false, false, SPLIT_PAIR>(a, s, 2);
    const int32_t st = c.tile == 256   ? launch_cfg2<256, 256, 2, 2, 64, 2, false, false, SPLIT_PARTS>(a, s, c.parts)
                       : c.tile == 192 ? launch_cfg2<192, 256, 2, 2, 64, 2, false, false, SPLIT_PARTS>(a, s, c.parts)
                                       : launch_cfg2<128, 128, 2, 2, 64, 3, false, false, SPLIT_PARTS>(a, s, c.parts);
    norm_done = norm != nullptr;
    return st != CASCADE_OK ? st : launch_splitk_finish(a, c.parts, norm, s);
}

// The same for a projection into heads, which has no norm behind it to take along and whose alternative below 65 rows is the
// few-row kernel: the second launch has to be earned.  Weights cold, one layer with an FFN of 256, split / unsplit by rows (main
// loop as for choose_split): K 4096
// (6144 columns, 48 tiles per row of tiles) 17 rows 0.99, 24 0.97, 32 0.96, 64 0.90, 128 0.90, 256 0.96; K 3072 (5120 columns, 40)
// 17 rows 1.01, 32 1.00, 64 0.94, 128 0.90, 256 0.93, 384 0.97; K 2048 (3072 columns, 24) 17 rows 1.04, 32 1.03, 33 0.97, 128 0.95, 256
// 0.99, whole layers of 72 tiles 102 / 105 us; K 1536 (2048 columns, 16) 33 rows 0.93, 128 0.95; K 1024 (3072 columns, 24) 33 rows
// 1.05, 64 1.03, 128 1.07, (1536 columns, 12) 64 rows 0.99, 128 1.01, two rows of tiles 1.03.  256 x 256 tiles: K 8192 (40 tiles) in
// six parts, 129 rows 0.98, 160 1.00, 200 1.02, 256 1.00; but K 4096 (48) in five, whole layer of 300 rows 240 / 242 us.
static SplitChoice choose_proj_split(int64_t M, int64_t N, int64_t K) {
    if (M <= (K > 3072 ? 16 : 32)) return {0, 1};
    const int64_t t128 = ((M + 127) / 128) * ((N + 127) / 128), p128 = parts128(M, N, K);
    const int64_t p256 = std::min({cu_count() / (((M + 255) / 256) * ((N + 255) / 256)), (int64_t)8});
    if (p128 >= 2 && K >= (t128 <= 24 ? 1536 : t128 <= 48 ? 2048 : 3072)) return {128, (int)p128};
    if (p128 < 2 && p256 >= 5 && K >= 8192) return {256, (int)p256};
    return {0, 1};
}
// Bytes of GemmArgs::planes that such a launch uses; 0: it does not split.
size_t gemm_bf16_proj_split_bytes(int32_t M, int32_t N, int32_t K) {
    if (M <= 0 || N <= 0 || N % 16 || K % 64) return 0;
    const SplitChoice c = choose_proj_split(M, N, K);
    return c.parts < 2 ? 0 : (size_t)c.parts * M * N * 4;
}
bool gemm_bf16_proj_split_takes(const GemmArgs &a) {
    if (a.dtype != CASCADE_BF16 || !v2_eligible(a) || (a.epilogue & ~CASCADE_EPI_BIAS) || a.ymap.map) return false;
    if (a.rope_table && (!gemm_bf16_rope_fusable(a) || (uintptr_t)a.rope_table % 16)) return false;
    for (int i = 0; i < 3; ++i)
        if (a.seg_end[i] % 16) return false;
    if (a.ldy % 8 || (uintptr_t)a.Y % 16) return false;
    const size_t need = gemm_bf16_proj_split_bytes(a.M, a.N, a.K);
    return need && a.planes && a.planes_bytes >= need && (uintptr_t)a.planes % 16 == 0;
}
int32_t launch_gemm_bf16_proj_split(const GemmArgs &a, hipStream_t s) {
    const SplitChoice c = choose_proj_split(a.M, a.N, a.K);
    const int32_t st = c.tile == 256 ? launch_cfg2<256, 256, 2, 2, 64, 2, false, false, SPLIT_PARTS>(a, s, c.parts)
                                     : launch_cfg2<128, 128, 2, 2, 64, 3, false, false, SPLIT_PARTS>(a, s, c.parts);
    return st != CASCADE_OK ? st : launch_splitk_heads(a, c.parts, s);
}

// Tiles of bm rows x bn_out output columns of a launch
static int64_t count_tiles(const GemmArgs &a, int bm, int bn_out) {
    int64_t t = 0;
    int col0 = 0;
    for (int i = 0; i < 3; ++i) {
        t += (std::max(0, a.seg_end[i] - col0) + bn_out - 1) / bn_out;
        col0 = std::max(col0, a.seg_end[i]);
    }
    return t * ((a.M + bm - 1) / bm);
}

// Returns CASCADE_EUNSUPPORTED when the shape is not eligible (the caller then uses the general kernel).
int32_t launch_gemm_bf16_v2(const GemmArgs &a, hipStream_t s) {
    if (!v2_eligible(a)) return a.rope_table ? CASCADE_EINVAL : CASCADE_EUNSUPPORTED;
    const bool swiglu = a.epilogue & CASCADE_EPI_SWIGLU;
    // Tile choice.  The cost of a launch is rounds of workgroups x columns per tile; candidates are
    // 256 rows x {256, 224, 192} columns (BK 64, two stages; the widths exist to fill whole rounds) and 256 x 128.  The
    // cheapest wins, the narrow one only by a margin.  Lower and narrower tiles follow below where those leave CUs idle.
    // 256 x 128, 8 wavefronts of 64 x 64 in two groups half a tile apart / one wavefront per SIMD with 64 x 128 (us):
    // 2048 x 4096 x 4096 with residual 66.1 / 60.3, x 14336 211 / 200, 4096 x 2048 x 2048 33.9 / 30.1, 8192 x 768 x 3072
    // 43.7 / 38.2, 4000 x 2048 x 8192 120 / 104, 2040 x 3000 x 1600 27.4 / 22.2 (128 x 64 per wavefront 60.4, 200, 30.4, 38.7, 106, 22.7);
    // 150 shapes 1.09 on average, behind by up to 5 % where two k-tiles in flight for three show: a short last row of tiles and all
    // tiles in one round (265 x 14336 x 4096 54.8 / 57.7, 1180 x 4096 x 4096 with bias 50.0 / 51.9).
    auto n_tiles = [&](int bn_out) { return count_tiles(a, 256, bn_out); };
    const int64_t cus = cu_count();
    auto cost = [&](int bne) { return ((n_tiles(swiglu ? bne / 2 : bne) + cus - 1) / cus) * bne; };
    const int64_t c256 = cost(256), c224 = cost(224), c192 = cost(192), c128 = cost(128);
    const bool gelu = a.epilogue & (CASCADE_EPI_GELU_ERF | CASCADE_EPI_GELU_TANH), bias = a.epilogue & CASCADE_EPI_BIAS;
    const int64_t best = swiglu ? std::min(c224, c256) : std::min(c192, std::min(c224, c256));
    // the 256 x 128 tile does ~15 % fewer flops per cycle than the wide ones: it has to be that much cheaper (8B layer of 1700
    // rows 681 us, with 5 % for 15 674, but 2500 rows 923 / 926, 2048 rows 742 / 744, 70B 2000 rows 2608 / 2617)
    const bool narrow = !swiglu && !a.rope_table && best * 20 > c128 * 23;
    // 128 x 128 tiles, when they all fit on the CUs at once with three k-tiles in flight each (few rows of tiles: the
    // 192 to 256 wide ones leave most CUs without a workgroup and multiply padding), or two workgroups to a CU where
    // there is one row of tiles (the weights are all that counts), where the wide tiles would fill less than 2/5 of the
    // CUs, or where a workgroup's start and end are a large part of it (short reductions).  For the last the areas a CU
    // computes are compared: `two` with both its places taken in every round, `one` with the last round half full, the
    // wide tiles' `area`.  The limits were set over 944 shapes of K 512 to 1536 and 257 to 1280 tiles, weights cold, with a
    // longer loop and epilogue in every tile and 256 x 128 on 8 wavefronts: within 0.3 to 1.4 % of the faster choice on average by
    // epilogue, at worst 8 % behind (all of them two to a CU, which the areas do not ask for, was up to 38 % behind).  As the
    // tiles are now, wide ones / 128 x 128 two to a CU (us): 300 x 50256 x 768 42.5 / 41.5, 3000 x 6144 x 768 with residual 46.6 /
    // 38.8; not 1000 x 11008 x 1536 34.0 / 47.7, 256 x 50256 x 768 27.1 / 38.0, SwiGLU 2048 x 4096 x 1536 41.3 / 53.3 (nor, by now,
    // SwiGLU 1400 x 2304 x 768 13.9 / 14.9, which takes them).  Against 256 x 128 up to K = 1024 and, beyond 512, for
    // moderately wide outputs (2048 x 2304 x 768 13.7 / 14.0, in 128 x 96 13.3; not 512 x 16384 x 1024 20.8 / 23.3); with a bias up
    // to 768 (2048 x 3072 x 1024 18.1 / 18.3, 128 x 96 17.1).  A bias costs the 192-wide tiles 2 us, one memory latency per column
    // block (4096 x 2304 x 768 19.3 / 22.1, with bias 21.2 / 22.9, 128 x 96 21.5; 4096 x 3072 x 768 with bias 22.3 / 24.4), GELU 7
    // (4096 x 3072 x 768 29.0 / 29.6; 256 columns 42.5).
    // One to a CU: 333 x 4096 x 4096 49.9 / 33.3, x 14336 162 / 115, SwiGLU 100 x 14336 x 4096 60.9 / 50.2; wide tiles on few CUs:
    // SwiGLU 256 x 11008 x 4096 58.8 / 73.5, 2048 x 2304 x 2048 34.3 / 42.4 and x 14336 213 / 341, hence its limits (by now also 1000 x
    // 2304 x 8192 95.8 / 104.6, which takes them); one row of the vocabulary projection: 32 x 128256 x 4096 207 / 191.
    const int64_t t128 = count_tiles(a, 128, swiglu ? 64 : 128), wide = n_tiles(swiglu ? 112 : 192);
    const int64_t two = (t128 + 2 * cus - 1) / (2 * cus) * 256, one = (t128 + cus - 1) / cus * 128;   // columns of 128 rows
    auto short_reduction = [&]() {
        if (a.K > 1536 || t128 > 5 * cus) return false;
        // areas in columns of 256 rows, times 20
        const int64_t area = narrow ? c128 * 23 : best * 20, two20 = two * 10, one20 = one * 10;
        if (gelu) return two20 <= area || (a.K <= 1024 && one20 <= area);
        if (narrow) return a.K <= (bias ? 768 : 1024) && (a.K <= 512 || a.N <= 8192) && two20 <= c128 * 20;
        const int width = swiglu ? (c224 == best ? 224 : 256) : c192 == best ? 192 : c224 == best ? 224 : 256;
        const bool several = best > width;                  // rounds of wide tiles
        if (two20 * 10 <= area * 9 || (several && two20 <= area)) return true;
        return bias && width == 192 && !several && a.K <= 1024 && a.N <= 4096 && one20 <= area;
    };
    const bool small_one = t128 <= cus;
    const bool small_two = !small_one && (a.M <= 128 || short_reduction() ||
                                          (t128 <= 2 * cus && wide * 5 <= 2 * cus && (swiglu ? t128 * 4 <= 5 * cus : a.K <= 4096)));
    // 128 x 96 tiles: a quarter less to load and to multiply, in place of 128 x 128 ones wherever they take as many rounds
    // (one to a CU: 4096 x 768 x 768 with residual 10.3 / 9.9, x 3072 23.7 / 22.8, 2048 rows 22.3 / 20.3, 500 x 6144 x 4096
    // 38.4 / 34.0; two: 4096 x 2304 x 768 with bias 23.1 / 22.2, 2048 x 3072 x 768 with bias and GELU 18.3 / 16.8, 6000 x
    // 768 x 768 with residual 16.2 / 15.4; not 3000 x 2304 x 768 16.2 / 19.4, which takes them a round more, nor 4096 x 3072 x
    // 1024 26.9 / 30.2, where both come to as many columns per CU; two to a CU from 15 % fewer columns per CU on).
    const int64_t t96 = count_tiles(a, 128, 96);
    // A tile saves less than it costs where the launches before and behind take another one: code that no recent launch ran is
    // fetched cold (~2 us).  So short reductions without activation and residual (a q/k/v projection, up to three quarters of
    // the width of the launch that follows) take 96 columns to a CU only if that one would too: a layer of width 768,
    // 1167 rows 88.7 whole / 90.4 with q/k/v alone, 1000 rows with both 87.4 / 80.9.  A projection on its own has no such
    // neighbours and stays with 128 columns too.
    const bool lone = !gelu && !(a.epilogue & CASCADE_EPI_RESIDUAL) && a.K <= 1536;
    const bool narrow_one = t96 * (lone ? 4 : 3) <= cus * 3, narrow_two = (t96 + cus - 1) / cus * 96 * 20 < one * 17;
    if (a.rope_table) {                  // rotary embedding in the epilogue: the one-wavefront kernels only
        if (!gemm_bf16_rope_fusable(a)) return CASCADE_EINVAL;
        if (small_one)
            return narrow_one ? launch_cfg2<128, 96, 4, 1, 64, 3, false, true>(a, s)
                              : launch_cfg2<128, 128, 2, 2, 64, 3, false, true>(a, s);
        // 256 x 96 where they fit on the CUs at once (8B, 800 to 1024 rows: half of them had a 256 x 192 tile, 82 us, now 52)
        if (count_tiles(a, 256, 96) <= cus) return launch_cfg2<256, 96, 4, 1, 64, 2, false, true>(a, s);
        if (small_two) return launch_cfg2<128, 128, 2, 2, 64, 2, false, true>(a, s);
        if (c256 * 100 <= best * 104 && n_tiles(256) > cus) return launch_cfg2<256, 256, 2, 2, 64, 2, false, true>(a, s);
        if (c192 == best) return launch_cfg2<256, 192, 2, 2, 64, 2, false, true>(a, s);
        if (c224 == best) return launch_cfg2<256, 224, 4, 1, 64, 2, false, true>(a, s);
        return launch_cfg2<256, 256, 2, 2, 64, 2, false, true>(a, s);
    }
    if (small_one) {
        if (swiglu) return launch_cfg2<128, 128, 2, 2, 64, 3, true>(a, s);
        return narrow_one ? launch_cfg2<128, 96, 2, 2, 64, 3, false>(a, s) : launch_cfg2<128, 128, 2, 2, 64, 3, false>(a, s);
    }
    if (small_two) {
        if (swiglu) return launch_cfg2<128, 128, 2, 2, 64, 2, true>(a, s);
        return narrow_two ? launch_cfg2<128, 96, 2, 2, 64, 2, false>(a, s) : launch_cfg2<128, 128, 2, 2, 64, 2, false>(a, s);
    }
    // 192 x 128 where they fit on the CUs at once and the 128 x 128 ones do not, for GELU (slow in the wide tiles) or rows that
    // fill the 256-row tiles: a short last row of those drops the loads of the rows it lacks, and they won with 256 x 128 on 8
    // wavefronts, from whose time the limits are (15/16: the worst of 60 shapes of K 1024 to 4096 2.5 % behind, with GELU of 90 0.6 %).
    // Weights cold, 256 x 128 now / 192 x 128 (us): 4096 x 4096, 1040 rows 50.6 / 50.0, 1250 52.3 / 51.0, 1344 51.6 / 51.0, 1536 53.4 /
    // 52.2; with bias and residual 1344 rows 54.7 / 53.2; 4096 x 2048, 1152 rows 23.5 / 21.7, 1200 24.4 / 22.7, with GELU 31.4 / 25.2 and
    // 32.3 / 26.9; 2560 x 2560, 2040 rows 31.8 / 28.1; 3072 x 3072, 1790 rows 36.8 / 33.0; 1536 x 2048, 3400 rows with bias and
    // residual 28.2 / 25.1; 1100 x 4096 x 14336 163.1 / 162.5.
    const bool full_rows = a.M * (int64_t)16 >= ((a.M + 255) / 256) * (int64_t)(256 * 15);
    if (!swiglu && a.K <= 4096 && (gelu || full_rows) && count_tiles(a, 192, 128) <= cus)
        return launch_cfg2<192, 128, 2, 2, 64, 2, false>(a, s);
    if (swiglu) {
        // Lower and narrower tiles for the rows and CUs that 256 x 224 leave over, priced by what a round of them takes
        // (224: one of 256 x 224).  14336 x 4096, 200 rows 256 x 224 / 256 x 128: 74 / 63, 333 rows 256 x 224 / 192 x 224
        // 88 / 79, 700 rows 155 / 142; 28672 x 8192, 160 rows 192 / 182, 333 rows 340 / 302; 13824 x 5120, 256 rows 106 / 89 (256 x 128).
        const int64_t c192r = (count_tiles(a, 192, 112) + cus - 1) / cus * 205, c64 = (n_tiles(64) + cus - 1) / cus * 175;   // of 64 output columns
        if (c64 < best && c64 <= c192r) return launch_cfg2<256, 128, 4, 1, 64, 2, true>(a, s);
        if (c192r < best) return launch_cfg2<192, 224, 4, 1, 64, 2, true>(a, s);
        if (c224 < c256) return launch_cfg2<256, 224, 4, 1, 64, 2, true>(a, s);
        return launch_cfg2<256, 256, 2, 2, 64, 2, true>(a, s);
    }
    if (!narrow) {
        // 256 columns: the one-wavefront schedule when a CU works through several tiles of a long reduction and
        // the epilogue is light (its 256 accumulators leave the GELU code no registers); measured on
        // 8192 x 4096 x 4096 with residual 200 against 232 us, x 14336 644 against 754 (1.49 and 1.28 PFLOP/s).  It goes before
        // the narrower tiles up to a 4 % higher cost: fewer tile-load instructions and operand reads per MFMA
        // (8192 x 32000 x 4096: 1470 against 1554 us for 192 columns at 1.6 % more rounds x width).
        const bool solo256 = n_tiles(256) > cus && a.K >= 2048 && !gelu;
        if (c256 * 100 <= best * 104 && solo256) return launch_cfg2<256, 256, 2, 2, 64, 2, false>(a, s);
        // 192 and 224 columns: always the one-wavefront schedule, the narrowest cost first (2048 x 6144 x 4096 in
        // one round of 256 tiles: 78 us, 256 columns with 8 wavefronts 101)
        if (c192 == best) return launch_cfg2<256, 192, 2, 2, 64, 2, false>(a, s);
        if (c224 == best)
            return gelu ? launch_cfg2<256, 224, 4, 2, 64, 2, false>(a, s)     // 8 wavefronts
                        : launch_cfg2<256, 224, 2, 2, 64, 2, false>(a, s);
        return launch_cfg2<256, 256, 4, 2, 64, 2, false>(a, s);   // 8 wavefronts
    }
    return launch_cfg2<256, 128, 4, 1, 64, 2, false>(a, s);
}
