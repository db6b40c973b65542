// bf16 partial attention (Algorithm 3): (m, e, u~) of every (query row, key/value shard), each shard on its own.
//
// What bounds it: u~ is fp32, rows x shards x heads x d, and dwarfs everything else (512 MB for 2048 rows, 16 shards, 32 heads of
// 128; stores alone reach 5.9 TB/s, 90 us).  A workgroup per (query tile, shard) spends most of its life starting up: row
// map, queries, first tiles, one after the other, then two tiles of work and the write-out.  So here a workgroup keeps its
// query tile (32 rows of a head per wavefront) and walks the visible tiles of many shards in one stream: queries are
// loaded once, the next tiles are always on their way to LDS, and a shard's 20 stores drain under the tiles that
// follow (the waits count them).  With vector instructions at ~2/3 of the issue slots the walk itself takes ~85 us of the 145.
// Measured, kernel per (query tile, shard) / this one, with V^T and the merge (us): 2048 rows in 16 shards, 32 heads of 128
// 328 / 251, 12 heads 173 / 110; 4 x 1000 in 8 shards, 12 heads of 64 81 / 69, 32 heads 190 / 130; 4096 in one shard,
// 12 heads of 64 140 / 115, 32 heads of 128 208 / 190; 300 rows in 8 shards, 32 heads of 128 33 / 30.
//
// The arithmetic is that of attn_bf16_kernel, 32 rows and 64 keys at a time in the same order (same bits): S^T = K Q^T, lazily
// moved exponent offset, P rounded to bf16, O^T += V^T P^T, m and e referred to the true maximum.
//
// Wavefronts, stages: head dimension 128 four wavefronts and two stages of 32 KB, so that two workgroups share a CU and one
// computes while the other stores; 64 three stages of 16 KB and eight wavefronts of at most 128 registers, two workgroups
// to a CU (150 registers, one workgroup: 80 us for 69), or four wavefronts where launches or shards are small.
#include <climits>
#include "attn_bf16.h"

namespace {

// Wait for a tile and for everybody: all but the youngest vector-memory operations of this wavefront complete (those of one
// younger tile, and the stores of up to two shards behind the awaited loads), its LDS reads returned, workgroup barrier.
// Loads and stores of a wavefront complete in order here.
template <int LPT, int ST>
__device__ __forceinline__ void wait_tile(bool younger, int flushes) {
    if (younger) {
        if (flushes == 0) phase_barrier<LPT, true>();
        else if (flushes == 1) phase_barrier<LPT + ST, true>();
        else phase_barrier<LPT + 2 * ST, true>();
    } else {
        if (flushes == 0) phase_barrier<0, true>();
        else if (flushes == 1) phase_barrier<ST, true>();
        else phase_barrier<2 * ST, true>();
    }
}

}   // namespace

template <int D, int NWV, int NST>
__global__ __launch_bounds__(NWV * 64, D == 128 ? 2 : NWV == 8 ? 4 : 3) void attn_partial_kernel(AttnBf16Params p, int shards_per_wg) {
    constexpr int TQ = 2, KS = D / 32, DB = D / 16;
    constexpr int K_ROW = D * 2, K_RPI = 1024 / K_ROW, K_CPR = K_ROW / 16;
    constexpr int K_BYTES = KV_TILE * K_ROW, V_BYTES = D * 128;
    constexpr int STAGE = K_BYTES + V_BYTES + KV_TILE * 4;
    constexpr int K_INSTR = KV_TILE / K_RPI / NWV, V_INSTR = D / 8 / NWV;
    constexpr int LPT = K_INSTR + V_INSTR + 1;         // tile loads per wavefront
    constexpr int ST = TQ * DB + 2 * TQ;               // stores of a shard's partial per wavefront
    static_assert(LPT + 2 * ST < 64, "vmcnt");
    typedef __attribute__((ext_vector_type(4))) int i32x4;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    i32x4 *list = (i32x4 *)(smem + NST * STAGE);                                   // [PARTS_MAX_TILES]
    uint64_t *vis = (uint64_t *)(smem + NST * STAGE + PARTS_MAX_TILES * 16);         // [PARTS_MAX_TILES / 64]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g4 = lane >> 4;
    const int hpb = 1 << p.hpb_log2, hsel = wave & (hpb - 1), rg = wave >> p.hpb_log2;
    const int q_tile = (int)div_by_magic(blockIdx.x, p.gy_magic), by = (int)blockIdx.x - q_tile * p.gy;
    const int b = (int)div_by_magic((uint32_t)by, p.heads_magic), gh = by - b * p.heads;
    const int g = (int)div_by_magic((uint32_t)gh, p.hblocks_magic);
    const int h = g * p.rep + (gh - g * p.hblocks) * hpb + hsel;

    const tile_cptr kvtiles = (tile_cptr)p.kvtiles;
    const tile_cptr qtp = (tile_cptr)p.qtiles + q_tile;
    const int_cptr first = (int_cptr)p.kv_shard_first;
    const int k0 = blockIdx.z * shards_per_wg, k1 = min(k0 + shards_per_wg, p.S);
    const int t0 = first[k0], nt = first[k1] - t0;     // at most PARTS_MAX_TILES
    const int q_row_start = qtp->row_start, q_n_rows = qtp->n_rows, q_pmax = qtp->pmax;
    const int wrow0 = rg * 16 * TQ;
    const bool active = wrow0 < q_n_rows;

    // ---- The visible tiles of the workgroup's shards, in order, as a list in LDS (one thread per tile): tile, first row,
    // rows | 1 << 16 on a shard's last visible tile, column block of V^T.  A shard's visible tiles are a prefix of its
    // tiles (ordered by smallest position).
    bool seen = false;
    int e_row = 0, e_rows = 0, e_index = 0, e_shard = 0;
    if (tid < PARTS_MAX_TILES) {
        if (tid < nt) {
            const CascadeTile *tp = p.kvtiles + t0 + tid;
            seen = !p.causal || tp->pmin <= q_pmax;
            e_row = tp->row_start; e_rows = tp->n_rows; e_index = tp->index; e_shard = tp->shard;
        }
        const uint64_t m = __ballot(seen);
        if (lane == 0) vis[wave] = m;
    }
    // ---- query fragments (B operand of S^T = K Q^T): lane holds row l16 of each 16-row block, chunk 32 ks + 8 g4
    bf16x8 qf[TQ][KS];
    int qlim[TQ];
    uint32_t row_off[TQ];                              // packed row; OOB_OFF: none (its stores fall outside, but are counted)
#pragma unroll
    for (int qb = 0; qb < TQ; ++qb) {
        const int rloc = wrow0 + 16 * qb + l16;
        const bool ok = rloc < q_n_rows;
        const int r = q_row_start + (ok ? rloc : q_n_rows - 1);
        const bf16_t *qp = p.q + b * p.qs_b + h * p.qs_h + (int64_t)(p.q_rowmap ? p.q_rowmap[r] : r) * p.qs_n + g4 * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[qb][ks] = *(const bf16x8 *)(qp + ks * 32);
        qlim[qb] = p.causal ? p.pos_packed[r] : (1 << 30) - 1;    // padding of a ragged tile: position 2^30
        row_off[qb] = ok ? (uint32_t)r : OOB_OFF;
    }
    int wq_hi = INT_MAX, wq_lo = INT_MAX;
    if (p.causal && active) {
        wq_hi = max(qtp->sub_max[2 * rg], qtp->sub_max[2 * rg + 1]);
        wq_lo = min(qtp->sub_min[2 * rg], qtp->sub_min[2 * rg + 1]);
    }
    __syncthreads();
    int n = 0;
#pragma unroll
    for (int w = 0; w < PARTS_MAX_TILES / 64; ++w) {
        n += __popcll(vis[w]);
    }
    n = __builtin_amdgcn_readfirstlane(n);
    if (seen) {
        int pos = __popcll(vis[wave] & ((1ull << lane) - 1));
        for (int w = 0; w < wave; ++w) pos += __popcll(vis[w]);
        const bool next_seen = tid + 1 < nt && ((vis[(tid + 1) >> 6] >> ((tid + 1) & 63)) & 1);
        const bool last = t0 + tid + 1 == p.kv_shard_first[e_shard + 1] || !next_seen;
        list[pos] = i32x4{t0 + tid, e_row, e_rows | (last ? 1 << 16 : 0), e_index};
    }
    __syncthreads();

    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(p.k + b * p.ks_b + g * p.ks_h), 0, p.k_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(p.vt + b * p.vts_b + g * p.vts_h), 0, p.vt_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int32_t *>(p.pos_kv_padded), 0, (uint32_t)p.n_kvtiles * KV_TILE * 4, 0x00020000);
    // direct-to-LDS loads, row and swizzle of each instruction as in attn_bf16_kernel
    uint32_t k_lane[K_INSTR], v_lane[V_INSTR];
    int k_rr[K_INSTR];
#pragma unroll
    for (int i = 0; i < K_INSTR; ++i) {
        const int rr = (wave * K_INSTR + i) * K_RPI + lane / K_CPR, slot = lane % K_CPR;
        const int c = D == 128 ? (slot ^ (rr & 15)) : (slot ^ ((rr >> 1) & 7));
        k_rr[i] = rr;
        k_lane[i] = (uint32_t)rr * (uint32_t)(p.ks_n * 2) + c * 16;
    }
#pragma unroll
    for (int i = 0; i < V_INSTR; ++i) {
        const int rr = (wave * V_INSTR + i) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ((rr >> 1) & 7);
        v_lane[i] = (uint32_t)rr * (uint32_t)(p.npad * 2) + c * 16;
    }
    auto entry = [&](int i) {
        const i32x4 e = list[i];
        return i32x4{__builtin_amdgcn_readfirstlane(e[0]), __builtin_amdgcn_readfirstlane(e[1]),
                     __builtin_amdgcn_readfirstlane(e[2]), __builtin_amdgcn_readfirstlane(e[3])};
    };
    auto issue = [&](const i32x4 &e, int stage) {
        unsigned char *sk = smem + stage * STAGE, *sv = sk + K_BYTES;
        const uint32_t k_tile = (uint32_t)e[1] * (uint32_t)(p.ks_n * 2), v_tile = (uint32_t)e[3] * (KV_TILE * 2);
        const int rows = e[2] & 0xffff;
#pragma unroll
        for (int i = 0; i < K_INSTR; ++i)
            load16_to_lds(rk, sk + (wave * K_INSTR + i) * K_RPI * K_ROW, k_rr[i] < rows ? k_tile + k_lane[i] : OOB_OFF);
#pragma unroll
        for (int i = 0; i < V_INSTR; ++i) load16_to_lds(rv, sv + (wave * V_INSTR + i) * 8 * 128, v_tile + v_lane[i]);
        load4_to_lds(rp, sv + V_BYTES, (uint32_t)(e[3] * KV_TILE + lane) * 4);
    };

    const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
    constexpr float RESCALE_LOG2 = 8.0f;
    f32x4 oacc[TQ][DB];
    float m_run[TQ], m_top[TQ], l_run[TQ];
    auto reset = [&]() {
#pragma unroll
        for (int qb = 0; qb < TQ; ++qb) {
            m_run[qb] = m_top[qb] = -INFINITY;
            l_run[qb] = 0.f;
#pragma unroll
            for (int db = 0; db < DB; ++db) oacc[qb][db] = zero4;
        }
    };
    // a shard's partial: exactly ST stores, whatever rows exist
    auto flush = [&](int kk) {
        const int64_t me = (((int64_t)b * p.H + h) * p.S + kk) * p.N;
        const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(p.m + me, 0, (uint32_t)p.N * 4, 0x00020000);
        const __amdgpu_buffer_rsrc_t re = __builtin_amdgcn_make_buffer_rsrc(p.e + me, 0, (uint32_t)p.N * 4, 0x00020000);
        const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc(
            p.u + (((int64_t)b * p.S + kk) * p.H + h) * (int64_t)p.N * D, 0, (uint32_t)p.N * D * 4, 0x00020000);
#pragma unroll
        for (int qb = 0; qb < TQ; ++qb) {
            const float l_tot = xor_sum_16_32(l_run[qb]);
            const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
            const float corr = m_top[qb] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run[qb] - m_top[qb]);
            const float f = p.u_mode == CASCADE_U_NORMALISED ? inv : corr;
            const uint32_t mo = g4 == 0 && row_off[qb] != OOB_OFF ? row_off[qb] * 4 : OOB_OFF;
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(m_top[qb] * LN2), rm, mo, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(l_tot * corr), re, mo, 0, 0);
            const uint32_t uo = row_off[qb] != OOB_OFF ? row_off[qb] * (D * 4) + 16 * g4 : OOB_OFF;
#pragma unroll
            for (int db = 0; db < DB; ++db)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, oacc[qb][db] * f), ru, uo + 64 * db, 0, 0);
        }
    };
    const int k_swz = D == 128 ? l16 : (l16 >> 1), v_swz = l16 >> 1;

    auto compute = [&](const i32x4 &e, int stage) {
        const tile_cptr tp = kvtiles + e[0];
        const int kn = e[2] & 0xffff;
        int skipm = 0, maskm = 0;
#pragma unroll
        for (int kvb = 0; kvb < 4; ++kvb) {
            skipm |= (int)((kvb * 16 >= kn) | (tp->sub_min[kvb] > wq_hi)) << kvb;
            maskm |= (int)((kvb * 16 + 16 > kn) | (tp->sub_max[kvb] > wq_lo)) << kvb;
        }
        if (skipm == 15) return;
        const bool both = (skipm & 12) != 12;          // the second half of the tile is needed
        const unsigned char *sk = smem + stage * STAGE, *sv = sk + K_BYTES;
        f32x4 s[TQ][4];
        auto scores = [&](int half) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const int kvb = 2 * half + kb;
                const unsigned char *kp = sk + (kvb * 16 + l16) * K_ROW;
                bf16x8 kf[KS];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) kf[ks] = *(const bf16x8 *)(kp + (((4 * ks + g4) ^ k_swz) * 16));
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int qb = 0; qb < TQ; ++qb)
                        s[qb][kvb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], qf[qb][ks], ks == 0 ? zero4 : s[qb][kvb], 0, 0, 0);
            }
        };
        scores(0);
        if (both) scores(1);
        else
#pragma unroll
            for (int qb = 0; qb < TQ; ++qb) s[qb][2] = s[qb][3] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        if (maskm) {
            i32x4 pk[4];
            const uint32_t pa = (uint32_t)(uintptr_t)(lds_void *)(sv + V_BYTES) + 16 * g4;
            asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:64\n\tds_read_b128 %2, %4 offset:128\n\t"
                         "ds_read_b128 %3, %4 offset:192\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(pk[0]), "=&v"(pk[1]), "=&v"(pk[2]), "=&v"(pk[3])
                         : "v"(pa)
                         : "memory");
#pragma unroll
            for (int kvb = 0; kvb < 4; ++kvb)
#pragma unroll
                for (int qb = 0; qb < TQ; ++qb)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (pk[kvb][r] > qlim[qb]) s[qb][kvb][r] = -INFINITY;
        }
        bf16x8 pf[TQ][2];
#pragma unroll
        for (int qb = 0; qb < TQ; ++qb) {
            float mx = -INFINITY;
#pragma unroll
            for (int kvb = 0; kvb < 4; ++kvb)
#pragma unroll
                for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s[qb][kvb][r]);
            mx = xor_max_16_32(mx) * p.scale_log2;
            m_top[qb] = fmaxf(m_top[qb], mx);
            if (__builtin_amdgcn_readfirstlane(__any(mx > m_run[qb] + RESCALE_LOG2))) {
                const float m_new = fmaxf(m_run[qb], mx);
                const float alpha = __builtin_amdgcn_exp2f(m_run[qb] - ((m_new == -INFINITY) ? 0.f : m_new));
                m_run[qb] = m_new;
                l_run[qb] *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db) oacc[qb][db] *= alpha;
            }
            const float m_sub = (m_run[qb] == -INFINITY) ? 0.f : m_run[qb];
            float psum = 0.f;
#pragma unroll
            for (int kvb = 0; kvb < 4; ++kvb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float pv = __builtin_amdgcn_exp2f(fmaf(s[qb][kvb][r], p.scale_log2, -m_sub));
                    psum += pv;
                    pf[qb][kvb >> 1][4 * (kvb & 1) + r] = (bf16_t)pv;
                }
            l_run[qb] += psum;
        }
        auto values = [&](int s2) {
            const int cv = ((4 * s2 + g4) ^ v_swz) * 16;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const bf16x8 vf = *(const bf16x8 *)(sv + (db * 16 + l16) * 128 + cv);
#pragma unroll
                for (int qb = 0; qb < TQ; ++qb)
                    oacc[qb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[qb][s2], oacc[qb][db], 0, 0, 0);
            }
        };
        values(0);
        if (both) values(1);
    };

    reset();
    if (n > 0) {
        // Tile i is multiplied while those up to i + NST - 1 are on their way.  The stage that iteration i requests into held
        // tile i - 1, whose last reads every wavefront had behind it at the barrier that ended iteration i - 1.
        i32x4 e0 = entry(0), e1 = entry(n > 1 ? 1 : 0), e2 = entry(n > 2 ? 2 : 0);
        issue(e0, 0);
        if (NST == 3 && n > 1) issue(e1, 1);
        if (NST == 3 && n > 1) phase_barrier<LPT, false>();
        else phase_barrier<0, false>();
        int stage = 0, f_prev = 0;
        for (int i = 0; i < n; ++i) {
            if (NST == 3) { if (i + 2 < n) issue(e2, stage == 0 ? 2 : stage - 1); }
            else if (i + 1 < n) issue(e1, stage ^ 1);
            const i32x4 e3 = entry(i + 3 < n ? i + 3 : 0);
            int f = 0;
            if (active) {
                compute(e0, stage);
                if (e0[2] >> 16) {
                    flush((kvtiles + e0[0])->shard);
                    reset();
                    f = 1;
                }
            }
            if (i + 1 < n) {
                if (NST == 3) wait_tile<LPT, ST>(i + 2 < n, f + f_prev);
                else wait_tile<LPT, ST>(false, f);
            }
            f_prev = f;
            e0 = e1; e1 = e2; e2 = e3;
            stage = stage == NST - 1 ? 0 : stage + 1;
        }
    }
    // shards of which the query tile sees nothing
    if (active)
        for (int k = k0; k < k1; ++k) {
            const int t = first[k] - t0;
            if (first[k + 1] - t0 > t && ((vis[t >> 6] >> (t & 63)) & 1)) continue;
            flush(k);
        }
}

template <int D, int NWV, int NST>
static int32_t launch_cfg(const AttnBf16Params &k, int n_qtiles, int shards_per_wg, hipStream_t s) {
    constexpr int lds = NST * (KV_TILE * D * 2 + D * 128 + KV_TILE * 4) + PARTS_MAX_TILES * 16 + PARTS_MAX_TILES / 8;
    auto kern = attn_partial_kernel<D, NWV, NST>;
    static std::atomic<uint64_t> lds_ready{0};
    CASCADE_HIP_TRY(ensure_dynamic_lds((const void *)kern, lds, lds_ready));
    const dim3 grid((unsigned)((int64_t)k.gy * n_qtiles), 1, (k.S + shards_per_wg - 1) / shards_per_wg);
    hipLaunchKernelGGL(kern, grid, dim3(NWV * 64), lds, s, k, shards_per_wg);
    CASCADE_HIP_TRY(hipGetLastError());
    return CASCADE_OK;
}

int32_t launch_attn_partial(const AttnBf16Params &k, int head_dim, int wavefronts, int n_qtiles, int shards_per_wg, hipStream_t s) {
    if (head_dim == 128) return wavefronts == 4 ? launch_cfg<128, 4, 2>(k, n_qtiles, shards_per_wg, s) : CASCADE_EINVAL;
    return wavefronts == 8 ? launch_cfg<64, 8, 3>(k, n_qtiles, shards_per_wg, s) : launch_cfg<64, 4, 3>(k, n_qtiles, shards_per_wg, s);
}
