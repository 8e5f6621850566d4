// Row-wise kernels of the verify step: RMSNorm (fused with the embedding gather or the split-K
// reduction and the residual add), rotary embedding + tree K/V write, SwiGLU gating, and the
// vocabulary argmax / top-k selection with wavefront-shuffle reductions.
#include "common.h"

// ---------------------------------------------------------------------------------------
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Which (row, column chunk) a workgroup of the kernels that write an activation slab takes.  A 128-byte line
// of the slab holds 16 bytes of each of eight rows, and consecutive workgroup ids go round-robin over the XCDs: with
// the row as the id eight L2s held an eighth of every line each and wrote it to memory piece by piece.  The 16 rows of
// a slab tile go to one XCD here, 8 ids apart (tile t of the (chunk, row tile) grid on XCD t % 8), so that their lines leave
// whole.  Norm kernel, row as the id / this (rocprofv3): 512 rows of 4096 12.4 -> 10.5 us, first layer 9.4 -> 9.1 (embeddings in
// cache); 272 rows 8.6 -> 7.7, 170 rows 7.0 -> 6.3; 68 rows of 8192 8.0 -> 6.8, of 4096 6.2 -> 5.6; fewer rows the same.
// Gating kernel, 7B widths: 102 rows 8.2 -> 7.1, 136 rows 9.4 -> 8.0.
// Workgroups beyond the last row or chunk have nothing to do (false).
__device__ __forceinline__ bool slab_block(int M, int chunks, int &row, int &chunk) {
    const int mt_n = (M + 15) >> 4, q = blockIdx.x >> 3, t = (q >> 4) * 8 + (blockIdx.x & 7);
    chunk = t / mt_n;
    row = (t - chunk * mt_n) * 16 + (q & 15);
    return row < M && chunk < chunks;
}
static dim3 slab_grid(int M, int chunks) { return dim3((unsigned)(((M + 15) / 16 * chunks + 7) / 8 * 128)); }

// RMSNorm, first half.  Per (row, 1024-column chunk): x += sum_s partial[s] (fixed order), then
// the *unnormalised* x * gain is written as two bf16 planes (hi, lo) in the GEMM's fragment
// order, and the chunk's sum of squares goes to ssq[row][chunk].  The row factor
// rsqrt(mean(x^2) + eps) is a scalar per row and commutes with the matrix product, so the GEMM
// applies it to its output rows; that keeps this kernel free of any row-wide reduction and
// lets all CUs share the split-K partial traffic.
// EMBED (the first layer's norm): x is the row's embedding instead of residual + partial sums, and is
// written here: tree rows take tok_emb[token], mask rows mask_emb[index] (Sec. 3.1), inactive rows
// (token < 0) the zero vector.  A launch and a pass over x less than an embedding kernel ahead of it
// (small shape, 2 layers 81.7 -> 80.0 us; 7B widths, 2 layers, 68 rows 340.4 -> 338.2, one row 246.8 -> 245.1).
template <bool EMBED>
__global__ __launch_bounds__(256) void rmsnorm_prep_kernel(float *__restrict__ x, const float *__restrict__ partial,
                                                           int splits, int M, int d,
                                                           const uint16_t *__restrict__ gain,
                                                           uint16_t *__restrict__ h_frag, float *__restrict__ ssq,
                                                           EmbedSource e, BuildSource build, TemplateDev t) {
    __shared__ float red[4];
    int row, chunk;
    if (!slab_block(M, (d + 1023) >> 10, row, chunk)) return;
    const int tid = threadIdx.x, n_ksteps = (d + 31) >> 5, m_tiles = (M + 15) >> 4;
    const int c = chunk * 256 + tid;                         // float4 column
    float ss = 0.f;
    if (c < (d >> 2)) {
        float4 *xr = reinterpret_cast<float4 *>(x + (int64_t)row * d);
        // Everything this thread reads is requested before anything is looked at (one memory
        // round trip): the residual, the gain and the first eight splits (the loads of a group
        // are independent; indices past the last split re-read it and are left out of the sum).
        // The partial sums are added in split order.
        float4 p[8];
        if (splits > 0) {
#pragma unroll
            for (int u = 0; u < 8; u++)
                p[u] = reinterpret_cast<const float4 *>(partial + ((int64_t)min(u, splits - 1) * M + row) * d)[c];
        }
        float4 v;
        if constexpr (EMBED) {
            const int b = row / e.rows, r = row - b * e.rows;
            int tok;
            if (build.root) {
                tok = tree_token(build, t, b, r);
                if (c == 0) build.token[row] = tok;
            } else {
                tok = e.token[row];
            }
            const uint16_t *src = nullptr;
            if (e.is_mask[r]) src = e.mask_emb + (int64_t)e.mask_index[r] * d;
            else if (tok >= 0 && tok < e.vocab) src = e.tok_emb + (int64_t)tok * d;
            const uint2 q = src ? reinterpret_cast<const uint2 *>(src)[c] : make_uint2(0u, 0u);
            v = make_float4(__uint_as_float(q.x << 16), __uint_as_float(q.x & 0xFFFF0000u), __uint_as_float(q.y << 16),
                            __uint_as_float(q.y & 0xFFFF0000u));
        } else {
            v = xr[c];
        }
        const uint2 gq = reinterpret_cast<const uint2 *>(gain)[c];
        if (splits > 0) {
#pragma unroll
            for (int u = 0; u < 8; u++)
                if (u < splits) { v.x += p[u].x; v.y += p[u].y; v.z += p[u].z; v.w += p[u].w; }
        }
        for (int s0 = 8; s0 < splits; s0 += 8) {
#pragma unroll
            for (int u = 0; u < 8; u++)
                p[u] = reinterpret_cast<const float4 *>(partial + ((int64_t)min(s0 + u, splits - 1) * M + row) * d)[c];
#pragma unroll
            for (int u = 0; u < 8; u++)
                if (s0 + u < splits) { v.x += p[u].x; v.y += p[u].y; v.z += p[u].z; v.w += p[u].w; }
        }
        if (EMBED || splits > 0) xr[c] = v;
        ss = v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        const float o[4] = {v.x * bf16_to_f32((uint16_t)(gq.x & 0xFFFFu)), v.y * bf16_to_f32((uint16_t)(gq.x >> 16)),
                            v.z * bf16_to_f32((uint16_t)(gq.y & 0xFFFFu)), v.w * bf16_to_f32((uint16_t)(gq.y >> 16))};
        uint16_t hi[4], lo[4];
#pragma unroll
        for (int e = 0; e < 4; e++) split_bf16(o[e], hi[e], lo[e]);
        uint2 ph, pl;
        ph.x = hi[0] | ((uint32_t)hi[1] << 16); ph.y = hi[2] | ((uint32_t)hi[3] << 16);
        pl.x = lo[0] | ((uint32_t)lo[1] << 16); pl.y = lo[2] | ((uint32_t)lo[3] << 16);
        const int pack_off = frag_pack_offset(M);
        *reinterpret_cast<uint2 *>(h_frag + frag_index(0, row, 4 * c, n_ksteps, m_tiles, pack_off)) = ph;
        *reinterpret_cast<uint2 *>(h_frag + frag_index(1, row, 4 * c, n_ksteps, m_tiles, pack_off)) = pl;
    }
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    if (tid == 0) ssq[(int64_t)row * RMS_MAX_CHUNKS + chunk] = red[0] + red[1] + red[2] + red[3];
}

// ---------------------------------------------------------------------------------------
// QKV epilogue: sum split-K partials, rotate q and k by the row's position
// ctx_len + depth(row) in the half-split pairing, write q [B][R][Hq][hd] and the rows'
// k/v into the per-pass tree scratch [B][Hkv][R][hd].  q, k and v are all written as hi and lo
// bf16 planes; only the hi planes of accepted rows are ever committed to the cache.
// A thread takes four neighbouring rotation pairs of a head: 16-byte loads, 8-byte stores.  What bounds it
// is the sums and planes it moves (512 rows of 96 heads: 50 MB); with one pair a thread, 4-byte loads and 2-byte
// stores, they moved at 2.1 TB/s, now at 4.8 (rocprofv3, 7B widths: 512 rows 23.9 -> 10.6 us, 272 rows in two
// k splits 14.2 -> 8.5, 170 rows 9.8 -> 6.1, 102 rows 7.5 -> 6.6; 13B 84 rows 7.6 -> 5.9; up to 84 rows of 7B, where the launch and
// two round trips are most of it, the same within 0.1: 68 rows 5.6.  Two pairs a thread: 68 rows 5.4, but 170 rows 8.0, 512 17.6).
#define ROPE_THREADS 128
template <int HD>
__global__ __launch_bounds__(ROPE_THREADS) void qkv_rope_kernel(
    // (what the first loads depend on sits in the first 14 dwords, which arrive in registers)
    const float *__restrict__ partial, const int32_t *__restrict__ ctx_len, const int32_t *__restrict__ depth,
    const float *__restrict__ rs_ssq, int splits, int M, int R, int Hq, int Hkv, int max_pos,
    const float *__restrict__ rope_cos, const float *__restrict__ rope_sin, uint16_t *__restrict__ q,
    uint16_t *__restrict__ q_lo, uint16_t *__restrict__ k_tree, uint16_t *__restrict__ v_tree,
    uint16_t *__restrict__ k_tree_lo, uint16_t *__restrict__ v_tree_lo, int rs_chunks, float rs_inv_d, float rs_eps) {
    constexpr int half = HD / 2, LANES = half / 4;           // threads per head
    const int row = blockIdx.x, head = blockIdx.y * (ROPE_THREADS / LANES) + threadIdx.x / LANES;   // head over Hq + 2*Hkv
    if (head >= Hq + 2 * Hkv) return;
    const int b = row / R, r = row % R;
    const int i = (threadIdx.x % LANES) * 4;
    // Two memory round trips: the row's position and the sums behind its norm factor, then the
    // rotary table entries together with the partial sums (the table is read for value heads too,
    // and ignored).
    const int row_ctx = ctx_len[b], row_depth = depth[r];
    const RowScale rs{rs_ssq, rs_chunks, rs_inv_d, rs_eps};
    const float sc = row_scale(rs, row);          // RMSNorm's row factor, deferred past the GEMM
    int pos = row_ctx + row_depth;
    pos = pos < max_pos ? pos : max_pos - 1;          // host checks capacity; stay in bounds
    const float4 tab_c = *reinterpret_cast<const float4 *>(rope_cos + (int64_t)pos * half + i);
    const float4 tab_s = *reinterpret_cast<const float4 *>(rope_sin + (int64_t)pos * half + i);
    const int64_t ncols = (int64_t)(Hq + 2 * Hkv) * HD;
    const int64_t col = (int64_t)head * HD + i;
    float lo[4] = {0.f, 0.f, 0.f, 0.f}, hi[4] = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < splits; s0 += 8) {     // eight splits per round trip, summed in split order
        float4 pl[8], ph[8];
#pragma unroll
        for (int u = 0; u < 8; u++) {
            if (u > 0 && s0 + u >= splits) continue;         // (reading the last one again instead cost 8 % of 512 rows in one split)
            const float *p = partial + ((int64_t)(s0 + u) * M + row) * ncols + col;
            pl[u] = *reinterpret_cast<const float4 *>(p);
            ph[u] = *reinterpret_cast<const float4 *>(p + half);
        }
#pragma unroll
        for (int u = 0; u < 8; u++)
            if (s0 + u < splits) {
                lo[0] += pl[u].x; lo[1] += pl[u].y; lo[2] += pl[u].z; lo[3] += pl[u].w;
                hi[0] += ph[u].x; hi[1] += ph[u].y; hi[2] += ph[u].z; hi[3] += ph[u].w;
            }
    }
    uint16_t *dst, *dst_lo;
    if (head < Hq) {
        dst = q + ((int64_t)row * Hq + head) * HD;
        dst_lo = q_lo + ((int64_t)row * Hq + head) * HD;
    } else if (head < Hq + Hkv) {
        const int64_t o = (((int64_t)b * Hkv + (head - Hq)) * R + r) * HD;
        dst = k_tree + o;
        dst_lo = k_tree_lo + o;      // the pass keeps the rounding residual of its own K/V rows
    } else {
        const int64_t o = (((int64_t)b * Hkv + (head - Hq - Hkv)) * R + r) * HD;
        dst = v_tree + o;
        dst_lo = v_tree_lo + o;
    }
    const float c[4] = {tab_c.x, tab_c.y, tab_c.z, tab_c.w}, sn[4] = {tab_s.x, tab_s.y, tab_s.z, tab_s.w};
    uint16_t a_hi[4], a_lo[4], b_hi[4], b_lo[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        float x = lo[e] * sc, y = hi[e] * sc;
        if (head < Hq + Hkv) rope_pair(x, y, c[e], sn[e]);
        split_bf16(x, a_hi[e], a_lo[e]);
        split_bf16(y, b_hi[e], b_lo[e]);
    }
    auto put = [](uint16_t *p, const uint16_t (&v)[4]) __attribute__((always_inline)) {
        *reinterpret_cast<uint2 *>(p) = make_uint2(v[0] | ((uint32_t)v[1] << 16), v[2] | ((uint32_t)v[3] << 16));
    };
    put(dst + i, a_hi);
    put(dst + i + half, b_hi);
    put(dst_lo + i, a_lo);
    put(dst_lo + i + half, b_lo);
}

// ---------------------------------------------------------------------------------------
// SwiGLU gating on the gate/up GEMM output whose 16-column tiles alternate gate, up.  One
// thread per 8 consecutive features: sums the split-K partials, writes both bf16 planes of
// silu(gate) * up as one 16-byte store each into the down-projection's activation slab
// (fragment order; features beyond d_ffn inside the last k-step are written as zeros).
__global__ void silu_mul_kernel(const float *__restrict__ partial, int splits, int M, int F,
                                uint16_t *__restrict__ act_frag, RowScale rs) {
    const int n_ksteps = (F + 31) >> 5, m_tiles = (M + 15) >> 4;
    int row, chunk;
    if (!slab_block(M, (n_ksteps * 4 + blockDim.x - 1) / blockDim.x, row, chunk)) return;
    const int f8 = chunk * blockDim.x + threadIdx.x;
    const int f = f8 * 8;
    if (f >= n_ksteps * 32) return;
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; e++) o[e] = 0.f;
    if (f < F) {
        const int64_t cg = (int64_t)(f >> 4) * 32 + (f & 15);
        float g[8], u[8];
#pragma unroll
        for (int e = 0; e < 8; e++) g[e] = u[e] = 0.f;
        for (int s = 0; s < splits; s++) {
            const float4 *p = reinterpret_cast<const float4 *>(partial + ((int64_t)s * M + row) * (2 * (int64_t)F) + cg);
            const float4 g0 = p[0], g1 = p[1], u0 = p[4], u1 = p[5];
            g[0] += g0.x; g[1] += g0.y; g[2] += g0.z; g[3] += g0.w; g[4] += g1.x; g[5] += g1.y; g[6] += g1.z; g[7] += g1.w;
            u[0] += u0.x; u[1] += u0.y; u[2] += u0.z; u[3] += u0.w; u[4] += u1.x; u[5] += u1.y; u[6] += u1.z; u[7] += u1.w;
        }
        const float sc = row_scale(rs, row);      // RMSNorm's row factor, deferred past the GEMM
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const float gs = g[e] * sc;
            o[e] = gs / (1.0f + expf(-gs)) * (u[e] * sc);
        }
    }
    uint16_t hi[8], lo[8];
#pragma unroll
    for (int e = 0; e < 8; e++) split_bf16(o[e], hi[e], lo[e]);
    uint4 ph, pl;
    ph.x = hi[0] | ((uint32_t)hi[1] << 16); ph.y = hi[2] | ((uint32_t)hi[3] << 16);
    ph.z = hi[4] | ((uint32_t)hi[5] << 16); ph.w = hi[6] | ((uint32_t)hi[7] << 16);
    pl.x = lo[0] | ((uint32_t)lo[1] << 16); pl.y = lo[2] | ((uint32_t)lo[3] << 16);
    pl.z = lo[4] | ((uint32_t)lo[5] << 16); pl.w = lo[6] | ((uint32_t)lo[7] << 16);
    const int pack_off = frag_pack_offset(M);
    *reinterpret_cast<uint4 *>(act_frag + frag_index(0, row, f, n_ksteps, m_tiles, pack_off)) = ph;
    *reinterpret_cast<uint4 *>(act_frag + frag_index(1, row, f, n_ksteps, m_tiles, pack_off)) = pl;
}

// ---------------------------------------------------------------------------------------
// Selection over the vocabulary.  Order: value descending, lower id first among equals.
// One workgroup per selected row.  Every thread scans its share of the row once and keeps its best
// entry; the workgroup's best is the first winner.  For the following ones (mask rows, k winners)
// only the wave whose thread owned the last winner looks again: its 64 lanes fetch that thread's
// share together, for the best entry below the winner, and the wave reduces again.  A further
// winner costs 0.6 us (one round trip to L2, one barrier) instead of a scan of the whole row (3 us).
// What bounds it: launch, one round trip for the row (128 KB at 32000 logits, through one CU) and
// the scan's vector instructions for the tree rows, the winners' chain for the mask rows.
// 68 rows x 32000 logits: 6.3 -> 4.4 us without mask rows, 15.3 -> 6.2 us with four winners per
// mask row, 27.2 -> 8.8 us with eight.
// (value, index) as one unsigned 64-bit key whose order is "larger value first, lower index on
// equal values": the float's bits made monotone (sign flip for positives, complement for
// negatives; -0 is first turned into +0) above the complemented index.  Logits are finite.
__device__ __forceinline__ uint32_t select_order(float v) {
    const uint32_t u = __float_as_uint(v + 0.0f);
    return max(u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u), 1u);     // (0 is kept for "no entry")
}
__device__ __forceinline__ unsigned long long select_key(uint32_t order, int i) {
    return ((unsigned long long)order << 32) | (uint32_t)(0x7FFFFFFF - i);
}
__device__ __forceinline__ float select_key_value(unsigned long long k) {
    uint32_t u = (uint32_t)(k >> 32);
    u ^= (u & 0x80000000u) ? 0x80000000u : 0xFFFFFFFFu;
    return __uint_as_float(u);
}
// Largest key of a wave, the same in every lane: the order words first, then the index words of the
// lanes that hold the largest.  Lane-to-lane moves inside the vector unit (row shifts, then the two
// row broadcasts) instead of 12 dependent trips through LDS (12.6 -> 8.1 us at four winners of 32000).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
#define DPP_MAX(ctrl) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, 0xF, 0xF, false))
    DPP_MAX(0x111); DPP_MAX(0x112); DPP_MAX(0x114); DPP_MAX(0x118);      // row_shr 1, 2, 4, 8
    DPP_MAX(0x142); DPP_MAX(0x143);                                      // row_bcast 15, 31
#undef DPP_MAX
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ unsigned long long wave_max_key(unsigned long long k) {
    const uint32_t order = (uint32_t)(k >> 32), top = wave_max_u32(order);
    return ((unsigned long long)top << 32) | wave_max_u32(order == top ? (uint32_t)k : 0u);
}
#define SELECT_THREADS 1024
// START: the sequences' lengths are copied too (launch_select); a branch on the pointer instead cost every launch 0.08 us.
template <bool START>
__global__ __launch_bounds__(SELECT_THREADS) void select_kernel(const float *__restrict__ logits, TemplateDev t,
                                                                int vocab, int kmax, int32_t *__restrict__ argmax,
                                                                int32_t *__restrict__ topk_ids,
                                                                float *__restrict__ topk_val,
                                                                const int32_t *__restrict__ ctx_len,
                                                                int32_t *__restrict__ ctx_start) {
    constexpr int NW = SELECT_THREADS / 64;
    __shared__ unsigned long long sk[2][NW];          // wave results, in turn: one barrier per winner
    const int b = blockIdx.y, wave = threadIdx.x >> 6;
    // mask rows (k winners) are dealt out first: theirs are the long workgroups
    const int n_mask_sel = gridDim.x - t.n_tree;
    if (START && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) ctx_start[b] = ctx_len[b];
    const int sel = (int)blockIdx.x < n_mask_sel ? t.n_tree + blockIdx.x : blockIdx.x - n_mask_sel;   // 0..T-1 tree rows, then G*n mask rows
    const bool is_tree = sel < t.n_tree;
    const int r = is_tree ? sel : t.mask_rows[sel - t.n_tree];
    const int k = is_tree ? 1 : kmax;
    const float4 *row = reinterpret_cast<const float4 *>(logits + ((int64_t)b * t.rows + r) * vocab);   // vocab % 16 == 0
    const int n4 = vocab >> 2;
    // this thread's best: its entries come in ascending index, so a strictly larger one replaces
    uint32_t best_order = 0;
    int best_i = 0x7FFFFFFF;                           // (key 0, below every real key: no entry yet)
    auto scan = [&](const float4 &q, int i4) __attribute__((always_inline)) {
        const float v[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const uint32_t o = select_order(v[e]);
            if (o > best_order) { best_order = o; best_i = 4 * i4 + e; }
        }
    };
    constexpr int BATCH = 8;                           // independent 16-byte loads per thread and round trip
    for (int base = 0; base < n4; base += BATCH * SELECT_THREADS) {
        float4 cq[BATCH];
#pragma unroll
        for (int j = 0; j < BATCH; j++) cq[j] = row[min(base + (int)threadIdx.x + j * SELECT_THREADS, n4 - 1)];   // (slots past the row are skipped below)
#pragma unroll
        for (int j = 0; j < BATCH; j++) {
            const int i4 = base + threadIdx.x + j * SELECT_THREADS;
            if (i4 < n4) scan(cq[j], i4);
        }
    }
    unsigned long long mine = select_key(best_order, best_i);
    unsigned long long wave_best = wave_max_key(mine);
    for (int p = 0; p < k; p++) {
        if ((threadIdx.x & 63) == 0) sk[p & 1][wave] = wave_best;
        __syncthreads();
        const unsigned long long best = wave_max_key(sk[p & 1][threadIdx.x & (NW - 1)]);
        if (threadIdx.x == 0) {
            const int bi = 0x7FFFFFFF - (int)(uint32_t)(best & 0xFFFFFFFFu);
            if (is_tree) {
                argmax[b * t.n_tree + sel] = bi;
            } else {
                const int64_t o = ((int64_t)b * (t.n_groups * t.n_mask) + (sel - t.n_tree)) * kmax + p;
                topk_ids[o] = bi;
                if (topk_val) topk_val[o] = select_key_value(best);
            }
        }
        if (p + 1 == k || wave_best != best) continue;           // wave-uniform: another wave's entry won
        // the owner's share of the row, one 16-byte piece per lane of its wave (from L2: one round trip)
        const int owner = __builtin_ctzll(__builtin_amdgcn_ballot_w64(mine == best));     // (keys are distinct: one lane)
        unsigned long long next = 0;
        for (int i4 = (wave << 6) + owner + (threadIdx.x & 63) * SELECT_THREADS; i4 < n4; i4 += 64 * SELECT_THREADS) {
            const float4 q = row[i4];
            const float v[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const unsigned long long key = select_key(select_order(v[e]), 4 * i4 + e);
                next = (key < best && key > next) ? key : next;
            }
        }
        next = wave_max_key(next);
        if ((threadIdx.x & 63) == owner) mine = next;
        wave_best = wave_max_key(mine);
    }
}

// ---------------------------------------------------------------------------------------
// One row per sequence out of a pass' slab (both planes, 16-byte granules) and residual stream.
// A few KB per row: nothing but launch and one round trip.
__global__ void gather_rows_kernel(const int32_t *__restrict__ sel_row, int rows, const uint16_t *__restrict__ a_frag, int K,
                                   const float *__restrict__ x, int d, uint16_t *__restrict__ a_out, float *__restrict__ x_out) {
    const int b = blockIdx.x, batch = gridDim.x, i = blockIdx.y * blockDim.x + threadIdx.x;
    const int row = b * rows + min(max(sel_row[b], 0), rows - 1), M = batch * rows;
    if (i < (K >> 3)) {
        const int ks = K >> 5, mt_in = (M + 15) >> 4, mt_out = (batch + 15) >> 4, off_in = frag_pack_offset(M), off_out = frag_pack_offset(batch);
#pragma unroll
        for (int plane = 0; plane < 2; plane++)
            *reinterpret_cast<uint4 *>(a_out + frag_index(plane, b, 8 * i, ks, mt_out, off_out)) =
                *reinterpret_cast<const uint4 *>(a_frag + frag_index(plane, row, 8 * i, ks, mt_in, off_in));
    }
    if (i < (d >> 2)) reinterpret_cast<float4 *>(x_out + (int64_t)b * d)[i] = reinterpret_cast<const float4 *>(x + (int64_t)row * d)[i];
}

// ---------------------------------------------------------------------------------------
void launch_gather_rows(const int32_t *sel_row, int batch, int rows, const void *a_frag, int k, const float *x, int d,
                        void *a_out, float *x_out, hipStream_t s) {
    const int n = (k >> 3) > (d >> 2) ? (k >> 3) : (d >> 2);
    hipLaunchKernelGGL(gather_rows_kernel, dim3(batch, (n + 255) / 256), dim3(256), 0, s, sel_row, rows, (const uint16_t *)a_frag, k,
                       x, d, (uint16_t *)a_out, x_out);
}
void launch_embed_prep(const int32_t *token, const BuildSource &build, const TemplateDev &t, int batch, const void *tok_emb, const void *mask_emb, int d,
                       int vocab, const void *gain, float *x, void *h_frag, float *ssq, hipStream_t s) {
    const EmbedSource e = {token, t.is_mask, t.mask_index, (const uint16_t *)tok_emb, (const uint16_t *)mask_emb, t.rows, vocab};
    hipLaunchKernelGGL(rmsnorm_prep_kernel<true>, slab_grid(batch * t.rows, (d + 1023) / 1024), dim3(256), 0, s, x, (const float *)nullptr, 0,
                       batch * t.rows, d, (const uint16_t *)gain, (uint16_t *)h_frag, ssq, e, build, t);
}
void launch_rmsnorm_prep(float *x, const float *partial, int splits, int M, int d, const void *gain,
                         void *h_frag, float *ssq, hipStream_t s) {
    hipLaunchKernelGGL(rmsnorm_prep_kernel<false>, slab_grid(M, (d + 1023) / 1024), dim3(256), 0, s, x, partial, splits, M, d,
                       (const uint16_t *)gain, (uint16_t *)h_frag, ssq, EmbedSource{}, BuildSource{}, TemplateDev{});
}
void launch_qkv_rope(const float *partial, int splits, int batch, const TemplateDev &t, int Hq,
                     int Hkv, int hd, const int32_t *ctx_len, const float *rope_cos,
                     const float *rope_sin, int max_pos, void *q, void *q_lo, void *k_tree, void *v_tree,
                     void *k_tree_lo, void *v_tree_lo, const RowScale &rs, hipStream_t s) {
    const int per_wg = ROPE_THREADS / (hd / 8);
    hipLaunchKernelGGL(hd == 128 ? qkv_rope_kernel<128> : qkv_rope_kernel<64>, dim3(batch * t.rows, (Hq + 2 * Hkv + per_wg - 1) / per_wg),
                       dim3(ROPE_THREADS), 0, s, partial, ctx_len, t.depth,
                       rs.ssq, splits, batch * t.rows, t.rows, Hq, Hkv, max_pos, rope_cos, rope_sin,
                       (uint16_t *)q, (uint16_t *)q_lo, (uint16_t *)k_tree, (uint16_t *)v_tree,
                       (uint16_t *)k_tree_lo, (uint16_t *)v_tree_lo, rs.chunks, rs.inv_d, rs.eps);
}
void launch_silu_mul(const float *partial, int splits, int M, int F, void *act_frag, const RowScale &rs,
                     hipStream_t s) {
    const int n8 = ((F + 31) / 32) * 4;                       // threads (8 features each) per row
    hipLaunchKernelGGL(silu_mul_kernel, slab_grid(M, (n8 + 127) / 128), dim3(128), 0, s, partial, splits, M, F,
                       (uint16_t *)act_frag, rs);
}
void launch_select(const float *logits, int batch, const TemplateDev &t, int vocab, int kmax,
                   int32_t *argmax, int32_t *topk_ids, float *topk_val, hipStream_t s, const int32_t *ctx_len, int32_t *ctx_start) {
    const int n_sel = t.n_tree + (topk_ids ? t.n_groups * t.n_mask : 0);
    hipLaunchKernelGGL(ctx_start ? select_kernel<true> : select_kernel<false>, dim3(n_sel, batch), dim3(SELECT_THREADS), 0, s, logits, t, vocab, kmax,
                       argmax, topk_ids, topk_val, ctx_len, ctx_start);
}
