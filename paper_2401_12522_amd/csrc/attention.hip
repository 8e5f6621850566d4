// Tree-masked attention of the verify pass (Sec. 3.2, "tree-based attention"): every row of
// the pass attends to all cached tokens and to its ancestors-or-self among the rows of the
// pass; mask-token rows additionally attend to the per-layer prompt prefix.
//
// Flash-style, one workgroup per (sequence, query head, 16 query rows, key split), or, where query heads share
// a K/V head, per 32 queries of several heads and correspondingly fewer rows:
//  * A workgroup owns one tile of 16 queries, or two, and walks the key axis
//    [prefix | cache | pass rows] in chunks of 32 key slots.  Its 8 wavefronts, or 4 of two workgroups
//    per CU (two per SIMD, so that one wave's softmax arithmetic overlaps the other's matrix instructions) take
//    chunks round-robin and never synchronise inside the loop: each keeps its own
//    online-softmax state, merged through LDS once at the end (fixed order, deterministic).  With 16 rows
//    per workgroup no split over the keys is needed to fill the chip at the verify shapes,
//    so the output is normalised and written in place (no partial results, no second kernel)
//    unless the context is long enough for the planner to ask for key splits.
//  * Where many workgroups of single heads would queue, two or four neighbouring row tiles of a head run as one workgroup
//    whose waves share every chunk (T below): each fetches its part of it into one of two buffers of the key group,
//    and a barrier per chunk keeps them in step.
//  * Workgroups that read the same K/V head are placed on the same XCD (consecutive workgroup
//    ids go round-robin over the 8 XCDs), so a head's K/V comes from HBM once and from that
//    XCD's L2 for the other m-tiles and query heads of the group.
//  * K and V chunks go straight into LDS with global->LDS loads, row-major with an XOR swizzle
//    of the 16-byte columns; K is read back as A-operand fragments, V transposed
//    (ds_read_tr16_b64) as the A operand of O^T = V^T P^T.  A wave owns one 16 KiB chunk buffer:
//    it pulls all fragments of a chunk into registers first and refills the buffer with the
//    next chunk while it multiplies, the loads interleaved with the QK^T matrix instructions.
//  * S^T = K Q^T is computed so that its accumulator layout is already the B-operand layout
//    of O^T = V^T P^T: the probabilities never leave registers.  Queries, probabilities and
//    the pass rows' K/V are each two bf16 planes (value and rounding residual).
//  * The K/V of the pass rows are not yet rounded to the cache format.  A chunk over the pass
//    rows holds 16 keys, each followed (4 slots later inside a lane's 8-slot group) by a
//    partner slot carrying the low plane; the two scores are added and the probability is
//    copied to the partner before P.V, all lane-locally.
//  * The tree mask is derived from per-row ancestor bitsets and only evaluated in chunks that
//    touch the prefix, the ragged end of the cache or the pass rows.  A parent always has a
//    smaller row index than its child, so a workgroup skips pass-row chunks beyond its rows.
#include "common.h"
#include <type_traits>

#define ATT_CHUNK 32            // key slots per chunk
#define ATT_GRID_Y_LG 15        // log2 of the grid's y extent where the K/V heads are more (65535 at most are launched)

// one all-zero K/V row (head dim <= 128): padding slots read it like any other row
static __device__ uint4 g_att_zero_row[16] = {};

// 2^x for x <= 0 or -inf (softmax arguments): the bare hardware instruction, without the
// denormal-range fix-up of exp2f (results below 2^-126 flush to zero, which is what we want)
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// two floats -> packed bf16 pair, round to nearest even (gfx950 has a native conversion)
__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
    typedef __attribute__((ext_vector_type(2))) float f32x2_t;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// max / sum over the 4 lanes l, l^16, l^32, l^48 (the 16-lane groups of a wave) with the
// gfx950 row swaps: permlane32_swap(a, b) returns ([a.lanes0-31, b.lanes0-31],
// [a.lanes32-63, b.lanes32-63]); permlane16_swap does the same with rows 1 and 2 of each half
__device__ __forceinline__ float max_over_lane_groups(float x) {
    typedef __attribute__((ext_vector_type(2))) unsigned u32x2_t;
    u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_over_lane_groups(float x) {
    typedef __attribute__((ext_vector_type(2))) unsigned u32x2_t;
    u32x2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// wait until at most N vector-memory operations of this wave are outstanding and all of its
// LDS reads have returned; nothing may be moved across it
template <int N>
__device__ __forceinline__ void att_wait() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0x0 << 8));
    asm volatile("" ::: "memory");
}
template <int I, int N, typename F>
__device__ __forceinline__ void att_static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        att_static_for<I + 1, N>(f);
    }
}

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// Transposed 16-bit LDS read (ds_read_b64_tr_b16): lane j of a 16-lane group receives, as
// element e, column j%4 of the four 16-bit values that lane 4e + j/4 of the group addressed.
// Issued as bare instructions: the V chunks reach LDS through global->LDS loads whose
// completion this kernel tracks itself (att_wait), and the compiler, unable to tell the ring
// slots apart, would otherwise drain every outstanding load before each such read.  The
// results are only valid after lds_wait_all().
template <int OFFSET>
__device__ __forceinline__ s16x4 lds_read_tr16(uint32_t lds_addr) {
    static_assert(OFFSET >= 0 && OFFSET < 65536, "ds offset field");
    s16x4 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(lds_addr), "n"(OFFSET));
    return v;
}
template <int OFFSET>
__device__ __forceinline__ u32x4 lds_read_b128(uint32_t lds_addr) {
    static_assert(OFFSET >= 0 && OFFSET < 65536, "ds offset field");
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(lds_addr), "n"(OFFSET));
    return v;
}
// wait for every LDS read of this wave; the registers pass through the statements so that no
// use of them can be scheduled ahead of the wait
template <int N, int M>
__device__ __forceinline__ void lds_wait_all(u32x4 (&k)[2][N], s16x4 (&v)[M][2]) {
    static_assert((N == 2 && M == 4) || (N == 4 && M == 8), "head dim 64 or 128");
    if constexpr (N == 4) {
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(k[0][0]), "+v"(k[0][1]), "+v"(k[0][2]), "+v"(k[0][3]), "+v"(k[1][0]), "+v"(k[1][1]),
                       "+v"(k[1][2]), "+v"(k[1][3]));
        asm volatile("" : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[1][0]), "+v"(v[1][1]), "+v"(v[2][0]), "+v"(v[2][1]),
                          "+v"(v[3][0]), "+v"(v[3][1]));
        asm volatile("" : "+v"(v[4][0]), "+v"(v[4][1]), "+v"(v[5][0]), "+v"(v[5][1]), "+v"(v[6][0]), "+v"(v[6][1]),
                          "+v"(v[7][0]), "+v"(v[7][1]));
    } else {
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(k[0][0]), "+v"(k[0][1]), "+v"(k[1][0]), "+v"(k[1][1]));
        asm volatile("" : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[1][0]), "+v"(v[1][1]), "+v"(v[2][0]), "+v"(v[2][1]),
                          "+v"(v[3][0]), "+v"(v[3][1]));
    }
}

// U tiles of 16 queries per wave, W waves per workgroup, of which T neighbours share every chunk
template <int HD, int U, int W, int T = 1>
struct AttCfg {
    static constexpr int KSN = HD / 32;                       // k-steps of the QK^T contraction
    static constexpr int NTN = HD / 16;                       // 16-wide tiles of the head dimension
    static constexpr int GPR = HD / 8;                        // 16-byte granules per K/V row
    static constexpr int RPI = 64 / GPR;                      // V rows per global->LDS instruction
    static constexpr int NVI = ATT_CHUNK / RPI;               // such instructions per chunk
    static constexpr int KV_BYTES = ATT_CHUNK * HD * 2;       // the K (or V) rows of one chunk
    static constexpr int CHUNK_BYTES = 2 * KV_BYTES;          // one ring slot: [K rows | V rows]
    static constexpr int G = W / T;                           // key groups: waves, or sets of T, with chunks of their own
    static constexpr int IPW = NVI / T;                       // load instructions (K, and V) per wave and chunk
    static constexpr int BUFS = T > 1 ? 2 : 1;                // chunk buffers per key group
    static constexpr int RING_BYTES = G * BUFS * CHUNK_BYTES;
    // the merge: every wave's tiles over the chunk buffers, and behind them its rows' maxima and sums
    static constexpr int MERGE_BYTES = U * W * NTN * 64 * 16, ML_BYTES = 2 * U * W * 16 * 4;
    static constexpr int ML = RING_BYTES > MERGE_BYTES ? RING_BYTES : MERGE_BYTES;
    static constexpr int SMEM = ML + ML_BYTES;
};

// LDS row of key slot s inside a V chunk: the two 4-slot halves of each lane group's 8 slots
// are kept 16 rows apart, so that one transposed read (16 rows x 32 bytes per half wave)
// touches 8 consecutive rows per 32 lanes.
__device__ __forceinline__ int att_slot_of_row(int rho) { return 8 * ((rho & 15) >> 2) + 4 * (rho >> 4) + (rho & 3); }
// XOR swizzle of the 32-byte column pairs of an LDS row (in 16-byte granules): 8 consecutive
// rows land on 8 different bank groups
template <int HD>
__device__ __forceinline__ constexpr int att_swizzle(int rho) { return HD == 128 ? 2 * (rho & 7) : 2 * ((rho >> 1) & 3); }
// The K rows are read as A-operand fragments, 16 lanes fetching the same 16-byte column of 16
// consecutive rows: there the granule index is XORed with 4 (3) bits of the row.
template <int HD>
__device__ __forceinline__ constexpr int att_swizzle_k(int rho) { return HD == 128 ? (rho & 15) : ((rho >> 1) & 7); }

// PAGED: the cache operands are page pools [n_pages][Hkv][page][HD] and key slot s of sequence b
// lives in page table[b][s >> page_lg] at row s & (page - 1); the sequence's table entries are
// copied to LDS (behind the chunk buffers) once per workgroup.
// RANKED: the sequences take their turns longest first (up to 8 of them).
template <int HD, int U, int W, int T, bool PAGED, bool RANKED>
__global__ __launch_bounds__(W * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void tree_attn_kernel(
    // the first 14 dwords arrive in scalar registers with the wave (kernel-argument preload):
    // what the workgroup needs to find its work and to issue its first loads comes first
    const int32_t *__restrict__ ctx_len, int batch, int qpk /* query heads per K/V head */, int Hkv, int n_mt_lg, int n_splits, int P, int R, int smax,
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ q_lo,
    TemplateDev t, const uint16_t *__restrict__ k_cache, const uint16_t *__restrict__ v_cache,
    const uint16_t *__restrict__ k_tree, const uint16_t *__restrict__ v_tree,
    const uint16_t *__restrict__ k_tree_lo, const uint16_t *__restrict__ v_tree_lo,
    const uint16_t *__restrict__ prompt_k, const uint16_t *__restrict__ prompt_v,
    const int32_t *__restrict__ token, float scale_log2, float *__restrict__ part_o, float *__restrict__ part_ml,
    uint16_t *__restrict__ out, uint16_t *__restrict__ out_lo, int as_fragments, int m_tiles_out, PageMap pm,
    const int32_t *__restrict__ only_row) {
    using C = AttCfg<HD, U, W, T>;
    constexpr int G = C::G, IPW = C::IPW;
    constexpr int KSN = C::KSN, NTN = C::NTN, GPR = C::GPR, RPI = C::RPI, NVI = C::NVI;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    const int Hq = qpk * Hkv;
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, and known to be
    // ---- workgroup id -> (kv group, query head of the group, m-tile, split), kv groups dealt
    //      round-robin to the XCDs (grid x runs over the XCDs first)
    const int group = (blockIdx.x & 7) + 8 * (blockIdx.y + (blockIdx.z << ATT_GRID_Y_LG));     // (sequence, kv head)
    if (group >= batch * Hkv) return;
    int w_in = blockIdx.x >> 3, split = 0;
    if (n_splits > 1) {                                      // (each integer division is 25 scalar instructions)
        split = w_in % n_splits;
        w_in /= n_splits;
    }
    // A tile's 16 query lanes are 2^lg_rows rows of 2^lg_ht heads (one head per workgroup: 16 rows of it); the
    // workgroup's second tile has the same rows of the next heads.
    const int n_mt = n_mt_lg & 0xFFFF, lg_ht = U > 1 ? (n_mt_lg >> 16) & 0xFF : 0, lg_rows = 4 - lg_ht;
    const int qh = w_in / n_mt;
    int mt = n_mt - 1 - (w_in - qh * n_mt);                                  // long m-tiles (sets of T of them) first
    const int kgrp = T > 1 ? wave / T : wave, tsub = T > 1 ? wave % T : 0;   // key group, tile of the set
    const int turn = group / Hkv, kvh = group - turn * Hkv;
    int b = turn, Lc;
    if constexpr (RANKED) {                                                     // lane 8i + j compares sequences i and j
        const int i = lane >> 3, j = lane & 7;
        const int mine = ctx_len[min(i, batch - 1)], other = ctx_len[min(j, batch - 1)];
        const uint64_t before = __builtin_amdgcn_ballot_w64(j < batch && (other > mine || (other == mine && j < i)));
        const int place = __popc((uint32_t)(before >> (8 * i)) & 0xFFu);
        const int at = __builtin_ctzll(__builtin_amdgcn_ballot_w64(i < batch && place == turn));
        b = at >> 3;
        Lc = __builtin_amdgcn_readlane(mine, at);
    } else {
        Lc = ctx_len[b];
    }
    // One row per sequence is asked for (bit 24, known without a load, so that other launches do not wait for one): only
    // its row tile is launched.  A prefill's last layer, 488 rows on 512, 32 heads: 27.7 -> 17.9 us, the other tiles'
    // workgroups leaving behind their first chunk before.  (Two tiles per workgroup have no registers for it: a spill, 1 %
    // of every launch.  They leave below.)
    if (U == 1 && T == 1 && (n_mt_lg >> 24)) mt = min(max(only_row[b], 0), R - 1) >> lg_rows;
    const int h0 = kvh * qpk + (U > 1 ? qh << (1 + lg_ht) : qh);                // the workgroup's first head

    const int32_t *tbl = reinterpret_cast<const int32_t *>(smem + C::SMEM);
    const int page_lg = pm.page_lg, page_mask = (1 << pm.page_lg) - 1;
    if (PAGED) {
        // never walk past the table entries the launch made room for; page ids are clamped to
        // the pool, so a bad table gives wrong data, not a fault
        Lc = min(Lc, pm.tbl_cap << page_lg);
        int32_t *dst = reinterpret_cast<int32_t *>(smem + C::SMEM);
        const int n_used = (Lc + page_mask) >> page_lg;
        for (int i = tid; i < n_used; i += W * 64)
            dst[i] = min(max(pm.table[(int64_t)b * pm.max_pages + i], 0), pm.n_pages - 1);
        __syncthreads();
    }
    const int row0 = (mt * T + tsub) << lg_rows, row_end = min(R, (mt + 1) * T << lg_rows);   // of the wave, of the workgroup
    const int n_ctx_keys = P + Lc;
    const int n_cc = (n_ctx_keys + ATT_CHUNK - 1) / ATT_CHUNK;           // chunks over [prefix | cache]
    const int n_tc = (row_end + 15) >> 4;                                // chunks over the pass rows
    const int n_chunks = n_cc + n_tc;
    const int per_split = (n_chunks + n_splits - 1) / n_splits;
    const int chunk_begin = split * per_split;
    const int chunk_end = min(n_chunks, chunk_begin + per_split);
    // this wave's chunks: chunk_begin + kgrp + G * i, i < n_my (waves that share go round as often as the first key group)
    const int n_my = max(0, (chunk_end - chunk_begin - kgrp + G - 1) / G);

    const uint16_t *pk = prompt_k + (int64_t)kvh * P * HD, *pv = prompt_v + (int64_t)kvh * P * HD;
    const int64_t page_stride = (int64_t)Hkv * HD << page_lg;           // elements per page (all kv heads)
    const uint16_t *ck = k_cache + (PAGED ? ((int64_t)kvh * HD << page_lg) : ((int64_t)b * Hkv + kvh) * smax * HD);
    const uint16_t *cv = v_cache + (PAGED ? ((int64_t)kvh * HD << page_lg) : ((int64_t)b * Hkv + kvh) * smax * HD);
    // element offset of cache slot j of this (sequence, kv head) from ck / cv
    auto slot_off = [&](int j) __attribute__((always_inline)) -> int64_t {
        if (!PAGED) return (int64_t)j * HD;
        return (int64_t)tbl[j >> page_lg] * page_stride + (int64_t)(j & page_mask) * HD;
    };
    // a chunk of cache slots j0 .. j0+ATT_CHUNK-1 has one base address (always, when contiguous)
    auto one_page = [&](int j0) __attribute__((always_inline)) -> bool {
        return !PAGED || (j0 >> page_lg) == ((j0 + ATT_CHUNK - 1) >> page_lg);
    };
    const int64_t tree_off = ((int64_t)b * Hkv + kvh) * R * HD;
    const uint16_t *tk = k_tree + tree_off, *tv = v_tree + tree_off;
    const uint16_t *tk_lo = k_tree_lo ? k_tree_lo + tree_off : nullptr;
    const uint16_t *tv_lo = v_tree_lo ? v_tree_lo + tree_off : nullptr;
    const uint16_t *zero = reinterpret_cast<const uint16_t *>(g_att_zero_row);

    // ---- query fragments (B operand of S^T = K Q^T) stay in registers: lane (g, c) holds
    //      Q[row0 + c][32ks + 8g .. +8] of both planes; rows beyond R are zero
    //      All loads of this prologue (mask byte, token, query fragments) are unconditional, from
    //      a clamped row, and their values are first looked at behind the wait for the first chunk:
    //      one memory round trip instead of one per dependent condition.
    const int rq = row0 + (c & ((1 << lg_rows) - 1)), hq = h0 + (c >> lg_rows);   // tile u: head hq + (u << lg_ht)
    const bool row_ok = rq < R;
    const int rqc = min(rq, R - 1);
    const uint32_t mask_byte = t.is_mask[rqc];
    const int32_t *tok_src = token ? token + (int64_t)b * R + rqc : reinterpret_cast<const int32_t *>(g_att_zero_row);
    const int32_t tok_val = *tok_src;
    bool row_mask = false;                               // set behind the first wait
    bf16x8 qf[U][2][KSN];
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
        for (int pl = 0; pl < 2; pl++) {
            const uint16_t *src = (pl && q_lo) ? q_lo : q;
            const bool live = row_ok && (pl == 0 || q_lo);
#pragma unroll
            for (int ks = 0; ks < KSN; ks++) {
                uint4 v = *reinterpret_cast<const uint4 *>(src + (((int64_t)b * R + rqc) * Hq + hq + (u << lg_ht)) * HD + ks * 32 + g * 8);
                if (!live) v = make_uint4(0, 0, 0, 0);
                qf[u][pl][ks] = __builtin_bit_cast(bf16x8, v);
            }
        }

    f32x4 o_acc[U][NTN];
    float m_run[U], base_m[U], l_run[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
#pragma unroll
        for (int nt = 0; nt < NTN; nt++) o_acc[u][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        m_run[u] = -INFINITY;
        base_m[u] = 0.f;
        l_run[u] = 0.f;
    }

    unsigned char *v_ring = smem + kgrp * (C::BUFS * C::CHUNK_BYTES);  // the key group's chunk buffer, or two that take turns
    // LDS addresses of this lane's transposed V reads inside ring slot 0: lane (g, c) addresses
    // V[slot 8g + 4half + c/4][16nt + 4(c%4) .. +4] and receives V[slots 8g + 4half .. +4][16nt + c]
    // ... and of its K fragment reads: sub-tile tt, k-step ks = row 16tt + c, granule 4ks + g
    // (both swizzles ignore bit 4 of the row, so the second sub-tile / half is the same address
    // plus 16 rows: an immediate offset of the read)
    static_assert(att_swizzle_k<HD>(16) == 0 && att_swizzle<HD>(16) == 0, "row bit 4 outside the swizzles");
    constexpr int ROWS16 = 16 * HD * 2;
    // The k-step and the head-dim tile sit in address bits that neither the row nor the ring slot
    // touches: one register each, the others an exclusive-or away (11 registers less, which two heads
    // per workgroup spilled before).
    const uint32_t k_addr = (uint32_t)(size_t)((__attribute__((address_space(3))) unsigned char *)v_ring) +
                            c * (HD * 2) + ((g ^ att_swizzle_k<HD>(c)) * 16);
    const uint32_t v_addr = (uint32_t)(size_t)((__attribute__((address_space(3))) unsigned char *)v_ring) + C::KV_BYTES +
                            (4 * g + (c >> 2)) * (HD * 2) + ((((c & 3) >> 1)) ^ att_swizzle<HD>(4 * g + (c >> 2))) * 16 + (c & 1) * 8;

    // Per-lane byte offsets of the fast path (a chunk that lies wholly inside the cache).  Both
    // operands are copied row-major, 1 KiB (RPI rows) per global->LDS instruction: instruction
    // iv fills LDS rows iv*RPI .., LDS row rho holds key slot att_slot_of_row(rho), and the lane
    // at granule position p of that row fetches granule p ^ swizzle(rho).  The swizzles depend
    // on iv only through iv%4 (K) and iv%2 (V).
    // In a chunk over the pass rows slot s is pass row 4*(s>>3) + (s&3) of the chunk's 16, plane
    // (s>>2)&1; the instruction's first slot and the lane's slot inside the instruction occupy
    // disjoint bits, so row and plane split the same way (the plane is uniform per instruction).
    const int v_lane_row = lane / GPR;                                  // row inside one instruction
    const int lane_slot = att_slot_of_row(v_lane_row);
    const int lane_tree_row = 4 * (lane_slot >> 3) + (lane_slot & 3);

    // The two global->LDS loads (one K, one V instruction) number iv < NVI of this wave's stage i,
    // the mask word riding with the last.  A chunk wholly inside the cache takes one uniform base
    // per operand plus the constant lane offsets; the other cases select per lane.
    typedef const __attribute__((address_space(1))) unsigned char *gptr;   // keeps the loads global, not flat
    uint64_t anc_next = 0;                                              // ancestor bits for the stage in flight
    auto emit = [&](int i, int j_iv) __attribute__((always_inline)) {
        const int iv = T > 1 ? tsub * IPW + j_iv : j_iv;
        unsigned char *buf = T > 1 ? v_ring + (i & 1) * C::CHUNK_BYTES : v_ring;
        const int chunk = chunk_begin + kgrp + G * i;
        const int base = chunk * ATT_CHUNK;
        const uint32_t k_gran_iv = ((lane % GPR) ^ att_swizzle_k<HD>((iv & 3) * RPI + v_lane_row)) * 16;
        const uint32_t v_gran_iv = ((lane % GPR) ^ att_swizzle<HD>((iv & 1) * RPI + v_lane_row)) * 16;
        const unsigned char *zero_b = reinterpret_cast<const unsigned char *>(zero);
        const int slot0 = att_slot_of_row(iv * RPI);                    // slot of the instruction's first row
        gptr k_src, v_src, a_src = (gptr)(zero_b + (lane & 1) * 8);
        if (base >= P && base + ATT_CHUNK <= n_ctx_keys && one_page(base - P)) {
            const int64_t row_bytes = (slot_off(base - P) + (int64_t)(slot0 + lane_slot) * HD) * 2;
            k_src = (gptr)(reinterpret_cast<const unsigned char *>(ck) + row_bytes + k_gran_iv);
            v_src = (gptr)(reinterpret_cast<const unsigned char *>(cv) + row_bytes + v_gran_iv);
        } else if (chunk >= n_cc) {
            // over the pass rows: one plane and 4-row group per instruction, rows beyond R are zero
            const int j_first = (chunk - n_cc) * 16;
            if (row_ok) a_src = (gptr)(t.anc + (int64_t)rq * t.words + (j_first >> 6));   // ancestor bits of these 16 rows
            const int j = j_first + 4 * (slot0 >> 3) + lane_tree_row;
            const uint16_t *kp = (slot0 & 4) ? tk_lo : tk, *vp = (slot0 & 4) ? tv_lo : tv;   // uniform
            const bool k_ok = j < R && kp, v_ok = j < R && vp;
            k_src = (gptr)(reinterpret_cast<const unsigned char *>(k_ok ? kp + (int64_t)j * HD : zero) + k_gran_iv);
            v_src = (gptr)(reinterpret_cast<const unsigned char *>(v_ok ? vp + (int64_t)j * HD : zero) + v_gran_iv);
        } else {
            // a chunk with prefix rows or the ragged end of the cache
            const int kidx = base + slot0 + lane_slot;
            const bool in_prefix = kidx < P, in_cache = kidx >= P && kidx < n_ctx_keys;
            const int64_t off = in_cache ? slot_off(kidx - P) : 0;
            const uint16_t *krow = in_prefix ? pk + (int64_t)kidx * HD : (in_cache ? ck + off : zero);
            const uint16_t *vrow = in_prefix ? pv + (int64_t)kidx * HD : (in_cache ? cv + off : zero);
            k_src = (gptr)(reinterpret_cast<const unsigned char *>(krow) + k_gran_iv);
            v_src = (gptr)(reinterpret_cast<const unsigned char *>(vrow) + v_gran_iv);
        }
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)k_src,
                                         (__attribute__((address_space(3))) void *)(buf + iv * 1024), 16, 0, 0);
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)v_src,
                                         (__attribute__((address_space(3))) void *)(buf + C::KV_BYTES + iv * 1024), 16, 0, 0);
        if (j_iv == IPW - 1) anc_next = *(const __attribute__((address_space(1))) uint64_t *)a_src;
    };

    // The same two loads for a chunk known to lie wholly inside the cache (all but a handful), as
    // buffer loads: a uniform descriptor per operand, the lane's constant offset in a register, the
    // chunk's and the instruction's first row in the scalar offset: no vector instruction per load
    // and no 64-bit lane addresses, so that two heads per workgroup have the registers for it too.
    // (Descriptors span the sequence's cached slots, or those of them a page can hold; the offsets stay
    // inside.  Slots from 2^23 on would leave their 32 bits and take the general path, by the one bound
    // below, kept in a scalar register.  Lc <= 2^23 as a condition of its own in the loop cost the
    // single-head forms up to 5 %: 32/32 heads of 128, 16 sequences of 512 with 25 rows 41.8 against
    // 39.8 us, 170 rows on 1024 25.9 against 25.0; two heads: 64/8, 8 sequences of 4096 204.8 against 203.0.)
    const int desc_slots = min(Lc, 1 << 23);
    int desc_end = P + desc_slots;
    asm("" : "+s"(desc_end));
    uint32_t k_off[4], v_off[2];
#pragma unroll
    for (int par = 0; par < 4; par++) {
        const int rho = ((T > 1 ? tsub * IPW : 0) + par) * RPI + v_lane_row;                         // (source granule, in bytes, at this lane's position)
        k_off[par] = (uint32_t)lane_slot * (HD * 2) + ((lane % GPR) ^ att_swizzle_k<HD>(rho)) * 16;
        if (par < 2) v_off[par] = (uint32_t)lane_slot * (HD * 2) + ((lane % GPR) ^ att_swizzle<HD>(rho)) * 16;
    }
    auto emit_cache = [&](__amdgpu_buffer_rsrc_t kr, __amdgpu_buffer_rsrc_t vr, uint32_t chunk_bytes, unsigned char *buf, int j) __attribute__((always_inline)) {
        const int iv = T > 1 ? tsub * IPW + j : j;
        const uint32_t at = chunk_bytes + (uint32_t)att_slot_of_row(iv * RPI) * (HD * 2);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, (__attribute__((address_space(3))) void *)(buf + iv * 1024), 16, k_off[j & 3], at, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, (__attribute__((address_space(3))) void *)(buf + C::KV_BYTES + iv * 1024), 16, v_off[j & 1], at, 0, 0);
    };

    // One chunk.  Its K and V fragments are all pulled into registers first, which frees the
    // wave's LDS buffer: the next chunk's loads are issued into it right away, interleaved
    // with the QK^T matrix instructions, and have the rest of the step to land.
    auto compute = [&](int i, bool more) __attribute__((always_inline)) {
        const uint64_t anc_cur = anc_next;
        const int chunk = chunk_begin + kgrp + G * i;
        const bool tree_chunk = chunk >= n_cc;
        const int base = chunk * ATT_CHUNK;
        u32x4 kf[2][KSN];
        uint32_t ka = k_addr, va = v_addr;
        if constexpr (T > 1) {
            ka += (i & 1) * C::CHUNK_BYTES;
            va += (i & 1) * C::CHUNK_BYTES;
        }
        if constexpr (U > 1 && HD == 128) asm volatile("" : "+v"(ka), "+v"(va));   // (the derived addresses are not kept across chunks)
#pragma unroll
        for (int ks = 0; ks < KSN; ks++) {
            kf[0][ks] = lds_read_b128<0>(ka ^ (64 * ks));
            kf[1][ks] = lds_read_b128<ROWS16>(ka ^ (64 * ks));
        }
        s16x4 vh[NTN][2];
#pragma unroll
        for (int nt = 0; nt < NTN; nt++) {
            vh[nt][0] = lds_read_tr16<0>(va ^ (32 * nt));
            vh[nt][1] = lds_read_tr16<ROWS16>(va ^ (32 * nt));
        }
        lds_wait_all(kf, vh);
        f32x4 s_acc[U][2];
#pragma unroll
        for (int u = 0; u < U; u++) s_acc[u][0] = s_acc[u][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        static_assert(NVI == 2 * KSN, "one (k-step, sub-tile) pair per load slot");
        auto qk = [&](int iv) __attribute__((always_inline)) {
            const int ks = iv >> 1, tt = iv & 1;
            const bf16x8 ka = __builtin_bit_cast(bf16x8, kf[tt][ks]);
#pragma unroll
            for (int u = 0; u < U; u++) {
                s_acc[u][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qf[u][0][ks], s_acc[u][tt], 0, 0, 0);
                s_acc[u][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qf[u][1][ks], s_acc[u][tt], 0, 0, 0);
            }
        };
        const int base_n = base + G * ATT_CHUNK;                 // the wave's next chunk
        if (more && base_n >= P && base_n + ATT_CHUNK <= desc_end && one_page(base_n - P)) {   // wave-uniform
            // contiguous: one descriptor for the sequence's slots; paged: one for the chunk's page
            const int64_t first = PAGED ? (int64_t)__builtin_amdgcn_readfirstlane(tbl[(base_n - P) >> page_lg]) * page_stride : 0;
            const uint32_t slot = PAGED ? (base_n - P) & page_mask : base_n - P;
            // (a page may be larger than a descriptor can span; what of it the sequence's first 2^23 slots
            // can lie in is not)
            const uint32_t span = (uint32_t)(PAGED ? min(1 << page_lg, desc_slots) : desc_slots) * (HD * 2);
            const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc((void *)(ck + first), 0, span, 0x00027000);
            const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc((void *)(cv + first), 0, span, 0x00027000);
            const uint32_t chunk_bytes = slot * (HD * 2);
            unsigned char *buf = T > 1 ? v_ring + ((i + 1) & 1) * C::CHUNK_BYTES : v_ring;
#pragma unroll
            for (int iv = 0; iv < NVI; iv++) {
                if (iv < IPW) emit_cache(kr, vr, chunk_bytes, buf, iv);
                __builtin_amdgcn_sched_barrier(0);
                qk(iv);
                __builtin_amdgcn_sched_barrier(0);
            }
            anc_next = 0;
        } else if constexpr (U == 1 || HD == 64) {
#pragma unroll
            for (int iv = 0; iv < NVI; iv++) {
                if (iv < IPW && more) emit(i + 1, iv);
                __builtin_amdgcn_sched_barrier(0);
                qk(iv);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            // (two heads of 128) one copy of the general loads ahead of the matrix instructions: unrolled
            // between them they cost the registers (a reload per chunk) and most of the instructions
            if (more) {
#pragma unroll 1
                for (int iv = 0; iv < IPW; iv++) emit(i + 1, iv);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int iv = 0; iv < NVI; iv++) qk(iv);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the visibility of a key depends on the row and the key only: one mask word for all heads
        const bool need_mask = tree_chunk || (base < P) || (base + ATT_CHUNK > n_ctx_keys);
        uint32_t bits = 0xFFu;
        if (need_mask) {
            // 8-bit visibility word for this lane's slots, built with integer selects only:
            // prefix -> mask rows, cache -> all rows, pass rows -> ancestor bits.
            bits = 0;
            if (row_ok) {
                if (tree_chunk) {
                    const int j0 = (chunk - n_cc) * 16 + 4 * g;          // this lane's 4 pass rows (4-aligned)
                    const uint32_t four = (uint32_t)(anc_cur >> (j0 & 63)) & 0xFu;
#pragma unroll
                    for (int e = 0; e < 4; e++) bits |= ((j0 + e < R) ? ((four >> e) & 1u) : 0u) << e;
                } else {
                    const int k0 = base + 8 * g;
#pragma unroll
                    for (int e = 0; e < 8; e++) {
                        const int kidx = k0 + e;
                        const uint32_t in_prefix = kidx < P ? 1u : 0u;
                        const uint32_t in_cache = (kidx >= P && kidx < n_ctx_keys) ? 1u : 0u;
                        bits |= ((in_prefix & (row_mask ? 1u : 0u)) | in_cache) << e;
                    }
                }
            }
        }
        s16x8 v8[NTN];
#pragma unroll
        for (int nt = 0; nt < NTN; nt++)
            v8[nt] = s16x8{vh[nt][0][0], vh[nt][0][1], vh[nt][0][2], vh[nt][0][3],
                           vh[nt][1][0], vh[nt][1][1], vh[nt][1][2], vh[nt][1][3]};
#pragma unroll
        for (int u = 0; u < U; u++) {
            // Scores in powers of two, scaled before anything else: the exponent of the largest is then exactly
            // zero.  With the scale in the exponent's multiply-add it was off by the product's rounding (1.5e-5
            // of a value at scores of 5e4) for 1 % of the two-head forms' time (64/8 heads, 8 sequences of
            // 4096: 207.4 against 209.6 us) and none of the others'.
            float sv[8];
#pragma unroll
            for (int tt = 0; tt < 2; tt++)
#pragma unroll
                for (int r = 0; r < 4; r++) sv[tt * 4 + r] = s_acc[u][tt][r] * scale_log2;
            if (tree_chunk) {                // score = q.k_hi + q.k_lo; partner slots leave the softmax
#pragma unroll
                for (int e = 0; e < 4; e++) sv[e] += sv[e + 4];
            }
            if (need_mask) {
#pragma unroll
                for (int e = 0; e < 8; e++) sv[e] = ((bits >> e) & 1u) ? sv[e] : -INFINITY;
            }
            float mx = sv[0];
#pragma unroll
            for (int e = 1; e < 8; e++) mx = fmaxf(mx, sv[e]);
            // The running maximum rarely moves after the first chunks: the lane groups are reduced and
            // the sums rescaled only where some lane's scores exceed it.  base_m is the number every
            // exponent is taken against (0 while a row has seen no key).
            float alpha = 1.f;
            if (__builtin_amdgcn_ballot_w64(mx > m_run[u]) != 0) {
                const float m_new = fmaxf(m_run[u], max_over_lane_groups(mx));
                base_m[u] = m_new == -INFINITY ? 0.f : m_new;
                alpha = fast_exp2(m_run[u] - base_m[u]);
                m_run[u] = m_new;
#pragma unroll
                for (int nt = 0; nt < NTN; nt++) o_acc[u][nt] *= alpha;
            }
            // probabilities as two bf16 planes (value and rounding residual), like every other
            // MFMA input of the pass
            float ps = 0.f;
            uint32_t pk2[4], pl2[4];
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                const float p0 = fast_exp2(sv[e] - base_m[u]), p1 = fast_exp2(sv[e + 1] - base_m[u]);
                ps += p0 + p1;
                const uint32_t hi = cvt_pk_bf16(p0, p1);
                pk2[e >> 1] = hi;
                pl2[e >> 1] = cvt_pk_bf16(p0 - __uint_as_float(hi << 16), p1 - __uint_as_float(hi & 0xFFFF0000u));
            }
            if (tree_chunk) {                // the low-plane value rows take the same probabilities
                pk2[2] = pk2[0];
                pk2[3] = pk2[1];
                pl2[2] = pl2[0];
                pl2[3] = pl2[1];
            }
            l_run[u] = l_run[u] * alpha + ps;
            // O^T[hd][q] += V^T[hd][slots 8g..8g+7] * P^T
            const bf16x8 pf = __builtin_bit_cast(bf16x8, make_uint4(pk2[0], pk2[1], pk2[2], pk2[3]));
            const bf16x8 pf_lo = __builtin_bit_cast(bf16x8, make_uint4(pl2[0], pl2[1], pl2[2], pl2[3]));
#pragma unroll
            for (int nt = 0; nt < NTN; nt++) {
                const bf16x8 vf = __builtin_bit_cast(bf16x8, v8[nt]);
                o_acc[u][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf, o_acc[u][nt], 0, 0, 0);
                o_acc[u][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf_lo, o_acc[u][nt], 0, 0, 0);
            }
        }
    };

    // ---- per-wave loop: one chunk in flight behind the one being multiplied -------------------
    if (n_my > 0) {
#pragma unroll
        for (int iv = 0; iv < IPW; iv++) emit(0, iv);
    }
    att_wait<0>();                                      // the first chunk and the prologue's loads have landed
    // (looked at here, where the prologue's loads have landed anyway: ahead of them it cost 0.5 % of
    // every launch; the whole workgroup leaves together)
    if (U > 1 && only_row && (min(max(only_row[b], 0), R - 1) >> lg_rows) != mt) return;
    // a tree row without a candidate (negative token) is absent from the pass: its output is zero
    int row_flags = (row_ok && mask_byte ? 1 : 0) | (row_ok && (mask_byte || tok_val >= 0) ? 2 : 0);
    asm volatile("" : "+v"(row_flags));                 // (looked at here, not inside the loop)
    row_mask = (row_flags & 1) != 0;
    const bool row_present = (row_flags & 2) != 0;
    if constexpr (T == 1) {
        for (int i = 0; i < n_my; i++) {
            compute(i, i + 1 < n_my);
            att_wait<0>();                              // the next chunk has landed
        }
    } else {
        // A barrier per chunk: every sharing wave's part of it has landed, and all have read the buffer that is refilled
        // next.  A wave whose rows are past the pass, or before all rows of a chunk, only loads its part.
        const int n_round = max(0, (chunk_end - chunk_begin + G - 1) / G);
        for (int i = 0; i < n_round; i++) {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            const int chunk = chunk_begin + kgrp + G * i;
            if (i < n_my && row0 < R && (chunk < n_cc || ((chunk - n_cc) << 4) < row0 + (1 << lg_rows))) {
                compute(i, i + 1 < n_my);
            } else if (i + 1 < n_my) {
#pragma unroll 1
                for (int iv = 0; iv < IPW; iv++) emit(i + 1, iv);
            }
            att_wait<0>();
        }
    }

    // ---- merge the wavefronts (disjoint key subsets): every wave leaves its maxima and sums, then its
    //      rescaled tiles in LDS, wave nt then sums tile nt of the head dimension over the waves in wave
    //      order (fixed order, deterministic) and finishes and stores those 16 columns.  All heads at a
    //      time: two barriers for the workgroup instead of three per head --------------------------------
    // (the lane's place is asked for again: kept through the loop it cost two heads per workgroup a spill)
    const int lane_m = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), g_m = lane_m >> 4, c_m = lane_m & 15;
    const int rq_m = row0 + (c_m & ((1 << lg_rows) - 1)), hq_m = h0 + (c_m >> lg_rows);
    float *sm = reinterpret_cast<float *>(smem + C::ML), *sl = sm + U * W * 16;   // [U][W][16]
    float4 *region = reinterpret_cast<float4 *>(smem);                            // [U][W][NTN][64]
#pragma unroll
    for (int u = 0; u < U; u++) {
        const float l = sum_over_lane_groups(l_run[u]);
        if (g_m == 0) {
            sm[(u * W + wave) * 16 + c_m] = m_run[u];
            sl[(u * W + wave) * 16 + c_m] = l;
        }
    }
    __syncthreads();                         // (every wave is past its chunk buffer, too)
    float m_tot[U], l_tot[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
        m_tot[u] = -INFINITY;
#pragma unroll
        for (int w = 0; w < G; w++) m_tot[u] = fmaxf(m_tot[u], sm[(u * W + w * T + tsub) * 16 + c_m]);
        const float m_use = (m_tot[u] == -INFINITY) ? 0.f : m_tot[u];
        l_tot[u] = 0.f;
#pragma unroll
        for (int w = 0; w < G; w++) l_tot[u] += sl[(u * W + w * T + tsub) * 16 + c_m] * fast_exp2(sm[(u * W + w * T + tsub) * 16 + c_m] - m_use);
        const float f = fast_exp2(m_run[u] - m_use);
#pragma unroll
        for (int nt = 0; nt < NTN; nt++)
            region[((u * W + wave) * NTN + nt) * 64 + lane_m] =
                make_float4(o_acc[u][nt][0] * f, o_acc[u][nt][1] * f, o_acc[u][nt][2] * f, o_acc[u][nt][3] * f);
    }
    __syncthreads();
    if (rq_m >= R) return;
#pragma unroll
    for (int u = 0; u < U; u++) {
        const int h = hq_m + (u << lg_ht);
#pragma unroll
        for (int nt = kgrp; nt < NTN; nt += G) {     // this wave's columns of the head, 16 at a time
            float4 o = region[((u * W + tsub) * NTN + nt) * 64 + lane_m];
#pragma unroll
            for (int w = 1; w < G; w++) {
                const float4 v = region[((u * W + w * T + tsub) * NTN + nt) * 64 + lane_m];
                o.x += v.x; o.y += v.y; o.z += v.z; o.w += v.w;
            }
            // ---- lane (g, c) holds O[row rq][hd 16nt + 4g .. +4] -----------------------------------
            if (n_splits > 1) {                  // unnormalised partial for attn_merge_kernel
                const int64_t prow = (((int64_t)b * Hq + h) * n_splits + split) * R + rq_m;
                *reinterpret_cast<float4 *>(part_o + prow * HD + nt * 16 + 4 * g_m) = o;
                if (nt == 0 && g_m == 0) {
                    part_ml[prow * 2] = m_tot[u];
                    part_ml[prow * 2 + 1] = row_present ? l_tot[u] : 0.f;      // (a zero sum makes the merge write zeros)
                }
                continue;
            }
            const float inv = (l_tot[u] > 0.f && row_present) ? 1.0f / l_tot[u] : 0.f;
            const int mrow = b * R + rq_m, n_ksteps = (Hq * HD) >> 5;
            const float ov[4] = {o.x * inv, o.y * inv, o.z * inv, o.w * inv};
            uint16_t hi[4], lo[4];
#pragma unroll
            for (int e = 0; e < 4; e++) split_bf16(ov[e], hi[e], lo[e]);
            uint2 ph, pl;
            ph.x = hi[0] | ((uint32_t)hi[1] << 16); ph.y = hi[2] | ((uint32_t)hi[3] << 16);
            pl.x = lo[0] | ((uint32_t)lo[1] << 16); pl.y = lo[2] | ((uint32_t)lo[3] << 16);
            const int k = h * HD + nt * 16 + 4 * g_m;
            if (as_fragments) {                  // two planes, the O-projection's activation slab
                const int pack_off = frag_pack_offset(batch * R);
                *reinterpret_cast<uint2 *>(out + frag_index(0, mrow, k, n_ksteps, m_tiles_out, pack_off)) = ph;
                *reinterpret_cast<uint2 *>(out + frag_index(1, mrow, k, n_ksteps, m_tiles_out, pack_off)) = pl;
            } else {
                *reinterpret_cast<uint2 *>(out + (int64_t)mrow * Hq * HD + k) = ph;
                if (out_lo) *reinterpret_cast<uint2 *>(out_lo + (int64_t)mrow * Hq * HD + k) = pl;
            }
        }
    }
}

// out[b][r][h*HD + 4i .. +4] = sum_s w_s O_s / sum_s w_s l_s,  w_s = 2^(m_s - max m).
// One thread per 4 head-dim elements; blockDim = (HD/4) * heads_per_block.
// only_row: one row per sequence (the others' partials were not written either), grid x 1.
__global__ void attn_merge_kernel(const float *__restrict__ part_o, const float *__restrict__ part_ml,
                                  int R, int Hq, int HD, int n_splits, uint16_t *__restrict__ out,
                                  uint16_t *__restrict__ out_lo, int as_fragments, int m_tiles,
                                  const int32_t *__restrict__ only_row) {
    const int per_head = HD >> 2;
    const int b = blockIdx.z, r = only_row ? min(max(only_row[b], 0), R - 1) : (int)blockIdx.x;
    const int h = blockIdx.y * (blockDim.x / per_head) + threadIdx.x / per_head, i4 = threadIdx.x % per_head;
    if (h >= Hq) return;
    const int64_t pbase = ((int64_t)b * Hq + h) * n_splits;
    float m = -INFINITY;
    for (int s = 0; s < n_splits; s++) m = fmaxf(m, part_ml[((pbase + s) * R + r) * 2]);
    const float m_use = (m == -INFINITY) ? 0.f : m;
    float l = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s = 0; s < n_splits; s++) {
        const float2 ml = *reinterpret_cast<const float2 *>(part_ml + ((pbase + s) * R + r) * 2);
        const float w = fast_exp2(ml.x - m_use);
        const float4 o = *reinterpret_cast<const float4 *>(part_o + ((pbase + s) * R + r) * HD + i4 * 4);
        l += w * ml.y;
        acc.x += w * o.x; acc.y += w * o.y; acc.z += w * o.z; acc.w += w * o.w;
    }
    const float inv = l > 0.f ? 1.0f / l : 0.f;
    const float v[4] = {acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv};
    uint16_t hi[4], lo[4];
#pragma unroll
    for (int e = 0; e < 4; e++) split_bf16(v[e], hi[e], lo[e]);
    uint2 ph, pl;
    ph.x = hi[0] | ((uint32_t)hi[1] << 16); ph.y = hi[2] | ((uint32_t)hi[3] << 16);
    pl.x = lo[0] | ((uint32_t)lo[1] << 16); pl.y = lo[2] | ((uint32_t)lo[3] << 16);
    if (as_fragments) {                     // two planes, the O-projection's activation slab
        const int mrow = b * R + r, k = h * HD + i4 * 4, n_ksteps = (Hq * HD) >> 5;
        const int pack_off = frag_pack_offset((int)gridDim.z * R);
        *reinterpret_cast<uint2 *>(out + frag_index(0, mrow, k, n_ksteps, m_tiles, pack_off)) = ph;
        *reinterpret_cast<uint2 *>(out + frag_index(1, mrow, k, n_ksteps, m_tiles, pack_off)) = pl;
    } else {
        *reinterpret_cast<uint2 *>(out + (((int64_t)b * R + r) * Hq + h) * HD + i4 * 4) = ph;
        if (out_lo) *reinterpret_cast<uint2 *>(out_lo + (((int64_t)b * R + r) * Hq + h) * HD + i4 * 4) = pl;
    }
}

AttnPlan attn_plan(int batch, int rows, int n_heads, int hd, int ctx_hint, int n_prompt) {
    AttnPlan p;
    const int n_mt = (rows + 15) / 16;
    const int n_chunks = (n_prompt + ctx_hint + ATT_CHUNK - 1) / ATT_CHUNK + n_mt;
    // (tiles of 16 rows of every head: heads that share a workgroup make fewer of them, see attn_tiles, and the split stays what
    // it is for heads by themselves)
    const int wgs = batch * n_heads * n_mt;
    // No key split while one workgroup's walk stays moderate (256 chunks = 8192 keys, 32 per
    // wave); beyond that, or when the row tiles alone leave most CUs idle on a long context,
    // split the key axis (partials + merge kernel) into shares of at least 16 chunks.
    int splits = (n_chunks + 255) / 256;
    if (wgs * splits < 128) {
        int fill = 256 / wgs;
        if (fill > n_chunks / 16) fill = n_chunks / 16;
        if (fill > splits) splits = fill;
    }
    if (splits < 1) splits = 1;
    if (splits > 64) splits = 64;
    const int per = (n_chunks + splits - 1) / splits;
    splits = (n_chunks + per - 1) / per;
    p.splits = splits;
    p.chunks = n_chunks;
    p.part_o_bytes = (size_t)batch * n_heads * splits * rows * hd * sizeof(float);
    p.part_ml_bytes = (size_t)batch * n_heads * splits * rows * 2 * sizeof(float);
    return p;
}

// How a launch is cut into workgroups, from nothing but its sizes.  table_entries: of a sequence's page table, 0 for a
// contiguous cache.
static size_t att_table_bytes(int entries) { return (size_t)((entries + 3) / 4) * 16; }
static size_t att_smem_four(int hd, int tiles) {
    return hd == 128 ? (tiles == 2 ? AttCfg<128, 2, 4>::SMEM : AttCfg<128, 1, 4>::SMEM) : (tiles == 2 ? AttCfg<64, 2, 4>::SMEM : AttCfg<64, 1, 4>::SMEM);
}
AttnTiles attn_tiles(int batch, int rows, int Hq, int Hkv, int hd, const AttnPlan &p, int table_entries, bool one_row) {
    // Grouped-query models: a workgroup's two tiles of 16 queries share its chunk loads.  The tiles take as many heads
    // of the K/V head's group as a power of two divides evenly, and so fewer rows: eight heads of 4 rows for 64/8 heads,
    // 17 workgroups per K/V head for the 68 rows of a 64-node tree where pairs of heads with 16 rows each took 20
    // (three of their four tiles over the last 16 rows held 4), a finer grain for the CUs, and fewer keys masked away at
    // a row tile's end.  Pairs of heads / this, us: 68 rows, 8 sequences of 1024 to 4096 keys 157.0 / 136.3, 2 of 1000
    // 28.4 / 27.1, one of 2048 29.6 / 28.3; 170 rows on 1024 34.1 / 29.6, 512 rows on 512 74.3 / 63.7, 25 rows, 4 of
    // 2000 28.9 / 26.6.
    // Fewer rows than a tile's are another matter: a pair's tile then has no more queries than rows, and a wave that
    // rescales only where one of its queries finds a new maximum does so less often.  Where the CUs of an XCD (32; its
    // K/V heads stay on it) take the pairs' workgroups at once there is nothing to gain for it, and heads share a tile up
    // to 4 queries only (pairs / shared as far as the heads go, warm: 64/8 heads, 5 rows on 1000 15.1 / 17.1, on 4096
    // 20.1 / 21.9, 4 sequences of 2048 22.6 / 24.1, 8 rows on 2048 16.8 / 18.0; 32/8 heads, 8 rows on 1000 15.8 / 17.2;
    // 32/1 heads, 3 rows on 1000 15.3 / 17.2; but one row 18.5 / 17.6 on 4096).  Where they queue, sharing wins
    // (32/1 heads, 5 rows on 4096 46.5 / 29.2), if it leaves fewer workgroups (12/1 heads, 9 rows on 8000, 3 of each
    // split either way: 45.8 / 48.7; from two full tiles on the finer grain pays by itself).
    const int qpk = Hq / Hkv;
    AttnTiles a;
    a.tiles = qpk % 2 == 0 ? 2 : 1;
    a.lg_ht = 0;
    while (a.tiles == 2 && a.lg_ht < 3 && qpk % (4 << a.lg_ht) == 0) a.lg_ht++;
    auto per_kv_head = [&](int lg) { return (int64_t)(qpk / 2 >> lg) * ((rows + (16 >> lg) - 1) / (16 >> lg)) * p.splits; };
    if (rows < 16 && ((int64_t)batch * Hkv + 7) / 8 * per_kv_head(0) <= 32)
        while (a.lg_ht > 0 && rows << a.lg_ht > 4) a.lg_ht--;
    if (rows < 32 && per_kv_head(a.lg_ht) >= per_kv_head(0)) a.lg_ht = 0;
    // Eight waves walk one workgroup's keys, or four: with four a CU holds two workgroups, one in its loop while the
    // other is in its prologue or merge (6 us of a workgroup's time together), and the merge is half as wide.
    // Four where the workgroups are more than the CUs, eight where each has a CU to itself and fewer waves would
    // only make its walk longer (eight / four, 68 rows unless stated: 64/8 heads, 8 sequences of 1024 to 4096 keys
    // 159.5 / 136.3 us, 3 of 300 26.3 / 19.8; 32 heads, 2 of 800 22.5 / 17.9, 4 of 700 to 1400 35.4 / 30.6, 8 of 2000
    // 111 / 94.5, 170 rows on 1024 25.1 / 21.8, 488 rows on 512 50.8 / 43.8; but one sequence, 136 and 160 workgroups:
    // 64/8 heads 28.3 / 33.2, 32 heads 13.0 / 15.5).  Where one row per sequence is asked for, one row tile of each
    // has work.
    // Two workgroups of four waves have to fit a CU's LDS: with a large page table they do not, and one by itself
    // takes half as long again as eight waves (a pass of 44 rows on 3841 pages of 16, 64/8 heads 653 / 436 us, on 3969 pages,
    // 32 heads 586 / 395).  The same at the end of a launch whose last workgroups, up to 256 in an odd round of 256, come
    // to one a CU: what that costs grows with the walk, what four waves save does not.  Paged walks lose beyond 17 chunks
    // a round (four / eight, passes of 32 heads, 3 rounds: 360 rows on 5000 307 / 282, 133 rows, 2 of 5630 320 / 293, 74
    // rows, 4 of 2367 195 / 186, 4 of 1292 136 / 137; 5 rounds: 127 rows, 5 of 4594 418 / 406, 204 rows, 3 of 1026 195 /
    // 198; 64/8 heads, 3 rounds: 360 rows on 5000 371 / 347, 5 rounds: 68 rows, 8 of 2000 278 / 290), contiguous ones of
    // one head per workgroup, unsplit, from 120 chunks in the upper half of the third round on (attention alone, 32 heads:
    // 357 rows on 5360 117 / 106, 351 on 3102 74 / 70; but 285 on 6309 110 / 113), with pairs never (64/8 heads, 351 rows on
    // 6806 187 / 195).
    const int rows_wg = 16 >> a.lg_ht, n_mt = one_row ? 1 : (rows + rows_wg - 1) / rows_wg;
    a.workgroups = (int64_t)batch * (a.tiles == 2 ? Hq >> (1 + a.lg_ht) : Hq) * n_mt * p.splits;
    const int64_t rounds = (a.workgroups + 255) / 256, walk = (p.chunks + p.splits - 1) / p.splits;
    const bool fits = 2 * (att_smem_four(hd, a.tiles) + att_table_bytes(table_entries)) <= 160 * 1024;
    const bool long_end = (rounds & 1) && (table_entries ? walk > 17 * rounds
                                                         : a.tiles == 1 && p.splits == 1 && rounds == 3 && a.workgroups >= 640 && walk >= 120);
    a.waves = rounds > 1 && fits && !long_end ? 4 : 8;
    // Where workgroups of one head and four waves queue (512 are held at once) two or four neighbouring row tiles of a head can
    // run as one workgroup whose waves share every chunk: half or a quarter of the loads, which bound these launches, and of
    // the workgroups, but a barrier per chunk, and a longer walk for every wave.  A round of such workgroups, full or not, takes
    // 1.5 or 2.55 times as long as one of single tiles (several sequences, 128-wide heads; of a single tiles' last round half counts
    // as its share), so two tiles pay where they save a round or most of one, four where two still queue.  single / shared, us, 32 heads
    // unless stated: 68 rows, 4 sequences up to 900 keys 31.8 / 26.6, 5 of 900 36.5 / 27.4, 5 of 2200 66.8 / 52.8, 8 of 900
    // (four tiles) 52.4 / 43.8, 40 rows, 8 of 900 38.8 / 29.2, 100 rows, 3 of 900 30.9 / 26.5, 256 rows, 2 of 1000 46.0 / 37.0, 40 heads,
    // 25 rows, 8 of 1000 36.1 / 31.4; but 68 rows, 6 of 900 (960 workgroups, 576 shared) 38.9 / 41.6 and, four tiles, 100 rows,
    // 5 of 2200 77.1 / 80.4, which the rule leaves out.  64-wide heads lose (4 heads, 32 sequences of 1000 21.4 / 22.2).
    // Up to 640 single tiles, few of which wait, what is saved is little, and one long sequence's tiles, walked at the joined pace,
    // are the launch's time: there only walks of up to 51 chunks share.  Shared / single, of equal lengths, lengths within a factor of
    // two and of four: up to 640, 900 keys 0.858, 0.917, 0.974, 1500 keys 0.884, 0.941, 1.086, 2200 keys 0.892, 1.007, 1.140, 4096 keys
    // 0.889, 1.020, 1.160 (up to 1.53); above 640, 900 keys 0.817, 0.841, 0.840, 2200 keys 0.841, 0.870, 0.959, 4096 keys 0.833, 0.903,
    // 0.957 (185 launches to 640, 160 of two tiles above).
    // One sequence's tiles differ in length and queue well by themselves (300 rows on 512 26.7 / 29.9): only where eight waves over four
    // tiles leave no queue do they gain, and from 960 on, where single tiles fill two rounds, enough to be told from a change of box (512
    // rows on 512 45.5 / 42.3, on 1500 66.5 / 60.9, on 6000 165 / 138, 40 heads, 384 rows on 512 40.7 / 36.3; but 32 heads, 384 rows, 768 tiles,
    // 36.4 / 35.6 and 56.4 / 54.3).
    a.share = 1;
    a.launched_workgroups = a.workgroups;
    if (a.tiles == 1 && a.waves == 4 && hd == 128 && p.splits == 1 && !one_row) {
        auto shared = [&](int t) { return (int64_t)batch * Hq * ((n_mt + t - 1) / t); };
        auto rounds_of = [](int64_t wgs) { return (double)((wgs + 511) / 512); };
        if (batch == 1) {
            if (a.workgroups >= 960 && shared(4) <= 256) a.share = 4;
        } else if (a.workgroups > (walk <= 51 ? 512 : 640)) {
            double best = 0.97 * 0.5 * ((double)a.workgroups / 512.0 + rounds_of(a.workgroups));
            for (int t : {2, 4}) {
                const double c = (t == 2 ? 1.5 : 2.55) * rounds_of(shared(t));
                if (c < best) { best = c; a.share = t; }
            }
        }
        a.launched_workgroups = shared(a.share);
    }
    a.share_waves = a.share == 4 && batch == 1 ? 8 : a.waves;
    // Where pairs of heads queue (512 workgroups of four waves are held at once, 256 of eight) and an XCD walks several sequences one
    // after the other, the longest start first, so that the last workgroups are short: instantiations of their own (as a branch
    // of the others the ranking cost every launch 0.5 %), up to 8 sequences (one comparison a lane; a loop over 64 cost a workgroup half a
    // microsecond), from walks of 64 chunks on.  Ranking costs a workgroup some 0.3 us: with 1024 keys that was 1.4 % of equal
    // lengths' time against 1 % that unequal ones gained, with 512 keys a loss for all, with one K/V head, whose sequences lie on an XCD each,
    // nothing but the cost.  From 2048 keys on, time of the batch's order, 64/8, 32/4 and 64/16 heads: equal lengths 1.004 (48 launches), lengths
    // within a factor of two 0.981 (58; 0.87 to 1.10 by the draw), of four 0.949 (38; 0.80 to 1.11); 64/8 heads, 68 rows, 8 of 1024 to
    // 4096 keys, 40 draws 0.957 (125 -> 120 us); paged, whole passes, 0.96 and equal lengths 0.995.  (One head per workgroup, whose launches
    // are bound by what they load, lost up to 8 % as often as it won; key splits are not measured.)
    a.ranked = a.tiles == 2 && p.splits == 1 && a.workgroups > (a.waves == 4 ? 512 : 256) && batch <= 8 && (int64_t)batch * Hkv > 8 && walk >= 64;
    return a;
}

// lg_ht: log2 of the heads that share a tile (two heads per workgroup and more)
template <int HD, int U, int W, int T, bool PAGED, bool RANKED = false>
static void launch_attn_t(const TemplateDev &t, const void *q, const void *q_lo, const void *k_cache, const void *v_cache,
                          const void *k_tree, const void *v_tree, const void *k_tree_lo, const void *v_tree_lo,
                          const void *prompt_k, const void *prompt_v, const int32_t *ctx_len, const int32_t *token,
                          int batch, int Hq,
                          int Hkv, int P, int smax, const AttnPlan &p, float *part_o, float *part_ml, void *out,
                          void *out_lo, bool out_as_fragments, const PageMap &pm, const int32_t *only_row, int lg_ht, hipStream_t s) {
    using C = AttCfg<HD, U, W, T>;
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)tree_attn_kernel<HD, U, W, T, PAGED, RANKED>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize,
                                  C::SMEM + (PAGED ? ATT_PAGE_TABLE_MAX * 4 : 0));
        attr_set = true;
    }
    const size_t smem_bytes = C::SMEM + (PAGED ? att_table_bytes(pm.tbl_cap) : 0);
    const int per_wg = T * 16 >> lg_ht, n_mt = U == 1 && T == 1 && only_row ? 1 : (t.rows + per_wg - 1) / per_wg;      // rows of a workgroup
    const float scale_log2 = 1.4426950408889634f / sqrtf((float)HD);
    const int groups = batch * Hkv, per_group = (Hq / Hkv / U >> lg_ht) * n_mt * p.splits;
    const int per_xcd = (groups + 7) / 8, grid_y = per_xcd < 1 << ATT_GRID_Y_LG ? per_xcd : 1 << ATT_GRID_Y_LG;
    const dim3 grid(8 * per_group, grid_y, (per_xcd + grid_y - 1) / grid_y);
    hipLaunchKernelGGL((tree_attn_kernel<HD, U, W, T, PAGED, RANKED>), grid, dim3(W * 64), smem_bytes, s,
                       ctx_len, batch, Hq / Hkv, Hkv, n_mt | lg_ht << 16 | (U == 1 && T == 1 && only_row ? 1 << 24 : 0), p.splits, P, t.rows, smax, (const uint16_t *)q, (const uint16_t *)q_lo, t,
                       (const uint16_t *)k_cache, (const uint16_t *)v_cache,
                       (const uint16_t *)k_tree, (const uint16_t *)v_tree, (const uint16_t *)k_tree_lo,
                       (const uint16_t *)v_tree_lo, (const uint16_t *)prompt_k, (const uint16_t *)prompt_v, token,
                       scale_log2, part_o, part_ml, (uint16_t *)out,
                       (uint16_t *)out_lo, out_as_fragments ? 1 : 0, (batch * t.rows + 15) / 16, pm, only_row);
}

void launch_tree_attention(const TemplateDev &t, const void *q, const void *q_lo, const void *k_cache, const void *v_cache,
                           const void *k_tree, const void *v_tree, const void *k_tree_lo, const void *v_tree_lo,
                           const void *prompt_k,
                           const void *prompt_v, const int32_t *ctx_len, const int32_t *token, int batch, int Hq, int Hkv, int hd,
                           int P, int smax, const AttnPlan &p, float *part_o, float *part_ml, void *out,
                           void *out_lo, bool out_as_fragments, const PageMap &pm, hipStream_t s, const int32_t *only_row) {
    const AttnTiles a = attn_tiles(batch, t.rows, Hq, Hkv, hd, p, pm.table ? pm.tbl_cap : 0, only_row != nullptr);
#define ATT_LAUNCH_P(HD_, U_, W_, T_, ...) launch_attn_t<HD_, U_, W_, T_, __VA_ARGS__>(t, q, q_lo, k_cache, v_cache, k_tree, v_tree, k_tree_lo, v_tree_lo, prompt_k, \
                                                   prompt_v, ctx_len, token, batch, Hq, Hkv, P, smax, p, part_o, part_ml, out, out_lo, out_as_fragments, pm, only_row, a.lg_ht, s)
#define ATT_LAUNCH(HD_, U_) do { \
        if (a.waves == 4) { if (pm.table) ATT_LAUNCH_P(HD_, U_, 4, 1, true); else ATT_LAUNCH_P(HD_, U_, 4, 1, false); } \
        else { if (pm.table) ATT_LAUNCH_P(HD_, U_, 8, 1, true); else ATT_LAUNCH_P(HD_, U_, 8, 1, false); } } while (0)
#define ATT_SHARED(W_, T_) do { if (pm.table) ATT_LAUNCH_P(128, 1, W_, T_, true); else ATT_LAUNCH_P(128, 1, W_, T_, false); } while (0)
#define ATT_RANKED(HD_) do { \
        if (a.waves == 4) { if (pm.table) ATT_LAUNCH_P(HD_, 2, 4, 1, true, true); else ATT_LAUNCH_P(HD_, 2, 4, 1, false, true); } \
        else { if (pm.table) ATT_LAUNCH_P(HD_, 2, 8, 1, true, true); else ATT_LAUNCH_P(HD_, 2, 8, 1, false, true); } } while (0)
    if (a.ranked && hd == 128) ATT_RANKED(128);
    else if (a.ranked) ATT_RANKED(64);
    else if (a.share == 2) ATT_SHARED(4, 2);
    else if (a.share == 4 && a.share_waves == 4) ATT_SHARED(4, 4);
    else if (a.share == 4) ATT_SHARED(8, 4);
    else if (hd == 128) {
        if (a.tiles == 2) ATT_LAUNCH(128, 2); else ATT_LAUNCH(128, 1);
    } else {
        if (a.tiles == 2) ATT_LAUNCH(64, 2); else ATT_LAUNCH(64, 1);
    }
#undef ATT_LAUNCH_P
#undef ATT_LAUNCH
#undef ATT_SHARED
#undef ATT_RANKED
    if (p.splits > 1) {
        const int heads_per_block = (256 / (hd / 4)) < Hq ? (256 / (hd / 4)) : Hq;
        hipLaunchKernelGGL(attn_merge_kernel, dim3(only_row ? 1 : t.rows, (Hq + heads_per_block - 1) / heads_per_block, batch),
                           dim3(heads_per_block * (hd / 4)), 0, s, part_o, part_ml, t.rows,
                           Hq, hd, p.splits, (uint16_t *)out, (uint16_t *)out_lo, out_as_fragments ? 1 : 0, (batch * t.rows + 15) / 16,
                           only_row);
    }
}
