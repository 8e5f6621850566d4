// Skinny weight-streaming GEMM for the verify step: Y[M][N] = A[M][K] * W[N][K]^T with
// M = (tree + mask rows) * batch, i.e. a few dozen rows, so the kernel is bound by the one
// pass over W in HBM (the paper's premise, Sec. 3.2: inference is memory-bandwidth bound,
// extra rows are nearly free).
//
// Layout choices for gfx950:
//  * W is pre-packed into 1 KiB blocks, each exactly one v_mfma_f32_16x16x32_bf16 B-operand
//    (16 rows x 32 k; lane l holds W[16t + l%16][32s + 8(l/16) .. +8]), so a wave loads its
//    fragments with fully coalesced 16-byte-per-lane loads straight into MFMA registers; W
//    never touches LDS.  Blocks are ordered k-major: [k-step pair][16-row tile][2 k-steps].
//    Waves that run side by side work on neighbouring tiles of the same k range, so what
//    the chip reads at any moment is one contiguous region (as in a plain copy), instead of
//    thousands of streams a power-of-two stride apart that would pile onto few HBM channels.
//  * The activation slab is small and shared by every wave.  Producers write it to global
//    memory already in A-operand fragment order (1 KiB per (plane, k-step, m-tile): lane l
//    holds A[16mt + l%16][32ks + 8(l/16) .. +8]), so one direct global->LDS load per
//    fragment reads 1 KiB contiguous, lands in LDS in operand order (conflict-free linear
//    reads) and spends no VGPRs on staging.  Each fragment read from LDS feeds NW weight
//    tiles; with two planes the slab traffic from L2 is what limits narrow NW.
//  * Activations may come as two bf16 planes (hi = bf16(x), lo = bf16(x - hi)); both are
//    multiplied with the same weight fragment.  That removes the activation rounding from
//    the error budget at the price of 2x MFMA work, which the kernel has to spare (at 68
//    rows it needs ~1/4 of the matrix-core rate the HBM stream could feed).
//  * A three-stage software pipeline keeps two stages of W (registers) and A (LDS ring) in
//    flight behind the one being multiplied; waits are on the oldest stage only.
//  * Parallelism comes from N (16*NW rows per wave) and, where N alone cannot fill 256 CUs,
//    from split-K with fp32 partial sums reduced in a fixed order by the consumer
//    (deterministic, no float atomics).
#include "common.h"
#include <string.h>
#include <stdlib.h>
#include <type_traits>

// index of the 1 KiB block holding rows 16t..16t+15, k 32ks..32ks+31 (k-major order)
__host__ __device__ __forceinline__ int64_t packed_block(int64_t t, int64_t ks, int64_t n_tiles) {
    return ((ks >> 1) * n_tiles + t) * 2 + (ks & 1);
}

// wait until at most N vector-memory operations of this wave are outstanding and all of its
// LDS reads have returned
template <int N>
__device__ __forceinline__ void wait_vmcnt_lds() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0x0 << 8));
}

// Workgroup barrier without the memory fences of __syncthreads(): those would drain every
// outstanding vector-memory operation (vmcnt(0)) and with it the prefetched stages.  The
// data hazards are covered explicitly by the wait that precedes it: the wave's own LDS-bound
// loads of the stage about to be read have landed, and its LDS reads of the previous stage
// (whose slot is refilled after the barrier) have returned.
__device__ __forceinline__ void wg_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// LDS reads of activation fragments as bare instructions with their own staged waits: the
// k-step's reads are all issued up front and each MFMA group waits only for the fragment it
// uses (the compiler's own placement was one wait for all of them).  lgkmcnt counts this
// wave's outstanding LDS reads, which return in order.
template <int OFFSET>
__device__ __forceinline__ bf16x8 lds_read_frag(uint32_t lds_addr) {
    static_assert(OFFSET >= 0 && OFFSET < 65536, "ds offset field");
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(lds_addr), "n"(OFFSET));
    return v;
}
template <int OUTSTANDING>
__device__ __forceinline__ void lds_wait_frag(bf16x8 &a) {
    static_assert(OUTSTANDING >= 0 && OUTSTANDING < 16, "lgkmcnt range");
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(a) : "n"(OUTSTANDING));
}

// (no use of the fragment is moved ahead of the wait before this)
__device__ __forceinline__ void frag_use(bf16x8 &a) { asm volatile("" : "+v"(a)); }

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// MT m-tiles of 16 rows, NW n-tiles per wave, SPLIT = two activation planes, KC k-steps (of 32)
// per pipeline stage, D stages in the ring (D-1 in flight behind the one being multiplied),
// WAVES wavefronts per workgroup, of which KG groups of WN = WAVES/KG waves each take one
// contiguous part of the workgroup's k range (with their own activation ring) and are summed
// through LDS at the end: twice the waves per partial sum written.
// PACK: the slab's last m-tile (the pass' tile MT-1) keeps both planes of its rows in its high
// plane's fragment (frag_pack_offset): the stage has one fragment less, the last of the list.
template <int MT, int NW, bool SPLIT, int KC, int D, int WAVES, int KG, bool PACK = false, bool ROPE = false>
struct GemmCfg {
    static_assert(!PACK || (SPLIT && KC == 1), "packing folds the low plane into the high one");
    static constexpr int WN = WAVES / KG;                       // waves side by side along N
    static constexpr int PL = SPLIT ? 2 : 1;
    static constexpr int NFRAG = PL * MT * KC - (PACK ? 1 : 0); // A fragments per stage
    static constexpr int FPW = (NFRAG + WN - 1) / WN;           // fetched per wave per stage
    static constexpr int LOADS = NW * KC + FPW;                 // vector-memory loads per wave per stage
    // every wave issues FPW fragment loads per stage (the vmcnt bookkeeping counts on it);
    // those beyond NFRAG land in one shared dump slot after the ring
    static constexpr int RING = KG * D * NFRAG * 1024;          // one ring per k group
    static constexpr int MERGE = KG > 1 ? WN * MT * NW * 1024 : 0;   // accumulators of one k group
    // outputs on their way out: the gated slab of the workgroup, or (three tiles per wave) each wave's
    // sums as rows of 48 floats, 4 floats apart from the next (rows 4g of the four lane groups then
    // start 16 banks apart)
    static constexpr int ROW3 = 52;
    static constexpr int STAGE = NW % 2 == 0 ? 2 * (WN * NW * 8 / 16) * MT * 512 : NW == 3 ? WN * MT * 16 * ROW3 * 4 : 0;
    // ... or (rotated QKV columns, any form of two k groups) each wave's sums as rows, 4 floats apart as above
    static constexpr int ROW = NW * 16 + 4, ROWS = ROPE ? WN * MT * 16 * ROW * 4 : 0;
    static constexpr int OUT = STAGE > ROWS ? STAGE : ROWS;
    static constexpr int SMEM = (RING > MERGE ? (RING > OUT ? RING : OUT) : (MERGE > OUT ? MERGE : OUT)) + 1024;
    static_assert((D - 2) * LOADS < 64, "vmcnt counter range");
};

// THROUGH: split-K partial sums are written through the L2 (store_through) from 8 MB on, where the launch
// leaves megabytes behind that would be written back between this kernel and the next (7B widths, 68 rows:
// 17 + 9 + 9 MB a layer: 3 us of the 340 of two layers and the head).  Below, and for a single split's
// plain sums, the write-back is short and the stores' way to memory costs the workgroups' tails more
// (68 rows x 22016, 6 MB: 45.2 us plain, 45.5).  The logits of a direct launch go through at every size,
// though it hardly matters there (one layer and the head, through / plain: 7B, 1 row 149.1 / 149.1 us,
// 48 rows 196.5 / 197.0, 68 rows 204.8 / 204.0, four sequences of 68 431.4 / 430.2; 13B, 25 rows 213.8 / 214.8).
// ROPE: a direct launch that rotates and stores the QKV columns (instantiations of their own: as one more case of the direct
// ones its code cost gate/up and the LM head of a 64-node step 0.5 %).
// TURNS: the two k groups take turns (below) instead of both at once; launch_gemm_t says where.
template <int MT, int NW, bool SPLIT, int KC, int D, int WAVES, int KG, bool DIRECT, bool PACK, bool THROUGH, bool ROPE, bool TURNS>
__global__ __launch_bounds__(WAVES * 64) void gemm_skinny_kernel(
    // The first 14 dwords of the argument block arrive in scalar registers with the wave
    // (kernel-argument preload); everything the first loads depend on is among them, the grid's
    // extent included: read through gridDim it costs one dependent scalar load per component
    // before the first weight load can be issued.
    const uint4 *__restrict__ A_frag, const uint4 *__restrict__ Wp, int planes_stride_f, int M, int m_tiles,
    int NT, int KS, int ksteps_per_split, int grid_x, int grid_y, int grid_z, int head_tiles,
    float *__restrict__ out, int64_t ldo, GemmOutput direct) {
    using C = GemmCfg<MT, NW, SPLIT, KC, D, WAVES, KG, PACK, ROPE>;
    constexpr int WN = C::WN;
    static_assert(!TURNS || (KG == 2 && KC == 1 && !PACK), "two k groups, whole fragments");
    constexpr int SUB = MT > 5 ? 2 : 1;                        // reads and multiplies of a k-step: all at once, or plane by plane
    extern __shared__ __attribute__((aligned(16))) uint4 smem_u4[];   // [KG][D][NFRAG][64] + dump slot

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, and known to be: addresses on the scalar unit
    const int kg = wave / WN, wn = wave % WN;                  // k group, position along N
    // (column group, k split, row pass) of this workgroup.  With several row passes (more rows
    // than one pass holds) the passes over the same weights are made neighbours on one XCD:
    // dispatch index L goes to XCD L % 8, so the passes of a (column group, split) pair take
    // indices 8 apart and run side by side on that XCD, the later ones finding the weight
    // blocks in its L2 instead of fetching them again.
    int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
    if (grid_z > 1) {
        const int X = grid_x, Z = grid_z, T = X * grid_y, Tb = T & ~7;
        const int L = bx + X * (by + grid_y * bz);
        int pair;
        if (L < Tb * Z) {
            const int q = L >> 3;
            bz = q % Z;
            pair = (q / Z) * 8 + (L & 7);
        } else {                                               // the last T % 8 pairs, pass-major
            const int r = L - Tb * Z;
            bz = r % Z;
            pair = Tb + r / Z;
        }
        bx = pair % X;
        by = pair / X;
    }
    else if (grid_y > 1) {
        // Split-K launch: workgroups of one k split read the same k range of the activation
        // slab.  With a power-of-two number of splits each split is given to its own XCD(s), so
        // that every k range is fetched into one L2 (or few) instead of all eight.
        const int X = grid_x, Y = grid_y, L = bx + X * by;
        if ((Y & (Y - 1)) == 0 && ((X * Y) & 7) == 0) {
            if (Y >= 8) {
                const int per = Y >> 3;                        // splits per XCD
                by = (L & 7) + 8 * ((L >> 3) % per);
                bx = (L >> 3) / per;
            } else {
                const int per = 8 / Y;                         // XCDs per split
                by = (L & 7) / per;
                bx = (L >> 3) * per + (L & 7) % per;
            }
        }
    }
    const int t0 = (bx * WN + wn) * NW;
    // The weight tile behind column tile t: itself, or, for columns that are rotated in pairs half a head apart, the two tiles of a
    // pair one after the other, so that a workgroup (an even number of tiles) holds whole pairs.
    int tile_of[NW];
#pragma unroll
    for (int j = 0; j < NW; j++) {
        const int t = min(t0 + j, NT - 1);
        tile_of[j] = t;
        if constexpr (ROPE) {
            const int r = t & (head_tiles - 1);
            tile_of[j] = t - r + (r >> 1) + (r & 1) * (head_tiles >> 1);
        }
    }
    // the workgroup's k range, cut into KG contiguous parts of equal stage count
    const int wg_begin = by * ksteps_per_split;
    const int wg_end = min(KS, wg_begin + ksteps_per_split);
    const int per_group = (wg_end - wg_begin + KG - 1) / KG;
    const int ks_begin = wg_begin + kg * per_group;
    const int ks_end = min(wg_end, ks_begin + per_group);
    const int m_base = bz * (MT * 16);
    const int n_stages = (per_group + KC - 1) / KC;            // same for every wave: barriers in lockstep
    uint4 *a_lds = smem_u4 + kg * (D * C::NFRAG * 64);         // this k group's ring
    uint4 *dump = smem_u4 + KG * D * C::NFRAG * 64;            // target of padding fetches

    // lane -> lane holding the same k granule of the last existing row of the slab's last m-tile
    // (packed tile: of the last existing row of the lane's plane)
    const int rows_last = M - (m_tiles - 1) * 16, pack_off = PACK ? frag_pack_offset(M) : 16;
    const int lane_row = lane & 15;
    const int lane_last = (lane & ~15) | (lane_row < pack_off ? min(lane_row, rows_last - 1)
                                                              : pack_off + min(lane_row - pack_off, rows_last - 1));

    f32x4 acc[MT][NW];
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
        for (int j = 0; j < NW; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    uint4 w[D][NW][KC];
    // byte address in LDS of this lane's 16 bytes of the k group's fragment 0
    const uint32_t lds_lane_base = (uint32_t)(size_t)((__attribute__((address_space(3))) uint4 *)a_lds) + lane * 16;

    // Issue all loads of pipeline stage `stage` into ring slot SLOT: NW*KC weight fragments to
    // registers and this wave's FPW activation fragments to LDS.  Every wave issues exactly
    // C::LOADS vector-memory operations, which is what the vmcnt waits below count on.
    // Every address is valid and computed without a select (all terms are wave-uniform but the
    // lane's 16 bytes): tiles past the matrix, k-steps past the group's range, m-tiles past the
    // slab and the padding fetches re-read the nearest existing fragment.  What they bring is
    // either never multiplied (k-steps: see compute) or lands in accumulators that are never
    // stored (rows and columns beyond the output).
    auto issue = [&](auto slot_c, int stage) {
        constexpr int SLOT = decltype(slot_c)::value;
        const int ks0 = ks_begin + stage * KC;
#pragma unroll
        for (int j = 0; j < NW; j++)
#pragma unroll
            for (int s = 0; s < KC; s++) {
                const int t = tile_of[j], ks = min(ks0 + s, KS - 1);
                typedef uint32_t __attribute__((ext_vector_type(4))) u32x4_t;
                const u32x4_t q = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(Wp + packed_block(t, ks, NT) * 64 + lane));
                w[SLOT][j][s] = make_uint4(q.x, q.y, q.z, q.w);
            }
#pragma unroll
        for (int i = 0; i < C::FPW; i++) {
            const int f = i * WN + wn;                            // fragment id inside the stage
            const int fc = min(f, C::NFRAG - 1);
            const int plane = fc / (MT * KC), mt = (fc / KC) % MT, s = fc % KC;
            const int mtg = min(bz * MT + mt, m_tiles - 1);   // m-tile in the whole slab
            const int ks = min(ks0 + s, KS - 1);
            // fragment (plane, ks, mtg) starts at ((plane * KS + ks) * m_tiles + mtg) * 64 uint4
            // The slab's last m-tile may hold fewer than 16 rows (4 of the 68 of a 64-node tree):
            // the lanes of its missing rows re-read the last row that exists, so the fragment
            // costs the L1 the cache lines of its real rows only (same-address lanes coalesce).
            // The copies land in accumulator rows that are never stored.
            const int src_lane = mtg == m_tiles - 1 ? lane_last : lane;   // wave-uniform choice
            const uint4 *src = A_frag + ((int64_t)plane * planes_stride_f + (int64_t)ks * m_tiles + mtg) * 64 + src_lane;
            uint4 *dst = f < C::NFRAG ? a_lds + (SLOT * C::NFRAG + f) * 64 : dump;   // wave-uniform; lane l lands at dst[l]
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                             (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
        }
    };
    auto compute = [&](auto slot_c, int stage) {
        constexpr int SLOT = decltype(slot_c)::value;
#pragma unroll
        for (int s = 0; s < KC; s++) {
            // a k group whose share of the range is shorter than the others' skips the k-steps
            // past its end (wave-uniform)
            if (ks_begin + stage * KC + s >= ks_end) continue;
            // the LDS reads of a batch are issued before its first MFMA; fragment f is waited for with the
            // batch's later reads still in flight.  Up to 5 m-tiles a k-step is one batch, above 4 fragments, so that the
            // accumulators (MT x NW tiles) leave room for them.
            constexpr int NF = C::PL * MT - (PACK ? 1 : 0), AB = MT > 5 ? 4 : NF, NB = (NF + AB - 1) / AB;
            static_assert(AB <= 16, "lgkmcnt range");
            static_for<0, NB>([&](auto b_c) {
                constexpr int B0 = decltype(b_c)::value * AB, BN = (NF - B0) < AB ? (NF - B0) : AB;
                bf16x8 a[BN];
                static_for<0, BN>([&](auto f_c) {
                    constexpr int F = B0 + decltype(f_c)::value;
                    a[F - B0] = lds_read_frag<((SLOT * C::NFRAG + F * KC) * 64) * 16>(lds_lane_base + s * 1024);
                });
                static_for<0, BN>([&](auto f_c) {
                    constexpr int F = B0 + decltype(f_c)::value, i = F % MT;
                    lds_wait_frag<BN - 1 - (F - B0)>(a[F - B0]);
#pragma unroll
                    for (int j = 0; j < NW; j++)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            a[F - B0], __builtin_bit_cast(bf16x8, w[SLOT][j][s]), acc[i][j], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);      // keeps the next fragment's wait behind these MFMAs
                });
            });
        }
    };
    // One pipeline step for stage c living in slot U: wait for its data (leaving the D-2 newer
    // stages in flight), make it visible to the workgroup, refill the slot freed by stage
    // c-1, multiply.  Every step issues exactly C::LOADS loads, also for stages past the end
    // (those read the zero granule), so the wait count is a compile-time constant and the
    // compiler's own wait-count analysis sees every register dependency satisfied by it; with
    // data-dependent counts it drains the whole ring at the loop head instead.
    // The k groups take the two halves of a step in opposite order: behind the barrier one
    // group queues its loads on the vector-memory path while the other is on LDS and the
    // matrix cores (waves of different groups share a SIMD), then they swap.  Two copies of the
    // loop, chosen once per wave: with both orders inside one body the compiler's wait-count
    // analysis loses track at the join and drains the ring (vmcnt(0)) before every multiply.
    auto main_loop = [&](auto multiply_first_c) __attribute__((always_inline)) {
        constexpr bool MULTIPLY_FIRST = decltype(multiply_first_c)::value;
        int c = 0;
        for (; c + D <= n_stages; c += D)        // branch-free body: D steps, slots 0..D-1
            static_for<0, D>([&](auto u_c) {
                constexpr int U = decltype(u_c)::value;
                constexpr int PRE = (U + D - 1) % D;
                wait_vmcnt_lds<(D - 2) * C::LOADS>();
                wg_barrier();
                if constexpr (MULTIPLY_FIRST) {
                    compute(u_c, c + U);
                    issue(std::integral_constant<int, PRE>{}, c + U + D - 1);
                } else {
                    issue(std::integral_constant<int, PRE>{}, c + U + D - 1);
                    compute(u_c, c + U);
                }
            });
        return c;
    };

    // A launch that finishes its own output needs the row factors of its rows at the end.  The sums
    // behind them are requested here, ahead of the first stages' loads (every thread fetches, from
    // a clamped row, and where there is nothing to fetch from the slab instead: no branch around
    // the loads), and reduced to the one factor right behind those loads, where the wave has to
    // wait for its first stage anyway: a single register lives through the loop.
    RowScaleSums my_row_sums;
    if constexpr (DIRECT) {
        const bool have = direct.kind != GEMM_OUT_PARTIAL && direct.rs.ssq != nullptr;
        const float4 *src = have ? reinterpret_cast<const float4 *>(direct.rs.ssq + (int64_t)min(m_base + (tid % (MT * 16)), M - 1) * RMS_MAX_CHUNKS)
                                 : reinterpret_cast<const float4 *>(A_frag);
        my_row_sums.q0 = src[0]; my_row_sums.q1 = src[1]; my_row_sums.q2 = src[2]; my_row_sums.q3 = src[3];
    }
    static_for<0, D - 1>([&](auto u_c) {
        issue(u_c, decltype(u_c)::value);
        if constexpr (TURNS) __builtin_amdgcn_sched_barrier(0);   // (stage by stage: the waits below count them)
    });
    float my_row_scale = 0.f;
    if constexpr (DIRECT) {
        if (direct.kind != GEMM_OUT_PARTIAL && m_base + (tid % (MT * 16)) < M) my_row_scale = row_scale_finish(direct.rs, my_row_sums);
    }
    if constexpr (TURNS) {
        // The k groups in turns: a phase ends at a barrier, and in each of them one group multiplies from registers while the
        // other, a phase behind, reads its next fragments from LDS and issues its loads.  Every SIMD holds waves of
        // both, so its matrix core always has one that waits for nothing (16 cycles an instruction, 58 cycles a phase
        // for barrier, wait and branch).  With both groups at once (the loop below) all waves read behind the same barrier and
        // the cores idled for that long, about 700 cycles of each k-step however many instructions it had.  Cycles per
        // k-step, at once / turns, of them multiplies: 9 m-tiles x 12 tiles 2490 / 1930, 1728; 9 x 16 3150 / 2470, 2304; 8 x 12
        // 2215 / 1690, 1536; 8 x 16 2800 / 2240, 2048.  What bounds it now is the card's power: the clock falls from 1.65-1.95 to
        // 1.4-1.65 GHz (with activations of zeros it is 2.35).  Calls, us: 22016 x 4096, 240 rows 93.8 / 75.8, 272 rows 101 / 90, 512
        // rows 165 / 151; 12288 x 4096, 512 rows 94.8 / 81.0; 57344 x 8192, 96 rows 180 / 169, 512 rows 781 / 698; 8192 x 28672, 272
        // rows 235 / 216; passes of 5: 8192 x 28672, 300 rows 268 / 250, 4096 x 11008, 340 rows 74.1 / 69.7, one plane:
        // 22016 x 4096, 20 rows 37 / 34.
        // What is in the multiplying phase besides its instructions costs the launch as it stands: 9 waits instead of one 7 %,
        // the next stage's addresses 17 %.  A higher wave priority there changes nothing.
        constexpr int NF = C::NFRAG, PER = (NF + SUB - 1) / SUB;     // fragments of a k-step, read at a time
        typedef const __attribute__((address_space(1))) unsigned char *gptr;
        typedef uint32_t __attribute__((ext_vector_type(4))) u32x4_t;
        bf16x8 a[PER];
        // Addresses: what stays the same from stage to stage here; a stage adds one offset per operand, worked out at the end
        // of a reading phase.
        gptr w_src[NW], a_src[C::FPW];
#pragma unroll
        for (int j = 0; j < NW; j++) w_src[j] = (gptr)(Wp + (int64_t)tile_of[j] * 128);
#pragma unroll
        for (int i = 0; i < C::FPW; i++) {
            const int fc = min(i * WN + wn, NF - 1), mtg = min(bz * MT + fc % MT, m_tiles - 1);
            a_src[i] = (gptr)(A_frag + ((int64_t)(fc / MT) * planes_stride_f + mtg) * 64 + (mtg == m_tiles - 1 ? lane_last : lane));
            asm("" : "+v"(a_src[i]));
        }
        int64_t w_at = 0, a_at = 0;                                  // of the next stage to issue
        auto place = [&](int stage) __attribute__((always_inline)) {
            const int ks = min(ks_begin + stage, KS - 1);
            w_at = packed_block(0, ks, NT) << 10;
            a_at = (int64_t)ks * m_tiles << 10;
            asm volatile("" : "+s"(w_at), "+s"(a_at));
        };
        auto fetch_a = [&](auto slot_c) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < C::FPW; i++) {
                const int f = i * WN + wn;
                uint4 *dst = f < NF ? a_lds + (decltype(slot_c)::value * NF + f) * 64 : dump;
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(a_src[i] + a_at),
                                                 (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
            }
        };
        auto fetch_w = [&](auto slot_c) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < NW; j++) {
                const u32x4_t q = __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x4_t *)(w_src[j] + w_at + lane * 16));
                w[decltype(slot_c)::value][j][0] = make_uint4(q.x, q.y, q.z, q.w);
            }
        };
        auto swap = [&]() __attribute__((always_inline)) {           // end of a phase
            __builtin_amdgcn_sched_barrier(0);
            wg_barrier();
            __builtin_amdgcn_sched_barrier(0);
        };
        auto read = [&](auto slot_c, auto sub_c) __attribute__((always_inline)) {
            constexpr int SLOT = decltype(slot_c)::value, F0 = decltype(sub_c)::value * PER;
            static_for<0, (NF - F0 < PER ? NF - F0 : PER)>([&](auto f_c) {
                constexpr int F = decltype(f_c)::value, AT = (SLOT * NF + F0 + F) * 1024, HIGH = AT < 65536 ? 0 : 32768;   // (16-bit offsets)
                a[F] = lds_read_frag<AT - HIGH>(lds_lane_base + HIGH);
            });
            __builtin_amdgcn_sched_barrier(0);
        };
        auto multiply = [&](auto slot_c, auto sub_c, bool live) __attribute__((always_inline)) {
            constexpr int SLOT = decltype(slot_c)::value, F0 = decltype(sub_c)::value * PER, N = NF - F0 < PER ? NF - F0 : PER;
            lds_wait_frag<0>(a[0]);                                  // (one wait for all)
            static_for<1, N>([&](auto f_c) { frag_use(a[decltype(f_c)::value]); });
            if (!live) return;                                       // (wave-uniform)
            static_for<0, N>([&](auto f_c) {
                constexpr int F = decltype(f_c)::value, I = (F0 + F) % MT;
#pragma unroll
                for (int j = 0; j < NW; j++)
                    acc[I][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[F], __builtin_bit_cast(bf16x8, w[SLOT][j][0]), acc[I][j], 0, 0, 0);
            });
        };
        // (LEFT: loads that may still be in flight behind the next stage's)
        auto step = [&](auto u_c, int stage, auto more_c, auto left_c) __attribute__((always_inline)) {
            constexpr int U = decltype(u_c)::value, PRE = (U + D - 1) % D;
            constexpr bool MORE = decltype(more_c)::value;
            const bool live = ks_begin + stage < ks_end;             // a k group whose share of the range is shorter than the other's
            static_for<0, SUB>([&](auto sub_c) {
                constexpr int S = decltype(sub_c)::value;
                read(u_c, sub_c);
                if constexpr (MORE && S == 0) fetch_a(std::integral_constant<int, PRE>{});
                if constexpr (MORE && S == SUB - 1) {
                    fetch_w(std::integral_constant<int, PRE>{});
                    place(stage + D);
                }
                swap();
                multiply(u_c, sub_c, live);
                if constexpr (S == SUB - 1) {
                    __builtin_amdgcn_sched_barrier(0);
                    wait_vmcnt_lds<decltype(left_c)::value>();
                }
                swap();
            });
        };
        place(D - 1);
        wait_vmcnt_lds<(D - 2) * C::LOADS>();
        swap();
        if (kg & 1) swap();
        int c = 0;
        for (; c + D <= n_stages; c += D)
            static_for<0, D>([&](auto u_c) {
                step(u_c, c + decltype(u_c)::value, std::true_type{}, std::integral_constant<int, (D - 2) * C::LOADS>{});
            });
        static_for<0, D - 1>([&](auto u_c) {
            constexpr int U = decltype(u_c)::value;
            if (c + U < n_stages)
                step(u_c, c + U, std::false_type{}, std::integral_constant<int, (D - 3 - U > 0 ? D - 3 - U : 0) * C::LOADS>{});
        });
        if (!(kg & 1)) swap();
    } else {
    int c;
    if (KG > 1 && (kg & 1)) c = main_loop(std::true_type{});
    else c = main_loop(std::false_type{});
    // Remaining n_stages % D steps: nothing more to fetch.  Stages c .. c+D-2 were issued by the
    // loop above (or the prologue) with C::LOADS loads each, so step U leaves D-2-U stages in
    // flight.  (Issuing dummy loads here instead would not keep the count: the compiler drops
    // the register loads whose values are never used, and the wait would then cover too little.)
    static_for<0, D - 1>([&](auto u_c) {
        constexpr int U = decltype(u_c)::value;
        if (c + U < n_stages) {
            wait_vmcnt_lds<(D - 2 - U) * C::LOADS>();
            wg_barrier();
            compute(u_c, c + U);
        }
    });
    }

    if constexpr (KG > 1) {
        // sum the k groups through LDS, group by group in a fixed order; group 0 stores
        wait_vmcnt_lds<0>();                                 // incl. this wave's fetches of stages past the end
        float4 *mrg = reinterpret_cast<float4 *>(smem_u4) + wn * (MT * NW * 64);
#pragma unroll
        for (int src = 1; src < KG; src++) {
            __syncthreads();
            if (kg == src) {
#pragma unroll
                for (int i = 0; i < MT; i++)
#pragma unroll
                    for (int j = 0; j < NW; j++)
                        mrg[(i * NW + j) * 64 + lane] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            }
            __syncthreads();
            if (kg == 0) {
#pragma unroll
                for (int i = 0; i < MT; i++)
#pragma unroll
                    for (int j = 0; j < NW; j++) {
                        const float4 v = mrg[(i * NW + j) * 64 + lane];
                        acc[i][j][0] += v.x; acc[i][j][1] += v.y; acc[i][j][2] += v.z; acc[i][j][3] += v.w;
                    }
            }
        }
        // (three tiles per wave: gate and up of a feature sit in different waves, the gating below is done
        // by all waves from LDS, as is the rotation)
        if (kg != 0 && !ROPE && !(NW == 3 && DIRECT && direct.kind == GEMM_OUT_SILU)) return;
    }
    if constexpr (PACK) {
        // the packed tile's low-plane products sit pack_off rows (pack_off / 4 lane groups)
        // further down: add them to the rows they belong to
#pragma unroll
        for (int j = 0; j < NW; j++)
#pragma unroll
            for (int r = 0; r < 4; r++) acc[MT - 1][j][r] += __shfl_down(acc[MT - 1][j][r], 4 * pack_off, 64);
    }
    // D layout: lane (g = lane/16, c = lane%16) holds rows 4g..4g+3, column c of each tile.
    const int g = lane >> 4, cc = lane & 15;
    // Three tiles per wave: the wave's sums as rows in LDS (its own region behind the merge; the same
    // wave wrote and reads, or a barrier follows).  A wave's region starts where its merge region
    // does not: the other waves of k group 0 are past theirs first.
    auto stage_rows3 = [&](float *stage, auto &&value) __attribute__((always_inline)) {
        __syncthreads();
        if (kg == 0) {
#pragma unroll
            for (int i = 0; i < MT; i++)
#pragma unroll
                for (int j = 0; j < NW; j++)
#pragma unroll
                    for (int r = 0; r < 4; r++) stage[(i * 16 + 4 * g + r) * C::ROW3 + j * 16 + cc] = value(i, j, r);
        }
    };
    // Stores of the wave's MT x NW tiles (k group 0 after the merge).  With k groups they go
    // through the wave's own LDS region (the one its partners wrote into, private since the
    // merge) and leave as 16 bytes per lane: whole NW*64-byte row segments instead of 64-byte
    // pieces.  Rows of 4-row group g sit in the half of the row given by g's parity (two-way
    // instead of four-way bank conflicts).
    auto store_tiles = [&](float *o, auto &&value) __attribute__((always_inline)) {
        // THROUGH: a store's 32-bit offset counts from the instruction's first row (16 rows at most)
        auto put = [&](int row0, int row, int chunk, const float4 &v) __attribute__((always_inline)) {
            if constexpr (!THROUGH) *reinterpret_cast<float4 *>(o + (int64_t)(m_base + row) * ldo + t0 * 16 + chunk * 4) = v;
            else store_through(through_rsrc(o + (int64_t)(m_base + row0) * ldo, 0xFFFFFFFCu),
                          ((uint32_t)(row - row0) * (uint32_t)ldo + (uint32_t)(t0 * 16 + chunk * 4)) * 4u, v);
        };
        if constexpr (NW == 3) {
            float *stage = reinterpret_cast<float *>(smem_u4) + wn * (MT * 16 * C::ROW3);
            stage_rows3(stage, value);
            for (int i0 = 0; i0 < MT * 16 * 12; i0 += 64) {       // (a multiple of 64)
                const int idx = i0 + lane, row = idx / 12, chunk = idx % 12, m = m_base + row, t = t0 + (chunk >> 2);
                const float4 v = *reinterpret_cast<const float4 *>(stage + row * C::ROW3 + chunk * 4);
                if (m < M && t < NT) put(i0 / 12, row, chunk, v);
            }
        } else if constexpr (KG > 1) {
            constexpr int CPR = NW * 4, RPI = 64 / CPR;       // 16-byte chunks per row, rows per store instruction
            float *stage = reinterpret_cast<float *>(smem_u4) + wn * (MT * NW * 256);
#pragma unroll
            for (int i = 0; i < MT; i++)
#pragma unroll
                for (int j = 0; j < NW; j++)
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const int row = i * 16 + 4 * g + r, chunk = (j * 4 + (cc >> 2)) ^ ((CPR / 2) * (g & 1));
                        stage[row * (NW * 16) + chunk * 4 + (cc & 3)] = value(i, j, r);
                    }
            // (the same wave wrote and reads: LDS keeps a wave's accesses in order)
#pragma unroll
            for (int k = 0; k < MT * 16 / RPI; k++) {
                const int row = k * RPI + lane / CPR, chunk = lane % CPR;
                const int phys = chunk ^ ((CPR / 2) * ((row >> 2) & 1));
                const float4 v = *reinterpret_cast<const float4 *>(stage + row * (NW * 16) + phys * 4);
                const int m = m_base + row, t = t0 + (chunk >> 2);
                if (m < M && t < NT) put(k * RPI, row, chunk, v);
            }
        } else {
#pragma unroll
            for (int j = 0; j < NW; j++) {
                const int t = t0 + j;
                if (t >= NT) continue;
#pragma unroll
                for (int i = 0; i < MT; i++)
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const int m = m_base + i * 16 + 4 * g + r;
                        if (m < M) o[(int64_t)m * ldo + t * 16 + cc] = value(i, j, r);
                    }
            }
        }
    };
    if (DIRECT && direct.kind != GEMM_OUT_PARTIAL) {
        // single split: the sums are complete.  The row factors of the block's rows are computed
        // once per workgroup (one thread per row) and handed out through LDS.
        float *scale_lds = reinterpret_cast<float *>(smem_u4 + (C::SMEM - 1024) / 16);   // the dump slot
        if constexpr (KG == 1) wait_vmcnt_lds<0>();          // (KG > 1: done before the merge)
        __syncthreads();
        if (tid < MT * 16) scale_lds[tid] = my_row_scale;
        __syncthreads();
        float sc[MT][4];
#pragma unroll
        for (int i = 0; i < MT; i++)
#pragma unroll
            for (int r = 0; r < 4; r++) sc[i][r] = scale_lds[i * 16 + 4 * g + r];
        if constexpr (ROPE) {
            // The workgroup's sums as rows in LDS, then eight rotation pairs of a row per item, the items of a row next to each
            // other: 16-byte stores, up to 128 contiguous bytes of a head's half.  The sums' trip through memory (25 MB at 512 rows of
            // 7B) and a launch less than qkv_rope_kernel behind a plain epilogue: prefill of 1000 tokens in chunks of 512, 2 layers
            // 1142 -> 1096 us; two narrow layers 81.4 -> 78.6 replayed, 82.5 -> 76.6 eager.
            static_assert(KG == 2, "the forms of two k groups");
            constexpr int PAIRS = WN * NW / 2, ITEMS = PAIRS * 2, PIECE = MT * 16 * C::ROW;
            static_assert(WN * NW % 2 == 0, "whole pairs");
            const RopeOutput &o = direct.rope;
            float *stage = reinterpret_cast<float *>(smem_u4);
            if (kg == 0) {
#pragma unroll
                for (int i = 0; i < MT; i++)
#pragma unroll
                    for (int j = 0; j < NW; j++)
#pragma unroll
                        for (int r = 0; r < 4; r++) stage[wn * PIECE + (i * 16 + 4 * g + r) * C::ROW + j * 16 + cc] = acc[i][j][r];
            }
            __syncthreads();
            const int half = o.hd >> 1, lg = o.hd == 128 ? 2 : 1;                       // (pairs of tiles per head: 4 or 2)
            for (int idx = tid; idx < MT * 16 * ITEMS; idx += WAVES * 64) {
                const int row = idx / ITEMS, item = idx % ITEMS, pr = item >> 1, oct = (item & 1) * 8;
                const int m = m_base + row, pair = bx * PAIRS + pr, head = pair >> lg, at = (pair & ((1 << lg) - 1)) * 16 + oct;
                if (m >= M || head >= o.Hq + 2 * o.Hkv) continue;
                const int b = m / o.R, r = m - b * o.R;
                int pos = o.ctx_len[b] + o.depth[r];
                pos = pos < o.max_pos ? pos : o.max_pos - 1;                            // host checks capacity; stay in bounds
                const float4 *ct = reinterpret_cast<const float4 *>(o.cos + (int64_t)pos * half + at), *st = reinterpret_cast<const float4 *>(o.sin + (int64_t)pos * half + at);
                const float4 c0 = ct[0], c1 = ct[1], s0 = st[0], s1 = st[1];
                const float c[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w}, sn[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
                const float *xs = stage + 2 * pr / NW * PIECE + row * C::ROW + 2 * pr % NW * 16 + oct;
                const float *ys = stage + (2 * pr + 1) / NW * PIECE + row * C::ROW + (2 * pr + 1) % NW * 16 + oct;
                const float4 x0 = *reinterpret_cast<const float4 *>(xs), x1 = *reinterpret_cast<const float4 *>(xs + 4);
                const float4 y0 = *reinterpret_cast<const float4 *>(ys), y1 = *reinterpret_cast<const float4 *>(ys + 4);
                const float xv[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w}, yv[8] = {y0.x, y0.y, y0.z, y0.w, y1.x, y1.y, y1.z, y1.w};
                const float rsc = scale_lds[row];
                uint32_t hi[2][4], lo[2][4];
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    uint16_t h[2][2], l[2][2];
#pragma unroll
                    for (int f = 0; f < 2; f++) {
                        float x = xv[e + f] * rsc, y = yv[e + f] * rsc;
                        if (head < o.Hq + o.Hkv) rope_pair(x, y, c[e + f], sn[e + f]);
                        split_bf16(x, h[0][f], l[0][f]);
                        split_bf16(y, h[1][f], l[1][f]);
                    }
#pragma unroll
                    for (int k = 0; k < 2; k++) {
                        hi[k][e >> 1] = h[k][0] | ((uint32_t)h[k][1] << 16);
                        lo[k][e >> 1] = l[k][0] | ((uint32_t)l[k][1] << 16);
                    }
                }
                uint16_t *dst, *dst_lo;
                if (head < o.Hq) {
                    const int64_t off = ((int64_t)m * o.Hq + head) * o.hd + at;
                    dst = o.q + off;
                    dst_lo = o.q_lo + off;
                } else {
                    const int kh = head - o.Hq;
                    const bool key = kh < o.Hkv;
                    const int64_t off = (((int64_t)b * o.Hkv + (key ? kh : kh - o.Hkv)) * o.R + r) * o.hd + at;
                    dst = (key ? o.k : o.v) + off;
                    dst_lo = (key ? o.k_lo : o.v_lo) + off;
                }
                *reinterpret_cast<uint4 *>(dst) = make_uint4(hi[0][0], hi[0][1], hi[0][2], hi[0][3]);
                *reinterpret_cast<uint4 *>(dst + half) = make_uint4(hi[1][0], hi[1][1], hi[1][2], hi[1][3]);
                *reinterpret_cast<uint4 *>(dst_lo) = make_uint4(lo[0][0], lo[0][1], lo[0][2], lo[0][3]);
                *reinterpret_cast<uint4 *>(dst_lo + half) = make_uint4(lo[1][0], lo[1][1], lo[1][2], lo[1][3]);
            }
        } else if (direct.kind == GEMM_OUT_SCALED) {
            // (the row factors sit in the dump slot behind the ring, outside the staging regions)
            store_tiles(out, [&](int i, int j, int r) { return acc[i][j][r] * sc[i][r]; });
        } else if constexpr (NW == 3) {
            // Gate and up tiles of the workgroup's 12 (WN * 3) alternate across the waves' regions; an
            // item is 8 features of one row: two pieces of gate, two of up, one 16-byte store per plane
            // (16 rows next to each other: 256 contiguous bytes of a fragment).
            constexpr int TILES = WN * 3, OCTS = TILES;               // 8 features per octet, 8 * TILES features
            // (8 * TILES features are whole k-steps: a d_ffn that ends inside one leaves its other half to the
            // workgroup that holds it, which stores zeros there)
            static_assert(TILES % 4 == 0, "whole k-steps of the next slab");
            float *stage = reinterpret_cast<float *>(smem_u4);
            stage_rows3(stage + wn * (MT * 16 * C::ROW3), [&](int i, int j, int r) { return acc[i][j][r]; });
            __syncthreads();
            const int F = direct.d_ffn, n_ksteps = (F + 31) >> 5, mt_all = (M + 15) >> 4;
            auto piece = [&](int tile, int row, int c4) __attribute__((always_inline)) {
                return *reinterpret_cast<const float4 *>(stage + (tile / 3) * (MT * 16 * C::ROW3) + row * C::ROW3 + (tile % 3) * 16 + c4);
            };
            for (int idx = tid; idx < MT * 16 * OCTS; idx += WAVES * 64) {
                const int row = idx % (MT * 16), oct = idx / (MT * 16);                  // octet inside the workgroup
                const int f = bx * (TILES * 8) + oct * 8, gate = 2 * (oct >> 1), c4 = (oct & 1) * 8;
                if ((f >> 5) >= n_ksteps || bz * MT + (row >> 4) >= mt_all) continue;
                const float sc = scale_lds[row];
                uint32_t hi[4], lo[4];
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    const float4 gv = piece(gate, row, c4 + 4 * q), uv = piece(gate + 1, row, c4 + 4 * q);
                    const float gs[4] = {gv.x * sc, gv.y * sc, gv.z * sc, gv.w * sc}, us[4] = {uv.x * sc, uv.y * sc, uv.z * sc, uv.w * sc};
                    uint16_t h[4], l[4];
#pragma unroll
                    for (int e = 0; e < 4; e++) split_bf16(f < F ? gs[e] / (1.0f + expf(-gs[e])) * us[e] : 0.f, h[e], l[e]);
                    hi[2 * q] = h[0] | ((uint32_t)h[1] << 16); hi[2 * q + 1] = h[2] | ((uint32_t)h[3] << 16);
                    lo[2 * q] = l[0] | ((uint32_t)l[1] << 16); lo[2 * q + 1] = l[2] | ((uint32_t)l[3] << 16);
                }
                uint16_t *dst = direct.act_frag + frag_index(0, m_base + row, f, n_ksteps, mt_all, 0);
                *reinterpret_cast<uint4 *>(dst) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
                *reinterpret_cast<uint4 *>(dst + (int64_t)n_ksteps * mt_all * 512) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            }
        } else if constexpr (NW % 2 == 0) {
            // Tiles alternate gate, up: accumulators (j, j+1) hold gate and up of the same 16
            // features for the same rows and lanes.  The workgroup's WN*NW*8 features are whole
            // k-steps of the next GEMM: the gated values are laid out as its fragments in LDS
            // (two planes) and leave as whole 1 KiB fragments, 16 bytes per lane.
            constexpr int FEATS = WN * NW * 8, HK = FEATS / 16;           // features, half k-steps per workgroup
            static_assert(FEATS % 16 == 0, "whole half fragments");
            static_assert(2 * HK * MT * 512 <= C::SMEM, "staging fits the ring");
            // a fragment (16 rows x 32 features) is two contiguous halves of 16 features
            // (512 bytes: [feature octet][row][8 features]); the workgroup's features are whole halves
            const int F = direct.d_ffn, n_ksteps = (F + 31) >> 5, mt_all = (M + 15) >> 4;
            uint16_t *stage = reinterpret_cast<uint16_t *>(smem_u4);     // [plane][HK][MT][256]
            // (every wave is past the ring and the merge area: synchronised above)
#pragma unroll
            for (int j = 0; j < NW; j += 2) {
                const int f_local = (wn * NW + j) * 8 + cc;              // feature inside the workgroup
                const int hk = f_local >> 4, pos = ((f_local >> 3) & 1) * 128 + (f_local & 7);
                const bool live = (t0 + j) < NT;
#pragma unroll
                for (int i = 0; i < MT; i++)
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const float gs = acc[i][j][r] * sc[i][r];
                        const float v = live ? gs / (1.0f + expf(-gs)) * (acc[i][j + 1][r] * sc[i][r]) : 0.f;
                        uint16_t hi, lo;
                        split_bf16(v, hi, lo);
                        const int at = pos + (4 * g + r) * 8;            // row 4g+r of m-tile i
                        if (PACK && i == MT - 1) {                       // the output slab packs its last tile the same way
                            if (4 * g + r < pack_off) stage[((0 * HK + hk) * MT + i) * 256 + at] = hi;
                            if (4 * g + r < rows_last) stage[((0 * HK + hk) * MT + i) * 256 + at + pack_off * 8] = lo;
                        } else {
                            stage[((0 * HK + hk) * MT + i) * 256 + at] = hi;
                            stage[((1 * HK + hk) * MT + i) * 256 + at] = lo;
                        }
                    }
            }
            __syncthreads();
            // fragment (plane, ks, mt) of the slab starts at ((plane * n_ksteps + ks) * mt_all + mt) KiB;
            // k-steps at or beyond n_ksteps and m-tiles beyond the slab do not exist.
            // One store instruction moves two halves (32 lanes x 16 bytes each).
            const int hk0 = bx * HK, mt0 = bz * MT, half_lane = lane >> 5, l32 = lane & 31;
            for (int pr = wn; pr < HK * MT * 2 / 2; pr += WN) {
                const int idx = pr * 2 + half_lane;                      // (plane, hk, i) flattened, as staged
                const int plane = idx / (HK * MT), hk = (idx / MT) % HK, i = idx % MT;
                const int hkg = hk0 + hk;                                // half k-step in the whole slab
                if ((hkg >> 1) >= n_ksteps || mt0 + i >= mt_all) continue;   // (a last half past F holds zeros)
                if (PACK && plane == 1 && i == MT - 1) continue;             // lives in the high plane's fragment
                const uint4 v = reinterpret_cast<const uint4 *>(stage)[idx * 32 + l32];
                reinterpret_cast<uint4 *>(direct.act_frag)[(((int64_t)plane * n_ksteps + (hkg >> 1)) * mt_all + mt0 + i) * 64 +
                                                           (hkg & 1) * 32 + l32] = v;
            }
            // A feature count that is an odd number of 16-feature halves leaves the second half of
            // the slab's last k-step without a feature.  Where the grid's columns run past F, the
            // loop above has stored zeros there (tiles beyond the matrix are not live); where they
            // end exactly at F, the workgroup that owns the last half clears it here: the down
            // projection multiplies it by zero-padded weights, and 0 x NaN of stale memory is NaN.
            const int n_half = F >> 4;
            if ((n_half & 1) && hk0 + HK == n_half && lane < 32) {
                for (int pr = wn; pr < 2 * MT; pr += WN) {
                    const int plane = pr / MT, i = pr % MT;
                    if (mt0 + i >= mt_all || (PACK && plane == 1 && i == MT - 1)) continue;
                    reinterpret_cast<uint4 *>(direct.act_frag)[(((int64_t)plane * n_ksteps + (n_half >> 1)) * mt_all + mt0 + i) * 64 +
                                                               32 + lane] = make_uint4(0u, 0u, 0u, 0u);
                }
            }
        }
        return;
    }
    store_tiles(out + (int64_t)by * M * ldo, [&](int i, int j, int r) { return acc[i][j][r]; });
}

// out[m][n] = rowscale(m) * sum over splits of partial[s][m][n], in split order.  Four columns per
// thread and eight splits' loads in flight (one load per split and column, each waited for, before: the
// 13B down product at 37 rows, 6 splits, single plane, 33.5 -> 32.2 us as a whole, with the second
// plane's empty fragments no longer written): launch plus one or two round trips.
// A workgroup takes 256 columns of four rows: workgroups go round the XCDs by their columns, and where
// a GEMM workgroup is 256 columns wide and N a multiple of 2048 the sums are read from the L2 that they
// were left in (1024 columns of one row instead, whole calls: 68 x 12288 x 4096, two planes, 35.1 us
// against 32.1; 400 x 2048 x 1024 22.2 against 18.3; single plane 128 x 4096 x 4096 26.3 against 20.3).
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float *__restrict__ partial, int splits, int M,
                                                              int64_t N, int64_t ld, float *__restrict__ out, RowScale rs) {
    const int64_t n4 = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
    const int m = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (m >= M || 4 * n4 >= N) return;                  // N is a multiple of 16
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < splits; s0 += 8) {
        float4 p[8];
#pragma unroll
        for (int u = 0; u < 8; u++)
            p[u] = reinterpret_cast<const float4 *>(partial + ((int64_t)min(s0 + u, splits - 1) * M + m) * ld)[n4];
#pragma unroll
        for (int u = 0; u < 8; u++)
            if (s0 + u < splits) { acc.x += p[u].x; acc.y += p[u].y; acc.z += p[u].z; acc.w += p[u].w; }
    }
    const float sc = row_scale(rs, m);
    reinterpret_cast<float4 *>(out + (int64_t)m * N)[n4] = make_float4(acc.x * sc, acc.y * sc, acc.z * sc, acc.w * sc);
}

// Pure permutation: row-major [N][K] bf16 -> packed tiles (see file header).
__global__ void pack_weight_kernel(const uint16_t *__restrict__ src, int64_t N, int64_t K, int64_t KS,
                                   uint4 *__restrict__ dst, int64_t tile0, int64_t tile_stride,
                                   int64_t total_tiles) {
    const int64_t blk = blockIdx.x;            // (source tile, k-step incl. the padding step)
    const int64_t t = blk / KS, s = blk % KS;
    const int lane = threadIdx.x;
    const int64_t n = t * 16 + (lane & 15), k = s * 32 + (lane >> 4) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (k < K) v = *reinterpret_cast<const uint4 *>(src + n * K + k);
    dst[packed_block(tile0 + t * tile_stride, s, total_tiles) * 64 + lane] = v;
}

// Row-major bf16 planes -> A-operand fragment order (used by the stand-alone GEMM entry point;
// inside the verify step the producing kernels write this layout directly).
__global__ void to_fragments_kernel(const uint16_t *__restrict__ a_hi, const uint16_t *__restrict__ a_lo, int M,
                                    int K, int64_t lda, int KS, int m_tiles, uint4 *__restrict__ dst) {
    const int ks = blockIdx.x, mt = blockIdx.y, plane = blockIdx.z, lane = threadIdx.x;
    const uint16_t *src = plane ? a_lo : a_hi;
    const int m = mt * 16 + (lane & 15), k = ks * 32 + (lane >> 4) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (src && m < M && k < K) v = *reinterpret_cast<const uint4 *>(src + (int64_t)m * lda + k);
    const int pack_off = a_lo ? frag_pack_offset(M) : 0;
    if (pack_off && mt == m_tiles - 1) {
        // both planes of a packed last tile share the high plane's fragment (disjoint rows)
        const int row = lane & 15;
        if (plane == 0 && row < pack_off) dst[((int64_t)ks * m_tiles + mt) * 64 + lane] = v;
        if (plane == 1 && m < M) dst[((int64_t)ks * m_tiles + mt) * 64 + lane + pack_off] = v;
        return;
    }
    dst[(((int64_t)plane * KS + ks) * m_tiles + mt) * 64 + lane] = v;
}

// Launch shapes.  Wide groups reuse each activation fragment for more weight tiles (the
// L2->LDS slab traffic is what limits narrow ones) but produce wider split-K partials; deep
// rings and more waves keep more weight bytes in flight per CU.
struct GemmVariant { int nw, waves, depth, kgroups; };
static const GemmVariant g_variants[] = {
    {1, 4, 4, 1}, {2, 4, 4, 1}, {4, 4, 4, 1}, {2, 8, 6, 1}, {4, 8, 6, 1},
    {2, 8, 4, 2}, {4, 8, 4, 2}, {1, 8, 4, 2}, {2, 8, 3, 2}, {2, 16, 3, 2}, {2, 6, 3, 2}, {2, 14, 3, 2},
    {4, 8, 3, 2},     // 12: tall passes (6 to 11 m-tiles per pass), 16 tiles per k group (or 12: GemmPlan::tall_tiles; always from 10 m-tiles on)
};
#define GEMM_N_VARIANTS ((int)(sizeof(g_variants) / sizeof(g_variants[0])))
static int g_force_variant = -1, g_force_splits = -1;
// variant: >= 0 forces that workgroup shape, -1 the heuristic, -2 the heuristic without tall passes
void gemm_force_plan(int variant, int splits) { g_force_variant = variant < -2 ? -1 : variant; g_force_splits = splits; }
bool gemm_plan_forced() { return g_force_variant != -1 || g_force_splits > 0; }

GemmPlan gemm_plan(int m_rows, int64_t n_rows, int64_t k, int planes) {
    GemmPlan p;
    const int64_t NT = n_rows / 16, KS = (k + 31) / 32;
    // Shapes measured on MI355X at 68 rows (7B- and 70B-like widths): 2 k groups of 4 waves
    // with 2 tiles per wave (128 columns per workgroup) or of 8 waves (256 columns); as many
    // splits as give one round of 256 equal workgroups, but no more than 8 for the narrow ones,
    // whose partial sums are re-read by a row-wise consumer.
    const int m_tiles = (m_rows + 15) / 16;
    p.variant = NT < 3000 ? 8 : 6;
    // 16 waves (256 columns per workgroup, half the activation-slab traffic per weight byte)
    // for the widest matrices, the QKV-like widths and narrow matrices with a very long k;
    // these and the 6- and 14-wave forms are instantiated for 1 and 5 m-tiles per pass
    const bool wide16 = NT >= 3000 || (NT >= 512 && NT < 1024 && (NT >= 640 || KS >= 512));
    const bool mt_1_or_5 = !(m_tiles == 2 || m_tiles == 3 || m_tiles == 6 || m_tiles == 7);
    if (wide16 && mt_1_or_5) p.variant = 9;
    // matrices wide enough for a single k split: the workgroup width (3, 4, 7 or 8 waves of 2
    // tiles per k group) that puts the most workgroups on the 256 CUs in one round
    if (NT >= 1024 && mt_1_or_5) {
        static const int wn_of[4] = {3, 4, 7, 8}, variant_of[4] = {10, 8, 11, 9};
        int64_t best = 0;
        for (int i = 0; i < 4; i++) {
            const int64_t wgs = (NT + 2 * wn_of[i] - 1) / (2 * wn_of[i]);
            if (wgs <= 256 && wgs >= best) { best = wgs; p.variant = variant_of[i]; }
        }
    }
    if (m_tiles == 6 || m_tiles == 7) p.variant = 8;            // one pass: 4 tiles per wave x 7 m-tiles of accumulators would spill
    // Many rows (prefill chunks, batches, per-node mask groups on large trees): the launch
    // makes `passes` row passes of 5 m-tiles over the weights, every pass its own set of
    // workgroups.  The passes fill the CUs, so fewer k splits are needed, and the widest
    // workgroups (16 waves, or 14 on the gate/up-like widths) share each activation fragment
    // among the most weight tiles.
    // A single-plane slab has no forms of 6 to 11 m-tiles, neither the one-pass nor the tall ones.  It was
    // given their plans and ran them in passes of 5; planned as what it is (whole calls, one plane,
    // splits and workgroups for two planes -> its own): 96 x 22016 x 4096 65.9 -> 56.0 us, 128 rows
    // 70.4 -> 58.8, 272 rows 108.6 -> 99.6; 272 x 12288 x 4096 66.4 -> 54.1; 170 x 4096 x 11008 51.9 -> 42.1.
    // The passes begin at 6 m-tiles, but below 256 weight tiles at 8: a 16-tile workgroup is most of such
    // a matrix (96 x 256 x 688 10.5 us in the 8-tile form, 12.9; 96 x 1024 x 4096 13.5 and 14.8).
    int passes = m_tiles > (planes == 1 && NT >= 256 ? 5 : 7) ? (m_tiles + 4) / 5 : 1;
    // What a launch is estimated to take: the traffic through one CU's vector L1 (weights + activation slab of the
    // workgroup's k range) times the number of rounds the workgroups take on the 256 CUs, plus the split-K
    // partial sums.
    auto estimate = [&](int mt, int n_pass, int tiles_wg, int *splits_out) {
        const int64_t wgs_n = (NT + tiles_wg - 1) / tiles_wg;
        int64_t sp = 256 / (wgs_n * n_pass);
        if (sp > KS / 8) sp = KS / 8;
        if (NT < 512 && sp > 8) sp = 8;
        if (sp > 32) sp = 32;
        if (g_force_splits > 0) sp = g_force_splits;
        if (sp < 1) sp = 1;
        const int64_t per = (KS + sp - 1) / sp;
        sp = (KS + per - 1) / per;
        const double per_wg = (double)(tiles_wg + planes * mt) * 1024.0 * (double)per;
        const double rounds = (double)((wgs_n * n_pass * sp + 255) / 256);
        double t = rounds * per_wg / 41e9;                              // ~17 B/clk through one CU's L1
        if (sp > 1) t += 2.0 * (double)sp * m_rows * (double)n_rows * 4.0 / 4e12;
        *splits_out = (int)sp;
        return t;
    };
    // 14 waves (14 tiles per workgroup) put more workgroups on the CUs than 16 from 1024 to 2999 tiles, 5 to 10 % where both
    // take as many rounds (22016 x 4096, 170 rows, 16 / 14 waves: 132 / 124 us; 272 rows 139 / 129), but a round more of
    // them costs far more than that: 32000 x 4096, 150 rows 84 / 129 us, 300 rows 149 / 192, 440 rows 214 / 256; 27648 x 5120,
    // 512 rows 260 / 308; 40960 x 2048, 240 rows 80 / 109; one plane 67 / 103, 119 / 148, 171 / 193, 202 / 228, 65 / 86.
    // (Passes of 5 by themselves: with two planes 440 and 512 rows take a tall form.)  The estimate ranks the two right
    // wherever they differ by more than 5 % (196 launches).
    double t_five = 0.0;                                     // passes of 5 m-tiles (or the one pass of 6 or 7)
    int sp_now = 1;
    if (passes >= 2) {
        p.variant = 9;
        t_five = estimate(5, passes, 16, &sp_now);
        if (NT >= 1024 && NT < 3000) {
            int sp14 = 1;
            const double t14 = estimate(5, passes, 14, &sp14);
            if (t14 <= t_five || sp_now > 1) { p.variant = 11; t_five = t14; }   // (more splits than one: not measured, and more scratch)
        }
    } else {
        t_five = estimate(m_tiles, 1, 8, &sp_now);
    }
    p.mt_pass = 0;
    p.tall_tiles = 16;
    // Tall passes (6 to 9 m-tiles per pass, variant 12): fewer passes over the weights and 16 weight tiles per
    // activation fragment, against fewer, fatter workgroups.  The tall form is taken where the same estimate promises a
    // fifth less than the others, or, with 10 us for what every launch costs besides, a seventh (what is less than that
    // it does not resolve.  A fifth alone left these behind, before / now: 13B gate/up, 81 rows 71 / 66 us, 117 rows 91 / 85, 409
    // rows 239 / 215; 70B QKV, 208 rows 83 / 79; 7088 x 16128, 164 rows 113 / 91.  Over 117 launches of 81 to 512 rows that a
    // seventh alone gives a tall form the median is 8 % less time; one pass of 7 m-tiles for two k splits instead of one
    // neither gains nor loses, 3 % either way).
    if (planes == 2 && m_tiles >= 6 && g_force_variant == -1) {
        const double launch = 10e-6;
        const int five_passes = passes, five_variant = p.variant, five_tiles = passes >= 2 ? 5 * passes : m_tiles;
        double t_ref = t_five;
        // (a launch of 14-wave workgroups is what the tall forms were measured against where that is what the width
        // suggests; what they have to beat where 16 waves are taken instead is below)
        if (passes >= 2 && NT >= 1024 && NT < 3000) {
            int sp14 = 1;
            t_ref = estimate(5, passes, 14, &sp14);
        }
        const double fifth = 0.8 * t_ref, seventh = 0.86 * (t_ref + launch) - launch;
        double t_best = fifth > seventh ? fifth : seventh;
        // 16 or 12 weight tiles per workgroup: a launch whose 16-tile workgroups leave CUs idle (172 of
        // 256 at 272 rows of the 7B gate/up, 9 m-tiles) or take a nearly empty last round is cut finer
        // where the estimate falls by a twentieth (gate/up, K = 4096: 170 rows 77.5 -> 72.1 us,
        // 272 rows 102.4 -> 95.7, 512 rows 198 -> 167 in passes of 8 instead of 5; K = 512, 265 rows:
        // 26.0 -> 23.9; 7B QKV at 512 rows 99.8 -> 91.5).  Between 81 and 144 rows that can mean two or
        // four k splits where passes of 5 or 7 m-tiles had one or two, and for gate/up the gating in a
        // kernel of its own, which the estimate leaves out; it pays all the same (one 7B layer and the
        // LM head, all reducers included, 12 tiles at one split only -> this rule: 84 rows 228 -> 223 us,
        // 96 243 -> 233, 105 260 -> 253, 112 261 -> 254, 120 267 -> 259, 128 271 -> 265, 134 300 -> 292,
        // 144 300 -> 294, four sequences of 68 454 -> 440).  Narrower workgroups were not built: at 12
        // tiles the activation reads already take five sixths of the LDS cycles that the multiplies last.
        // More splits need more scratch: where they would not fit the static one of bita_gemm_noalloc a form is
        // left out, so that it takes no shape away from that call (none of the 7B, 13B and 70B matrices up to 544 rows
        // comes near), but for 16-tile forms that promise a fifth, which never fitted.
        for (int cap = 9; cap >= 6; cap--) {
            const int n_pass = (m_tiles + cap - 1) / cap, mt = (m_tiles + n_pass - 1) / n_pass;
            if (mt < 6) continue;
            int sp = 1;
            for (int tiles : {16, 12}) {
                // (small matrices, fewer than half the CUs at 16 tiles, are latency: the shorter epilogue wins)
                if (tiles == 12 && (NT + 15) / 16 * n_pass * sp < 128) continue;
                const double t = estimate(mt, n_pass, tiles, &sp);
                if (sp > 1 && (tiles == 12 || t > fifth) &&
                    (((size_t)sp * m_rows * n_rows * 4 + 255) & ~(size_t)255) + frag_bytes(m_rows, k) > BITA_NOALLOC_SCRATCH_BYTES)
                    continue;
                // (in two passes 12 tiles that promise a fifth stand against 16 that promise a seventh: 12 of 15 such launches of
                // 169 to 221 rows lost 1 to 6 % with 16, three gained 3 to 4; in one pass or three 16 gain more than they lose)
                const bool stands = n_pass == 2 && t < fifth && t_best >= fifth;
                if (t < (tiles == 12 && p.mt_pass && !stands ? 0.95 : 1.0) * t_best) { t_best = t; p.mt_pass = mt; passes = n_pass; p.variant = 12; p.tall_tiles = tiles; }
            }
        }
        // Against the form that would run instead the estimate errs with the m-tiles that the passes execute.  Where the tall
        // ones execute no more, a tie goes to them (19440 x 4552, 211 rows, 14 m-tiles for 15, estimates alike, tall / passes
        // of 5 84 / 88 us; as many, 16720 x 2240, 508 rows 85 / 89, 17504 x 744, 490 rows 45.8 / 45.0).  Where they execute more
        // it promises them too much: with a tenth or less the passes of 5 are 1 to 7 % faster (32000 x 8192, 301 rows, 21 for 20,
        // estimates alike, 309 / 288; 40960 x 2048, 460 rows, 32 for 30, 0.92 of the other, 164 / 155), and with 0.87 of it
        // from k = 2560 on (27648 x 5120, 538 rows, 36 for 35, 281 / 267; but 26928 x 1496, 547 rows 99 / 103, and with 0.865 of
        // it 33312 x 3472, 524 rows 240 / 245).  Short k's, below 24 k-steps, are its own again (32048 x 432, 295 rows 33 / 35).
        const bool more = p.mt_pass && passes * p.mt_pass > five_tiles;
        if (t_best >= (!more || KS < 24 ? 1.01 : KS < 80 ? 0.9 : 0.87) * t_five) {
            p.mt_pass = 0;
            p.tall_tiles = 16;
            passes = five_passes;
            p.variant = five_variant;
        }
        // Passes of 10 and 11 m-tiles, on 12 weight tiles, where the estimate falls by another tenth: row counts that 6 to 9 fill
        // badly.  Without / with them, us: 22016 x 4096, 300 rows (2 passes of 10 for 4 of 5) 132.1 / 100.0, 340 (2 of 11 for 5) 136.2 /
        // 109.0, 145 to 160 rows (one of 10 in two k splits for 2 passes of 5 in one) 75.0 / 66.5; 12288 x 4096, 150 rows (4 splits for 2)
        // 48.7 / 46.8, 289 rows 73.6 / 66.6; 27648 x 5120, 480 rows 243 / 222; 40960 x 2048, 152 rows 76.1 / 58.7, 170 (one of 11 for two
        // of 6) 69.9 / 63.1; 11008 x 8192, 147 rows 84.8 / 64.1.  Of 34 launches that take them the slowest are 1 to 2 % behind, within
        // what one plan differs from itself (16720 x 2240, 145 rows 41.0 / 41.9).  More k splits mean a gating or a rotation in a kernel
        // of its own, which the estimate leaves out, and it pays all the same in place of passes of 5 (two 7B layers and a small head, 145
        // rows 413 / 397, 150 418 / 405, 160 423 / 410, 289 646 / 567; of 13B widths, 470 rows 1198 / 1153), but not in place of two passes of 6
        // (22016 x 4096, 161 rows 67.4 / 69.3, 166 rows 68.0 / 71.9, the two layers 414 / 418 and 416 / 422; 19440 x 4552, 176 rows
        // 72.8 / 78.1; but 20480 x 6144, 170 rows 96.0 / 92.5): a tall form gives way only to one of no more splits.
        const GemmVariant &v = g_variants[p.variant];
        int sp = 1;
        double t_now = estimate(p.mt_pass ? p.mt_pass : 5, passes, p.mt_pass ? p.tall_tiles : v.nw * v.waves / v.kgroups, &sp);
        t_now *= 0.9;
        const int tall_splits = p.mt_pass ? sp : 32;
        for (int mt = 10; mt <= 11 && passes >= 2; mt++) {
            const int n_pass = (m_tiles + mt - 1) / mt;
            if ((m_tiles + n_pass - 1) / n_pass != mt) continue;
            const double t = estimate(mt, n_pass, 12, &sp);
            if ((NT + 15) / 16 * n_pass * sp < 128 || t >= t_now || sp > tall_splits) continue;
            if (sp > 1 && (((size_t)sp * m_rows * n_rows * 4 + 255) & ~(size_t)255) + frag_bytes(m_rows, k) > BITA_NOALLOC_SCRATCH_BYTES) continue;
            t_now = t; p.mt_pass = mt; passes = n_pass; p.variant = 12; p.tall_tiles = 12;
        }
    }
    if (g_force_variant >= 0 && g_force_variant < GEMM_N_VARIANTS) p.variant = g_force_variant;
    const GemmVariant &v = g_variants[p.variant];
    const int tiles_wg = p.mt_pass ? p.tall_tiles : v.nw * v.waves / v.kgroups;
    const int64_t wgs_n = (NT + tiles_wg - 1) / tiles_wg;
    int64_t splits = (v.waves > 4 ? 256 : 512) / (wgs_n * passes);
    const int64_t max_splits = KS / 8;                          // at least 8 stages per split
    if (splits > max_splits) splits = max_splits;
    if (NT < 512 && splits > 8) splits = 8;
    if (splits > 32) splits = 32;
    if (g_force_splits > 0) splits = g_force_splits;
    if (splits < 1) splits = 1;
    const int64_t per = (KS + splits - 1) / splits;
    p.ksteps_per_split = (int)per;
    p.splits = (int)((KS + per - 1) / per);
    return p;
}

// Which loop: the two k groups in turns, or both at once.
// Turns always: two planes and complete sums from 6 m-tiles on (38 products of 81 to 512 rows 0.85 to 1.01 of the time), passes of 10 and 11; one
// plane in passes of 5 on fewer than 14 waves (20 to 80 rows of wide matrices 5 to 9 % faster, narrow ones the same: 99 launches of 4 to 32
// k-steps a group 0.998 of the time).
// Never: the packed 5 of a 64-node tree and the forms that 73 to 80 rows of two planes take (68 rows, both at once / turns: 12288 x
// 4096 30.4 / 30.9 us, 32000 x 4096 54.2 / 54.5, 57344 x 8192 154 / 153; 80 rows: 32000 x 4096 56.0 / 56.6, 8192 x 8192 37.5 / 38.2); one
// plane on 14 and 16 waves (40 launches 1.000, five rows of the long ones 1.02).
// The rest by gemm_turns_pay.  Passes of 5 with complete sums need 40 k-steps and more workgroups than half of the CUs (31 products 0.975 of
// the time, 8192 x 28672, 300 rows 270 -> 251 us, 12288 x 4096, 300 rows 76.8 -> 73.5; the other 147 1.000, 12432 x 1040, 166 rows 25.5 -> 27.1).
// Split sums gain by turns as products alone; inside a layer, between kernels that leave the clock high, only where the m-tiles times a
// split's k-steps are more than 150 times the splits.  What turns cost a layer's time (two layers of 7B and 13B widths, one of 70B, each product
// by itself, us): below the line 81 to 128 rows QKV of 26 k-steps in 5 splits +2 to +8, of 40 in 4 +10, down of 43 in 8 (161 to 256 rows) +13, of 72 in
// 6 +2, of 112 in 8 (105 to 128 rows) +7, O of 54 in 3 +10, of 64 in 4 +4; above it QKV of 64 and 80 in 2 (161 to 272 rows) -2 to -9, of 86 in 3
// -5, down of 108 in 4 (400 rows) -12, of 224 in 4 -4 to -15, of 448 in 2 -25.  One pass of 6 m-tiles is below it at any length (gate/up at 81
// and 96 rows, 64 and 80 in 2, 0 to +6).  Cards differ below the line: of five, three lose 1 to 5 % of a layer by turns there, two gain up to 2.
// With this rule 43 row counts of the three widths take 0.86 to 1.003 of what they took with both groups at once everywhere.
static bool gemm_turns_pay(int mt, int passes, int64_t workgroups, const GemmPlan &p) {
    if (p.splits == 1) return mt > 5 || (p.ksteps_per_split >= 40 && workgroups > 128);
    return mt * p.ksteps_per_split > 150 * p.splits && workgroups > 128 && (mt > 6 || passes > 1);
}
constexpr bool gemm_either_loop(int MT, bool SPLIT, int WAVES, int KG, bool DIRECT, bool PACK) {
    return KG == 2 && SPLIT && !PACK && ((MT == 5 && WAVES >= 14) || (MT > 5 && MT < 10 && !DIRECT));
}
constexpr bool gemm_turns(int MT, bool SPLIT, int WAVES, int KG, bool DIRECT, bool PACK) {
    return KG == 2 && !gemm_either_loop(MT, SPLIT, WAVES, KG, DIRECT, PACK) && (MT > 5 || (MT == 5 && !SPLIT && WAVES < 14));
}
template <int MT, int NW, bool SPLIT, int WAVES, int D, int KG, bool DIRECT, bool PACK = false, bool THROUGH = DIRECT, bool ROPE = false,
          bool TURNS = gemm_turns(MT, SPLIT, WAVES, KG, DIRECT, PACK)>
static void launch_gemm_t(const void *a_frag, int M, int64_t K, const void *w, int64_t N, float *out, int64_t ldo,
                          const GemmPlan &p, hipStream_t s, const GemmOutput &direct) {
    if constexpr (gemm_either_loop(MT, SPLIT, WAVES, KG, DIRECT, PACK) && !TURNS) {
        constexpr int TILES = GemmCfg<MT, NW, SPLIT, 1, D, WAVES, KG>::WN * NW;
        const int passes = (M + 16 * MT - 1) / (16 * MT);
        if (M > 80 && gemm_turns_pay(MT, passes, (N / 16 + TILES - 1) / TILES * p.splits * passes, p)) {
            launch_gemm_t<MT, NW, SPLIT, WAVES, D, KG, DIRECT, PACK, THROUGH, ROPE, true>(a_frag, M, K, w, N, out, ldo, p, s, direct);
            return;
        }
    }
    if constexpr (DIRECT && SPLIT && KG == 2 && !ROPE && (NW > 2 || WAVES == 8 || WAVES == 16) && D == 3) {
        if (direct.kind == GEMM_OUT_ROPE) {                    // (the forms that gemm_direct_output_possible says)
            launch_gemm_t<MT, NW, SPLIT, WAVES, D, KG, DIRECT, PACK, THROUGH, true, TURNS>(a_frag, M, K, w, N, out, ldo, p, s, direct);
            return;
        }
    }
    if constexpr (MT > 1 && SPLIT && KG > 1 && !THROUGH) {
        if (p.splits > 1 && (int64_t)p.splits * M * ldo * 4 >= (8 << 20) && ldo <= GEMM_THROUGH_MAX_LD) {
            launch_gemm_t<MT, NW, SPLIT, WAVES, D, KG, DIRECT, PACK, true, ROPE, TURNS>(a_frag, M, K, w, N, out, ldo, p, s, direct);
            return;
        }
    }
    constexpr int KC = 1;
    using C = GemmCfg<MT, NW, SPLIT, KC, D, WAVES, KG, PACK, ROPE>;
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)gemm_skinny_kernel<MT, NW, SPLIT, KC, D, WAVES, KG, DIRECT, PACK, THROUGH, ROPE, TURNS>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, C::SMEM);
        attr_set = true;
    }
    const int NT = (int)(N / 16), KS = (int)((K + 31) / 32), m_tiles = (M + 15) / 16;
    dim3 grid((NT + C::WN * NW - 1) / (C::WN * NW), p.splits, (m_tiles + MT - 1) / MT);
    hipLaunchKernelGGL((gemm_skinny_kernel<MT, NW, SPLIT, KC, D, WAVES, KG, DIRECT, PACK, THROUGH, ROPE, TURNS>), grid, dim3(WAVES * 64), C::SMEM, s,
                       (const uint4 *)a_frag, (const uint4 *)w, KS * m_tiles, M, m_tiles, NT, KS, p.ksteps_per_split,
                       (int)grid.x, (int)grid.y, (int)grid.z, ROPE ? direct.rope.hd / 16 : 0, out, ldo, direct);
}

template <int MT, bool SPLIT>
static void launch_gemm_v(const void *a_frag, int M, int64_t K, const void *w, int64_t N, float *out, int64_t ldo,
                          const GemmPlan &p, hipStream_t s, const GemmOutput &direct) {
    // the instantiations with an output epilogue exist for the k-group shapes only
    // a two-plane slab whose last m-tile is packed (frag_pack_offset) takes the instantiation
    // that reads it so; both exist for one and five m-tiles, the only slabs that pack
    constexpr bool CAN_PACK = SPLIT && (MT == 1 || MT == 5);
    const bool pack = CAN_PACK && frag_pack_offset(M) != 0;
#define T(nw, waves, d, kg, dir) do { \
        if constexpr (CAN_PACK) { \
            if (pack) { launch_gemm_t<MT, nw, SPLIT, waves, d, kg, dir, true>(a_frag, M, K, w, N, out, ldo, p, s, direct); break; } \
        } \
        launch_gemm_t<MT, nw, SPLIT, waves, d, kg, dir, false>(a_frag, M, K, w, N, out, ldo, p, s, direct); \
    } while (0)
#define V(i, nw, waves, d, kg) case i: T(nw, waves, d, kg, false); break;
#define W(i, nw, waves, d, kg) case i: \
        if (direct.kind != GEMM_OUT_PARTIAL) T(nw, waves, d, kg, true); \
        else T(nw, waves, d, kg, false); \
        break;
    switch (p.variant) {
        V(0, 1, 4, 4, 1) V(1, 2, 4, 4, 1) V(2, 4, 4, 4, 1) V(3, 2, 8, 6, 1) V(4, 4, 8, 6, 1)
        W(5, 2, 8, 4, 2) W(6, 4, 8, 4, 2) V(7, 1, 8, 4, 2) W(8, 2, 8, 3, 2) W(9, 2, 16, 3, 2) W(10, 2, 6, 3, 2) W(11, 2, 14, 3, 2)
    }
#undef V
#undef W
#undef T
}

// two planes, the planner's variants (6 and 8) only; more than 5 m-tiles with variant 8 alone (registers, LDS ring)
template <int MT>
static void launch_gemm_k(const void *a_frag, int M, int64_t K, const void *w, int64_t N, float *out, int64_t ldo,
                          const GemmPlan &p, hipStream_t s, const GemmOutput &direct) {
    const bool d = direct.kind != GEMM_OUT_PARTIAL;
    if constexpr (MT <= 5) {
        if (p.variant == 6) {
            if (d) launch_gemm_t<MT, 4, true, 8, 4, 2, true>(a_frag, M, K, w, N, out, ldo, p, s, direct);
            else launch_gemm_t<MT, 4, true, 8, 4, 2, false>(a_frag, M, K, w, N, out, ldo, p, s, direct);
            return;
        }
    }
    if (d) launch_gemm_t<MT, 2, true, 8, 3, 2, true>(a_frag, M, K, w, N, out, ldo, p, s, direct);
    else launch_gemm_t<MT, 2, true, 8, 3, 2, false>(a_frag, M, K, w, N, out, ldo, p, s, direct);
}

// a_frag: activations in fragment order, [planes][k-steps][m-tiles][64] x 16 bytes;
// out_partial: [splits][M][ldo] fp32.
void launch_gemm(const void *a_frag, bool two_planes, int M, int64_t K, const void *w, int64_t N,
                 float *out, int64_t ldo, const GemmPlan &p, hipStream_t s, const GemmOutput *directp) {
    GemmOutput direct;
    memset(&direct, 0, sizeof(direct));
    // direct outputs need complete sums and, for the gating, gate/up tile pairs inside one workgroup
    if (directp && gemm_direct_output_possible(p, directp->kind)) direct = *directp;
    const int m_tiles = (M + 15) / 16;
    if (p.mt_pass >= 6 && two_planes) {
        const bool d = direct.kind != GEMM_OUT_PARTIAL;
#define TALL(MT_) case MT_: \
            if (p.tall_tiles == 12) { \
                if (d) launch_gemm_t<MT_, 3, true, 8, 3, 2, true>(a_frag, M, K, w, N, out, ldo, p, s, direct); \
                else launch_gemm_t<MT_, 3, true, 8, 3, 2, false>(a_frag, M, K, w, N, out, ldo, p, s, direct); \
            } else if (d) launch_gemm_t<MT_, 4, true, 8, 3, 2, true>(a_frag, M, K, w, N, out, ldo, p, s, direct); \
            else launch_gemm_t<MT_, 4, true, 8, 3, 2, false>(a_frag, M, K, w, N, out, ldo, p, s, direct); \
            return;
#define TALL12(MT_) case MT_: \
            if (d) launch_gemm_t<MT_, 3, true, 8, 3, 2, true>(a_frag, M, K, w, N, out, ldo, p, s, direct); \
            else launch_gemm_t<MT_, 3, true, 8, 3, 2, false>(a_frag, M, K, w, N, out, ldo, p, s, direct); \
            return;
        switch (p.mt_pass) { TALL(6) TALL(7) TALL(8) TALL(9) TALL12(10) TALL12(11) }
#undef TALL12
#undef TALL
    }
    if (M <= 16) {
        if (two_planes) launch_gemm_v<1, true>(a_frag, M, K, w, N, out, ldo, p, s, direct);
        else launch_gemm_v<1, false>(a_frag, M, K, w, N, out, ldo, p, s, direct);
        return;
    }
    // Row counts other than the 65..80 of the 64-node tree (Sec. 4.3.4, Table 4: 16 or 21 tree rows for
    // the efficient tree, 105 rows with a mask group behind each of its nodes): one pass over
    // the weights with 2, 3 or 7 m-tiles, for the planner's two variants.  Beyond 7 m-tiles
    // the weight stream no longer bounds the kernel: tall passes (above), or passes of 5 m-tiles (grid z) where the
    // planner finds those as fast.
    const bool planner_variant = p.variant == 6 || p.variant == 8;
    if (two_planes && planner_variant && (m_tiles <= 3 || (m_tiles >= 6 && m_tiles <= 7 && p.variant == 8))) {
        if (m_tiles == 2) launch_gemm_k<2>(a_frag, M, K, w, N, out, ldo, p, s, direct);
        else if (m_tiles == 3) launch_gemm_k<3>(a_frag, M, K, w, N, out, ldo, p, s, direct);
        else launch_gemm_k<7>(a_frag, M, K, w, N, out, ldo, p, s, direct);
        return;
    }
    GemmPlan q = p;
    if (q.variant == 12) q.variant = 9;     // (12 exists as tall passes alone, which a forced variant does not plan)
    if (two_planes) launch_gemm_v<5, true>(a_frag, M, K, w, N, out, ldo, q, s, direct);
    else launch_gemm_v<5, false>(a_frag, M, K, w, N, out, ldo, q, s, direct);
}
bool gemm_direct_output_possible(const GemmPlan &p, int kind) {
    // rotated columns: the forms that plans with a single split and QKV-like widths take
    if (kind == GEMM_OUT_ROPE) return p.splits == 1 && (p.variant == 8 || p.variant == 9 || p.variant == 12);
    // the k-group shapes with whole gate/up tile pairs per wave, or (12, tall) per workgroup: its waves
    // hold four tiles, or three that are gated from LDS
    return p.splits == 1 && (p.variant == 5 || p.variant == 6 || p.variant >= 8);
}

size_t frag_bytes(int m_rows, int64_t k) {                     // two planes
    return (size_t)2 * ((k + 31) / 32) * ((m_rows + 15) / 16) * 1024;
}

void launch_to_fragments(const void *a_hi, const void *a_lo, int M, int64_t K, int64_t lda, void *dst,
                         hipStream_t s) {
    const int KS = (int)((K + 31) / 32), m_tiles = (M + 15) / 16;
    hipLaunchKernelGGL(to_fragments_kernel, dim3(KS, m_tiles, a_lo ? 2 : 1), dim3(64), 0, s, (const uint16_t *)a_hi,
                       (const uint16_t *)a_lo, M, (int)K, lda, KS, m_tiles, (uint4 *)dst);
}

void launch_reduce_partials(const float *partial, int splits, int M, int64_t N, int64_t ld,
                            float *out, const RowScale &rs, hipStream_t s) {
    dim3 grid((unsigned)((N + 255) / 256), (M + 3) / 4);
    hipLaunchKernelGGL(reduce_partials_kernel, grid, dim3(256), 0, s, partial, splits, M, N, ld, out, rs);
}

void launch_pack(const void *src, int64_t N, int64_t K, void *dst, int64_t tile0, int64_t tile_stride,
                 int64_t total_tiles, hipStream_t s) {
    const int64_t KS = ((K + 63) / 64) * 2;                 // k-steps incl. zero padding to a pair
    hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)((N / 16) * KS)), dim3(64), 0, s,
                       (const uint16_t *)src, N, K, KS, (uint4 *)dst, tile0, tile_stride, total_tiles);
}
