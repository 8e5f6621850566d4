// Internal declarations shared by the HIP sources of libbita (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <map>
#include <mutex>
#include <vector>
#include "../../include/bita.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

#define BITA_WAVE 64

// bf16 <-> fp32 on raw bits (round to nearest even; inputs are finite)
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
// x ~= hi + lo with both parts bf16: the pair carries ~16 mantissa bits of x
__device__ __forceinline__ void split_bf16(float x, uint16_t &hi, uint16_t &lo) {
    hi = f32_to_bf16(x);
    lo = f32_to_bf16(x - bf16_to_f32(hi));
}
// Position (in bf16 elements) of A[m][k] of plane p inside an activation slab kept in MFMA
// A-operand fragment order: 1 KiB per (plane, k-step of 32, m-tile of 16), lane l of a
// fragment holding A[16mt + l%16][32ks + 8(l/16) .. +8].
// A last m-tile that is at most half full keeps BOTH planes of its rows in the high plane's
// fragment: the low plane of row r sits at row r + off (off = 4 for up to 4 rows, 8 for up to 8).
// One fragment and one matrix instruction per weight tile then serve both planes of those rows;
// the two partial products come out as different accumulator rows and are added once, after the
// k loop.  frag_pack_offset gives off (0 = not packed) from the slab's row count alone, so
// producers and the GEMM agree; it applies to the slabs whose GEMM always takes every m-tile in
// one pass with as many accumulator tiles: one m-tile (M <= 8: the one-row pass) or five
// (65..72 rows: the 64-node tree with its mask rows).
__host__ __device__ __forceinline__ int frag_pack_offset(int M) {
    const int m_tiles = (M + 15) >> 4, v = M - 16 * (m_tiles - 1);
    if ((m_tiles != 1 && m_tiles != 5) || v > 8) return 0;
    return v <= 4 ? 4 : 8;
}
__device__ __forceinline__ int64_t frag_index(int plane, int m, int k, int n_ksteps, int m_tiles, int pack_off) {
    if (pack_off && plane == 1 && (m >> 4) == m_tiles - 1) {
        plane = 0;
        m += pack_off;
    }
    const int ks = k >> 5, kq = (k >> 3) & 3, e = k & 7;
    return ((((int64_t)plane * n_ksteps + ks) * m_tiles + (m >> 4)) * 64 + kq * 16 + (m & 15)) * 8 + e;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}

// 16-byte store that is written through the XCD's L2 instead of staying there dirty until the end of
// the kernel: what a kernel leaves dirty is written back between it and the next one, when nothing
// else runs (256 workgroups that store 9 / 17 MB and end: 3.1 -> 2.5 / 4.6 -> 3.6 us).  For row pieces of
// 128 bytes and more; the 192-byte ones of three-tile waves, one and a half cache lines, still gain (whole
// calls, plain / through: 272 x 12288 x 4096 66.7 / 65.8 us, 140 x 6144 x 16384 77.4 / 76.6, 170 x 12288 x 4096 51.1 / 50.2).
// (A buffer store with the scope bit, so that the compiler knows the instruction: as inline assembly
// it does not keep the store's data registers untouched for the wait state a 16-byte store needs.)
// Its offset has 32 bits: the 16 rows that one instruction may span have at most this many floats each.
#define GEMM_THROUGH_MAX_LD (1 << 26)
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t through_rsrc(void *base, uint32_t bytes) {      // base: wave-uniform
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00027000);
}
__device__ __forceinline__ void store_through(__amdgpu_buffer_rsrc_t r, uint32_t byte_offset, float4 v) {
    const f32x4 q = {v.x, v.y, v.z, v.w};
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, q), r, byte_offset, 0, /* sc1 */ 16);
}

// ---- host-side error plumbing -------------------------------------------------
int  bita_set_error(int code, const char *fmt, ...);
#define BITA_HIP_CHECK(expr)                                                                 \
    do {                                                                                     \
        hipError_t _e = (expr);                                                              \
        if (_e != hipSuccess)                                                                \
            return bita_set_error(BITA_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(_e)); \
    } while (0)

// ---- device mirror of a pass layout ---------------------------------------------
struct TemplateDev {
    int32_t rows, n_tree, n_mask, n_groups, depth_max, kmax, words;
    const int32_t *parent;        // [R]
    const int32_t *depth;         // [R]
    const int32_t *rank;          // [R] sibling rank of a tree row
    const int32_t *mask_index;    // [R] index inside its group, -1 for tree rows
    const int32_t *group_of_node; // [T] group attached to a tree row or -1
    const int32_t *mask_rows;     // [G*n] row of mask i of group g
    const uint8_t *is_mask;       // [R]
    const uint64_t *anc;          // [R][words] ancestor-or-self bitsets
};
struct bita_tree_template {
    TemplateDev dev;
    void *blob;                   // one device allocation backing all arrays
};

// ---- the model handle: borrowed weight pointers plus the rotary table it owns --------
struct bita_model {
    bita_config cfg;
    const void *tok_emb, *mask_emb, *final_norm, *lm_head;
    std::vector<const void *> attn_norm, ffn_norm, wqkv, wo, w_gate_up, w_down, prompt_k, prompt_v;
    float *rope_cos = nullptr, *rope_sin = nullptr;     // [max_pos][hd/2]
    // chain templates of the prefill chunks by row count, created once and kept until the
    // handle is destroyed (the enqueued kernels read their device arrays)
    mutable std::mutex chain_mutex;
    std::map<int, bita_tree_template *> chains;
    mutable std::map<std::pair<int, int>, size_t> chunk_bytes;   // workspace of a prefill's passes by (batch, chunk rows)
};

// ---- kernel launchers (each only enqueues) --------------------------------------
#define RMS_MAX_CHUNKS 16          // 1024 columns each: d_model <= 16384
struct RowScale { const float *ssq; int chunks; float inv_d, eps; };   // ssq == nullptr: no scaling
// second half of RMSNorm: rsqrt(mean(x^2) + eps) of row m from the per-chunk sums of squares.
// In two steps, so that a kernel can request the sums early and look at them late: all 16 slots of
// the row are fetched at once (independent loads, one round trip) and summed in chunk order;
// slots at or beyond rs.chunks are never written and are left out.
struct RowScaleSums { float4 q0, q1, q2, q3; };
__device__ __forceinline__ RowScaleSums row_scale_fetch(const RowScale &rs, int m) {
    RowScaleSums r;
    r.q0 = r.q1 = r.q2 = r.q3 = make_float4(0.f, 0.f, 0.f, 0.f);
    if (!rs.ssq) return r;
    const float4 *p = reinterpret_cast<const float4 *>(rs.ssq + (int64_t)m * RMS_MAX_CHUNKS);
    r.q0 = p[0]; r.q1 = p[1]; r.q2 = p[2]; r.q3 = p[3];
    return r;
}
__device__ __forceinline__ float row_scale_finish(const RowScale &rs, const RowScaleSums &r) {
    if (!rs.ssq) return 1.0f;
    const float v[RMS_MAX_CHUNKS] = {r.q0.x, r.q0.y, r.q0.z, r.q0.w, r.q1.x, r.q1.y, r.q1.z, r.q1.w,
                                     r.q2.x, r.q2.y, r.q2.z, r.q2.w, r.q3.x, r.q3.y, r.q3.z, r.q3.w};
    float tot = 0.f;
#pragma unroll
    for (int ch = 0; ch < RMS_MAX_CHUNKS; ch++) tot += ch < rs.chunks ? v[ch] : 0.f;
    return 1.0f / sqrtf(tot * rs.inv_d + rs.eps);
}
__device__ __forceinline__ float row_scale(const RowScale &rs, int m) { return row_scale_finish(rs, row_scale_fetch(rs, m)); }
// mt_pass: m-tiles per row pass of a tall launch (6..11), 0 = the variant's own row handling;
// tall_tiles: weight tiles per workgroup of a tall launch (16 or 12)
struct GemmPlan { int splits, ksteps_per_split, variant, mt_pass, tall_tiles; };
// What a GEMM launch with a single split (complete sums in its accumulators) may do instead of
// storing fp32 partials: apply the deferred RMSNorm row factor and store the result, or apply it
// and the SwiGLU gating to its tile-interleaved gate/up columns and store the next GEMM's
// activation slab (two bf16 planes, fragment order).
// GEMM_OUT_ROPE: apply it to the QKV columns, rotate q and k by the row's position and store both planes of q, k and v where
// qkv_rope_kernel would (the same arithmetic, bit for bit).
enum { GEMM_OUT_PARTIAL = 0, GEMM_OUT_SCALED = 1, GEMM_OUT_SILU = 2, GEMM_OUT_ROPE = 3 };
struct RopeOutput {
    const int32_t *ctx_len, *depth;                 // [B], [R]
    const float *cos, *sin;                         // [max_pos][hd/2]
    uint16_t *q, *q_lo, *k, *v, *k_lo, *v_lo;       // [B][R][Hq][hd], [B][Hkv][R][hd]
    int R, Hq, Hkv, hd, max_pos;
};
struct GemmOutput { int kind; RowScale rs; uint16_t *act_frag; int d_ffn; RopeOutput rope; };
// one rotation pair, rounded the same wherever it is done
__device__ __forceinline__ void rope_pair(float &x, float &y, float c, float s) {
    const float nx = __builtin_fmaf(x, c, -(y * s)), ny = __builtin_fmaf(y, c, x * s);
    x = nx;
    y = ny;
}
bool gemm_direct_output_possible(const GemmPlan &p, int kind);
void gemm_force_plan(int variant, int splits);   // tuning aid: < 0 restores the heuristic
bool gemm_plan_forced();
// Device bytes of the static scratch behind bita_gemm_noalloc.  The planner knows it because a shape's
// plan, and with it the result's last bits, is the same for every caller.
#define BITA_NOALLOC_SCRATCH_BYTES (32u << 20)
// planes: of the activations (every launch of a step has two); a plan holds for that number only
GemmPlan gemm_plan(int m_rows, int64_t n_rows, int64_t k, int planes = 2);
size_t frag_bytes(int m_rows, int64_t k);        // bytes of a two-plane activation slab
// a_frag: activations in fragment order (see frag_index); out_partial: [splits][m_rows][ldo] fp32
void launch_gemm(const void *a_frag, bool two_planes, int m_rows, int64_t k, const void *w_packed,
                 int64_t n_rows, float *out_partial, int64_t ldo, const GemmPlan &p, hipStream_t s,
                 const GemmOutput *direct = nullptr);
void launch_to_fragments(const void *a_hi, const void *a_lo, int m_rows, int64_t k, int64_t lda, void *dst,
                         hipStream_t s);
void launch_reduce_partials(const float *partial, int splits, int m_rows, int64_t n, int64_t ld,
                            float *out, const RowScale &rs, hipStream_t s);
void launch_pack(const void *src, int64_t n_rows, int64_t k, void *dst, int64_t tile0,
                 int64_t tile_stride, int64_t total_tiles, hipStream_t s);

// Where the first layer's norm takes its rows from (see rmsnorm_prep_kernel).
// A whole step (bita_decode_step) has the first layer's norm work out the rows' tokens itself, from what
// bita_build_tree takes (root == nullptr: they are in `token` already).
struct BuildSource { const int32_t *root, *cand, *group, *shift; int cand_rows, kmax; int32_t *token; };
struct EmbedSource { const int32_t *token; const uint8_t *is_mask; const int32_t *mask_index; const uint16_t *tok_emb, *mask_emb; int rows, vocab; };
// x = embeddings of the pass' rows, and the first norm's slab and sums of squares
void launch_embed_prep(const int32_t *token, const BuildSource &build, const TemplateDev &t, int batch, const void *tok_emb, const void *mask_emb, int d,
                       int vocab, const void *gain, float *x, void *h_frag, float *ssq, hipStream_t s);
// x += sum of partials (optional), then h = rmsnorm(x) * gain as bf16 with row stride ldh
// RMSNorm is split: the prep kernel writes x*gain (two planes, fragment order) and per-chunk
// sums of squares ssq[m_rows][RMS_MAX_CHUNKS]; the row factor rsqrt(sum(ssq)/d + eps) commutes
// with the matrix product and is applied by the kernel that consumes the GEMM output.
void launch_rmsnorm_prep(float *x, const float *partial, int splits, int m_rows, int d,
                         const void *gain, void *h_frag, float *ssq, hipStream_t s);
void launch_qkv_rope(const float *partial, int splits, int batch, const TemplateDev &t,
                     int n_heads, int n_kv_heads, int hd, const int32_t *ctx_len,
                     const float *rope_cos, const float *rope_sin, int max_pos,
                     void *q, void *q_lo, void *k_tree, void *v_tree, void *k_tree_lo, void *v_tree_lo,
                     const RowScale &rs, hipStream_t s);
void launch_silu_mul(const float *partial, int splits, int m_rows, int d_ffn, void *act_frag,
                     const RowScale &rs, hipStream_t s);
// ctx_start: where a step that goes on to change the lengths has them copied to (nullptr: nowhere)
void launch_select(const float *logits, int batch, const TemplateDev &t, int vocab, int kmax,
                   int32_t *argmax, int32_t *topk_ids, float *topk_val, hipStream_t s,
                   const int32_t *ctx_len = nullptr, int32_t *ctx_start = nullptr);

// Where the cache rows live: contiguous per sequence (table == nullptr) or in pages of
// 1 << page_lg key slots, page ids per sequence in table[b][0 .. max_pages).  tbl_cap: table
// entries per sequence a launch makes room for (covers the call's ctx_hint).
#define ATT_PAGE_TABLE_MAX 4096
struct PageMap { const int32_t *table; int page_lg, n_pages, max_pages, tbl_cap; };
struct AttnPlan { int splits, chunks; size_t part_o_bytes, part_ml_bytes; };
AttnPlan attn_plan(int batch, int rows, int n_heads, int hd, int ctx_hint, int n_prompt);
// tiles of 16 queries per workgroup, log2 of the heads that share one, waves per workgroup; one_row: of each sequence.
// share: how many neighbouring workgroups of a head are launched as one of share_waves waves that share chunks (1: none, and
// launched_workgroups = workgroups, share_waves = waves).  ranked: the longest sequences' workgroups start first
struct AttnTiles { int tiles, lg_ht, waves, share, share_waves; bool ranked; int64_t workgroups, launched_workgroups; };
AttnTiles attn_tiles(int batch, int rows, int n_heads, int n_kv_heads, int hd, const AttnPlan &p, int table_entries, bool one_row);
// k_tree_lo / v_tree_lo: low bf16 plane of the pass rows' K/V (nullable); out_lo: low plane of
// the row-major output (nullable; unused when the output is written as fragments)
void launch_tree_attention(const TemplateDev &t, const void *q, const void *q_lo, const void *k_cache,
                           const void *v_cache, const void *k_tree, const void *v_tree,
                           const void *k_tree_lo, const void *v_tree_lo,
                           const void *prompt_k, const void *prompt_v, const int32_t *ctx_len,
                           const int32_t *token /* [B][R] or nullptr: rows with a negative token are absent */,
                           int batch, int n_heads, int n_kv_heads, int hd, int n_prompt, int smax,
                           const AttnPlan &p, float *part_o, float *part_ml, void *out, void *out_lo,
                           bool out_as_fragments, const PageMap &pm, hipStream_t s,
                           const int32_t *only_row = nullptr /* [B]: only this row of each sequence is asked for (its row tile is computed) */);

// A prefill chunk needs from its pass the rows' K/V and, where a sequence may end in the chunk, the
// greedy token after one row per sequence (sel_row [B], row inside the chunk): the last layer then
// goes on with those rows alone behind the K/V projection.  sel_row == nullptr: K/V only.  ws: a
// workspace of bita_workspace_bytes(m, batch, 1).
struct PassTail { const int32_t *sel_row; void *ws; };
// bita_verify_step, with an optional tail (argmax is then [B], one per sequence; no top-k, no logits), or working
// the rows' tokens out itself (build; the lengths at the start of the step are then found at *ctx_start)
int verify_pass(bita_model *m, const bita_kv *kv, const bita_tree_template *t, const int32_t *d_token,
                const int32_t *d_ctx_len, int32_t batch, void *d_workspace, size_t ws_bytes, int32_t kmax,
                int32_t *d_argmax, int32_t *d_topk_ids, float *d_topk_val, float *d_logits, void *stream,
                const PassTail *tail, const BuildSource *build = nullptr, int32_t **ctx_start = nullptr);
int page_map_of(const bita_kv *kv, int ctx_upper, PageMap *pm, const char *who);
// token of row v of sequence b (bita_build_tree)
__device__ __forceinline__ int tree_token(const BuildSource &s, const TemplateDev &t, int b, int v) {
    if (v == 0) return s.root[b];
    if (v >= t.n_tree) return t.mask_index[v];
    const int g = s.group ? s.group[b] : 0, lvl = t.depth[v] - 1 + (s.shift ? s.shift[b] : 0), rank = t.rank[v];
    const int row = g * t.n_mask + lvl;
    // g < 0: the previous pass had no mask group to offer (accept writes -1 then): no drafts
    return (g >= 0 && lvl >= 0 && lvl < t.n_mask && row < s.cand_rows && rank < s.kmax)
               ? s.cand[((int64_t)b * s.cand_rows + row) * s.kmax + rank] : -1;
}
// row sel_row[b] of each sequence of `rows`: its columns of a two-plane slab (fragment order) and of
// the residual stream, into a slab and a stream of `batch` rows
void launch_gather_rows(const int32_t *sel_row, int batch, int rows, const void *a_frag, int k, const float *x, int d,
                        void *a_out, float *x_out, hipStream_t s);
