// Integer kernels of the streamlined generation-and-verification loop (Sec. 3.2, Algorithm 1):
// next-tree token assignment, the greedy acceptance walk, and the K/V commit of accepted rows.
#include "common.h"

// token[v] of the next pass: draft row at depth dv with sibling rank j carries the j-th
// ranked prediction of mask (dv-1+shift) of the chosen group; rows without a prediction
// are inactive (-1); mask rows carry their index in the group; row 0 is the last emitted token.
__global__ void build_tree_kernel(TemplateDev t, BuildSource src) {
    const int b = blockIdx.x;
    for (int v = threadIdx.x; v < t.rows; v += blockDim.x) src.token[(int64_t)b * t.rows + v] = tree_token(src, t, b, v);
}

// One wavefront per sequence.  At node v with greedy token a, the lanes test rows
// v+1.. in parallel for "tree child of v, active, token == a"; the lowest such row wins.
__global__ __launch_bounds__(64) void accept_kernel(TemplateDev t, const int32_t *__restrict__ token,
                                                    const int32_t *__restrict__ argmax,
                                                    int32_t *__restrict__ path, int32_t *__restrict__ n_acc,
                                                    int32_t *__restrict__ bonus, int32_t *__restrict__ emitted,
                                                    int32_t *__restrict__ next_group,
                                                    int32_t *__restrict__ next_shift) {
    const int b = blockIdx.x, lane = threadIdx.x;
    const int32_t *tok = token + (int64_t)b * t.rows;
    const int32_t *am = argmax + (int64_t)b * t.n_tree;
    const int stride = t.depth_max + 1;
    int32_t *p = path + (int64_t)b * stride, *e = emitted + (int64_t)b * stride;
    for (int i = lane; i < stride; i += 64) { p[i] = -1; e[i] = -1; }
    __syncthreads();
    int v = 0, len = 1;
    if (lane == 0) p[0] = 0;
    int a = am[0];
    while (len <= t.depth_max) {
        int found = -1;
        for (int base = v + 1; base < t.n_tree && found < 0; base += 64) {
            const int c = base + lane;
            const bool hit = c < t.n_tree && t.parent[c] == v && tok[c] >= 0 && tok[c] == a;
            const unsigned long long m = __ballot(hit);
            if (m) found = base + __ffsll((long long)m) - 1;
        }
        if (found < 0) break;
        if (lane == 0) { p[len] = found; e[len - 1] = a; }
        v = found;
        len++;
        a = am[v];
    }
    if (lane == 0) {
        e[len - 1] = a;
        n_acc[b] = len;
        bonus[b] = a;
        const int g = t.group_of_node[v];
        if (next_group) next_group[b] = g >= 0 ? g : t.group_of_node[0];
        if (next_shift) next_shift[b] = g >= 0 ? 0 : len - 1;
    }
}

// Where a pass' K/V rows are and where the cache rows go.
struct KvRows { uint4 *k_cache, *v_cache; const uint4 *k_tree, *v_tree; int batch, Hkv, smax, rows, row_u4; PageMap pm; };
// cache[l][b][h][slot][j] <- tree[l][b][h][row][j], 16 bytes
__device__ __forceinline__ void commit_granule(const KvRows &kv, int lh, int b, int row, int slot, int j) {
    const int l = lh / kv.Hkv, h = lh - l * kv.Hkv;
    const int64_t src = ((((int64_t)l * kv.batch + b) * kv.Hkv + h) * kv.rows + row) * kv.row_u4 + j;
    int64_t dst = ((((int64_t)l * kv.batch + b) * kv.Hkv + h) * kv.smax + slot) * kv.row_u4 + j;
    if (kv.pm.table) {                                  // page pools [L][n_pages][Hkv][page][hd]
        const int page = min(max(kv.pm.table[(int64_t)b * kv.pm.max_pages + (slot >> kv.pm.page_lg)], 0), kv.pm.n_pages - 1);
        dst = (((((int64_t)l * kv.pm.n_pages + page) * kv.Hkv + h) << kv.pm.page_lg) + (slot & ((1 << kv.pm.page_lg) - 1))) * kv.row_u4 + j;
    }
    const uint4 k = kv.k_tree[src], v = kv.v_tree[src];
    kv.k_cache[dst] = k;
    kv.v_cache[dst] = v;
}

#define COMMIT_THREADS 256
// cache[l][b][h][ctx_len + i][:] <- tree[l][b][h][path[i]][:], 16 bytes per lane.
// grid: (layer * kv-head, rows of the path, sequence).  ctx_len is advanced by a second tiny kernel so
// every workgroup of this one reads the old value.
__global__ __launch_bounds__(COMMIT_THREADS) void compact_kv_kernel(KvRows kv, const int32_t *__restrict__ path, int path_stride,
                                                                    const int32_t *__restrict__ n_acc, const int32_t *__restrict__ ctx_len) {
    const int per_wg = COMMIT_THREADS / kv.row_u4, b = blockIdx.z;
    const int i = blockIdx.y * per_wg + (int)threadIdx.x / kv.row_u4, j = threadIdx.x % kv.row_u4;
    const int n = n_acc[b], lc = ctx_len[b];
    if (i >= n || i >= path_stride || lc + n > kv.smax) return;
    const int src_row = path[(int64_t)b * path_stride + i];
    if (src_row < 0 || src_row >= kv.rows) return;
    commit_granule(kv, blockIdx.x, b, src_row, lc + i, j);
}
__global__ void advance_ctx_kernel(const int32_t *__restrict__ n_acc, int32_t *__restrict__ ctx_len,
                                   int batch, int smax) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < batch && ctx_len[b] + n_acc[b] <= smax) ctx_len[b] += n_acc[b];
}

// Acceptance and commit in one launch (bita_decode_step): every workgroup walks the tree for itself, from copies in
// LDS, and copies its share of the accepted rows; the first one of a sequence writes what the walk found and the
// new length.  Nobody reads what another workgroup writes: the length comes from ctx_start, which the
// selection filled.  Three launches (acceptance walk, copies, lengths) and the first one's memory round
// trip per level before.
__global__ __launch_bounds__(COMMIT_THREADS) void accept_commit_kernel(TemplateDev t, const int32_t *__restrict__ token, const int32_t *__restrict__ argmax,
                                                                       int32_t *__restrict__ path, int32_t *__restrict__ n_acc, int32_t *__restrict__ bonus,
                                                                       int32_t *__restrict__ emitted, int32_t *__restrict__ next_group,
                                                                       int32_t *__restrict__ next_shift, const int32_t *__restrict__ ctx_start,
                                                                       int32_t *__restrict__ ctx_len, int n_lh, KvRows kv) {
    __shared__ int32_t s_parent[BITA_MAX_ROWS], s_token[BITA_MAX_ROWS], s_argmax[BITA_MAX_ROWS], s_path[BITA_MAX_ROWS];
    __shared__ int32_t s_len;
    const int b = blockIdx.z, tid = threadIdx.x;
    const int lc = ctx_start[b];
    for (int i = tid; i < t.n_tree; i += COMMIT_THREADS) {
        s_parent[i] = t.parent[i];
        s_token[i] = token[(int64_t)b * t.rows + i];
        s_argmax[i] = argmax[(int64_t)b * t.n_tree + i];
    }
    __syncthreads();
    if (tid < 64) {
        // as accept_kernel: the lowest active child of v that carries v's greedy token
        int v = 0, len = 1;
        if (tid == 0) s_path[0] = 0;
        while (len <= t.depth_max) {
            const int a = s_argmax[v];
            int found = -1;
            for (int base = v + 1; base < t.n_tree && found < 0; base += 64) {
                const int c = base + tid;
                const bool hit = c < t.n_tree && s_parent[c] == v && s_token[c] >= 0 && s_token[c] == a;
                const unsigned long long m = __ballot(hit);
                if (m) found = base + __ffsll((long long)m) - 1;
            }
            if (found < 0) break;
            if (tid == 0) s_path[len] = found;
            v = found;
            len++;
        }
        if (tid == 0) s_len = len;
    }
    __syncthreads();
    const int n = s_len, last = s_path[n - 1];
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        const int stride = t.depth_max + 1;
        for (int i = tid; i < stride; i += COMMIT_THREADS) {
            path[(int64_t)b * stride + i] = i < n ? s_path[i] : -1;
            emitted[(int64_t)b * stride + i] = i < n ? s_argmax[s_path[i]] : -1;
        }
        if (tid == 0) {
            n_acc[b] = n;
            bonus[b] = s_argmax[last];
            const int g = t.group_of_node[last];
            if (next_group) next_group[b] = g >= 0 ? g : t.group_of_node[0];
            if (next_shift) next_shift[b] = g >= 0 ? 0 : n - 1;
            if (lc + n <= kv.smax) ctx_len[b] = lc + n;
        }
    }
    const int per_wg = COMMIT_THREADS / kv.row_u4;
    const int lh = blockIdx.x * per_wg + tid / kv.row_u4, j = tid % kv.row_u4;
    if (lh >= n_lh || lc + n > kv.smax) return;
    for (int i = blockIdx.y; i < n; i += gridDim.y) commit_granule(kv, lh, b, s_path[i], lc + i, j);
}

static int build_check(const bita_tree_template *t, const int32_t *d_root_token, const int32_t *d_cand, int32_t cand_rows, int32_t kmax,
                       int32_t batch, const int32_t *d_token) {
    if (!t || !d_root_token || !d_token || batch <= 0)
        return bita_set_error(BITA_ERR_INVALID_ARG, "bita_build_tree: null argument or batch <= 0");
    if (t->dev.n_tree > 1 && (!d_cand || cand_rows <= 0 || kmax <= 0 || kmax > BITA_MAX_TOPK))
        return bita_set_error(BITA_ERR_INVALID_ARG,
                              "bita_build_tree: candidates needed, cand_rows > 0, 1 <= kmax <= %d",
                              BITA_MAX_TOPK);
    return BITA_OK;
}

static void launch_build_tree(const TemplateDev &t, const BuildSource &src, int batch, hipStream_t s) {
    hipLaunchKernelGGL(build_tree_kernel, dim3(batch), dim3(64), 0, s, t, src);
}
extern "C" int bita_build_tree(const bita_tree_template *t, const int32_t *d_root_token,
                               const int32_t *d_cand, int32_t cand_rows, int32_t kmax,
                               const int32_t *d_group, const int32_t *d_shift, int32_t batch,
                               int32_t *d_token, void *stream) {
    if (int rc = build_check(t, d_root_token, d_cand, cand_rows, kmax, batch, d_token)) return rc;
    const BuildSource src = {d_root_token, d_cand, d_group, d_shift, cand_rows, kmax, d_token};
    launch_build_tree(t->dev, src, batch, (hipStream_t)stream);
    BITA_HIP_CHECK(hipGetLastError());
    return BITA_OK;
}

extern "C" int bita_accept(const bita_tree_template *t, const int32_t *d_token, const int32_t *d_argmax,
                           int32_t batch, int32_t *d_path, int32_t *d_n_acc, int32_t *d_bonus,
                           int32_t *d_emitted, int32_t *d_next_group, int32_t *d_next_shift,
                           void *stream) {
    if (!t || !d_token || !d_argmax || !d_path || !d_n_acc || !d_bonus || !d_emitted || batch <= 0)
        return bita_set_error(BITA_ERR_INVALID_ARG, "bita_accept: null argument or batch <= 0");
    hipLaunchKernelGGL(accept_kernel, dim3(batch), dim3(64), 0, (hipStream_t)stream, t->dev, d_token,
                       d_argmax, d_path, d_n_acc, d_bonus, d_emitted, d_next_group, d_next_shift);
    BITA_HIP_CHECK(hipGetLastError());
    return BITA_OK;
}

static KvRows kv_rows(const bita_config &cfg, const bita_kv *kv, const PageMap &pm, int batch) {
    return KvRows{(uint4 *)kv->k_cache, (uint4 *)kv->v_cache, (const uint4 *)kv->k_tree, (const uint4 *)kv->v_tree, batch,
                  cfg.n_kv_heads, kv->smax, kv->rows, cfg.head_dim * 2 / 16, pm};
}
int compact_kv_launch(const bita_config &cfg, const bita_kv *kv, const PageMap &pm, const int32_t *d_path,
                      int path_stride, const int32_t *d_n_acc, int32_t *d_ctx_len, int batch, hipStream_t s) {
    const KvRows rows = kv_rows(cfg, kv, pm, batch);
    const int per_wg = COMMIT_THREADS / rows.row_u4;
    hipLaunchKernelGGL(compact_kv_kernel, dim3(cfg.n_layers * cfg.n_kv_heads, (path_stride + per_wg - 1) / per_wg, batch), dim3(COMMIT_THREADS),
                       0, s, rows, d_path, path_stride, d_n_acc, d_ctx_len);
    hipLaunchKernelGGL(advance_ctx_kernel, dim3((batch + 63) / 64), dim3(64), 0, s, d_n_acc, d_ctx_len,
                       batch, kv->smax);
    return BITA_OK;
}

// The four calls of a step with three launches less: the tokens are worked out by the first layer's norm, and
// acceptance, copies and lengths are one kernel.  Each of the three cost 1.5 to 2 us whatever it did (four calls / one,
// in turn in one process, eager: two narrow layers, 12 rows 80.8 / 74.7 us, of which the host issues 73.6 / 59.4; two layers of 7B
// widths and the head, 68 rows 341 / 335, one row 245.6 / 240.3; a layer of 13B widths and the head, 25 rows 203.8 / 199.2, of 70B,
// 68 rows 458 / 453; replayed from a graph two narrow layers 83.9 / 80.2, 13B 211.3 / 206.5).
extern "C" int bita_decode_step(bita_model *m, const bita_kv *kv, const bita_tree_template *t, const int32_t *d_root_token,
                                const int32_t *d_cand, int32_t cand_rows, int32_t cand_kmax, const int32_t *d_group, const int32_t *d_shift,
                                int32_t *d_ctx_len, int32_t batch, void *d_workspace, size_t ws_bytes, int32_t kmax,
                                const bita_step_out *out, void *stream) {
    if (!out) return bita_set_error(BITA_ERR_INVALID_ARG, "bita_decode_step: null output descriptor");
    if (int rc = build_check(t, d_root_token, d_cand, cand_rows, cand_kmax, batch, out->d_token)) return rc;
    const bool outputs = out->d_argmax && out->d_path && out->d_n_acc && out->d_bonus && out->d_emitted;
    const int stride = t->dev.depth_max + 1;
    PageMap pm;
    const bool commits = m && kv && d_ctx_len && outputs && kv->batch == batch && stride <= kv->rows && kv->ctx_hint >= 0 &&
                         kv->ctx_hint <= kv->smax - stride && page_map_of(kv, kv->ctx_hint + stride, &pm, "bita_compact_kv") == BITA_OK;
    if (!commits) {
        // something of it will be refused: the calls before that one do their work, as they do one by one
        if (int rc = bita_build_tree(t, d_root_token, d_cand, cand_rows, cand_kmax, d_group, d_shift, batch, out->d_token, stream)) return rc;
        if (int rc = bita_verify_step(m, kv, t, out->d_token, d_ctx_len, batch, d_workspace, ws_bytes, kmax, out->d_argmax, out->d_topk_ids,
                                      out->d_topk_val, out->d_logits, stream)) return rc;
        if (int rc = bita_accept(t, out->d_token, out->d_argmax, batch, out->d_path, out->d_n_acc, out->d_bonus, out->d_emitted,
                                 out->d_next_group, out->d_next_shift, stream)) return rc;
        return bita_compact_kv(m, kv, out->d_path, stride, out->d_n_acc, d_ctx_len, batch, stream);
    }
    int32_t *ctx_start = nullptr;
    const BuildSource build = {d_root_token, d_cand, d_group, d_shift, cand_rows, cand_kmax, out->d_token};
    if (int rc = verify_pass(m, kv, t, out->d_token, d_ctx_len, batch, d_workspace, ws_bytes, kmax, out->d_argmax, out->d_topk_ids,
                             out->d_topk_val, out->d_logits, stream, nullptr, &build, &ctx_start)) {
        // refused ahead of its first kernel, which would have written the tokens: bita_build_tree had nothing against them
        launch_build_tree(t->dev, build, batch, (hipStream_t)stream);
        (void)hipGetLastError();
        return rc;
    }
    const KvRows rows = kv_rows(m->cfg, kv, pm, batch);
    const int n_lh = m->cfg.n_layers * m->cfg.n_kv_heads, per_wg = COMMIT_THREADS / rows.row_u4;
    hipLaunchKernelGGL(accept_commit_kernel, dim3((n_lh + per_wg - 1) / per_wg, stride < 4 ? stride : 4, batch), dim3(COMMIT_THREADS), 0,
                       (hipStream_t)stream, t->dev, out->d_token, out->d_argmax, out->d_path, out->d_n_acc, out->d_bonus, out->d_emitted,
                       out->d_next_group, out->d_next_shift, ctx_start, d_ctx_len, n_lh, rows);
    BITA_HIP_CHECK(hipGetLastError());
    return BITA_OK;
}
