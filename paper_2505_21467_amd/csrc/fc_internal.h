// Internal declarations shared by the host layer and the kernel files of libfreecache.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "freecache.h"

#define FC_VTILE 64  // rows per transposed V tile; Spad is a multiple of it

// Launch plan of the split-KV attention (host, pure function of the shape).
struct FcAttnPlan {
    int kind;            // 0 = k_attn_tile (fp32, head_dim 64, bf16 head_dim 128 over up to 96 keys); bf16 head_dim 128: 1 = k_attn_ranges,
                         // split-KV, 2 = k_attn_groups, all keys in one launch
    int splits;          // key ranges per (sequence, kv head); every one is non-empty
    int keys_per_split;  // multiple of 64 (kind 0: of 32)
    int row_tiles;       // 16-row (kind 1: 32-row) tiles of the flattened (head-in-group, a) rows per (b, kv head)
    int tiles_per_wg;    // row tiles handled by one workgroup
    int waves;           // waves per workgroup
    int v_parts;         // kind 2: parts the columns of V are cut into
};

// A cache handle: written by fc_cache_alloc only.
struct fc_cache {
    fc_config cfg;
    int32_t spad;        // max_seq rounded up to FC_VTILE
    size_t layer_elems;  // elements of one layer's K (== V) storage: B * Hkv * spad * Dh
    size_t esize;        // bytes per element
    void *k;             // device
    void *v;             // device
    bool owned;
    double inv_freq[64]; // rotary frequencies rope_base^(-2i/Dh), i < Dh/2, computed once on the host
    // Device scratch owned by the handle (nullptr when no GPU was present at creation): space for the
    // partial sums that the short-window projection hands from its first kernel to its second.
    void *scratch;
};

#define FC_SCRATCH_BYTES (32u * 1024u * 1024u)

// Tuning knobs: defaults (0 / -1 = the planner decides), overridden once from the environment
// variables of the same names at first use and afterwards only through fc_tuning_set.  Planners and
// launchers read this struct; nothing on a launch path calls getenv.
struct FcKnobs {
    int attn_r, attn_w;     // FC_ATTN_TILES=R,W      row tiles and waves per attention workgroup
    int attn_wgs;           // FC_ATTN_WGS=n          workgroups the split heuristic aims for
    int lin_wgs;            // FC_LIN_WGS=n           workgroups of the weight-streaming linear kernels
    int lin_no_rows;        // FC_LIN_NO_ROWS         slice-wise instead of whole-row weight streaming
    int lin_wide_shape;     // FC_LIN_WIDE_SHAPE=0..11 (4..8, 11: gated layer only) one tile shape for the tiled linear GEMM (-1 = planned)
    int lin_ksplit;         // FC_LIN_KSPLIT=n        parts of the hidden dimension
    int gemm_no_split;      // FC_GEMM_NO_SPLIT       never cut a GEMM into two launches
    int proj_gemm_shape;    // FC_PROJ_GEMM_SHAPE=0..11 one tile shape for the projection GEMM (-1 = planned)
    int proj_no_headsplit;  // FC_PROJ_NO_HEADSPLIT   short-window projection without the head-split kernels
    int version;            // changes with every fc_tuning_set
    int accept_wgs;         // FC_ACCEPT_WGS=n        workgroups of the acceptance scan
};
const FcKnobs &fc_knobs();

// Geometry handed to kernels by value.
struct FcGeom {
    int32_t B, d, Hq, Hkv, Dh, max_seq, spad, g;
    bool once;        // weights and rows of a pass exceed the memory-side cache (fc_read_once)
    float scale;      // softmax scale
    double log_base;  // ln(rope_base)
};

// Whether a pass over so many bytes finds nothing of them in the memory-side cache (256 MB) when it comes round again.  Streams
// that a single workgroup reads are then loaded with the non-temporal hint: they do not go through that cache on their way.
// Per launch, without and with, us: 36 head slots, hidden 3584, 8 / 32 rows 9.9 / 11.6 and 9.1 / 11.0; gated 3584 x 18944, 32 rows 48.5 and
// 44.1 (5.6 and 6.2 TB/s); 18944 x 3584 27.2 and 24.7; 136 MB of keys and values 52.5 and 47.1.  Where the bytes would have been
// in that cache the hint loses: the same projection over one or two layers 8.6 and 11.0; and it loses where several
// workgroups share a stream by way of L2 (attention with two groups of row tiles, 16800 keys 17.3 and 19.3; tiles of 48 rows,
// three to a run, 17.9 and 19.1).  Just above the line that cache would still hold a part: steps of 4 .. 8 layers, hidden 3584, as fast
// as without the hint x 0.96 .. 1.14 (mean 1.017, 50 of them) at 268 .. 320 MB, 0.97 .. 1.18 (1.025) to 420 MB, 0.99 .. 1.18 (1.047) above.
inline bool fc_read_once(double bytes_per_pass) { return bytes_per_pass > 256.0 * 1024 * 1024; }

// Bytes of a pass over all layers: projection weights, `keys` keys and values per sequence, and the layers' other weights (d_ff; 0: none of
// them).  What the cache has room for does not count: 36 head slots, hidden 3584, 32 rows, 1056 keys, room for 131072, one / two
// layers 15.8 / 16.4 us per layer with the hint that the room would ask for, 14.4 / 14.8 without.
inline double fc_pass_bytes(const fc_config &c, int32_t d_ff, int32_t keys)
{
    const double d = c.hidden, e = (double)c.n_q_heads * c.head_dim, kv = (double)c.n_kv_heads * c.head_dim;
    const double rest = d_ff > 0 ? d * e + 3.0 * d * d_ff : 0.0;
    return c.n_layers * ((e + 2.0 * kv) * d + 2.0 * c.batch * kv * keys + rest) * (c.dtype == FC_F32 ? 4.0 : 2.0);
}

// Element offset of K[b][j][row][i] inside one layer.
__host__ __device__ inline size_t fc_k_index(const FcGeom &G, int b, int j, int row, int i)
{
    return (((size_t)b * G.Hkv + j) * G.spad + row) * G.Dh + i;
}
// Element offset of V[b][j][row][i] inside one layer (64-row tiles, key index fastest).
__host__ __device__ inline size_t fc_v_index(const FcGeom &G, int b, int j, int row, int i)
{
    return ((size_t)b * G.Hkv + j) * G.spad * G.Dh + (size_t)(row / FC_VTILE) * (FC_VTILE * G.Dh) +
           (size_t)i * FC_VTILE + (row % FC_VTILE);
}

FcAttnPlan fc_plan_attention(const fc_config &cfg, int A, int kv_len, size_t cap = SIZE_MAX);  // cap: bytes of partial results
size_t fc_plan_workspace(const fc_config &cfg, const FcAttnPlan &p);

// Kernel launchers (defined in the .hip kernel files).  All return hipGetLastError() after launch.
hipError_t fc_launch_copy_rows(const FcGeom &G, int dtype, void *k_layer, void *v_layer, void *k_rows,
                               void *v_rows, int start, int rows, bool to_cache, hipStream_t s);
hipError_t fc_launch_project_tile(const FcGeom &G, const double *inv_freq, int dtype, const void *x, const void *w,
                                  const void *bias, const int32_t *pos, int win_start, int A,
                                  void *q_out, void *k_layer, void *v_layer, hipStream_t s);
hipError_t fc_launch_attention_tile(const FcGeom &G, const FcAttnPlan &p, int dtype, const void *q, const void *k_layer,
                                    const void *v_layer, const int32_t *pos, int A, int kv_len,
                                    void *out, void *workspace, hipStream_t s);
bool fc_project_mfma_supported(const fc_config &cfg);
bool fc_project_prefers_gemm(const fc_config &cfg, int M, bool scratch);
bool fc_project_prefers_tile(const fc_config &cfg, int M);
hipError_t fc_launch_project_mfma(const FcGeom &G, const void *x, const void *w, const void *bias,
                                  const int32_t *pos, int win_start, int A, void *q_out,
                                  void *k_layer, void *v_layer, void *scratch, hipStream_t s);
bool fc_project_gemm_supported(const fc_config &cfg, int M);
double fc_project_gemm_us(int slots, int M, int K);
hipError_t fc_launch_project_gemm(const FcGeom &G, const void *x, const void *w, const void *bias,
                                  const int32_t *pos, int win_start, int A, void *q_out, void *k_layer,
                                  void *v_layer, hipStream_t s);
hipError_t fc_launch_attention_mfma(const FcGeom &G, const FcAttnPlan &p, const void *q,
                                    const void *k_layer, const void *v_layer, const int32_t *pos,
                                    int A, int kv_len, void *out, void *workspace, hipStream_t s);

// Rest of the layer on the window rows: RMS normalisation and the linear layers around attention.
enum { FC_LIN_RESIDUAL = 0, FC_LIN_GATE_UP = 1, FC_LIN_VOCAB = 2 };
// Vocabulary mode: per (part of the vocabulary, row) the largest logit, its index and the sum of
// exp(logit - largest) over the part, in groups of eight rows, [ceil(M / 8)][parts][8]: the merge reads a group's parts
// in one piece.
struct FcArgmax {
    float mx;
    int32_t arg;
    float sm;
};
struct FcArgmaxPart {
    FcArgmax *p;
    int parts;
    __host__ __device__ FcArgmax &at(int part, int m) const { return p[((size_t)(m >> 3) * parts + part) * 8 + (m & 7)]; }
};
// (largest, index, sum) of a union of two parts; equal maxima keep the smaller index.
__host__ __device__ inline void fc_argmax_merge(float &mx, int &arg, float &sm, float mx2, int arg2, float sm2)
{
    if (mx2 > mx || (mx2 == mx && arg2 < arg)) {
        const float t = mx;
        mx = mx2;
        mx2 = t;
        const float u = sm;
        sm = sm2;
        sm2 = u;
        arg = arg2;
    }
    // now mx >= mx2; a part that is still empty has mx2 = -inf and sm2 = 0
    if (sm2 != 0.f) sm += sm2 * expf(mx2 - mx);
}
hipError_t fc_launch_rmsnorm(int dtype, const void *x, const void *weight, float eps, int rows, int d,
                             void *out, hipStream_t s);
// Linear layer for any dtype and shape.  FC_LIN_RESIDUAL: out = aux + x w^T (aux = residual
// or nullptr); FC_LIN_GATE_UP: out = silu(x w^T) * (x aux^T) (aux = up matrix).
hipError_t fc_launch_linear_tile(int dtype, int mode, const void *x, const void *w, const void *aux,
                                    int M, int K, int N, void *out, hipStream_t s);
// Launch plan of the weight-streaming linear kernels (host, pure function of the shape).
struct FcSkinnyPlan {
    int kind;    // 0 = plain kernel (no workspace), 1 = streaming kernels, 2 = whole-row kernel (T = half items, G)
    int mt;      // 16-row tiles per pass (1 or 2)
    int chunks;  // passes of up to 32 rows
    int slabs;   // 128-row slabs of the weight matrix (64 gate + 64 up rows in gated mode)
    int S;       // hidden-dimension slices per slab
    int T;       // work items = slabs * S
    int G;       // workgroups
    int maxseg;  // upper bound of the workgroups that meet one slab
    size_t reserve;  // kind 2: workspace asked of the caller and not used
};
// Layers of up to 8192 outputs and 256 rows, one launch, no workspace: whether the kernel can, and the launch.
bool fc_linear_lines_cover(int dtype, int mode, int M, int K, int N);
// The same for a small vocabulary: parts of the arg-max it writes, `parts` at most (0: not for it), and the launch.
int fc_lmhead_lines_parts(int dtype, int M, int K, int V, int parts);
hipError_t fc_launch_lmhead_lines(const void *x, const void *w, int M, int K, int V, const FcArgmaxPart &am, hipStream_t s);
// And for a large one.
int fc_lmhead_runs_parts(int dtype, int M, int K, int V, int parts);
hipError_t fc_launch_lmhead_runs(const void *x, const void *w, int M, int K, int V, const FcArgmaxPart &am, hipStream_t s);
hipError_t fc_launch_linear_lines(int mode, const void *x, const void *w, const void *w2, const void *res, int M, int K, int N,
                                  void *out, bool once, hipStream_t s);
FcSkinnyPlan fc_plan_skinny(int dtype, int mode, int M, int K, int N);
size_t fc_skinny_workspace(const FcSkinnyPlan &p);
hipError_t fc_launch_linear_skinny(const FcSkinnyPlan &pl, int mode, const void *x, const void *w,
                                   const void *w2, const void *res, int M, int K, int N, void *out,
                                   void *workspace, hipStream_t s, const FcArgmaxPart *am = nullptr);
// Unmasking step: vocabulary projection for any dtype and shape, merge of the vocabulary parts, and
// the confidence-ranked fill.
hipError_t fc_launch_lmhead_tile(int dtype, const void *x, const void *w, int M, int K, int V,
                                 const FcArgmaxPart &am, hipStream_t s);
#define FC_LMHEAD_TILE_PART 32  // vocabulary entries per part of that kernel
hipError_t fc_launch_lmhead_reduce(const FcArgmaxPart &am, int M, int32_t *tok, float *conf,
                                   hipStream_t s);
#define FC_UNMASK_MAX_ROWS 8192
hipError_t fc_launch_unmask_select(const int32_t *tok, const float *conf, const int32_t *pos, int win_start,
                                   int B, int A, int n_unmask, int mask_id, int32_t *tokens, int L,
                                   int32_t *pos_next, int32_t *count_next, hipStream_t s);
// Tiled-GEMM plan of the same linear layers on more than 32 rows.
struct FcWidePlan {
    int kind;    // 0 = not covered, 1 = tiled GEMM
    int shape;   // tile shape where ksplit > 1 or a tuning knob forces one (numbered in fc_proj_gemm.hip)
    int ksplit;  // parts of the hidden dimension (1 = epilogue inside the GEMM, no workspace)
    size_t required;  // bytes of workspace a call must bring (the plan keeps within `cap` bytes from there on)
};
FcWidePlan fc_plan_wide(int dtype, int mode, int M, int K, int N, size_t cap = SIZE_MAX);
size_t fc_wide_workspace(const FcWidePlan &p, int M, int N);
hipError_t fc_launch_linear_wide(const FcWidePlan &pl, int mode, const void *x, const void *w, const void *w2,
                                 const void *res, int M, int K, int N, void *out, void *workspace, bool once, hipStream_t s,
                                 const FcArgmaxPart *am = nullptr);
hipError_t fc_launch_gather_rows(const void *table, int64_t R, int row_bytes, const int32_t *idx, int64_t n, void *out,
                                 hipStream_t s);
#define FC_ACCEPT_MAX_TOPK 8
size_t fc_accept_workspace(int B, int A, int V);
hipError_t fc_launch_guided_accept(const float *dlm, const float *ar, const int32_t *pos, int win_start, int B, int A,
                                   int V, int topk, float tau, int mask_id, int32_t *tokens, int L, int32_t *n_accept,
                                   int32_t *pos_next, int32_t *count_next, void *workspace, hipStream_t s);
hipError_t fc_launch_kv_similarity(const FcGeom &G, int dtype, const void *k_layer, const void *v_layer,
                                   const void *k_prev, const void *v_prev, int start, int rows, float *sim_k,
                                   float *sim_v, hipStream_t s);
