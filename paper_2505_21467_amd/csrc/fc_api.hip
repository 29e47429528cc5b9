// C-ABI host layer of libfreecache: argument validation, launch planning, kernel enqueue.
// Every check happens before the first HIP call of an entry point.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <new>

#include "fc_internal.h"

namespace {

thread_local char g_err[512] = "";

fc_status fail(fc_status st, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return st;
}

size_t esize_of(int dtype) { return dtype == FC_F32 ? 4 : 2; }

// Validate a configuration; on failure fills the error text and returns the status.
fc_status check_config(const fc_config *c)
{
    if (!c) return fail(FC_ERR_INVALID_ARG, "config is NULL");
    if (c->dtype != FC_F32 && c->dtype != FC_BF16)
        return fail(FC_ERR_INVALID_ARG, "dtype %d is neither FC_F32 nor FC_BF16", c->dtype);
    if (c->n_layers < 1 || c->batch < 1 || c->hidden < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1 ||
        c->head_dim < 1 || c->max_seq < 1)
        return fail(FC_ERR_INVALID_ARG, "config sizes must be positive");
    if (!(c->rope_base > 1.0f) || !isfinite(c->rope_base))
        return fail(FC_ERR_INVALID_ARG, "rope_base must be finite and > 1");
    if (c->softmax_scale < 0.0f || !isfinite(c->softmax_scale))
        return fail(FC_ERR_INVALID_ARG, "softmax_scale must be finite and >= 0");
    if (c->n_q_heads % c->n_kv_heads != 0)
        return fail(FC_ERR_UNSUPPORTED, "n_q_heads %d is not a multiple of n_kv_heads %d", c->n_q_heads,
                    c->n_kv_heads);
    if (c->head_dim != 64 && c->head_dim != 128)
        return fail(FC_ERR_UNSUPPORTED, "head_dim %d not supported (64 or 128)", c->head_dim);
    if (c->hidden % 8 != 0) return fail(FC_ERR_UNSUPPORTED, "hidden %d is not a multiple of 8", c->hidden);
    if (c->max_seq > (1 << 24)) return fail(FC_ERR_UNSUPPORTED, "max_seq %d exceeds 2^24", c->max_seq);
    if (c->batch > 65535 || c->n_q_heads > 65535)
        return fail(FC_ERR_UNSUPPORTED, "batch and n_q_heads are limited to 65535");
    return FC_OK;
}

int spad_of(const fc_config &c) { return (c.max_seq + FC_VTILE - 1) / FC_VTILE * FC_VTILE; }

// keys: of each layer that the pass around the call reads, as far as the call can know (`once` is a hint)
FcGeom geom_of(const fc_cache *cache, int32_t d_ff = 0, int32_t keys = 0)
{
    const fc_config &c = cache->cfg;
    FcGeom G;
    G.B = c.batch;
    G.d = c.hidden;
    G.Hq = c.n_q_heads;
    G.Hkv = c.n_kv_heads;
    G.Dh = c.head_dim;
    G.max_seq = c.max_seq;
    G.spad = cache->spad;
    G.g = c.n_q_heads / c.n_kv_heads;
    G.once = fc_read_once(fc_pass_bytes(c, d_ff, keys));
    G.scale = c.softmax_scale > 0.f ? c.softmax_scale : (float)(1.0 / sqrt((double)c.head_dim));
    G.log_base = log((double)c.rope_base);
    return G;
}

void *layer_ptr(const fc_cache *c, void *base, int layer)
{
    return (char *)base + (size_t)layer * c->layer_elems * c->esize;
}

fc_status check_cache_layer(const fc_cache *cache, int32_t layer)
{
    if (!cache) return fail(FC_ERR_INVALID_ARG, "cache is NULL");
    if (layer < 0 || layer >= cache->cfg.n_layers)
        return fail(FC_ERR_BOUNDS, "layer %d outside [0, %d)", layer, cache->cfg.n_layers);
    return FC_OK;
}

fc_status hip_fail(hipError_t e, const char *what)
{
    return fail(FC_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// Launch planning (pure host functions).

// Tuning knobs (see FcKnobs): read from the environment once, then changed only by fc_tuning_set.
namespace {

void knobs_defaults(FcKnobs &k)
{
    memset(&k, 0, sizeof k);
    k.lin_wide_shape = -1;
    k.proj_gemm_shape = -1;
}

// Apply one "NAME", "value" pair (value NULL = back to the default).  False for an unknown name.
bool knob_apply(FcKnobs &k, const char *name, const char *value)
{
    FcKnobs d;
    knobs_defaults(d);
    const int v = value ? atoi(value) : 0;
    if (!strcmp(name, "FC_ATTN_TILES")) {
        k.attn_r = k.attn_w = 0;
        if (value) sscanf(value, "%d,%d", &k.attn_r, &k.attn_w);
    } else if (!strcmp(name, "FC_ATTN_WGS")) k.attn_wgs = value ? v : d.attn_wgs;
    else if (!strcmp(name, "FC_LIN_WGS")) k.lin_wgs = value ? v : d.lin_wgs;
    else if (!strcmp(name, "FC_LIN_NO_ROWS")) k.lin_no_rows = value ? 1 : 0;
    else if (!strcmp(name, "FC_LIN_WIDE_SHAPE")) k.lin_wide_shape = value ? v : d.lin_wide_shape;
    else if (!strcmp(name, "FC_LIN_KSPLIT")) k.lin_ksplit = value ? v : d.lin_ksplit;
    else if (!strcmp(name, "FC_GEMM_NO_SPLIT")) k.gemm_no_split = value ? 1 : 0;
    else if (!strcmp(name, "FC_PROJ_GEMM_SHAPE")) k.proj_gemm_shape = value ? v : d.proj_gemm_shape;
    else if (!strcmp(name, "FC_PROJ_NO_HEADSPLIT")) k.proj_no_headsplit = value ? 1 : 0;
    else if (!strcmp(name, "FC_ACCEPT_WGS")) k.accept_wgs = value ? v : d.accept_wgs;
    else return false;
    return true;
}

const char *const KNOB_NAMES[] = {"FC_ATTN_TILES", "FC_ATTN_WGS", "FC_LIN_WGS", "FC_LIN_NO_ROWS", "FC_LIN_WIDE_SHAPE",
                                  "FC_LIN_KSPLIT", "FC_GEMM_NO_SPLIT", "FC_PROJ_GEMM_SHAPE", "FC_PROJ_NO_HEADSPLIT",
                                  "FC_ACCEPT_WGS"};

FcKnobs knobs_from_environment()
{
    FcKnobs k;
    knobs_defaults(k);
    for (const char *n : KNOB_NAMES)
        if (const char *e = getenv(n)) knob_apply(k, n, e);
    return k;
}

FcKnobs &knobs_mut()
{
    static FcKnobs k = knobs_from_environment();  // (once, whichever thread comes first)
    return k;
}

}  // namespace

const FcKnobs &fc_knobs() { return knobs_mut(); }

namespace {

// Row tiles and waves of a workgroup of k_attn_ranges (one on a compute unit) and what it takes (us): its start and end, and each
// stage of 64 keys, on an otherwise idle chip and what a full one adds.
struct AttnShape {
    int R, W;
    double start, stage, full;
};
const AttnShape ATTN_SHAPES[] = {{8, 4, 5.99, 1.239, 0.158}, {4, 4, 4.11, 0.796, 0.072}, {2, 4, 3.24, 0.514, 0.041},
                                 {8, 8, 4.44, 1.393, 0.240}, {4, 8, 4.36, 0.640, 0.238}};

// Estimated time of the attention call (us): the rounds of workgroups and the stream from HBM (6.86 TB/s), joined by a 2-norm, a fixed
// part, and the merge kernel, which reads what the first one wrote (2.44 TB/s both ways).  Fitted to 18000 measured (shape, plan) pairs, 748 shapes
// (1 .. 8 sequences, 1 .. 32 kv heads, 1 .. 8 query heads each, 2 .. 2304 window rows, 100 .. 17000 keys from HBM; rms error 5.6 %) with the kernel as it
// was when its references did not move; the figures of the five shapes above then by what each measured before and since, 2 .. 72 stages on 64 and 256
// compute units.  (20 of 114 drawn plans changed by that, 1.018 x in the mean.)  The plan it picks was 0.8 % slower than the best measured one
// in the mean, 2.7 % in nine of ten shapes, 22 % at most (4 x 10 rows, 64 / 8 heads, 9727 keys, bound by HBM, where two runs of one plan
// may differ by as much).  Eight waves against four with as many rows: 4 x 555 rows of 28 / 4, 215 keys 18.0 -> 16.9, 6 x 183 rows of 32 / 32, 191 keys 15.2 -> 14.1,
// 860 rows of 28 / 4, 929 keys 19.7 -> 19.0.
// (Returns some value >= limit where the terms without the norm reach it.)
double attn_cost(const AttnShape &sh, int64_t pairs, int row_tiles, int kv_len, int64_t splits, int64_t stages, double limit)
{
    const int64_t n = pairs * ((row_tiles + sh.R - 1) / sh.R) * splits, rounds = n / 256, rest = n % 256;
    const double wg = (double)rounds * (sh.start + stages * (sh.stage + sh.full)) +
                      (rest ? sh.start + stages * (sh.stage + sh.full * (double)rest / 256.0) : 0.0);
    const double hbm = (double)pairs * kv_len * 512.0 / 6.86e6;
    const double rest_us = 2.35 + (splits > 1 ? 2.39 + 0.059 * splits + (double)pairs * row_tiles * splits * 8704.0 / 2.44e6 : 0.0);
    const double least = rest_us + fmax(wg, hbm);
    if (least >= limit) return least;
    return rest_us + sqrt(wg * wg + hbm * hbm);
}

// The same for the tile kernel where its operands come straight into registers (bf16 of head_dim 128, up to 96 keys): `wgs`
// workgroups (at most 256: one round), one per sequence, kv head and 16 query rows, each over `groups` groups of 32 keys of
// `group_bytes` bytes.  What counts is what one compute unit can pull that way, 38 B/ns; with up to 64 / 128 workgroups the
// head dimension of V is cut in four / two (the launch does that).
double attn_tile_cost(int64_t wgs, int64_t groups, int64_t group_bytes)
{
    const double g = (double)groups * (double)group_bytes / 16384.0;
    if (wgs <= 64) return 3.58 + 0.275 * g;
    if (wgs <= 128) return 3.92 + 0.341 * g;
    return 4.28 + (0.229 + 1.18e-3 * (double)wgs) * g;
}

// The tile kernel of fp32 and of bf16 of head_dim 64, one tile per workgroup and at most 128 of them, over `groups` groups of 32 keys
// per workgroup: start + each group + each round of groups over the eight waves + what the other workgroups cost + each key
// range (uncut: operands by way of LDS; in ranges: straight into registers, and a second kernel).  Rows: V in four parts (up to 64
// workgroups), in two; in ranges.  fp32 is fitted to 64 .. 2100 keys (rms error 3 .. 5 %), bf16 to 100 .. 16800.  What they choose
// against the best number of ranges, 111 shapes of each of 4 .. 128 workgroups x 100 .. 16800 keys: 0.6 % slower in the mean and 8 % at
// most for fp32 of head_dim 64 (beyond 2100 keys 1.0 and 7 %), 1.7 and 18 % for 128 (2.3 and 9 %), 0.4 and 11 % for bf16 (fitted to
// the short ones only, it was 2.1 and 25 %: it cut 96 workgroups over 4200 keys in two, 20.6 us instead of 16.5).
struct TileCost {
    double start, group, round, load, range;
};
const TileCost TILE_F32_64[] = {{3.53, 0.187, 0.320, 0.203, 0}, {3.68, 0.210, 0.488, 0.075, 0}, {5.75, 0.156, 0.565, 0.320, 0.296}};
const TileCost TILE_F32_128[] = {{4.00, 0.487, 0.092, 0.562, 0}, {4.99, 0.340, 1.076, 0.189, 0}, {6.24, 0.543, 0.031, 0.751, 0.411}};
const TileCost TILE_BF16_64[] = {{3.76, 0.084, 0, 0.039, 0}, {3.93, 0.091, 0, 0.018, 0}, {6.15, 0.111, 0, 0.129, 0.285}};
double attn_tile_ranges_cost(bool f32, int head_dim, int64_t wgs, int64_t groups, int64_t splits)
{
    const int i = splits > 1 ? 2 : wgs <= 64 ? 0 : 1;
    const TileCost &c = !f32 ? TILE_BF16_64[i] : head_dim == 64 ? TILE_F32_64[i] : TILE_F32_128[i];
    return c.start + c.group * (double)groups + c.round * (double)((groups + 7) / 8) + c.load * (double)groups * (double)wgs / 256.0 + c.range * (double)splits;
}

// k_attn_groups: 16-row tiles of a workgroup, parts of the columns of V, waves, and its time (us) in up to one round of
// workgroups: start + h (group + load x) for h groups of 32 keys per wave and x of the compute units in use, or the
// stream from HBM, the longer of the two and a fifth of the shorter.  Fitted to 1380 measured (shape, workgroup) pairs (1 .. 8
// sequences, 1 .. 32 kv heads, 4 .. 64 rows, 64 .. 4500 keys; rms error 6 .. 9 %).  Against the best of 30 plans of k_attn_ranges: 28 / 4 heads,
// 32 rows, 256 / 480 / 768 / 1056 keys 4.6 and 7.6 / 5.4 and 8.5 / 6.0 and 9.1 / 7.1 and 9.6; 64 rows, 1056 keys 8.0 and 10.7; 3 x 19 rows,
// 1581 keys 11.9 and 12.7.
struct GroupsShape {
    int tiles, v_parts, waves;
    double start, start_x, group, load;
};
const GroupsShape GROUPS_SHAPES[] = {{1, 4, 8, 3.25, 0.0, 0.69, 0.105},
                                     {1, 2, 8, 3.05, 0.0, 0.85, 0.125},
                                     {1, 1, 6, 3.04, 0.22, 0.92, 0.09},
                                     {2, 2, 8, 3.80, 0.1, 1.04, 0.21}};
double attn_groups_cost(const GroupsShape &sh, int64_t pairs, int64_t wgs, int kv_len)
{
    const int64_t stages = ((int64_t)kv_len + 63) / 64, n = (stages + sh.waves - 1) / sh.waves;
    const bool half = (kv_len + 31) / 32 % 2 && stages % sh.waves == 1;  // only one wave has n stages, and half of the last
    const double x = (double)wgs / 256.0, work = (double)(2 * n - half) * (sh.group + sh.load * x);
    const double hbm = (double)pairs * kv_len * 512.0 / 5.73e6;
    return sh.start + sh.start_x * x + fmax(work, hbm) + 0.19 * fmin(work, hbm);
}

// Most key ranges the planner considers for this many row tiles: one round of workgroups in some shape, or about 32 MB
// of partial results where a round has few ranges.
int64_t attn_splits_bound(int64_t pairs, int row_tiles, int64_t by_len)
{
    int64_t bound = 1;
    for (const AttnShape &sh : ATTN_SHAPES) {
        const int64_t b = 256 / (pairs * ((row_tiles + sh.R - 1) / sh.R));
        if (b > bound) bound = b;
    }
    if (pairs * row_tiles >= 200 && 3800 / (pairs * row_tiles) > bound) bound = 3800 / (pairs * row_tiles);
    if (bound > 96) bound = 96;  // (more never came out best)
    return bound < by_len ? bound : by_len;
}

// Stages of a range when the keys are cut into `splits`: eight waves take them by twos (fewer ranges, as fast).
int64_t stages_per_range(int W, int64_t splits, int64_t n_stages)
{
    const int64_t stages = (n_stages + splits - 1) / splits;
    return W == 8 && splits > 1 ? (stages + 1) / 2 * 2 : stages;
}

void set_attn_plan(FcAttnPlan &p, int R, int W, int64_t splits, int64_t n_stages)
{
    p.tiles_per_wg = R;
    p.waves = W;
    const int64_t stages = stages_per_range(W, splits, n_stages);
    p.keys_per_split = (int)(stages * 64);
    p.splits = (int)((n_stages + stages - 1) / stages);
}

// Key ranges with which `base` (sequence, kv head, tile group) triples come nearest to `target` workgroups.
int64_t nearest_splits(int64_t target, int64_t base, int64_t by_len)
{
    int64_t splits = (target + base / 2) / base;
    if (splits > by_len) splits = by_len;
    return splits < 1 ? 1 : splits;
}

// At least 128 keys per range.
int64_t splits_by_len(int kv_len)
{
    const int64_t n_stages = ((int64_t)kv_len + 63) / 64;
    return n_stages / 2 > 1 ? n_stages / 2 : 1;
}

// Tiles and number of ranges the tuning knobs ask for (FC_ATTN_TILES, FC_ATTN_WGS).
struct ForcedTiles {
    int R, W;
    int64_t splits;
};
bool attn_forced() { return fc_knobs().attn_r > 0 || fc_knobs().attn_wgs > 0; }
ForcedTiles forced_tiles(int64_t pairs, int row_tiles, int64_t by_len)
{
    int R = fc_knobs().attn_r, W = fc_knobs().attn_w;
    int64_t target = fc_knobs().attn_wgs;
    if (W != 8) W = 4;
    if (R != 2 && R != 4 && R != 8) R = row_tiles <= 2 ? 2 : (row_tiles <= 7 ? 4 : 8);
    if (R == 2) W = 4;
    if (target <= 0) target = 256;
    return ForcedTiles{R, W, nearest_splits(target, pairs * ((row_tiles + R - 1) / R), by_len)};
}

// Bytes of partial results per row tile and key range: 32 x 128 half floats and 32 x 4 floats of row state.
constexpr size_t ATTN_PART_BYTES = 32 * (128 * 2 + 4 * sizeof(float));

// Workspace a call must bring (bytes), a bound that callers rely on: the partial results of 256 units of two, four or eight
// 32-row tiles by the row count, of 512 units of two where the cache is too short to give 256 of four, or those of the plan that a
// tuning knob forces.  It is not the launch (every shape there puts one workgroup on a compute unit): the planner often takes
// fewer ranges, and more only where the caller brings more (fc_workspace_bytes says how much is of use).
size_t attn_required(const fc_config &cfg, int A, int kv_len)
{
    if (cfg.dtype != FC_BF16 || cfg.head_dim != 128) return 0;  // those cut the keys only where there is space for it
    const int64_t pairs = (int64_t)cfg.batch * cfg.n_kv_heads, by_len = splits_by_len(kv_len);
    const int row_tiles = (int)(((int64_t)(cfg.n_q_heads / cfg.n_kv_heads) * A + 31) / 32);
    int64_t splits;
    if (attn_forced()) {
        splits = forced_tiles(pairs, row_tiles, by_len).splits;
    } else {
        const int R = row_tiles <= 2 ? 2 : (row_tiles <= 7 ? 4 : 8);
        const int64_t base = pairs * ((row_tiles + R - 1) / R);
        splits = nearest_splits(256, base, by_len);
        if (R == 4 && base * splits < 256) splits = nearest_splits(512, pairs * ((row_tiles + 1) / 2), by_len);
    }
    return splits > 1 ? (size_t)pairs * row_tiles * splits * ATTN_PART_BYTES : 0;
}

}  // namespace

FcAttnPlan fc_plan_attention(const fc_config &cfg, int A, int kv_len, size_t cap)
{
    FcAttnPlan p;
    memset(&p, 0, sizeof p);
    p.splits = 1;
    const int g = cfg.n_q_heads / cfg.n_kv_heads;
    if (cfg.dtype != FC_BF16 || cfg.head_dim != 128) {
        // kind 0: one workgroup per (sequence, kv head, one or two 16-row tiles); two tiles share the key
        // and value loads and are taken once they still fill half the chip (head_dim 64 only: with fp32 rows
        // of 128 the operands of two tiles do not fit in registers).  The keys are cut into ranges, one round of workgroups
        // at most, where their shorter chains pay for the second launch that merges them (3 to 5 us).
        const bool f32 = cfg.dtype == FC_F32;
        const int64_t rows = (int64_t)g * A, pairs = (int64_t)cfg.batch * cfg.n_kv_heads;
        p.row_tiles = (int)((rows + 15) / 16);
        p.waves = 8;
        p.tiles_per_wg = cfg.head_dim == 64 && pairs * ((rows + 31) / 32) >= 128 ? 2 : 1;
        const int64_t base = pairs * ((p.row_tiles + p.tiles_per_wg - 1) / p.tiles_per_wg);
        const int64_t groups = ((int64_t)kv_len + 31) / 32;
        auto cut = [&](int64_t n) {
            FcAttnPlan c = p;
            const int64_t per = (groups + n - 1) / n;
            c.splits = (int)((groups + per - 1) / per);
            c.keys_per_split = (int)(32 * per);
            return c;
        };
        FcAttnPlan chosen = cut(1);
        if (p.tiles_per_wg == 2) {
            // Two tiles fill half a round at least: just half of one leaves a choice, and two ranges pay from 13 / 53 groups on
            // (us uncut and in two, fp32: 200 keys 9.7 and 11.0, 384 13.0 and 13.4, 448 15.6 and 13.7, 700 20.7 and 16.9, 2100 46.5 and 33.1;
            // bf16: 1000 keys 10.2 and 11.5, 1664 13.4 and 13.5, 1800 14.9 and 14.3, 4000 27.4 and 21.8).
            const FcAttnPlan two = cut(2);
            if (base == 128 && groups >= (f32 ? 13 : 53) && fc_plan_workspace(cfg, two) <= cap) chosen = two;
            return chosen;
        }
        double best = 1e30;
        for (int64_t n = 1; n <= groups && n * base <= 256; ++n) {
            const FcAttnPlan c = cut(n);
            const double t = attn_tile_ranges_cost(f32, cfg.head_dim, base * c.splits, c.keys_per_split / 32, c.splits);
            if (t < best && fc_plan_workspace(cfg, c) <= cap) {
                best = t;
                chosen = c;
            }
        }
        return chosen;
    }
    p.kind = 1;
    p.row_tiles = (int)(((int64_t)g * A + 31) / 32);
    const int64_t pairs = (int64_t)cfg.batch * cfg.n_kv_heads;
    const int64_t n_stages = ((int64_t)kv_len + 63) / 64;
    const int64_t by_len = splits_by_len(kv_len);
    if (attn_forced()) {  // (whatever the space: the caller checks)
        const ForcedTiles f = forced_tiles(pairs, p.row_tiles, by_len);
        set_attn_plan(p, f.R, f.W, f.splits, n_stages);
        return p;
    }
    const int64_t bound = attn_splits_bound(pairs, p.row_tiles, by_len);
    const int64_t within = (int64_t)(cap / ((size_t)pairs * p.row_tiles * ATTN_PART_BYTES));
    double best = 1e30;
    for (const AttnShape &sh : ATTN_SHAPES) {
        const int64_t base = pairs * ((p.row_tiles + sh.R - 1) / sh.R);
        // the first few splits, whole rounds of workgroups, and steps of a third between
        static const int STEPS[] = {1, 2, 3, 4, 5, 6, 7, 8, 12, 16, 24, 32, 48, 64, 96};
        constexpr int NS = sizeof STEPS / sizeof STEPS[0];
        for (int c = 0; c < NS + 3; ++c) {
            const int64_t splits = c < NS ? STEPS[c] : 256 * (c - NS + 1) / base;
            if (splits < 1 || splits > bound) continue;
            const int64_t stages = stages_per_range(sh.W, splits, n_stages), ranges = (n_stages + stages - 1) / stages;
            if (ranges > 1 && ranges > within) continue;
            const double limit = best * (1 - 1e-9);
            const double t = attn_cost(sh, pairs, p.row_tiles, kv_len, ranges, stages, limit);
            if (t < limit) {
                best = t;
                set_attn_plan(p, sh.R, sh.W, splits, n_stages);
            }
        }
    }
    // one launch: 16 or 32 rows per workgroup, or (short keys only) the tile kernel
    const int64_t row_tiles = ((int64_t)g * A + 15) / 16;
    auto one_launch = [&](int kind, int tiles, int v_parts, int waves) {
        p.kind = kind;
        p.splits = 1;
        p.keys_per_split = kind == 0 ? (kv_len + 31) / 32 * 32 : (int)(n_stages * 64);
        p.row_tiles = (int)row_tiles;
        p.tiles_per_wg = tiles;
        p.waves = waves;
        p.v_parts = v_parts;
    };
    if (pairs * row_tiles > 512) return p;
    // Six waves beyond 1200 keys: the estimate takes them where the other shapes are as fast or faster.  60 drawn shapes of
    // 1201 .. 3500 keys that would change, in the geometric mean 0.955 x (us without and with: 8 x 10 rows, 28 / 4 heads, 1425 keys 13.3 and
    // 14.8; 3 x 45 rows, 1220 keys 11.8 and 12.5; 2 x 42 rows, 32 / 32 heads, 2716 keys 23.6 and 28.5); the others, most of them against
    // the split-KV kernel, gain (6 x 13 rows, 32 / 32 heads, 1250 keys 27.2 and 23.2).
    for (const GroupsShape &sh : GROUPS_SHAPES) {
        const int64_t wgs = pairs * ((row_tiles + sh.tiles - 1) / sh.tiles) * sh.v_parts;
        if (wgs > 256 || (sh.waves == 6 && kv_len > 1200)) continue;
        // (Beside k_attn_ranges the estimate is 6 % short: of 4000 drawn shapes 144 are decided by it, and 120 of those measured
        // 0.947 x without it, those between 1.03 and 1.06 0.954 x.)
        const double t = 1.06 * attn_groups_cost(sh, pairs, wgs, kv_len);
        if (t < best) {
            best = t;
            one_launch(2, sh.tiles, sh.v_parts, sh.waves);
        }
    }
    // (32 rows x 28 heads, 32 / 64 keys 4.0 and 4.7 us; from 100 keys on the same or slower)
    if (kv_len <= 96 && pairs * row_tiles <= 256 && attn_tile_cost(pairs * row_tiles, ((int64_t)kv_len + 31) / 32, 16384) < best)
        one_launch(0, 1, 0, 8);
    return p;
}

size_t fc_plan_workspace(const fc_config &cfg, const FcAttnPlan &p)
{
    if (p.splits <= 1) return 0;
    if (p.kind == 0)  // per (workgroup tile, split): rows x Dh partial outputs + rows x 2 floats of row state
        return (size_t)cfg.batch * cfg.n_kv_heads * ((p.row_tiles + p.tiles_per_wg - 1) / p.tiles_per_wg) * p.splits *
               (16 * p.tiles_per_wg) * (cfg.head_dim + 2) * sizeof(float);
    return (size_t)cfg.batch * cfg.n_kv_heads * p.row_tiles * p.splits * ATTN_PART_BYTES;
}

namespace {

// The last few results of a pure planning function, per host thread: a step asks for the same shapes in every layer, and
// a plan takes a microsecond or two.  Keys are plain values without padding.
template <typename Key, typename Value>
struct Memo {
    static constexpr int N = 4;
    Key key[N];
    Value value[N];
    int used = 0, next = 0;
    template <typename Make>
    const Value &get(const Key &k, Make make)
    {
        for (int i = 0; i < used; ++i)
            if (!memcmp(&key[i], &k, sizeof k)) return value[i];
        const int at = next;
        next = (next + 1) % N;
        value[at] = make();
        key[at] = k;
        if (used < N) ++used;
        return value[at];
    }
};

struct AttnPlanKey {
    size_t bytes;
    int32_t batch, n_q_heads, n_kv_heads, head_dim, dtype, A, kv_len, knobs;
};
static_assert(sizeof(AttnPlanKey) == sizeof(size_t) + 8 * sizeof(int32_t), "no padding");

struct WidePlanKey {
    size_t bytes;
    int32_t dtype, mode, M, K, N, knobs;
};
static_assert(sizeof(WidePlanKey) == sizeof(size_t) + 6 * sizeof(int32_t), "no padding");

// The plan of one call that brings `bytes` of workspace.
FcAttnPlan plan_with_workspace(const fc_config &c, int A, int kv_len, size_t bytes)
{
    static thread_local Memo<AttnPlanKey, FcAttnPlan> memo;
    const AttnPlanKey k = {bytes, c.batch, c.n_q_heads, c.n_kv_heads, c.head_dim, c.dtype, A, kv_len, fc_knobs().version};
    return memo.get(k, [&] { return fc_plan_attention(c, A, kv_len, bytes); });
}

}  // namespace

// Workspace (bytes) of the attention of windows of up to max_rows rows over up to max_seq keys: what a call must bring,
// and (`useful`) what the plan for the full length takes where that is more.  Shorter caches make do with as much.
static size_t attn_workspace(const fc_config &cfg, int max_rows, bool useful)
{
    const int64_t pairs = (int64_t)cfg.batch * cfg.n_kv_heads, g = cfg.n_q_heads / cfg.n_kv_heads;
    size_t most = 0;
    int64_t tiles = 0;
    for (int a = 1; a <= max_rows; ++a) {
        const int64_t t = (g * a + 15) / 16;
        if (t == tiles) continue;  // plans depend on the 16-row tiles only
        tiles = t;
        size_t b = attn_required(cfg, a, cfg.max_seq);
        if (useful && pairs * t <= 4000) {  // (beyond 1900 32-row tiles no plan cuts the keys)
            const size_t u = fc_plan_workspace(cfg, fc_plan_attention(cfg, a, cfg.max_seq));
            if (u > b) b = u;
        }
        if (b > most) most = b;
    }
    return most;
}

extern "C" {

const char *fc_last_error(void) { return g_err; }

fc_status fc_tuning_set(const char *name, const char *value)
{
    if (!name) return fail(FC_ERR_INVALID_ARG, "name is NULL");
    if (!knob_apply(knobs_mut(), name, value)) return fail(FC_ERR_INVALID_ARG, "unknown tuning knob %s", name);
    ++knobs_mut().version;
    return FC_OK;
}

fc_status fc_attention_plan(const fc_config *cfg, int32_t A, int32_t kv_len, int32_t *plan)
{
    fc_status st = check_config(cfg);
    if (st != FC_OK) return st;
    if (!plan) return fail(FC_ERR_INVALID_ARG, "plan is NULL");
    if (A < 1) return fail(FC_ERR_INVALID_ARG, "A %d must be >= 1", A);
    if (kv_len < 1 || kv_len > cfg->max_seq) return fail(FC_ERR_BOUNDS, "kv_len %d outside [1, %d]", kv_len, cfg->max_seq);
    const FcAttnPlan p = fc_plan_attention(*cfg, A, kv_len, attn_workspace(*cfg, A, true));
    plan[0] = p.kind;
    plan[1] = p.splits;
    plan[2] = p.keys_per_split;
    plan[3] = p.row_tiles;
    plan[4] = p.tiles_per_wg;
    plan[5] = p.waves;
    return FC_OK;
}

size_t fc_cache_storage_bytes(const fc_config *cfg)
{
    if (check_config(cfg) != FC_OK) return 0;
    return (size_t)cfg->n_layers * cfg->batch * cfg->n_kv_heads * spad_of(*cfg) * cfg->head_dim *
           esize_of(cfg->dtype);
}

fc_status fc_cache_alloc(const fc_config *cfg, void *k_storage, void *v_storage, fc_cache **out)
{
    if (!out) return fail(FC_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    fc_status st = check_config(cfg);
    if (st != FC_OK) return st;
    if ((k_storage == nullptr) != (v_storage == nullptr))
        return fail(FC_ERR_INVALID_ARG, "k_storage and v_storage must both be given or both be NULL");
    if (k_storage && (((uintptr_t)k_storage | (uintptr_t)v_storage) & 15))
        return fail(FC_ERR_INVALID_ARG, "cache storage must be 16-byte aligned");
    fc_cache *c = new (std::nothrow) fc_cache;
    if (!c) return fail(FC_ERR_OOM, "host allocation failed");
    c->cfg = *cfg;
    c->spad = spad_of(*cfg);
    c->esize = esize_of(cfg->dtype);
    c->layer_elems = (size_t)cfg->batch * cfg->n_kv_heads * c->spad * cfg->head_dim;
    c->k = k_storage;
    c->v = v_storage;
    c->owned = false;
    for (int i = 0; i < 64; ++i)
        c->inv_freq[i] = i < cfg->head_dim / 2 ? pow((double)cfg->rope_base, -2.0 * i / cfg->head_dim) : 0.0;
    if (!k_storage) {
        const size_t bytes = fc_cache_storage_bytes(cfg);
        void *k = nullptr, *v = nullptr;
        if (hipMalloc(&k, bytes) != hipSuccess || hipMalloc(&v, bytes) != hipSuccess ||
            hipMemset(k, 0, bytes) != hipSuccess || hipMemset(v, 0, bytes) != hipSuccess) {
            (void)hipGetLastError();
            if (k) (void)hipFree(k);
            if (v) (void)hipFree(v);
            delete c;
            return fail(FC_ERR_OOM, "could not allocate 2 x %zu bytes of cache storage", bytes);
        }
        c->k = k;
        c->v = v;
        c->owned = true;
    }
    // Scratch for kernels that hand partial results between workgroups.  On a host without a GPU
    // (argument-validation tests) the handle is still created; compute calls then fail at launch.
    c->scratch = nullptr;
    {
        void *s = nullptr;
        const hipError_t e = hipMalloc(&s, FC_SCRATCH_BYTES);
        if (e == hipSuccess) {
            c->scratch = s;
        } else {
            (void)hipGetLastError();
            if (s) (void)hipFree(s);
            int ndev = 0;
            if (hipGetDeviceCount(&ndev) == hipSuccess && ndev > 0) {
                if (c->owned) {
                    (void)hipFree(c->k);
                    (void)hipFree(c->v);
                }
                delete c;
                return fail(FC_ERR_OOM, "could not allocate %u bytes of device scratch", FC_SCRATCH_BYTES);
            }
            (void)hipGetLastError();
        }
    }
    *out = c;
    return FC_OK;
}

fc_status fc_cache_free(fc_cache *cache)
{
    if (!cache) return FC_OK;
    fc_status st = FC_OK;
    if (cache->owned) {
        hipError_t e1 = hipFree(cache->k), e2 = hipFree(cache->v);
        if (e1 != hipSuccess || e2 != hipSuccess) st = hip_fail(e1 != hipSuccess ? e1 : e2, "hipFree");
    }
    if (cache->scratch) {
        hipError_t e = hipFree(cache->scratch);
        if (e != hipSuccess && st == FC_OK) st = hip_fail(e, "hipFree");
    }
    delete cache;
    return st;
}

fc_status fc_cache_ptrs(const fc_cache *cache, int32_t layer, void **k, void **v)
{
    fc_status st = check_cache_layer(cache, layer);
    if (st != FC_OK) return st;
    if (!k || !v) return fail(FC_ERR_INVALID_ARG, "k or v is NULL");
    *k = layer_ptr(cache, cache->k, layer);
    *v = layer_ptr(cache, cache->v, layer);
    return FC_OK;
}

static fc_status copy_rows(const fc_cache *cache, int32_t layer, void *k_rows, void *v_rows,
                           int32_t start, int32_t rows, void *stream, bool to_cache)
{
    fc_status st = check_cache_layer(cache, layer);
    if (st != FC_OK) return st;
    if (!k_rows || !v_rows) return fail(FC_ERR_INVALID_ARG, "k_rows or v_rows is NULL");
    if (rows < 1) return fail(FC_ERR_INVALID_ARG, "rows %d must be >= 1", rows);
    if (start < 0 || start > cache->cfg.max_seq - rows)
        return fail(FC_ERR_BOUNDS, "rows [%d, %d+%d) outside the cache of %d rows", start, start, rows,
                    cache->cfg.max_seq);
    hipError_t e = fc_launch_copy_rows(geom_of(cache), cache->cfg.dtype, layer_ptr(cache, cache->k, layer),
                                       layer_ptr(cache, cache->v, layer), k_rows, v_rows, start, rows,
                                       to_cache, (hipStream_t)stream);
    return e == hipSuccess ? FC_OK : hip_fail(e, "row copy launch");
}

fc_status fc_cache_write_rows(fc_cache *cache, int32_t layer, const void *k_rows, const void *v_rows,
                              int32_t start, int32_t rows, void *stream)
{
    return copy_rows(cache, layer, (void *)k_rows, (void *)v_rows, start, rows, stream, true);
}

fc_status fc_cache_read_rows(const fc_cache *cache, int32_t layer, void *k_rows, void *v_rows,
                             int32_t start, int32_t rows, void *stream)
{
    return copy_rows(cache, layer, k_rows, v_rows, start, rows, stream, false);
}

fc_status fc_window(int32_t step, int32_t P, int32_t G, int32_t Bk, int32_t steps_per_block,
                    int32_t refresh_every, int32_t mode, int32_t *win_start, int32_t *rows,
                    int32_t *refresh_after)
{
    if (!win_start || !rows || !refresh_after) return fail(FC_ERR_INVALID_ARG, "output pointer is NULL");
    if (step < 0 || P < 0 || G < 1 || Bk < 1 || steps_per_block < 1 || refresh_every < 0)
        return fail(FC_ERR_INVALID_ARG, "step/P >= 0, G/Bk/steps_per_block >= 1, refresh_every >= 0 required");
    if (mode != 0 && mode != 1) return fail(FC_ERR_INVALID_ARG, "mode %d is neither 0 nor 1", mode);
    const int64_t n_blocks = ((int64_t)G + Bk - 1) / Bk;
    const int64_t blk = step / steps_per_block;
    if (blk >= n_blocks)
        return fail(FC_ERR_BOUNDS, "step %d lies past the last of %lld blocks", step, (long long)n_blocks);
    const int64_t first = blk * Bk;  // offset of the block inside the generation region
    const int64_t rest = (int64_t)G - first;
    if ((int64_t)P + G > INT32_MAX) return fail(FC_ERR_INVALID_ARG, "P + G overflows int32");
    *win_start = (int32_t)(P + first);
    *rows = (int32_t)(mode == 1 ? rest : (rest < Bk ? rest : Bk));
    *refresh_after = (refresh_every > 0 && ((int64_t)step + 1) % refresh_every == 0) ? 1 : 0;
    return FC_OK;
}

// d_ff: of the layer the call is a part of (0: projections and attention alone); keys: that its attention reads (0: not known)
static fc_status project_scatter(fc_cache *cache, int32_t layer, int32_t d_ff, int32_t keys, const void *x, const void *w_qkv, const void *b_qkv,
                                 int32_t win_start, int32_t A, const int32_t *pos, void *q_out, void *stream)
{
    fc_status st = check_cache_layer(cache, layer);
    if (st != FC_OK) return st;
    if (!x || !w_qkv || !q_out) return fail(FC_ERR_INVALID_ARG, "x, w_qkv or q_out is NULL");
    if (A < 1) return fail(FC_ERR_INVALID_ARG, "A %d must be >= 1", A);
    if ((int64_t)A * cache->cfg.batch > (1 << 24))
        return fail(FC_ERR_UNSUPPORTED, "batch * A exceeds 2^24 rows");
    if (!pos && (win_start < 0 || win_start > cache->cfg.max_seq - A))
        return fail(FC_ERR_BOUNDS, "window [%d, %d+%d) outside the cache of %d rows", win_start, win_start,
                    A, cache->cfg.max_seq);
    // Not told, the keys up to the window's end count; where rows are listed on the device, all there is room for.
    const FcGeom G = geom_of(cache, d_ff, keys > 0 ? keys : pos ? cache->cfg.max_seq : win_start + A);
    void *kl = layer_ptr(cache, cache->k, layer), *vl = layer_ptr(cache, cache->v, layer);
    // wide windows: tiled GEMM; short windows: weight-streaming kernels; small problems, other shapes and fp32: tile kernel
    hipError_t e;
    if (fc_project_prefers_tile(cache->cfg, cache->cfg.batch * A))
        e = fc_launch_project_tile(G, cache->inv_freq, cache->cfg.dtype, x, w_qkv, b_qkv, pos, win_start, A, q_out, kl, vl,
                                   (hipStream_t)stream);
    else if (fc_project_prefers_gemm(cache->cfg, cache->cfg.batch * A, cache->scratch != nullptr))
        e = fc_launch_project_gemm(G, x, w_qkv, b_qkv, pos, win_start, A, q_out, kl, vl, (hipStream_t)stream);
    else if (fc_project_mfma_supported(cache->cfg))
        e = fc_launch_project_mfma(G, x, w_qkv, b_qkv, pos, win_start, A, q_out, kl, vl,
                                   cache->scratch, (hipStream_t)stream);
    else
        e = fc_launch_project_tile(G, cache->inv_freq, cache->cfg.dtype, x, w_qkv, b_qkv, pos, win_start, A, q_out, kl,
                                   vl, (hipStream_t)stream);
    return e == hipSuccess ? FC_OK : hip_fail(e, "projection launch");
}

fc_status fc_qkv_project_scatter(fc_cache *cache, int32_t layer, const void *x, const void *w_qkv,
                                 const void *b_qkv, int32_t win_start, int32_t A, const int32_t *pos,
                                 void *q_out, void *stream)
{
    return project_scatter(cache, layer, 0, 0, x, w_qkv, b_qkv, win_start, A, pos, q_out, stream);
}

size_t fc_workspace_bytes(const fc_config *cfg, int32_t max_rows)
{
    if (check_config(cfg) != FC_OK || max_rows < 1) return 0;
    return attn_workspace(*cfg, max_rows, true);
}

static fc_status run_attention(fc_cache *cache, int32_t layer, int32_t d_ff, const FcAttnPlan &plan, const void *q, int32_t A,
                               int32_t kv_len, const int32_t *pos, void *out, void *workspace, size_t space, void *stream)
{
    const size_t bytes = fc_plan_workspace(cache->cfg, plan);
    if (bytes > space)  // (not reached: the planner keeps within the space, and the plan of a tuning knob is required space)
        return fail(FC_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", bytes, space);
    const FcGeom G = geom_of(cache, d_ff, kv_len);
    void *kl = layer_ptr(cache, cache->k, layer), *vl = layer_ptr(cache, cache->v, layer);
    hipError_t e = plan.kind != 0
                       ? fc_launch_attention_mfma(G, plan, q, kl, vl, pos, A, kv_len, out, workspace,
                                                  (hipStream_t)stream)
                       : fc_launch_attention_tile(G, plan, cache->cfg.dtype, q, kl, vl, pos, A, kv_len, out, workspace,
                                                  (hipStream_t)stream);
    return e == hipSuccess ? FC_OK : hip_fail(e, "attention launch");
}

static fc_status active_attention(fc_cache *cache, int32_t layer, int32_t d_ff, const void *q, int32_t A, int32_t kv_len,
                                  const int32_t *pos, void *out, void *workspace, size_t workspace_bytes, void *stream)
{
    fc_status st = check_cache_layer(cache, layer);
    if (st != FC_OK) return st;
    if (!q || !out) return fail(FC_ERR_INVALID_ARG, "q or out is NULL");
    if (A < 1) return fail(FC_ERR_INVALID_ARG, "A %d must be >= 1", A);
    if ((int64_t)A * cache->cfg.batch > (1 << 24))
        return fail(FC_ERR_UNSUPPORTED, "batch * A exceeds 2^24 rows");
    if (kv_len < 1 || kv_len > cache->cfg.max_seq)
        return fail(FC_ERR_BOUNDS, "kv_len %d outside [1, %d]", kv_len, cache->cfg.max_seq);
    const size_t need = attn_required(cache->cfg, A, kv_len), given = workspace ? workspace_bytes : 0;
    if (given < need) return fail(FC_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", need, given);
    const FcAttnPlan plan = plan_with_workspace(cache->cfg, A, kv_len, given);
    return run_attention(cache, layer, d_ff, plan, q, A, kv_len, pos, out, workspace, given, stream);
}

fc_status fc_active_attention(fc_cache *cache, int32_t layer, const void *q, int32_t A, int32_t kv_len,
                              const int32_t *pos, void *out, void *workspace, size_t workspace_bytes,
                              void *stream)
{
    return active_attention(cache, layer, 0, q, A, kv_len, pos, out, workspace, workspace_bytes, stream);
}

// ---------------------------------------------------------------------------------------------
// Attention for callers that cannot allocate: the split-KV partial results live in a static device
// array instead of a caller-provided workspace.  The array's name is only a host-side stand-in for
// the symbol; its device address is looked up once per device and kept.
}  // extern "C"

#define FC_STATIC_SCRATCH_BYTES (16u * 1024u * 1024u)
#define FC_MAX_DEVICES 64
static __device__ __align__(256) unsigned char fc_static_scratch[FC_STATIC_SCRATCH_BYTES];

namespace {

// Device address of fc_static_scratch on the current device (each GPU holds its own copy of the
// array at its own address).  On failure *out stays nullptr and the status (error text set) is returned.
fc_status static_scratch_ptr(void **out)
{
    *out = nullptr;
    static void *ptrs[FC_MAX_DEVICES];  // zero-initialised; a slot is written once and then only read
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= FC_MAX_DEVICES)
        return fail(FC_ERR_UNSUPPORTED, "device ordinal %d outside [0, %d)", dev, FC_MAX_DEVICES);
    void *p = __atomic_load_n(&ptrs[dev], __ATOMIC_ACQUIRE);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(fc_static_scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(fc_static_scratch)");
        if (!p) return fail(FC_ERR_HIP, "hipGetSymbolAddress(fc_static_scratch) returned a null address");
        __atomic_store_n(&ptrs[dev], p, __ATOMIC_RELEASE);
    }
    *out = p;
    return FC_OK;
}

}  // namespace

extern "C" {

size_t fc_active_attention_static_max_bytes(void) { return FC_STATIC_SCRATCH_BYTES; }

fc_status fc_active_attention_static(fc_cache *cache, int32_t layer, const void *q, int32_t A, int32_t kv_len,
                                     const int32_t *pos, void *out, void *stream)
{
    fc_status st = check_cache_layer(cache, layer);
    if (st != FC_OK) return st;
    if (!q || !out) return fail(FC_ERR_INVALID_ARG, "q or out is NULL");
    if (A < 1) return fail(FC_ERR_INVALID_ARG, "A %d must be >= 1", A);
    if ((int64_t)A * cache->cfg.batch > (1 << 24))
        return fail(FC_ERR_UNSUPPORTED, "batch * A exceeds 2^24 rows");
    if (kv_len < 1 || kv_len > cache->cfg.max_seq)
        return fail(FC_ERR_BOUNDS, "kv_len %d outside [1, %d]", kv_len, cache->cfg.max_seq);
    const size_t need = attn_required(cache->cfg, A, kv_len);
    if (need > FC_STATIC_SCRATCH_BYTES)
        return fail(FC_ERR_WORKSPACE, "this shape needs %zu bytes of partial results, the static scratch holds %u", need,
                    FC_STATIC_SCRATCH_BYTES);
    const FcAttnPlan plan = plan_with_workspace(cache->cfg, A, kv_len, FC_STATIC_SCRATCH_BYTES);
    void *scratch = nullptr;
    if (plan.splits > 1) {
        st = static_scratch_ptr(&scratch);
        if (st != FC_OK) return st;
    }
    // Nothing in the scratch has to start at zero: every (row tile, split) slot the merge kernel
    // reads is written by the first kernel of the same call.
    return run_attention(cache, layer, 0, plan, q, A, kv_len, pos, out, scratch, FC_STATIC_SCRATCH_BYTES, stream);
}

fc_status fc_refresh(fc_cache *cache, int32_t layer, const void *x, const void *w_qkv, const void *b_qkv,
                     int32_t start, int32_t R, int32_t kv_len, void *q_scratch, void *out,
                     void *workspace, size_t workspace_bytes, void *stream)
{
    fc_status st = check_cache_layer(cache, layer);
    if (st != FC_OK) return st;
    if (!x || !w_qkv || !q_scratch) return fail(FC_ERR_INVALID_ARG, "x, w_qkv or q_scratch is NULL");
    if (R < 1) return fail(FC_ERR_INVALID_ARG, "R %d must be >= 1", R);
    if (start < 0 || start > cache->cfg.max_seq - R)
        return fail(FC_ERR_BOUNDS, "rows [%d, %d+%d) outside the cache of %d rows", start, start, R,
                    cache->cfg.max_seq);
    if (out) {
        // validate the attention half before anything is enqueued, so a failure has no side effects
        if (kv_len < 1 || kv_len > cache->cfg.max_seq)
            return fail(FC_ERR_BOUNDS, "kv_len %d outside [1, %d]", kv_len, cache->cfg.max_seq);
        if (start + R > kv_len)
            return fail(FC_ERR_BOUNDS, "refreshed rows end at %d, beyond kv_len %d", start + R, kv_len);
        const size_t need = attn_required(cache->cfg, R, kv_len), given = workspace ? workspace_bytes : 0;
        if (given < need) return fail(FC_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", need, given);
    }
    st = project_scatter(cache, layer, 0, out ? kv_len : 0, x, w_qkv, b_qkv, start, R, nullptr, q_scratch, stream);
    if (st != FC_OK || !out) return st;
    return fc_active_attention(cache, layer, q_scratch, R, kv_len, nullptr, out, workspace, workspace_bytes,
                               stream);
}

// ---------------------------------------------------------------------------------------------
// The rest of the layer on the window rows.

static fc_status check_dtype(int32_t dtype)
{
    if (dtype != FC_F32 && dtype != FC_BF16)
        return fail(FC_ERR_INVALID_ARG, "dtype %d is neither FC_F32 nor FC_BF16", dtype);
    return FC_OK;
}

fc_status fc_rmsnorm(int32_t dtype, const void *x, const void *weight, float eps, int32_t rows,
                     int32_t hidden, void *out, void *stream)
{
    fc_status st = check_dtype(dtype);
    if (st != FC_OK) return st;
    if (!x || !weight || !out) return fail(FC_ERR_INVALID_ARG, "x, weight or out is NULL");
    if (rows < 1 || hidden < 1) return fail(FC_ERR_INVALID_ARG, "rows and hidden must be >= 1");
    if (!(eps >= 0.0f) || !isfinite(eps)) return fail(FC_ERR_INVALID_ARG, "eps must be finite and >= 0");
    hipError_t e = fc_launch_rmsnorm(dtype, x, weight, eps, rows, hidden, out, (hipStream_t)stream);
    return e == hipSuccess ? FC_OK : hip_fail(e, "rmsnorm launch");
}

static fc_status check_linear_shape(int32_t M, int32_t K, int32_t N)
{
    if (M < 1 || K < 1 || N < 1) return fail(FC_ERR_INVALID_ARG, "M, K and N must be >= 1");
    if (K % 8 != 0) return fail(FC_ERR_UNSUPPORTED, "K %d is not a multiple of 8", K);
    if (M > (1 << 24) || N > (1 << 22)) return fail(FC_ERR_UNSUPPORTED, "M is limited to 2^24 rows, N to 2^22");
    return FC_OK;
}

// Workspace of a linear call: what it must bring, and what its best plan takes where that is more.
struct LinearSpace {
    size_t least, useful;
    uint64_t plan;  // what of the plan the two sizes depend on besides the rows (a word per mode)
};

// Tiled GEMM where it is planned, streaming kernels otherwise.
static LinearSpace linear_need(int dtype, int mode, int M, int K, int N)
{
    const FcWidePlan wide = fc_plan_wide(dtype, mode, M, K, N);
    if (wide.kind != 1) {
        const size_t n = fc_skinny_workspace(fc_plan_skinny(dtype, mode, M, K, N));
        return LinearSpace{n, n, 0};
    }
    const size_t best = fc_wide_workspace(wide, M, N), part = (size_t)M * N * sizeof(float);
    return LinearSpace{wide.required, best > wide.required ? best : wide.required, 1 + (wide.required / part) * 32 + (uint64_t)wide.ksplit * 1024};
}

// ... of the layer whose output is N wide and of the gated one of N / 2 outputs.
static LinearSpace linear_workspace(int32_t dtype, int32_t M, int32_t K, int32_t N)
{
    // the gated W_1 is planned on its F = N / 2 outputs; its slabs hold half as many outputs, so the
    // two plans need the same space and one query serves both calls
    LinearSpace a = linear_need(dtype, FC_LIN_RESIDUAL, M, K, N);
    if (N % 2 == 0) {
        const LinearSpace b = linear_need(dtype, FC_LIN_GATE_UP, M, K, N / 2);
        if (b.least > a.least) a.least = b.least;
        if (b.useful > a.useful) a.useful = b.useful;
        a.plan = a.plan << 1 | (b.plan != 0);  // (a gated layer is never cut into parts)
    }
    return a;
}

size_t fc_linear_workspace_bytes(int32_t dtype, int32_t M, int32_t K, int32_t N)
{
    if ((dtype != FC_F32 && dtype != FC_BF16) || M < 1 || K < 1 || N < 1) return 0;
    return linear_workspace(dtype, M, K, N).useful;
}

// Small bf16 problems run in the tile kernel: it is one launch, and short as long as the products are few, where the
// tiled GEMM walks the hidden dimension stage by stage in a few workgroups and cuts it only with a second launch, and
// the slice-wise kernel always has one.  But its waves walk the hidden dimension as a chain, and its workgroups pull X for 16
// weight rows each.  Both sides measured, weights from HBM (us, tile kernel first):
//   against the tiled GEMM, 33 .. 256 rows: 1024 x 1024 outputs, 64 rows 4.4 and 6.9, 128 rows 5.4 and 8.1; 2048 x 1024, 64 rows
//   6.4 and 8.3, 74 rows 9.2 and 8.8; 4096 x 256, 33 rows 9.2 and 8.3; 8192 x 256 16.4 and 11.1: up to hidden 2048, by
//   products;
//   against the slice-wise kernel, 1 .. 32 rows, 30 matrices of 0.5 to 68 million weights: 1024 x 512 4.9 and 9.1 at any row
//   count; 2048 x 8192, 8 / 16 / 32 rows 11.0 and 13.5 / 12.9 and 13.6 / 17.2 and 14.8; 8192 x 1024 12.8 and 10.9 at 4 rows;
//   18944 x 3584 28.1 and 29.4 at 4 rows, 36 and 30 at 12.  The estimate is wrong by more than 3 % (at most 8) in 4 of 386 measured
//   cases (by products alone it was wrong in 94, by up to a factor of two).
// Estimate of the tile kernel at up to 32 rows (us).
static double linear_tile_us(bool gated, int M, int K, int N)
{
    const double weights = (gated ? 2e-6 : 1e-6) * K * (double)N;  // millions
    const int tiles = gated ? (N + 7) / 8 : (N + 15) / 16, passes = M > 16 && tiles < 256 ? 2 : 1;  // over the weights
    const int wgs = tiles * passes;
    const double uneven = wgs > 256 ? (double)((wgs + 255) / 256 * 256) / wgs : 1.0, chain = K / 1024.0;
    return fmax(4.7, 3.5 + fmax(1.1 * chain, 0.31 * weights * passes * uneven) + (M - 1) * fmax(0.052 * chain, 0.0125 * weights * uneven));
}

static double linear_slices_us(bool gated, int M, int K, int N)
{
    return 8.3 + (gated ? 0.62e-6 : 0.31e-6) * K * (double)N + (M > 16 ? 0.5 : 0.0);
}

static bool linear_prefers_tile(int dtype, int mode, int M, int K, int N, const FcWidePlan &wide, const FcSkinnyPlan &skinny)
{
    if (dtype != FC_BF16 || fc_knobs().lin_wide_shape >= 0 || fc_knobs().lin_ksplit > 0 || fc_knobs().lin_wgs > 0 ||
        fc_knobs().lin_no_rows)  // tuning knobs name the kernels
        return false;
    const bool gated = mode == FC_LIN_GATE_UP;
    const double weights = (gated ? 2e-6 : 1e-6) * K * (double)N;  // millions
    if (wide.kind == 1)
        return K <= 2048 && fmax(4.4, 3.2 + 0.027 * M * weights) < 0.97 * (3.5 + 0.0034 * (K < 1024 ? K : 1024));
    if (skinny.kind != 1) return false;
    return linear_tile_us(gated, M, K, N) < 0.97 * linear_slices_us(gated, M, K, N);
}

// The kernel for few outputs, one launch with every window row in every workgroup, against what the problem would take
// otherwise.  Both sides measured, weights from HBM, hidden 512 .. 18944, 256 .. 8192 outputs, 4 .. 256 rows (us, this kernel
// first):
//   up to 32 rows it takes the whole-row kernel's place (3584 x 3584 7.0 / 7.1 / 8.1 and 7.8 / 8.5 / 9.9 at 4 / 16 / 32 rows; hidden
//   512 with less than two million weights is a draw), and the tiled GEMM's except gated at hidden 4096 beyond 7168 outputs
//   (8192: 27.7 and 24.0) and where the window rows outweigh the weights (18944 x 3584, 32 rows: 36.3 and 29.9); the tile and
//   the slice-wise kernel by estimate (2048 x 4096, 32 rows 5.7 and 8.4; 8192 x 3584, 4 rows 14.9 and 13.9; 12288 x 2048
//   18.6 and 15.4; 18944 x 8192, 16 rows 52.2 and 57.9), small problems at hidden 1024 stay in the tile kernel (1024 x 1024
//   4.5 and 4.3);
//   beyond 32 rows the tiled GEMM cuts the hidden dimension of W_out and W_2, and gains where it is long or the outputs many
//   (3584 x 3584, 64 / 128 / 256 rows 9.4 / 12.1 / 16.5 and 11.3 / 13.8 / 17.7; 2048 x 2048, 64 rows 6.1 and 8.3; 5120 x 5120 18.5 and 17.2;
//   8192 x 2048, 256 rows 24.4 and 20.6; 3584 x 8192, 64 rows 17.5 and 16.8); gated layers of few outputs leave it few
//   workgroups at any hidden size (2048 x 2048, 64 rows 7.2 and 13.7; 3584 x 4096, 128 rows 20.8 and 27.2; 4096 x 6144, 48 rows 21.5
//   and 24.3; 3584 x 8192 24.4 and 23.7); and widths that are no whole slabs would go to the tile kernel (3584 x 6000,
//   40 rows 12.3 and 29.0).
static bool linear_prefers_lines(int dtype, int mode, int M, int K, int N, const FcWidePlan &wide, const FcSkinnyPlan &skinny, bool tile)
{
    if (!fc_linear_lines_cover(dtype, mode, M, K, N) || fc_knobs().lin_wide_shape >= 0 || fc_knobs().lin_ksplit > 0 ||
        fc_knobs().lin_wgs > 0 || fc_knobs().lin_no_rows)  // tuning knobs name the kernels
        return false;
    const bool gated = mode == FC_LIN_GATE_UP;
    const double weights = (gated ? 2e-6 : 1e-6) * K * (double)N;  // millions
    if (M > 32) {
        if ((K <= 1024 && tile) || (K <= 512 && (M > 64 || weights > 2.7))) return false;
        if (wide.kind == 0 && K > 1024) return true;  // else the tile kernel
        if (gated) return N <= 4096 || (N <= 6144 && K >= 3072 && M <= 48);
        if (M > 64 && weights < 2.0) return false;
        if (N > 5120) return M <= 96 && (int64_t)((M + 15) / 16) * K <= 12288;
        return K <= 4096 || (K <= 5120 && N <= 3584 && M <= 192) || (K <= 8192 && N <= 1024);
    }
    if (wide.kind == 1) return gated ? K % 4096 != 0 || N <= 7168 : K <= 8192;
    if (skinny.kind == 2) return K > 512 || weights >= 2.0;
    if (K > 8192) return (M <= 16 && N >= 5120) || skinny.kind == 0;
    const double tile_us = linear_tile_us(gated, M, K, N);
    if (K <= 1024 && tile_us <= 5.7) return false;
    const double us = 2.28 + (M + 15) / 16 * (0.2 + 0.000265 * K) + 0.28 * weights + 0.00018 * K + 0.035 * fmax(0.0, weights - 33.0);
    return us < (skinny.kind == 1 ? fmin(tile_us, linear_slices_us(gated, M, K, N)) : tile_us);
}

static fc_status linear_common(int32_t dtype, int mode, const void *x, const void *w, const void *w2,
                               const void *res, int32_t M, int32_t K, int32_t N, void *out, void *workspace,
                               size_t workspace_bytes, bool once, void *stream)
{
    fc_status st = check_dtype(dtype);
    if (st != FC_OK) return st;
    if (!x || !w || !out || (mode == FC_LIN_GATE_UP && !w2))
        return fail(FC_ERR_INVALID_ARG, "x, a weight matrix or out is NULL");
    st = check_linear_shape(M, K, N);
    if (st != FC_OK) return st;
    if (((uintptr_t)x | (uintptr_t)w | (uintptr_t)w2 | (uintptr_t)res | (uintptr_t)out | (uintptr_t)workspace) & 15)
        return fail(FC_ERR_INVALID_ARG, "pointers must be 16-byte aligned");
    static thread_local Memo<WidePlanKey, FcWidePlan> memo;  // (planning weighs a hundred tiles and parts)
    const WidePlanKey key = {workspace ? workspace_bytes : 0, dtype, mode, M, K, N, fc_knobs().version};
    const FcWidePlan wide = memo.get(key, [&] { return fc_plan_wide(dtype, mode, M, K, N, key.bytes); });
    const FcSkinnyPlan plan = fc_plan_skinny(dtype, mode, M, K, N);
    const size_t need = wide.kind == 1 ? wide.required : fc_skinny_workspace(plan);
    if (need > 0 && (!workspace || workspace_bytes < need))
        return fail(FC_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", need,
                    workspace ? workspace_bytes : (size_t)0);
    hipError_t e;
    const bool tile = linear_prefers_tile(dtype, mode, M, K, N, wide, plan);
    if (linear_prefers_lines(dtype, mode, M, K, N, wide, plan, tile))
        e = fc_launch_linear_lines(mode, x, w, w2, res, M, K, N, out, once, (hipStream_t)stream);
    else if (wide.kind == 1 && !tile)
        e = fc_launch_linear_wide(wide, mode, x, w, w2, res, M, K, N, out, workspace, once, (hipStream_t)stream);
    else if (plan.kind >= 1 && !tile)
        e = fc_launch_linear_skinny(plan, mode, x, w, w2, res, M, K, N, out, workspace, (hipStream_t)stream);
    else
        e = fc_launch_linear_tile(dtype, mode, x, w, mode == FC_LIN_GATE_UP ? w2 : res, M, K, N, out,
                                  (hipStream_t)stream);
    return e == hipSuccess ? FC_OK : hip_fail(e, "linear launch");
}

// A layer called by itself: its matrix comes round again behind those of the other layers, and the call takes it that there are four
// such matrices at least.  us without and with the hint, one matrix again and again / two in turn / four in turn: gated 3584 x 8192
// (117 MB), 32 rows 18.7 and 19.4 / 18.6 and 20.2 / 22.7 and 20.8, 128 rows 21.6 and 28.5 / 25.8 and 29.1 / 30.8 and 29.5; gated
// 3584 x 9472, 256 rows 43.4 and 49.9 / 47.1 and 49.0 / 51.4 and 49.2; 18944 x 3584 (136 MB), 32 rows 27.6 and 28.3 / 28.2 and 28.2 /
// 31.0 and 28.4.  (A program that goes over one such matrix only is the one that loses.)
static bool layer_read_once(double K, double N) { return fc_read_once(4.0 * 2.0 * K * N); }

fc_status fc_linear_residual(int32_t dtype, const void *x, const void *w, const void *residual, int32_t M,
                             int32_t K, int32_t N, void *out, void *workspace, size_t workspace_bytes,
                             void *stream)
{
    return linear_common(dtype, FC_LIN_RESIDUAL, x, w, nullptr, residual, M, K, N, out, workspace,
                         workspace_bytes, layer_read_once(K, N), stream);
}

fc_status fc_ffn_gate_up(int32_t dtype, const void *x, const void *w_gate, const void *w_up, int32_t M,
                         int32_t K, int32_t F, void *out, void *workspace, size_t workspace_bytes, void *stream)
{
    return linear_common(dtype, FC_LIN_GATE_UP, x, w_gate, w_up, nullptr, M, K, F, out, workspace,
                         workspace_bytes, layer_read_once(K, 2.0 * F), stream);
}

namespace {

// Carve-up of the whole-layer workspace for M = B * A rows (every part 256-byte aligned).
struct LayerWs {
    size_t h, q, o, x2, act, lin, attn;  // attn: last
    size_t least;                        // bytes a call must bring
    size_t lin_end, attn_end;            // where the best plans' partial sums and partial results end
};

struct LayerWsKey {
    int32_t batch, hidden, n_q_heads, n_kv_heads, head_dim, max_seq, dtype, d_ff, A, knobs;
};

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Space of the three linear layers together.
LinearSpace layer_linear_space(const fc_config &c, int32_t d_ff, int32_t M)
{
    LinearSpace all = {0, 0, 0};
    const int32_t E = c.n_q_heads * c.head_dim;
    for (const LinearSpace &l : {linear_workspace(c.dtype, M, E, c.hidden), linear_workspace(c.dtype, M, c.hidden, 2 * d_ff),
                                 linear_workspace(c.dtype, M, d_ff, c.hidden)}) {
        if (l.least > all.least) all.least = l.least;
        if (l.useful > all.useful) all.useful = l.useful;
        all.plan = all.plan << 20 | l.plan;  // (17 bits each)
    }
    return all;
}

// The activations' places; `lin` is where they end.
LayerWs layer_activations(const fc_config &c, int32_t d_ff, int32_t A)
{
    LayerWs w = {};
    const size_t es = esize_of(c.dtype);
    const size_t M = (size_t)c.batch * A, d = c.hidden, E = (size_t)c.n_q_heads * c.head_dim;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align256(bytes);
        return at;
    };
    w.h = take(M * d * es);
    w.q = take(M * E * es);
    w.o = take(M * E * es);
    w.x2 = take(M * d * es);
    w.act = take(M * (size_t)d_ff * es);
    w.lin = off;
    return w;
}

LayerWs layer_ws(const fc_config &c, int32_t d_ff, int32_t A)
{
    LayerWs w = layer_activations(c, d_ff, A);
    // The linear layers' partial sums may run on over the attention's space, which is free again by then.
    const LinearSpace lin = layer_linear_space(c, d_ff, c.batch * A);
    w.attn = w.lin + align256(lin.least);
    w.lin_end = w.lin + align256(lin.useful);
    w.least = w.attn + align256(attn_workspace(c, A, false));
    w.attn_end = w.attn + align256(attn_workspace(c, A, true));
    return w;
}

// (planning it walks every window size up to A; a thread asks for the size and then calls)
LayerWs layer_ws_of(const fc_config &c, int32_t d_ff, int32_t A)
{
    static thread_local Memo<LayerWsKey, LayerWs> memo;
    const LayerWsKey key = {c.batch, c.hidden, c.n_q_heads, c.n_kv_heads, c.head_dim, c.max_seq, c.dtype, d_ff, A, fc_knobs().version};
    return memo.get(key, [&] { return layer_ws(c, d_ff, A); });
}

// The most that a layer call of up to max_rows rows requires or makes use of.  Narrower windows may ask for more than wider ones, whose layers go
// in fewer parts: 28 / 4 heads, d_ff 18944, 256 rows require 68 MB, 257 rows 50.  Between two multiples of 64 rows the number of tiles is the same
// in every shape, so that the estimate of a number of parts is a constant and a term of rows x parts: the cheapest number does not rise
// with the rows, and where it is the same at both ends of an interval the widest window takes the most.
size_t layer_workspace_most(const fc_config &c, int32_t d_ff, int32_t max_rows)
{
    const LayerWs widest = layer_ws_of(c, d_ff, max_rows);
    const size_t attn = align256(attn_workspace(c, max_rows, false));  // at least that of any narrower window
    size_t most = widest.lin_end > widest.attn_end ? widest.lin_end : widest.attn_end;
    auto take = [&](int32_t A, const LinearSpace &lin) {
        const size_t at = layer_activations(c, d_ff, A).lin, least = at + align256(lin.least) + attn, useful = at + align256(lin.useful);
        if (least > most) most = least;
        if (useful > most) most = useful;
    };
    auto space = [&](int32_t A) { return layer_linear_space(c, d_ff, c.batch * A); };
    struct Interval {
        int32_t lo, hi;
        LinearSpace at_lo, at_hi;
    } todo[32];  // (halved each time, at most 64 windows wide)
    for (int64_t last = (int64_t)c.batch * max_rows; last >= 1;) {
        const int64_t before = last > 64 ? (last - 1) / 64 * 64 : last > 32 ? 32 : last > 16 ? 16 : 0;  // rows before + 1 .. last
        const int32_t lo = (int32_t)(before / c.batch + 1), hi = (int32_t)(last / c.batch);
        last = before;
        if (lo > hi) continue;
        // 256 compute units' partial sums of 256 x 256 are 64 MB; beyond that only the slice-wise kernel goes, which rises with the rows
        if (layer_activations(c, d_ff, hi).lin + ((size_t)64 << 20) + attn <= most) break;
        int n = 0;
        todo[n++] = Interval{lo, hi, space(lo), space(hi)};
        take(hi, todo[0].at_hi);
        while (n > 0) {
            const Interval v = todo[--n];
            if (v.at_lo.plan == v.at_hi.plan) continue;  // (the wider end is taken already)
            if (v.hi - v.lo <= 1) {
                take(v.lo, v.at_lo);
                continue;
            }
            const int32_t mid = v.lo + (v.hi - v.lo) / 2;
            const LinearSpace at_mid = space(mid);
            take(mid, at_mid);
            todo[n++] = Interval{v.lo, mid, v.at_lo, at_mid};
            todo[n++] = Interval{mid, v.hi, at_mid, v.at_hi};
        }
    }
    return most;
}

}  // namespace

size_t fc_full_layer_workspace_bytes(const fc_config *cfg, int32_t d_ff, int32_t max_rows)
{
    if (check_config(cfg) != FC_OK || d_ff < 1 || max_rows < 1 || (int64_t)max_rows * cfg->batch > (1 << 24))
        return 0;
    static thread_local Memo<LayerWsKey, size_t> memo;
    const LayerWsKey key = {cfg->batch, cfg->hidden, cfg->n_q_heads, cfg->n_kv_heads, cfg->head_dim, cfg->max_seq, cfg->dtype, d_ff, max_rows,
                            fc_knobs().version};
    return memo.get(key, [&] { return layer_workspace_most(*cfg, d_ff, max_rows); });
}

fc_status fc_full_layer_step(fc_cache *cache, int32_t layer, const fc_layer_weights *wt, const void *x,
                             int32_t win_start, int32_t A, const int32_t *pos, int32_t kv_len, void *y,
                             void *workspace, size_t workspace_bytes, void *stream)
{
    fc_status st = check_cache_layer(cache, layer);
    if (st != FC_OK) return st;
    if (!wt || !x || !y) return fail(FC_ERR_INVALID_ARG, "weights, x or y is NULL");
    if (!wt->norm1 || !wt->w_qkv || !wt->w_out || !wt->norm2 || !wt->w_gate || !wt->w_up || !wt->w_down)
        return fail(FC_ERR_INVALID_ARG, "a required weight pointer is NULL");
    if (wt->d_ff < 1 || wt->d_ff % 8 != 0) return fail(FC_ERR_INVALID_ARG, "d_ff %d must be a positive multiple of 8", wt->d_ff);
    if (!(wt->eps >= 0.0f) || !isfinite(wt->eps)) return fail(FC_ERR_INVALID_ARG, "eps must be finite and >= 0");
    if (A < 1) return fail(FC_ERR_INVALID_ARG, "A %d must be >= 1", A);
    const fc_config &c = cache->cfg;
    if ((int64_t)A * c.batch > (1 << 24)) return fail(FC_ERR_UNSUPPORTED, "batch * A exceeds 2^24 rows");
    if ((c.n_q_heads * c.head_dim) % 8 != 0) return fail(FC_ERR_UNSUPPORTED, "Hq * Dh must be a multiple of 8");
    if (!pos && (win_start < 0 || win_start > c.max_seq - A))
        return fail(FC_ERR_BOUNDS, "window [%d, %d+%d) outside the cache of %d rows", win_start, win_start, A,
                    c.max_seq);
    if (kv_len < 1 || kv_len > c.max_seq) return fail(FC_ERR_BOUNDS, "kv_len %d outside [1, %d]", kv_len, c.max_seq);
    const LayerWs w = layer_ws_of(c, wt->d_ff, A);
    if (!workspace || workspace_bytes < w.least)
        return fail(FC_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", w.least,
                    workspace ? workspace_bytes : (size_t)0);
    if ((uintptr_t)workspace & 15) return fail(FC_ERR_INVALID_ARG, "workspace must be 16-byte aligned");
    char *ws = (char *)workspace;
    const int M = c.batch * A, d = c.hidden, E = c.n_q_heads * c.head_dim;
    void *h = ws + w.h, *q = ws + w.q, *o = ws + w.o, *x2 = ws + w.x2, *act = ws + w.act;
    // (no more than what is of use, so that what a caller has to spare changes no plan, and with it no rounding)
    const size_t attn_bytes = (workspace_bytes < w.attn_end ? workspace_bytes : w.attn_end) - w.attn;
    const size_t lin_bytes = (workspace_bytes < w.lin_end ? workspace_bytes : w.lin_end) - w.lin;
    void *lin = lin_bytes ? ws + w.lin : nullptr, *attn = attn_bytes ? ws + w.attn : nullptr;

    const bool once = fc_read_once(fc_pass_bytes(c, wt->d_ff, kv_len));
    st = fc_rmsnorm(c.dtype, x, wt->norm1, wt->eps, M, d, h, stream);
    if (st == FC_OK) st = project_scatter(cache, layer, wt->d_ff, kv_len, h, wt->w_qkv, wt->b_qkv, win_start, A, pos, q, stream);
    if (st == FC_OK) st = active_attention(cache, layer, wt->d_ff, q, A, kv_len, pos, o, attn, attn_bytes, stream);
    if (st == FC_OK)
        st = linear_common(c.dtype, FC_LIN_RESIDUAL, o, wt->w_out, nullptr, x, M, E, d, x2, lin, lin_bytes, once, stream);
    if (st == FC_OK) st = fc_rmsnorm(c.dtype, x2, wt->norm2, wt->eps, M, d, h, stream);
    if (st == FC_OK)
        st = linear_common(c.dtype, FC_LIN_GATE_UP, h, wt->w_gate, wt->w_up, nullptr, M, d, wt->d_ff, act, lin, lin_bytes, once, stream);
    if (st == FC_OK)
        st = linear_common(c.dtype, FC_LIN_RESIDUAL, act, wt->w_down, nullptr, x2, M, wt->d_ff, d, y, lin, lin_bytes, once, stream);
    return st;
}

// ---------------------------------------------------------------------------------------------
// Unmasking step.

namespace {

// Carve-up of the lm-head workspace: [partial tiles of the streaming kernels][(largest, index, sum) per part and row].
struct LmHeadWs {
    FcWidePlan wide;
    FcSkinnyPlan plan;
    int parts;
    size_t tiles, am, total;
};

LmHeadWs lm_head_ws(int dtype, int M, int K, int V)
{
    LmHeadWs w;
    w.wide = fc_plan_wide(dtype, FC_LIN_VOCAB, M, K, V);  // tiled GEMM
    w.plan = fc_plan_skinny(dtype, FC_LIN_VOCAB, M, K, V);
    if (w.wide.kind == 1) w.plan.kind = 0;
    w.parts = w.wide.kind == 1 ? V / 128
                               : (w.plan.kind == 1 ? w.plan.slabs
                                                   : (w.plan.kind == 2 ? w.plan.G  // one running triple per workgroup
                                                                       : (V + FC_LMHEAD_TILE_PART - 1) / FC_LMHEAD_TILE_PART));
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align256(bytes);
        return at;
    };
    w.tiles = take(fc_skinny_workspace(w.plan));
    w.am = take((size_t)w.parts * ((M + 7) / 8 * 8) * sizeof(FcArgmax));
    w.total = off;
    return w;
}

}  // namespace

size_t fc_lm_head_workspace_bytes(int32_t dtype, int32_t M, int32_t K, int32_t V)
{
    if ((dtype != FC_F32 && dtype != FC_BF16) || M < 1 || K < 1 || V < 1 || M > (1 << 24) || V > (1 << 24)) return 0;
    return lm_head_ws(dtype, M, K, V).total;
}

fc_status fc_lm_head_argmax(int32_t dtype, const void *x, const void *w_vocab, int32_t M, int32_t K, int32_t V,
                            int32_t *tok, float *conf, void *workspace, size_t workspace_bytes, void *stream)
{
    fc_status st = check_dtype(dtype);
    if (st != FC_OK) return st;
    if (!x || !w_vocab || !tok || !conf) return fail(FC_ERR_INVALID_ARG, "x, w_vocab, tok or conf is NULL");
    if (M < 1 || K < 1 || V < 1) return fail(FC_ERR_INVALID_ARG, "M, K and V must be >= 1");
    if (K % 8 != 0) return fail(FC_ERR_UNSUPPORTED, "K %d is not a multiple of 8", K);
    if (M > (1 << 24) || V > (1 << 24)) return fail(FC_ERR_UNSUPPORTED, "M and V are limited to 2^24");
    if (((uintptr_t)x | (uintptr_t)w_vocab | (uintptr_t)workspace) & 15)
        return fail(FC_ERR_INVALID_ARG, "pointers must be 16-byte aligned");
    const LmHeadWs w = lm_head_ws(dtype, M, K, V);
    if (!workspace || workspace_bytes < w.total)
        return fail(FC_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", w.total,
                    workspace ? workspace_bytes : (size_t)0);
    char *ws = (char *)workspace;
    FcArgmaxPart am;
    am.p = (FcArgmax *)(ws + w.am);
    am.parts = w.parts;
    hipError_t e;
    const bool knobs = fc_knobs().lin_wide_shape >= 0 || fc_knobs().lin_wgs > 0 || fc_knobs().lin_no_rows;  // they name the kernels
    const int runs = knobs || w.wide.kind == 1 || w.plan.kind == 1 ? 0 : fc_lmhead_lines_parts(dtype, M, K, V, w.parts);
    const int long_runs = knobs || w.wide.kind == 1 || w.plan.kind != 2 ? 0 : fc_lmhead_runs_parts(dtype, M, K, V, w.parts);
    if (runs > 0) {
        am.parts = runs;
        e = fc_launch_lmhead_lines(x, w_vocab, M, K, V, am, (hipStream_t)stream);
    } else if (long_runs > 0) {
        am.parts = long_runs;
        e = fc_launch_lmhead_runs(x, w_vocab, M, K, V, am, (hipStream_t)stream);
    } else if (w.wide.kind == 1)
        e = fc_launch_linear_wide(w.wide, FC_LIN_VOCAB, x, w_vocab, nullptr, nullptr, M, K, V, nullptr, nullptr,
                                  fc_read_once(2.0 * K * V), (hipStream_t)stream, &am);
    else if (w.plan.kind >= 1)
        e = fc_launch_linear_skinny(w.plan, FC_LIN_VOCAB, x, w_vocab, nullptr, nullptr, M, K, V, nullptr, ws + w.tiles,
                                    (hipStream_t)stream, &am);
    else
        e = fc_launch_lmhead_tile(dtype, x, w_vocab, M, K, V, am, (hipStream_t)stream);
    if (e == hipSuccess) e = fc_launch_lmhead_reduce(am, M, tok, conf, (hipStream_t)stream);
    return e == hipSuccess ? FC_OK : hip_fail(e, "lm-head launch");
}

fc_status fc_unmask_select(const int32_t *tok, const float *conf, const int32_t *pos, int32_t win_start, int32_t B,
                           int32_t A, int32_t n_unmask, int32_t mask_id, int32_t *tokens, int32_t L,
                           int32_t *pos_next, int32_t *count_next, void *stream)
{
    if (!tok || !conf || !tokens || !pos_next || !count_next)
        return fail(FC_ERR_INVALID_ARG, "tok, conf, tokens, pos_next or count_next is NULL");
    if (B < 1 || A < 1 || L < 1 || n_unmask < 0) return fail(FC_ERR_INVALID_ARG, "B, A, L >= 1 and n_unmask >= 0 required");
    if (B > 65535) return fail(FC_ERR_UNSUPPORTED, "B is limited to 65535");
    if (A > FC_UNMASK_MAX_ROWS) return fail(FC_ERR_UNSUPPORTED, "A %d exceeds %d rows", A, FC_UNMASK_MAX_ROWS);
    if (pos == pos_next) return fail(FC_ERR_INVALID_ARG, "pos_next must not be pos");
    if (!pos && (win_start < 0 || win_start > L - A))
        return fail(FC_ERR_BOUNDS, "window [%d, %d+%d) outside the sequence of %d tokens", win_start, win_start, A, L);
    hipError_t e = fc_launch_unmask_select(tok, conf, pos, win_start, B, A, n_unmask, mask_id, tokens, L, pos_next,
                                           count_next, (hipStream_t)stream);
    return e == hipSuccess ? FC_OK : hip_fail(e, "unmask launch");
}

fc_status fc_gather_rows(int32_t dtype, const void *table, int32_t rows, int32_t width, const int32_t *idx, int32_t n,
                         void *out, void *stream)
{
    fc_status st = check_dtype(dtype);
    if (st != FC_OK) return st;
    if (!table || !idx || !out) return fail(FC_ERR_INVALID_ARG, "table, idx or out is NULL");
    if (rows < 1 || width < 1 || n < 1) return fail(FC_ERR_INVALID_ARG, "rows, width and n must be >= 1");
    const size_t row_bytes = (size_t)width * esize_of(dtype);
    if (row_bytes % 16 != 0) return fail(FC_ERR_UNSUPPORTED, "row size %zu is not a multiple of 16 bytes", row_bytes);
    if (((uintptr_t)table | (uintptr_t)out) & 15) return fail(FC_ERR_INVALID_ARG, "pointers must be 16-byte aligned");
    hipError_t e = fc_launch_gather_rows(table, rows, (int)row_bytes, idx, n, out, (hipStream_t)stream);
    return e == hipSuccess ? FC_OK : hip_fail(e, "gather launch");
}

size_t fc_guided_accept_workspace_bytes(int32_t B, int32_t A, int32_t V)
{
    if (B < 1 || A < 1 || V < 1 || B > 65535 || A > 65535) return 0;
    return fc_accept_workspace(B, A, V);
}

fc_status fc_guided_accept(const float *dlm, const float *ar, const int32_t *pos, int32_t win_start, int32_t B, int32_t A,
                           int32_t V, int32_t topk, float tau, int32_t mask_id, int32_t *tokens, int32_t L,
                           int32_t *n_accept, int32_t *pos_next, int32_t *count_next, void *workspace,
                           size_t workspace_bytes, void *stream)
{
    if (!dlm || !ar || !tokens || !n_accept || !pos_next || !count_next)
        return fail(FC_ERR_INVALID_ARG, "dlm, ar, tokens, n_accept, pos_next or count_next is NULL");
    if (B < 1 || A < 1 || V < 1 || L < 1 || topk < 1 || topk > V) return fail(FC_ERR_INVALID_ARG, "B, A, V, L >= 1 and 1 <= topk <= V required");
    if (!isfinite(tau)) return fail(FC_ERR_INVALID_ARG, "tau must be finite");
    if (topk > FC_ACCEPT_MAX_TOPK) return fail(FC_ERR_UNSUPPORTED, "topk %d exceeds %d", topk, FC_ACCEPT_MAX_TOPK);
    if (B > 65535 || A > 65535) return fail(FC_ERR_UNSUPPORTED, "B and A are limited to 65535");
    if (pos == pos_next) return fail(FC_ERR_INVALID_ARG, "pos_next must not be pos");
    if (!pos && (win_start < 0 || win_start > L - A))
        return fail(FC_ERR_BOUNDS, "window [%d, %d+%d) outside the sequence of %d tokens", win_start, win_start, A, L);
    const size_t need = fc_guided_accept_workspace_bytes(B, A, V);
    if (!workspace || workspace_bytes < need)
        return fail(FC_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", need, workspace ? workspace_bytes : (size_t)0);
    if (((uintptr_t)dlm | (uintptr_t)ar | (uintptr_t)workspace) & 15)
        return fail(FC_ERR_INVALID_ARG, "dlm, ar and workspace must be 16-byte aligned");
    hipError_t e = fc_launch_guided_accept(dlm, ar, pos, win_start, B, A, V, topk, tau, mask_id, tokens, L, n_accept,
                                           pos_next, count_next, workspace, (hipStream_t)stream);
    return e == hipSuccess ? FC_OK : hip_fail(e, "acceptance launch");
}

fc_status fc_kv_similarity(const fc_cache *cache, int32_t layer, const void *k_prev, const void *v_prev, int32_t start,
                           int32_t rows, float *sim_k, float *sim_v, void *stream)
{
    fc_status st = check_cache_layer(cache, layer);
    if (st != FC_OK) return st;
    if (!k_prev || !v_prev || !sim_k || !sim_v) return fail(FC_ERR_INVALID_ARG, "k_prev, v_prev, sim_k or sim_v is NULL");
    if (rows < 1) return fail(FC_ERR_INVALID_ARG, "rows %d must be >= 1", rows);
    if (start < 0 || start > cache->cfg.max_seq - rows)
        return fail(FC_ERR_BOUNDS, "rows [%d, %d+%d) outside the cache of %d rows", start, start, rows,
                    cache->cfg.max_seq);
    hipError_t e = fc_launch_kv_similarity(geom_of(cache), cache->cfg.dtype, layer_ptr(cache, cache->k, layer),
                                           layer_ptr(cache, cache->v, layer), k_prev, v_prev, start, rows, sim_k, sim_v,
                                           (hipStream_t)stream);
    return e == hipSuccess ? FC_OK : hip_fail(e, "similarity launch");
}

}  // extern "C"
