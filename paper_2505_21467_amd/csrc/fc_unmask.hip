// Unmasking step of a diffusion language model on the window rows (paper, section 3.1: the masked set
// M_t, the logits z_t of the masked positions, the arg-max fill of the selected subset U_t; with
// FreeCache, section 3.2.1, only the rows of the active window are evaluated).
//
// The vocabulary projection never writes its logits: every kernel that produces a part of a row's
// logits keeps (largest, its index, sum of exp(logit - largest)) of that part; k_lmhead_reduce merges
// the parts into the arg-max token and its softmax probability 1 / sum.  k_unmask_select then fills,
// per sequence, the n most confident still-masked window positions and lists the positions that stay
// masked (the next step's active rows).
#include <stdlib.h>

#include "fc_device.h"
#include "fc_internal.h"

namespace {

// Merge of the vocabulary parts: a workgroup takes a group of eight rows, whose (part, row) triples lie in one piece, 128
// parts at a time.  (One row per workgroup and triples in three [part][row] arrays touched a line per value: 256 parts
// x 32 rows 4.6 us, 1188 x 256 11.1; now 4.3 and 6.6.)
constexpr int RED_ROWS = 8, RED_GROUPS = 128, RED_WAVES = RED_ROWS * RED_GROUPS / 64;
__global__ __launch_bounds__(RED_ROWS * RED_GROUPS) void k_lmhead_reduce(FcArgmaxPart am, int M, int32_t *tok, float *conf)
{
    __shared__ float s_mx[RED_WAVES][RED_ROWS], s_sm[RED_WAVES][RED_ROWS];
    __shared__ int s_arg[RED_WAVES][RED_ROWS];
    const int tid = threadIdx.x, lane = tid & 63, row = tid % RED_ROWS, group = tid / RED_ROWS, parts = am.parts;
    const int m = blockIdx.x * RED_ROWS + row, mm = min(m, M - 1);
    float mx = -INFINITY, sm = 0.f;
    int arg = 0x7fffffff;
    auto merge_lanes = [&]() {  // over the lanes of a row
#pragma unroll
        for (int off = RED_ROWS; off < 64; off <<= 1) {
            const float mx2 = __shfl_xor(mx, off, 64), sm2 = __shfl_xor(sm, off, 64);
            const int arg2 = __shfl_xor(arg, off, 64);
            fc_argmax_merge(mx, arg, sm, mx2, arg2, sm2);
        }
    };
    constexpr int U = 4;  // parts per thread in flight at a time
    for (int base = 0; base < parts; base += RED_GROUPS * U) {
        FcArgmax v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = am.at(min(base + RED_GROUPS * u + group, parts - 1), mm);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (base + RED_GROUPS * u + group < parts) fc_argmax_merge(mx, arg, sm, v[u].mx, v[u].arg, v[u].sm);
    }
    merge_lanes();
    if (lane < RED_ROWS) {
        s_mx[tid >> 6][lane] = mx;
        s_sm[tid >> 6][lane] = sm;
        s_arg[tid >> 6][lane] = arg;
    }
    __syncthreads();
    if (tid >= 64) return;
    mx = s_mx[group][row];
    sm = s_sm[group][row];
    arg = s_arg[group][row];
#pragma unroll
    for (int w2 = 8; w2 < RED_WAVES; w2 += 8) fc_argmax_merge(mx, arg, sm, s_mx[group + w2][row], s_arg[group + w2][row], s_sm[group + w2][row]);
    merge_lanes();
    if (tid < RED_ROWS && m < M) {
        tok[m] = arg;
        conf[m] = 1.0f / sm;
    }
}

// Confidence-ranked fill, one block per sequence.  A candidate is a window row whose position is valid
// and whose token is still the mask.  Its rank is the number of candidates that come before it in the
// order (larger confidence first, then smaller row); ranks below n_unmask are filled.  The remaining
// candidates are listed in row order (ballots within the waves, their counts through LDS).  The kernel is a chain of
// latencies: position, token, rank, so everything else is fetched beside it, and windows of up to 64 rows take one wave,
// without barriers (40 rows: 4.0 us with a scan over 256 threads, now 2.8).
template <int NW>
__global__ __launch_bounds__(NW * 64) void k_unmask_select(const int32_t *__restrict__ tok, const float *__restrict__ conf,
                                                           const int32_t *__restrict__ pos, int win_start, int A,
                                                           int n_unmask, int mask_id, int32_t *tokens, int L,
                                                           int32_t *pos_next, int32_t *count_next)
{
    constexpr int NT = NW * 64;
    extern __shared__ __align__(16) unsigned char sm_raw[];
    float *s_conf = (float *)sm_raw;            // [A, rounded up to 4]; -1 marks "not a candidate" (confidences are > 0)
    __shared__ int s_count[NW];
    const int b = blockIdx.x, tid = threadIdx.x;
    int32_t *seq = tokens + (size_t)b * L;
    const size_t at = (size_t)b * A;
    auto position = [&](int a) { return pos ? pos[at + a] : win_start + a; };

    const int A4 = (A + 3) & ~3;
    int p0 = -1, t0 = 0;  // position and token of the first chunk's row
    for (int a = tid; a < A4; a += NT) {
        float c = -1.0f;
        if (a < A) {
            const int p = position(a), t = tok[at + a];
            const float cv = conf[at + a];
            const bool inside = p >= 0 && p < L;
            const int now = seq[inside ? p : 0];  // (asked for with the others, not behind a test)
            __builtin_amdgcn_sched_barrier(0);
            if (inside && now == mask_id) c = cv;
            if (a == tid) {
                p0 = p;
                t0 = t;
            }
        }
        s_conf[a] = c;
    }
    __syncthreads();

    int n = 0;  // rows listed so far
    for (int a0 = 0; a0 < A; a0 += NT) {
        const int a = a0 + tid;
        bool keep = false;  // candidate that stays masked
        int p = -1;
        if (a < A && s_conf[a] >= 0.f) {
            p = a0 ? position(a) : p0;
            const float c = s_conf[a];
            int rank = 0;
            for (int o = 0; o < A4; o += 4) {
                const float4 co = *(const float4 *)(s_conf + o);  // non-candidates hold -1 and never count
                rank += (co.x > c || (co.x == c && o < a)) ? 1 : 0;
                rank += (co.y > c || (co.y == c && o + 1 < a)) ? 1 : 0;
                rank += (co.z > c || (co.z == c && o + 2 < a)) ? 1 : 0;
                rank += (co.w > c || (co.w == c && o + 3 < a)) ? 1 : 0;
            }
            if (rank < n_unmask)
                seq[p] = a0 ? tok[at + a] : t0;
            else
                keep = true;
        }
        const unsigned long long kept = __ballot(keep);
        int before = n + __popcll(kept & ((1ull << (tid & 63)) - 1));
        if (NW > 1) {
            if ((tid & 63) == 0) s_count[tid >> 6] = __popcll(kept);
            __syncthreads();
#pragma unroll
            for (int w2 = 0; w2 < NW; ++w2) {
                if (w2 < tid >> 6) before += s_count[w2];
                n += s_count[w2];
            }
            __syncthreads();
        } else {
            n += __popcll(kept);
        }
        if (keep) pos_next[at + before] = p;
    }
    for (int a = n + tid; a < A; a += NT) pos_next[at + a] = -1;
    if (tid == 0) count_next[b] = n;
}

// -------------------------------------------------------------------------------------------------
// Guided Diffusion acceptance (paper, section 3.2.2, Algorithm 1; Top-K match and threshold tau from the
// implementation details).  A row matches if the DLM's token t is among the topk best AR entries, that is, if ar[t] is a number and
// fewer than topk AR entries come before (ar[t], t) in the order (larger value first, then smaller id).  No list of the
// topk best is needed for that:
//  - k_accept_scan cuts every still masked row's vocabulary into parts, a wave each, and keeps for every four parts the
//    best DLM entry with the AR's value there and, of the other entries, the best AR entry and the second largest AR value.
//    These are running maxima per lane, so the scan is bound by reading the logits.
//  - accept_rows (half a wave per row) merges these records and counts.  Only a record whose best AR entry, or entry at its
//    best DLM entry, comes before (ar[t], t) holds any that does, and just these if its second largest value is below ar[t];
//    with topk of them or more the row does not match.  A record is read again only where fewer are certain and its second
//    value counts or ties.
//    With parts that held the two best entries alone, ar[t] and the parts' exact counts were two more memory round trips (us,
//    32 rows x 2 x 152064: topk 2 18.0 -> 15.1, topk 8 22.3 -> 14.9; 64 rows 28.5 -> 22.8; 32 x 2 x 15999 13.2 -> 10.9).
// Sorted lists per lane, merged by rounds of arg-max, took 14.8 us for the scan of 32 rows x 2 x 152064 floats (39 MB):
// some lane of a wave updates its list at almost every step, and the whole wave pays for it.
// Then the prefix: the longest run of matching masked rows is filled (or the first masked row), the rest listed.
// Blocks of up to 64 rows do the last two in one kernel, one workgroup per sequence.
constexpr int ACC_MAXK = 8;
constexpr int ACC_PARTS = 128;      // at most, per row
constexpr int ACC_REC = 4;          // parts per record and workgroup of the scan: at most 32 records per row
constexpr int ACC_FUSED_ROWS = 64;

// (value, id) order: larger value first, then smaller id
__device__ __forceinline__ bool acc_before(float v1, int i1, float v2, int i2) { return v1 > v2 || (v1 == v2 && i1 < i2); }

struct AccRec {  // of four parts of a row; ids int max where there is no entry
    float dv;        // best DLM entry,
    int di;
    float dx;        // the AR's value there;
    float av;        // of the other entries: best AR entry
    int ai;
    float a2;        // and second largest AR value (its id is not known)
};
__device__ __forceinline__ AccRec acc_none()
{
    return AccRec{-INFINITY, 0x7fffffff, __builtin_nanf(""), -INFINITY, 0x7fffffff, -INFINITY};
}
__device__ __forceinline__ void acc_insert(AccRec &x, float v, int i)  // an AR entry (not a number: none)
{
    x.a2 = __builtin_amdgcn_fmed3f(x.av, x.a2, fmaxf(v, -INFINITY));
    if (acc_before(v, i, x.av, x.ai)) {
        x.av = v;
        x.ai = i;
    }
}
// The AR's entry at the lesser of the two DLM entries joins the others.
__device__ __forceinline__ void acc_merge(AccRec &x, const AccRec &y)
{
    const bool second = acc_before(y.dv, y.di, x.dv, x.di);
    const float v = second ? x.dx : y.dx;
    const int i = second ? x.di : y.di;
    if (second) {
        x.dv = y.dv;
        x.di = y.di;
        x.dx = y.dx;
    }
    x.a2 = fmaxf(fmaxf(x.a2, y.a2), fminf(x.av, y.av));
    if (acc_before(y.av, y.ai, x.av, x.ai)) {
        x.av = y.av;
        x.ai = y.ai;
    }
    acc_insert(x, v, i);
}

// Over the wave or each half: every lane ends with the merged record.  Neighbours within 16 lanes by DPP (once the lanes of a quad, or
// of half a row, agree, the mirror image is as good a partner as lane ^ 4 or lane ^ 8), then the halves by permlane swaps;
// through LDS (ds_bpermute) the six dependent steps cost 0.2 us more.
template <int CTRL>
__device__ __forceinline__ AccRec acc_dpp(const AccRec &x)
{
    auto mv = [](int v) { return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true); };
    return AccRec{__int_as_float(mv(__float_as_int(x.dv))), mv(x.di), __int_as_float(mv(__float_as_int(x.dx))),
                  __int_as_float(mv(__float_as_int(x.av))), mv(x.ai), __int_as_float(mv(__float_as_int(x.a2)))};
}
template <int HALF>
__device__ __forceinline__ void acc_swap(const AccRec &x, AccRec &lo, AccRec &hi)
{
    auto sw = [](unsigned v, unsigned &a, unsigned &b) {
        if constexpr (HALF == 16) {
            const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
            a = r[0];
            b = r[1];
        } else {
            const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
            a = r[0];
            b = r[1];
        }
    };
    unsigned a[6], b[6];
    const unsigned v[6] = {__float_as_uint(x.dv), (unsigned)x.di, __float_as_uint(x.dx), __float_as_uint(x.av), (unsigned)x.ai, __float_as_uint(x.a2)};
#pragma unroll
    for (int i = 0; i < 6; ++i) sw(v[i], a[i], b[i]);
    lo = AccRec{__uint_as_float(a[0]), (int)a[1], __uint_as_float(a[2]), __uint_as_float(a[3]), (int)a[4], __uint_as_float(a[5])};
    hi = AccRec{__uint_as_float(b[0]), (int)b[1], __uint_as_float(b[2]), __uint_as_float(b[3]), (int)b[4], __uint_as_float(b[5])};
}
// ALL: whole records, over 64 lanes; else only the best DLM entry and the largest AR value (in av), over 32.
template <bool ALL>
__device__ __forceinline__ void acc_reduce(AccRec &x)
{
    auto merge = [](AccRec &p, const AccRec &q) {
        if constexpr (ALL) {
            acc_merge(p, q);
        } else {
            if (acc_before(q.dv, q.di, p.dv, p.di)) {
                p.dv = q.dv;
                p.di = q.di;
                p.dx = q.dx;
            }
            p.av = fmaxf(p.av, q.av);
        }
    };
    merge(x, acc_dpp<0xB1>(x));   // quad_perm [1, 0, 3, 2]
    merge(x, acc_dpp<0x4E>(x));   // quad_perm [2, 3, 0, 1]
    merge(x, acc_dpp<0x141>(x));  // row_half_mirror
    merge(x, acc_dpp<0x140>(x));  // row_mirror
    AccRec y;
    acc_swap<16>(AccRec(x), x, y);
    merge(x, y);
    if constexpr (ALL) {
        acc_swap<32>(AccRec(x), x, y);
        merge(x, y);
    }
}

struct AccArgs {
    const float *dlm, *ar;
    const int32_t *pos;
    int32_t *tokens;
    AccRec *recs;                  // [B][A][n_recs]
    int win_start, A, V, chunk, n_parts, n_recs, topk, mask_id, L;
    float tau;
};

__device__ __forceinline__ int acc_position(const AccArgs &p, int b, int a)
{
    return p.pos ? p.pos[(size_t)b * p.A + a] : p.win_start + a;
}

// grid (records, A, B): each wave scans entries [part * chunk, (part + 1) * chunk) of row (b, a), normally in one step
// with every load in flight at once.
constexpr int ACC_LANES = 64, ACC_VEC_LOADS = 5;
static_assert(ACC_REC * ACC_LANES == 256 && ACC_PARTS / ACC_REC <= 32, "a wave per part; a lane of half a wave per record");
constexpr int ACC_STEP = ACC_LANES * 4 * ACC_VEC_LOADS;  // entries per step with 16-byte loads
template <bool VEC>
__global__ __launch_bounds__(256) void k_accept_scan(AccArgs p)
{
    const int a = blockIdx.y, b = blockIdx.z, l = threadIdx.x % ACC_LANES;
    const int wave = threadIdx.x / ACC_LANES, part = blockIdx.x * ACC_REC + wave;
    __shared__ AccRec s_rec[ACC_REC];
    const size_t at = (size_t)b * p.A + a;
    const int ps = acc_position(p, b, a);
    if (!(ps >= 0 && ps < p.L && p.tokens[(size_t)b * p.L + ps] == p.mask_id)) return;  // not a candidate: nothing to scan
    const float *zd = p.dlm + at * p.V, *za = p.ar + at * p.V;
    const int v0 = min(part, p.n_parts) * p.chunk, v1 = min(p.V, v0 + p.chunk);
    constexpr int W = VEC ? 4 : 1, U = VEC ? ACC_VEC_LOADS : 10;  // entries per lane and load; loads of each array in flight
    AccRec r = acc_none();
    for (int s0 = v0 + l * W; s0 < v1; s0 += ACC_LANES * W * U) {
        float d[U][W], x[U][W];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = min(s0 + u * ACC_LANES * W, p.V - W);  // (past the end: re-read and dropped)
            if constexpr (VEC) {
                *(float4 *)d[u] = *(const float4 *)(zd + v);
                *(float4 *)x[u] = *(const float4 *)(za + v);
            } else {
                d[u][0] = zd[v];
                x[u][0] = za[v];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < W; ++e) {
                const int v = s0 + u * ACC_LANES * W + e;
                const bool in = v < v1, best = in && acc_before(d[u][e], v, r.dv, r.di);
                const float ov = best ? r.dx : in ? x[u][e] : -INFINITY;
                const int oi = best ? r.di : in ? v : 0x7fffffff;
                if (best) {
                    r.dv = d[u][e];
                    r.di = v;
                    r.dx = x[u][e];
                }
                acc_insert(r, ov, oi);
            }
    }
    acc_reduce<true>(r);
    if (l == 0) s_rec[wave] = r;
    __syncthreads();
    if (threadIdx.x) return;
#pragma unroll
    for (int w = 1; w < ACC_REC; ++w) acc_merge(r, s_rec[w]);
    p.recs[at * p.n_recs + blockIdx.x] = r;
}

// One wave decides 2 N rows, half a wave each: rows a0 + n step + (lane >> 5).  The DLM's token, and 1 / 0 for a match or none,
// -1 for a row that is not a candidate.
template <int N>
__device__ __forceinline__ void accept_rows(const AccArgs &p, int b, int a0, int step, int lane, int (&tok)[N], int (&match)[N])
{
    AccRec rec[N];
    bool cand[N];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const int row = a0 + n * step + (lane >> 5), a = min(row, p.A - 1);
        const int ps = acc_position(p, b, a);
        const bool in = ps >= 0 && ps < p.L;
        cand[n] = p.tokens[(size_t)b * p.L + (in ? ps : 0)] == p.mask_id && in && row < p.A;
        rec[n] = (lane & 31) < p.n_recs ? p.recs[((size_t)b * p.A + a) * p.n_recs + (lane & 31)] : acc_none();
    }
#pragma unroll
    for (int n = 0; n < N; ++n) {
        AccRec all = rec[n];
        all.av = fmaxf(all.av, all.dx);
        acc_reduce<false>(all);
        const float z = all.dx;  // the AR's value of the DLM's token
        tok[n] = all.di;
        const bool want = cand[n] && (!(p.tau > 0.0f) || all.dv > p.tau * all.av);
        const bool at_dlm = want && rec[n].di != tok[n] && acc_before(rec[n].dx, rec[n].di, z, tok[n]);
        const bool ahead = want && acc_before(rec[n].av, rec[n].ai, z, tok[n]);
        const uint64_t open = __ballot(ahead && rec[n].a2 >= z), closed = __ballot(ahead) & ~open, dlm = __ballot(at_dlm);
        const int sh = lane & 32;
        int count = __builtin_popcount((uint32_t)(open >> sh)) + __builtin_popcount((uint32_t)(closed >> sh)) +
                    __builtin_popcount((uint32_t)(dlm >> sh)) + __builtin_popcount((uint32_t)(__ballot(ahead && rec[n].a2 > z) >> sh));  // certain
        const uint64_t todo = __ballot(want && (uint32_t)(open >> sh) && count < p.topk);
        if (todo) {
#pragma unroll 1
            for (int h = 0; h < 64; h += 32) {
                if (!((todo >> h) & 1)) continue;
                const float zh = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z), h));
                const int th = __builtin_amdgcn_readlane(tok[n], h);
                const float *za = p.ar + ((size_t)b * p.A + a0 + n * step + (h >> 5)) * p.V;
                int total = __builtin_popcount((uint32_t)(closed >> h)) + __builtin_popcount((uint32_t)((dlm & ~open) >> h));
                for (uint32_t w = (uint32_t)(open >> h); w && total < p.topk; w &= w - 1) {
                    const int rc = __builtin_ctz(w);
                    const int v0 = rc * ACC_REC * p.chunk, v1 = min((int64_t)p.V, (int64_t)min((rc + 1) * ACC_REC, p.n_parts) * p.chunk);
                    int c = 0;
                    for (int s0 = v0; s0 < v1; s0 += 2 * ACC_STEP) {  // half a record's loads in flight at once
                        constexpr int U = 2 * ACC_STEP / 64;
                        float x[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) x[u] = za[min(s0 + 64 * u + lane, p.V - 1)];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int v = s0 + 64 * u + lane;
                            c += v < v1 && acc_before(x[u], v, zh, th);
                        }
                    }
                    // Up to ACC_MAXK of a lane count: topk is no more, so that the decision is the same.  (A lane of a large record
                    // meets thousands.)
                    c = min(c, ACC_MAXK);
#pragma unroll
                    for (int bit = 1; bit <= ACC_MAXK; bit <<= 1) total += bit * __builtin_popcountll(__ballot(c & bit));
                }
                if (sh == h) count = total;
            }
        }
        // A NaN comes before nothing and nothing before it: counting alone would let it match.  (Token V and beyond: a DLM
        // row of NaNs, no arg-max.)
        match[n] = !cand[n] ? -1 : want && count < p.topk && z == z && tok[n] < p.V ? 1 : 0;
    }
}

// Rows of a block that is too long for the fused kernel, two to a wave.  Token and match take the place of the row's first
// record, which this wave alone has read.
__global__ __launch_bounds__(64) void k_accept_rowmerge(AccArgs p)
{
    const int b = blockIdx.y;
    int a = 2 * blockIdx.x, tok[1], match[1];
    accept_rows<1>(p, b, a, 1, threadIdx.x, tok, match);
    if (threadIdx.x % 32 == 0 && a + (int)threadIdx.x / 32 < p.A) {
        a += threadIdx.x / 32;
        int32_t *row = (int32_t *)(p.recs + ((size_t)b * p.A + a) * p.n_recs);
        row[0] = tok[0];
        row[1] = match[0];
    }
}

// Blocks of at most 64 rows: one workgroup per sequence, 2 N rows per wave; its first wave, a lane per row, finds the prefix.
template <int N>
__global__ __launch_bounds__(1024) void k_accept_block(AccArgs p, int32_t *n_accept, int32_t *pos_next, int32_t *count_next)
{
    __shared__ int s_tok[ACC_FUSED_ROWS], s_match[ACC_FUSED_ROWS];
    const int b = blockIdx.x, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_waves = blockDim.x >> 6;
    int tok[N], match[N];
    accept_rows<N>(p, b, 2 * wave, 2 * n_waves, lane, tok, match);
    if ((lane & 31) == 0) {
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int a = 2 * wave + n * 2 * n_waves + (lane >> 5);
            if (a < p.A) {
                s_tok[a] = tok[n];
                s_match[a] = match[n];
            }
        }
    }
    __syncthreads();
    if (wave) return;
    const bool row = lane < p.A;
    const int mt = row ? s_match[lane] : -1;
    const uint64_t masked = __ballot(mt >= 0), missed = __ballot(mt == 0);
    const int m = __builtin_popcountll(masked);
    const int k = missed ? __builtin_popcountll(masked & ((missed & -missed) - 1)) : m;  // longest matching prefix
    const int n = m == 0 ? 0 : (k > 0 ? k : 1);
    const int j = __builtin_popcountll(masked & (((uint64_t)1 << lane) - 1));           // index among the masked rows
    if (mt >= 0) {
        const int ps = acc_position(p, b, lane);
        if (j < n) p.tokens[(size_t)b * p.L + ps] = s_tok[lane];
        else pos_next[(size_t)b * p.A + (j - n)] = ps;
    }
    if (row && lane >= m - n) pos_next[(size_t)b * p.A + lane] = -1;
    if (lane == 0) {
        n_accept[b] = n;
        count_next[b] = m - n;
    }
}

// Prefix of a longer block, one workgroup per sequence over the rows' results.
__global__ __launch_bounds__(256) void k_accept_seq(const int32_t *__restrict__ rows, int stride,
                                                    const int32_t *__restrict__ pos, int win_start, int A,
                                                    int32_t *tokens, int L, int32_t *n_accept, int32_t *pos_next,
                                                    int32_t *count_next)
{
    __shared__ int s_scan[256];
    __shared__ int s_base, s_first_miss;
    const int b = blockIdx.x, tid = threadIdx.x;
    int32_t *seq = tokens + (size_t)b * L;
    auto position = [&](int a) { return pos ? pos[(size_t)b * A + a] : win_start + a; };
    if (tid == 0) {
        s_base = 0;
        s_first_miss = 0x7fffffff;
    }
    __syncthreads();
    // pass 1: index j of every masked row among the masked rows; the first j that does not match
    for (int a0 = 0; a0 < A; a0 += 256) {
        const int a = a0 + tid;
        const int mt = a < A ? rows[((size_t)b * A + a) * stride + 1] : -1;
        s_scan[tid] = mt >= 0 ? 1 : 0;
        __syncthreads();
        for (int off = 1; off < 256; off <<= 1) {
            const int v = tid >= off ? s_scan[tid - off] : 0;
            __syncthreads();
            s_scan[tid] += v;
            __syncthreads();
        }
        if (mt == 0) atomicMin(&s_first_miss, s_base + s_scan[tid] - 1);
        __syncthreads();
        if (tid == 255) s_base += s_scan[255];
        __syncthreads();
    }
    const int m = s_base;                                  // masked rows
    const int k = min(s_first_miss, m);                    // longest matching prefix
    const int n = m == 0 ? 0 : (k > 0 ? k : 1);
    __syncthreads();
    if (tid == 0) s_base = 0;
    __syncthreads();
    // pass 2: fill the first n masked rows, list the others
    for (int a0 = 0; a0 < A; a0 += 256) {
        const int a = a0 + tid;
        const int mt = a < A ? rows[((size_t)b * A + a) * stride + 1] : -1;
        s_scan[tid] = mt >= 0 ? 1 : 0;
        __syncthreads();
        for (int off = 1; off < 256; off <<= 1) {
            const int v = tid >= off ? s_scan[tid - off] : 0;
            __syncthreads();
            s_scan[tid] += v;
            __syncthreads();
        }
        if (mt >= 0) {
            const int j = s_base + s_scan[tid] - 1;
            if (j < n)
                seq[position(a)] = rows[((size_t)b * A + a) * stride];
            else
                pos_next[(size_t)b * A + (j - n)] = position(a);
        }
        __syncthreads();
        if (tid == 255) s_base += s_scan[255];
        __syncthreads();
    }
    for (int a = m - n + tid; a < A; a += 256) pos_next[(size_t)b * A + a] = -1;
    if (tid == 0) {
        n_accept[b] = n;
        count_next[b] = m - n;
    }
}

// Row gather in 16-byte pieces: out[i] = table[idx[i]], zeros for a negative or too large index.
__global__ __launch_bounds__(256) void k_gather_rows(const uint4 *__restrict__ table, int64_t R, int pieces,
                                                     const int32_t *__restrict__ idx, uint4 *__restrict__ out)
{
    const int64_t i = blockIdx.x;
    const int32_t r = idx[i];
    const bool ok = r >= 0 && r < R;
    for (int c = threadIdx.x; c < pieces; c += 256)
        out[i * pieces + c] = ok ? table[(int64_t)r * pieces + c] : make_uint4(0, 0, 0, 0);
}

}  // namespace

// Parts a row's vocabulary is cut into: one step of the scan each (32 rows x 152064: 11 us for 39 MB),
// at most two per lane of the merging wave; chunks of whole float4s.
int fc_accept_parts(int B, int A, int V)
{
    int64_t parts = (V + ACC_STEP - 1) / ACC_STEP;
    if (fc_knobs().accept_wgs > 0) parts = fc_knobs().accept_wgs / ((int64_t)B * A);  // tuning knob
    if (parts > ACC_PARTS) parts = ACC_PARTS;
    if (parts > V) parts = V;
    if (parts < 1) parts = 1;
    return (int)parts;
}

size_t fc_accept_workspace(int B, int A, int V)
{
    // (a record of 24 bytes per four parts is at most this much)
    return (size_t)B * A * (8 + 16 * (size_t)fc_accept_parts(B, A, V));
}

hipError_t fc_launch_guided_accept(const float *dlm, const float *ar, const int32_t *pos, int win_start, int B, int A,
                                   int V, int topk, float tau, int mask_id, int32_t *tokens, int L, int32_t *n_accept,
                                   int32_t *pos_next, int32_t *count_next, void *workspace, hipStream_t s)
{
    if (topk < 1 || topk > ACC_MAXK || !workspace) return hipErrorInvalidValue;
    AccArgs p;
    p.dlm = dlm;
    p.ar = ar;
    p.pos = pos;
    p.tokens = tokens;
    p.win_start = win_start;
    p.A = A;
    p.V = V;
    p.n_parts = fc_accept_parts(B, A, V);
    p.chunk = (((V + p.n_parts - 1) / p.n_parts) + 3) & ~3;
    p.topk = topk;
    p.mask_id = mask_id;
    p.L = L;
    p.tau = tau;
    p.recs = (AccRec *)workspace;
    p.n_recs = (p.n_parts + ACC_REC - 1) / ACC_REC;
    const dim3 grid((unsigned)p.n_recs, (unsigned)A, (unsigned)B);
    // rows of V floats are 16-byte aligned when V is a multiple of 4
    if ((V & 3) == 0) k_accept_scan<true><<<grid, dim3(256), 0, s>>>(p);
    else k_accept_scan<false><<<grid, dim3(256), 0, s>>>(p);
    if (A <= 32) k_accept_block<1><<<dim3((unsigned)B), dim3((unsigned)(A + 1) / 2 * 64), 0, s>>>(p, n_accept, pos_next, count_next);
    else if (A <= ACC_FUSED_ROWS) k_accept_block<2><<<dim3((unsigned)B), dim3(1024), 0, s>>>(p, n_accept, pos_next, count_next);
    else {
        k_accept_rowmerge<<<dim3((unsigned)(A + 1) / 2, (unsigned)B), dim3(64), 0, s>>>(p);
        k_accept_seq<<<dim3((unsigned)B), dim3(256), 0, s>>>((const int32_t *)p.recs, p.n_recs * (int)(sizeof(AccRec) / 4), pos, win_start,
                                                             A, tokens, L, n_accept, pos_next, count_next);
    }
    return hipGetLastError();
}

hipError_t fc_launch_gather_rows(const void *table, int64_t R, int row_bytes, const int32_t *idx, int64_t n, void *out,
                                 hipStream_t s)
{
    k_gather_rows<<<dim3((unsigned)n), dim3(256), 0, s>>>((const uint4 *)table, R, row_bytes / 16, idx, (uint4 *)out);
    return hipGetLastError();
}

hipError_t fc_launch_lmhead_reduce(const FcArgmaxPart &am, int M, int32_t *tok, float *conf,
                                   hipStream_t s)
{
    k_lmhead_reduce<<<dim3((unsigned)((M + RED_ROWS - 1) / RED_ROWS)), dim3(RED_ROWS * RED_GROUPS), 0, s>>>(am, M, tok, conf);
    return hipGetLastError();
}

hipError_t fc_launch_unmask_select(const int32_t *tok, const float *conf, const int32_t *pos, int win_start,
                                   int B, int A, int n_unmask, int mask_id, int32_t *tokens, int L,
                                   int32_t *pos_next, int32_t *count_next, hipStream_t s)
{
    if (A > FC_UNMASK_MAX_ROWS) return hipErrorInvalidValue;
    const size_t lds = (size_t)((A + 3) & ~3) * sizeof(float);
    if (A <= 64)
        k_unmask_select<1><<<dim3((unsigned)B), dim3(64), lds, s>>>(tok, conf, pos, win_start, A, n_unmask, mask_id, tokens,
                                                                     L, pos_next, count_next);
    else
        k_unmask_select<4><<<dim3((unsigned)B), dim3(256), lds, s>>>(tok, conf, pos, win_start, A, n_unmask, mask_id, tokens,
                                                                      L, pos_next, count_next);
    return hipGetLastError();
}
