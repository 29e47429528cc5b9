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
            if (p >= 0 && p < L && seq[p] == mask_id) c = cv;
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
//  - k_accept_scan cuts every still masked row's vocabulary into parts, 64 lanes each, and finds each part's best DLM and
//    best AR entry: two running maxima per lane, so the scan is bound by reading the logits;
//  - accept_rows (a wave per row) merges the parts, fetches ar[t], and counts.  Only parts whose best AR entry comes
//    before (ar[t], t) hold any entry that does; with topk of them or more the row does not match, and else
//    those few parts (usually none or one) are read again and counted exactly.
// Sorted lists per lane, merged by rounds of arg-max, took 14.8 us for the scan of 32 rows x 2 x 152064 floats (39 MB):
// some lane of a wave updates its list at almost every step, and the whole wave pays for it.
// Then the prefix: the longest run of matching masked rows is filled (or the first masked row), the rest listed.
// Blocks of up to 64 rows do the last two in one kernel, one workgroup per sequence.
constexpr int ACC_MAXK = 8;
constexpr int ACC_PARTS = 128;      // at most, per row: two per lane of the merging wave
constexpr int ACC_FUSED_ROWS = 64;

// (value, id) order: larger value first, then smaller id
__device__ __forceinline__ bool acc_before(float v1, int i1, float v2, int i2) { return v1 > v2 || (v1 == v2 && i1 < i2); }

struct AccPart {  // best entries of one part of a row; (-inf, int max) where there is none
    float dv;
    int di;
    float av;
    int ai;
};

struct AccArgs {
    const float *dlm, *ar;
    const int32_t *pos;
    int32_t *tokens;
    AccPart *parts;                // [B][A][n_parts]
    int win_start, A, V, chunk, n_parts, topk, mask_id, L;
    float tau;
};

__device__ __forceinline__ int acc_position(const AccArgs &p, int b, int a)
{
    return p.pos ? p.pos[(size_t)b * p.A + a] : p.win_start + a;
}

// grid (parts / 4, A, B): 64 lanes scan entries [part * chunk, (part + 1) * chunk) of row (b, a), normally in one step
// with every load in flight at once.
constexpr int ACC_LANES = 64, ACC_VEC_LOADS = 5;
constexpr int ACC_STEP = ACC_LANES * 4 * ACC_VEC_LOADS;  // entries per step with 16-byte loads
template <bool VEC>
__global__ __launch_bounds__(256) void k_accept_scan(AccArgs p)
{
    const int a = blockIdx.y, b = blockIdx.z, l = threadIdx.x % ACC_LANES;
    const int part = blockIdx.x * (256 / ACC_LANES) + threadIdx.x / ACC_LANES;
    const size_t at = (size_t)b * p.A + a;
    const int ps = acc_position(p, b, a);
    if (!(ps >= 0 && ps < p.L && p.tokens[(size_t)b * p.L + ps] == p.mask_id)) return;  // not a candidate: nothing to scan
    const float *zd = p.dlm + at * p.V, *za = p.ar + at * p.V;
    const int v0 = min(part, p.n_parts) * p.chunk, v1 = min(p.V, v0 + p.chunk);
    constexpr int W = VEC ? 4 : 1, U = VEC ? ACC_VEC_LOADS : 10;  // entries per lane and load; loads of each array in flight
    float dv = -INFINITY, av = -INFINITY;
    int di = 0x7fffffff, ai = 0x7fffffff;
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
                if (v < v1 && acc_before(d[u][e], v, dv, di)) {
                    dv = d[u][e];
                    di = v;
                }
                if (v < v1 && acc_before(x[u][e], v, av, ai)) {
                    av = x[u][e];
                    ai = v;
                }
            }
    }
#pragma unroll
    for (int off = ACC_LANES / 2; off > 0; off >>= 1) {
        const float d2 = __shfl_xor(dv, off, 64), a2 = __shfl_xor(av, off, 64);
        const int i2 = __shfl_xor(di, off, 64), j2 = __shfl_xor(ai, off, 64);
        if (acc_before(d2, i2, dv, di)) {
            dv = d2;
            di = i2;
        }
        if (acc_before(a2, j2, av, ai)) {
            av = a2;
            ai = j2;
        }
    }
    if (l == 0 && part < p.n_parts) p.parts[at * p.n_parts + part] = AccPart{dv, di, av, ai};
}

// One wave decides rows a0, a0 + step, .. (N of them at most) of sequence b: the DLM's token, and 1 / 0 for a match or
// none, -1 for a row that is not a candidate.  The rows' memory round trips run together.
template <int N>
__device__ __forceinline__ void accept_rows(const AccArgs &p, int b, int a0, int step, int lane, int (&tok)[N], int (&match)[N])
{
    AccPart pt[N][ACC_PARTS / 64];
    float z[N], zmax[N];
    bool cand[N];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const int a = min(a0 + n * step, p.A - 1);
        const int ps = acc_position(p, b, a);
        const bool in = ps >= 0 && ps < p.L;
        cand[n] = p.tokens[(size_t)b * p.L + (in ? ps : 0)] == p.mask_id && in && a0 + n * step < p.A;
#pragma unroll
        for (int g = 0; g < ACC_PARTS / 64; ++g)
            pt[n][g] = 64 * g + lane < p.n_parts ? p.parts[((size_t)b * p.A + a) * p.n_parts + 64 * g + lane]
                                                 : AccPart{-INFINITY, 0x7fffffff, -INFINITY, 0x7fffffff};
    }
#pragma unroll
    for (int n = 0; n < N; ++n) {
        float dv = pt[n][0].dv;
        int di = pt[n][0].di;
        float am = pt[n][0].av;
#pragma unroll
        for (int g = 1; g < ACC_PARTS / 64; ++g) {
            if (acc_before(pt[n][g].dv, pt[n][g].di, dv, di)) {
                dv = pt[n][g].dv;
                di = pt[n][g].di;
            }
            am = fmaxf(am, pt[n][g].av);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const float v2 = __shfl_xor(dv, off, 64);
            const int i2 = __shfl_xor(di, off, 64);
            am = fmaxf(am, __shfl_xor(am, off, 64));
            if (acc_before(v2, i2, dv, di)) {
                dv = v2;
                di = i2;
            }
        }
        tok[n] = di;
        zmax[n] = am;
        match[n] = !cand[n] ? -1 : (!(p.tau > 0.0f) || dv > p.tau * am) ? 1 : 0;
        // the AR's value of the DLM's token (rows that are no candidates hold anything: stay inside the row)
        z[n] = p.ar[((size_t)b * p.A + min(a0 + n * step, p.A - 1)) * p.V + (di >= 0 && di < p.V ? di : 0)];
    }
#pragma unroll
    for (int n = 0; n < N; ++n) {
        if (match[n] != 1) continue;  // wave-uniform
        uint64_t ahead[ACC_PARTS / 64];
        int count = 0;
#pragma unroll
        for (int g = 0; g < ACC_PARTS / 64; ++g) {
            ahead[g] = __ballot(acc_before(pt[n][g].av, pt[n][g].ai, z[n], tok[n]));
            count += __builtin_popcountll(ahead[g]);
        }
        if (count > 0 && count < p.topk) {
            // at least one entry in each of these parts: count them all
            const float *za = p.ar + ((size_t)b * p.A + a0 + n * step) * p.V;
            count = 0;
#pragma unroll
            for (int g = 0; g < ACC_PARTS / 64; ++g)
                for (uint64_t w = ahead[g]; w && count < p.topk; w &= w - 1) {
                    const int v0 = (64 * g + __builtin_ctzll(w)) * p.chunk, v1 = min(p.V, v0 + p.chunk);
                    for (int v = v0; v < v1; v += ACC_STEP) {  // a part is one step: every load in flight at once
                        float x[ACC_STEP / 64];
#pragma unroll
                        for (int u = 0; u < ACC_STEP / 64; ++u) x[u] = za[min(v + 64 * u + lane, p.V - 1)];
#pragma unroll
                        for (int u = 0; u < ACC_STEP / 64; ++u) {
                            const int vv = v + 64 * u + lane;
                            count += __builtin_popcountll(__ballot(vv < v1 && acc_before(x[u], vv, z[n], tok[n])));
                        }
                    }
                }
        }
        // A NaN comes before nothing and nothing before it: counting alone would let it match.  (Token V and beyond: a DLM
        // row of NaNs, no arg-max.)  Not an early `continue` at the top: hipcc 7.2 then dropped the assignment here.
        if (count >= p.topk || !(z[n] == z[n]) || tok[n] >= p.V) match[n] = 0;
    }
}

// Rows of a block that is too long for the fused kernel: one wave per row.
__global__ __launch_bounds__(64) void k_accept_rowmerge(AccArgs p, int32_t *row_tok, int32_t *row_match)
{
    const int a = blockIdx.x, b = blockIdx.y;
    int tok[1], match[1];
    accept_rows<1>(p, b, a, 1, threadIdx.x, tok, match);
    if (threadIdx.x == 0) {
        row_tok[(size_t)b * p.A + a] = tok[0];
        row_match[(size_t)b * p.A + a] = match[0];
    }
}

// Blocks of at most 64 rows: one workgroup per sequence, N rows per wave; its first wave, a lane per row, finds the prefix.
template <int N>
__global__ __launch_bounds__(1024) void k_accept_block(AccArgs p, int32_t *n_accept, int32_t *pos_next, int32_t *count_next)
{
    __shared__ int s_tok[ACC_FUSED_ROWS], s_match[ACC_FUSED_ROWS];
    const int b = blockIdx.x, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_waves = blockDim.x >> 6;
    int tok[N], match[N];
    accept_rows<N>(p, b, wave, n_waves, lane, tok, match);
    if (lane == 0) {
#pragma unroll
        for (int n = 0; n < N; ++n)
            if (wave + n * n_waves < p.A) {
                s_tok[wave + n * n_waves] = tok[n];
                s_match[wave + n * n_waves] = match[n];
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
__global__ __launch_bounds__(256) void k_accept_seq(const int32_t *__restrict__ row_tok, const int32_t *__restrict__ row_match,
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
        const int mt = a < A ? row_match[(size_t)b * A + a] : -1;
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
        const int mt = a < A ? row_match[(size_t)b * A + a] : -1;
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
                seq[position(a)] = row_tok[(size_t)b * A + a];
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
    return (size_t)2 * B * A * sizeof(int32_t) + (size_t)B * A * fc_accept_parts(B, A, V) * sizeof(AccPart);
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
    p.parts = (AccPart *)workspace;
    int32_t *row_tok = (int32_t *)(p.parts + (size_t)B * A * p.n_parts), *row_match = row_tok + (size_t)B * A;
    const dim3 grid((unsigned)((p.n_parts + 256 / ACC_LANES - 1) / (256 / ACC_LANES)), (unsigned)A, (unsigned)B);
    // rows of V floats are 16-byte aligned when V is a multiple of 4
    if ((V & 3) == 0) k_accept_scan<true><<<grid, dim3(256), 0, s>>>(p);
    else k_accept_scan<false><<<grid, dim3(256), 0, s>>>(p);
    if (A <= 16) k_accept_block<1><<<dim3((unsigned)B), dim3((unsigned)A * 64), 0, s>>>(p, n_accept, pos_next, count_next);
    else if (A <= 32) k_accept_block<2><<<dim3((unsigned)B), dim3(1024), 0, s>>>(p, n_accept, pos_next, count_next);
    else if (A <= ACC_FUSED_ROWS) k_accept_block<4><<<dim3((unsigned)B), dim3(1024), 0, s>>>(p, n_accept, pos_next, count_next);
    else {
        k_accept_rowmerge<<<dim3((unsigned)A, (unsigned)B), dim3(64), 0, s>>>(p, row_tok, row_match);
        k_accept_seq<<<dim3((unsigned)B), dim3(256), 0, s>>>(row_tok, row_match, pos, win_start, A, tokens, L, n_accept,
                                                             pos_next, count_next);
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
