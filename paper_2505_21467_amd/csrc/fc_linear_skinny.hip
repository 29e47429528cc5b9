// Weight-streaming linear layers for short windows (bf16, at most 32 rows per pass): the output
// projection and the two feed-forward matrices of the layer evaluated on the window rows only
// (paper, Table 1, rows "Output projection", "FFN W_1", "FFN W_2" with the row count L replaced by
// the window size A).
//
// With a few dozen rows the product Y^T = W X^T is bound by reading W once from HBM.  Three kernels:
// the slice-wise one described here, for any hidden size that is a multiple of 512, a whole-row
// one (k_linear_rows, further down) for the hidden sizes whose X block fits in registers, and one for layers
// of few outputs (k_linear_lines).  The weight
// matrix is cut into work items of 128 rows x KSL hidden elements (every row piece is 1 KB, or 512 B,
// of contiguous memory); the items, ordered row slab by row slab, are dealt out in equal contiguous
// runs to one workgroup per compute unit, so the matrix streams once, evenly, whatever its shape.
// Inside an item the eight waves own 16 weight rows each and load them straight into the operand
// registers of v_mfma_f32_16x16x32_bf16 (8 consecutive k per lane); the matching slice of X goes
// through LDS (direct-to-LDS loads, swizzled) and is shared by the waves.  Loads of item i+1 are
// issued before the multiplies of item i.
//
// A run of items may start and end inside a row slab, so every (slab, workgroup) pair that meet
// writes an fp32 partial tile; a second kernel sums a slab's partial tiles (a kernel boundary is
// the only cross-workgroup ordering used) and applies the epilogue: residual add, or the SiLU gate.
// For the gated W_1 a slab holds 64 rows of the gate matrix and the same 64 rows of the up matrix,
// laid out so that g and u of one output sit in lanes 32 apart of the same accumulator register.
#include <stdlib.h>
#include <string.h>

#include <type_traits>

#include "fc_device.h"
#include "fc_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

struct LinArgs {
    const uint16_t *X;    // [M][K]
    const uint16_t *W;    // [N][K]  (gate matrix in gated mode)
    const uint16_t *W2;   // up matrix [N][K] in gated mode
    const uint16_t *res;  // [M][N] or nullptr
    uint16_t *out;        // [M][N]
    FcArgmaxPart am;      // vocabulary mode: per (slab, row) running maximum, its index, sum of exponentials
    float *partials;      // [m chunk][slab][maxseg][wave][mt][4][64]
    int M, K, N;          // N = output columns
    int S, T, G, maxseg, slabs;
    int wave_bytes;       // k_linear_lines: LDS of a wave,
    uint32_t div_grid;    // reciprocal of the grid,
    bool once;            // weights with the non-temporal hint
};


__device__ __forceinline__ bf16x8 ld8(const uint16_t *p)
{
    union { uint4 u; bf16x8 v; } x;
    x.u = *(const uint4 *)p;
    return x.v;
}

__device__ __forceinline__ float swap32(float v)
{
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return (threadIdx.x & 32) ? __uint_as_float(r[0]) : __uint_as_float(r[1]);
}

// Workgroup that owns unit u when U units are dealt to G workgroups as runs
// [floor(w U / G), floor((w + 1) U / G)).  A unit is one k-step (32 hidden elements) of one slab.
__host__ __device__ __forceinline__ int owner_of(int64_t u, int64_t U, int G)
{
    return (int)(((u + 1) * G - 1) / U);
}

template <int MT, int KSL, int MODE>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(KSL >= 512 ? 2 : 4, KSL >= 512 ? 2 : 4))) void k_linear_stream(LinArgs p)
{
    constexpr int KS = KSL / 32;        // k-steps of 32 per item
    constexpr int ROWB = KSL * 2;       // bytes of one X row of a slice
    constexpr int RPL = 1024 / ROWB;    // X rows per wave-wide 1 KB load
    constexpr int NLD = 16 * MT / RPL / 8;
    static_assert(NLD >= 1, "slice too narrow for this row count");
    __shared__ __align__(1024) unsigned char xs[2][16 * MT * ROWB];

    const int wg = blockIdx.x, m0 = blockIdx.y * 32;
    // this workgroup's run of k-steps [ulo, uhi): whole items except possibly the first and the last
    const int64_t U = (int64_t)p.T * KS;
    const int64_t ulo = (int64_t)wg * U / p.G, uhi = ((int64_t)wg + 1) * U / p.G;
    const int lo = (int)(ulo / KS), hi = (int)((uhi + KS - 1) / KS);
    const int s_first = (int)(ulo - (int64_t)lo * KS);        // first k-step of item lo
    const int s_last = (int)(uhi - (int64_t)(hi - 1) * KS);   // end of the k-steps of item hi - 1
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho = lane & 15, q = lane >> 4;

    auto issue = [&](int item, bf16x8(&wf)[KS], unsigned char *xb) {
        const int slab = item / p.S, sl = item - slab * p.S;
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int ld = wave * NLD + i;
            const int mrow = ld * RPL + lane / (64 / RPL);
            const int c = (lane % (64 / RPL)) ^ (mrow & 15);  // chunk c of row m is stored at c ^ (m & 15)
            const int mg = min(m0 + mrow, p.M - 1);            // padding rows read a valid row
            fc_load_lds16(p.X + (size_t)mg * p.K + (size_t)sl * KSL + c * 8, xb + ld * 1024);
        }
        const uint16_t *wrow;
        if (MODE == FC_LIN_GATE_UP)
            wrow = (rho < 8 ? p.W : p.W2) + (size_t)(slab * 64 + wave * 8 + (rho & 7)) * p.K;
        else
            wrow = p.W + (size_t)(slab * 128 + wave * 16 + rho) * p.K;
        wrow += (size_t)sl * KSL + 8 * q;
        const int sa = item == lo ? s_first : 0, sb = item == hi - 1 ? s_last : KS;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (s >= sa && s < sb)
                wf[s] = ld8(wrow + 32 * s);
            else
                wf[s] = bf16x8{};  // k-steps of a neighbouring run: contribute nothing
        }
    };

    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto compute = [&](const bf16x8(&wf)[KS], const unsigned char *xb) {
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int m = 16 * mt + rho;
                const bf16x8 xf = *(const bf16x8 *)(xb + m * ROWB + (((4 * s + q) ^ (m & 15)) << 4));
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s], xf, acc[mt], 0, 0, 0);
            }
    };

    // hand the partial tile over when the run leaves the slab (or ends)
    auto tail = [&](int item) {
        if (item + 1 < hi && (item + 1) % p.S != 0) return;
        const int slab = item / p.S;
        const int seg = wg - owner_of((int64_t)slab * p.S * KS, U, p.G);
        float *part = p.partials +
                      ((((size_t)blockIdx.y * p.slabs + slab) * p.maxseg + seg) * 8 + wave) * (MT * 256);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                part[mt * 256 + r * 64 + lane] = acc[mt][r];
                acc[mt][r] = 0.f;
            }
    };

    if (ulo >= uhi) return;
    bf16x8 wa[KS], wb[KS];
    issue(lo, wa, xs[0]);
    int item = lo;
    for (;;) {
        __syncthreads();  // the loads of `item` have landed; every wave is done with the other buffers
        if (item + 1 < hi) issue(item + 1, wb, xs[1]);
        compute(wa, xs[0]);
        tail(item);
        if (++item >= hi) break;
        __syncthreads();
        if (item + 1 < hi) issue(item + 1, wa, xs[0]);
        compute(wb, xs[1]);
        tail(item);
        if (++item >= hi) break;
    }
}

// Sum of a slab's partial tiles + epilogue; one wave per (slab, 16-row tile of W, m chunk, 16 rows of X).  One memory
// round trip long where a slab met at most twelve runs, whose partial tiles are then all in flight (28 slabs,
// hidden 18944, 32 rows: 4.6 us with both row tiles in one wave and four in flight, now 4.0).
template <int MT, int KSL, int MODE>
__global__ __launch_bounds__(64) void k_linear_finish(LinArgs p)
{
    constexpr int KS = KSL / 32, SEGS = 12;
    const int64_t U = (int64_t)p.T * KS;
    const int slab = blockIdx.x >> 3, wave = blockIdx.x & 7, mt = blockIdx.z;
    const int lane = threadIdx.x, rho = lane & 15, q = lane >> 4;
    const int m = blockIdx.y * 32 + 16 * mt + rho;
    const bool mvalid = m < p.M;
    const int first = owner_of((int64_t)slab * p.S * KS, U, p.G);
    const int nseg = owner_of((int64_t)(slab + 1) * p.S * KS - 1, U, p.G) - first + 1;
    const float *base = p.partials + ((((size_t)blockIdx.y * p.slabs + slab) * p.maxseg) * 8 + wave) * (MT * 256) + mt * 256 + lane;
    const size_t seg_stride = (size_t)8 * MT * 256;

    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    uint2 rv = make_uint2(0, 0);
    for (int s0 = 0; s0 < nseg; s0 += SEGS) {
        float v[SEGS][4];
#pragma unroll
        for (int u = 0; u < SEGS; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[u][r] = base[(size_t)min(s0 + u, nseg - 1) * seg_stride + r * 64];
        if (MODE == FC_LIN_RESIDUAL && s0 == 0 && p.res && mvalid)
            rv = *(const uint2 *)(p.res + (size_t)m * p.N + slab * 128 + wave * 16 + 4 * q);
#pragma unroll
        for (int u = 0; u < SEGS; ++u)
            if (s0 + u < nseg) {
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r] += v[u][r];
            }
    }

    float y[4];
    int n;
    if (MODE == FC_LIN_GATE_UP) {
        // lanes q = 0, 1 hold the gate products of outputs 4q + r, lanes q = 2, 3 the up products
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float other = swap32(acc[r]);
            y[r] = acc[r] / (1.0f + expf(-acc[r])) * other;
        }
        if (!mvalid || q >= 2) return;
        n = slab * 64 + wave * 8 + 4 * q;
    } else {
        if (!mvalid) return;
        n = slab * 128 + wave * 16 + 4 * q;
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = acc[r];
        if (p.res) {
            y[0] += __uint_as_float(rv.x << 16);
            y[1] += __uint_as_float(rv.x & 0xffff0000u);
            y[2] += __uint_as_float(rv.y << 16);
            y[3] += __uint_as_float(rv.y & 0xffff0000u);
        }
    }
    uint2 w;
    w.x = (uint32_t)fc_bf16_bits(y[0]) | ((uint32_t)fc_bf16_bits(y[1]) << 16);
    w.y = (uint32_t)fc_bf16_bits(y[2]) | ((uint32_t)fc_bf16_bits(y[3]) << 16);
    *(uint2 *)(p.out + (size_t)m * p.N + n) = w;
}

// Vocabulary mode (the unmasking step, section 3.1): the outputs of a slab are 128 logits per row, of
// which only the largest, its index and the sum of exp(logit - largest) are kept, per (slab, row); a
// last kernel merges the slabs.  One workgroup per slab: wave wt sums the partial tiles of the slab's
// weight tile wt, the lanes that share a row merge, and one thread per row merges the eight tiles
// (the merge keeps the smaller index on equal maxima, so its order does not matter).
template <int MT, int KSL>
__global__ __launch_bounds__(512) void k_lmhead_finish(LinArgs p)
{
    constexpr int KS = KSL / 32;
    __shared__ float s_mx[8][16 * MT], s_sm[8][16 * MT];
    __shared__ int s_arg[8][16 * MT];
    const int64_t U = (int64_t)p.T * KS;
    const int slab = blockIdx.x, m0 = blockIdx.y * 32;
    const int lane = threadIdx.x & 63, wt = threadIdx.x >> 6;  // wave wt sums the slab's weight tile wt
    const int rho = lane & 15, q = lane >> 4;
    const int first = owner_of((int64_t)slab * p.S * KS, U, p.G);
    const int nseg = owner_of((int64_t)(slab + 1) * p.S * KS - 1, U, p.G) - first + 1;
    const size_t seg_stride = (size_t)8 * MT * 256;
    const float *base = p.partials + ((((size_t)blockIdx.y * p.slabs + slab) * p.maxseg) * 8 + wt) * (MT * 256);
    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int sg = 0; sg < nseg; ++sg)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[mt][r] += base[(size_t)sg * seg_stride + mt * 256 + r * 64 + lane];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        // lane (rho, q) holds logits 4q .. 4q + 3 of the tile for row rho, in ascending order
        float mx = -INFINITY, sm = 0.f;
        int arg = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) fc_argmax_merge(mx, arg, sm, acc[mt][r], slab * 128 + wt * 16 + 4 * q + r, 1.0f);
#pragma unroll
        for (int off = 16; off < 64; off <<= 1) {
            const float mx2 = __shfl_xor(mx, off, 64), sm2 = __shfl_xor(sm, off, 64);
            const int arg2 = __shfl_xor(arg, off, 64);
            fc_argmax_merge(mx, arg, sm, mx2, arg2, sm2);
        }
        if (q == 0) {
            s_mx[wt][16 * mt + rho] = mx;
            s_sm[wt][16 * mt + rho] = sm;
            s_arg[wt][16 * mt + rho] = arg;
        }
    }
    __syncthreads();
    const int row = threadIdx.x;  // one thread per row merges the eight tiles
    if (row < 16 * MT && m0 + row < p.M) {
        float mx = s_mx[0][row], sm = s_sm[0][row];
        int arg = s_arg[0][row];
        for (int w2 = 1; w2 < 8; ++w2) fc_argmax_merge(mx, arg, sm, s_mx[w2][row], s_arg[w2][row], s_sm[w2][row]);
        p.am.at(slab, m0 + row) = FcArgmax{mx, arg, sm};
    }
}


// -------------------------------------------------------------------------------------------------
// Hidden sizes of 512, 3584 and 4096 (the whole activation block fits in registers): whole rows.
//
// A work item is 16 rows of W over the whole hidden dimension (16 x 2K bytes, contiguous in memory);
// the eight waves of a workgroup cut the hidden dimension in eight, and every wave keeps its part of
// the X block (at most 32 rows) in operand registers for the whole kernel, so X is read once per
// workgroup and never again.  It comes by way of LDS, 16 rows at a time, in whole cache lines (direct loads,
// chunks permuted against bank conflicts), with the first item's weights behind it: loaded straight into
// operand registers, half a line per row and load, X cost 3.6 us per 16 rows, none of it hidden (gated W_1 at
// hidden 3584, 18944 outputs, 32 rows: 54.5 us, now 51.2; 4096 x 4096: 16.4, now 11.5).  The weight fragments of a wave are refilled one by one, right behind
// the multiply that consumed them, with the same fragment of the next item: a full item of loads
// stays in flight and the wave never drains its queue.  The eight partial 16 x 32 tiles of an item
// are summed through LDS (double-buffered: one barrier per item) by the first MT waves, which apply
// the epilogue -- residual add, SiLU gate (an item being 8 gate rows and the same 8 up rows), or the
// running (largest logit, index, sum of exponentials) per row, written once per workgroup at the end.
// No partial sums leave the workgroup and there is no second kernel.  Items are dealt in contiguous
// runs measured in half items (8 rows, or 4 gated features), so runs differ by at most half an item;
// a lane whose half of an item belongs to the neighbouring run re-reads the row of the other half
// (same cache lines: no extra traffic) and its results are dropped.  A vocabulary may have any size: rows past its
// end re-read the last one.  Bound by the weights: 5.9 TB/s and about 6 us of launch, X and last items.
template <int MT, int NKW, int MODE>
__global__ __launch_bounds__(512) void k_linear_rows(LinArgs p)
{
    extern __shared__ __align__(1024) unsigned char lds[];
    float(*red)[8][MT * 4][64] = (float(*)[8][MT * 4][64])lds;  // [2]
    constexpr int XROW = NKW * 64;  // bytes of a wave's part of an X row
    // The 16-byte chunks of a row are permuted so that 16 rows' chunks of one column fall into 16 different bank groups.
    auto xswz = [](int r) { return NKW % 4 == 0 ? r & 15 : (r >> 1) & 7; };
    const int wg = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho = lane & 15, q = lane >> 4;
    const int U = p.T;  // half items
    const int u0 = (int)((int64_t)wg * U / p.G), u1 = (int)(((int64_t)wg + 1) * U / p.G);
    if (u0 >= u1) return;
    const int it0 = u0 >> 1, it1 = (u1 + 1) >> 1;
    const size_t kw0 = (size_t)wave * (NKW * 32) + 8 * q;  // this lane's first hidden element

    bf16x8 xr[NKW][MT], wf[NKW];

    // this lane's weight row of item `it`
    auto wrow_of = [&](int it) -> const uint16_t * {
        if (MODE == FC_LIN_GATE_UP) {
            int fi = rho & 7;  // feature of the item; half item = 4 features
            const int uu = 2 * it + (fi >> 2);
            if (uu < u0 || uu >= u1) fi ^= 4;
            return (rho < 8 ? p.W : p.W2) + (size_t)(8 * it + fi) * p.K + kw0;
        }
        int r = rho;  // row of the item; half item = 8 rows
        const int uu = 2 * it + (r >> 3);
        if (uu < u0 || uu >= u1) r ^= 8;
        const int n = MODE == FC_LIN_VOCAB ? min(16 * it + r, p.N - 1) : 16 * it + r;
        return p.W + (size_t)n * p.K + kw0;
    };

    // X block -> operand registers, 16 rows at a time by way of LDS
    unsigned char *xw = lds + wave * (16 * XROW);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int i = 0; i < NKW; ++i) {
            const int byte = 1024 * i + 16 * lane, r = byte / XROW, c = (byte - r * XROW) >> 4;
            const int m = min(16 * mt + r, p.M - 1);  // padding rows read a valid row
            fc_load_lds16(p.X + (size_t)m * p.K + wave * (NKW * 32) + 8 * (c ^ xswz(r)), xw + 1024 * i);
        }
        if (mt == MT - 1) {
            __builtin_amdgcn_sched_barrier(0);
            const uint16_t *cur = wrow_of(it0);
#pragma unroll
            for (int s = 0; s < NKW; ++s) wf[s] = ld8(cur + 32 * s);
            __builtin_amdgcn_sched_barrier(0);
            fc_wait_vm<NKW>();  // everything before the weights
        } else {
            fc_wait_vm<0>();
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < NKW; ++s)
            xr[s][mt] = *(const bf16x8 *)(xw + rho * XROW + (((4 * s + q) ^ xswz(rho)) << 4));
        __builtin_amdgcn_sched_barrier(0);
        fc_wait_lds();  // lgkmcnt(0): the LDS rows may be overwritten
        __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_barrier();  // the partial tiles reuse the area
    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float run_mx = -INFINITY, run_sm = 0.f;  // vocabulary mode: running state of row 16 mt + rho (lanes q = 0 of wave mt)
    int run_arg = 0x7fffffff;
    int buf = 0;

    // Outputs are collected in LDS and leave as whole row segments (flush): an item gives a row only 16 or
    // 32 bytes, and written item by item those pieces cost the streaming a tenth of its rate (memory
    // switching between reading and writing for every piece); a run's segment of a row is one or two
    // cache lines.  Wave mt stages and flushes its own 16 rows, so no barrier is involved.
    constexpr int HALF_EL = MODE == FC_LIN_GATE_UP ? 4 : 8;  // output columns of a half item
    constexpr int STG_ITEMS = 16;                            // items staged between two flushes
    constexpr int STG_CH = STG_ITEMS * 2 * HALF_EL / 4;      // 8-byte pieces of a staged row (at most 64)
    uint2(*stage)[STG_CH + 1] = (uint2(*)[STG_CH + 1])(lds + 2 * 8 * MT * 4 * 64 * sizeof(float));  // [16 MT]
    int stage_it0 = it0;  // item in the first staging slot
    auto flush = [&](int it_end) {  // items stage_it0 .. it_end - 1 are staged
        const int c0 = max(u0 * HALF_EL, stage_it0 * 2 * HALF_EL), c1 = min(u1 * HALF_EL, it_end * 2 * HALF_EL);
        const int nch = (c1 - c0) >> 2, ch0 = (c0 - stage_it0 * 2 * HALF_EL) >> 2;
#pragma unroll 4
        for (int r = 0; r < 16; ++r) {
            const int m = 16 * wave + r;
            if (m < p.M && lane < nch) *(uint2 *)(p.out + (size_t)m * p.N + c0 + 4 * lane) = stage[m][ch0 + lane];
        }
    };

    // Sum of the eight partial tiles of item `it` (in red[rb]) and epilogue, by wave mt < MT for tile mt.
    auto finish_item = [&](int it, int rb) {
        if (MODE != FC_LIN_VOCAB && it - stage_it0 == STG_ITEMS) {
            flush(it);
            stage_it0 = it;
        }
        // wave mt sums tile mt: lane (rho, q) = X row 16 mt + rho, item rows 4 q .. 4 q + 3
        const int mt = wave, m = 16 * mt + rho;
        float sum[4] = {0.f, 0.f, 0.f, 0.f}, sum2[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w2 = 0; w2 < 8; ++w2)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                sum[r] += red[rb][w2][mt * 4 + r][lane];
                if (MODE == FC_LIN_GATE_UP) sum2[r] += red[rb][w2][mt * 4 + r][lane ^ 32];  // up rows: 8 item rows on
            }
        if (MODE == FC_LIN_GATE_UP) {
            const int uu = 2 * it + (q & 1);
            if (q < 2 && m < p.M && uu >= u0 && uu < u1) {
                float y[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) y[r] = sum[r] / (1.0f + expf(-sum[r])) * sum2[r];
                uint2 o;
                o.x = (uint32_t)fc_bf16_bits(y[0]) | ((uint32_t)fc_bf16_bits(y[1]) << 16);
                o.y = (uint32_t)fc_bf16_bits(y[2]) | ((uint32_t)fc_bf16_bits(y[3]) << 16);
                stage[m][(it - stage_it0) * 2 + q] = o;
            }
        } else if (MODE == FC_LIN_RESIDUAL) {
            const int uu = 2 * it + (q >> 1);
            if (m < p.M && uu >= u0 && uu < u1) {
                const size_t at = (size_t)m * p.N + 16 * it + 4 * q;
                if (p.res) {
                    const uint2 rv = *(const uint2 *)(p.res + at);
                    sum[0] += __uint_as_float(rv.x << 16);
                    sum[1] += __uint_as_float(rv.x & 0xffff0000u);
                    sum[2] += __uint_as_float(rv.y << 16);
                    sum[3] += __uint_as_float(rv.y & 0xffff0000u);
                }
                uint2 o;
                o.x = (uint32_t)fc_bf16_bits(sum[0]) | ((uint32_t)fc_bf16_bits(sum[1]) << 16);
                o.y = (uint32_t)fc_bf16_bits(sum[2]) | ((uint32_t)fc_bf16_bits(sum[3]) << 16);
                stage[m][(it - stage_it0) * 4 + q] = o;
            }
        } else {
            // the item's 16 logits of a row: four per lane in ascending order, then the four lanes of the row
            const int uu = 2 * it + (q >> 1);
            float mx = -INFINITY, sm = 0.f;
            int arg = 0x7fffffff;
            if (uu >= u0 && uu < u1) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (16 * it + 4 * q + r < p.N) fc_argmax_merge(mx, arg, sm, sum[r], 16 * it + 4 * q + r, 1.0f);
            }
#pragma unroll
            for (int off = 16; off < 64; off <<= 1) {
                const float mx2 = __shfl_xor(mx, off, 64), sm2 = __shfl_xor(sm, off, 64);
                const int arg2 = __shfl_xor(arg, off, 64);
                fc_argmax_merge(mx, arg, sm, mx2, arg2, sm2);
            }
            fc_argmax_merge(run_mx, run_arg, run_sm, mx, arg, sm);
        }
    };

    auto item = [&](int it, auto more) {
        constexpr bool MORE = decltype(more)::value;
        // The previous item is finished here, one iteration late: what it loads or stores is then issued
        // behind the wait for this item's fragments and never part of it.
        fc_wait_vm<0>();  // vmcnt(0): this item's fragments have landed
        __builtin_amdgcn_sched_barrier(0);
        if (it > it0 && wave < MT) finish_item(it - 1, buf ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        // Fragment s of the next item goes into its register as soon as the multiplies of fragment s are
        // issued.
        const uint16_t *nxt = MORE ? wrow_of(it + 1) : nullptr;
#pragma unroll
        for (int s = 0; s < NKW; ++s) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s], xr[s][mt], acc[mt], 0, 0, 0);
            if (MORE) wf[s] = ld8(nxt + 32 * s);
        }
        float *mine = &red[buf][wave][0][lane];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                mine[(mt * 4 + r) * 64] = acc[mt][r];
                acc[mt][r] = 0.f;
            }
        fc_wait_lds();  // lgkmcnt(0): the tile is in LDS
        __builtin_amdgcn_s_barrier();
        buf ^= 1;
    };
    for (int it = it0; it < it1 - 1; ++it) item(it, std::true_type());
    item(it1 - 1, std::false_type());
    if (wave < MT) {
        finish_item(it1 - 1, buf ^ 1);
        if (MODE != FC_LIN_VOCAB) flush(it1);
    }
    if (MODE == FC_LIN_VOCAB && wave < MT && q == 0 && 16 * wave + rho < p.M)
        p.am.at(wg, 16 * wave + rho) = FcArgmax{run_mx, run_arg, run_sm};
}

template <int MT, int NKW, int MODE>
hipError_t launch_rows_mode(const dim3 &g, const LinArgs &a, hipStream_t s)
{
    constexpr int X = 8 * 16 * NKW * 64, OUT = 2 * 8 * MT * 4 * 64 * 4 + (MODE == FC_LIN_VOCAB ? 0 : MT * 16 * 65 * 8);
    constexpr int LDS = X > OUT ? X : OUT;
    static hipError_t attr = hipFuncSetAttribute((const void *)k_linear_rows<MT, NKW, MODE>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (attr != hipSuccess) return attr;
    k_linear_rows<MT, NKW, MODE><<<g, dim3(512), LDS, s>>>(a);
    return hipGetLastError();
}

// -------------------------------------------------------------------------------------------------
// Layers of at most 8192 outputs (two matrices: as many pairs) and 256 rows, hidden sizes that are multiples of 512.
//
// Every workgroup owns an equal run of outputs and a tile of up to 64 window rows over the whole hidden dimension; its eight waves cut the hidden dimension, and
// each streams its part of the run's weight rows and of the window rows through LDS of its own, 64 hidden elements (one
// line of every row) a stage, waiting for nobody until the waves' tiles are summed.  One launch, no partial tiles in memory.
//   * Bound by what a compute unit takes in: weights from HBM, all window rows from L2.  Direct-to-LDS loads whose lanes lie
//     in eight whole lines run at 64 bytes per clock; straight into operand registers, sixteen rows to an instruction, a
//     quarter of that.  So a long hidden dimension with few outputs, where the window rows outweigh the weights, is
//     better off in parts (18944 x 3584, 32 rows: 36 us here, 30 in the tiled GEMM with its second launch).
//   * Where weight rows lie a multiple of 8 KB apart the workgroups of a die start at eight different stages: all at the
//     same offset they meet in a part of the memory channels.
//   * The epilogue goes by tasks of 16 outputs of four rows, dealt to all waves; the residual is asked for at the start.
// us at 4 / 16 / 32 / 64 rows: 3584 x 3584 7.0 / 7.1 / 8.1 / 9.4 (k_linear_rows 7.8 / 8.5 / 9.9, tiled GEMM in parts 11.3);
// gated 3584 x 4096 11.7 / 11.9 / 13.2 / 16.8 (13.9 / 14.8 / 16.3, 21.5); gated 2048 x 2048 5.0 / 5.1 / 5.5 / 7.2 (tile kernel 5.8 /
// 6.3, slice-wise 8.3, tiled GEMM 13.7); 8192 x 2048 11.3 / 11.6 / 12.9 (14.3 / 14.4 / 15.5).
//
constexpr int LINES_K = 64;  // hidden elements per stage: one 128-byte line of every row

template <int MT, int NR, int MODE>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_linear_lines(LinArgs p)
{
    constexpr int NF = MODE == FC_LIN_GATE_UP ? 2 : 1, TASKS = (NR * MT + 1) / 2;
    extern __shared__ __align__(1024) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho = lane & 15, q = lane >> 4;
    const int m0 = 16 * MT * blockIdx.y;  // (the runs are whole eights: the tiles of one are on one die)
    const int n0 = (int)fc_quotient(blockIdx.x * (uint32_t)p.N, p.div_grid);
    const int R = (int)fc_quotient((blockIdx.x + 1) * (uint32_t)p.N, p.div_grid) - n0;  // outputs of this workgroup
    const int n_stages = p.K / (8 * LINES_K);
    const int n_wl = (R + 7) >> 3;  // loads of a stage and matrix
    unsigned char *xbuf = lds + wave * p.wave_bytes, *wbuf = xbuf + MT * 2048;

    const unsigned char *wbase[NF];
    wbase[0] = (const unsigned char *)(p.W + (size_t)n0 * p.K) + (size_t)wave * n_stages * 128;
    if (NF == 2) wbase[NF - 1] = (const unsigned char *)(p.W2 + (size_t)n0 * p.K) + (size_t)wave * n_stages * 128;
    const unsigned char *xbase = (const unsigned char *)p.X + (size_t)wave * n_stages * 128;
    uint32_t woff[2 * NR], xoff[2 * MT];
#pragma unroll
    for (int i = 0; i < 2 * NR; ++i) {
        const int r = 8 * i + (lane >> 3);
        woff[i] = (uint32_t)min(r, R - 1) * (uint32_t)(2 * p.K) + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) {
        const int r = 8 * i + (lane >> 3);
        xoff[i] = (uint32_t)min(m0 + r, p.M - 1) * (uint32_t)(2 * p.K) + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
    const int turn0 = p.K % 4096 == 0 ? (blockIdx.x >> 3) & 7 : 0;  // n_stages is a multiple of 8 there
    auto issue = [&](int st) {
        st += turn0;
        if (st >= n_stages) st -= n_stages;
        fc_with_hint(p.once, [&](auto once) {
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int i = 0; i < 2 * NR; ++i)
                    if (i < n_wl) fc_load_lds16<decltype(once)::value>(wbase[f] + (size_t)st * 128 + woff[i], wbuf + f * (NR * 2048) + 1024 * i);
        });
#pragma unroll
        for (int i = 0; i < 2 * MT; ++i) fc_load_lds16(xbase + (size_t)st * 128 + xoff[i], xbuf + 1024 * i);
    };
    auto task_row = [&](int j) { return 4 * ((wave + 8 * j) % (4 * MT)) + q; };
    auto task_col = [&](int j) { return 16 * ((wave + 8 * j) / (4 * MT)) + rho; };
    // Residuals, all under way at once and waited for with the first stage (as 16-bit values, each behind its own test of the
    // pointer, the compiler waited for them one by one: eight trips to memory ahead of the weights in the tile of 64 rows).
    uint32_t res[TASKS];
#pragma unroll
    for (int j = 0; j < TASKS; ++j) res[j] = 0;
    if (MODE == FC_LIN_RESIDUAL && p.res) {
#pragma unroll
        for (int j = 0; j < TASKS; ++j) res[j] = p.res[(size_t)min(m0 + task_row(j), p.M - 1) * p.N + n0 + min(task_col(j), R - 1)];
    }
    __builtin_amdgcn_sched_barrier(0);
    issue(0);
    __builtin_amdgcn_sched_barrier(0);

    auto frag = [&](const unsigned char *buf, int row, int s) {
        return *(const bf16x8 *)(buf + row * 128 + (((4 * s + q) ^ ((row >> 1) & 7)) << 4));
    };
    f32x4 acc[NR][NF][MT];
#pragma unroll
    for (int t = 0; t < NR; ++t)
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[t][f][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int st = 0; st < n_stages; ++st) {
        fc_wait_vm<0>();
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 xf[2][MT], wf[2][NR][NF];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) xf[s][mt] = frag(xbuf, 16 * mt + rho, s);
#pragma unroll
            for (int t = 0; t < NR; ++t)
#pragma unroll
                for (int f = 0; f < NF; ++f) wf[s][t][f] = frag(wbuf + f * (NR * 2048), min(16 * t + rho, R - 1), s);
        }
        fc_wait_lds();  // lgkmcnt(0): the areas may be overwritten
        __builtin_amdgcn_sched_barrier(0);
        if (st + 1 < n_stages) issue(st + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int t = 0; t < NR; ++t)
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[t][f][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s][t][f], xf[s][mt], acc[t][f][mt], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < NR; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int f = 0; f < NF; ++f) *(f32x4 *)(xbuf + ((t * MT + mt) * NF + f) * 1280 + q * 320 + rho * 16) = acc[t][f][mt];
    __syncthreads();
    if constexpr (MODE == FC_LIN_VOCAB) {  // a wave per four rows, over all tiles of outputs
        static_assert(MODE != FC_LIN_VOCAB || 4 * MT <= 8, "rows");
        const int ml = 4 * wave + q;
        if (wave >= 4 * MT || 4 * wave >= p.M) return;
        float mx = -INFINITY, sm = 0.f;
        int arg = 0x7fffffff;
#pragma unroll
        for (int t = 0; t < NR; ++t) {
            if (16 * t >= R) break;
            const unsigned char *part = lds + (t * MT + (ml >> 4)) * 1280 + (rho >> 2) * 320 + (ml & 15) * 16 + (rho & 3) * 4;
            float y = 0.f;
#pragma unroll
            for (int w2 = 0; w2 < 8; ++w2) y += *(const float *)(part + w2 * p.wave_bytes);
            if (16 * t + rho < R) fc_argmax_merge(mx, arg, sm, y, n0 + 16 * t + rho, 1.0f);
        }
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const float mx2 = __shfl_xor(mx, off, 64), sm2 = __shfl_xor(sm, off, 64);
            const int arg2 = __shfl_xor(arg, off, 64);
            fc_argmax_merge(mx, arg, sm, mx2, arg2, sm2);
        }
        if (rho == 0 && ml < p.M) p.am.at(blockIdx.x, ml) = FcArgmax{mx, arg, sm};
        return;
    }
#pragma unroll
    for (int j = 0; j < TASKS; ++j) {
        const int ml = task_row(j), m = m0 + ml, c = task_col(j);
        if (m0 + 4 * ((wave + 8 * j) % (4 * MT)) >= p.M || (wave + 8 * j) / (4 * MT) >= NR) continue;
        const unsigned char *part = lds + (((c >> 4) * MT + (ml >> 4)) * NF) * 1280 + ((c & 15) >> 2) * 320 + (ml & 15) * 16 + (c & 3) * 4;
        float y[NF] = {};
#pragma unroll
        for (int w2 = 0; w2 < 8; ++w2)
#pragma unroll
            for (int f = 0; f < NF; ++f) y[f] += *(const float *)(part + w2 * p.wave_bytes + f * 1280);
        if (m >= p.M || c >= R) continue;
        asm volatile("" : "+v"(res[j]));  // (its conversion stays here: ahead of the loop it would wait there)
        p.out[(size_t)m * p.N + n0 + c] = fc_bf16_bits(MODE == FC_LIN_GATE_UP ? y[0] / (1.0f + expf(-y[0])) * y[NF - 1] : y[0] + __uint_as_float(res[j] << 16));
    }
}

template <int MT, int NR, int MODE>
hipError_t launch_lines(LinArgs a, int runs, hipStream_t s)
{
    constexpr int NF = MODE == FC_LIN_GATE_UP ? 2 : 1;
    const int ring = MT * 2048 + NF * NR * 2048, state = NR * NF * MT * 1280;
    a.wave_bytes = ring > state ? ring : state;
    if ((a.N + runs - 1) / runs > 16 * NR || a.wave_bytes > 20 * 1024) return hipErrorInvalidValue;
    a.div_grid = fc_reciprocal(runs);
    a.once = a.once && a.M <= 16 * MT;
    static hipError_t attr = hipFuncSetAttribute((const void *)k_linear_lines<MT, NR, MODE>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return attr;
    k_linear_lines<MT, NR, MODE><<<dim3((unsigned)runs, (unsigned)((a.M + 16 * MT - 1) / (16 * MT))), dim3(512), 8 * a.wave_bytes, s>>>(a);
    return hipGetLastError();
}

// -------------------------------------------------------------------------------------------------
// Large vocabularies, at most 32 rows: a workgroup per compute unit owns an equal run of entries, takes it in passes of up to
// 256 and keeps (largest, index, sum of exponentials) per row to itself until the end.
//   * Bound by the weights from HBM.  Four waves only load: each takes every fourth stage of 64 hidden elements, whole lines of
//     all the pass's rows, into the slot of its own in the ring, so it has to wait for nothing but its own last loads and the loads of
//     three stages (90 KB in a full pass, less where the run is short) are always on their way, over the end of a pass as well.  The
//     lines carry the non-temporal hint where the matrix exceeds the memory-side cache.
//   * Four waves multiply, 64 entries each; what they have to do takes a quarter of the time the loads take.
//   * Logits are summed in eight chains along the hidden dimension, and those by twos.  Relative error (rms) of the confidences against 64
//     bits, whole-row kernel / this one, 32 rows: 512 x 152064 1.18e-7 / 1.11e-7 (chains over 512 elements 2.58e-7), 3584 x 152064 4.26e-7 / 3.35e-7,
//     3584 x 40001 3.32e-7 / 2.90e-7, 4096 x 152064 4.45e-7 / 3.68e-7; with expf in place of the hardware's exponential of a rounded product the same.
//   * Where weight rows lie a multiple of 4 KB apart, workgroups in step would all ask for the same 128 bytes of all those rows, which share
//     a few memory channels.  They take the chains there in four orders, c ^ mix: the pairs, and the pairs of pairs, are the same ones, so a
//     weight row gives the same bits in every workgroup and equal logits go to the smaller index.  Hidden 4096, 32 rows, us in one order / four
//     (/ every workgroup from a stage of its own on, where equal logits went either way): 32001 entries 65.3 / 53.4 (/ 50.1), 50304 81.0 / 68.6
//     (/ 68.8), 100001 139.2 / 124.2 (/ 129.9), 152064 192.5 / 190.8 (/ 189.9).
// us with the merge, whole-row kernel / this one: 3584 x 152064, 4 rows 185.4 / 162.8 (6.7 TB/s), 32 rows 187.9 / 164.9; 3584 x 40001, 32 rows
// 59.0 / 51.4; 4096 x 152064, 32 rows 210.5 / 190.8; 512 x 152064, 32 rows 70.0 / 36.8.
constexpr int RUN_ENTRIES = 256, RUN_WAVES = 4, RUN_SLOTS = 4;  // entries of a pass, multiplying waves, slots = loading waves
__host__ __device__ constexpr int run_slot(int MT) { return (RUN_ENTRIES + 16 * MT) * 128; }

template <int MT, bool ONCE>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_vocab_runs(LinArgs p)
{
    extern __shared__ __align__(1024) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int first = (int)((int64_t)blockIdx.x * p.N / p.G), R = (int)(((int64_t)blockIdx.x + 1) * p.N / p.G) - first;
    const int n_pass = (R + RUN_ENTRIES - 1) / RUN_ENTRIES;
    const int per_pass = ((R + n_pass - 1) / n_pass + 7) & ~7;  // whole blocks of eight rows
    const int n_st = p.K / 64, chain = n_st / 8, total = (R + per_pass - 1) / per_pass * n_st;

    if (wave >= RUN_WAVES) {
        const int lw = wave - RUN_WAVES, lr = lane >> 3;
        const int mix = p.K % 2048 == 0 ? (blockIdx.x >> 3 & 3) * 2 : 0;
        unsigned char *slot = lds + lw * run_slot(MT);
        int pass = 0, st = lw;  // of this wave's next stage
        auto issue = [&]() {
            for (; st >= n_st; st -= n_st) ++pass;
            const int at = mix ? ((st / chain) ^ mix) * chain + st % chain : st;
            const int rows = min(per_pass, R - pass * per_pass);
            const unsigned char *w = (const unsigned char *)(p.W + (size_t)(first + pass * per_pass) * p.K) + (size_t)at * 128;
            const unsigned char *x = (const unsigned char *)p.X + (size_t)at * 128;
#pragma unroll
            for (int i = 0; i < 2 * MT; ++i) {
                const int r = 8 * i + lr;
                fc_load_lds16(x + (uint32_t)min(r, p.M - 1) * (uint32_t)(2 * p.K) + (((lane & 7) ^ (r >> 1 & 7)) << 4), slot + RUN_ENTRIES * 128 + i * 1024);
            }
#pragma unroll 4
            for (int i = 0; 8 * i < rows; ++i) {
                const int r = 8 * i + lr;
                fc_load_lds16<ONCE>(w + (uint32_t)min(r, rows - 1) * (uint32_t)(2 * p.K) + (((lane & 7) ^ (r >> 1 & 7)) << 4), slot + i * 1024);
            }
            st += RUN_SLOTS;
        };
        // Barrier `it` (it = 0 .. total - 2): stage it + 1 is complete and every multiplying wave has left stage it.
        if (lw < total) issue();
        if (lw == 0) fc_wait_vm<0>();
        __builtin_amdgcn_s_barrier();  // stage 0 is complete
        for (int it = 0; it + 1 < total; ++it) {
            if ((it + 1) % RUN_SLOTS == lw) fc_wait_vm<0>();
            __builtin_amdgcn_s_barrier();
            if (it % RUN_SLOTS == lw && it + RUN_SLOTS < total) issue();
        }
        return;
    }

    const int l = lane & 15, q = lane >> 4;
    float run_mx[MT], run_sm[MT];
    int run_arg[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        run_mx[i] = -INFINITY;
        run_sm[i] = 0.f;
        run_arg[i] = 0x7fffffff;
    }
    f32x4 acc[MT][4];
    auto add = [&](f32x4 (&kept)[MT][4]) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][t][r] += kept[i][t][r];
    };
    auto keep = [&](f32x4 (&kept)[MT][4]) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                kept[i][t] = acc[i][t];
                asm volatile("" : "+v"(kept[i][t]));  // summed here and not where it is used, or all eight chains wait in registers
            }
    };
    __builtin_amdgcn_s_barrier();  // stage 0 is complete
    int it = 0;
    auto one_chain = [&]() {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int end = it + chain;
        do {
            const unsigned char *slot = lds + (it % RUN_SLOTS) * run_slot(MT);
            bf16x8 xf[2][MT], wf[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int off = l * 128 + (((4 * h + q) ^ (l >> 1 & 7)) << 4);
#pragma unroll
                for (int i = 0; i < MT; ++i) xf[h][i] = *(const bf16x8 *)(slot + RUN_ENTRIES * 128 + i * 2048 + off);
#pragma unroll
                for (int t = 0; t < 4; ++t) wf[h][t] = *(const bf16x8 *)(slot + wave * 8192 + t * 2048 + off);
            }
            fc_wait_lds();  // lgkmcnt(0): the slot may be overwritten
            __builtin_amdgcn_sched_barrier(0);
            if (it + 1 < total) __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[h][t], xf[h][i], acc[i][t], 0, 0, 0);
        } while (++it < end);
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int done = 0; done < R; done += per_pass) {
        const int rows = min(per_pass, R - done) - 64 * wave;  // of this wave, if positive
        if (rows <= 0) {
            for (int end = it + n_st; it < end; ++it)
                if (it + 1 < total) __builtin_amdgcn_s_barrier();
            continue;
        }
        f32x4 one[MT][4], two[MT][4], four[MT][4];  // sums of so many chains
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            one_chain();
            if ((c & 1) == 0) {
                keep(one);
                continue;
            }
            add(one);
            if ((c & 2) == 0) {
                keep(two);
                continue;
            }
            add(two);
            if ((c & 4) == 0) keep(four);
            else add(four);
        }
        // lane (l, q): window row 16 i + l, entries 16 t + 4 q + r of the wave, ascending; the largest first, then the sum against it
        const int base = first + done + 64 * wave + 4 * q;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            float mx = -INFINITY, sm = 0.f;
            int arg = base;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool more = 16 * t + 4 * q + r < rows && acc[i][t][r] > mx;
                    mx = more ? acc[i][t][r] : mx;
                    arg = more ? base + 16 * t + r : arg;
                }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                float e[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float part = __builtin_amdgcn_exp2f((acc[i][t][r] - mx) * 1.4426950408889634f);
                    // the largest adds 1 whatever it is (an infinite logit: inf - inf)
                    e[r] = 16 * t + 4 * q + r >= rows ? 0.f : base + 16 * t + r == arg ? 1.f : part;
                }
                sm += (e[0] + e[1]) + (e[2] + e[3]);
            }
            if (4 * q < rows) fc_argmax_merge(run_mx[i], run_arg[i], run_sm[i], mx, arg, sm);
        }
    }
    // over the lanes of a row, then over the waves
    FcArgmax *state = (FcArgmax *)lds;  // [multiplying wave][16 MT]; every slot has been left and no load is on its way
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < MT; ++i) {
#pragma unroll
        for (int off = 16; off < 64; off <<= 1) {
            const float mx2 = __shfl_xor(run_mx[i], off, 64), sm2 = __shfl_xor(run_sm[i], off, 64);
            const int arg2 = __shfl_xor(run_arg[i], off, 64);
            fc_argmax_merge(run_mx[i], run_arg[i], run_sm[i], mx2, arg2, sm2);
        }
        if (q == 0) state[wave * 16 * MT + 16 * i + l] = FcArgmax{run_mx[i], run_arg[i], run_sm[i]};
    }
    fc_wait_lds();
    __builtin_amdgcn_s_barrier();
    if (tid < 16 * MT && tid < p.M) {
        FcArgmax a = state[tid];
#pragma unroll
        for (int w = 1; w < RUN_WAVES; ++w) {
            const FcArgmax b = state[w * 16 * MT + tid];
            fc_argmax_merge(a.mx, a.arg, a.sm, b.mx, b.arg, b.sm);
        }
        p.am.at(blockIdx.x, tid) = a;
    }
}

template <int MT>
hipError_t launch_vocab_runs(const LinArgs &a, hipStream_t s)
{
    constexpr int LDS = RUN_SLOTS * run_slot(MT);
    static_assert(LDS <= 160 * 1024 && RUN_SLOTS == 4 && RUN_WAVES == 4, "512 threads");
    auto start = [&](auto once) {
        constexpr auto kernel = k_vocab_runs<MT, decltype(once)::value>;
        static hipError_t attr = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (attr != hipSuccess) return attr;
        kernel<<<dim3((unsigned)a.G), dim3(512), LDS, s>>>(a);
        return hipGetLastError();
    };
    return a.once ? start(std::true_type()) : start(std::false_type());
}

// Tiles of 16 mt window rows and runs of outputs, one workgroup per compute unit; runs of at least four outputs: with fewer
// the window rows are fetched for too little.
struct LinesShape {
    int row_tiles, runs, run;
};
LinesShape lines_shape(int N, int M, int mt)
{
    LinesShape s;
    s.row_tiles = (M + 16 * mt - 1) / (16 * mt);
    const int most = s.row_tiles > 32 ? 8 : 256 / s.row_tiles / 8 * 8;
    s.runs = N >= 4 * most ? most : N >= 32 ? N / 32 * 8 : (N + 3) / 4;
    s.run = (N + s.runs - 1) / s.runs;
    return s;
}

template <int MT>
hipError_t launch_lines_mt(int mode, const LinArgs &a, hipStream_t s)
{
    const LinesShape sh = lines_shape(a.N, a.M, MT);
    if (mode == FC_LIN_GATE_UP) return sh.run <= 16 ? launch_lines<MT, 1, FC_LIN_GATE_UP>(a, sh.runs, s) : launch_lines<MT, 2, FC_LIN_GATE_UP>(a, sh.runs, s);
    if constexpr (MT < 4)  // (lines_tile takes four row tiles for longer runs only)
        if (sh.run <= 16) return launch_lines<MT, 1, FC_LIN_RESIDUAL>(a, sh.runs, s);
    if constexpr (MT == 1) return launch_lines<MT, 2, FC_LIN_RESIDUAL>(a, sh.runs, s);  // (256 runs for one row tile: 32 outputs at most)
    else return sh.run <= 32 ? launch_lines<MT, 2, FC_LIN_RESIDUAL>(a, sh.runs, s) : launch_lines<MT, 4, FC_LIN_RESIDUAL>(a, sh.runs, s);
}

#ifndef FC_LIN_KSL
#define FC_LIN_KSL 512
#endif
constexpr int KSL = FC_LIN_KSL;  // hidden elements per work item

template <int MODE>
hipError_t launch_mode(const FcSkinnyPlan &pl, const LinArgs &a, hipStream_t s)
{
    const dim3 g1((unsigned)pl.G, (unsigned)pl.chunks), g2((unsigned)pl.slabs * 8, (unsigned)pl.chunks, (unsigned)pl.mt);
    if (pl.mt == 1) {
        k_linear_stream<1, KSL, MODE><<<g1, dim3(512), 0, s>>>(a);
        k_linear_finish<1, KSL, MODE><<<g2, dim3(64), 0, s>>>(a);
    } else {
        k_linear_stream<2, KSL, MODE><<<g1, dim3(512), 0, s>>>(a);
        k_linear_finish<2, KSL, MODE><<<g2, dim3(64), 0, s>>>(a);
    }
    return hipGetLastError();
}

template <int MT, int NKW>
hipError_t launch_rows(int mode, const FcSkinnyPlan &pl, const LinArgs &a, hipStream_t s)
{
    const dim3 g((unsigned)pl.G);
    if (mode == FC_LIN_GATE_UP) return launch_rows_mode<MT, NKW, FC_LIN_GATE_UP>(g, a, s);
    if (mode == FC_LIN_VOCAB) return launch_rows_mode<MT, NKW, FC_LIN_VOCAB>(g, a, s);
    return launch_rows_mode<MT, NKW, FC_LIN_RESIDUAL>(g, a, s);
}

// hidden sizes the whole-row kernel is built for (256 x the fragments per wave)
bool rows_kernel_covers(int K) { return K == 512 || K == 3584 || K == 4096; }

}  // namespace

// Runs of work items for the slice-wise kernel.
static FcSkinnyPlan plan_slices(int dtype, int mode, int M, int K, int N, int target)
{
    FcSkinnyPlan p;
    memset(&p, 0, sizeof p);
    const int rows_per_slab = mode == FC_LIN_GATE_UP ? 64 : 128;  // FC_LIN_VOCAB: slabs of 128 vocabulary rows
    if (dtype != FC_BF16 || M < 1 || K < KSL || K % KSL != 0 || N < rows_per_slab || N % rows_per_slab != 0)
        return p;  // kind 0: plain kernel, no workspace
    p.kind = 1;
    p.mt = M <= 16 ? 1 : 2;
    p.chunks = M <= 16 ? 1 : (M + 31) / 32;
    p.slabs = N / rows_per_slab;
    p.S = K / KSL;
    const int64_t T = (int64_t)p.slabs * p.S;
    if (T > (1 << 26) || p.chunks > 65535) {
        p.kind = 0;
        return p;
    }
    p.T = (int)T;
    p.G = p.T < target ? p.T : target;
    // runs are measured in k-steps of 32 hidden elements, so every workgroup streams the same
    // amount to within one k-step; a slab of S * KS k-steps meets at most this many runs
    const int64_t per_slab = (int64_t)p.S * (KSL / 32), upw = T * (KSL / 32) / p.G;
    const int64_t bound = (per_slab + upw - 1) / upw + 1;
    p.maxseg = (int)(bound < p.G ? bound : p.G);
    return p;
}

FcSkinnyPlan fc_plan_skinny(int dtype, int mode, int M, int K, int N)
{
    int target = 256;  // one workgroup per compute unit
    if (fc_knobs().lin_wgs > 0) target = fc_knobs().lin_wgs;  // tuning and test knob: runs of any length
    // whole-row kernel: at most 32 rows, a hidden size it is built for, whole half items (a vocabulary of any size)
    const bool off = fc_knobs().lin_no_rows != 0;  // tuning knob
    const int per_half = mode == FC_LIN_GATE_UP ? 4 : 8;
    const int halves = mode == FC_LIN_VOCAB || N % per_half == 0 ? (N + per_half - 1) / per_half : 0;
    const int items = N >= per_half ? (halves + 1) / 2 : 0;
    if (off || dtype != FC_BF16 || M < 1 || M > 32 || !rows_kernel_covers(K) || items < 1)
        return plan_slices(dtype, mode, M, K, N, target);
    FcSkinnyPlan p;
    memset(&p, 0, sizeof p);
    // Fewer items than compute units are no reason for the slice-wise kernel (hidden 3584, 224 / 64 items: 10.0 / 9.3 us
    // against 12.6 / 11.4, its second launch included), but what these shapes ask of a caller's workspace stays what it
    // has been with it.
    if (items < 256 && K >= 2048) p.reserve = fc_skinny_workspace(plan_slices(dtype, mode, M, K, N, target));
    p.kind = 2;
    p.mt = M <= 16 ? 1 : 2;
    p.chunks = 1;
    p.T = halves;
    p.G = items < target ? items : target;  // at least one item each
    return p;
}

size_t fc_skinny_workspace(const FcSkinnyPlan &p)
{
    if (p.kind != 1) return p.reserve;  // the whole-row kernel keeps its partial sums inside the workgroup
    return (size_t)p.chunks * p.slabs * p.maxseg * 8 * p.mt * 256 * sizeof(float);
}

hipError_t fc_launch_linear_skinny(const FcSkinnyPlan &pl, int mode, const void *x, const void *w, const void *w2,
                                   const void *res, int M, int K, int N, void *out, void *workspace,
                                   hipStream_t s, const FcArgmaxPart *am)
{
    if (pl.kind == 2) {
        if (M < 1 || M > 32 || !rows_kernel_covers(K) || pl.G < 1 || pl.T < 1 || pl.G > (pl.T + 1) / 2 ||
            (mode == FC_LIN_VOCAB && !am))
            return hipErrorInvalidValue;
        LinArgs a;
        memset(&a, 0, sizeof a);
        a.X = (const uint16_t *)x;
        a.W = (const uint16_t *)w;
        a.W2 = (const uint16_t *)w2;
        a.res = (const uint16_t *)res;
        a.out = (uint16_t *)out;
        if (am) a.am = *am;
        a.M = M;
        a.K = K;
        a.N = N;
        a.T = pl.T;
        a.G = pl.G;
        const int nkw = K / 256;
        if (pl.mt == 1) {
            if (nkw == 2) return launch_rows<1, 2>(mode, pl, a, s);
            if (nkw == 14) return launch_rows<1, 14>(mode, pl, a, s);
            return launch_rows<1, 16>(mode, pl, a, s);
        }
        if (nkw == 2) return launch_rows<2, 2>(mode, pl, a, s);
        if (nkw == 14) return launch_rows<2, 14>(mode, pl, a, s);
        return launch_rows<2, 16>(mode, pl, a, s);
    }
    // The kernels index the partial tiles by (slab, position of the workgroup among those that meet
    // the slab); make sure on the host that no slab meets more workgroups than the plan reserved.
    for (int slab = 0; slab < pl.slabs; ++slab) {
        const int64_t per_slab = (int64_t)pl.S * (KSL / 32), U = (int64_t)pl.T * (KSL / 32);
        const int first = owner_of(slab * per_slab, U, pl.G), last = owner_of((slab + 1) * per_slab - 1, U, pl.G);
        if (last - first + 1 > pl.maxseg) return hipErrorInvalidValue;
    }
    if (pl.kind != 1 || pl.G < 1 || pl.G > pl.T || M > pl.chunks * 32 || !workspace) return hipErrorInvalidValue;
    LinArgs a;
    memset(&a, 0, sizeof a);
    a.X = (const uint16_t *)x;
    a.W = (const uint16_t *)w;
    a.W2 = (const uint16_t *)w2;
    a.res = (const uint16_t *)res;
    a.out = (uint16_t *)out;
    a.partials = (float *)workspace;
    a.M = M;
    a.K = K;
    a.N = N;
    a.S = pl.S;
    a.T = pl.T;
    a.G = pl.G;
    a.maxseg = pl.maxseg;
    a.slabs = pl.slabs;
    if (mode == FC_LIN_VOCAB) {
        if (!am) return hipErrorInvalidValue;
        a.am = *am;
        const dim3 g1((unsigned)pl.G, (unsigned)pl.chunks), g2((unsigned)pl.slabs, (unsigned)pl.chunks);
        if (pl.mt == 1) {
            k_linear_stream<1, KSL, FC_LIN_RESIDUAL><<<g1, dim3(512), 0, s>>>(a);
            k_lmhead_finish<1, KSL><<<g2, dim3(512), 0, s>>>(a);
        } else {
            k_linear_stream<2, KSL, FC_LIN_RESIDUAL><<<g1, dim3(512), 0, s>>>(a);
            k_lmhead_finish<2, KSL><<<g2, dim3(512), 0, s>>>(a);
        }
        return hipGetLastError();
    }
    return mode == FC_LIN_GATE_UP ? launch_mode<FC_LIN_GATE_UP>(pl, a, s) : launch_mode<FC_LIN_RESIDUAL>(pl, a, s);
}

// Tiles of 16 window rows a workgroup takes; 0: not for this kernel.  Beyond 32 rows by an estimate (us: the window rows' and
// the weights' way into a compute unit, the epilogue, the weights' from HBM; 11 % from 1200 measured times in the mean)
// that picks within 1 % of the best of 32, 48 and 64 rows in the mean: 3584 x 3584, 64 / 96 / 128 / 176 rows 9.4 / 11.1 / 12.1 / 14.2, one tile of
// all rows 10.9 / 14.2, tiled GEMM in parts 11.3 / 12.8 / 13.8 / 16.9.
static int lines_tile(int mode, int M, int K, int N)
{
    const bool gated = mode == FC_LIN_GATE_UP;
    if (M <= 32) return (M + 15) / 16;
    double best = 1e30;
    int mt = 0;
    for (int t = 2; t <= 4; ++t) {
        const LinesShape s = lines_shape(N, M, t);
        if (s.run > (gated ? 32 : 64)) continue;
        const double rows = M / (16.0 * s.row_tiles) < t ? M / (16.0 * s.row_tiles) : t, w = gated ? 2.0 : 1.0;
        const double tail = 0.066 * w * t * (s.run <= 16 ? 1 : s.run <= 32 ? 2 : 4);
        const double us = 1e-3 * K * (0.258 * rows + 0.0183 * w * s.run + 2.24e-4 * w * N) + tail;
        if (us < best) {
            best = us;
            mt = t;
        }
    }
    return mt;
}

template <int MT>
static hipError_t launch_lines_vocab(const LinArgs &a, int runs, hipStream_t s)
{
    const int run = (a.N + runs - 1) / runs;
    if (run <= 16) return launch_lines<MT, 1, FC_LIN_VOCAB>(a, runs, s);
    if (run <= 32) return launch_lines<MT, 2, FC_LIN_VOCAB>(a, runs, s);
    return launch_lines<MT, 4, FC_LIN_VOCAB>(a, runs, s);
}

// Vocabularies of up to 64 entries per workgroup: faster than what they took before at every size measured, 301 .. 16384 entries,
// hidden 512 .. 5120, 1 .. 32 rows, the reduction included (us at 17 rows: hidden 3584, 2049 / 9001 / 15999 entries 15.7 / 22.4 / 31.8 in
// the whole-row kernel, 10.7 / 18.6 / 26.9 here; hidden 1024, 5001 12.6 in the tile kernel, 9.2 here).
int fc_lmhead_lines_parts(int dtype, int M, int K, int V, int parts)
{
    const int runs = parts < 256 ? parts : 256;
    return dtype == FC_BF16 && M >= 1 && M <= 32 && K >= 512 && K % 512 == 0 && runs >= 1 && V >= runs && (V + runs - 1) / runs <= 64 ? runs : 0;
}

hipError_t fc_launch_lmhead_lines(const void *x, const void *w, int M, int K, int V, const FcArgmaxPart &am, hipStream_t s)
{
    if (fc_lmhead_lines_parts(FC_BF16, M, K, V, am.parts) != am.parts) return hipErrorInvalidValue;
    LinArgs a;
    memset(&a, 0, sizeof a);
    a.X = (const uint16_t *)x;
    a.W = (const uint16_t *)w;
    a.am = am;
    a.M = M;
    a.K = K;
    a.N = V;
    return M <= 16 ? launch_lines_vocab<1>(a, am.parts, s) : launch_lines_vocab<2>(a, am.parts, s);
}

// Parts of the arg-max the kernel for large vocabularies writes, `parts` at most (0: not for it), and the launch.  From runs of 90
// entries on (hidden 512: 64, where it takes over from k_linear_lines; hidden 4096, whose rows share memory channels: 120); a shorter run has
// too few bytes on their way.  us, whole-row kernel / this one, weights from HBM, 4 / 32 rows: hidden 3584, 16385 entries 28.0 and 29.5 / 32.9 and
// 35.3, 20001 34.4 and 36.3 / 36.0 and 38.6, 22017 35.7 and 37.7 / 38.4 and 41.2, 23040 38.3 and 40.0 / 36.9 and 39.0, 26497 41.3 and 43.3 / 39.9
// and 41.4, 32771 47.4 and 48.7 / 47.9 and 48.4, 50304 68.7 and 70.7 / 59.9 and 61.0; hidden 4096, 23041 42.1 and 44.2 / 43.8 and 44.5, 26497 44.2
// and 46.2 / 46.3 and 47.0, 29001 49.8 and 52.1 / 51.2 and 52.4, 32001 55.1 and 57.9 / 51.9 and 53.4, 32771 52.9 and 53.3 / 52.8 and 53.3, 40001 66.1
// and 69.5 / 57.6 and 58.3, 65537 (257 entries, two passes) 92.3 and 96.2 / 95.9 and 98.9, 131072 183.3 and 187.7 / 160.5 and 161.1; hidden 512,
// 16391 13.3 and 14.6 / 12.2 and 13.7, 32771 19.9 and 21.5 / 14.7 and 16.3.
int fc_lmhead_runs_parts(int dtype, int M, int K, int V, int parts)
{
    const int runs = parts < 256 ? parts : 256;
    return dtype == FC_BF16 && M >= 1 && M <= 32 && K >= 512 && K % 512 == 0 && runs == 256 && V >= (K <= 512 ? 64 : K % 2048 == 0 ? 120 : 90) * 256 ? runs : 0;
}

hipError_t fc_launch_lmhead_runs(const void *x, const void *w, int M, int K, int V, const FcArgmaxPart &am, hipStream_t s)
{
    if (fc_lmhead_runs_parts(FC_BF16, M, K, V, am.parts) != am.parts) return hipErrorInvalidValue;
    LinArgs a;
    memset(&a, 0, sizeof a);
    a.X = (const uint16_t *)x;
    a.W = (const uint16_t *)w;
    a.am = am;
    a.M = M;
    a.K = K;
    a.N = V;
    a.G = am.parts;
    a.once = fc_read_once(2.0 * K * V);
    return M <= 16 ? launch_vocab_runs<1>(a, s) : launch_vocab_runs<2>(a, s);
}

bool fc_linear_lines_cover(int dtype, int mode, int M, int K, int N)
{
    return dtype == FC_BF16 && mode != FC_LIN_VOCAB && M >= 1 && M <= 256 && K >= 512 && K % 512 == 0 && N >= 1 && N <= 8192 &&
           lines_tile(mode, M, K, N) > 0;
}

hipError_t fc_launch_linear_lines(int mode, const void *x, const void *w, const void *w2, const void *res, int M, int K, int N,
                                  void *out, bool once, hipStream_t s)
{
    if (!fc_linear_lines_cover(FC_BF16, mode, M, K, N)) return hipErrorInvalidValue;
    LinArgs a;
    memset(&a, 0, sizeof a);
    a.X = (const uint16_t *)x;
    a.W = (const uint16_t *)w;
    a.W2 = (const uint16_t *)w2;
    a.res = (const uint16_t *)res;
    a.out = (uint16_t *)out;
    a.M = M;
    a.K = K;
    a.N = N;
    a.once = once;
    switch (lines_tile(mode, M, K, N)) {
    case 1: return launch_lines_mt<1>(mode, a, s);
    case 2: return launch_lines_mt<2>(mode, a, s);
    case 3: return launch_lines_mt<3>(mode, a, s);
    default: return launch_lines_mt<4>(mode, a, s);
    }
}
