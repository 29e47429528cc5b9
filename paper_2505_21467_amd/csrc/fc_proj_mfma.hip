// QKV projection of the active rows on the matrix cores (bf16, head_dim 128), fused with bias, rotary
// embedding and the scatter into the cache.
//
// The window is short (tens to a few hundred rows), so the product Y^T = W X^T is bound by streaming
// the weight matrix once from HBM.  Both operands are contiguous along the hidden dimension, which is
// exactly the per-lane operand layout of v_mfma_f32_16x16x32_bf16 (8 consecutive k per lane).  Three kernels: runs of
// rotary pairs over the whole hidden dimension for at most 256 window rows (k_proj_stream), few head slots cut along a long
// hidden dimension for 33 .. 128 rows (k_proj_headsplit), both at multiples of 512, and k_proj_skinny, described here, for
// what is left.
//
// A workgroup owns 16 rows of W -- 8 rows i0..i0+7 of one head and their rotary partners
// i0+64..i0+71 -- and up to 32 rows of X.  Its waves split the hidden dimension, load both operands straight into
// registers, and the partial tiles are summed through LDS.  In the
// 16x16 accumulator layout a lane holds 4 consecutive head-dim indices of one window row, and the
// rotary partner of every value sits in the lane 32 away, so the rotation needs one cross-lane swap.
// The rotated q goes to q_out; k and v go directly to their cache rows (v into the transposed tiles).
#include <math.h>

#include <type_traits>

#include "fc_device.h"
#include "fc_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

struct ProjArgs {
    const uint16_t *X;     // [M][K]
    const uint16_t *W;     // [N][K]
    const uint16_t *bias;  // [N] or nullptr
    const int32_t *pos;    // [M] or nullptr
    uint16_t *Q;           // [B][Hq][A][128]
    uint16_t *Kc;          // one layer
    uint16_t *Vc;          // one layer
    FcGeom G;
    int M, A, K, win_start, n_tiles;
    double log2_base_64;   // log2(rope_base) / 64
    double rot[6];         // rope_base^(-i/64), i = 1, 2, 4, .. 32
    float *partials;       // cache scratch: partial tiles of the hidden-dimension slices
    int mt;                // 16-row window tiles of a partial
    int wave_bytes;        // k_proj_stream: LDS of a wave,
    uint32_t div_runs, div_a;  // reciprocals of the number of runs and of A
    bool once;             // k_proj_stream: weights with the non-temporal hint
};

__device__ __forceinline__ bf16x8 ld8(const uint16_t *p)
{
    union { uint4 u; bf16x8 v; } x;
    x.u = *(const uint4 *)p;
    return x.v;
}

__device__ __forceinline__ float swap32f(float v)
{
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    // r[0] = lower half in all lanes, r[1] = upper half in all lanes
    return (threadIdx.x & 32) ? __uint_as_float(r[0]) : __uint_as_float(r[1]);
}

// NW = waves per workgroup (they split the hidden dimension).
template <int MT, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_proj_skinny(ProjArgs p)
{
    __shared__ float red[NW - 1][MT][4][64];
    __shared__ float2 cs[16 * MT][8];  // (cos, sin) for (window row of this chunk, rotary index i0 + e)
    const FcGeom &G = p.G;
    // workgroup id -> (m chunk, n tile): chunks of one n tile have ids equal modulo 8 (same XCD)
    const int tiles8 = (p.n_tiles + 7) & ~7;
    const int mc = blockIdx.x / tiles8, tile = blockIdx.x % tiles8;
    if (tile >= p.n_tiles) return;
    const int hs = tile >> 3, i0 = (tile & 7) * 8;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho = lane & 15, q = lane >> 4;
    const int n = hs * 128 + (rho < 8 ? i0 + rho : 64 + i0 + rho - 8);
    const int kq = p.K / NW;  // hidden elements per wave
    const int m0 = mc * (16 * MT);

    const uint16_t *wrow = p.W + (size_t)n * p.K + (size_t)wave * kq + 8 * q;
    const uint16_t *xrow[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        int m = m0 + 16 * mt + rho;
        if (m >= p.M) m = p.M - 1;  // padding rows of the last chunk read a valid row; never stored
        xrow[mt] = p.X + (size_t)m * p.K + (size_t)wave * kq + 8 * q;
    }

    // Rotary factors for this workgroup's rows and its 8 rotary indices, one (or two) per thread.
    // The angle pos * inv_freq is formed and reduced to a fraction of a turn in double; the
    // hardware sine/cosine take their argument in turns.  Called once the loads are in flight: the
    // table does not depend on them and their latency covers it.
    auto rope_table = [&]() {
        if (hs >= G.Hq + G.Hkv) return;
        for (int idx = tid; idx < 16 * MT * 8; idx += NW * 64) {
            const int lr = idx >> 3, e = idx & 7;
            const int m = min(m0 + lr, p.M - 1);
            const int pp = p.pos ? p.pos[m] : p.win_start + (m % p.A);
            // rope_base^(-2i/128) = 2^(-i * log2(base) / 64), evaluated in double
            const double inv_freq = exp2(-(double)(i0 + e) * p.log2_base_64);
            const double turns = (double)pp * inv_freq * 0.15915494309189533576888;
            const float fr = (float)(turns - rint(turns));
            cs[lr][e] = make_float2(__builtin_amdgcn_cosf(fr), __builtin_amdgcn_sinf(fr));
        }
    };

    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int ks = kq >> 5;
    rope_table();
    for (int s = 0; s < ks; ++s) {
        const bf16x8 wfrag = ld8(wrow + 32 * s);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wfrag, ld8(xrow[mt] + 32 * s), acc[mt], 0, 0, 0);
    }

    // sum the partial tiles of the NW waves in wave 0
    if (wave > 0) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wave - 1][mt][r][lane] = acc[mt][r];
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int w2 = 0; w2 < NW - 1; ++w2) acc[mt][r] += red[w2][mt][r][lane];

    // lane (rho, q) holds W rows 4q..4q+3 of the tile for window row rho of each m tile:
    // q = 0,1 -> head-dim i0 + 4q + r; q = 2,3 -> 64 + i0 + 4(q-2) + r (the rotary partners)
    const bool second = q >= 2;
    const int ib = i0 + 4 * (q & 1);           // rotary index of r = 0
    const int d0 = (second ? 64 : 0) + ib;     // head-dim index of r = 0
    float bs[4] = {0.f, 0.f, 0.f, 0.f};
    if (p.bias) {
#pragma unroll
        for (int r = 0; r < 4; ++r) bs[r] = fc_to_float(bf16_t{p.bias[hs * 128 + d0 + r]});
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = m0 + 16 * mt + rho;
        const bool mvalid = m < p.M;
        const int mm = mvalid ? m : 0;
        const int b = mm / p.A, a = mm - b * p.A;
        const int pp = p.pos ? p.pos[mm] : p.win_start + a;
        const bool valid = mvalid && pp >= 0 && pp < G.max_seq;
        float y[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = acc[mt][r] + bs[r];
        if (hs < G.Hq + G.Hkv) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float other = swap32f(y[r]);
                const float2 f = cs[16 * mt + rho][4 * (q & 1) + r];
                y[r] = second ? y[r] * f.x + other * f.y : y[r] * f.x - other * f.y;
            }
        }
        uint2 w;
        w.x = (uint32_t)fc_bf16_bits(y[0]) | ((uint32_t)fc_bf16_bits(y[1]) << 16);
        w.y = (uint32_t)fc_bf16_bits(y[2]) | ((uint32_t)fc_bf16_bits(y[3]) << 16);
        if (hs < G.Hq) {
            if (mvalid) {
                if (!valid) w = make_uint2(0, 0);
                *(uint2 *)(p.Q + (((size_t)b * G.Hq + hs) * p.A + a) * 128 + d0) = w;
            }
        } else if (valid) {
            if (hs < G.Hq + G.Hkv) {
                *(uint2 *)(p.Kc + fc_k_index(G, b, hs - G.Hq, pp, d0)) = w;
            } else {
                const int j = hs - G.Hq - G.Hkv;
#pragma unroll
                for (int r = 0; r < 4; ++r) p.Vc[fc_v_index(G, b, j, pp, d0 + r)] = fc_bf16_bits(y[r]);
            }
        }
    }
}

// -------------------------------------------------------------------------------------------------
// Head-split kernel for windows of 33 .. 128 rows and hidden sizes that are multiples of 512.
//
// A workgroup owns one whole head slot (128 rows of W: 8 waves x 16 rows) and one 512-wide slice of
// the hidden dimension, so the 512-wide slice of X is fetched once per workgroup (direct-to-LDS,
// swizzled) and shared by the 8 waves instead of being re-read by every 16-row tile.  The partial
// tiles of the hidden-dimension slices of a head go to the cache's device scratch and are summed
// by k_proj_finish.  Bound by one pass over the weights and its first latency: at 36 head slots and hidden 3584
// (252 workgroups, one per compute unit) 9.2 us for 33 MB.
constexpr int HS_K = 512;  // hidden elements per workgroup

template <int MT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_proj_headsplit(ProjArgs p)
{
    extern __shared__ __align__(1024) unsigned char xs[];  // X slice: [16 MT rows][64 chunks of 16 B]
    const int S = p.K / HS_K;
    const int hs = blockIdx.x / S, ks = blockIdx.x % S;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho = lane & 15, q = lane >> 4;
    const int i0 = wave * 8;
    const int n = hs * 128 + (rho < 8 ? i0 + rho : 64 + i0 + rho - 8);

    // X slice -> LDS: one 1 KB row per wave-wide load; chunk c of row m is stored at c ^ (m & 15)
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) {
        const int m = wave * 2 * MT + i;
        const int mg = min(m, p.M - 1);
        const int c = lane ^ (m & 15);
        fc_load_lds16(p.X + (size_t)mg * p.K + (size_t)ks * HS_K + c * 8, xs + m * 1024);
    }
    // W fragments of this wave's 16 rows: all 16 k-steps in flight
    const uint16_t *wrow = p.W + (size_t)n * p.K + (size_t)ks * HS_K + 8 * q;
    bf16x8 wf[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) wf[s] = ld8(wrow + 32 * s);
    __builtin_amdgcn_sched_barrier(0);

    __syncthreads();  // waits for every load of the workgroup, X slice included

    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 16; ++s)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int m = 16 * mt + rho;
            const bf16x8 xf = *(const bf16x8 *)(xs + m * 1024 + (((4 * s + q) ^ (m & 15)) << 4));
            acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s], xf, acc[mt], 0, 0, 0);
        }

    // hand the partial tile over: [head][slice][wave][mt][r][lane]
    float *part = p.partials + ((((size_t)hs * S + ks) * 8 + wave) * MT) * 256;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[mt * 256 + r * 64 + lane] = acc[mt][r];
}

// Second half of the head-split projection: one wave per (head slot, 16-row tile, 16 window rows) sums the partial
// tiles of the hidden-dimension slices (a kernel boundary is the only cross-workgroup ordering used:
// device-scope fences inside a kernel cost an L2 write-back per workgroup on this multi-die part),
// then applies bias and rotary embedding and scatters q, k and v.  Rotary factors are computed per
// lane: base^(-i/64) by binary powering in double (the powers come from the host), the angle reduced to a
// fraction of a turn in double, hardware sine/cosine (argument in turns).  The kernel is one memory round
// trip long, so all of that runs while the partial tiles are on their way.
__global__ __launch_bounds__(64) void k_proj_finish(ProjArgs p)
{
    const FcGeom &G = p.G;
    const int S = p.K / HS_K;
    const int hs = blockIdx.x >> 3, wave = blockIdx.x & 7;  // the wave index of the first kernel = tile
    const int lane = threadIdx.x;
    const int rho = lane & 15, q = lane >> 4;
    const int i0 = wave * 8;
    const int m = 16 * blockIdx.y + rho;
    const bool mvalid = m < p.M;
    const int mm = mvalid ? m : p.M - 1;

    // the first eight slices' loads go out, then everything the epilogue needs besides is fetched and computed
    float v[8][4];
    auto load = [&](int kb) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k2 = min(kb + u, S - 1);
            const float *pp2 = p.partials + ((((size_t)hs * S + k2) * 8 + wave) * p.mt + blockIdx.y) * 256;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[u][r] = pp2[r * 64 + lane];
        }
    };
    load(0);
    const bool second = q >= 2, rotate = hs < G.Hq + G.Hkv;
    const int ib = i0 + 4 * (q & 1);
    const int d0 = (second ? 64 : 0) + ib;
    float bs[4] = {0.f, 0.f, 0.f, 0.f};
    if (p.bias) {
#pragma unroll
        for (int r = 0; r < 4; ++r) bs[r] = fc_to_float(bf16_t{p.bias[hs * 128 + d0 + r]});
    }
    const int pp = p.pos ? p.pos[mm] : p.win_start + mm % p.A;
    __builtin_amdgcn_sched_barrier(0);
    float2 cs[4];
    if (rotate) {
        double f = 0.15915494309189533576888;  // base^(-(ib + r)/64) / (2 pi): turns per position
#pragma unroll
        for (int bit = 0; bit < 6; ++bit)
            if (ib & (1 << bit)) f *= p.rot[bit];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double turns = (double)pp * f;
            const float fr = (float)(turns - rint(turns));
            cs[r] = make_float2(__builtin_amdgcn_cosf(fr), __builtin_amdgcn_sinf(fr));
            f *= p.rot[0];
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int kb = 0; kb < S; kb += 8) {  // eight slices at a time
        if (kb) load(kb);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (kb + u < S) {
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r] += v[u][r];
            }
    }

    const int b = mm / p.A, a = mm - b * p.A;
    const bool valid = mvalid && pp >= 0 && pp < G.max_seq;
    float y[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = acc[r] + bs[r];
    if (rotate) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float other = swap32f(y[r]);
            y[r] = second ? y[r] * cs[r].x + other * cs[r].y : y[r] * cs[r].x - other * cs[r].y;
        }
    }
    uint2 w;
    w.x = (uint32_t)fc_bf16_bits(y[0]) | ((uint32_t)fc_bf16_bits(y[1]) << 16);
    w.y = (uint32_t)fc_bf16_bits(y[2]) | ((uint32_t)fc_bf16_bits(y[3]) << 16);
    if (hs < G.Hq) {
        if (mvalid) {
            if (!valid) w = make_uint2(0, 0);
            *(uint2 *)(p.Q + (((size_t)b * G.Hq + hs) * p.A + a) * 128 + d0) = w;
        }
    } else if (valid) {
        if (hs < G.Hq + G.Hkv) {
            *(uint2 *)(p.Kc + fc_k_index(G, b, hs - G.Hq, pp, d0)) = w;
        } else {
            const int j = hs - G.Hq - G.Hkv;
#pragma unroll
            for (int r = 0; r < 4; ++r) p.Vc[fc_v_index(G, b, j, pp, d0 + r)] = fc_bf16_bits(y[r]);
        }
    }
}

// -------------------------------------------------------------------------------------------------
// Whole-row kernel: at most 256 window rows, hidden sizes that are multiples of 512.
//
// Every workgroup owns an equal run of rotary pairs (rows i and i + 64 of a head; 9 pairs at 36 head slots) and a tile of up
// to 64 window rows over the whole hidden dimension, so no partial tiles leave it.  Its eight waves cut the hidden dimension; each streams its part of the
// run's weight rows and of the window rows through LDS of its own, 64 hidden elements (one line of every row) per
// stage, and waits for nobody until the waves' tiles are summed.
//   * Bound by what a compute unit takes in, weights from HBM and all window rows from L2.  Loads whose lanes lie in eight
//     whole lines run at 64 bytes per clock; loaded straight into operand registers, sixteen rows to an instruction,
//     weights alone came at a quarter of that.
//   * Where weight rows lie a multiple of 8 KB apart the workgroups of a die start at eight different stages: all at the
//     same offset they meet in a part of the memory channels (96 slots, hidden 4096, 8 / 32 rows 20.2 / 22.1 -> 19.4 / 20.9).
//   * The epilogue's tasks go by 16 pairs of four rows: more waves share it, a row is stored 32 bytes at a time, and its
//     operands and first angle are at hand when the sums are (16 / 32 / 64 rows 9.1 / 10.5 / 14.3 -> 8.7 / 10.0 / 13.8 us).
//   * NP = 2: runs of 17 .. 32 pairs.
// Against the kernel it replaced (X kept in operand registers, at most 32 rows) and the head-split kernels, us: 36 head slots,
// hidden 3584, 4 / 16 / 32 rows 9.4 / 9.6 / 11.1 -> 8.3 / 8.6 / 9.8, 48 / 64 / 96 / 128 rows 13.6 / 15.0 / 17.4 / 19.2 -> 11.8 / 12.5 / 14.2 /
// 16.1; 96 slots, hidden 4096, 32 rows 23.3 -> 21.1; 24 slots, hidden 2048, 32 / 64 / 128 rows 9.5 / 11.8 / 10.5 -> 5.5 / 6.2 / 7.6.

constexpr int STREAM_K = 64;  // hidden elements per stage: one 128-byte line of every row
template <int MT, int NP>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_proj_stream(ProjArgs p)
{
    extern __shared__ __align__(1024) unsigned char lds[];
    const FcGeom &G = p.G;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho = lane & 15, q = lane >> 4;
    // (run of pairs, tile of window rows): the runs are whole eights, so the tiles of one are on one die, which reads its
    // weights from HBM once.  (Taken from one index by division this cost 0.25 us.)
    const int run = blockIdx.x, m0 = 16 * MT * blockIdx.y;
    const uint32_t n_pairs = (uint32_t)p.n_tiles * 8;
    const int g0 = (int)fc_quotient(run * n_pairs, p.div_runs);
    const int R = (int)fc_quotient((run + 1) * n_pairs, p.div_runs) - g0;  // pairs of this workgroup
    const int n_stages = p.K / (8 * STREAM_K);
    const int n_wl = (2 * R + 7) >> 3;  // weight loads of a stage
    unsigned char *xbuf = lds + wave * p.wave_bytes, *wbuf = xbuf + MT * 2048;

    // row r of the workgroup's weight rows: the first rows of its pairs, then their partners
    const int row0 = (g0 >> 6) * 128 + (g0 & 63);
    const unsigned char *wbase = (const unsigned char *)(p.W + (size_t)row0 * p.K) + (size_t)wave * n_stages * 128;
    const unsigned char *xbase = (const unsigned char *)p.X + (size_t)wave * n_stages * 128;
    // A run has fewer than 64 pairs and meets the end of a head once at most, at pair `turn`: 64 rows on from there, as for the partners.
    const int turn = 64 - (g0 & 63);
    const uint32_t chunk = (uint32_t)((lane & 7) ^ (lane >> 4)) << 4;  // swizzled by bits 1..3 of the row
    uint32_t woff[4 * NP], xoff[2 * MT];
#pragma unroll
    for (int i = 0; i < 4 * NP; ++i) {
        const int r = min(8 * i + (lane >> 3), 2 * R - 1), e = r < R ? r : r - R;
        const int row = e + (e < turn ? 0 : 64) + (r < R ? 0 : 64);
        woff[i] = __umul24(row, 2 * p.K) + (chunk ^ (i & 1) << 6);
    }
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) xoff[i] = (uint32_t)min(m0 + 8 * i + (lane >> 3), p.M - 1) * (uint32_t)(2 * p.K) + (chunk ^ (i & 1) << 6);
    const int turn0 = p.K % 4096 == 0 ? (run >> 3) & 7 : 0;  // n_stages is a multiple of 8 there
    auto issue = [&](int st) {
        st += turn0;
        if (st >= n_stages) st -= n_stages;
        fc_with_hint(p.once, [&](auto once) {
#pragma unroll
            for (int i = 0; i < 4 * NP; ++i)
                if (i < n_wl) fc_load_lds16<decltype(once)::value>(wbase + (size_t)st * 128 + woff[i], wbuf + 1024 * i);
        });
#pragma unroll
        for (int i = 0; i < 2 * MT; ++i) fc_load_lds16(xbase + (size_t)st * 128 + xoff[i], xbuf + 1024 * i);
    };
    // The epilogue goes by tasks of 16 pairs in four window rows, lane = (row, pair), dealt to the waves.  Positions and
    // bias are asked for first; the first task's angle comes while the last stage is on its way.
    constexpr int TASKS = (NP * MT + 1) / 2;
    int pp[TASKS];
    uint32_t bs[TASKS][2];  // (as 16 bits the compiler packs a pair, and waits for both here: a trip to HBM ahead of the weights)
    auto task_row = [&](int j) { return 4 * ((wave + 8 * j) % (4 * MT)) + q; };
    auto task_pair = [&](int j) { return 16 * ((wave + 8 * j) / (4 * MT)) + rho; };
#pragma unroll
    for (int j = 0; j < TASKS; ++j) {
        const int mm = min(m0 + task_row(j), p.M - 1);
        pp[j] = p.pos ? p.pos[mm] : p.win_start + mm - (int)fc_quotient(mm, p.div_a) * p.A;
        bs[j][0] = bs[j][1] = 0;
    }
    if (p.bias) {
#pragma unroll
        for (int j = 0; j < TASKS; ++j) {
            const int gp = g0 + min(task_pair(j), R - 1);
            bs[j][0] = p.bias[(gp >> 6) * 128 + (gp & 63)];
            bs[j][1] = p.bias[(gp >> 6) * 128 + (gp & 63) + 64];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    issue(0);
    __builtin_amdgcn_sched_barrier(0);
    auto angle = [&](int j) {
        const int i = (g0 + task_pair(j)) & 63;
        double f = 0.15915494309189533576888;  // base^(-i/64) / (2 pi): turns per position of pair i
#pragma unroll
        for (int bit = 0; bit < 6; ++bit)
            if (i & (1 << bit)) f *= p.rot[bit];
        const double turns = (double)pp[j] * f;
        return (float)(turns - rint(turns));
    };
    float first_angle = 0.f;

    auto frag = [&](const unsigned char *buf, int row, int s) {
        return *(const bf16x8 *)(buf + row * 128 + (((4 * s + q) ^ ((row >> 1) & 7)) << 4));
    };
    f32x4 acc[NP][2][MT];
#pragma unroll
    for (int t = 0; t < NP; ++t)
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[t][f][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int st = 0; st < n_stages; ++st) {
        if (st == n_stages - 1) first_angle = angle(0);
        fc_wait_vm<0>();
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 xf[2][MT], wf[2][NP][2];
        auto read = [&](int s) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) xf[s][mt] = frag(xbuf, 16 * mt + rho, s);
#pragma unroll
            for (int t = 0; t < NP; ++t) {
                const int row = min(16 * t + rho, R - 1);
                wf[s][t][0] = frag(wbuf, row, s);
                wf[s][t][1] = frag(wbuf, R + row, s);
            }
        };
        auto multiply = [&](int s) {
#pragma unroll
            for (int t = 0; t < NP; ++t)
#pragma unroll
                for (int f = 0; f < 2; ++f)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[t][f][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s][t][f], xf[s][mt], acc[t][f][mt], 0, 0, 0);
        };
        read(0);
        read(1);
        fc_wait_lds();  // lgkmcnt(0): the areas may be overwritten
        __builtin_amdgcn_sched_barrier(0);
        if (st + 1 < n_stages) issue(st + 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(0);
        multiply(1);
    }
    // [pair tile][window tile][first / partner][lane] in the wave's own area, quarters 64 bytes apart for the reads below
#pragma unroll
    for (int t = 0; t < NP; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int f = 0; f < 2; ++f) *(f32x4 *)(xbuf + ((t * MT + mt) * 2 + f) * 1280 + q * 320 + rho * 16) = acc[t][f][mt];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TASKS; ++j) {
        const int ml = task_row(j), m = m0 + ml, pr = task_pair(j);
        if (m0 + 4 * ((wave + 8 * j) % (4 * MT)) >= p.M || (wave + 8 * j) / (4 * MT) >= NP) continue;
        const unsigned char *part = lds + (((pr >> 4) * MT + (ml >> 4)) * 2) * 1280 + ((pr & 15) >> 2) * 320 + (ml & 15) * 16 + (pr & 3) * 4;
        float y0 = 0.f, y1 = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < 8; ++w2) {
            y0 += *(const float *)(part + w2 * p.wave_bytes);
            y1 += *(const float *)(part + w2 * p.wave_bytes + 1280);
        }
        if (m >= p.M || pr >= R) continue;
        const int gp = g0 + pr, hs = gp >> 6, i = gp & 63;
        asm volatile("" : "+v"(bs[j][0]), "+v"(bs[j][1]));  // (their conversion stays here: ahead of the loop it would wait there)
        y0 += __uint_as_float(bs[j][0] << 16);
        y1 += __uint_as_float(bs[j][1] << 16);
        if (hs < G.Hq + G.Hkv) {
            const float turn = j ? angle(j) : first_angle;
            const float cs = __builtin_amdgcn_cosf(turn), sn = __builtin_amdgcn_sinf(turn);
            const float r0 = y0 * cs - y1 * sn, r1 = y1 * cs + y0 * sn;
            y0 = r0;
            y1 = r1;
        }
        const int b = (int)fc_quotient(m, p.div_a), a = m - b * p.A;
        const bool valid = pp[j] >= 0 && pp[j] < G.max_seq;
        const uint16_t o0 = fc_bf16_bits(y0), o1 = fc_bf16_bits(y1);
        if (hs < G.Hq) {
            uint16_t *d = p.Q + (((size_t)b * G.Hq + hs) * p.A + a) * 128 + i;
            d[0] = valid ? o0 : 0;
            d[64] = valid ? o1 : 0;
        } else if (valid) {
            const bool is_k = hs < G.Hq + G.Hkv;
            const int kv = hs - G.Hq - (is_k ? 0 : G.Hkv);
            uint16_t *base = is_k ? p.Kc : p.Vc;
            base[is_k ? fc_k_index(G, b, kv, pp[j], i) : fc_v_index(G, b, kv, pp[j], i)] = o0;
            base[is_k ? fc_k_index(G, b, kv, pp[j], i + 64) : fc_v_index(G, b, kv, pp[j], i + 64)] = o1;
        }
    }
}

template <int MT, int NP>
hipError_t launch_stream(ProjArgs a, int runs, hipStream_t s)
{
    const int run = (a.n_tiles * 8 + runs - 1) / runs;
    const int ring = MT * 2048 + (2 * run + 7) / 8 * 1024;
    const int state = NP * 2 * MT * 1280;
    a.wave_bytes = ring > state ? ring : state;
    if (run > 16 * NP || runs % 8 || a.wave_bytes > 20 * 1024) return hipErrorInvalidValue;
    a.div_runs = fc_reciprocal(runs);
    a.div_a = fc_reciprocal(a.A);
    a.once = a.G.once && a.M <= 16 * MT;
    static hipError_t attr = hipFuncSetAttribute((const void *)k_proj_stream<MT, NP>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return attr;
    k_proj_stream<MT, NP><<<dim3((unsigned)runs, (unsigned)((a.M + 16 * MT - 1) / (16 * MT))), dim3(512), 8 * a.wave_bytes, s>>>(a);
    return hipGetLastError();
}

// Tiles of 16 mt window rows and runs of pairs, one workgroup per compute unit; runs of at least four pairs: with fewer the
// window rows are fetched for too little.
struct StreamShape {
    int mt, row_tiles, runs, run;
};
StreamShape stream_shape(int slots, int M, int mt)
{
    StreamShape s;
    s.mt = mt;
    s.row_tiles = (M + 16 * mt - 1) / (16 * mt);
    const int n_pairs = slots * 64, most = s.row_tiles > 32 ? 8 : 256 / s.row_tiles / 8 * 8;
    s.runs = n_pairs < 4 * most ? n_pairs / 32 * 8 : most;  // whole eights, one of each on every die
    s.run = (n_pairs + s.runs - 1) / s.runs;
    return s;
}

template <int MT>
hipError_t launch_stream_mt(const ProjArgs &a, int slots, hipStream_t s)
{
    const StreamShape sh = stream_shape(slots, a.M, MT);
    return sh.run <= 16 ? launch_stream<MT, 1>(a, sh.runs, s) : launch_stream<MT, 2>(a, sh.runs, s);
}

size_t headsplit_bytes(int slots, int M, int K)
{
    return (size_t)slots * (K / HS_K) * 8 * ((M + 15) / 16) * 256 * sizeof(float);
}

bool headsplit_covers(int slots, int M, int K)
{
    return !fc_knobs().proj_no_headsplit && M > 32 && M <= 128 && K % HS_K == 0 && headsplit_bytes(slots, M, K) <= FC_SCRATCH_BYTES;
}

template <int MT>
hipError_t launch_headsplit(const ProjArgs &a, int slots, hipStream_t s)
{
    constexpr int LDS = 16 * MT * 2 * HS_K;
    static hipError_t attr = hipFuncSetAttribute((const void *)k_proj_headsplit<MT>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (attr != hipSuccess) return attr;
    k_proj_headsplit<MT><<<dim3((unsigned)(slots * (a.K / HS_K))), dim3(512), LDS, s>>>(a);
    k_proj_finish<<<dim3((unsigned)slots * 8, (unsigned)MT), dim3(64), 0, s>>>(a);
    return hipGetLastError();
}

template <int MT>
hipError_t launch_mt(const ProjArgs &a, int m_chunks, hipStream_t s)
{
    const unsigned grid = (unsigned)(((a.n_tiles + 7) & ~7) * m_chunks);
    if (a.K % 256 == 0) k_proj_skinny<MT, 8><<<dim3(grid), dim3(512), 0, s>>>(a);  // eight waves split the hidden dimension
    else k_proj_skinny<MT, 4><<<dim3(grid), dim3(256), 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace

bool fc_project_mfma_supported(const fc_config &cfg)
{
    return cfg.dtype == FC_BF16 && cfg.head_dim == 128 && cfg.hidden % 128 == 0;
}

// Estimates (us).
// Head-split: weights at 5 TB/s after 4 us of launch and first latency, but no less than two short kernels; for every 16 rows
// the partial tiles, written and read back at 5.5 TB/s, and the window rows.  Measured at 48 / 64 / 96 / 128 rows: 36 head
// slots, hidden 3584: 13.7 / 15.1 / 17.5 / 19.2, the tiled GEMM, whose 72 half-slab tiles leave most of the chip idle,
// 20.9 / 21.6 / 22.8 / 23.6.  96 slots, hidden 4096 (three workgroups per compute unit), 64 rows: 38.4 against 27.9.
static double headsplit_us(int slots, int M, int K)
{
    const double weights = 256.0 * slots * K, part = (double)headsplit_bytes(slots, 16, K);
    return fmax(8.5, 4.0 + weights / 5.0e6) + (M + 15) / 16 * (0.5 + 2.0 * part / 5.5e6);
}

// Tile kernel of small problems: a wave's chain along the hidden dimension rules it out where that is long.
static double tile_us(int slots, int M, int K)
{
    const double weights = 128e-6 * (double)K * slots;  // millions
    return K > 3072 || weights > 13.0 ? 1e30 : fmax(4.0, 3.2 + 0.032 * M * weights);
}

// Runs of pairs: launch, the window rows' and the weights' way into a compute unit, the epilogue, the weights' from HBM (7 %
// from the measured times in the mean at hidden 512 .. 5120, 24 .. 96 head slots, 33 .. 144 rows).  Rows in tiles of 32, 48 or
// 64 by the same estimate, which picks within 0.1 % of the best of the three: 36 slots, hidden 3584, 64 / 96 / 128 rows 12.3 / 14.0 /
// 16.9 us where one tile of all rows took 13.6 / 17.8 / 20.4.  (1e30: runs of more than 32 pairs.)
static double stream_us(int slots, int M, int K, int *mt)
{
    double best = 1e30;
    for (int t = M <= 32 ? (M + 15) / 16 : 2; t <= (M <= 32 ? (M + 15) / 16 : 4); ++t) {
        const StreamShape s = stream_shape(slots, M, t);
        if (s.run > 32) continue;
        const double rows = fmin(t, M / (16.0 * s.row_tiles));
        const double us = 2.52 + 1e-3 * K * (0.311 * rows + 0.0362 * s.run + 0.0312 * slots) + 0.36 * t * ((s.run + 15) / 16);
        if (us < best) {
            best = us;
            *mt = t;
        }
    }
    return best;
}

// Up to 32 rows nothing else is faster by more than 0.1 us, except past 96 head slots (two operands) the tiled GEMM at small
// hidden sizes (128 slots, 16 rows, hidden 2048 / 3584 16.3 / 22.0 us and 13.9 / 24).  From 33 rows on by estimates.  Head-split keeps
// few slots with a hidden dimension beyond 8192 (6 slots, hidden 12288, 64 rows 17.8 and 13.9); more than 80 slots, or 64
// from 65 rows on, the tiled GEMM (96 slots, hidden 2048, 48 rows 15.3 and 14.2; 48 slots, hidden 4096, 160 rows 25.7 and 24.0;
// 36 slots, hidden 3584, 144 / 160 rows 16.4 / 18.2 and 17.5 / 17.9; 24 slots, hidden 5120, 192 rows 19.2 and 25.0; 12 slots, hidden
// 3584, 256 rows 10.3 and 15.5).
static bool stream_wins(int slots, int M, int K, int *mt)
{
    if (K % 512 != 0 || M > 256 || slots > (M > (K >= 3072 ? 64 : 48) ? 64 : M > 32 ? 80 : K >= 3584 ? 128 : 96) || (M > 128 && K <= 1024)) return false;
    const double us = stream_us(slots, M, K, mt);
    if (M <= 32) return us < 1e30;
    if (M > 128) return us < 0.95 * fc_project_gemm_us(slots, M, K);
    if (slots > 64) return us < fc_project_gemm_us(slots, M, K);
    return us < fmin(0.94 * headsplit_us(slots, M, K), tile_us(slots, M, K));
}

bool fc_project_prefers_gemm(const fc_config &cfg, int M, bool scratch)
{
    if (!fc_project_gemm_supported(cfg, M)) return false;
    if (fc_knobs().proj_gemm_shape >= 0 && M > 32) return true;  // tuning knob
    const int slots = cfg.n_q_heads + 2 * cfg.n_kv_heads;
    int stream_mt;
    if (stream_wins(slots, M, cfg.hidden, &stream_mt)) return false;
    if (!scratch || !headsplit_covers(slots, M, cfg.hidden)) return M > 32 || cfg.hidden % HS_K == 0;
    return headsplit_us(slots, M, cfg.hidden) > fc_project_gemm_us(slots, M, cfg.hidden);
}

// Small problems: the tile kernel, by estimate.  Measured with weights from HBM (us, tile kernel first), hidden 256 .. 8192, 6 .. 48
// head slots, 1 .. 128 rows: against the tiled GEMM, hidden 512, 12 slots, 128 rows 5.7 and 5.8; against k_proj_skinny
// (hidden no multiple of 512), hidden 768, 12 slots 4.9 and 4.3 at 16 rows, 4.9 and 5.3 at 24.
bool fc_project_prefers_tile(const fc_config &cfg, int M)
{
    const int slots = cfg.n_q_heads + 2 * cfg.n_kv_heads;
    int stream_mt;
    if (cfg.dtype != FC_BF16 || cfg.head_dim != 128 || fc_knobs().proj_gemm_shape >= 0 || stream_wins(slots, M, cfg.hidden, &stream_mt))
        return false;
    const bool skinny = M <= 32 && cfg.hidden % HS_K != 0;
    if (skinny && M <= 16) return false;
    const double other = skinny ? 3.55 + 0.002 * cfg.hidden : 3.9 + 0.0043 * (cfg.hidden < 1024 ? cfg.hidden : 1024);
    return tile_us(slots, M, cfg.hidden) < 0.97 * other;
}

hipError_t fc_launch_project_mfma(const FcGeom &G, const void *x, const void *w, const void *bias,
                                  const int32_t *pos, int win_start, int A, void *q_out, void *k_layer,
                                  void *v_layer, void *scratch, hipStream_t s)
{
    ProjArgs a;
    a.X = (const uint16_t *)x;
    a.W = (const uint16_t *)w;
    a.bias = (const uint16_t *)bias;
    a.pos = pos;
    a.Q = (uint16_t *)q_out;
    a.Kc = (uint16_t *)k_layer;
    a.Vc = (uint16_t *)v_layer;
    a.G = G;
    a.M = G.B * A;
    a.A = A;
    a.K = G.d;
    a.win_start = win_start;
    a.n_tiles = (G.Hq + 2 * G.Hkv) * 8;
    a.log2_base_64 = G.log_base * 1.4426950408889634074 / 64.0;
    a.partials = (float *)scratch;
    for (int i = 0; i < 6; ++i) a.rot[i] = exp(-G.log_base * (1 << i) / 64.0);
    const int slots = G.Hq + 2 * G.Hkv, mt = (a.M + 15) / 16;
    int stream_mt;
    if (stream_wins(slots, a.M, a.K, &stream_mt)) {
        switch (stream_mt) {
        case 1: return launch_stream_mt<1>(a, slots, s);
        case 2: return launch_stream_mt<2>(a, slots, s);
        case 3: return launch_stream_mt<3>(a, slots, s);
        default: return launch_stream_mt<4>(a, slots, s);
        }
    }
    if (scratch && headsplit_covers(slots, a.M, a.K)) {
        a.mt = mt;
        switch (mt) {
        case 3: return launch_headsplit<3>(a, slots, s);
        case 4: return launch_headsplit<4>(a, slots, s);
        case 5: return launch_headsplit<5>(a, slots, s);
        case 6: return launch_headsplit<6>(a, slots, s);
        case 7: return launch_headsplit<7>(a, slots, s);
        default: return launch_headsplit<8>(a, slots, s);
        }
    }
    if (a.M <= 16) return launch_mt<1>(a, 1, s);
    return launch_mt<2>(a, (a.M + 31) / 32, s);
}
