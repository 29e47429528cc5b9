// QKV projection of the active rows on the matrix cores (bf16, head_dim 128), fused with bias, rotary
// embedding and the scatter into the cache.
//
// The window is short (tens to a few hundred rows), so the product Y^T = W X^T is bound by streaming
// the weight matrix once from HBM.  Both operands are contiguous along the hidden dimension, which is
// exactly the per-lane operand layout of v_mfma_f32_16x16x32_bf16 (8 consecutive k per lane), so W
// fragments are loaded straight from global memory into operand registers.  Three kernels: whole rows for at most 32
// window rows at the hidden sizes it is built for (k_proj_rows), head slots cut along the hidden dimension for
// at most 128 rows (k_proj_headsplit), and the one described here for what is left.
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
// Head-split kernel for windows of at most 128 rows and hidden sizes that are multiples of 512.
//
// A workgroup owns one whole head slot (128 rows of W: 8 waves x 16 rows) and one 512-wide slice of
// the hidden dimension, so the 512-wide slice of X is fetched once per workgroup (direct-to-LDS,
// swizzled) and shared by the 8 waves instead of being re-read by every 16-row tile.  The partial
// tiles of the hidden-dimension slices of a head go to the cache's device scratch and are summed
// by k_proj_finish.  Bound by one pass over the weights and its first latency: at 36 head slots and hidden 3584
// (252 workgroups, one per compute unit) 9.2 us for 33 MB.
constexpr int HS_K = 512;  // hidden elements per workgroup

__device__ __forceinline__ void load_lds16p(const void *g, void *l)
{
    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)g,
                                     (void __attribute__((address_space(3))) *)l, 16, 0, 0);
}

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
        load_lds16p(p.X + (size_t)mg * p.K + (size_t)ks * HS_K + c * 8, xs + m * 1024);
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
// Whole-row kernel for windows of at most 32 rows at the hidden sizes it was measured at, 512, 3584 and 4096.  The window rows
// would fit in registers at every multiple of 256 up to 4096; at other sizes the kernels above run.
//
// Every workgroup owns an equal run of rotary pairs (rows i and i + 64 of a head; 9 pairs at 36 head slots) and takes
// them in items of 8 NF pairs over the whole hidden dimension, so no partial tiles leave the workgroup: its eight
// waves cut the hidden dimension, keep their part of X in operand registers, and sum their tiles through LDS.
//   NF = 1: one operand of 16 weight rows, lanes 0 .. 7 the first rows of 8 pairs, 8 .. 15 their partners
//   NF = 2: two operands, the first rows of up to 16 pairs and their partners
// X comes by way of LDS in whole cache lines (direct-to-LDS, 16 rows at a time, chunks permuted against bank conflicts):
// loaded straight into operand registers, half a line per row and load, it was 7 us of the kernel at 32 rows.  One launch:
// 36 head slots, hidden 3584, 16 / 32 rows 9.9 / 11.3 us (head-split and its finish 11.5 / 12.6); 96 slots, hidden 4096,
// 32 rows 22.8 us (26.7 in the tiled GEMM); 12 slots, hidden 512, 4.2 (6.6).
template <int N>
__device__ __forceinline__ void wait_vm()
{
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

template <int MT, int NKW, int NF>
__global__ __launch_bounds__(512) void k_proj_rows(ProjArgs p)
{
    extern __shared__ __align__(1024) unsigned char lds[];
    float(*red)[8][NF][MT * 4][64] = (float(*)[8][NF][MT * 4][64])lds;  // [2]
    constexpr int XROW = NKW * 64;  // bytes of a wave's part of an X row
    auto xswz = [](int r) { return NKW % 4 == 0 ? r & 15 : (r >> 1) & 7; };
    const FcGeom &G = p.G;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho = lane & 15, q = lane >> 4;
    const int n_pairs = p.n_tiles * 8;
    int g0 = (int)((int64_t)blockIdx.x * n_pairs / gridDim.x);
    const int g1 = (int)(((int64_t)blockIdx.x + 1) * n_pairs / gridDim.x);
    const int kw0 = wave * (NKW * 32) + 8 * q;

    // weight row of this lane in operand f of the item that starts at pair g (past the end: the run's last pair)
    auto wrow_of = [&](int g, int f) -> const uint16_t * {
        const int gp = min(g + (NF == 1 ? rho & 7 : rho), g1 - 1);
        const bool partner = NF == 1 ? rho >= 8 : f == 1;
        return p.W + ((size_t)(gp >> 6) * 128 + (gp & 63) + (partner ? 64 : 0)) * p.K + kw0;
    };
    bf16x8 xr[NKW][MT], wf[NKW][NF];
    unsigned char *xw = lds + wave * (16 * XROW);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int i = 0; i < NKW; ++i) {
            const int byte = 1024 * i + 16 * lane, r = byte / XROW, c = (byte - r * XROW) >> 4;
            const int m = min(16 * mt + r, p.M - 1);  // padding rows read a valid row
            load_lds16p(p.X + (size_t)m * p.K + wave * (NKW * 32) + 8 * (c ^ xswz(r)), xw + 1024 * i);
        }
        if (mt == MT - 1) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const uint16_t *w = wrow_of(g0, f);
#pragma unroll
                for (int s = 0; s < NKW; ++s) wf[s][f] = ld8(w + 32 * s);
            }
            __builtin_amdgcn_sched_barrier(0);
            wait_vm<NKW * NF>();  // everything before the weights
        } else {
            wait_vm<0>();
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < NKW; ++s)
            xr[s][mt] = *(const bf16x8 *)(xw + rho * XROW + (((4 * s + q) ^ xswz(rho)) << 4));
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the LDS rows may be overwritten
        __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_barrier();  // the partial tiles reuse the area

    // In the epilogue wave e < 4 MT finishes register r = e & 3 of window tile e >> 2; its lanes hold pair 4 q + r of an
    // item (NF = 1: pair 4 (q & 1) + r, lanes q >= 2 the partner).
    const int mt_e = wave >> 2, r_e = wave & 3;
    const int m = 16 * mt_e + rho, mm = min(m, p.M - 1);
    const int b = mm / p.A, a = mm - b * p.A;
    const int pp = p.pos ? p.pos[mm] : p.win_start + a;
    const bool valid = pp >= 0 && pp < G.max_seq;
    const int pair_e = NF == 1 ? 4 * (q & 1) + r_e : 4 * q + r_e;

    f32x4 acc[NF][MT];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[f][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    int buf = 0;
    auto item = [&](int g, auto more) {
        constexpr bool MORE = decltype(more)::value;
        // what the epilogue needs besides, while the weights are on their way
        const int gp = min(g + pair_e, g1 - 1), hs = gp >> 6, i = gp & 63;
        float bs[2] = {0.f, 0.f};
        if (p.bias) {
            bs[0] = fc_to_float(bf16_t{p.bias[hs * 128 + i]});
            bs[1] = fc_to_float(bf16_t{p.bias[hs * 128 + i + 64]});
        }
        double f = 0.15915494309189533576888;  // base^(-i/64) / (2 pi): turns per position
#pragma unroll
        for (int bit = 0; bit < 6; ++bit)
            if (i & (1 << bit)) f *= p.rot[bit];
        const double turns = (double)pp * f;
        const float fr = (float)(turns - rint(turns));
        const bool rotate = hs < G.Hq + G.Hkv;
        const float cs = rotate ? __builtin_amdgcn_cosf(fr) : 1.f, sn = rotate ? __builtin_amdgcn_sinf(fr) : 0.f;
        __builtin_amdgcn_sched_barrier(0);

        const uint16_t *nxt[NF];
#pragma unroll
        for (int f2 = 0; f2 < NF; ++f2)
            if (MORE) nxt[f2] = wrow_of(g + 8 * NF, f2);
#pragma unroll
        for (int s = 0; s < NKW; ++s)
#pragma unroll
            for (int f2 = 0; f2 < NF; ++f2) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[f2][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s][f2], xr[s][mt], acc[f2][mt], 0, 0, 0);
                if (MORE) wf[s][f2] = ld8(nxt[f2] + 32 * s);
            }
#pragma unroll
        for (int f2 = 0; f2 < NF; ++f2)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    red[buf][wave][f2][mt * 4 + r][lane] = acc[f2][mt][r];
                    acc[f2][mt][r] = 0.f;
                }
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the tile is in LDS
        __builtin_amdgcn_s_barrier();
        if (wave < 4 * MT) {
            float y0 = 0.f, y1 = 0.f;  // NF = 1: own value and partner's; NF = 2: first row and partner
#pragma unroll
            for (int w2 = 0; w2 < 8; ++w2) {
                y0 += red[buf][w2][0][wave][lane];
                y1 += NF == 1 ? red[buf][w2][0][wave][lane ^ 32] : red[buf][w2][NF - 1][wave][lane];
            }
            const bool second = NF == 1 && q >= 2;
            y0 += second ? bs[1] : bs[0];
            y1 += second ? bs[0] : bs[1];
            const uint16_t o0 = fc_bf16_bits(second ? y0 * cs + y1 * sn : y0 * cs - y1 * sn);
            const uint16_t o1 = fc_bf16_bits(y1 * cs + y0 * sn);
            const int d0 = i + (second ? 64 : 0);
            if (m < p.M && g + pair_e < g1) {
                if (hs < G.Hq) {
                    uint16_t *d = p.Q + (((size_t)b * G.Hq + hs) * p.A + a) * 128;
                    d[d0] = valid ? o0 : 0;
                    if (NF == 2) d[i + 64] = valid ? o1 : 0;
                } else if (valid) {
                    const bool is_k = hs < G.Hq + G.Hkv;
                    const int j = hs - G.Hq - (is_k ? 0 : G.Hkv);
                    uint16_t *base = is_k ? p.Kc : p.Vc;
                    base[is_k ? fc_k_index(G, b, j, pp, d0) : fc_v_index(G, b, j, pp, d0)] = o0;
                    if (NF == 2) base[is_k ? fc_k_index(G, b, j, pp, i + 64) : fc_v_index(G, b, j, pp, i + 64)] = o1;
                }
            }
        }
        buf ^= 1;
    };
    if constexpr (NF == 1)
        for (; g0 + 8 < g1; g0 += 8) item(g0, std::true_type());
    item(g0, std::false_type());
}

template <int MT, int NKW, int NF>
hipError_t launch_rows(const ProjArgs &a, hipStream_t s)
{
    constexpr int X = 8 * 16 * NKW * 64, RED = 2 * 8 * NF * MT * 4 * 64 * 4, LDS = X > RED ? X : RED;
    static hipError_t attr = hipFuncSetAttribute((const void *)k_proj_rows<MT, NKW, NF>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (attr != hipSuccess) return attr;
    const int groups = a.n_tiles;  // of eight pairs
    k_proj_rows<MT, NKW, NF><<<dim3((unsigned)(groups < 256 ? groups : 256)), dim3(512), LDS, s>>>(a);
    return hipGetLastError();
}

// Two operands (one item of up to 16 pairs) where the runs are of 9 .. 16 pairs: with one they would be two items, the
// second nearly empty (36 head slots, hidden 3584, 32 rows: 11.3 against 11.9 us).  At hidden 4096 they do not fit in
// registers.
template <int MT>
hipError_t launch_rows_mt(const ProjArgs &a, hipStream_t s)
{
    const int run = (a.n_tiles * 8 + 255) / 256;
    if (a.K == 512) return launch_rows<MT, 2, 1>(a, s);
    if (a.K == 4096) return launch_rows<MT, 16, 1>(a, s);
    return run > 8 && run <= 16 ? launch_rows<MT, 14, 2>(a, s) : launch_rows<MT, 14, 1>(a, s);
}

bool rows_covers(int M, int K) { return M <= 32 && (K == 512 || K == 3584 || K == 4096); }

size_t headsplit_bytes(int slots, int M, int K)
{
    return (size_t)slots * (K / HS_K) * 8 * ((M + 15) / 16) * 256 * sizeof(float);
}

bool headsplit_covers(int slots, int M, int K)
{
    return !fc_knobs().proj_no_headsplit && M <= 128 && K % HS_K == 0 && headsplit_bytes(slots, M, K) <= FC_SCRATCH_BYTES;
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

// The head-split kernels against the tiled GEMM, by estimate (us): weights at 5 TB/s after 4 us of launch and first
// latency, but no less than two short kernels; for every 16 rows the partial tiles, written and read back at 5.5 TB/s,
// and the window rows.  Measured at 16 / 32 / 64 / 96 / 128 rows: 36 head slots, hidden 3584: 11.5 / 12.7 / 15.3 / 17.8 /
// 19.6, the GEMM, whose 72 half-slab tiles leave most of the chip idle, 19.5 / 20.6 / 21.6 / 22.8 / 23.6.  96 slots,
// hidden 4096 (three workgroups per compute unit): 27.4 / 29.9 / 38.4 at 16 / 32 / 64 rows against 25.8 / 26.5 / 27.9.
// 12 slots, hidden 512: 9.1 / 9.5 / 10.8 against 6.2 / 6.6 / 6.8.
bool fc_project_prefers_gemm(const fc_config &cfg, int M, bool scratch)
{
    if (!fc_project_gemm_supported(cfg, M)) return false;
    if (fc_knobs().proj_gemm_shape >= 0 && M > 32) return true;  // tuning knob
    if (rows_covers(M, cfg.hidden)) return false;
    const int slots = cfg.n_q_heads + 2 * cfg.n_kv_heads, mt = (M + 15) / 16;
    if (!scratch || !headsplit_covers(slots, M, cfg.hidden)) return M > 32;
    const double weights = 256.0 * slots * cfg.hidden, part = (double)headsplit_bytes(slots, 16, cfg.hidden);
    const double us = fmax(8.5, 4.0 + weights / 5.0e6) + mt * (0.5 + 2.0 * part / 5.5e6);
    return us > fc_project_gemm_us(slots, M, cfg.hidden);
}

// Small problems: the tile kernel, by estimate.  Measured with weights from HBM (us, tile kernel first), hidden 256 .. 8192, 6 .. 48
// head slots, 1 .. 128 rows: against the tiled GEMM, hidden 512, 12 slots, 48 / 128 rows 5.0 and 5.7 / 6.0 and 5.8;
// against the head-split kernels, two launches, hidden 1024, 24 slots, 16 / 32 rows 5.0 and 7.6 / 6.6 and 7.8, hidden 2048 6.9 and
// 9.6 / 10.5 and 10.0; against k_proj_skinny (hidden no multiple of 512), hidden 768, 12 slots 4.9 and 4.3 at 16 rows, 4.9 and 5.3
// at 24.  A wave's chain along the hidden dimension is what it loses by: 6 slots, 8 rows, hidden 3072 7.5 and 9.2, 5120 10.8
// and 10.2, 8192 14.6 and 10.1; 48 slots, hidden 2560 13.2 and 11.2.
bool fc_project_prefers_tile(const fc_config &cfg, int M)
{
    if (cfg.dtype != FC_BF16 || cfg.head_dim != 128 || fc_knobs().proj_gemm_shape >= 0 || rows_covers(M, cfg.hidden)) return false;
    const double weights = 128e-6 * (double)cfg.hidden * (cfg.n_q_heads + 2 * cfg.n_kv_heads);  // millions
    const bool skinny = M <= 32 && cfg.hidden % HS_K != 0;
    if (cfg.hidden > 3072 || weights > 13.0 || (skinny && M <= 16)) return false;
    const double other = skinny ? 3.55 + 0.002 * cfg.hidden : 3.9 + 0.0043 * (cfg.hidden < 1024 ? cfg.hidden : 1024);
    return fmax(4.0, 3.2 + 0.032 * M * weights) < 0.97 * other;
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
    if (rows_covers(a.M, a.K)) return mt == 1 ? launch_rows_mt<1>(a, s) : launch_rows_mt<2>(a, s);
    if (scratch && headsplit_covers(slots, a.M, a.K)) {
        a.mt = mt;
        switch (mt) {
        case 1: return launch_headsplit<1>(a, slots, s);
        case 2: return launch_headsplit<2>(a, slots, s);
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
