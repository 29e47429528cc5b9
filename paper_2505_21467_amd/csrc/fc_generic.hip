// Kernels for fp32 caches (the small full-precision configuration) and for the bf16 shapes that the
// weight-streaming and tiled-GEMM kernels do not cover (head_dim 64, hidden sizes and widths that are
// not whole stages or slabs), plus row copies, RMS normalisation and the drift diagnostic.
// Arithmetic: products on the matrix cores with fp32 accumulation (fp32 operands use the fp32 MFMA:
// full-precision products), rotary angles reduced in double, results rounded once to the storage dtype.
#include <string.h>

#include "fc_device.h"
#include "fc_internal.h"

namespace {

__device__ __forceinline__ float wave_sum(float v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// ---------------------------------------------------------------------------------------------
// Row copies between the plain [B][Hkv][rows][Dh] layout and the cache layout.
template <typename T>
__global__ __launch_bounds__(256) void k_copy_rows(FcGeom G, T *__restrict__ kc, T *__restrict__ vc,
                                                   T *__restrict__ kr, T *__restrict__ vr, int start,
                                                   int rows, bool to_cache)
{
    const size_t total = (size_t)G.B * G.Hkv * rows * G.Dh;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (size_t)gridDim.x * blockDim.x) {
        const int i = (int)(e % G.Dh);
        size_t r = e / G.Dh;
        const int row = (int)(r % rows);
        r /= rows;
        const int j = (int)(r % G.Hkv);
        const int b = (int)(r / G.Hkv);
        const size_t ki = fc_k_index(G, b, j, start + row, i);
        const size_t vi = fc_v_index(G, b, j, start + row, i);
        if (to_cache) {
            kc[ki] = kr[e];
            vc[vi] = vr[e];
        } else {
            kr[e] = kc[ki];
            vr[e] = vc[vi];
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Operand fragments of the 16x16 matrix instructions: a lane (rho = lane & 15, q = lane >> 4) holds 16
// bytes of row rho, the hidden elements KB q .. KB q + KB - 1 of a block of 4 KB.  For fp32 the four
// elements feed four v_mfma_f32_16x16x4_f32 (each takes one element per lane, so the hidden index is
// permuted, the same way in both operands); for bf16 the eight feed one v_mfma_f32_16x16x32_bf16.
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

template <typename T>
struct Op;
template <>
struct Op<float> {
    static constexpr int KB = 4;
    typedef f32x4 frag;
    static __device__ __forceinline__ f32x4 mfma(const frag &a, const frag &b, f32x4 acc)
    {
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], acc, 0, 0, 0);
        return acc;
    }
};
template <>
struct Op<bf16_t> {
    static constexpr int KB = 8;
    typedef bf16x8 frag;
    static __device__ __forceinline__ f32x4 mfma(const frag &a, const frag &b, f32x4 acc)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
    }
};

__device__ __forceinline__ float partner32(float v)  // the value of lane ^ 32
{
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return (threadIdx.x & 32) ? __uint_as_float(r[0]) : __uint_as_float(r[1]);
}

// Over the four lanes l, l ^ 16, l ^ 32, l ^ 48 that share a column.
__device__ __forceinline__ float max_rows(float v)
{
    unsigned u = __float_as_uint(v);
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    u = __float_as_uint(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
    r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_rows(float v)
{
    unsigned u = __float_as_uint(v);
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    u = __float_as_uint(__uint_as_float(r[0]) + __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ void store4(float *p, const float (&y)[4]) { fc_store_any(p, make_float4(y[0], y[1], y[2], y[3])); }
__device__ __forceinline__ void store4(bf16_t *p, const float (&y)[4])
{
    uint2 w;
    w.x = (uint32_t)fc_bf16_bits(y[0]) | ((uint32_t)fc_bf16_bits(y[1]) << 16);
    w.y = (uint32_t)fc_bf16_bits(y[2]) | ((uint32_t)fc_bf16_bits(y[3]) << 16);
    fc_store_any(p, w);
}

// ---------------------------------------------------------------------------------------------
// Linear layers of any shape: Y^T = W X^T for a block of 16 NT weight rows and 16 MT window rows per
// workgroup.  These problems are small (a few MB of weights at most), so what bounds them is latency:
// the eight waves cut the hidden dimension, each streams its part of both operands from global memory
// (U blocks at a time, the next U in flight behind the multiplies of these), and the partial tiles are summed
// through LDS, tile t by wave t mod 8, which applies the epilogue.  The operands come by way of LDS (an area of its own per
// wave, direct-to-LDS loads of 64 bytes per row): straight into registers, with neighbouring lanes in different rows, a
// compute unit takes one lane a clock, 38 B/ns.  108 problems of 4 .. 160 rows, hidden 256 .. 2048 in fp32, 256 / 512 in bf16:
// 0.78 of the time (fp32 32 x 1024 x 512 6.4 -> 4.4 us, gated 160 x 512 x 1024 11.7 -> 8.6, projection 32 x 512 x 1024 4.7 -> 4.1; the
// same bits).  Pointers off 16 bytes and rows that are no whole blocks still go straight into registers (bf16 4 x 2056 x 2056
// 4.9 that way, 5.1 with pieces that straddle lines).
// Plain-ALU kernels with one dot product per wave took 36 us for the tiny configuration's projection (32
// rows, hidden 256, 768 outputs; 0.3 TFLOP/s); this one takes about 5.
//   EPI_QKV       bias, rotary embedding, scatter: a 16-row weight tile is the rotary indices i0 .. i0 + 7
//                 of a head and their partners, so the two members of a pair sit 32 lanes apart
//   EPI_RESIDUAL  out = aux + x w^T (aux may be nullptr)
//   EPI_GATE_UP   out = silu(x w^T) * (x w2^T): a tile is eight gate rows and the same eight up rows
//   EPI_VOCAB     per (workgroup of weight rows, window row): largest logit, its index, sum of exponentials
enum { EPI_QKV, EPI_RESIDUAL, EPI_GATE_UP, EPI_VOCAB };

struct TileArgs {
    const void *X, *W, *W2, *aux;  // aux: bias [N] (EPI_QKV) or residual [M][N]
    void *out;                     // [M][N], or q
    int M, K, N, n_blocks;         // n_blocks: workgroups along the weight rows
    FcDivisor by_blocks, by_a;
    // EPI_QKV
    FcGeom G;
    const int32_t *pos;
    int win_start, A;
    void *Kc, *Vc;
    double inv_freq[64];
    FcArgmaxPart am;               // EPI_VOCAB
};

constexpr int TW = 8;  // waves per workgroup
// LDS of a wave: its partial tiles, before that (LDS) a step's blocks of both operands
constexpr size_t tile_wave(int NT, int MT, int U, bool lds) { return (size_t)1024 * (lds && U * (NT + MT) > NT * MT ? U * (NT + MT) : NT * MT); }
constexpr size_t tile_lds(int NT, int MT, int U, bool lds) { return TW * tile_wave(NT, MT, U, lds) + (size_t)MT * 16 * NT * 8 * sizeof(float2); }

template <typename T, int NT, int MT, int U, int EPI, bool LDS>
__global__ __launch_bounds__(TW * 64) void k_linear_tile(TileArgs p)
{
    typedef Op<T> O;
    typedef typename O::frag frag;
    constexpr int KB = O::KB;  // U blocks of 4 KB hidden elements per load step
    extern __shared__ __align__(16) unsigned char tile_smem[];
    constexpr size_t WAVE = tile_wave(NT, MT, U, LDS);
    float2 *cs = (float2 *)(tile_smem + TW * WAVE);                // EPI_QKV: [window row][8 NT rotary indices]
    const FcGeom &G = p.G;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho = lane & 15, q = lane >> 4;
    const int m_blk = (int)p.by_blocks.over(blockIdx.x), n_blk = (int)blockIdx.x - m_blk * p.n_blocks, m0 = m_blk * (16 * MT);
    const int half = G.Dh / 2, head_shift = G.Dh == 128 ? 3 : 2;
    // EPI_QKV: tiles per head = Dh / 16, four or eight
    auto head_of = [&](int tile) { return tile >> head_shift; };
    auto i0_of = [&](int tile) { return (tile & ((1 << head_shift) - 1)) * 8; };

    // What the lane loads: row lr, elements KB lq of a block.  Into registers the operand's own; by way of LDS four
    // neighbouring lanes take 64 bytes of a row, chunks permuted against bank conflicts.
    const int lr = LDS ? lane >> 2 : rho, lq = LDS ? (lane & 3) ^ (lane >> 4) : q;
    const T *wrow[NT], *xrow[MT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int tile = n_blk * NT + t;
        if (EPI == EPI_QKV) {
            const int hs = min(head_of(tile), G.Hq + 2 * G.Hkv - 1), i0 = i0_of(tile);
            wrow[t] = (const T *)p.W + (size_t)(hs * G.Dh + (lr < 8 ? i0 + lr : half + i0 + lr - 8)) * p.K;
        } else if (EPI == EPI_GATE_UP) {
            wrow[t] = (const T *)(lr < 8 ? p.W : p.W2) + (size_t)min(tile * 8 + (lr & 7), p.N - 1) * p.K;
        } else {
            wrow[t] = (const T *)p.W + (size_t)min(tile * 16 + lr, p.N - 1) * p.K;
        }
        wrow[t] += KB * lq;
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) xrow[t] = (const T *)p.X + (size_t)min(m0 + 16 * t + lr, p.M - 1) * p.K + KB * lq;

    // this wave's blocks of the hidden dimension
    const int n_kb = (p.K + 4 * KB - 1) / (4 * KB);
    const int b0 = wave * n_kb / TW, b1 = (wave + 1) * n_kb / TW;
    unsigned char *buf = tile_smem + wave * WAVE;
    auto issue = [&](int b) {  // LDS: the next U blocks at most
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (b + u >= b1) break;
            const int at = (b + u) * 4 * KB;
#pragma unroll
            for (int t = 0; t < NT; ++t) fc_load_lds16(wrow[t] + at, buf + (u * (NT + MT) + t) * 1024);
#pragma unroll
            for (int t = 0; t < MT; ++t) fc_load_lds16(xrow[t] + at, buf + (u * (NT + MT) + NT + t) * 1024);
        }
    };
    auto load = [&](int b, frag(&wf)[U][NT], frag(&xf)[U][MT]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // past this wave's blocks or past the hidden dimension (K is a multiple of 8, a block 16 or 32):
            // read the row's first elements and drop them
            const int k = (b + u) * 4 * KB;
            const bool ok = b + u < b1 && k + KB * q < p.K;
            const int at = ok ? k : -KB * q;
#pragma unroll
            for (int t = 0; t < NT; ++t) wf[u][t] = fc_load_any<frag>(wrow[t] + at);
#pragma unroll
            for (int t = 0; t < MT; ++t) xf[u][t] = fc_load_any<frag>(xrow[t] + at);
            if (!ok) {
#pragma unroll
                for (int t = 0; t < NT; ++t) wf[u][t] = frag{};
#pragma unroll
                for (int t = 0; t < MT; ++t) xf[u][t] = frag{};
            }
        }
    };
    f32x4 acc[NT][MT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const frag(&wf)[U][NT], const frag(&xf)[U][MT]) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[t][m] = O::mfma(wf[u][t], xf[u][m], acc[t][m]);
    };

    frag wa[U][NT], xa[U][MT], wb[U][NT], xb[U][MT];
    if constexpr (LDS) issue(b0);
    else load(b0, wa, xa);
    if (EPI == EPI_QKV) {
        // rotary factors of this workgroup's rows and indices, while the first loads are in flight
        const int hs0 = head_of(n_blk * NT);
        if (hs0 < G.Hq + G.Hkv) {
            for (int idx = tid; idx < 16 * MT * 8 * NT; idx += TW * 64) {
                const int row = idx / (8 * NT), e = idx % (8 * NT);
                const int m = min(m0 + row, p.M - 1);
                const int pp = p.pos ? p.pos[m] : p.win_start + m - (int)p.by_a.over(m) * p.A;
                double turns = (double)pp * p.inv_freq[i0_of(n_blk * NT + e / 8) + e % 8] * 0.15915494309189533576888;
                turns -= rint(turns);
                float c, s;
                sincosf((float)(turns * 6.283185307179586476925286766559), &s, &c);
                cs[idx] = make_float2(c, s);
            }
        }
    }
    if constexpr (LDS) {
        const int at = rho * 64 + ((q ^ (rho >> 2)) << 4);
        for (int b = b0; b < b1; b += U) {
            fc_wait_vm<0>();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int t = 0; t < NT; ++t) wa[u][t] = *(const frag *)(buf + (u * (NT + MT) + t) * 1024 + at);
#pragma unroll
                for (int t = 0; t < MT; ++t) xa[u][t] = *(const frag *)(buf + (u * (NT + MT) + NT + t) * 1024 + at);
            }
            fc_wait_lds();  // lgkmcnt(0): the area may be overwritten
            __builtin_amdgcn_sched_barrier(0);
            if (b + U < b1) issue(b + U);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (b + u >= b1) break;
                // fp32: with several waves per SIMD a pause behind each four matrix instructions lets another wave in
                // (700 x 512 x 2048 26.3 -> 22.5 us, gated 160 x 512 x 2048 14.9 -> 13.4; without rivals it is not felt)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        acc[t][m] = O::mfma(wa[u][t], xa[u][m], acc[t][m]);
                        if constexpr (sizeof(T) == 4) asm volatile("s_nop 7");
                    }
            }
        }
    } else {
        for (int b = b0;; b += 2 * U) {  // (a wave without blocks multiplies zeros once)
            if (b + U >= b1) {
                multiply(wa, xa);
                break;
            }
            load(b + U, wb, xb);
            multiply(wa, xa);
            if (b + 2 * U >= b1) {
                multiply(wb, xb);
                break;
            }
            load(b + 2 * U, wa, xa);
            multiply(wb, xb);
        }
    }

#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) ((float *)buf)[((t * MT + m) * 4 + r) * 64 + lane] = acc[t][m][r];
    __syncthreads();

    float run_mx = -INFINITY, run_sm = 0.f;
    int run_arg = 0x7fffffff;
    // EPI_VOCAB: the NT tiles of a window-row tile are merged by one wave
    for (int ti = wave; ti < (EPI == EPI_VOCAB ? MT : NT * MT); ti += TW) {
#pragma unroll
        for (int tv = 0; tv < (EPI == EPI_VOCAB ? NT : 1); ++tv) {
            const int t = EPI == EPI_VOCAB ? tv : ti / MT, mt = EPI == EPI_VOCAB ? ti : ti % MT;
            float y[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w2 = 0; w2 < TW; ++w2)
#pragma unroll
                for (int r = 0; r < 4; ++r) y[r] += ((const float *)(tile_smem + w2 * WAVE))[((t * MT + mt) * 4 + r) * 64 + lane];
            // lane (rho, q) holds weight rows 4 q .. 4 q + 3 of the tile for window row rho
            const int m = m0 + 16 * mt + rho, tile = n_blk * NT + t;
            const bool mvalid = m < p.M;
            if constexpr (EPI == EPI_QKV) {
                const int hs = head_of(tile), i0 = i0_of(tile);
                if (hs >= G.Hq + 2 * G.Hkv) continue;
                const int d0 = (q >= 2 ? half : 0) + i0 + 4 * (q & 1);
                const int mm = mvalid ? m : 0;
                const int b = (int)p.by_a.over(mm), a = mm - b * p.A;
                const int pp = p.pos ? p.pos[mm] : p.win_start + a;
                const bool valid = mvalid && pp >= 0 && pp < G.max_seq;
                if (p.aux) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) y[r] += fc_to_float(((const T *)p.aux)[hs * G.Dh + d0 + r]);
                }
                if (hs < G.Hq + G.Hkv) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float other = partner32(y[r]);
                        const float2 f = cs[(16 * mt + rho) * (8 * NT) + 8 * t + 4 * (q & 1) + r];
                        y[r] = q >= 2 ? y[r] * f.x + other * f.y : y[r] * f.x - other * f.y;
                    }
                }
                if (hs < G.Hq) {
                    if (!valid) y[0] = y[1] = y[2] = y[3] = 0.f;
                    if (mvalid) store4((T *)p.out + (((size_t)b * G.Hq + hs) * p.A + a) * G.Dh + d0, y);
                } else if (valid) {
                    if (hs < G.Hq + G.Hkv) {
                        store4((T *)p.Kc + fc_k_index(G, b, hs - G.Hq, pp, d0), y);
                    } else {
                        T *v = (T *)p.Vc + fc_v_index(G, b, hs - G.Hq - G.Hkv, pp, d0);
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[r * FC_VTILE] = fc_from_float<T>(y[r]);
                    }
                }
            } else if constexpr (EPI == EPI_GATE_UP) {
                // lanes q = 0, 1 hold the gate products of features 4 q + r, lanes q = 2, 3 the up products
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float up = partner32(y[r]);
                    y[r] = y[r] / (1.0f + expf(-y[r])) * up;
                }
                const int f0 = tile * 8 + 4 * q;
                if (!mvalid || q >= 2) continue;
                T *o = (T *)p.out + (size_t)m * p.N + f0;
                if ((p.N & 3) == 0) {
                    if (f0 < p.N) store4(o, y);
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (f0 + r < p.N) o[r] = fc_from_float<T>(y[r]);
                }
            } else if constexpr (EPI == EPI_RESIDUAL) {
                const int n0 = tile * 16 + 4 * q;
                if (!mvalid) continue;
                T *o = (T *)p.out + (size_t)m * p.N + n0;
                if (p.aux) {
                    const T *res = (const T *)p.aux + (size_t)m * p.N + n0;
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (n0 + r < p.N) y[r] += fc_to_float(res[r]);
                }
                if ((p.N & 3) == 0) {
                    if (n0 < p.N) store4(o, y);
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (n0 + r < p.N) o[r] = fc_from_float<T>(y[r]);
                }
            } else {
                const int n0 = tile * 16 + 4 * q;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (n0 + r < p.N) fc_argmax_merge(run_mx, run_arg, run_sm, y[r], n0 + r, 1.0f);
            }
        }
        if constexpr (EPI == EPI_VOCAB) {
#pragma unroll
            for (int off = 16; off < 64; off <<= 1) {
                const float mx2 = __shfl_xor(run_mx, off, 64), sm2 = __shfl_xor(run_sm, off, 64);
                const int arg2 = __shfl_xor(run_arg, off, 64);
                fc_argmax_merge(run_mx, run_arg, run_sm, mx2, arg2, sm2);
            }
            const int m = m0 + 16 * ti + rho;
            if (q == 0 && m < p.M) p.am.at(n_blk, m) = FcArgmax{run_mx, run_arg, run_sm};
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Attention of any supported shape: 16 QT query rows of a (sequence, kv head) per workgroup, its eight
// waves take the 32-key groups of the workgroup's key range in turn and are merged through LDS.
//
// S^T = K Q^T and O^T += V^T P^T on the 16x16 matrix instructions.  K rows and transposed V tiles are both in operand
// order, 16 bytes per lane.  Uncut (LDS), they come by way of LDS, where every wave has areas of its own: loaded straight
// into registers, with neighbouring lanes in different rows, a compute unit takes one lane a clock, 38 B/ns, and by direct-to-LDS
// loads of 64 bytes or more per row up to 138.  700 drawn shapes of 64 .. 2100 keys, with the ranges planned anew: fp32 rows of 64 / 128
// 1.075 / 1.14 x, bf16 rows of 64 1.13 x (288 keys, 8 heads x 16 rows: 6.4 -> 6.2, 11.1 -> 8.8, 4.6 -> 4.2 us); of it 1.03 x from dealing
// the workgroups to the XCDs by what they read.  fp32 is bound by its matrix rate (a group of 32 keys, rows of 64: 1024 clocks of scores).
// In ranges, a wave has one group or two and the longer way costs more than it brings (2 .. 9 %): straight into registers, and so for
// the up to three groups of bf16 rows of 128.  The queries come to LDS once per workgroup: operand-shaped, by each of its waves, they
// took as long as the keys (4 to 8 KB x 8 at a lane a clock, behind the keys and in two trips).  With that, without integer divisions
// ahead of the first load and with the last groups of fp32 dealt by halves, us: fp32 32 rows x 4 heads of 64, 256 / 288 / 544 keys
// 5.04 / 6.00 / 7.75 -> 4.79 / 5.48 / 7.42, in ranges 1056 keys 8.00 -> 7.36; 4 x 30 rows, 8 / 4 heads of 128, 400 keys 13.5 -> 11.8; bf16 rows of 128,
// 64 keys 3.78 -> 3.09.  (A second pair of areas, a group ahead: no gain.)  The accumulator of S^T
// puts keys 4 q + r of a 16-key group into register r of lane (query, q): for fp32 that is the operand
// layout of P^T (four 16x16x4 instructions, keys 4 q + j); for bf16 the K rows of the two groups are read
// permuted, so that the eight probabilities of a lane are the keys 8 q .. 8 q + 7.  No exchange for P.
//
// These caches are small: the kernel is bound by latency with few query rows and by the fp32 matrix
// rate with many.  A cache with a single workgroup per (head, tile) is cut into key ranges ("splits",
// planned on the host) whose partial states k_attn_tile_merge combines.  The plain-ALU kernel it replaces
// (a thread per key, then a thread per output column) took 22 us for the tiny configuration.
struct AttnTileArgs {
    const void *Q, *Kc, *Vc;
    const int32_t *pos;
    void *out;
    float *part_o, *part_ml;  // splits > 1: [bj][tile][split][16 QT][Dh], [bj][tile][split][16 QT][2]
    FcGeom G;
    int A, kv_len, tiles, splits, groups_per_split;
    float c;                  // softmax scale * log2(e)
    FcDivisor by_splits, by_tiles, by_hkv, by_a;
};

constexpr int AT_STRIDE = 4;  // padding floats per row of the exchange area

// Probabilities are fp32: for bf16 values of head_dim 64 they go into the output products as sums of three bf16 numbers,
// which hold all 24 bits (error against 64 bits 1.65e-3, what rounding the result costs; with probabilities in bf16
// 2.0e-3 and 1 to 4 % less time: 32 rows x 4 heads x 288 keys 4.32 against 4.2 us).  For bf16 of head_dim 128 they are
// rounded to bf16 as in the split-KV kernel; the planner chooses between the two by length.  The exponential is the
// hardware's, of a rounded product: over 40 fp32 shapes of 64 .. 2048 keys the error against 64 bits is 1.004 times
// that with expf (5e-7 at 288 keys, all from the sums), and the tiny configuration's step takes 10.6 us instead of 11.2.
template <typename T, int DH>
constexpr int prob_terms() { return Op<T>::KB == 8 && DH == 64 ? 3 : 1; }

template <typename T>
__device__ __forceinline__ void attn_store_row4(const AttnTileArgs &p, int bj, int row, int d0, float4 v)
{
    const FcGeom &G = p.G;
    if (row >= G.g * p.A) return;
    const int b = (int)p.by_hkv.over(bj), j = bj - b * G.Hkv, hg = (int)p.by_a.over(row), a = row - hg * p.A;
    if (p.pos) {  // padded row: same rule as the projection (negative or beyond the cache)
        const int pp = p.pos[b * p.A + a];
        if (pp < 0 || pp >= G.max_seq) v = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    const float y[4] = {v.x, v.y, v.z, v.w};
    store4((T *)p.out + ((size_t)b * p.A + a) * ((size_t)G.Hq * G.Dh) + (size_t)(j * G.g + hg) * G.Dh + d0, y);
}

// LDS of k_attn_tile: a wave's area holds KG keys and VG values of a group, or its results at the end.  20 KB at most, so that
// eight waves fit; fp32 rows of 128 come in halves of 16 keys where that takes it.
template <typename T, int DH, int QT, int DS, bool LDS>
struct AttnTileLds {
    static constexpr int KROW = DH * sizeof(T), VKEY = DH / DS * sizeof(T), MOST = 20 * 1024;
    static constexpr int KG = 32 * (KROW + VKEY) <= MOST ? 32 : 16;
    static constexpr int VG = KG * KROW + 32 * VKEY <= MOST ? 32 : 16;
    static constexpr int VROW = VG * sizeof(T);
    static constexpr int NK = KG * KROW / 1024, NVL = VG * VKEY / 1024;  // 1 KB loads
    static constexpr int STAGE = KG * KROW + VG * VKEY, STATE = QT * 16 * (DH / DS + AT_STRIDE + 2) * (int)sizeof(float);
    static constexpr int WAVE = ((LDS && STAGE > STATE ? STAGE : STATE) + 127) / 128 * 128;
    // The queries: 1 KB pieces, one per wave, behind the areas (BEHIND) or, where they do not fit there (fp32 rows of 128 with V in
    // four parts), at the start in the waves' areas for the values.  (Behind them it is 0.1 us less, 8 x 64 rows, 800 keys 0.3.)
    static constexpr int NQ = QT * 16 * KROW / 1024;
    static constexpr bool BEHIND = LDS && TW * WAVE + NQ * 1024 <= 160 * 1024;
    static constexpr int QAT = BEHIND ? TW * WAVE : LDS ? KG * KROW : 0, QSTEP = BEHIND ? 1024 : WAVE, BYTES = TW * WAVE + (BEHIND ? NQ * 1024 : 0);
    static_assert(NQ <= TW && (BEHIND || QAT + 1024 <= WAVE), "a piece of the queries per wave");
    static_assert(STAGE <= MOST && NVL >= 1, "areas");
    template <int ROWB>
    static __device__ __forceinline__ int swizzle(int row)
    {
        return ROWB >= 256 ? row & 15 : ROWB == 128 ? (row >> 1) & 7 : (row >> 2) & 3;
    }
};

template <typename T, int DH, int QT, int DS, bool LDS>
__global__ __launch_bounds__(TW * 64) void k_attn_tile(AttnTileArgs p)
{
    typedef Op<T> O;
    typedef typename O::frag frag;
    typedef AttnTileLds<T, DH, QT, DS, LDS> L;
    constexpr int KB = O::KB, NKB = DH / (4 * KB), DV = DH / DS, ND = DV / 16, ROW = DV + AT_STRIDE;
    constexpr bool F32 = KB == 4;
    constexpr int NV = F32 ? 2 : 1;  // V fragments per 16 head-dim rows and 32 keys
    constexpr int NP = prob_terms<T, DH>();
    extern __shared__ __align__(1024) unsigned char attn_smem[];
    const FcGeom &G = p.G;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho = lane & 15, q = lane >> 4;
    unsigned char *kbuf = attn_smem + wave * L::WAVE, *vbuf = kbuf + L::KG * L::KROW;
    // at the end: [16 QT][ROW] partial outputs and [16 QT][2] row states of every wave, in its area
    auto xo = [&](int w) { return (float *)(attn_smem + w * L::WAVE); };
    auto xml = [&](int w) { return xo(w) + QT * 16 * ROW; };
    // workgroup ids equal modulo 8 share an XCD: the workgroups, ordered by what they read, are dealt in equal contiguous runs
    const uint32_t n_wgs = (uint32_t)G.B * G.Hkv * p.tiles * p.splits * DS, xcd = blockIdx.x & 7;
    const uint32_t id = (uint32_t)((uint64_t)xcd * n_wgs >> 3) + (blockIdx.x >> 3);
    if (id >= (uint32_t)((uint64_t)(xcd + 1) * n_wgs >> 3)) return;
    const int dv0 = (int)(id % DS) * DV;  // this workgroup's part of the head dimension of V
    const int bt = (int)p.by_splits.over(id / DS), split = id / DS - bt * p.splits;
    const int bj = (int)p.by_tiles.over(bt), tile = bt - bj * p.tiles;
    const int b = (int)p.by_hkv.over(bj), j = bj - b * G.Hkv;
    const T *kc = (const T *)p.Kc + (size_t)bj * G.spad * DH, *vc = (const T *)p.Vc + (size_t)bj * G.spad * DH;

    const int n_groups = (p.kv_len + 31) / 32;
    const int g0 = split * p.groups_per_split, g1 = min(n_groups, g0 + p.groups_per_split);
    // The wave's groups: every eighth.  fp32, which the matrix rate binds: up to four groups left for the last round are dealt by halves,
    // so that a SIMD has half a group more than another and not a whole one.
    const int rest = (g1 - g0) % TW;
    const bool halves = LDS && F32 && rest >= 1 && rest <= TW / 2;
    const int rounds = (g1 - g0) / TW, last0 = g0 + rounds * TW;
    const int n = rounds + (halves ? 32 * last0 + 16 * wave < min(p.kv_len, 32 * g1) : wave < rest);
    auto group_of = [&](int i) { return halves && i == rounds ? last0 + (wave >> 1) : g0 + wave + i * TW; };
    // key of row i of 16-key half h: fp32 in order; bf16 so that register pairs of the two halves are 8 keys in a row
    auto key_of = [&](int h, int i) { return F32 ? 16 * h + i : 8 * (i >> 2) + 4 * h + (i & 3); };
    // Part `part` of group g to LDS, in pieces of 1 KB; a row's 16-byte chunks are permuted so that 16 rows' chunks of one
    // column fall into 16 different bank groups.
    auto issue_k = [&](int i, int part) {
        const int g = group_of(i);
#pragma unroll
        for (int l = 0; l < L::NK; ++l) {
            const int at = 1024 * l + 16 * lane, row = at / L::KROW, c = (at % L::KROW) >> 4, r = part * L::KG + row;
            const unsigned char *src = (const unsigned char *)kc + (size_t)(32 * g + key_of(r >> 4, r & 15)) * L::KROW;
            fc_load_lds16(src + 16 * (c ^ L::template swizzle<L::KROW>(row)), kbuf + 1024 * l);
        }
    };
    auto issue_v = [&](int i, int part) {
        const int g = group_of(i);
        const unsigned char *vt = (const unsigned char *)(vc + (size_t)(g >> 1) * (FC_VTILE * DH) + 32 * (g & 1) + L::VG * part);
#pragma unroll
        for (int l = 0; l < L::NVL; ++l) {
            const int at = 1024 * l + 16 * lane, row = at / L::VROW, c = (at % L::VROW) >> 4;
            fc_load_lds16(vt + (size_t)(dv0 + row) * (FC_VTILE * sizeof(T)) + 16 * (c ^ L::template swizzle<L::VROW>(row)), vbuf + 1024 * l);
        }
    };
    frag kd[2][NKB], vd[ND][NV];  // without LDS
    auto load_k = [&](int g) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int k = 0; k < NKB; ++k)
                kd[h][k] = *(const frag *)(kc + (size_t)(32 * g + key_of(h, rho)) * DH + 4 * KB * k + KB * q);
    };
    // Queries (rows past the end take row 0's, their results are never stored): a wave brings 1 KB of them to LDS, ahead of its keys, and all
    // read them there.  Loaded by every wave straight into registers they took a compute unit 0.86 us, a lane a clock.
    auto query_row = [&](int at) {
        const int row = at < G.g * p.A ? at : 0, hg = (int)p.by_a.over(row), a = row - hg * p.A;
        return (const unsigned char *)p.Q + (((size_t)b * G.Hq + j * G.g + hg) * p.A + a) * L::KROW;
    };
    if (wave < L::NQ) {
        const int at = 1024 * wave + 16 * lane, row = at / L::KROW, c = (at % L::KROW) >> 4;
        const unsigned char *src = query_row(tile * (16 * QT) + row) + 16 * (c ^ L::template swizzle<L::KROW>(row));
        unsigned char *dst = attn_smem + L::QAT + wave * L::QSTEP;
        if (((uintptr_t)p.Q & 15) == 0) fc_load_lds16(src, dst);
        else *(uint4 *)(dst + 16 * lane) = fc_load_any<uint4>(src);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (n > 0) {
        if (LDS) issue_k(0, 0);
        else load_k(g0 + wave);
        if (L::BEHIND) issue_v(0, 0);
        __builtin_amdgcn_sched_barrier(0);
        fc_wait_vm<!LDS ? 2 * NKB : L::BEHIND ? L::NK + L::NVL : L::NK, true>();
    } else {
        fc_wait_vm<0, true>();
    }
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    frag qf[QT][NKB];
#pragma unroll
    for (int u = 0; u < QT; ++u)
#pragma unroll
        for (int k = 0; k < NKB; ++k) {
            const int row = 16 * u + rho, at = row * L::KROW + 16 * ((4 * k + q) ^ L::template swizzle<L::KROW>(row));
            qf[u][k] = *(const frag *)(attn_smem + L::QAT + (at >> 10) * L::QSTEP + (at & 1023));
        }
    fc_wait_lds();
    if constexpr (!L::BEHIND) {  // (without LDS: the areas are written at the end only, by then every wave may be past its reads)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (LDS && n > 0) issue_v(0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    f32x4 o[QT][ND];
    float m[QT], l[QT];
#pragma unroll
    for (int u = 0; u < QT; ++u) {
#pragma unroll
        for (int d = 0; d < ND; ++d) o[u][d] = f32x4{0.f, 0.f, 0.f, 0.f};
        m[u] = -INFINITY;
        l[u] = 0.f;
    }
    // The wave's groups from .. to - 1, WHOLE or the HALF of one that it got, in a loop of their own: with tests for halves among the matrix
    // instructions those no longer go beside the softmax (fp32 rows of 128, two layers, us before / with the tests / now: 16 / 4 heads, 92 rows,
    // 1969 keys 91 / 96.6 / 90.5, 60 rows 62.4 / 56.5 / 57.2; 16 / 8 heads, 400 rows, 1900 keys 234 / 244 / 234).
    constexpr int WHOLE = 0, HALF = 1;
    auto take = [&](int from, int to, auto form) {
        constexpr int FORM = decltype(form)::value;
        for (int i = from; i < to; ++i) {
            const int g = group_of(i), half = FORM == HALF ? wave & 1 : -1;  // -1: both
            const bool more = FORM == WHOLE && i + 1 < n;
            if constexpr (!LDS) {
                const T *vt = vc + (size_t)(g >> 1) * (FC_VTILE * DH) + 32 * (g & 1);
#pragma unroll
                for (int d = 0; d < ND; ++d)
#pragma unroll
                    for (int h = 0; h < NV; ++h)
                        vd[d][h] = *(const frag *)(vt + (dv0 + 16 * d + rho) * FC_VTILE + (F32 ? 16 * h : 0) + KB * q);
            }
            f32x4 s[QT][2];
#pragma unroll
            for (int u = 0; u < QT; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h) s[u][h] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (LDS) {
#pragma unroll
                for (int part = 0; part < 32 / L::KG; ++part) {
                    if (part == 0) fc_wait_vm<L::NVL>();  // these keys are here; the values behind them may stay in flight
                    else fc_wait_vm<0>();
                    __builtin_amdgcn_sched_barrier(0);
                    frag kf[L::KG / 16][NKB];
#pragma unroll
                    for (int h = 0; h < L::KG / 16; ++h)
#pragma unroll
                        for (int k = 0; k < NKB; ++k)
                            kf[h][k] = *(const frag *)(kbuf + (16 * h + rho) * L::KROW + 16 * ((4 * k + q) ^ L::template swizzle<L::KROW>(16 * h + rho)));
                    fc_wait_lds();  // lgkmcnt(0): the area may be overwritten
                    __builtin_amdgcn_sched_barrier(0);
                    if (part + 1 < 32 / L::KG) issue_k(i, part + 1);
                    else if (more) issue_k(i + 1, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    auto scores = [&](auto first, auto last) {  // 16-key halves first .. last - 1 of the part
#pragma unroll
                        for (int k = 0; k < NKB; ++k)
#pragma unroll
                            for (int u = 0; u < QT; ++u)
#pragma unroll
                                for (int h = decltype(first)::value; h < decltype(last)::value; ++h)
                                    s[u][part * (L::KG / 16) + h] = O::mfma(kf[h][k], qf[u][k], s[u][part * (L::KG / 16) + h]);
                    };
                    const std::integral_constant<int, 0> c0;
                    const std::integral_constant<int, 1> c1;
                    const std::integral_constant<int, L::KG / 16> c2;
                    if (half < 0) scores(c0, c2);
                    else if (L::KG == 16) {
                        if (half == part) scores(c0, c1);
                    } else if (half == 0) scores(c0, c1);
                    else scores(c1, c2);
                }
            } else {
#pragma unroll
                for (int u = 0; u < QT; ++u)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int k = 0; k < NKB; ++k) s[u][h] = O::mfma(kd[h][k], qf[u][k], s[u][h]);
                if (more) load_k(g + TW);  // the next group's keys travel behind the softmax and the output products
            }
            if (half >= 0) {
#pragma unroll
                for (int u = 0; u < QT; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (half == 1) s[u][0][r] = -INFINITY;
                        else s[u][1][r] = -INFINITY;
                    }
            }
            const bool past = 32 * g + 32 > p.kv_len;  // keys past the end may hold anything: no score, and zero values (0 * V stays 0)
            if (past) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (32 * g + key_of(h, 4 * q + r) >= p.kv_len) {
#pragma unroll
                            for (int u = 0; u < QT; ++u) s[u][h][r] = -INFINITY;
                        }
            }
            frag pf[QT][F32 ? NV : NP];
#pragma unroll
            for (int u = 0; u < QT; ++u) {
                float mx = s[u][0][0];
#pragma unroll
                for (int r = 1; r < 8; ++r) mx = fmaxf(mx, s[u][r >> 2][r & 3]);
                const float m_new = fmaxf(m[u], max_rows(mx));
                const float alpha = __builtin_amdgcn_exp2f((m[u] - m_new) * p.c);
                m[u] = m_new;
                l[u] *= alpha;
                float pr[8];
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    pr[r] = __builtin_amdgcn_exp2f((s[u][r >> 2][r & 3] - m_new) * p.c);
                    l[u] += pr[r];
                }
#pragma unroll
                for (int d = 0; d < ND; ++d)
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[u][d][r] *= alpha;
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    if constexpr (F32) {
                        pf[u][r >> 2][r & 3] = pr[r];
                    } else {
#pragma unroll
                        for (int h = 0; h < NP; ++h) {
                            pf[u][h][r] = (__bf16)pr[r];
                            pr[r] -= (float)pf[u][h][r];  // (exact)
                        }
                    }
                }
            }
            if constexpr (LDS) {
#pragma unroll
                for (int part = 0; part < 32 / L::VG; ++part) {
                    if (part == 0 && more) fc_wait_vm<L::NK>();  // these values are here; the next keys may stay in flight
                    else fc_wait_vm<0>();
                    __builtin_amdgcn_sched_barrier(0);
                    constexpr int NVP = NV * L::VG / 32;  // fragments per 16 rows
                    frag vf[ND][NVP];
#pragma unroll
                    for (int d = 0; d < ND; ++d)
#pragma unroll
                        for (int h = 0; h < NVP; ++h)
                            vf[d][h] = *(const frag *)(vbuf + (16 * d + rho) * L::VROW + 16 * ((4 * h + q) ^ L::template swizzle<L::VROW>(16 * d + rho)));
                    fc_wait_lds();
                    __builtin_amdgcn_sched_barrier(0);
                    if (part + 1 < 32 / L::VG) issue_v(i, part + 1);
                    else if (more) issue_v(i + 1, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    if (past) {
#pragma unroll
                        for (int d = 0; d < ND; ++d)
#pragma unroll
                            for (int h = 0; h < NVP; ++h)
#pragma unroll
                                for (int e = 0; e < KB; ++e)
                                    if (32 * g + L::VG * part + (F32 ? 16 * h : 0) + KB * q + e >= p.kv_len) vf[d][h][e] = {};
                    }
#pragma unroll
                    for (int h = 0; h < (F32 ? NVP : NP); ++h) {
                        if (half >= 0 && half != NVP * part + h) continue;
#pragma unroll
                        for (int u = 0; u < QT; ++u)
#pragma unroll
                            for (int d = 0; d < ND; ++d) o[u][d] = O::mfma(vf[d][F32 ? h : 0], pf[u][F32 ? NVP * part + h : h], o[u][d]);
                    }
                }
            } else {
                if (past) {
#pragma unroll
                    for (int d = 0; d < ND; ++d)
#pragma unroll
                        for (int h = 0; h < NV; ++h)
#pragma unroll
                            for (int e = 0; e < KB; ++e)
                                if (32 * g + (F32 ? 16 * h : 0) + KB * q + e >= p.kv_len) vd[d][h][e] = {};
                }
#pragma unroll
                for (int u = 0; u < QT; ++u)
#pragma unroll
                    for (int d = 0; d < ND; ++d)
#pragma unroll
                        for (int h = 0; h < (F32 ? NV : NP); ++h) o[u][d] = O::mfma(vd[d][F32 ? h : 0], pf[u][h], o[u][d]);
            }
        }
    };
    take(0, halves ? rounds : n, std::integral_constant<int, WHOLE>());
    if constexpr (F32 && LDS)
        if (halves) take(rounds, n, std::integral_constant<int, HALF>());

    // ---- merge the eight waves through LDS
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        const float lu = sum_rows(l[u]);
        float *row = xo(wave) + (16 * u + rho) * ROW + 4 * q;
#pragma unroll
        for (int d = 0; d < ND; ++d) *(f32x4 *)(row + 16 * d) = o[u][d];
        if (q == 0) {
            float *ml = xml(wave) + (16 * u + rho) * 2;
            ml[0] = m[u];
            ml[1] = lu;
        }
    }
    __syncthreads();
    for (int idx = tid; idx < QT * 16 * (DV / 4); idx += TW * 64) {
        const int row = idx / (DV / 4), d0 = 4 * (idx % (DV / 4));
        float mm = -INFINITY;
#pragma unroll
        for (int w = 0; w < TW; ++w) mm = fmaxf(mm, xml(w)[row * 2]);
        float den = 0.f;
        float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < TW; ++w) {
            const float *ml = xml(w) + row * 2;
            const float k = __builtin_amdgcn_exp2f((ml[0] - mm) * p.c);
            const float4 v = *(const float4 *)(xo(w) + row * ROW + d0);
            den += k * ml[1];
            num.x += k * v.x;
            num.y += k * v.y;
            num.z += k * v.z;
            num.w += k * v.w;
        }
        if (p.splits > 1) {
            const size_t at = ((size_t)bt * p.splits + split) * (QT * 16) + row;
            *(float4 *)(p.part_o + at * DH + dv0 + d0) = num;
            if (dv0 + d0 == 0) *(float2 *)(p.part_ml + at * 2) = make_float2(mm, den);
        } else {
            attn_store_row4<T>(p, bj, tile * (16 * QT) + row, dv0 + d0, make_float4(num.x / den, num.y / den, num.z / den, num.w / den));
        }
    }
}

// Merge of the key ranges: one workgroup per (sequence, kv head, tile), a thread per four output values.
template <typename T, int DH, int QT>
__global__ __launch_bounds__(256) void k_attn_tile_merge(AttnTileArgs p)
{
    const int bt = blockIdx.x / (QT * DH / 64), idx = (blockIdx.x % (QT * DH / 64)) * 256 + threadIdx.x;
    const int row = idx / (DH / 4), d0 = 4 * (idx % (DH / 4));
    const size_t at = (size_t)bt * p.splits * (QT * 16) + row;
    float mm = -INFINITY, den = 0.f;
    float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
    constexpr int U = 8;  // ranges whose loads are in flight together
    for (int s0 = 0; s0 < p.splits; s0 += U) {
        float2 ml[U];
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t as = at + (size_t)min(s0 + u, p.splits - 1) * (QT * 16);
            ml[u] = *(const float2 *)(p.part_ml + as * 2);
            v[u] = *(const float4 *)(p.part_o + as * DH + d0);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + u >= p.splits) break;
            const float m_new = fmaxf(mm, ml[u].x);
            const float k0 = __builtin_amdgcn_exp2f((mm - m_new) * p.c), k1 = __builtin_amdgcn_exp2f((ml[u].x - m_new) * p.c);
            mm = m_new;
            den = den * k0 + ml[u].y * k1;
            num.x = num.x * k0 + v[u].x * k1;
            num.y = num.y * k0 + v[u].y * k1;
            num.z = num.z * k0 + v[u].z * k1;
            num.w = num.w * k0 + v[u].w * k1;
        }
    }
    const int bj = (int)p.by_tiles.over(bt);
    attn_store_row4<T>(p, bj, (bt - bj * p.tiles) * (16 * QT) + row, d0,
                       make_float4(num.x / den, num.y / den, num.z / den, num.w / den));
}

// ---------------------------------------------------------------------------------------------
// RMS normalisation, one block per row: out = x / sqrt(mean(x^2) + eps) * weight.
template <typename T>
__global__ __launch_bounds__(256) void k_rmsnorm(const T *X, const T *__restrict__ w, float eps, int d, T *out)
{
    __shared__ float red[4];
    const size_t row = blockIdx.x;
    const T *x = X + row * d;
    const int tid = threadIdx.x;
    float ss = 0.f;
    for (int k = tid; k < d; k += 256) {
        const float v = fc_to_float(x[k]);
        ss += v * v;
    }
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    const float tot = (red[0] + red[1]) + (red[2] + red[3]);
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
    // out may be x: element k is read and written by the same thread only
    for (int k = tid; k < d; k += 256) out[row * d + k] = fc_from_float<T>(fc_to_float(x[k]) * inv * fc_to_float(w[k]));
}

// fp32 rows whose length is a multiple of 4 and at most 1024 NJ: as below.  (Hidden 384, 40 rows: 3.4 us with a second
// pass over the row and the weight behind the sum, now 2.9.)
template <int NJ>
__global__ __launch_bounds__(256) void k_rmsnorm_f32_row(const float *X, const float *__restrict__ w, float eps, int d, float *out)
{
    __shared__ float red[4];
    const size_t row = blockIdx.x;
    const int tid = threadIdx.x, chunks = d >> 2;
    float4 v[NJ], g[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int c = tid + 256 * j;
        v[j] = c < chunks ? *(const float4 *)(X + row * d + 4 * c) : make_float4(0.f, 0.f, 0.f, 0.f);
        g[j] = c < chunks ? *(const float4 *)(w + 4 * c) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) ss += (v[j].x * v[j].x + v[j].y * v[j].y) + (v[j].z * v[j].z + v[j].w * v[j].w);
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    const float tot = (red[0] + red[1]) + (red[2] + red[3]);
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int c = tid + 256 * j;
        if (c < chunks)
            *(float4 *)(out + row * d + 4 * c) = make_float4(v[j].x * inv * g[j].x, v[j].y * inv * g[j].y, v[j].z * inv * g[j].z,
                                                             v[j].w * inv * g[j].w);
    }
}

// bf16 rows whose length is a multiple of 8 and at most 2048 * NJ: every thread keeps its NJ 16-byte
// pieces of the row in registers, so the row is read once.
template <int NJ>
__global__ __launch_bounds__(256) void k_rmsnorm_bf16_row(const uint16_t *X, const uint16_t *__restrict__ w, float eps,
                                                          int d, uint16_t *out)
{
    __shared__ float red[4];
    const size_t row = blockIdx.x;
    const int tid = threadIdx.x, chunks = d >> 3;
    uint4 v[NJ], g[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int c = tid + 256 * j;
        v[j] = c < chunks ? *(const uint4 *)(X + row * d + 8 * c) : make_uint4(0, 0, 0, 0);
        g[j] = c < chunks ? *(const uint4 *)(w + 8 * c) : make_uint4(0, 0, 0, 0);
    }
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const uint32_t u[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float a = __uint_as_float(u[e] << 16), b = __uint_as_float(u[e] & 0xffff0000u);
            ss += a * a;
            ss += b * b;
        }
    }
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    const float tot = (red[0] + red[1]) + (red[2] + red[3]);
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int c = tid + 256 * j;
        if (c >= chunks) continue;
        const uint32_t u[4] = {v[j].x, v[j].y, v[j].z, v[j].w}, gw[4] = {g[j].x, g[j].y, g[j].z, g[j].w};
        uint32_t o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float a = __uint_as_float(u[e] << 16) * inv * __uint_as_float(gw[e] << 16);
            const float b = __uint_as_float(u[e] & 0xffff0000u) * inv * __uint_as_float(gw[e] & 0xffff0000u);
            o[e] = (uint32_t)fc_bf16_bits(a) | ((uint32_t)fc_bf16_bits(b) << 16);
        }
        *(uint4 *)(out + row * d + 8 * c) = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

// ---------------------------------------------------------------------------------------------
// KV drift diagnostic: cosine similarity over the head dimension between rows of the cache and an
// earlier snapshot of the same rows in the plain [B][Hkv][rows][Dh] layout.  One wave per
// (sequence, kv head, row); lanes run along the head dimension.
template <typename T>
__global__ __launch_bounds__(64) void k_kv_similarity(FcGeom G, const T *__restrict__ kc, const T *__restrict__ vc,
                                                      const T *__restrict__ k_prev, const T *__restrict__ v_prev,
                                                      int start, int rows, float *sim_k, float *sim_v)
{
    const int r = blockIdx.x, j = blockIdx.y, b = blockIdx.z, lane = threadIdx.x;
    const size_t old = (((size_t)b * G.Hkv + j) * rows + r) * G.Dh;
    float dk = 0.f, nk = 0.f, pk = 0.f, dv = 0.f, nv = 0.f, pv = 0.f;
    for (int i = lane; i < G.Dh; i += 64) {
        const float xk = fc_to_float(kc[fc_k_index(G, b, j, start + r, i)]), yk = fc_to_float(k_prev[old + i]);
        const float xv = fc_to_float(vc[fc_v_index(G, b, j, start + r, i)]), yv = fc_to_float(v_prev[old + i]);
        dk += xk * yk;
        nk += xk * xk;
        pk += yk * yk;
        dv += xv * yv;
        nv += xv * xv;
        pv += yv * yv;
    }
    dk = wave_sum(dk);
    nk = wave_sum(nk);
    pk = wave_sum(pk);
    dv = wave_sum(dv);
    nv = wave_sum(nv);
    pv = wave_sum(pv);
    if (lane == 0) {
        const size_t o = ((size_t)b * G.Hkv + j) * rows + r;
        sim_k[o] = (nk > 0.f && pk > 0.f) ? dk / (sqrtf(nk) * sqrtf(pk)) : 0.f;
        sim_v[o] = (nv > 0.f && pv > 0.f) ? dv / (sqrtf(nv) * sqrtf(pv)) : 0.f;
    }
}

}  // namespace

hipError_t fc_launch_kv_similarity(const FcGeom &G, int dtype, const void *k_layer, const void *v_layer,
                                   const void *k_prev, const void *v_prev, int start, int rows, float *sim_k,
                                   float *sim_v, hipStream_t s)
{
    const dim3 grid((unsigned)rows, (unsigned)G.Hkv, (unsigned)G.B);
    if (dtype == FC_F32)
        k_kv_similarity<float><<<grid, dim3(64), 0, s>>>(G, (const float *)k_layer, (const float *)v_layer,
                                                         (const float *)k_prev, (const float *)v_prev, start, rows, sim_k,
                                                         sim_v);
    else
        k_kv_similarity<bf16_t><<<grid, dim3(64), 0, s>>>(G, (const bf16_t *)k_layer, (const bf16_t *)v_layer,
                                                          (const bf16_t *)k_prev, (const bf16_t *)v_prev, start, rows,
                                                          sim_k, sim_v);
    return hipGetLastError();
}

hipError_t fc_launch_copy_rows(const FcGeom &G, int dtype, void *k_layer, void *v_layer, void *k_rows,
                               void *v_rows, int start, int rows, bool to_cache, hipStream_t s)
{
    const size_t total = (size_t)G.B * G.Hkv * rows * G.Dh;
    size_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks == 0) return hipSuccess;
    if (dtype == FC_F32)
        k_copy_rows<float><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(
            G, (float *)k_layer, (float *)v_layer, (float *)k_rows, (float *)v_rows, start, rows, to_cache);
    else
        k_copy_rows<bf16_t><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(
            G, (bf16_t *)k_layer, (bf16_t *)v_layer, (bf16_t *)k_rows, (bf16_t *)v_rows, start, rows,
            to_cache);
    return hipGetLastError();
}

hipError_t fc_launch_rmsnorm(int dtype, const void *x, const void *weight, float eps, int rows, int d,
                             void *out, hipStream_t s)
{
    const bool aligned = (((uintptr_t)x | (uintptr_t)weight | (uintptr_t)out) & 15) == 0;
    if (dtype == FC_F32 && d % 4 == 0 && d <= 4096 && aligned) {
        const float *xf = (const float *)x, *wf = (const float *)weight;
        if (d <= 1024)
            k_rmsnorm_f32_row<1><<<dim3((unsigned)rows), dim3(256), 0, s>>>(xf, wf, eps, d, (float *)out);
        else
            k_rmsnorm_f32_row<4><<<dim3((unsigned)rows), dim3(256), 0, s>>>(xf, wf, eps, d, (float *)out);
    } else if (dtype == FC_F32)
        k_rmsnorm<float><<<dim3((unsigned)rows), dim3(256), 0, s>>>((const float *)x, (const float *)weight, eps,
                                                                    d, (float *)out);
    else if (d % 8 == 0 && d <= 8192 && aligned) {
        const uint16_t *xb = (const uint16_t *)x, *wb = (const uint16_t *)weight;
        if (d <= 2048)
            k_rmsnorm_bf16_row<1><<<dim3((unsigned)rows), dim3(256), 0, s>>>(xb, wb, eps, d, (uint16_t *)out);
        else if (d <= 4096)
            k_rmsnorm_bf16_row<2><<<dim3((unsigned)rows), dim3(256), 0, s>>>(xb, wb, eps, d, (uint16_t *)out);
        else
            k_rmsnorm_bf16_row<4><<<dim3((unsigned)rows), dim3(256), 0, s>>>(xb, wb, eps, d, (uint16_t *)out);
    } else
        k_rmsnorm<bf16_t><<<dim3((unsigned)rows), dim3(256), 0, s>>>((const bf16_t *)x, (const bf16_t *)weight,
                                                                     eps, d, (bf16_t *)out);
    return hipGetLastError();
}

namespace {

template <typename T, int NT, int MT, int U, int EPI, bool LDS>
hipError_t launch_tile_u(TileArgs a, int n_tiles, hipStream_t s)
{
    constexpr size_t BYTES = tile_lds(NT, MT, U, LDS);
    static hipError_t attr = hipFuncSetAttribute((const void *)k_linear_tile<T, NT, MT, U, EPI, LDS>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)BYTES);
    if (attr != hipSuccess) return attr;
    a.n_blocks = (n_tiles + NT - 1) / NT;
    a.by_blocks.set(a.n_blocks);
    const int64_t grid = (int64_t)a.n_blocks * ((a.M + 16 * MT - 1) / (16 * MT));
    if (grid > INT32_MAX) return hipErrorInvalidValue;
    k_linear_tile<T, NT, MT, U, EPI, LDS><<<dim3((unsigned)grid), dim3(TW * 64), BYTES, s>>>(a);
    return hipGetLastError();
}

// Tile choice.  These problems are bound by the latency of a wave's chain of loads and multiplies, so what counts is
// that every compute unit has a workgroup and that several share one: 16 or 32 window rows per workgroup (about 60
// registers: four workgroups per compute unit; 138 rows x 3072 x 512 took 28 us in tiles of 64 rows, 200 registers),
// and 64 rows x two weight tiles, which halve the traffic, only for many rounds of workgroups.  A long hidden dimension
// with few workgroups keeps four blocks in flight per wave instead of two (with two weight tiles as well that costs more
// than it brings: 20 x 3584 x 9001 in bf16 27.1 us with two, 32.3 with four).  Not so bf16 in tiles of 32 rows: with four
// blocks the compiler (clang 22, ROCm 7.2) hands registers of waiting X fragments to address arithmetic (v[10:17] in the
// loop of the residual layer), and every result is wrong.  The vocabulary takes two weight tiles always: its parts are
// workspace.
template <typename T, int EPI>
hipError_t launch_tile_t(const TileArgs &a, int n_tiles, hipStream_t s)
{
    constexpr int NT = EPI == EPI_VOCAB ? 2 : 1;
    const int64_t blocks = (n_tiles + NT - 1) / NT;
    auto wgs = [&](int mt) { return blocks * ((a.M + 16 * mt - 1) / (16 * mt)); };
    // By way of LDS: two blocks a step always (four leave one workgroup per compute unit where there were two: 6 % slower), and
    // the tile with the fewest rounds of 256 workgroups by what a workgroup takes, 1 : 1.7 for 16 and 32 rows; bf16, which its
    // matrix rate does not bind, also 64 rows x two weight tiles, 3 (fp32 would be 7; us at 16 / 32 / 64 rows: gated
    // fp32 160 x 512 x 2048 13.9 / 12.8, 160 x 512 x 1024 8.6 / 9.0; 700 x 512 x 2048 25.8 / 23.0 / 25.5; bf16 64 x 1000 x 6000
    // 12.8 / 10.2 / 8.2).
    if (a.K % (4 * Op<T>::KB) == 0 && (((uintptr_t)a.X | (uintptr_t)a.W | (uintptr_t)a.W2) & 15) == 0) {
        auto rounds = [&](int64_t n) { return (double)((n + 255) / 256); };
        const double one = rounds(wgs(1)), two = 1.7 * rounds(wgs(2));
        if constexpr (sizeof(T) == 2)
            if (a.M > 32 && 3.0 * rounds((n_tiles + 1) / 2 * (int64_t)((a.M + 63) / 64)) < fmin(one, two))
                return launch_tile_u<T, 2, 4, 2, EPI, true>(a, n_tiles, s);
        return a.M > 16 && two < one ? launch_tile_u<T, NT, 2, 2, EPI, true>(a, n_tiles, s) : launch_tile_u<T, NT, 1, 2, EPI, true>(a, n_tiles, s);
    }
    const bool deep = (a.K + 4 * Op<T>::KB - 1) / (4 * Op<T>::KB) >= 8 * TW;
    if (a.M > 32 && wgs(2) >= 4096) return launch_tile_u<T, 2, 4, 2, EPI, false>(a, n_tiles, s);
    if (a.M > 16 && wgs(2) >= 256) {
        if constexpr (sizeof(T) == 4 && NT == 1)
            if (deep && wgs(2) <= 512) return launch_tile_u<T, NT, 2, 4, EPI, false>(a, n_tiles, s);
        return launch_tile_u<T, NT, 2, 2, EPI, false>(a, n_tiles, s);
    }
    if constexpr (NT == 1)
        if (deep && wgs(1) <= 512) return launch_tile_u<T, NT, 1, 4, EPI, false>(a, n_tiles, s);
    return launch_tile_u<T, NT, 1, 2, EPI, false>(a, n_tiles, s);
}

template <int EPI>
hipError_t launch_tile(int dtype, const TileArgs &a, int n_tiles, hipStream_t s)
{
    return dtype == FC_F32 ? launch_tile_t<float, EPI>(a, n_tiles, s) : launch_tile_t<bf16_t, EPI>(a, n_tiles, s);
}

template <typename T, int DH, int QT, int DS, bool LDS>
hipError_t launch_attn_tile(const AttnTileArgs &a, hipStream_t s)
{
    constexpr size_t BYTES = AttnTileLds<T, DH, QT, DS, LDS>::BYTES;
    static hipError_t attr = hipFuncSetAttribute((const void *)k_attn_tile<T, DH, QT, DS, LDS>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)BYTES);
    if (attr != hipSuccess) return attr;
    const int64_t bt = (int64_t)a.G.B * a.G.Hkv * a.tiles;
    if (bt * a.splits > (1 << 30) || bt * (QT * DH / 64) > (1 << 30)) return hipErrorInvalidValue;
    k_attn_tile<T, DH, QT, DS, LDS><<<dim3((unsigned)((bt * a.splits * DS + 7) / 8 * 8)), dim3(TW * 64), BYTES, s>>>(a);
    if constexpr (!LDS && (Op<T>::KB != 8 || DH != 128))  // (the others are never cut)
        if (a.splits > 1) k_attn_tile_merge<T, DH, QT><<<dim3((unsigned)(bt * (QT * DH / 64))), dim3(256), 0, s>>>(a);
    return hipGetLastError();
}

// With a quarter or half of the compute units at most, the head dimension of V is cut in four or two: every part
// repeats the scores, but the values it loads, its output products and the merge of its waves shrink (fp32, head_dim 64,
// 8 workgroups, 288 keys: 8.4 us uncut, 6.5 in four; 861 keys in two ranges, with the merge 11.4 and 9.5).  With more workgroups
// it costs more than it brings (144 of head_dim 128, 305 keys: 12.3 us, 18.5 in halves).
template <typename T, int DH, bool LDS>
hipError_t launch_attn_tile_t(int qt, const AttnTileArgs &a, hipStream_t s)
{
    if constexpr (DH == 64)
        if (qt == 2) return launch_attn_tile<T, DH, 2, 1, LDS>(a, s);
    if (qt != 1) return hipErrorInvalidValue;
    const int64_t wgs = (int64_t)a.G.B * a.G.Hkv * a.tiles * a.splits;
    if (wgs <= 64) return launch_attn_tile<T, DH, 1, 4, LDS>(a, s);
    if (wgs <= 128) return launch_attn_tile<T, DH, 1, 2, LDS>(a, s);
    return launch_attn_tile<T, DH, 1, 1, LDS>(a, s);
}

}  // namespace

hipError_t fc_launch_project_tile(const FcGeom &G, const double *inv_freq, int dtype, const void *x, const void *w,
                                  const void *bias, const int32_t *pos, int win_start, int A, void *q_out, void *k_layer,
                                  void *v_layer, hipStream_t s)
{
    TileArgs a;
    memset(&a, 0, sizeof a);
    a.X = x;
    a.W = w;
    a.aux = bias;
    a.out = q_out;
    a.M = G.B * A;
    a.K = G.d;
    a.N = (G.Hq + 2 * G.Hkv) * G.Dh;
    a.G = G;
    a.pos = pos;
    a.win_start = win_start;
    a.A = A;
    a.by_a.set(A);
    a.Kc = k_layer;
    a.Vc = v_layer;
    memcpy(a.inv_freq, inv_freq, sizeof a.inv_freq);
    return launch_tile<EPI_QKV>(dtype, a, a.N / 16, s);
}

hipError_t fc_launch_linear_tile(int dtype, int mode, const void *x, const void *w, const void *aux, int M, int K, int N,
                                 void *out, hipStream_t s)
{
    TileArgs a;
    memset(&a, 0, sizeof a);
    a.X = x;
    a.W = w;
    a.out = out;
    a.M = M;
    a.K = K;
    a.N = N;
    a.G.Dh = 64;  // not used
    if (mode == FC_LIN_GATE_UP) {
        a.W2 = aux;
        return launch_tile<EPI_GATE_UP>(dtype, a, (N + 7) / 8, s);
    }
    a.aux = aux;
    return launch_tile<EPI_RESIDUAL>(dtype, a, (N + 15) / 16, s);
}

hipError_t fc_launch_lmhead_tile(int dtype, const void *x, const void *w, int M, int K, int V, const FcArgmaxPart &am,
                                 hipStream_t s)
{
    TileArgs a;
    memset(&a, 0, sizeof a);
    a.X = x;
    a.W = w;
    a.M = M;
    a.K = K;
    a.N = V;
    a.G.Dh = 64;  // not used
    a.am = am;
    return launch_tile<EPI_VOCAB>(dtype, a, (V + 15) / 16, s);
}

hipError_t fc_launch_attention_tile(const FcGeom &G, const FcAttnPlan &pl, int dtype, const void *q, const void *k_layer,
                                    const void *v_layer, const int32_t *pos, int A, int kv_len, void *out,
                                    void *workspace, hipStream_t s)
{
    AttnTileArgs a;
    memset(&a, 0, sizeof a);
    a.Q = q;
    a.Kc = k_layer;
    a.Vc = v_layer;
    a.pos = pos;
    a.out = out;
    a.G = G;
    a.A = A;
    a.kv_len = kv_len;
    a.tiles = (int)(((int64_t)G.g * A + 16 * pl.tiles_per_wg - 1) / (16 * pl.tiles_per_wg));
    a.splits = pl.splits;
    a.groups_per_split = pl.keys_per_split / 32;
    a.c = G.scale * 1.4426950408889634f;
    a.by_splits.set(a.splits);
    a.by_tiles.set(a.tiles);
    a.by_hkv.set(G.Hkv);
    a.by_a.set(A);
    if (pl.splits > 1) {
        if (!workspace) return hipErrorInvalidValue;
        a.part_o = (float *)workspace;
        a.part_ml = a.part_o + (size_t)G.B * G.Hkv * a.tiles * pl.splits * 16 * pl.tiles_per_wg * G.Dh;
    }
    const int qt = pl.tiles_per_wg;
    if (pl.splits == 1) {
        if (dtype == FC_F32) return G.Dh == 64 ? launch_attn_tile_t<float, 64, true>(qt, a, s) : G.Dh == 128 ? launch_attn_tile_t<float, 128, true>(qt, a, s) : hipErrorInvalidValue;
        if (G.Dh == 64) return launch_attn_tile_t<bf16_t, 64, true>(qt, a, s);
        return G.Dh == 128 ? launch_attn_tile_t<bf16_t, 128, false>(qt, a, s) : hipErrorInvalidValue;  // (up to three groups)
    }
    if (dtype == FC_F32) return G.Dh == 64 ? launch_attn_tile_t<float, 64, false>(qt, a, s) : G.Dh == 128 ? launch_attn_tile_t<float, 128, false>(qt, a, s) : hipErrorInvalidValue;
    return G.Dh == 64 ? launch_attn_tile_t<bf16_t, 64, false>(qt, a, s) : hipErrorInvalidValue;
}
