// QKV projection of a wide window (hundreds to thousands of rows: refreshes, batched blocks) as a
// tiled matrix-core GEMM (bf16, head_dim 128), fused with bias, rotary embedding and the scatter into
// the cache.  Table 1's "W_Q, W_K, W_V projections" row with L replaced by the window length.
//
// Y^T = W X^T: the weight rows are the A operand of v_mfma_f32_16x16x32_bf16 and the window rows the B
// operand, so a lane of the accumulator holds four output features of ONE window row.  The weight rows go by pairs -- the two
// members of a rotary pair, or gate and up row -- and the pairs of all slabs, laid end to end, are dealt to the workgroups in
// equal runs: 128, 96, 80, 64, 48 or 32 pairs, so that a grid a little over one round of workgroups in one width fits a round in another.
//
// Both operands are contiguous along the hidden dimension.  64 (or 128) hidden elements of every row
// of the tile (128- or 256-byte row pieces) stream HBM/L2 -> LDS with direct-to-LDS 16-byte loads into
// a ring of two to four stages; the 16-byte chunks of a row piece are XOR-swizzled with bits 1..3 (or
// 0..3) of the row (applied to the global address of the loading lane), which spreads the 16 lanes the
// LDS serves per clock over 16 different bank groups.
//
// k_gemm_wide (256 window rows) issues its loads between its multiplies.  A wave that issues a direct-to-LDS load waits until the
// memory pipeline has taken it (about 46 cycles per load measured back to back); k_proj_gemm (64 or 128 window rows, where the
// weights' way in counts and not the multiplies) carries more waves that do nothing but issue the loads.
#include <math.h>
#include <string.h>

#include <type_traits>

#include "fc_device.h"
#include "fc_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int KS_MIN = 64;      // hidden elements per stage: 64 or 128 (template parameter KS)

struct GemmArgs {
    const uint16_t *X;     // [M][K]
    const uint16_t *W;     // [N][K]
    const uint16_t *bias;  // [N] or nullptr
    const int32_t *pos;    // [M] or nullptr
    uint16_t *Q;           // [B][Hq][A][128]
    uint16_t *Kc;          // one layer
    uint16_t *Vc;          // one layer
    FcGeom G;
    int M, A, K, win_start;
    int n_mt;              // tiles of window rows
    int n_units;           // tiles of pairs of weight rows
    uint32_t rot_step;     // ROTATE: stages / (units of a round of workgroups) in 1/65536
    int n_slots;           // 128-row slabs of W: head slots (EPI 0), N / 128 (EPI 1, 3), d_ff / 64 (EPI 2)
    // The part of the problem this launch covers (a problem may be cut into two launches with different
    // tile shapes, see launch_pieces): slabs [slot_base, slot_base + slots_here), rows [m_base, m_end).
    int slot_base, slots_here, m_base, m_end;
    double rot1, rot8, rot16, rot32;  // rope_base^(-i/64), i = 1, 8, 16, 32
    // plain linear layers of the rest of the layer (EPI != 0)
    const uint16_t *W2;    // EPI 2: the up matrix [N][K] (W is the gate matrix)
    const uint16_t *res;   // EPI 1: residual [M][N] or nullptr
    uint16_t *out;         // EPI 1, 2: [M][N]
    float *part;           // EPI 3: partial sums [ksplit][M][N]
    int N;                 // output columns
    bool once;             // weights with the non-temporal hint, where there is one tile of rows
    int ksplit;            // EPI 3: parts the hidden dimension is cut into
    FcDivisor by_mt, by_parts, by_a;  // n_mt, ksplit, A
    FcArgmaxPart am;       // EPI 4: per (slab, row) largest logit, its index, sum of exponentials
};


// fc_wait_vm with N = k * PER for a run-time k in 0..3
template <int PER, bool LGKM0>
__device__ __forceinline__ void wait_stages(int k)
{
    if (k >= 3) fc_wait_vm<3 * PER, LGKM0>();
    else if (k == 2) fc_wait_vm<2 * PER, LGKM0>();
    else if (k == 1) fc_wait_vm<PER, LGKM0>();
    else fc_wait_vm<0, LGKM0>();
}

// silu(g) * u in fp32, in front of the rounding to bf16, with the hardware's exponential and reciprocal (gates below
// -87 give 0 instead of some 1e-36).  Against expf and a division, which the kernels for few rows use: over 16 shapes of 33 ..
// 600 rows the same error against 64 bits (1.66e-3, the rounding), 2 results in 10000 off by a rounding either way;
// 2304 rows of a layer 2122 us per two layers instead of 2164, 256 rows 425.5 instead of 428.5.
__device__ __forceinline__ float silu_mul(float g, float u)
{
    return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.4426950408889634f)) * u;
}

__device__ __forceinline__ uint4 pack8(const float (&y)[8])
{
    uint4 w;
    w.x = (uint32_t)fc_bf16_bits(y[0]) | ((uint32_t)fc_bf16_bits(y[1]) << 16);
    w.y = (uint32_t)fc_bf16_bits(y[2]) | ((uint32_t)fc_bf16_bits(y[3]) << 16);
    w.z = (uint32_t)fc_bf16_bits(y[4]) | ((uint32_t)fc_bf16_bits(y[5]) << 16);
    w.w = (uint32_t)fc_bf16_bits(y[6]) | ((uint32_t)fc_bf16_bits(y[7]) << 16);
    return w;
}

// Window rows a wave's epilogue takes at a time, and the LDS it needs for them: fp32, 16 bytes of padding each
__host__ __device__ constexpr int epi_rows(int MT) { return MT >= 4 ? 64 : 32; }
__host__ __device__ constexpr int epi_bytes(int MT, int NT) { return epi_rows(MT) * (NT * 64 + 16); }

// The workgroup's bias goes to LDS at the very start: nothing else asks for it before the end, and a layer's bias
// comes from HBM (2.5 us with the matrix core idle when the epilogue fetched it).  npw pairs from `first` on: the first
// members, then their partners.  One wave calls this.
// A direct load takes two values from a 4-byte address; a bias that starts at an odd element goes through registers.
constexpr int BIAS_LDS = 512;
__device__ __forceinline__ void load_bias(const GemmArgs &p, unsigned char *dst, int first, int npw, int pair_end, int lane)
{
    if (!p.bias) return;
    for (int d0 = 0; d0 < npw; d0 += 64) {
        const int d = d0 + lane;
        if (d >= npw) break;
        const bool high = d >= npw / 2;
        const int pr = min(first + 2 * (high ? d - npw / 2 : d), pair_end - 2);
        const uint16_t *src = p.bias + (pr >> 6) * 128 + (pr & 63) + (high ? 64 : 0);
        if (((uintptr_t)p.bias & 3) == 0)
            __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)src,
                                             (void __attribute__((address_space(3))) *)(dst + d0 * 4), 4, 0, 0);
        else
            *(uint32_t *)(dst + d * 4) = (uint32_t)src[0] | ((uint32_t)src[1] << 16);
    }
    fc_wait_lds();  // LDS writes done, if any
}

// A workgroup's weight rows are pairs: (i, i + 64) of a slab of 128 rows -- the two members of a rotary pair -- or (gate row,
// up row) of a gated layer.  The pairs of all slabs, laid end to end, are dealt to the workgroups in runs of whole eights, and a wave's
// tile holds the first members of its 8 NT pairs in its first 8 NT rows and their partners in the others.
//
// Epilogue of a wave.  Lane (l, q) = (lane & 15, lane >> 4) of tile (i, t) holds rows 16 t + 4 q + r of the wave's weight rows for
// window row m_first + 16 i + l.  The values go through LDS, 64 (or 32) window rows at a time in the wave's own area: in the
// accumulator layout a store instruction covers 8 bytes of 16 different rows, read back as rows it covers 128
// or 256 contiguous bytes.  The loop over eight-value pieces is not unrolled where it holds the rotation or the gate: this code
// runs once per tile, and unrolled it costs more in instruction fetches than in work.
// With one wave per SIMD nothing hides a wait, so a piece's operands are fetched before the arithmetic of the one before it, and
// residuals before the values go to LDS.  What a workgroup takes beside its stages (one stage instead of 56; us, 32 rows a step, fetched
// when due -> this): projection 2048 rows of 36 slots 21.0 -> 13.4, a start off a multiple of eight 20.6 -> 16.4, with bias 24.4 -> 16.9;
// gated 256 rows 9.3 -> 8.6, residual 2304 rows 9.6 -> 8.3; 4.9 of each is the launch and the first stage.  It was the wave with the last
// query or key rows and the first value rows that all others waited for: value rows by single keys (6 us) and the rotation for all its pieces.
template <int MT, int NT, int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs &p, f32x4 (&acc)[MT][NT], unsigned char *area, const uint16_t *bias_low,
                                              const uint16_t *bias_high, int pair0, int pair_end, int m_first, int lane, int kpart)
{
    constexpr int P = 8 * NT;               // pairs of the wave
    constexpr int PITCH = NT * 64 + 16;     // bytes per window row: first members, partners, padding
    constexpr int ROWS = epi_rows(MT), TI = ROWS / 16, TASKS = ROWS * NT / 64;  // pieces per lane
    const FcGeom &G = p.G;
    const int l = lane & 15, q = lane >> 4;
    const int first_v = G.Hq + G.Hkv;       // EPI 0: first value slab
    const bool has_v = EPI == 0 && pair0 + P > first_v * 64;
    static_assert(MT % TI == 0 && ROWS * NT % 64 == 0, "whole steps");
#pragma unroll
    for (int i = 0; i < MT; i += TI) {
        const int m_i = m_first + 16 * i;
        // EPI 0: sequence, window row and position of row m_i + lane % ROWS (pp < 0: padded or past the end)
        int b_l = 0, a_l = 0, pp_l = -1;
        if (EPI == 0) {
            const int m = m_i + lane % ROWS;
            if (m < p.m_end) {
                b_l = (int)p.by_a.over(m);
                a_l = m - b_l * p.A;
                pp_l = p.pos ? p.pos[m] : p.win_start + a_l;
                if (pp_l >= G.max_seq) pp_l = -1;
            }
        }
        if (has_v) {
            // Value rows go to the transposed tiles.  Where these 64 rows are consecutive positions of one sequence by way of LDS, [weight
            // row][window row], rounded, as far from a multiple of eight there as in the tile: they leave in pieces of eight keys, 16 bytes, and
            // single keys at both ends: eight of 64 rows, eight weight rows at a time (by sixteens, half of the lanes idle, a start off a
            // multiple of eight cost 2 us: 1280 rows of 36 slots from 67 on 44.0 -> 42.8, 2304 rows 69.3 -> 67.9; 1581 rows of 96 slots, hidden
            // 4096, 153.8 -> 151.8, straight from the accumulators 151.2).  Otherwise straight from the accumulators, lanes along the keys
            // (32 rows of 128 x 80-pair tiles by way of LDS: 6 x 100 rows 28.7 -> 29.5 us).
            constexpr int VPITCH = ROWS * 2 + 16, GROUPS = ROWS / 8;
            const int64_t per_head = (int64_t)G.spad * 128;
            const int n_in = min(ROWS, p.m_end - m_i), r_l = lane % ROWS;
            const int pp0 = __builtin_amdgcn_readfirstlane(pp_l), b0 = __builtin_amdgcn_readfirstlane(b_l);
            if (ROWS == 64 && n_in >= 16 && pp0 >= 0 && __all(r_l >= n_in || (pp_l == pp0 + r_l && b_l == b0))) {
                const int shift = pp0 & 7;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int j = 16 * t + 4 * q;
                    float bs[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) bs[e] = p.bias ? fc_to_float(bf16_t{(j >= P ? bias_high + j - P : bias_low + j)[e]}) : 0.f;
#pragma unroll
                    for (int h = 0; h < TI; ++h)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            *(uint16_t *)(area + (j + e) * VPITCH + (16 * h + l + shift) * 2) = fc_bf16_bits(acc[i + h][t][e] + bs[e]);
                }
                __builtin_amdgcn_wave_barrier();
                fc_wait_lds();
                // elements from value 0 of the sequence's first head to value row j's; -1: none of this wave's
                auto offset_of = [&](int j) -> int64_t {
                    const int pr = pair0 + (j >= P ? j - P : j);
                    if (pr < first_v * 64 || pr >= pair_end) return -1;
                    return ((pr >> 6) - first_v) * per_head + ((pr & 63) + (j >= P ? 64 : 0)) * FC_VTILE;
                };
                auto key_at = [&](int pp) -> int64_t { return (int64_t)(pp / FC_VTILE) * (FC_VTILE * 128) + pp % FC_VTILE; };
                uint16_t *const vb = p.Vc + (size_t)b0 * G.Hkv * per_head;
                const int c_lo = (shift + 7) & ~7, c_hi = (shift + n_in) & ~7, base = pp0 - shift;  // whole pieces: columns c_lo .. c_hi - 1
                {
                    const int c = c_lo + 8 * (lane % GROUPS);
                    const int64_t at = key_at(base + c);
#pragma unroll 2
                    for (int j = lane / GROUPS; j < 16 * NT; j += 64 / GROUPS) {
                        const uint4 v8 = *(const uint4 *)(area + j * VPITCH + 2 * c);
                        const int64_t o = offset_of(j);
                        if (o >= 0 && c < c_hi) *(uint4 *)(vb + o + at) = v8;
                    }
                }
                const int before = c_lo - shift, single = before + shift + n_in - c_hi;  // 8 of 64 rows, at most 7 + 7 of fewer
                if (single) {
                    const int wide = single > 8 ? 4 : 3, e = lane & ((1 << wide) - 1), c = e < before ? shift + e : c_hi + e - before;
                    const int64_t at = key_at(base + c);
#pragma unroll 4
                    for (int j = lane >> wide; j < 16 * NT; j += 64 >> wide) {
                        const uint16_t v1 = *(const uint16_t *)(area + j * VPITCH + 2 * min(c, ROWS + 7));
                        const int64_t o = offset_of(j);
                        if (o >= 0 && e < single) vb[o + at] = v1;
                    }
                }
            } else {
#pragma unroll
                for (int h = 0; h < TI; ++h) {
                    const int b = __shfl(b_l, 16 * h + l, 64), pp = __shfl(pp_l, 16 * h + l, 64);
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const int j = 16 * t + 4 * q;
                        const bool high = j >= P;
                        const int pr = pair0 + (high ? j - P : j), hs = pr >> 6;
                        if (hs < first_v || pr >= pair_end || pp < 0) continue;
                        uint16_t *v = p.Vc + fc_v_index(G, b, hs - first_v, pp, (pr & 63) + (high ? 64 : 0));
                        const uint16_t *bs = high ? bias_high + j - P : bias_low + j;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            v[e * FC_VTILE] = fc_bf16_bits(acc[i + h][t][e] + (p.bias ? fc_to_float(bf16_t{bs[e]}) : 0.f));
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
            fc_wait_lds();
            if (pair0 >= first_v * 64) continue;
        }
        // Piece k of a lane: eight first members and their partners of one row.  (EPI 0, a wave with value slabs behind others: the others)
        const int eights = EPI == 0 && has_v ? min(NT, (first_v * 64 - pair0) / 8) : NT;
        const int n_pieces = EPI == 0 && has_v ? (ROWS * eights + 63) / 64 : TASKS;
        auto piece_row = [&](int k) { return EPI == 0 && has_v ? (lane + 64 * k) / eights : (lane + 64 * k) / NT; };
        auto piece_eight = [&](int k) { return lane + 64 * k - piece_row(k) * (EPI == 0 && has_v ? eights : NT); };
        // EPI 1: the residual is asked for before the values go to LDS
        uint4 rl[EPI == 1 ? TASKS : 1], rh[EPI == 1 ? TASKS : 1];
        if constexpr (EPI == 1) {
            if (p.res) {
#pragma unroll
                for (int k = 0; k < TASKS; ++k) {
                    const int m = min(m_i + piece_row(k), p.m_end - 1), pr = min(pair0 + 8 * piece_eight(k), pair_end - 8);
                    const uint16_t *r = p.res + (size_t)m * p.N + (size_t)(pr >> 6) * 128 + (pr & 63);
                    rl[k] = *(const uint4 *)r;
                    rh[k] = *(const uint4 *)(r + 64);
                }
            } else {
#pragma unroll
                for (int k = 0; k < TASKS; ++k) rl[k] = rh[k] = make_uint4(0, 0, 0, 0);
            }
        }
        // ---- to LDS
#pragma unroll
        for (int h = 0; h < TI; ++h)
#pragma unroll
            for (int t = 0; t < NT; ++t) *(f32x4 *)(area + (16 * h + l) * PITCH + 64 * t + 16 * q) = acc[i + h][t];
        __builtin_amdgcn_wave_barrier();
        fc_wait_lds();
        // ---- and back as rows
        struct Eight {
            float lo[8], hv[8];
            int row, s, b, a, pp;
        };
        auto fetch = [&](int k, Eight &x) {
            x.row = piece_row(k);
            x.s = piece_eight(k);
            if (EPI == 0) {
                x.b = __shfl(b_l, x.row, 64);
                x.a = __shfl(a_l, x.row, 64);
                x.pp = __shfl(pp_l, x.row, 64);
            }
            const float *src = (const float *)(area + (EPI == 0 ? min(x.row, ROWS - 1) : x.row) * PITCH) + 8 * x.s;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                *(float4 *)(x.lo + 4 * h) = *(const float4 *)(src + 4 * h);
                *(float4 *)(x.hv + 4 * h) = *(const float4 *)(src + P + 4 * h);
            }
        };
        auto finish = [&](int k, Eight &x) {
            float (&lo)[8] = x.lo, (&hv)[8] = x.hv;
            const int s = x.s, m = m_i + x.row, b = x.b, a = x.a, pp = x.pp;
            const int pr = pair0 + 8 * s;                 // first of the eight pairs
            if (m >= p.m_end || pr >= pair_end || (EPI == 0 && x.row >= ROWS)) return;
            const int hs = pr >> 6, lf = pr & 63;         // slab, and place among its first members
            if constexpr (EPI == 0) {
                const bool valid = pp >= 0;
                if (p.bias) {
                    union { uint4 u4; uint16_t h[8]; } bl, bh;
                    bl.u4 = *(const uint4 *)(bias_low + 8 * s);
                    bh.u4 = *(const uint4 *)(bias_high + 8 * s);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        lo[e] += fc_to_float(bf16_t{bl.h[e]});
                        hv[e] += fc_to_float(bf16_t{bh.h[e]});
                    }
                }
                // the angle is reduced to a fraction of a turn in double, then hardware sine / cosine
                // (argument in turns)
                double f = 0.15915494309189533576888;  // base^(-i/64) / (2 pi): turns per position of pair i
                if (lf & 8) f *= p.rot8;
                if (lf & 16) f *= p.rot16;
                if (lf & 32) f *= p.rot32;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const double turns = (double)pp * f;
                    const float ph = (float)(turns - rint(turns));
                    const float c = __builtin_amdgcn_cosf(ph), sn = __builtin_amdgcn_sinf(ph);
                    const float xv = lo[e], y = hv[e];
                    lo[e] = xv * c - y * sn;
                    hv[e] = y * c + xv * sn;
                    f *= p.rot1;
                }
                if (hs < G.Hq) {
                    uint16_t *d = p.Q + (((size_t)b * G.Hq + hs) * p.A + a) * 128 + lf;
                    const uint4 ql = valid ? pack8(lo) : make_uint4(0, 0, 0, 0), qh = valid ? pack8(hv) : make_uint4(0, 0, 0, 0);
                    fc_store_any(d, ql);
                    fc_store_any(d + 64, qh);
                } else if (valid) {
                    uint16_t *kr = p.Kc + fc_k_index(G, b, hs - G.Hq, pp, lf);
                    *(uint4 *)kr = pack8(lo);
                    *(uint4 *)(kr + 64) = pack8(hv);
                }
            } else if constexpr (EPI == 2) {
                float y[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) y[e] = silu_mul(lo[e], hv[e]);
                *(uint4 *)(p.out + (size_t)m * p.N + pr) = pack8(y);
            } else {
                const size_t at = (size_t)m * p.N + (size_t)hs * 128 + lf;  // partners 64 on
                if constexpr (EPI == 3) {
                    float *o = p.part + (size_t)kpart * p.M * p.N + at;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        *(float4 *)(o + 4 * h) = *(float4 *)(lo + 4 * h);
                        *(float4 *)(o + 64 + 4 * h) = *(float4 *)(hv + 4 * h);
                    }
                } else {
                    union { uint4 u4; uint16_t h[8]; } xl, xh;
                    xl.u4 = rl[k];
                    xh.u4 = rh[k];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        lo[e] += fc_to_float(bf16_t{xl.h[e]});
                        hv[e] += fc_to_float(bf16_t{xh.h[e]});
                    }
                    *(uint4 *)(p.out + at) = pack8(lo);
                    *(uint4 *)(p.out + at + 64) = pack8(hv);
                }
            }
        };
        if constexpr (EPI == 0 || EPI == 2) {
            Eight x[2];
            fetch(0, x[0]);
#pragma unroll 1
            for (int k = 0; k + 1 < n_pieces; ++k) {
                fetch(k + 1, x[1]);
                __builtin_amdgcn_sched_barrier(0);
                finish(k, x[0]);
                x[0] = x[1];
            }
            finish(n_pieces - 1, x[0]);
        } else {
#pragma unroll
            for (int k = 0; k < TASKS; ++k) {
                Eight x;
                fetch(k, x);
                finish(k, x);
            }
        }
        __builtin_amdgcn_wave_barrier();
        fc_wait_lds();
    }
}

// Vocabulary mode (EPI 4): a wave's 128 weight rows are slab hs, a lane holds its logits 16 t + 4 q + r for window row 16 i + l,
// ascending in (t, r), so that ties keep the smaller index; the others are in lanes 16, 32 and 48 on.  First the
// maximum and its place, then the sum of exponentials against it, by the hardware's exponential of a rounded product.
// On logits that are exact in fp32 the error of the confidences against 64 bits is 5 .. 10e-8, 0.87 times that of a running
// maximum with expf and 0.89 times that of expf in this form, which also takes longer (256 rows x 152064: 309.0 us, this
// 303.9); on others the logits' own error covers it.
template <int MT>
__device__ __forceinline__ void gemm_epilogue_vocab(const GemmArgs &p, const f32x4 (&acc)[MT][8], int hs, int m_first, int lane)
{
    const int l = lane & 15, q = lane >> 4;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int m = m_first + 16 * i + l;
        float mx = -INFINITY, sm = 0.f;
        int arg = 0;
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool more = acc[i][t][r] > mx;
                mx = more ? acc[i][t][r] : mx;
                arg = more ? 16 * t + r : arg;
            }
        arg += hs * 128 + 4 * q;
#pragma unroll
        for (int t = 0; t < 8; t += 2) {
            float e[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) e[r] = __builtin_amdgcn_exp2f((acc[i][t + r / 4][r % 4] - mx) * 1.4426950408889634f);
            sm += ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]));
        }
#pragma unroll
        for (int off = 16; off < 64; off <<= 1) {
            const float mx2 = __shfl_xor(mx, off, 64), sm2 = __shfl_xor(sm, off, 64);
            const int arg2 = __shfl_xor(arg, off, 64);
            fc_argmax_merge(mx, arg, sm, mx2, arg2, sm2);
        }
        if (q == 0 && m < p.m_end) p.am.at(hs, m) = FcArgmax{mx, arg, sm};
    }
}

// Weight row of place `j` of a wave tile of 8 NT pairs from pair0 on, and the matrix it is of (EPI 2: first members gate, partners up).
// Pairs past the end re-read the last one; they are never stored.
template <int NT, int EPI>
__device__ __forceinline__ uint32_t weight_row(int pair0, int pair_end, int j)
{
    const bool high = j >= 8 * NT;
    const int pr = min(pair0 + (high ? j - 8 * NT : j), pair_end - 1);
    return EPI == 2 ? pr : (uint32_t)((pr >> 6) * 128 + (pr & 63) + (high ? 64 : 0));
}

// Workgroup -> (tile of pairs and rows, part of the hidden dimension).  Workgroup ids that are equal modulo 8 land on the same XCD; the
// tiles, ordered unit by unit, are dealt to the eight XCDs in equal contiguous runs, so the workgroups that stream the same weight
// rows share an L2 and every XCD gets the same number of tiles (dealing whole units instead left 35 tiles on four XCDs and 28
// on the others for 36 head slots x 7 row tiles: two rounds of 32 compute units instead of one, 100 us instead of 62).
// The parts of the hidden dimension (EPI 3) count as tiles too.
struct TilePlace {
    int unit, mt, kpart;
};
template <int EPI>
__device__ __forceinline__ bool tile_place(const GemmArgs &p, TilePlace &w)
{
    const int xcd = blockIdx.x & 7, qd = blockIdx.x >> 3;
    const int n_kp = EPI == 3 ? p.ksplit : 1;
    const int64_t n_tiles = (int64_t)p.n_units * p.n_mt * n_kp;
    const int tile_k = (int)(xcd * n_tiles / 8) + qd;
    if (tile_k >= (int)((xcd + 1) * n_tiles / 8)) return false;
    const int tile = EPI == 3 ? (int)p.by_parts.over(tile_k) : tile_k;
    w.kpart = tile_k - tile * n_kp;
    w.unit = (int)p.by_mt.over(tile);
    w.mt = tile - w.unit * p.n_mt;
    return true;
}

// -------------------------------------------------------------------------------------------------
// At most 128 window rows per workgroup: NW waves that multiply, 32 window rows each and all 32 NSUB weight rows, and NL that
// only load.
// EPI selects the epilogue: 0 = QKV (bias, rotary embedding, scatter into the cache); the others are
// the plain linear layers of the rest of the layer, whose 128-row slabs of W take the place of the
// head slots: 1 = out = residual + x w^T; 2 = out = silu(x w_gate^T) * (x w_up^T), a slab being 64
// gate rows and the same 64 up rows; 3 = fp32 partial sums of one part of the hidden dimension
// (the parts are tiles of their own), for matrices with too few slabs to fill the chip; 4 = vocabulary projection of the
// unmasking step: of the 128 logits of a slab only the largest, its index and the sum of
// exp(logit - largest) are kept per row (NSUB = 4 only).
// SLOTS: stages in the LDS ring.  ONCE: the weights with the non-temporal hint.
template <int KS, int NW, int NSUB, int SLOTS, int NL, int EPI, bool ROTATE, bool ONCE>
__global__ __launch_bounds__((NW + NL) * 64) __attribute__((amdgpu_waves_per_eu((EPI == 4 && NW == 2) || NW + NL > 4 ? 2 : 1))) void k_proj_gemm(GemmArgs p)
{
    constexpr int ROWB = KS * 2;               // bytes of one row piece: 128 or 256
    constexpr int CPR = ROWB / 16;             // 16-byte chunks per row piece
    constexpr int RPB = 1024 / ROWB;           // row pieces per 1 KB block (= one wave-wide load)
    constexpr int NKK = KS / 32;               // k-steps per stage
    constexpr int MT = 2, NT = 2 * NSUB;       // tiles of 16 window rows and weight rows of a wave
    constexpr int WROWS = 16 * NT, XROWS = 32 * NW, PAIRS = WROWS / 2;
    constexpr int WBYTES = WROWS * ROWB, STAGE = (WROWS + XROWS) * ROWB;
    constexpr int NBLK = (WROWS + XROWS) / RPB, WBLK = WROWS / RPB;  // 1 KB blocks per stage, weight blocks first
    constexpr int LBW = NBLK / NL, WBW = WBLK / NL;                  // per loading wave
    static_assert(KS == 64 || KS == 128, "stage depth");
    static_assert(NBLK % NL == 0 && WBLK % NL == 0 && PAIRS % RPB == 0 && (EPI != 4 || NSUB == 4), "tile shape");
    static_assert((SLOTS - 1) * LBW < 64 && SLOTS >= 2 && SLOTS <= 4, "vmcnt range");
    extern __shared__ __align__(1024) unsigned char smem[];

    TilePlace at;
    if (!tile_place<EPI>(p, at)) return;
    const int m0 = p.m_base + at.mt * XROWS;
    const int pair0 = p.slot_base * 64 + at.unit * PAIRS, pair_end = (p.slot_base + p.slots_here) * 64;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = lane & 15, q = lane >> 4;
    const int lw = wave - NW;                  // index among the loading waves

    // part of the hidden dimension this workgroup covers (EPI 3 only: part kpart of p.ksplit)
    const int all_stages = p.K / KS;
    const int st0 = EPI == 3 ? (int)p.by_parts.over((uint32_t)(at.kpart * all_stages)) : 0;
    const int n_stages = EPI == 3 ? (int)p.by_parts.over((uint32_t)((at.kpart + 1) * all_stages)) - st0 : all_stages;
    unsigned char *bias_area = smem + SLOTS * STAGE;  // behind the ring

    if (wave >= NW) {
        // ---- loading waves: per-lane source offsets (bytes from W / X, hidden offset 0) of this wave's blocks
        uint32_t goff[LBW];
#pragma unroll
        for (int i = 0; i < LBW; ++i) {
            const int bid = lw + NL * i;
            const int rl = RPB * (i < WBW ? bid : bid - WBLK) + lane / CPR;  // row of the W / X tile
            // logical 16-byte chunk that lands at position lane % CPR of the row piece: 128-byte pieces are
            // swizzled with bits 1..3 of the row, 256-byte pieces with bits 0..3
            const int c = (lane % CPR) ^ (KS == 64 ? (rl >> 1) & 7 : rl & 15);
            const uint32_t row = i < WBW ? weight_row<NT, EPI>(pair0, pair_end, rl)
                                         : (uint32_t)min(m0 + rl, p.m_end - 1);  // rows past the end: never stored
            goff[i] = row * (uint32_t)(p.K * 2) + c * 16;
        }
        // Rows of W that lie a multiple of 4 KB apart: workgroup `unit` starts unit / n_units of the way along the hidden
        // dimension and goes round.  In step, all workgroups ask for the same 128 bytes of all those rows, and these share a few
        // memory channels.  One row tile of up to 128 rows, us without and with: gated 4096 x 12288, 64 / 128 rows 40.3 and 32.7 /
        // 44.4 and 39.7; 4096 x 14336 50.0 and 41.9 / 52.4 and 46.7; 2048 x 16384, 48 rows 28.0 and 23.2; 6144 x 16384 78 and 69; 8192 x 8192,
        // 64 rows 51.8 and 45.1; vocabulary 4096 x 32000, 64 rows 60.4 and 51.0; projection, 96 slots, hidden 4096, 64 rows 27.3 and 24.9.
        // At other distances it gives nothing or costs (hidden 5120 34.6 and 35.6, 7168 44.1 and 45.7, 1024 15.0 and 15.3), and so it
        // does with more row tiles, whose window rows then come from L2 at two places at a time (256 rows of gated 4096 x
        // 12288 66.9 and 70.3), and with the last rows of a problem, behind the launch that has just read the weights (300 rows of
        // the same 102.8 and 107.0).
        // More than one round of workgroups: by the place among the 256 that run together, 32 on each XCD.  (By unit / n_units
        // those together cover a fifth of the hidden dimension at 1188 units; 96 rows, vocabulary of 65536 4.7 us slower.)  Vocabularies, us
        // without and with: hidden 4096, 64 rows, 50304 entries 81.2 and 76.2; 65536 101.9 and 83.6; 152064 198.3 and 195.5; 96 rows, 50304 96.0
        // and 87.0; 65536 120.9 and 95.4; 128 rows, 152064 247.9 and 243.4; hidden 2048, 64 rows, 131072 104.2 and 86.7; hidden 8192, 32000 108.5
        // and 83.3.  From four rounds on the workgroups drift apart by themselves and it is a few per cent either way.
        const int per_round = min(p.n_units, 256);
        const int place = (int)(blockIdx.x & 7) * per_round / 8 + (int)(blockIdx.x >> 3 & 31);
        const int rot = ROTATE ? (int)(((uint32_t)place * p.rot_step) >> 16) : 0;
        auto issue_stage = [&](int st) {
            const int sr = st + rot, hidden = st0 + (ROTATE && sr >= n_stages ? sr - n_stages : sr);
            unsigned char *dst = smem + (st % SLOTS) * STAGE;
#pragma unroll
            for (int i = 0; i < LBW; ++i) {
                // EPI 2: the partners (whole blocks) are rows of the up matrix
                const uint16_t *mat = i >= WBW ? p.X : EPI == 2 && RPB * (lw + NL * i) >= PAIRS ? p.W2 : p.W;
                const unsigned char *src = (const unsigned char *)mat + (size_t)hidden * ROWB;
                if (ONCE && i < WBW) fc_load_lds16<true>(src + goff[i], dst + (lw + NL * i) * 1024);
                else fc_load_lds16(src + goff[i], dst + (lw + NL * i) * 1024);
            }
        };
        if (EPI == 0 && lw == 0) load_bias(p, bias_area, pair0, PAIRS, pair_end, lane);
        // One barrier per stage, shared with the multiplying waves.  Barrier `it` (it = 0 .. n_stages - 2) means: stage it+1 is
        // complete and every multiplying wave has left stage it, whose slot takes stage it + SLOTS.
        const int n_pro = min(SLOTS, n_stages);
        for (int st = 0; st < n_pro; ++st) issue_stage(st);
        wait_stages<LBW, false>(n_pro - 1);
        __builtin_amdgcn_s_barrier();  // stage 0 is complete
        for (int it = 0; it + 1 < n_stages; ++it) {
            // stages requested so far: min(n_stages, it + SLOTS); those after it+1 may stay in flight
            wait_stages<LBW, false>(min(n_stages, it + SLOTS) - (it + 2));
            __builtin_amdgcn_s_barrier();
            if (it + SLOTS < n_stages) issue_stage(it + SLOTS);
        }
        return;
    }

    // ---- operand read offsets inside a stage (bytes): row l of a 16-row tile, k-step kk
    uint32_t foff[NKK];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
        foff[kk] = (uint32_t)(l * ROWB + (((4 * kk + q) ^ (KS == 64 ? (l >> 1) & 7 : l)) << 4));
    const uint32_t x_base = (uint32_t)(WBYTES + wave * 32 * ROWB);

    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Logits of up to 64 rows are summed in two levels, chains over 512 elements and those.  Relative error of the confidences against
    // 64 bits, 32 rows x 152064, hidden 3584 / 4096: 7.8e-7 / 6.2e-7 in one chain over all elements, 2.1e-7 / 1.7e-7 in two levels, 2.4e-7 / 2.3e-7
    // in the whole-row kernel, whose waves cut the hidden dimension in eight.
    constexpr bool LEVELS = EPI == 4 && XROWS == 64;
    constexpr int RUN = 512 / KS;
    f32x4 total[LEVELS ? MT : 1][LEVELS ? NT : 1];
    auto fold = [&]() {
        if constexpr (LEVELS) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        total[i][t][r] += acc[i][t][r];
                        acc[i][t][r] = 0.f;
                    }
        }
    };
    if constexpr (LEVELS) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t) total[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // Fragments are double-buffered in registers: the LDS reads of k-step kk+1 are issued before the
    // multiplies of k-step kk, and the first reads of the next stage go out (behind that stage's
    // barrier) before the last multiplies of this one, so the matrix core never waits for LDS.
    bf16x8 xf[2][MT], wf[2][NT];
    auto read_frags = [&](int slot, int kk, int buf) {
        const unsigned char *st = smem + slot * STAGE;
#pragma unroll
        for (int i = 0; i < MT; ++i) xf[buf][i] = *(const bf16x8 *)(st + x_base + i * (16 * ROWB) + foff[kk]);
#pragma unroll
        for (int t = 0; t < NT; ++t) wf[buf][t] = *(const bf16x8 *)(st + t * (16 * ROWB) + foff[kk]);
    };
    auto multiply = [&](int buf) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[buf][t], xf[buf][i], acc[i][t], 0, 0, 0);
    };
    __builtin_amdgcn_s_barrier();  // stage 0 is complete
    read_frags(0, 0, 0);
    int slot = 0;
    for (int it = 0; it < n_stages; ++it) {
#pragma unroll
        for (int kk = 0; kk < NKK - 1; ++kk) {
            read_frags(slot, kk + 1, (kk + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            multiply(kk & 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        const int nslot = slot == SLOTS - 1 ? 0 : slot + 1;
        if (it + 1 < n_stages) {
            fc_wait_lds();  // lgkmcnt(0): the reads of stage `it` have returned
            __builtin_amdgcn_s_barrier();
            read_frags(nslot, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        multiply((NKK - 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
        if (LEVELS && it % RUN == RUN - 1) fold();
        slot = nslot;
    }

    // ---- epilogue; the LDS ring is its staging area, once every wave has left it
    if constexpr (EPI == 4) {
        if constexpr (LEVELS) {
            fold();
            gemm_epilogue_vocab<MT>(p, total, pair0 >> 6, m0 + 32 * wave, lane);
        } else {
            gemm_epilogue_vocab<MT>(p, acc, pair0 >> 6, m0 + 32 * wave, lane);
        }
    } else {
        static_assert(NW * epi_bytes(MT, NT) <= SLOTS * STAGE, "epilogue staging");
        __builtin_amdgcn_s_barrier();
        const uint16_t *bias_low = (const uint16_t *)bias_area;
        gemm_epilogue<MT, NT, EPI>(p, acc, smem + wave * epi_bytes(MT, NT), bias_low, bias_low + PAIRS, pair0, pair_end, m0 + 32 * wave, lane, at.kpart);
    }
}

// -------------------------------------------------------------------------------------------------
// 256 window rows: four waves, one per SIMD, WN of them along the weight rows, each with MT x NT tiles of 16 x 16 (128 x 128, 128 x 96,
// 128 x 80 or 64 x 128).
//
// One wave per SIMD keeps up to 256 accumulators and reads the fewest operand bytes from LDS: 131 KB per 64 hidden
// elements of a 256 x 256 tile against 196 KB with eight waves of 64 x 128, beside 64 KB of loads (free of conflicts LDS gives
// 240 to 250 B per clock: 540 and 800 clocks of reads beside 2048 of multiplies).  v_mfma 16x16x32 instead of 32x32x16: under the
// power limit, multiplies alone, 2024 against 1780 TFLOP/s (the accumulators are read and written half as often).  A stage of 64
// hidden elements is two phases of MT * NT multiplies; between them go the fragment reads of the next phase and the loads of later
// stages, one every few multiplies, so nothing is waited for but the stage's barrier in the middle:
//
//   barrier(s)   stage s+1 has arrived, every wave has read all of stage s: its slots are free
//   phase B(s)   multiplies the second half of stage s; reads the first half of stage s+1, issues the first loads of batch s
//   phase A(s+1) multiplies the first half of stage s+1; reads the second half, issues the other loads of batch s
//
// Batch s is window rows of stage s + XS and weight rows of stage s + WS, into the slots just freed.
// Against eight waves and 32x32x16 multiplies, us: gated 3584 x 18944, 2304 rows (256 x 256) 492 -> 431 + 37, 256 rows (256 x 160, weights
// from HBM) 83 -> 71; 18944 x 3584, 2304 rows (256 x 128) 470 -> 405; vocabulary 3584 x 152064, 256 rows 325 -> 283.  In the loop a
// 256 x 256 x 64 stage takes 2460 clocks of which 2048 are multiplies; the clock is what the power limit leaves, 1.8 GHz.
// Weights from HBM: a compute unit has some 64 KB of loads under way, taken in order, so window rows that are in L2 wait behind
// weights that are not (256 x 160: loads alone 0.97 us a stage, weights alone 0.75, with the non-temporal hint both 0.86).
template <int MT, int NT, int WN, int WS, int XS, int EPI, bool ONCE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_gemm_wide(GemmArgs p)
{
    constexpr int WROWS = 16 * NT * WN, XROWS = 16 * MT * 4 / WN, PAIRS = WROWS / 2;
    constexpr int WBYTES = WROWS * 128, XBYTES = XROWS * 128;       // a stage of 64 hidden elements
    constexpr int WL = WROWS / 32, XL = XROWS / 32, BATCH = WL + XL;  // 1 KB loads per wave
    constexpr int NM = MT * NT, NR = MT + NT;                       // multiplies and reads of a phase
    // loads that may still be on their way when stage s + 1 has to be there: those behind X(s + 1) and behind W(s + 1)
    constexpr int BEHIND_X = (XS - 2) * BATCH + WL, BEHIND_W = (WS - 2) * BATCH;
    constexpr int AHEAD = BEHIND_X < BEHIND_W ? BEHIND_X : BEHIND_W;
    static_assert(XROWS == 256 && XS >= 2 && WS >= XS && WS <= 4 && AHEAD + BATCH < 64, "ring");
    static_assert(WS * WBYTES + XS * XBYTES >= 4 * epi_bytes(MT, NT) + 1024, "epilogue staging, bias");
    static_assert(EPI != 4 || NT == 8, "a slab per wave");
    extern __shared__ __align__(1024) unsigned char smem[];
    unsigned char *const wring = smem, *const xring = smem + WS * WBYTES;

    TilePlace at;
    if (!tile_place<EPI>(p, at)) return;
    const int m0 = p.m_base + at.mt * XROWS;
    const int pair0 = p.slot_base * 64 + at.unit * PAIRS, pair_end = (p.slot_base + p.slots_here) * 64;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = WN == 1 ? 0 : wave >> 1, wm = WN == 1 ? wave : wave & 1;
    const int l = lane & 15, q = lane >> 4;

    // The workgroup's bias, one weight row per thread, is asked for here and waits in a register (the ring takes all of LDS):
    // fetched by the epilogue it cost 2.5 us with the matrix cores idle.
    uint16_t bias = 0;
    if (EPI == 0 && p.bias && tid < WROWS) bias = p.bias[weight_row<NT, EPI>(pair0 + (tid / (16 * NT)) * 8 * NT, pair_end, tid % (16 * NT))];

    // ---- loads: 8 rows x 128 B each, the 16-byte chunks of a row permuted by bits 1..3 of the row
    uint32_t woff[WL], xoff[XL];
#pragma unroll
    for (int i = 0; i < WL; ++i) {
        const int r = 8 * (wave + 4 * i) + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
        woff[i] = weight_row<NT, EPI>(pair0 + (r / (16 * NT)) * 8 * NT, pair_end, r % (16 * NT)) * (uint32_t)(p.K * 2) + c * 16;
    }
#pragma unroll
    for (int i = 0; i < XL; ++i) {
        const int r = 8 * (wave + 4 * i) + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
        xoff[i] = (uint32_t)min(m0 + r, p.m_end - 1) * (uint32_t)(p.K * 2) + c * 16;  // rows past the end: never stored
    }
    // part of the hidden dimension this workgroup covers (EPI 3 only: part kpart of p.ksplit)
    const int all_stages = p.K / 64;
    const int st0 = EPI == 3 ? (int)p.by_parts.over((uint32_t)(at.kpart * all_stages)) : 0;
    const int n_stages = EPI == 3 ? (int)p.by_parts.over((uint32_t)((at.kpart + 1) * all_stages)) - st0 : all_stages;
    auto load_w = [&](int st, int slot, int i) {
        const bool up = EPI == 2 && 8 * (wave + 4 * i) % (16 * NT) >= 8 * NT;  // (whole blocks)
        const unsigned char *src = (const unsigned char *)(up ? p.W2 : p.W) + (size_t)(st0 + st) * 128;
        fc_load_lds16<ONCE>(src + woff[i], wring + slot * WBYTES + (wave + 4 * i) * 1024);
    };
    auto load_x = [&](int st, int slot, int i) {
        const unsigned char *src = (const unsigned char *)p.X + (size_t)(st0 + st) * 128;
        fc_load_lds16(src + xoff[i], xring + slot * XBYTES + (wave + 4 * i) * 1024);
    };

    // ---- operand fragments
    uint32_t foff[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) foff[h] = (uint32_t)(l * 128 + (((4 * h + q) ^ ((l >> 1) & 7)) << 4));
    bf16x8 xf[2][MT], wf[2][NT];
    auto read = [&](int h, int wslot, int xslot, int j) {
        if (j < MT) xf[h][j] = *(const bf16x8 *)(xring + xslot * XBYTES + wm * (MT * 2048) + j * 2048 + foff[h]);
        else wf[h][j - MT] = *(const bf16x8 *)(wring + wslot * WBYTES + wn * (NT * 2048) + (j - MT) * 2048 + foff[h]);
    };
    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // The multiplies of half h; read_at(j) and load_at(j) go between them, load_at for loads first .. last - 1.  (Loops with conditions
    // that unrolling decides: as a recursion of templates over the same places the file took 16 minutes to compile.)
    auto phase = [&](auto hc, auto first, auto last, auto read_at, auto load_at) {
        constexpr int H = decltype(hc)::value, L0 = decltype(first)::value, L1 = decltype(last)::value, SPAN = NM * 7 / 8, LOADS = L1 > L0 ? L1 - L0 : 1;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
#pragma unroll
            for (int j = 0; j < NR; ++j)
                if (j * SPAN / NR == m) {
                    read_at(j);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
            for (int j = L0; j < L1; ++j)
                if ((j - L0) * SPAN / LOADS + 1 == m) {
                    load_at(j);
                    __builtin_amdgcn_sched_barrier(0);
                }
            acc[m / NT][m % NT] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[H][m % NT], xf[H][m / NT], acc[m / NT][m % NT], 0, 0, 0);
            if ((m & 1) == 1) __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    using std::integral_constant;
    const integral_constant<int, 0> none;
    const integral_constant<int, 1> half1;
    const integral_constant<int, XS == 2 ? XL : (BATCH + 1) / 2> mid;
    const integral_constant<int, BATCH> all;
    auto no_load = [](int) {};

    // ---- fill the ring in the order of the batches, then the first half of stage 0
#pragma unroll
    for (int b = -WS; b < 0; ++b) {
        if (b + XS >= 0 && b + XS < n_stages)
#pragma unroll
            for (int i = 0; i < XL; ++i) load_x(b + XS, b + XS, i);
        if (b + WS < n_stages)
#pragma unroll
            for (int i = 0; i < WL; ++i) load_w(b + WS, b + WS, i);
    }
    if (n_stages >= WS) fc_wait_vm<AHEAD + BATCH>();
    else fc_wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    int ws = 0, xs = 0;  // slots of stage s
#pragma unroll
    for (int j = 0; j < NR; ++j) read(0, 0, 0, j);
    fc_wait_lds();
    __builtin_amdgcn_sched_barrier(0);
    phase(none, none, none, [&](int j) { read(1, 0, 0, j); }, no_load);

    auto stage = [&](int s, auto tail) {
        constexpr bool TAIL = decltype(tail)::value;  // the ring drains: loads that there are, by comparison
        if (!TAIL || s - 1 + WS < n_stages) fc_wait_vm<AHEAD, true>();
        else fc_wait_vm<0, true>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const int ws1 = ws == WS - 1 ? 0 : ws + 1, xs1 = xs == XS - 1 ? 0 : xs + 1;
        auto load = [&](int j) {
            if (j < XL) {
                if (!TAIL || s + XS < n_stages) load_x(s + XS, xs, j);
            } else if (!TAIL) {
                load_w(s + WS, ws, j - XL);
            }
        };
        phase(half1, none, mid, [&](int j) { read(0, ws1, xs1, j); }, load);
        fc_wait_lds();
        __builtin_amdgcn_sched_barrier(0);
        phase(none, mid, all, [&](int j) { read(1, ws1, xs1, j); }, load);
        ws = ws1;
        xs = xs1;
    };
    int s = 0;
    for (; s + WS < n_stages; ++s) stage(s, std::false_type());
    for (; s + 1 < n_stages; ++s) stage(s, std::true_type());
    fc_wait_vm<0, true>();
    phase(half1, none, none, [](int) {}, no_load);

    // ---- epilogue; the LDS ring is its staging area, once every wave has left it
    if constexpr (EPI == 4) {
        const int hs = (pair0 >> 6) + wn;
        if (hs < p.slot_base + p.slots_here)  // an odd number of slabs leaves the last pair half empty
            gemm_epilogue_vocab<MT>(p, acc, hs, m0 + 16 * MT * wm, lane);
    } else {
        uint16_t *bias_area = (uint16_t *)(smem + 4 * epi_bytes(MT, NT));
        __builtin_amdgcn_s_barrier();
        if (EPI == 0) {
            if (tid < WROWS) bias_area[tid] = bias;
            fc_wait_lds();
            __builtin_amdgcn_s_barrier();
        }
        bias_area += wn * 16 * NT;
        gemm_epilogue<MT, NT, EPI>(p, acc, smem + wave * epi_bytes(MT, NT), bias_area, bias_area + 8 * NT, pair0 + wn * 8 * NT, pair_end,
                                   m0 + 16 * MT * wm, lane, at.kpart);
    }
}

// Tiles of `pairs` pairs x `rows` window rows; the grid, a multiple of eight, or 0: not a launch.
template <int EPI>
unsigned set_tiles(GemmArgs &a, int pairs, int rows)
{
    if (a.slots_here < 1 || a.slot_base < 0 || a.slot_base + a.slots_here > a.n_slots || a.m_base < 0 || a.m_end > a.M || a.m_end <= a.m_base ||
        (EPI == 3 && a.ksplit < 1))
        return 0;
    a.n_units = (int)(((int64_t)a.slots_here * 64 + pairs - 1) / pairs);
    a.n_mt = (a.m_end - a.m_base + rows - 1) / rows;
    a.by_mt.set(a.n_mt);
    a.by_parts.set(a.ksplit);
    a.by_a.set(a.A);
    const int64_t n_tiles = (int64_t)a.n_units * a.n_mt * (EPI == 3 ? a.ksplit : 1);
    return n_tiles > (1 << 30) ? 0 : (unsigned)((n_tiles + 7) / 8 * 8);
}

template <int MT, int NT, int WN, int WS, int XS, int EPI>
hipError_t launch_wide(GemmArgs a, hipStream_t s)
{
    constexpr int LDS = (WS * 16 * NT * WN + XS * 256) * 128;
    static_assert(LDS <= 160 * 1024, "LDS ring too large");
    const unsigned grid = set_tiles<EPI>(a, 8 * NT * WN, 256);
    if (grid == 0 || a.K % 64 != 0) return hipErrorInvalidValue;
    auto start = [&](auto once) {
        constexpr auto kernel = k_gemm_wide<MT, NT, WN, WS, XS, EPI, decltype(once)::value>;
        static hipError_t attr = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (attr != hipSuccess) return attr;
        kernel<<<dim3(grid), dim3(256), LDS, s>>>(a);
        return hipGetLastError();
    };
    // One tile of rows: its workgroups are the only ones to read their weights.
    return a.once && a.M <= 256 ? start(std::true_type()) : start(std::false_type());
}

template <int KS, int NW, int NSUB, int SLOTS, int NL, int EPI>
hipError_t launch_gemm(GemmArgs a, hipStream_t s)
{
    constexpr int XROWS = 32 * NW;
    constexpr int LDS = SLOTS * (32 * NSUB + XROWS) * KS * 2 + (EPI == 0 ? BIAS_LDS : 0);
    static_assert(LDS <= 160 * 1024, "LDS ring too large");
    const unsigned grid = set_tiles<EPI>(a, 16 * NSUB, XROWS);
    if (grid == 0 || a.K % KS != 0) return hipErrorInvalidValue;
    auto start = [&](auto rotate, auto once) {
        constexpr auto kernel = k_proj_gemm<KS, NW, NSUB, SLOTS, NL, EPI, decltype(rotate)::value, decltype(once)::value>;
        static hipError_t attr = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (attr != hipSuccess) return attr;
        kernel<<<dim3(grid), dim3((NW + NL) * 64), LDS, s>>>(a);
        return hipGetLastError();
    };
    // One tile of rows: its workgroups are the only ones to read their weights.
    auto with_hint = [&](auto rotate) {
        return a.once && a.M <= XROWS ? start(rotate, std::true_type()) : start(rotate, std::false_type());
    };
    // (the 128-row half slab of the projection is here for a hidden size that is no multiple of 128)
    if constexpr (EPI != 3 && !(EPI == 0 && NW == 4 && NSUB == 2 && KS == 64))
        if (a.n_mt == 1 && a.m_base == 0 && a.K % 2048 == 0 && a.K / KS < 65536) {
            a.rot_step = (uint32_t)(((int64_t)(a.K / KS) << 16) / (a.n_units < 256 ? a.n_units : 256));  // (place * rot_step stays below 2^32)
            return with_hint(std::true_type());
        }
    return with_hint(std::false_type());
}

// Sum of the KS hidden-dimension parts of an EPI 3 launch + residual, four outputs per thread, all its loads under way at once: the
// kernel is a launch and one memory round trip.
template <int KS>
__global__ __launch_bounds__(256) void k_splitk_finish(const float *__restrict__ part, const uint16_t *res,
                                                       uint16_t *out, size_t quads, size_t plane)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= quads) return;
    float4 v[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) v[k] = *(const float4 *)(part + (size_t)k * plane + 4 * i);
    const uint2 rv = res ? *(const uint2 *)(res + 4 * i) : make_uint2(0, 0);
    __builtin_amdgcn_sched_barrier(0);
    float4 a = v[0];
#pragma unroll
    for (int k = 1; k < KS; ++k) {
        a.x += v[k].x;
        a.y += v[k].y;
        a.z += v[k].z;
        a.w += v[k].w;
    }
    if (res) {
        a.x += __uint_as_float(rv.x << 16);
        a.y += __uint_as_float(rv.x & 0xffff0000u);
        a.z += __uint_as_float(rv.y << 16);
        a.w += __uint_as_float(rv.y & 0xffff0000u);
    }
    uint2 w;
    w.x = (uint32_t)fc_bf16_bits(a.x) | ((uint32_t)fc_bf16_bits(a.y) << 16);
    w.y = (uint32_t)fc_bf16_bits(a.z) | ((uint32_t)fc_bf16_bits(a.w) << 16);
    *(uint2 *)(out + 4 * i) = w;
}

constexpr int MAX_PARTS = 16;
template <int KS = 2>
hipError_t launch_finish(const GemmArgs &a, hipStream_t s)
{
    if constexpr (KS > MAX_PARTS) return hipErrorInvalidValue;
    else {
        if (a.ksplit != KS) return launch_finish<KS + 1>(a, s);
        const size_t quads = (size_t)a.M * a.N / 4;
        k_splitk_finish<KS><<<dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s>>>(a.part, a.res, a.out, quads, (size_t)a.M * a.N);
        return hipGetLastError();
    }
}

// A launch in one tile shape (numbered below).  Loads of the 128-row shapes are issued by four extra waves: their four
// multiplying waves are alone on their SIMDs.  The half-head shape of the projection takes 128 hidden elements per
// stage where it can.
template <int EPI>
hipError_t launch_shape(int shape, const GemmArgs &a, hipStream_t s)
{
    switch (shape) {
    case 0: return launch_wide<4, 8, 1, 4, 3, EPI>(a, s);
    case 1: return launch_gemm<64, 4, 4, 4, 4, EPI>(a, s);
    case 2:
        if constexpr (EPI == 0)
            if (a.K % 128 == 0) return launch_gemm<128, 4, 2, 3, 4, EPI>(a, s);
        if constexpr (EPI != 4) return launch_gemm<64, 4, 2, 4, 4, EPI>(a, s);
        return hipErrorInvalidValue;
    case 3:
        return launch_wide<8, 8, 2, 3, 2, EPI>(a, s);
    case 4:
        if constexpr (EPI == 0 || EPI == 2) return launch_wide<8, 5, 2, 3, 3, EPI>(a, s);
        return hipErrorInvalidValue;
    case 5:
        if constexpr (EPI == 0 || EPI == 2) return launch_gemm<64, 4, 3, 4, 4, EPI>(a, s);
        return hipErrorInvalidValue;
    case 6:
        if constexpr (EPI == 0 || EPI == 2) return launch_gemm<64, 2, 5, 4, 4, EPI>(a, s);
        return hipErrorInvalidValue;
    case 7:
        if constexpr (EPI == 0 || EPI == 2) return launch_gemm<64, 2, 3, 4, 4, EPI>(a, s);
        return hipErrorInvalidValue;
    case 8:
        if constexpr (EPI == 0 || EPI == 2) return launch_gemm<64, 4, 5, 4, 4, EPI>(a, s);
        return hipErrorInvalidValue;
    case 9: return launch_gemm<64, 2, 4, 3, 2, EPI>(a, s);
    case 10:
        if constexpr (EPI == 4) return hipErrorInvalidValue;
        else return launch_gemm<64, 2, 2, 4, 4, EPI>(a, s);
    case 11:
        if constexpr (EPI == 0 || EPI == 2) return launch_wide<8, 6, 2, 3, 2, EPI>(a, s);
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

// Tile shapes of the tiled GEMM and what workgroups take per 64 hidden elements (us): the first round of them, one on every compute
// unit, nearly empty and full, a further round, and the share of one that its emptiest part takes.  One row tile, whose weights come from
// HBM, and several, which share them by way of L2, have figures of their own.  Fitted to 6000 measured launches, 917 problems: 24 .. 96
// head slots, gated layers of 2048 .. 22016 outputs, vocabularies of 32000 .. 152064, plain layers of 8192 .. 18944 outputs, hidden 1024 ..
// 8192, 8 .. 2304 rows, weights from HBM; rms error 8 %, and the shape it picks is 0.1 % slower than the best measured one in the
// mean, more than 4 % in three problems; the same on problems left out of the fit.  Per tile area the larger shapes are cheaper -- they
// move fewer bytes into the compute unit per product -- but leave the chip emptier at the end.
//   0: 256 rows x slab   1: 128 rows x slab   2: 128 rows x half slab   3: 256 rows x two slabs
//   4: 256 rows x 80 dealt pairs   5: 128 rows x 48 dealt pairs
//   6: 64 rows x 80 dealt pairs   7: 64 rows x 48 dealt pairs   8: 128 rows x 80 dealt pairs
//   9: 64 rows x slab   10: 64 rows x half slab   11: 256 rows x 96 dealt pairs
// 11 is for what fills one round in it and in no other, between the 160 and the 256 weight rows of 4 and 3 (us without and with): 36 head
// slots, hidden 3584, 2100 / 2200 / 2304 rows 73.0 / 75.5 / 74.7 and 67.1 / 67.6 / 67.3; 96 slots, hidden 4096, 780 / 1000 rows 89.4 / 89.3 and 80.3 /
// 80.6; gated 4096 x 12288, 260 / 400 rows 90.5 / 89.9 and 84.8 / 84.7, 3584 x 11008, 350 rows 76.4 and 68.9; 36 such problems 1.056 x in the mean. In
// several rounds 3 is as good (fitted to those too, it was taken for 3584 x 18944, 2304 rows: 470 -> 484), so its further rounds are
// set to cost what keeps it out of them.
// 6 .. 10 are for few rows, where the weights alone should count: in the 128-row half slab, for 40 or 64 rows the shape with
// the most tiles, the compute units pulled three bytes for every byte of weights (two thirds of them window rows, most
// of those padding); 64 rows x 160 weight rows pull 1.4.  Gated W_1 of 18944 outputs at hidden 3584, 64 / 128 rows:
// 65 / 80 us in the half slab, 44.7 / 50.3 in those (shapes 6 and 8; the weights alone 46 at 5.9 TB/s).
constexpr int N_SHAPES = 12;
struct ShapeCost {
    double least, first, further, start;
};
constexpr ShapeCost SHAPE_US[2][N_SHAPES] = {  // one row tile, several
    {{0.60, 0.87, 0.80, 0.75}, {0.41, 0.52, 0.66, 0.95}, {0.24, 0.36, 0.38, 0.87}, {0.85, 1.34, 1.36, 0.79},
     {0.63, 1.01, 1.04, 0.80}, {0.36, 0.45, 0.48, 0.95}, {0.47, 0.49, 0.67, 0.96}, {0.31, 0.31, 0.39, 1.00},
     {0.58, 0.58, 0.79, 0.87}, {0.47, 0.47, 0.45, 0.93}, {0.21, 0.24, 0.25, 0.99}, {0.75, 1.17, 1.17, 0.80}},
    {{0.58, 0.82, 0.90, 0.59}, {0.50, 0.53, 0.58, 0.76}, {0.25, 0.34, 0.37, 0.79}, {1.07, 1.35, 1.52, 0.79},
     {0.77, 0.99, 1.05, 0.73}, {0.33, 0.43, 0.47, 0.85}, {0.46, 0.51, 0.53, 0.85}, {0.26, 0.35, 0.31, 0.70},
     {0.55, 0.64, 0.70, 0.80}, {0.51, 0.51, 0.36, 0.67}, {0.17, 0.22, 0.22, 0.77}, {0.90, 1.16, 1.60, 0.90}}};
constexpr bool shape_dealt(int shape) { return (shape >= 4 && shape <= 8) || shape == 11; }
constexpr bool shape_half(int shape) { return shape == 2 || shape == 10; }

int64_t tiles_of(int shape, int64_t slots, int64_t rows)
{
    const int64_t t256 = (rows + 255) / 256, t128 = (rows + 127) / 128, t64 = (rows + 63) / 64;
    switch (shape) {
    case 0: return slots * t256;
    case 1: return slots * t128;
    case 2: return 2 * slots * t128;
    case 3: return (slots + 1) / 2 * t256;
    case 4: return (slots * 64 + 79) / 80 * t256;
    case 5: return (slots * 64 + 47) / 48 * t128;
    case 6: return (slots * 64 + 79) / 80 * t64;
    case 7: return (slots * 64 + 47) / 48 * t64;
    case 8: return (slots * 64 + 79) / 80 * t128;
    case 9: return slots * t64;
    case 11: return (slots * 64 + 95) / 96 * t256;
    default: return 2 * slots * t64;
    }
}

// Estimated time of one launch per 64 hidden elements: the workgroups and the weights, from HBM at 7.2 TB/s (several row tiles: 5.0),
// joined by a 4-norm.
double launch_cost(int shape, int64_t slots, int64_t rows)
{
    const int tile_rows = shape == 0 || shape == 3 || shape == 4 || shape == 11 ? 256 : shape == 6 || shape == 7 || shape >= 9 ? 64 : 128;
    const bool several = rows > tile_rows;
    const ShapeCost c = SHAPE_US[several][shape];
    const int64_t n = tiles_of(shape, slots, rows), full = n / 256;
    const double part = (double)(n % 256) / 256.0;
    const double tiles = full == 0 ? c.least + (c.first - c.least) * part
                                   : c.first + c.further * ((double)(full - 1) + (part > 0.0 ? c.start + (1.0 - c.start) * part : 0.0));
    const double weights = (double)slots * 128 * 128 / (several ? 5.0e6 : 7.2e6);
    const double t2 = tiles * tiles, w2 = weights * weights;
    return sqrt(sqrt(t2 * t2 + w2 * w2));
}

// A problem is covered by one launch, or cut in two where the last round of workgroups would be nearly empty:
// the first launch takes whole rounds and the second, in a smaller tile, the other slabs or the last rows.
// The cut, the second launch (about 3 us) and the shapes are the cheapest by the estimate above: 2304 rows x 296
// gated slabs, hidden 3584: 284 slabs in 1278 tiles of shape 3 (4.99 rounds) and 12 in shape 1; 256
// rows x 296: 237 tiles of shape 4 in one round; 2048 rows x 36 head slots: 232 tiles of shape 4.
struct GemmPiece {
    int shape, slot_base, slots, m_base, m_end;
};
int plan_pieces(int slots, int M, int K, bool allow_half, bool allow_dealt, GemmPiece out[2])
{
    const bool no_split = fc_knobs().gemm_no_split != 0;  // tuning knob
    // Two 64-row half slabs on a compute unit against one 128-row slab: more than 512 rows, 257 .. 512 such tiles.  The half slabs start and end
    // sooner, and the slabs move fewer bytes, so that the hidden dimension decides (us, half slabs first): 2048 x 2176, 930 rows
    // 16.9 and 19.4, 2560 x 2816, 704 rows 24.3 and 27.2, 3584 x 3584, 525 rows 29.2 and 29.9, but 8192 x 2176, 930 rows 59.8 and 58.3, 10240 x 1280,
    // 1537 rows 82.4 and 70.7, 18944 x 3584, 525 rows 135 and 127.
    const bool no64 = M > 512 && K > 4096 && tiles_of(10, slots, M) > 256;
    double best = 1e30;
    int n = 1;
    for (int sh = 0; sh < N_SHAPES; ++sh) {
        if ((shape_half(sh) && !allow_half) || (shape_dealt(sh) && !allow_dealt) || (no64 && (sh == 9 || sh == 10))) continue;
        const double c = launch_cost(sh, slots, M);
        if (c < best) {
            best = c;
            out[0] = GemmPiece{sh, 0, slots, 0, M};
        }
    }
    if (no_split) return 1;
    const double extra = 3.0 / (K / 64), short_by = 1.03;  // (estimates of two launches come out short: 130 measured cuts)
    for (int sh = 0; sh <= 3; sh += 3) {
        const int64_t per = sh == 3 ? 2 : 1, t256 = (M + 255) / 256, units = (slots + per - 1) / per;
        for (int64_t rounds = units * t256 / 256; rounds >= 1 && rounds >= units * t256 / 256 - 1; --rounds) {
            const int64_t u1 = rounds * 256 / t256, s1 = u1 * per;          // slabs of the first launch
            const int64_t r1 = rounds * 256 / units, m1 = r1 * 256;         // or its row tiles
            for (int s2 = 0; s2 <= 3; ++s2) {
                if (s2 == sh || (s2 == 2 && !allow_half)) continue;  // (two launches of one shape take what one does, and the second's start)
                if (u1 >= 1 && s1 < slots) {
                    const double c = short_by * (launch_cost(sh, s1, M) + launch_cost(s2, slots - s1, M)) + extra;
                    if (c < best) {
                        best = c;
                        n = 2;
                        out[0] = GemmPiece{sh, 0, (int)s1, 0, M};
                        out[1] = GemmPiece{s2, (int)s1, (int)(slots - s1), 0, M};
                    }
                }
                if (r1 >= 1 && m1 < M) {
                    const double c = short_by * (launch_cost(sh, slots, m1) + launch_cost(s2, slots, M - m1)) + extra;
                    if (c < best) {
                        best = c;
                        n = 2;
                        out[0] = GemmPiece{sh, 0, slots, 0, (int)m1};
                        out[1] = GemmPiece{s2, 0, slots, (int)m1, M};
                    }
                }
            }
        }
    }
    return n;
}

template <int EPI>
hipError_t launch_pieces(GemmArgs a, hipStream_t s)
{
    GemmPiece pc[2];
    const int n = plan_pieces(a.n_slots, a.M, a.K, EPI != 4, EPI == 0 || EPI == 2, pc);
    for (int i = 0; i < n; ++i) {
        a.slot_base = pc[i].slot_base;
        a.slots_here = pc[i].slots;
        a.m_base = pc[i].m_base;
        a.m_end = pc[i].m_end;
        const hipError_t e = launch_shape<EPI>(pc[i].shape, a, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// At most 32 rows of a gated layer or a vocabulary: the tiled GEMM streams the weights a little faster than the whole-row
// kernel (6.3 TB/s instead of 6) where its tiles fill one round of workgroups, and more slowly otherwise.  Both sides measured, weights from HBM (us at 16 / 32 rows, tiled GEMM first):
//   gated, hidden 3584: 6400 outputs (200 half slabs) 20.3 and 21.7 / 20.8 and 23.5, 8192 (256) 22.1 and 24.0 / 22.8 and 25.4,
//   9472 (198 tiles of 48 dealt pairs) 26.3 and 29.1 / 27.4 and 31.0, 12288 (256) 32.3 and 33.2 / 32.7 and 34.7, 13312 (208 slabs)
//   35.5 and 36.5 / 36.5 and 38.1, 16384 (256) 41.2 and 42.5 / 41.8 and 44.2, 18944 (237 tiles of 80 dealt pairs) 47.5 and 49.7 /
//   48.5 and 51.3, 22016 63.4 and 59.8 / 66.0 and 62.0;
//   gated, hidden 4096: 6400 23.2 and 24.1 / 23.8 and 26.2, 8192 24.2 and 33.6 / 24.3 and 33.8, 11008 (230 tiles of 48) 32.1 and 36.5 /
//   32.4 and 38.5, 12288 35.5 and 37.9 / 35.8 and 40.2, 14336 41.0 and 42.7 / 41.7 and 45.4, 16384 47.3 and 46.1 / 47.6 and 49.1, 18944
//   52.8 and 56.0 / 53.7 and 58.7, 22016 71.3 and 68.7 / 73.7 and 70.7;
//   vocabulary, against the runs of entries (k_vocab_runs; hidden 4096 up to 30719 entries: whole rows), with the merge, us at 4 / 32 rows: hidden
//   3584, 26624 (208 slabs) 40.4 and 39.0 / 41.4 and 41.0, 29056 42.3 and 43.6 / 43.0 and 45.7, 32000 (250) 45.2 and 46.2 / 45.6 and 47.0, 32768 45.9 and
//   46.6 / 46.4 and 47.7; hidden 4096, 26624 42.0 and 44.2 / 42.7 and 46.2, 29056 44.7 and 49.8 / 45.1 and 52.1, 32000 49.3 and 51.9 / 49.7 and 53.4, 32768 49.7
//   and 52.8 / 49.7 and 53.3.
//   Two rounds of tiles (hidden 3584, 59392 .. 65536 entries) are within 2 % of them either way, the runs ahead at most sizes (59392 69.1
//   and 68.4 / 71.4 and 69.6, 62080 71.4 and 71.7 / 73.1 and 73.1, 65536 75.1 and 74.5 / 75.8 and 75.9), and so left to them.
bool wide_beats_rows(int mode, int M, int64_t slabs)
{
    auto in = [](int64_t n, int64_t lo) { return n >= lo && n <= 256; };
    if (mode == FC_LIN_VOCAB) return in(slabs, 208);
    const int64_t pairs48 = tiles_of(7, slabs, M);
    return in(tiles_of(10, slabs, M), 200) || in(tiles_of(9, slabs, M), 208) || in(pairs48, 192) ||
           (slabs > 256 && in(tiles_of(6, slabs, M), 208));
}

// Layers without pairs (EPI 1, 3): a launch of at most one round of workgroups, the hidden dimension in `parts` parts (1: uncut, without the
// sum).  A workgroup takes `start` and each 64 hidden elements, a + b x with x of the compute units in use, for one row tile (weights
// from HBM at 6.8 TB/s) and several (by way of L2, 5.3); the partial sums are written and read at 2 TB/s together, and their sum is a launch
// of its own.  Fitted to 8000 measured launches of this kind: 14 matrices of 2048 x 2048 .. 18944 x 3584, 24 .. 2304 rows, weights from
// HBM; rms error 7 % for those near the best.  The tile and number of parts it picks are 1.2 % slower than the best in the mean.
struct PartCost {
    int shape;
    double start, one_a, one_b, more_a, more_b;
};
constexpr PartCost PART_US[] = {{0, 2.18, 0.490, 0.363, 0.544, 0.235}, {1, 2.21, 0.405, 0.209, 0.413, 0.116},
                                {2, 1.56, 0.291, 0.090, 0.269, 0.071}, {3, 0.00, 0.929, 0.451, 0.944, 0.338},
                                {9, 2.01, 0.523, 0.001, 0.512, 0.001}, {10, 1.13, 0.290, 0.003, 0.208, 0.063}};
double part_cost(const PartCost &c, int64_t tiles, int64_t M, int64_t K, int64_t N, int parts)
{
    const bool several = M > (c.shape == 0 || c.shape == 3 ? 256 : c.shape < 9 ? 128 : 64);
    const double x = (double)(tiles * parts) / 256.0, weights = (double)K * N * 2.0 / (several ? 5.30e6 : 6.81e6);
    const double loop = c.start + (double)K / KS_MIN / parts * (several ? c.more_a + c.more_b * x : c.one_a + c.one_b * x);
    const double l2 = loop * loop, w2 = weights * weights;
    return sqrt(sqrt(l2 * l2 + w2 * w2)) + (parts > 1 ? 3.71 + (double)parts * M * N * 4.0 / 1.96e6 : 1.83);
}

// The tile and the parts that a layer takes with so many bytes for partial sums.  A few row tiles of a long hidden dimension fill a round
// well in parts only: 18944 x 3584, 480 / 580 / 760 rows, uncut 128-row half slabs 111 / 142 / 166 us, 256-row slabs in 4 / 3 / 3 parts 77 / 98 /
// 101; 12288 x 4096, 360 / 760 rows 75 / 113 and 57 / 86; 1200 rows, more than one round of any tile, 256 x 256 in three parts 144 -> 113.  The
// estimate of the uncut launches is that of plan_pieces, or that of one round here where it is the larger; it has to be beaten by 7 %,
// and where a round would be less than three quarters full may be missed by 5 %.  Against parts for fewer than 192 workgroups
// of 128 rows x half a slab, by fill rates (the rule that says what space a call must bring), over 211 drawn problems where the two
// differ: 1.14 x in the mean, up to 1.64 x, 21 slower by more than 3 % (worst: 5120 x 6144, 99 rows 23.1 -> 25.6; 13824 x 5120, 120 rows
// 37.0 -> 39.7).  The better of both by measurement would be 1.147 x; a fit to these as well leaves 16 slower at the same mean.
void choose_parts(FcWidePlan &p, int M, int K, int N, size_t cap)
{
    const int64_t units = N / 128;
    const int stages = K / KS_MIN;
    GemmPiece pc[2];
    const int pieces = plan_pieces((int)units, M, K, true, false, pc);
    double uncut = 0.0, round = 1e30;
    for (int i = 0; i < pieces; ++i) uncut += launch_cost(pc[i].shape, pc[i].slots, pc[i].m_end - pc[i].m_base) * stages;
    uncut = uncut * 0.99 + 3.45 * pieces;
    for (const PartCost &c : PART_US) {
        const int64_t tiles = tiles_of(c.shape, units, M);
        if (tiles <= 256) round = fmin(round, part_cost(c, tiles, M, K, N, 1));
    }
    if (round < 1e30) uncut = fmax(uncut, round);
    double best = uncut * (2 * units * ((M + 127) / 128) >= 192 ? 0.93 : 1.05);
    for (const PartCost &c : PART_US) {
        const int64_t tiles = tiles_of(c.shape, units, M);
        for (int parts = 2; parts <= MAX_PARTS && parts <= stages / 8 && tiles * parts <= 256; ++parts) {
            if ((size_t)parts * M * N * sizeof(float) > cap) break;
            const double t = part_cost(c, tiles, M, K, N, parts);
            if (t < best) {
                best = t;
                p.shape = c.shape;
                p.ksplit = parts;
            }
        }
    }
}

// The parts for which a call has to bring space: of layers that fill less than three quarters of a round uncut, by a workgroup's fill
// rate and the rate of the partial sums.  (With that much a call may find a better plan, with more a better one still.)
void required_parts(FcWidePlan &p, int mode, int M, int K, int N)
{
    const int64_t units = N / (mode == FC_LIN_GATE_UP ? 64 : 128), t256 = (M + 255) / 256, t128 = (M + 127) / 128;
    if (M <= 128 && units >= 192) p.shape = mode == FC_LIN_VOCAB ? 1 : 2;
    else if (units * t256 >= 192) p.shape = 0;
    else if (units * t128 >= 144 || mode == FC_LIN_VOCAB) p.shape = 1;
    else p.shape = 2;
    if (mode != FC_LIN_RESIDUAL || p.shape != 2 || 2 * units * t128 >= 192) return;
    const int64_t stages = K / KS_MIN;
    double best = 1e30;
    for (const int sh : {0, 1, 2, 9, 10}) {
        const int64_t rows = sh == 0 ? 256 : sh < 3 ? 128 : 64, wrows = shape_half(sh) ? 64 : 128;
        if (rows == 64 && M > 64) continue;
        const int64_t tiles = tiles_of(sh, units, M);
        for (int64_t ks = 1; ks <= MAX_PARTS; ++ks) {
            if (ks > 1 && ks > stages / 8) break;
            const int64_t wg = tiles * ks;
            if (wg > 288) break;
            const double fill_us = (double)((wg + 255) / 256) * (double)(rows + wrows) * (double)(K / ks) * 2.0 / 50e3;
            const double part_us = ks > 1 ? (double)ks * M * N * 8.0 / 3e6 : 0.0;
            if (fill_us + part_us < best) {
                best = fill_us + part_us;
                p.shape = sh;
                p.ksplit = (int)ks;
            }
        }
    }
}

}  // namespace

// Tiled-GEMM plan of a plain linear layer (host, pure function of the shape and the space for partial sums); kind 0: not for this kernel.
FcWidePlan fc_plan_wide(int dtype, int mode, int M, int K, int N, size_t cap)
{
    FcWidePlan p;
    p.kind = 0;
    p.shape = 0;
    p.ksplit = 1;
    p.required = 0;
    const int per_slab = mode == FC_LIN_GATE_UP ? 64 : 128;  // FC_LIN_VOCAB: slabs of 128 vocabulary rows
    if (dtype != FC_BF16 || M < 1 || K < 4 * KS_MIN || K % KS_MIN != 0 || N < per_slab || N % per_slab != 0) return p;
    // 32-bit byte offsets inside X and each weight matrix
    if ((int64_t)N * K * 2 >= ((int64_t)1 << 32) || (int64_t)M * K * 2 >= ((int64_t)1 << 32)) return p;
    // At most 32 rows: gated layers and vocabularies see above.  W_out and W_2 in parts against the slice-wise kernel, which has
    // a second launch too and pulls a window slice per 128 weight rows: a large matrix, more than 16 rows (us at 24 rows,
    // tiled GEMM first: 18944 x 3584 30.1 and 31.2, 16384 x 4096 37.0 and 43.1, 8192 x 8192 35.6 and 41.7, 24576 x 4096 41.0 and 42.0;
    // 16 rows of the first 29.7 and 29.6).  Below the line it is mixed: 16384 x 3584 30.7 and 27.4, 12288 x 4096 25.0 and 25.0,
    // 12288 x 3584 22.6 and 23.2, 10240 x 5120 24.2 and 26.3.
    const FcKnobs &knobs = fc_knobs();
    if (M <= 32) {
        const FcSkinnyPlan rows = fc_plan_skinny(dtype, mode, M, K, N);
        const bool knob = knobs.lin_wide_shape >= 6;
        if (!knob && (knobs.lin_wgs > 0 || knobs.lin_no_rows)) return p;  // tuning knobs of the streaming kernels
        if (!knob && !(mode == FC_LIN_RESIDUAL ? rows.kind == 1 && M > 16 && (double)K * N >= 60e6
                                               : rows.kind == 2 && K >= 2048 && wide_beats_rows(mode, M, N / per_slab)))
            return p;
    }
    p.kind = 1;
    // (The shape counts only where the hidden dimension is cut into parts or a tuning knob asks for one shape;
    // everything else goes through plan_pieces at launch.)
    required_parts(p, mode, M, K, N);
    if (knobs.lin_wide_shape >= 0 || knobs.lin_ksplit > 0) {  // tuning knobs
        const int v = knobs.lin_wide_shape, ks = knobs.lin_ksplit;
        if (v >= 0 && v < N_SHAPES && (!shape_half(v) || mode != FC_LIN_VOCAB) && (!shape_dealt(v) || mode == FC_LIN_GATE_UP)) p.shape = v;
        if (ks >= 1 && ks <= MAX_PARTS && ks <= K / KS_MIN / 4 && mode == FC_LIN_RESIDUAL) p.ksplit = ks;
        p.required = fc_wide_workspace(p, M, N);
        return p;
    }
    p.required = fc_wide_workspace(p, M, N);
    if (mode == FC_LIN_RESIDUAL && cap >= p.required) {
        p.ksplit = 1;
        choose_parts(p, M, K, N, cap);
    }
    return p;
}

size_t fc_wide_workspace(const FcWidePlan &p, int M, int N)
{
    return p.kind == 1 && p.ksplit > 1 ? (size_t)p.ksplit * M * N * sizeof(float) : 0;
}

hipError_t fc_launch_linear_wide(const FcWidePlan &pl, int mode, const void *x, const void *w, const void *w2,
                                 const void *res, int M, int K, int N, void *out, void *workspace, bool once, hipStream_t s,
                                 const FcArgmaxPart *am)
{
    if (pl.kind != 1 || (pl.ksplit > 1 && !workspace)) return hipErrorInvalidValue;
    GemmArgs a;
    memset(&a, 0, sizeof a);
    a.X = (const uint16_t *)x;
    a.W = (const uint16_t *)w;
    a.W2 = (const uint16_t *)w2;
    a.res = (const uint16_t *)res;
    a.out = (uint16_t *)out;
    a.part = (float *)workspace;
    a.M = M;
    a.A = M;
    a.K = K;
    a.N = N;
    a.n_slots = mode == FC_LIN_GATE_UP ? N / 64 : N / 128;
    a.ksplit = pl.ksplit;
    a.once = once;
    a.slot_base = 0;
    a.slots_here = a.n_slots;
    a.m_base = 0;
    a.m_end = M;
    const bool forced = fc_knobs().lin_wide_shape >= 0;  // a forced shape is used for the whole problem
    if (mode == FC_LIN_VOCAB) {
        if (!am) return hipErrorInvalidValue;
        a.am = *am;
        return forced ? launch_shape<4>(pl.shape, a, s) : launch_pieces<4>(a, s);
    }
    if (mode == FC_LIN_GATE_UP) return forced ? launch_shape<2>(pl.shape, a, s) : launch_pieces<2>(a, s);
    if (pl.ksplit <= 1) return forced ? launch_shape<1>(pl.shape, a, s) : launch_pieces<1>(a, s);
    hipError_t e = launch_shape<3>(pl.shape, a, s);
    if (e != hipSuccess) return e;
    return launch_finish(a, s);
}

bool fc_project_gemm_supported(const fc_config &cfg, int M)
{
    // 32-bit byte offsets inside X and W; the hidden dimension in whole stages
    const int64_t n = (int64_t)(cfg.n_q_heads + 2 * cfg.n_kv_heads) * cfg.head_dim;
    return cfg.dtype == FC_BF16 && cfg.head_dim == 128 && cfg.hidden % KS_MIN == 0 && M >= 1 &&
           n * cfg.hidden * 2 < ((int64_t)1 << 32) && (int64_t)M * cfg.hidden * 2 < ((int64_t)1 << 32);
}

// Estimated time of the tiled projection of up to 256 rows (us; 24 .. 96 head slots, hidden 1024 .. 8192, 40 .. 240 rows: within a tenth
// of the measured times in the mean).
double fc_project_gemm_us(int slots, int M, int K)
{
    GemmPiece pc[2];
    double c = 0.0;
    const int n = plan_pieces(slots, M, K, true, true, pc);
    for (int i = 0; i < n; ++i) c += launch_cost(pc[i].shape, pc[i].slots, pc[i].m_end - pc[i].m_base) * (K / 64);
    return 3.0 * n + M / 64.0 + (M <= 128 ? 1.12 : 1.0) * c;
}

hipError_t fc_launch_project_gemm(const FcGeom &G, const void *x, const void *w, const void *bias,
                                  const int32_t *pos, int win_start, int A, void *q_out, void *k_layer,
                                  void *v_layer, hipStream_t s)
{
    GemmArgs a;
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
    a.n_mt = a.n_units = 0;
    a.n_slots = G.Hq + 2 * G.Hkv;
    a.W2 = a.res = nullptr;
    a.out = nullptr;
    a.part = nullptr;
    a.N = 0;
    a.once = G.once;
    a.ksplit = 1;
    a.rot1 = exp(-G.log_base / 64.0);
    a.rot8 = exp(-G.log_base / 8.0);
    a.rot16 = exp(-G.log_base / 4.0);
    a.rot32 = exp(-G.log_base / 2.0);
    a.slot_base = 0;
    a.slots_here = a.n_slots;
    a.m_base = 0;
    a.m_end = a.M;
    if (fc_knobs().proj_gemm_shape >= 0) return launch_shape<0>(fc_knobs().proj_gemm_shape, a, s);  // tuning knob: one shape for all
    return launch_pieces<0>(a, s);
}
