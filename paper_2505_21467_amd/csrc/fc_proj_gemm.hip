// QKV projection of a wide window (hundreds to thousands of rows: refreshes, batched blocks) as a
// tiled matrix-core GEMM (bf16, head_dim 128), fused with bias, rotary embedding and the scatter into
// the cache.  Table 1's "W_Q, W_K, W_V projections" row with L replaced by the window length.
//
// Y^T = W X^T: the weight rows are the A operand of v_mfma_f32_32x32x16_bf16 and the window rows the B
// operand, so a lane of the accumulator holds 16 output features of ONE window row.  A wave owns 32
// window rows and all NSUB 32-feature sub-tiles of its workgroup; with NSUB = 4 the workgroup covers a
// whole head (features i and i + 64 of a rotary pair sit in sub-tiles t and t + 2, same lane, same
// register), with NSUB = 2 it covers the rotary-paired half head {32 h .. 32 h + 31} u {64 + 32 h ..}
// (more, smaller workgroups when the window is too short to fill the chip).  The rotation, the bias and
// the stores to q_out / the K rows / the transposed V tiles therefore need no exchange between lanes.
// A second kernel, k_gemm_pp, covers 256 window rows x two heads.  Two more shapes (NSUB = 5, 3) deal the rotary pairs of all head slots, laid end to end, 80 or 48 to a
// workgroup (16 per sub-tile, low rows then high rows: the partner of register r is register r + 8): a
// quarter more work per workgroup than a head for grids that would otherwise be a little more than one
// round, a quarter less for grids well short of one.
//
// Both operands are contiguous along the hidden dimension.  64 (or 128) hidden elements of every row
// of the tile (128- or 256-byte row pieces) stream HBM/L2 -> LDS with direct-to-LDS 16-byte loads into
// a ring of two to four stages; the 16-byte chunks of a row piece are XOR-swizzled with bits 1..3 (or
// 0..3) of the row (applied to the global address of the loading lane), which spreads the 16 lanes the
// LDS serves per clock over 16 different bank groups.
//
// A wave that issues a direct-to-LDS load waits until the memory pipeline has taken it (about 46
// cycles per load measured), and that wait is not hidden when the wave is alone on its SIMD.  The
// 128-row shapes (four multiplying waves) therefore carry four more waves that do nothing but issue
// the loads; in the 256-row shapes (two multiplying waves per SIMD) every wave issues its share, a
// quarter at a time between its multiplies.
#include <math.h>
#include <string.h>

#include <type_traits>

#include "fc_device.h"
#include "fc_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

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
    int n_mt;              // row tiles of 32 * NW window rows
    int n_units;           // head slots (NSUB = 4) or half-head slots (NSUB = 2)
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

// bytes of LDS a wave needs for its epilogue: 32 rows of NT sub-tiles in fp32, 16 bytes of padding each
__host__ __device__ constexpr int epi_bytes(int NT) { return 32 * (NT * 128 + 16); }

// The workgroup's bias goes to LDS at the very start: nothing else asks for it before the end, and a layer's bias
// comes from HBM (2.5 us with the matrix core idle when the epilogue fetched it).  NPW pairs: the low values, then
// the high ones; pairs (2 d, 2 d + 1) of all slabs laid end to end, from pair `first` on.  One wave calls this.
// A direct load takes two values from a 4-byte address; a bias that starts at an odd element goes through registers.
constexpr int BIAS_LDS = 512;
__device__ __forceinline__ void load_bias(const GemmArgs &p, unsigned char *dst, int first, int npw, int n_pairs, int lane)
{
    if (!p.bias) return;
    for (int d0 = 0; d0 < npw; d0 += 64) {
        const int d = d0 + lane;
        if (d >= npw) break;
        const bool high = d >= npw / 2;
        const int pr = min(first + 2 * (high ? d - npw / 2 : d), n_pairs - 2);
        const uint16_t *src = p.bias + (pr >> 6) * 128 + (pr & 63) + (high ? 64 : 0);
        if (((uintptr_t)p.bias & 3) == 0)
            __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)src,
                                             (void __attribute__((address_space(3))) *)(dst + d0 * 4), 4, 0, 0);
        else
            *(uint32_t *)(dst + d * 4) = (uint32_t)src[0] | ((uint32_t)src[1] << 16);
    }
    fc_wait_lds();  // LDS writes done, if any
}

// Epilogue of a wave.  Lane (col, hi) of sub-tile i holds window row m_first + 32 i + col; register r of
// sub-tile t is row 8 (r >> 2) + 4 hi + (r & 3) of the sub-tile.  Sub-tiles are, in units of 32 features of slab hs:
// t for a whole slab (NT = 4), {half, half + 2} for a half slab (NT = 2); or (DEALT) 16 pairs each, the low rows in
// registers 0..7 and the high rows in 8..15, starting with pair pair0 of all slabs laid end to end, nt of them.
// Either way the tile is a row of "low" and a row of "high" values per window row; the two members of a pair
// (rotary pair, gate and up product) have the same place in the two.
//
// The values go through LDS, 32 window rows at a time in the wave's own area: in the accumulator layout a
// store instruction covers 16 bytes of 32 different rows (128 KB of a 256 x 256 tile took 7.6 us to leave),
// read back as rows it covers 128 or 256 contiguous bytes.  The loop over eight-value pieces is not
// unrolled: this code runs once per tile, and unrolled it costs more in instruction fetches than in work.
template <int NT, int MW, int EPI, bool DEALT>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs &p, f32x16 (&acc)[MW][NT], unsigned char *area,
                                              const uint16_t *bias_low, const uint16_t *bias_high, int hs, int half, int pair0,
                                              int nt, int m_first, int lane, int kpart)
{
    constexpr int PITCH = NT * 128 + 16;         // bytes per window row: low values, high values, padding
    constexpr int HIGH = NT * 64;                // offset of the high values
    const FcGeom &G = p.G;
    const int col = lane & 31, hi = lane >> 5;
    const int first_v = G.Hq + G.Hkv;            // EPI 0: first value slab
#pragma unroll
    for (int i = 0; i < MW; ++i) {
        const int m_i = m_first + 32 * i;
        // EPI 0: sequence, window row and position of row m_i + col (pp < 0: padded or past the end)
        int b_l = 0, a_l = 0, pp_l = -1;
        if (EPI == 0 && m_i + col < p.m_end) {
            b_l = (m_i + col) / p.A;
            a_l = m_i + col - b_l * p.A;
            pp_l = p.pos ? p.pos[m_i + col] : p.win_start + a_l;
            if (pp_l >= G.max_seq) pp_l = -1;
        }
        if (EPI == 0 && (DEALT || hs >= first_v)) {
            // value rows go to the transposed tiles straight from the accumulators: lanes run along the keys
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int pr = pair0 + 16 * t, hs_t = DEALT ? pr >> 6 : hs;
                if (DEALT && (t >= nt || hs_t < first_v || hs_t >= p.n_slots)) continue;
                if (pp_l < 0) continue;
#pragma unroll
                for (int rq = 0; rq < 4; ++rq) {
                    const int d0 = DEALT ? (pr & 63) + 8 * (rq & 1) + 4 * hi + 64 * (rq >> 1)
                                         : 32 * (NT == 4 ? t : half + 2 * t) + 8 * rq + 4 * hi;
                    uint16_t *v = p.Vc + fc_v_index(G, b_l, hs_t - first_v, pp_l, d0);
                    // (the same place in the wave's low or high values as below)
                    const uint16_t *bs = DEALT ? (rq >= 2 ? bias_high : bias_low) + 16 * t + 8 * (rq & 1) + 4 * hi
                                               : (t >= NT / 2 ? bias_high : bias_low) + 32 * (t % (NT / 2 > 0 ? NT / 2 : 1)) + 8 * rq + 4 * hi;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        v[e * FC_VTILE] = fc_bf16_bits(acc[i][t][4 * rq + e] + (p.bias ? fc_to_float(bf16_t{bs[e]}) : 0.f));
                }
            }
            if (!DEALT) continue;
        }
        // ---- to LDS
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const bool high = DEALT ? rq >= 2 : t >= NT / 2;
                const int at = (DEALT ? 64 * t + 32 * (rq & 1) : 128 * (t % (NT / 2 > 0 ? NT / 2 : 1)) + 32 * rq) + 16 * hi;
                if (!DEALT || t < nt)
                    *(float4 *)(area + col * PITCH + (high ? HIGH : 0) + at) =
                        make_float4(acc[i][t][4 * rq], acc[i][t][4 * rq + 1], acc[i][t][4 * rq + 2], acc[i][t][4 * rq + 3]);
            }
        __builtin_amdgcn_wave_barrier();
        fc_wait_lds();
        // ---- and back as rows, eight low and eight high values per lane and step
        const int per_row = DEALT ? 2 * nt : NT * 2;  // pieces of eight pairs per row
#pragma unroll 1
        for (int u = lane; u < 32 * per_row; u += 64) {
            const int row = u / per_row, s = u - row * per_row;
            const int m = m_i + row;
            int b = 0, a = 0, pp = 0;
            if (EPI == 0) {
                b = __shfl(b_l, row, 64);
                a = __shfl(a_l, row, 64);
                pp = __shfl(pp_l, row, 64);
            }
            float lo[8], hv[8];
            const float *src = (const float *)(area + row * PITCH) + 8 * s;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                *(float4 *)(lo + 4 * h) = *(const float4 *)(src + 4 * h);
                *(float4 *)(hv + 4 * h) = *(const float4 *)(src + HIGH / 4 + 4 * h);
            }
            if (m >= p.m_end) continue;
            const int pr = pair0 + 8 * s;                     // DEALT: pair
            const int lf = DEALT ? pr & 63 : NT == 4 ? 8 * s : 32 * half + 8 * s;  // first low feature of the slab
            const int hs_t = DEALT ? pr >> 6 : hs;
            if (DEALT && hs_t >= p.n_slots) continue;
            if constexpr (EPI == 0) {
                if (DEALT && hs_t >= first_v) continue;
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
                    const float l = lo[e], h = hv[e];
                    lo[e] = l * c - h * sn;
                    hv[e] = h * c + l * sn;
                    f *= p.rot1;
                }
                if (hs_t < G.Hq) {
                    uint16_t *q = p.Q + (((size_t)b * G.Hq + hs_t) * p.A + a) * 128 + lf;
                    const uint4 ql = valid ? pack8(lo) : make_uint4(0, 0, 0, 0), qh = valid ? pack8(hv) : make_uint4(0, 0, 0, 0);
                    fc_store_any(q, ql);
                    fc_store_any(q + 64, qh);
                } else if (valid) {
                    uint16_t *k = p.Kc + fc_k_index(G, b, hs_t - G.Hq, pp, lf);
                    *(uint4 *)k = pack8(lo);
                    *(uint4 *)(k + 64) = pack8(hv);
                }
            } else if constexpr (EPI == 2) {
                float y[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) y[e] = silu_mul(lo[e], hv[e]);
                *(uint4 *)(p.out + (size_t)m * p.N + hs_t * 64 + lf) = pack8(y);
            } else {
                const size_t at = (size_t)m * p.N + (size_t)hs * 128 + lf;  // low features at `at`, high ones 64 on
                if constexpr (EPI == 3) {
                    float *o = p.part + (size_t)kpart * p.M * p.N + at;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        *(float4 *)(o + 4 * h) = *(float4 *)(lo + 4 * h);
                        *(float4 *)(o + 64 + 4 * h) = *(float4 *)(hv + 4 * h);
                    }
                } else {
                    if (p.res) {
                        union { uint4 u4; uint16_t h[8]; } rl, rh;
                        rl.u4 = *(const uint4 *)(p.res + at);
                        rh.u4 = *(const uint4 *)(p.res + at + 64);
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            lo[e] += fc_to_float(bf16_t{rl.h[e]});
                            hv[e] += fc_to_float(bf16_t{rh.h[e]});
                        }
                    }
                    *(uint4 *)(p.out + at) = pack8(lo);
                    *(uint4 *)(p.out + at + 64) = pack8(hv);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        fc_wait_lds();
    }
}

// Vocabulary mode (EPI 4): lane (col, hi) holds, for window row col, the logits 32 t + 8 (r >> 2) + 4 hi + (r & 3)
// of slab hs, ascending in (t, r), so that ties keep the smaller index; the other half is in lane ^ 32.  First the
// maximum and its place, then the sum of exponentials against it, by the hardware's exponential of a rounded product.
// On logits that are exact in fp32 the error of the confidences against 64 bits is 5 .. 10e-8, 0.87 times that of a running
// maximum with expf and 0.89 times that of expf in this form, which also takes longer (256 rows x 152064: 309.0 us, this
// 303.9); on others the logits' own error covers it.
template <int MW>
__device__ __forceinline__ void gemm_epilogue_vocab(const GemmArgs &p, const f32x16 (&acc)[MW][4], int hs, int m_first, int lane)
{
    const int col = lane & 31, hi = lane >> 5;
#pragma unroll
    for (int i = 0; i < MW; ++i) {
        const int m = m_first + 32 * i + col;
        float mx = -INFINITY, sm = 0.f;
        int arg = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const bool more = acc[i][t][r] > mx;
                mx = more ? acc[i][t][r] : mx;
                arg = more ? 32 * t + 8 * (r >> 2) + (r & 3) : arg;
            }
        arg += hs * 128 + 4 * hi;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) sm += __builtin_amdgcn_exp2f((acc[i][t][r] - mx) * 1.4426950408889634f);
        const float mx2 = __shfl_xor(mx, 32, 64), sm2 = __shfl_xor(sm, 32, 64);
        const int arg2 = __shfl_xor(arg, 32, 64);
        fc_argmax_merge(mx, arg, sm, mx2, arg2, sm2);
        if (hi == 0 && m < p.m_end) p.am.at(hs, m) = FcArgmax{mx, arg, sm};
    }
}

// Workgroup tile: NG head groups x WM row groups of waves (NW = NG * WM waves).  A wave owns MW
// 32-row sub-tiles of window rows and the NSUB 32-feature sub-tiles of one head (NSUB = 4) or of one
// rotary-paired half head (NSUB = 2).  SLOTS = stages in the LDS ring.
// NL = 0: every wave also issues its share of the loads; NL > 0: NL extra waves do nothing but issue
// the loads, so that the multiplying waves never wait for the memory pipeline to take a load.
// EPI selects the epilogue: 0 = QKV (bias, rotary embedding, scatter into the cache); the others are
// the plain linear layers of the rest of the layer, whose 128-row slabs of W take the place of the
// head slots: 1 = out = residual + x w^T; 2 = out = silu(x w_gate^T) * (x w_up^T), a slab being 64
// gate rows (sub-tiles 0, 1) and the same 64 up rows (sub-tiles 2, 3), so that both products of an
// output sit in one lane like a rotary pair; 3 = fp32 partial sums of one part of the hidden dimension
// (the parts are tiles of their own), for matrices with too few slabs to fill the chip; 4 = vocabulary projection of the
// unmasking step: of the 128 logits of a slab only the largest, its index and the sum of
// exp(logit - largest) are kept per row (NSUB = 4 only).
template <int KS, int NW, int NSUB, int MW, int NG, int SLOTS, int NL, int EPI, bool ROTATE, bool ONCE>
__global__ __launch_bounds__((NW + NL) * 64) void k_proj_gemm(GemmArgs p)
{
    constexpr int ROWB = KS * 2;               // bytes of one row piece: 128 or 256
    constexpr int CPR = ROWB / 16;             // 16-byte chunks per row piece
    constexpr int RPB = 1024 / ROWB;           // row pieces per 1 KB block (= one wave-wide load)
    constexpr int NKK = KS / 16;               // k-steps per stage
    constexpr int WM = NW / NG;
    constexpr int NLW = NL > 0 ? NL : NW;      // waves that issue loads
    constexpr bool DEALT = NSUB == 5 || NSUB == 3;
    constexpr int PPU = 16 * NSUB;             // DEALT: pairs per workgroup
    constexpr int WROWS = DEALT ? 32 * NSUB : 32 * NSUB * NG, XROWS = 32 * MW * WM;
    constexpr int WBYTES = WROWS * ROWB, STAGE = (WROWS + XROWS) * ROWB;
    constexpr int NBLK = (WROWS + XROWS) / RPB;  // 1 KB blocks per stage
    // NSUB = 5 or 3 ("dealt pairs", EPI 0 and 2 only): the workgroup takes 16 NSUB consecutive PAIRS of weight rows
    // -- rotary pairs (i, i + 64) of the head slots laid end to end, or (gate row, up row) pairs -- 16
    // pairs per sub-tile: the low rows in rows 0..15 of the sub-tile, the high rows in rows 16..31, so
    // that the two members of a pair sit in one lane, registers r and r + 8.  The 52 blocks of a stage
    // of the 80-pair shape do not divide by its eight waves: waves 0..3 issue seven loads per stage, waves
    // 4..7 six (the 48-pair shape has four loading waves of seven blocks each).
    // With NG = 2 the five sub-tiles are split between the two waves of a SIMD (sub-tiles 0..2 and 3..4),
    // each wave taking MW = 2 row sub-tiles: the pair of waves reads 5 + 4 fragments for its 6 + 4
    // multiplies of a k-step instead of 2 x 6 for 2 x 5 with 32-row waves (same time measured, less LDS
    // traffic).
    constexpr int NT = DEALT && NG == 2 ? (NSUB + 1) / 2 : NSUB;  // sub-tiles a wave owns (at most)
    constexpr int WBLK = WROWS / RPB;          // weight blocks of a stage (the first ones)
    constexpr int LBW = (NBLK + NLW - 1) / NLW;  // blocks per loading wave and stage (DEALT: at most)
    constexpr int WBW = WBLK / NLW;            // of which weight blocks (not DEALT)
    static_assert(KS == 64 || KS == 128, "stage depth");
    static_assert(NW % NG == 0 && (DEALT || (NBLK % NLW == 0 && WBLK % NLW == 0)) && (NSUB >= 4 || NG == 1), "tile shape");
    static_assert(!DEALT || ((EPI == 0 || EPI == 2) && (NG == 1 || NG == 2) &&
                             (NL == 0 ? NBLK - (LBW - 1) * NLW == NLW / 2 : (NBLK % NLW == 0 && WBLK % NLW == 0))),
                  "dealt pairs: QKV or gated epilogue");
    static_assert((SLOTS - 1) * LBW < 64 && SLOTS >= 2 && SLOTS <= 4, "vmcnt range");
    static_assert(EPI == 0 || NG == 1 || DEALT, "the plain linear layers use one slab per workgroup");
    extern __shared__ __align__(1024) unsigned char smem[];

    // Workgroup -> (unit, row tile).  Workgroup ids that are equal modulo 8 land on the same XCD; the
    // tiles, ordered unit by unit, are dealt to the eight XCDs in equal contiguous runs, so the
    // workgroups that stream the same weight rows share an L2 and every XCD gets the same number of
    // tiles (dealing whole units instead left 35 tiles on four XCDs and 28 on the others for 36 head
    // slots x 7 row tiles: two rounds of 32 compute units instead of one, 100 us instead of 62).
    const int id = blockIdx.x;
    const int xcd = id & 7, qd = id >> 3;
    // (EPI 3: the parts of the hidden dimension count as tiles too, so that they are dealt evenly as well)
    const int n_kp = EPI == 3 ? p.ksplit : 1;
    const int64_t n_tiles = (int64_t)p.n_units * p.n_mt * n_kp;
    const int tile_k = (int)(xcd * n_tiles / 8) + qd;
    if (tile_k >= (int)((xcd + 1) * n_tiles / 8)) return;
    const int tile = tile_k / n_kp, kpart = tile_k - tile * n_kp;
    const int unit = tile / p.n_mt, mt = tile - unit * p.n_mt;
    const int m0 = p.m_base + mt * XROWS;
    const int n_slots = p.n_slots;             // EPI 0: Hq query heads, Hkv key heads, Hkv value heads

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, hi = lane >> 5;
    const bool is_loader = NL > 0 && wave >= NW;  // wave-uniform
    const int lw = NL > 0 ? wave - NW : wave;     // index among the loading waves
    const int wn = (wave % NW) / WM, wm = wave % WM;  // this wave's head group and row group
    const int hs = p.slot_base + (NSUB >= 4 ? unit * NG + wn : unit >> 1);  // (DEALT: not used)
    const int half = NSUB >= 4 ? 0 : unit & 1;  // which rotary-paired half of the head
    const bool head_valid = DEALT || hs < n_slots;  // an odd number of heads leaves the last pair half empty
    const int n_pairs = n_slots * 64;           // DEALT: pairs of the whole problem
    const int my_blocks = DEALT && NL == 0 && lw >= NLW / 2 ? LBW - 1 : LBW;  // wave-uniform
    const int t0 = DEALT && NG == 2 && wn ? NT : 0;              // DEALT: first sub-tile of this wave
    const int nt_mine = DEALT && NG == 2 && wn ? NSUB - NT : NT;  // and how many it owns (wave-uniform)

    // ---- loader: per-lane source offsets (bytes from W / X, hidden offset 0) of this wave's blocks
    uint32_t goff[LBW];
#pragma unroll
    for (int i = 0; i < LBW; ++i) {
        const int bid = lw + NLW * i;               // block of the stage: weight blocks first (junk for lw < 0)
        const bool is_w = DEALT ? bid < WBLK : i < WBW;
        const int rl = RPB * (is_w ? bid : bid - WBLK) + lane / CPR;  // row of the W / X tile
        // logical 16-byte chunk that lands at position lane % CPR of the row piece: 128-byte pieces are
        // swizzled with bits 1..3 of the row, 256-byte pieces with bits 0..3
        const int c = (lane % CPR) ^ (KS == 64 ? (rl >> 1) & 7 : rl & 15);
        if (is_w) {
            int n;
            if (DEALT) {
                const int pr = min(PPU * unit + 16 * (rl >> 5) + (rl & 15), n_pairs - 1);  // pairs past the end are never stored
                if (EPI == 2) n = pr;  // row pr of the gate matrix (low) or of the up matrix (high)
                else n = (pr >> 6) * 128 + (pr & 63) + ((rl & 16) ? 64 : 0);
            } else if (EPI == 2) {  // row of the gate or of the up matrix (which of the two: see issue_stage)
                const int u = min(hs, n_slots - 1);  // NG = 1 here: hs is the slab of the whole workgroup
                n = u * 64 + (NSUB == 4 ? rl & 63 : 32 * half + (rl & 31));
            } else if (NSUB == 4) {
                n = min(p.slot_base + unit * NG + rl / 128, n_slots - 1) * 128 + (rl & 127);
            } else {
                n = min(hs, n_slots - 1) * 128 + (rl >> 5) * 64 + 32 * half + (rl & 31);
            }
            goff[i] = (uint32_t)n * (uint32_t)(p.K * 2) + c * 16;
        } else {
            const int m = min(m0 + rl, p.m_end - 1);  // rows past the end re-read the last row; never stored
            goff[i] = (uint32_t)m * (uint32_t)(p.K * 2) + c * 16;
        }
    }
    // The loads of a stage are issued in four parts spread over the multiplies of the stage before,
    // because a wave that issues many of them back to back waits for the memory pipeline to take
    // them before it can issue anything else.  part < 0: all of them.
    // part of the hidden dimension this workgroup covers (EPI 3 only: part kpart of p.ksplit)
    const int all_stages = p.K / KS;
    const int st0 = EPI == 3 ? (int)((int64_t)kpart * all_stages / p.ksplit) : 0;
    const int n_stages = EPI == 3 ? (int)(((int64_t)kpart + 1) * all_stages / p.ksplit) - st0 : all_stages;
    // Rows of W that lie a multiple of 4 KB apart: workgroup `unit` starts unit / n_units of the way along the hidden
    // dimension and goes round.  In step, all workgroups ask for the same 128 bytes of all those rows, and these share a few
    // memory channels.  One row tile of up to 128 rows, us without and with: gated 4096 x 12288, 64 / 128 rows 47.1 and
    // 35.8 / 49.0 and 41.3; 4096 x 14336 53.2 and 41.7 / 55.9 and 47.9; 2048 x 16384, 48 rows 34.0 and 26.0; 6144 x 16384 90 and 70;
    // 8192 x 8192 60 and 45; vocabulary 4096 x 32000, 64 rows 64.6 and 49.6; projection, 96 slots, hidden 4096, 64 rows 27.3
    // and 24.9.  At other distances it gives nothing or costs (hidden 5120 34.6 and 35.6, 7168 44.1 and 45.7, 1024 15.0 and
    // 15.3), and so it does with more row tiles, whose window rows then come from L2 at two places at a time (256 rows of
    // gated 4096 x 12288 66.9 and 70.3), and with the last rows of a problem, behind the launch that has just read the
    // weights (300 rows of the same 102.8 and 107.0).
    // More than one round of workgroups: by the place among the 256 that run together, 32 on each XCD.  (By unit / n_units
    // those together cover a fifth of the hidden dimension at 1188 units.)  Vocabularies at hidden 4096, us without, by the
    // unit, by the place: 64 rows, 33024 entries (258 units) 86.2, 72.8, 72.6; 50304 86.6, 82.1, 81.9; 65536 110.5, 92.5, 92.4; 98304 144.1,
    // 140.8, 138.7; 152064 219.5, 217.2, 216.2; 196608 278.0, 270.0, 269.5; 96 rows, 65536 125.6, 100.7, 95.9; 106496 194.6, 177.9, 177.8.
    // From four rounds on the workgroups drift apart by themselves and it is a few per cent either way: 96 rows,
    // 128256 189.6, 196.3, 193.5 (the largest loss; 131072 192.3, 196.1, 197.4), 152064 234.0, 232.8, 231.4, 163840 255.4, 254.2, 249.9;
    // 64 rows at hidden 2048, 131072 114.9, 96.1, 95.2; 96 rows at hidden 8192, 131072 377.0, 376.2, 380.2, 147456 445.4, 450.8, 456.0.
    const int per_round = min(p.n_units, 256);
    const int rot = ROTATE ? (int)(((uint32_t)(xcd * per_round / 8 + (qd & 31)) * p.rot_step) >> 16) : 0;
    auto issue_stage = [&](int st, int part) {
        const int sr = st + rot, at = st0 + (ROTATE && sr >= n_stages ? sr - n_stages : sr);
        unsigned char *dst = smem + (st % SLOTS) * STAGE;
#pragma unroll
        for (int i = 0; i < LBW; ++i) {
            if (part >= 0 && (i & 3) != part) continue;
            if (DEALT && i >= my_blocks) continue;
            static_assert(!ONCE || NL > 0, "weight blocks known at compile time");
            const uint16_t *mat = p.X;
            if (DEALT) {
                // rows 16..31 of a sub-tile are the high rows: EPI 2 takes them from the up matrix
                const int bid = lw + NLW * i;
                if (bid < WBLK) mat = (EPI == 2 && ((RPB * bid) & 16)) ? p.W2 : p.W;
            } else if (i < WBW) {
                // EPI 2: the second half of the tile rows (a whole number of 1 KB blocks) is the up matrix
                const bool up = EPI == 2 && RPB * (lw + NLW * i) >= (NSUB == 4 ? 64 : 32);
                mat = up ? p.W2 : p.W;
            }
            const unsigned char *src = (const unsigned char *)mat + (size_t)at * ROWB;
            if (ONCE && i < WBW) fc_load_lds16<true>(src + goff[i], dst + (lw + NLW * i) * 1024);
            else fc_load_lds16(src + goff[i], dst + (lw + NLW * i) * 1024);
        }
    };

    // bias, behind the ring
    constexpr int NPW = DEALT ? PPU : NSUB == 4 ? 64 * NG : 32;  // pairs per workgroup
    unsigned char *bias_area = smem + SLOTS * STAGE;
    if (EPI == 0 && lw == 0)
        load_bias(p, bias_area, DEALT ? PPU * unit : NSUB == 4 ? (p.slot_base + unit * NG) * 64 : hs * 64 + 32 * half, NPW, n_pairs, lane);

    // ---- operand read offsets inside a stage (bytes): row `col` of a 32-row sub-tile, k-step kk
    uint32_t foff[NKK];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk)
        foff[kk] = (uint32_t)(col * ROWB + (((2 * kk + hi) ^ (KS == 64 ? (col >> 1) & 7 : col & 15)) << 4));
    const uint32_t w_base = (uint32_t)((DEALT ? t0 : wn * NSUB) * 32 * ROWB);
    const uint32_t x_base = (uint32_t)(WBYTES + wm * MW * 32 * ROWB);

    f32x16 acc[MW][NT];
#pragma unroll
    for (int i = 0; i < MW; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][t][r] = 0.f;

    // Fragments are double-buffered in registers: the LDS reads of k-step kk+1 are issued before the
    // multiplies of k-step kk, and the first reads of the next stage go out (behind that stage's
    // barrier) before the last multiplies of this one, so the matrix core never waits for LDS.
    bf16x8 xf[2][MW], wf[2][NT];
    auto read_frags = [&](int slot, int kk, int buf) {
        const unsigned char *st = smem + slot * STAGE;
#pragma unroll
        for (int i = 0; i < MW; ++i) xf[buf][i] = *(const bf16x8 *)(st + x_base + i * (32 * ROWB) + foff[kk]);
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (t < nt_mine) wf[buf][t] = *(const bf16x8 *)(st + w_base + t * (32 * ROWB) + foff[kk]);
    };
    auto multiply = [&](int buf) {
#pragma unroll
        for (int i = 0; i < MW; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if (t < nt_mine)
                    acc[i][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[buf][t], xf[buf][i], acc[i][t], 0, 0, 0);
    };

    const int n_pro = min(SLOTS, n_stages);
    if (NL > 0) {
        // ---- loading waves: one barrier per stage, shared with the multiplying waves.  Barrier `it`
        // (it = 0 .. n_stages - 2) means: stage it+1 is complete and every multiplying wave has left
        // stage it, whose slot takes stage it + SLOTS.
        if (is_loader) {
            for (int st = 0; st < n_pro; ++st) issue_stage(st, -1);
            wait_stages<LBW, false>(n_pro - 1);
            __builtin_amdgcn_s_barrier();  // stage 0 is complete
            for (int it = 0; it + 1 < n_stages; ++it) {
                // stages requested so far: min(n_stages, it + SLOTS); those after it+1 may stay in flight
                wait_stages<LBW, false>(min(n_stages, it + SLOTS) - (it + 2));
                __builtin_amdgcn_s_barrier();
                if (it + SLOTS < n_stages) issue_stage(it + SLOTS, -1);
            }
            return;
        }
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
            multiply(1);
            __builtin_amdgcn_sched_barrier(0);
            slot = nslot;
        }
    } else {
    for (int st = 0; st < n_pro; ++st) issue_stage(st, -1);
    if (my_blocks == LBW) wait_stages<LBW, false>(n_pro - 1);
    else wait_stages<LBW - 1, false>(n_pro - 1);
    __builtin_amdgcn_s_barrier();  // stage 0 is complete for every wave
    read_frags(0, 0, 0);
    int slot = 0;
    for (int it = 0; it < n_stages; ++it) {
        // The slot of stage it-1 was released by the barrier in the middle of the previous iteration;
        // stage it-1+SLOTS goes there: its first quarter was issued behind that barrier, the rest now.
        const int refill = it - 1 + SLOTS;
        const bool do_refill = it > 0 && refill < n_stages;
#pragma unroll
        for (int kk = 0; kk < NKK - 1; ++kk) {
            read_frags(slot, kk + 1, (kk + 1) & 1);
            if (do_refill && kk < 3) issue_stage(refill, kk + 1);
            __builtin_amdgcn_sched_barrier(0);
            multiply(kk & 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        const int nslot = slot == SLOTS - 1 ? 0 : slot + 1;
        if (it + 1 < n_stages) {
            // This wave's reads of stage `it` have all returned (lgkmcnt 0); behind the barrier that
            // holds for every wave, and stage it+1 is complete (later stages may still be in flight).
            if (my_blocks == LBW) wait_stages<LBW, true>(min(n_stages, it + SLOTS) - (it + 2));
            else wait_stages<LBW - 1, true>(min(n_stages, it + SLOTS) - (it + 2));
            __builtin_amdgcn_s_barrier();
            if (it + SLOTS < n_stages) issue_stage(it + SLOTS, 0);
            read_frags(nslot, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        multiply(1);
        __builtin_amdgcn_sched_barrier(0);
        slot = nslot;
    }
    }

    // ---- epilogue; the LDS ring is its staging area, once every wave has left it
    if constexpr (EPI == 4) {
        if (head_valid) gemm_epilogue_vocab<MW>(p, acc, hs, m0 + 32 * wm * MW, lane);
    } else {
        static_assert(NW * epi_bytes(NT) <= SLOTS * STAGE, "epilogue staging");
        __builtin_amdgcn_s_barrier();
        if (!head_valid) return;
        const uint16_t *bias_low = (const uint16_t *)bias_area + (DEALT ? 16 * t0 : NSUB == 4 ? 64 * wn : 0);
        gemm_epilogue<NT, MW, EPI, DEALT>(p, acc, smem + wave * epi_bytes(NT), bias_low, bias_low + NPW, hs, half, PPU * unit + 16 * t0, nt_mine,
                                          m0 + 32 * wm * MW, lane, kpart);
    }
}

// -------------------------------------------------------------------------------------------------
// 256 window rows x two slabs (256 weight rows), for problems with enough such tiles to fill the chip.
//
// A workgroup has eight waves in two groups of four, one wave of each group per SIMD; group wn owns slab wn
// and its wave wm the window rows 64 wm .. 64 wm + 63 (MW = 2, NT = 4 sub-tiles of 32 x 32).  The loop over
// 64 hidden elements (a stage) alternates between reading operand fragments from LDS (and issuing loads)
// and multiplying, with a workgroup barrier behind each such interval, and group 1 runs one interval behind
// group 0: on every SIMD one wave multiplies while the other reads, so that LDS results never have to
// wait for the register ports of a running multiply and the matrix core always has a wave to run.  The loads
// of an interval are issued behind its reads: in front of them they held the reads back (1.74 us per stage at half
// the compute units, 1.32 behind).  2304 rows x 296 gated slabs, hidden 3584: 635 us in tiles of one slab, 560 in
// this one, 551 with the last round cut off (1135 TFLOP/s); with all compute units multiplying and no loads at
// all the same loop runs at 1380 TFLOP/s, which is what the clock allows under that load.
//
//   interval   M0            C0          M1         C1          M2            C2          M3               C3
//   reads      W sub 0,1                 X sub 1                W sub 2,3                 X sub 0 (next)
//   multiplies               X0 W01                 X1 W01                    X0 W23                       X1 W23
//
// LDS holds two stages of 64 KB in four parts (X0, W01, X1, W23: 128 rows x 128 B, swizzled like the other
// shapes).  A part is refilled, for the stage after the next, one or two intervals after its last reader:
// group 0 issues its half of W23, X0, W01, X1 in M0 .. M3, group 1 its half of X0, W01, X1, W23, so a
// load has eleven intervals (about 1.4 us) to arrive, and some 88 KB are always in flight.  Each wave
// waits for its own loads of the part that group 0 reads next at the end of every second interval; the count of
// younger loads is the same every time (five parts in group 0, six in group 1, two loads each).  Past the last
// stage the loads go on, from the last stage's addresses, into parts nobody reads: the counts stay exact.
template <int GRP, typename Issue, typename Read, typename Mul>
__device__ __forceinline__ void gemm_pp_loop(int n_stages, Issue issue, Read read, Mul mul)
{
    constexpr int AHEAD = 2 * (GRP == 0 ? 5 : 6);
    auto end_m = [&]() {  // end of a memory interval
        fc_wait_vm<GRP == 1 ? AHEAD : 63, true>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto compute = [&](int i, int tp) {
        mul(i, tp);
        __builtin_amdgcn_sched_barrier(0);
        if (GRP == 0) fc_wait_vm<AHEAD>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    // parts: 0 X0, 1 W01, 2 X1, 3 W23
#pragma unroll
    for (int part = 0; part < 4; ++part) issue(0, part);
#pragma unroll
    for (int part = 0; part < (GRP == 0 ? 3 : 4); ++part) issue(1, part);
    fc_wait_vm<AHEAD>();  // X0 and W01 of stage 0
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read(0, 0);
    if (GRP == 1) {
        fc_wait_lds();
        __builtin_amdgcn_s_barrier();  // one interval behind
        __builtin_amdgcn_sched_barrier(0);
    }
    for (int st = 0; st < n_stages; ++st) {
        // M0
        read(st, 1);
        issue(GRP == 0 ? st + 1 : st + 2, GRP == 0 ? 3 : 0);
        end_m();
        compute(0, 0);
        // M1
        read(st, 2);
        issue(st + 2, GRP == 0 ? 0 : 1);
        end_m();
        compute(1, 0);
        // M2
        read(st, 3);
        issue(st + 2, GRP == 0 ? 1 : 2);
        end_m();
        compute(0, 1);
        // M3
        read(st + 1, 0);  // (behind the last stage: not used)
        issue(st + 2, GRP == 0 ? 2 : 3);
        end_m();
        compute(1, 1);
    }
    if (GRP == 0) __builtin_amdgcn_s_barrier();
    fc_wait_vm<0>();  // no load may still arrive in LDS when the epilogue uses it
    __builtin_amdgcn_s_barrier();
}

constexpr int PP_LDS = 8 * epi_bytes(4) > 128 * 1024 ? 8 * epi_bytes(4) : 128 * 1024;  // the loop's two stages; the epilogue
template <int EPI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_pp(GemmArgs p)
{
    constexpr int PART = 128 * 128, STAGE = 4 * PART;
    extern __shared__ __align__(1024) unsigned char smem[];
    // workgroup -> (slab pair, row tile), dealt to the XCDs as in k_proj_gemm
    const int id = blockIdx.x;
    const int xcd = id & 7, qd = id >> 3;
    const int64_t n_tiles = (int64_t)p.n_units * p.n_mt;
    const int tile = (int)(xcd * n_tiles / 8) + qd;
    if (tile >= (int)((xcd + 1) * n_tiles / 8)) return;
    const int unit = tile / p.n_mt, mt = tile - unit * p.n_mt;
    const int m0 = p.m_base + mt * 256;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, hi = lane >> 5;
    const int wn = wave >> 2, wm = wave & 3;

    // ---- loads: two 1 KB blocks (8 rows x 128 B) of each part per wave
    uint32_t goff[4][2];
#pragma unroll
    for (int part = 0; part < 4; ++part)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = 8 * (2 * wave + i) + (lane >> 3);  // row of the part
            const int c = (lane & 7) ^ ((r >> 1) & 7);
            int row;
            if ((part & 1) == 0) {
                row = min(m0 + 64 * (r >> 5) + 16 * part + (r & 31), p.m_end - 1);  // rows past the end: never stored
            } else {
                const int slab = min(p.slot_base + 2 * unit + (r >> 6), p.n_slots - 1);
                row = EPI == 2 ? slab * 64 + (r & 63) : slab * 128 + (part == 3 ? 64 : 0) + (r & 63);
            }
            goff[part][i] = (uint32_t)row * (uint32_t)(p.K * 2) + c * 16;
        }
    const int n_stages = p.K / 64;
    auto issue = [&](int st, int part) {
        __builtin_amdgcn_sched_barrier(0);
        const uint16_t *mat = (part & 1) == 0 ? p.X : (EPI == 2 && part == 3) ? p.W2 : p.W;
        const unsigned char *src = (const unsigned char *)mat + (size_t)min(st, n_stages - 1) * 128;
        unsigned char *dst = smem + (st & 1) * STAGE + part * PART + wave * 2048;
#pragma unroll
        for (int i = 0; i < 2; ++i) fc_load_lds16(src + goff[part][i], dst + i * 1024);
    };

    // bias, behind everything else
    unsigned char *bias_area = smem + PP_LDS;
    if (EPI == 0 && wave == 0) load_bias(p, bias_area, (p.slot_base + 2 * unit) * 64, 128, p.n_slots * 64, lane);

    // ---- operand fragments
    uint32_t foff[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) foff[kk] = (uint32_t)(col * 128 + (((2 * kk + hi) ^ ((col >> 1) & 7)) << 4));
    bf16x8 xf[2][4], wf[2][4];
    auto read = [&](int st, int part) {
        const unsigned char *base = smem + (st & 1) * STAGE + part * PART;
        if ((part & 1) == 0) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) xf[part >> 1][kk] = *(const bf16x8 *)(base + wm * 4096 + foff[kk]);
        } else {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                for (int t = 0; t < 2; ++t) wf[t][kk] = *(const bf16x8 *)(base + wn * 8192 + t * 4096 + foff[kk]);
        }
    };
    f32x16 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][t][r] = 0.f;
    auto mul = [&](int i, int tp) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                acc[i][2 * tp + t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[t][kk], xf[i][kk], acc[i][2 * tp + t], 0, 0, 0);
    };
    if (wn == 0) gemm_pp_loop<0>(n_stages, issue, read, mul);
    else gemm_pp_loop<1>(n_stages, issue, read, mul);

    const int hs = p.slot_base + 2 * unit + wn;
    if (hs >= p.slot_base + p.slots_here) return;  // an odd number of slabs leaves the last pair half empty
    if constexpr (EPI == 4) gemm_epilogue_vocab<2>(p, acc, hs, m0 + 64 * wm, lane);
    else gemm_epilogue<4, 2, EPI, false>(p, acc, smem + wave * epi_bytes(4), (const uint16_t *)bias_area + 64 * wn,
                                         (const uint16_t *)bias_area + 128 + 64 * wn, hs, 0, 0, 4, m0 + 64 * wm, lane, 0);
}

template <int EPI>
hipError_t launch_gemm_pp(GemmArgs a, hipStream_t s)
{
    constexpr int LDS = PP_LDS + (EPI == 0 ? BIAS_LDS : 0);
    static hipError_t attr = hipFuncSetAttribute((const void *)k_gemm_pp<EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (attr != hipSuccess) return attr;
    a.n_units = (a.slots_here + 1) / 2;
    a.n_mt = (a.m_end - a.m_base + 255) / 256;
    if (a.slots_here < 1 || a.n_mt < 1 || a.slot_base < 0 || a.slot_base + a.slots_here > a.n_slots || a.m_base < 0 ||
        a.m_end > a.M || a.K % 64 != 0)
        return hipErrorInvalidValue;
    const int64_t n_tiles = (int64_t)a.n_units * a.n_mt;
    if (n_tiles > (1 << 30)) return hipErrorInvalidValue;
    k_gemm_pp<EPI><<<dim3((unsigned)((n_tiles + 7) / 8 * 8)), dim3(512), LDS, s>>>(a);
    return hipGetLastError();
}

template <int KS, int NW, int NSUB, int MW, int NG, int SLOTS, int NL, int EPI = 0>
hipError_t launch_gemm(GemmArgs a, hipStream_t s)
{
    constexpr int XROWS = 32 * MW * (NW / NG);
    constexpr bool DEALT = NSUB == 5 || NSUB == 3;
    constexpr int LDS = SLOTS * ((DEALT ? 32 * NSUB : 32 * NSUB * NG) + XROWS) * KS * 2 + (EPI == 0 ? BIAS_LDS : 0);
    static_assert(LDS <= 160 * 1024, "LDS ring too large");
    const int slots = a.slots_here;
    a.n_units = DEALT ? (a.n_slots * 64 + 16 * NSUB - 1) / (16 * NSUB) : NSUB == 4 ? (slots + NG - 1) / NG : 2 * slots;
    if (DEALT && (a.slot_base != 0 || slots != a.n_slots)) return hipErrorInvalidValue;  // dealt pairs cover every slab
    a.n_mt = (a.m_end - a.m_base + XROWS - 1) / XROWS;
    if (slots < 1 || a.n_mt < 1 || a.slot_base < 0 || a.slot_base + slots > a.n_slots || a.m_base < 0 || a.m_end > a.M)
        return hipErrorInvalidValue;
    const int64_t n_tiles = (int64_t)a.n_units * a.n_mt * (EPI == 3 ? a.ksplit : 1);
    if (n_tiles > (1 << 30) || (EPI == 3 && a.ksplit < 1)) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)((n_tiles + 7) / 8 * 8);
    auto start = [&](auto rotate, auto once) {
        constexpr auto kernel = k_proj_gemm<KS, NW, NSUB, MW, NG, SLOTS, NL, EPI, decltype(rotate)::value, decltype(once)::value>;
        static hipError_t attr = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (attr != hipSuccess) return attr;
        kernel<<<dim3(grid), dim3((NW + NL) * 64), LDS, s>>>(a);
        return hipGetLastError();
    };
    // One tile of rows: its workgroups are the only ones to read their weights.
    auto with_hint = [&](auto rotate) {
        if constexpr (XROWS <= 128)
            if (a.once && a.M <= XROWS) return start(rotate, std::true_type());
        return start(rotate, std::false_type());
    };
    if constexpr (XROWS <= 128 && EPI != 3)
        if (a.n_mt == 1 && a.m_base == 0 && a.K % 2048 == 0 && a.K / KS < 65536) {
            a.rot_step = (uint32_t)(((int64_t)(a.K / KS) << 16) / (a.n_units < 256 ? a.n_units : 256));  // (place * rot_step stays below 2^32)
            return with_hint(std::true_type());
        }
    return with_hint(std::false_type());
}

// Sum of the hidden-dimension parts of an EPI 3 launch + residual, four outputs per thread.
__global__ __launch_bounds__(256) void k_splitk_finish(const float *__restrict__ part, const uint16_t *res,
                                                       uint16_t *out, size_t quads, size_t plane, int ksplit)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= quads) return;
    float4 a = *(const float4 *)(part + 4 * i);
    for (int k = 1; k < ksplit; ++k) {
        const float4 b = *(const float4 *)(part + (size_t)k * plane + 4 * i);
        a.x += b.x;
        a.y += b.y;
        a.z += b.z;
        a.w += b.w;
    }
    if (res) {
        const uint2 rv = *(const uint2 *)(res + 4 * i);
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

// A launch in one tile shape (numbered below).  Loads of the 128-row shapes are issued by four extra waves: their four
// multiplying waves are alone on their SIMDs.  The half-head shape of the projection takes 128 hidden elements per
// stage where it can.
template <int EPI>
hipError_t launch_shape(int shape, const GemmArgs &a, hipStream_t s)
{
    switch (shape) {
    case 0: return launch_gemm<64, 8, 4, 1, 1, 3, 0, EPI>(a, s);
    case 1: return launch_gemm<64, 4, 4, 1, 1, 4, 4, EPI>(a, s);
    case 2:
        if constexpr (EPI == 0)
            if (a.K % 128 == 0) return launch_gemm<128, 4, 2, 1, 1, 3, 4, EPI>(a, s);
        if constexpr (EPI != 4) return launch_gemm<64, 4, 2, 1, 1, 4, 4, EPI>(a, s);
        return hipErrorInvalidValue;
    case 3:
        if constexpr (EPI == 3) return hipErrorInvalidValue;
        else return launch_gemm_pp<EPI>(a, s);
    case 4:
        if constexpr (EPI == 0 || EPI == 2) return launch_gemm<64, 8, 5, 2, 2, 3, 0, EPI>(a, s);
        return hipErrorInvalidValue;
    case 5:
        if constexpr (EPI == 0 || EPI == 2) return launch_gemm<64, 4, 3, 1, 1, 4, 4, EPI>(a, s);
        return hipErrorInvalidValue;
    case 6:
        if constexpr (EPI == 0 || EPI == 2) return launch_gemm<64, 2, 5, 1, 1, 4, 4, EPI>(a, s);
        return hipErrorInvalidValue;
    case 7:
        if constexpr (EPI == 0 || EPI == 2) return launch_gemm<64, 2, 3, 1, 1, 4, 4, EPI>(a, s);
        return hipErrorInvalidValue;
    case 8:
        if constexpr (EPI == 0 || EPI == 2) return launch_gemm<64, 4, 5, 1, 1, 4, 4, EPI>(a, s);
        return hipErrorInvalidValue;
    case 9: return launch_gemm<64, 2, 4, 1, 1, 3, 2, EPI>(a, s);
    case 10:
        if constexpr (EPI == 4) return hipErrorInvalidValue;
        else return launch_gemm<64, 2, 2, 1, 1, 4, 4, EPI>(a, s);
    default: return hipErrorInvalidValue;
    }
}

// Tile shapes of the tiled GEMM and what a full round of 256 workgroups takes per 64 hidden elements (us, measured at
// hidden 3584 and 4096 with 150..768 workgroups).  Per tile area the larger ones are cheaper -- they move fewer
// bytes into the compute unit per product -- but leave the chip emptier at the end.
//   0: 256 rows x slab   1: 128 rows x slab   2: 128 rows x half slab   3: 256 rows x two slabs
//   4: 256 rows x 80 dealt pairs   5: 128 rows x 48 dealt pairs
//   6: 64 rows x 80 dealt pairs   7: 64 rows x 48 dealt pairs   8: 128 rows x 80 dealt pairs
//   9: 64 rows x slab   10: 64 rows x half slab
// 6 .. 10 are for few rows, where the weights alone should count: in the 128-row half slab, for 40 or 64 rows the shape with
// the most tiles, the compute units pulled three bytes for every byte of weights (two thirds of them window rows, most
// of those padding); 64 rows x 160 weight rows pull 1.4.  Gated W_1 of 18944 outputs at hidden 3584, 64 / 128 rows:
// 67.5 / 81.6 us, now 50.4 / 58.3 (the weights alone 46 at 5.9 TB/s).
constexpr int N_SHAPES = 11;
constexpr double ROUND_US[N_SHAPES] = {1.03, 0.62, 0.39, 1.84, 1.30, 0.54, 0.75, 0.53, 0.95, 0.52, 0.34};
// The same for up to one round of one row tile of the 64-row shapes (6, 7, 9, 10), where a workgroup's own pull counts and not how many there are:
// line 0.85 + 0.15 x (gated hidden 3584, 32 rows, us per stage: shape 7 with 134 / 198 tiles 0.40 / 0.435, shape 9 with 100 / 148
// 0.50 / 0.53, shape 6 with 80 / 119 0.54 / 0.57, shape 10 with 72 / 200 0.30 / 0.32).
constexpr double SINGLE_US[N_SHAPES] = {0, 0, 0, 0, 0, 0, 0.60, 0.45, 0, 0.55, 0.33};
constexpr bool shape_dealt(int shape) { return shape >= 4 && shape <= 8; }
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
    default: return 2 * slots * t64;
    }
}

// Estimated time of one launch per 64 hidden elements.  A round that fills half the chip was measured at 0.78 to
// 0.9 of a full one (the clock is higher and the memory path less loaded), hence the line 0.6 + 0.4 x.  The weights
// come from HBM at 5.8 TB/s at best.
double launch_cost(int shape, int64_t slots, int64_t rows)
{
    const int64_t n = tiles_of(shape, slots, rows), part = n % 256;
    const double tiles = SINGLE_US[shape] > 0 && rows <= 64 && n <= 256 ? SINGLE_US[shape] * (0.85 + 0.15 * n / 256.0)
                                                          : ROUND_US[shape] * ((double)(n / 256) + (part ? 0.6 + 0.4 * part / 256.0 : 0.0));
    const double weights = (double)slots * 128 * 128 / 5.8e6;
    return (tiles > weights ? tiles : weights) + 0.02 * tiles;  // (equally bound by the weights: the smaller tiles)
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
    double best = 1e30;
    int n = 1;
    for (int sh = 0; sh < N_SHAPES; ++sh) {
        if ((shape_half(sh) && !allow_half) || (shape_dealt(sh) && !allow_dealt)) continue;
        const double c = launch_cost(sh, slots, M);
        if (c < best) {
            best = c;
            out[0] = GemmPiece{sh, 0, slots, 0, M};
        }
    }
    if (no_split) return 1;
    const double extra = 3.0 / (K / 64);
    for (int sh = 0; sh <= 3; sh += 3) {
        const int64_t per = sh == 3 ? 2 : 1, t256 = (M + 255) / 256, units = (slots + per - 1) / per;
        for (int64_t rounds = units * t256 / 256; rounds >= 1 && rounds >= units * t256 / 256 - 1; --rounds) {
            const int64_t u1 = rounds * 256 / t256, s1 = u1 * per;          // slabs of the first launch
            const int64_t r1 = rounds * 256 / units, m1 = r1 * 256;         // or its row tiles
            for (int s2 = 0; s2 <= 3; ++s2) {
                if (s2 == 2 && !allow_half) continue;
                if (u1 >= 1 && s1 < slots) {
                    const double c = launch_cost(sh, s1, M) + launch_cost(s2, slots - s1, M) + extra;
                    if (c < best) {
                        best = c;
                        n = 2;
                        out[0] = GemmPiece{sh, 0, (int)s1, 0, M};
                        out[1] = GemmPiece{s2, (int)s1, (int)(slots - s1), 0, M};
                    }
                }
                if (r1 >= 1 && m1 < M) {
                    const double c = launch_cost(sh, slots, m1) + launch_cost(s2, slots, M - m1) + extra;
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
// kernel (6.3 TB/s instead of 6) where its tiles fill one round of workgroups (vocabulary: or two), and more slowly otherwise.  Both sides measured, weights from HBM (us at 16 / 32 rows, tiled GEMM first):
//   gated, hidden 3584: 6400 outputs (200 half slabs) 20.3 and 21.7 / 20.8 and 23.5, 8192 (256) 22.1 and 24.0 / 22.8 and 25.4,
//   9472 (198 tiles of 48 dealt pairs) 26.3 and 29.1 / 27.4 and 31.0, 12288 (256) 32.3 and 33.2 / 32.7 and 34.7, 13312 (208 slabs)
//   35.5 and 36.5 / 36.5 and 38.1, 16384 (256) 41.2 and 42.5 / 41.8 and 44.2, 18944 (237 tiles of 80 dealt pairs) 47.5 and 49.7 /
//   48.5 and 51.3, 22016 63.4 and 59.8 / 66.0 and 62.0;
//   gated, hidden 4096: 6400 23.2 and 24.1 / 23.8 and 26.2, 8192 24.2 and 33.6 / 24.3 and 33.8, 11008 (230 tiles of 48) 32.1 and 36.5 /
//   32.4 and 38.5, 12288 35.5 and 37.9 / 35.8 and 40.2, 14336 41.0 and 42.7 / 41.7 and 45.4, 16384 47.3 and 46.1 / 47.6 and 49.1, 18944
//   52.8 and 56.0 / 53.7 and 58.7, 22016 71.3 and 68.7 / 73.7 and 70.7;
//   vocabulary, hidden 3584: 16000 35.0 and 30.1 / 35.3 and 31.6, 32000 (250 slabs) 44.7 and 48.2 / 45.0 and 50.3, 50304 70.5 and
//   69.3 / 72.6 and 71.2, 65536 (512) 84.0 and 85.2 / 84.0 and 86.4, 152064 188.1 and 184.6 / 189.2 and 186.9; hidden 4096: 16000 38.5
//   and 34.1 / 39.1 and 36.5, 32000 49.0 and 56.8 / 48.7 and 59.9, 65536 92.2 and 93.2 / 92.4 and 94.3, 152064 215 and 203 / 216 and 210
//   (two rounds there gain 2 % and would ask for a larger workspace than the whole-row kernel: left to it).
bool wide_beats_rows(int mode, int M, int K, int64_t slabs)
{
    auto in = [](int64_t n, int64_t lo) { return n >= lo && n <= 256; };
    if (mode == FC_LIN_VOCAB) return in(slabs, 208) || (K % 4096 != 0 && in(slabs - 256, 208));
    const int64_t pairs48 = tiles_of(7, slabs, M);
    return in(tiles_of(10, slabs, M), 200) || in(tiles_of(9, slabs, M), 208) || in(pairs48, 192) ||
           (slabs > 256 && in(tiles_of(6, slabs, M), 208));
}

}  // namespace

// Tiled-GEMM plan of a plain linear layer (host, pure function of the shape); kind 0: not for this kernel.
FcWidePlan fc_plan_wide(int dtype, int mode, int M, int K, int N)
{
    FcWidePlan p;
    p.kind = 0;
    p.shape = 0;
    p.ksplit = 1;
    const int per_slab = mode == FC_LIN_GATE_UP ? 64 : 128;  // FC_LIN_VOCAB: slabs of 128 vocabulary rows
    if (dtype != FC_BF16 || M < 1 || K < 4 * KS_MIN || K % KS_MIN != 0 || N < per_slab || N % per_slab != 0) return p;
    // 32-bit byte offsets inside X and each weight matrix
    if ((int64_t)N * K * 2 >= ((int64_t)1 << 32) || (int64_t)M * K * 2 >= ((int64_t)1 << 32)) return p;
    // At most 32 rows: gated layers and vocabularies see above.  W_out and W_2 in parts against the slice-wise kernel, which has
    // a second launch too and pulls a window slice per 128 weight rows: a large matrix, more than 16 rows (us at 24 rows,
    // tiled GEMM first: 18944 x 3584 30.1 and 31.2, 16384 x 4096 37.0 and 43.1, 8192 x 8192 35.6 and 41.7, 24576 x 4096 41.0 and 42.0;
    // 16 rows of the first 29.7 and 29.6).  Below the line it is mixed: 16384 x 3584 30.7 and 27.4, 12288 x 4096 25.0 and 25.0,
    // 12288 x 3584 22.6 and 23.2, 10240 x 5120 24.2 and 26.3.
    if (M <= 32) {
        const FcSkinnyPlan rows = fc_plan_skinny(dtype, mode, M, K, N);
        const bool knob = fc_knobs().lin_wide_shape >= 6;
        if (!knob && (fc_knobs().lin_wgs > 0 || fc_knobs().lin_no_rows)) return p;  // tuning knobs of the streaming kernels
        if (!knob && !(mode == FC_LIN_RESIDUAL ? rows.kind == 1 && M > 16 && (double)K * N >= 60e6
                                               : rows.kind == 2 && K >= 2048 && wide_beats_rows(mode, M, K, N / per_slab)))
            return p;
    }
    p.kind = 1;
    const int64_t units = N / per_slab, t256 = (M + 255) / 256, t128 = (M + 127) / 128;
    // (The shape counts only where the hidden dimension is cut into parts or a tuning knob asks for one shape;
    // everything else goes through plan_pieces at launch.)
    if (M <= 128 && units >= 192) p.shape = mode == FC_LIN_VOCAB ? 1 : 2;
    else if (units * t256 >= 192) p.shape = 0;
    else if (units * t128 >= 144 || mode == FC_LIN_VOCAB) p.shape = 1;
    else p.shape = 2;
    // Too few slabs even for the smallest tile: also cut the hidden dimension (partial sums in fp32).
    // Tile and number of parts are chosen together by a two-term estimate that reproduces the measured
    // order (256 rows, 28 slabs, hidden 18944: 53 us for the 256-row tile in 8 parts, 58 for the 128-row
    // tile in 4, 68 for the half slab in 2; hidden 3584: 24, 20, 18): a workgroup pulls the rows of
    // both its operands at about 50 GB/s, and the partial sums are written and read at about 3 TB/s.
    const int64_t wgs = 2 * units * t128;
    if (mode == FC_LIN_RESIDUAL && p.shape == 2 && wgs < 192) {
        const int64_t stages = K / KS_MIN;
        double best = 1e30;
        for (const int sh : {0, 1, 2, 9, 10}) {
            const int64_t rows = sh == 0 ? 256 : sh < 3 ? 128 : 64, wrows = shape_half(sh) ? 64 : 128;
            if (rows == 64 && M > 64) continue;  // (256 rows in four such tiles, uncut: 25.0 us for W_out, 19.8 as chosen here)
            const int64_t tiles = tiles_of(sh, units, M);
            for (int64_t ks = 1; ks <= 16; ++ks) {
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
    {  // tuning knobs
        const int v = fc_knobs().lin_wide_shape;
        if (v >= 0 && v < N_SHAPES && (!shape_half(v) || mode != FC_LIN_VOCAB) && (!shape_dealt(v) || mode == FC_LIN_GATE_UP)) p.shape = v;
        const int ks = fc_knobs().lin_ksplit;
        if (ks >= 1 && ks <= 16 && ks <= K / KS_MIN / 4 && mode == FC_LIN_RESIDUAL) p.ksplit = ks;
        if (p.shape == 3) p.ksplit = 1;  // (forced: 256 rows x two slabs come in one piece only)
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
    const size_t quads = (size_t)M * N / 4;
    k_splitk_finish<<<dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s>>>((const float *)workspace, a.res, a.out,
                                                                                  quads, (size_t)M * N, pl.ksplit);
    return hipGetLastError();
}

bool fc_project_gemm_supported(const fc_config &cfg, int M)
{
    // 32-bit byte offsets inside X and W; the hidden dimension in whole stages
    const int64_t n = (int64_t)(cfg.n_q_heads + 2 * cfg.n_kv_heads) * cfg.head_dim;
    return cfg.dtype == FC_BF16 && cfg.head_dim == 128 && cfg.hidden % KS_MIN == 0 && M >= 1 &&
           n * cfg.hidden * 2 < ((int64_t)1 << 32) && (int64_t)M * cfg.hidden * 2 < ((int64_t)1 << 32);
}

// Estimated time of the tiled projection of M <= 128 rows (us; within a tenth of the measured times at hidden 1024 ..
// 8192, 12 .. 96 head slots, 4 .. 128 rows).
double fc_project_gemm_us(int slots, int M, int K)
{
    GemmPiece pc[2];
    double c = 4.0 + M / 64.0;
    const int n = plan_pieces(slots, M, K, true, true, pc);
    for (int i = 0; i < n; ++i) c += launch_cost(pc[i].shape, pc[i].slots, pc[i].m_end - pc[i].m_base) * (K / 64);
    return n == 2 ? c + 3.0 : c;
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
