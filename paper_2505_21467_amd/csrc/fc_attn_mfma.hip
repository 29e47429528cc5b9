// Active-query attention on the matrix cores (bf16, head_dim 128).
//
// For one (sequence, kv head) the g*A query rows (head-in-group major, then window row) are cut into 16-row tiles.  Two kernels:
//
// k_attn_ranges  a workgroup owns a number of row tiles and one contiguous range of keys; with several ranges each writes
//                unnormalised partial outputs with their reference maximum and sum, which k_attn_combine merges.
// k_attn_groups  a workgroup owns one or two row tiles and all keys; its waves take the keys in turn.
//
// Both compute S^T = K Q^T with v_mfma_f32_16x16x32_bf16 (K rows are the A operand: a lane (rho, q) = (lane & 15, lane >> 4) holds
// scores of ONE query row rho) and feed the probabilities, converted to bf16 in place, back as the B operand of
// O^T += V^T P^T.  Within a block of 32 keys the K rows are read in the order in which a lane ends up with keys 8 q .. 8 q + 7,
// the operand layout of P^T for natural-order V^T rows: no shuffles and no LDS round trip for P.
//
// K rows and transposed V tiles stream HBM -> LDS with 16-byte direct-to-LDS loads (no registers in between).  The LDS image is
// XOR-swizzled at 16-byte granularity (the swizzle is applied to the global address of each lane, since direct loads land
// in lane order) so that the 16 lanes the LDS serves per clock hit 16 different 16-byte bank groups: K rows (256 B) by the low
// four bits of the row, V^T rows (128 B, two per 256 B of banks) by bits 1..3 of the row.
#include <stdlib.h>

#include "fc_device.h"
#include "fc_internal.h"

namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int DH = 128;
constexpr int KT = 64;                 // keys per stage (= one transposed V tile)
constexpr int K_BYTES = KT * DH * 2;   // 16384
constexpr int OROW = 132;              // floats per row of the output staging area (128 + 4 padding)

// k_attn_groups: LDS of a wave, a group of keys and a stage of values, or its state of 16 QT rows at the end
__host__ __device__ constexpr int groups_wave_bytes(int QT, int VP)
{
    const int ring = 8192 + 16384 / VP, state = QT * (8192 / VP + 128);
    return ring > state ? ring : state;
}

struct AttnArgs {
    const uint16_t *Q;    // [B][Hq][A][128]
    const uint16_t *Kc;   // one layer, [B][Hkv][spad][128]
    const uint16_t *Vc;   // one layer, [B][Hkv][spad/64][128][64]
    const int32_t *pos;   // [B][A] or nullptr
    uint16_t *out;        // [B][A][Hq*128]
    float *part_o;        // [B*Hkv*row_tiles][splits][8 slots][64 lanes][8 halves]: accumulators as the lanes hold them
    float *part_ml;       // [B*Hkv*row_tiles][splits][32 rows][4]  (max in the log2 domain, sum, scaling exponent, -)
    int B, Hq, Hkv, g, A, kv_len, spad, max_seq;
    int row_tiles, n_rg, splits, keys_per_split, n_units;
    float c;              // softmax scale * log2(e)
    uint32_t div_pair, div_hkv, div_a;  // k_attn_groups: reciprocals (its launch bounds what they divide)
    bool once;            // k_attn_ranges: keys and values with the non-temporal hint
    // k_attn_ranges and k_attn_combine, any size; five divisions ahead of the first load took 0.3 us of a call.  (In k_attn_groups, which
    // has its quotients for a multiply each, these cost 0.2 us more: three arguments and four instructions more apiece.)
    FcDivisor by_rg, by_splits, by_tiles, by_hkv, by_a;
};

// Lanes l and l^32 hold the two halves of a query row.  v_permlane32_swap exchanges the upper 32
// lanes of its first operand with the lower 32 lanes of its second; fed the same value twice it
// returns (lower half in all lanes, upper half in all lanes), so one instruction pairs the halves.
__device__ __forceinline__ float row_max2(float v)
{
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float row_sum2(float v)
{
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The same over lanes l and l ^ 16.
__device__ __forceinline__ float row_max16(float v)
{
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float row_sum16(float v)
{
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ bool row_is_padded(const int32_t *pos, int idx, int max_seq)
{
    if (!pos) return false;
    const int p = pos[idx];
    return p < 0 || p >= max_seq;
}

// -------------------------------------------------------------------------------------------------
// 16 QT NW query rows per workgroup over one range of keys: NW waves, each with QT tiles of 16 rows and all keys of the range.
//
// One wave per SIMD (NW = 4) has to hide its own latencies, so the arithmetic is one stream in which every multiply has other work beside
// it: while the weights (exponentials) of a tile and block of 32 keys are computed, the matrix core forms the scores of the
// next block and the output products of the tile before, and the fragments of the keys and values are replaced one by one
// behind the last multiply that reads them.  Weights are exp2(c (s - m)) with m the row's maximum over the first stage of the range; where a
// lane's eight weights of a block sum to more than MOST (one comparison per tile and block), the references of the tile's rows move to
// the block's maxima before the weights are used.  So weights stay below 2^8, and the largest ones of a row are near a power of
// two, where rounding to bf16 takes little or nothing.  MOST is what keeps the error against 64 bits at or below that of the kernel named below, scores
// of deviation 1 .. 4, 23 shapes (1 / 1.2 / 2 / 4: 8 x 256 rows, 2304 keys 2.340 / 2.334 / 2.277 / 2.084e-3 against 2.342 / 2.338 / 2.290 / 2.132; 32 rows, 16800
// keys 2.312 / 2.300 / 2.014 / 1.756 against 2.316 / 2.304 / 2.157 / 1.785), with as few moves as that takes: a
// move is 80 VALU instructions (16 rows a wave) or 145, and its workgroup waits.  At 16 everywhere 8 x 256 rows take 3 / 8 / 8 / 9 us more at
// deviation 1.4 / 2 / 3 / 4; never moving saves them 0.4 / 0.8 / 5.6 / 9.4 and costs 2.33e-3 at every deviation.  The first stage of ranges of few
// rows counts to 16 bits of its weights, by a second product with what rounding took (0.35 us): few rows go in fewer ranges per row than in
// that kernel, whose every wave had a reference of its own and so the largest weight of its first block exact; without, 32 rows, 16800
// keys 2.333 / 2.316e-3 at 1 / 1.2.
// What bounds it: a multiply keeps the VALU of its SIMD for 8 of its 16 clocks, an exponential takes 8, other VALU instructions 4.4, an LDS
// read 6: 2690 clocks for 64 rows x 64 keys per wave against 2048 of multiplies.
// Against eight waves of 32x32x16 multiplies with a maximum per block (in phase, each stage the sum of both), us per call on one card at
// deviation 1.2, at 4 in brackets: 8 x 256 rows of 28 / 4 heads, 2304 keys 70.1 -> 63.6 (73.9 -> 75.0); 2304 rows 72.3 -> 64.0 (76.4 -> 74.6); 2 x 300
// rows, 1001 keys 22.8 -> 18.9 (24.5 -> 22.9); 2 x 256 rows of 32 / 32, 2000 keys 32.3 -> 26.8 (33.2 -> 28.9); 32 rows, 16800 keys 21.0 -> 20.0 (21.6
// -> 21.7); 8 x 32 rows, 2304 keys 22.2 -> 20.5 (23.0 -> 22.4); 4 x 64 rows of 32 / 32, 4160 keys 49.7 -> 46.7 (49.8 -> 46.8).  Slower: 3 x 527
// rows of 32 / 32, 1531 keys 56.8 -> 59.3.
// 16 rows a wave fit into the VALU's half of the registers, where a move is 32 multiplies and not 96 instructions (32 rows, 16800 keys, deviation 4
// 23.9 -> 21.7).  Others have the accumulators of the output and the queries in the other half, and the scores' multiplies are inline assembly to
// have those in the VALU's: the compiler puts every accumulator into the other half and moves 64 scores per stage and lane across (62.0 ->
// 63.4 us; for 16 rows 2 x 200 rows, 1500 keys 17.4 -> 18.6).  Its hazard rules do not see them, so: a score is read no sooner than three
// multiplies (48 clocks) behind its last one, or behind s_nops; a test holds the compiled code to it.
template <int QT, int NW, bool ONCE>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(QT == 1 ? 2 : NW / 4, QT == 1 ? 2 : NW / 4))) void k_attn_ranges(AttnArgs p)
{
    // Sum of a lane's eight weights from which the references of a tile's rows move
    constexpr float MOST = QT == 4 ? 128.0f : QT == 2 ? 64.0f : NW == 8 ? 24.0f : 16.0f;
    constexpr int LB = 16 / NW;  // 1 KB loads of a stage's keys, and of its values, per wave
    extern __shared__ __align__(1024) unsigned char smem[];
    unsigned char *const kring = smem, *const vring = smem + 4 * K_BYTES;  // four stages each

    const int id = blockIdx.x;
    const int xcd = id & 7, qd = id >> 3;
    const int64_t n_tiles = (int64_t)p.n_units * p.n_rg;
    const int tile = (int)(xcd * n_tiles / 8) + qd;
    if (tile >= (int)((xcd + 1) * n_tiles / 8)) return;
    const int unit = (int)p.by_rg.over(tile), rg = tile - unit * p.n_rg;
    const int bj = (int)p.by_splits.over(unit), split = unit - bj * p.splits;
    const int b = (int)p.by_hkv.over(bj), j = bj - b * p.Hkv;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho = lane & 15, q = lane >> 4;
    const int nrows = p.g * p.A;
    const int row0 = (rg * NW + wave) * (16 * QT);  // first query row of this wave
    auto head_of = [&](int row) { return (int)p.by_a.over(row); };

    // ---- query rows (past the end: the last row, never stored)
    bf16x8 qf[QT][4];
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        const int row = min(row0 + 16 * u + rho, nrows - 1);
        const int hg = head_of(row), a = row - hg * p.A;
        const uint16_t *qrow = p.Q + (((size_t)b * p.Hq + j * p.g + hg) * p.A + a) * DH + 8 * q;
#pragma unroll
        for (int k = 0; k < 4; ++k) qf[u][k] = fc_load_any<bf16x8>(qrow + 32 * k);
    }
    __builtin_amdgcn_sched_barrier(0);

    const int k0 = split * p.keys_per_split;
    const int k1 = min(p.kv_len, k0 + p.keys_per_split);
    const int n_stages = (k1 - k0 + KT - 1) / KT;

    // ---- loads of a stage: 16 KB of key rows and 16 KB of transposed values
    const unsigned char *ksrc = (const unsigned char *)(p.Kc + ((size_t)bj * p.spad + k0) * DH);
    const unsigned char *vsrc = (const unsigned char *)(p.Vc + ((size_t)bj * p.spad + k0) * DH);
    uint32_t kgo[LB], vgo[LB];
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int rr = 4 * (LB * wave + i) + (lane >> 4), r = rr & 15;  // LDS row, 256 bytes: row r of 16-key half (rr >> 4) & 1 of a block
        kgo[i] = (uint32_t)(((rr & 32) + 8 * (r >> 2) + 4 * ((rr >> 4) & 1) + (r & 3)) * 256 + (((lane & 15) ^ r) << 4));
        const int dh = 8 * (LB * wave + i) + (lane >> 3);  // LDS row, 128 bytes
        vgo[i] = (uint32_t)(dh * 128 + (((lane & 7) ^ ((dh >> 1) & 7)) << 4));
    }
    auto load_k = [&](int st, int slot, int i) {
        const unsigned char *src = ksrc + (size_t)st * K_BYTES;
        uint32_t at = kgo[i];
        asm("" : "+s"(src), "+v"(at));  // (a scalar base and the lane's 32-bit offset, not a 64-bit sum per load and lane)
        fc_load_lds16<ONCE>(src + at, kring + slot * K_BYTES + (LB * wave + i) * 1024);
    };
    auto load_v = [&](int st, int slot, int i) {
        const unsigned char *src = vsrc + (size_t)st * K_BYTES;
        uint32_t at = vgo[i];
        asm("" : "+s"(src), "+v"(at));
        fc_load_lds16<ONCE>(src + at, vring + slot * K_BYTES + (LB * wave + i) * 1024);
    };
    // keys of stages 0 .. 3, values of 0 .. 2 (past the end the last one again, never read)
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        const int have = min(st, n_stages - 1);
#pragma unroll
        for (int i = 0; i < LB; ++i) load_k(have, st, i);
        if (st < 3)
#pragma unroll
            for (int i = 0; i < LB; ++i) load_v(have, st, i);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- operand fragments: row rho of a tile, step k of the head dimension / half of a stage
    uint32_t kfo[4], vfo[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) kfo[k] = (uint32_t)(rho * 256 + (((4 * k + q) ^ rho) << 4));
#pragma unroll
    for (int h = 0; h < 2; ++h) vfo[h] = (uint32_t)(rho * 128 + (((4 * h + q) ^ ((rho >> 1) & 7)) << 4));
    const float c = p.c;
    // A register's half: the matrix core's for what only it touches, except where the VALU's holds everything.
    auto hold = [](auto &x) {
        if constexpr (QT == 1) asm volatile("" : "+v"(x));
        else asm volatile("" : "+a"(x));
    };
    bf16x8 kf[2][4], vf[8], pf[QT];
    f32x4 s[2][QT][2], o[QT][8];
    float l[QT], nm[QT];  // sum of weights, -c times the reference maximum
    auto read_k = [&](const unsigned char *slot, int half, int i) {  // in the order in which `score` takes them
        kf[i & 1][i >> 1] = *(const bf16x8 *)(slot + half * 8192 + (i & 1) * 4096 + kfo[i >> 1]);
    };
    auto read_v = [&](const unsigned char *slot, int half, int d) { vf[d] = *(const bf16x8 *)(slot + d * 2048 + vfo[half]); };
    // Multiply i of eight: scores of tile u.
    auto score = [&](int buf, int u, int i) {
        f32x4 &d = s[buf][u][i & 1];
        if constexpr (QT == 1) {
            if (i < 2) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=v"(d) : "v"(kf[i & 1][i >> 1]), "v"(qf[u][i >> 1]));
            else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(kf[i & 1][i >> 1]), "v"(qf[u][i >> 1]));
        } else if (i < 2) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=v"(d) : "v"(kf[i & 1][i >> 1]), "a"(qf[u][i >> 1]));
        else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(kf[i & 1][i >> 1]), "a"(qf[u][i >> 1]));
    };
    auto output = [&](int u, int d) { o[u][d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[d], pf[u], o[u][d], 0, 0, 0); };

    auto mask_values = [&](int d, int base) {  // values of keys past the end may hold anything (also NaN): their weights are 0
        union { uint32_t w[4]; bf16x8 v; } x;
        x.v = vf[d];
#pragma unroll
        for (int r = 0; r < 4; ++r) x.w[r] &= (base + 2 * r < k1 ? 0xffffu : 0u) | (base + 2 * r + 1 < k1 ? 0xffff0000u : 0u);
        vf[d] = x.v;
    };

    // ---- first stage: its scores and their maxima (those of the second block are formed again in the loop)
    fc_wait_vm<6 * LB>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < QT; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) hold(qf[u][k]);
#pragma unroll
    for (int i = 0; i < 8; ++i) read_k(kring, 0, i);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
        for (int u = 0; u < QT; ++u) score(0, u, i);
        read_k(kring, 1, i);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int u = 0; u < QT; ++u) score(1, u, i);
    asm volatile("s_nop 15\n\ts_nop 15");  // the last products have left the matrix core
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        float mx = -INFINITY;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 8; ++r) mx = fmaxf(mx, k0 + 32 * h + 8 * q + r < k1 ? s[h][u][r >> 2][r & 3] : -INFINITY);
        nm[u] = -row_max2(row_max16(mx)) * c;
        l[u] = 0.f;
#pragma unroll
        for (int d = 0; d < 8; ++d) o[u][d] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // What rounding takes from the first stage's weights.  (Two tiles: in several ranges only, with one the error is no larger without.)
    if (QT == 1 || (QT == 2 && NW == 4 && p.splits > 1)) {
        fc_wait_vm<5 * LB>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int base = k0 + 32 * h + 8 * q;
#pragma unroll
            for (int d = 0; d < 8; ++d) read_v(vring, h, d);
            if (k1 - k0 < KT)
#pragma unroll
                for (int d = 0; d < 8; ++d) mask_values(d, base);
#pragma unroll
            for (int u = 0; u < QT; ++u) {
                bf16x8 rest;
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const float w = __builtin_amdgcn_exp2f(base + r < k1 ? __builtin_fmaf(s[h][u][r >> 2][r & 3], c, nm[u]) : -INFINITY);
                    rest[r] = (__bf16)(w - (float)(__bf16)w);
                }
#pragma unroll
                for (int d = 0; d < 8; ++d) o[u][d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[d], rest, o[u][d], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        pf[QT - 1][r] = (__bf16)0.f;
#pragma unroll
        for (int d = 0; d < 8; ++d) vf[d][r] = (__bf16)0.f;
    }

    float t[8], e[8], sum = 0.f;
    bf16x8 pw;  // weights of the tile at hand (one tile: those of the block before are still being multiplied)
    auto weight_end = [&](int u) {
        pw[7] = (__bf16)e[7];
        sum += e[7];
    };
    // The weights of tile u and the block at `base`, its scores in s[B], are about to be multiplied.  Where a lane's eight sum to more than
    // MOST, the references of the tile's rows move to the block's maxima first and its weights are formed anew.
    auto weight_use = [&](int B, int u, int base, bool cut) {
        if (__builtin_expect(__any(sum > MOST), 0)) {
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 8; ++r) mx = fmaxf(mx, !cut || base + r < k1 ? s[B][u][r >> 2][r & 3] : -INFINITY);
            const float to = fminf(nm[u], -row_max2(row_max16(mx)) * c), alpha = __builtin_amdgcn_exp2f(to - nm[u]);
            nm[u] = to;
            l[u] *= alpha;
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                hold(o[u][d]);
#pragma unroll
                for (int r = 0; r < 4; ++r) o[u][d][r] *= alpha;
                hold(o[u][d]);  // (back to the matrix core's half of the registers here, not behind the branch)
            }
            sum = 0.f;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                float w = __builtin_amdgcn_exp2f(__builtin_fmaf(s[B][u][r >> 2][r & 3], c, to));
                if (cut) w = base + r < k1 ? w : 0.f;
                pw[r] = (__bf16)w;
                sum += w;
            }
        }
#pragma unroll
        for (int d = 0; d < 8; ++d) hold(o[u][d]);
        pf[u] = pw;
        l[u] += sum;
    };
    // A stage.  LOADS: with all its loads, keys of stage st + 4 and values of stage st + 3; LAST: the last one, with keys past the end.
    auto stage = [&](int st, auto loads, auto last) {
        constexpr bool LOADS = decltype(loads)::value, LAST = decltype(last)::value;
        // the values of stage st and the keys of stage st + 1 have arrived; every wave has read the keys of stage st and the values
        // of stage st - 1
        if (LAST) fc_wait_vm<0, true>();
        else if (LOADS || st + 3 < n_stages) fc_wait_vm<4 * LB, true>();
        else if (st + 2 < n_stages) fc_wait_vm<3 * LB, true>();
        else fc_wait_vm<LB, true>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const unsigned char *const keys = kring + ((st + 1) & 3) * K_BYTES, *const values = vring + (st & 3) * K_BYTES;
        // A block of 32 keys, tile by tile: weights of block i, tile u; beside them the scores of block i + 1, tile u, and the output
        // products of the tile before; fragments of the keys of block i + 2 and of the values of block i, each right behind the last
        // multiply by the one before.
        auto block = [&](auto bc) {
            constexpr int B = decltype(bc)::value, N = B ^ 1;
            constexpr bool SCORES = !LAST || B == 0;
            const int base = k0 + st * KT + 32 * B + 8 * q;
            auto weight = [&](int u, int i) {  // step i of 16 of the weights of tile u
                const int k = i >> 1;
                if ((i & 1) == 0) {
                    t[k] = __builtin_fmaf(s[B][u][k >> 2][k & 3], c, nm[u]);
                    if (LAST) t[k] = base + k < k1 ? t[k] : -INFINITY;
                } else {
                    e[k] = __builtin_amdgcn_exp2f(t[k]);
                    if (k >= 1) {
                        pw[k - 1] = (__bf16)e[k - 1];
                        sum = k == 1 ? e[0] : sum + e[k - 1];
                    }
                }
            };
#pragma unroll
            for (int u = 0; u < QT; ++u)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int before = u == 0 ? QT - 1 : u - 1;  // tile, of this block or the one before
                    const bool behind = u > 0 || B > 0;          // ... whose weights are not in use yet
                    if (i == 0 && behind) weight_end(before);
                    // (one tile: ahead of the score that replaces its first)
                    if (i == (QT == 1 ? 0 : 1) && behind) weight_use(u == 0 ? N : B, before, u == 0 ? base - 32 : base, LAST);
                    if ((i & 1) == 0) {
                        if (SCORES) score(N, u, i >> 1);
                        if (!LAST && u == QT - 1) read_k(keys, B, i >> 1);
                    } else {
                        if (LAST && QT > 1 && u == 1) mask_values(i >> 1, base);
                        if (LAST && QT == 1 && B == 1) mask_values(i >> 1, base - 32);
                        output(before, i >> 1);
                        if (u == 0) read_v(values, B, i >> 1);
                    }
                    weight(u, i);
                    const int g = 16 * u + i, step = 16 * QT / LB;  // a load every `step` multiplies: keys in the first block, values in the other
                    if (g % step == step / 2) {
                        if (B == 0) {
                            if (LOADS || (!LAST && st + 3 < n_stages)) load_v(st + 3, (st + 3) & 3, g / step);
                        } else if (LOADS) {
                            load_k(st + 4, st & 3, g / step);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
        };
        block(std::integral_constant<int, 0>());
        block(std::integral_constant<int, 1>());
        weight_end(QT - 1);
        weight_use(1, QT - 1, k0 + st * KT + 32 + 8 * q, LAST);
    };
    // what goes round the loops keeps its half of the registers
    auto pin = [&]() {
#pragma unroll
        for (int i = 0; i < 8; ++i) asm("" : "+v"(kf[i & 1][i >> 1]), "+v"(vf[i]));
#pragma unroll
        for (int u = 0; u < QT; ++u) {
            asm("" : "+v"(s[0][u][0]), "+v"(s[0][u][1]));
#pragma unroll
            for (int d = 0; d < 8; ++d) hold(o[u][d]);
        }
    };
    pin();
    int st = 0;
    for (; st + 4 < n_stages; ++st) stage(st, std::true_type(), std::false_type()), pin();
    for (; st + 1 < n_stages; ++st) stage(st, std::false_type(), std::false_type()), pin();
    stage(st, std::false_type(), std::true_type());
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        if (QT == 1) mask_values(d, k0 + st * KT + 32 + 8 * q);
        output(QT - 1, d);
    }
    __syncthreads();  // every wave is done with the rings; LDS is reused below

#pragma unroll
    for (int u = 0; u < QT; ++u) l[u] = row_sum2(row_sum16(l[u]));

    if (p.splits > 1) {
        // ---- partial output, in accumulator order, as scaled half floats: the partial of a row is normalised by its own sum (a convex
        // combination of V rows, so it is no larger than the largest |V|) and by a power of two that brings the row's largest
        // magnitude into [2^14, 2^15); eleven significant bits per value, with the row's maximum, sum and exponent in fp32.  That halves
        // the one traffic this kernel adds on top of the key/value stream.  Slot 4 h + d2 of a tile of 32 rows: lane (rho, q) holds of
        // row 16 h + rho the head-dim elements 32 d2 + 4 q .. + 3 and those 16 on.
#pragma unroll
        for (int u = 0; u < QT; ++u) {
            const int t16 = (rg * NW + wave) * QT + u, tt = t16 >> 1, h = t16 & 1;
            if (tt >= p.row_tiles) continue;
            const size_t ts = ((size_t)bj * p.row_tiles + tt) * p.splits + split;
            uint4 *po = (uint4 *)p.part_o + ts * (8 * 64) + h * 256 + lane;
            float amax = 0.f;
#pragma unroll
            for (int d = 0; d < 8; ++d)
#pragma unroll
                for (int r = 0; r < 4; ++r) amax = fmaxf(amax, fabsf(o[u][d][r]));
            const float inv_l = 1.0f / l[u];
            const int k = 15 - __builtin_amdgcn_frexp_expf(row_max2(row_max16(amax)) * inv_l);  // 15 for an all-zero row
#pragma unroll
            for (int d2 = 0; d2 < 4; ++d2) {
                union { _Float16 h[8]; uint4 u4; } x;
#pragma unroll
                for (int e2 = 0; e2 < 8; ++e2) x.h[e2] = (_Float16)__builtin_amdgcn_ldexpf(o[u][2 * d2 + (e2 >> 2)][e2 & 3] * inv_l, k);
                po[d2 * 64] = x.u4;
            }
            if (q == 0) ((float4 *)p.part_ml)[ts * 32 + 16 * h + rho] = make_float4(-nm[u], l[u], (float)k, 0.f);
        }
        return;
    }

    // ---- final output, through the wave's own area: written as whole rows of 256 bytes
    float *stg = (float *)(smem + wave * (QT * 16 * OROW * 4));
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        const float inv = 1.0f / l[u];
#pragma unroll
        for (int d = 0; d < 8; ++d)
            *(float4 *)(stg + (16 * u + rho) * OROW + 16 * d + 4 * q) = make_float4(o[u][d][0] * inv, o[u][d][1] * inv, o[u][d][2] * inv, o[u][d][3] * inv);
    }
    __builtin_amdgcn_wave_barrier();
    fc_wait_lds();
    const int c8 = (lane & 15) * 8;
#pragma unroll 4
    for (int i = 0; i < 4 * QT; ++i) {
        const int r = 4 * i + q, row = row0 + r;
        const float4 x = *(const float4 *)(stg + r * OROW + c8), y = *(const float4 *)(stg + r * OROW + c8 + 4);
        if (row >= nrows) continue;
        const int hg = head_of(row), a = row - hg * p.A;
        const bool padded = row_is_padded(p.pos, b * p.A + a, p.max_seq);
        uint4 w;
        w.x = padded ? 0u : ((uint32_t)fc_bf16_bits(x.x) | ((uint32_t)fc_bf16_bits(x.y) << 16));
        w.y = padded ? 0u : ((uint32_t)fc_bf16_bits(x.z) | ((uint32_t)fc_bf16_bits(x.w) << 16));
        w.z = padded ? 0u : ((uint32_t)fc_bf16_bits(y.x) | ((uint32_t)fc_bf16_bits(y.y) << 16));
        w.w = padded ? 0u : ((uint32_t)fc_bf16_bits(y.z) | ((uint32_t)fc_bf16_bits(y.w) << 16));
        fc_store_any(p.out + ((size_t)b * p.A + a) * ((size_t)p.Hq * DH) + (size_t)(j * p.g + hg) * DH + c8, w);
    }
}

// -------------------------------------------------------------------------------------------------
// 16 QT query rows per workgroup, all keys, a 32-key group per wave at a time: one launch, no partial results.
//
// The waves take stages of 64 keys in turn, each with rings of its own in LDS that it fills itself (direct-to-LDS,
// swizzled as above), so that nothing synchronises them before the end, where their states are merged through LDS.  Every
// workgroup pulls all keys, but from L2.  VP > 1: the columns of V are cut into VP parts, each with the scores of its own: more,
// shorter workgroups where there are few tiles.  16x16 matrix instructions (v_mfma_f32_16x16x32_bf16): a lane (rho, q) holds 8 scores of
// query row rho, the keys 8 q .. 8 q + 7 of the group (the K rows are read in that order), which is the operand layout of P^T.
template <int QT, int VP, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu((NW + 3) / 4, (NW + 3) / 4))) void k_attn_groups(AttnArgs p)
{
    constexpr int ND = 8 / VP;               // 16-column tiles of the output
    constexpr int NK = 8, NV = 16 / VP;      // 1 KB loads of a group's keys and of a stage's values
    constexpr int RS = groups_wave_bytes(QT, VP);  // LDS per wave
    extern __shared__ __align__(1024) unsigned char smem[];

    const int id = blockIdx.x;
    const int xcd = id & 7, qd = id >> 3;
    const uint32_t per_pair = (uint32_t)p.row_tiles * VP, n_tiles = (uint32_t)p.n_units * per_pair;
    const uint32_t tile = xcd * n_tiles / 8 + qd;
    if (tile >= (xcd + 1) * n_tiles / 8) return;
    const int bj = (int)fc_quotient(tile, p.div_pair), mine = (int)(tile - bj * per_pair);
    const int rt = mine / VP, vp = mine - rt * VP;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho = lane & 15, q = lane >> 4;

    // stages of this wave: wave, wave + NW, ..; of the last one of all there may be only the first half
    const int n_stages = (p.kv_len + 63) >> 6;
    const int n = wave < n_stages ? (n_stages - wave + NW - 1) / NW : 0;
    unsigned char *kbuf = smem + wave * RS, *vbuf = kbuf + NK * 1024;

    const unsigned char *kbase = (const unsigned char *)(p.Kc + (size_t)bj * p.spad * DH);
    const unsigned char *vbase = (const unsigned char *)(p.Vc + (size_t)bj * p.spad * DH) + vp * (ND * 16 * 128);
    uint32_t koff[NK], voff[NV];
#pragma unroll
    for (int i = 0; i < NK; ++i) {
        const int row = 4 * i + (lane >> 4), h = row >> 4, r = row & 15;  // LDS row, 256 bytes: row r of 16-key half h
        koff[i] = (uint32_t)((8 * (r >> 2) + 4 * h + (r & 3)) * 256 + (((lane & 15) ^ r) << 4));
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int dh = 8 * i + (lane >> 3);  // LDS row, 128 bytes
        voff[i] = (uint32_t)(dh * 128 + (((lane & 7) ^ ((dh >> 1) & 7)) << 4));
    }
    auto issue_k = [&](int i) {  // half i & 1 of the wave's stage i >> 1
        const unsigned char *src = kbase + (size_t)(wave + NW * (i >> 1)) * (64 * 256) + (i & 1) * (32 * 256);
#pragma unroll
        for (int l = 0; l < NK; ++l) fc_load_lds16(src + koff[l], kbuf + l * 1024);
    };
    auto issue_v = [&](int t) {
        const unsigned char *src = vbase + (size_t)(wave + NW * t) * (FC_VTILE * 256);
#pragma unroll
        for (int l = 0; l < NV; ++l) fc_load_lds16(src + voff[l], vbuf + l * 1024);
    };
    if (n > 0) {
        issue_k(0);
        issue_v(0);
    }
    __builtin_amdgcn_sched_barrier(0);

    // query rows (past the end: the last row, never stored)
    const int b = (int)fc_quotient(bj, p.div_hkv), j = bj - b * p.Hkv;
    bf16x8 qf[QT][4];
    size_t orow[QT];  // output row (element offset)
    int pp[QT];
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        const int row = min(rt * (16 * QT) + 16 * u + rho, p.g * p.A - 1);
        const int hg = (int)fc_quotient(row, p.div_a), a = row - hg * p.A, hq = j * p.g + hg;
        const uint16_t *qrow = p.Q + (((size_t)b * p.Hq + hq) * p.A + a) * DH + 8 * q;
#pragma unroll
        for (int s = 0; s < 4; ++s) qf[u][s] = fc_load_any<bf16x8>(qrow + 32 * s);
        pp[u] = p.pos ? p.pos[b * p.A + a] : 0;
        orow[u] = ((size_t)b * p.A + a) * ((size_t)p.Hq * DH) + (size_t)hq * DH + vp * (ND * 16) + 4 * q;
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
    uint32_t kfo[4], vfo[2];
#pragma unroll
    for (int s = 0; s < 4; ++s) kfo[s] = (uint32_t)(rho * 256 + (((4 * s + q) ^ rho) << 4));
#pragma unroll
    for (int h = 0; h < 2; ++h) vfo[h] = (uint32_t)(rho * 128 + (((4 * h + q) ^ ((rho >> 1) & 7)) << 4));

    bf16x8 vf[2][ND];
    for (int t = 0; t < n; ++t) {
        const int ks0 = 64 * (wave + NW * t);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int i = 2 * t + half, kb = ks0 + 32 * half;
            // this group has arrived, with the first one the stage's values too; the next stage's values may stay in flight
            if (half == 1 && t + 1 < n) fc_wait_vm<NV>();
            else fc_wait_vm<0>();
            __builtin_amdgcn_sched_barrier(0);
            bf16x8 kf[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int s = 0; s < 4; ++s) kf[h][s] = *(const bf16x8 *)(kbuf + h * 4096 + kfo[s]);
            if (half == 0) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int d = 0; d < ND; ++d) vf[h][d] = *(const bf16x8 *)(vbuf + d * 2048 + vfo[h]);
            }
            fc_wait_lds();  // lgkmcnt(0): the areas may be overwritten
            __builtin_amdgcn_sched_barrier(0);
            if (half == 0 || t + 1 < n) issue_k(i + 1);
            if (half == 0 && t + 1 < n) issue_v(t + 1);
            __builtin_amdgcn_sched_barrier(0);
            if (half == 1 && kb >= p.kv_len) break;  // nothing in this half
            f32x4 s[QT][2];
#pragma unroll
            for (int u = 0; u < QT; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h) s[u][h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int u = 0; u < QT; ++u)
#pragma unroll
                    for (int h = 0; h < 2; ++h) s[u][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[h][k], qf[u][k], s[u][h], 0, 0, 0);
            if (kb + 32 > p.kv_len) {  // keys past the end may hold anything (also NaN): no score, and values of 0
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (kb + 8 * q + 4 * h + r >= p.kv_len) {
#pragma unroll
                            for (int u = 0; u < QT; ++u) s[u][h][r] = -INFINITY;
#pragma unroll
                            for (int d = 0; d < ND; ++d) vf[half][d][4 * h + r] = (__bf16)0.f;
                        }
            }
            // The exact running maximum: the largest probabilities are then 1, which bf16 holds exactly (with one that moves only
            // when a probability would pass 2^8, the error over 100 .. 600 keys is 7 % larger).
#pragma unroll
            for (int u = 0; u < QT; ++u) {
                float mx = s[u][0][0];
#pragma unroll
                for (int r = 1; r < 8; ++r) mx = fmaxf(mx, s[u][r >> 2][r & 3]);
                mx = fmaxf(m[u], row_max2(row_max16(mx)));
                const float alpha = __builtin_amdgcn_exp2f((m[u] - mx) * p.c);
                m[u] = mx;
                l[u] *= alpha;
#pragma unroll
                for (int d = 0; d < ND; ++d)
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[u][d][r] *= alpha;
            }
            bf16x8 pf[QT];
#pragma unroll
            for (int u = 0; u < QT; ++u) {
                const float mc = m[u] * p.c;
                float sum[2] = {0.f, 0.f};
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const float pr = __builtin_amdgcn_exp2f(s[u][r >> 2][r & 3] * p.c - mc);
                    sum[r & 1] += pr;
                    pf[u][r] = (__bf16)pr;
                }
                l[u] += sum[0] + sum[1];
            }
#pragma unroll
            for (int d = 0; d < ND; ++d)
#pragma unroll
                for (int u = 0; u < QT; ++u) o[u][d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[half][d], pf[u], o[u][d], 0, 0, 0);
        }
    }

    // ---- merge: every wave leaves its state in its own area; wave w takes accumulators w, w + NW, .. of all of them
    constexpr int NS = QT * ND;
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        const float lu = row_sum2(row_sum16(l[u]));
#pragma unroll
        for (int d = 0; d < ND; ++d) *(f32x4 *)(kbuf + ((u * ND + d) * 64 + lane) * 16) = o[u][d];
        if (q == 0) *(float2 *)(kbuf + NS * 1024 + (16 * u + rho) * 8) = make_float2(m[u], lu);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < QT; ++u)
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            if ((u * ND + d) % NW != wave || rt * (16 * QT) + 16 * u + rho >= p.g * p.A) continue;
            float2 ml[NW];
            float mm = -INFINITY, den = 0.f, y[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                ml[w] = *(const float2 *)(smem + w * RS + NS * 1024 + (16 * u + rho) * 8);
                mm = fmaxf(mm, ml[w].x);
            }
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float k = __builtin_amdgcn_exp2f((ml[w].x - mm) * p.c);  // (0 for a wave without keys)
                const f32x4 v = *(const f32x4 *)(smem + w * RS + ((u * ND + d) * 64 + lane) * 16);
                den += k * ml[w].y;
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] += k * v[e];
            }
            const float inv = 1.0f / den;
            const bool padded = p.pos && (pp[u] < 0 || pp[u] >= p.max_seq);
            uint2 w2;
            w2.x = padded ? 0u : ((uint32_t)fc_bf16_bits(y[0] * inv) | ((uint32_t)fc_bf16_bits(y[1] * inv) << 16));
            w2.y = padded ? 0u : ((uint32_t)fc_bf16_bits(y[2] * inv) | ((uint32_t)fc_bf16_bits(y[3] * inv) << 16));
            fc_store_any(p.out + orow[u] + 16 * d, w2);
        }
}

// Merge the per-range partials: one workgroup of NWV waves per (tile of 32 rows, slot).  Lane (rho, q) owns one row of the tile
// and two groups of four consecutive head-dim elements, exactly as in the first kernel's accumulators, so every load is a
// wave-wide contiguous 1 KB.  Each wave merges an equal share of the ranges, CB of them per batch with all their loads in
// flight together (the launch picks NWV and CB so that one batch per wave covers every range up to 128: the merge is one
// memory round trip); the waves' states are then merged through LDS.
template <int CB, int NWV>
__global__ __launch_bounds__(64 * NWV) void k_attn_combine(AttnArgs p)
{
    __shared__ float xw[NWV > 1 ? NWV : 1][10][64];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per = (p.splits + NWV - 1) / NWV;
    const int s_lo = min(wv * per, p.splits), s_hi = min(s_lo + per, p.splits);
    const int q2 = blockIdx.x & 7;           // slot
    const int col = 16 * (q2 >> 2) + (lane & 15);
    const size_t tg = blockIdx.x >> 3;       // (b * Hkv + j) * row_tiles + rt
    const int bj = (int)p.by_tiles.over(blockIdx.x >> 3), rt = (int)(blockIdx.x >> 3) - bj * p.row_tiles;
    const int b = (int)p.by_hkv.over(bj), j = bj - b * p.Hkv;
    const u32x4 *po = (const u32x4 *)p.part_o + tg * p.splits * (8 * 64) + q2 * 64 + lane;
    const float4 *ml = (const float4 *)p.part_ml + tg * p.splits * 32 + col;

    const int rho = rt * 32 + col, row = min(rho, p.g * p.A - 1);
    const int hg = (int)p.by_a.over(row), a = row - hg * p.A;
    const int pos = p.pos ? p.pos[b * p.A + a] : 0;

    float m_run = -INFINITY, den = 0.f;
    float num[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) num[e] = 0.f;
    for (int sb = s_lo; sb < s_hi; sb += CB) {
        u32x4 v[CB];
        float4 mlv[CB];  // (max in the log2 domain, sum, exponent of the half-float scaling, -)
#pragma unroll
        for (int u = 0; u < CB; ++u) {
            const int s = min(sb + u, s_hi - 1);
            v[u] = po[(size_t)s * (8 * 64)];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < CB; ++u) mlv[u] = ml[(size_t)min(sb + u, s_hi - 1) * 32];
        __builtin_amdgcn_sched_barrier(0);
        // (left to itself the compiler asks for half of these, waits for them, and asks for the other half then)
#pragma unroll
        for (int u = 0; u < CB; ++u) asm volatile("" : "+v"(v[u]));
        float mb = mlv[0].x;
#pragma unroll
        for (int u = 1; u < CB; ++u) mb = fmaxf(mb, mlv[u].x);
        const float m_new = fmaxf(m_run, mb);
        const float keep = __builtin_amdgcn_exp2f(m_run - m_new);  // 0 on the first batch
#pragma unroll
        for (int e = 0; e < 8; ++e) num[e] *= keep;
        den *= keep;
#pragma unroll
        for (int u = 0; u < CB; ++u) {
            // weight of the split's sum; its stored values are (partial / sum) * 2^k
            const float w = (sb + u < s_hi) ? __builtin_amdgcn_exp2f(mlv[u].x - m_new) * mlv[u].y : 0.f;
            const float wn = __builtin_amdgcn_ldexpf(w, -(int)mlv[u].z);
            union { u32x4 u4; _Float16 h[8]; } x;
            x.u4 = v[u];
#pragma unroll
            for (int e = 0; e < 8; ++e) num[e] += wn * (float)x.h[e];
            den += w;
        }
        m_run = m_new;
    }
    if (NWV > 1) {
        // wave 0 (which always has a split) merges the states; a wave without splits holds (-inf, 0, 0)
        xw[wv][0][lane] = m_run;
        xw[wv][1][lane] = den;
#pragma unroll
        for (int e = 0; e < 8; ++e) xw[wv][2 + e][lane] = num[e];
        __syncthreads();
        if (wv != 0) return;
        float m_all = m_run;
#pragma unroll
        for (int w2 = 1; w2 < NWV; ++w2) m_all = fmaxf(m_all, xw[w2][0][lane]);
        const float k0 = __builtin_amdgcn_exp2f(m_run - m_all);
        den *= k0;
#pragma unroll
        for (int e = 0; e < 8; ++e) num[e] *= k0;
#pragma unroll
        for (int w2 = 1; w2 < NWV; ++w2) {
            const float kw2 = __builtin_amdgcn_exp2f(xw[w2][0][lane] - m_all);
            den += kw2 * xw[w2][1][lane];
#pragma unroll
            for (int e = 0; e < 8; ++e) num[e] += kw2 * xw[w2][2 + e][lane];
        }
    }

    if (rho >= p.g * p.A) return;  // row past the end of the last tile
    const int hq = j * p.g + hg;
    const bool padded = p.pos && (pos < 0 || pos >= p.max_seq);
    uint16_t *orow = p.out + ((size_t)b * p.A + a) * ((size_t)p.Hq * DH) + (size_t)hq * DH;
#pragma unroll
    for (int g2 = 0; g2 < 2; ++g2) {
        uint2 w;
        w.x = padded ? 0u : ((uint32_t)fc_bf16_bits(num[4 * g2] / den) | ((uint32_t)fc_bf16_bits(num[4 * g2 + 1] / den) << 16));
        w.y = padded ? 0u : ((uint32_t)fc_bf16_bits(num[4 * g2 + 2] / den) | ((uint32_t)fc_bf16_bits(num[4 * g2 + 3] / den) << 16));
        const int dh = 32 * (q2 & 3) + 16 * g2 + 4 * (lane >> 4);
        *(uint2 *)(orow + dh) = w;
    }
}

// 16 QT NW rows per workgroup
template <int QT, int NW>
hipError_t launch_ranges(AttnArgs a, hipStream_t s)
{
    constexpr int STAGING = NW * QT * 16 * OROW * 4, LDS_BYTES = STAGING > 8 * K_BYTES ? STAGING : 8 * K_BYTES;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
    auto start = [&](auto once) {
        constexpr auto kernel = k_attn_ranges<QT, NW, decltype(once)::value>;
        static hipError_t attr = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (attr != hipSuccess) return attr;
        const unsigned grid = (unsigned)(((int64_t)a.n_units * a.n_rg + 7) / 8 * 8);
        kernel<<<dim3(grid), dim3(NW * 64), LDS_BYTES, s>>>(a);
        return hipGetLastError();
    };
    return a.once ? start(std::true_type()) : start(std::false_type());
}

template <int QT, int VP, int NW>
hipError_t launch_groups(AttnArgs a, hipStream_t s)
{
    constexpr int LDS_BYTES = NW * groups_wave_bytes(QT, VP);
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
    static hipError_t attr = hipFuncSetAttribute((const void *)k_attn_groups<QT, VP, NW>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
    if (attr != hipSuccess) return attr;
    const int64_t rows = (int64_t)a.g * a.A, row_tiles = (rows + 16 * QT - 1) / (16 * QT), pairs = (int64_t)a.B * a.Hkv;
    const int64_t n = pairs * row_tiles * VP;
    if (n > 4096 || rows > 32768) return hipErrorInvalidValue;
    a.row_tiles = (int)row_tiles;
    a.n_units = (int)pairs;
    a.div_pair = fc_reciprocal(row_tiles * VP);
    a.div_hkv = fc_reciprocal(a.Hkv);
    a.div_a = fc_reciprocal(a.A);
    k_attn_groups<QT, VP, NW><<<dim3((unsigned)((n + 7) / 8 * 8)), dim3(NW * 64), LDS_BYTES, s>>>(a);
    return hipGetLastError();
}

}  // namespace

hipError_t fc_launch_attention_mfma(const FcGeom &G, const FcAttnPlan &pl, const void *q, const void *k_layer,
                                    const void *v_layer, const int32_t *pos, int A, int kv_len, void *out,
                                    void *workspace, hipStream_t s)
{
    AttnArgs a;
    a.Q = (const uint16_t *)q;
    a.Kc = (const uint16_t *)k_layer;
    a.Vc = (const uint16_t *)v_layer;
    a.pos = pos;
    a.out = (uint16_t *)out;
    // workspace: per (row tile, split) 32 x 128 scaled half floats, then 32 x (max, sum, exponent, -)
    const size_t tiles = (size_t)G.B * G.Hkv * pl.row_tiles;
    a.part_o = (float *)workspace;
    a.part_ml = workspace ? (float *)workspace + tiles * pl.splits * (32 * DH / 2) : nullptr;
    a.B = G.B;
    a.Hq = G.Hq;
    a.Hkv = G.Hkv;
    a.g = G.g;
    a.A = A;
    a.kv_len = kv_len;
    a.spad = G.spad;
    a.max_seq = G.max_seq;
    a.row_tiles = pl.row_tiles;
    a.n_rg = (pl.row_tiles + pl.tiles_per_wg - 1) / pl.tiles_per_wg;
    a.splits = pl.splits;
    a.keys_per_split = pl.keys_per_split;
    a.n_units = G.B * G.Hkv * pl.splits;
    a.once = G.once && a.n_rg == 1;
    a.c = G.scale * 1.4426950408889634f;
    a.by_rg.set(a.n_rg);
    a.by_splits.set(pl.splits);
    a.by_tiles.set(pl.row_tiles);
    a.by_hkv.set(G.Hkv);
    a.by_a.set(A);
    hipError_t e;
    const int R = pl.tiles_per_wg;
    if (pl.kind == 2) {  // all keys in one launch
        if (pl.splits != 1) return hipErrorInvalidValue;
        if (R == 2) return launch_groups<2, 2, 8>(a, s);
        if (pl.v_parts == 4) return launch_groups<1, 4, 8>(a, s);
        if (pl.v_parts == 2) return launch_groups<1, 2, 8>(a, s);
        if (pl.v_parts == 1) return launch_groups<1, 1, 6>(a, s);
        return hipErrorInvalidValue;
    }
    if (pl.waves == 4) {  // a wave per SIMD
        if (R == 8) e = launch_ranges<4, 4>(a, s);
        else if (R == 4) e = launch_ranges<2, 4>(a, s);
        else if (R == 2) e = launch_ranges<1, 4>(a, s);
        else return hipErrorInvalidValue;
    } else {              // two
        if (R == 8) e = launch_ranges<2, 8>(a, s);
        else if (R == 4) e = launch_ranges<1, 8>(a, s);
        else return hipErrorInvalidValue;
    }
    if (e != hipSuccess || pl.splits == 1) return e;
    const dim3 cgrid((unsigned)(tiles * 8));
    if (pl.splits <= 2) k_attn_combine<2, 1><<<cgrid, dim3(64), 0, s>>>(a);
    else if (pl.splits <= 8) k_attn_combine<8, 1><<<cgrid, dim3(64), 0, s>>>(a);
    else if (pl.splits <= 16) k_attn_combine<8, 2><<<cgrid, dim3(128), 0, s>>>(a);
    else if (pl.splits <= 32) k_attn_combine<8, 4><<<cgrid, dim3(256), 0, s>>>(a);
    else if (pl.splits <= 64) k_attn_combine<16, 4><<<cgrid, dim3(256), 0, s>>>(a);
    else k_attn_combine<32, 4><<<cgrid, dim3(256), 0, s>>>(a);
    return hipGetLastError();
}
