// ec_prefill_score / ec_chunk_score for fp32 inputs: fp32 matrix instructions, fp32 arithmetic throughout.
// Geometry (ScoreGeom): Tq queries over L = P + Tq key rows, query m sees rows n <= P + m.
//
// The same two passes as for bf16, on v_mfma_f32_16x16x4_f32:
//   attn_fwd_f32 : S^T = K.Q^T per block of 16 keys x 16 queries, so that a lane owns one query and 4 keys; its online
//                  softmax and O^T += V^T.P^T, whose B operand the probabilities are as they stand: instruction j of
//                  a block contracts the keys 4h + j that the four quarters h of the wave hold.
//   colsum_f32   : the K operands of 16 keys stay in registers, queries stream through LDS, p = exp(s - lse_row) is
//                  summed per key over a lane's queries and over the lanes at the end.  One workgroup owns a column:
//                  no atomics, deterministic.
// Bound: the matrix pipe at its fp32 rate (a sixteenth of the bf16 one; 149 TFLOP/s in a large product here).  A tile of 32
// keys costs a wave 128 instructions of 32 clocks (D = 128); while two waves share a SIMD the vector work fills the gaps, but the
// longest workgroups end alone, and there everything between the matrix instructions adds up: 6.9 thousand clocks a tile
// with the compiler's order, of which 4.1 matrix time.  Operands requested ahead at constant addresses, loads among the matrix
// instructions and the bare exponential instruction took that down.  Measured (graph replay), vector ALU -> matrix
// instructions -> now: whole call at B1 H32 T1024 D128 694 -> 148 -> 128 us (100 TFLOP/s; a workgroup loops over up to 32 tiles
// while the mean is 16), T2048 496 -> 450, T512 58.5 -> 51.7, H8 T1024 81 -> 69.5, B1 H32 T1024 D64 88 -> 76.
// Eight waves on 64 queries, two on the keys of each 16: 168 us at T1024 (81 at D64), all of them in step.
// The operands that stay in registers come through LDS (whole call, graph replay, straight from memory / now): B1 H32 D128 T1024
// 126.9 / 126.1, T512 49.3 / 47.2, H4 T100 14.7 / 13.5, B8 T130 51.1 / 48.8, B4 D64 T300 39.5 / 37.4, H4 D64 T256 14.2 / 13.5.
// Error of out against 64 bits at T1024 6.3e-7 (vector ALU) -> 2.8e-7, of the scores 1.3e-7 -> 1.1e-7, no change by the order.
// Operands are read from LDS 16 bytes at a time, each read feeding four instructions: both operands of a contraction
// enumerate it in the same permuted order.
//
// Operand layout (wave64, lane l, quarter h = l / 16): A (16 x 4): lane holds A[l % 16][h];  B (4 x 16): B[h][l % 16];
//   C (16 x 16): lane holds C[4h + r][l % 16] in register r.
#include <type_traits>

#include "tile_lds.h"

namespace ec {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((address_space(3))) const f32x4 lds_f32x4;

constexpr int kF32Waves = 4;

struct Swizzle16 {  // operand reads of 16 consecutive rows at one chunk number touch every bank once
    static constexpr int kPeriod = 16;
    static __device__ __forceinline__ int at(int r) { return r & 15; }
};

__device__ __forceinline__ f32x4 lds_read(uint32_t at) { return *(lds_f32x4*)(uintptr_t)at; }

// Item of a launch whose heads have n_tiles tiles each.  One XCD works on every eighth head; inside it the tiles come
// longest first over all heads, every second run of 32 (a workgroup for each of the XCD's compute units) backwards: a
// launch that fits on the chip at once then gives every compute unit a long tile and a short one.
struct F32Item {
    int bh, rank;  // rank 0: the longest tile of its head; bh < 0: nothing to do
};
__device__ __forceinline__ F32Item f32_item(int linear_id, int n_tiles, int n_heads)
{
    const int xcd = linear_id % kXcds, nth = linear_id / kXcds;
    const int heads = (n_heads - xcd + kXcds - 1) / kXcds;  // of this XCD
    const int total = heads * n_tiles;
    if (nth >= total) return {-1, 0};
    const int run = nth / 32, first = run * 32, len = min(32, total - first);
    const int place = (run % 2) ? first + len - 1 - (nth - first) : nth;
    return {place % heads * kXcds + xcd, place / heads};
}
inline int f32_grid(int n_tiles, int n_heads) { return (n_heads + kXcds - 1) / kXcds * n_tiles * kXcds; }

// A wave that has the SIMD to itself, as the longest workgroup of a launch does at the end, pays for every vector instruction
// and every wait between its matrix instructions (a 16x16x4 takes 32 clocks, two additions behind it make that 44).  So operands
// are requested kAhead reads before the four matrix instructions that use them, at addresses that differ by constants, the next
// tile's loads are issued in between, and the order is fixed by hand.
constexpr int kAhead = 4;

// Maximum over the four quarters of the wave.
__device__ __forceinline__ float quarters_max(float x)
{
    const auto y = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(y[0]), __uint_as_float(y[1]));
    const auto z = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(z[0]), __uint_as_float(z[1]));
}

// ------------------------------------------------------------------ forward
// QW waves of 16 queries each x KS waves that share a tile's blocks of 16 keys (QW * KS = 4).  Tiles of 16 * 2 * max(1,
// KS / 2) keys, double-buffered.  KS = 4: launches that would leave most of the chip idle; the four partial (max, sum,
// O) of a query meet in LDS at the end, in ascending order.  KS = 2 lies between.
template <int D, int QW, int KS, bool OUT>
__global__ __launch_bounds__(kF32Waves * kWave, KS == 1 ? 2 : 1) void attn_fwd_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, float* __restrict__ out,
    float* __restrict__ lse, float lse_unit, ScoreGeom geo, float scale_log2e, int n_qtiles, int n_heads,
    const int32_t* __restrict__ seq_len, int H)
{
    static_assert(QW * KS == kF32Waves, "four waves");
    constexpr int BM = QW * 16;
    constexpr int NBLK = KS == 1 ? 2 : 1;     // blocks of a tile per wave
    constexpr int TN = 16 * NBLK * KS;        // keys per tile
    constexpr int KB = D / 16, DB = D / 16;
    constexpr int TILE = TN * D * 4;          // bytes
    using Mover = TileToLds<2 * D, TN, kF32Waves, Swizzle16>;
    __shared__ __align__(16) float tiles[4 * TN * D];  // K even, K odd, V even, V odd
    __shared__ float stats[KS > 1 ? 2 * kF32Waves * 16 : 1];

    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int qw = wave % QW, ks = wave / QW;
    const int r16 = lane % 16, h = lane / 16;
    const F32Item item = f32_item(blockIdx.x, n_qtiles, n_heads);
    if (item.bh < 0) return;
    const int bh = item.bh;
    const int Tq = ragged_rows(seq_len, bh / H, geo.Tq), P = geo.P, L = P + Tq;
    const int m0 = (n_qtiles - 1 - item.rank) * BM;
    if (m0 >= Tq) return;  // ragged batch: this sequence ends before the tile (whole workgroup)
    const int mw = m0 + qw * 16, m = mw + r16;  // first query of the wave, this lane's
    const Mover k_move(tile_rsrc(k + (size_t)bh * geo.kv_rows * D, (uint32_t)L * (D * 4)), wave, lane);
    const Mover v_move(tile_rsrc(v + (size_t)bh * geo.kv_rows * D, (uint32_t)L * (D * 4)), wave, lane);
    const uint32_t base = lds_address(tiles);
    constexpr int LOADS = OUT ? 2 * Mover::NI : Mover::NI;  // of a wave per tile
    auto fetch = [&](int t, int from, int to) __attribute__((always_inline)) {
        const uint32_t at = base + t % 2 * TILE;
#pragma unroll
        for (int j = from; j < to; ++j) {
            if (j < Mover::NI)
                k_move.issue(at, t * TN, j);
            else
                v_move.issue(at + 2 * TILE, t * TN, j - Mover::NI);
        }
    };
    const int n_end = min(L, P + m0 + BM);
    const int n_tiles = (n_end + TN - 1) / TN;
    fetch(0, 0, LOADS);

    // The queries, a row per lane, are read from LDS, where they come in at the places of the odd tiles: straight from memory each of a
    // load's 64 lanes would be a request of its own, 64 clocks of the compute unit's cache instead of 16.
    {
        const Mover q_move(tile_rsrc(q + (size_t)bh * geo.q_rows * D, (uint32_t)Tq * (D * 4)), wave, lane);
#pragma unroll
        for (int half = 0; half < (BM + TN - 1) / TN; ++half)
            if (q_move.w0 < BM) {
#pragma unroll
                for (int j = 0; j < Mover::NI; ++j) q_move.issue(base + (half == 0 ? 1 : 3) * TILE, m0 + half * TN, j);
            }
    }
    f32x4 qf[KB];  // B operand: element e of block kb is feature 16 kb + 4 h + e of this lane's query
    f32x4 o[DB];  // O^T: register r of block db is feature 64 (db / 4) + 4 (4h + r) + db % 4
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Maximum of the scores before scaling: the largest one's exponent is then exactly 0, however large the scores are,
    // where a scaled maximum would leave the rounding of its product.  l_run: this lane's share of the row sum.
    float m_run = kLowest, l_run = 0.f;

    wait_loads();
    meet();
    {
        const uint32_t row = base + (BM > TN && qw * 16 >= TN ? 3 : 1) * TILE + (qw * 16 % TN + r16) * (D * 4);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) qf[kb] = lds_read(row + ((4 * kb + h) ^ r16) * 16);
    }
    // Byte addresses of this lane's operands in the even tiles.  K: contraction block kb of key r16 of the wave's first block.
    // V: 4 features (of every 64) of key 4h + j there.
    constexpr int VC = D / 64;
    uint32_t k_at[KB], v_at[4];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) k_at[kb] = one_register(base + (ks * 16 + r16) * (D * 4) + ((4 * kb + h) ^ r16) * 16);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        v_at[j] = one_register(base + 2 * TILE + (ks * 16 + 4 * h + j) * (D * 4) + (r16 ^ (4 * h + j)) * 16);

    auto body = [&](int t, auto odd) __attribute__((always_inline)) {
        constexpr int PAR = odd.value ? TILE : 0;
        constexpr int NF = KB * NBLK, NV = NBLK * 4 * VC;  // operands of S^T: (block kb, key block); of O^T: (key block, j, 64 features)
        constexpr bool SPREAD = NF >= 16;  // loads between the matrix instructions: B8 T300 H32 D128 127 -> 121 us; D64 76.4 -> 78.5
        wait_loads();
        wait_lds();
        meet();  // tile t has landed, tile t - 1 has been read
        const bool more = t + 1 < n_tiles;
        const int n0 = t * TN + ks * 16;  // the wave's blocks start 16 KS keys apart
        const bool idle = n0 > P + mw + 15;  // every key is in the future of the wave's queries
        if (more && (!SPREAD || idle)) fetch(t + 1, 0, LOADS);
        if (idle) return;
        auto operand_k = [&](int f) __attribute__((always_inline)) { return lds_read(k_at[f / NBLK] + (PAR + f % NBLK * KS * 16 * D * 4)); };
        auto operand_v = [&](int g) __attribute__((always_inline)) {
            return lds_read(v_at[g / VC % 4] + (PAR + g / VC / 4 * KS * 16 * D * 4 + g % VC * 256));
        };
        // S^T in four chains per block: shorter sums, and no instruction waits for the one before it
        f32x4 c[NBLK][4], ka[NF], va[NV], s[NBLK];
#pragma unroll
        for (int f = 0; f < kAhead; ++f) ka[f] = operand_k(f);
#pragma unroll
        for (int b = 0; b < NBLK; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) c[b][e] = f32x4{0.f, 0.f, 0.f, 0.f};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                c[f % NBLK][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(ka[f][e], qf[f / NBLK][e], c[f % NBLK][e], 0, 0, 0);
            if (f + kAhead < NF)
                ka[f + kAhead] = operand_k(f + kAhead);
            else if (OUT)
                va[f + kAhead - NF] = operand_v(f + kAhead - NF);  // on their way during the softmax
            if (SPREAD && more) fetch(t + 1, f * LOADS / NF, (f + 1) * LOADS / NF);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int b = 0; b < NBLK; ++b) s[b] = (c[b][0] + c[b][1]) + (c[b][2] + c[b][3]);
        float mn = INFINITY;
#pragma unroll
        for (int b = 0; b < NBLK; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) mn = fminf(mn, s[b][r]);
        if (n0 + (NBLK - 1) * 16 * KS + 15 > P + mw) {
#pragma unroll
            for (int b = 0; b < NBLK; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (n0 + b * 16 * KS + 4 * h + r > P + m) s[b][r] = -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int b = 0; b < NBLK; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s[b][r]);
        mx = quarters_max(mx);
        const float m_new = fmaxf(m_run, mx);
        const float corr = exp2f((m_run - m_new) * scale_log2e);
        m_run = m_new;
#pragma unroll
        for (int b = 0; b < NBLK; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) s[b][r] = (s[b][r] - m_new) * scale_log2e;
        // the exponential instruction gives zero where the result is subnormal; exp2f, which is six times as long, does not
        if (__builtin_expect(__any((mn - m_new) * scale_log2e < -126.f), 0)) {
#pragma unroll
            for (int b = 0; b < NBLK; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) s[b][r] = exp2f(s[b][r]);
        } else {
#pragma unroll
            for (int b = 0; b < NBLK; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) s[b][r] = __builtin_amdgcn_exp2f(s[b][r]);
        }
        float psum = 0.f;
#pragma unroll
        for (int b = 0; b < NBLK; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) psum += s[b][r];
        l_run = fmaf(l_run, corr, psum);
        if constexpr (OUT) {
            // a tile is summed by itself and then added: the rounding errors of a long chain stay small
            f32x4 ot[DB];
#pragma unroll
            for (int db = 0; db < DB; ++db) ot[db] = f32x4{0.f, 0.f, 0.f, 0.f};
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < NV; ++g) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    ot[g % VC * 4 + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(va[g][e], s[g / VC / 4][g / VC % 4], ot[g % VC * 4 + e], 0, 0, 0);
                if (g + kAhead < NV) va[g + kAhead] = operand_v(g + kAhead);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 4; ++r) o[db][r] = fmaf(o[db][r], corr, ot[db][r]);
        }
    };
    for (int t = 0; t < n_tiles; t += 2) {
        body(t, std::false_type{});
        if (t + 1 < n_tiles) body(t + 1, std::true_type{});
    }

    l_run += __shfl_xor(l_run, 16, kWave);
    l_run += __shfl_xor(l_run, 32, kWave);
    if constexpr (KS > 1) {
        wait_lds();
        meet();  // the tiles have been read
        // wave w leaves word j of its lane l at (w * DB * 4 + j) * 64 + l
        if constexpr (OUT) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 4; ++r) tiles[(wave * DB * 4 + db * 4 + r) * kWave + lane] = o[db][r];
        }
        if (h == 0) {
            stats[wave * 16 + r16] = m_run;
            stats[(kF32Waves + wave) * 16 + r16] = l_run;
        }
        __syncthreads();
        if (ks > 0) return;
        float m_all = m_run;
#pragma unroll
        for (int w = 1; w < KS; ++w) m_all = fmaxf(m_all, stats[(w * QW + qw) * 16 + r16]);
        const float f0 = exp2f((m_run - m_all) * scale_log2e);
        l_run *= f0;
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db] *= f0;
#pragma unroll
        for (int w = 1; w < KS; ++w) {
            const float f = exp2f((stats[(w * QW + qw) * 16 + r16] - m_all) * scale_log2e);
            l_run = fmaf(stats[(kF32Waves + w * QW + qw) * 16 + r16], f, l_run);
            if constexpr (OUT) {
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        o[db][r] = fmaf(tiles[((w * QW + qw) * DB * 4 + db * 4 + r) * kWave + lane], f, o[db][r]);
            }
        }
        m_run = m_all;
    }
    if (m < Tq) {
        if (h == 0) lse[(size_t)bh * geo.q_rows + m] = fmaf(m_run, scale_log2e, log2f(l_run)) * lse_unit;
        if constexpr (OUT) {
            const float inv = 1.f / l_run;
            float* orow = out + ((size_t)bh * geo.q_rows + m) * D;
#pragma unroll
            for (int c = 0; c < D / 64; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    f32x4 y;
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = o[4 * c + e][r] * inv;
                    *reinterpret_cast<f32x4*>(orow + c * 64 + h * 16 + r * 4) = y;
                }
        }
    }
}

// ------------------------------------------------------------------ column mass
// KW waves of 16 keys each x QG waves that take the blocks of 16 queries in turn (KW * QG = 4); tiles of 16 QG queries,
// double-buffered.
template <int D, int KW, int QG>
__global__ __launch_bounds__(kF32Waves * kWave, 2) void colsum_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ lse, float lse_unit,
    float* __restrict__ head_imp, ScoreGeom geo, float scale_log2e, int n_ktiles, int n_heads,
    const int32_t* __restrict__ seq_len, int H)
{
    static_assert(KW * QG == kF32Waves, "four waves");
    constexpr int BN = KW * 16;
    constexpr int TQ = 16 * QG;  // queries per tile
    constexpr int KB = D / 16;
    constexpr int TILE = TQ * D * 4;
    using Mover = TileToLds<2 * D, TQ, kF32Waves, Swizzle16>;
    __shared__ __align__(16) float tiles[2 * TQ * D];
    __shared__ float red[kF32Waves][16];

    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int kw = wave % KW, qg = wave / KW;
    const int r16 = lane % 16, h = lane / 16;
    const F32Item item = f32_item(blockIdx.x, n_ktiles, n_heads);
    if (item.bh < 0) return;
    const int bh = item.bh;
    const int Tq = ragged_rows(seq_len, bh / H, geo.Tq), P = geo.P, L = P + Tq;
    const int n0 = item.rank * BN;  // low keys have the most queries
    if (n0 >= L) return;  // ragged batch: this sequence ends before the tile (whole workgroup)
    const int nw = n0 + kw * 16;
    const Mover q_move(tile_rsrc(q + (size_t)bh * geo.q_rows * D, (uint32_t)Tq * (D * 4)), wave, lane);
    const float* lh = lse + (size_t)bh * geo.q_rows;
    const uint32_t base = lds_address(tiles);
    const int m_begin = max(n0 - P, 0) / TQ * TQ;  // first tile with a query that sees key n0
    const int n_tiles = (Tq - m_begin + TQ - 1) / TQ;
    float l2_next;  // log-sum-exp of the lane's query in the tile being fetched
    auto fetch = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < Mover::NI; ++j) q_move.issue(base + t % 2 * TILE, m_begin + t * TQ, j);
        l2_next = lh[min(m_begin + t * TQ + qg * 16 + r16, Tq - 1)];
    };
    fetch(0);

    // the keys come in where the odd tiles go, as the queries of the forward pass do
    {
        const Mover k_move(tile_rsrc(k + (size_t)bh * geo.kv_rows * D, (uint32_t)L * (D * 4)), wave, lane);
        if (k_move.w0 < BN) {
#pragma unroll
            for (int j = 0; j < Mover::NI; ++j) k_move.issue(base + TILE, n0, j);
        }
    }
    f32x4 kf[KB];  // A operand: element e of block kb is feature 16 kb + 4 h + e of key nw + r16
    f32x4 col = f32x4{0.f, 0.f, 0.f, 0.f};  // keys nw + 4 h + r
    static_assert(BN <= TQ, "an odd tile holds the keys");
    wait_loads();
    meet();
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) kf[kb] = lds_read(base + TILE + (kw * 16 + r16) * (D * 4) + ((4 * kb + h) ^ r16) * 16);
    uint32_t q_at[KB];  // byte address of this lane's operand of contraction block kb in the even tiles
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) q_at[kb] = one_register(base + (qg * 16 + r16) * (D * 4) + ((4 * kb + h) ^ r16) * 16);
    auto body = [&](int t, auto odd) __attribute__((always_inline)) {
        constexpr int PAR = odd.value ? TILE : 0;
        const int m0 = m_begin + t * TQ + qg * 16;  // first query of the wave's block
        wait_loads();
        wait_lds();
        meet();  // tile t has landed, tile t - 1 has been read
        const float l2 = l2_next * lse_unit;
        if (t + 1 < n_tiles) fetch(t + 1);
        if (P + m0 + 15 < nw) return;  // no query of the tile sees a key of this wave
        f32x4 s[4], a[KB];
#pragma unroll
        for (int kb = 0; kb < kAhead; ++kb) a[kb] = lds_read(q_at[kb] + PAR);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = f32x4{0.f, 0.f, 0.f, 0.f};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kb][e], a[kb][e], s[e], 0, 0, 0);
            if (kb + kAhead < KB) a[kb + kAhead] = lds_read(q_at[kb + kAhead] + PAR);
            __builtin_amdgcn_sched_barrier(0);
        }
        f32x4 p;
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r] = fmaf((s[0][r] + s[1][r]) + (s[2][r] + s[3][r]), scale_log2e, -l2);
        // as in the forward pass
        if (__any(fminf(fminf(p[0], p[1]), fminf(p[2], p[3])) < -126.f)) {
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r] = exp2f(p[r]);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(p[r]);
        }
        if (m0 + 16 > Tq || P + m0 < nw + 15) {  // uniform: a query behind the last one, or a key behind its query
            const int m = m0 + r16;
            const int last = m < Tq ? P + m - nw - 4 * h : -1;  // last of the lane's keys that its query sees
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r] = r <= last ? p[r] : 0.f;
        }
        col += p;
    };
    for (int t = 0; t < n_tiles; t += 2) {
        body(t, std::false_type{});
        if (t + 1 < n_tiles) body(t + 1, std::true_type{});
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float x = group_sum<16>(col[r]);
        if (r16 == 0) red[wave][4 * h + r] = x;
    }
    __syncthreads();
    const int key = threadIdx.x;
    if (key < BN && n0 + key < L) {
        float sum = 0.f;
#pragma unroll
        for (int g = 0; g < QG; ++g) sum += red[g * KW + key / 16][key % 16];
        head_imp[(size_t)bh * geo.imp_rows + n0 + key] = sum;
    }
}

template <int D>
static int launch_f32(const float* q, const float* k, const float* v, float* out, float* lse, bool lse_wanted,
                      float* head_imp, int B, int H, ScoreGeom geo, const int32_t* seq_len, float scale, hipStream_t stream)
{
    const float sl = scale * kLog2e;
    // between the two passes the log-sum-exp stays in base-2 units (two roundings less) unless the caller reads it
    const float unit_out = lse_wanted ? kLn2 : 1.f, unit_in = lse_wanted ? kLog2e : 1.f;
    const int BH = B * H;
    const dim3 block(kF32Waves * kWave);
    const int qt64 = (geo.Tq + 63) / 64, qt32 = (geo.Tq + 31) / 32, qt16 = (geo.Tq + 15) / 16;
#define EC_FWD_F32(QW_, KS_, QT_)                                                                                        \
    do {                                                                                                              \
        if (out != nullptr)                                                                                           \
            hipLaunchKernelGGL((attn_fwd_f32_kernel<D, QW_, KS_, true>), dim3(f32_grid(QT_, BH)), block, 0, stream, q, \
                               k, v, out, lse, unit_out, geo, sl, QT_, BH, seq_len, H);                                         \
        else                                                                                                          \
            hipLaunchKernelGGL((attn_fwd_f32_kernel<D, QW_, KS_, false>), dim3(f32_grid(QT_, BH)), block, 0, stream,  \
                               q, k, v, out, lse, unit_out, geo, sl, QT_, BH, seq_len, H);                                      \
    } while (0)
    // us of the whole call for 64 / 32 / 16 queries per workgroup (one / two / four waves on the keys of 16 queries), H32
    // D128, the column pass alike:
    //   B1 T256 34.0 / 28.2 / 29.8   B1 T512 61.0 / 52.2 / 67.0   B1 T1024 130 / 143 / 186   B4 T256 47.2 / 52.9 / 80.4
    //   B1 T2048 451 / 476 / 642   H16 B1 T1024 105 / 82.6 / 104   H8 B1 T512 50.2 / 38.3 / 29.2
    const long long wide = (long long)qt64 * BH;
    if (wide >= 512)
        EC_FWD_F32(4, 1, qt64);
    else if (wide >= 128)
        EC_FWD_F32(2, 2, qt32);
    else
        EC_FWD_F32(1, 4, qt16);
#undef EC_FWD_F32
    int rc = status_from_hip(hipGetLastError());
    if (rc != EC_OK) return rc;
    const int kt32 = (geo.L + 31) / 32, kt16 = (geo.L + 15) / 16;
    // us of the whole call for 32 / 16 keys per workgroup:
    //   B1 T256 29.2 / 28.5   B1 T512 51.9 / 55.5   B1 T1024 131 / 144   B4 T256 47.7 / 57.2   H8 B1 T512 34.0 / 29.1
    if ((long long)kt32 * BH >= 512)
        hipLaunchKernelGGL((colsum_f32_kernel<D, 2, 2>), dim3(f32_grid(kt32, BH)), block, 0, stream, q, k, lse, unit_in,
                           head_imp, geo, sl, kt32, BH, seq_len, H);
    else
        hipLaunchKernelGGL((colsum_f32_kernel<D, 1, 4>), dim3(f32_grid(kt16, BH)), block, 0, stream, q, k, lse, unit_in,
                           head_imp, geo, sl, kt16, BH, seq_len, H);
    return status_from_hip(hipGetLastError());
}

// Per-head importance into head_imp [B,H,L]; out may be NULL (then v is not read).  lse is a scratch row unless lse_wanted.
int score_f32_dispatch(const void* q, const void* k, const void* v, void* out, float* lse, bool lse_wanted,
                       float* head_imp, int B, int H, ScoreGeom geo, const int32_t* seq_len, int D, float scale,
                       hipStream_t stream)
{
    if (D == 128)
        return launch_f32<128>((const float*)q, (const float*)k, (const float*)v, (float*)out, lse, lse_wanted, head_imp,
                               B, H, geo, seq_len, scale, stream);
    if (D == 64)
        return launch_f32<64>((const float*)q, (const float*)k, (const float*)v, (float*)out, lse, lse_wanted, head_imp,
                              B, H, geo, seq_len, scale, stream);
    return EC_EUNSUPPORTED;
}

}  // namespace ec
