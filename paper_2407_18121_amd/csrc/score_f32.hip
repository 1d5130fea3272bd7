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
// Bound: the matrix pipe at its fp32 rate (a sixteenth of the bf16 one; 149 TFLOP/s in a large product here); a block costs
// 64 instructions of 32 clocks (D = 128) against some 30 vector instructions, so the phases simply follow each other and
// the other wave of the SIMD fills the gaps.  Measured, before (vector ALU) -> after: whole call at B1 H32 T1024 D128
// 694 -> 143 us (90 TFLOP/s; a workgroup loops over up to 32 tiles while the mean is 16).  By the profiler, which times
// every launch by itself and adds its start, the two passes take 498 + 221 -> 103 + 53 us there (109 + 52 us with the
// waits for the operands inside the loop) and 61 + 22 -> 7.9 + 4.8 us at B1 H4 T256 D64.
// Error of out against 64 bits at T1024 6.3e-7 -> 2.7e-7, of the scores 1.3e-7 -> 0.7e-7.
// Operands are read from LDS 16 bytes at a time, each read feeding four instructions: both operands of a contraction
// enumerate it in the same permuted order.
//
// Operand layout (wave64, lane l, quarter h = l / 16): A (16 x 4): lane holds A[l % 16][h];  B (4 x 16): B[h][l % 16];
//   C (16 x 16): lane holds C[4h + r][l % 16] in register r.
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

// S^T = K.Q^T of NBLK blocks of 16 keys against the wave's 16 queries, in four chains per block: shorter sums, and no
// instruction waits for the one before it.
template <int D, int NBLK>
__device__ __forceinline__ void score_blocks(const uint32_t (&at)[NBLK], const f32x4 (&qf)[D / 16], int swz, int h,
                                             f32x4 (&s)[NBLK])
{
    f32x4 t[NBLK][4];
#pragma unroll
    for (int b = 0; b < NBLK; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) t[b][e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < D / 16; ++kb) {
        f32x4 a[NBLK];
#pragma unroll
        for (int b = 0; b < NBLK; ++b) a[b] = lds_read(at[b] + ((4 * kb + h) ^ swz) * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int b = 0; b < NBLK; ++b)
                t[b][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b][e], qf[kb][e], t[b][e], 0, 0, 0);
    }
#pragma unroll
    for (int b = 0; b < NBLK; ++b) s[b] = (t[b][0] + t[b][1]) + (t[b][2] + t[b][3]);
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
    auto fetch = [&](int t) __attribute__((always_inline)) {
        const uint32_t at = base + t % 2 * TILE;
#pragma unroll
        for (int j = 0; j < Mover::NI; ++j) k_move.issue(at, t * TN, j);
        if constexpr (OUT) {
#pragma unroll
            for (int j = 0; j < Mover::NI; ++j) v_move.issue(at + 2 * TILE, t * TN, j);
        }
    };
    const int n_end = min(L, P + m0 + BM);
    const int n_tiles = (n_end + TN - 1) / TN;
    fetch(0);

    f32x4 qf[KB];  // B operand: element e of block kb is feature 16 kb + 4 h + e of this lane's query
    {
        const float* qrow = q + ((size_t)bh * geo.q_rows + min(m, Tq - 1)) * D;  // rows beyond Tq are not stored
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) qf[kb] = *reinterpret_cast<const f32x4*>(qrow + kb * 16 + h * 4);
    }
    f32x4 o[DB];  // O^T: register r of block db is feature 64 (db / 4) + 4 (4h + r) + db % 4
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Maximum of the scores before scaling: the largest one's exponent is then exactly 0, however large the scores are,
    // where a scaled maximum would leave the rounding of its product.  l_run: this lane's share of the row sum.
    float m_run = kLowest, l_run = 0.f;

    // The compiler learns here that the operand has arrived: the waits it would otherwise put before its uses inside the loop
    // would be waits for the tile in flight.
    wait_loads();
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) asm volatile("" : "+v"(qf[kb]));
    for (int t = 0; t < n_tiles; ++t) {
        wait_loads();
        wait_lds();
        meet();  // tile t has landed, tile t - 1 has been read
        if (t + 1 < n_tiles) fetch(t + 1);
        const int n0 = t * TN + ks * 16;  // the wave's blocks start 16 KS keys apart
        if (n0 > P + mw + 15) continue;   // every key is in the future of the wave's queries
        const uint32_t at = base + t % 2 * TILE;
        uint32_t rows[NBLK];
#pragma unroll
        for (int b = 0; b < NBLK; ++b) rows[b] = at + ((b * KS + ks) * 16 + r16) * (D * 4);
        f32x4 s[NBLK];
        score_blocks<D, NBLK>(rows, qf, r16, h, s);
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
        mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
        mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
        const float m_new = fmaxf(m_run, mx);
        const float corr = exp2f((m_run - m_new) * scale_log2e);
        m_run = m_new;
        float psum = 0.f;
#pragma unroll
        for (int b = 0; b < NBLK; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[b][r] = exp2f((s[b][r] - m_new) * scale_log2e);
                psum += s[b][r];
            }
        l_run = fmaf(l_run, corr, psum);
        if constexpr (OUT) {
            // a tile is summed by itself and then added: the rounding errors of a long chain stay small
            f32x4 ot[DB];
#pragma unroll
            for (int db = 0; db < DB; ++db) ot[db] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int b = 0; b < NBLK; ++b)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int row = (b * KS + ks) * 16 + 4 * h + j;
                    f32x4 a[D / 64];
#pragma unroll
                    for (int c = 0; c < D / 64; ++c)
                        a[c] = lds_read(at + 2 * TILE + row * (D * 4) + ((c * 16 + r16) ^ (row & 15)) * 16);
#pragma unroll
                    for (int db = 0; db < DB; ++db)
                        ot[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[db / 4][db % 4], s[b][j], ot[db], 0, 0, 0);
                }
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 4; ++r) o[db][r] = fmaf(o[db][r], corr, ot[db][r]);
        }
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

    f32x4 kf[KB];  // A operand: element e of block kb is feature 16 kb + 4 h + e of key nw + r16
    {
        const float* krow = k + ((size_t)bh * geo.kv_rows + min(nw + r16, L - 1)) * D;  // keys beyond L are not stored
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) kf[kb] = *reinterpret_cast<const f32x4*>(krow + kb * 16 + h * 4);
    }
    f32x4 col = f32x4{0.f, 0.f, 0.f, 0.f};  // keys nw + 4 h + r
    wait_loads();  // as in the forward pass: no wait for the operand inside the loop
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) asm volatile("" : "+v"(kf[kb]));
    for (int t = 0; t < n_tiles; ++t) {
        const int m0 = m_begin + t * TQ + qg * 16;  // first query of the wave's block
        wait_loads();
        wait_lds();
        meet();  // tile t has landed, tile t - 1 has been read
        const float l2 = l2_next * lse_unit;
        if (t + 1 < n_tiles) fetch(t + 1);
        if (P + m0 + 15 < nw) continue;  // no query of the tile sees a key of this wave
        f32x4 s[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const f32x4 a = lds_read(base + t % 2 * TILE + (qg * 16 + r16) * (D * 4) + ((4 * kb + h) ^ r16) * 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kb][e], a[e], s[e], 0, 0, 0);
        }
        const int m = m0 + r16;
        const int last = m < Tq ? P + m - nw - 4 * h : -1;  // last of the lane's keys that its query sees
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float x = (s[0][r] + s[1][r]) + (s[2][r] + s[3][r]);
            const float p = exp2f(fmaf(x, scale_log2e, -l2));
            col[r] += r <= last ? p : 0.f;
        }
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
    //   B1 T256 38.7 / 32.2 / 32.8   B1 T512 68.7 / 56.6 / 71.5   B1 T1024 143 / 151 / 208   B4 T256 50.3 / 54.1 / 85.7
    //   B1 T2048 496 / 523 / 733   H16 B1 T1024 124 / 95 / 118   H8 B1 T512 64.8 / 49.7 / 38.2
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
    // us of the whole call for 32 / 16 keys per workgroup, 64 queries per workgroup in the forward pass:
    //   B1 T256 38.7 / 37.4   B1 T512 68.7 / 70.9   B1 T1024 143 / 155   B4 T256 50.3 / 58.9   H8 B1 T512 64.8 / 58.8
    //   (64 keys, column pass alone at T1024: 62 against 53)
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
