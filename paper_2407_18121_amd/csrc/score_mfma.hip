// ec_prefill_score / ec_chunk_score, matrix-core path for bf16 inputs (Sec. 3.3, Eq. 1 and I_n = sum_m A_mn).
// Geometry (ScoreGeom): Tq queries over L = P + Tq key rows, query m sees rows n <= P + m; the first-turn
// prompt pass is P = 0.
//
// Two kernels, neither of which stores the T x T matrix:
//   attn_fwd     : one workgroup = 128 queries (4 waves x 32) at a time, key tiles of 64 double-buffered in
//                  LDS.  The score tile is computed TRANSPOSED, S^T = K.Q^T, with v_mfma_f32_32x32x16_bf16: in the
//                  accumulator layout a lane then owns one query (column) and 16 keys (rows), so the row max / row
//                  sum of the online softmax are in-lane reductions plus one exchange between the two half-waves,
//                  the rescale factor is a per-lane scalar, and the fp32 accumulators -- rounded to bf16 -- are
//                  directly the B operand of O^T += V^T.P^T (the contraction index is permuted the same way on both
//                  operands).  V tiles are staged as they lie in memory and transposed by the LDS transpose read on
//                  their way to the registers, so no V^T copy is made.  Emits out (optional) and the row log-sum-exp.
//   colsum       : one workgroup = 128 or 256 keys (4 waves x 32 or 64) whose K fragments stay in registers; query
//                  tiles at or below the diagonal are streamed through LDS, S^T = K.Q^T is recomputed and p =
//                  exp(s - lse_row) is summed per key, over a lane's queries first and over the lanes at the end.
//                  One workgroup owns a column, so there are no atomics and the result is deterministic.
// Causal work is uneven: the last query tile sees every key, the first one only itself.  Where a launch has enough of
// them, a workgroup takes two tiles of a head, the n-th from either end, so that all workgroups do the same work and
// the start of the second tile travels while the first is written out.
//
// MFMA operand layout used throughout (wave64, lane l, half h = l / 32):
//   A (32 x 16): lane holds A[l % 32][8h .. 8h+7]      B (16 x 32): lane holds B[8h .. 8h+7][l % 32]
//   C (32 x 32): lane holds C[8g + 4h + t][l % 32] in register 4g + t, g,t in 0..3
#include <type_traits>

#include "score_route.h"
#include "tile_lds.h"

namespace ec {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef bf16x8 __attribute__((aligned(2))) bf16x8_any;  // in memory: at any element
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;

constexpr int kFwdBN = 64;   // keys per LDS tile
constexpr int kSplitMaxWorkgroups = 256;  // launches of at most this many workgroups divide a workgroup's loop over two wave groups

// Chunk permutations of the LDS tiles (see TileToLds).
template <int D> struct SwizzleRows {  // operand reads of 16 consecutive rows at one chunk number touch every bank once
    static constexpr int kPeriod = 16;  // rows after which it repeats
    static __device__ __forceinline__ int at(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
};
template <int D> struct SwizzleTr {  // four rows at the same 64 bytes (a transposed read's half) land in different banks
    static constexpr int kPeriod = 4;
    static __device__ __forceinline__ int at(int r) { return D == 128 ? (r & 3) << 2 : ((r >> 1) & 1) << 2; }
};

// ------------------------------------------------------------------ forward
// One workgroup = QW * 32 queries (one wave per 32); key tiles of 64, K and V double-buffered in LDS and moved there
// without passing through registers.  Per tile a wave issues 16 matrix instructions for S^T = K.Q^T and 16 for
// O^T += V^T.P^T (D = 128), and per 32 x 32 block 8 max, 16 scale-and-shift, 16 exponential, 16 add and 8 convert
// instructions.  Bound: both pipes, so they have to run at the same time: the scores of tile i + 1 are multiplied while
// tile i is turned into probabilities (phase A), and their row maximum is taken while tile i is multiplied with V
// (phase B).  The issue order inside a phase is fixed by hand: some vector work behind every matrix instruction, LDS
// operands four fragments ahead, the loads of later tiles in between.  Measured at B16 H32 T8192 D128: 9.2 ms before
// (phases one after the other, tiles through registers, 256 queries per workgroup), 8.3 ms with this loop, 8.0 ms with
// PAIR; B8 T2048: 400 -> 340 -> 290 us (the last 40 of them by the coalesced ways in and out).  The clock follows the
// power: 19.2 M cycles at 2.05 GHz became 13.7 M at 1.7 GHz.  256 queries per workgroup took 8.8 ms; six or eight
// fragments ahead changed nothing.
// PAIR: the workgroup takes query tiles n - 1 - i and i of its head, one after the other.
// KSPLIT = 2 (short prompts that give the chip one workgroup per compute unit or less): two groups of QW waves share
// the workgroup's queries and take alternate key tiles, each group moving its own tiles; their (max, sum, O) are merged
// through LDS at the end.  The key loop of a workgroup, which is what bounds such launches, is half as long.
// DIRECT = false: q, k or v does not start on a 16-byte boundary, and tiles pass through registers.
constexpr int kFwdAhead = 4;  // LDS fragments requested ahead of the matrix pipe
template <int D, int QW, int KSPLIT, bool PAIR, bool OUT, bool DIRECT>
__global__ __launch_bounds__(QW * KSPLIT * kWave, 2) void attn_fwd_mfma_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    uint16_t* __restrict__ out, float* __restrict__ lse, ScoreGeom geo, float scale_log2e, int n_qtiles,
    int n_heads, const int32_t* __restrict__ seq_len, int H)
{
    constexpr int BM = QW * 32;   // queries per workgroup
    constexpr int KB = D / 16;    // contraction blocks of Q.K
    constexpr int DB = D / 32;    // 32-row blocks of O^T
    constexpr int NA = 2 * KB;    // matrix instructions of phase A: (kb, 32-key block)
    constexpr int NP = 4 * DB;    // of phase B: (16-key block, db)
    constexpr int EV = 32 / NA;   // elements turned into probabilities per matrix instruction of phase A
    constexpr int TILE = kFwdBN * D;
    using KMove = TileToLds<D, kFwdBN, QW, SwizzleRows<D>, DIRECT>;
    using VMove = TileToLds<D, kFwdBN, QW, SwizzleTr<D>, DIRECT>;
    constexpr int NI = KMove::NI;
    // per group: K of even tiles, K of odd tiles, V of even tiles, V of odd tiles
    __shared__ __align__(16) uint16_t tiles[KSPLIT][4 * TILE];
    __shared__ float stats[KSPLIT == 2 ? 2 * QW * kWave : 1];

    const int lane = threadIdx.x % kWave;
    const int wave_wg = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int grp = wave_wg / QW;   // scalar: which key tiles (tile number mod KSPLIT)
    const int wave = wave_wg % QW;  // scalar: which 32 queries
    const int c32 = lane % 32, h = lane / 32;
    const int n_items = PAIR ? (n_qtiles + 1) / 2 : n_qtiles;  // per head
    const XcdItem item = xcd_item(blockIdx.x, n_items, n_heads);
    if (item.bh < 0) return;
    const int bh = item.bh;
    const int Tq = seq_len ? ragged_rows(seq_len, bh / H, geo.Tq) : geo.Tq, P = geo.P, L = P + Tq;
    const int own_tiles = (Tq + BM - 1) / BM;  // query tiles of this sequence
    const int early = PAIR ? item.tile : n_qtiles - 1 - item.tile;
    int qtile = PAIR ? own_tiles - 1 - early : early;  // the longer tile of a pair first
    if (qtile < (PAIR ? early : 0) || qtile >= own_tiles) return;  // ragged batch: the sequence is shorter (whole workgroup)
    const uint16_t* qh = q + (size_t)bh * geo.q_rows * D;
    // tiles are fetched through descriptors that end at the sequence's last row: rows beyond it arrive as zeros
    const KMove k_move(tile_rsrc(k + (size_t)bh * geo.kv_rows * D, (uint32_t)L * (D * 2)), wave, lane);
    const VMove v_move(tile_rsrc(v + (size_t)bh * geo.kv_rows * D, (uint32_t)L * (D * 2)), wave, lane);
    constexpr int K0 = 0, K1 = TILE, V0 = 2 * TILE, V1 = 3 * TILE;  // elements
    const uint32_t mine_at = lds_address(tiles[grp]);
    auto row_of = [&](int i) { return (i * KSPLIT + grp) * kFwdBN; };  // first key of the group's i-th tile
    auto move_k = [&](int at, int i) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NI; ++j) k_move.issue(mine_at + at * 2, row_of(i), j);
    };
    auto move_v = [&](int at, int i) __attribute__((always_inline)) {
        if constexpr (OUT) {
#pragma unroll
            for (int j = 0; j < NI; ++j) v_move.issue(mine_at + at * 2, row_of(i), j);
        }
    };
    // A wave's 32 query rows travel through the place of its own share of the V tiles (16 rows each), so that no other wave
    // has to be waited for, and K of the first tile goes with them.
    const uint32_t q_at = mine_at + V0 * 2 + wave * (16 * D * 2);
    const TileToLds<D, 32, 1, SwizzleRows<D>, DIRECT> q_move(tile_rsrc(qh, (uint32_t)Tq * (D * 2)), 0, lane);
    auto first_loads = [&](int mw) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < q_move.NI; ++j)
            q_move.issue(q_at + (j < q_move.NI / 2 ? 0 : (TILE - 16 * D) * 2), mw, j);
        move_k(K0, 0);
    };
    first_loads(qtile * BM + wave * 32);

    // A operand of S^T: row i of a 32-key block is key swap23(i) (bits 2 and 3 of i exchanged), i.e. key
    // 16(i/16) + 8((i/4)%2) + 4((i/8)%2) + i%4.  In the accumulator layout (register 4g+t of half h = row 8g+4h+t)
    // registers 8G..8G+7 of a lane then hold the 8 CONSECUTIVE keys 16G + 8h .. +7: the P fragment of a P.V matrix
    // instruction is a run of registers.
    bf16x8 qf[KB];  // B operand: this lane's query
    const int krow = (c32 & ~12) | ((c32 & 4) << 1) | ((c32 & 8) >> 1);
    uint32_t k_at[KB];  // byte address of this lane's 16 bytes of contraction block kb in tile K0
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
        k_at[kb] = one_register(mine_at + krow * (D * 2) + ((2 * kb + h) ^ SwizzleRows<D>::at(krow)) * 16);
    auto k_frag = [&](int kt, int f) __attribute__((always_inline)) {  // f = 2 kb + 32-key block
        return *(lds_bf16x8*)(uintptr_t)(k_at[f / 2] + (kt + f % 2 * 32 * D) * 2);
    };
    // V rows sit in LDS key-major; the operand of O^T += V^T.P^T needs, per lane, 8 keys of ONE feature.
    // ds_read_b64_tr_b16 does that transposition on the way out of LDS: in a group of 16 lanes, lane r points at 4
    // consecutive features of key r/4 (features 4(r%4).. of the group's 16), and lane j receives feature j of keys
    // 0..3.  Two such reads (keys +0..3, +4..7) make one 8-key fragment.  Groups 0,1 (half h = 0) take keys 0..7 of a
    // 16-key contraction block, groups 2,3 keys 8..15.
    uint32_t v_at[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) {
        const int row = h * 8 + (lane % 16) / 4, chunk = db * 4 + (lane / 16) % 2 * 2 + lane % 4 / 2;
        v_at[db] = one_register(mine_at + row * (D * 2) + (chunk ^ SwizzleTr<D>::at(row)) * 16 + lane % 2 * 8);
    }
    auto v_frag = [&](int vt, int g) __attribute__((always_inline)) {  // g = DB * (16-key block) + db
        const uint32_t src = v_at[g % DB] + (vt + g / DB * 16 * D) * 2;
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(uintptr_t)src);
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(uintptr_t)(src + 4 * D * 2));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };

    for (;;) {  // one query tile after the other
        const int m0 = qtile * BM;
        const int mw = m0 + wave * 32;  // first query of this wave
        const int m = mw + c32;         // this lane's query
        f32x16 o[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
        // m_run: running maximum of the scaled scores, base 2, of every tile whose scores have been computed (one tile
        // ahead of o and l_run, which are already scaled to it).  A group that does not start at key 0 can meet a tile in
        // which a query sees no key at all, and any tile can hold nothing but scores of -inf.  l_run: this half-wave's share
        // of the row sum.
        float m_run = kLowest, l_run = 0.f;
        f32x16 sA[2], sB[2];
        bf16x8 pf[4];

        auto mask = [&](f32x16 (&s)[2], int n0) __attribute__((always_inline)) {
            if (n0 + kFwdBN - 1 > P + mw || n0 + kFwdBN > L) {  // tile with keys behind one of the wave's queries
                const int last = min(P + m, L - 1) - n0 - h * 8;
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (nb * 32 + (r / 8) * 16 + (r % 8) > last) s[nb][r] = -INFINITY;
            }
        };
        // the other half-wave holds the other 32 keys of each query: exchange through the lane-swap instruction (a shuffle
        // would go through LDS and its latency sits on the critical path)
        auto raise_max = [&](float mx) __attribute__((always_inline)) {
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * scale_log2e;
            const float m_new = fmaxf(m_run, mx);
            const float corr = __builtin_amdgcn_exp2f(m_run - m_new);  // 0 from kLowest to a score
            const bool grew = m_new > m_run;
            m_run = m_new;
            l_run *= corr;
            if (OUT && __any(grew)) {  // wave-uniform
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[db][r] *= corr;
            }
        };
        auto pin = [&](bf16x8 (&p)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                u32x4 w = __builtin_bit_cast(u32x4, p[kk]);
                asm volatile("" : "+v"(w));
                p[kk] = __builtin_bit_cast(bf16x8, w);
            }
        };
        // Phase A: probabilities of the tile in s (into pf and the row sum) beside sn = K.Q^T of the next one; extra(f) is
        // issued behind the f-th matrix instruction.
        auto phase_a = [&](auto next, f32x16 (&s)[2], f32x16 (&sn)[2], int kt, auto&& extra) __attribute__((always_inline)) {
            // of the SIMD's two waves the one with the vector work issues first, the other's matrix instructions are long
            // enough to wait (B16 H32 T8192 with the column pass: 12.00 -> 11.89 ms; the other way round 12.15)
            __builtin_amdgcn_s_setprio(1);
            bf16x8 ka[NA];
            if constexpr (next.value) {
#pragma unroll
                for (int f = 0; f < kFwdAhead; ++f) ka[f] = k_frag(kt, f);
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) sn[nb][r] = 0.f;
                __builtin_amdgcn_sched_barrier(0);
            }
            float x[EV], y[EV], ps[2] = {0.f, 0.f};
#pragma unroll
            for (int f = 0; f < NA + 2; ++f) {
                if constexpr (next.value)
                    if (f < NA) {
                        sn[f % 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[f], qf[f / 2], sn[f % 2], 0, 0, 0);
                        if (f + kFwdAhead < NA) ka[f + kFwdAhead] = k_frag(kt, f + kFwdAhead);
                    }
                extra(f);
                if (f >= 2) {  // third stage of the elements of two instructions ago: sum and round
#pragma unroll
                    for (int e = 0; e < EV; ++e) {
                        const int el = (f - 2) * EV + e;
                        ps[e % 2] += y[e];
                        pf[el / 8][el % 8] = (__bf16)y[e];
                    }
                }
                if (f >= 1 && f <= NA) {
#pragma unroll
                    for (int e = 0; e < EV; ++e) y[e] = __builtin_amdgcn_exp2f(x[e]);
                }
                if (f < NA) {
#pragma unroll
                    for (int e = 0; e < EV; ++e) {
                        const int el = f * EV + e;
                        x[e] = fmaf(s[el / 16][el % 16], scale_log2e, -m_run);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            l_run += ps[0] + ps[1];
            asm volatile("" : "+v"(l_run));
            pin(pf);  // sum and probabilities are formed here, beside the matrix instructions, not where they are used
        };
        // Phase B: O^T += V^T.P^T of the tile in pf beside the row maximum of the scores in sn.
        auto phase_b = [&](auto next, f32x16 (&sn)[2], int vt) __attribute__((always_inline)) {
            __builtin_amdgcn_s_setprio(0);
            float mx[2] = {-INFINITY, -INFINITY};
            bf16x8 va[NP];
            if constexpr (OUT) {
#pragma unroll
                for (int g = 0; g < kFwdAhead; ++g) va[g] = v_frag(vt, g);
                __builtin_amdgcn_sched_barrier(0);
            }
            constexpr int MV = 32 / NP;
#pragma unroll
            for (int g = 0; g < NP; ++g) {
                if constexpr (OUT) {
                    o[g % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[g], pf[g / DB], o[g % DB], 0, 0, 0);
                    if (g + kFwdAhead < NP) va[g + kFwdAhead] = v_frag(vt, g + kFwdAhead);
                }
                if constexpr (next.value) {
#pragma unroll
                    for (int e = 0; e < MV; e += 2) {
                        const int el = g * MV + e;
                        mx[(e / 2 + g) % 2] = fmaxf(fmaxf(mx[(e / 2 + g) % 2], sn[el / 16][el % 16]), sn[el / 16][el % 16 + 1]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (next.value) raise_max(fmaxf(mx[0], mx[1]));
        };

        const int n_end = min(L, P + m0 + BM);  // the workgroup's last query sees rows up to P + m0 + BM - 1
        const int n_iter = ((n_end + kFwdBN - 1) / kFwdBN + KSPLIT - 1) / KSPLIT;  // same for both groups: one barrier each
        // tiles of this wave: the group's tiles with a key that one of its queries sees
        const int seen = (mw < Tq) ? (min(P + mw + 32, n_end) + kFwdBN - 1) / kFwdBN : 0;
        const int count = max(seen - grp + KSPLIT - 1, 0) / KSPLIT;

        wait_loads();  // this wave's queries and its share of the first K tile
        {
            const int row = anew(c32);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
                qf[kb] = *(lds_bf16x8*)(uintptr_t)(q_at + row / 16 * (TILE * 2) + row % 16 * (D * 2) +
                                                   ((2 * kb + h) ^ SwizzleRows<D>::at(row)) * 16);
        }
        wait_lds();  // their place is free
        move_v(V0, 0);
        move_k(K1, 1);
        meet();
        if (count > 0) {  // scores of the first tile
            bf16x8 ka[NA];
#pragma unroll
            for (int f = 0; f < NA; ++f) ka[f] = k_frag(K0, f);
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r) sA[nb][r] = 0.f;
#pragma unroll
            for (int f = 0; f < NA; ++f) sA[f % 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[f], qf[f / 2], sA[f % 2], 0, 0, 0);
            mask(sA, row_of(0));
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(fmaxf(mx, sA[0][r]), sA[1][r]);
            raise_max(mx);
        }
        // One tile with a successor: K of tile i + 1 and V of tile i have landed; K of tile i + 2 goes where K of tile i was, V
        // of tile i + 1 where V of tile i - 1 was, both read for the last time before the barrier.
        auto body = [&](int i, f32x16 (&s)[2], f32x16 (&sn)[2], int k_old, int k_next, int v_cur, int v_next) __attribute__((always_inline)) {
            tile_barrier();
            const int k_row = (i + 2 < n_iter) ? row_of(i + 2) : L;  // L: nothing is fetched
            const int v_row = row_of(i + 1);
            phase_a(std::true_type{}, s, sn, k_next, [&](int f) __attribute__((always_inline)) {
                constexpr int EVERY = NA / (2 * NI);
                static_assert(EVERY >= 1, "a phase has room for its loads");
                if (f < NA && f % EVERY == 0) {
                    if (f / EVERY < NI)
                        k_move.begin(mine_at + k_old * 2, k_row, f / EVERY);
                    else if (OUT)
                        v_move.begin(mine_at + v_next * 2, v_row, f / EVERY - NI);
                }
            });
#pragma unroll
            for (int j = 0; j < NI; ++j) k_move.finish(mine_at + k_old * 2, j);
            mask(sn, row_of(i + 1));
            phase_b(std::true_type{}, sn, v_cur);
            if constexpr (OUT) {
#pragma unroll
                for (int j = 0; j < NI; ++j) v_move.finish(mine_at + v_next * 2, j);
            }
        };
        int i = 0;
        for (; i + 2 < count; i += 2) {
            body(i, sA, sB, K0, K1, V0, V1);
            body(i + 1, sB, sA, K1, K0, V1, V0);
        }
        const bool odd = i + 1 < count;
        if (odd) {
            body(i, sA, sB, K0, K1, V0, V1);
            ++i;
        }
        // the wave's last tile, then nothing but its share of the loads that other waves still need
        for (bool work = i < count; i < n_iter; ++i, work = false) {
            tile_barrier();
            const bool even = i % 2 == 0;
            if (i + 2 < n_iter) move_k(even ? K0 : K1, i + 2);
            if (i + 1 < n_iter) move_v(even ? V1 : V0, i + 1);
            if (work) {
                if (odd) {
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) sA[nb] = sB[nb];
                }
                phase_a(std::false_type{}, sA, sB, K0, [](int) {});
                phase_b(std::false_type{}, sB, even ? V0 : V1);
            }
        }

        if (KSPLIT == 2) {
            // group 1 hands its state over through group 0's tiles; word j of thread t sits at j * THREADS + t: consecutive
            // lanes, consecutive words
            constexpr int THREADS = QW * kWave;
            static_assert(KSPLIT == 1 || !OUT || sizeof(tiles) >= sizeof(float) * THREADS * DB * 16, "hand-over area");
            float* xch = reinterpret_cast<float*>(&tiles[0][0]);
            const int tid = threadIdx.x % THREADS;
            tile_barrier();
            if (grp == 1) {
                stats[tid] = m_run;
                stats[THREADS + tid] = l_run;
                if constexpr (OUT) {
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            xch[(db * 16 + r) * THREADS + tid] = o[db][r];
                }
            }
            __syncthreads();
            if (grp == 1) return;
            const float m1 = stats[tid], l1 = stats[THREADS + tid];
            const float m_all = fmaxf(m_run, m1);
            const float f0 = __builtin_amdgcn_exp2f(m_run - m_all), f1 = __builtin_amdgcn_exp2f(m1 - m_all);
            l_run = l_run * f0 + l1 * f1;
            m_run = m_all;
            if constexpr (OUT) {
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        o[db][r] = o[db][r] * f0 + xch[(db * 16 + r) * THREADS + tid] * f1;
            }
        }
        const int next_tile = PAIR ? own_tiles - 1 - qtile : qtile;
        const bool more = PAIR && next_tile < qtile;
        if (more) {  // what the second tile starts with travels while the first one is written out
            tile_barrier();
            first_loads(next_tile * BM + wave * 32);
        }
        const int el = anew(lane), ec = el % 32, eh = el / 32;  // lane, row and half of the way out
        const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
        if (mw + ec < Tq && eh == 0) lse[(size_t)bh * geo.q_rows + mw + ec] = (m_run + log2f(l_tot)) * kLn2;
        if constexpr (OUT) {
            // The accumulators hold 8-byte pieces of 32 rows per register pair.  Half a row at a time they are turned through
            // this wave's share of tile K1 (every wave has read K for the last time), so that a store instruction writes
            // whole 128-byte (D = 64: 64-byte) stretches.
            constexpr int HC = D / 16;        // 16-byte chunks in half a row
            constexpr int RPS = kWave / HC;   // rows per store instruction
            const float inv = 1.f / l_tot;
            const uint32_t stage = lds_address(tiles[KSPLIT - 1]) + K1 * 2 + wave * (16 * D * 2);
            auto place = [&](int row, int chunk) { return row * (HC * 16) + (chunk ^ (D == 128 ? row & 7 : (row >> 2) & 3)) * 16; };
#pragma unroll
            for (int half = 0; half < 2; ++half) {
#pragma unroll
                for (int d2 = 0; d2 < DB / 2; ++d2)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        bf16x4 y;
#pragma unroll
                        for (int t = 0; t < 4; ++t) y[t] = (__bf16)(o[half * (DB / 2) + d2][g * 4 + t] * inv);
                        *(lds_bf16x4*)(uintptr_t)(stage + place(ec, d2 * 4 + g) + eh * 8) = y;
                    }
#pragma unroll
                for (int j = 0; j < 32 / RPS; ++j) {
                    const int row = j * RPS + el / HC;
                    const bf16x8 y = *(lds_bf16x8*)(uintptr_t)(stage + place(row, el % HC));
                    if (mw + row < Tq)
                        *reinterpret_cast<bf16x8_any*>(out + ((size_t)bh * geo.q_rows + mw + row) * D + half * (D / 2) + el % HC * 8) = y;
                }
            }
        }
        if (!more) return;
        qtile = next_tile;
    }
}

// ------------------------------------------------------------------ column mass
// One workgroup owns KW * 32 * NB keys of a head; KW * QG waves.  A wave keeps the K fragments of its 32 * NB keys in
// registers and takes every QG-th step of 32 queries; the Q rows of QT queries at a time are moved straight into
// LDS (two tiles, one being read while the other lands).  S^T = K.Q^T, so a lane owns ONE query: its log-sum-exp is
// a single value per step, and p = exp2(s c - lse) is added to the lane's own partial column sums, 16 per block of
// 32 keys, which are reduced over the lanes once at the end.  No workgroup shares a column: deterministic.
// Bound: vector issue and matrix pipe together.  Per 32 x 32 block 8 matrix instructions (256 clocks) stand against 16
// scale-and-shift, 16 exponential (two issue slots each) and 16 add instructions (256 clocks): the exponentials of a
// step are issued between the matrix instructions of the next one (its score block stays pending for one step).  Q
// fragments are reloaded for the next step right after their last use, so no LDS latency is exposed.  Measured at
// B16 H32 T8192 D128: 4.4 ms before (compiler's order, a lane per key), 4.35 ms in this order, 4.1 ms with PAIR, 3.9 ms
// without waits for memory inside the loop and with the second key tile's start under the end of the first; B8 T2048:
// 200 -> 186 -> 160 us.
// PAIR: the workgroup takes key tiles i and n - 1 - i of its head, one after the other.
// QG = 2 (launches of one workgroup per compute unit or less): twice the waves on the same keys.
template <int D, int NB, int KW, int QG, int QT, bool PAIR, bool DIRECT>
__global__ __launch_bounds__(KW * QG * kWave, 2) void colsum_mfma_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const float* __restrict__ lse,
    float* __restrict__ head_imp, ScoreGeom geo, float scale_log2e, int n_ktiles, int n_heads,
    const int32_t* __restrict__ seq_len, int H)
{
    constexpr int KB = D / 16;
    constexpr int WAVES = KW * QG;
    constexpr int KEYS_W = 32 * NB;     // keys per wave
    constexpr int BN = KW * KEYS_W;     // keys per workgroup
    constexpr int SPT = QT / 32 / QG;  // steps of one wave per tile
    constexpr int kNoStep = 0x3fffff00;  // "first query" of a block that holds no step: behind every sequence
    // The keys of a wave, a row per lane, are read from LDS: straight from memory each of a load's 64 rows would be a request of its
    // own, 64 clocks of the compute unit's cache instead of 16.  They come in where the second query tile goes afterwards (one
    // wave group) or have a place of their own (two).  64 keys per wave would need twice the place, which is not there.  us of the
    // whole call before / now: B1 H32 D128 T1000 36.9 / 35.7, T300 18.8 / 18.1, B16 H40 T512 136.9 / 134.5, B4 H32 T1100 98.1 /
    // 98.1, D64 B2 H40 T700 28.4 / 27.9; two groups at D 64, whose rows are half as long: B1 H32 T1000 28.4 / 28.8, so not there.
    constexpr bool STAGED = NB == 1 && DIRECT && (D == 128 || QG == 1);
    constexpr int kKeysAt = QG == 1 ? QT * D : 2 * QT * D;  // element
    static_assert(!STAGED || !PAIR, "one key tile");
    __shared__ __align__(16) uint16_t qs[STAGED ? kKeysAt + BN * D : 2 * QT * D];  // two tiles
    __shared__ __align__(16) float ls[2 * QT];
    __shared__ __align__(16) float red[WAVES][4][KEYS_W / 2];  // [wave][half-wave, 16-lane row][16 sums per 32 keys]

    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int qg = wave / KW, kw = wave % KW;
    const int c32 = lane % 32, h = lane / 32;
    const int n_items = PAIR ? (n_ktiles + 1) / 2 : n_ktiles;  // per head
    const XcdItem item = xcd_item(blockIdx.x, n_items, n_heads);
    if (item.bh < 0) return;
    const int bh = item.bh;
    const int Tq = seq_len ? ragged_rows(seq_len, bh / H, geo.Tq) : geo.Tq, P = geo.P, L = P + Tq;
    const int own_tiles = (L + BN - 1) / BN;  // key tiles of this sequence
    int ktile = item.tile;                    // low tiles have the most queries: first
    if (ktile >= (PAIR ? (own_tiles + 1) / 2 : own_tiles)) return;  // ragged batch: the sequence is shorter (whole workgroup)
    const uint16_t* qh = q + (size_t)bh * geo.q_rows * D;
    const uint16_t* kh = k + (size_t)bh * geo.kv_rows * D;
    const u32x4 q_rsrc = tile_rsrc(qh, (uint32_t)Tq * (D * 2));
    const u32x4 l_rsrc = tile_rsrc(lse + (size_t)bh * geo.q_rows, (uint32_t)Tq * 4);

    // Single key tiles take their query tiles from the first one with a query that sees key n0 (m sees n <= P + m) upwards;
    // pairs from the sequence's last one down, so that all workgroups of a head start at the same queries and the first
    // two query tiles of the second key tile can travel before it begins.
    const int m_last = (Tq - 1) / QT * QT;
    auto first_seen = [&](int tile) __attribute__((always_inline)) { return max(tile * BN - P, 0) / QT * QT; };
    constexpr int DIR = PAIR ? -1 : 1;
    using Mover = TileToLds<D, QT, WAVES, SwizzleRows<D>, DIRECT>;
    const uint32_t qs_at = lds_address(qs), ls_at = lds_address(ls);
    auto fetch_lse = [&](int buf, int m) __attribute__((always_inline)) {
        if (wave < QT / kWave)
            load_lds_4(l_rsrc, ls_at + (buf * QT + wave * kWave) * 4, (m + wave * kWave + anew(lane)) * 4);
    };
    auto first_tile = [&](int t) __attribute__((always_inline)) {
        const Mover mover(q_rsrc, wave, anew(lane));
        const int m = PAIR ? max(m_last - t * QT, 0) : first_seen(ktile) + t * QT;
#pragma unroll
        for (int j = 0; j < Mover::NI; ++j) mover.issue(qs_at + t * QT * D * 2, m, j);
        fetch_lse(t, m);
    };
    if constexpr (STAGED) {
        const TileToLds<D, BN, WAVES, SwizzleRows<D>> k_move(tile_rsrc(kh, (uint32_t)L * (D * 2)), wave, anew(lane));
#pragma unroll
        for (int j = 0; j < k_move.NI; ++j) k_move.issue(qs_at + kKeysAt * 2, ktile * BN, j);
    }
    first_tile(0);
    if (!STAGED || QG == 2) first_tile(1);
    bf16x8 kf[NB][KB];
    auto load_keys = [&](int tile) __attribute__((always_inline)) {
        const int lk = anew(lane);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int n = min(tile * BN + kw * KEYS_W + nb * 32 + lk % 32, L - 1);  // sums of keys beyond L are not stored
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
                kf[nb][kb] = *reinterpret_cast<const bf16x8_any*>(kh + (size_t)n * D + kb * 16 + lk / 32 * 8);
        }
    };
    if constexpr (!STAGED) load_keys(ktile);

    for (;;) {  // one key tile after the other
        const int n0 = ktile * BN;
        const int nw = n0 + kw * KEYS_W;  // first key of this wave
        const int m_begin = first_seen(ktile);
        const int n_tiles = (m_last - m_begin) / QT + 1;
        const int next_tile = PAIR ? own_tiles - 1 - ktile : ktile;
        const bool more = PAIR && next_tile > ktile;
        const int m_first = PAIR ? m_last : m_begin;
        const Mover mover(q_rsrc, wave, anew(lane));
        // What is fetched as tile t: behind the last tile of a pair's first half the first two of the second half, behind
        // the very last rows behind the sequence, for which nothing is read.
        auto first_query = [&](int buf, int t) __attribute__((always_inline)) {
            if (!PAIR || t < n_tiles) return m_first + DIR * t * QT;
            return more ? max(m_last - buf * QT, 0) : m_last + QT;
        };

        // A and B take turns: one is being computed while the other is pending
        f32x16 sA[NB], sB[NB];
        float lA = -INFINITY, lB = -INFINITY;  // minus the log-sum-exp of the lane's query, base 2; -inf: no mass
        int mA = kNoStep, mB = kNoStep;  // first query of the step in A, B
        f32x16 col[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) sA[nb][r] = sB[nb][r] = col[nb][r] = 0.f;

        // this lane's address inside a step: row c32, chunk 2 kb + h, swizzled
        const int lq = anew(lane), swz = SwizzleRows<D>::at(lq % 32);
        uint32_t q_at[KB];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) q_at[kb] = one_register(qs_at + (qg * 32 + lq % 32) * (D * 2) + ((2 * kb + lq / 32) ^ swz) * 16);
        auto frag = [&](int u, int kb) __attribute__((always_inline)) {  // u: step of 32 queries inside the two tiles
            return *(lds_bf16x8*)(uintptr_t)(q_at[kb] + u * 32 * D * 2);
        };
        // pairs that the mask takes out (keys behind the query, queries behind the end): score -inf, mass zero.  A
        // log-sum-exp that would turn -inf into a number other than -inf (NaN, or that of a row of -inf) goes into the scores
        // of the keys that the query sees, so that it does not reach the others.
        auto mask = [&](f32x16 (&sp)[NB], float& lp, int mp) __attribute__((always_inline)) {
            if (!(lp < INFINITY)) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) sp[nb][r] += lp;
                lp = 0.f;
            }
            const int last = (mp + c32 < Tq) ? P + mp + c32 - nw - h * 4 : -1;  // last key this lane's query sees
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (nb * 32 + (r / 4) * 8 + (r % 4) > last) sp[nb][r] = -INFINITY;
        };
        bf16x8 qa[KB];
        bool loaded = false;  // qa, ln hold this wave's next step
        float ln = 0.f;  // log-sum-exp of the step in qa
        // One step: S^T of the step held in qa into sn while the pending block (sp, lp) is turned into mass; qa is
        // refilled with step u_next of tile qs_next.
        auto step = [&](f32x16 (&sn)[NB], float& l_n, int& m_n, int mq, f32x16 (&sp)[NB], float& lp, int& mp,
                        int u_next, auto&& extra) __attribute__((always_inline)) {
            l_n = -ln * kLog2e;
            m_n = mq;
            ln = ls[(u_next + qg) * 32 + c32];
            if (P + mp < nw + KEYS_W - 1 || mp + 32 > Tq) mask(sp, lp, mp);  // some pair of the pending step is masked
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r) sn[nb][r] = 0.f;
            // Issue order, fixed by hand: per matrix instruction EV elements are scaled, the EV before them exponentiated and
            // the EV before those added, so that no instruction waits for the one in front of it.
            constexpr int EV = 16 / KB;
            constexpr int NM = NB * KB;
            float x[EV], y[EV];
#pragma unroll
            for (int i = 0; i < NM + 2; ++i) {
                if (i < NM) {
                    const int kb = i / NB, nb = i % NB;
                    sn[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[nb][kb], qa[kb], sn[nb], 0, 0, 0);
                    if (nb == NB - 1) qa[kb] = frag(u_next, kb);
                    extra(i);
                }
                if (i >= 2) {
#pragma unroll
                    for (int e = 0; e < EV; ++e) {
                        const int el = (i - 2) * EV + e;
                        col[el / 16][el % 16] += y[e];
                    }
                }
                if (i >= 1 && i <= NM) {
#pragma unroll
                    for (int e = 0; e < EV; ++e) y[e] = __builtin_amdgcn_exp2f(x[e]);
                }
                if (i < NM) {
#pragma unroll
                    for (int e = 0; e < EV; ++e) {
                        const int el = i * EV + e;
                        x[e] = fmaf(sp[el / 16][el % 16], scale_log2e, lp);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) asm volatile("" : "+v"(col[nb]));  // added here, beside the matrix instructions
            lp = -INFINITY;  // retired
            mp = kNoStep;
        };

        const int mq_first = nw - P - 31;  // the last query of a step has to see the wave's first key
        static_assert(SPT % 2 == 0, "A and B alternate through a tile");
        constexpr auto nothing = [](int) {};
        auto tile = [&](int buf, int t) __attribute__((always_inline)) {
            const int m0 = m_first + DIR * t * QT + qg * 32, m_refill = first_query(buf, t + 2);
            const int u0 = buf * (QT / 32);  // steps are counted from the wave's first one
#pragma unroll
            for (int i = 0; i < SPT; ++i) {
                const int at = PAIR ? SPT - 1 - i : i, u = u0 + at * QG, mq = m0 + at * QG * 32;
                const bool last = i == SPT - 1;
                const bool active = mq >= mq_first && mq < Tq;  // some query of the step sees a key of this wave (wave-uniform)
                if (active && !loaded) {  // its first step: nothing has been loaded ahead
#pragma unroll
                    for (int kb = 0; kb < KB; ++kb) qa[kb] = frag(u, kb);
                    ln = ls[(u + qg) * 32 + c32];
                    loaded = true;
                }
                if (last) {
                    tile_barrier();  // the other tile has landed, and every wave has read this one for the last time
                    fetch_lse(buf, m_refill);
                }
                if (!active) {
                    if (last) {
#pragma unroll
                        for (int j = 0; j < Mover::NI; ++j) mover.issue(qs_at + buf * QT * D * 2, m_refill, j);
                    }
                    continue;
                }
                if (i % 2 == 0)
                    step(sA, lA, mA, mq, sB, lB, mB, u + DIR * QG, nothing);
                else if (!last)
                    step(sB, lB, mB, mq, sA, lA, mA, u + DIR * QG, nothing);
                else {  // the tile after the next one takes this one's place, its loads spread over the matrix instructions
                    step(sB, lB, mB, mq, sA, lA, mA, (buf ^ 1) * (QT / 32) + (PAIR ? (SPT - 1) * QG : 0), [&](int g) __attribute__((always_inline)) {
                        constexpr int EVERY = NB * KB / Mover::NI;
                        if (g % EVERY == 0) mover.begin(qs_at + buf * QT * D * 2, m_refill, g / EVERY);
                    });
#pragma unroll
                    for (int j = 0; j < Mover::NI; ++j) mover.finish(qs_at + buf * QT * D * 2, j);
                }
            }
        };
        tile_barrier();
        if constexpr (STAGED) {
            const int row = kw * 32 + lq % 32;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
                kf[0][kb] = *(lds_bf16x8*)(uintptr_t)(qs_at + kKeysAt * 2 + row * (D * 2) + ((2 * kb + lq / 32) ^ swz) * 16);
            if constexpr (QG == 1) {
                wait_lds();
                meet();  // the keys have been read: their place is free
                first_tile(1);
            }
        }
        // The compiler learns here that the keys have arrived: the waits it would otherwise put before their uses inside the
        // loop would be waits for the tiles in flight (4.13 -> 3.86 ms at T8192, 56 -> 53 us with 32 keys per wave).  The few
        // steps of a two-group launch are 0.6 us slower without them (B1 T1024 13.5 / 14.1 us).
        if constexpr (QG == 1) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) asm volatile("" : "+v"(kf[nb][kb]));
        }
        for (int t = 0; t < n_tiles; t += 2) {
            tile(0, t);
            if (t + 1 < n_tiles) tile(1, t + 1);
        }

        if (more) load_keys(next_tile);  // travels while this tile's sums are brought together
        // at most one of the two is still pending
        auto retire = [&](f32x16 (&sp)[NB], float lp, int mp) __attribute__((always_inline)) {
            mask(sp, lp, mp);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r) col[nb][r] += __builtin_amdgcn_exp2f(fmaf(sp[nb][r], scale_log2e, lp));
        };
        if (mA != kNoStep)
            retire(sA, lA, mA);
        else if (mB != kNoStep)
            retire(sB, lB, mB);
        const int el = anew(lane);
        // over the 16 lanes of a row by DPP, over the rows and the query groups through LDS, always in the same order
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float4 y;
                y.x = group_sum<16>(col[nb][4 * g]);
                y.y = group_sum<16>(col[nb][4 * g + 1]);
                y.z = group_sum<16>(col[nb][4 * g + 2]);
                y.w = group_sum<16>(col[nb][4 * g + 3]);
                if (el % 16 == 0) *reinterpret_cast<float4*>(&red[wave][el / 16][nb * 16 + 4 * g]) = y;
            }
        __syncthreads();
        const int key = anew(threadIdx.x);
        if (key < BN && n0 + key < L) {
            const int w = key / KEYS_W, j = key % 32, slot = (key % KEYS_W) / 32 * 16 + j / 8 * 4 + j % 4, hh = (j / 4) % 2;
            float sum = 0.f;
#pragma unroll
            for (int g = 0; g < QG; ++g) sum += red[g * KW + w][2 * hh][slot] + red[g * KW + w][2 * hh + 1][slot];
            head_imp[(size_t)bh * geo.imp_rows + n0 + key] = sum;
        }
        if (!more) return;
        ktile = next_tile;
        __syncthreads();  // the sums have been read
    }
}

template <int D>
static int launch_mfma(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* out, float* lse,
                       float* head_imp, int B, int H, ScoreGeom geo, const int32_t* seq_len, float scale, bool direct,
                       hipStream_t stream)
{
    const float sl = scale * kLog2e;
    const int Tq = geo.Tq, L = geo.L;
    const int BH = B * H;
    const int qt128 = (Tq + 127) / 128;
#define EC_FWD(KS_, PAIR_, DIRECT_)                                                                                  \
    do {                                                                                                             \
        const dim3 grid(xcd_grid((PAIR_ ? (qt128 + 1) / 2 : qt128) * BH)), block(4 * KS_ * kWave);                    \
        if (out != nullptr)                                                                                          \
            hipLaunchKernelGGL((attn_fwd_mfma_kernel<D, 4, KS_, PAIR_, true, DIRECT_>), grid, block, 0, stream, q, k, \
                               v, out, lse, geo, sl, qt128, BH, seq_len, H);                                         \
        else                                                                                                         \
            hipLaunchKernelGGL((attn_fwd_mfma_kernel<D, 4, KS_, PAIR_, false, DIRECT_>), grid, block, 0, stream, q,   \
                               k, v, out, lse, geo, sl, qt128, BH, seq_len, H);                                      \
    } while (0)
    // Launch shapes of the forward pass, us (pairs / single tiles / two wave groups per tile), H 32, D 128:
    //   B1 T512 18.2 / 13.7 / 14.7    B1 T1024 26.4 / 22.6 / 22.2   B1 T2048 46.5 / 60.1 / 61.8   B2 T1024 29.0 / 33.3 / 39.9
    //   B4 T1024 47.0 / 63.4 / 75.9   B8 T1536 180 / 204 / 234      B2 T8192 1068 / 1112 / 1172   B16 H40 T256 35.9 / 33.2 / 49.1
    //   H8 B1: T1024 25.3 / 20.3 / 19.7   T2048 39.3 / 34.6 / 32.8   T4096 70.0 / 65.4 / 61.7
    // Pairs by the rule of score_route.h; below it two groups per tile once the key loop is long enough to pay for merging
    // them.
    // Off the 16-byte grid one shape serves all sizes: the loads themselves, two requests for every 128 bytes, set the pace
    // (whole call on / off the grid, B1 H32 T1024 D128 37 / 64 us, B8 T2048 503 / 831 us, B4 T8192 3.05 / 4.11 ms; in
    // pairs the latter two take 814 us and 4.13 ms).
    if (!direct)
        EC_FWD(1, false, false);
    else if (pair_query_tiles(D, qt128, BH, Tq, geo.P))
        EC_FWD(1, true, true);
    else if ((long long)qt128 * BH <= kSplitMaxWorkgroups && L >= 1024)
        EC_FWD(2, false, true);
    else
        EC_FWD(1, false, true);
#undef EC_FWD
    int rc = status_from_hip(hipGetLastError());
    if (rc != EC_OK) return rc;
    const int kt256 = (L + 255) / 256, kt128 = (L + 127) / 128;
#define EC_COLSUM(NB_, QG_, QT_, PAIR_, DIRECT_)                                                                     \
    do {                                                                                                             \
        const int kt = (L + 128 * NB_ - 1) / (128 * NB_);                                                            \
        hipLaunchKernelGGL((colsum_mfma_kernel<D, NB_, 4, QG_, QT_, PAIR_, DIRECT_>),                                \
                           dim3(xcd_grid((PAIR_ ? (kt + 1) / 2 : kt) * BH)), dim3(4 * QG_ * kWave), 0, stream, q, k, \
                           lse, head_imp, geo, sl, kt, BH, seq_len, H);                                              \
    } while (0)
    // Launch shapes of the column pass, us (64 keys per wave in pairs / 32 keys per wave / 32 keys, two query groups):
    //   H32 D128: B1 T512 22.7 / 11.3 / 9.0   B1 T1024 30.4 / 14.9 / 13.2   B2 T1024 31.9 / 22.3 / 25.8   B1 T2048 46.4 / 37.1 / 37.8
    //   B2 T2048 53.8 / 54.5 / 66.2   B4 T1024 35.2 / 39.6 / 47.0   B8 T1536 107 / 111 / 156   B2 T8192 524 / 591 / 647
    //   B16 H40 T512 63.5 / 50.0 / 82.5; a chunk of 1024 over 640 rows, B8: 117 / 99 (its first tiles are equally long: nothing to pair)
    if (!direct)
        EC_COLSUM(1, 1, 64, false, false);
    else if (pair_key_tiles(D, kt256, BH, Tq, geo.P))
        EC_COLSUM(2, 1, 128, true, true);
    else if ((long long)kt128 * BH <= kSplitMaxWorkgroups)
        EC_COLSUM(1, 2, 128, false, true);
    else
        EC_COLSUM(1, 1, 64, false, true);
#undef EC_COLSUM
    return status_from_hip(hipGetLastError());
}

// Per-head importance into head_imp [B,H,L]; out may be NULL (then v is not read).  direct: q, k and v start on 16-byte
// boundaries.
int score_mfma_dispatch(const void* q, const void* k, const void* v, void* out, float* lse, float* head_imp,
                        int B, int H, ScoreGeom geo, const int32_t* seq_len, int D, int dt, float scale, bool direct,
                        hipStream_t stream)
{
    if (dt != EC_BF16) return EC_EUNSUPPORTED;
    if (D == 128)
        return launch_mfma<128>((const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (uint16_t*)out, lse,
                                head_imp, B, H, geo, seq_len, scale, direct, stream);
    if (D == 64)
        return launch_mfma<64>((const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (uint16_t*)out, lse,
                               head_imp, B, H, geo, seq_len, scale, direct, stream);
    return EC_EUNSUPPORTED;
}

}  // namespace ec
