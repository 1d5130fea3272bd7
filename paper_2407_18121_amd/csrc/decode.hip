// ec_decode_step: single-query attention over the compressed cache, with the
// append of the new key/value row and the fixed-point elimination folded into
// the same launch (Sec. 3.1 Output Generation; Sec. 3.3; Alg. 1's last branch).
//
// Every K and V row of the cache is read exactly once with 16-byte loads.  What bounds it: memory, from about 200 (batch, head)
// pairs on (6 TB/s); below that what one compute unit can have in flight, 54 GB/s, and at short caches the launch itself.
//   one workgroup per (batch, head): nothing is exchanged between workgroups.
//   divided: few pairs with long caches; the rows of one pair are spread over several workgroups of the same launch, whose
//            partial results meet in lines of memory that belong to the library (below).
// As many lanes as a row has 16-byte chunks own one row per load, so a wave load covers 1 KB of contiguous cache; each keeps
// its own running (max, sum, weighted V) inside the streaming loop.  The next tile travels while one is used: its loads are issued
// first and without conditions, so that the wait for one tile is not a wait for both, and scalar bases keep addresses out of
// the vector unit, which 366 instructions per 16 rows of a wave used to fill (bf16: now about 130, with the dot instruction).
// Tiles are aligned to the END of the cache, so when the loop finishes the registers still hold the newest rows: after the
// workgroup barrier that ends all reads, the rows behind the evicted one are stored one slot up straight from those registers,
// and so is the new row -- the elimination costs no extra read.
#include <algorithm>
#include <cmath>

#include "decode_split.h"
#include "ec_common.h"

namespace ec {

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// How a wave reads: a row is owned by as many lanes as it has 16-byte chunks, so that a load covers 1 KB of contiguous cache and
// the sum of a score is a few full-rate lane moves.
template <int DT, int D, int WAVES, int UNROLL> struct DecodeShape {
    static constexpr int kThreads = WAVES * kWave;
    static constexpr int kRowBytes = D * Elem<DT>::kBytes;
    static constexpr int kLPR = kRowBytes / 16;                 // lanes per row
    static constexpr int kRPW = kWave / kLPR;                   // rows per wave load
    static constexpr int kEPL = Elem<DT>::kPerChunk;            // features per lane
    static constexpr int kTile = WAVES * kRPW * UNROLL;         // rows per workgroup iteration
};

// ------------------------------------------------------------------ meeting place of a divided (batch, head)
// A line carries one share's partial result from the workgroup that formed it (a helper) to the one that owns the
// (batch, head), inside one launch.  Lines belong to the library (2.2 MB) and are shared by everything that runs on the
// device, so a line is claimed before it is used and is empty again when the launch ends:
//   state   0 -> open (owner) -> joined (helper) -> 0 (owner, the data read and cleared), or open -> 0 (owner gives up on it)
// "Open" and "joined" carry the address of the head's rows in the K cache, which a launch in flight has to itself, since it writes
// them (an output row may be a throw-away that several share), and the share's number.
// Nobody ever waits for a workgroup that may not be running: an owner that cannot claim a line, or whose helper has not
// joined by the time it is needed, forms that share itself, with the same instructions in the same order; a helper that finds its
// line not open leaves without a trace.  Once a helper has joined it is running and waits for nothing, so the owner's wait for
// its data ends; that wait is bounded all the same, and a line that exceeded it is never given back.
// The data words carry their own validity (upper half not 0): no fence, no cache write-back.
//
// All workgroups of one (batch, head) are launched on one XCD (their linear ids are equal modulo eight), every XCD has lines of its
// own, and a workgroup looks at those of the XCD that it finds itself on: one that was placed elsewhere merely never meets its owner.
// Exchanges and compare-exchanges are carried out by the L2 that they arrive at, and lines that one XCD alone touches stay in its L2
// (loads and stores of device scope, by which words were passed before, go past it).  A helper joins when it starts, not when it is done; the owner takes words and
// empties them in one access, so that it gives its lines back as soon as it has everything and not when the launch has been
// written out; and each wave weighs the shares with a lane for each.  What the exchange adds to a launch was 3.3 us with loads and
// stores past the L2, a join at the end and a separate clearing, and is 2.6: B*H 32, 640 rows of bf16 D128 8.46 -> 7.82 us, B*H 8, 4096 rows (16
// shares) 11.9 -> 10.3.  Stamps at B*H 32, 640 rows, us after the first workgroup's start: rows streamed 3.6, waves brought together 4.0,
// helpers' words sent 4.3, all of them taken 5.9, written out 6.7.  Looking first by plain loads is slower (all taken 6.6).
constexpr int kMaxShares = 64;
constexpr int kLineWords = 136;  // D + 2, padded to whole 64 bytes
constexpr int kJoinTries = 4;    // of a helper that finds its line not open yet
// Looks of the owner at missing data before it asks whether the helper has joined.  Where owners alone do not fill the chip helpers are
// there or about to be: 4 to 24 looks are alike in launches of one workgroup a compute unit, and in larger ones, which only the shaped entry
// point makes, 24 are better than 8 (160 pairs of 640 rows in 2 shares 16.2 / 18.8 us, 48 of 4400 in 24 28.1 / 35.5).  Where
// they do, and all workgroups have no room at once, helpers wait until owners have left: 24 looks / 1, 256 pairs in 16 shares 68.4 / 62.2, 512
// pairs in 2 39.1 / 28.2, 1536 in 2 95 / 61.
__device__ __forceinline__ int patience(int BH) { return BH >= kComputeUnits && gridDim.x > 3 * kComputeUnits ? 1 : 24; }
constexpr int kStuck = 1 << 20;  // looks after that
constexpr unsigned long long kOpen = 1, kJoined = 2;
__device__ __align__(128) static unsigned long long line_state[kXcds * kLines];
__device__ __align__(128) static unsigned long long line_data[kXcds * kLines][kLineWords];

// An exchange takes what it finds and leaves the word empty.  Device scope, as the two sides are different workgroups; for these two
// operations the instructions are those of workgroup scope.
__device__ __forceinline__ unsigned long long line_swap(unsigned long long* p, unsigned long long x)
{
    return __hip_atomic_exchange(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long line_cas(unsigned long long* p, unsigned long long from, unsigned long long to)
{
    __hip_atomic_compare_exchange_strong(p, &from, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return from;  // what was there
}
__device__ __forceinline__ unsigned xcd_id()
{
    unsigned x;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(x));
    return x % kXcds;
}

// The rows of one (batch, head) as shares: share s is the s-th run of `chunk` rows from the END of the cache, so that share
// 0, which the owner takes, holds the rows that an elimination usually moves.  A share has at least `least` rows (a ragged
// batch's launch is laid out for the longest cache).
struct Shares {
    int n_rows, chunk, count;
    __device__ __forceinline__ Shares(int n_rows_, int splits, int least)
        : n_rows(n_rows_), chunk(max((n_rows_ + splits - 1) / splits, least)), count((n_rows_ + chunk - 1) / chunk) {}
    __device__ __forceinline__ int end(int s) const { return n_rows - s * chunk; }
    __device__ __forceinline__ int begin(int s) const { return max(n_rows - (s + 1) * chunk, 0); }
};

// All of x has arrived in registers: what follows neither waits for it nor runs before it.
template <typename T, int N> __device__ __forceinline__ void arrived(T (&x)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));
}

// 16 bytes of data that is read once: the non-temporal hint keeps the stream from displacing cache lines, which measurably
// raises the rate of large one-pass reads on this chip.
__device__ __forceinline__ u32x4 load_once(const char* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}
constexpr int kNonTemporal = 2;  // the same hint of a buffer load
typedef __attribute__((address_space(1))) const char global_char;
typedef __attribute__((address_space(1))) const u32x4 global_u32x4;
__device__ __forceinline__ u32x4 load_once(global_char* p) { return __builtin_nontemporal_load((global_u32x4*)p); }

// The scale in base-2 units, log2(e) * scale, as a factor of q and one of the sums of products.  fp32: q takes all of it.  bf16: q
// takes the power of two that leaves 1 .. 2, so that no sum leaves the range that the score itself stays in.
struct ScoreScale {
    float of_q, of_sum;
};
static ScoreScale score_scale(float scale, int dt)
{
    const float log2 = scale * kLog2e;
    if (dt == EC_F32) return {log2, 1.f};
    int n;
    const float rest = std::frexp(log2, &n);  // 0.5 .. 1
    return {std::ldexp(1.f, n - 1), 2.f * rest};
}

// A chunk of q as the products need it.  A bf16 chunk with an element that its power of two would push below bf16's range (2^-123 and
// less at usual scales) stays as it is.  The first scores wait for this, so that the usual case is short.
struct PreparedQ {
    u32x4 chunk;
    float of_sum;
};
template <int DT> __device__ __forceinline__ PreparedQ prepared_q(const uint4& c, ScoreScale scale)
{
    constexpr int N = Elem<DT>::kPerChunk;
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    float x[N], y[N], smallest = INFINITY;
    unpack<DT>(c, x);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        y[i] = x[i] * scale.of_q;
        smallest = fminf(smallest, fabsf(y[i]));
    }
    PreparedQ p;
    p.of_sum = scale.of_sum;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (DT == EC_F32)
            p.chunk[i] = __float_as_uint(y[i]);
        else
            p.chunk[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{y[2 * i], y[2 * i + 1]}), bf16x2));
    }
    if (DT == EC_BF16 && __builtin_expect(smallest < 0x1p-126f, 0)) {
        bool exact = true;
#pragma unroll
        for (int i = 0; i < N; ++i) exact = exact && (x[i] == 0.f || fabsf(y[i]) >= 0x1p-126f);
        if (!exact) {
            p.chunk = u32x4{c.x, c.y, c.z, c.w};
            p.of_sum *= scale.of_q;
        }
    }
    return p;
}

// Product of a chunk of K with the chunk of q.  bf16: the dot instruction adds two products at a time, each exact in fp32.
template <int DT> __device__ __forceinline__ float chunk_dot(const u32x4& k, const u32x4& q)
{
    float d = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t a = k[i], b = q[i];
        if constexpr (DT == EC_F32)
            d = fmaf(__uint_as_float(b), __uint_as_float(a), d);
        else
            d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), d, false);
    }
    return d;
}

// Maximum over the lane's row of 16.
__device__ __forceinline__ float row_max(float x)
{
    x = fmaxf(x, dpp_mov<kDppQuadXor1>(x));
    x = fmaxf(x, dpp_mov<kDppQuadXor2>(x));
    x = fmaxf(x, dpp_mov<kDppRowHalfMirror>(x));
    return fmaxf(x, dpp_mov<kDppRowMirror>(x));
}

// x[i] <- 2^x[i].  The exponential instruction gives zero where the result is subnormal; exp2f, which is six times as long, does not,
// and is taken only where there is one (-149.. < x < -126; what lies below is zero either way, lanes without rows included).
template <int N> __device__ __forceinline__ void exp2_all(float (&x)[N])
{
    bool subnormal = false;
#pragma unroll
    for (int i = 0; i < N; ++i) subnormal = subnormal | (fabsf(x[i] + 138.5f) < 12.5f);
    if (__builtin_expect(__any(subnormal), 0)) {
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = exp2f(x[i]);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = __builtin_amdgcn_exp2f(x[i]);
    }
}

// Values of a lane and of its partner `off` lanes away (8, 16 or 32), the one with the lower lane number first, in both of them.
struct Pair {
    float lower, upper;
};
__device__ __forceinline__ Pair lane_pair(float x, int off)
{
    const uint32_t u = __float_as_uint(x);
    if (off == 32) {
        const auto y = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        return {__uint_as_float(y[0]), __uint_as_float(y[1])};
    }
    if (off == 16) {
        const auto y = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        return {__uint_as_float(y[0]), __uint_as_float(y[1])};
    }
    const float other = dpp_mov<kDppRowRor8>(x);
    const bool low = threadIdx.x % 16 < 8;
    return {low ? x : other, low ? other : x};
}

// EMIT (frequency discard policy): the kernel also stores every row's scaled score (base-2 units) into
// raw [B,H,cap] and the head's softmax maximum and denominator into stats [B,H,2], from which
// freq_accumulate_kernel forms this step's probabilities.
// SPLIT: the grid holds `splits` workgroups per (batch, head); the first B * H of them are the owners.
template <int DT, int D, int WAVES, int UNROLL, bool DEEP, bool EMIT, bool SPLIT>
__global__ __launch_bounds__(WAVES * kWave) void decode_step_kernel(
    const uint4* __restrict__ q, const uint4* __restrict__ k_new, const uint4* __restrict__ v_new,
    uint4* k_cache, uint4* v_cache, int32_t* pos, uint4* __restrict__ out, int BH, int H, int G, int cap,
    int cache_len, int evict_idx, int32_t new_pos, ScoreScale scale, float* __restrict__ raw,
    float* __restrict__ stats, const int32_t* __restrict__ len_b, const int32_t* __restrict__ evict_b,
    const int32_t* __restrict__ new_pos_b, int splits, int least)
{
    using S = DecodeShape<DT, D, WAVES, UNROLL>;
    const int stride = SPLIT ? split_stride(BH) : BH;
    const int own_share = SPLIT ? blockIdx.x / stride : 0;
    const int bh = SPLIT ? blockIdx.x - own_share * stride : blockIdx.x;
    if (SPLIT && bh >= BH) return;
    if (len_b) {  // ragged batch: every batch element has its own cache length, victim and position
        const int b = bh / H;
        cache_len = min(max(len_b[b], 0), cap - 1);
        evict_idx = evict_b ? min(max(evict_b[b], -1), cache_len) : -1;
        if (new_pos_b) new_pos = new_pos_b[b];
    }
    constexpr int THREADS = S::kThreads, TILE = S::kTile, ROW = S::kRowBytes;
    constexpr int LPR = S::kLPR, RPW = S::kRPW, NR = UNROLL, EPL = S::kEPL;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid % kWave;
    const int sub = lane % LPR, rgrp = lane / LPR;  // which chunk of a row, which row of a load

    const Shares shares(cache_len + 1, SPLIT ? splits : 1, SPLIT ? least : 1);  // row cache_len is the new one, still in k_new/v_new
    if (SPLIT && own_share >= shares.count) return;

    char* kc = reinterpret_cast<char*>(k_cache) + (size_t)bh * cap * ROW;
    char* vc = reinterpret_cast<char*>(v_cache) + (size_t)bh * cap * ROW;
    const char* kn = reinterpret_cast<const char*>(k_new) + (size_t)bh * ROW;
    const char* vn = reinterpret_cast<const char*>(v_new) + (size_t)bh * ROW;

    const unsigned long long row_key = (unsigned long long)(uintptr_t)kc << 8;
    const unsigned line0 = first_line((uintptr_t)out / ROW + bh, splits);
    const unsigned xcd_lines = SPLIT ? xcd_id() * kLines : 0;
    auto line_of = [&](int s) { return xcd_lines + (line0 + (unsigned)(s - 1)) % kLines; };
    auto key_of = [&](int s) { return row_key | (unsigned long long)s << 2; };
    bool claimed = false;  // owner, lane s of wave 0: the line of share s is this launch's
    if (SPLIT && own_share == 0 && wave == 0 && lane >= 1 && lane < shares.count)
        claimed = line_cas(&line_state[line_of(lane)], 0, key_of(lane) | kOpen) == 0;
    unsigned long long seen = 0;  // helper: what its line held
    if (SPLIT && own_share > 0 && tid == 0) seen = line_cas(&line_state[line_of(own_share)], key_of(own_share) | kOpen, key_of(own_share) | kJoined);

    // positions of the rows behind the victim, fetched early (stored after the barrier)
    const bool owns_pos = own_share == 0 && pos != nullptr && (G == H || (bh % H) == 0);
    int32_t* pp = owns_pos ? pos + ((size_t)(bh / H) * G + (G == 1 ? 0 : bh % H)) * cap : nullptr;
    const int n_move = (evict_idx >= 0) ? max(cache_len - 1 - evict_idx, 0) : 0;
    int32_t pos_pref = 0;
    if (owns_pos && tid < n_move) pos_pref = pp[evict_idx + 1 + tid];

    PreparedQ qp;
    const uint4 q_in = q[(size_t)bh * LPR + sub];

    // two tiles, one being used while the other lands
    struct Rows {
        u32x4 k[NR], v[NR];
    } ta, tb;
    const int lane_row = wave * (RPW * NR) + rgrp;  // this lane's rows of a tile: lane_row + u * RPW
    const uint32_t lane_at = lane_row * ROW + sub * 16;

    // A tile is rows first .. first + TILE - 1.  The first of a share may start before its first row r0, the last may end with
    // the new row; the ones between are loaded without a condition, so that waiting for one never means waiting for the next.
    // The outer ones, which is all there is of a short cache, do without branches too: rows before r0 are offsets behind the end of
    // the buffer, which read nothing and give zeros.  Only the last load of a lane can be the new row's, from an address of its
    // own; there a row before r0 is r0 again, and attend() drops its V.  (Each load under a condition -> this, us, bf16 D128: B*H
    // 128, 120 rows 5.2 -> 4.5; B*H 256, 120 rows 6.4 -> 5.7, 250 rows 8.7 -> 8.1.)
    auto load_inner = [&](int first, Rows& x) __attribute__((always_inline)) {
        global_char *k0 = (global_char*)kc + (size_t)first * ROW, *v0 = (global_char*)vc + (size_t)first * ROW;
        asm volatile("" : "+s"(k0), "+s"(v0));  // scalar base, constant lane offset: no address arithmetic per load
#pragma unroll
        for (int u = 0; u < NR; ++u) x.k[u] = load_once(k0 + (lane_at + u * RPW * ROW));
        __builtin_amdgcn_sched_barrier(0);  // K is needed first
#pragma unroll
        for (int u = 0; u < NR; ++u) x.v[u] = load_once(v0 + (lane_at + u * RPW * ROW));
        __builtin_amdgcn_sched_barrier(0);
    };
    // An inner tile or the last one, by the same instructions: a branch between two kinds of loads makes the waits behind it waits
    // for everything.
    auto load_any = [&](int first, Rows& x) __attribute__((always_inline)) {
        global_char *k0 = (global_char*)kc + (ptrdiff_t)first * ROW, *v0 = (global_char*)vc + (ptrdiff_t)first * ROW;
        asm volatile("" : "+s"(k0), "+s"(v0));
        const bool is_new = first + (NR - 1) * RPW + lane_row == cache_len;
        const uint32_t at = lane_at + (NR - 1) * RPW * ROW;
        global_char* ks = is_new ? (global_char*)kn + sub * 16 : k0 + at;
        global_char* vs = is_new ? (global_char*)vn + sub * 16 : v0 + at;
#pragma unroll
        for (int u = 0; u < NR - 1; ++u) x.k[u] = load_once(k0 + (lane_at + u * RPW * ROW));
        x.k[NR - 1] = load_once(ks);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < NR - 1; ++u) x.v[u] = load_once(v0 + (lane_at + u * RPW * ROW));
        x.v[NR - 1] = load_once(vs);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto load_outer = [&](int first, int r0, Rows& x) __attribute__((always_inline)) {
        const auto k_rows = __builtin_amdgcn_make_buffer_rsrc(kc + (ptrdiff_t)first * ROW, 0, TILE * ROW, 0x00020000);
        const auto v_rows = __builtin_amdgcn_make_buffer_rsrc(vc + (ptrdiff_t)first * ROW, 0, TILE * ROW, 0x00020000);
        const int r = max(first + (NR - 1) * RPW + lane_row, r0);
        const char* ks = (r == cache_len ? kn : kc + (ptrdiff_t)r * ROW) + sub * 16;
        const char* vs = (r == cache_len ? vn : vc + (ptrdiff_t)r * ROW) + sub * 16;
        auto load = [&](auto rows, int u) __attribute__((always_inline)) {
            const uint32_t at = first + u * RPW + lane_row >= r0 ? lane_at + u * RPW * ROW : TILE * ROW;
            return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, at, 0, kNonTemporal));
        };
#pragma unroll
        for (int u = 0; u < NR - 1; ++u) x.k[u] = load(k_rows, u);
        x.k[NR - 1] = load_once(ks);
        __builtin_amdgcn_sched_barrier(0);  // K is needed first
#pragma unroll
        for (int u = 0; u < NR - 1; ++u) x.v[u] = load(v_rows, u);
        x.v[NR - 1] = load_once(vs);
        __builtin_amdgcn_sched_barrier(0);
    };

    __shared__ __align__(16) float sh_acc[WAVES][D];
    __shared__ float sh_m[WAVES];
    __shared__ float sh_l[WAVES];
    __shared__ float part[SPLIT ? kMaxShares : 1][D + 2];  // of every share: weighted V, maximum, sum of weights
    __shared__ unsigned long long sh_claimed, sh_lost, sh_missing[2];
    __shared__ int sh_joined;
    if (SPLIT && tid < 2) sh_missing[tid] = 0;

    // ---- fixed-point elimination + append ----
    // With a victim, rows evict_idx+1 .. cache_len (the last being the new row) move up by one; the new row is dropped if it
    // is the victim itself.  Without one, the new row lands at cache_len.  The last tile of share 0 is still in registers when
    // its scores have been formed: rows held .. cache_len are stored from there.
    const int tail_first = shares.end(0) - TILE, held = max(tail_first, shares.begin(0));
    // Nothing moves but what the registers hold, and all of it to rows of share 0: the row before them belongs to a share that a
    // helper may still be reading or that has yet to be formed.
    const bool moved_early = evict_idx < 0 || (evict_idx >= shares.begin(0) && evict_idx + 1 >= held);
    auto move_held = [&]() __attribute__((always_inline)) {
        const int lowest = evict_idx >= 0 ? max(evict_idx + 1, held) : cache_len, up = evict_idx >= 0 ? 1 : 0;
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int r = tail_first + u * RPW + lane_row;
            if (r >= lowest) {
                const ptrdiff_t at = (ptrdiff_t)(r - up) * ROW + sub * 16;
                *reinterpret_cast<u32x4*>(kc + at) = ta.k[u];
                *reinterpret_cast<u32x4*>(vc + at) = ta.v[u];
            }
        }
    };

    unsigned long long todo = 0;
    for (int s = own_share;;) {
        const int r0 = shares.begin(s), r1 = shares.end(s);
        const int n_tiles = (r1 - r0 + TILE - 1) / TILE;
        const int first_row = r1 - n_tiles * TILE;
        const int last_first = r1 - TILE;
        // per lane: maximum (base-2 units), sum of weights and weighted V of the rows it holds V of
        float m_run = kLowest, l_run = 0.f;
        float acc[EPL];
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = 0.f;

        auto attend = [&](int first, Rows& x) __attribute__((always_inline)) {
            float sc[NR];
            float m_tile = kLowest, least_score = INFINITY;
#pragma unroll
            for (int u = 0; u < NR; ++u) {
                const float d = chunk_dot<DT>(x.k[u], qp.chunk);
                sc[u] = group_sum<LPR>(DT == EC_F32 ? d : d * qp.of_sum);
                least_score = fminf(least_score, sc[u]);
            }
            if (first < r0) {  // uniform
#pragma unroll
                for (int u = 0; u < NR; ++u)
                    if (first + u * RPW + lane_row < r0) sc[u] = -INFINITY;
                if (first + (NR - 1) * RPW + lane_row < r0) x.v[NR - 1] = u32x4{0, 0, 0, 0};  // read from another row
            }
            if constexpr (EMIT) {
                const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(raw + ((ptrdiff_t)bh * cap + first), 0, TILE * 4, 0x00020000);
                float y = sc[0];
#pragma unroll
                for (int u = 1; u < NR; ++u) y = sub == u ? sc[u] : y;
                const int r = sub * RPW + lane_row;
                // not under a condition either: lanes with nothing to store point behind the descriptor's end
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y), rsrc, sub < NR && first + r >= r0 ? r * 4 : TILE * 4, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < NR; ++u) m_tile = fmaxf(m_tile, sc[u]);
            __builtin_amdgcn_sched_barrier(0);  // V is not waited for before the scores are there
            if (__any(m_tile > m_run)) {  // wave-uniform
                const float m_new = fmaxf(m_run, m_tile);
                const float corr = exp2f(m_run - m_new);
                m_run = m_new;
                l_run *= corr;
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[e] *= corr;
            }
            float weight[NR];  // as exp2_all(), with a shorter question
            if (__builtin_expect(__any(least_score - m_run < -126.f), 0)) {  // wave-uniform
#pragma unroll
                for (int u = 0; u < NR; ++u) weight[u] = exp2f(sc[u] - m_run);
            } else {
#pragma unroll
                for (int u = 0; u < NR; ++u) weight[u] = __builtin_amdgcn_exp2f(sc[u] - m_run);
            }
            // fp32: a tile is summed by itself and then added, which keeps the rounding errors of a long chain small
            float part_l = 0.f, part_v[EPL];
#pragma unroll
            for (int u = 0; u < NR; ++u) {
                const float p = weight[u];
                float vx[EPL];
                unpack<DT>(__builtin_bit_cast(uint4, x.v[u]), vx);
                if (DT == EC_F32) {
                    part_l += p;
#pragma unroll
                    for (int e = 0; e < EPL; ++e) part_v[e] = u == 0 ? p * vx[e] : fmaf(p, vx[e], part_v[e]);
                } else {
                    l_run += p;
#pragma unroll
                    for (int e = 0; e < EPL; ++e) acc[e] = fmaf(p, vx[e], acc[e]);
                }
            }
            if (DT == EC_F32) {
                l_run += part_l;
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[e] += part_v[e];
            }
            // summed here, before the registers of the tile are loaded again
            asm volatile("" : "+v"(l_run));
            arrived(acc);
        };

        load_outer(first_row, r0, ta);
        if (s == own_share) qp = prepared_q<DT>(q_in, scale);
        int first = first_row;
        if constexpr (DEEP) {
            for (; first < last_first - TILE; first += 2 * TILE) {
                load_inner(first + TILE, tb);
                attend(first, ta);
                load_any(first + 2 * TILE, ta);
                attend(first + TILE, tb);
            }
            if (first != last_first) {
                load_any(last_first, tb);
                attend(first, ta);
                attend(last_first, tb);
                ta = tb;
            } else {
                attend(last_first, ta);
            }
        } else {
            while (first != last_first) {
                attend(first, ta);
                first += TILE;
                load_any(first, ta);
            }
            attend(last_first, ta);
        }
        // ta holds the last tile: of share 0, the newest rows

        // ---- merge the lanes of each wave that hold the same features: the maximum first, then plain sums ----
        {
            float m_wave = m_run;
#pragma unroll
            for (int off = LPR; off < kWave; off <<= 1) {
                const Pair m = lane_pair(m_wave, off);
                m_wave = fmaxf(m.lower, m.upper);
            }
            const float corr = exp2f(m_run - m_wave);
            m_run = m_wave;
            l_run *= corr;
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[e] *= corr;
#pragma unroll
            for (int off = LPR; off < kWave; off <<= 1) {
                const Pair l = lane_pair(l_run, off);
                l_run = l.lower + l.upper;
#pragma unroll
                for (int e = 0; e < EPL; ++e) {
                    const Pair x = lane_pair(acc[e], off);
                    acc[e] = x.lower + x.upper;
                }
            }
        }

        // ---- merge the waves through LDS ----
        if (lane < LPR) {
#pragma unroll
            for (int e = 0; e < EPL; e += 4)
                *reinterpret_cast<float4*>(&sh_acc[wave][sub * EPL + e]) = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
            if (sub == 0) {
                sh_m[wave] = m_run;
                sh_l[wave] = l_run;
            }
        }
        if (SPLIT && own_share > 0 && tid == 0) {
            for (int i = 0; seen == 0 && i < kJoinTries; ++i)
                seen = line_cas(&line_state[line_of(s)], key_of(s) | kOpen, key_of(s) | kJoined);
            sh_joined = seen == (key_of(s) | kOpen);
        }
        if (SPLIT && own_share == 0 && s == 0 && wave == 0) {
            const unsigned long long c = __ballot(claimed);
            if (tid == 0) sh_claimed = c;
        }
        __syncthreads();  // also: every wave of this workgroup has finished reading its rows

        if (own_share == 0 && s == 0) {
            if (moved_early) move_held();  // to rows of share 0 only: the other shares' workgroups do not read them
            if (owns_pos) {  // one copy of the positions per score group
                if (tid < n_move) pp[evict_idx + tid] = pos_pref;  // fetched before the barrier above
                for (int c0 = THREADS; c0 < n_move; c0 += THREADS) {  // beyond one workgroup's worth
                    const int c = c0 + tid;
                    int32_t pv = 0;
                    if (c < n_move) pv = pp[evict_idx + 1 + c];
                    __syncthreads();
                    if (c < n_move) pp[evict_idx + c] = pv;
                }
                const int new_row = (evict_idx < 0) ? cache_len : ((evict_idx == cache_len) ? -1 : cache_len - 1);
                if (new_row >= 0 && tid == 0) pp[new_row] = new_pos;
            }
        }

        float M = kLowest, L = 0.f, o_d = 0.f;
        if (tid < D) {
            float wt[WAVES], l[WAVES], x[WAVES];  // read together
#pragma unroll
            for (int w = 0; w < WAVES; ++w) wt[w] = sh_m[w], l[w] = sh_l[w], x[w] = sh_acc[w][tid];
            arrived(wt), arrived(l), arrived(x);
#pragma unroll
            for (int w = 0; w < WAVES; ++w) M = fmaxf(M, wt[w]);
#pragma unroll
            for (int w = 0; w < WAVES; ++w) wt[w] -= M;
            exp2_all(wt);
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                L = fmaf(l[w], wt[w], L);
                o_d = fmaf(x[w], wt[w], o_d);
            }
        }
        if constexpr (SPLIT) {
            if (own_share > 0) {
                if (sh_joined && tid < D) {
                    unsigned long long* line = line_data[line_of(s)];
                    const unsigned long long valid = 1ull << 32;
                    line_swap(line + tid, valid | __float_as_uint(o_d));
                    if (tid < 2) line_swap(line + D + tid, valid | __float_as_uint(tid == 0 ? M : L));
                }
                return;
            }
            if (tid < D) {
                part[s][tid] = o_d;
                if (tid < 2) part[s][D + tid] = tid == 0 ? M : L;
            }
            if (s == 0) {
                // word j of the claimed lines belongs to thread j % THREADS, which remembers the ones still to come
                constexpr int kBatch = 4;
                const int total = (shares.count - 1) * (D + 2);
                unsigned long long pending = 0;
                for (int j = tid, i = 0; j < total; j += THREADS, ++i)
                    if (sh_claimed >> (1 + j / (D + 2)) & 1) pending |= 1ull << i;
                auto look = [&](int patience) {
                    for (int i0 = 0; i0 * THREADS + tid < total; i0 += kBatch)
                        for (int n = 0; (pending >> i0 & ((1ull << kBatch) - 1)) && n < patience; ++n) {
                            unsigned long long x[kBatch] = {};
#pragma unroll
                            for (int u = 0; u < kBatch; ++u) {
                                const int j = (i0 + u) * THREADS + tid;
                                if (pending >> (i0 + u) & 1) x[u] = line_swap(&line_data[line_of(1 + j / (D + 2))][j % (D + 2)], 0);
                            }
#pragma unroll
                            for (int u = 0; u < kBatch; ++u)
                                if (x[u] >> 32) {
                                    const int j = (i0 + u) * THREADS + tid;
                                    part[1 + j / (D + 2)][j % (D + 2)] = __uint_as_float((uint32_t)x[u]);
                                    pending &= ~(1ull << (i0 + u));
                                }
                        }
                };
                auto missing = [&](int round) {  // shares with a word still to come
                    for (int i = 0; i < 64 && pending >> i; ++i)
                        if (pending >> i & 1) atomicOr(&sh_missing[round], 1ull << (1 + (i * THREADS + tid) / (D + 2)));
                    __syncthreads();
                    return sh_missing[round];
                };
                look(patience(BH));
                const unsigned long long all = (shares.count < 64 ? 1ull << shares.count : 0ull) - 2;
                unsigned long long given_up = 0;
                if (const unsigned long long late = missing(0)) {  // uniform
                    if (wave == 0) {
                        const unsigned long long open = key_of(lane) | kOpen;
                        const bool lost = (late >> lane & 1) && line_cas(&line_state[line_of(lane)], open, 0) == open;
                        const unsigned long long l = __ballot(lost);
                        if (tid == 0) sh_lost = l;
                    }
                    __syncthreads();
                    given_up = sh_lost;
                    for (int i = 0; i < 64 && pending >> i; ++i)
                        if (given_up >> (1 + (i * THREADS + tid) / (D + 2)) & 1) pending &= ~(1ull << i);
                    look(kStuck);
                    given_up |= missing(1);
                }
                todo = all & (~sh_claimed | given_up);
                // Every word of the lines that were joined has been taken (all threads have passed missing()): whoever claims one
                // next finds it empty.
                if (wave == 0 && claimed && !(given_up >> lane & 1)) line_swap(&line_state[line_of(lane)], 0);
            } else {
                todo &= ~(1ull << s);
                __syncthreads();  // sh_acc is written again
            }
            if (todo) {
                s = __ffsll((long long)todo) - 1;
                continue;
            }
            if (!moved_early && s != 0) {  // another share was formed after share 0: its rows again
                load_outer(tail_first, shares.begin(0), ta);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // arrived before any wave overwrites them
                __syncthreads();
            }
            // Every wave weighs the shares, a lane each, and adds their rows up in ascending order (every thread all of them: 16 shares
            // 10.8 us, so 10.3).
            const bool has = lane < shares.count;
            const int of = has ? lane : 0;
            const float m_share = has ? part[of][D] : kLowest, l_share = has ? part[of][D + 1] : 0.f;
            auto first = [](float x) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x))); };
            M = first(shares.count > 16 ? wave_max(m_share) : row_max(m_share));
            float wt[1] = {m_share - M};
            exp2_all(wt);
            L = first(shares.count > 16 ? group_sum<kWave>(l_share * wt[0]) : group_sum<16>(l_share * wt[0]));
            o_d = 0.f;
            if (tid < D) {
                constexpr int N = 8;  // reads that overlap
                for (int i0 = 0; i0 < shares.count; i0 += N) {
                    float x[N];
#pragma unroll
                    for (int i = 0; i < N; ++i) x[i] = i0 + i < shares.count ? part[i0 + i][tid] : 0.f;
                    arrived(x);
#pragma unroll
                    for (int i = 0; i < N; ++i)  // lanes behind the last share: x is 0
                        o_d = fmaf(x[i], __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wt[0]), i0 + i)), o_d);
                }
            }
        }
        if (tid < D) {
            if (EMIT && tid == 0) {
                stats[(size_t)bh * 2] = M;
                stats[(size_t)bh * 2 + 1] = L;
            }
            const float r = o_d / L;
            typename Elem<DT>::type* o = reinterpret_cast<typename Elem<DT>::type*>(out) + (size_t)bh * D;
            if constexpr (DT == EC_F32)
                o[tid] = r;
            else
                o[tid] = f32_to_bf16(r);
        }
        break;
    }

    if (!moved_early) {
        // Rows behind the victim that left the registers long ago, through memory: slab by slab, each read completely before any
        // of it is overwritten.  No other workgroup's reads count any more: a helper that still has some going was given up on, cannot
        // join, and drops its sums.
        const int total = (held - (evict_idx + 1)) * LPR;
        u32x4* kd = reinterpret_cast<u32x4*>(kc + (size_t)evict_idx * ROW);
        u32x4* vd = reinterpret_cast<u32x4*>(vc + (size_t)evict_idx * ROW);
        for (int c0 = 0; c0 < total; c0 += THREADS) {
            const int c = c0 + tid;
            u32x4 kk, vv;
            if (c < total) {
                kk = kd[LPR + c];
                vv = vd[LPR + c];
            }
            __syncthreads();
            if (c < total) {
                kd[c] = kk;
                vd[c] = vv;
            }
        }
        __syncthreads();
        move_held();
    }
}

template <int DT, int D, int WAVES, int UNROLL, bool DEEP, bool EMIT, bool SPLIT>
static int launch_decode_w(const void* q, const void* k_new, const void* v_new, void* k_cache,
                           void* v_cache, int32_t* pos, int B, int H, int G, int cap, int cache_len,
                           int evict_idx, int32_t new_pos, float scale, void* out, float* raw, float* stats,
                           const int32_t* len_b, const int32_t* evict_b, const int32_t* new_pos_b, int splits, int least,
                           hipStream_t stream)
{
    using S = DecodeShape<DT, D, WAVES, UNROLL>;
    hipLaunchKernelGGL((decode_step_kernel<DT, D, WAVES, UNROLL, DEEP, EMIT, SPLIT>), dim3(SPLIT ? split_stride(B * H) * splits : B * H),
                       dim3(S::kThreads), 0, stream, (const uint4*)q, (const uint4*)k_new, (const uint4*)v_new,
                       (uint4*)k_cache, (uint4*)v_cache, pos, (uint4*)out, B * H, H, G, cap, cache_len, evict_idx, new_pos,
                       score_scale(scale, DT), raw, stats, len_b, evict_b, new_pos_b, splits, least);
    return status_from_hip(hipGetLastError());
}

constexpr int kLeastShareBytes = 48 << 10;  // of K and V

// Shape of a workgroup when the caller leaves it to the library: waves, loads of K and of V per lane and tile, and whether the next
// tile travels while one is used (deep).  Up to one workgroup per compute unit wants as much in flight as it can have.  Beyond
// that the limit is memory, and the more pairs there are the fewer bytes should be asked for at a time; batches of sequences that
// differ in length want more than their pairs say, as the short ones end and leave the rest alone.  A cache of one tile has only
// one round of loads.  us, four waves 4 deep / four 2 deep / four 4 / two 4 / two 2 (the kernel before the deep loop), D128:
//   bf16 B*H  320  250 rows 10.8 / 10.8 / 10.6 / 11.8 / 17.2 (11.3)       900 rows 29.3 / 28.7 / 28.2 / 32.0 / 47.7 (28.4)
//   bf16 B*H  640  250 rows 17.7 / 17.7 / 17.7 / 17.2 / 20.0 (18.2)       900 rows 52.8 / 52.8 / 53.5 / 50.2 / 55.0 (52.6)
//   bf16 B*H 1024  400 rows 39.9 / 39.6 / 39.7 / 36.8 / 37.9 (36.8)     B*H 1536  640 rows 91.8 / 92.0 / 92.0 / 90.6 / 83.6 (85.8)
//   bf16 B*H 1536   32 rows 10.9 / 10.5 / 10.2 / 10.9 / 12.6 (10.3)     B*H 512 ragged 900 rows 32.6 / 32.5 / 32.8 / 35.8 / 48.6 (33.1)
//   f32  B*H  512  250 rows 25.8 / 27.3 / 24.9 / 28.2 / 34.2 (25.2)     B*H 1920  400 rows 151 / 155 / 150 / 147 / 141 (142)
// Rows of 128 bytes (bf16 D64): up to 1023 pairs like bf16 D128; then two waves, 2 deep for short caches (B*H 1024, 64 rows 6.7 us,
// four waves 2 deep 6.8) and not deep for long ones (B*H 1536, 900 rows 57.9, deep 61.5).
// Over both types and sizes, 320 to 1920 pairs, 32 to 4096 rows the choice is 2 % faster than that kernel; what it loses, 3 to 7 % at
// single points and 10 % for 1920 ragged caches of up to 33 rows, it loses on caches of one to three tiles and at 88 KB of 1536
// pairs, where no shape here does better by more than 2 %.
constexpr long long kKiB = 1 << 10;
struct DecodeAuto {
    int waves, unroll;
    bool deep;
};
static DecodeAuto decode_auto_shape(int BH, int n_rows, int row_bytes, bool half, bool ragged)
{
    const long long bytes = 2LL * n_rows * row_bytes;             // of K and V, of the longest sequence
    const long long typical = ragged ? bytes - bytes / 4 : bytes;  // lengths from half of it to all of it
    const bool crowd = BH >= (ragged ? 1400 : 1200);
    if (BH <= kComputeUnits) return {4, 4, true};
    if (row_bytes >= 512) {
        if (typical < 140 * kKiB) return {4, 4, true};
        if (BH < 1024 || typical < (crowd ? 200 : 300) * kKiB) return {4, 4, false};
        return crowd ? DecodeAuto{2, 2, false} : DecodeAuto{2, 4, false};
    }
    if (row_bytes >= 256 && bytes <= 32 * kKiB) return {4, 4, false};
    if (BH < (half ? 512 : 513))  // at 512 two waves and four are alike
        return bytes >= 320 * kKiB ? DecodeAuto{4, 4, false} : DecodeAuto{4, 2, true};
    if (BH < 1024) {
        const bool is_long = !ragged && bytes >= (row_bytes >= 256 ? 160 : 320) * kKiB;
        return is_long ? DecodeAuto{2, 4, false} : DecodeAuto{4, 2, true};
    }
    if (row_bytes >= 256) {
        if (typical < 80 * kKiB) return {4, 2, true};
        return crowd && typical >= 110 * kKiB ? DecodeAuto{2, 2, false} : DecodeAuto{2, 4, false};
    }
    return {2, 2, typical < 80 * kKiB || (ragged && !crowd)};
}
// the shapes above but the first
#define EC_DECODE_AUTO_SHAPES(CASE_) CASE_(4, 4, false) CASE_(4, 2, true) CASE_(2, 4, false) CASE_(2, 2, true) CASE_(2, 2, false)

// splits: 0 = choose, n = n workgroups per (batch, head).
template <int DT, int D>
static int launch_decode(const void* q, const void* k_new, const void* v_new, void* k_cache,
                         void* v_cache, int32_t* pos, int B, int H, int G, int cap, int cache_len,
                         int evict_idx, int32_t new_pos, float scale, void* out, int forced_waves,
                         int forced_unroll, int splits, bool strict, size_t part_floats,
                         const int32_t* len_b, const int32_t* evict_b, const int32_t* new_pos_b, hipStream_t stream)
{
    constexpr int kRow = D * Elem<DT>::kBytes;
    const int n_rows = cache_len + 1;  // ragged batches pass the longest length the buffers allow
    int waves = forced_waves, unroll = forced_unroll <= 0 ? 4 : forced_unroll, least = 1;
    // an explicit request has to bring a workspace, as the interface says
    if (strict && splits > 1 && part_floats < (size_t)B * H * splits * (D + 2)) return EC_EWORKSPACE;
    const bool choose = forced_waves <= 0 && forced_unroll <= 0 && splits <= 0;
    if (splits <= 0) {  // with a width or a depth given, one workgroup takes everything
        splits = choose ? decode_auto_splits(B * H, n_rows, kRow, DT == EC_BF16) : 1;
        least = kLeastShareBytes / (2 * kRow);
    }
#define EC_DECODE_W(W_, U_, DEEP_, SPLIT_)                                                                                 \
    return launch_decode_w<DT, D, W_, U_, DEEP_, false, SPLIT_>(q, k_new, v_new, k_cache, v_cache, pos, B, H, G, cap, cache_len, \
                                                                evict_idx, new_pos, scale, out, nullptr, nullptr, len_b,   \
                                                                evict_b, new_pos_b, splits, least, stream)
    if (choose && splits == 1) {
        const DecodeAuto a = decode_auto_shape(B * H, n_rows, kRow, DT == EC_BF16, len_b != nullptr);
#define EC_DECODE_AUTO(W_, U_, DEEP_) \
    if (a.waves == W_ && a.unroll == U_ && a.deep == DEEP_) EC_DECODE_W(W_, U_, DEEP_, false);
        EC_DECODE_AUTO_SHAPES(EC_DECODE_AUTO)
#undef EC_DECODE_AUTO
    }
    if (waves <= 0) waves = 4;
    const bool known = splits > 1 ? ((waves == 2 || waves == 4) && (unroll == 4 || unroll == 8)) || (waves == 8 && unroll == 4)
                                  : (waves == 2 && (unroll == 4 || unroll == 8)) ||
                                        (waves == 4 && (unroll == 4 || unroll == 6 || unroll == 8 || unroll == 12)) ||
                                        (waves == 8 && (unroll == 4 || unroll == 8 || unroll == 12)) ||
                                        (waves == 16 && (unroll == 4 || unroll == 6));
    if (!known) return EC_EINVAL;
    // what the kernel is built for: up to 8 waves, 4 or 8 loads of K and of V
#define EC_DECODE_U(W_, SPLIT_)                            \
    do {                                                   \
        if (unroll == 4) EC_DECODE_W(W_, 4, true, SPLIT_); \
        EC_DECODE_W(W_, 8, true, SPLIT_);                  \
    } while (0)
    if (splits > 1) {
        if (waves == 2) EC_DECODE_U(2, true);
        if (waves == 4) EC_DECODE_U(4, true);
        EC_DECODE_W(8, 4, true, true);
    }
    splits = 1;
    if (waves == 2) EC_DECODE_U(2, false);
    if (waves == 4) EC_DECODE_U(4, false);
    EC_DECODE_U(8, false);
#undef EC_DECODE_U
#undef EC_DECODE_W
}

// strict: the launch shape is an explicit request; a split without enough workspace is then an error instead
// of falling back to the fused kernel.
int decode_dispatch(const void* q, const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                    int32_t* pos, int B, int H, int G, int D, int cap, int cache_len, int evict_idx,
                    int32_t new_pos, float scale, int dt, void* out, int forced_waves, int forced_unroll,
                    int splits, bool strict, size_t part_floats, const int32_t* len_b,
                    const int32_t* evict_b, const int32_t* new_pos_b, hipStream_t stream)
{
#define EC_DECODE_CASE(DT_, D_)                                                                       \
    if (dt == DT_ && D == D_)                                                                         \
        return launch_decode<DT_, D_>(q, k_new, v_new, k_cache, v_cache, pos, B, H, G, cap, cache_len,    \
                                      evict_idx, new_pos, scale, out, forced_waves, forced_unroll, splits, \
                                      strict, part_floats, len_b, evict_b, new_pos_b, stream);
    EC_DECODE_CASE(EC_BF16, 128)
    EC_DECODE_CASE(EC_BF16, 64)
    EC_DECODE_CASE(EC_F32, 128)
    EC_DECODE_CASE(EC_F32, 64)
#undef EC_DECODE_CASE
    return EC_EUNSUPPORTED;
}

// ------------------------------------------------------------------ frequency discard policy
// freq[b,g,j] += this step's attention mass of row j (head mean when G == 1); the row just appended
// (j = n - 1) starts at its own mass.  A workgroup covers 64 rows; its 4 thread groups each add up a quarter
// of the heads (ascending), and the quarters are added in ascending order: the result does not depend on
// scheduling.
constexpr int kFreqRows = 64;
constexpr int kFreqParts = 4;
constexpr int kFreqHeads = 8;
__global__ __launch_bounds__(kFreqRows * kFreqParts) void freq_accumulate_kernel(const float* __restrict__ raw,
                                                                                const float* __restrict__ stats,
                                                                                float* __restrict__ freq, int H, int G,
                                                                                int n, int cap)
{
    __shared__ float part[kFreqParts][kFreqRows];
    const int bg = blockIdx.y;
    const int r = threadIdx.x % kFreqRows, grp = threadIdx.x / kFreqRows;
    const int j = blockIdx.x * kFreqRows + r;
    const int b = bg / G, g = bg % G;
    const int h_first = (G == H) ? g : 0, h_count = (G == H) ? 1 : H;
    const int per = (h_count + kFreqParts - 1) / kFreqParts;
    const int h0 = h_first + grp * per, h1 = min(h0 + per, h_first + h_count);
    float acc = 0.f;
    auto mass = [&](float x, float m, float l) { return exp2f(x - m) / l; };
    if (per < kFreqHeads / 2) {  // head-wise counts, few heads
        if (j < n)
            for (int h = h0; h < h1; ++h) {
                const size_t bh = (size_t)b * H + h;
                acc += mass(raw[bh * cap + j], stats[bh * 2], stats[bh * 2 + 1]);
            }
    } else {
        // Eight heads at a time, all their reads in flight together (the last one again where there are fewer).  A trip to memory
        // per head, one after the other, made a whole step (decode, masses, removal) 27.2 us at B8 H32 640 rows, now 25.8, and 15.4
        // at B1 300 rows, now 13.9; below four heads a thread the reads for nothing cost more (H8: 16.1, 16.4).
        for (int h = h0; h < h1; h += kFreqHeads) {
            float x[kFreqHeads], m[kFreqHeads], l[kFreqHeads];
#pragma unroll
            for (int i = 0; i < kFreqHeads; ++i) {
                const size_t bh = (size_t)b * H + min(h + i, h1 - 1);
                x[i] = raw[bh * cap + min(j, n - 1)], m[i] = stats[bh * 2], l[i] = stats[bh * 2 + 1];
            }
            arrived(x);
#pragma unroll
            for (int i = 0; i < kFreqHeads; ++i)
                if (h + i < h1) acc += mass(x[i], m[i], l[i]);
        }
    }
    part[grp][r] = acc;
    __syncthreads();
    if (grp == 0 && j < n) {
        float mass = part[0][r];
#pragma unroll
        for (int p = 1; p < kFreqParts; ++p) mass += part[p][r];
        mass /= (float)h_count;
        float* f = freq + (size_t)bg * cap + j;
        *f = (j == n - 1) ? mass : *f + mass;
    }
}

template <int DT, int D>
static int launch_decode_score(const void* q, const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                               int32_t* pos, float* freq, int B, int H, int G, int cap, int cache_len,
                               int32_t new_pos, float scale, void* out, float* raw, float* stats,
                               hipStream_t stream)
{
    constexpr int kRow = D * Elem<DT>::kBytes;
    const int n = cache_len + 1, splits = decode_auto_splits(B * H, n, kRow, DT == EC_BF16), least = kLeastShareBytes / (2 * kRow);
#define EC_DSCORE(W_, U_, DEEP_, SPLIT_)                                                                                       \
    rc = launch_decode_w<DT, D, W_, U_, DEEP_, true, SPLIT_>(q, k_new, v_new, k_cache, v_cache, pos, B, H, G, cap, cache_len, -1, \
                                                             new_pos, scale, out, raw, stats, nullptr, nullptr, nullptr, splits, \
                                                             least, stream)
#define EC_DSCORE_AUTO(W_, U_, DEEP_) else if (a.waves == W_ && a.unroll == U_ && a.deep == DEEP_) EC_DSCORE(W_, U_, DEEP_, false);
    const DecodeAuto a = decode_auto_shape(B * H, n, kRow, DT == EC_BF16, false);
    int rc;
    if (splits > 1) EC_DSCORE(4, 4, true, true);
    EC_DECODE_AUTO_SHAPES(EC_DSCORE_AUTO)
    else EC_DSCORE(4, 4, true, false);
#undef EC_DSCORE_AUTO
#undef EC_DSCORE
    if (rc != EC_OK) return rc;
    hipLaunchKernelGGL(freq_accumulate_kernel, dim3((n + kFreqRows - 1) / kFreqRows, B * G),
                       dim3(kFreqRows * kFreqParts), 0, stream, raw, stats, freq, H, G, n, cap);
    return status_from_hip(hipGetLastError());
}

int decode_score_dispatch(const void* q, const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                          int32_t* pos, float* freq, int B, int H, int G, int D, int cap, int cache_len,
                          int32_t new_pos, float scale, int dt, void* out, float* raw, float* stats,
                          hipStream_t stream)
{
#define EC_DSCORE_CASE(DT_, D_)                                                                                          \
    if (dt == DT_ && D == D_)                                                                                            \
        return launch_decode_score<DT_, D_>(q, k_new, v_new, k_cache, v_cache, pos, freq, B, H, G, cap, cache_len, new_pos, \
                                            scale, out, raw, stats, stream);
    EC_DSCORE_CASE(EC_BF16, 128)
    EC_DSCORE_CASE(EC_BF16, 64)
    EC_DSCORE_CASE(EC_F32, 128)
    EC_DSCORE_CASE(EC_F32, 64)
#undef EC_DSCORE_CASE
    return EC_EUNSUPPORTED;
}

// ec_evict_min in two launches: one workgroup per score group finds the least-mass row and closes the gap in the group's
// masses and positions, then two workgroups per (batch, head), one for K and one for V, move the rows behind it up by
// one.  The first launch is a chain of latencies (load, reduction, load, store), the second moves 2 * row bytes * rows
// behind the victim, half the cache for a victim anywhere.  What a round moves (256 rows of 256 bytes) is held in
// registers between the two sides of a barrier, all its loads in flight at once: threads past the end read the last
// element again instead of branching around the load, which would make every load wait for the one before it.
// Measured at H32 D128, bf16, victims anywhere, whole call (four caches in turn): B8 640 rows 42.8 -> 21.2 us, B16 900 rows
// 110 -> 58.5 us, B1 640 rows 13.2 -> 7.4 us from 512 rows a round, which went through scratch memory one by one.
// Threads x loads 256 x 8 to 1024 x 8 differ by 5 %; more than 8 loads cost small caches up to 30 %.

constexpr int kEvictMetaThreads = 1024;
constexpr int kEvictMetaUnroll = 4;
__global__ __launch_bounds__(kEvictMetaThreads) void evict_min_meta_kernel(float* freq, int32_t* pos,
                                                                          int32_t* __restrict__ victim, int cap, int len,
                                                                          int lo, int hi)
{
    constexpr int WAVES = kEvictMetaThreads / kWave;
    __shared__ unsigned long long sh_best[WAVES];
    const int bg = blockIdx.x, tid = threadIdx.x;
    float* f = freq + (size_t)bg * cap;
    int32_t* p = pos ? pos + (size_t)bg * cap : nullptr;
    // (mass, index) as one integer whose order is the fp32 order, -0 equal to +0, NaN of either sign behind +inf, the lower
    // index first
    unsigned long long best = ~0ull;
    for (int j = lo + tid; j <= hi; j += kEvictMetaThreads) {
        uint32_t u = __float_as_uint(f[j]);
        if (u == 0x80000000u) u = 0u;
        if ((u & 0x7fffffffu) > 0x7f800000u) u = 0x7fffffffu;
        u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
        best = min(best, ((unsigned long long)u << 32) | (uint32_t)j);
    }
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) best = min(best, __shfl_xor(best, off, kWave));
    if (tid % kWave == 0) sh_best[tid / kWave] = best;
    __syncthreads();
    best = sh_best[tid % WAVES];
#pragma unroll
    for (int off = 1; off < WAVES; off <<= 1) best = min(best, __shfl_xor(best, off, kWave));
    const int vic = (int)(uint32_t)best;
    if (tid == 0) victim[bg] = vic;

    const int total = len - 1 - vic;
    for (int c0 = 0; c0 < total; c0 += kEvictMetaThreads * kEvictMetaUnroll) {
        float fv[kEvictMetaUnroll];
        int32_t pv[kEvictMetaUnroll];
#pragma unroll
        for (int u = 0; u < kEvictMetaUnroll; ++u) {
            const int c = min(c0 + u * kEvictMetaThreads + tid, total - 1);
            fv[u] = f[vic + 1 + c];
            pv[u] = p ? p[vic + 1 + c] : 0;
        }
        arrived(fv);
        arrived(pv);
        __syncthreads();  // read completely before any of it is overwritten
#pragma unroll
        for (int u = 0; u < kEvictMetaUnroll; ++u) {
            const int c = c0 + u * kEvictMetaThreads + tid;
            if (c < total) {
                f[vic + c] = fv[u];
                if (p) p[vic + c] = pv[u];
            }
        }
        __syncthreads();  // and written before the next slab, which overlaps it by one element, is read
    }
}

constexpr int kEvictThreads = 512;
constexpr int kEvictUnroll = 8;
__global__ __launch_bounds__(kEvictThreads) void evict_min_rows_kernel(u32x4* k_cache, u32x4* v_cache,
                                                                       const int32_t* __restrict__ victim, int H, int G,
                                                                       int cap, int len, int lpr)
{
    const int bh = blockIdx.x, tid = threadIdx.x;
    const int b = bh / H, h = bh % H;
    const int vic = victim[(size_t)b * G + (G == 1 ? 0 : h)];
    u32x4* dst = (blockIdx.y == 0 ? k_cache : v_cache) + ((size_t)bh * cap + vic) * lpr;
    const u32x4* src = dst + lpr;
    const int total = (len - 1 - vic) * lpr;  // 16-byte chunks that move, in ascending address order
    for (int c0 = 0; c0 < total; c0 += kEvictThreads * kEvictUnroll) {
        u32x4 x[kEvictUnroll];
#pragma unroll
        for (int u = 0; u < kEvictUnroll; ++u) {
            const int c = min(c0 + u * kEvictThreads + tid, total - 1);
            x[u] = src[c];
        }
        arrived(x);
        __syncthreads();  // the slab is read completely before any of it is overwritten
#pragma unroll
        for (int u = 0; u < kEvictUnroll; ++u) {
            const int c = c0 + u * kEvictThreads + tid;
            if (c < total) dst[c] = x[u];
        }
        __syncthreads();  // and written before the next slab, which overlaps it by one row, is read
    }
}

int evict_min_dispatch(void* k_cache, void* v_cache, int32_t* pos, float* freq, int B, int H, int G, int D, int cap,
                       int len, int protect_first, int protect_recent, int dt, int32_t* victim, hipStream_t stream)
{
    const int lpr = D * (dt == EC_F32 ? 4 : 2) / 16;
    hipLaunchKernelGGL(evict_min_meta_kernel, dim3(B * G), dim3(kEvictMetaThreads), 0, stream, freq, pos, victim, cap, len,
                       protect_first, len - 1 - protect_recent);
    int rc = status_from_hip(hipGetLastError());
    if (rc != EC_OK) return rc;
    hipLaunchKernelGGL(evict_min_rows_kernel, dim3(B * H, 2), dim3(kEvictThreads), 0, stream, (u32x4*)k_cache,
                       (u32x4*)v_cache, victim, H, G, cap, len, lpr);
    return status_from_hip(hipGetLastError());
}

}  // namespace ec
