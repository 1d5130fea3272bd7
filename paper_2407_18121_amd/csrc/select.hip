// ec_select_anchors: per (batch, score group) choice of the N_I highest-scoring
// positions (Sec. 3.3), protected first/last positions always kept (Sec. 4.1),
// equal scores resolved toward the lower position, output ascending.
//
// One workgroup per problem.  Scores are mapped to 32-bit keys whose unsigned order equals the fp32 order (-0 folded onto +0).  A
// radix select from the top finds the key of the last selected element and how many elements equal to it are needed; an
// ordered sweep over the positions then emits the selected indices in ascending order, taking equal keys
// lowest-position-first.  Pure integer work: the result is bit-exact by construction.
#include <type_traits>

#include "ec_common.h"

namespace ec {

// Least and largest value of the lane's row of 16, in every lane of it.
__device__ __forceinline__ void row_range(uint32_t& lo, uint32_t& hi)
{
    auto step = [&](auto ctrl) __attribute__((always_inline)) {
        lo = min(lo, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, ctrl.value, 0xf, 0xf, true));
        hi = max(hi, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, ctrl.value, 0xf, 0xf, true));
    };
    step(std::integral_constant<int, kDppQuadXor1>{});
    step(std::integral_constant<int, kDppQuadXor2>{});
    step(std::integral_constant<int, kDppRowHalfMirror>{});
    step(std::integral_constant<int, kDppRowMirror>{});
}

// Sum over the lanes up to and including this one.
__device__ __forceinline__ int prefix_sum(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // the last lane of a row to the next one (rows 1, 3)
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // lane 31 to rows 2, 3
    return x;
}

__device__ __forceinline__ uint32_t score_key(float s)
{
    uint32_t u = __float_as_uint(s);
    if (u == 0x80000000u) u = 0u;  // -0 compares equal to +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// What the two kernels make of their arguments.  Ragged batches: seq_len[b] positions and n_anchor_b[b] anchors for batch element b
// (both clamped), rows of score and anchor_idx stay T_max and n_max apart.
struct SelectProblem {
    int T, n_anchor, free_lo, free_hi, n_free;  // unprotected: [free_lo, free_hi)
    __device__ __forceinline__ SelectProblem(int b, int T_max, int n_max, int protect_first, int protect_last,
                                             const int32_t* __restrict__ seq_len, const int32_t* __restrict__ n_anchor_b)
    {
        T = ragged_rows(seq_len, b, T_max);
        n_anchor = n_anchor_b ? min(max(n_anchor_b[b], 0), min(T, n_max)) : n_max;
        protect_first = min(protect_first, n_anchor);
        protect_last = min(protect_last, n_anchor - protect_first);
        free_lo = protect_first, free_hi = T - protect_last;
        n_free = n_anchor - protect_first - protect_last;
    }
};

// Up to THREADS * KEYS positions: a thread holds KEYS consecutive ones in registers.
// Bound: a chain of short steps with a barrier behind each.  The first digit starts at the highest bit in which two keys differ,
// which spreads them over its 256 values whatever their range (a fixed one puts usual scores on few of them); the histogram has
// copies for the lanes of a wave, whose neighbouring positions tend to score alike and would wait for each other's
// atomics; as soon as one wave can hold the keys that share the digits found so far, every wave ranks them by itself; and all
// positions are emitted in one sweep.  As many threads as there is work for: a barrier and the instructions between two
// cost more the more waves share a SIMD.
// us per call (graph replay, scores like a prompt's), four fixed digits over keys in LDS by 1024 threads -> this: T128 5.2 -> 4.7,
// T1024 6.3 -> 5.0, 32 groups of T2048 8.5 -> 5.8, T4096 12.1 -> 6.4, 16 of T8192 20.4 -> 8.9.  One / four / eight copies: T256
// 4.8 / 5.2 / 5.6, T2048 6.5 / 5.8 / 5.8, T8192 13.1 / 9.4 / 8.9.  Sixteen keys a thread and a quarter of the threads: T1024 7.8.
template <int THREADS, int KEYS>
__global__ __launch_bounds__(THREADS) void select_anchors_kernel(
    const float* __restrict__ score, int T_max, int n_max, int protect_first, int protect_last,
    int32_t* __restrict__ anchor_idx, const int32_t* __restrict__ seq_len, const int32_t* __restrict__ n_anchor_b, int G)
{
    constexpr int WAVES = THREADS / kWave;
    constexpr int kCopies = THREADS * KEYS <= 256 ? 1 : THREADS * KEYS <= 2048 ? 4 : 8;
    __shared__ int hist[kCopies][256 + 1];
    __shared__ uint32_t wave_lo[WAVES], wave_hi[WAVES];
    __shared__ int wave_tot[WAVES];
    __shared__ __align__(16) uint32_t few[kWave];  // keys that share all digits found so far, once one wave can hold them
    __shared__ uint32_t sh_prefix;
    __shared__ int sh_need, sh_count, sh_few;

    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const SelectProblem p(blockIdx.x / G, T_max, n_max, protect_first, protect_last, seq_len, n_anchor_b);
    if (p.T == 0 || p.n_anchor == 0) return;  // whole workgroup
    const float* s = score + (size_t)blockIdx.x * T_max;
    int32_t* dst = anchor_idx + (size_t)blockIdx.x * n_max;

    const int t0 = tid * KEYS;
    uint32_t key[KEYS], lo = ~0u, hi = 0u;  // lo, hi: of the unprotected keys
    static_assert(KEYS % 4 == 0, "whole 16-byte chunks");
    if (((uintptr_t)s & 15) == 0 && t0 + KEYS <= p.T) {
#pragma unroll
        for (int i = 0; i < KEYS; i += 4) {
            const float4 x = *reinterpret_cast<const float4*>(s + t0 + i);
            key[i] = score_key(x.x), key[i + 1] = score_key(x.y), key[i + 2] = score_key(x.z), key[i + 3] = score_key(x.w);
        }
    } else {
#pragma unroll
        for (int i = 0; i < KEYS; ++i) key[i] = score_key(s[min(t0 + i, p.T - 1)]);
    }
    auto is_free = [&](int i) { return t0 + i >= p.free_lo && t0 + i < p.free_hi; };
#pragma unroll
    for (int i = 0; i < KEYS; ++i)
        if (is_free(i)) lo = min(lo, key[i]), hi = max(hi, key[i]);
    row_range(lo, hi);
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, 16, kWave)), hi = max(hi, (uint32_t)__shfl_xor((int)hi, 16, kWave));
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, 32, kWave)), hi = max(hi, (uint32_t)__shfl_xor((int)hi, 32, kWave));
    if (lane == 0) wave_lo[wave] = lo, wave_hi[wave] = hi;
    for (int i = tid; i < kCopies * 257; i += THREADS) hist[0][i] = 0;
    if (tid < kWave) few[tid] = 0;
    if (tid == 0) sh_few = 0;
    __syncthreads();
    lo = wave_lo[lane % WAVES], hi = wave_hi[lane % WAVES];  // 1, 4, 8 or 16 of them: a row of lanes holds them all
    row_range(lo, hi);

    // ---- radix select of the n_free-th largest unprotected key ----
    uint32_t kth = lo;        // key of the last selected unprotected element
    int need_eq = p.n_free;   // how many elements equal to kth are selected (lowest positions)
    if (p.n_free > 0 && lo != hi) {
        int top = 32 - __clz((int)(lo ^ hi));  // the bits of the keys below `top` are still open
        uint32_t prefix = top < 32 ? hi >> top << top : 0u;
        int need = p.n_free;
        for (;;) {
            const int shift = max(top - 8, 0);
            const uint32_t known = top < 32 ? ~0u << top : 0u;
#pragma unroll
            for (int i = 0; i < KEYS; ++i)
                if (is_free(i) && (key[i] & known) == prefix) atomicAdd(&hist[lane % kCopies][(key[i] & ~known) >> shift], 1);
            __syncthreads();
            // One wave finds the digit: lane l owns digits 4l .. 4l + 3; the candidates above them are those of the lanes above,
            // and the four digits of a lane are walked in registers.
            if (wave == 0) {
                int c[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    c[i] = 0;
#pragma unroll
                    for (int k = 0; k < kCopies; ++k) {
                        c[i] += hist[k][4 * lane + i];
                        hist[k][4 * lane + i] = 0;  // ready for the next digit
                    }
                }
                const int upto = prefix_sum(c[0] + c[1] + c[2] + c[3]);
                int above = __builtin_amdgcn_readlane(upto, kWave - 1) - upto;
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    if (above < need && need <= above + c[i]) {  // exactly one digit satisfies this
                        sh_prefix = prefix | ((uint32_t)(4 * lane + i) << shift);
                        sh_need = need - above;
                        sh_count = c[i];
                    }
                    above += c[i];
                }
            }
            __syncthreads();
            prefix = sh_prefix, need = sh_need, top = shift;
            if (top == 0 || sh_count <= kWave) break;
        }
        kth = prefix, need_eq = need;
        if (top > 0) {
            const uint32_t known = ~0u << top;
#pragma unroll
            for (int i = 0; i < KEYS; ++i)
                if (is_free(i) && (key[i] & known) == prefix) few[atomicAdd(&sh_few, 1)] = key[i];
            __syncthreads();
            // A lane each: the keys above it; the least key with fewer than `need` above it is the threshold.
            const int count = sh_count;
            const uint32_t mine = few[min(lane, count - 1)];
            int above = 0;
            for (int i = 0; i < count; i += 4) {
                const uint4 x = *reinterpret_cast<const uint4*>(&few[i]);  // 0 behind the last one
                above += (x.x > mine) + (x.y > mine) + (x.z > mine) + (x.w > mine);
            }
            uint32_t least = above < need ? mine : ~0u, unused = 0u;
            row_range(least, unused);
            least = min(least, (uint32_t)__shfl_xor((int)least, 16, kWave));
            kth = min(least, (uint32_t)__shfl_xor((int)least, 32, kWave));
            need_eq = need - __builtin_amdgcn_readlane(above, __ffsll((unsigned long long)__ballot(mine == kth)) - 1);
        }
    }

    // ---- ordered emission ----
    // One scan carries two counts, packed into one word: elements that are kept outright (protected or above the threshold
    // key) and elements equal to it.  Of the equal ones the first need_eq are kept, so an element's output slot is
    // (kept outright before it) + min(equal before it, need_eq).
    bool keep[KEYS], eq[KEYS];
    int mine = 0;
#pragma unroll
    for (int i = 0; i < KEYS; ++i) {
        const bool open = is_free(i) && p.n_free > 0;
        keep[i] = t0 + i < p.T && (!is_free(i) || (open && key[i] > kth));
        eq[i] = open && key[i] == kth;
        mine += (int)keep[i] + ((int)eq[i] << 16);
    }
    const int upto = prefix_sum(mine);
    if (lane == kWave - 1) wave_tot[wave] = upto;
    __syncthreads();
    const int waves = prefix_sum(lane < WAVES ? wave_tot[lane % WAVES] : 0);
    const int before = upto - mine + (wave > 0 ? __builtin_amdgcn_readlane(waves, max(wave - 1, 0)) : 0);
    int kept = before & 0xffff, equal = before >> 16;
#pragma unroll
    for (int i = 0; i < KEYS; ++i) {
        const int o = kept + min(equal, need_eq);
        if ((keep[i] || (eq[i] && equal < need_eq)) && o < p.n_anchor) dst[o] = t0 + i;
        kept += keep[i], equal += eq[i];
    }
}

// More positions: the scores are read again for every digit and for the sweep.
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;
__global__ __launch_bounds__(kSelThreads) void select_anchors_long_kernel(
    const float* __restrict__ score, int T_max, int n_max, int protect_first, int protect_last,
    int32_t* __restrict__ anchor_idx, const int32_t* __restrict__ seq_len, const int32_t* __restrict__ n_anchor_b, int G)
{
    __shared__ int hist[256];
    __shared__ int wave_tot[2][kSelWaves];  // two sets, used in turn: one barrier per sweep step
    __shared__ uint32_t sh_prefix;
    __shared__ int sh_need;

    const int tid = threadIdx.x;
    const int lane = tid % kWave, wave = tid / kWave;
    const SelectProblem p(blockIdx.x / G, T_max, n_max, protect_first, protect_last, seq_len, n_anchor_b);
    const int T = p.T, n_anchor = p.n_anchor, free_lo = p.free_lo, free_hi = p.free_hi, n_free = p.n_free;
    if (T == 0 || n_anchor == 0) return;  // whole workgroup
    const float* s = score + (size_t)blockIdx.x * T_max;
    int32_t* dst = anchor_idx + (size_t)blockIdx.x * n_max;
    if (tid < 256) hist[tid] = 0;
    if (tid == 0) {
        sh_prefix = 0u;
        sh_need = n_free;
    }
    __syncthreads();

    // ---- radix select of the n_free-th largest unprotected key ----
    if (n_free > 0) {
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
            const uint32_t hi_mask = (pass == 0) ? 0u : (0xffffffffu << (shift + 8));
            const uint32_t prefix = sh_prefix;
            const int need = sh_need;
            for (int t = free_lo + tid; t < free_hi; t += kSelThreads) {
                const uint32_t key = score_key(s[t]);
                if ((key & hi_mask) == prefix) atomicAdd(&hist[(key >> shift) & 0xffu], 1);
            }
            __syncthreads();
            // One wave finds the digit: lane l owns digits 4l..4l+3; a shuffle scan from the top gives the
            // number of candidates in the lanes above, and the four digits of a lane are walked in registers.
            if (wave == 0) {
                int c[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) c[i] = hist[4 * lane + i];
#pragma unroll
                for (int i = 0; i < 4; ++i) hist[4 * lane + i] = 0;  // ready for the next pass
                const int mine = c[0] + c[1] + c[2] + c[3];
                int incl = mine;  // candidates in lanes >= this one
#pragma unroll
                for (int off = 1; off < kWave; off <<= 1) {
                    const int x = __shfl_down(incl, off, kWave);
                    if (lane + off < kWave) incl += x;
                }
                int above = incl - mine;  // candidates with a digit above this lane's four
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    if (above < need && need <= above + c[i]) {  // exactly one digit satisfies this
                        sh_prefix = prefix | ((uint32_t)(4 * lane + i) << shift);
                        sh_need = need - above;
                    }
                    above += c[i];
                }
            }
            __syncthreads();
        }
    }
    const uint32_t kth = sh_prefix;  // key of the last selected unprotected element
    const int need_eq = sh_need;     // how many elements equal to kth are selected (lowest positions)

    // ---- ordered emission ----
    // One workgroup scan per 1024 positions carries two counts, packed into one word: elements that are
    // kept outright (protected or above the threshold key) and elements equal to it.  Of the equal ones the
    // first need_eq are kept, so an element's output slot is (kept outright before it) + min(equal before
    // it, need_eq).
    int base_keep = 0, base_eq = 0, set = 0;
    for (int t0 = 0; t0 < T; t0 += kSelThreads, set ^= 1) {
        const int t = t0 + tid;
        bool keep = false, eq = false;
        if (t < T) {
            keep = (t < free_lo) || (t >= free_hi);
            if (!keep && n_free > 0) {
                const uint32_t key = score_key(s[t]);
                keep = key > kth;
                eq = key == kth;
            }
        }
        const unsigned long long ball_keep = __ballot(keep), ball_eq = __ballot(eq);
        const unsigned long long below = (1ull << lane) - 1ull;
        if (lane == 0) wave_tot[set][wave] = __popcll(ball_keep) | (__popcll(ball_eq) << 16);
        __syncthreads();
        int before = 0, tot = 0;
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w) {
            const int c = wave_tot[set][w];
            before += (w < wave) ? c : 0;
            tot += c;
        }
        const int keep_before = base_keep + (before & 0xffff) + __popcll(ball_keep & below);
        const int eq_before = base_eq + (before >> 16) + __popcll(ball_eq & below);
        const int o = keep_before + min(eq_before, need_eq);
        if ((keep || (eq && eq_before < need_eq)) && o < n_anchor) dst[o] = t;
        base_keep += tot & 0xffff;
        base_eq += tot >> 16;
    }
}

int select_dispatch(const float* score, int B, int G, int T, int n_anchor, int protect_first,
                    int protect_last, int32_t* anchor_idx, const int32_t* seq_len, const int32_t* n_anchor_b,
                    hipStream_t stream)
{
#define EC_SELECT(THREADS_, KEYS_)                                                                                         \
    if (T <= THREADS_ * KEYS_) {                                                                                           \
        hipLaunchKernelGGL((select_anchors_kernel<THREADS_, KEYS_>), dim3(B * G), dim3(THREADS_), 0, stream, score, T, n_anchor, \
                           protect_first, protect_last, anchor_idx, seq_len, n_anchor_b, G);                               \
        return status_from_hip(hipGetLastError());                                                                        \
    }
    EC_SELECT(64, 4)
    EC_SELECT(256, 4)
    EC_SELECT(512, 4)
    EC_SELECT(1024, 4)
    EC_SELECT(1024, 8)
#undef EC_SELECT
    hipLaunchKernelGGL(select_anchors_long_kernel, dim3(B * G), dim3(kSelThreads), 0, stream, score, T, n_anchor, protect_first,
                       protect_last, anchor_idx, seq_len, n_anchor_b, G);
    return status_from_hip(hipGetLastError());
}

// ------------------------------------------------------------------ retention test on the device
// Per-sequence bookkeeping of a ragged generation loop (Alg. 1's del_num and fix_idx in integer arithmetic,
// the same rules as the host function ec_evict_index), one thread per batch element.
__global__ __launch_bounds__(256) void retention_step_kernel(int32_t* __restrict__ n_seen_b,
                                                             int32_t* __restrict__ cache_len_b,
                                                             int32_t* __restrict__ evict_idx_b,
                                                             int32_t* __restrict__ new_pos_b,
                                                             int32_t* __restrict__ pending_b, int B, int gamma_num,
                                                             int gamma_den, int budget_mode, int fixed_len,
                                                             int trunc_mode, int recent, int n_tl, int protect_first,
                                                             int flush_only)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    int len = cache_len_b[b];
    if (pending_b[b]) {  // the step prepared by the previous call has run: a row was appended, maybe one removed
        len += (evict_idx_b[b] < 0) ? 1 : 0;
        pending_b[b] = 0;
    }
    if (!flush_only) {
        const long long seen = (long long)n_seen_b[b] + 1;
        const long long after = (long long)len + 1;
        long long keep;
        if (budget_mode == EC_BUDGET_RATIO) {
            const long long prod = (long long)gamma_num * seen;
            keep = prod / gamma_den + ((prod % gamma_den) ? 1 : 0);
        } else {
            keep = fixed_len;
        }
        long long victim = -1;
        if (after > keep) {
            victim = (trunc_mode == EC_TRUNC_RECENT) ? after - 1 - recent : (long long)n_tl;
            if (victim < protect_first) victim = protect_first;
            if (victim >= after - 1) victim = -1;
        }
        n_seen_b[b] = (int32_t)seen;
        evict_idx_b[b] = (int32_t)victim;
        new_pos_b[b] = (int32_t)(seen - 1);
        pending_b[b] = 1;
    }
    cache_len_b[b] = len;
}

int retention_step_launch(int32_t* n_seen_b, int32_t* cache_len_b, int32_t* evict_idx_b, int32_t* new_pos_b,
                          int32_t* pending_b, int B, int gamma_num, int gamma_den, int budget_mode, int fixed_len,
                          int trunc_mode, int recent, int n_tl, int protect_first, int flush_only, hipStream_t stream)
{
    hipLaunchKernelGGL(retention_step_kernel, dim3((B + 255) / 256), dim3(256), 0, stream, n_seen_b, cache_len_b,
                       evict_idx_b, new_pos_b, pending_b, B, gamma_num, gamma_den, budget_mode, fixed_len, trunc_mode,
                       recent, n_tl, protect_first, flush_only);
    return status_from_hip(hipGetLastError());
}

}  // namespace ec
