// ec_merge_compact / ec_remerge_compact: bucket division (Sec. 3.3, Eq. 2), cache merging
// (Eq. 3) and compaction (Alg. 1's gather) in one pass over K and V.
//
// Every prompt K/V row is read once, every cache row written once: HBM-bound where the launch fills the chip, bound by the
// longest chain of loads that wait for each other where it does not.  Buckets are contiguous position ranges, so the rows of
// bucket j are one contiguous slab of memory.  A group of LPR = row_bytes/16 lanes streams rows with 16-byte loads,
// accumulates in fp32, divides by the count once and stores the row.
// Importance scores put most anchors next to each other and leave buckets of tens to thousands of rows between the others, so
//   - a workgroup's buckets are runs of a wave's width (1 KB of single rows) from all over the head: with one stretch of the
//     head each, a few workgroups had all the long buckets.  Runs of 4 / one stretch of 16 buckets, bf16 D128, us: B1 H8 T512 half
//     the rows kept 8.0 / 10.3, B8 T1664 54 % kept 76 / 87, B16 T8192 a tenth kept 425 / 464; anchors every second row, B16 T4096, 319 / 315;
//   - buckets are dealt out in pieces of at most an even share of the workgroup's rows, two rounds of pieces at the most.  The
//     smallest share of 4 / 8 / 16 / 32 rows: B1 H32 T1024 10.8 / 10.8 / 10.8 / 10.5 us, B1 H8 T512 6.6 / 6.6 / 7.2 / 5.9, B8 H32 T2048
//     63.4 / 63.6 / 65.8 / 67, B16 H32 T8192 420 / 422 / 430 / 454, the same with random anchors 449 / 459 / 464 / 481;
//   - loads stand under wave-uniform conditions, or have no others behind them;
//   - short buckets are bound by vector instructions, of which rounding and dividing had half: rows are rounded by the conversion
//     instruction and divided by products where those give the same bits (B8 T1664 76.0 -> 68.7 -> 68.1 us, B16 T4096 every second
//     row 320 -> 308 -> 305).
// us per call, against one bucket per lane group with conditional loads and buckets of more than 128 rows summed by the workgroup,
// prompt-like anchors: B1 H32 T1024 12.8 -> 10.8, B1 H8 T512 7.2 -> 6.6, B8 H32 T2048 70.5 -> 63.4, B16 H40 T624 65.5 -> 60.3, B16 H32 T8192
// 433 -> 420 (5.6 TB/s), fp32 D64 B8 H8 T2048 26.6 -> 20.1.  Random anchors: B1 T1024 half kept 9.06 -> 8.95, B8 T2048 a quarter
// 62.3 -> 60.3, half 75.2 -> 78.2, B16 T4096 half 301 -> 309, T8192 a tenth 418 -> 449.  Every second row: B16 T4096 286 -> 296, bf16 D64
// B8 T4096 71.7 -> 81.5: every bucket is alike and nothing is gained by what the others need.
#include "ec_common.h"

namespace ec {

constexpr int kMergeThreads = 256;
constexpr int kMergeUnroll = 8;  // rows of K and of V in flight per bucket (16 loads per lane)
// Rows up to which buckets are not divided if no other one of the workgroup has more (8 / 16: scattered anchors, which have many
// buckets of 9 to 16 rows, B8 T2048 77.9 / 63.7 us; prompt-like ones alike).
constexpr int kMergeWhole = 16;
constexpr int kMergePiece = 4;   // the smallest share
constexpr int kMergeAssign = 128;  // buckets with more rows have their assignment written by the whole workgroup
constexpr int kMergeMostRows = 1 << 30;

// Inclusive bounds of bucket j for ascending anchors a[0..n), t = a[j].  Clamped so that a
// malformed anchor list can never index outside [0,T).
__device__ __forceinline__ void bucket_bounds(const int32_t* __restrict__ a, int j, int n, int T,
                                              int& t, int& lo, int& hi)
{
    t = a[j];
    const int before = a[max(j - 1, 0)], behind = a[min(j + 1, n - 1)];
    lo = (j == 0) ? 0 : ((before + t) >> 1) + 1;
    hi = (j == n - 1) ? T - 1 : ((t + behind) >> 1);
    lo = max(lo, 0);
    hi = min(hi, T - 1);
}

// Rows of K and V on their way.
template <int N_> struct Rows {
    static constexpr int N = N_;
    u32x4 k[N], v[N];
    int w[N];
};

// fp32 -> bf16 by the conversion instruction, two values at a time; the same bits as f32_to_bf16() for all 2^32 values.
template <int DT> __device__ __forceinline__ uint4 round_row(const float* f)
{
    if constexpr (DT == EC_F32) return pack<DT>(f);
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    u32x4 c;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        c[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{f[2 * i], f[2 * i + 1]}), bf16x2));
    return __builtin_bit_cast(uint4, c);
}

// x / n rounded once, for n = 2 .. kMergeCount and |x| = kMergeLeast .. largest, unit being 1 / n rounded: the first product is off by
// an ulp or two, what it leaves of x is exact, and adding that part rounds as a division does.  Compared with the division for all
// 2^23 significands and every such n.  3 instructions for 10.
constexpr int kMergeCount = 1 << 16;
constexpr float kMergeLeast = 0x1p-90f;
__device__ __forceinline__ float quotient(float x, float n, float unit)
{
    const float q = x * unit;
    return fmaf(fmaf(-n, q, x), unit, q);
}

// Inclusive sums over the first N lanes of a wave, N = 8, 16 or 32; they saturate at kMergeMostRows.
template <int N> __device__ __forceinline__ int bucket_scan(int x)
{
    auto add = [&](int y) __attribute__((always_inline)) { x = min(x + y, kMergeMostRows); };
    // shifts inside a row of 16 lanes bring zeros in
    add(__builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true));
    add(__builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true));
    add(__builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true));
    if (N >= 16) add(__builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true));
    if (N >= 32) {
        const int first_row = __builtin_amdgcn_readlane(x, 15);
        add(threadIdx.x % kWave >= 16 ? first_row : 0);
    }
    return x;
}

// WEIGHTED: every source row t carries an integer weight w_t (the number of original tokens it already
// stands for, when rows of an earlier merge are merged again); the cache row is sum w_t x_t / sum w_t
// and counts receives sum w_t.  Without it every row weighs 1 (Eq. 3).  src_rows is the distance in rows
// between the heads of k/v (>= T); src_pos, if given, maps a source row to its original position.
template <int DT, int D, bool WEIGHTED>
__global__ __launch_bounds__(kMergeThreads, WEIGHTED ? 3 : 4) void merge_compact_kernel(
    const u32x4* __restrict__ k, const u32x4* __restrict__ v, const int32_t* __restrict__ anchor_idx,
    const int32_t* __restrict__ weights, const int32_t* __restrict__ src_pos,
    uint4* __restrict__ k_cache, uint4* __restrict__ v_cache, int32_t* __restrict__ counts,
    int32_t* __restrict__ assign, int32_t* __restrict__ pos, int H, int G, int T_max, int src_rows, int n_max,
    int cap, int evict_only, const int32_t* __restrict__ seq_len, const int32_t* __restrict__ n_anchor_b)
{
    constexpr int LPR = D * Elem<DT>::kBytes / 16;
    constexpr int EPL = Elem<DT>::kPerChunk;
    constexpr int GROUPS = kMergeThreads / LPR;
    constexpr int RUN = kWave / LPR;        // neighbouring buckets of a wave
    constexpr int PIECES = 2 * GROUPS;  // at most: one per bucket and one more per full share of the rows
    __shared__ float sh_part[PIECES][LPR * EPL * 2];
    __shared__ int sh_wsum[PIECES];
    __shared__ int4 sh_bucket[GROUPS];  // first and last row, pieces, pieces up to and including it

    const int bh = blockIdx.y;
    const int b = bh / H, h = bh % H;
    const int tid = threadIdx.x;
    const int sub = tid % LPR, grp = tid / LPR;
    // Long and short buckets sit at the same chunk numbers in every head, and workgroups go to the 8
    // XCDs round-robin by linear id: rotating the chunk number by the head index keeps the heavy chunks
    // from piling onto the same XCDs.
    const int chunk = (blockIdx.x + blockIdx.y) % gridDim.x;
    // ragged batches: batch element b has T positions and n_anchor anchors; array rows stay T_max / n_max apart
    const int T = ragged_rows(seq_len, b, T_max);
    const int n_anchor = n_anchor_b ? min(max(n_anchor_b[b], 0), min(T, n_max)) : n_max;
    const int n_chunks = (n_anchor + GROUPS - 1) / GROUPS;
    if (chunk >= n_chunks) return;  // whole workgroup
    // the workgroup's buckets: ascending, so that those the head has come first
    auto bucket = [&](int i) __attribute__((always_inline)) { return (i / RUN * n_chunks + chunk) * RUN + i % RUN; };

    const size_t bg = (size_t)b * G + (G == 1 ? 0 : h);
    const int32_t* a = anchor_idx + bg * n_max;
    const int32_t* wrow = WEIGHTED ? weights + bg * T_max : nullptr;
    const bool owner = (G == H || h == 0);  // writes the bookkeeping of its score group
    // K and V of a bucket are streamed side by side: two independent load streams per lane
    const char* src_k = (const char*)(k + (size_t)bh * src_rows * LPR);
    const char* src_v = (const char*)(v + (size_t)bh * src_rows * LPR);

    asm volatile("" ::"s"(src_k), "s"(src_v), "s"(k_cache), "s"(v_cache));  // arguments in scalar registers before the loads

    // ---- the buckets of the workgroup: lane l of every wave holds bucket number l of them, and beside it (loaded together,
    // which costs no time) its lane group's own, for the usual case that none is divided ----
    const int lane = tid % kWave;
    int at, lo, hi, own_at, own_lo, own_hi;
    const int j = lane < GROUPS ? bucket(lane) : n_anchor;
    const int n_here = __popcll(__ballot(j < n_anchor));
    const bool own = bucket(grp) < n_anchor;
    bucket_bounds(a, min(bucket(grp), n_anchor - 1), n_anchor, T, own_at, own_lo, own_hi);
    bucket_bounds(a, min(j, n_anchor - 1), n_anchor, T, at, lo, hi);
    if (!own) own_lo = 0, own_hi = -1;
    if (lane >= n_here) at = lo = 0, hi = -1;
    const int blo = lo, bhi = hi;  // the bucket, for the assignment
    if (evict_only) {  // eviction-only ablation: the anchor's own row
        if (own) own_lo = own_hi = min(max(own_at, 0), T - 1);
        if (lane < n_here) lo = hi = min(max(at, 0), T - 1);
    }
    // Pieces: a bucket of more rows than an even share of the workgroup's is divided.  All sums saturate, so that a malformed
    // anchor list, whose buckets overlap, cannot wrap them.
    const int rows = max(hi - lo + 1, 0);
    int n_parts = lane < n_here ? 1 : 0, parts_end = 0;  // pieces of the lane's bucket; of the ones up to and including it
    int n_pieces = n_here;
    if (__any(rows > kMergeWhole)) {  // the same in every wave
        const int all_rows = __builtin_amdgcn_readlane(bucket_scan<GROUPS>(min(rows, kMergeMostRows)), GROUPS - 1);
        const int share = ((all_rows + GROUPS - 1) / GROUPS + kMergePiece - 1) / kMergePiece * kMergePiece;
        if (lane < n_here) n_parts = max((rows + share - 1) / share, 1);
        parts_end = bucket_scan<GROUPS>(n_parts);
        n_pieces = __builtin_amdgcn_readlane(parts_end, GROUPS - 1);
        // every wave leaves the same values and needs no other wave's: from here on they cost no registers
        if (lane < GROUPS) sh_bucket[lane] = make_int4(lo, hi, n_parts, parts_end);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }

    if (owner && tid < n_here) {  // bookkeeping of the score group, one store for the workgroup's buckets
        if (!WEIGHTED && counts) counts[bg * n_max + j] = hi - lo + 1;
        if (pos) pos[bg * cap + j] = src_pos ? src_pos[bg * T_max + min(max(at, 0), T - 1)] : at;
    }

    if (owner && assign) {
        // short buckets by their lane groups, long ones by the workgroup
        const int b_lo = __shfl(blo, grp, kWave), b_hi = __shfl(bhi, grp, kWave), row = __shfl(lo, grp, kWave);
        if (grp < n_here && b_hi - b_lo < kMergeAssign)
            for (int t = b_lo + sub; t <= b_hi; t += LPR) assign[bg * T_max + t] = (!evict_only || t == row) ? bucket(grp) : -1;
        for (unsigned long long todo = __ballot(bhi - blo >= kMergeAssign); todo != 0; todo &= todo - 1) {
            const int i = __ffsll((long long)todo) - 1;
            const int l_lo = __shfl(blo, i, kWave), l_hi = __shfl(bhi, i, kWave), l_row = __shfl(lo, i, kWave);
            for (int t = l_lo + tid; t <= l_hi; t += kMergeThreads)
                assign[bg * T_max + t] = (!evict_only || t == l_row) ? bucket(i) : -1;
        }
    }

    float acc_k[EPL], acc_v[EPL];
    int wsum;
    u32x4 row_k, row_v;  // of a bucket of one row, as they were read: the sum of a signalling NaN and nothing is a quiet one
    // Rows first, first + step, ... <= last of every lane group; `most` rows of the group of the wave that has the most.  All
    // loads stand under wave-uniform conditions and are the same for every way through a loop: behind a load that some lanes
    // or some ways skip, a wait for one row is a wait for all of them, which took one trip to memory per row.  Groups that
    // have fewer rows than their neighbours read their last one again, out of the cache.  use_w: rows carry their weights.
    auto stream = [&](int first, int last, int step, int most, bool use_w) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc_k[e] = acc_v[e] = -0.f;  // leaves what is added to it as it is, -0 too
        wsum = 0;
        constexpr uint32_t kMinus = DT == EC_F32 ? 0x80000000u : 0x80008000u;
        const u32x4 nothing = {kMinus, kMinus, kMinus, kMinus};
        int r_load = first, r_use = first;
        auto load = [&](auto& x) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < x.N; ++u) {
                const int r = max(min(r_load, last), 0);  // an empty bucket of a malformed list reads row 0 and drops it
                const ptrdiff_t at = ((ptrdiff_t)r * LPR + sub) * 16;
                if (WEIGHTED) x.w[u] = wrow[r];
                x.k[u] = __builtin_nontemporal_load((const u32x4*)(src_k + at));
                x.v[u] = __builtin_nontemporal_load((const u32x4*)(src_v + at));
                r_load += step;
                asm volatile("" : "+v"(r_load));  // the next row's address is formed when it is needed
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto use = [&](auto& x, int n) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < x.N; ++u) {
                if (u > 0 && u >= n) return;  // uniform
                const bool in = r_use <= last;
                float xk[EPL], xv[EPL];
                unpack<DT>(__builtin_bit_cast(uint4, in ? x.k[u] : nothing), xk);
                unpack<DT>(__builtin_bit_cast(uint4, in ? x.v[u] : nothing), xv);
                if (WEIGHTED) {
                    const int wt = max(x.w[u], 1);
                    wsum += in ? wt : 0;
                    const float w = use_w ? (float)wt : 1.f;
#pragma unroll
                    for (int e = 0; e < EPL; ++e) {
                        acc_k[e] = fmaf(w, xk[e], acc_k[e]);
                        acc_v[e] = fmaf(w, xv[e], acc_v[e]);
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < EPL; ++e) {
                        acc_k[e] += xk[e];
                        acc_v[e] += xv[e];
                    }
                }
                r_use += step;
                asm volatile("" : "+v"(r_use));
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (most <= 1) {
            Rows<1> x;
            load(x);
            use(x, 1);
            row_k = x.k[0], row_v = x.v[0];
        } else if (most <= kMergeUnroll) {
            // nothing is loaded behind these, so that each lane group can leave out the rows it does not have
            Rows<kMergeUnroll> x;
#pragma unroll
            for (int u = 0; u < kMergeUnroll; ++u) {
                const int r = first + u * step;
                if (r <= last) {
                    const ptrdiff_t at = ((ptrdiff_t)r * LPR + sub) * 16;
                    if (WEIGHTED) x.w[u] = wrow[r];
                    x.k[u] = __builtin_nontemporal_load((const u32x4*)(src_k + at));
                    x.v[u] = __builtin_nontemporal_load((const u32x4*)(src_v + at));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            use(x, most);
            row_k = x.k[0], row_v = x.v[0];
        } else {
            constexpr int N = kMergeUnroll / 2;
            Rows<N> xa, xb;
            load(xa);
            int left = (most + N - 1) / N;  // blocks that have not been used
            for (; left > 2; left -= 2) {
                load(xb);
                use(xa, N);
                load(xa);
                use(xb, N);
            }
            if (left == 2) {
                load(xb);
                use(xa, N);
                use(xb, N);
                row_k = xb.k[N - 1], row_v = xb.v[N - 1];  // a bucket of one row has it in every slot
            } else {
                use(xa, N);
                row_k = xa.k[N - 1], row_v = xa.v[N - 1];
            }
        }
    };
    // divide by the count, round once, store cache row jj
    auto finish = [&](int jj, int n_rows, int w_total) __attribute__((always_inline)) {
        const int count = WEIGHTED ? w_total : n_rows;
        if (n_rows > 1) {
            const float cf = (float)count;
            float least = INFINITY, most = 0.f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) {
                least = fminf(least, fminf(fabsf(acc_k[e]), fabsf(acc_v[e])));
                most = fmaxf(most, fmaxf(fabsf(acc_k[e]), fabsf(acc_v[e])));
            }
            if (__any(least < kMergeLeast || most == INFINITY || count > kMergeCount)) {
#pragma unroll
                for (int e = 0; e < EPL; ++e) {
                    acc_k[e] = acc_k[e] / cf;
                    acc_v[e] = acc_v[e] / cf;
                }
            } else {
                const float unit = 1.f / cf;
#pragma unroll
                for (int e = 0; e < EPL; ++e) {
                    acc_k[e] = quotient(acc_k[e], cf, unit);
                    acc_v[e] = quotient(acc_v[e], cf, unit);
                }
            }
        } else if (n_rows == 1) {
            unpack<DT>(__builtin_bit_cast(uint4, row_k), acc_k);
            unpack<DT>(__builtin_bit_cast(uint4, row_v), acc_v);
        }
        k_cache[((size_t)bh * cap + jj) * LPR + sub] = round_row<DT>(acc_k);
        v_cache[((size_t)bh * cap + jj) * LPR + sub] = round_row<DT>(acc_v);
        if (WEIGHTED && owner && sub == 0 && counts) counts[bg * n_max + jj] = count;
    };

    // ---- piece p goes to lane group p % GROUPS; a bucket's pieces take its rows in turn ----
#pragma unroll 1
    for (int p0 = 0; p0 < min(n_pieces, PIECES); p0 += GROUPS) {
        const int p = p0 + grp;
        int i = grp, part = 0, parts = 1, p_lo, p_hi, most = 0;  // the piece's bucket, which part of how many, rows of the wave
        if (n_pieces > n_here) {  // uniform
            i = 0;
#pragma unroll
            for (int step = GROUPS / 2; step > 0; step >>= 1)
                if (sh_bucket[i + step - 1].w <= p) i += step;
            const int4 y = sh_bucket[i];
            p_lo = y.x, p_hi = y.y, parts = max(y.z, 1);
            part = p - (y.w - parts);
            most = p < n_pieces ? (p_hi - p_lo - part) / parts + 1 : 0;
#pragma unroll
            for (int off = LPR; off < kWave; off <<= 1) most = max(most, __shfl_xor(most, off, kWave));
            most = __builtin_amdgcn_readfirstlane(most);
            if (most <= 0 && p0 > 0) continue;  // uniform: no piece for this wave
        } else {  // every bucket is one piece
            p_lo = own_lo, p_hi = own_hi;
            const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
#pragma unroll
            for (int g = 0; g < kWave / LPR; ++g) most = max(most, __builtin_amdgcn_readlane(rows, wave * (kWave / LPR) + g));
        }
        // a bucket of one row is copied (weight 1 whatever it carries), so it stays bit-exact
        stream(p_lo + part, p < n_pieces ? p_hi : -1, parts, most, WEIGHTED && p_lo != p_hi);
        if (p < n_pieces) {
            if (parts == 1) {
                finish(bucket(i), p_hi - p_lo + 1, wsum);
            } else {
#pragma unroll
                for (int e = 0; e < EPL; ++e) {
                    sh_part[p][e * LPR + sub] = acc_k[e];
                    sh_part[p][(EPL + e) * LPR + sub] = acc_v[e];
                }
                if (sub == 0) sh_wsum[p] = wsum;
            }
        }
    }
    if (n_pieces > n_here) {  // uniform: partial sums in ascending order, by the lane group of the bucket's number
        __syncthreads();
        const int4 y = sh_bucket[grp];
        const int parts = y.z, first = y.w - parts, n_rows = y.y - y.x + 1;
        if (parts > 1) {
            int w_total = 0;
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc_k[e] = acc_v[e] = 0.f;
            for (int p = first; p < min(first + parts, PIECES); ++p) {
                w_total += sh_wsum[p];
#pragma unroll
                for (int e = 0; e < EPL; ++e) {
                    acc_k[e] += sh_part[p][e * LPR + sub];
                    acc_v[e] += sh_part[p][(EPL + e) * LPR + sub];
                }
            }
            finish(bucket(grp), n_rows, w_total);
        }
    }
}

template <int DT, int D>
static int launch_merge(const void* k, const void* v, const int32_t* anchor_idx, const int32_t* weights,
                        const int32_t* src_pos, int B, int H, int G, int T, int src_rows, int n_anchor, void* k_cache,
                        void* v_cache, int cap, int32_t* counts, int32_t* assign, int32_t* pos, int evict_only,
                        const int32_t* seq_len, const int32_t* n_anchor_b, hipStream_t stream)
{
    constexpr int LPR = D * Elem<DT>::kBytes / 16;
    constexpr int GROUPS = kMergeThreads / LPR;
    dim3 grid((n_anchor + GROUPS - 1) / GROUPS, B * H);
    if (weights != nullptr && !evict_only)
        hipLaunchKernelGGL((merge_compact_kernel<DT, D, true>), grid, dim3(kMergeThreads), 0, stream,
                           (const u32x4*)k, (const u32x4*)v, anchor_idx, weights, src_pos, (uint4*)k_cache,
                           (uint4*)v_cache, counts, assign, pos, H, G, T, src_rows, n_anchor, cap, evict_only, seq_len,
                           n_anchor_b);
    else
        hipLaunchKernelGGL((merge_compact_kernel<DT, D, false>), grid, dim3(kMergeThreads), 0, stream,
                           (const u32x4*)k, (const u32x4*)v, anchor_idx, weights, src_pos, (uint4*)k_cache,
                           (uint4*)v_cache, counts, assign, pos, H, G, T, src_rows, n_anchor, cap, evict_only, seq_len,
                           n_anchor_b);
    return status_from_hip(hipGetLastError());
}

int merge_dispatch(const void* k, const void* v, const int32_t* anchor_idx, const int32_t* weights,
                   const int32_t* src_pos, int B, int H, int G, int T, int src_rows, int D, int n_anchor, int dt,
                   int evict_only, void* k_cache, void* v_cache, int cap, int32_t* counts, int32_t* assign,
                   int32_t* pos, const int32_t* seq_len, const int32_t* n_anchor_b, hipStream_t stream)
{
#define EC_MERGE_CASE(DT_, D_)                                                                               \
    if (dt == DT_ && D == D_)                                                                                \
        return launch_merge<DT_, D_>(k, v, anchor_idx, weights, src_pos, B, H, G, T, src_rows, n_anchor, k_cache, \
                                     v_cache, cap, counts, assign, pos, evict_only, seq_len, n_anchor_b, stream);
    EC_MERGE_CASE(EC_BF16, 128)
    EC_MERGE_CASE(EC_BF16, 64)
    EC_MERGE_CASE(EC_F32, 128)
    EC_MERGE_CASE(EC_F32, 64)
#undef EC_MERGE_CASE
    return EC_EUNSUPPORTED;
}

}  // namespace ec
