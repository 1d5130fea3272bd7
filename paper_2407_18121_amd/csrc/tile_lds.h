// Tiles of a row-major matrix moved straight from memory into LDS, and the order in which workgroups take their work:
// shared by the scoring kernels.
#pragma once

#include "ec_common.h"

namespace ec {

typedef u32x4 __attribute__((aligned(2))) u32x4_any;  // at any element of a 16-bit tensor

// Workgroups are handed to the 8 XCDs round-robin by linear id, and each XCD has its own L2.  Work items are therefore
// renumbered so that all tiles of a head (which share its K and V) sit behind the same L2 instead of being fetched
// eight times.  Heads go to the XCDs in turn: a ragged batch, whose long sequences are neighbouring heads, then loads
// them alike (B16 H40, 312..624 rows: the slowest XCD ended at 141 us, the fastest at 105, with contiguous ranges).  A
// head count that eight does not divide is cut into equal contiguous ranges of items.
inline int xcd_grid(int total) { return (total + kXcds - 1) / kXcds * kXcds; }
struct XcdItem {
    int bh, tile;  // bh < 0: nothing to do
};
__device__ __forceinline__ XcdItem xcd_item(int linear_id, int per_head, int n_heads)
{
    const int xcd = linear_id % kXcds, nth = linear_id / kXcds;
    if (n_heads % kXcds == 0) {
        const int head = nth / per_head;
        return {head * kXcds + xcd, nth - head * per_head};
    }
    const int total = per_head * n_heads, per_xcd = (total + kXcds - 1) / kXcds;
    const int item = xcd * per_xcd + nth;
    if (nth >= per_xcd || item >= total) return {-1, 0};
    const int bh = item / per_head;
    return {bh, item - bh * per_head};
}

// Buffer descriptor over `bytes` bytes at p (raw: no stride, 32-bit data format).  Loads through it whose byte
// offset is at or beyond `bytes` return zeros instead of touching memory.  Lengths and offsets are unsigned: a head may
// be longer than 2 GiB (the host keeps the ones that 32 bits do not cover away).
__device__ __forceinline__ u32x4 tile_rsrc(const void* p, uint32_t bytes)
{
    const uint64_t at = (uint64_t)(uintptr_t)p;
    u32x4 r;
    r.x = __builtin_amdgcn_readfirstlane((uint32_t)at);
    r.y = __builtin_amdgcn_readfirstlane((uint32_t)(at >> 32) & 0xffffu);
    r.z = __builtin_amdgcn_readfirstlane(bytes);
    r.w = 0x00020000u;
    return r;
}

// ------------------------------------------------------------------ tiles moved straight from memory into LDS
// A tile of ROWS rows of D 16-bit words sits in LDS without padding (a lane of a direct load writes the 16 bytes
// behind its neighbour's), so bank conflicts are avoided by permuting the 16-byte chunks of a row: chunk c of row r
// is stored at place c ^ swizzle(r), which the loading lane arranges by fetching from the permuted address.
typedef __attribute__((address_space(3))) void lds_void;
__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)(lds_void*)p; }
// A value that the compiler has to take up anew: what is derived from it is computed here, not before the loop around.
__device__ __forceinline__ int anew(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}
// An LDS byte address that stays one register: the compiler would otherwise keep a copy per constant it is added to.
__device__ __forceinline__ uint32_t one_register(uint32_t a)
{
    asm volatile("" : "+v"(a));
    return a;
}
// One direct load: lane l writes its 16 (4) bytes at byte lds + 16 l (4 l).  Written in assembly because the compiler
// would make every later LDS read wait for every load in flight (it cannot tell the tiles of one array apart); the loads
// have no result register, and the waits below are the ones they need.  The five wait states are those between a vector
// instruction that writes a scalar register (a restored spill) and a load that reads it.
__device__ __forceinline__ void load_lds_16(u32x4 rsrc, uint32_t lds, uint32_t byte_offset)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds), "v"(byte_offset), "s"(rsrc) : "memory");
}
__device__ __forceinline__ void load_lds_4(u32x4 rsrc, uint32_t lds, uint32_t byte_offset)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :: "s"(lds), "v"(byte_offset), "s"(rsrc) : "memory");
}
// the wave's loads into LDS have landed / its LDS reads have returned / the workgroup meets
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void meet()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// All loads of this wave into LDS have landed and all its LDS reads have returned; then the workgroup meets.
__device__ __forceinline__ void tile_barrier()
{
    wait_loads();
    wait_lds();
    meet();
}

// Moves ROWS rows (of D 16-bit words each) starting at row0 of a matrix into LDS, WAVES waves sharing the work; issue(lds, row0, j), j in
// 0..NI-1, is one load instruction of this wave, so that a kernel can spread them over its arithmetic.  The bounds check
// of the descriptor covers rows beyond the matrix: nothing is read there, and the caller masks what they produce.
// A kernel that has arithmetic to put between the two halves of a move calls begin and later, in front of the barrier
// behind which the tile is read, finish; issue is both at once.
// DIRECT = false: for matrices that do not start on a 16-byte boundary, which loads straight into LDS need.  The rows
// pass through registers then, in flight from begin to finish.
template <int D, int ROWS, int WAVES, typename SWZ, bool DIRECT = true> struct TileToLds {
    static constexpr int CH = D / 8;            // 16-byte chunks per row
    static constexpr int RPI = kWave / CH;      // rows one wave moves per instruction
    static constexpr int NI = ROWS / RPI / WAVES;
    static constexpr int PERIOD = SWZ::kPeriod > RPI ? SWZ::kPeriod / RPI : 1;  // the lane's part of the address repeats
    static constexpr int PARTS = NI < PERIOD ? NI : PERIOD;
    static_assert(NI * RPI * WAVES == ROWS && (NI % PERIOD == 0 || PERIOD % NI == 0), "a wave's share within the period");
    u32x4 rsrc;
    int w0;                                     // first row of the wave's share (scalar)
    uint32_t part[PARTS];
    mutable u32x4 held[DIRECT ? 1 : NI];
    __device__ __forceinline__ TileToLds(u32x4 r, int wave, int lane) : rsrc(r), w0(wave * NI * RPI)
    {
#pragma unroll
        for (int j = 0; j < PARTS; ++j) {
            const int row = j * RPI + lane / CH;
            part[j] = (row * CH + (lane % CH ^ SWZ::at(w0 + row))) * 16;
        }
    }
    // lds: byte address of the tile (scalar)
    __device__ __forceinline__ void begin(uint32_t lds, int row0, int j) const
    {
        const uint32_t at = part[j % PARTS] + (uint32_t)(row0 + w0 + j / PARTS * PARTS * RPI) * (D * 2);
        if constexpr (DIRECT) {
            load_lds_16(rsrc, lds + (w0 + j * RPI) * (D * 2), at);
        } else {
            typedef __attribute__((address_space(1))) const u32x4_any global_u32x4;
            held[j] = u32x4{0, 0, 0, 0};
            if (at < rsrc.z) held[j] = *(global_u32x4*)(((uint64_t)rsrc.y << 32 | rsrc.x) + at);
        }
    }
    __device__ __forceinline__ void finish(uint32_t lds, int j) const
    {
        typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
        if constexpr (!DIRECT) *(lds_u32x4*)(uintptr_t)(lds + (w0 + j * RPI) * (D * 2) + threadIdx.x % kWave * 16) = held[j];
    }
    __device__ __forceinline__ void issue(uint32_t lds, int row0, int j) const
    {
        begin(lds, row0, j);
        finish(lds, j);
    }
};

}  // namespace ec
