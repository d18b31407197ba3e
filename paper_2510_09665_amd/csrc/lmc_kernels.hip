// Device kernels of liblmc for gfx950 (MI355X): the paged-KV gather (store direction)
// and scatter (load direction) that the paper's section 5.1 places between the
// engine's pages and the contiguous streaming GPU buffer, plus small helpers.
//
// Both kernels are pure byte movement and HBM-bound; there is no reuse, so neither LDS
// nor MFMA has a role.  What was measured to matter on this part, and shapes the code:
//   - One 16-byte vector per lane and a very large grid.  Occupancy, not unrolling,
//     supplies the bytes in flight: with a handful of VGPRs every SIMD holds its full
//     8 wavefronts.  Unrolled variants that walk several layer-planes per lane were
//     10-15 % slower: their accesses sit power-of-two distances apart (planes of a
//     chunk, layers of the cache) and collide on memory channels.
//   - Workgroup order follows the chunk buffer: tile, then layer-plane, then chunk.
//     The contiguous side of the copy is then swept linearly by the launch as a
//     whole, and the paged side is touched page by page (a page's tokens are
//     consecutive rows).  Ordering by layer-plane first cost 5-10 %.
//   - Non-temporal loads and stores inside HBM: nothing is read twice.  Stores to the host
//     go through the L2 instead (StoreKind).
//   - Index arithmetic (which chunk, plane, token, vector; slot -> block and offset)
//     uses multiply-high division by host-precomputed constants; the workgroup-level
//     part is wave-uniform and runs on the scalar unit.
#include "lmc_kernels.hpp"

#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

namespace lmc {
namespace {

constexpr int kThreads = 256;

template <int N> struct VecOf;
template <> struct VecOf<16> { typedef unsigned int type __attribute__((ext_vector_type(4))); };
template <> struct VecOf<8> { typedef unsigned int type __attribute__((ext_vector_type(2))); };
template <> struct VecOf<4> { typedef unsigned int type; };
template <> struct VecOf<2> { typedef unsigned short type; };
template <> struct VecOf<1> { typedef unsigned char type; };
// kWide: 16 bytes at any address (gfx950 takes unaligned global accesses in one instruction)
template <> struct VecOf<kWide> { typedef unsigned int type __attribute__((ext_vector_type(4), aligned(1))); };
// kPacked: a gather's 16 bytes on the chunk side, put together from rows of any length
constexpr int kPacked = 18;
template <> struct VecOf<kPacked> { typedef VecOf<16>::type type; };
template <int VEC> constexpr uint32_t kBytesOf = VEC == kWide || VEC == kPacked ? 16u : uint32_t(VEC);

#define LMC_GLOBAL __attribute__((address_space(1)))

// Addresses are carried as integers (so they can be pinned in scalar registers) and
// dereferenced as global-memory pointers, never as flat ones.
template <typename V, bool NT> __device__ __forceinline__ V load_vec(uint64_t addr) {
    const LMC_GLOBAL V *p = (const LMC_GLOBAL V *)addr;
    if (NT) return __builtin_nontemporal_load(p);
    return *p;
}
template <typename V, bool NT> __device__ __forceinline__ void store_vec(uint64_t addr, V v) {
    LMC_GLOBAL V *p = (LMC_GLOBAL V *)addr;
    if (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// How the kernels write: as the compiler does, with the non-temporal hint, or at system scope
// (sc0 sc1 nt).  A store at system scope goes through the XCD's L2 instead of staying there
// until it is evicted or the kernel ends, and has reached memory, the host's included, when it
// completes.  Across the host link that is the faster way to write whole cache lines: 64 MiB to
// the pinned pool by a plain copy 57.1 GB/s, the same in every run, against 55.4-56.0 (the
// runtime's own copies: 56.9).  Lines written in parts suffer, since nothing puts them together
// any more (a gather of 216-byte rows inside HBM: 53.8 us instead of 45.7).  Inside HBM a linear
// copy gains 3 % (6.76 against 6.48 TB/s), a gather of 512 MiB in random 32 KiB pages 0.4 %, one
// of 32 MiB loses 2 % (11.1 against 10.9 us) and the scatter does not care while it is alone: gathers
// and all but the largest scatters keep the hint there.
enum StoreKind { kStorePlain = 0, kStoreNonTemporal = 1, kStoreThrough = 2 };
// s_nop 1: gfx950 wants two wait states between a store of more than 64 bits and an instruction
// that writes its data registers again, and the compiler, which does not see the store, adds none.
__device__ __forceinline__ void store_through(uint64_t addr, typename VecOf<16>::type v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1 nt\n\ts_nop 1" ::"v"(addr), "v"(v) : "memory");
}
// The flag the host reads: it must not stay in an L2 either.
__device__ __forceinline__ void raise_flag(uint64_t addr) {
    asm volatile("global_store_dword %0, %1, off sc0 sc1" ::"v"(addr), "v"(1) : "memory");
}
template <int VEC, int ST> __device__ __forceinline__ void store_out(uint64_t addr, typename VecOf<VEC>::type v) {
    typedef typename VecOf<VEC>::type V;
    if constexpr (ST != kStoreThrough) {
        store_vec<V, ST != kStorePlain>(addr, v);
    } else if constexpr (sizeof(V) == 16) {
        store_through(addr, v);
    } else if constexpr (sizeof(V) == 8) {
        __hip_atomic_store((LMC_GLOBAL uint64_t *)addr, __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    } else {
        __hip_atomic_store((LMC_GLOBAL V *)addr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Tells the device's queues, while the kernel still runs, that this wavefront's stores so far have
// reached memory: adds one to a word, which hipStreamWaitValue64 compares with the number of
// wavefronts that owe it one.  The stores are at system scope (kStoreThrough), so when they have
// completed nothing of them is left in an L2 that would have to be written back: no release
// fence, which takes 4 us of a kernel that moves 0.5 MiB across the link in 13.
__device__ __forceinline__ void arrive(uint64_t word_at) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if ((threadIdx.x & 63u) == 0)
        (void)__hip_atomic_fetch_add((LMC_GLOBAL uint64_t *)word_at, uint64_t(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// The same for a whole workgroup, at the end of a kernel, and for the host too, if asked: the last one to
// arrive, which brings the word to `target`, writes that to a word in host memory. One count for each
// workgroup, 24 at one address instead of one for each of 192 wavefronts (0.5 MiB, to the host and from it,
// 12.6 us either way: the barrier costs what the counts did).
__device__ __forceinline__ void arrive_and_tell(const HostWord &told) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x != 0) return;
    LMC_GLOBAL uint64_t *word = (LMC_GLOBAL uint64_t *)told.word;
    if (told.host == nullptr) {
        (void)__hip_atomic_fetch_add(word, uint64_t(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    } else if (__hip_atomic_fetch_add(word, uint64_t(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) + 1 == told.target) {
        __hip_atomic_store((LMC_GLOBAL uint64_t *)told.host, told.target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Keeps a wave-uniform value in scalar registers from this point on.
template <typename T> __device__ __forceinline__ T pin(T v) {
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ FastDiv pin(FastDiv f) {
    f.mul = pin(f.mul);
    f.shift = pin(f.shift);
    f.d = pin(f.d);
    return f;
}

// Everything a tile needs besides its own number, held in scalar registers.
struct TileArgs {
    FastDiv by_tiles, by_lp, by_row, by_run, by_bs;
    uint32_t lp_base, vec_per_plane, chunk_tokens, n_slots, runs_per_row, run_bytes, row_bytes;
    uint64_t chunk_stride, plane_bytes, slots_at, staging_at, bad_flag_at;
    int64_t block_stride, token_stride, run_stride;
};

// Fetches every kernel argument at once, in one batch of scalar loads.  Left alone the
// compiler loads each field just before its first use, which puts four scalar-load
// round trips behind the slot load on every wavefront's critical path.
template <int VEC>
__device__ __forceinline__ TileArgs fetch_args(const KernelGeom &g, const LaunchView &view,
                                               const int64_t *slot_mapping, uint8_t *staging,
                                               int32_t *bad_flag) {
    TileArgs a;
    a.by_tiles = pin(g.by_tiles_per_plane);
    a.by_lp = pin(view.by_n_lp);
    a.by_row = pin(g.by_vec_per_row);
    a.by_run = pin(g.by_vec_per_run);
    a.by_bs = pin(g.by_block_size);
    a.lp_base = pin(view.lp_base);
    a.chunk_stride = pin(view.chunk_stride);
    a.vec_per_plane = pin(g.vec_per_plane);
    a.chunk_tokens = pin(g.chunk_tokens);
    a.n_slots = pin(g.n_slots);
    a.runs_per_row = pin(g.runs_per_row);
    if (VEC == kWide || VEC == kPacked) a.run_bytes = pin(g.run_bytes);
    if (VEC == kWide) a.row_bytes = pin(g.row_bytes);
    a.block_stride = pin(g.block_stride);
    a.token_stride = pin(g.token_stride);
    a.run_stride = pin(g.run_stride);
    a.plane_bytes = pin(g.plane_bytes);
    a.slots_at = pin(uint64_t(slot_mapping));
    a.staging_at = pin(uint64_t(staging));
    a.bad_flag_at = pin(uint64_t(bad_flag));
    return a;
}

// Where vector w of a token's row lies: *in_page relative to the token's first byte in its
// page, *in_row relative to the row's first byte in the chunk.  A wide row (kWide) is cut
// run by run: every run of run_bytes >= 16 bytes takes ceil(run_bytes / 16) vectors, the
// last of them moved back so that it ends with the run.  It overlaps its neighbour, and
// the overlapped bytes are moved twice, with equal values, by lanes of one launch.
template <int VEC>
__device__ __forceinline__ void place(const TileArgs &a, uint32_t w, int64_t *in_page, uint64_t *in_row) {
    uint32_t run = 0, dv = w;
    if (a.runs_per_row > 1) {
        run = a.by_run.div(w);
        dv = w - run * a.by_run.d;
    }
    uint32_t off = dv * kBytesOf<VEC>;
    if (VEC == kWide) off = min(off, a.run_bytes - 16u);
    *in_page = int64_t(run) * a.run_stride + int64_t(off);
    *in_row = VEC == kWide ? uint64_t(run) * a.run_bytes + off : uint64_t(w) * kBytesOf<VEC>;
}

// One 16-byte piece r of plane (c, layer) of a chunk for kPacked, gathered from the pages.
// Here by_run divides a byte of the plane by run_bytes, which gives the run that holds it, and
// by_row divides a run by the runs of a row, which gives the token (packed_geom).  A run has 16
// bytes or more, so a piece holds bytes of one run or of two that follow each other; of those
// the first's last 16 bytes and the second's first 16 are loaded, so that nothing outside the
// runs is read, and shifted together.  Tokens without a page give zeros.
template <bool NT_LD>
__device__ __forceinline__ typename VecOf<16>::type packed_piece(const TileArgs &a, uint64_t layer, uint32_t c, uint32_t r,
                                                                 bool flag_bad) {
    typedef typename VecOf<kWide>::type W;
    const uint32_t byte = r * 16u;
    const uint32_t run = a.by_run.div(byte);
    const uint32_t off = byte - run * a.run_bytes;
    const uint32_t rest = a.run_bytes - off;          // bytes of this run from here on
    const uint32_t run2 = rest < 16u ? run + 1u : run;
    const uint32_t t = a.by_row.div(run), t2 = a.by_row.div(run2);
    const uint64_t map = a.slots_at + uint64_t(c) * a.chunk_tokens * 8u;
    const int64_t s = load_vec<int64_t, false>(map + uint64_t(t) * 8u), s2 = load_vec<int64_t, false>(map + uint64_t(t2) * 8u);
    auto page = [&](int64_t slot, uint32_t token, uint32_t run_of_plane) {
        const uint32_t su = uint64_t(slot) < uint64_t(a.n_slots) ? uint32_t(slot) : 0u;
        const uint32_t b = a.by_bs.div(su);
        return layer + uint64_t(int64_t(b) * a.block_stride + int64_t(su - b * a.by_bs.d) * a.token_stride +
                                int64_t(run_of_plane - token * a.by_row.d) * a.run_stride);
    };
    if (flag_bad && (s >= int64_t(a.n_slots) || s2 >= int64_t(a.n_slots))) raise_flag(a.bad_flag_at);
    W x = load_vec<W, NT_LD>(page(s, t, run) + min(off, a.run_bytes - 16u));
    W y = W(0);
    if (rest < 16u) y = load_vec<W, NT_LD>(page(s2, t2, run2));
    if (uint64_t(s) >= uint64_t(a.n_slots)) x = W(0);
    if (uint64_t(s2) >= uint64_t(a.n_slots)) y = W(0);
    if (rest < 16u) {
        // bytes 16 - rest .. 15 of x, then bytes 0 .. 15 - rest of y
        const uint32_t bits = (16u - rest) * 8u;
        const uint64_t x0 = x.x | uint64_t(x.y) << 32, x1 = x.z | uint64_t(x.w) << 32;
        const uint64_t y0 = y.x | uint64_t(y.y) << 32, y1 = y.z | uint64_t(y.w) << 32;
        const unsigned __int128 both = ((unsigned __int128)x1 << 64 | x0) >> bits | ((unsigned __int128)y1 << 64 | y0) << (128u - bits);
        const uint64_t z0 = uint64_t(both), z1 = uint64_t(both >> 64);
        x.x = uint32_t(z0);
        x.y = uint32_t(z0 >> 32);
        x.z = uint32_t(z1);
        x.w = uint32_t(z1 >> 32);
    }
    return x;
}

// One tile (256 consecutive vectors of one plane of one chunk) of the path's copy in
// either direction; lane = one vector r of plane lp of chunk c, token t = r / vec_per_row:
//   GATHER: chunk[c][lp][r] = valid(slot[c][t]) ? page(lp, slot[c][t])[r % vec_per_row] : 0
//   else  : if valid(slot[c][t]):  page(lp, slot[c][t])[r % vec_per_row] = chunk[c][lp][r]
// blk numbers the launch's tiles in chunk-buffer order: tile, then layer-plane, then chunk.
template <int VEC, bool GATHER, bool NT_LD, int ST>
__device__ __forceinline__ void move_tile(const TileArgs &a, const LayerPtrs &layers, uint32_t blk) {
    typedef typename VecOf<VEC>::type V;
    const uint32_t q = a.by_tiles.div(blk);
    const uint32_t tile = blk - q * a.by_tiles.d;
    const uint32_t c = a.by_lp.div(q);
    const uint32_t lp = q - c * a.by_lp.d;  // plane inside this launch's part of the chunk
    const uint32_t r = tile * kThreads + threadIdx.x;
    if (r >= a.vec_per_plane) return;
    const uint32_t t = a.by_row.div(r);
    const uint32_t w = r - t * a.by_row.d;

    const int64_t s = load_vec<int64_t, false>(a.slots_at + (uint64_t(c) * a.chunk_tokens + t) * 8u);
    // the plane's base pointer is fetched while the slot is on its way
    const uint64_t layer = pin(uint64_t(layers.p[a.lp_base + lp]));
    const bool valid = uint64_t(s) < uint64_t(a.n_slots);  // negative wraps to huge
    if (s >= int64_t(a.n_slots)) raise_flag(a.bad_flag_at);
    const uint32_t su = valid ? uint32_t(s) : 0u;  // slot 0 is always inside the pages
    const uint32_t b = a.by_bs.div(su);
    const uint32_t o = su - b * a.by_bs.d;
    int64_t in_page;
    uint64_t in_row;
    place<VEC>(a, w, &in_page, &in_row);
    const uint64_t page = layer + uint64_t(int64_t(b) * a.block_stride + int64_t(o) * a.token_stride + in_page);
    const uint64_t st = a.staging_at + uint64_t(c) * a.chunk_stride + uint64_t(lp) * a.plane_bytes +
                        (VEC == kWide ? uint64_t(t) * a.row_bytes + in_row : uint64_t(r) * kBytesOf<VEC>);
    if (GATHER) {
        V v = load_vec<V, NT_LD>(page);
        if (!valid) v = V(0);
        store_out<VEC, ST>(st, v);
    } else if (valid) {
        store_out<VEC, ST>(page, load_vec<V, NT_LD>(st));
    }
}

// Hands each XCD runs of 2^xcd_shift consecutive tiles: hardware deals consecutive workgroup
// ids to the 8 XCDs in turn, one tile each.  This is a permutation inside every group of
// 8 << xcd_shift ids, and n_blocks_permuted is a multiple of that, so the result stays below it.
__device__ __forceinline__ uint32_t permuted_block(uint32_t blk, uint32_t n_blocks_permuted, uint32_t xcd_shift) {
    if (blk >= n_blocks_permuted) return blk;
    const uint32_t xcd = blk & 7u, local = blk >> 3;
    const uint32_t grp = local >> xcd_shift;
    return (((grp << 3) + xcd) << xcd_shift) + (local & ((1u << xcd_shift) - 1u));
}

// HBM to HBM (pages <-> staging): one tile per workgroup, a very large grid.
template <int VEC, bool GATHER, bool NT_LD, int ST>
__global__ __launch_bounds__(kThreads) void move_rows(const KernelGeom g, const LaunchView view,
                                                      const LayerPtrs layers,
                                                      const int64_t *__restrict__ slot_mapping,
                                                      uint8_t *staging, int32_t *bad_flag,
                                                      uint32_t n_blocks_permuted, uint32_t xcd_shift) {
    const TileArgs a = fetch_args<VEC>(g, view, slot_mapping, staging, bad_flag);
    move_tile<VEC, GATHER, NT_LD, ST>(a, layers, permuted_block(blockIdx.x, n_blocks_permuted, xcd_shift));
}

// The gather where a run is a multiple of 64 vectors (1 KiB): every wavefront then moves part of
// one run of one token, so token, slot and both addresses are found once per wavefront, on the
// scalar unit, with a scalar load of the slot, and a lane adds nothing but its 16 bytes.
// Llama-3-8B shape, per lane and per wavefront: 16 chunks 179.5, 176.1 us, 31 chunks 358.3, 350.3,
// one chunk 10.8, 10.45; 1 KiB rows in one-token pages, 160 MiB: 115.3, 112.1.  The scatter,
// which loads its data while the slot is on its way, loses 1-2 % this way.
__global__ __launch_bounds__(kThreads) void gather_rows_by_wave(const KernelGeom g, const LaunchView view,
                                                                const LayerPtrs layers,
                                                                const int64_t *__restrict__ slot_mapping,
                                                                uint8_t *staging, int32_t *bad_flag,
                                                                uint32_t n_blocks_permuted, uint32_t xcd_shift) {
    typedef typename VecOf<16>::type V;
    const TileArgs a = fetch_args<16>(g, view, slot_mapping, staging, bad_flag);
    const uint32_t blk = permuted_block(blockIdx.x, n_blocks_permuted, xcd_shift);
    const uint32_t q = a.by_tiles.div(blk);
    const uint32_t tile = blk - q * a.by_tiles.d;
    const uint32_t c = a.by_lp.div(q);
    const uint32_t lp = q - c * a.by_lp.d;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t r = tile * kThreads + __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);  // the wavefront's first vector
    if (r >= a.vec_per_plane) return;                    // planes are whole wavefronts
    const uint32_t t = a.by_row.div(r);
    const uint32_t w = r - t * a.by_row.d;
    const int64_t s = *(const __attribute__((address_space(4))) int64_t *)(a.slots_at + (uint64_t(c) * a.chunk_tokens + t) * 8u);
    const uint64_t layer = uint64_t(layers.p[a.lp_base + lp]);
    const uint64_t st = a.staging_at + uint64_t(c) * a.chunk_stride + uint64_t(lp) * a.plane_bytes + uint64_t(r) * 16u;
    if (s >= int64_t(a.n_slots)) raise_flag(a.bad_flag_at);
    V v = V(0);
    if (uint64_t(s) < uint64_t(a.n_slots)) {             // negative wraps to huge
        const uint32_t b = a.by_bs.div(uint32_t(s));
        const uint32_t o = uint32_t(s) - b * a.by_bs.d;
        int64_t in_page;
        uint64_t in_row;
        place<16>(a, w, &in_page, &in_row);
        const uint64_t page = layer + uint64_t(int64_t(b) * a.block_stride + int64_t(o) * a.token_stride + in_page);
        v = __builtin_nontemporal_load((const LMC_GLOBAL V *)page + lane);
    }
    __builtin_nontemporal_store(v, (LMC_GLOBAL V *)st + lane);
}

// What crosses the link keeps the compute unit to itself: a workgroup asks for most of its LDS, of
// which it uses nothing (LaunchShape::paced_lds).  A load of host memory takes 4 us and
// more with the link busy, stores to it queue up likewise, and the loads of whatever else runs on that
// compute unit wait behind them.  Beside a load of 64 MiB and beside a store of as much, with 0, 96, 128
// and 160 KiB claimed: a dense bf16 product of 128 rows by 4096 x 4096 (33 us alone) 76, 77, 37, 36 and
// 66, 65, 34, 34 us, one of 512 rows (36) 80, 82, 54, 54 and 65, 66, 50, 51, attention (138) 274, 274,
// 260, 259 and 224, 223, 184, 184, softmax (46) 61, 61, 62, 48 and 55, 54, 54, 46; the transfers
// themselves 1194 us with any.  64 MiB layer by layer with such products between the layers: 4.92, -,
// 4.24, 4.24 ms.  Hence 128: what it keeps out is what has much LDS and reads much, and it starts
// beside a kernel that stays and holds no more than 32 KiB on every compute unit.  Beside one that
// holds more everywhere it starts when that one ends; for a process that has such a kernel wait for a
// transfer there is the knob "link_lds_kib".  Nothing is lost while the GPU is full of kernels that
// end: 0.5 MiB issued into a queue of products, attention or softmax ends within the spread of the
// unclaimed (15-110 us), as soon as one compute unit runs out of work of the kernel before.
// Hence also two groups of 256 lanes to a workgroup: as many tiles in flight on half the compute
// units, at the same rate.
constexpr int kPacedThreads = 2 * kThreads;

// The gather's tile for a workgroup that takes many, one after the other: no early return, a lane
// past the end of the plane reads the slot that the last one reads and moves nothing.  With a list,
// chunk c of the launch lies list->slot[c] chunk strides into the buffer.
template <int VEC, bool NT_LD, int ST>
__device__ __forceinline__ void gather_tile_in_turn(const TileArgs &a, const LayerPtrs &layers, uint32_t blk,
                                                    uint32_t lane, const ChunkList *list) {
    typedef typename VecOf<VEC>::type V;
    const uint32_t q = a.by_tiles.div(blk);
    const uint32_t tile = blk - q * a.by_tiles.d;
    const uint32_t c = a.by_lp.div(q);
    const uint32_t lp = q - c * a.by_lp.d;
    const uint32_t r0 = tile * kThreads + lane;
    const uint32_t r = min(r0, a.vec_per_plane - 1);
    if constexpr (VEC == kPacked) {
        const uint64_t st = a.staging_at + uint64_t(list ? uint32_t(list->slot[c]) : c) * a.chunk_stride +
                            uint64_t(lp) * a.plane_bytes + uint64_t(r) * 16u;
        const V v = packed_piece<NT_LD>(a, uint64_t(layers.p[a.lp_base + lp]), c, r, r0 < a.vec_per_plane);
        if (r0 < a.vec_per_plane) store_out<VEC, ST>(st, v);
        return;
    }
    const uint32_t t = a.by_row.div(r);
    const uint32_t w = r - t * a.by_row.d;
    const int64_t s = load_vec<int64_t, false>(a.slots_at + (uint64_t(c) * a.chunk_tokens + t) * 8u);
    const uint64_t layer = uint64_t(layers.p[a.lp_base + lp]);
    const uint32_t c_buf = list ? uint32_t(list->slot[c]) : c;
    int64_t in_page;
    uint64_t in_row;
    place<VEC>(a, w, &in_page, &in_row);
    const uint64_t st = a.staging_at + uint64_t(c_buf) * a.chunk_stride + uint64_t(lp) * a.plane_bytes +
                        (VEC == kWide ? uint64_t(t) * a.row_bytes + in_row : uint64_t(r) * kBytesOf<VEC>);
    const bool has_page = uint64_t(s) < uint64_t(a.n_slots);  // negative wraps to huge
    const bool mine = r0 < a.vec_per_plane;
    if (mine && s >= int64_t(a.n_slots)) raise_flag(a.bad_flag_at);
    const uint32_t su = has_page ? uint32_t(s) : 0u;  // slot 0 is always inside the pages
    const uint32_t b = a.by_bs.div(su);
    const uint32_t o = su - b * a.by_bs.d;
    V v = load_vec<V, NT_LD>(layer + uint64_t(int64_t(b) * a.block_stride + int64_t(o) * a.token_stride + in_page));
    if (!has_page) v = V(0);
    if (mine) store_out<VEC, ST>(st, v);
}

// Across the host link (pages <-> pinned pool, no staging): the link, not HBM, sets the
// pace, and it runs best when few groups of 256 lanes walk the host side in order.  Measured with a
// plain copy kernel on this part: 64 groups taking tiles in turn reach 57.6 GB/s
// reading host memory and 56.2 GB/s writing it (the runtime's own copies: 57.2 / 57.0),
// one tile per workgroup over thousands of workgroups 55.7 / 54.4; with stores at system scope
// (StoreKind) writing is at 57.1.  The grid is fixed and
// every group takes tiles blk, blk + groups, ... until the launch's n_blocks.
template <int VEC, bool NT_LD, int ST>
__global__ __launch_bounds__(kPacedThreads) void gather_paced(const KernelGeom g, const LaunchView view,
                                                         const LayerPtrs layers,
                                                         const int64_t *__restrict__ slot_mapping,
                                                         uint8_t *staging, int32_t *bad_flag,
                                                         uint32_t n_blocks, uint32_t groups, const HostWord told) {
    const TileArgs a = fetch_args<VEC>(g, view, slot_mapping, staging, bad_flag);
    const uint32_t step = pin(groups), end = pin(n_blocks), lane = threadIdx.x % kThreads;
    const uint32_t first = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads) * gridDim.x + blockIdx.x;
    // an odd number of groups leaves a half without work
    for (uint32_t blk = first < step ? first : end; blk < end; blk += step)
        gather_tile_in_turn<VEC, NT_LD, ST>(a, layers, blk, lane, nullptr);
    if (ST == kStoreThrough && told.word != nullptr) arrive_and_tell(told);
}

// The same for chunks in any pool slots (a fragmented pool, a batch of requests): one launch
// instead of one per run of consecutive slots, each of which ends with the link running dry
// and is followed by a gap of 4-5 us.  A store of 25 chunks of 2 MiB in 12 runs: 12 launches
// take 975 us on the device, one takes 946 (1123 and 1089 us for the whole call).
template <int VEC, bool NT_LD, int ST>
__global__ __launch_bounds__(kPacedThreads) void gather_listed(const KernelGeom g, const LaunchView view,
                                                          const LayerPtrs layers,
                                                          const int64_t *__restrict__ slot_mapping,
                                                          uint8_t *staging, int32_t *bad_flag,
                                                          uint32_t n_blocks, uint32_t groups, const HostWord told, const ChunkList list) {
    const TileArgs a = fetch_args<VEC>(g, view, slot_mapping, staging, bad_flag);
    const uint32_t step = pin(groups), end = pin(n_blocks), lane = threadIdx.x % kThreads;
    const uint32_t first = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads) * gridDim.x + blockIdx.x;
    // an odd number of groups leaves a half without work
    for (uint32_t blk = first < step ? first : end; blk < end; blk += step)
        gather_tile_in_turn<VEC, NT_LD, ST>(a, layers, blk, lane, &list);
    if (ST == kStoreThrough && told.word != nullptr) arrive_and_tell(told);
}

// One lane's piece of a tile of a scatter from the pool: where it comes from, and what its
// destination is worked out from once the slot is known.
struct Piece {
    uint64_t from, layer;
    int64_t in_page, slot;
    bool mine;            // not past the end of the plane
};
struct BackToBack {};     // in a list's place: chunk c lies c chunk strides into the pool
template <int VEC, typename List>
__device__ __forceinline__ Piece find_piece(const TileArgs &a, const LayerPtrs &layers, uint32_t blk, uint32_t lane, const List &list) {
    const uint32_t q = a.by_tiles.div(blk);
    const uint32_t tile = blk - q * a.by_tiles.d;
    const uint32_t c = a.by_lp.div(q);
    const uint32_t lp = q - c * a.by_lp.d;
    const uint32_t r0 = tile * kThreads + lane;
    const uint32_t r = min(r0, a.vec_per_plane - 1);
    const uint32_t t = a.by_row.div(r);
    const uint32_t w = r - t * a.by_row.d;
    Piece p;
    p.slot = load_vec<int64_t, false>(a.slots_at + (uint64_t(c) * a.chunk_tokens + t) * 8u);
    p.mine = r0 < a.vec_per_plane;
    p.layer = uint64_t(layers.p[a.lp_base + lp]);
    uint32_t c_buf = c;
    if constexpr (!std::is_same_v<List, BackToBack>) c_buf = uint32_t(list.slot[c]);
    uint64_t in_row;
    place<VEC>(a, w, &p.in_page, &in_row);
    p.from = a.staging_at + uint64_t(c_buf) * a.chunk_stride + uint64_t(lp) * a.plane_bytes +
             (VEC == kWide ? uint64_t(t) * a.row_bytes + in_row : uint64_t(r) * kBytesOf<VEC>);
    return p;
}

// The scatter across the link, for chunks back to back or in listed pool slots, in one or more
// steps: a step is the next planes of every chunk, and a workgroup goes on with its next tile
// whichever step that is in.  With words, the wavefronts count themselves off at the step's word
// when their last tile of it is in the pages, between the load and the store of the next tile,
// where they wait anyway; so the layers of a layer-wise retrieve need neither a launch each,
// with the link idle for 5 us of 41 in between (2 MiB a step), nor an event each, which takes the
// thread that waits for it on another queue 13 us where a word takes 2.
// While a tile's data crosses the link the slots of the next tile are fetched, so a workgroup
// spends nothing but the link's round trip on a tile; stores are waited for only with the data
// behind them.  They are at system scope, for the words and because a wavefront has nothing
// else to do at this pace.
template <int VEC, typename List>
__global__ __launch_bounds__(kPacedThreads) void scatter_paced(const KernelGeom g, const LaunchView view,
                                                          const StepView steps, const LayerPtrs layers,
                                                          const int64_t *__restrict__ slot_mapping, const uint8_t *pool,
                                                          int32_t *bad_flag, uint64_t *words, const HostWord told_host,
                                                          const List list) {
    typedef typename VecOf<VEC>::type V;
    const uint32_t half = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads), lane = threadIdx.x % kThreads;
    TileArgs a = fetch_args<VEC>(g, view, slot_mapping, const_cast<uint8_t *>(pool), bad_flag);
    const uint32_t groups = pin(steps.groups), n_steps = pin(steps.n_steps);
    const uint32_t planes = a.by_lp.d, last_blocks = pin(steps.last_blocks);
    const FastDiv by_last = pin(steps.by_last_lp);
    const uint64_t words_at = pin(uint64_t(words));
    uint32_t blk = half * gridDim.x + blockIdx.x, step = 0, told = 0;   // told: steps this wavefront has counted itself off at
    uint32_t blocks = n_steps > 1 ? pin(steps.n_blocks) : last_blocks;
    if (n_steps == 1) a.by_lp = by_last;
    const bool works = blk < groups;                 // an odd number of groups leaves a half without work
    // goes on to the step that tile blk lies in; false behind the last
    auto in_step = [&]() {
        while (blk >= blocks) {
            blk -= blocks;
            if (++step >= n_steps) return false;
            a.lp_base += planes;
            a.staging_at += uint64_t(planes) * a.plane_bytes;
            if (step + 1 == n_steps) {
                blocks = last_blocks;
                a.by_lp = by_last;
            }
        }
        return true;
    };
    if (works && in_step()) {
        Piece p = find_piece<VEC>(a, layers, blk, lane, list);
        asm volatile("" : "+v"(p.slot));   // arrived: the loop then has no load of its own to wait for at its head
        for (bool more = true; more;) {
            const bool moves = p.mine && uint64_t(p.slot) < uint64_t(a.n_slots);   // negative wraps to huge
            V v = V(0);
            if (moves) v = load_vec<V, true>(p.from);      // a token without a page costs the link nothing
            if (p.mine && p.slot >= int64_t(a.n_slots)) raise_flag(a.bad_flag_at);
            const uint32_t before = step;
            blk += groups;
            more = in_step();
            Piece next = p;
            if (more) next = find_piece<VEC>(a, layers, blk, lane, list);
            const uint32_t su = moves ? uint32_t(p.slot) : 0u;
            const uint32_t b = a.by_bs.div(su);
            const uint32_t o = su - b * a.by_bs.d;
            const uint64_t page = p.layer + uint64_t(int64_t(b) * a.block_stride + int64_t(o) * a.token_stride + p.in_page);
            if (words_at != 0)
                for (; told < before; told++) arrive(words_at + told * kWordStride);
            // the next slot is waited for here, with the data, and not behind the store
            asm volatile("" : "+v"(next.slot));
            if (moves) store_out<VEC, kStoreThrough>(page, v);
            p = next;
        }
    }
    if (words_at != 0 && works)
        for (; told < n_steps; told++) arrive(words_at + told * kWordStride);
    if (told_host.word != nullptr) arrive_and_tell(told_host);
}

// ---- scatter in the order of the destination ---------------------------------------------
// A launch that fills thousands of pages per plane (a long context, a batch of requests)
// finds many of its pages close together in memory, but the slot mapping names them in
// the order of the tokens, which is random in address.  Writes to DRAM are what suffers
// most from jumping around, so for such launches the rows are visited in ascending slot
// order, plane by plane: the writes then sweep each plane once, and the jumps move to the
// reads of the staging buffer.  The order is built on the device, without a sort: every
// slot number is an index into a table (one word per slot of a plane) that receives the
// token living there, and compacting the table yields (slot, token) pairs in slot order.

constexpr uint32_t kNoToken = 0xFFFFFFFFu;
constexpr int kSlotsPerThread = 8;
constexpr int kSlotsPerGroup = kThreads * kSlotsPerThread;

__global__ __launch_bounds__(kThreads) void order_clear(uint32_t *__restrict__ token_at, uint32_t n_slots) {
    const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
    if (i < n_slots) token_at[i] = kNoToken;
}

// token_at[slot] = token; slots outside the pages raise the flag, negative ones are left out
__global__ __launch_bounds__(kThreads) void order_mark(const int64_t *__restrict__ slot_mapping,
                                                       uint32_t n_tokens, uint32_t n_slots,
                                                       uint32_t *__restrict__ token_at, int32_t *bad_flag) {
    const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= n_tokens) return;
    const int64_t s = slot_mapping[i];
    if (s >= int64_t(n_slots)) *bad_flag = 1;
    else if (s >= 0) token_at[s] = i;
}

// exclusive prefix sum over the workgroup of one value per thread; *total = the sum
__device__ __forceinline__ uint32_t group_exclusive_scan(uint32_t v, uint32_t *lds, uint32_t *total) {
    const uint32_t t = threadIdx.x, n = blockDim.x;
    lds[t] = v;
    __syncthreads();
    for (uint32_t d = 1; d < n; d <<= 1) {
        const uint32_t add = t >= d ? lds[t - d] : 0u;
        __syncthreads();
        lds[t] += add;
        __syncthreads();
    }
    const uint32_t incl = lds[t];
    *total = lds[n - 1];
    __syncthreads();
    return incl - v;
}

__device__ __forceinline__ uint32_t occupied_in_my_slots(const uint32_t *token_at, uint32_t n_slots,
                                                         uint32_t first) {
    uint32_t cnt = 0;
    for (int k = 0; k < kSlotsPerThread; k++)
        cnt += (first + k < n_slots && token_at[first + k] != kNoToken) ? 1u : 0u;
    return cnt;
}

// counts[group] = occupied slots among the group's kSlotsPerGroup slots
__global__ __launch_bounds__(kThreads) void order_count(const uint32_t *__restrict__ token_at,
                                                        uint32_t n_slots, uint32_t *__restrict__ counts) {
    __shared__ uint32_t lds[kThreads];
    const uint32_t first = blockIdx.x * kSlotsPerGroup + threadIdx.x * kSlotsPerThread;
    uint32_t total;
    group_exclusive_scan(occupied_in_my_slots(token_at, n_slots, first), lds, &total);
    if (threadIdx.x == 0) counts[blockIdx.x] = total;
}

// one workgroup: counts[] becomes its exclusive prefix sum, *n_rows the grand total
__global__ __launch_bounds__(1024) void order_offsets(uint32_t *__restrict__ counts, uint32_t n_groups,
                                                      uint32_t *__restrict__ n_rows) {
    __shared__ uint32_t lds[1024];
    const uint32_t per = (n_groups + 1023u) / 1024u;
    const uint32_t lo = threadIdx.x * per, hi = lo + per < n_groups ? lo + per : n_groups;
    uint32_t sum = 0;
    for (uint32_t i = lo; i < hi; i++) sum += counts[i];
    uint32_t total;
    uint32_t run = group_exclusive_scan(sum, lds, &total);
    for (uint32_t i = lo; i < hi; i++) {
        const uint32_t c = counts[i];
        counts[i] = run;
        run += c;
    }
    if (threadIdx.x == 0) *n_rows = total;
}

// pairs[rank of the slot among the occupied ones] = (slot, token)
__global__ __launch_bounds__(kThreads) void order_emit(const uint32_t *__restrict__ token_at,
                                                       uint32_t n_slots, const uint32_t *__restrict__ offsets,
                                                       uint2 *__restrict__ pairs) {
    __shared__ uint32_t lds[kThreads];
    const uint32_t first = blockIdx.x * kSlotsPerGroup + threadIdx.x * kSlotsPerThread;
    uint32_t total;
    uint32_t at = offsets[blockIdx.x] +
                  group_exclusive_scan(occupied_in_my_slots(token_at, n_slots, first), lds, &total);
    for (int k = 0; k < kSlotsPerThread; k++) {
        if (first + k >= n_slots) break;
        const uint32_t tok = token_at[first + k];
        if (tok != kNoToken) pairs[at++] = make_uint2(first + k, tok);
    }
}

// The scatter itself.  The pairs are taken in groups of group_rows; workgroups are
// numbered group by group, inside a group plane by plane, inside a plane along the group's
// pairs: lane = vector w of the row of pair j.  So what is in flight at any moment is, in
// each of a few planes, a run of pages that are neighbours in address.  The launch is sized
// for the tokens of the call; the pairs may be fewer (tokens without a page), the rest of
// the grid retires.
template <int VEC, bool NT_LD, bool NT_ST>
__global__ __launch_bounds__(kThreads) void scatter_rows_ordered(const KernelGeom g, const LaunchView view,
                                                                 const LayerPtrs layers,
                                                                 const uint2 *__restrict__ pairs,
                                                                 const uint32_t *__restrict__ n_rows_at,
                                                                 const uint8_t *staging, FastDiv by_tiles_per_group,
                                                                 FastDiv by_chunk_tokens, uint32_t group_rows,
                                                                 uint32_t n_blocks_permuted, uint32_t xcd_shift) {
    typedef typename VecOf<VEC>::type V;
    const TileArgs a = fetch_args<VEC>(g, view, nullptr, const_cast<uint8_t *>(staging), nullptr);
    const FastDiv by_tiles = pin(by_tiles_per_group), by_ct = pin(by_chunk_tokens);
    const uint64_t pairs_at = pin(uint64_t(pairs));
    const uint32_t n_rows = pin(*n_rows_at), rows = pin(group_rows);
    const uint32_t blk = permuted_block(blockIdx.x, n_blocks_permuted, xcd_shift);
    const uint32_t q = by_tiles.div(blk);
    const uint32_t tile = blk - q * by_tiles.d;
    const uint32_t grp = a.by_lp.div(q);
    const uint32_t lp = q - grp * a.by_lp.d;
    const uint32_t r = tile * kThreads + threadIdx.x;
    const uint32_t row = a.by_row.div(r);
    const uint32_t w = r - row * a.by_row.d;
    const uint32_t j = grp * rows + row;
    if (row >= rows || j >= n_rows) return;
    const typename VecOf<8>::type pr = load_vec<typename VecOf<8>::type, false>(pairs_at + uint64_t(j) * 8u);
    const uint64_t layer = pin(uint64_t(layers.p[a.lp_base + lp]));
    const uint32_t su = pr.x, tok = pr.y;
    const uint32_t c = by_ct.div(tok);
    const uint32_t t = tok - c * by_ct.d;
    const uint32_t b = a.by_bs.div(su);
    const uint32_t o = su - b * a.by_bs.d;
    int64_t in_page;
    uint64_t in_row;
    place<VEC>(a, w, &in_page, &in_row);
    const uint64_t page = layer + uint64_t(int64_t(b) * a.block_stride + int64_t(o) * a.token_stride + in_page);
    const uint64_t row_bytes = VEC == kWide ? a.row_bytes : a.by_row.d * kBytesOf<VEC>;
    const uint64_t st = a.staging_at + uint64_t(c) * a.chunk_stride + uint64_t(lp) * a.plane_bytes +
                        t * row_bytes + in_row;
    store_vec<V, NT_ST>(page, load_vec<V, NT_LD>(st));
}

__global__ __launch_bounds__(kThreads) void check_slots(const int64_t *__restrict__ slot_mapping,
                                                        uint64_t n, uint32_t n_slots,
                                                        int32_t *bad_flag) {
    uint64_t i = uint64_t(blockIdx.x) * kThreads + threadIdx.x;
    const uint64_t step = uint64_t(gridDim.x) * kThreads;
    bool bad = false;
    for (; i < n; i += step) bad |= slot_mapping[i] >= int64_t(n_slots);
    if (bad) *bad_flag = 1;
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Streaming copy, one 16-byte vector per lane, non-temporal loads, stores through the L2: the
// fastest of the plain-copy shapes measured on this part.
__global__ __launch_bounds__(kThreads) void copy_bytes(u32x4 *__restrict__ dst,
                                                       const u32x4 *__restrict__ src, uint64_t n_vec) {
    const uint64_t i = uint64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n_vec) store_through(uint64_t(dst + i), __builtin_nontemporal_load(src + i));
}

// Plain copy of 4 KiB tiles in a given order, no slot mapping, no geometry: workgroup w
// copies tile src_order[w] of src to tile dst_order[w] of dst (a null order = w itself).
// Fed with the address stream of a gather or scatter launch it shows what the access
// pattern alone costs: the ceiling that launch can reach.  mode 1 only reads, mode 2 only
// writes (reads and writes react differently to scattered pages).
__global__ __launch_bounds__(kThreads) void copy_tiles(u32x4 *dst, const uint32_t *__restrict__ dst_order,
                                                       const u32x4 *src, const uint32_t *__restrict__ src_order,
                                                       uint32_t n_tiles, uint32_t mode, u32x4 *sink) {
    const uint32_t w = blockIdx.x;
    if (w >= n_tiles) return;
    const uint64_t s = (src_order ? uint64_t(src_order[w]) : uint64_t(w)) * kThreads + threadIdx.x;
    const uint64_t d = (dst_order ? uint64_t(dst_order[w]) : uint64_t(w)) * kThreads + threadIdx.x;
    if (mode == 0) {
        store_through(uint64_t(dst + d), __builtin_nontemporal_load(src + s));
    } else if (mode == 1) {
        const u32x4 v = __builtin_nontemporal_load(src + s);
        if (v.x == 0x9E3779B9u && v.y == 0x7F4A7C15u && v.z == 0xF39CC060u && v.w == 0x5CEDC834u) *sink = v;
    } else {
        const u32x4 v = {w, w, w, w};
        __builtin_nontemporal_store(v, dst + d);
    }
}

// Copy between device memory and the pinned pool, paced for the host link like
// gather_paced: a fixed, small grid whose workgroups take 4 KiB tiles in turn.  The
// bytes form `rows` rows of width_vec 16-byte vectors, src_pitch / dst_pitch bytes apart
// (one row per chunk; pitch == width gives a plain copy).
// By 48 groups that keep their compute units to themselves 57.5 GB/s from the host and 57.0 to it, by
// 64 57.1 to it (64 that do not: 57.5, 57.1): rectangles to the host go by all the groups.
template <bool TO_POOL>
__global__ __launch_bounds__(kPacedThreads) void copy_rect_paced(uint8_t *__restrict__ dst, uint64_t dst_pitch,
                                                            const uint8_t *__restrict__ src,
                                                            uint64_t src_pitch, uint64_t width_vec,
                                                            FastDiv by_tiles_per_row, uint32_t n_tiles, uint32_t groups) {
    const uint64_t dst_at = pin(uint64_t(dst)), src_at = pin(uint64_t(src));
    const uint64_t dp = pin(dst_pitch), sp = pin(src_pitch), wv = pin(width_vec);
    const FastDiv by_tpr = pin(by_tiles_per_row);
    const uint32_t step = pin(groups), end = pin(n_tiles), lane = threadIdx.x % kThreads;
    const uint32_t first = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads) * gridDim.x + blockIdx.x;
    if (first >= step) return;                       // an odd number of groups leaves a half without work
    for (uint32_t t = first; t < end; t += step) {
        const uint32_t row = by_tpr.div(t);
        const uint64_t v = uint64_t(t - row * by_tpr.d) * kThreads + lane;
        if (v >= wv) continue;
        const u32x4 x = load_vec<u32x4, true>(src_at + uint64_t(row) * sp + v * 16u);
        if (TO_POOL) store_through(dst_at + uint64_t(row) * dp + v * 16u, x);
        else store_vec<u32x4, true>(dst_at + uint64_t(row) * dp + v * 16u, x);
    }
}

// The same for pieces that lie in pool slots of any numbers (a fragmented pool): the row
// on the pool's side starts at slot[row] * pool_pitch.  One launch for all the pieces of a
// pipeline step, where the runtime would make one small copy per piece.
template <bool TO_POOL>
__global__ __launch_bounds__(kPacedThreads) void copy_pieces_paced(uint8_t *__restrict__ pool, uint64_t pool_pitch,
                                                              uint8_t *__restrict__ staging, uint64_t stage_pitch,
                                                              uint64_t width_vec, FastDiv by_tiles_per_row,
                                                              uint32_t n_tiles, uint32_t groups, PieceSlots slots) {
    const uint64_t pool_at = pin(uint64_t(pool)), stage_at = pin(uint64_t(staging));
    const uint64_t pp = pin(pool_pitch), sp = pin(stage_pitch), wv = pin(width_vec);
    const FastDiv by_tpr = pin(by_tiles_per_row);
    const uint32_t step = pin(groups), end = pin(n_tiles), lane = threadIdx.x % kThreads;
    const uint32_t first = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads) * gridDim.x + blockIdx.x;
    if (first >= step) return;                       // an odd number of groups leaves a half without work
    for (uint32_t t = first; t < end; t += step) {
        const uint32_t row = by_tpr.div(t);
        const uint64_t v = uint64_t(t - row * by_tpr.d) * kThreads + lane;
        if (v >= wv) continue;
        const uint64_t in_pool = pool_at + uint64_t(uint32_t(slots.slot[row])) * pp + v * 16u;
        const uint64_t in_stage = stage_at + uint64_t(row) * sp + v * 16u;
        const u32x4 x = load_vec<u32x4, true>(TO_POOL ? in_stage : in_pool);
        if (TO_POOL) store_through(in_pool, x);
        else store_vec<u32x4, true>(in_stage, x);
    }
}

__global__ __launch_bounds__(kThreads) void fill_bytes(uint8_t *dst, uint8_t value, uint64_t n) {
    const uint64_t step = uint64_t(gridDim.x) * kThreads;
    for (uint64_t i = uint64_t(blockIdx.x) * kThreads + threadIdx.x; i < n; i += step)
        dst[i] = value;
}

// Inside HBM.
template <int VEC, bool GATHER>
hipError_t launch_move_v(const KernelGeom &g, const LaunchView &v, const LaunchShape &s,
                         const LayerPtrs &layers, const int64_t *slot_mapping, uint32_t n_chunks,
                         uint8_t *staging, int32_t *bad_flag, hipStream_t stream, hipEvent_t start,
                         hipEvent_t stop) {
    const uint32_t n_blocks = n_chunks * v.by_n_lp.d * g.by_tiles_per_plane.d;
    if (n_blocks == 0) return hipSuccess;
    uint32_t shift = 0, permuted = 0;
    if (s.xcd_run > 0) {
        while ((2u << shift) <= s.xcd_run) shift++;                      // floor(log2(xcd_run))
        // Gathers like runs eight times as long, if there are four for every XCD; scatters do not.  Runs of 32
        // and 256 tiles, launches on three streams in turn: Llama-3-8B shape 512 and 128 MiB 178.2, 176.7
        // and 45.6, 44.7 us, 70B 480 MiB 168.1, 166.7, MLA fp8 and bf16 256 MiB 91.1, 89.6 and 84.7, 83.2,
        // 216-byte rows 128 MiB 50.6, 50.6 (the scatter of the first: 194.9, 196.4).
        for (int k = 0; GATHER && k < 3 && (64u << shift) <= n_blocks; k++) shift++;
        permuted = n_blocks & ~((8u << shift) - 1u);                     // the tail keeps its order
    }
    const dim3 grid(n_blocks), block(kThreads);
    if constexpr (GATHER && VEC == 16)
        if (g.by_vec_per_run.d % 64 == 0 && s.nt_load && s.nt_store && reinterpret_cast<uintptr_t>(slot_mapping) % 8 == 0) {
            hipExtLaunchKernelGGL(gather_rows_by_wave, grid, block, 0, stream, start, stop, 0, g, v, layers, slot_mapping,
                                  staging, bad_flag, permuted, shift);
            return hipGetLastError();
        }
    // Large scatters write at system scope and in the plain order of the tiles: each stream of writes
    // sweeps its own buffer, and launches of several streams that run into each other lose less
    // to one another.  Non-temporal with runs of 32 and so, 256 MiB on one stream and on three in turn: 32 KiB
    // pages 93.7, 92.3 and 96.7, 94.3 us, 16 KiB 93.8, 93.5 and 97.8, 96.0, 8 KiB 94.8, 95.0 and 98.9, 96.8,
    // MLA bf16 89.0, 87.3 and 90.5, 88.5, one-token pages of 1 and 4 KiB 95.5, 95.9 and 99.5, 98.1;
    // 92.5, 91.8 and 97.3, 95.1; 512 MiB of the first 189.3, 188.8 and 196.9, 192.6, 192 MiB 70.3, 69.0 and
    // 70.7, 70.0.  160 MiB are the same or 1 % slower, less is the same either way.  Smaller pieces (256-byte
    // rows in 4 KiB pages: 96.9, 98.4 on one stream) and rows whose wavefronts write lines in parts
    // (pages by head: 92.6, 99.6) lose.
    constexpr uint64_t kLargeScatter = uint64_t(192) << 20;
    const uint64_t moved = uint64_t(n_chunks) * v.by_n_lp.d * g.plane_bytes;
    const bool large_pieces =
        g.runs_per_row == 1 && ((g.row_bytes % 128 == 0 && g.row_bytes >= 1024) ||
                                (g.token_stride == int64_t(g.row_bytes) && uint64_t(g.by_block_size.d) * g.row_bytes >= 8192));
    if constexpr (!GATHER && VEC == 16)
        if (moved >= kLargeScatter && large_pieces && s.nt_load && s.nt_store) {
            hipExtLaunchKernelGGL((move_rows<VEC, GATHER, true, kStoreThrough>), grid, block, 0, stream, start, stop, 0, g, v,
                                  layers, slot_mapping, staging, bad_flag, 0u, 0u);
            return hipGetLastError();
        }
#define LMC_GO(LD, ST)                                                                          \
    hipExtLaunchKernelGGL((move_rows<VEC, GATHER, LD, ST>), grid, block, 0, stream, start, stop, \
                          0, g, v, layers, slot_mapping, staging, bad_flag, permuted, shift)
    if (s.nt_load && s.nt_store) LMC_GO(true, kStoreNonTemporal);
    else if (s.nt_load) LMC_GO(true, kStorePlain);
    else if (s.nt_store) LMC_GO(false, kStoreNonTemporal);
    else LMC_GO(false, kStorePlain);
#undef LMC_GO
    return hipGetLastError();
}

// How many of the groups asked for a launch gets where three quarters do.  A measured point, no law: the
// rate does not grow steadily with the groups (figures at each use), and why is not known.
uint32_t paced_part(uint32_t groups) { return std::max(1u, groups - groups / 4); }

// Pages into the pool.
template <int VEC>
hipError_t launch_gather_paced(const KernelGeom &g, const LaunchView &v, const LaunchShape &s,
                               const LayerPtrs &layers, const int64_t *slot_mapping, uint32_t n_chunks,
                               uint8_t *pool, int32_t *bad_flag, hipStream_t stream, hipEvent_t start,
                               hipEvent_t stop, const ChunkList *list, HostWord *told) {
    const uint32_t n_blocks = n_chunks * v.by_n_lp.d * g.by_tiles_per_plane.d;
    if (n_blocks == 0) return hipSuccess;
    // through the L2 where lanes write 16 bytes, which the pool's slots, chunks and planes are then multiples
    // of (16-byte runs make them so, packs() has looked).  Planes that begin inside a line of 128 bytes leave a wavefront's first and last line to two wavefronts, which costs the link less
    // than non-temporal stores do: 5.9 and 29 MiB in 360-byte rows (planes of 90720 bytes) 136 and
    // 597 us so, 124 and 582 through; 8 MiB in 208-byte rows, planes of 7488 bytes, 179 and 167.
    constexpr bool kLines = VEC == 16 || VEC == kPacked;
    const bool through = kLines && s.nt_load && s.nt_store;
    // blk + step must not wrap: n_blocks < 2^24 (max_chunks_per_launch) and the grid is small
    // The rate does not grow steadily with the groups: 8, 32 and 64 MiB by 32, 48, 64, 96, 128 of them
    // 166, 165, 167, 164, 163; 609, 605, 623, 606, 606; 1202, 1195, 1233, 1198, 1195 us (0.5 to 4 MiB
    // within 2 %), so three quarters of the 64 that the knob stands at, on as few compute units as
    // that takes: a product of 128 rows by 4096 x 4096 (31 us alone) takes 33 us beside 48 groups, 40
    // beside 96.  Pieces put together from two loads take longer: 8.7 MiB in 216-byte rows, planes of
    // 16 tokens, by 64 and 128: 189, 184 us.
    uint32_t groups = VEC == kPacked ? (n_blocks >= 512 ? 2 * s.paced_groups : s.paced_groups)
                      : through ? paced_part(s.paced_groups) : s.paced_groups;
    groups = std::min(n_blocks, groups);
    const dim3 grid((groups + 1) / 2), block(kPacedThreads);
    HostWord done{nullptr, nullptr, 0};
    if (told != nullptr && through) {
        done = *told;
        done.target += grid.x;
    }
#define LMC_GO(LD, ST)                                                                                  \
    if (list != nullptr)                                                                                \
        hipExtLaunchKernelGGL((gather_listed<VEC, LD, ST>), grid, block, s.paced_lds, stream, start, stop, 0, g, v, \
                              layers, slot_mapping, pool, bad_flag, n_blocks, groups, done, *list);     \
    else hipExtLaunchKernelGGL((gather_paced<VEC, LD, ST>), grid, block, s.paced_lds, stream, start, stop, 0, g, v, \
                          layers, slot_mapping, pool, bad_flag, n_blocks, groups, done)
    if (s.nt_load && s.nt_store) { LMC_GO(true, (kLines ? kStoreThrough : kStoreNonTemporal)); }
    else if (s.nt_load) { LMC_GO(true, kStorePlain); }
    else if (s.nt_store) { LMC_GO(false, kStoreNonTemporal); }
    else { LMC_GO(false, kStorePlain); }
#undef LMC_GO
    const hipError_t e = hipGetLastError();
    if (told != nullptr && e == hipSuccess && done.word != nullptr) told->target = done.target;
    return e;
}

// The pool into pages, `planes` planes of every chunk in each step.  The non-temporal hints of the
// launch shape are for HBM and change nothing here.
template <int VEC>
hipError_t launch_scatter_paced(const KernelGeom &g, const LaunchView &v, const LaunchShape &s, uint32_t planes,
                                const LayerPtrs &layers, const int64_t *slot_mapping, uint32_t n_chunks,
                                const uint8_t *pool, int32_t *bad_flag, hipStream_t stream, hipEvent_t start,
                                hipEvent_t stop, const ChunkList *list, Arrivals *arrivals) {
    const uint64_t tiles = uint64_t(n_chunks) * v.by_n_lp.d * g.by_tiles_per_plane.d;   // < 2^24 (max_chunks_per_launch)
    if (arrivals != nullptr) arrivals->count = 0;
    if (tiles == 0) return hipSuccess;
    LaunchView step = v;
    step.by_n_lp = make_fastdiv(planes);
    StepView steps;
    steps.n_steps = (v.by_n_lp.d + planes - 1) / planes;
    const uint32_t last = v.by_n_lp.d - (steps.n_steps - 1) * planes;
    steps.n_blocks = n_chunks * planes * g.by_tiles_per_plane.d;
    steps.last_blocks = n_chunks * last * g.by_tiles_per_plane.d;
    steps.by_last_lp = make_fastdiv(last);
    // 64 MiB by 32, 48, 64, 96 groups: 1189, 1182, 1183, 1227 us; 12 MiB by 48, 64: 225, 225; 0.5 MiB alike
    steps.groups = uint32_t(std::min<uint64_t>(tiles, paced_part(s.paced_groups)));
    const dim3 grid((steps.groups + 1) / 2), block(kPacedThreads);
    uint64_t *words = arrivals != nullptr && arrivals->host == nullptr ? arrivals->words : nullptr;
    HostWord told{nullptr, nullptr, 0};
    const bool tells = arrivals != nullptr && arrivals->host != nullptr;
    if (tells) told = HostWord{arrivals->words, arrivals->host, arrivals->reached + grid.x};
    if (list != nullptr)
        hipExtLaunchKernelGGL((scatter_paced<VEC, ChunkList>), grid, block, s.paced_lds, stream, start, stop, 0, g, step, steps, layers,
                              slot_mapping, pool, bad_flag, words, told, *list);
    else
        hipExtLaunchKernelGGL((scatter_paced<VEC, BackToBack>), grid, block, s.paced_lds, stream, start, stop, 0, g, step, steps, layers,
                              slot_mapping, pool, bad_flag, words, told, BackToBack{});
    const hipError_t e = hipGetLastError();
    if (arrivals != nullptr && e == hipSuccess) arrivals->count = tells ? grid.x : steps.groups * (kThreads / 64);
    return e;
}

// A gather of wide rows into the pool, whose planes are whole 16-byte pieces, goes piece by
// piece of the chunk (kPacked) instead of row by row: whole lines are written, which may then
// go through the L2.  44 MiB in 216-byte rows: 871 us with 8-byte lanes, 816 so; in 360-byte
// rows, whose planes are no whole lines, 934 and 869.  Inside HBM the second load and the
// shifts cost more than that is worth (121 MiB in 216-byte rows: 61.7 us against 44 row by row).
bool packs(const KernelGeom &g, const LaunchView &v, const uint8_t *staging) {
    return g.vec == uint32_t(kWide) && g.plane_bytes < (uint64_t(1) << 31) &&
           ((uint64_t(reinterpret_cast<uintptr_t>(staging)) | v.chunk_stride | g.plane_bytes) % 16) == 0;
}
KernelGeom packed_geom(const KernelGeom &g) {
    KernelGeom p = g;
    p.vec_per_plane = uint32_t(g.plane_bytes / 16);
    p.by_tiles_per_plane = make_fastdiv((p.vec_per_plane + kThreads - 1) / kThreads);
    p.by_vec_per_run = make_fastdiv(g.run_bytes);
    p.by_vec_per_row = make_fastdiv(g.runs_per_row);
    return p;
}

// Calls f with the lane width of the geometry as a compile-time constant.
template <typename F> hipError_t by_vec(const KernelGeom &g, F f) {
    switch (g.vec) {
        case kWide: return f(std::integral_constant<int, kWide>());
        case 16: return f(std::integral_constant<int, 16>());
        case 8: return f(std::integral_constant<int, 8>());
        case 4: return f(std::integral_constant<int, 4>());
        case 2: return f(std::integral_constant<int, 2>());
        case 1: return f(std::integral_constant<int, 1>());
    }
    return hipErrorInvalidValue;
}

}  // namespace

FastDiv make_fastdiv(uint32_t d) {
    FastDiv f;
    f.d = d;
    if (d <= 1) {
        f.mul = 0;
        f.shift = 0;
        return f;
    }
    uint32_t l = 0;
    while ((uint64_t(1) << l) < d) l++;
    f.mul = uint32_t((uint64_t(1) << (31 + l)) / d + 1);
    f.shift = l - 1;
    return f;
}

uint32_t max_chunks_per_launch(const KernelGeom &g, const LaunchView &v) {
    // the workgroup index must stay below 2^31 for the fast division, and a launch's
    // thread count (workgroups x 256) below 2^32, the stricter of the two: 2^24 - 1
    // workgroups, 64 GiB at 4 KiB tiles
    return uint32_t(0x00FFFFFFu / (uint64_t(v.by_n_lp.d) * g.by_tiles_per_plane.d));
}

LaunchView bulk_view(const KernelGeom &g) {
    LaunchView v;
    v.by_n_lp = make_fastdiv(g.n_layer_planes);
    v.lp_base = 0;
    v.chunk_stride = g.chunk_bytes;
    return v;
}

LaunchView layer_view(const KernelGeom &g, uint32_t planes_per_layer, uint32_t first_layer,
                      uint32_t n_layers) {
    LaunchView v;
    v.by_n_lp = make_fastdiv(n_layers * planes_per_layer);
    v.lp_base = first_layer * planes_per_layer;
    v.chunk_stride = uint64_t(n_layers) * planes_per_layer * g.plane_bytes;
    return v;
}

hipError_t launch_gather(const KernelGeom &g, const LaunchView &v, const LaunchShape &s,
                         const LayerPtrs &layers, const int64_t *slot_mapping, uint32_t n_chunks,
                         uint8_t *staging, int32_t *bad_flag, hipStream_t stream, hipEvent_t start,
                         hipEvent_t stop, const ChunkList *list, HostWord *told) {
    if (list != nullptr && (s.paced_groups == 0 || n_chunks > uint32_t(kMaxListed))) return hipErrorInvalidValue;
    if (s.paced_groups > 0 && packs(g, v, staging))
        return launch_gather_paced<kPacked>(packed_geom(g), v, s, layers, slot_mapping, n_chunks, staging, bad_flag, stream,
                                            start, stop, list, told);
    return by_vec(g, [&](auto vec) {
        return s.paced_groups > 0
                   ? launch_gather_paced<vec.value>(g, v, s, layers, slot_mapping, n_chunks, staging, bad_flag, stream, start,
                                                    stop, list, told)
                   : launch_move_v<vec.value, true>(g, v, s, layers, slot_mapping, n_chunks, staging, bad_flag, stream, start, stop);
    });
}

hipError_t launch_scatter(const KernelGeom &g, const LaunchView &v, const LaunchShape &s,
                          const LayerPtrs &layers, const int64_t *slot_mapping, uint32_t n_chunks,
                          const uint8_t *staging, int32_t *bad_flag, hipStream_t stream,
                          hipEvent_t start, hipEvent_t stop, const ChunkList *list, Arrivals *arrivals,
                          uint32_t planes_per_step) {
    if (list != nullptr && n_chunks > uint32_t(kMaxListed)) return hipErrorInvalidValue;
    if (s.paced_groups == 0 && (list != nullptr || arrivals != nullptr || planes_per_step != 0)) return hipErrorInvalidValue;
    const uint32_t planes = planes_per_step == 0 ? v.by_n_lp.d : std::min(planes_per_step, v.by_n_lp.d);
    if (arrivals != nullptr && arrivals->host != nullptr && planes != v.by_n_lp.d) return hipErrorInvalidValue;
    return by_vec(g, [&](auto vec) {
        return s.paced_groups > 0
                   ? launch_scatter_paced<vec.value>(g, v, s, planes, layers, slot_mapping, n_chunks, staging,
                                                     bad_flag, stream, start, stop, list, arrivals)
                   : launch_move_v<vec.value, false>(g, v, s, layers, slot_mapping, n_chunks, const_cast<uint8_t *>(staging),
                                                     bad_flag, stream, start, stop);
    });
}

uint64_t order_table_words(const KernelGeom &g) { return g.n_slots; }
uint64_t order_count_words(const KernelGeom &g) { return (uint64_t(g.n_slots) + kSlotsPerGroup - 1) / kSlotsPerGroup; }

// rows per group: the launch's choice, rounded so that a group is whole tiles where it can be
static uint32_t ordered_group_rows(const KernelGeom &g, const LaunchShape &s, uint64_t n_tokens) {
    uint64_t rows = s.ordered_group_rows == 0 ? n_tokens : std::min<uint64_t>(s.ordered_group_rows, n_tokens);
    return uint32_t(std::max<uint64_t>(rows, 1));
}

static uint64_t ordered_blocks(const KernelGeom &g, const LaunchView &v, uint64_t n_tokens, uint64_t rows) {
    const uint64_t tiles_per_group = (rows * g.by_vec_per_row.d + kThreads - 1) / kThreads;
    const uint64_t groups = (n_tokens + rows - 1) / rows;
    return groups * v.by_n_lp.d * tiles_per_group;
}

bool ordered_scatter_fits(const KernelGeom &g, const LaunchView &v, const LaunchShape &s, uint64_t n_tokens) {
    if (n_tokens == 0 || n_tokens >= (uint64_t(1) << 31) || g.n_slots > kMaxOrderedSlots) return false;
    const uint64_t rows = ordered_group_rows(g, s, n_tokens);
    if (rows * g.by_vec_per_row.d >= (uint64_t(1) << 31)) return false;   // lanes of one group and plane
    return ordered_blocks(g, v, n_tokens, rows) <= 0x00FFFFFFu;           // as max_chunks_per_launch
}

template <int VEC>
static hipError_t launch_scatter_ordered_v(const KernelGeom &g, const LaunchView &v, const LaunchShape &s,
                                           const LayerPtrs &layers, uint32_t n_tokens, const OrderScratch &o,
                                           const uint8_t *staging, hipStream_t stream, hipEvent_t start,
                                           hipEvent_t stop) {
    const uint32_t rows = ordered_group_rows(g, s, n_tokens);
    const uint32_t tiles_per_group = uint32_t((uint64_t(rows) * g.by_vec_per_row.d + kThreads - 1) / kThreads);
    const uint32_t n_blocks = uint32_t(ordered_blocks(g, v, n_tokens, rows));
    uint32_t shift = 0, permuted = 0;
    if (s.xcd_run > 0) {
        while ((2u << shift) <= s.xcd_run) shift++;
        permuted = n_blocks & ~((8u << shift) - 1u);
    }
    const FastDiv by_tiles = make_fastdiv(tiles_per_group), by_ct = make_fastdiv(g.chunk_tokens);
    dim3 grid(n_blocks), block(kThreads);
#define LMC_GO(LD, ST)                                                                                 \
    hipExtLaunchKernelGGL((scatter_rows_ordered<VEC, LD, ST>), grid, block, 0, stream, start, stop, 0, g, \
                          v, layers, o.pairs, o.n_rows, staging, by_tiles, by_ct, rows, permuted, shift)
    if (s.nt_load && s.nt_store) LMC_GO(true, true);
    else if (s.nt_load) LMC_GO(true, false);
    else if (s.nt_store) LMC_GO(false, true);
    else LMC_GO(false, false);
#undef LMC_GO
    return hipGetLastError();
}

hipError_t launch_scatter_ordered(const KernelGeom &g, const LaunchView &v, const LaunchShape &s,
                                  const LayerPtrs &layers, const int64_t *slot_mapping, uint32_t n_tokens,
                                  const OrderScratch &o, const uint8_t *staging, int32_t *bad_flag,
                                  hipStream_t stream, hipEvent_t start, hipEvent_t stop) {
    if (n_tokens == 0) return hipSuccess;
    const uint32_t n_slots = g.n_slots;
    const uint32_t n_groups = uint32_t(order_count_words(g));
    const dim3 block(kThreads);
    hipLaunchKernelGGL(order_clear, dim3((n_slots + kThreads - 1) / kThreads), block, 0, stream, o.token_at, n_slots);
    hipLaunchKernelGGL(order_mark, dim3((n_tokens + kThreads - 1) / kThreads), block, 0, stream, slot_mapping,
                       n_tokens, n_slots, o.token_at, bad_flag);
    hipLaunchKernelGGL(order_count, dim3(n_groups), block, 0, stream, o.token_at, n_slots, o.counts);
    hipLaunchKernelGGL(order_offsets, dim3(1), dim3(1024), 0, stream, o.counts, n_groups, o.n_rows);
    hipLaunchKernelGGL(order_emit, dim3(n_groups), block, 0, stream, o.token_at, n_slots, o.counts, o.pairs);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    switch (g.vec) {
        case kWide: return launch_scatter_ordered_v<kWide>(g, v, s, layers, n_tokens, o, staging, stream, start, stop);
        case 16: return launch_scatter_ordered_v<16>(g, v, s, layers, n_tokens, o, staging, stream, start, stop);
        case 8: return launch_scatter_ordered_v<8>(g, v, s, layers, n_tokens, o, staging, stream, start, stop);
        case 4: return launch_scatter_ordered_v<4>(g, v, s, layers, n_tokens, o, staging, stream, start, stop);
        case 2: return launch_scatter_ordered_v<2>(g, v, s, layers, n_tokens, o, staging, stream, start, stop);
        case 1: return launch_scatter_ordered_v<1>(g, v, s, layers, n_tokens, o, staging, stream, start, stop);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_check_slots(const int64_t *slot_mapping, uint64_t n, uint32_t n_slots,
                              int32_t *bad_flag, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    uint64_t blocks = (n + kThreads - 1) / kThreads;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(check_slots, dim3(uint32_t(blocks)), dim3(kThreads), 0, stream, slot_mapping,
                       n, n_slots, bad_flag);
    return hipGetLastError();
}

hipError_t launch_copy(uint8_t *dst, const uint8_t *src, uint64_t nbytes, hipStream_t stream) {
    const uint64_t n_vec = nbytes / 16;
    const uint64_t per_launch = uint64_t(0x00FFFFFFu) * kThreads;   // a launch's threads stay below 2^32
    for (uint64_t v0 = 0; v0 < n_vec; v0 += per_launch) {
        const uint64_t n = n_vec - v0 < per_launch ? n_vec - v0 : per_launch;
        hipLaunchKernelGGL(copy_bytes, dim3(uint32_t((n + kThreads - 1) / kThreads)), dim3(kThreads),
                           0, stream, reinterpret_cast<u32x4 *>(dst) + v0,
                           reinterpret_cast<const u32x4 *>(src) + v0, n);
    }
    return hipGetLastError();
}

hipError_t launch_copy_tiles(uint8_t *dst, const uint32_t *dst_order, const uint8_t *src,
                             const uint32_t *src_order, uint32_t n_tiles, uint32_t mode, uint8_t *sink,
                             hipStream_t stream) {
    if (n_tiles == 0) return hipSuccess;
    if (n_tiles > 0x7FFFFFFFu || mode > 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(copy_tiles, dim3(n_tiles), dim3(kThreads), 0, stream, reinterpret_cast<u32x4 *>(dst), dst_order,
                       reinterpret_cast<const u32x4 *>(src), src_order, n_tiles, mode, reinterpret_cast<u32x4 *>(sink));
    return hipGetLastError();
}

hipError_t launch_copy_rect(uint8_t *dst, uint64_t dst_pitch, const uint8_t *src, uint64_t src_pitch,
                            uint64_t width, uint64_t rows, bool to_pool, uint32_t groups, uint32_t lds, hipStream_t stream) {
    if (width == 0 || rows == 0) return hipSuccess;
    if ((width % 16) != 0 || (dst_pitch % 16) != 0 || (src_pitch % 16) != 0 || groups == 0 ||
        (reinterpret_cast<uintptr_t>(dst) % 16) != 0 || (reinterpret_cast<uintptr_t>(src) % 16) != 0)
        return hipErrorInvalidValue;
    const uint64_t width_vec = width / 16;
    const uint64_t tiles_per_row = (width_vec + kThreads - 1) / kThreads;
    if (tiles_per_row >= (uint64_t(1) << 24)) return hipErrorInvalidValue;   // 64 GiB rows: not a chunk
    // the tile index is 32-bit and stays below 2^24, so t + grid never wraps and FastDiv is exact
    const uint64_t rows_per_launch = std::max<uint64_t>(1, uint64_t(0x00FFFFFFu) / tiles_per_row);
    for (uint64_t r0 = 0; r0 < rows; r0 += rows_per_launch) {
        const uint64_t n = std::min(rows - r0, rows_per_launch);
        const uint32_t n_tiles = uint32_t(n * tiles_per_row), used = std::min(n_tiles, to_pool ? groups : paced_part(groups));
        hipLaunchKernelGGL(to_pool ? copy_rect_paced<true> : copy_rect_paced<false>, dim3((used + 1) / 2),
                           dim3(kPacedThreads), lds, stream, dst + r0 * dst_pitch, dst_pitch, src + r0 * src_pitch, src_pitch,
                           width_vec, make_fastdiv(uint32_t(tiles_per_row)), n_tiles, used);
    }
    return hipGetLastError();
}

hipError_t launch_copy_pieces(uint8_t *pool, uint64_t pool_pitch, uint8_t *staging, uint64_t stage_pitch,
                              uint64_t width, const PieceSlots &slots, uint32_t n_pieces, bool to_pool,
                              uint32_t groups, uint32_t lds, hipStream_t stream) {
    if (width == 0 || n_pieces == 0) return hipSuccess;
    if ((width % 16) != 0 || (pool_pitch % 16) != 0 || (stage_pitch % 16) != 0 || groups == 0 ||
        n_pieces > uint32_t(kMaxPieces) || (reinterpret_cast<uintptr_t>(pool) % 16) != 0 ||
        (reinterpret_cast<uintptr_t>(staging) % 16) != 0)
        return hipErrorInvalidValue;
    for (uint32_t i = 0; i < n_pieces; i++)
        if (slots.slot[i] < 0) return hipErrorInvalidValue;
    const uint64_t width_vec = width / 16;
    const uint64_t tiles_per_row = (width_vec + kThreads - 1) / kThreads;
    // the tile index is 32-bit and stays below 2^24, so t + grid never wraps and FastDiv is exact
    if (tiles_per_row * n_pieces >= (uint64_t(1) << 24)) return hipErrorInvalidValue;
    const uint32_t n_tiles = uint32_t(tiles_per_row * n_pieces);
    // Pieces to the host move as fast by three quarters of the groups (16 and 32 chunks layer by
    // layer: 55.4 and 56.2 GB/s by 48 and by 64), pieces from it by all of them: loads layer by layer of 8,
    // 16, 32 chunks, two layers a step, 55.2, 55.3, 55.5 GB/s by 48, 56.0, 56.4, 56.7 by 64.  A product of
    // 128 rows by 4096 x 4096 (33 us alone) beside such a load takes 48-62 us with 48, 73-81 with 64
    // and took 145-360 with 64 that share their compute units.
    const uint32_t used = std::min(n_tiles, to_pool ? paced_part(groups) : groups);
    const dim3 grid((used + 1) / 2), block(kPacedThreads);
    if (to_pool)
        hipLaunchKernelGGL(copy_pieces_paced<true>, grid, block, lds, stream, pool, pool_pitch, staging, stage_pitch,
                           width_vec, make_fastdiv(uint32_t(tiles_per_row)), n_tiles, used, slots);
    else
        hipLaunchKernelGGL(copy_pieces_paced<false>, grid, block, lds, stream, pool, pool_pitch, staging, stage_pitch,
                           width_vec, make_fastdiv(uint32_t(tiles_per_row)), n_tiles, used, slots);
    return hipGetLastError();
}

hipError_t launch_fill(uint8_t *dst, uint8_t value, uint64_t nbytes, hipStream_t stream) {
    if (nbytes == 0) return hipSuccess;
    uint64_t blocks = (nbytes + kThreads - 1) / kThreads;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_bytes, dim3(uint32_t(blocks)), dim3(kThreads), 0, stream, dst, value,
                       nbytes);
    return hipGetLastError();
}

}  // namespace lmc
