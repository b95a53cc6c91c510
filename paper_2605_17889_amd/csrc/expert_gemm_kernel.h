// Grouped expert GEMM kernels for gfx950 (device code; included by expert_gemm.hip).
//
//   C[p, n] = sum_k A[p, k] * B_e[n, k]           for the rows p of expert e's group,
// both operands contiguous along k ("NT"), bf16 in, fp32 accumulation on
// v_mfma_f32_16x16x32_bf16, bf16 out. With DUAL, a tile carries BN/2 rows of W1 and the
// matching BN/2 rows of W3 (interleaved in blocks of 32 or 16) and stores SiLU(gate)*up.
//
// Data path: global memory -> LDS by direct-to-LDS loads (no VGPR staging); LDS -> VGPR by
// 16-byte reads of a swizzled layout; MFMA. Tiles are enumerated on the device from `offsets`.
//
// The 16x16x32 instruction is used instead of 32x32x16 because it does the same work per cycle
// with half the accumulator updates per multiply-add: under the board's power limit a loop of
// it sustains ~13 % more FLOP/s on random operands. The weight fragment is the first MFMA
// operand, so a lane ends up with four consecutive output columns of one row (one 8-byte store).
//
// Four kernels share the tile mapping, the LDS layout and the fragment plan:
//   grouped_gemm_kernel       ring of NSTAGE LDS stages, compiler-scheduled k-step (small tiles:
//                           decode and micro-batch sized expert groups, HBM-bound);
//   grouped_gemm_routed_kernel  the same tiles for gate/up of a few tokens, which finds its groups
//                           in the selected experts instead of a permutation's tables;
//   grouped_gemm_1w_kernel    the large compute-bound tiles, one wavefront per SIMD: hand-placed
//                           software pipeline with at most a few other instructions behind every
//                           MFMA, tiles of five heights, in short reductions persistent workgroups;
//   grouped_gemm_ring_kernel  the large tiles with two wavefronts per SIMD (by moe_set_gemm_config,
//                           and what the one before does not take): the fragments of the next half
//                           k-step are read from LDS while the MFMAs of the current one issue, and
//                           the direct-to-LDS loads are spread between the MFMAs.
// In the last two the workgroup barrier sits in the middle of a k-step, so that MFMAs are ready on
// both sides of it, and the two operands have LDS rings of different depth.
#pragma once
#include <type_traits>

#include "common.h"
#include "permute_block.h"
#include "route_select.h"

namespace moe {
namespace gemm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kGroupM = 8;   // at most this many m-tiles that sweep the n-tiles together (share weight tiles)

struct TileCoord {
    int expert;      // negative: no tile for this workgroup (kNoTile, kEmptySlot)
    int row0;        // first row (in the permuted matrix) of the tile
    int rows;        // valid rows in the tile (1..BM)
    int nt;          // n-tile index
    int height;      // rows that its workgroup computes: BM / 2 to BM (see tile_in_expert)
};

// Map a workgroup to its tile. Logical tile order: expert by expert; inside an expert, groups
// of kGroupM m-tiles; inside a group the n-tiles, each visited by all m-tiles of the group in
// turn. XCD x is handed the x-th contiguous eighth of that order, so the workgroups resident
// together on one XCD share A rows and weight tiles in its L2.
//
// Every wavefront works the map out by itself, without LDS: lane l takes the four experts 4l..4l+3
// (five loads of their offsets in flight together), the tile counts are prefix-summed inside the
// lane and across the lanes (six row moves of the vector unit), and the lane whose range holds the
// tile number hands its expert to all. The cost does not grow with the number of experts (a scalar
// loop over 128 experts would cost more than a tile of a small expert). A lookup is a chain of
// latencies that nothing hides, paid by every tile: with the prefix sum through LDS, one 64-expert
// group after the other, and full integer divisions, 37 tokens through 128 experts took 243 us
// for the layer; in this form, and with the row indices of source_rows() fetched together, 231 us.
//
// split_cus > 0 (the pipelined kernel passes the number of compute units): a launch of `total`
// tiles runs in rounds of split_cus tiles, one per compute unit; when the last round is less
// than half full, each of its tiles is handed to two workgroups as an upper and a lower half
// of BM/2 rows, so that the round ends after a half-height tile instead of a full one. The
// halves are the highest slots of every XCD's range, hence the last workgroups dispatched.
//
// The tile is named by (xcd, slot): slot-th entry of XCD xcd's range; the kernels take both from
// the workgroup index. Result: expert >= 0: a tile of at least one row; kNoTile: the range is exhausted (every later
// slot is too); kEmptySlot: this slot holds nothing (the lower half of a tile that has none).
constexpr int kNoTile = -1, kEmptySlot = -2;

// a / b and a % b for a >= 0, b >= 1. A wavefront-uniform integer division takes some forty
// instructions of the vector unit; below 2^22 the float quotient is off by at most one.
__host__ __device__ __forceinline__ int div_small(int a, int b, int& rem) {
#if defined(__HIP_DEVICE_COMPILE__)
    if (a >= (1 << 22)) {
        const int q = a / b;
        rem = a - q * b;
        return q;
    }
    int q = static_cast<int>(static_cast<float>(a) * __builtin_amdgcn_rcpf(static_cast<float>(b)));
    q = __builtin_amdgcn_readfirstlane(q);
    int r = a - q * b;
    if (r < 0) { --q; r += b; }
    if (r >= b) { ++q; r -= b; }
    rem = r;
    return q;
#else
    rem = a % b;
    return a / b;
#endif
}

// The slots of one XCD's range of `total` tiles. A lookup gives a slot's place in the logical order, or -1 past
// the end of the range; `half` is 0 / 1 for the upper / lower half of a split tile, else -1.
struct SlotRange {
    int first, whole, slots;       // first tile; tiles that are not split, each one slot; all slots
    __device__ __forceinline__ void init(int total, int split_cus, int xcd) {
        const int per = (total + kXcds - 1) / kXcds;
        const int len = max(0, min(per, total - xcd * per));   // tiles in this XCD's range
        int halved = 0;                                        // of those, the last `halved` are split
        if (split_cus > 0) {
            int rem;
            div_small(total, split_cus, rem);
            if (rem > 0 && 2 * rem <= split_cus) halved = min(len, (rem + kXcds - 1) / kXcds);
        }
        first = xcd * per;
        whole = len - halved;
        slots = len + halved;
    }
    __device__ __forceinline__ int tile(int slot, int& half) const {
        half = -1;
        if (slot < whole) return first + slot;
        if (slot >= slots) return -1;
        half = (slot - whole) & 1;
        return first + whole + ((slot - whole) >> 1);
    }
};

constexpr int kLongK = 4096;         // reductions of this and more are long

// Whether the mt m-tiles of an expert of m_e rows share its rows evenly (see tile_in_expert). Short reductions always:
// 16384 skewed tokens through 128 experts of 2048 x 768 687 us whole, with experts of nine and fewer m-tiles cut 673,
// with all 665 (in quarters). In long ones a workgroup that ends early is out of step with those whose rows and
// weights it shares in L2, which costs more than a saving of few rows; with more than kLongCutTiles m-tiles the saving
// is small, and with six or eight little is gained by one tail less. Experts of at most four m-tiles are cut, whole ->
// cut: layers of 2500 tokens through 8 experts of 6144 x 16384 (625 rows each) 2658 -> 2488 us. Those of five to seven
// where the last tile would hold few rows, whole -> cut: 4200 tokens (1050) 4128 -> 3877, 4400 (1100) 4332 -> 3947,
// 5200 (1300, six) 4770 -> 4647, 6400 (1600, seven) 6059 -> 5677, 5300 at 4096 x 14336 2875 -> 2793. Past the lines,
// whole -> cut: six m-tiles with tails to 96 (5600) 4999 -> 5009, tails of 129 to 192 in five (4800) 4220 -> 4303, eight
// with tails to 64 (7200) 6352 -> 6513, eight and nine (8192) 7168 -> 7295. The lines at other shapes, 8 experts, exact
// groups, expert stage alone: 1050 rows of 4096 x 14336 2437 -> 2247, of 8192 x 8192 2742 -> 2520; 1320 of 8192 x 8192
// 3244 -> 3012; 1660 of 5120 x 12800 4339 -> 4207; 1850 (eight) of 8192 x 8192 4358 -> 4421, 2100 (nine) of 5120 x 12800
// 5428 -> 5311. Six m-tiles with tails of 65 to 128: where all groups are alike cutting them gains up to 1.1 % (1376 of
// 5120 x 12800) or nothing, but a layer's groups are not, and cut ones among whole ones lose: layers of 5500 or 5600 tokens
// 4948 -> 5052 (6144 x 16384), 2843 -> 2861 (4096 x 14336), 3263 -> 3301 (8192 x 8192), 3528 -> 3568 (5120 x 12800).
enum class Cut { kNever, kLong, kAlways };
constexpr int kLongCutTiles = 7;
template <int BM>
__host__ __device__ __forceinline__ bool tiles_are_cut(int m_e, int mt, Cut cut) {
    if (cut != Cut::kLong) return cut == Cut::kAlways;
    const int tail = m_e - (mt - 1) * BM;
    return mt <= 4 || (mt <= kLongCutTiles && tail <= (mt == 6 ? BM / 4 : BM / 2));
}

// Coordinates of tile `local` of the expert whose group is rows [row_e, row_e + m_e). The expert's
// mt m-tiles form ceil(mt / kGroupM) groups of nearly equal height (the first `extra` groups hold
// one tile more), so that a short tail tile sweeps the n-tiles together with full tiles of its
// expert and finds the weight tiles in L2.
//
// Tiles that are cut share the expert's rows in units of an eighth of a tile: 576 rows
// are 3 x 192 instead of 2 x 256 and a tail of 64, 520 are 192, 192 and 160. No tile is lower than half of one: a
// k-step of 192 rows takes 1536 cycles of matrix instructions and 56 loads, one of 128 rows, bound by its 48
// loads, hardly less than that. Rows that are padding cost time and, under the board's power limit, clock.
// Units of a quarter -> of an eighth, gate/up and down: 8192 tokens through 64 experts of 2048 x 1408 (664 to 871 rows
// each) 462 -> 431 and 257 -> 241 us, 5003 282 -> 270 and 196 -> 191 (fp32 outputs), 8192 through 128 of 2048 x 768
// 336 -> 325 and 234 -> 222, 1200 through 8 of 4096 x 14336 515 -> 520 and 295 -> 274 (those of short reductions
// together with the persistent workgroups, see grouped_gemm_1w_kernel).
template <int BM>
__host__ __device__ __forceinline__ TileCoord tile_in_expert(int expert, int row_e, int m_e, int local, int NT,
                                                             int half, Cut cut) {
    TileCoord tc{kNoTile, 0, 0, 0, 0};
    const int mt = (m_e + BM - 1) / BM;
    const int ngroups = (mt + kGroupM - 1) / kGroupM;
    int gm = mt, head = 0, in = local;
    if (ngroups > 1) {
        int extra;
        const int base = div_small(mt, ngroups, extra);
        const int big = extra * (base + 1) * NT;           // tiles in the taller groups
        if (local < big) {
            gm = base + 1;
            head = div_small(local, gm * NT, in) * gm;
        } else {
            gm = base;
            head = extra * (base + 1) + div_small(local - big, gm * NT, in) * gm;
        }
    }
    int mi;                                                // m-tile: first inside its group, then of the expert
    tc.nt = div_small(in, gm, mi);
    mi += head;
    int first = mi * BM;
    tc.height = BM;
    if (tiles_are_cut<BM>(m_e, mt, cut)) {
        constexpr int U = BM / 8;
        int extra;
        const int base = div_small((m_e + U - 1) / U, mt, extra);   // in units of U rows; `extra` tiles one more
        tc.height = max(BM / 2, (base + (mi < extra ? 1 : 0)) * U);
        first = (mi * base + min(mi, extra)) * U;
    }
    tc.row0 = row_e + first;
    tc.rows = min(tc.height, m_e - first);
    tc.expert = expert;
    if (half >= 0) {
        const int h0 = half * (BM / 2);
        tc.rows = max(0, min(BM / 2, tc.rows - h0));
        tc.row0 += tc.rows > 0 ? h0 : 0;
        if (tc.rows == 0) tc.expert = kEmptySlot;
    }
    if (tc.rows <= BM / 2) tc.height = BM / 2;
    return tc;
}

// Value of lane l - (move of CTRL) or 0, for the prefix sum below.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int row_move(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}
// Inclusive prefix sum over the 64 lanes: shifts by 1, 2, 4, 8 inside rows of 16 lanes, then lane 15
// of every row is added to the row behind it and lane 31 to the upper half.
__device__ __forceinline__ int lane_prefix_sum(int v) {
    v += row_move<0x111, 0xf>(v);
    v += row_move<0x112, 0xf>(v);
    v += row_move<0x114, 0xf>(v);
    v += row_move<0x118, 0xf>(v);
    v += row_move<0x142, 0xa>(v);
    v += row_move<0x143, 0xc>(v);
    return v;
}

// The same map for exactly 8 experts, on the scalar unit: the nine offsets are wavefront-uniform
// reads of memory that the kernel never writes, so they come through the scalar cache (a hit
// for every workgroup of a compute unit after the first) and the search is a handful of scalar
// instructions instead of vector loads, a prefix sum across lanes and a ballot.
template <int BM>
__device__ __forceinline__ TileCoord locate_tile_scalar8(const int32_t* __restrict__ offsets, int NT,
                                                         int split_cus, Cut cut, int xcd, int slot) {
    int off[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) off[e] = offsets[e];
    int incl[8];
    int total = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        total += ((off[e + 1] - off[e] + BM - 1) / BM) * NT;
        incl[e] = total;
    }
    SlotRange range;
    range.init(total, split_cus, xcd);
    int half;
    const int L = range.tile(slot, half);
    if (L < 0) return TileCoord{kNoTile, 0, 0, 0, 0};
    int e = 0;
#pragma unroll
    for (int i = 0; i < 7; ++i) e += (L >= incl[i]) ? 1 : 0;      // first expert whose range holds L
    int start = 0, m_e = 0, row_e = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (i == e) {
            start = i == 0 ? 0 : incl[i - 1];
            m_e = off[i + 1] - off[i];
            row_e = off[i];
        }
    return tile_in_expert<BM>(e, row_e, m_e, L - start, NT, half, cut);
}

// An XCD's range of the tiles, prepared for lookups: the tile counts of all experts over the lanes of a
// wavefront (lane l holds experts 4 l to 4 l + 3) and the range's slots.
template <int BM>
struct TileTable {
    static constexpr int EPL = kMaxExperts / kWave;        // experts per lane
    int off[EPL + 1], start[EPL + 1];                      // offsets; number of the first tile of each expert
    SlotRange range;
    __device__ __forceinline__ void init(const int32_t* __restrict__ offsets, int E, int NT, int split_cus, int xcd,
                                         int lane) {
        static_assert(EPL == 4, "in-lane search");
#pragma unroll
        for (int w = 0; w <= EPL; ++w) off[w] = offsets[min(lane * EPL + w, E)];
        init_tiles(NT, split_cus, xcd);
    }
    // the same from the number of rows of each expert
    __device__ __forceinline__ void init_from_counts(const int32_t* cnt, int E, int NT, int xcd, int lane) {
        off[0] = 0;
#pragma unroll
        for (int w = 0; w < EPL; ++w) off[w + 1] = off[w] + (lane * EPL + w < E ? cnt[lane * EPL + w] : 0);
        const int before = lane_prefix_sum(off[EPL]) - off[EPL];
#pragma unroll
        for (int w = 0; w <= EPL; ++w) off[w] += before;
        init_tiles(NT, 0, xcd);
    }
    __device__ __forceinline__ int first_row(int expert) const {
        int v = off[0];
#pragma unroll
        for (int w = 1; w < EPL; ++w) v = (expert & (EPL - 1)) == w ? off[w] : v;
        return __builtin_amdgcn_readlane(v, expert / EPL);
    }
    __device__ __forceinline__ void init_tiles(int NT, int split_cus, int xcd) {
        start[0] = 0;
#pragma unroll
        for (int w = 0; w < EPL; ++w) start[w + 1] = start[w] + ((off[w + 1] - off[w] + BM - 1) / BM) * NT;
        const int incl = lane_prefix_sum(start[EPL]), before = incl - start[EPL];
#pragma unroll
        for (int w = 0; w <= EPL; ++w) start[w] += before;
        range.init(__builtin_amdgcn_readlane(incl, kWave - 1), split_cus, xcd);
    }
    // `magic`: lane g holds floor(2^32 / g) + 1, so that a / g == (a * magic) >> 32 for 2 <= g and a * g < 2^32.
    __device__ __forceinline__ TileCoord find(int NT, Cut cut, int slot, uint32_t magic) const {
        int half;
        const int L = range.tile(slot, half);
        if (L < 0) return TileCoord{kNoTile, 0, 0, 0, 0};
        // The last lane whose first expert starts at or before tile L holds it. From there on everything is the
        // same in all lanes and computed on the scalar unit.
        const int src = 63 - __builtin_clzll(__ballot(L >= start[0]));
        int e = 0, first = __builtin_amdgcn_readlane(start[0], src);
        int row_e = __builtin_amdgcn_readlane(off[0], src), next = __builtin_amdgcn_readlane(off[1], src);
#pragma unroll
        for (int w = 1; w < EPL; ++w) {
            const int s = __builtin_amdgcn_readlane(start[w], src), o = __builtin_amdgcn_readlane(off[w + 1], src);
            const bool on = L >= s;
            e = on ? w : e;
            first = on ? s : first;
            row_e = on ? next : row_e;
            next = on ? o : next;
        }
        e += src * EPL;
        const int m_e = next - row_e, mt = (m_e + BM - 1) / BM;
        if (mt > kGroupM || half >= 0) return tile_in_expert<BM>(e, row_e, m_e, L - first, NT, half, cut);
        // tile_in_expert where the expert's tiles are one group and nothing is split
        constexpr uint32_t U = BM / 8;
        const uint32_t in = L - first, mul = __builtin_amdgcn_readlane(magic, mt), one = mt == 1 ? ~0u : 0u;
        const uint32_t nt = __umulhi(in, mul) + (in & one), mi = in - nt * mt;
        uint32_t base = 8, extra = 0;
        if (tiles_are_cut<BM>(m_e, mt, cut)) {
            const uint32_t units = (m_e + U - 1) / U;
            base = __umulhi(units, mul) + (units & one);
            extra = units - base * mt;
        }
        const int at = (mi * base + min(mi, extra)) * U, height = max(4u, base + (mi < extra ? 1u : 0u)) * U;
        const int rows = min(height, m_e - at);
        return TileCoord{e, row_e + at, rows, static_cast<int>(nt), rows <= BM / 2 ? BM / 2 : height};
    }
};
__device__ __forceinline__ uint32_t division_magic(int lane) { return lane < 2 ? 0u : 0xffffffffu / lane + 1u; }

// The same in every lane: into scalar registers, where the load addresses are formed.
__device__ __forceinline__ TileCoord uniform_tile(TileCoord tc) {
    tc.expert = __builtin_amdgcn_readfirstlane(tc.expert);
    tc.row0 = __builtin_amdgcn_readfirstlane(tc.row0);
    tc.rows = __builtin_amdgcn_readfirstlane(tc.rows);
    tc.nt = __builtin_amdgcn_readfirstlane(tc.nt);
    tc.height = __builtin_amdgcn_readfirstlane(tc.height);
    return tc;
}

// The tile of this workgroup where every workgroup has one.
template <int BM>
__device__ __forceinline__ TileCoord locate_tile(const int32_t* __restrict__ offsets, int E, int NT, int split_cus = 0,
                                                 Cut cut = Cut::kNever) {
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
    if (E == 8) return uniform_tile(locate_tile_scalar8<BM>(offsets, NT, split_cus, cut, xcd, slot));
    TileTable<BM> table;
    table.init(offsets, E, NT, split_cus, xcd, threadIdx.x & (kWave - 1));
    return uniform_tile(table.find(NT, cut, slot, division_magic(threadIdx.x & (kWave - 1))));
}

// LDS tile layout: rows of BK bf16 in 16-byte chunks; logical chunk c of row r is stored at
// chunk position c ^ swz(r). LDS has 64 four-byte banks and a 16-byte read is served 16 lanes
// at a time; the 16 lanes of a fragment read the same logical chunk of 16 consecutive rows,
// which the swizzle spreads over 16 distinct 16-byte slots of a 256-byte bank window.
template <int BK>
__device__ __forceinline__ int swz(int row) {
    if (BK == 64) return (row >> 1) & 7;     // 128-byte rows: 2 rows per bank window
    return (row >> 2) & 3;                   // 64-byte rows: 4 rows per bank window
}

// One direct-to-LDS load: every lane fetches 16 bytes from sbase + voff and the wavefront's
// 64 x 16 bytes land contiguously at LDS byte offset lds_off (wave-uniform, passed in M0).
// The compiler is not told that this is a memory operation with a counter: the kernels place
// their own s_waitcnt vmcnt(n) before the barrier that publishes a stage.
// STREAM marks the line non-temporal: for operand bytes that no other tile will ask for again
// (weights when every expert has a single m-tile), so that they do not displace reusable lines.
template <bool STREAM = false>
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff, uint32_t lds_off) {
    if constexpr (STREAM)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     :: "s"(lds_off), "v"(voff), "s"(sbase) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :: "s"(lds_off), "v"(voff), "s"(sbase) : "memory", "m0");
}

template <int N> __device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// SiLU with the hardware exponential and reciprocal (about 1 ulp each): the result is rounded
// to bf16 right away, and the exact division costs three times as many instructions in the
// epilogue of every gate/up tile.
__device__ __forceinline__ float silu(float a) { return a * __builtin_amdgcn_rcpf(1.0f + __expf(-a)); }

template <int BM_, int BN_, int BK_, int WM_, int WN_, int NSTAGE_, bool DUAL_,
          bool STREAM_B_ = false>
struct Config {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, NSTAGE = NSTAGE_;
    static constexpr bool DUAL = DUAL_;
    static constexpr bool STREAM_B = STREAM_B_;            // weights loaded as non-temporal
    static constexpr int NW = WM * WN, NTHREADS = NW * 64;
    static constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 16, TN = WTN / 16;
    static constexpr int KSUB = BK / 32;                   // MFMA k-substeps per stage
    static constexpr int ROW_BYTES = BK * 2;
    static constexpr int CPR = BK / 8;                     // 16-byte chunks per row
    static constexpr int RPI = 64 / CPR;                   // rows one wavefront load covers
    static constexpr int TILE_STEP = 16 * ROW_BYTES;       // LDS bytes between 16-row tiles
    static constexpr int A_BYTES = BM * ROW_BYTES, B_BYTES = BN * ROW_BYTES;
    static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int SMEM = NSTAGE * STAGE_BYTES;
    static constexpr int NIA = BM / RPI, NIB = BN / RPI;   // wavefront loads per stage
    static constexpr int LPW = (NIA + NIB) / NW;           // ... per wavefront
    static constexpr int BN_OUT = DUAL ? BN / 2 : BN;      // output columns per tile
    static constexpr int DB = WTN % 64 == 0 ? 32 : 16;     // DUAL: rows of W1, then as many of W3, in turn
    static_assert(BK == 64 || BK == 32, "LDS rows of 128 or 64 bytes");
    static_assert(BM % (WM * 16) == 0 && BN % (WN * 16) == 0, "wave tile");
    static_assert(!DUAL || WTN % (2 * DB) == 0, "gate and up of a column must live in one wave");
    static_assert(NIA % NW == 0 && NIB % NW == 0, "loads must split evenly over wavefronts");
    static_assert(NSTAGE >= 2 && SMEM <= 160 * 1024, "LDS budget");
};

// The same tiling with fp32 outputs: C is then a float matrix. Used for the down projection
// when the layer keeps the expert outputs in fp32 until the gate-weighted sum (one bf16
// rounding fewer per output element); the accumulation is identical.
template <class Cfg>
struct F32Out : Cfg {
    static constexpr bool OUT_F32 = true;
    static_assert(!Cfg::DUAL, "the gate/up intermediate stays bf16");
};
// The same tile with H rows.
template <class Cfg, int H> struct WithHeight;
template <int BM, int BN, int BK, int WM, int WN, int NSTAGE, bool DUAL, bool STREAM_B, int H>
struct WithHeight<Config<BM, BN, BK, WM, WN, NSTAGE, DUAL, STREAM_B>, H> {
    using type = Config<H, BN, BK, WM, WN, NSTAGE, DUAL, STREAM_B>;
};
template <class Cfg, int H>
struct WithHeight<F32Out<Cfg>, H> { using type = F32Out<typename WithHeight<Cfg, H>::type>; };
template <class Cfg, int H> using AtHeight = typename WithHeight<Cfg, H>::type;
template <class Cfg, class = void>
struct out_is_f32 : std::false_type {};
template <class Cfg>
struct out_is_f32<Cfg, std::void_t<decltype(Cfg::OUT_F32)>> : std::bool_constant<Cfg::OUT_F32> {};

// ---- pieces shared by the kernels ---------------------------------------------------------

// MFMA 16x16x32 operand fragment: lane l supplies 8 consecutive k (k-group l >> 4) of operand
// row l & 15. Per-lane LDS byte offsets inside a stage of the fragment of this wavefront's
// first A / B tile at each k-substep; tile i of the wave is 16 rows (TILE_STEP bytes) further on
// (the swizzle only depends on row & 15, so it is the same for every tile).
template <class Cfg>
struct FragPlan {
    uint32_t a_off[Cfg::KSUB], b_off[Cfg::KSUB];
    int frag_row, frag_kg;
    __device__ __forceinline__ void init(int lane, int wm, int wn) {
        frag_row = lane & 15;
        frag_kg = lane >> 4;
#pragma unroll
        for (int kk = 0; kk < Cfg::KSUB; ++kk) {
            const uint32_t chunk =
                static_cast<uint32_t>(((kk * 4 + frag_kg) ^ swz<Cfg::BK>(frag_row)) << 4);
            a_off[kk] = (wm * Cfg::WTM + frag_row) * Cfg::ROW_BYTES + chunk;
            b_off[kk] = Cfg::A_BYTES + (wn * Cfg::WTN + frag_row) * Cfg::ROW_BYTES + chunk;
        }
    }
};

__device__ __forceinline__ bf16x8 lds16(const unsigned char* p) {
    return *reinterpret_cast<const bf16x8*>(p);
}

// acc (16x16, transposed: rows = weight rows, columns = activation rows) += W_frag * X_frag
__device__ __forceinline__ f32x4 mma16(const bf16x8& w, const bf16x8& x, const f32x4& acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x, acc, 0, 0, 0);
}

// The same instruction with the accumulator pinned to the accumulation registers (AGPRs). The
// pipelined kernel uses it so that its 128 or 256 accumulator registers never compete with the
// fragment registers (left to itself the register allocator shuffles accumulators between the
// two register classes inside the k-loop). The compiler does not know that this is an MFMA:
// it still waits for the LDS reads that feed it, but the kernel must pad by hand before
// anything other than an MFMA touches the accumulators (see mfma_drain()).
__device__ __forceinline__ void mma16_agpr(const bf16x8& w, const bf16x8& x, f32x4& acc) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(w), "v"(x));
}
// Wait states between the last MFMA and the first ordinary read of its result. `last` are the
// accumulators of the last MFMAs: the empty statements keep the compiler from reading them ahead of
// the wait (older ones have left the matrix pipe by then, whenever they are read).
template <int N>
__device__ __forceinline__ void mfma_drain(f32x4 (&last)[N]) {
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int j = 0; j < N; ++j) asm volatile("" : "+a"(last[j]));
}

// Epilogue. Result layout of the transposed 16x16 tile: lane holds activation row (lane & 15)
// and the four output columns 4 * (lane >> 4) + r in registers r = 0..3. With DUAL, B-tile rows
// come in blocks of DB W1 rows followed by the DB W3 rows of the same output columns, so accumulator
// tiles j and j + P (P = DB / 16, j & P == 0) are gate and up of the same columns.
template <class Cfg>
__device__ __forceinline__ void store_tile(const f32x4 (&acc)[Cfg::TM][Cfg::TN], const TileCoord& tc,
                                           const FragPlan<Cfg>& fp, int wm, int wn,
                                           uint16_t* __restrict__ C, int ldc) {
    constexpr bool DUAL = Cfg::DUAL;
    constexpr int DB = Cfg::DB, P = DB / 16;
#pragma unroll
    for (int i = 0; i < Cfg::TM; ++i) {
        const int row = wm * Cfg::WTM + i * 16 + fp.frag_row;
        if (row >= tc.rows) continue;
        uint16_t* crow = C + static_cast<size_t>(tc.row0 + row) * ldc + tc.nt * Cfg::BN_OUT + 4 * fp.frag_kg;
#pragma unroll
        for (int j = 0; j < Cfg::TN; ++j) {
            if (DUAL && (j & P)) continue;
            const int r0 = wn * Cfg::WTN + j * 16;                 // first B-tile row of tile j
            const int col = DUAL ? r0 / (2 * DB) * DB + r0 % DB : r0;
            if constexpr (out_is_f32<Cfg>::value) {
                float* frow = reinterpret_cast<float*>(C) + static_cast<size_t>(tc.row0 + row) * ldc +
                              tc.nt * Cfg::BN_OUT + 4 * fp.frag_kg;
                *reinterpret_cast<f32x4*>(frow + col) = acc[i][j];
                continue;
            }
            bf16x4 o;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = DUAL ? silu(acc[i][j][r]) * acc[i][DUAL ? j + P : j][r] : acc[i][j][r];
                o[r] = static_cast<__bf16>(v);                     // round to nearest even
            }
            *reinterpret_cast<bf16x4*>(crow + col) = o;
        }
    }
}

// Division of a flat id (below 2^31) by the number of experts per token as a multiplication:
// id / div == (id * mul) >> (32 + shift) with mul = floor(2^(32 + shift) / div) + 1 and
// 2^shift < div <= 2^(shift + 1): the error term id * (mul * div - 2^(32 + shift)) stays below
// 2^31 * 2^(shift + 1). mul == 0 stands for div == 1.
struct RowDiv {
    uint32_t mul;
    int shift;
    explicit RowDiv(int div) : mul(0), shift(0) {
        if (div <= 1) return;
        while ((2 << shift) < div) ++shift;
        mul = static_cast<uint32_t>((1ull << (32 + shift)) / static_cast<unsigned>(div) + 1);
    }
};

// Rows of A, relative to a_origin(), that feed rows r0 + i * RPI + lrow of the tile, lrow < RPI by lane (rows past
// the end of the group read its last row). Without an index the A matrix is already grouped: the origin is
// the tile's first row and the answer is the row itself. With one, A holds one row per token, the
// origin is A itself and grouped row p reads the token row_index[p] / div (the permutation's flat
// id t*k+s divided by k) — the row gather fused into the operand load. Offsets from the origin
// are 32-bit: the caller guarantees that the token matrix is smaller than 4 GiB when it passes
// an index. The index comes through the scalar cache, RPI entries together, and a lane picks its own: a
// vector load would be counted with the direct-to-LDS loads, and to wait for it would be to wait for all of those
// that are on their way. A group shorter than RPI rows reads past its end, up to RPI - 1 entries past the end of
// the index, which the caller's buffer has to hold.
template <int COUNT, int RPI>
__device__ __forceinline__ void source_rows(int (&src)[COUNT], const TileCoord& tc, int r0, int lrow,
                                            const int32_t* __restrict__ row_index, RowDiv div) {
#pragma unroll
    for (int i = 0; i < COUNT; ++i) src[i] = min(r0 + i * RPI + lrow, tc.rows - 1);
    if (row_index != nullptr) {
        int ids[COUNT][RPI];
        int at[COUNT];
#pragma unroll
        for (int i = 0; i < COUNT; ++i) {
            at[i] = max(0, min(r0 + i * RPI, tc.rows - RPI));
#pragma unroll
            for (int q = 0; q < RPI; ++q) ids[i][q] = row_index[tc.row0 + at[i] + q];
        }
#pragma unroll
        for (int i = 0; i < COUNT; ++i) {
            int id = ids[i][0];
#pragma unroll
            for (int q = 1; q < RPI; ++q) id = src[i] - at[i] >= q ? ids[i][q] : id;
            src[i] = div.mul == 0 ? id : static_cast<int>(__umulhi(static_cast<uint32_t>(id), div.mul) >> div.shift);
        }
    }
}
__device__ __forceinline__ const uint16_t* a_origin(const uint16_t* A, const TileCoord& tc,
                                                    const int32_t* row_index, int K) {
    return row_index ? A : A + static_cast<size_t>(tc.row0) * K;
}

// Direct-to-LDS load plan of one wavefront. Wavefront load q of a stage covers tile rows
// [q*RPI, (q+1)*RPI); lane l lands at row q*RPI + l/CPR, chunk position l%CPR, so it must
// fetch logical chunk (l%CPR) ^ swz(row). A rows past the group's end are clamped to its last
// row (always in bounds; masked at the store).
template <class Cfg>
struct LoadPlan {
    static constexpr int LA = Cfg::NIA / Cfg::NW, LB = Cfg::NIB / Cfg::NW;
    // The B-tile rows of a wavefront come in blocks of Cfg::DB from W1 and W3 in turn with DUAL.
    static constexpr int BLOCKS = Cfg::DUAL && LB * Cfg::RPI > Cfg::DB ? LB * Cfg::RPI / Cfg::DB : 1;
    const uint16_t* a_base;
    const uint16_t* b_base[BLOCKS];     // the n-tile's first row in the block's matrix
    uint32_t a_voff[LA], b_voff[LB], a_lds, b_lds;      // a_lds, b_lds: this wavefront's first load inside a stage
    bool a_on[LA];      // false: every row of this A load lies past the end of the group
    __device__ __forceinline__ void init_a(const TileCoord& tc, int wave, int lane, const uint16_t* A,
                                           const int32_t* row_index, RowDiv index_div, int K) {
        const int lrow = lane / Cfg::CPR, lpos = lane % Cfg::CPR;
        a_base = a_origin(A, tc, row_index, K);
        int src[LA];
        source_rows<LA, Cfg::RPI>(src, tc, wave * LA * Cfg::RPI, lrow, row_index, index_div);
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int q = wave * LA + i;
            const int r = q * Cfg::RPI + lrow;
            a_voff[i] = (static_cast<uint32_t>(src[i]) * K + ((lpos ^ swz<Cfg::BK>(r)) * 8)) * 2u;
            a_on[i] = q * Cfg::RPI < tc.rows;
        }
    }
    // A rows one by one from row_of(row of the tile)
    template <class RowOf>
    __device__ __forceinline__ void init_a_from(const TileCoord& tc, int wave, int lane, const uint16_t* A, int K,
                                                RowOf&& row_of) {
        const int lrow = lane / Cfg::CPR, lpos = lane % Cfg::CPR;
        a_base = A;
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int r = (wave * LA + i) * Cfg::RPI + lrow;
            a_voff[i] = (static_cast<uint32_t>(row_of(min(r, tc.rows - 1))) * K + ((lpos ^ swz<Cfg::BK>(r)) * 8)) * 2u;
        }
    }
    // what is the same for every tile
    __device__ __forceinline__ void init_fixed(int wave, int lane, int K) {
        static_assert(!Cfg::DUAL || LB * Cfg::RPI % Cfg::DB == 0 || Cfg::DB % (LB * Cfg::RPI) == 0, "whole blocks");
        const int lrow = lane / Cfg::CPR, lpos = lane % Cfg::CPR;
        a_lds = wave * LA * 1024;
        b_lds = Cfg::A_BYTES + wave * LB * 1024;
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            const int q = wave * LB + i, r0 = q * Cfg::RPI;
            const int col0 = Cfg::DUAL ? r0 / (2 * Cfg::DB) * Cfg::DB + r0 % Cfg::DB : r0;
            b_voff[i] = (static_cast<uint32_t>(col0 + lrow) * K + ((lpos ^ swz<Cfg::BK>(r0 + lrow)) * 8)) * 2u;
        }
    }
    __device__ __forceinline__ void init_b(const TileCoord& tc, int wave, const uint16_t* B0, const uint16_t* B1,
                                           int N, int K) {
        const size_t first = (static_cast<size_t>(tc.expert) * N + static_cast<size_t>(tc.nt) * Cfg::BN_OUT) * K;
#pragma unroll
        for (int b = 0; b < BLOCKS; ++b)
            b_base[b] = (Cfg::DUAL && ((wave * LB * Cfg::RPI / Cfg::DB + b) & 1) ? B1 : B0) + first;
    }
    __device__ __forceinline__ void init(const TileCoord& tc, int wave, int lane, const uint16_t* A,
                                         const uint16_t* B0, const uint16_t* B1,
                                         const int32_t* row_index, RowDiv index_div, int N, int K) {
        init_b(tc, wave, B0, B1, N, K);
        init_a(tc, wave, lane, A, row_index, index_div, K);
    }
    __device__ __forceinline__ const uint16_t* b_src(int i) const { return b_base[i * BLOCKS / LB]; }
    // load number n (0 <= n < LA + LB) of k-step kt into the stage at LDS byte offset sbase
    __device__ __forceinline__ void issue_one(int n, uint32_t sbase, size_t koff) const {
        if (n < LA) dma16(a_base + koff, a_voff[n], sbase + a_lds + n * 1024);
        else dma16<Cfg::STREAM_B>(b_src(n - LA) + koff, b_voff[n - LA], sbase + b_lds + (n - LA) * 1024);
    }
    // single loads with explicit LDS region bases (operand rings of different depth)
    __device__ __forceinline__ void issue_a(int i, uint32_t region, size_t koff) const {
        dma16(a_base + koff, a_voff[i], region + a_lds + i * 1024);
    }
    __device__ __forceinline__ void issue_b(int i, uint32_t region, size_t koff) const {
        dma16(b_src(i) + koff, b_voff[i], region + (b_lds - Cfg::A_BYTES) + i * 1024);
    }
    __device__ __forceinline__ void issue_a_all(uint32_t sbase, size_t koff) const {
#pragma unroll
        for (int n = 0; n < LA; ++n) issue_one(n, sbase, koff);
    }
    __device__ __forceinline__ void issue_b_all(uint32_t sbase, size_t koff) const {
#pragma unroll
        for (int n = LA; n < LA + LB; ++n) issue_one(n, sbase, koff);
    }
    __device__ __forceinline__ void issue_all(uint32_t sbase, size_t koff) const {
#pragma unroll
        for (int n = 0; n < LA + LB; ++n) issue_one(n, sbase, koff);
    }
};

// ---- kernel 1: ring of stages, every wavefront loads and computes ---------------------------
// Workgroups that start together stay at the same k, where weight rows whose pitch is a multiple of 4 KB fall on
// few memory channels. In long reductions the first workgroup of every compute unit starts later by its place in its
// XCD: they then stream different k, and what a late start costs is less than what the channels gain; the
// order of the sums is the same. `spread` is the step in units of 768 cycles (spread_steps in expert_gemm.hip).
constexpr int kSpreadSlots = 32;     // compute units of an XCD
__device__ __forceinline__ void spread_start(int spread) {
    const int slot = blockIdx.x / kXcds;
    if (slot >= kSpreadSlots) return;
    for (int i = slot * spread; i > 0; --i) __builtin_amdgcn_s_sleep(12);
}

// One tile: `init_a` sets the A addresses of the load plan, after the first weights have gone out.
template <class Cfg, class InitA>
__device__ __forceinline__ void ring_of_stages(const TileCoord& tc, LoadPlan<Cfg>& lp, InitA&& init_a, unsigned char* smem,
                                               int wave, int lane, const uint16_t* __restrict__ B0,
                                               const uint16_t* __restrict__ B1, uint16_t* __restrict__ C, int N,
                                               int K) {
    constexpr int BK = Cfg::BK, TM = Cfg::TM, TN = Cfg::TN, LPW = Cfg::LPW, NSTAGE = Cfg::NSTAGE;
    static_assert(Cfg::KSUB == 2, "two k-substeps a stage");
    const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
    // ---- first loads: the first weights go out under the latency of the row index (layer call of 64 tokens through
    // 8 experts of 512 x 1024 20.5 us, with two stages of weights 21.0; one token through 8 of 128 of 2048 x 768 29.2, 29.4)
    const int KT = K / BK;
    lp.init_fixed(wave, lane, K);
    lp.init_b(tc, wave, B0, B1, N, K);
    lp.issue_b_all(0, 0);
    init_a();
    lp.issue_a_all(0, 0);
#pragma unroll
    for (int s = 1; s < NSTAGE - 1; ++s)
        if (s < KT) lp.issue_all(s * Cfg::STAGE_BYTES, static_cast<size_t>(s) * BK);

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    FragPlan<Cfg> fp;
    fp.init(lane, wm, wn);

    // ---- main loop: ring of NSTAGE stages, NSTAGE-1 k-steps of loads in flight.
    int stage = 0;
    for (int kt = 0; kt < KT; ++kt) {
        // The loads of k-step kt are the oldest in flight; up to NSTAGE-2 newer steps may stay
        // pending. Near the tail fewer are in flight, so wait for everything.
        if (kt + NSTAGE - 2 < KT) wait_vmcnt<(NSTAGE - 2) * LPW>(); else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();          // stage `stage` is complete for every wavefront
                                               // and stage (stage-1) is no longer being read
        const int nk = kt + NSTAGE - 1;
        const unsigned char* st = smem + stage * Cfg::STAGE_BYTES;
        const uint32_t into = (stage == 0 ? NSTAGE - 1 : stage - 1) * Cfg::STAGE_BYTES;
        const size_t koff = static_cast<size_t>(nk) * BK;
        // Fragments of the first k-substep are asked for ahead of the loads, which leave a wavefront some 100 cycles
        // apart, those of the second ahead of the first one's MFMAs (layer calls with the loads first -> so: one token
        // through 8 experts of 512 x 1024 20.0 -> 19.6 us, 5 through 6 of 64 of 2048 x 1408 93.9 -> 92.3, 37 through 8 of 128
        // of 2048 x 768 191.0 -> 190.4; large experts within 0.5 %).
        bf16x8 af[2][TM], bfr[2][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) af[0][i] = lds16(st + fp.a_off[0] + i * Cfg::TILE_STEP);
#pragma unroll
        for (int j = 0; j < TN; ++j) bfr[0][j] = lds16(st + fp.b_off[0] + j * Cfg::TILE_STEP);
        if (nk < KT) lp.issue_all(into, koff);
#pragma unroll
        for (int i = 0; i < TM; ++i) af[1][i] = lds16(st + fp.a_off[1] + i * Cfg::TILE_STEP);
#pragma unroll
        for (int j = 0; j < TN; ++j) bfr[1][j] = lds16(st + fp.b_off[1] + j * Cfg::TILE_STEP);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = mma16(bfr[0][j], af[0][i], acc[i][j]);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = mma16(bfr[1][j], af[1][i], acc[i][j]);
        stage = (stage + 1 == NSTAGE) ? 0 : stage + 1;
    }
    store_tile<Cfg>(acc, tc, fp, wm, wn, C, N);
}

template <class Cfg>
__global__ __launch_bounds__(Cfg::NTHREADS) void grouped_gemm_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B0,
    const uint16_t* __restrict__ B1, uint16_t* __restrict__ C,
    const int32_t* __restrict__ offsets, const int32_t* __restrict__ row_index, RowDiv index_div,
    int E, int N, int K, int spread) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const TileCoord tc = locate_tile<Cfg::BM>(offsets, E, N / Cfg::BN_OUT);
    if (tc.expert < 0) return;
    spread_start(spread);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    LoadPlan<Cfg> lp;
    ring_of_stages<Cfg>(tc, lp, [&] { lp.init_a(tc, wave, lane, A, row_index, index_div, K); }, smem, wave, lane, B0, B1,
                        C, N, K);
}

// ---- kernel 1, few tokens: tiles straight from the selected experts ---------------------------
// Gate/up of a call whose permutation no launch has made: every workgroup derives the groups from the R = T * k
// flat ids by itself (a histogram in LDS, its prefix sums, then the ids of its own tile by ballots), and the
// first workgroup of the grid, which has no tile, writes the tables for the kernels behind this one. EW > 0: the
// selection too, from the logits of at most NTHREADS / 16 tokens and at most 16 * EW experts. What that costs a
// workgroup is less than a launch with the latencies around it; layer calls with the separate launch -> without, see
// gateup_routes in expert_gemm.hip.
constexpr int kRoutedIds = 1024;         // ids at most: sixteen per lane
template <int WAVES> constexpr int kMaxKeepRouted = kRoutedIds / (WAVES * kWave);
struct Routing {
    const float* logits;                 // [T, E], with EW > 0
    int32_t* topk_idx;                   // [T, k]: read, written with EW > 0
    float* topk_w;                       // [T, k], written with EW > 0
    int32_t *counts, *offsets, *perm, *inv_perm;      // written
    int T, k;
};

template <class Cfg, int EW>
__global__ __launch_bounds__(Cfg::NTHREADS) void grouped_gemm_routed_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B0, const uint16_t* __restrict__ B1,
    uint16_t* __restrict__ C, Routing rt, RowDiv index_div, int E, int N, int K) {
    constexpr int BM = Cfg::BM, ROUNDS = kRoutedIds / kWave;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    // scratch in the stage that no load reaches before the first barrier of the k-loop
    static_assert((kMaxExperts + kRoutedIds + BM) * 4 <= Cfg::STAGE_BYTES, "fits a stage");
    static_assert(sizeof(SmallTables<Cfg::NW>) <= (Cfg::NSTAGE - 1) * Cfg::STAGE_BYTES, "fits in front of it");
    static_assert(Cfg::NW * kWave * kMaxKeepRouted<Cfg::NW> >= kRoutedIds, "ids of the tables' workgroup");
    int32_t* cnt = reinterpret_cast<int32_t*>(smem + (Cfg::NSTAGE - 1) * Cfg::STAGE_BYTES);
    int32_t *ids = cnt + kMaxExperts, *list = ids + kRoutedIds;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int R = rt.T * rt.k, NT = N / Cfg::BN_OUT;
    const bool tables = blockIdx.x == 0;             // tiles start at slot 1 of every XCD
    if (tid < E) cnt[tid] = 0;
    int my[ROUNDS];                      // every wavefront holds all ids, 64 a round
    if constexpr (EW > 0) {
        const int at = wave * rt.k;
        if (wave < rt.T) {
            if (tables)
                select_by_wavefront<EW>(rt.logits, wave, lane, E, rt.k, [&](int s, int e, float w) {
                    ids[at + s] = e;
                    rt.topk_idx[at + s] = e;
                    rt.topk_w[at + s] = w;
                });
            else                         // the gates drop out of this one
                select_by_wavefront<EW>(rt.logits, wave, lane, E, rt.k, [&](int s, int e, float) { ids[at + s] = e; });
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        my[r] = -1;
        if (r * kWave >= R) continue;    // the same for all lanes: rounds without ids cost a branch
        const int i = r * kWave + lane;
        if (i < R) my[r] = (EW > 0 ? ids : rt.topk_idx)[i];
    }
    if constexpr (EW == 0) __syncthreads();          // the counters are clear
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
        if (r * kWave < R && r % Cfg::NW == wave && my[r] >= 0) atomicAdd(&cnt[my[r]], 1);   // counts: any order
    __syncthreads();
    if (blockIdx.x < kXcds) {
        if (tables)
            permute_block<Cfg::NW, kMaxKeepRouted<Cfg::NW>, false>(
                *reinterpret_cast<SmallTables<Cfg::NW>*>(smem), EW > 0 ? ids : rt.topk_idx, 0, R, E, rt.counts,
                rt.offsets, rt.perm, rt.inv_perm);
        return;
    }
    TileTable<BM> table;
    table.init_from_counts(cnt, E, NT, blockIdx.x % kXcds, lane);
    const TileCoord tc = uniform_tile(table.find(NT, Cut::kNever, blockIdx.x / kXcds - 1, division_magic(lane)));
    if (tc.expert < 0) return;
    LoadPlan<Cfg> lp;
    ring_of_stages<Cfg>(tc, lp, [&] {
        // each wavefront lists the tile's ids for itself (all write the same values)
        const int first = tc.row0 - table.first_row(tc.expert);
        int found = 0;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (r * kWave >= R) continue;
            const uint64_t m = __ballot(my[r] == tc.expert);
            const int at = found + __popcll(m & ((1ull << lane) - 1ull)) - first;
            if (my[r] == tc.expert && at >= 0 && at < tc.rows) list[at] = r * kWave + lane;
            found += __popcll(m);
        }
        __builtin_amdgcn_wave_barrier();
        lp.init_a_from(tc, wave, lane, A, K, [&](int row) {
            const int id = list[row];
            return index_div.mul == 0 ? id : static_cast<int>(__umulhi(static_cast<uint32_t>(id), index_div.mul) >> index_div.shift);
        });
    }, smem, wave, lane, B0, B1, C, N, K);
}

// ---- kernel 2: operand rings of different depth, hand-placed software pipeline ---------------
// A k-step (64 k) is two half-steps of one MFMA k-substep each. While the MFMAs of a half-step
// issue, the fragments of the next half-step are read from LDS into the registers that the
// MFMAs just consumed. The barrier of k-step kt sits between its two half-steps: when a
// wavefront arrives it has read all of k-step kt (the fragments of the second half are in
// registers) and its loads of k-step kt+1 have landed, so after the barrier the stages of
// k-step kt may be refilled and k-step kt+1 may be read, and the MFMAs of the second half-step
// are ready to issue at once. Scheduling fences keep each group of MFMAs, LDS reads and
// direct-to-LDS loads where it is written.
//
// LDS holds NA stages of the A tile and NB stages of the B tile (BM or BN rows of 64 k each;
// for 256 x 256 tiles NA + NB = 5 stages of 32 KB fill the 160 KB). After the barrier of k-step
// kt the A stage is refilled with k-step kt+NA and the B stage with k-step kt+NB, so the
// operand with the deeper ring has NB-1 (or NA-1) k-steps to arrive: with two stages each the
// kernel waits about a third of every k-step for the slowest cache line of the next one. The
// operand with the shallower ring is issued first within a k-step: loads complete in order, so
// the wait for it then leaves only the newest loads of the deeper operand pending.
#define MOE_FENCE() __builtin_amdgcn_sched_barrier(0)

template <class Cfg, int NA, int NB>
struct RingCfg {
    static constexpr int A_RING = NA * Cfg::A_BYTES, SMEM = NA * Cfg::A_BYTES + NB * Cfg::B_BYTES;
    static constexpr bool A_FIRST = NA <= NB;                 // issue order inside a k-step
    static constexpr int LA = Cfg::NIA / Cfg::NW, LB = Cfg::NIB / Cfg::NW;
    // loads that may stay pending when k-step kt+1 must have landed
    static constexpr int PENDING = (NA == NB) ? 0 : (NA < NB ? (NB - NA) * LB : (NA - NB) * LA);
    static_assert(SMEM <= 160 * 1024 && NA >= 2 && NB >= 2, "LDS budget");
    static_assert(NA - NB <= 1 && NB - NA <= 1, "pending count assumes rings that differ by one");
    static_assert(NA * LA + NB * LB < 64, "loads in flight must fit the 6-bit load counter");
};

// One k-step of one wavefront.
//   COMPUTE  false for a wavefront whose rows all lie past the end of a partial tile: it only
//            issues its loads and meets the others at the barrier.
//   PARTIAL  the tile has fewer than BM rows: A loads whose rows all lie past the end are
//            skipped (what the MFMAs read there only reaches output rows that are never stored).
//   RUNTIME  tail of the k-loop: dma_a / dma_b say whether k-steps kt+NA / kt+NB exist,
//            read_next whether kt+1 does, and the wait for loads is total.
//
// Fragment registers: A tile i of the next half-step replaces fa[i] right after the MFMAs that
// consumed it, except the last tile, which alternates between fa[TM-1] (first half-steps) and
// fx (second half-steps) so that it can be read at the start of the half-step: no LDS read is
// issued in the last chunk and the wait for all reads before the barrier costs nothing. B
// fragments alternate between fb0 and fb1 and are read in the first chunks.
template <class Cfg, int NA, int NB, bool COMPUTE, bool PARTIAL, bool RUNTIME>
__device__ __forceinline__ void ring_kstep(f32x4 (&acc)[Cfg::TM][Cfg::TN], bf16x8 (&fa)[Cfg::TM],
                                           bf16x8& fx, bf16x8 (&fb0)[Cfg::TN],
                                           bf16x8 (&fb1)[Cfg::TN], const unsigned char* pa_h1,
                                           const unsigned char* pb_h1, const unsigned char* pa_n0,
                                           const unsigned char* pb_n0, const LoadPlan<Cfg>& lp,
                                           uint32_t a_region, uint32_t b_region, size_t a_koff,
                                           size_t b_koff, bool dma_a, bool dma_b, bool read_next) {
    using R = RingCfg<Cfg, NA, NB>;
    constexpr int TM = Cfg::TM, TN = Cfg::TN, LA = R::LA, LB = R::LB, LPW = LA + LB;
    constexpr int BPC = (TN + TM / 2 - 1) / (TM / 2);      // B reads per chunk (first chunks)
    static_assert(TN <= TM, "interleave plan");
    static_assert(!PARTIAL || R::A_FIRST, "skipping A loads needs the B loads to be the newest");
    // ---- first half: MFMAs on (fa, fb0); read the second-half fragments of this k-step
    if (COMPUTE) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int j = 0; j < TN; ++j) mma16_agpr(fb0[j], fa[i], acc[i][j]);
            MOE_FENCE();    // the reads below reuse the registers of fa[i]: after its MFMAs
            if (i == 0) fx = lds16(pa_h1 + (TM - 1) * Cfg::TILE_STEP);
            if (i < TM - 1) fa[i] = lds16(pa_h1 + i * Cfg::TILE_STEP);
#pragma unroll
            for (int b = i * BPC; b < (i + 1) * BPC && b < TN; ++b)
                fb1[b] = lds16(pb_h1 + b * Cfg::TILE_STEP);
            MOE_FENCE();
        }
    }
    if (RUNTIME) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(R::PENDING) : "memory");
    __builtin_amdgcn_s_barrier();      // k-step kt+1 complete in LDS; this k-step's stages are free
    MOE_FENCE();
    // ---- second half: MFMAs on (fa[0..TM-2], fx, fb1); read the first-half fragments of k-step
    //      kt+1; refill the freed stages
    auto issue = [&](int n) {          // n-th load of this k-step in issue order
        const bool is_a = R::A_FIRST ? (n < LA) : (n >= LB);
        const int idx = R::A_FIRST ? (is_a ? n : n - LA) : (is_a ? n - LB : n);
        if (is_a) {
            if ((!RUNTIME || dma_a) && (!PARTIAL || lp.a_on[idx])) lp.issue_a(idx, a_region, a_koff);
        } else {
            if (!RUNTIME || dma_b) lp.issue_b(idx, b_region, b_koff);
        }
    };
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if (COMPUTE) {
#pragma unroll
            for (int j = 0; j < TN; ++j) mma16_agpr(fb1[j], i == TM - 1 ? fx : fa[i], acc[i][j]);
            MOE_FENCE();
            if (!RUNTIME || read_next) {
                if (i == 0) fa[TM - 1] = lds16(pa_n0 + (TM - 1) * Cfg::TILE_STEP);
                if (i < TM - 1) fa[i] = lds16(pa_n0 + i * Cfg::TILE_STEP);
#pragma unroll
                for (int b = i * BPC; b < (i + 1) * BPC && b < TN; ++b)
                    fb0[b] = lds16(pb_n0 + b * Cfg::TILE_STEP);
            }
        }
        // the LPW loads of the k-step are spread evenly over the TM chunks
#pragma unroll
        for (int n = (i * LPW + TM - 1) / TM; n < ((i + 1) * LPW + TM - 1) / TM; ++n) issue(n);
        MOE_FENCE();
    }
}

// One tile of the pipelined kernel (all wavefronts of the workgroup call it together).
template <class Cfg, int NA, int NB>
__device__ __forceinline__ void ring_tile(const TileCoord& tc, unsigned char* smem,
                                          const uint16_t* __restrict__ A,
                                          const uint16_t* __restrict__ B0,
                                          const uint16_t* __restrict__ B1, uint16_t* __restrict__ C,
                                          const int32_t* __restrict__ row_index, RowDiv index_div,
                                          int N, int K) {
    using R = RingCfg<Cfg, NA, NB>;
    constexpr int BM = Cfg::BM, BK = Cfg::BK, WN = Cfg::WN, TM = Cfg::TM, TN = Cfg::TN;
    constexpr int LA = R::LA, LB = R::LB, AB = Cfg::A_BYTES, BB = Cfg::B_BYTES;
    static_assert(BK == 64, "64-k stages");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    LoadPlan<Cfg> lp;
    lp.init_fixed(wave, lane, K);
    lp.init(tc, wave, lane, A, B0, B1, row_index, index_div, N, K);
    FragPlan<Cfg> fp;
    fp.init(lane, wm, wn);
    // fragment addresses of the two k-halves inside stage 0 of each ring
    const unsigned char* pa[2] = {smem + fp.a_off[0], smem + fp.a_off[1]};
    const unsigned char* pb[2] = {smem + R::A_RING + (fp.b_off[0] - AB), smem + R::A_RING + (fp.b_off[1] - AB)};

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");   // accumulator writes settle before MFMAs

    const int KT = K / BK;                           // >= max(NA, NB) (checked by the launcher)
    constexpr int NMAX = NA < NB ? NB : NA;

    auto run = [&](auto compute_tag, auto partial_tag) {
        constexpr bool COMPUTE = decltype(compute_tag)::value, PARTIAL = decltype(partial_tag)::value;
        // prologue: fill both rings in the order the k-loop would have issued them
#pragma unroll
        for (int s = 0; s < NMAX; ++s) {
            const size_t koff = static_cast<size_t>(s) * BK;
            if (R::A_FIRST) {
                if (s < NA) for (int i = 0; i < LA; ++i) if (!PARTIAL || lp.a_on[i]) lp.issue_a(i, s * AB, koff);
                if (s < NB) for (int i = 0; i < LB; ++i) lp.issue_b(i, R::A_RING + s * BB, koff);
            } else {
                if (s < NB) for (int i = 0; i < LB; ++i) lp.issue_b(i, R::A_RING + s * BB, koff);
                if (s < NA) for (int i = 0; i < LA; ++i) lp.issue_a(i, s * AB, koff);
            }
        }
        constexpr int TOTAL = NA * LA + NB * LB;
        if (PARTIAL) wait_vmcnt<0>();                // fewer loads than TOTAL were issued
        else wait_vmcnt<TOTAL - (LA + LB)>();        // k-step 0 landed
        __builtin_amdgcn_s_barrier();
        bf16x8 fa[TM], fx, fb0[TN], fb1[TN];
        if (COMPUTE) {
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[i] = lds16(pa[0] + i * Cfg::TILE_STEP);
#pragma unroll
            for (int j = 0; j < TN; ++j) fb0[j] = lds16(pb[0] + j * Cfg::TILE_STEP);
            fx = fa[TM - 1];
        }
        MOE_FENCE();

        int ra = 0, rb = 0;                          // ring positions of k-step kt
        auto step = [&](auto runtime_tag, int kt) {
            constexpr bool RT = decltype(runtime_tag)::value;
            const int ra1 = (ra + 1 == NA) ? 0 : ra + 1, rb1 = (rb + 1 == NB) ? 0 : rb + 1;
            ring_kstep<Cfg, NA, NB, COMPUTE, PARTIAL, RT>(
                acc, fa, fx, fb0, fb1, pa[1] + ra * AB, pb[1] + rb * BB, pa[0] + ra1 * AB,
                pb[0] + rb1 * BB, lp, ra * AB, R::A_RING + rb * BB,
                static_cast<size_t>(kt + NA) * BK, static_cast<size_t>(kt + NB) * BK, kt + NA < KT,
                kt + NB < KT, kt + 1 < KT);
            ra = ra1; rb = rb1;
        };
        int kt = 0;
        for (; kt + NMAX < KT; ++kt) step(std::false_type{}, kt);
        for (; kt < KT; ++kt) step(std::true_type{}, kt);
    };
    using T = std::true_type;
    using F = std::false_type;
    if (tc.rows == BM) {
        run(T{}, F{});
    } else if (wm * Cfg::WTM < tc.rows) {
        run(T{}, T{});
    } else {
        run(F{}, T{});                               // no row of this wavefront is in the tile
        return;
    }
    mfma_drain(acc[TM - 1]);
    store_tile<Cfg>(acc, tc, fp, wm, wn, C, N);
}

// Epilogue of the one-wavefront-per-SIMD tile: the outputs go through LDS so that global memory
// sees whole cache lines. In the accumulator layout a lane holds four consecutive columns of one
// row per fragment, so a direct store writes sixteen separate 32-byte pieces; 256 compute units
// finishing their tiles together then queue at the L2 for thousands of cycles. Here a wavefront
// writes the sixteen rows of fragment row i (of half of it with fp32 outputs) into a 4 KB region of
// its own (`stage`) and reads them back 16 bytes per lane, whole rows at a time, so that each store
// instruction covers full 128-byte lines; the region is reused for the next fragment row. LDS serves
// a wavefront's requests in order, so neither the read after the write nor the next write after the
// read needs a wait, and the next row is converted and written while the reads of this one are on
// their way. The 16-byte chunks of a row are XOR-swizzled by the row so that both the writes (16 rows
// at one column) and the reads (whole rows) spread over all banks. `before_stores` runs once, ahead of
// the first store.
//
// The accumulators are read where they are converted: left to the compiler, all of a tile's were copied to
// ordinary registers ahead of the first conversion, which took 222 of those and spilled what lives from tile to tile.
__device__ __forceinline__ float read_acc(const f32x4& acc, int r) {
    float v;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(acc[r]));
    return v;
}
constexpr int kEpilogueBytes = 4096;                 // LDS that a wavefront stages its outputs through
// Bytes from a wavefront's first output row to behind its last one inside the tile. The tile has rows_from_here rows
// from the first one on, which may be more than the wavefront's own: 256 rows of 2^22 floats would be 2^32 bytes, while
// 128 rows of any width that offsets_fit_1w() lets in are less.
__host__ __device__ constexpr uint32_t store_bytes(int rows_from_here, int wave_rows, uint32_t row_bytes) {
    const int rows = rows_from_here < wave_rows ? rows_from_here : wave_rows;
    return (rows < 0 ? 0 : rows) * row_bytes;
}
template <class Cfg, class Before>
__device__ __forceinline__ void store_tile_via_lds(const f32x4 (&acc)[Cfg::TM][8], const TileCoord& tc,
                                                   const FragPlan<Cfg>& fp, int wave, int lane,
                                                   unsigned char* stage, uint16_t* __restrict__ C,
                                                   int ldc, Before&& before_stores) {
    constexpr bool DUAL = Cfg::DUAL, F32 = out_is_f32<Cfg>::value;
    constexpr int WN = Cfg::WN;
    constexpr int PASSES = F32 ? 2 : 1;              // pieces that a fragment row is staged in
    constexpr int COLS = DUAL ? 64 : 128;            // output columns of this wavefront
    constexpr int ESZ = F32 ? 4 : 2;                 // bytes per output element
    constexpr int ROWB = COLS * ESZ / PASSES;        // bytes of one output row of a piece
    constexpr int CP = ROWB / 16;                    // 16-byte chunks per row
    constexpr int RSH = CP == 8 ? 1 : 0;             // log2 of the rows that share 256 bytes of LDS
    constexpr int SWM = CP - 1;                      // the swizzle permutes chunks inside 256 bytes
    constexpr int NJ = (DUAL ? 4 : 8) / PASSES;      // output fragments per piece
    constexpr int RPI = 64 / CP;                     // rows per store instruction
    constexpr int PIECES = Cfg::TM * PASSES;
    static_assert(Cfg::TN == 8 && 16 * ROWB <= kEpilogueBytes && CP <= 16, "fits the region");
    const int wm = wave / WN, wn = wave % WN;
    const uint32_t wswz = (fp.frag_row >> RSH) & SWM;
    unsigned char* wbase = stage + fp.frag_row * ROWB;
    const int rrow = lane / CP, rchunk = lane % CP;
    // Stores through a buffer resource that ends behind the wavefront's last row: those of rows past the end of
    // the group are dropped by its bounds check, with no comparison, branch or 64-bit address per store (of the
    // 700 cycles that a fragment row of the down projection took, those were half).
    const uint32_t row_bytes = static_cast<uint32_t>(ldc) * ESZ;
    // to a scalar register: left alone, the comparisons become one vector instruction, and a resource that is not
    // known to be uniform puts a loop around every store (8192 tokens through 128 experts of 2048 x 768 680 -> 689 us a layer)
    const uint32_t bytes = __builtin_amdgcn_readfirstlane(store_bytes(tc.rows - wm * Cfg::WTM, Cfg::WTM, row_bytes));
    const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<unsigned char*>(C) + static_cast<size_t>(tc.row0 + wm * Cfg::WTM) * row_bytes, 0,
        static_cast<int>(bytes), 0x00027000);
    const uint32_t ccol = static_cast<uint32_t>(tc.nt * Cfg::BN_OUT + wn * COLS) * ESZ + rchunk * 16;
    uint32_t coff[16 / RPI];
#pragma unroll
    for (int q = 0; q < 16 / RPI; ++q) coff[q] = (q * RPI + rrow) * row_bytes + ccol;
    auto write_piece = [&](int u) {
        const int i = u / PASSES, j0 = (u % PASSES) * NJ;
        auto frag = [&](int jj) { return j0 + (DUAL ? (jj & 1) + (jj >> 1) * 4 : jj); };   // gate; up = + 2
        if constexpr (F32) {
#pragma unroll
            for (int jj = 0; jj < NJ; ++jj) {
                const uint32_t chunk = (static_cast<uint32_t>(jj * 4 + fp.frag_kg) ^ wswz) * 16;
                *reinterpret_cast<f32x4*>(wbase + chunk) = acc[i][frag(jj)];
            }
        } else {
            f32x4 v[NJ], up[NJ];                     // all reads first: the conversions then interleave
#pragma unroll
            for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[jj][r] = read_acc(acc[i][frag(jj)], r);
                    if constexpr (DUAL) up[jj][r] = read_acc(acc[i][frag(jj) + 2], r);
                }
#pragma unroll
            for (int jj = 0; jj < NJ; ++jj) {
                bf16x4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r)          // round to nearest even
                    o[r] = static_cast<__bf16>(DUAL ? silu(v[jj][r]) * up[jj][r] : v[jj][r]);
                const uint32_t chunk = (static_cast<uint32_t>(jj * 2 + (fp.frag_kg >> 1)) ^ wswz) * 16;
                *reinterpret_cast<bf16x4*>(wbase + chunk + (fp.frag_kg & 1) * 8) = o;
            }
        }
        MOE_FENCE();                                 // one piece's registers at a time
    };
    write_piece(0);
#pragma unroll
    for (int u = 0; u < PIECES; ++u) {
        u32x4 v[16 / RPI];
#pragma unroll
        for (int q = 0; q < 16 / RPI; ++q) {
            const int rl = q * RPI + rrow;                          // row inside the fragment row
            const uint32_t chunk = (static_cast<uint32_t>(rchunk) ^ ((rl >> RSH) & SWM)) * 16;
            v[q] = *reinterpret_cast<const u32x4*>(stage + rl * ROWB + chunk);
        }
        MOE_FENCE();
        if (u + 1 < PIECES) write_piece(u + 1);
        if (u == 0) before_stores();
#pragma unroll
        for (int q = 0; q < 16 / RPI; ++q) {
            __builtin_amdgcn_raw_buffer_store_b128(v[q], out, coff[q] + (u % PASSES) * ROWB, 0, 0);
            if (u % PASSES == PASSES - 1) coff[q] += 16 * row_bytes;
        }
        MOE_FENCE();
    }
}

template <class T> struct type_tag { using type = T; };

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>) in order
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

// ---- the large tiles with ONE wavefront per SIMD (4 wavefronts, 128 x 128 outputs each) -------
// Four wavefronts read 128 KB of fragments from LDS per k-step where eight read 192 KB, and hold
// all 256 accumulator registers of a lane's SIMD, so every fragment set can be double-buffered
// in the other 256 registers. With a single wavefront per SIMD nothing covers for it: a wavefront
// issues one instruction every four cycles, an MFMA occupies the matrix pipe for sixteen, so at
// most three other instructions fit between two MFMAs before the pipe runs dry. The k-step below
// therefore places every LDS read, every direct-to-LDS load and every scalar update behind an
// MFMA of its own: per half-step of 64 MFMAs, 16 fragment reads (after every fourth MFMA), 8
// loads (in every group of eight MFMAs: M0 is written before one MFMA and the load issued after
// it, the MFMA serving as the wait state that a write to M0 needs) and the pointer updates.
// The A loads of k-step kt+2 go out in the second half of k-step kt, the B loads of k-step
// kt+3 in the first half of k-step kt+1, so the texture-address unit sees one load per SIMD
// every 128 cycles throughout instead of all sixteen within one half.
//
// The workgroup is PERSISTENT: it runs one tile after the other, and the loads go on in
// between. (Gate/up through a row index waits for all that are on their way once per tile, where the load pointers
// move on: the next tile's index entries come by vector loads, which are counted with the others.) In the last two k-steps of a tile the load pointers already stand on the next tile, so
// those k-steps fill the rings with its first two k-steps (nothing else is left to load there), and
// they arrive under the conversion and stores of the finished tile. A workgroup per tile paid for its
// lookup (2.6 k cycles), its first loads (4.6 k, bound by their issue: 32 per wavefront about 100
// cycles apart), the launch gap and the last two k-steps' loads of nothing: a tile of 256 rows takes 35.6 k
// cycles at K = 768 (45 before) and 79.5 k at 2048 (89). About half of that arrives as time, the rest as a
// lower clock under the board's power limit: 8192 tokens through 128 experts of 2048 x 768 gate/up 354 -> 337
// and down 241 -> 218 us, 5003 through 64 of 2048 x 1408 294 -> 277 and 197 -> 189 (fp32 outputs), 8192 479 -> 432 and
// 262 -> 237, lower tiles (tile_in_expert) included.
// Long reductions keep a workgroup per tile (PERSISTENT false): the dispatcher starts workgroups in order, which
// brings those that share rows and weights in L2 back into step at every tile; persistent ones drift apart by
// what lower tiles save, and a k-step out of step is fetched again (8192 tokens at 6144 x 16384 7276 -> 7464 us
// a layer, at a clock 2 % lower for the same power).
//
// The LDS layout is that of the full tile whatever the height of a tile: A stages of Full::A_BYTES.
// Load i of wavefront w fetches tile rows 8 * (4 i + w) to + 7 of A, so that the first TM loads of
// all wavefronts are the rows of a tile of TM * 32 rows for every height, and a lower tile can fetch
// the first rows of a higher one (the others follow before its first store, see ring_tile_1w).
template <class Full>
struct Ring1W {
    static constexpr int NA = 2, NB = 3;
    static constexpr int AB = Full::A_BYTES, BB = Full::B_BYTES, A_RING = NA * AB, SMEM = A_RING + NB * BB;
    static constexpr int LA = Full::NIA / Full::NW, LB = Full::NIB / Full::NW;     // loads per wavefront and k-step
    static_assert(Full::NW == 4 && Full::TN == 8 && Full::BK == 64 && Full::RPI == 8 && LA == 8 && LB == 8 &&
                  SMEM <= 160 * 1024, "256 x 256 x 64, rings of 2 + 3 stages");
};

// Whether the byte offsets of a tile fit 32 bits, for matrices of N weight rows of K per expert: those of weight rows
// from the expert's matrix, and with K >= 256 those of a wavefront's 128 output rows of N floats.
__host__ __device__ constexpr bool offsets_fit_1w(int N, int K) {
    return static_cast<unsigned long long>(N) * static_cast<unsigned long long>(K) * 2ull < (1ull << 32);
}

// Loads of one tile: pointers that advance by a k-step at a time, byte offsets per lane.
struct LoadPlan1W {
    const uint16_t* a_ptr;          // A origin + current k offset of the A loads
    const uint16_t* b_ptr[2];       // first row of the n-tile in W (and W3 with DUAL) + current k offset
    uint32_t a_voff[8], b_voff[8];  // of A load i (this tile's rows); of B load i (the same for every tile)
};

// The A row that lane l looks up for its wavefront: row 8 * (4 i + w) + r of the tile with i = l / 8, r = l % 8
// (rows past the end of the group: its last one).
__device__ __forceinline__ int a_row_1w(const TileCoord& tc, int wave, int lane) {
    return min((lane >> 3) * 32 + wave * 8 + (lane & 7), max(tc.rows, 1) - 1);
}

// lp becomes the plan of tile tc at its first k. With an index (gate/up only), `id` is its entry for every lane's
// a_row_1w.
template <class Full>
__device__ __forceinline__ void start_loads_1w(LoadPlan1W& lp, const TileCoord& tc, int id, int wave, int lane,
                                               const uint16_t* A, const uint16_t* B0, const uint16_t* B1,
                                               const int32_t* row_index, RowDiv div, int N, int K) {
    uint32_t row_off = a_row_1w(tc, wave, lane);
    if (Full::DUAL && row_index != nullptr) {
        asm volatile("" : "+v"(id));   // keeps what waits for the index load where this stands
        row_off = id;
        if (div.mul != 0) row_off = __umulhi(row_off, div.mul) >> div.shift;
    }
    row_off *= static_cast<uint32_t>(K) * 2u;
    lp.a_ptr = a_origin(A, tc, row_index, K);
    const size_t first = (static_cast<size_t>(tc.expert) * N + static_cast<size_t>(tc.nt) * Full::BN_OUT) * K;
    lp.b_ptr[0] = B0 + first;
    lp.b_ptr[1] = Full::DUAL ? B1 + first : lp.b_ptr[0];
    const uint32_t chunk = static_cast<uint32_t>((lane & 7) ^ swz<64>(wave * 8 + (lane >> 3))) * 16u;
#pragma unroll
    for (int i = 0; i < 8; ++i)        // lane l needs row l / 8 of load i, which lane 8 i + l / 8 looked up
        lp.a_voff[i] = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute((i * 8 + (lane >> 3)) * 4,
                                                                         static_cast<int>(row_off))) + chunk;
}
template <class Full>
__device__ __forceinline__ void init_b_offsets(LoadPlan1W& lp, int wave, int lane, int K) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r0 = (wave * 8 + i) * 8;                      // first tile row of the load
        const int col0 = Full::DUAL ? (r0 >> 6) * 32 + (r0 & 31) : r0;
        lp.b_voff[i] = (static_cast<uint32_t>(col0 + (lane >> 3)) * K + (((lane & 7) ^ swz<64>(r0 + (lane >> 3))) * 8)) * 2u;
    }
}

// acc += W_frag * X_frag with the accumulator pinned to AGPRs; then one direct-to-LDS load whose
// LDS address (lds_base + LDS_OFF) was put into M0 before the MFMA.
template <int LDS_OFF>
__device__ __forceinline__ void mma16_then_dma(const bf16x8& w, const bf16x8& x, f32x4& acc,
                                               uint32_t lds_base, uint32_t voff, const void* sbase) {
    asm volatile("s_add_u32 m0, %3, %4\n\t"
                 "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\t"
                 "global_load_lds_dwordx4 %5, %6"
                 : "+a"(acc)
                 : "v"(w), "v"(x), "s"(lds_base), "n"(LDS_OFF), "v"(voff), "s"(sbase)
                 : "memory", "m0", "scc");
}

// One k-step of one wavefront. On entry f[0] holds the first-half fragments of this k-step.
// Every k-step runs exactly this code, without a branch: the accumulators are operands of inline
// assembly, which the compiler does not know to be MFMAs, so it must never find a reason (a join
// of two paths, a second loop) to move them between registers next to one. The first half issues
// the B loads of k-step kt+2, the second half the A loads of k-step kt+2 (in the last two k-steps of
// a tile: those of the next tile's first two, or these two's again where there is no next one),
// which keeps the number of loads in flight, and with it the load-counter value to wait for, the
// same in every k-step. Likewise the last k-step reads "next" fragments that are never used.
// LDS addresses of one k-step: fragment pointers of this k-step's second half (h1) and of the
// next k-step's first half (n0), the stages that this k-step's loads refill, and the ring
// positions (as byte offsets) they derive from.
struct RingState1W {
    const unsigned char *pa_h1, *pb_h1, *pa_n0, *pb_n0;
    uint32_t a_region, b_region;    // M0 bases of the A loads (stage kt) / B loads (stage kt-1)
    uint32_t sa, sb;                // byte offsets of k-step kt's stages inside the A / B ring
};

// MFMA number m of a half-step with its load, if it has one: load n = m / STRIDE goes out behind
// MFMA m when m % STRIDE == 3 and n < NLOADS; it lands LDS_STEP bytes behind load n - 1.
template <int M, int STRIDE, int NLOADS, int LDS_STEP>
__device__ __forceinline__ void mma16_slot(const bf16x8& w, const bf16x8& x, f32x4& acc,
                                           uint32_t lds_base, const uint32_t* voff,
                                           const void* sbase) {
    if constexpr (M % STRIDE == 3 && M / STRIDE < NLOADS)
        mma16_then_dma<(M / STRIDE) * LDS_STEP>(w, x, acc, lds_base, voff[M / STRIDE], sbase);
    else
        mma16_agpr(w, x, acc);
}

template <class Cfg, class R>
__device__ __forceinline__ void kstep_1w(f32x4 (&acc)[Cfg::TM][8], bf16x8 (&fa)[2][Cfg::TM],
                                         bf16x8 (&fb)[2][8], RingState1W& rs, LoadPlan1W& lp,
                                         int wave, const unsigned char* pa0, const unsigned char* pa1,
                                         const unsigned char* pb0, const unsigned char* pb1) {
    constexpr int TM = Cfg::TM, NM = TM * 8, NR = TM + 8;      // MFMAs and fragment reads per half
    constexpr int LA = TM, LB = R::LB;
    constexpr uint32_t AB = R::AB, BB = R::BB;
    static_assert(TM >= 4 && TM <= 8 && Cfg::TN == 8, "64 to 128 rows x 128 columns per wavefront");
    const uint32_t a_region = rs.a_region, b_region = rs.b_region;
    const unsigned char *pa_h1 = rs.pa_h1, *pb_h1 = rs.pb_h1, *pa_n0 = rs.pa_n0, *pb_n0 = rs.pb_n0;
    // fragment read r of a half goes out behind MFMA r * SPAN / NR: B fragments first (every MFMA
    // row needs all of them), then the A fragments in the order the MFMA rows use them. The reads
    // of the first half must all have returned at the barrier in the middle of the k-step, so
    // they are spread over its first part only (three quarters of it at full height); those of the second half have
    // until their MFMA in the next k-step and are spread over the whole half.
    constexpr int SPAN1 = (3 * NR <= NM - 4) ? 3 * NR : 2 * NR;
    auto read_behind = [&](auto mtag, auto spantag, bf16x8 (&dfb)[8], bf16x8 (&dfa)[TM],
                           const unsigned char* pbq, const unsigned char* paq) {
        constexpr int m = decltype(mtag)::value, SPAN = decltype(spantag)::value;
        constexpr int r = (m * NR + SPAN - 1) / SPAN;           // first read index with r * SPAN / NR >= m
        if constexpr (r < NR && (r * SPAN) / NR == m) {
            if constexpr (r < 8) dfb[r] = lds16(pbq + r * Cfg::TILE_STEP);
            else dfa[r - 8] = lds16(paq + (r - 8) * Cfg::TILE_STEP);
            MOE_FENCE();
        }
    };
    // ---- first half: MFMAs on f[0]; read f[1] (second half of this k-step); the eight B loads
    //      (with DUAL: four loads of W1 rows, then four of W3 rows)
    auto first = [&](auto mtag) {
        constexpr int m = decltype(mtag)::value, i = m >> 3, j = m & 7, n = m / (NM / 8);
        const void* src = lp.b_ptr[Cfg::DUAL ? (n >> 2) & 1 : 0];
        mma16_slot<m, NM / 8, 8, 1024>(fb[0][j], fa[0][i], acc[i][j], b_region, lp.b_voff, src);
        MOE_FENCE();
        read_behind(mtag, std::integral_constant<int, SPAN1>{}, fb[1], fa[1], pb_h1, pa_h1);
        // the B pointers move on behind the last B load (MFMA 7 * NM / 8 + 3)
        constexpr int after_loads = 7 * (NM / 8) + 4;
        if constexpr (m == (after_loads + 1 < NM ? after_loads + 1 : NM - 1)) {
            lp.b_ptr[0] += Cfg::BK;
            if (Cfg::DUAL) lp.b_ptr[1] += Cfg::BK;
            MOE_FENCE();
        }
    };
    // ---- second half: MFMAs on f[1]; read f[0] of k-step kt+1; the A loads; the next k-step's
    //      ring addresses, one small step behind an MFMA at a time
    uint32_t sb1 = 0, sb2 = 0, sa1 = 0;
    RingState1W nx;
    auto second = [&](auto mtag) {
        constexpr int m = decltype(mtag)::value, i = m >> 3, j = m & 7;
        mma16_slot<m, 8, LA, 4096>(fb[1][j], fa[1][i], acc[i][j], a_region, lp.a_voff, lp.a_ptr);
        MOE_FENCE();
        read_behind(mtag, std::integral_constant<int, NM>{}, fb[0], fa[0], pb_n0, pa_n0);
        if constexpr (m == 1) { sb1 = rs.sb + BB; MOE_FENCE(); }
        if constexpr (m == 2) { sb1 = (sb1 == R::NB * BB) ? 0u : sb1; MOE_FENCE(); }     // stage of k-step kt+1
        if constexpr (m == 5) { sb2 = sb1 + BB; MOE_FENCE(); }
        if constexpr (m == 6) { sb2 = (sb2 == R::NB * BB) ? 0u : sb2; MOE_FENCE(); }     // ... of kt+2
        if constexpr (m == 9) { sa1 = rs.sa ^ AB; MOE_FENCE(); }                         // two A stages
        if constexpr (m == 10) { nx.pa_h1 = pa1 + sa1; MOE_FENCE(); }
        if constexpr (m == 13) { nx.pb_h1 = pb1 + sb1; MOE_FENCE(); }
        if constexpr (m == 14) { nx.pa_n0 = pa0 + rs.sa; MOE_FENCE(); }
        if constexpr (m == 17) { nx.pb_n0 = pb0 + sb2; MOE_FENCE(); }
        if constexpr (m == 18) { nx.a_region = sa1 + wave * 1024; MOE_FENCE(); }
        if constexpr (m == 21) { nx.b_region = R::A_RING + rs.sb + wave * (LB * 1024); MOE_FENCE(); }
        if constexpr (m == NM - 3) { lp.a_ptr += Cfg::BK; MOE_FENCE(); }
    };
    static_for<NM>(first);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(LB) : "memory");
    __builtin_amdgcn_s_barrier();      // k-step kt+1 complete in LDS; this k-step's stages are free
    MOE_FENCE();
    static_for<NM>(second);
    nx.sa = sa1;
    nx.sb = sb1;
    rs = nx;
}

// One tile of a persistent workgroup. On entry its first two k-steps are in the rings (stages 0 and 1 of
// A, sb and the one behind it of B) and every wavefront knows it; on return those of the next tile are
// in the rings or on their way, sb is its B stage, and the stores of this one are on their way.
//   lp        loads of this tile at k-step 2, then of the next one
//   nxt       the next tile, id as for start_loads_1w; this one if it is the last
//   draw      called once in each wavefront two k-steps before the end; drawn() before the first store, when
//             all loads of the wavefront have landed
template <class Cfg, class Full, class Draw, class Drawn>
__device__ __forceinline__ void ring_tile_1w(const TileCoord& tc, const TileCoord& nxt, LoadPlan1W& lp,
                                             int id, bool last, uint32_t& sb, unsigned char* smem, int wave, int lane,
                                             const uint16_t* __restrict__ A, const uint16_t* __restrict__ B0,
                                             const uint16_t* __restrict__ B1, uint16_t* __restrict__ C,
                                             const int32_t* __restrict__ row_index, RowDiv index_div, int N, int K,
                                             Draw&& draw, Drawn&& drawn) {
    using R = Ring1W<Full>;
    constexpr int TM = Cfg::TM, TN = Cfg::TN;
    constexpr uint32_t AB = R::AB, BB = R::BB;
    static_assert(Cfg::NW == 4 && Cfg::BN == Full::BN && Cfg::BK == 64, "same n-tiling");
    FragPlan<Cfg> fp;
    fp.init(lane, wave / Cfg::WN, wave % Cfg::WN);
    const unsigned char* pa[2] = {smem + fp.a_off[0], smem + fp.a_off[1]};
    const unsigned char* pb[2] = {smem + R::A_RING + (fp.b_off[0] - Cfg::A_BYTES),
                                  smem + R::A_RING + (fp.b_off[1] - Cfg::A_BYTES)};
    bf16x8 fa[2][TM], fb[2][TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[0][j] = lds16(pb[0] + sb + j * Cfg::TILE_STEP);
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[0][i] = lds16(pa[0] + i * Cfg::TILE_STEP);
    MOE_FENCE();
    // The accumulators start as the result of an MFMA, 0 * 0 + 0, not as ordinary register
    // writes: the compiler may sink those to just in front of the k-loop, where it cannot
    // know that the inline assembly there is an MFMA that needs wait states after them.
    // MFMA after MFMA on the same registers needs nothing.
    f32x4 acc[TM][TN];
    {
        const bf16x4 zero = {0, 0, 0, 0};
        asm volatile("s_nop 4" :: "v"(zero));
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)             // four registers in half the time of the 16x16x32 instruction
                asm volatile("v_mfma_f32_4x4x4_16b_bf16 %0, %1, %1, 0" : "=a"(acc[i][j]) : "v"(zero));
    }
    const uint32_t sb_next = sb + BB == R::NB * BB ? 0u : sb + BB;
    RingState1W rs{pa[1], pb[1] + sb, pa[0] + AB, pb[0] + sb_next, wave * 1024u,
                   R::A_RING + (sb == 0 ? (R::NB - 1) * BB : sb - BB) + wave * (R::LB * 1024u), 0u, sb};
    // two k-steps per trip (K is a multiple of 128 for every supported shape): the loop's own
    // compare-and-branch then falls between MFMAs half as often
    int left = K / Cfg::BK - 2;                      // k-steps whose loads are this tile's
    for (;; left -= 2) {
        if (left == 0) {                             // from here on the loads are the next tile's
            if (last) {                              // or the last two k-steps again, from L2 and to no use
                lp.a_ptr -= 2 * Cfg::BK;
                lp.b_ptr[0] -= 2 * Cfg::BK;
                if (Cfg::DUAL) lp.b_ptr[1] -= 2 * Cfg::BK;
            } else {
                start_loads_1w<Full>(lp, nxt, id, wave, lane, A, B0, B1, row_index, index_div, N, K);
                draw();
            }
        }
        kstep_1w<Cfg, R>(acc, fa, fb, rs, lp, wave, pa[0], pa[1], pb[0], pb[1]);
        kstep_1w<Cfg, R>(acc, fa, fb, rs, lp, wave, pa[0], pa[1], pb[0], pb[1]);
        if (left == 0) break;
    }
    mfma_drain(acc[TM - 1]);                         // before anything else touches the accumulators
    sb = rs.sb;                                      // B stage of the next tile's first k-step
    // rows of a higher next tile that this one's loads did not reach, of both its k-steps
    if constexpr (TM < 8) {
        if (!last && nxt.height > Cfg::BM) {
#pragma unroll
            for (int i = TM; i < 8; ++i) {
                dma16(lp.a_ptr - 2 * Cfg::BK, lp.a_voff[i], wave * 1024 + i * 4096);
                dma16(lp.a_ptr - Cfg::BK, lp.a_voff[i], AB + wave * 1024 + i * 4096);
            }
        }
    }
    // The B stage of the last k-step is idle: every wavefront had read it at that k-step's barrier, and the
    // next load into it is the next tile's first. A wavefront stages its outputs in the 8 KB that it will
    // then fill by itself.
    unsigned char* idle = smem + R::A_RING + (sb == 0 ? (R::NB - 1) * BB : sb - BB);
    store_tile_via_lds<Cfg>(acc, tc, fp, wave, lane, idle + wave * (R::LB * 1024), C, N, [&] {
        __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0): the next tile's first loads, and what draw() asked for
        drawn(idle);
    });
}

constexpr int kCounterInts = 32;                     // a counter per XCD, on a cache line of its own

// Tiles are enumerated at Cfg::BM rows and run at the height that tile_in_expert gives them, half of that and
// up in steps of an eighth (an expert's short tail, or a half of a tile of the last, partial round, at half).
// Every output element is one accumulator chain over k, so the bits do not depend on which height computed it.
//
// PERSISTENT: workgroup b of P per XCD serves XCD b % 8's range of tiles: its slots b / 8 and b / 8 + P, then whichever
// slot it draws, one tile ahead of the one it computes, so that workgroups even out tiles of unequal cost among themselves as
// the dispatcher did. No workgroup waits for another one; each ends when it has drawn past the end of its
// range. Draws: of a range of S slots, S - 2 P are drawn, and every workgroup that has a second tile, min(P, S - P) of
// them, draws until it is past the end: S - P draws in all, whose last one sets the counter back to zero for
// the next launch.
template <class Cfg, bool PERSISTENT>
__global__ __launch_bounds__(Cfg::NTHREADS) void grouped_gemm_1w_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B0,
    const uint16_t* __restrict__ B1, uint16_t* __restrict__ C,
    const int32_t* __restrict__ offsets, const int32_t* __restrict__ row_index, RowDiv index_div,
    int E, int N, int K, int split_cus, int32_t* __restrict__ counters) {
    using R = Ring1W<Cfg>;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int xcd = blockIdx.x % kXcds, workgroups = gridDim.x / kXcds;
    int32_t* counter = counters + xcd * kCounterInts;
    const int NT = N / Cfg::BN_OUT;
    const Cut cut = K < kLongK ? Cut::kAlways : Cut::kLong;
    TileTable<Cfg::BM> table;                        // kept over the tiles: a lookup then reads no memory
    TileCoord tc;
    const uint32_t magic = division_magic(lane);
    if constexpr (PERSISTENT) {
        table.init(offsets, E, NT, split_cus, xcd, lane);
        tc = uniform_tile(table.find(NT, cut, blockIdx.x / kXcds, magic));
    } else {
        tc = locate_tile<Cfg::BM>(offsets, E, NT, split_cus, cut);
    }
    if (PERSISTENT ? tc.expert == kNoTile : tc.expert < 0) return;     // uniform for the whole workgroup
    // to a persistent one an empty slot is a tile without rows and without k-steps: it has to go on to its next one
    if (tc.expert == kEmptySlot) tc = TileCoord{0, 0, 0, 0, Cfg::BM / 2};
    bool last = !PERSISTENT;
    int ahead = 0;                                   // lane 0 of wavefront 0: the latest draw
    auto draw = [&] {
        if (PERSISTENT && threadIdx.x == 0) {
            // an address that the compiler does not know to be uniform: of one that is it makes a sum over
            // the lanes, and waits for the result on the spot to hand it to them
            int at = 0;
            asm volatile("" : "+v"(at));
            ahead = __hip_atomic_fetch_add(counter + at, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    // handed to the other wavefronts in the 4 KB of the idle B stage behind each one's staging region
    auto drawn = [&](unsigned char* idle) {
        if (PERSISTENT && wave == 0) {
            const int v = __builtin_amdgcn_readfirstlane(ahead);
            if (lane < 4) *reinterpret_cast<int*>(idle + lane * (R::LB * 1024) + kEpilogueBytes) = v;
        }
    };
    auto row_id = [&](const TileCoord& t) {          // without an index some load, so that no path sets it otherwise
        if constexpr (!Cfg::DUAL) return 0;
        return row_index != nullptr ? row_index[t.row0 + a_row_1w(t, wave, lane)] : offsets[0];
    };
    LoadPlan1W lp;
    uint32_t sb = 0;
    // the first two k-steps of tile t into the rings: stages 0 and 1 of A, sb and the one behind it of B
    auto first_loads = [&](const TileCoord& t, int id) {
        start_loads_1w<Cfg>(lp, t, id, wave, lane, A, B0, B1, row_index, index_div, N, K);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const uint32_t b_stage = s == 0 ? sb : sb + R::BB == R::NB * R::BB ? 0u : sb + R::BB;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i < 4 || i * 32 < t.height) dma16(lp.a_ptr, lp.a_voff[i], s * R::AB + wave * 1024 + i * 4096);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                dma16(lp.b_ptr[Cfg::DUAL ? i >> 2 : 0], lp.b_voff[i], R::A_RING + b_stage + wave * (R::LB * 1024) + i * 1024);
            lp.a_ptr += Cfg::BK;
            lp.b_ptr[0] += Cfg::BK;
            if (Cfg::DUAL) lp.b_ptr[1] += Cfg::BK;
        }
    };
    init_b_offsets<Cfg>(lp, wave, lane, K);
    first_loads(tc, row_id(tc));
    if (tc.height == Cfg::BM) wait_vmcnt<R::LA + R::LB>();   // k-step 0 landed
    else wait_vmcnt<4 + R::LB>();
    int slot = blockIdx.x / kXcds + workgroups;      // of the next tile
    unsigned char* idle = nullptr;                   // the B stage in which the latest draw lies, once there is one
    while (true) {
        // lane-dependent addresses are formed anew for every tile: kept over the loop they would take the
        // registers of fragments
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(lane) :: "memory");
        __builtin_amdgcn_s_barrier();                // the tile's first k-step has landed for every wavefront
        TileCoord nxt = tc;
        if constexpr (PERSISTENT) {
            if (idle != nullptr)
                slot = 2 * workgroups + __builtin_amdgcn_readfirstlane(
                    *reinterpret_cast<const int*>(idle + wave * (R::LB * 1024) + kEpilogueBytes));
            const TileCoord found = uniform_tile(table.find(NT, cut, slot, magic));
            last = found.expert == kNoTile;
            if (found.expert == kEmptySlot)
                nxt = TileCoord{tc.expert, tc.row0, 0, tc.nt, Cfg::BM / 2};
            else if (!last)
                nxt = found;
            else if (idle != nullptr && slot == table.range.slots + workgroups - 1 && threadIdx.x == 0)
                __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const int id = row_id(nxt);
        auto run = [&](auto cfg_tag) {
            using TileCfg = typename decltype(cfg_tag)::type;
            ring_tile_1w<TileCfg, Cfg>(tc, nxt, lp, id, last, sb, smem, wave, lane, A, B0, B1, C, row_index, index_div,
                                       N, K, draw, drawn);
        };
        if (PERSISTENT && tc.rows == 0) {            // nothing to compute: the next tile's first loads, as at the start
            wait_vmcnt<0>();                         // this one's have landed where they go
            __builtin_amdgcn_s_barrier();            // every wavefront has read the draw that the next one replaces
            if (!last) {
                draw();
                first_loads(nxt, id);
                wait_vmcnt<0>();
                drawn(smem + R::A_RING + (sb == 0 ? (R::NB - 1) * R::BB : sb - R::BB));
            }
        } else switch (tc.height) {
            case 128: run(type_tag<AtHeight<Cfg, 128>>{}); break;
            case 160: run(type_tag<AtHeight<Cfg, 160>>{}); break;
            case 192: run(type_tag<AtHeight<Cfg, 192>>{}); break;
            case 224: run(type_tag<AtHeight<Cfg, 224>>{}); break;
            default: run(type_tag<Cfg>{}); break;
        }
        if (last) break;
        tc = nxt;
        idle = smem + R::A_RING + (sb == 0 ? (R::NB - 1) * R::BB : sb - R::BB);
    }
}

// The 256-row tiles of eight wavefronts, a workgroup per tile; tiles of at most HalfCfg::BM rows run at half
// the height.
template <class Cfg, class HalfCfg, int NA, int NB>
__global__ __launch_bounds__(Cfg::NTHREADS) void grouped_gemm_ring_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B0,
    const uint16_t* __restrict__ B1, uint16_t* __restrict__ C,
    const int32_t* __restrict__ offsets, const int32_t* __restrict__ row_index, RowDiv index_div,
    int E, int N, int K, int split_cus) {
    static_assert(HalfCfg::BM * 2 == Cfg::BM && HalfCfg::BN == Cfg::BN && HalfCfg::BK == Cfg::BK &&
                  HalfCfg::NTHREADS == Cfg::NTHREADS && HalfCfg::DUAL == Cfg::DUAL, "same n-tiling");
    static_assert(RingCfg<HalfCfg, NA, NB>::SMEM <= RingCfg<Cfg, NA, NB>::SMEM, "LDS of the full tile");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

    const TileCoord tc = locate_tile<Cfg::BM>(offsets, E, N / Cfg::BN_OUT, split_cus);
    if (tc.expert < 0) return;                       // uniform for the whole workgroup
    if (tc.height == HalfCfg::BM)
        ring_tile<HalfCfg, NA, NB>(tc, smem, A, B0, B1, C, row_index, index_div, N, K);
    else
        ring_tile<Cfg, NA, NB>(tc, smem, A, B0, B1, C, row_index, index_div, N, K);
}

}  // namespace gemm
}  // namespace moe
