// Grouped expert GEMMs on the gfx950 matrix cores (paper Table 1 row 3: per expert three
// d_h x d_e bf16 matrices, 6*rows*d_h*d_e FLOPs; Section 4.1: each expert is a gated FFN).
//
//   gate/up : H[p, j]  = bf16( SiLU(sum_i Xp[p,i] W1_e[j,i]) * (sum_i Xp[p,i] W3_e[j,i]) )
//   down    : Yp[p, c] = bf16( sum_j H[p,j] W2_e[c,j] )
// for every row p of expert e's group, offsets[e] <= p < offsets[e+1].
//
// A workgroup owns a BM x BN output tile of ONE expert; tiles are enumerated on the device
// from `offsets` (no host synchronisation, variable rows per expert, empty experts produce no
// tile). Every output element is one accumulator chain over k = 0,16,32,... with the same
// MFMA instruction in every tile configuration, so results do not depend on how many rows an
// expert has, on its place among the experts of a call or on which configuration is picked
// (coalesced == micro-batched, some experts == all of them, bit for bit).
#include <algorithm>
#include <atomic>
#include <cmath>

#include "expert_gemm_kernel.h"

namespace moe {

constexpr int kCounterSets = 64;
static __device__ __align__(256) int32_t tile_counter_sets[kCounterSets][kTileCounterBytes / sizeof(int32_t)];
static std::atomic<uint64_t> counter_sets_taken[64];         // one bit per set and device
static std::atomic<int32_t*> counter_sets_at[64];

int32_t* take_tile_counters(int device, int* set) {
    *set = -1;
    int32_t* base = counter_sets_at[device].load(std::memory_order_acquire);
    if (base == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(tile_counter_sets)) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        base = static_cast<int32_t*>(p);
        counter_sets_at[device].store(base, std::memory_order_release);
    }
    uint64_t taken = counter_sets_taken[device].load(std::memory_order_relaxed);
    while (~taken != 0) {
        const int n = __builtin_ctzll(~taken);
        if (counter_sets_taken[device].compare_exchange_weak(taken, taken | (1ull << n), std::memory_order_acq_rel)) {
            *set = n;
            return base + n * (kTileCounterBytes / sizeof(int32_t));
        }
    }
    return nullptr;
}

void give_tile_counters(int device, int set) {
    if (set >= 0) counter_sets_taken[device].fetch_and(~(1ull << set), std::memory_order_acq_rel);
}

int compute_units(int device) {
    static std::atomic<int> cached[64];
    int n = cached[device].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || n <= 0) {
            (void)hipGetLastError();
            n = 256;
        }
        cached[device].store(n, std::memory_order_relaxed);
    }
    return n;
}

namespace {

using gemm::Config;
template <bool F32, class Cfg>
using Out = std::conditional_t<F32, gemm::F32Out<Cfg>, Cfg>;

template <class Kernel, class... Args>
int launch_tiles(const GemmEnv& env, std::atomic<uint64_t>& attr_set, Kernel kern, int smem,
                 int threads, long long grid, hipStream_t s, Args... args) {
    // The attribute belongs to the kernel's code object on ONE device: one bit per device, set
    // by whichever thread launches this kernel there first (setting it twice is harmless).
    if (env.device < 0 || env.device >= 64) return MOE_ERR_INVALID_ARG;
    const uint64_t bit = 1ull << env.device;
    if (!(attr_set.load(std::memory_order_acquire) & bit)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess)
            return MOE_ERR_HIP;
        attr_set.fetch_or(bit, std::memory_order_release);
    }
    grid = (grid + kXcds - 1) / kXcds * kXcds;
    if (grid > 0x7fffffffLL) return MOE_ERR_UNSUPPORTED_SHAPE;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(grid)), dim3(threads), smem, s, args...);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

// Most row tiles that R rows in E groups can make: a group of m > 0 rows has ceil(m / BM) of them, so
// all groups together have at most R / BM + min(E, R). The bound sizes the grid, and a workgroup
// without a tile still occupies a compute unit's LDS while it finds that out (about 1 us, one at
// a time per compute unit with the deep rings): one token through 8 of 128 experts used to launch
// 4096 workgroups for the 256 tiles of the down projection, 25.0 us for 25 MB of weights; with
// min(E, R) in place of E it takes 9.0 us (gate/up 18.5 -> 16.5 us).
long long most_row_tiles(int R, int E, int BM) { return R / BM + std::min(E, R); }

// Experts that R rows are expected to touch.
double touched_experts(int R, int E) { return E * (1.0 - std::exp(-static_cast<double>(R) / E)); }

// Step of the staggered first starts of the weight-bound tiles (gemm::spread_start), 0: together. Together -> steps of
// 1 -> of 2, in us: pitch of 32 KB (down, 8 experts of 6144 x 16384) 16 tokens 257, 251, 246; 64 261, 256, 252; 256 291, 279,
// 271; 420 314, 306, 297. Pitch of 12 KB (gate/up there) 489, 485, 480; 501, 501, 501; 549, 547, 543; 594, 594, 590; 200 tokens
// 582, 536, 531. Pitch of 28 KB (down, 4096 x 14336) 64 tokens 154, 152, 150; 128 160, 160, 159; 200 188, 187, 186; but 256, a tile
// per compute unit, 168, 169, 176, so steps of 2 only at the worst pitch. A reduction of 4096 ends too soon for it: gate/up,
// 16 tokens at 4096 x 14336 279 together, 290 with eight starts over the same span; nor does a launch of few weights pay for
// the last starts, 11 us late with steps of 1 (one token through 2 of 8 experts of 4096 x 14336, 235 MB of W2: layer call
// 126.8 us together, 137.5; of 6144 x 16384, 403 MB, 202.7 and 211). Other reductions, both projections of 8 experts with
// the same rows each, together -> as here: 8192 x 8192 4 rows 514 -> 506, 60 531 -> 519; 10240 x 10240 4 775 -> 738, 32
// 803 -> 790; 12288 x 8192 32 754 -> 747; 7168 x 18432 60 1101 -> 1072; within 1 % of each other where the pitch is no multiple
// of 4 KB (11008, 6656, 7680, 17920). A gate/up reduction of 5120 gains nothing: 4 rows 485 -> 487 with steps of 1, 60 593 -> 595.
int spread_steps(int R, int E, int N, int K, bool dual) {
    const double bytes = touched_experts(R, E) * (dual ? 4.0 : 2.0) * N * K;
    return K < 6144 || bytes < 0.8e9 ? 0 : K % 16384 == 0 ? 2 : 1;
}

// The generic kernel with Cfg::NSTAGE stages.
template <class Cfg>
int launch_grouped(const GemmEnv& env, const moe_bf16* A, const moe_bf16* B0, const moe_bf16* B1, moe_bf16* C,
                   const int32_t* offsets, const int32_t* row_index, int index_div,
                   int R, int E, int N, int K, hipStream_t s) {
    if (N % Cfg::BN_OUT != 0 || K % Cfg::BK != 0) return MOE_ERR_UNSUPPORTED_SHAPE;
    static std::atomic<uint64_t> attr_set{0};
    const long long max_mt = most_row_tiles(R, E, Cfg::BM);
    return launch_tiles(env, attr_set, gemm::grouped_gemm_kernel<Cfg>, Cfg::SMEM, Cfg::NTHREADS,
                        max_mt * (N / Cfg::BN_OUT), s, A, B0, B1, C, offsets, row_index,
                        gemm::RowDiv(index_div), E, N, K, spread_steps(R, E, N, K, Cfg::DUAL));
}

// Slots of all tiles that R rows in E groups can make: the tiles, and where the last round is split two slots
// per tile there, at most ceil(cus / 2 / 8) more in every XCD's range.
long long most_slots(int R, int E, int BM, int NT, int split_cus) {
    return most_row_tiles(R, E, BM) * NT + kXcds * ((split_cus / 2 + kXcds - 1) / kXcds + 1);
}

// The pipelined kernel of eight wavefronts with operand rings of NA and NB stages; tiles of at most HalfCfg::BM
// rows and the tiles of a last round that is less than half full run at half the height.
template <class Cfg, class HalfCfg, int NA, int NB>
int launch_ring(const GemmEnv& env, const moe_bf16* A, const moe_bf16* B0, const moe_bf16* B1, moe_bf16* C,
                const int32_t* offsets, const int32_t* row_index, int index_div,
                int R, int E, int N, int K, hipStream_t s) {
    if (N % Cfg::BN_OUT != 0 || K % Cfg::BK != 0) return MOE_ERR_UNSUPPORTED_SHAPE;
    if (K / Cfg::BK < (NA > NB ? NA : NB)) return MOE_ERR_UNSUPPORTED_SHAPE;
    static std::atomic<uint64_t> attr_set{0};
    const int cus = env.split_last_round ? compute_units(env.device) : 0;
    return launch_tiles(env, attr_set, gemm::grouped_gemm_ring_kernel<Cfg, HalfCfg, NA, NB>,
                        gemm::RingCfg<Cfg, NA, NB>::SMEM, Cfg::NTHREADS,
                        most_slots(R, E, Cfg::BM, N / Cfg::BN_OUT, cus), s, A, B0, B1, C,
                        offsets, row_index, gemm::RowDiv(index_div), E, N, K, cus);
}

// Expected row tiles of height h: groups one standard deviation below and above the mean.
double mean_row_tiles(double avg, double sigma, int h) {
    return 0.5 * (std::ceil(std::max(1.0, avg - sigma) / h) + std::ceil((avg + sigma) / h));
}

// Expected row tiles of height h of a launch.
double row_tiles(int R, int E, int h) {
    const double avg = static_cast<double>(R) / (E > 0 ? E : 1);
    return E * mean_row_tiles(avg, std::sqrt(avg), h);
}

// The pipelined kernel of one wavefront per SIMD: a persistent workgroup per compute unit where the reduction is
// short and most of them get two tiles and more, else a workgroup per tile (4000 tokens through 8 experts of 512 x 1024,
// one tile per compute unit, 62.4 us a layer with persistent ones, 60.9 without).
template <class Cfg>
int launch_1w(const GemmEnv& env, const moe_bf16* A, const moe_bf16* B0, const moe_bf16* B1, moe_bf16* C,
              const int32_t* offsets, const int32_t* row_index, int index_div,
              int R, int E, int N, int K, hipStream_t s) {
    if (N % Cfg::BN_OUT != 0 || K % (2 * Cfg::BK) != 0 || K < 4 * Cfg::BK) return MOE_ERR_UNSUPPORTED_SHAPE;
    static std::atomic<uint64_t> attr_set[2];
    const int cus = compute_units(env.device), split = env.split_last_round ? cus : 0;
    const long long slots = most_slots(R, E, Cfg::BM, N / Cfg::BN_OUT, split);
    if (K < gemm::kLongK && row_tiles(R, E, Cfg::BM) * (N / Cfg::BN_OUT) > 1.5 * cus)
        return launch_tiles(env, attr_set[0], gemm::grouped_gemm_1w_kernel<Cfg, true>, gemm::Ring1W<Cfg>::SMEM,
                            Cfg::NTHREADS, std::min<long long>(slots, cus), s, A, B0, B1, C, offsets, row_index,
                            gemm::RowDiv(index_div), E, N, K, split, env.tile_counters);
    return launch_tiles(env, attr_set[1], gemm::grouped_gemm_1w_kernel<Cfg, false>, gemm::Ring1W<Cfg>::SMEM,
                        Cfg::NTHREADS, slots, s, A, B0, B1, C, offsets, row_index, gemm::RowDiv(index_div), E, N, K,
                        split, env.tile_counters);
}

// The n-tiles of one projection in each kind of tile, and what the small tiles of config 2 cost.
struct NTiles {
    int large, mid, small;
    double mid_step;             // k-step of the 96- and 128-row tiles, of a 256-row tile's
    double small_alone, small_pair;   // k-step of a 64-row tile alone on a compute unit / of two on one
    double weight_mb;            // of the launched experts
    int ksteps;                  // of the reduction
};

// Tile configuration by average rows per expert. All configurations give identical bits.
//
// The measured constants of this rule and of the variants in launch_gateup and launch_down, and what each stands
// on ("cold": a graph of calls with other weights every time, 1.2 GB and more of them; else the same ones):
//   0.82, 0.6   k-step of a 96- or 128-row tile (256 or 128 columns), 0.41 / 0.58 and 0.27 / 0.38 of one 64-row
//               tile alone on a compute unit / of two: one expert of 4096 x 14336, 512 rows (below)
//   0.56, 0.8   k-step of a 256-row tile where at most half the compute units have one, weights from cache / from
//   (64 MB)     memory. The line only has to keep large weights from the lower price: 512 rows through one
//               expert of 4096 x 14336 234 us a layer cold with 0.8, 293 with 0.56. Layers of up to 64 MB differ
//               by -4 to +5 % either way, cold or not (1024 rows through 4 of 2048 x 1408 cold 82.7 us with 0.56,
//               80.8 with 0.8; 1600 through 8 of 2048 x 768 61.6 and 64.5), and of three such layers, 256 to 6000
//               rows, none is over 1 % slower cold than with the 128- or the 256-row tiles throughout
//   + 3, + 6    a tile's cost outside its reduction, in k-steps, and 0.9 the margin that small tiles have to win by:
//               512 and 900 tokens through 8 experts of 512 x 1024 (below)
//   0.93        seven stages against four, 2.5 narrow gate/up tiles, 3.5 128 columns down: where they are used
int pick_config(const GemmEnv& env, int R, int E, const NTiles& nt) {
    if (env.forced_config >= 0) return env.forced_config;
    // 0: pipelined 256-row tiles (lower ones at the end). 1: 128-row tiles (generic kernel).
    // 2: up to 64 rows per expert (64-row tiles, two workgroups per compute unit). 3: up to 32
    // (32-row tiles). 4: 96-row tiles of four wavefronts side by side (groups of 65 to 96 rows: a
    // quarter fewer matrix instructions and fragment reads per k-step than the 128-row tile, and
    // room for a deeper weight ring in the down projection). Per-expert counts are not known on
    // the host, so the choice prices a uniform routing: the average group and its standard deviation.
    const double avg = static_cast<double>(R) / (E > 0 ? E : 1);
    const double sigma = std::sqrt(avg);
    const double upper = avg + 2.0 * sigma;
    if (upper <= 32.0) return 3;
    // The 64-row tiles against the 96-row ones, gate/up + down: 500 tokens through 128 experts of
    // 2048 x 768 205 us against 218; with a few experts past 64 rows (560 tokens through 64 experts of
    // 2048 x 1408) 226 against 211. Layers on the same weights: 195 tokens through 8 of 4096 x 14336 502 against 524, of
    // 6144 x 16384 830 against 817; past the line, 205 there 905 against 849, 810 through 128 of 2048 x 768 281 against 268.
    if (upper <= 64.0) return 2;
    const int cus = compute_units(env.device);
    // The 96- and 128-row tiles only where the largest group is expected to fit one: a second tile costs more than
    // they gain. The largest of E groups lies about sqrt(2 ln E) standard deviations above the mean (two for the
    // 8 experts that the lines were drawn at). Gate/up and down, 96- / 128- / 256-row tiles: 800 tokens through 64 experts
    // of 2048 x 1408 (75 rows each) 154 and 79, 154 and 79, 154 and 77 us; 280 through 8 of 6144 x 16384 (70) 517 and 277,
    // 520 and 276, 543 and 336. 128- / 256-row: 1700 through 128 of 2048 x 768 (106) 174 and 111, 158 and 103;
    // 420 through 8 of 4096 x 14336 (105) 354 and 185, 358 and 232; 460 (115) 370 and 306, 362 and 234. With more rows the
    // 256-row tiles and their lower tails are the faster ones (4096 x 14336, 600 tokens 479 and 313, 393 and 240, 2048 1000
    // and 725, 761 and 498; two experts of 4096 x 14336 with 300 rows each, gate/up 179 and 147).
    const double largest = avg + std::max(2.0, std::sqrt(2.0 * std::log(static_cast<double>(E)))) * sigma;
    int config = largest <= 96.0 ? 4 : largest <= 128.0 ? 1 : 0;
    // Groups around 256 rows, where one 256-row tile per expert leaves compute units idle and the few groups of more
    // than 256 rows start a second round: two or three 128-row tiles per expert are two rounds too, of half the
    // height. Down, 8 experts of 6144 x 16384, 256- against 128-row tiles: 1000 tokens 656 and 544 us, 1024 671 and 547;
    // below the lines, one large round, 975 472 and 528; above, three of the others, 1050 633 and 742. With reductions of
    // 12288, 8192, 6144 438 and 407, 290 and 261, 229 and 217 (1024 tokens); below that a wrong guess of the groups costs as
    // much as a right one gains (12 experts, K = 4096 102 and 134 or 143 and 132, as the routing falls).
    const double past256 = 0.5 * E * std::erfc((256.0 - avg) / (std::sqrt(2.0) * sigma));   // groups, expected
    if (config == 0 && nt.ksteps >= 96 && E * nt.large <= cus && (E + past256) * nt.large > cus &&
        (2.0 * E + past256) * nt.mid <= 0.95 * 2.0 * cus)
        config = 1;
    // A launch of at most one such tile per compute unit takes one tile's time however many compute
    // units idle: small tiles are worth their extra loads if they use the idle ones. Units of a
    // k-step of a full 256-row tile (about 1 us), measured on one expert of 4096 x 14336 (512 rows,
    // down projection: 125 us with large tiles, 94 and 87 us with 64-row ones of 128 and 64 columns;
    // 181 against 124 us when the weights come from memory, which a compute unit reads at 60 GB/s). What a
    // tile costs outside its reduction is added in k-steps, and decides where that is short (layer call of
    // 512 tokens through 8 experts of 512 x 1024 27.9 us with large gate/up tiles, 26.6 with 64-row ones; 900
    // tokens 29.1 and 28.1).
    const int rows = config == 0 ? 256 : config == 1 ? 128 : 96;
    const double tiles = E * mean_row_tiles(avg, sigma, rows) * (config == 0 ? nt.large : nt.mid);
    if (tiles <= cus) {
        const double step = config != 0 ? nt.mid_step : tiles <= 0.5 * cus ? (nt.weight_mb > 64.0 ? 0.8 : 0.56) : 1.0;
        const double small = E * mean_row_tiles(avg, sigma, 64) * nt.small;
        const double rounds = std::floor(small / (2.0 * cus)), rem = small - rounds * 2.0 * cus;
        const double fill = rounds * nt.small_pair + (rem <= 0.0 ? 0.0 : rem <= cus ? nt.small_alone : nt.small_pair);
        if ((nt.ksteps + 3.0) * fill < 0.9 * (nt.ksteps + 6.0) * step) return 2;
    }
    return config;
}

NTiles gateup_tiles(int E, int d, int f) {
    return NTiles{f / 128, f / 128, f / 64, 0.82, 0.41, 0.58, 4e-6 * E * d * f, d / 64};
}

// Tiles of half the width while up to two and a half of them go to a compute unit, gate/up against
// the 128-column ones: one token through 8 of 128 experts of 2048 x 768 (0.75 per compute unit) 14.2
// and 18.2 us, 2 (1.4) 21.6 and 22.3, 2 through 6 of 64 of 2048 x 1408 (2.1) 23.9 and 25.0, 64 through
// 2 of 8 of 512 x 1024 (1.0) 7.7 and 8.7. Longer reductions than those below lose past the line: layers of 4096 x 14336,
// one token through 2 of 8 (3.3) 142 and 129, of 6144 x 16384 (3.7) 229 and 220
bool narrow_gateup_tiles(int R, int E, int f, int cus) { return 2.0 * touched_experts(R, E) * (f / 64) <= 2.5 * cus; }

// Workgroups of `tiles` tiles that find a free slot per round, over the slots of those rounds.
double last_round_use(double tiles, double slots) { return tiles / (slots * std::ceil(tiles / slots)); }

// Short reductions, more than that: a tile of half the width leaves half as much of the last round empty, except
// where both widths take two rounds (three to four narrow tiles per compute unit) or the wide ones fill theirs. Layers
// through 8 of 128 experts of 2048 x 768, wide -> narrow: 4 tokens (2.6) 66.6 -> 62.8 us, 5 (3.3) 69.8 -> 72.7, 7 (4.4)
// 99.4 -> 88.6, 20 (8.7) 155 -> 150, 37 (10.8) 184 -> 180, 120 (12, all full) 209 -> 213; 6 of 64 of 2048 x 1408, 4 tokens
// (3.6) 70.0 -> 70.8, 16 (8.7) 151 -> 145, 80 (11) 182 -> 178; 4 of 60 of 1536 x 1536, 30 tokens 133 -> 127.
bool narrow_short_gateup_tiles(int R, int E, int d, int f, int cus) {
    const double wide = touched_experts(R, E) * (f / 64);
    return d <= 2048 && (2.0 * wide <= 3.0 * cus || wide > 2.0 * cus) && last_round_use(wide, cus) <= 0.97;
}

// The deep ring where no compute unit gets a second tile, whichever experts are touched: one
// token through 8 of 128 of 2048 x 768 (192 tiles) 14.3 against 14.9 us, through 4 of 32 of 2048 x 2048
// (256) 16.7 against 17.5; through 6 of 64 of 2048 x 1408 (264) 20.2 against 18.2
bool one_tile_per_cu(int R, int E, int f, int cus) { return std::min(E, R) * (f / 32) <= cus; }

// Large tiles: four wavefronts of 128 x 128 outputs (one per SIMD) or eight of 128 x 64.
bool use_one_wave_per_simd(const GemmEnv& env, int N, int K) {
    if (!gemm::offsets_fit_1w(N, K)) return false;
    if (K % 128 != 0) return false;       // its k-loop takes two 64-wide steps per trip
    if (env.large_tile_waves != 0) return env.large_tile_waves == 4;
    return true;     // faster at every shape measured (reductions of 768 to 16384)
}

// Weights may be loaded as non-temporal when (almost) every expert has a single m-tile: then no
// other tile asks for the same weight bytes and keeping them cached only displaces the rows.
bool single_m_tile(const GemmEnv& env, int R, int E, int BM) {
    if (env.stream_mode >= 0) return env.stream_mode != 0;
    const double avg = static_cast<double>(R) / (E > 0 ? E : 1);
    return avg + 2.0 * std::sqrt(avg) <= BM;
}

//                      BM   BN  BK WM WN NSTAGE DUAL [STREAM_B]
using GateUpLarge = Config<256, 256, 64, 2, 4, 2, true>;
// one wavefront per SIMD: 2 x 2 wavefronts of 128 x 128 outputs, fewer rows in lower tiles
using GateUpLarge1W = Config<256, 256, 64, 2, 2, 2, true>;
using DownLarge1W   = Config<256, 256, 64, 2, 2, 2, false>;
using GateUpMid   = Config<128, 256, 64, 2, 4, 3, true>;   // also the half-height tile of GateUpLarge
// 64 rows: four wavefronts of 32 rows share a workgroup, and its ring leaves room for a second
// workgroup on the compute unit, so that one streams weights while the other looks its tile up,
// waits for its first loads or stores; the two-wavefront tile with a four-stage ring of its own
// (one workgroup per compute unit) took 134 us at 500 tokens through 128 experts of 2048 x 768, gate/up,
// this one 126.5 us, and the down projection 86 -> 74 us
using GateUpSmall  = Config<64, 128, 64, 2, 2, 3, true>;
using GateUpSmallS = Config<64, 128, 64, 2, 2, 3, true, true>;
using DownSmallWide  = Config<64, 128, 64, 2, 2, 3, false>;
using DownSmallWideS = Config<64, 128, 64, 2, 2, 3, false, true>;
using DownSmall  = Config<64, 64, 64, 2, 2, 5, false>;    // more tiles
using DownSmallS = Config<64, 64, 64, 2, 2, 5, false, true>;
using DownLarge   = Config<256, 256, 64, 2, 4, 2, false>;
using DownMid     = Config<128, 128, 64, 2, 2, 4, false>;
using DownMidWide = Config<128, 256, 64, 2, 4, 3, false>;
using GateUpMidS   = Config<128, 256, 64, 2, 4, 3, true, true>;
using DownMidS     = Config<128, 128, 64, 2, 2, 4, false, true>;
using DownMidWideS = Config<128, 256, 64, 2, 4, 3, false, true>;
using GateUpMid96  = Config<96, 256, 64, 1, 4, 3, true>;
using GateUpMid96S = Config<96, 256, 64, 1, 4, 3, true, true>;
using DownMid96      = Config<96, 128, 64, 1, 4, 5, false>;
using DownMid96S     = Config<96, 128, 64, 1, 4, 5, false, true>;
using DownMid96Wide  = Config<96, 256, 64, 1, 4, 3, false>;
using DownMid96WideS = Config<96, 256, 64, 1, 4, 3, false, true>;
// A handful of rows per expert (decode). Four stages let two gate/up workgroups (three of the narrow
// down tiles) share a compute unit: at 2048 x 768 and 128 experts a tile has 32 or 12 k-steps, and with
// one workgroup per compute unit its lookup and first loads were a fifth of its time (37 tokens:
// gate/up 122 -> 114 us, down 72 -> 54 us). Seven stages where one workgroup per compute unit divides
// into whole rounds and two do not.
using GateUpTiny      = Config<32, 128, 64, 2, 2, 4, true>;
using GateUpTinyS     = Config<32, 128, 64, 2, 2, 4, true, true>;
using GateUpTinyDeepS = Config<32, 128, 64, 2, 2, 7, true, true>;
// A few tokens: more, narrower tiles. Four wavefronts (two, down) share their loads, which leave a wavefront
// one by one, some 100 cycles apart: one wavefront per tile took 15.8 us for gate/up of one token through 8 of
// 128 experts of 2048 x 768, four take 14.9, and 14.2 with the deep ring where no second tile has to fit; down
// of one token through 2 of 8 of 4096 x 14336 51.4 -> 45.5 us, of 6144 x 16384 73.1 -> 72.3.
using GateUpFewS     = Config<32, 64, 64, 2, 2, 4, true, true>;
using GateUpFewDeepS = Config<32, 64, 64, 2, 2, 6, true, true>;
using DownTiny     = Config<32, 64, 64, 2, 2, 4, false>;
using DownTinyS    = Config<32, 64, 64, 2, 2, 4, false, true>;
using DownFew      = Config<16, 32, 64, 1, 2, 6, false>;
using DownFewS     = Config<16, 32, 64, 1, 2, 6, false, true>;

// Tile of a gate/up launch that derives the groups from the selected experts (grouped_gemm_routed_kernel): those of
// launch_gateup's choice that leave every workgroup one tile or two. Beyond that each tile would pay for the
// derivation again.
enum class RoutedTile { none, few_deep, few, small_stream, small };
RoutedTile routed_tile(const GemmEnv& env, int R, int E, int d, int f) {
    if (R > gemm::kRoutedIds || env.forced_config >= 0 || env.stream_mode >= 0) return RoutedTile::none;
    const int cus = compute_units(env.device);
    switch (pick_config(env, R, E, gateup_tiles(E, d, f))) {
        case 3:
            if (!single_m_tile(env, R, E, 32) || !narrow_gateup_tiles(R, E, f, cus)) return RoutedTile::none;
            return one_tile_per_cu(R, E, f, cus) ? RoutedTile::few_deep : RoutedTile::few;
        case 2:
            if (most_row_tiles(R, E, 64) * (f / 64) > 2 * cus) return RoutedTile::none;
            return single_m_tile(env, R, E, 64) ? RoutedTile::small_stream : RoutedTile::small;
        default: return RoutedTile::none;
    }
}

template <class Cfg, int EW>
int launch_routed(const GemmEnv& env, const moe_bf16* x, const gemm::Routing& rt, int d, int f, int E,
                  const moe_bf16* W1, const moe_bf16* W3, moe_bf16* H, hipStream_t s) {
    static std::atomic<uint64_t> attr_set{0};
    const long long tiles = most_row_tiles(rt.T * rt.k, E, Cfg::BM) * (f / Cfg::BN_OUT);
    return launch_tiles(env, attr_set, gemm::grouped_gemm_routed_kernel<Cfg, EW>, Cfg::SMEM, Cfg::NTHREADS,
                        tiles + kXcds, s, x, W1, W3, H, rt, gemm::RowDiv(rt.k), E, f, d);
}

}  // namespace

bool gateup_routes(const GemmEnv& env, int T, int d, int f, int E, int k) {
    const RoutedTile t = routed_tile(env, T * k, E, d, f);
    if (t == RoutedTile::none) return false;
    // Ids at hand (device time of a layer call, separate launch -> without): 8 experts of 512 x 1024, 1 token 19.3 -> 17.4 us,
    // 16 20.1 -> 18.9, 256 24.8 -> 23.0, 500 27.9 -> 26.5. With the selection on the way, about one tile per compute unit: one
    // token through 8 of 128 experts of 2048 x 768 33.8 -> 32.2, 6 of 64 of 2048 x 1408 (1.03) 37.4 -> 36.7; two through 8 of 128
    // (1.5) 41.8 -> 43.1. Up to a token per wavefront.
    return E <= 16 || (T <= GateUpFewS::NW && (t == RoutedTile::few || t == RoutedTile::few_deep) &&
                       4 * most_row_tiles(T * k, E, 32) * (f / 32) <= 5 * compute_units(env.device));
}

int launch_gateup_routed(const GemmEnv& env, const moe_bf16* x, const float* logits, int32_t* topk_idx, float* topk_w,
                         int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* inv_perm, int T, int d, int f,
                         int E, int k, const moe_bf16* W1, const moe_bf16* W3, moe_bf16* H, hipStream_t s) {
    const gemm::Routing rt{logits, topk_idx, topk_w, counts, offsets, perm, inv_perm, T, k};
    const RoutedTile tile = routed_tile(env, T * k, E, d, f);
    auto with = [&](auto cfg) {
        using Cfg = decltype(cfg);
        if (E <= 16) return launch_routed<Cfg, 0>(env, x, rt, d, f, E, W1, W3, H, s);
        if (E <= 64) return launch_routed<Cfg, 1>(env, x, rt, d, f, E, W1, W3, H, s);
        if (E <= 128) return launch_routed<Cfg, 2>(env, x, rt, d, f, E, W1, W3, H, s);
        return launch_routed<Cfg, 4>(env, x, rt, d, f, E, W1, W3, H, s);
    };
    switch (tile) {
        case RoutedTile::few_deep: return with(GateUpFewDeepS{});
        case RoutedTile::few: return with(GateUpFewS{});
        case RoutedTile::small_stream: return launch_routed<GateUpSmallS, 0>(env, x, rt, d, f, E, W1, W3, H, s);
        case RoutedTile::small: return launch_routed<GateUpSmall, 0>(env, x, rt, d, f, E, W1, W3, H, s);
        default: return MOE_ERR_UNSUPPORTED_SHAPE;
    }
}

// `a` is the grouped activation matrix [R, d] when row_index is NULL; otherwise it is the
// token matrix [T, d] and grouped row p reads token row_index[p] / index_div (the caller makes
// sure that T * d * 2 bytes fit a 32-bit offset). R bounds the rows of the E launched experts
// (it sizes the grid); R_hint is how many rows they are expected to hold together (it picks the
// tile configuration): the two differ when a call covers a subset of a layer's experts.
int launch_gateup(const GemmEnv& env, const moe_bf16* a, const int32_t* row_index, int index_div,
                  const int32_t* offsets, int R, int R_hint, int d, int f, int E,
                  const moe_bf16* W1, const moe_bf16* W3, moe_bf16* H, hipStream_t s) {
    if (R == 0) return MOE_OK;
    const moe_bf16* x_perm = a;
    int config = pick_config(env, R_hint, E, gateup_tiles(E, d, f));
    if (config == 0 && d / 64 < 3) config = 1;     // the pipelined kernel needs three k-steps
    // Row counts that lead to 96- or 128-row tiles let every group fit one, so their weights are streamed; the cached forms
    // (GateUpMid96, DownMid96 and DownMid96Wide) run under the tuning knob, those of 128 rows also where groups of about
    // 256 rows take two tiles and where a reduction is too short for the pipelined kernel.
    switch (config) {
        case 0:
            if (use_one_wave_per_simd(env, f, d))
                return launch_1w<GateUpLarge1W>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
            return launch_ring<GateUpLarge, GateUpMid, 2, 3>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
        case 1:
            if (single_m_tile(env, R_hint, E, 128))
                return launch_grouped<GateUpMidS>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
            return launch_grouped<GateUpMid>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
        case 4:
            if (single_m_tile(env, R_hint, E, 96))
                return launch_grouped<GateUpMid96S>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
            return launch_grouped<GateUpMid96>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
        case 3:
            if (single_m_tile(env, R_hint, E, 32)) {
                const double nt = touched_experts(R_hint, E) * (f / 64);
                const int cus = compute_units(env.device);
                if (narrow_gateup_tiles(R_hint, E, f, cus) || narrow_short_gateup_tiles(R_hint, E, d, f, cus)) {
                    if (one_tile_per_cu(R_hint, E, f, cus))
                        return launch_grouped<GateUpFewDeepS>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
                    return launch_grouped<GateUpFewS>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
                }
                // 16 tokens through 8 experts of 4096 x 14336, 7 rounds of one workgroup per compute unit or
                // 3.5 of two: 280 against 284 us; 4 tokens at 6144 x 16384, 6 or 3 rounds: 397 against 367
                if (last_round_use(nt, 2.0 * cus) < 0.93 * last_round_use(nt, cus))
                    return launch_grouped<GateUpTinyDeepS>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
                return launch_grouped<GateUpTinyS>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
            }
            return launch_grouped<GateUpTiny>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
        default:
            if (single_m_tile(env, R_hint, E, 64))
                return launch_grouped<GateUpSmallS>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
            return launch_grouped<GateUpSmall>(env, x_perm, W1, W3, H, offsets, row_index, index_div, R, E, f, d, s);
    }
}

namespace {

// F32: the same tilings with a float output matrix (gemm::F32Out).
template <bool F32>
int launch_down_as(const GemmEnv& env, const moe_bf16* H, const int32_t* offsets, int R, int R_hint,
                   int d, int f, int E, const moe_bf16* W2, moe_bf16* y_perm, hipStream_t s) {
    if (R == 0) return MOE_OK;
    const bool wide_mid = static_cast<long long>(E) * (d / 256) >= 160 && d % 256 == 0;
    const int cus = compute_units(env.device);
    int config = pick_config(env, R_hint, E, NTiles{d / 256, wide_mid ? d / 256 : d / 128, d / 64,
                                                    wide_mid ? 0.82 : 0.6, 0.27, 0.38, 2e-6 * E * d * f, f / 64});
    if (config == 0 && f / 64 < 3) config = 1;     // the pipelined kernel needs three k-steps
    switch (config) {
        case 0:
            if (use_one_wave_per_simd(env, d, f))
                return launch_1w<Out<F32, DownLarge1W>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
            return launch_ring<Out<F32, DownLarge>, Out<F32, DownMidWide>, 2, 3>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
        case 1:
            // HBM-bound: wide tiles stream more bytes per workgroup, but only if there are
            // enough of them to occupy the 256 compute units (about one m-tile per expert).
            if (wide_mid) {
                if (single_m_tile(env, R_hint, E, 128))
                    return launch_grouped<Out<F32, DownMidWideS>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
                return launch_grouped<Out<F32, DownMidWide>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
            }
            if (single_m_tile(env, R_hint, E, 128))
                return launch_grouped<Out<F32, DownMidS>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
            return launch_grouped<Out<F32, DownMid>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
        case 4:
            // wide tiles where there are enough of them for the 256 compute units, as for case 1
            if (wide_mid) {
                if (single_m_tile(env, R_hint, E, 96))
                    return launch_grouped<Out<F32, DownMid96WideS>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
                return launch_grouped<Out<F32, DownMid96Wide>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
            }
            if (single_m_tile(env, R_hint, E, 96))
                return launch_grouped<Out<F32, DownMid96S>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
            return launch_grouped<Out<F32, DownMid96>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
        case 3:
            // 32-column tiles where 64-column ones would leave compute units without any: one token through 2 of
            // 8 experts of 4096 x 14336 45.5 against 61.7 us; and while all of their row tiles find one: 64 tokens
            // through 2 of 8 of 512 x 1024 7.9 against 9.1 us
            if (touched_experts(R_hint, E) * (d / 64) < cus) {
                if (single_m_tile(env, R_hint, E, 16))
                    return launch_grouped<Out<F32, DownFewS>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
                if (row_tiles(R_hint, E, 16) * (d / 32) <= cus)
                    return launch_grouped<Out<F32, DownFew>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
            }
            if (single_m_tile(env, R_hint, E, 32))
                return launch_grouped<Out<F32, DownTinyS>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
            return launch_grouped<Out<F32, DownTiny>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
        default:
            // 32-row tiles where the 64-row ones would leave half of the compute units without any: 256 tokens through
            // 2 of 8 experts of 512 x 1024 (96 tiles) 9.2 against 9.9 us, 600 (192 tiles) 10.9 against 10.2
            if (row_tiles(R_hint, E, 64) * (d / 64) <= 0.5 * cus)
                return launch_grouped<Out<F32, DownTiny>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
            // 128 columns where that makes about two rounds of two workgroups per compute unit, else 64. Layer calls
            // with cold weights, 128 against 64 columns: 500 tokens through 128 experts of 2048 x 768 (8 tiles of 128
            // columns per compute unit) 239 and 243 us, 448 through 56 of 2048 x 1024, 4 per token (3.5) 149.2 and
            // 150.5; 110 tokens through 8 of 6144 x 16384 (1.5) 806 and 783. In between the sides are mixed (3.0: 384
            // tokens through 48 of 2048 x 1024 128.7 and 134.6, 192 through 24 of 4096 x 2048 242 and 238)
            if (touched_experts(R_hint, E) * (d / 128) >= 3.5 * cus) {
                if (single_m_tile(env, R_hint, E, 64))
                    return launch_grouped<Out<F32, DownSmallWideS>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
                return launch_grouped<Out<F32, DownSmallWide>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
            }
            if (single_m_tile(env, R_hint, E, 64))
                return launch_grouped<Out<F32, DownSmallS>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
            return launch_grouped<Out<F32, DownSmall>>(env, H, W2, nullptr, y_perm, offsets, nullptr, 1, R, E, d, f, s);
    }
}

}  // namespace

// y_perm is [R, d] bf16, or [R, d] fp32 when y_f32 is set.
int launch_down(const GemmEnv& env, const moe_bf16* H, const int32_t* offsets, int R, int R_hint,
                int d, int f, int E, const moe_bf16* W2, void* y_perm, bool y_f32, hipStream_t s) {
    moe_bf16* out = static_cast<moe_bf16*>(y_perm);
    return y_f32 ? launch_down_as<true>(env, H, offsets, R, R_hint, d, f, E, W2, out, s)
                 : launch_down_as<false>(env, H, offsets, R, R_hint, d, f, E, W2, out, s);
}

}  // namespace moe
