// adacomp_plan.h -- host-side plan (tile tables, workspace layout) and the structures the
// kernels read from device memory.  Internal to libadacomp.
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

#include "adacomp.h"

namespace adacomp {

constexpr uint32_t kWG = 256;            // threads per workgroup in every kernel (4 wave64)
constexpr uint32_t kMaxTileBins = 1024;  // bins per compress tile (LDS arrays)
constexpr uint32_t kFoldTiles = 512;     // tables up to this many compress tiles and
constexpr uint32_t kFoldLayers = 16;     // this many layers: the placement kernel does the scan itself
constexpr uint32_t kComputeUnits = 256;  // of an MI355X: what a small table's tiles are sized against
// elements per unpack tile: 16 KB of LDS accumulators (8192 was 10 % faster for the plain sum but
// 12 % slower with the optimizer epilogue)
constexpr uint32_t kUnpackTileElems = 4096;
constexpr uint32_t kMaxBatch = 32;  // learners per launch of the compress kernels
constexpr uint32_t kMaxPacketArgs = 64;  // packet pointers passed by value per unpack launch

// A layer as the kernels see it (64 bytes).
struct LayerDev {
    uint64_t elem_offset;
    uint64_t counts_offset;  // byte offsets inside a packet; fixed by the layer table alone
    uint64_t chunks_offset;
    uint32_t n_elems, L_T, n_bins, word_bytes;
    uint32_t ctile_start, n_ctiles;  // this layer's compress tiles in the tile table
    uint32_t bin_start, chunk_start; // first global bin / chunk index (g_max, chunk scratch arrays)
    uint32_t n_chunks, pad0;
};
static_assert(sizeof(LayerDev) == 64, "LayerDev layout");

// One workgroup's share of adacomp_compress: whole bins of one layer (32 bytes).
struct TileDev {
    uint64_t elem_base;   // first element in grad / residue (layer offset included)
    uint32_t stage_base;  // first entry of the tile's stretch of the staging array: the tiles' element counts,
                          // each rounded up to 4, summed over the tiles before it (so a multiple of 4)
    uint32_t L_T;
    uint32_t magic;       // floor(2^32 / L_T) + 1: bin = umulhi(e, magic) for e < 16384 (L_T > 1)
    uint16_t n_elems;     // elements in the tile, <= 4096 or 16384 by register class
    uint16_t n_bins;      // bins in the tile, <= kMaxTileBins
    uint32_t first_bin;   // index of the tile's first bin inside the layer
    uint32_t layer_flags; // bits 0..23 layer, bit 24 register class (0: 4096-element tiles, 1: 16384), bits 25..26 skip, bit 31 aligned
    __host__ __device__ uint32_t layer() const { return layer_flags & 0xFFFFFFu; }
    __host__ __device__ uint32_t jcode() const { return (layer_flags >> 24) & 1u; }
    // skip: for a tile of the larger class that is not 16-byte aligned but fits its class with the
    // misalignment added, the number of elements (1..3) between the 16-byte boundary below the tile
    // and its first element; 0 for aligned tiles and for unaligned ones that take 4-byte accesses
    __host__ __device__ uint32_t skip() const { return (layer_flags >> 25) & 3u; }
    __host__ __device__ bool aligned() const { return (layer_flags >> 31) != 0; }
};
static_assert(sizeof(TileDev) == 32, "TileDev layout");

// One workgroup's share of adacomp_unpack_accumulate: up to 64 whole bins inside one 64-bin
// chunk, or a slice [idx_lo, idx_lo + n_elems) of a single bin longer than the tile (32 bytes).  With what the kernels need to
// know about the layer, so that they do not have to fetch its record behind this one.
struct UTileDev {
    uint64_t elem_base;
    uint32_t first_bin;
    uint32_t layer_flags; // bits 0..23 layer, 24..27 log2(lanes per bin), bit 31 aligned
    uint32_t counts_offset, chunks_offset;   // of the layer, in a packet (which stays below 2^32 bytes)
    uint16_t n_elems;     // <= kUnpackTileElems
    uint16_t L_T;
    uint16_t idx_lo;
    uint8_t n_bins;       // <= 64
    uint8_t chunk_bins;   // bins of the layer in the tile's 64-bin chunk
    __host__ __device__ uint32_t layer() const { return layer_flags & 0xFFFFFFu; }
    __host__ __device__ uint32_t group_log2() const { return (layer_flags >> 24) & 15u; }
    __host__ __device__ bool aligned() const { return (layer_flags >> 31) != 0; }
    __host__ __device__ bool words8() const { return L_T <= 64u; }
};
static_assert(sizeof(UTileDev) == 32, "UTileDev layout");

// Consecutive unpack tiles served by one workgroup: tiles of one 64-bin chunk, or slices of one bin.
struct UGroupDev {
    uint32_t first_tile, n_tiles;
};
static_assert(sizeof(UGroupDev) == 8, "UGroupDev layout");
// The tile of group g where every group is a tile.  Workgroups are dealt to the 8 XCDs round-robin, so inside each 64 the
// order is transposed and the 8 tiles of a chunk, which read the same count and offset lines of every packet, share an L2.
__host__ __device__ inline uint32_t single_tile(uint32_t g, uint32_t n_tiles)
{
    return g < (n_tiles & ~63u) ? ((g & ~63u) | ((g & 7u) << 3) | ((g >> 3) & 7u)) : g;
}
constexpr uint32_t kUnpackGroupTiles = 8;   // at most this many tiles per group
constexpr uint32_t kUnpackMinGroups = 2048;  // groups of more than one tile only while this many workgroups remain (8 per compute unit)
// Tables with both word widths: one launch per width on tables of more tiles than this and with more packets than
// that: two launches are two ends, and the kernel for both and 16 packets had registers for fewer workgroups than those for one width.
// It has 75 now, as few as those, and one launch would be the faster one for more packets too, up to some 60 M elements.  Two / one, in us:
//   up to 8 packets: ResNet-50's table, SGD, 8 91 / 85, 1 77 / 72; 30 M, L_T 64 and 500, sum of 8 42 / 35; 10 M, 50 and 500, SGD with 8 43.6 / 37.4, sum of 6 18.5 / 13.6;
//   more, as it is / as one: 4 M, 50, and 8 M, 500, sum of 9 27.1 / 21.8, 16 31.1 / 24.1, SGD 51.2 / 44.5, Adam 71.6 / 64.3; 10 M and 15 M, sum of 16 61.3 / 48.9, SGD 91.5 / 84.0;
//   30 M, 64, and 30 M, 500, 16 110.3 / 99.7, 187.5 / 183.5, 267.7 / 267.6; 60 M, 50, and 65 M, 500, 16 241 / 232, 382 / 386, 553 / 573.
constexpr uint32_t kUnpackSplitTiles = 2048;
constexpr uint32_t kUnpackTogether = 8;
constexpr uint32_t kUnpackLdsFull = 27306;  // bytes of LDS that leave six workgroups on a compute unit
// Launches over the 16-bit layers of large tables are bound by HBM, which serves them better with fewer bytes in
// flight than the workgroups that fit put there (as it does k_fused, below): LDS that no kernel touches holds them to 5
// or 4 to a compute unit.  That needs full tiles, since a workgroup in one of 2080 elements (L_T 65; 2400 at 150 and 300, 2800 at
// 700, 3000 at 3000 and 9000, 3200 at 100 and 200, 4000 at 500) has half of them in flight, and few words to each: what hides the
// adds is other workgroups.  As many as fit (8, 7 or 6: up to 4, 8 or more packets) / 5 / 4, in us, 40 M elements (SGD and
// Adam: behind the adds, one slot after the other, as these launches were when this was measured; as they are, below):
//   sum    L_T 65, 1 packet 34 / 43 / 51, 4 50 / 63 / 74, 8 76 / 86 / 98; 100, 1 38.6 / 35.3 / 36.2, 4 37.9 / 46.9 / 54; 200, 4
//          42.2 / 39.2 / 39.3, 8 40.6 / 43.4 / 48.7; 300, 4 42.3 / 41.6 / 39.6, 8 41.5 / 44.4 / 51.6; 500, 1 42.2 / 41.5 / 40.5, 4 43.4 /
//          41.8 / 41.8, 8 46.6 / 42.0 / 42.2, 16 47.9 / 48.8 / 53; 9000, 4 38.5 / 36.3 / 36.1, 8 38.0 / 39.2 / 42.8; 24 M, L_T 500, 4 25.2 /
//          24.1 / 23.5, 8 25.5 / 26.2 / 28.1; 13 M, 4 11.9 / 12.6 / 14.1
//   SGD    L_T 65, 1 115 / 123 / 135, 8 127 / 144 / 163; 100, 1 120 / 118 / 122, 8 123 / 126 / 137; 200, 1 121 / 117 / 121, 4 121 / 123 /
//          128; 300, 4 116 / 121 / 129; 500, 1 126 / 117 / 117, 8 125 / 120 / 122, 16 126 / 127 / 133; 700, 4 117 / 115 / 118, 8 117.5 /
//          118.5 / 125; 3000, 8 118 / 116 / 119; 13 M, L_T 500, 4 41.8 / 41.1 / 43.1
//   Adam   L_T 65, 4 185 / 189 / 205, 8 193 / 207 / 228; 100, 4 194 / 189 / 191, 8 191 / 193 / 202; 200, 8 192 / 190 / 194; 300, 4 184 / 182 /
//          187, 8 183 / 185 / 194; 500, 1 205 / 203 / 188, 8 204 / 195 / 189, 16 202 / 198 / 193 (125 M 519 / 512 / 520); 9000, 8 193 / 189 /
//          186, 16 194 / 190 / 189; 13 M, L_T 500, 8 65.4 / 64.2 / 65.3
//   launches that fetch ahead, and those of 1 and 2 packets, are held to 4 where others are held to 5 (as many as fit: 5 or 4, for 1 and 2 packets 6 or 7).  60 M
//   elements: SGD    300, 1 154.2 / 150.0 / 151.3; 500, 1 156.3 / 154.4 / 152.1, 8 154.5 / 154.7 / 152.7, 16 155.5 / 155.8 / 156.0; 700, 1 170.1 / 161.2 / 160.8, 4 167.8 / 161.0 / 158.9; 3000, 1
//          182.9 / 172.3 / 168.1, 8 163.6 / 163.3 / 160.1; 9000, 4 172.1 / 164.9 / 160.7; 125 M, 500, 4 332 / 339 / 334, 8 326 / 326 / 319
//          Adam   500, 1 243.0 / 239.2 / 236.7, 4 243.0 / 243.0 / 239.5, 8 238.3 / 238.1 / 237.8; 3000, 4 258.4 / 258.7 / 252.1; 125 M, 500, 1 521 / 512 / 500, 4 520 / 520 / 508, 16 498 / 502 / 498
//   others, not held by the lines of tiles and bins: SGD 700, 8 170.5 / 168.0 / 164.5; Adam 300, 8 244.9 / 237.8 / 240.0, 700, 8 263.5 / 263.9 / 257.3
constexpr uint32_t kResidentLds[2] = {32000, 40900};   // bytes of LDS that leave five, four workgroups on a compute unit
constexpr uint64_t kResidentElems = 11600000, kResidentElemsSum = 23200000, kResidentElemsSumMany = 32000000;   // from which on: with the optimizer; sums of up to 4 packets; of more
constexpr uint64_t kHoldSum8Elems = 18000000;   // elements of layers with 8-bit words from which on sums of one or two packets over nothing else are held (unpack_hold_sum8_alone)
constexpr uint64_t kEarlyElems = 1500000;   // elements of a launch from which on the optimizer's state is fetched ahead of the adds (unpack_early_for)
// Groups up to which a plain sum of few packets waits for all packets' records together (k_unpack_few).  Together / not, in us: 4 packets, L_T 500, 2 M elements
// 4.46 / 4.58, 4 M (1000 groups) 5.67 / 5.79, 8 M 7.89 / 7.87, 25 M 22.8 / 22.5; 100, 4 M 7.65 / 7.64; 1 M, L_T 50, and 1.5 M, 500 6.34 / 6.47; 2.4 M and 3.6 M (1670) 9.17 / 8.30, 6.4 M and
// 9.6 M 17.9 / 17.4.
constexpr uint32_t kFewTilesTogether = 1024;
constexpr uint32_t kUnpackTaperTiles = 768;  // tiles at the end of the table that go alone (3 per compute unit)

// What k_fused leaves per tile for k_scan and k_place: one 16-byte record, so that a tile makes one
// small store here instead of three.
struct TileOut {
    double gmax_sum;  // sum of the tile's g_max values
    uint32_t count;   // words the tile sends
    uint32_t base;    // words of the layer before this tile (written by k_scan); after a lazy call the bits of the layer's scale
};
static_assert(sizeof(TileOut) == 16, "TileOut layout");

// Byte offsets inside the caller's workspace.  The tables come first; then one scratch block per
// learner of a batched call (a single-learner call uses block 0).
struct WorkspaceLayout {
    size_t layers = 0, ctiles = 0, cclass = 0, utiles = 0, ugroups = 0, usingles = 0;  // tables written by workspace_init
    size_t scratch = 0;                                 // first scratch block
    size_t scratch_stride = 0;                          // bytes per learner
    // offsets inside a scratch block
    size_t tile_out = 0;                                // TileOut per compress tile
    size_t layer_nsel = 0, layer_scale = 0;             // per layer
    size_t gmax = 0, chunk_rel = 0;                     // per bin / per chunk
    size_t stage = 0;                                   // uint16 per element of the layers (not of the address span): words before placement
    // The exchange areas of the one-launch compress, one per learner of a launch, lie at the end of the
    // workspace (SyncPlace); offsets inside one.  A workspace without room for them takes the staged launches.
    size_t sync_rec = 0, sync_tile = 0, sync_layer = 0, sync_epoch = 0;
    size_t sync_stride = 0;
    size_t least(size_t n_learners) const { return scratch + scratch_stride * n_learners; }   // what a call needs
    // and exchange areas for a launch of as many learners, as far as those take less than one more learner's block
    size_t total(size_t n_learners) const
    {
        const size_t most = (scratch_stride - 1) / sync_stride, n = n_learners < kMaxBatch ? n_learners : kMaxBatch;
        return least(n_learners) + sync_stride * (n < most ? n : most);
    }
};

// Where a registered workspace keeps its exchange areas: `learners` of them, which a call's launches use one
// after the other.  They are cleared when the workspace is initialised and from then on belong to the kernels,
// also to those of captured calls that are replayed any time later: so they begin behind the scratch block of
// the last learner that any call on this workspace could have.  In workspace_bytes_batch(n) bytes that is learner
// n.  An area takes 52 bytes per compress tile (packed to 44, which one of the two forms makes do with, and
// without sections on lines of their own, calls took 0.8 % longer over 41 tables), a scratch block 2 per element and some: areas for 32 learners fit in
// less than a block where tiles have a thousand elements and are not few, for 16 where they have 400.  Calls of
// more learners take the staged launches there (30 k elements in 14 layers, 32 learners: 15.7 us, one launch
// 14.1, two of 16 learners each 23.5).
struct SyncPlace {
    size_t offset = 0, learners = 0;
};
SyncPlace sync_place(const WorkspaceLayout &ws, size_t workspace_bytes, size_t most_learners);

// A tile's workgroup of a one-launch call takes the count of the calls before it, plus one, as its epoch and
// counts itself at the end of its exchange, wherever it stands then.  Stored instead, the epoch would fall
// behind that of other tiles for good when two calls overlap on one workspace (which is refused by contract, and
// spoils both): every later call would wait in vain.
__host__ __device__ inline void count_call(uint32_t *calls)
{
#ifdef __HIP_DEVICE_COMPILE__
    (void)__hip_atomic_fetch_add(calls, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#else
    (void)__atomic_fetch_add(calls, 1u, __ATOMIC_RELAXED);
#endif
}

// Polls (0.4 us each) before a workgroup works out what it waits for; in a call that has the GPU for itself waits
// are 10 to 20 us long.  Captured on the whole GPU, replayed on 64 / 32 compute units, in us, by 64, 256 and 4096
// polls: ResNet-50's table 820, 1060, 7700 / 1430, 2090, 15400; one layer of 1000 tiles 196, 263, 1590 / 275, 346, 1680.
constexpr uint32_t kWaitPolls = 256;
constexpr uint32_t kWaitPollsKnown = 4096;   // polls for what this workgroup has published itself
constexpr uint32_t kWaitPollsMax = 1u << 16;   // of adacomp_debug_wait_polls

struct Plan {
    uint32_t n_layers = 0;
    uint32_t n_ctiles = 0, n_utiles = 0, n_ugroups = 0;
    uint32_t n_ugroups8 = 0, n_usingles8 = 0;  // groups of layers with 8-bit words: they come first in both tables
    uint32_t crowd_tiles = 0;   // compress tiles, for the lines between staged and one-launch calls of many workgroups (kOneLaunchCrowd*): as
                                // many as a table makes before build_plan rounds them down to the compute units, with which the lines were measured
    uint32_t n_bins_total = 0, n_chunks_total = 0;
    uint64_t n_elems16 = 0, n_bins16 = 0;   // of the layers with 16-bit words
    uint64_t elem_span = 0;     // max over layers of elem_offset + n_elems
    uint64_t n_elems_total = 0;
    uint64_t n_elems8_lines = 0;  // of the layers with 8-bit words that begin on a line of 128 bytes: all of their tiles do then
    uint64_t stage_entries = 0; // entries of the staging array: sum over the compress tiles of their element counts rounded up to 4
    uint64_t fixed_bytes = 0;   // packet bytes before the first word
    uint64_t bound_bytes = 0;   // packet bytes with every element sent
    uint32_t n_class_tiles[2] = {0, 0};  // compress tiles of 4096 / of 16384 elements
    std::vector<uint32_t> cclass;        // compress tile indices, the 4096-element ones first (tables with both kinds)
    bool has_short_bins = false;  // some layer has L_T <= 64 (8-bit words, many words per tile)
    uint32_t layer_tiles_max = 0;  // compress tiles of the layer that has most
    uint32_t short_bin_max = 0;    // longest L_T <= 64
    bool has_tiny_bins = false;    // some layer has L_T < 4
    bool groups_single = false;    // the groups of the plain sum are single tiles too (of a plan with tables)
    bool has_shifted_tiles = false;  // some tile of the larger class has skip != 0
    WorkspaceLayout ws;
    SyncPlace sync;   // of a registered workspace
    uint32_t wait_polls = kWaitPolls;
    std::vector<LayerDev> layers;
    std::vector<TileDev> ctiles;
    std::vector<UTileDev> utiles;
    std::vector<UGroupDev> ugroups, usingles;
};

// Validates the table (ADACOMP_E* on failure) and, with tables = true, fills the tile tables.
int build_plan(const adacomp_layer_t *layers, uint32_t n_layers, bool tables, Plan &plan);
uint32_t bin_magic(uint32_t L_T);
// Host bookkeeping of adacomp_workspace_init (which workspace holds the tile tables of which layer
// table) and the look-up every compute call starts with: ADACOMP_EWORKSPACE unless `workspace` was
// registered for exactly this list of layers and is large enough for n_learners scratch blocks.
void register_workspace(const adacomp_layer_t *layers, uint32_t n_layers, const void *workspace, size_t workspace_bytes,
                        Plan &&plan);
int find_plan(const adacomp_layer_t *layers, uint32_t n_layers, const void *workspace, size_t workspace_bytes,
              size_t n_learners, Plan &out);

// ---- kernel launchers (adacomp_kernels.hip) ---------------------------------------------------
constexpr uint64_t kSplitElems = 32u * 1000u * 1000u;  // gradients at least this long: one k_fused launch per learner

// Dynamic LDS that no kernel touches, asked for with the launches of the eager 256-thread streaming
// kernel in calls that launch it once per learner, for many learners: with its 8.5 KB of arrays that leaves room for 6 workgroups per
// compute unit instead of the 8 its registers allow.  The kernel is bound by HBM, and HBM serves it
// better with fewer bytes in flight (a bare triad of the same shape gains up to 7 % between 8 and 4
// resident workgroups); since the layer record is fetched at the start of a workgroup and not in its
// tail, 6 workgroups still cover the LDS phases.  Measured per learner of the 125 M-element table,
// uncapped / capped: 235.5 / 247.9 us in calls of 1 learner, 243.3 / 251.2 of 2, 240.2 / 245.9 of 4,
// 242.1 / 239.0 of 8, 242.4 / 237.3 of 12, 243.8 / 238.0 of 16: a launch that follows another
// streaming launch gains, one that follows a placement and an unpack loses, hence the learner count.
// The kernel that first applies waiting corrections is longer per tile and loses with any cap.
constexpr uint32_t kFusedIdleLds = 18000;
constexpr uint32_t kFusedIdleMinLearners = 8;

// How adacomp_compress covers a table in one launch (see k_pack): not at all, with every workgroup
// reading the records of the whole table, or with one workgroup per layer doing so.
constexpr uint32_t kOneLaunchNever = 0, kOneLaunchTable = 1, kOneLaunchLayers = 2;
// Tiles of a layer up to which its workgroups wait for each other: 2048 are resident, and the longer a
// layer, the longer its first tiles hold their place.  Three launches / one, in us, one layer: L_T 50, 1000 tiles, 1 learner
// 29.3 / 19.5, 8 learners 119 / 94; L_T 500, 525 tiles, 2 learners 23.1 / 14.7, 8 50 / 41; 625 tiles, 4 35 / 28; 1000 tiles, 2
// 30.9 / 20.0, 4 47.9 / 39.5, 8 81 / 78; the character LSTM, 8 learners with unpack 73.4 / 70.3.  Where little is sent the
// placement that one launch saves is cheap, and the gain shrinks with the rounds of resident workgroups: without short bins
// half as many tiles from more than four rounds on.
constexpr size_t kOneLaunchRounds = 4;
constexpr uint32_t kOneLaunchTiles = 1024;
constexpr uint32_t kOneLaunchTilesLong = 512;
// ... and per compute unit that the stream may use, half of what is resident there: workgroups of a layer that
// does not fit wait for others that cannot start until they work those out themselves.  Streams masked to 64 and
// 32 units, one launch (before there was this line) / three, in us: ResNet-50's table (layers of up to 583
// tiles) 21400 / 243 and 62000 / 450, the character LSTM's 2060 / 43 and 11300 / 66.
constexpr uint32_t kOneLaunchTilesPerUnit = 4;
// Calls with more workgroups than are resident (8 per compute unit): the form in which every workgroup reads
// all records is for latency, and costs more than it saves there; with a quarter as many again and small tiles
// neither form pays, but where staged calls of tables with short bins take three launches.  Staged / all records / per layer, in us: 6 layers, L_T 50 and 500, 16 learners: 227 k elements
// (1000 a tile) 24.9 / 24.4 / 25.6, 14 layers 26.8 / 31.8 / 26.9; 500 k (1900) 37.7 / 49.2 / 34.0; 1.5 M 80 / 87 / 57.
// L_T 500, 32 learners: 500 k 59.5 / 96.8 / 65.0, 943 k (3500) 82 / 121 / 71; L_T 3608, 8 learners, 1.5 M 36 / 48 / 33;
// 20 layers, L_T 2240, 1.1 M (2200 a tile), 4 learners (2060 workgroups) 24.9 / - / 21.0; 20 layers, L_T 50 and
// 500, 227 k, 16 learners 31.9 / - / 29.0, but L_T 500 alone, 14 learners 24.9 / - / 26.7, 12 (2800 workgroups), 14
// layers 21.8 / - / 23.0.
constexpr uint32_t kOneLaunchCrowdElems = 1536, kOneLaunchCrowdElemsLong = 2048;   // elements per tile from which on one launch pays
// Tables with bins of the larger tile class have all layers in tiles of that class (build_plan), if none takes more of
// them than there are compute units (two workgroups are resident on each).  Three staged launches or more (one over
// each class) / one, in us: 4 M elements, L_T 50 and 9000, 1 learner 36.5 / 19.7, 16 with unpack 242 / 201; 9 M, 1 learner 51 /
// 30; 20 M in 40 layers, 50 and 7000 86 / 60; 8 M, 64 and 1501, another rule 55 / 31.  Without short bins the staged
// calls are the shorter ones from 3 workgroups per unit on: L_T 5000, 2 M, 4 learners (536 workgroups) 36.8 / 34.2, 16
// 88 / 96; 5 M, 4 learners 64 / 70; L_T 12001, 300 k, 16 learners (480) 31.7 / 22.8, 5 M, 4 63 / 70.
constexpr uint32_t kOneLaunchTilesLarge = 256;
// ... nor does one launch pay with many workgroups whose tiles are half empty, since one bin fills little more than half
// of them: a workgroup holds its place for all that a full one waits, and loads less in that time.  Staged / one launch
// / staged over tiles of both classes, in us: L_T 50 and 9000, 80 % of the elements in long bins (9900 to a tile), 10 M, 1
// learner 54 / 38 / 48, 2 (2022 workgroups) 79 / 68 / 72, 4 130 / 129 / 122, 8 247 / 258 / 240; 20 M, 2 127 / 133 / 122; 4 M, 16 176 /
// 196 / 183; 95 %, 20 M, 1 (2170) 76 / 70 / 70, 4 234 / 264 / 230; L_T 8200, 95 %, 4 242 / 283 / 239; but 60 % (11000 to a tile), 10 M, 8
// 270 / 249 / 249, L_T 11000, 80 %, 8 240 / 230 / 232.
constexpr uint32_t kOneLaunchLargeFill = 10000, kOneLaunchLargePerUnit = 12;   // elements per tile below which, workgroups per unit beyond which
// Lazy calls save the placement's pass over the residue in either form, so that one launch pays by what it does without
// launches and staged words, not by bytes: up to as many elements in all, and with small tiles up to the 6 workgroups
// that its registers leave on a compute unit.  Staged / one launch, in us: 100 k elements, L_T 50 and 500, 1 learner 13.4 /
// 8.3, 16 with unpack (1700 workgroups of 1000) 32.2 / 34.3; 1.2 M, 1 16.4 / 11.2, 16 71 / 70; 4 M, 4 58 / 50, 16 164 / 170;
// 12 M, 1 40.5 / 33.9, 2 63.4 / 63.0, 4 129 / 140; ResNet-50's table, 1 66.8 / 66.2, 8 415 / 475.
constexpr uint64_t kLazyOneLaunchElems = 24u * 1000u * 1000u;
// ... and half as many where tiles of the larger class are a third empty or more.  Staged / one launch / staged over tiles of
// both classes: L_T 50 and 9000, 60 % of the elements in long bins (11000 to a tile), 4 M in all 27.8 / 20.8 / 31.7, 8 M 40.0 / 35.9 /
// 40.9, 10 M, 1 learner 46.4 / 44.9 / 45.4, 2 42.0 / 38.2 / 45.7, 16 M 58.5 / 62.2 / 62.3, 20 M, 1 71.2 / 78.6 / 73.8, 2 70.9 / 81.3 /
// 73.6, 4 66.5 / 74.1 / 73.6; but 20 % (14000 to a tile), 20 M 68 / 66 / 71, L_T 5000 (15000) 68 / 63 / 72.
constexpr uint32_t kLazyLargeFill = 12288;   // elements per tile
// Every tile looks at every layer before its own: 300 layers, 8 M elements, 4 learners 86 / 120.
constexpr uint32_t kOneLaunchLayersMax = 512;

// A tile by 512 threads instead of 256, up to as many workgroups as leave two to a compute unit: the phases of a
// workgroup that has a unit to itself are chains of dependent instructions, half as long with half as many slots
// to a thread.  256 / 512 threads, in us: 32 workgroups 7.2 / 6.7, 205 8.3 / 7.5, 488 (8 learners) 8.8 / 8.3, 596 10.4
// / 10.4, and 1192, of which 1024 are resident with 512 threads, 13.4 / 17.9.
constexpr uint32_t kPackWidePerUnit = 2;

// k_pack takes whole rows of 16-byte slots, its threads times four elements each, as far as the tile has elements in
// them.  `bin` is what the index of a slot's first element gives; the slots past the tile would lie in bins that it has
// not (5120 elements in 1024 bins of five: the second row of 1024 threads ends in bin 1637), so the larger class takes
// them for bin n_bins, which has an entry of its own and no elements.  They send nothing.  In the smaller class 4096
// elements in bins of four or more are 1024 bins at most, with nothing to look at.
constexpr uint32_t kPackBins = kMaxTileBins + 4u;   // entries of k_pack's arrays of bins: of a slot, its bin and the one after
template <bool LARGE>
__host__ __device__ inline uint32_t pack_bin(const uint32_t bin, const uint32_t n_bins)
{
    return LARGE && bin > n_bins ? n_bins : bin;
}

struct CompressArgs {
    const TileDev *tiles;
    const LayerDev *layers;
    uint8_t *scratch;         // scratch block of learner 0 of this launch
    uint64_t scratch_stride;
    uint8_t *sync;            // exchange area of learner 0 of this launch (one-launch calls)
    uint64_t sync_stride;
    uint32_t o_sync_rec, o_sync_tile, o_sync_layer, o_sync_epoch;
    uint32_t one_launch, wait_polls;    // kOneLaunch*; polls before a waiting workgroup helps itself
    uint32_t o_tile_out, o_layer_nsel, o_layer_scale, o_gmax, o_chunk_rel;
    uint32_t n_tiles, n_layers, n_learners, keep_gmax;
    uint32_t fused_first, fused_count;  // learners covered by one k_fused launch
    const uint32_t *class_tiles;        // tile indices by register class, or null: the launch covers tiles 0 .. class_count - 1
    uint32_t class_first, class_count;  // this launch's stretch of class_tiles
    uint32_t place_lanes;               // lanes per tile in k_place: 16 or 64
    uint32_t place_mode;                // kPlaceEager / kPlaceWords / kPlaceResidue
    uint32_t fold_scan;                 // no k_scan launch: k_place computes word offsets and layer scales itself
    uint32_t place_tiled;               // the placement is k_place_tiled: one workgroup per tile, residue corrected line by line
    uint32_t lazy;                      // k_fused applies the waiting residue corrections of the previous call
    uint32_t shift;                     // the launch over the larger tiles uses the kernel that honours TileDev::skip
    uint32_t fused_idle_lds;            // bytes of dynamic LDS for the eager 256-thread k_fused launches (kFusedIdleLds or 0)
    uint32_t rule;                      // ADACOMP_RULE_*
    uint32_t pack_wide;                 // one_launch == kOneLaunchTable: 512 threads to a tile instead of 256
    float soft_factor_minus_1;          // 1 for the paper's factor 2
    uint64_t o_stage;
    uint64_t capacity;        // bytes available in each packet buffer
    uint64_t fixed_bytes;
    const float *grad[kMaxBatch];
    float *residue[kMaxBatch];
    uint8_t *packet[kMaxBatch];
};

// A launch whose kernel arguments take 1224 bytes, these and the 256 hidden ones that gridDim, blockDim or
// __syncthreads_or bring along, waits 100 us or more on the host when hundreds of other launches went
// before it (968, and 1184, do not): the kernels do without the hidden ones.
static_assert(sizeof(CompressArgs) <= 1024, "kernel arguments");

// What an unpack kernel has behind its three scalar arguments (the tiles' records, the table of groups, null: a tile each, single_tile,
// and the number of groups, kind 3: of the layers with 16-bit words), which take 24 bytes.
struct UnpackHead {
    float *dense;
    uint32_t n_groups8;                // kind 3: groups of the layers with 8-bit words, a chunk each, the first of the table
    uint32_t n_layers, n_learners, accumulate;
    uint32_t write_dense;              // 0: the sum is only consumed by the update
    uint32_t mode;                     // 0: sum only; 1: SGD with momentum; 2: Adam (applied by this launch)
    float *weights, *state1, *state2;  // momentum buffer, or Adam's m and v
    float n_average;                   // learner count the sum is divided by
    float lr, p1, p2, one_minus_p1, one_minus_p2, eps, bias1, bias2;
    uint32_t chunk_lds;                // kind 3: floats of LDS per chunk, 64 times the longest of the 8-bit layers' bins, + log2 of the chunks per workgroup
    uint32_t first16;                  // kind 3: where in the table the groups of the layers with 16-bit words begin
};
// With N packets: a kernel takes no more of them than it can have.  Small sums are bound by what a launch costs the host, which
// goes by its arguments too: 144 bytes of them for 1 and 2 packets, 640 for 64.  256 and 704, with this structure aligned to 64 bytes and
// the scalar arguments in it a second time / as it is, in us: 0.4 M elements, L_T 50, and 0.6 M, 500, 2 packets 4.64 / 4.46, 4 5.88 /
// 5.68; 4 M and 4 M, 1 packet 7.70 / 7.50, SGD with 2 23.65 / 22.52.  k_unpack8 for two packets had 66 vector registers instead of 32.
template <uint32_t N>
struct UnpackPackets : UnpackHead {
    const uint8_t *packets[N];
};
// What the host fills.
struct UnpackArgs : UnpackPackets<kMaxPacketArgs> {
    const UTileDev *tiles;
    const UGroupDev *groups;
    uint32_t n_groups;                 // workgroups that take a group each
};
// Workgroups start with the scalar loads of these arguments, and the first of a launch wait for every line
// of them.  With 16 bytes more before `packets`, whose lines then no longer began with it, k_unpack took
// 1.5 to 2 % longer (4 M elements, 4 packets 8.85 -> 9.04 us; 20 M, 8 packets 31.5 -> 32.1).
static_assert(24 + sizeof(UnpackHead) == 128 && alignof(UnpackHead) == 8, "a line of kernel arguments ends where the packets begin");
static_assert(sizeof(UnpackPackets<2>) == sizeof(UnpackHead) + 16 && sizeof(UnpackPackets<4>) == sizeof(UnpackHead) + 32 &&
              sizeof(UnpackPackets<8>) == sizeof(UnpackHead) + 64, "kernel arguments end with the last packet");

uint32_t one_launch_for(const Plan &p, size_t n_learners, size_t workspace_bytes, uint32_t compute_units, bool lazy = false);
bool pack_wide_for(const Plan &p, size_t n_learners, uint32_t compute_units);
uint32_t place_lanes_for(const Plan &p);
uint32_t resident_for(uint64_t n_elems, uint64_t n_bins, uint64_t n_tiles, uint32_t n_learners, uint32_t mode);
uint32_t unpack_hold_sum8_alone(uint64_t elems8, uint64_t tiles8, bool on_lines, uint32_t n_learners);
uint32_t unpack_hold_sum8(uint64_t elems8, uint64_t tiles8, uint64_t elems16, uint64_t bins16, uint32_t n_learners);
bool unpack_early_for(uint64_t n_elems, uint64_t n_bins, uint64_t n_tiles, bool words8, uint32_t n_learners, uint32_t mode);
uint32_t unpack8_wg_log(const Plan &p, uint32_t n_chunks, uint32_t n_groups16, uint32_t n_learners);
int launch_fused(const CompressArgs &a, int jcode, void *stream);
int launch_scan(const CompressArgs &a, void *stream);
int launch_place(const CompressArgs &a, void *stream);
// what a k_place launch does: everything (the default); the words, offsets and header only, leaving
// the residue corrections waiting; or those corrections only
constexpr uint32_t kPlaceEager = 0, kPlaceWords = 1, kPlaceResidue = 2;
int launch_unpack(const UnpackArgs &a, int kind, uint32_t resident, bool early, void *stream);  // kind 0: 16-bit words, 1: 8-bit, 2: both, 3: both, k_unpack8
int launch_copy(float *dst, const float *src, size_t n, void *stream);
int launch_triad(float *x, const float *y, size_t n, uint32_t resident, void *stream);   // n a multiple of 4, below 2^44; resident 3 .. 8
int launch_fill(float *x, float value, size_t n, void *stream);

}  // namespace adacomp
