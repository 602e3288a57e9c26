// adacomp_api.hip -- the C ABI of libadacomp: argument checks, the plan (tile tables and
// workspace layout) and the launch sequences.  No arithmetic of the method lives here.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <unordered_map>

#include "adacomp_debug.h"
#include "adacomp_plan.h"

namespace adacomp {

static uint64_t pad16(uint64_t x) { return (x + 15u) & ~uint64_t(15); }
static size_t pad256(size_t x) { return (x + 255u) & ~size_t(255); }
static uint32_t gcd_u32(uint32_t a, uint32_t b) { while (b) { uint32_t t = a % b; a = b; b = t; } return a; }

uint32_t bin_magic(uint32_t L_T)
{
    // floor(2^32 / L_T) + 1; exact for every index below 2^32 / L_T >= 2^18 (see the self-test).
    // L_T == 1 would need 2^32 + 1: the kernels special-case it (bin == index).
    return L_T <= 1 ? 0u : uint32_t((uint64_t(1) << 32) / L_T) + 1u;
}

static int validate(const adacomp_layer_t *layers, uint32_t n_layers)
{
    if (!layers || n_layers == 0 || n_layers >= (1u << 24)) return ADACOMP_EINVAL;
    for (uint32_t l = 0; l < n_layers; ++l) {
        if (layers[l].n_elems == 0 || layers[l].n_elems >= (uint64_t(1) << 31)) return ADACOMP_EINVAL;
        if (layers[l].L_T == 0 || layers[l].L_T > ADACOMP_LT_MAX) return ADACOMP_EBADLT;
        if (layers[l].elem_offset % 4 != 0) return ADACOMP_EALIGN;
        if (layers[l].elem_offset + layers[l].n_elems < layers[l].elem_offset) return ADACOMP_EINVAL;
    }
    // overlap check: sort-free O(n^2) is fine for a few hundred layers; use a sorted copy beyond that
    if (n_layers <= 512) {
        for (uint32_t l = 0; l < n_layers; ++l)
            for (uint32_t m = 0; m < l; ++m) {
                uint64_t a0 = layers[l].elem_offset, a1 = a0 + layers[l].n_elems;
                uint64_t b0 = layers[m].elem_offset, b1 = b0 + layers[m].n_elems;
                if (a0 < b1 && b0 < a1) return ADACOMP_EINVAL;
            }
    } else {
        std::vector<std::pair<uint64_t, uint64_t>> iv(n_layers);
        for (uint32_t l = 0; l < n_layers; ++l) iv[l] = {layers[l].elem_offset, layers[l].elem_offset + layers[l].n_elems};
        std::sort(iv.begin(), iv.end());
        for (uint32_t l = 1; l < n_layers; ++l)
            if (iv[l].first < iv[l - 1].second) return ADACOMP_EINVAL;
    }
    return ADACOMP_OK;
}

// process-wide tuning and diagnostic flags (adacomp_debug.h): atomics, so that a compute call on one
// thread reads a whole value while another thread sets it; no ordering beyond that is promised
static std::atomic<uint32_t> g_unpack_min_groups{kUnpackMinGroups};
static std::atomic<bool> g_fold_scan{true};
static std::atomic<bool> g_place_tiled{true};

int build_plan(const adacomp_layer_t *layers, uint32_t n_layers, bool tables, Plan &p)
{
    int rc = validate(layers, n_layers);
    if (rc != ADACOMP_OK) return rc;
    p = Plan();
    p.n_layers = n_layers;
    p.layers.resize(n_layers);

    uint64_t fixed = sizeof(adacomp_packet_header_t) + uint64_t(sizeof(adacomp_packet_layer_t)) * n_layers;
    uint64_t words_bound = 0;
    uint64_t n_ctiles = 0, n_utiles = 0, bins_total = 0, chunks_total = 0;

    // A table that makes fewer tiles of 4096 elements than there are compute units cannot fill the GPU,
    // and the time of a launch is then the time of one tile: such tables get smaller tiles, down to
    // 1024 elements (the 397 k-element table: 97 tiles become 265, 23 -> 19 us per compress call).
    uint64_t elems_all = 0;
    for (uint32_t l = 0; l < n_layers; ++l) elems_all += layers[l].n_elems;
    uint32_t small_cap = uint32_t(std::min<uint64_t>(4096u, std::max<uint64_t>(1024u, elems_all / kComputeUnits)));
    // ... and, where a somewhat larger tile does it, as many as there are compute units, less the one for the header:
    // a few more share units with others (397 k elements, 266 tiles of 1500 / 199 of 2000: 7.8 / 6.6 us; 600 k, 9.2 / 7.5; 1.02 M, 263 of
    // 3900 / 255 of 4000: 8.35 / 7.25, 4 learners with unpack 22.5 / 22.1).
    uint64_t tiles_before = 0;
    for (uint32_t cap = small_cap;; cap = std::min(cap + cap / 16u, 4096u)) {
        uint64_t tiles = 0;
        for (uint32_t l = 0; l < n_layers; ++l) {
            const uint64_t bins = (layers[l].n_elems + layers[l].L_T - 1u) / layers[l].L_T;
            const uint64_t a = 4u / gcd_u32(layers[l].L_T, 4u);
            uint64_t bpt = std::min<uint64_t>(std::max<uint64_t>(cap / layers[l].L_T, 1u), kMaxTileBins);
            if (bpt < a) bpt = a;
            tiles += (bins + bpt / a * a - 1u) / (bpt / a * a);
        }
        if (tiles_before == 0) tiles_before = tiles;
        if (tiles < kComputeUnits) { small_cap = cap; break; }
        if (cap >= 4096u) break;
    }

    // Tables with layers of the larger tile class that can go in one launch (one_launch_for) have all their layers in
    // tiles of that class: up to a million elements smaller ones, so that there are some.  A 256th / 128th / 64th of
    // the elements to a tile, in us: 1.2 M elements, L_T 800 and 8000, 1 learner 10.1 / 10.4 / 11.1, 4 learners with unpack
    // 27.6 / 27.6 / 21.7; 1 M, 50 and 9000, 1 learner 10.6 / 10.0 / 11.9, 4 33.0 / 31.0 / 25.7, 16 108 / 75 / 68; 2 M, 5000, 1 learner
    // 13.4 / 12.1 / 12.1, 4 50 / 34 / 34 (in staged launches over tiles of both classes 24, 35, 24, 42, 87, 18 and 37).
    auto large_class = [](uint32_t T) { const uint64_t a = 4u / gcd_u32(T, 4u); return T > 4096u || (a * T > 4096u && a * T <= 16384u); };
    const uint32_t large_cap = uint32_t(std::min<uint64_t>(16384u, std::max<uint64_t>(4096u, elems_all / 64u)));
    bool all_large = false, fits = n_layers <= kOneLaunchLayersMax, short_bins = false;
    uint64_t large_tiles = 0, long_elems = 0;   // tiles if all have that class; elements of the layers that need it
    for (uint32_t l = 0; l < n_layers && fits; ++l) {
        const uint32_t T = layers[l].L_T;
        const uint64_t a = 4u / gcd_u32(T, 4u), bpt = std::min<uint64_t>(std::max<uint64_t>(large_cap / T, 1u), kMaxTileBins);
        const uint64_t at_least = a * T <= 16384u ? (bpt < a ? a : bpt / a * a) : bpt;
        all_large = all_large || large_class(T);
        fits = T >= 4u && layers[l].n_elems <= at_least * T * kOneLaunchTilesLarge;
        short_bins = short_bins || T <= 64u;
        if (large_class(T)) long_elems += layers[l].n_elems;
        large_tiles += (layers[l].n_elems + at_least * T - 1u) / (at_least * T);
    }
    // Tables that are staged whoever calls, also one learner (one_launch_for), keep the smaller tiles for the bins that fit
    // them, unless the long bins hold two fifths of the elements and the others are not short: larger tiles save a launch over
    // one of the classes (7 us), smaller ones stream faster.  Smaller / larger, us: L_T 500 and 8000, a quarter in long bins,
    // 20 M, 4 learners 212 / 214, 16 869 / 914; 28 M, 1 85 / 83, 4 283 / 297, 8 578 / 610; 200, 4 310 / 342, 8 649 / 711; 60 M, 100, 1 189 / 201;
    // half: 20 M, 500, 1 69 / 63, 8 395 / 404; 40 M, 1 113 / 109, 8 1004 / 960; 200, 1 122 / 124, 4 495 / 499; three quarters: 40 M, 100, 1
    // 120 / 115, 4 484 / 464.  L_T 50, tiles half empty, 40 M, four fifths in bins of 9000, 1 learner 123 / 126, of 8200 126 / 131.
    const bool staged = short_bins ? large_tiles > kOneLaunchLargePerUnit * kComputeUnits && elems_all < large_tiles * kOneLaunchLargeFill
                                   : large_tiles > 3u * kComputeUnits;
    all_large = all_large && fits && (!staged || (!short_bins && 5u * long_elems >= 2u * elems_all));

    for (uint32_t l = 0; l < n_layers; ++l) {
        const uint32_t T = layers[l].L_T;
        const uint32_t n = uint32_t(layers[l].n_elems);
        const uint32_t n_bins = (n + T - 1) / T;
        const uint32_t n_chunks = (n_bins + ADACOMP_CHUNK_BINS - 1) / ADACOMP_CHUNK_BINS;
        const uint32_t wb = T <= 64 ? 1u : 2u;
        LayerDev &ld = p.layers[l];
        ld.elem_offset = layers[l].elem_offset;
        ld.n_elems = n; ld.L_T = T; ld.n_bins = n_bins; ld.word_bytes = wb; ld.n_chunks = n_chunks; ld.pad0 = 0;
        ld.counts_offset = fixed;
        ld.chunks_offset = fixed + pad16(uint64_t(n_bins) * wb);
        fixed = ld.chunks_offset + pad16(uint64_t(n_chunks) * 4);
        words_bound += pad16(uint64_t(n) * wb);
        ld.bin_start = uint32_t(bins_total);
        ld.chunk_start = uint32_t(chunks_total);
        bins_total += n_bins;
        if (wb == 2u) { p.n_elems16 += n; p.n_bins16 += n_bins; }
        else if (layers[l].elem_offset % 32u == 0u) p.n_elems8_lines += n;
        chunks_total += n_chunks;
        if (bins_total >= (uint64_t(1) << 32)) return ADACOMP_EINVAL;
        p.elem_span = std::max<uint64_t>(p.elem_span, layers[l].elem_offset + n);
        p.n_elems_total += n;

        // ---- compress tiles: whole bins, as many as fit the registers of a workgroup ------------
        // up to 4096 elements (256 threads with 16 each) unless a bin is longer: then up to 16384 (1024 threads).
        // With all_large every layer takes the larger class, those of short bins too: tiles of up to large_cap
        // elements, and of up to kMaxTileBins bins like the others, which with bins of fewer than 16 elements end
        // inside a row of the threads' slots (see pack_bin).  Tiles of 8192 elements streamed at less than half the rate of
        // either on MI355X (measured on a plain triad), so there is no class in between.
        // Tile starts are float4-aligned when a tile holds a multiple of a = 4 / gcd(L_T, 4) bins.  Bin
        // lengths that are odd (a = 4) or twice an odd number (a = 2) and too long for a such bins to fit
        // 4096 elements take the larger class when they fit there: unaligned tiles fall back to 4-byte
        // accesses, which stream at 44 % of the HBM peak instead of 71-77 %.
        const uint32_t a = 4u / gcd_u32(T, 4u);
        const int cls = (all_large || large_class(T)) ? 1 : 0;
        const uint32_t cap = cls ? 16384u : 4096u;
        uint32_t bpt = (all_large ? large_cap : cls ? cap : small_cap) / T;
        if (bpt == 0) bpt = 1;                        // a bin of up to cap elements always fits its class
        if (bpt > kMaxTileBins) bpt = kMaxTileBins;
        if (bpt < a && uint64_t(a) * T <= cap) bpt = a;
        if (bpt >= a) bpt -= bpt % a;
        const uint32_t nt = (n_bins + bpt - 1) / bpt;
        ld.ctile_start = uint32_t(n_ctiles);
        ld.n_ctiles = nt;
        p.n_class_tiles[cls] += nt;
        p.layer_tiles_max = std::max(p.layer_tiles_max, nt);
        if (T <= 64u) { p.has_short_bins = true; p.short_bin_max = std::max(p.short_bin_max, T); }
        if (T < 4u) p.has_tiny_bins = true;
        // The staging array is indexed by position in the tile table, not by address: a tile's stretch
        // starts where the stretches of the tiles before it end (each rounded up to 4 entries, which keeps
        // every stretch 8-byte aligned), so its size follows the element count whatever holes the table has.
        const uint64_t full_tile = uint64_t(bpt) * T, full_stretch = (full_tile + 3u) & ~uint64_t(3);
        if (tables) {
            for (uint32_t t = 0; t < nt; ++t) {
                TileDev td;
                const uint32_t first_bin = t * bpt;
                const uint64_t e0 = uint64_t(first_bin) * T;
                td.elem_base = layers[l].elem_offset + e0;
                td.stage_base = uint32_t(p.stage_entries + full_stretch * t);
                td.n_elems = uint16_t(std::min<uint64_t>(full_tile, n - e0));
                td.L_T = T;
                td.magic = bin_magic(T);
                td.n_bins = uint16_t((uint32_t(td.n_elems) + T - 1) / T);
                td.first_bin = first_bin;
                td.layer_flags = l | (uint32_t(cls) << 24) | ((e0 % 4 == 0) ? 0x80000000u : 0u);
                p.ctiles.push_back(td);
            }
        }
        // unaligned tiles of the larger class keep 16-byte accesses when the tile still fits with its
        // misalignment added (all but bins of 16382 or 16383 elements); independent of `tables`, so
        // that every plan of a table says the same
        if (cls == 1 && (uint64_t(bpt) * T) % 4 != 0) {
            for (uint32_t t = 0; t < nt; ++t) {
                const uint64_t e0 = uint64_t(t) * bpt * T;
                const uint32_t sk = uint32_t(e0 % 4), ne = uint32_t(std::min<uint64_t>(uint64_t(bpt) * T, n - e0));
                if (sk != 0 && ne + sk <= 16384u) {
                    p.has_shifted_tiles = true;
                    if (tables) p.ctiles[p.ctiles.size() - nt + t].layer_flags |= sk << 25;
                }
            }
        }
        p.stage_entries += full_stretch * (nt - 1) + ((n - full_tile * (nt - 1) + 3u) & ~uint64_t(3));
        if (p.stage_entries >= (uint64_t(1) << 32)) return ADACOMP_EINVAL;
        n_ctiles += nt;

        // ---- unpack tiles: a power-of-two number of bins inside one 64-bin chunk, or slices of
        //      one long bin --------------------------------------------------------------------
        const uint32_t glog = T <= 64 ? 3u : 4u;      // lanes that share a bin: 8 or 16
        if (T <= kUnpackTileElems) {
            uint32_t nb = 1;
            while (nb * 2 <= ADACOMP_CHUNK_BINS && uint64_t(nb) * 2 * T <= kUnpackTileElems) nb *= 2;
            const uint32_t nut = (n_bins + nb - 1) / nb;
            if (tables) {
                for (uint32_t t = 0; t < nut; ++t) {
                    UTileDev ut;
                    const uint32_t first_bin = t * nb;
                    const uint64_t e0 = uint64_t(first_bin) * T;
                    ut.elem_base = layers[l].elem_offset + e0;
                    ut.n_elems = uint16_t(std::min<uint64_t>(uint64_t(nb) * T, n - e0));
                    ut.L_T = uint16_t(T);
                    ut.n_bins = uint8_t((ut.n_elems + T - 1) / T);
                    ut.first_bin = first_bin;
                    ut.idx_lo = 0;
                    ut.chunk_bins = uint8_t(std::min<uint32_t>(ADACOMP_CHUNK_BINS, n_bins - (first_bin & ~(ADACOMP_CHUNK_BINS - 1u))));
                    ut.counts_offset = uint32_t(ld.counts_offset); ut.chunks_offset = uint32_t(ld.chunks_offset);
                    ut.layer_flags = l | (glog << 24) | ((e0 % 4 == 0) ? 0x80000000u : 0u);
                    p.utiles.push_back(ut);
                }
            }
            n_utiles += nut;
        } else {
            for (uint32_t b = 0; b < n_bins; ++b) {
                const uint64_t b0 = uint64_t(b) * T;
                const uint32_t blen = uint32_t(std::min<uint64_t>(T, n - b0));
                for (uint32_t lo = 0; lo < blen; lo += kUnpackTileElems) {
                    if (tables) {
                        UTileDev ut;
                        ut.elem_base = layers[l].elem_offset + b0 + lo;
                        ut.n_elems = uint16_t(std::min(kUnpackTileElems, blen - lo));
                        ut.L_T = uint16_t(T);
                        ut.n_bins = 1;
                        ut.first_bin = b;
                        ut.idx_lo = uint16_t(lo);
                        ut.chunk_bins = uint8_t(std::min<uint32_t>(ADACOMP_CHUNK_BINS, n_bins - (b & ~(ADACOMP_CHUNK_BINS - 1u))));
                        ut.counts_offset = uint32_t(ld.counts_offset); ut.chunks_offset = uint32_t(ld.chunks_offset);
                        ut.layer_flags = l | (glog << 24) | (((b0 + lo) % 4 == 0) ? 0x80000000u : 0u);
                        p.utiles.push_back(ut);
                    }
                    ++n_utiles;
                }
            }
        }
        if (n_ctiles >= (1u << 31) || n_utiles >= (1u << 31)) return ADACOMP_EINVAL;
    }
    p.n_ctiles = uint32_t(n_ctiles);
    p.crowd_tiles = all_large ? p.n_ctiles : std::max(p.n_ctiles, uint32_t(std::min<uint64_t>(tiles_before, UINT32_MAX)));
    p.n_utiles = uint32_t(n_utiles);
    if (tables && p.n_class_tiles[0] && p.n_class_tiles[1]) {
        // both tile sizes: each gets its own k_fused launch over its own tiles
        p.cclass.reserve(p.n_ctiles);
        for (uint32_t c = 0; c < 2u; ++c)
            for (uint32_t i = 0; i < p.n_ctiles; ++i)
                if (p.ctiles[i].jcode() == c) p.cclass.push_back(i);
    }
    if (tables) {
        // ---- unpack groups: runs of tiles that share phase 1 (same layer and 64-bin chunk, or the
        //      same long bin).  Longer runs save more table work but leave fewer workgroups, so the
        //      run length halves until at least kUnpackMinGroups workgroups remain.  Workgroups
        //      start in index order, so the runs get shorter towards the end of the table (the last
        //      kUnpackTaperTiles tiles go alone, twice as many before them in pairs, ...): the
        //      launch then ends with short workgroups instead of a few long stragglers. -----------
        uint32_t run = kUnpackGroupTiles;
        const uint32_t min_groups = g_unpack_min_groups.load(std::memory_order_relaxed);
        while (run > 1u && n_utiles / run < min_groups) run /= 2u;
        const uint32_t taper = kUnpackTaperTiles;
        const uint32_t run_max = run;
        for (uint32_t i = 0; i < p.n_utiles; ++i) {
            const UTileDev &ut = p.utiles[i];
            const uint32_t left = p.n_utiles - i;
            run = run_max;
            for (uint32_t r = 1u, span = taper; r < run_max; r *= 2u, span += taper * r)
                if (left <= span) { run = r; break; }
            bool fresh = p.ugroups.empty() || p.ugroups.back().n_tiles >= run;
            if (!fresh) {
                const UTileDev &first = p.utiles[p.ugroups.back().first_tile];
                fresh = first.layer() != ut.layer() ||
                        (ut.L_T <= kUnpackTileElems ? (first.first_bin >> 6) != (ut.first_bin >> 6) : first.first_bin != ut.first_bin);
            }
            if (fresh) p.ugroups.push_back(UGroupDev{i, 1u});
            else ++p.ugroups.back().n_tiles;
        }
        // Single tiles, for the launches that also apply the optimizer: those are bound by the
        // traffic of their epilogue, gain nothing from shared tables, and with runs of tiles they
        // were up to 15 % slower on some machines.
        p.usingles.resize(p.n_utiles);
        for (uint32_t i = 0; i < p.n_utiles; ++i) p.usingles[i] = UGroupDev{single_tile(i, p.n_utiles), 1u};
        p.groups_single = run_max == 1u;
        if (run_max == 1u) p.ugroups = p.usingles;
        // groups of 8-bit layers first: the two kinds go to different kernels
        auto is8 = [&p](const UGroupDev &g) { return p.utiles[g.first_tile].L_T <= 64u; };
        p.n_ugroups8 = uint32_t(std::stable_partition(p.ugroups.begin(), p.ugroups.end(), is8) - p.ugroups.begin());
        p.n_usingles8 = uint32_t(std::stable_partition(p.usingles.begin(), p.usingles.end(), is8) - p.usingles.begin());
        p.n_ugroups = uint32_t(p.ugroups.size());
    }
    p.n_bins_total = uint32_t(bins_total);
    p.n_chunks_total = uint32_t(chunks_total);
    p.fixed_bytes = fixed;
    p.bound_bytes = fixed + words_bound;
    if (p.bound_bytes >= (uint64_t(1) << 32)) return ADACOMP_EINVAL;  // word positions are 32-bit in k_unpack

    WorkspaceLayout &w = p.ws;
    size_t off = 256;  // first 256 bytes: reserved
    w.layers = off;      off = pad256(off + sizeof(LayerDev) * size_t(n_layers));
    w.ctiles = off;      off = pad256(off + sizeof(TileDev) * size_t(p.n_ctiles));
    w.cclass = off;      off = pad256(off + 4 * size_t(p.n_ctiles));
    w.utiles = off;      off = pad256(off + sizeof(UTileDev) * size_t(p.n_utiles));
    w.ugroups = off;     off = pad256(off + sizeof(UGroupDev) * size_t(p.n_utiles));  // at most one group per tile
    w.usingles = off;    off = pad256(off + sizeof(UGroupDev) * size_t(p.n_utiles));
    w.scratch = off;
    off = 0;             // offsets inside one learner's scratch block
    w.tile_out = off;    off = pad256(off + sizeof(TileOut) * size_t(p.n_ctiles));
    w.layer_nsel = off;  off = pad256(off + 4 * size_t(n_layers));
    w.layer_scale = off; off = pad256(off + 4 * size_t(n_layers));
    w.gmax = off;        off = pad256(off + 4 * size_t(p.n_bins_total));
    w.chunk_rel = off;   off = pad256(off + 4 * size_t(p.n_chunks_total));
    if (off >= (size_t(1) << 32)) return ADACOMP_EINVAL;
    w.stage = off;       off = pad256(off + 2 * size_t(p.stage_entries) + 128);  // slack: k_place reads up to 64 entries from a tile's start
    w.scratch_stride = off;
    off = 0;             // offsets inside one learner's exchange area
    w.sync_rec = off;    off = (off + 16 * size_t(p.n_ctiles) + 127u) & ~size_t(127);
    w.sync_tile = off;   off = (off + 32 * size_t(p.n_ctiles) + 127u) & ~size_t(127);
    w.sync_layer = off;  off = (off + 32 * size_t(n_layers) + 127u) & ~size_t(127);
    w.sync_epoch = off;  off = (off + 4 * (size_t(p.n_ctiles) + 1u) + 127u) & ~size_t(127);
    if (off >= (size_t(1) << 32)) return ADACOMP_EINVAL;
    w.sync_stride = off;
    return ADACOMP_OK;
}

SyncPlace sync_place(const WorkspaceLayout &ws, size_t workspace_bytes, size_t most_learners)
{
    SyncPlace at;
    const size_t end = workspace_bytes & ~size_t(127);
    if (end < ws.least(1)) return at;
    const size_t accepted = std::min((end - ws.scratch) / ws.scratch_stride, most_learners);   // by find_plan
    at.learners = std::min((end - ws.least(accepted)) / ws.sync_stride, size_t(kMaxBatch));
    at.offset = end - at.learners * ws.sync_stride;
    return at;
}

// Workspaces that adacomp_workspace_init has filled, by address.
// waiting: the residue buffers, by learner slot, whose corrections of the last lazy call have not
// been written yet (empty: none).  Kept at enqueue time, which is stream order for a workspace that
// one stream uses at a time.
struct Registered {
    Plan plan;
    size_t bytes = 0;
    std::vector<adacomp_layer_t> table;  // the layer table the tile tables in the workspace were built for
    std::vector<float *> waiting;
};

static bool same_table(const std::vector<adacomp_layer_t> &have, const adacomp_layer_t *layers, uint32_t n_layers)
{
    if (have.size() != n_layers) return false;
    for (uint32_t l = 0; l < n_layers; ++l)
        if (have[l].elem_offset != layers[l].elem_offset || have[l].n_elems != layers[l].n_elems ||
            have[l].L_T != layers[l].L_T)
            return false;
    return true;
}
static std::mutex g_mu;
static std::unordered_map<const void *, Registered> g_ws;

int find_plan(const adacomp_layer_t *layers, uint32_t n_layers, const void *workspace,
              size_t workspace_bytes, size_t n_learners, Plan &out)
{
    if (!layers || n_layers == 0 || !workspace) return ADACOMP_EINVAL;
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_ws.find(workspace);
    if (it == g_ws.end()) return ADACOMP_EWORKSPACE;
    const Plan &p = it->second.plan;
    // the kernels index the tile tables in the workspace without further checks: the table of this
    // call must be, entry by entry, the one those tables were built for
    if (!same_table(it->second.table, layers, n_layers)) return ADACOMP_EWORKSPACE;
    if (workspace_bytes < p.ws.least(n_learners) || it->second.bytes < p.ws.least(n_learners)) return ADACOMP_EWORKSPACE;
    // copy the scalars only; the tables already live on the device
    out.n_layers = p.n_layers; out.n_ctiles = p.n_ctiles; out.crowd_tiles = p.crowd_tiles; out.n_utiles = p.n_utiles; out.n_ugroups = p.n_ugroups; out.n_ugroups8 = p.n_ugroups8; out.n_usingles8 = p.n_usingles8;
    out.n_bins_total = p.n_bins_total; out.n_chunks_total = p.n_chunks_total;
    out.n_elems16 = p.n_elems16; out.n_bins16 = p.n_bins16; out.n_elems8_lines = p.n_elems8_lines;
    out.elem_span = p.elem_span; out.n_elems_total = p.n_elems_total; out.stage_entries = p.stage_entries;
    out.fixed_bytes = p.fixed_bytes; out.bound_bytes = p.bound_bytes;
    for (int c = 0; c < 2; ++c) out.n_class_tiles[c] = p.n_class_tiles[c];
    out.layer_tiles_max = p.layer_tiles_max; out.has_tiny_bins = p.has_tiny_bins; out.short_bin_max = p.short_bin_max;
    out.has_short_bins = p.has_short_bins; out.has_shifted_tiles = p.has_shifted_tiles; out.groups_single = p.groups_single;
    out.ws = p.ws;
    out.sync = p.sync;
    out.wait_polls = p.wait_polls;
    return ADACOMP_OK;
}

void register_workspace(const adacomp_layer_t *layers, uint32_t n_layers, const void *workspace, size_t workspace_bytes,
                        Plan &&plan)
{
    Registered reg;
    reg.plan = std::move(plan);
    Plan &p = reg.plan;
    // the host copies of the tile tables are not needed once they are on the device
    p.ctiles.clear(); p.ctiles.shrink_to_fit();
    p.cclass.clear(); p.cclass.shrink_to_fit();
    p.utiles.clear(); p.utiles.shrink_to_fit();
    p.ugroups.clear(); p.ugroups.shrink_to_fit();
    p.usingles.clear(); p.usingles.shrink_to_fit();
    reg.table.assign(layers, layers + n_layers);
    reg.bytes = workspace_bytes;
    std::lock_guard<std::mutex> lk(g_mu);
    g_ws[workspace] = std::move(reg);
}

// Workgroups per compute unit for launches over the 16-bit layers, by what those have (see kResidentLds); 0: as many as fit.
uint32_t resident_for(uint64_t n_elems, uint64_t n_bins, uint64_t n_tiles, uint32_t n_learners, uint32_t mode)
{
    auto tiles_of = [&](uint32_t at_least) { return n_elems >= at_least * n_tiles; };                    // elements
    auto bins_of = [&](uint32_t per_learner) { return n_elems >= per_learner * n_learners * n_bins; };   // elements, for every packet
    const bool few = n_learners <= 4u;
    if (mode == 2u) {
        if (n_elems < kResidentElems) return 0u;
        if ((tiles_of(3800u) && bins_of(60u)) || (tiles_of(2900u) && bins_of(300u))) return 4u;
        return tiles_of(few ? 2300u : 2900u) && bins_of(25u) ? 5u : 0u;
    }
    if (n_learners > 8u || !bins_of(mode == 1u ? 60u : 50u)) return 0u;
    if (mode == 1u) return n_elems >= kResidentElems && tiles_of(few ? 2700u : 2900u) ? 5u : 0u;
    if (few) return n_elems >= kResidentElemsSum && (tiles_of(2700u) || (tiles_of(2300u) && bins_of(70u))) ? 5u : 0u;
    return n_elems >= kResidentElemsSumMany && tiles_of(3800u) ? 5u : 0u;
}

// Does a launch with the optimizer's step ask for weights and moments when the words have been asked for, ahead of the adds
// (k_unpack's and k_unpack_few's EARLY), or behind the adds?  Ahead, they are on their way while the adds run, and take 32 or 48 registers
// through them, which leaves fewer workgroups: 7 instead of 8 with up to 4 packets (Adam 5 / 6), 4 or 5 instead of 6 or 7 with more.  That
// pays in full tiles with few words, and where there is work for all compute units.  Behind / ahead, in us:
//   1 and 2 packets: 0.4 M elements, L_T 500, SGD, 1 packet 5.9 / 5.9; 2 M, 50 6.7 / 5.7, 65 8.5 / 7.4, 500 6.8 / 6.6; 1.6 M, 20 5.5 / 5.7; 4 M, 65
//     12.3 / 12.7; 8 M, 20 22.4 / 23.7, 50 and 500, 2 packets 23.3 / 22.6; 13 M, 500 35.2 / 36.6.  With SGD the larger ones are ahead behind them, as far as bins are
//     short: 25 M, 16 68.1 / 72.0, 50 64.4 / 65.6, 100 64.5 / 66.8, 500 65.0 / 67.0; 60 M, 65 152.9 / 162.4, 500 153.9 / 161.5; 125 M, 500 323 / 340; 40 M, 1000
//     103.9 / 108.5, 1100 117.7 / 112.9, 1365 113.4 / 107.3, 2100 118.7 / 112.3, 4096 103.8 / 103.5, 5000 136.9 / 131.9.  With Adam: 25 M, 14 107.8 / 115.6, 20 100.8 / 102.4,
//     50 100.5 / 100.2, 65 100.9 / 104.7, 9000 112.2 / 109.4; 8 M, 50 and 500 36.9 / 36.0; 125 M, 500 502 / 496;
//   3 and 4: 2 M, 50 and 500, SGD, 4 9.3 / 8.6; 25 M, 500, 4 73.0 / 70.6, Adam 114.0 / 110.8; tiles of 2080 elements (L_T 65), Adam, 4 110.7 / 112.1; of 1280
//     (L_T 20, and 200), SGD, 4 85.1 / 80.2, Adam, 4 122 / 120, 60 M 286 / 287.  8-bit words, Adam: 2 M, 18, 3 14.7 / 13.6; 25 M, 18, 3 123.7 / 116.1, 4 124.4 / 125.9,
//     28, 3 103.7 / 100.2, 4 106.7 / 102.3; 60 M, 18, 3 289.6 / 276.5, 4 292.1 / 299.4; with 16-bit ones, 3: 20 M, 18, and 5 M, 65 122.6 / 117.0; 12 M, 20, and 13 M,
//     500 110.7 / 107.0, 65 110.0 / 108.1; 7 M, 20, and 18 M, 65 109.9 / 112.7;
//   8: 25 M, L_T 500 73.8 / 70.6, L_T 50 85.7 / 75.9, 65 76.1 / 80.4, 20 and 200 106 / 128; Adam 116.6 / 113.8, 123 / 114, 113 / 124, 152 / 165;
//   16: 25 M, 500 78.4 / 72.8, 250 75.7 / 74.3, 170 75.7 / 82.7, 100 83.6 / 95.6, 50 101 / 122; Adam 121 / 117, 118 / 114, 114 / 115, 121 /
//     130, 132 / 154; 24 packets, 10 M, 170 45.6 / 52.8.
// (words8: the launch's words, or of a launch over both widths and up to 8 packets those of a third of its elements, have 8 bits)
bool unpack_early_for(uint64_t n_elems, uint64_t n_bins, uint64_t n_tiles, bool words8, uint32_t n_learners, uint32_t mode)
{
    if (mode == 0u || n_elems < kEarlyElems) return false;
    if (n_learners <= 2u && mode == 1u) return n_elems < kResidentElems ? n_elems >= 1700u * n_tiles : n_elems >= 1050u * n_bins;
    if (n_learners <= 2u) return n_elems >= 2300u * n_tiles;
    if (n_learners <= 4u) return mode == 1u || words8 || n_elems >= 2300u * n_tiles;
    if (n_learners <= 8u) return n_elems >= 2900u * n_tiles;
    return n_learners <= 16u && !words8 && n_elems >= 2900u * n_tiles && n_elems >= 200u * n_bins;
}

// Is a launch of up to 4 packets with 8-bit words and the optimizer's step, whose kernels leave 5 or 6 workgroups to a compute unit, held to
// 4?  As many as fit / 4, in us: 25 M elements, L_T 50, SGD, 4 packets 71.8 / 70.3, Adam 111.5 / 109.1; 50 and 500 71.0 / 69.5,
// 111.0 / 109.3; 60 M, Adam 260 / 256, 260 / 256; tiles of 2080 elements, 25 M, SGD 70.7 / 78.3.
static bool unpack_hold_few(uint64_t n_elems, uint64_t n_tiles, uint32_t n_learners)
{
    return n_learners <= 4u && n_elems >= kResidentElems && n_elems >= 2900u * n_tiles;
}

// Plain sums of one or two packets over layers with 8-bit words and nothing else, in k_unpack_few: how many workgroups per compute unit they are
// held to.  Full tiles and few words to add: the launch is a stream of stores, which HBM takes at a higher rate with fewer in flight, if the
// workgroups' tiles share lines of 128 bytes above all (layers that do not begin on one).  As many as fit / 5 / 4, in us:
//   tiles on lines, 1 packet: L_T 64, 14 M elements 11.3 / 11.2 / 12.2, 20 M 15.5 / 14.5 / 16.0, 25 M 18.9 / 17.1 / 18.9, 60 M 42.5 / 36.5 / 39.8, 125 M 90.8 / 76.5 / 80.9; 58, 60 M
//     43.8 / 36.6 / 42.6; 55 43.1 / 37.9 / 44.2.  2 packets: 64, 25 M 17.6 / 20.4 / 22.9, 60 M 36.5 / 43.7 / 50.4, 125 M 76.2 / 98.6 / 117; 55, 60 M 40.4 / 49.7 / 58.3;
//   off lines, 1 packet: 64, 14 M 12.9 / 12.3 / 12.7, 20 M 18.0 / 17.1 / 16.5, 25 M 22.0 / 21.0 / 19.7, 60 M 51.7 / 49.9 / 44.8, 125 M 107 / 104 / 94; 58, 60 M 52.1 / 50.1 /
//     43.0; 55 51.8 / 49.8 / 44.6; 54, 33 M 28.8 / 26.2 / 26.6, 60 M 52.0 / 47.2 / 45.2, 125 M 107 / 89 / 100.  2 packets: 64, 14 M 12.5 / 13.4 / 15.0, 20 M 18.7 / 17.8 / 19.6, 25 M
//     22.7 / 20.7 / 23.1, 60 M 50.9 / 43.7 / 50.5, 125 M 98.5 / 98.2 / 117; 60, 60 M 54.9 / 45.9 / 53.0; 58 48.1 / 47.6 / 55.4, 125 M 92 / 108 / 129; 55, 60 M 46.5 / 49.4 / 57.7.
uint32_t unpack_hold_sum8_alone(uint64_t elems8, uint64_t tiles8, bool on_lines, uint32_t n_learners)
{
    if (elems8 < kHoldSum8Elems || elems8 < 3200u * tiles8) return 0u;   // (emptier tiles have more words to add: unpack_hold_sum8)
    if (n_learners == 1u) return !on_lines && elems8 >= 3500u * tiles8 ? 4u : 5u;
    return n_learners == 2u && !on_lines && elems8 >= 3800u * tiles8 ? 5u : 0u;
}

// ... and over them together with 16-bit layers, in one launch (tiles8 .. bins16: of either).  As many as fit / 5 / 4, in us (or as 1):
//   Tiles of fewer elements have bins of fewer, and more words to add, which other workgroups cover: 95 % at L_T 20 and 5 % at 64, 1 packet, 25 M
//     1 / 1.16 / 1.35, 60 M 1 / 1.32 / 1.56; half and half (1950 to a tile), 60 M 1 / 1.11 / 1.18; 33 and 64 (2830) 1 / 1.06 / 1.12; 45 % at 20, 5 % at 64 and the
//     rest at 500 1 / 1.05 / 1.14.
//   With 16-bit layers, 5 % at L_T 64, 60 M, 1 packet: the rest at 65 51.9 / 49.4 / 57.5, 72 1 / 0.85 / 0.98, 84 1 / 0.89 / 0.88, 129 59.3 / 55.7 / 48.9, 500 59.4 /
//     56.9 / 55.1; half of them at 65 52.2 / 47.7 / 50.5, 80 51.3 / 48.9 / 45.8, a quarter at 65 51.7 / 47.4 / 46.4.  2 packets: 65 46.6 / 59.7, 72 1 / 1.08, 76 1 / 0.99, 84 1 / 0.85,
//     129 59.2 / 54.7; half of them at 65 45.1 / 51.5, 84 1 / 0.93, 129 50.4 / 52.3; 25 M, 72 1 / 0.91, 84 1 / 0.88, 500 27.4 / 26.6, a quarter of the
//     elements at 64 26.8 / 25.7, half of them 23.9 / 24.6.
uint32_t unpack_hold_sum8(uint64_t elems8, uint64_t tiles8, uint64_t elems16, uint64_t bins16, uint32_t n_learners)
{
    const uint64_t n = elems8 + elems16;
    if (n_learners == 0u || n_learners > 2u || n < (n_learners == 1u || 4u * elems8 <= n ? kResidentElemsSum : kResidentElemsSumMany)) return 0u;
    if (8u * elems8 > n && elems8 < 3200u * tiles8) return 0u;
    // bins not far beyond 64 elements in more than a third of the table, or an eighth
    const bool short16 = n_learners == 1u ? 3u * elems16 > n && elems16 < 78u * bins16 : 8u * elems16 > n && elems16 < 71u * bins16;
    if (n_learners == 2u) return !short16 && (elems8 >= 3900u * tiles8 || 4u * elems8 <= n) ? 5u : 0u;
    return !short16 && elems8 >= 3700u * tiles8 ? 4u : 5u;
}

// Layers with 8-bit words in k_unpack8 (a wave per chunk of 64 bins), or in k_unpack and k_unpack_few (a workgroup)?
// A wave adds learner after learner, about a microsecond each, which pays where there are chunks enough to cover
// it (256 bytes of LDS to each element of L_T: 12 chunks are on a compute unit at L_T 50, 10 at 64, more
// below).  A workgroup / a wave per chunk, in us:
//   plain sum, 1 packet: L_T 16, 700 chunks 5.2 / 5.2, 1500 6.7 / 5.5, 6000 15.8 / 7.9; L_T 32, 700 5.6 / 5.9, 1500 7.2 /
//     6.9, 6000 16.9 / 11.7; L_T 50, 100 5.0 / 5.7, 700 6.2 / 6.8, 1500 8.4 / 8.1, 3000 11.5 / 11.0, 6000 17.5 / 18.2 (ResNet-50's
//     table, with 16-bit groups, 22.0 / 20.0); L_T 64, 700 6.3 / 7.3, 3000 11.5 / 13.1, 6000 21.6 / 22.6;
//   4 packets: L_T 16, 3000 chunks 14.7 / 9.2; L_T 32, 1000 8.2 / 8.8, 3000 15.7 / 10.5, 5000 21.8 / 16.5; L_T 50, 3000
//     16.8 / 14.0, 5000 23.0 / 21.2, 9000 37.1 / 31.8; L_T 64, 5000 24.0 / 27.9;
//   8 packets: L_T 16, 1000 9.1 / 11.7, 3000 18.2 / 13.2; L_T 32, 1000 9.6 / 12.9, 3000 19.0 / 14.8, 9000 48 / 34; L_T 50, 3000
//     20.0 / 18.0, 5000 29.0 / 29.6, 9000 49.9 / 43.5; L_T 64, 9000 51.6 / 62.7;
//   16 packets, L_T 50, 8000: 87 / 68 at 4 words to a bin, but 129 / 202 with the dense packets of first mini-batches (L_T
//     32: 101 / 112): beyond 32 elements left with k_unpack, and with fewer packets where chunks are many.
// With the optimizer a wave also has its tile's weights and moments to carry, with too few loads in flight:
//   SGD, L_T 8, 5000 chunks, 1 / 8 packets 14.8 / 9.7 and 27 / 17; L_T 12 16.6 / 13.4 and 29 / 19; L_T 16, 1 packet 5000 18.5 /
//   18.9, 12000 37.6 / 40.5, 8 packets 29.6 / 24.8 and 62 / 50; 20 M elements, L_T 32 75 / 84, 50 77 / 93.
static bool unpack8_for(const Plan &p, uint32_t n_chunks, uint32_t n_learners, uint32_t mode)
{
    if (mode != 0u) return p.short_bin_max <= (n_learners <= 2u ? 13u : 16u) && n_learners <= 8u && n_chunks >= 3072u;
    if (n_learners <= 2u) return p.short_bin_max <= 53u && n_chunks >= (p.short_bin_max <= 24u ? 800u : 1300u);
    if (p.short_bin_max <= 32u) return n_chunks >= 3072u;
    if (n_learners <= 4u) return n_chunks >= 5120u && p.short_bin_max <= 53u;
    if (n_learners <= 8u) return p.short_bin_max <= 40u ? n_chunks >= 4096u : p.short_bin_max <= 53u && n_chunks >= 6144u;
    return false;
}

// Chunks (waves at work) per workgroup of k_unpack8, as a power of two.  All workgroups of a launch have the
// same LDS, so the 16-bit groups that ride along get that of the chunks: with four chunks always (51 KB at
// L_T 50, 64 KB at 64) they had 3 or 2 workgroups on a compute unit instead of the 6 of k_unpack.
// k_unpack (two launches, or one on small tables) / four / two / one chunks, in us, 1 packet; elements, share
// of those with 8-bit words, L_T of both:
//   4 M, 2 %, 64 and 500:    8.6 / 15.1 / 11.2 / 8.3     60 M, 30 %, 64 and 500:    71.5 / 80.7 / 58.1 / 60.7
//   60 M, 10 %, 64 and 4272: 74.9 / 161 / 88.6 / 65.8    60 M, 85 %, 64 and 4272:   70.5 / 69.6 / 58.7 / 66.0
//   30 M, 30 %, 50 and 4272: 45.9 / 52.5 / 34.8 / 37.0   12 M, 15 %, 50 and 500:    20.9 / 21.1 / 14.8 / -
//   60 M, 15 %, 40 and 4272: 78.3 / 86.2 / 63.9 / -      60 M, 60 %, 40 and 500:    86.4 / 60.6 / 60.5 / -
// Hence: up to L_T 40, where four chunks still leave 4 workgroups, fewer only if 16-bit groups dominate;
// beyond, two, and from L_T 54 on, where two leave 5, one if the 16-bit groups are many.  The exception:
// where those are long runs of tiles, 3 workgroups keep the memory busy and four chunks are 3 to 5 % ahead
// (60 M, 30, 60 and 85 %, 50 and 500: four 60.0, 59.0 and 55.3, two 63.3, 61.6 and 57.0).
uint32_t unpack8_wg_log(const Plan &p, uint32_t n_chunks, uint32_t n_groups16, uint32_t n_learners)
{
    const uint64_t n8 = n_chunks, n16 = n_groups16;
    if (n16 == 0u || 4u * 256u * p.short_bin_max <= kUnpackLdsFull) return 2u;
    if (p.short_bin_max <= 40u) return n16 > 3u * n8 ? 1u : 2u;
    const uint64_t tiles16 = p.n_utiles - p.n_usingles8;
    if (p.short_bin_max <= 53u) return n_learners <= 2u && tiles16 >= 3u * n16 && 4u * n16 <= 3u * n8 ? 2u : 1u;
    return 2u * n16 > n8 ? 0u : 1u;
}

// One launch for everything, where the tiles of each layer are on the GPU together (see k_pack): tables of
// one tile class, with bins of at least four elements, in a
// workspace that has exchange areas for all learners of a launch.  compute_units: what the stream may use.
uint32_t one_launch_for(const Plan &p, size_t n_learners, size_t workspace_bytes, uint32_t compute_units, bool lazy)
{
    if (std::min(n_learners, size_t(kMaxBatch)) > p.sync.learners || workspace_bytes < p.sync.offset + p.sync.learners * p.ws.sync_stride) return kOneLaunchNever;
    if (!g_fold_scan.load(std::memory_order_relaxed) || p.has_tiny_bins || (p.n_class_tiles[0] != 0 && p.n_class_tiles[1] != 0)) return kOneLaunchNever;
    const bool large = p.n_class_tiles[1] != 0;
    const uint32_t room = (large ? kOneLaunchTilesLarge / kComputeUnits : kOneLaunchTilesPerUnit) * compute_units;
    const size_t workgroups = std::min(n_learners, size_t(kMaxBatch)) * p.crowd_tiles;
    const bool filled = !large || p.n_elems_total >= p.crowd_tiles * uint64_t(kLazyLargeFill);
    if (lazy && (n_learners * p.n_elems_total > (filled ? kLazyOneLaunchElems : kLazyOneLaunchElems / 2u) ||
                 (4 * workgroups > 6 * size_t(room) && p.n_elems_total < p.crowd_tiles * uint64_t(kOneLaunchCrowdElems)))) return kOneLaunchNever;
    const bool crowd = workgroups > 2 * size_t(room);   // more than are resident
    const bool folds = p.n_ctiles <= kFoldTiles && p.n_layers <= kFoldLayers;   // two staged launches, not three
    const uint64_t pays = !p.has_short_bins ? kOneLaunchCrowdElemsLong : folds ? kOneLaunchCrowdElems : 0u;
    if (large && !p.has_short_bins && workgroups > 3 * size_t(room)) return kOneLaunchNever;
    if (large && workgroups > kOneLaunchLargePerUnit * size_t(room) && p.n_elems_total < p.crowd_tiles * uint64_t(kOneLaunchLargeFill)) return kOneLaunchNever;
    if (2 * workgroups > 5 * size_t(room) && p.n_elems_total < p.crowd_tiles * pays) return kOneLaunchNever;
    if (!crowd && p.n_ctiles <= std::min(kFoldTiles, room) && p.n_layers <= kFoldLayers) return kOneLaunchTable;
    const uint32_t most = large ? kOneLaunchTilesLarge : (n_learners == 1 || p.has_short_bins || workgroups <= kOneLaunchRounds * 2 * size_t(room)) ? kOneLaunchTiles : kOneLaunchTilesLong;
    return (p.layer_tiles_max <= std::min(most, room) && p.n_layers <= kOneLaunchLayersMax) ? kOneLaunchLayers : kOneLaunchNever;
}

// Lanes per tile in k_place: 64 for tables with short bins, whose tiles send several hundred words,
// and for small tables, where the launch is far from filling the GPU and the words of a tile are
// better spread over more lanes (the 397 k-element table sends 440 words per tile in its first
// steps: 37 -> 23 us per compress call); and for tables in tiles of the larger class, of which a tile sends four times
// the words.  16 otherwise.  The larger class, 16 / 64 lanes, us: bins of 8000 and others, 40 M elements, L_T 100 in half of
// them, 1 learner 144 / 129, 4 536 / 524; 200 130 / 124, 506 / 499; 500 113 / 109, 457 / 451; 60 M, 100 191 / 181, 826 / 780; bins of 8000
// alone, 40 M, 97.2 / 96.2, 8 learners 804 / 797.
uint32_t place_lanes_for(const Plan &p)
{
    const bool large = p.n_class_tiles[0] == 0u && p.n_class_tiles[1] != 0u;
    return (p.has_short_bins || large || p.n_ctiles <= 2048u) ? 64u : 16u;
}

// 512 threads to a tile instead of 256 (see kPackWidePerUnit)?
bool pack_wide_for(const Plan &p, size_t n_learners, uint32_t compute_units)
{
    return std::min(n_learners, size_t(kMaxBatch)) * (size_t(p.n_ctiles) + 1u) <= size_t(kPackWidePerUnit) * compute_units;
}

// ---- optional event timing of the streaming kernel ---------------------------------------------
// The records are guarded by g_timing_mu; `on` alone is read without it, so that calls pay nothing
// while timing is off.
struct Timing {
    std::atomic<bool> on{false};
    std::vector<std::pair<hipEvent_t, hipEvent_t>> pool;
    size_t used = 0;
    uint64_t learners = 0;  // learners covered by the recorded launches
    uint32_t stride = 1;    // every stride-th launch is recorded
    uint64_t seen = 0;      // launches since recording started
};
static Timing g_timing;
static std::mutex g_timing_mu;
static std::atomic<bool> g_keep_gmax{false};

}  // namespace adacomp

using namespace adacomp;

extern "C" {

size_t adacomp_packet_bound(const adacomp_layer_t *layers, uint32_t n_layers)
{
    Plan p;
    return build_plan(layers, n_layers, false, p) == ADACOMP_OK ? size_t(p.bound_bytes) : 0;
}

size_t adacomp_packet_fixed_bytes(const adacomp_layer_t *layers, uint32_t n_layers)
{
    Plan p;
    return build_plan(layers, n_layers, false, p) == ADACOMP_OK ? size_t(p.fixed_bytes) : 0;
}

size_t adacomp_workspace_bytes(const adacomp_layer_t *layers, uint32_t n_layers)
{
    Plan p;
    return build_plan(layers, n_layers, false, p) == ADACOMP_OK ? p.ws.total(1) : 0;
}

size_t adacomp_workspace_bytes_batch(const adacomp_layer_t *layers, uint32_t n_layers, uint32_t n_learners)
{
    Plan p;
    if (n_learners == 0) return 0;
    return build_plan(layers, n_layers, false, p) == ADACOMP_OK ? p.ws.total(n_learners) : 0;
}

int adacomp_workspace_gmax(const adacomp_layer_t *layers, uint32_t n_layers, size_t *byte_offset,
                           size_t *n_bins_total, size_t *learner_stride)
{
    if (!byte_offset || !n_bins_total) return ADACOMP_EINVAL;
    Plan p;
    int rc = build_plan(layers, n_layers, false, p);
    if (rc != ADACOMP_OK) return rc;
    *byte_offset = p.ws.scratch + p.ws.gmax;
    *n_bins_total = p.n_bins_total;
    if (learner_stride) *learner_stride = p.ws.scratch_stride;
    return ADACOMP_OK;
}

static int init_workspace(const adacomp_layer_t *layers, uint32_t n_layers, void *workspace, size_t workspace_bytes,
                          size_t most_learners, void *hip_stream)
{
    if (!workspace) return ADACOMP_EINVAL;
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return ADACOMP_EALIGN;
    Registered reg;
    int rc = build_plan(layers, n_layers, true, reg.plan);
    if (rc != ADACOMP_OK) return rc;
    Plan &p = reg.plan;
    if (workspace_bytes < p.ws.least(1)) return ADACOMP_EWORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (hipStreamSynchronize(s) != hipSuccess) return ADACOMP_EHIP;
    char *ws = static_cast<char *>(workspace);
    if (hipMemcpy(ws + p.ws.layers, p.layers.data(), sizeof(LayerDev) * p.layers.size(), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(ws + p.ws.ctiles, p.ctiles.data(), sizeof(TileDev) * p.ctiles.size(), hipMemcpyHostToDevice) != hipSuccess ||
        (!p.cclass.empty() && hipMemcpy(ws + p.ws.cclass, p.cclass.data(), 4 * p.cclass.size(), hipMemcpyHostToDevice) != hipSuccess) ||
        hipMemcpy(ws + p.ws.utiles, p.utiles.data(), sizeof(UTileDev) * p.utiles.size(), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(ws + p.ws.ugroups, p.ugroups.data(), sizeof(UGroupDev) * p.ugroups.size(), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(ws + p.ws.usingles, p.usingles.data(), sizeof(UGroupDev) * p.usingles.size(), hipMemcpyHostToDevice) != hipSuccess)
        return ADACOMP_EHIP;
    p.sync = sync_place(p.ws, workspace_bytes, most_learners);
    if (p.sync.learners != 0 && (hipMemset(ws + p.sync.offset, 0, p.sync.learners * p.ws.sync_stride) != hipSuccess ||
                                 hipStreamSynchronize(nullptr) != hipSuccess))
        return ADACOMP_EHIP;
    register_workspace(layers, n_layers, workspace, workspace_bytes, std::move(reg.plan));
    return ADACOMP_OK;
}

int adacomp_workspace_init(const adacomp_layer_t *layers, uint32_t n_layers, void *workspace,
                           size_t workspace_bytes, void *hip_stream)
{
    return init_workspace(layers, n_layers, workspace, workspace_bytes, SIZE_MAX, hip_stream);
}

int adacomp_workspace_release(void *workspace)
{
    std::lock_guard<std::mutex> lk(g_mu);
    return g_ws.erase(workspace) ? ADACOMP_OK : ADACOMP_EINVAL;
}

// Small tables: no k_scan launch, the placement kernel does the scan itself (see k_place).
static bool fold_scan_for(const Plan &p)
{
    return g_fold_scan.load(std::memory_order_relaxed) && place_lanes_for(p) == 64u && p.n_ctiles <= kFoldTiles && p.n_layers <= kFoldLayers;
}

// Compute units that work on this stream can get: those of its mask (hipExtStreamCreateWithCUMask; without
// one, and on the GPU's partitions, all there are).  Asked for at every call, 0.2 us: a stream may be
// destroyed and another one get its handle.
static uint32_t compute_units_of(hipStream_t s)
{
    uint32_t mask[32] = {0};
    // (the runtime has no mask for the handle that stands for the null stream)
    if (hipExtStreamGetCUMask(s == hipStreamLegacy ? nullptr : s, 32, mask) != hipSuccess) { (void)hipGetLastError(); return 0; }
    uint32_t n = 0;
    for (uint32_t m : mask) n += uint32_t(__builtin_popcount(m));
    return n;
}

static int compress_common(const adacomp_layer_t *layers, uint32_t n_layers, uint32_t n_learners,
                           const float *const *grads, float *const *residues, void *const *packets_out,
                           size_t packet_capacity, uint32_t rule, float soft_factor, bool lazy, void *workspace,
                           size_t workspace_bytes, void *hip_stream)
{
    if (n_learners == 0 || !grads || !residues || !packets_out) return ADACOMP_EINVAL;
    if (rule > ADACOMP_RULE_LOCAL_SELECTION || !(soft_factor >= 1.0f && soft_factor <= 16.0f)) return ADACOMP_EINVAL;
    for (uint32_t k = 0; k < n_learners; ++k) {
        if (!grads[k] || !residues[k] || !packets_out[k] || grads[k] == residues[k]) return ADACOMP_EINVAL;
        if (reinterpret_cast<uintptr_t>(grads[k]) % 16 || reinterpret_cast<uintptr_t>(residues[k]) % 16 ||
            reinterpret_cast<uintptr_t>(packets_out[k]) % 16)
            return ADACOMP_EALIGN;
        for (uint32_t m = 0; m < k; ++m)
            if (residues[k] == residues[m] || packets_out[k] == packets_out[m]) return ADACOMP_EINVAL;
    }
    Plan p;
    int rc = find_plan(layers, n_layers, workspace, workspace_bytes, n_learners, p);
    if (rc != ADACOMP_OK) return rc;
    if (packet_capacity < p.fixed_bytes) return ADACOMP_ENOSPC;

    // Corrections that wait belong to the residue buffers of the call that left them: a lazy call
    // goes on with exactly those buffers, anything else has to wait for adacomp_residue_sync.
    bool corrections_wait = false;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_ws.find(workspace);
        if (it == g_ws.end()) return ADACOMP_EWORKSPACE;  // released by another thread meanwhile
        const std::vector<float *> &waiting = it->second.waiting;
        if (!waiting.empty()) {
            if (!lazy || waiting.size() != n_learners) return ADACOMP_EPENDING;
            for (uint32_t k = 0; k < n_learners; ++k)
                if (waiting[k] != residues[k]) return ADACOMP_EPENDING;
            corrections_wait = true;
        }
    }

    char *ws = static_cast<char *>(workspace);
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    CompressArgs a;
    a.lazy = corrections_wait ? 1u : 0u;
    a.place_mode = lazy ? kPlaceWords : kPlaceEager;
    a.tiles = reinterpret_cast<const TileDev *>(ws + p.ws.ctiles);
    a.layers = reinterpret_cast<const LayerDev *>(ws + p.ws.layers);
    a.scratch_stride = p.ws.scratch_stride;
    a.o_tile_out = uint32_t(p.ws.tile_out); a.o_layer_nsel = uint32_t(p.ws.layer_nsel);
    a.o_layer_scale = uint32_t(p.ws.layer_scale); a.o_gmax = uint32_t(p.ws.gmax);
    a.o_chunk_rel = uint32_t(p.ws.chunk_rel); a.o_stage = p.ws.stage;
    a.o_sync_rec = uint32_t(p.ws.sync_rec); a.o_sync_tile = uint32_t(p.ws.sync_tile);
    a.o_sync_layer = uint32_t(p.ws.sync_layer); a.o_sync_epoch = uint32_t(p.ws.sync_epoch);
    a.one_launch = one_launch_for(p, n_learners, workspace_bytes, kComputeUnits, lazy);
    a.pack_wide = 0u;
    if (a.one_launch != kOneLaunchNever) {
        const uint32_t units = compute_units_of(s);
        a.one_launch = one_launch_for(p, n_learners, workspace_bytes, units, lazy);
        a.pack_wide = pack_wide_for(p, n_learners, units) ? 1u : 0u;
    }
    a.sync = reinterpret_cast<uint8_t *>(ws + p.sync.offset);   // the launches of a call take turns with the areas
    a.sync_stride = p.ws.sync_stride;
    a.wait_polls = p.wait_polls;
    a.n_tiles = p.n_ctiles;
    a.n_layers = p.n_layers;
    a.keep_gmax = g_keep_gmax.load(std::memory_order_relaxed) ? 1u : 0u;
    a.class_tiles = (p.n_class_tiles[0] && p.n_class_tiles[1]) ? reinterpret_cast<const uint32_t *>(ws + p.ws.cclass) : nullptr;
    a.place_lanes = place_lanes_for(p);
    a.fold_scan = fold_scan_for(p) ? 1u : 0u;
    // tables with short bins send a large share of their elements: the eager placement then corrects
    // the residue tile by tile, whole lines at a time (k_place_tiled), instead of word by word
    a.place_tiled = (g_place_tiled.load(std::memory_order_relaxed) && p.has_short_bins && !a.fold_scan && !lazy) ? 1u : 0u;
    a.shift = (p.has_shifted_tiles && !corrections_wait) ? 1u : 0u;
    a.rule = rule;
    a.soft_factor_minus_1 = soft_factor - 1.0f;
    a.capacity = packet_capacity;
    a.fixed_bytes = p.fixed_bytes;

    // The streaming kernel runs a few percent faster per byte in launches of one learner than in one
    // launch over 16 learners of the 125 M-element workload (240 vs 246 us per learner), so large
    // gradients get one k_fused launch per learner and small ones share a launch; the scan and
    // placement kernels always cover all learners of the call.  The lazy variant of the kernel does
    // more before its first store and loses more at every launch boundary: two learners per launch
    // (or four) are 1.5 % faster per step there, and 0.3 % (1 %) slower on the eager path.
    const uint32_t per_launch_max = p.n_elems_total >= kSplitElems ? (lazy ? 2u : 1u) : kMaxBatch;
    a.fused_idle_lds = (per_launch_max == 1u && n_learners >= kFusedIdleMinLearners) ? kFusedIdleLds : 0u;
    auto enqueue = [&]() -> int {
    int rc = ADACOMP_OK;
    for (uint32_t done = 0; done < n_learners; done += kMaxBatch) {
        const uint32_t now = std::min(n_learners - done, kMaxBatch);
        a.n_learners = now;
        a.scratch = reinterpret_cast<uint8_t *>(ws + p.ws.scratch + p.ws.scratch_stride * done);
        for (uint32_t k = 0; k < kMaxBatch; ++k) {
            a.grad[k] = k < now ? grads[done + k] : nullptr;
            a.residue[k] = k < now ? residues[done + k] : nullptr;
            a.packet[k] = k < now ? static_cast<uint8_t *>(packets_out[done + k]) : nullptr;
        }
        for (uint32_t f = 0; f < now; f += per_launch_max) {
            a.fused_first = f;
            a.fused_count = std::min(per_launch_max, now - f);
            hipEvent_t ev_end = nullptr;   // set: this launch is bracketed by an event pair
            if (g_timing.on.load(std::memory_order_relaxed)) {
                std::lock_guard<std::mutex> lk(g_timing_mu);
                if (g_timing.on.load(std::memory_order_relaxed) && (g_timing.seen++ % g_timing.stride) == 0) {
                    if (g_timing.used == g_timing.pool.size()) {
                        hipEvent_t e0, e1;
                        if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return ADACOMP_EHIP;
                        g_timing.pool.emplace_back(e0, e1);
                    }
                    const std::pair<hipEvent_t, hipEvent_t> &ev = g_timing.pool[g_timing.used++];
                    g_timing.learners += a.fused_count;
                    if (hipEventRecord(ev.first, s) != hipSuccess) return ADACOMP_EHIP;
                    ev_end = ev.second;   // the handle itself: the pool may grow under another thread
                }
            }
            for (int c = 0; c < 2; ++c) {
                if (p.n_class_tiles[c] == 0) continue;
                a.class_first = c ? p.n_class_tiles[0] : 0u;
                a.class_count = p.n_class_tiles[c];
                if ((rc = launch_fused(a, c, hip_stream)) != ADACOMP_OK) return rc;
            }
            if (ev_end && hipEventRecord(ev_end, s) != hipSuccess) return ADACOMP_EHIP;
        }
        if (a.one_launch) continue;
        if (!a.fold_scan && (rc = launch_scan(a, hip_stream)) != ADACOMP_OK) return rc;
        if ((rc = launch_place(a, hip_stream)) != ADACOMP_OK) return rc;
    }
    return ADACOMP_OK;
    };
    rc = enqueue();
    if (lazy || corrections_wait) {
        // After a failure part of the way through, some kernels of this call may have applied and
        // overwritten the corrections that waited while others did not run: nothing can be said to
        // wait any more, and the residues are unspecified (as after a failed adacomp_residue_sync).
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_ws.find(workspace);
        if (it != g_ws.end()) {
            if (rc == ADACOMP_OK) it->second.waiting.assign(residues, residues + n_learners);
            else it->second.waiting.clear();
        }
    }
    return rc;
}

int adacomp_compress_variant(const adacomp_layer_t *layers, uint32_t n_layers, uint32_t n_learners,
                             const float *const *grads, float *const *residues, void *const *packets_out,
                             size_t packet_capacity, uint32_t rule, float soft_factor, void *workspace,
                             size_t workspace_bytes, void *hip_stream)
{
    return compress_common(layers, n_layers, n_learners, grads, residues, packets_out, packet_capacity, rule,
                           soft_factor, false, workspace, workspace_bytes, hip_stream);
}

int adacomp_compress_batch_lazy(const adacomp_layer_t *layers, uint32_t n_layers, uint32_t n_learners,
                                const float *const *grads, float *const *residues, void *const *packets_out,
                                size_t packet_capacity, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return compress_common(layers, n_layers, n_learners, grads, residues, packets_out, packet_capacity,
                           ADACOMP_RULE_ADACOMP, 2.0f, true, workspace, workspace_bytes, hip_stream);
}

int adacomp_residue_sync(void *workspace, void *hip_stream)
{
    if (!workspace) return ADACOMP_EINVAL;
    Plan p;
    std::vector<float *> waiting;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_ws.find(workspace);
        if (it == g_ws.end()) return ADACOMP_EWORKSPACE;
        if (it->second.waiting.empty()) return ADACOMP_OK;
        waiting = it->second.waiting;
        p.n_layers = it->second.plan.n_layers; p.n_ctiles = it->second.plan.n_ctiles;
        p.has_short_bins = it->second.plan.has_short_bins; p.ws = it->second.plan.ws;
        for (int c = 0; c < 2; ++c) p.n_class_tiles[c] = it->second.plan.n_class_tiles[c];
    }
    char *ws = static_cast<char *>(workspace);
    CompressArgs a = {};
    a.tiles = reinterpret_cast<const TileDev *>(ws + p.ws.ctiles);
    a.layers = reinterpret_cast<const LayerDev *>(ws + p.ws.layers);
    a.scratch_stride = p.ws.scratch_stride;
    a.o_tile_out = uint32_t(p.ws.tile_out); a.o_layer_nsel = uint32_t(p.ws.layer_nsel);
    a.o_layer_scale = uint32_t(p.ws.layer_scale); a.o_gmax = uint32_t(p.ws.gmax);
    a.o_chunk_rel = uint32_t(p.ws.chunk_rel); a.o_stage = p.ws.stage;
    a.n_tiles = p.n_ctiles;
    a.n_layers = p.n_layers;
    a.place_lanes = place_lanes_for(p);
    a.place_mode = kPlaceResidue;
    const uint32_t n_learners = uint32_t(waiting.size());
    int rc = ADACOMP_OK;
    for (uint32_t done = 0; done < n_learners; done += kMaxBatch) {
        const uint32_t now = std::min(n_learners - done, kMaxBatch);
        a.n_learners = now;
        a.scratch = reinterpret_cast<uint8_t *>(ws + p.ws.scratch + p.ws.scratch_stride * done);
        for (uint32_t k = 0; k < kMaxBatch; ++k) a.residue[k] = k < now ? waiting[done + k] : nullptr;
        if ((rc = launch_place(a, hip_stream)) != ADACOMP_OK) break;
    }
    // after a failed launch some corrections may be applied and others not: nothing waits either way
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_ws.find(workspace);
    if (it != g_ws.end()) it->second.waiting.clear();
    return rc;
}

int adacomp_compress_batch(const adacomp_layer_t *layers, uint32_t n_layers, uint32_t n_learners,
                           const float *const *grads, float *const *residues, void *const *packets_out,
                           size_t packet_capacity, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return adacomp_compress_variant(layers, n_layers, n_learners, grads, residues, packets_out, packet_capacity,
                                    ADACOMP_RULE_ADACOMP, 2.0f, workspace, workspace_bytes, hip_stream);
}

int adacomp_compress(const adacomp_layer_t *layers, uint32_t n_layers, const float *grad,
                     float *residue, void *packet_out, size_t packet_capacity, void *workspace,
                     size_t workspace_bytes, void *hip_stream)
{
    return adacomp_compress_batch(layers, n_layers, 1, &grad, &residue, &packet_out, packet_capacity,
                                  workspace, workspace_bytes, hip_stream);
}

// ---- the entry point that allocates nothing -----------------------------------------------------
// Its workspace is a file-scope device array.  Host code never uses the array's name as an address
// (on the host the name is only a handle for the runtime): the device address of this GPU's copy
// comes from hipGetSymbolAddress, once per device, and that pointer is what is registered as the
// workspace, copied to and handed to the kernels.
constexpr size_t kStaticScratchBytes = ADACOMP_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
static std::mutex g_static_mu;
static void *g_static_ptr[kMaxDevices];  // per device: where that device holds `scratch`

static int static_scratch(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return ADACOMP_EHIP;
    std::lock_guard<std::mutex> lk(g_static_mu);
    if (!g_static_ptr[dev]) {   // first call on this device, which is current
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return ADACOMP_EHIP;
        if (reinterpret_cast<uintptr_t>(ptr) % 256 != 0) return ADACOMP_EALIGN;
        g_static_ptr[dev] = ptr;
    }
    *out = g_static_ptr[dev];
    return ADACOMP_OK;
}

int adacomp_compress_static(const adacomp_layer_t *layers, uint32_t n_layers, const float *grad, float *residue,
                            void *packet_out, size_t packet_capacity, void *hip_stream)
{
    if (!layers || n_layers == 0 || !grad || !residue || !packet_out) return ADACOMP_EINVAL;
    void *ws = nullptr;
    const int rc_dev = static_scratch(&ws);
    if (rc_dev == ADACOMP_OK) {
        // the usual case: this device's array already holds the tile tables of this layer table
        const int rc = adacomp_compress(layers, n_layers, grad, residue, packet_out, packet_capacity, ws,
                                        kStaticScratchBytes, hip_stream);
        if (rc != ADACOMP_EWORKSPACE) return rc;
    }
    // another layer table than the last call's on this device (or the first call): check it, see that
    // it fits, and write its tile tables into the array
    Plan p;
    int rc = build_plan(layers, n_layers, false, p);
    if (rc != ADACOMP_OK) return rc;
    if (p.ws.least(1) > kStaticScratchBytes) return ADACOMP_ETOOBIG;
    if (rc_dev != ADACOMP_OK) return rc_dev;
    if ((rc = init_workspace(layers, n_layers, ws, kStaticScratchBytes, 1, hip_stream)) != ADACOMP_OK) return rc;   // one learner: no other call knows this array
    return adacomp_compress(layers, n_layers, grad, residue, packet_out, packet_capacity, ws, kStaticScratchBytes,
                            hip_stream);
}

static int unpack_common(const adacomp_layer_t *layers, uint32_t n_layers, const void *const *packets,
                         uint32_t n_learners, float *dense_out, float *weights, float *state1, float *state2,
                         const adacomp_optimizer_t *opt, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (n_learners > 0 && !packets) return ADACOMP_EINVAL;
    if (reinterpret_cast<uintptr_t>(dense_out) % 16) return ADACOMP_EALIGN;
    for (uint32_t k = 0; k < n_learners; ++k) {
        if (!packets[k]) return ADACOMP_EINVAL;
        if (reinterpret_cast<uintptr_t>(packets[k]) % 16) return ADACOMP_EALIGN;
    }
    Plan p;
    int rc = find_plan(layers, n_layers, workspace, workspace_bytes, 1, p);
    if (rc != ADACOMP_OK) return rc;

    char *ws = static_cast<char *>(workspace);
    UnpackArgs a;
    a.tiles = reinterpret_cast<const UTileDev *>(ws + p.ws.utiles);
    a.dense = dense_out;
    a.n_layers = p.n_layers;
    a.weights = weights; a.state1 = state1; a.state2 = state2;
    a.n_average = float(n_learners);
    a.lr = a.p1 = a.p2 = a.one_minus_p1 = a.one_minus_p2 = a.eps = 0.f;
    a.bias1 = a.bias2 = 1.f;
    if (opt) {
        a.lr = opt->lr;
        if (opt->kind == ADACOMP_OPT_SGD_MOMENTUM) a.p1 = opt->momentum;
        else {
            a.p1 = opt->beta1; a.p2 = opt->beta2;
            a.one_minus_p1 = 1.0f - opt->beta1; a.one_minus_p2 = 1.0f - opt->beta2;
            a.eps = opt->eps; a.bias1 = opt->bias1; a.bias2 = opt->bias2;
        }
    }
    uint32_t done = 0;
    do {  // 64 learners per launch; later launches add onto the stored partial sum, same order;
          // the update is applied by the last launch, when the sum is complete
        const uint32_t now = std::min(n_learners - done, kMaxPacketArgs);
        const bool last = done + now == n_learners;
        a.n_learners = now;
        a.accumulate = done > 0;
        a.mode = (opt && last) ? opt->kind : 0u;
        a.write_dense = dense_out != nullptr;
        for (uint32_t k = 0; k < kMaxPacketArgs; ++k)
            a.packets[k] = k < now ? static_cast<const uint8_t *>(packets[done + k]) : nullptr;
        // runs of tiles per workgroup for the plain sum, single tiles when the optimizer step follows
        const UGroupDev *table = reinterpret_cast<const UGroupDev *>(ws + (a.mode == 0u ? p.ws.ugroups : p.ws.usingles));
        const uint32_t n_all = a.mode == 0u ? p.n_ugroups : p.n_utiles, n8 = a.mode == 0u ? p.n_ugroups8 : p.n_usingles8;
        // What the launches over one word width or both have, whether they fetch the optimizer's state ahead, and to how many
        // workgroups per compute unit they are held.
        const uint64_t tiles16 = p.n_utiles - p.n_usingles8, elems8 = p.n_elems_total - p.n_elems16, bins8 = p.n_bins_total - p.n_bins16;
        const bool early16 = unpack_early_for(p.n_elems16, p.n_bins16, tiles16, false, now, a.mode), early8 = unpack_early_for(elems8, bins8, p.n_usingles8, true, now, a.mode);
        const bool early_both = now <= 8u && unpack_early_for(p.n_elems_total, p.n_bins_total, p.n_utiles, 3u * elems8 >= p.n_elems_total, now, a.mode);
        uint32_t resident16 = resident_for(p.n_elems16, p.n_bins16, tiles16, now, a.mode);
        if (resident16 != 0u && a.mode != 0u && (early16 || now <= 2u)) resident16 = 4u;
        uint32_t resident8 = unpack_hold_few(elems8, p.n_usingles8, now) ? 4u : 0u;
        // Over both widths: early as over one (behind / ahead, us, 12 M, L_T 50, and 13 M, 500: SGD, 4 packets 71.3 / 66.3, 8 76.1 / 69.9, Adam, 8 112.2 / 107.6); and held where the
        // 16-bit layers have few words to a bin (as many as fit / 4: 12 M and 13 M, SGD, 4 67.5 / 66.3; 30 M, 50, and 30 M, 4000, SGD, 4 161.0 / 156.0, Adam, 3 241.5 / 238.3; 5 M, 50,
        // and 45 M, 500, Adam, 3 205.0 / 201.1; not by this line, 20 M, 50, and 20 M, 200, SGD, 4 107.0 / 103.5; with tiles less full 5 M, 20, and 20 M, 65, SGD, 2 65.9 / 71.1).
        uint32_t resident_both = unpack_hold_few(p.n_elems_total, p.n_utiles, now) && p.n_elems16 >= 60u * uint64_t(now) * p.n_bins16 ? 4u : 0u;
        if (a.mode == 0u) {
            const bool on_lines = 2u * p.n_elems8_lines >= elems8 && reinterpret_cast<uintptr_t>(dense_out) % 128u == 0u;
            resident8 = p.n_elems16 == 0u ? unpack_hold_sum8_alone(elems8, p.n_usingles8, on_lines, now) : 0u;
            resident_both = unpack_hold_sum8(elems8, p.n_usingles8, p.n_elems16, p.n_bins16, now);
        }
        // Launches over all groups take single tiles without a look at the table, a round of scalar loads; over both word widths only
        // while every tile has a compute unit to itself, since those of short bins, which take longest, stand first in it (2 M elements,
        // 50 and 500, 16 packets: by the table 13.8 us, without 14.4; 0.4 M 13.0 / 12.6).
        const bool singles = a.mode != 0u || p.groups_single;
        const UGroupDev *const whole_table = singles ? nullptr : table, *const both_table = singles && p.n_utiles <= kComputeUnits ? nullptr : table;
        a.groups = table;
        a.n_groups = n_all;
        a.n_groups8 = a.first16 = a.chunk_lds = 0u;
        if (n8 != 0u && unpack8_for(p, n8, now, a.mode)) {
            a.groups = reinterpret_cast<const UGroupDev *>(ws + p.ws.ugroups);   // single chunks in either table, here in order
            a.n_groups8 = n8;
            a.n_groups = n_all - n8;
            a.first16 = uint32_t(table - a.groups) + n8;
            a.chunk_lds = 64u * p.short_bin_max + unpack8_wg_log(p, n8, a.n_groups, now);
            if ((rc = launch_unpack(a, 3, 0u, false, hip_stream)) != ADACOMP_OK) return rc;
        } else if (n8 == 0u || n8 == n_all) {  // one word width
            a.groups = whole_table;
            if ((rc = launch_unpack(a, n8 ? 1 : 0, n8 ? resident8 : resident16, n8 ? early8 : early16, hip_stream)) != ADACOMP_OK) return rc;
        } else if (p.n_utiles <= kUnpackSplitTiles || now <= kUnpackTogether) {  // mixed, and small or of few packets: one launch that handles both
            a.groups = both_table;
            if ((rc = launch_unpack(a, 2, resident_both, early_both, hip_stream)) != ADACOMP_OK) return rc;
        } else {  // large and mixed: the 8-bit groups come first in the table
            a.n_groups = n8;
            if ((rc = launch_unpack(a, 1, resident8, early8, hip_stream)) != ADACOMP_OK) return rc;
            a.groups = table + n8;
            a.n_groups = n_all - n8;
            if ((rc = launch_unpack(a, 0, resident16, early16, hip_stream)) != ADACOMP_OK) return rc;
        }
        done += now;
    } while (done < n_learners);
    return ADACOMP_OK;
}

int adacomp_unpack_accumulate(const adacomp_layer_t *layers, uint32_t n_layers,
                              const void *const *packets, uint32_t n_learners, float *dense_out,
                              void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!dense_out) return ADACOMP_EINVAL;
    return unpack_common(layers, n_layers, packets, n_learners, dense_out, nullptr, nullptr, nullptr, nullptr,
                         workspace, workspace_bytes, hip_stream);
}

int adacomp_unpack_update(const adacomp_layer_t *layers, uint32_t n_layers, const void *const *packets,
                          uint32_t n_learners, float *dense_out, float *weights, float *state1, float *state2,
                          const adacomp_optimizer_t *opt, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!opt || !weights || !state1 || n_learners == 0) return ADACOMP_EINVAL;
    if (opt->kind != ADACOMP_OPT_SGD_MOMENTUM && opt->kind != ADACOMP_OPT_ADAM) return ADACOMP_EINVAL;
    if (opt->kind == ADACOMP_OPT_ADAM && (!state2 || !(opt->bias1 > 0.f) || !(opt->bias2 > 0.f))) return ADACOMP_EINVAL;
    if (!dense_out && n_learners > kMaxPacketArgs) return ADACOMP_EINVAL;  // the partial sums need a home
    if (reinterpret_cast<uintptr_t>(weights) % 16 || reinterpret_cast<uintptr_t>(state1) % 16 ||
        reinterpret_cast<uintptr_t>(state2) % 16)
        return ADACOMP_EALIGN;
    if (weights == state1 || weights == state2 || state1 == state2 || dense_out == weights || dense_out == state1 ||
        (dense_out && dense_out == state2))
        return ADACOMP_EINVAL;
    return unpack_common(layers, n_layers, packets, n_learners, dense_out, weights, state1, state2, opt, workspace,
                         workspace_bytes, hip_stream);
}

const char *adacomp_strerror(int code)
{
    switch (code) {
    case ADACOMP_OK: return "ok";
    case ADACOMP_EINVAL: return "invalid argument (null pointer, empty or overlapping layer, aliasing buffers)";
    case ADACOMP_EBADLT: return "L_T must be in 1..16384";
    case ADACOMP_EALIGN: return "elem_offset must be a multiple of 4 and buffers 16-byte aligned (workspace 256)";
    case ADACOMP_ENOSPC: return "packet capacity below the fixed part of the packet";
    case ADACOMP_EHIP: return "HIP runtime error (no device or failed launch)";
    case ADACOMP_EWORKSPACE: return "workspace too small or not initialised for this layer table";
    case ADACOMP_EPENDING: return "residue corrections of a lazy call wait in this workspace: go on with the same lazy call or call adacomp_residue_sync";
    case ADACOMP_ETOOBIG: return "layer table needs more workspace than the static scratch array holds (16 MiB): use adacomp_compress with a workspace of the caller's";
    default: return "unknown adacomp error";
    }
}

int adacomp_copy_f32(float *dst, const float *src, size_t n, void *hip_stream)
{
    if (!dst || !src) return ADACOMP_EINVAL;
    if (reinterpret_cast<uintptr_t>(dst) % 16 || reinterpret_cast<uintptr_t>(src) % 16) return ADACOMP_EALIGN;
    return n == 0 ? ADACOMP_OK : launch_copy(dst, src, n, hip_stream);
}

int adacomp_triad_resident_f32(float *x, const float *y, size_t n, uint32_t workgroups_per_cu, void *hip_stream)
{
    if (!x || !y || x == y || workgroups_per_cu < 3 || workgroups_per_cu > 8) return ADACOMP_EINVAL;
    if (reinterpret_cast<uintptr_t>(x) % 16 || reinterpret_cast<uintptr_t>(y) % 16 || n % 4 != 0) return ADACOMP_EALIGN;
    if (n >= (size_t(1) << 43)) return ADACOMP_EINVAL;
    return n == 0 ? ADACOMP_OK : launch_triad(x, y, n, workgroups_per_cu, hip_stream);
}

int adacomp_triad_f32(float *x, const float *y, size_t n, void *hip_stream)
{
    return adacomp_triad_resident_f32(x, y, n, 8, hip_stream);
}

int adacomp_fill_f32(float *x, float value, size_t n, void *hip_stream)
{
    if (!x) return ADACOMP_EINVAL;
    if (reinterpret_cast<uintptr_t>(x) % 16 || n % 4 != 0) return ADACOMP_EALIGN;
    if (n >= (size_t(1) << 43)) return ADACOMP_EINVAL;
    return n == 0 ? ADACOMP_OK : launch_fill(x, value, n, hip_stream);
}

int adacomp_selftest_binindex(void)
{
    for (uint32_t T = 2; T <= ADACOMP_LT_MAX; ++T) {
        const uint32_t m = bin_magic(T);
        uint32_t q = 0, r = 0;  // running e / T, e % T
        for (uint32_t e = 0; e < 16384u; ++e) {
            if (uint32_t((uint64_t(e) * m) >> 32) != q) return -1;
            if (++r == T) { r = 0; ++q; }
        }
    }
    return 0;
}

int adacomp_debug_keep_gmax(int enable)
{
    g_keep_gmax = enable != 0;
    return ADACOMP_OK;
}

int adacomp_debug_wait_polls(void *workspace, uint32_t polls)
{
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_ws.find(workspace);
    if (it == g_ws.end()) return ADACOMP_EWORKSPACE;
    it->second.plan.wait_polls = std::min(polls, kWaitPollsMax);   // every wait ends
    return ADACOMP_OK;
}

int adacomp_debug_one_launch(const void *workspace, size_t n_learners, int lazy)
{
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_ws.find(workspace);
    if (it == g_ws.end() || n_learners == 0 || it->second.bytes < it->second.plan.ws.least(n_learners)) return ADACOMP_EWORKSPACE;
    return one_launch_for(it->second.plan, n_learners, it->second.bytes, kComputeUnits, lazy != 0) != kOneLaunchNever ? 1 : 0;
}

int adacomp_tuning_fold_scan(int enable)
{
    g_fold_scan = enable != 0;
    return ADACOMP_OK;
}

int adacomp_tuning_place_tiled(int enable)
{
    g_place_tiled = enable != 0;
    return ADACOMP_OK;
}

int adacomp_tuning_unpack_min_groups(uint32_t n_groups)
{
    g_unpack_min_groups = n_groups ? n_groups : kUnpackMinGroups;
    return ADACOMP_OK;
}

int adacomp_timing_enable(int enable)
{
    std::lock_guard<std::mutex> lk(g_timing_mu);
    g_timing.on = enable != 0;
    g_timing.stride = enable > 0 ? uint32_t(enable) : 1u;
    g_timing.used = 0;
    g_timing.learners = 0;
    g_timing.seen = 0;
    return ADACOMP_OK;
}

int adacomp_timing_read(double *total_ms, uint64_t *n_launches, uint64_t *n_learners)
{
    if (!total_ms || !n_launches || !n_learners) return ADACOMP_EINVAL;
    std::lock_guard<std::mutex> lk(g_timing_mu);
    double sum = 0.0;
    for (size_t i = 0; i < g_timing.used; ++i) {
        float ms = 0.f;
        if (hipEventSynchronize(g_timing.pool[i].second) != hipSuccess ||
            hipEventElapsedTime(&ms, g_timing.pool[i].first, g_timing.pool[i].second) != hipSuccess)
            return ADACOMP_EHIP;
        sum += ms;
    }
    *total_ms = sum;
    *n_launches = g_timing.used;
    *n_learners = g_timing.learners;
    g_timing.used = 0;
    g_timing.learners = 0;
    return ADACOMP_OK;
}

}  // extern "C"
