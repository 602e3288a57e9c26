// Exercises the host-only parts of libadacomp (table validation, plan and size arithmetic, error
// paths that return before any HIP call) under AddressSanitizer / UBSan on the host side.
// Built and run by tests/test_sanitizers.py; no GPU is touched.
#include <algorithm>
#include <cstdio>
#include <cstdint>
#include <cstdlib>
#include <utility>
#include <vector>

#include <hip/hip_runtime.h>

#include "adacomp.h"
#include "adacomp_debug.h"
#include "adacomp_plan.h"

// Invariants of the tile tables that the kernels index without further checks: every table is
// built on the host, so everything the kernels assume about it can be verified here.
static uint64_t g_tiles_checked = 0, g_groups_checked = 0;

static int check_plan(const std::vector<adacomp_layer_t> &t)
{
    using namespace adacomp;
    Plan p;
    if (build_plan(t.data(), uint32_t(t.size()), true, p) != ADACOMP_OK) return 100;
    if (p.ctiles.size() != p.n_ctiles || p.utiles.size() != p.n_utiles || p.ugroups.size() != p.n_ugroups ||
        p.usingles.size() != p.n_utiles)
        return 101;
    // compress tiles: whole bins, in order, covering each layer exactly; sizes fit the register class
    uint32_t ct = 0;
    uint64_t stage_next = 0;   // stretches of the staging array: one after the other in tile order, each a multiple of 4 entries
    for (uint32_t l = 0; l < p.n_layers; ++l) {
        const LayerDev &ld = p.layers[l];
        if (ld.ctile_start != ct) return 102;
        uint64_t e = 0;
        uint32_t bin = 0;
        for (uint32_t i = 0; i < ld.n_ctiles; ++i, ++ct) {
            const TileDev &td = p.ctiles[ct];
            const uint32_t cap = td.jcode() ? 16384u : 4096u;
            if (td.layer() != l || td.L_T != ld.L_T || td.first_bin != bin || td.elem_base != ld.elem_offset + e) return 103;
            if (td.n_elems == 0 || td.n_elems > cap || td.n_bins == 0 || td.n_bins > kMaxTileBins) return 104;
            if (td.n_bins != (td.n_elems + td.L_T - 1) / td.L_T) return 105;
            if (td.aligned() != (td.elem_base % 4 == 0)) return 106;
            // a tile that keeps 16-byte accesses although it is not aligned: larger class only, skip is its
            // misalignment, and the tile still fits its class with the misalignment added
            if (td.skip() != 0 && (td.aligned() || td.jcode() != 1 || td.skip() != td.elem_base % 4 || td.n_elems + td.skip() > 16384u)) return 119;
            if (td.skip() == 0 && !td.aligned() && td.jcode() == 1 && td.n_elems + td.elem_base % 4 <= 16384u) return 146;
            if (td.skip() != 0 && !p.has_shifted_tiles) return 147;
            if (td.magic != bin_magic(td.L_T)) return 107;
            if (td.n_elems > 16384u) return 108;  // the multiply-shift bin index is checked below this
            if (td.stage_base % 4u != 0 || td.stage_base < stage_next) return 117;   // stretches do not overlap
            stage_next = uint64_t(td.stage_base) + td.n_elems;
            if (stage_next > p.stage_entries) return 118;
            e += td.n_elems;
            bin += td.n_bins;
            if (i + 1 < ld.n_ctiles && td.n_elems % td.L_T != 0) return 109;  // only the last tile may end in a short bin
        }
        if (e != ld.n_elems || bin != ld.n_bins) return 110;
    }
    if (ct != p.n_ctiles) return 111;
    // tables with both tile sizes list the tile indices by size, each size in ascending order
    if (p.n_class_tiles[0] + p.n_class_tiles[1] != p.n_ctiles) return 112;
    if (p.n_class_tiles[0] && p.n_class_tiles[1]) {
        if (p.cclass.size() != p.n_ctiles) return 113;
        for (uint32_t i = 0; i < p.n_ctiles; ++i) {
            const uint32_t want = i < p.n_class_tiles[0] ? 0u : 1u;
            if (p.cclass[i] >= p.n_ctiles || p.ctiles[p.cclass[i]].jcode() != want) return 114;
            if (i && i != p.n_class_tiles[0] && p.cclass[i] <= p.cclass[i - 1]) return 115;
        }
    } else if (!p.cclass.empty()) return 116;
    // unpack tiles: cover each layer exactly, at most kUnpackTileElems each, whole bins inside one
    // 64-bin chunk or a slice of one long bin
    std::vector<uint64_t> covered(p.n_layers, 0);
    for (uint32_t i = 0; i < p.n_utiles; ++i) {
        const UTileDev &ut = p.utiles[i];
        if (ut.layer() >= p.n_layers) return 120;
        const LayerDev &ld = p.layers[ut.layer()];
        if (ut.L_T != ld.L_T || ut.n_elems == 0 || ut.n_elems > kUnpackTileElems) return 121;
        const uint64_t local = uint64_t(ut.first_bin) * ut.L_T + ut.idx_lo;
        if (ut.elem_base != ld.elem_offset + local || local != covered[ut.layer()]) return 122;
        covered[ut.layer()] += ut.n_elems;
        if (ut.L_T <= kUnpackTileElems) {
            if (ut.idx_lo != 0 || ut.n_bins == 0 || ut.n_bins > 64) return 123;
            if ((ut.first_bin >> 6) != ((ut.first_bin + ut.n_bins - 1) >> 6)) return 124;
            if (ut.n_bins != (ut.n_elems + ut.L_T - 1) / ut.L_T) return 125;
        } else {
            if (ut.n_bins != 1 || ut.idx_lo + ut.n_elems > ut.L_T) return 126;
        }
        if (ut.group_log2() < 3 || ut.group_log2() > 6) return 127;
        if (ut.aligned() != (ut.elem_base % 4 == 0)) return 128;
        // what the record holds of its layer, whose own the unpack kernels do not read
        if (ut.counts_offset != ld.counts_offset || ut.chunks_offset != ld.chunks_offset || ut.words8() != (ld.word_bytes == 1)) return 151;
        if (ut.chunk_bins != std::min<uint32_t>(64u, ld.n_bins - (ut.first_bin & ~63u)) || (ut.first_bin & 63u) + ut.n_bins > ut.chunk_bins) return 152;
    }
    for (uint32_t l = 0; l < p.n_layers; ++l)
        if (covered[l] != p.layers[l].n_elems) return 129;
    // groups: consecutive tiles, every tile in exactly one group, at most kUnpackGroupTiles, all in
    // one layer and one chunk (or one long bin): the kernel's table rows stay below 64
    std::vector<uint8_t> seen(p.n_utiles, 0);
    for (const UGroupDev &g : p.ugroups) {
        if (g.n_tiles == 0 || g.n_tiles > kUnpackGroupTiles || uint64_t(g.first_tile) + g.n_tiles > p.n_utiles) return 130;
        const UTileDev &a = p.utiles[g.first_tile];
        for (uint32_t i = 0; i < g.n_tiles; ++i) {
            const UTileDev &ut = p.utiles[g.first_tile + i];
            if (seen[g.first_tile + i]++) return 131;
            if (ut.layer() != a.layer()) return 132;
            if (ut.L_T <= kUnpackTileElems ? (ut.first_bin >> 6) != (a.first_bin >> 6) : ut.first_bin != a.first_bin) return 133;
            if (ut.first_bin < a.first_bin || ut.first_bin + ut.n_bins - a.first_bin > 64) return 134;
        }
        // the end of the group's bins, as k_unpack works it out from the first tile's record
        const UTileDev &last = p.utiles[g.first_tile + g.n_tiles - 1u];
        const uint32_t bins = a.L_T > kUnpackTileElems ? 1u : a.n_bins * g.n_tiles;
        if (std::min(a.first_bin + bins, (a.first_bin & ~63u) + a.chunk_bins) != last.first_bin + last.n_bins) return 153;
    }
    for (uint32_t i = 0; i < p.n_utiles; ++i)
        if (seen[i] != 1) return 135;
    // both tables list the groups of layers with 8-bit words first (they go to their own kernel)
    if (p.n_ugroups8 > p.n_ugroups || p.n_usingles8 > p.n_utiles) return 137;
    for (uint32_t i = 0; i < p.n_ugroups; ++i)
        if ((p.utiles[p.ugroups[i].first_tile].L_T <= 64u) != (i < p.n_ugroups8)) return 138;
    for (uint32_t i = 0; i < p.n_utiles; ++i)
        if ((p.utiles[p.usingles[i].first_tile].L_T <= 64u) != (i < p.n_usingles8)) return 139;
    std::fill(seen.begin(), seen.end(), 0);
    for (const UGroupDev &g : p.usingles) {
        if (g.n_tiles != 1 || g.first_tile >= p.n_utiles || seen[g.first_tile]++) return 136;
    }
    // launches without a table of groups: the tile from the workgroup's number, each tile once; of one word width in the table's order
    std::fill(seen.begin(), seen.end(), 0);
    const bool mixed = p.n_usingles8 != 0 && p.n_usingles8 != p.n_utiles;
    for (uint32_t i = 0; i < p.n_utiles; ++i) {
        const uint32_t t = single_tile(i, p.n_utiles);
        if (t >= p.n_utiles || seen[t]++ || (!mixed && p.usingles[i].first_tile != t)) return 154;
    }
    if (p.groups_single) {
        if (p.n_ugroups != p.n_utiles) return 155;
        for (uint32_t i = 0; i < p.n_ugroups; ++i)
            if (p.ugroups[i].n_tiles != 1 || p.ugroups[i].first_tile != p.usingles[i].first_tile) return 156;
    }
    if (p.ws.sync_stride >> 32) return 157;   // k_pack takes it in 32 bits
    // workspace layout: sections in order, inside the advertised size
    const WorkspaceLayout &w = p.ws;
    if (w.cclass + 4 * size_t(p.n_ctiles) > w.utiles) return 144;
    if (!(w.layers < w.ctiles && w.ctiles <= w.cclass && w.cclass <= w.utiles && w.utiles <= w.ugroups && w.ugroups <= w.usingles && w.usingles <= w.scratch)) return 140;
    if (w.usingles + sizeof(UGroupDev) * size_t(p.n_utiles) > w.scratch) return 141;
    if (w.stage + 2 * size_t(p.stage_entries) + 128 > w.scratch_stride) return 142;  // k_place reads 64 entries from a tile's start
    if (p.stage_entries > p.n_elems_total + 3ull * p.n_ctiles) return 145;       // the array follows the element count, not the address span
    // exchange areas of the one-launch compress: sections in order, behind the scratch blocks of as many
    // learners, inside the workspace, and none where there is no room; k_pack takes aligned tiles only
    if (!(w.sync_rec + 16 * size_t(p.n_ctiles) <= w.sync_tile && w.sync_tile + 32 * size_t(p.n_ctiles) <= w.sync_layer &&
          w.sync_layer + 32 * size_t(p.n_layers) <= w.sync_epoch && w.sync_epoch + 4 * (size_t(p.n_ctiles) + 1) <= w.sync_stride))   // (epochs: the header's workgroup has one too)
        return 148;
    // no call that the workspace accepts has a scratch block that reaches an area: a captured call may be
    // replayed after any of them
    for (size_t n = 1; n <= 70; n += n < 6 ? 1 : 8)
        for (size_t bytes : {w.least(n), w.least(n) + w.sync_stride - 1, w.total(n) - 1, w.total(n), w.total(n) + 1000, w.least(n + 1) - 1})
            for (size_t most : {size_t(1), SIZE_MAX}) {
                const SyncPlace at = sync_place(w, bytes, most);
                size_t accepted = 0;   // learners of the largest call
                while (accepted < most && w.least(accepted + 1) <= bytes) ++accepted;
                if (at.learners > kMaxBatch || (at.learners && (at.offset % 128 || at.offset < w.least(accepted) || at.offset + at.learners * w.sync_stride > bytes))) return 150;
                const size_t most_areas = std::min({n, size_t(kMaxBatch), (w.scratch_stride - 1) / w.sync_stride});
                if (bytes == w.total(n) && (most > n ? accepted != n : false)) return 153;
                if (accepted == n && bytes >= w.total(n) && at.learners < most_areas) return 149;
                if (accepted == n && bytes < w.least(n) + w.sync_stride && at.learners) return 152;
            }
    for (const TileDev &td : p.ctiles)
        if (td.jcode() == 0 && !td.aligned()) return 151;
    // k_pack: the bins of every slot of the rows that a tile begins, those past the tile too, have entries in its
    // arrays; those of the tile's elements are what their index says
    for (const TileDev &td : p.ctiles) {
        if (td.L_T < 4u) continue;   // staged
        for (const uint32_t threads : {256u, 512u, 1024u}) {
            if ((threads == 1024u) != (td.jcode() == 1u)) continue;
            for (uint32_t e0 = 0; e0 < (td.jcode() ? 16384u : 4096u); e0 += 4u) {
                if (threads > 256u && e0 >= 4u * threads && e0 / (4u * threads) * (4u * threads) >= td.n_elems) break;   // rows that are left out
                const uint32_t bin = uint32_t((uint64_t(e0) * td.magic) >> 32);
                const uint32_t b0 = td.jcode() ? pack_bin<true>(bin, td.n_bins) : pack_bin<false>(bin, td.n_bins);
                if (b0 + 1u >= kPackBins || (e0 < td.n_elems && b0 != bin)) return 154;
            }
        }
    }
    if (w.total(3) != adacomp_workspace_bytes_batch(t.data(), uint32_t(t.size()), 3)) return 143;
    g_tiles_checked += p.n_ctiles + p.n_utiles;
    g_groups_checked += p.n_ugroups;
    return 0;
}

int main()
{
    uint64_t lcg = 12345;
    auto next = [&lcg]() { lcg = lcg * 6364136223846793005ull + 1442695040888963407ull; return uint32_t(lcg >> 33); };
    const uint32_t lts[] = {1, 2, 3, 7, 50, 63, 64, 65, 500, 4095, 4096, 4097, 8192, 16383, 16384};
    uint64_t checksum = 0;
    for (int rep = 0; rep < 200; ++rep) {
        const uint32_t n_layers = 1 + next() % 40;
        std::vector<adacomp_layer_t> t(n_layers);
        uint64_t off = 0;
        for (auto &l : t) {
            l.elem_offset = off;
            l.n_elems = 1 + next() % (rep % 10 == 0 ? 3000000u : 20000u);
            l.L_T = lts[next() % (sizeof lts / sizeof lts[0])];
            l.reserved = 0;
            off += (l.n_elems + 3) / 4 * 4 + 4 * (next() % 3);
        }
        const size_t bound = adacomp_packet_bound(t.data(), n_layers), fixed = adacomp_packet_fixed_bytes(t.data(), n_layers);
        const size_t ws1 = adacomp_workspace_bytes(t.data(), n_layers), ws5 = adacomp_workspace_bytes_batch(t.data(), n_layers, 5);
        if (!bound || !fixed || fixed > bound || !ws1 || ws5 <= ws1) return 2;
        size_t goff = 0, gn = 0, gstride = 0;
        if (adacomp_workspace_gmax(t.data(), n_layers, &goff, &gn, &gstride) != ADACOMP_OK || goff + 4 * gn > ws1) return 3;
        checksum += bound + fixed + ws1 + gn;
        // tile tables, with the default grouping of unpack tiles and with runs forced on small tables
        adacomp_tuning_unpack_min_groups(rep % 2 ? 1u : 0u);
        const int pc = check_plan(t);
        adacomp_tuning_unpack_min_groups(0);
        if (pc) { std::printf("plan check failed with %d at rep %d\n", pc, rep); return pc; }
        // calls on a workspace that was never initialised return before touching any device
        alignas(256) static char fake[4096];
        const float *g = reinterpret_cast<const float *>(fake);
        float *r = reinterpret_cast<float *>(fake + 1024);
        void *pk = fake + 2048;
        if (adacomp_compress(t.data(), n_layers, g, r, pk, bound, fake + 3072, ws1, nullptr) != ADACOMP_EWORKSPACE) return 4;
        const void *pks[1] = {pk};
        if (adacomp_unpack_accumulate(t.data(), n_layers, pks, 1, r, fake + 3072, ws1, nullptr) != ADACOMP_EWORKSPACE) return 5;
        void *pko[1] = {pk};
        if (adacomp_compress_batch_lazy(t.data(), n_layers, 1, &g, &r, pko, bound, fake + 3072, ws1, nullptr) != ADACOMP_EWORKSPACE) return 9;
        if (adacomp_residue_sync(fake + 3072, nullptr) != ADACOMP_EWORKSPACE || adacomp_residue_sync(nullptr, nullptr) != ADACOMP_EINVAL) return 10;
        // a broken copy of the table is refused
        std::vector<adacomp_layer_t> b = t;
        b[next() % n_layers].L_T = 16385;
        if (adacomp_packet_bound(b.data(), n_layers) != 0) return 6;
        b = t;
        b[0].elem_offset += 2;
        if (adacomp_packet_bound(b.data(), n_layers) != 0) return 7;
        if (n_layers > 1) { b = t; b[1].elem_offset = b[0].elem_offset; if (adacomp_packet_bound(b.data(), n_layers) != 0) return 8; }
    }
    for (uint64_t elems : {1000ull, 5000ull, 397000ull, 2000000ull})
        for (uint32_t lt : {50u, 500u}) {   // workspace_bytes_batch has areas for all learners of the call, up to a launch's
            std::vector<adacomp_layer_t> t = {{0, elems, lt, 0}, {(elems + 3) / 4 * 4, elems / 3, 500, 0}};
            adacomp::Plan p;
            if (adacomp::build_plan(t.data(), 2, false, p) != ADACOMP_OK) return 12;
            for (uint32_t n : {1u, 2u, 8u, 16u, 32u, 56u, 57u, 150u, 300u}) {
                if (elems <= 5000 && n > 2) continue;   // areas for all take more than a scratch block
                const size_t bytes = adacomp_workspace_bytes_batch(t.data(), 2, n);
                if (adacomp::sync_place(p.ws, bytes, SIZE_MAX).learners < std::min(n, adacomp::kMaxBatch)) return 13;
                if (p.ws.least(n + 1) <= bytes) return 14;
            }
        }
    for (uint64_t elems = 240000; elems < 1100000; elems += 3571)   // fewer tiles than compute units wherever tiles of up to 4096 elements make so few
        for (uint32_t lt : {50u, 52u, 500u, 1000u}) {
            const adacomp_layer_t t = {0, elems, lt, 0};
            adacomp::Plan p;
            if (adacomp::build_plan(&t, 1, false, p) != ADACOMP_OK) return 16;
            const uint64_t of_4096 = 4096u / lt / (lt % 4u ? 2u : 1u) * (lt % 4u ? 2u : 1u), least = ((elems + lt - 1u) / lt + of_4096 - 1u) / of_4096;
            if (least < 256u && p.n_ctiles >= 256u) return 17;
        }
    for (uint32_t lt = 4; lt <= 50; ++lt) {   // short bins in tiles of the larger class, as many as such a tile takes
        std::vector<adacomp_layer_t> t = {{0, 9001 * 3 + 1, 9001, 0}, {27008, 1024ull * 70 * lt + 7, lt, 0}};
        adacomp::Plan p;
        if (adacomp::build_plan(t.data(), 2, true, p) != ADACOMP_OK || p.n_class_tiles[0] != 0 || (lt <= 16) != (p.ctiles[4].n_bins == adacomp::kMaxTileBins)) return 15;
        const int pc = check_plan(t);
        if (pc) { std::printf("plan check failed with %d, bins of %u among long ones\n", pc, lt); return pc; }
    }
    {   // the 125 M-element table of the benchmark: runs of 8 tiles that shorten towards the end
        std::vector<adacomp_layer_t> t(7);
        uint64_t off = 0;
        for (int l = 0; l < 7; ++l) { t[l] = adacomp_layer_t{off, l < 6 ? 4096ull * 4096 : 4096ull * 5999, 500, 0}; off += t[l].n_elems; }
        const int pc = check_plan(t);
        if (pc) { std::printf("plan check of the large table failed with %d\n", pc); return pc; }
        adacomp::Plan p;
        adacomp::build_plan(t.data(), 7, true, p);
        uint32_t longest = 0;
        for (const auto &g : p.ugroups) longest = g.n_tiles > longest ? g.n_tiles : longest;
        if (longest != adacomp::kUnpackGroupTiles || p.ugroups.back().n_tiles != 1) return 11;
    }
    {   // a workspace registered for one layer table serves that list of layers and no other: the
        // same table is found, tables of the same length that differ in one field of one layer are
        // refused (the kernels would index the tile tables of the wrong geometry otherwise)
        using namespace adacomp;
        std::vector<adacomp_layer_t> a = {{0, 5000, 50, 0}, {5000, 70000, 500, 0}, {75000, 130, 64, 0}};
        alignas(256) static char fake_ws[256];
        Plan p, found;
        if (build_plan(a.data(), 3, true, p) != ADACOMP_OK) return 20;
        const size_t bytes = p.ws.total(2);
        p.sync = sync_place(p.ws, bytes, SIZE_MAX);
        register_workspace(a.data(), 3, fake_ws, bytes, std::move(p));
        if (find_plan(a.data(), 3, fake_ws, bytes, 2, found) != ADACOMP_OK) return 21;
        if (found.n_ctiles == 0 || found.ws.total(2) != bytes) return 22;
        if (find_plan(a.data(), 3, fake_ws, bytes, 3, found) != ADACOMP_EWORKSPACE) return 23;  // too small for 3 learners
        if (find_plan(a.data(), 3, fake_ws + 16, bytes, 2, found) != ADACOMP_EWORKSPACE) return 24;
        for (int field = 0; field < 3; ++field)
            for (int l = 0; l < 3; ++l) {
                std::vector<adacomp_layer_t> b = a;
                if (field == 0) b[l].L_T += 1;
                if (field == 1) b[l].n_elems -= 1;
                if (field == 2) b[2].elem_offset += 4 * (l + 1);   // the last layer moved up: still no overlap
                if (adacomp_packet_bound(b.data(), 3) == 0) return 25;   // b is a valid table in its own right
                if (find_plan(b.data(), 3, fake_ws, bytes, 2, found) != ADACOMP_EWORKSPACE) return 26;
                const float *g = reinterpret_cast<const float *>(fake_ws);
                if (adacomp_compress(b.data(), 3, g + 4, const_cast<float *>(g) + 8, fake_ws + 64, 1 << 20, fake_ws, bytes, nullptr) !=
                    ADACOMP_EWORKSPACE)
                    return 27;
            }
        if (find_plan(a.data(), 2, fake_ws, bytes, 2, found) != ADACOMP_EWORKSPACE) return 28;  // a prefix of the list
        // polls before a waiting workgroup helps itself: whatever is asked for, the wait ends
        for (uint32_t polls : {0u, 7u, kWaitPollsMax, kWaitPollsMax + 1u, 0xFFFFFFFFu}) {
            if (adacomp_debug_wait_polls(fake_ws, polls) != ADACOMP_OK || find_plan(a.data(), 3, fake_ws, bytes, 2, found) != ADACOMP_OK) return 31;
            if (found.wait_polls != std::min(polls, kWaitPollsMax)) return 32;
        }
        if (adacomp_debug_wait_polls(fake_ws + 16, 1) != ADACOMP_EWORKSPACE) return 33;
        // the route of a call: in one launch, unless that is switched off; nothing for more learners than there is room for
        if (adacomp_debug_one_launch(fake_ws, 2, 0) != 1 || adacomp_debug_one_launch(fake_ws, 1, 1) != 1 || adacomp_debug_one_launch(fake_ws, 3, 0) != ADACOMP_EWORKSPACE ||
            adacomp_debug_one_launch(fake_ws, 0, 0) != ADACOMP_EWORKSPACE || adacomp_debug_one_launch(fake_ws + 16, 1, 0) != ADACOMP_EWORKSPACE) return 34;
        adacomp_tuning_fold_scan(0);
        const int staged = adacomp_debug_one_launch(fake_ws, 1, 0);
        adacomp_tuning_fold_scan(1);
        if (staged != 0) return 35;
        if (adacomp_workspace_release(fake_ws) != ADACOMP_OK) return 29;
        if (find_plan(a.data(), 3, fake_ws, bytes, 2, found) != ADACOMP_EWORKSPACE) return 30;
    }
    {   // one launch only where half of the workgroups that are resident on the stream's compute units (8 on each)
        // hold the tiles that wait for each other: one layer, L_T 500, tiles of 4000 elements
        using namespace adacomp;
        auto route = [](uint32_t tiles, uint32_t layers, uint32_t lt, size_t learners, uint32_t units, bool lazy = false) {
            std::vector<adacomp_layer_t> t(layers);
            for (uint32_t l = 0; l < layers; ++l) t[l] = adacomp_layer_t{uint64_t(l) * 4000 * tiles, 4000ull * tiles, lt, 0};
            Plan p;
            if (build_plan(t.data(), layers, false, p) != ADACOMP_OK) return 99u;
            if (tiles >= 256 && p.layer_tiles_max != tiles) return 98u;
            p.sync = sync_place(p.ws, p.ws.total(learners), SIZE_MAX);
            return one_launch_for(p, learners, p.ws.total(learners), units, lazy);
        };
        if (route(1024, 1, 500, 1, 256) != kOneLaunchLayers || route(1025, 1, 500, 1, 256) != kOneLaunchNever) return 50;
        if (route(512, 2, 500, 8, 256) != kOneLaunchLayers || route(513, 2, 500, 8, 256) != kOneLaunchNever) return 51;
        if (route(512, 1, 500, 1, 128) != kOneLaunchTable || route(513, 1, 500, 1, 128) != kOneLaunchNever) return 52;
        if (route(512, 4, 500, 1, 128) != kOneLaunchLayers || route(513, 4, 50, 4, 128) != kOneLaunchNever) return 53;
        if (route(256, 9, 50, 2, 64) != kOneLaunchLayers || route(257, 9, 50, 2, 64) != kOneLaunchNever) return 54;
        if (route(1024, 1, 50, 1, 32) != kOneLaunchNever || route(300, 2, 500, 1, 32) != kOneLaunchNever) return 55;
        if (route(300, 2, 500, 1, 0) != kOneLaunchNever) return 56;   // the runtime did not say
        // more workgroups than are resident: not the form that reads all records, and none with small tiles
        if (route(256, 2, 500, 4, 256) != kOneLaunchTable || route(256, 2, 500, 5, 256) != kOneLaunchLayers) return 58;
        if (route(512, 1, 500, 4, 256) != kOneLaunchTable || route(512, 1, 50, 40, 256) != kOneLaunchLayers) return 59;
        if (route(60, 1, 500, 8, 256) != kOneLaunchTable || route(60, 1, 500, 10, 256) != kOneLaunchLayers || route(60, 1, 500, 11, 256) != kOneLaunchNever) return 60;   // 240,000 elements: 240 tiles of 1000
        if (route(120, 1, 50, 7, 256) != kOneLaunchTable || route(120, 1, 50, 8, 256) != kOneLaunchLayers || route(120, 1, 50, 30, 256) != kOneLaunchLayers) return 61;    // 267 tiles of 1800
        if (route(120, 1, 500, 6, 256) != kOneLaunchTable || route(120, 1, 500, 8, 256) != kOneLaunchLayers || route(120, 1, 500, 9, 256) != kOneLaunchNever) return 62;   // 320 of 1500
        if (route(3, 20, 50, 32, 256) != kOneLaunchLayers || route(3, 16, 50, 32, 256) != kOneLaunchNever) return 63;   // three staged launches or two
        // several learners without short bins: layers of more than 512 tiles up to four rounds of resident workgroups (8192)
        if (route(1024, 1, 500, 8, 256) != kOneLaunchLayers || route(1024, 1, 500, 9, 256) != kOneLaunchNever || route(600, 1, 500, 13, 256) != kOneLaunchLayers || route(600, 1, 500, 14, 256) != kOneLaunchNever) return 64;
        // lazy calls: up to 24 M elements in all, with tiles of fewer than 1536 elements up to 6 workgroups on a compute unit
        if (route(600, 10, 500, 1, 256, true) != kOneLaunchLayers || route(601, 10, 500, 1, 256, true) != kOneLaunchNever || route(600, 2, 50, 5, 256, true) != kOneLaunchLayers || route(600, 2, 50, 6, 256, true) != kOneLaunchNever) return 65;
        if (route(60, 1, 500, 6, 256, true) != kOneLaunchTable || route(60, 1, 500, 7, 256, true) != kOneLaunchNever || route(60, 1, 500, 7, 256) != kOneLaunchTable || route(120, 1, 50, 6, 256, true) != kOneLaunchTable || route(120, 1, 50, 10, 256, true) != kOneLaunchLayers) return 66;
        // tables of the larger tile class: layers of up to 256 tiles and of as many as the stream has compute units; without
        // short bins up to 3 workgroups on each
        auto large = [](uint32_t tiles, uint32_t layers, uint32_t lt, size_t learners, uint32_t units, bool lazy = false) {
            std::vector<adacomp_layer_t> t(layers + 1);
            for (uint32_t l = 0; l < layers; ++l) t[l] = adacomp_layer_t{uint64_t(l) * 16384 * tiles, 16384ull * tiles, 16384, 0};
            t[layers] = adacomp_layer_t{uint64_t(layers) * 16384 * tiles, 2 * lt, lt, 0};
            Plan p;
            if (build_plan(t.data(), layers + 1, false, p) != ADACOMP_OK) return 99u;
            p.sync = sync_place(p.ws, p.ws.total(learners), SIZE_MAX);
            return one_launch_for(p, learners, p.ws.total(learners), units, lazy);
        };
        if (large(255, 1, 500, 2, 256) != kOneLaunchTable || large(256, 1, 500, 2, 256) != kOneLaunchLayers || large(257, 1, 500, 1, 256) != kOneLaunchNever) return 76;
        if (large(255, 3, 500, 1, 256) != kOneLaunchLayers || large(256, 3, 500, 1, 256) != kOneLaunchNever || large(128, 2, 500, 2, 256) != kOneLaunchLayers || large(128, 2, 500, 3, 256) != kOneLaunchNever) return 77;
        if (large(256, 5, 50, 1, 256) != kOneLaunchLayers || large(257, 5, 50, 1, 256) != kOneLaunchNever || large(100, 3, 50, 32, 256) != kOneLaunchLayers) return 78;
        if (large(100, 1, 50, 1, 128) != kOneLaunchTable || large(128, 2, 50, 1, 128) != kOneLaunchLayers || large(129, 2, 50, 1, 128) != kOneLaunchNever) return 79;
        // tiles half empty: 11 layers of 9000-element bins, 40 bins of L_T 50
        auto half = [](uint32_t tiles, uint32_t lt, size_t learners, bool lazy = false) {
            std::vector<adacomp_layer_t> t(12);
            for (uint32_t l = 0; l < 11; ++l) t[l] = adacomp_layer_t{uint64_t(l) * lt * tiles, uint64_t(lt) * tiles, lt, 0};
            t[11] = adacomp_layer_t{11ull * lt * tiles, 2000, 50, 0};
            Plan p;
            if (build_plan(t.data(), 12, false, p) != ADACOMP_OK || p.n_ctiles != 11 * tiles + 1) return 99u;
            p.sync = sync_place(p.ws, p.ws.total(learners), SIZE_MAX);
            return one_launch_for(p, learners, p.ws.total(learners), 256, lazy);
        };
        if (half(121, 9000, 1, true) != kOneLaunchLayers || half(122, 9000, 1, true) != kOneLaunchNever || half(122, 12300, 1, true) != kOneLaunchLayers) return 86;
        if (half(139, 9000, 2) != kOneLaunchLayers || half(140, 9000, 2) != kOneLaunchNever || half(140, 10012, 2) != kOneLaunchLayers || half(200, 12000, 4) != kOneLaunchLayers) return 85;
        if (large(244, 6, 50, 1, 256, true) != kOneLaunchLayers || large(245, 6, 50, 1, 256, true) != kOneLaunchNever) return 80;   // 24 M elements
    }
    {   // tiles of both classes where no call goes in one launch, but not if long bins hold two fifths of the elements of a table without short ones
        using namespace adacomp;
        auto both = [](uint32_t layers, uint32_t n_long, uint32_t tiles, uint32_t lt, uint32_t lt_long) {   // the same number of elements to each layer
            std::vector<adacomp_layer_t> t(layers);
            for (uint32_t l = 0; l < layers; ++l) t[l] = adacomp_layer_t{16000ull * tiles * l, 16000ull * tiles, l < n_long ? lt_long : lt, 0};
            Plan p;
            if (build_plan(t.data(), layers, true, p) != ADACOMP_OK || check_plan(t)) return 99;
            return p.n_class_tiles[0] != 0u && p.n_class_tiles[1] != 0u ? 1 : p.n_class_tiles[1] != 0u ? 0 : 98;
        };
        if (both(4, 1, 192, 500, 8000) != 0 || both(4, 1, 193, 500, 8000) != 1 || both(4, 2, 193, 500, 8000) != 0 || both(5, 2, 193, 500, 8000) != 0 || both(8, 3, 193, 500, 8000) != 1) return 87;
        if (both(4, 1, 193, 50, 8000) != 0 || both(20, 1, 200, 50, 8000) != 0) return 88;
        if (both(20, 19, 139, 50, 9000) != 1 || both(20, 5, 139, 50, 9000) != 0 || both(10, 9, 139, 50, 9000) != 0) return 89;
    }
    {   // lanes per tile in the placement: 64 with few tiles, with short bins, and in tables of the larger tile class
        using namespace adacomp;
        auto lanes = [](uint64_t elems, uint32_t lt, uint64_t elems_b, uint32_t lt_b) {
            const adacomp_layer_t t[2] = {{0, elems, lt, 0}, {elems, elems_b, lt_b, 0}};
            Plan p;
            return build_plan(t, 2, true, p) == ADACOMP_OK ? place_lanes_for(p) : 0u;
        };
        if (lanes(2047 * 4000, 500, 400, 500) != 64 || lanes(2048 * 4000, 500, 400, 500) != 16 || lanes(5000 * 4000, 500, 400, 50) != 64) return 83;
        if (lanes(3000 * 16000, 8000, 16000, 8000) != 64 || lanes(3000 * 16000, 8000, 5000 * 4000, 500) != 16) return 84;   // (of both classes: layers too long for one launch)
    }
    {   // 512 threads to a tile up to two workgroups on a compute unit, one per learner for the header; bins of 2052: a tile each
        using namespace adacomp;
        auto wide = [](uint64_t tiles, size_t learners, uint32_t units) {
            const adacomp_layer_t t = {0, 2052 * tiles, 2052, 0};
            Plan p;
            return build_plan(&t, 1, false, p) == ADACOMP_OK && p.n_ctiles == tiles && pack_wide_for(p, learners, units);
        };
        if (!wide(511, 1, 256) || wide(512, 1, 256) || !wide(255, 2, 256) || wide(256, 2, 256) || !wide(169, 3, 256) || wide(170, 3, 256) || !wide(15, 32, 256) || !wide(15, 40, 256) || wide(16, 32, 256)) return 81;
        if (!wide(127, 1, 64) || wide(128, 1, 64) || wide(1, 1, 0)) return 82;
    }
    {   // the epochs of an exchange area after two calls that overlapped (both refused results, nothing else): in
        // whatever order the calls read and count, each tile has counted two, and the next call's tiles agree
        uint32_t calls[3] = {7, 7, 7}, a[3], b[3];
        a[0] = calls[0] + 1; adacomp::count_call(calls + 0); b[0] = calls[0] + 1; adacomp::count_call(calls + 0);   // one after the other
        a[1] = calls[1] + 1; b[1] = calls[1] + 1; adacomp::count_call(calls + 1); adacomp::count_call(calls + 1);   // both read first
        b[2] = calls[2] + 1; a[2] = calls[2] + 1; adacomp::count_call(calls + 2); adacomp::count_call(calls + 2);
        for (int t = 0; t < 3; ++t)
            if (calls[t] != 9 || a[t] > 9 || b[t] > 9) return 57;
    }
    {   // k_unpack8: a workgroup's LDS is that of its chunks (256 bytes per element of the longest 8-bit bin each), and
        // the 16-bit groups beside them have the same: where those are many they keep 5 of the 6 workgroups that
        // k_unpack has on a compute unit (160 KB), and the launch stays inside the 64 KB of a workgroup
        using namespace adacomp;
        Plan p;
        for (uint32_t T = 1; T <= 64; ++T)
            for (uint32_t n8 : {1u, 17u, 1000u, 20000u})
                for (uint32_t n16 : {0u, 1u, 60u, 900u, 3500u, 70000u})
                    for (uint32_t tiles_per_group : {1u, 2u, 4u}) {
                        p.short_bin_max = T;
                        p.n_usingles8 = n8;
                        p.n_utiles = n8 + n16 * tiles_per_group;
                        const uint32_t log = unpack8_wg_log(p, n8, n16, 1), lds = std::max(24644u, 256u * T << log);
                        if (log > 2 || lds > 65536 || (n16 == 0 && log != 2)) return 40;
                        if (n16 > 3 * n8 && 163840 / lds < 5) return 41;
                        if (T > 40 && n16 > n8 && 163840 / lds < 5) return 42;
                        if (163840 / lds < 3) { if (T <= 53 || 2 * n16 > n8) return 43; }
                    }
    }
    {   // workgroups per compute unit of the launches over 16-bit layers: fewer than fit only where tiles are full and bins
        // have elements enough for the packets (one layer; n_bins of L_T elements, a power of two of them to a tile of up to 4096)
        using namespace adacomp;
        auto held = [](uint64_t elems, uint32_t lt, uint32_t learners, uint32_t mode) {
            const adacomp_layer_t t = {0, elems, lt, 0};
            Plan p;
            if (build_plan(&t, 1, true, p) != ADACOMP_OK || p.n_elems16 != elems || p.n_usingles8 != 0) return 99u;
            return resident_for(p.n_elems16, p.n_bins16, p.n_utiles, learners, mode);
        };
        const uint64_t M = 1000000;
        if (held(40 * M, 500, 8, 2) != 4 || held(40 * M, 500, 9, 2) != 5 || held(40 * M, 500, 16, 2) != 5 || held(40 * M, 500, 21, 2) != 0 || held(11 * M, 500, 1, 2) != 0) return 70;
        if (held(40 * M, 100, 4, 2) != 5 || held(40 * M, 100, 5, 2) != 0 || held(40 * M, 65, 1, 2) != 0 || held(40 * M, 300, 4, 2) != 5 || held(40 * M, 300, 5, 2) != 0 || held(40 * M, 9000, 16, 2) != 4 || held(40 * M, 3000, 16, 2) != 5) return 71;
        if (held(40 * M, 500, 8, 1) != 5 || held(40 * M, 500, 9, 1) != 0 || held(40 * M, 200, 3, 1) != 5 || held(40 * M, 200, 4, 1) != 0 || held(40 * M, 65, 1, 1) != 0) return 72;
        if (held(40 * M, 700, 4, 1) != 5 || held(40 * M, 700, 5, 1) != 0 || held(40 * M, 3000, 8, 1) != 5 || held(11 * M, 500, 1, 1) != 0 || held(12 * M, 500, 1, 1) != 5) return 73;
        if (held(24 * M, 500, 4, 0) != 5 || held(24 * M, 500, 5, 0) != 0 || held(40 * M, 500, 8, 0) != 5 || held(40 * M, 500, 9, 0) != 0 || held(23 * M, 500, 4, 0) != 0) return 74;
        if (held(40 * M, 100, 2, 0) != 5 || held(40 * M, 100, 3, 0) != 0 || held(40 * M, 65, 1, 0) != 0 || held(40 * M, 200, 4, 0) != 5 || held(40 * M, 9000, 5, 0) != 0 || held(40 * M, 300, 4, 0) != 5 || held(40 * M, 150, 4, 0) != 0) return 75;
    }
    {   // ... and of sums of one or two packets over 8-bit layers, alone or with 16-bit ones in the launch: fewer only where the tiles of
        // the former are full, and 4 (with two packets any) only where bins of the latter are not short too
        using namespace adacomp;
        auto held = [](uint64_t elems8, uint32_t lt8, uint64_t elems16, uint32_t lt16, uint32_t learners, uint64_t elems8b = 0, uint32_t lt8b = 64) {
            std::vector<adacomp_layer_t> t;
            uint64_t off = 0;
            for (auto l : {std::make_pair(elems8, lt8), std::make_pair(elems16, lt16), std::make_pair(elems8b, lt8b)})
                if (l.first != 0) { t.push_back(adacomp_layer_t{off, l.first, l.second, 0}); off += (l.first + 3) / 4 * 4; }
            Plan p;
            if (build_plan(t.data(), uint32_t(t.size()), true, p) != ADACOMP_OK) return 99u;
            return unpack_hold_sum8(p.n_elems_total - p.n_elems16, p.n_usingles8, p.n_elems16, p.n_bins16, learners);
        };
        const uint64_t M = 1000000;
        if (held(25 * M, 64, 0, 0, 1) != 4 || held(25 * M, 54, 0, 0, 1) != 5 || held(23 * M, 64, 0, 0, 1) != 0 || held(33 * M, 64, 0, 0, 2) != 5 || held(25 * M, 64, 0, 0, 2) != 0 || held(2 * M, 64, 22 * M, 500, 2) != 5 || held(2 * M, 64, 21 * M, 500, 2) != 0 || held(8 * M, 64, 17 * M, 500, 2) != 0 || held(60 * M, 60, 0, 0, 2) != 0 || held(8 * M, 33, 32 * M, 500, 2) != 0 || held(60 * M, 64, 0, 0, 3) != 0 || held(60 * M, 64, 0, 0, 0) != 0) return 76;
        if (held(30 * M, 20, 0, 0, 1, 30 * M) != 0 || held(57 * M, 20, 0, 0, 1, 3 * M) != 0 || held(20 * M, 33, 0, 0, 1, 20 * M) != 0 || held(27 * M, 20, 30 * M, 500, 1, 3 * M) != 0 || held(6 * M, 20, 53 * M, 2000, 1, M) != 5) return 77;
        if (held(2 * M, 64, 38 * M, 65, 1) != 5 || held(2 * M, 64, 38 * M, 77, 1) != 5 || held(2 * M, 64, 38 * M, 79, 1) != 4 || held(30 * M, 64, 10 * M, 65, 1) != 4 || held(2 * M, 64, 38 * M, 129, 1) != 4 || held(20 * M, 64, 20 * M, 65, 1) != 5 || held(38 * M, 64, 2 * M, 65, 1) != 4) return 78;
        if (held(2 * M, 64, 38 * M, 65, 2) != 0 || held(20 * M, 64, 20 * M, 70, 2) != 0 || held(2 * M, 64, 38 * M, 76, 2) != 5 || held(2 * M, 64, 38 * M, 500, 2) != 5 || held(38 * M, 64, 2 * M, 65, 2) != 5) return 79;
    }
    {   // ... over 8-bit layers alone: by the lines of 128 bytes that the layers begin on, the tiles' fill and the number of elements
        using namespace adacomp;
        auto held = [](uint64_t elems, uint32_t lt, uint32_t layers, uint64_t first, uint32_t learners) {   // layers of equal size, the next `first` elements after the end of one
            std::vector<adacomp_layer_t> t;
            const uint64_t each = elems / layers / 32 * 32;
            for (uint32_t i = 0; i < layers; ++i) t.push_back(adacomp_layer_t{first + i * (each + first), each, lt, 0});
            Plan p;
            if (build_plan(t.data(), layers, true, p) != ADACOMP_OK) return 99u;
            return unpack_hold_sum8_alone(p.n_elems_total, p.n_usingles8, 2 * p.n_elems8_lines >= p.n_elems_total, learners);
        };
        const uint64_t M = 1000000;
        for (uint64_t on : {uint64_t(0), uint64_t(32), uint64_t(64)})
            if (held(19 * M, 64, 10, on, 1) != 5 || held(17 * M, 64, 10, on, 1) != 0 || held(60 * M, 55, 10, on, 1) != 5 || held(125 * M, 64, 3, on, 2) != 0 || held(25 * M, 48, 10, on, 1) != 0) return 168;
        for (uint64_t off : {uint64_t(4), uint64_t(20)}) {
            if (held(19 * M, 64, 1, off, 1) != 4 || held(60 * M, 55, 1, off, 1) != 4 || held(60 * M, 54, 1, off, 1) != 5 || held(17 * M, 64, 1, off, 1) != 0) return 169;
            if (held(19 * M, 64, 1, off, 2) != 5 || held(17 * M, 64, 1, off, 2) != 0 || held(60 * M, 60, 1, off, 2) != 5 || held(60 * M, 59, 1, off, 2) != 0 || held(60 * M, 64, 1, off, 3) != 0 || held(60 * M, 64, 1, off, 0) != 0) return 170;
        }
        if (held(25 * M, 64, 8, 4, 2) != 5 || held(25 * M, 64, 2, 4, 2) != 5 || held(25 * M, 20, 4, 4, 1) != 0) return 171;
    }
    {   // launches that fetch weights and moments ahead of the adds, of which there are none: refused before anything is launched
        using namespace adacomp;
        UnpackArgs a{};
        a.n_groups = 1;
        auto refused = [&a](uint32_t learners, uint32_t mode, int kind) { a.n_learners = learners; a.mode = mode; return launch_unpack(a, kind, 0u, true, nullptr) == ADACOMP_EINVAL; };
        if (!refused(17, 1, 0) || !refused(64, 2, 0) || !refused(9, 1, 1) || !refused(9, 2, 2) || !refused(0, 1, 0) || !refused(4, 0, 0) || !refused(4, 1, 3)) return 164;
    }
    {   // where weights and moments are fetched ahead of the adds: tables of one layer, both sides of each line
        using namespace adacomp;
        auto early = [](uint64_t elems, uint32_t lt, uint32_t learners, uint32_t mode) {
            std::vector<adacomp_layer_t> t{{0, elems, lt, 0}};
            Plan p;
            if (build_plan(t.data(), 1, true, p) != ADACOMP_OK) return false;
            return unpack_early_for(elems, p.n_bins_total, p.n_utiles, lt <= 64, learners, mode);
        };
        const uint64_t M = 1000000;
        for (uint32_t n = 1; n <= 16; ++n) if (early(M, 500, n, 1) || early(M, 500, n, 2) || early(2 * M, 500, n, 0)) return 160;
        for (uint32_t n = 1; n <= 2; ++n) {
            if (!early(2 * M, 500, n, 1) || !early(11 * M, 500, n, 1) || early(12 * M, 500, n, 1) || early(125 * M, 500, n, 1) || early(25 * M, 1023, n, 1) || !early(25 * M, 1365, n, 1) || !early(60 * M, 9000, n, 1)) return 161;
            if (early(8 * M, 20, n, 1) || !early(8 * M, 33, n, 1) || early(25 * M, 14, n, 1) || early(25 * M, 64, n, 1)) return 162;
            if (!early(2 * M, 500, n, 2) || !early(125 * M, 500, n, 2) || early(25 * M, 20, n, 2) || !early(25 * M, 50, n, 2) || early(25 * M, 65, n, 2) || !early(25 * M, 100, n, 2)) return 163;
        }
        for (uint32_t n = 3; n <= 4; ++n) if (!early(2 * M, 18, n, 1) || !early(2 * M, 18, n, 2) || !early(60 * M, 64, n, 2) || early(60 * M, 65, n, 2) || !early(60 * M, 65, n, 1) || !early(60 * M, 100, n, 2)) return 165;
        for (uint32_t n = 5; n <= 8; ++n) for (uint32_t m = 1; m <= 2; ++m) if (early(25 * M, 33, n, m) || !early(25 * M, 50, n, m) || early(25 * M, 65, n, m) || !early(25 * M, 500, n, m)) return 166;
        for (uint32_t n : {9u, 16u}) for (uint32_t m = 1; m <= 2; ++m) if (early(25 * M, 64, n, m) || early(25 * M, 150, n, m) || !early(25 * M, 500, n, m) || early(25 * M, 500, 17, m)) return 167;
    }
    if (adacomp_selftest_binindex() != 0) return 9;
    for (int c = 1; c > -9; --c) if (!adacomp_strerror(c)) return 10;
    std::printf("api sanitizer driver ok, checksum %llu, %llu tiles and %llu groups checked\n", (unsigned long long)checksum,
                (unsigned long long)g_tiles_checked, (unsigned long long)g_groups_checked);
    return 0;
}
