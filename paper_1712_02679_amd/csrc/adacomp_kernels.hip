// adacomp_kernels.hip -- the hot path of libadacomp as hand-written HIP for gfx950 (CDNA4,
// wave64).  Everything here is bound by HBM traffic, not arithmetic: there is no dense
// contraction, hence no MFMA.  The floating-point work of the default method is single additions
// and subtractions in float32 (no multiplies, nothing to contract) plus one float64 sum and divide
// per layer; the soft-threshold factor of the variant entry point adds one multiply per element,
// the fused optimizer step a handful of separate float32 operations per element.
//
// adacomp_compress runs one launch, k_pack, on tables whose layers are small enough that the tiles of
// a layer are on the GPU together (see there), and three on the others:
//   k_fused  (streaming, dominant)  one pass over dW and the residue: G = R + dW, H = G + dW, the
//            per-bin maximum of |G|, the selection compare, and R <- G, all while the tile sits
//            in registers (Algorithm 2 of the AdaComp paper, both loops; selection is local to a
//            bin, so nothing outside the tile is needed).  Selected elements leave as 16-bit
//            (tile-local index, sign) entries in a staging area, counts per bin go straight into
//            the packet, g_max and its per-tile float64 sum go to scratch.
//   k_scan   one workgroup per layer: the layer scale = average of the g_max vector (section
//            "Pseudo code") and the exclusive scan of per-tile word counts.  (Small tables: no
//            launch; every k_place workgroup works these out itself.)
//   k_place  16 or 64 lanes per tile: moves the staged entries to their final place in the packet
//            as (index-in-bin, ternary code) words and applies the only step that needs the
//            layer-wide scale, residue <- G - Gq at the sent elements (a read-modify-write of
//            about 0.3-10 % of the elements); one extra workgroup writes header and records.
//            Large tables with short bins (L_T <= 64), which send several percent of their elements,
//            use k_place_tiled instead: a workgroup per tile, the residue corrected line by line.
// adacomp_compress_batch_lazy runs the same three, or k_pack on small tables and few learners, but leaves the
// residue corrections out; the next call's k_fused or k_pack applies them to the residue values while it has
// them in registers (same arithmetic, same results; adacomp_residue_sync writes them on request).
// adacomp_unpack_accumulate is one launch: k_unpack, up to four packets k_unpack_few, and where layers with short
// bins have many chunks k_unpack8 (large tables of both word widths and more than eight packets take two launches of
// k_unpack): a workgroup owns a tile of the dense output in LDS, a lane group owns each bin and adds the learners' +-scale in learner order, then the
// tile is written out once with coalesced float4 stores; neighbouring tiles share a workgroup
// and the per-bin bookkeeping.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "adacomp_plan.h"

namespace adacomp {

// ---- small device helpers --------------------------------------------------------------------
// Streaming (non-temporal) 16-byte accesses: every element of dW and the residue is touched once
// per call, so nothing is gained by keeping it in L2, and on MI355X the streaming hint is worth
// about 15 % of bandwidth on a read-read-write pass.
typedef float vfloat4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ vfloat4 load_stream4(const float *p) { return __builtin_nontemporal_load(reinterpret_cast<const vfloat4 *>(p)); }
__device__ __forceinline__ void store_stream4(float *p, vfloat4 v) { __builtin_nontemporal_store(v, reinterpret_cast<vfloat4 *>(p)); }

// The same accesses as raw buffer instructions, for k_pack and for the optimizer's epilogues, which stream two or three arrays in and out per
// tile: addressing through a descriptor (scalar base, 32-bit offset) takes fewer registers there than 64-bit addresses, and needs no
// alignment but the element's (k_fused and the plain sum measured the same with them).  A descriptor covers one tile:
// base = the tile's first element, size = its bytes; an access past the tile is dropped by the
// hardware.
typedef uint32_t vuint4 __attribute__((ext_vector_type(4)));
constexpr int kAuxStream = 2;  // cache-policy bits of a buffer access on gfx94x / gfx950: 1 = sc0, 2 = nt, 16 = sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_buffer(const float *base, uint32_t n_elems)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, int(n_elems * 4u), 0x00020000);
}
__device__ __forceinline__ vfloat4 buffer_load_stream4(__amdgpu_buffer_rsrc_t rsrc, uint32_t elem)
{
    return __builtin_bit_cast(vfloat4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, int(elem * 4u), 0, kAuxStream));
}
__device__ __forceinline__ void buffer_store_stream4(__amdgpu_buffer_rsrc_t rsrc, uint32_t elem, vfloat4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(vuint4, v), rsrc, int(elem * 4u), 0, kAuxStream);
}
// a slot at byte offset `lane_at` (per lane) + `row_at` (uniform) of a tile
__device__ __forceinline__ vfloat4 buffer_load_slot(__amdgpu_buffer_rsrc_t rsrc, uint32_t lane_at, uint32_t row_at)
{
    return __builtin_bit_cast(vfloat4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, int(lane_at), int(row_at), kAuxStream));
}
// A store of 16 bytes reads its registers after it has been issued.  The compiler keeps what overwrites them two wait states away, but not
// from a store that has its offset in a scalar register, as these have: built with such an overwrite right behind the store, lanes
// 12 .. 15 of each 16 stored the new value in place of the first of their four now and then, on a busy GPU.  The s_nop is those wait
// states, and names the registers, so that nothing can write them before it.
__device__ __forceinline__ void buffer_store_slot(__amdgpu_buffer_rsrc_t rsrc, uint32_t lane_at, uint32_t row_at, vfloat4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(vuint4, v), rsrc, int(lane_at), int(row_at), kAuxStream);
    asm volatile("s_nop 1" :: "v"(v));
}
// one element through the same descriptor (the first and last slot of a tile that is not 16-byte aligned)
__device__ __forceinline__ float buffer_load1(__amdgpu_buffer_rsrc_t rsrc, uint32_t elem)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, int(elem * 4u), 0, 0));
}
__device__ __forceinline__ void buffer_store1(__amdgpu_buffer_rsrc_t rsrc, uint32_t elem, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rsrc, int(elem * 4u), 0, 0);
}

// A record of a table that does not change while a kernel runs, the same for all threads: scalar loads.
// (Behind a store the compiler takes a vector register per word otherwise.)
typedef uint32_t vuint2 __attribute__((ext_vector_type(2)));
typedef uint32_t vuint8 __attribute__((ext_vector_type(8)));
typedef uint32_t vuint16 __attribute__((ext_vector_type(16)));
template <class V, class T>
__device__ __forceinline__ T table_record(const T *p)
{
    static_assert(sizeof(V) == sizeof(T), "record size");
    return __builtin_bit_cast(T, *(const __attribute__((address_space(4))) V *)p);
}
template <class V>
__device__ __forceinline__ V packet_field(const uint8_t *p) { return *(const __attribute__((address_space(4))) V *)p; }


__device__ __forceinline__ uint32_t bin_of(uint32_t e, uint32_t L_T, uint32_t magic)
{
    return L_T == 1u ? e : __umulhi(e, magic);
}

// Inclusive prefix sum over the 64 lanes of a wave with DPP moves (no LDS traffic): four
// shift-and-add steps inside each row of 16 lanes, then the row totals are carried over with the
// two row broadcasts (lane 15 of rows 0 and 2 into rows 1 and 3, lane 31 into rows 2 and 3).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x111, 0xF, 0xF, false));  // row_shr:1
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x112, 0xF, 0xF, false));  // row_shr:2
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x114, 0xF, 0xF, false));  // row_shr:4
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x118, 0xF, 0xF, false));  // row_shr:8
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x142, 0xA, 0xF, false));  // row_bcast:15 -> rows 1, 3
    v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x143, 0xC, 0xF, false));  // row_bcast:31 -> rows 2, 3
    return v;
}

// Sum over the 64 lanes, in every lane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return uint32_t(__builtin_amdgcn_readlane(int(wave_incl_scan(v)), 63)); }

// Maximum over the 64 lanes, in every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    auto take = [&](int o) { v = uint32_t(o) > v ? uint32_t(o) : v; };
    take(__builtin_amdgcn_update_dpp(0, int(v), 0x111, 0xF, 0xF, true));   // row_shr:1, 2, 4, 8: lane 15 of a row has the row's
    take(__builtin_amdgcn_update_dpp(0, int(v), 0x112, 0xF, 0xF, true));
    take(__builtin_amdgcn_update_dpp(0, int(v), 0x114, 0xF, 0xF, true));
    take(__builtin_amdgcn_update_dpp(0, int(v), 0x118, 0xF, 0xF, true));
    take(__builtin_amdgcn_update_dpp(0, int(v), 0x142, 0xA, 0xF, false));  // row_bcast:15 -> rows 1, 3
    take(__builtin_amdgcn_update_dpp(0, int(v), 0x143, 0xC, 0xF, false));  // row_bcast:31 -> rows 2, 3
    return uint32_t(__builtin_amdgcn_readlane(int(v), 63));
}

// Sum of one double per lane, in every lane, in a fixed order: lane i with lane i ^ 32, then ^ 16, ^ 8, ^ 4, ^ 2,
// ^ 1.  Moves inside the vector registers and no LDS, since a sum stands in every chain that other workgroups wait
// for (with ds_bpermute / with these, in us: 397 k elements 9.7 / 8.9, the CIFAR table 11.5 / 10.6, ResNet-50's 64.0 / 62.5).
__device__ __forceinline__ double f64_of(uint32_t lo, uint32_t hi) { return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo); }
template <int ROR>
__device__ __forceinline__ double row_turned(double v)   // of the lane ROR further in the same row of 16
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return f64_of(uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(b)), 0x120 | ROR, 0xF, 0xF, false)),
                  uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(b >> 32)), 0x120 | ROR, 0xF, 0xF, false)));
}
__device__ __forceinline__ double wave_sum_f64(double v)
{
    uint64_t b = __builtin_bit_cast(uint64_t, v);
    auto lo = __builtin_amdgcn_permlane32_swap(uint32_t(b), uint32_t(b), false, false);
    auto hi = __builtin_amdgcn_permlane32_swap(uint32_t(b >> 32), uint32_t(b >> 32), false, false);
    v = f64_of(lo[0], hi[0]) + f64_of(lo[1], hi[1]);
    b = __builtin_bit_cast(uint64_t, v);
    lo = __builtin_amdgcn_permlane16_swap(uint32_t(b), uint32_t(b), false, false);
    hi = __builtin_amdgcn_permlane16_swap(uint32_t(b >> 32), uint32_t(b >> 32), false, false);
    v = f64_of(lo[0], hi[0]) + f64_of(lo[1], hi[1]);
    v += row_turned<8>(v);   // from here on the values repeat every 8, 4, 2 lanes, so that turning the row is the exchange
    v += row_turned<4>(v);
    v += row_turned<2>(v);
    v += row_turned<1>(v);
    return v;
}

// ==============================================================================================
// k_fused: Algorithm 2, both loops, on a tile of whole bins held in registers.
// Thread t owns float4 slots t, t + WG, ...: element e = 4 * (j * WG + t) + c of the tile, with WG = 256
// threads and 4 slots each for tiles of 4096 elements, 1024 threads and 4 slots each for tiles of 16384.
// ==============================================================================================
// VARIANT = false is the method as built by default (union rule, factor 2: additions only);
// VARIANT = true takes the selection rule and the soft-threshold factor from the arguments.
// LAZY = true: the residue corrections of the learner's previous call (residue <- G - Gq at the
// elements it sent) are still waiting in the scratch block instead of having been written (the host
// knows); they are applied here, to the residue values in registers, before anything else.
// SHIFT = true (launches over tiles of 16384 elements that hold bins of an odd length, or of twice an
// odd length): a tile that starts `skip` = 1..3 elements past a 16-byte boundary still moves whole
// 16-byte slots.  Slot q of the tile then covers the elements 4 q - skip .. 4 q + 3 - skip: the first
// slot begins in the tile before (those elements are left alone: loaded as zero, never stored) and
// everything after it is aligned.  With 4-byte accesses such tiles streamed at 44 % of the HBM peak.
template <int J, int WAVES, bool VARIANT, bool LAZY, bool SHIFT>
__device__ __forceinline__ void fused_tile(const CompressArgs &a)
{
    static_assert(!(SHIFT && LAZY), "the lazy kernel keeps 4-byte accesses on unaligned tiles");
    constexpr uint32_t WG = uint32_t(WAVES) * 64u;  // threads of the workgroup: a tile is J * WG float4 slots
    static_assert(J * WAVES <= 64, "the per-row word totals are scanned by one wave");
    // one-dimensional grid, learner-major: workgroups are dispatched in index order, so a batched
    // call streams one learner's buffers after the other instead of all of them at once.  A launch
    // covers the class_count tiles of one register class (all tiles, for most tables).
    const uint32_t lq = blockIdx.x / a.class_count;
    uint32_t pos = blockIdx.x - lq * a.class_count;
    const uint32_t lr = a.fused_first + lq;
    // Workgroups go to the 8 XCDs round-robin by index.  Inside each run of 64 the mapping is
    // transposed, so that the 8 workgroups landing on one XCD take 8 consecutive tiles (128 KB of
    // each stream): measured 6-9 % faster than the identity on a plain triad with these tiles,
    // and free of the slowdown of long launches.
    if (pos < (a.class_count & ~63u)) pos = (pos & ~63u) | ((pos & 7u) << 3) | ((pos >> 3) & 7u);
    const uint32_t tile = a.class_tiles ? a.class_tiles[a.class_first + pos] : pos;
    const TileDev td = a.tiles[tile];
    // The layer's record is needed only at the end, for the tile's outputs, but a dependent load in
    // the tail adds its whole latency to the life of the workgroup, so it is fetched early.  The
    // 256-thread kernel fetches it here, which holds its streaming loads back until the record is in
    // (they wait for the same counter as the buffer pointers); measured, that is as fast or faster
    // than the fetch behind the loads.  The 1024-thread kernel, of which a compute unit holds two
    // workgroups, cannot hide that wait (a third longer per launch) and fetches behind its loads
    // (2-4 % faster than in the tail).
    LayerDev ld;
    if (WAVES == 4) ld = a.layers[td.layer()];
    uint8_t *const sb = a.scratch + uint64_t(lr) * a.scratch_stride;
    TileOut *const tile_out = reinterpret_cast<TileOut *>(sb + a.o_tile_out);
    float *const gmax_out = reinterpret_cast<float *>(sb + a.o_gmax);
    uint32_t *const chunk_rel = reinterpret_cast<uint32_t *>(sb + a.o_chunk_rel);
    uint16_t *const stage_all = reinterpret_cast<uint16_t *>(sb + a.o_stage);
    uint8_t *const packet = a.packet[lr];

    __shared__ uint32_t s_gmax[kMaxTileBins];  // bit pattern of max |G|: for non-negative floats the
    __shared__ uint32_t s_cnt[kMaxTileBins];   // unsigned integer order is the float order
    __shared__ uint32_t s_wtot[64];
    __shared__ double s_red[WAVES];

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform across the wave
    const uint32_t n = td.n_elems, T = td.L_T, M = td.magic, nb = td.n_bins;
    const uint32_t skip = SHIFT ? td.skip() : 0u;         // elements of the first slot that belong to the tile before
    const bool vec = td.aligned() || (SHIFT && skip != 0u);

    for (uint32_t i = tid; i < nb; i += WG) { s_gmax[i] = 0u; s_cnt[i] = 0u; }

    const float *__restrict__ gr = a.grad[lr] + td.elem_base;
    float *__restrict__ rs = a.residue[lr] + td.elem_base;

    // ---- G <- residue + dW ; H <- G + dW ; residue <- G (the "no transmission" value) ----------
    float r[J][4], w[J][4];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const uint32_t f0 = (uint32_t(j) * WG + tid) * 4u;
        const uint32_t e0 = f0 - skip;   // wraps to a huge value in the first slot of a shifted tile: its valid elements wrap back
        if (vec && f0 >= skip && e0 + 4u <= n) {
            const vfloat4 rv = load_stream4(rs + e0);
            const vfloat4 wv = load_stream4(gr + e0);
            r[j][0] = rv.x; r[j][1] = rv.y; r[j][2] = rv.z; r[j][3] = rv.w;
            w[j][0] = wv.x; w[j][1] = wv.y; w[j][2] = wv.z; w[j][3] = wv.w;
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const bool ok = e0 + uint32_t(c) < n;
                r[j][c] = ok ? rs[e0 + c] : 0.f;
                w[j][c] = ok ? gr[e0 + c] : 0.f;
            }
        }
    }
    if (WAVES != 4) ld = a.layers[td.layer()];
    if (LAZY) {
        // The previous call left, for this tile, its staged entries (tile-local index, sign), their
        // number and the layer's scale.  An entry becomes a code byte in LDS at the element's place;
        // every thread then reads the four codes of each of its slots and corrects its residues:
        // the same single float32 subtraction or addition that the eager placement performs.
        __shared__ __attribute__((aligned(16))) uint8_t s_fix[J * WG * 4];
        const TileOut prev = tile_out[tile];
        const uint32_t prev_count = prev.count;
        const float prev_scale = __uint_as_float(prev.base);
        for (uint32_t i = tid; i < uint32_t(J) * WG / 4u; i += WG) reinterpret_cast<uint4 *>(s_fix)[i] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        // four entries per load: a tile's stretch of the staging area starts on an 8-byte boundary
        // (stretches are multiples of 4 entries) and what lies behind its last entry is readable
        const uint2 *prev_stage = reinterpret_cast<const uint2 *>(stage_all + td.stage_base);
        const uint32_t prev_n = prev_count < n ? prev_count : n;
        for (uint32_t q = tid; 4u * q < prev_n; q += WG) {
            const uint2 v = prev_stage[q];
            const uint32_t entry[4] = {v.x & 0xFFFFu, v.x >> 16, v.y & 0xFFFFu, v.y >> 16};
#pragma unroll
            for (uint32_t i = 0; i < 4u; ++i)
                if (4u * q + i < prev_n && (entry[i] >> 2) < n) s_fix[entry[i] >> 2] = uint8_t(entry[i] & 3u);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const uint32_t e0 = (uint32_t(j) * WG + tid) * 4u;
            const uint32_t codes = *reinterpret_cast<const uint32_t *>(&s_fix[e0]);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t code = (codes >> (8 * c)) & 3u;
                if (code == 1u) r[j][c] = r[j][c] - prev_scale;
                else if (code == 3u) r[j][c] = r[j][c] + prev_scale;
            }
        }
    }
    uint32_t gb[J][4];  // bits of G (sign included)
    uint32_t mb[J][4];  // bits of max(|G|, |H|): what is compared with g_max
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const uint32_t f0 = (uint32_t(j) * WG + tid) * 4u;
        const uint32_t e0 = f0 - skip;
        float G[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            G[c] = r[j][c] + w[j][c];
            float H;
            if (VARIANT) {
                const float extra = a.soft_factor_minus_1 * w[j][c];  // residue + f dW = G + (f - 1) dW
                H = G[c] + extra;
            } else {
                H = G[c] + w[j][c];
            }
            gb[j][c] = __float_as_uint(G[c]);
            const uint32_t ag = gb[j][c] & 0x7FFFFFFFu, ah = __float_as_uint(H) & 0x7FFFFFFFu;
            if (VARIANT && a.rule == ADACOMP_RULE_PRINTED_COMPARE) mb[j][c] = ah;          // |H| alone
            else if (VARIANT && a.rule == ADACOMP_RULE_LOCAL_SELECTION) mb[j][c] = ag;     // bin maxima only
            else mb[j][c] = ag > ah ? ag : ah;
        }
        if (vec && f0 >= skip && e0 + 4u <= n) {
            store_stream4(rs + e0, vfloat4{G[0], G[1], G[2], G[3]});
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (e0 + uint32_t(c) < n) rs[e0 + c] = G[c];
        }
    }

    __syncthreads();  // LDS arrays are zeroed

    // ---- first loop of Algorithm 2: g_max(i) per bin -------------------------------------------
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const uint32_t f0 = (uint32_t(j) * WG + tid) * 4u;
        const uint32_t e0 = f0 - skip;
        if (WAVES == 16) {
            // Long bins: the 256 elements of a wave's row of slots nearly always lie in one bin, and
            // 64 lanes that bring their maxima to one LDS address are served one after the other
            // (2 cycles each, measured).  The wave reduces first; one lane goes to the LDS.
            const uint32_t w0f = (uint32_t(j) * WG + wave * 64u) * 4u;  // uniform: first slot of the row
            const uint32_t w0 = w0f - skip;                              // its first element (the row that holds a shifted tile's first slot takes the path below)
            if (w0f >= skip && w0 < n) {
                const uint32_t w1 = w0 + 255u < n ? w0 + 255u : n - 1u;
                const uint32_t bw = bin_of(w0, T, M);
                if (bw == bin_of(w1, T, M)) {
                    uint32_t m = gb[j][0] & 0x7FFFFFFFu;   // elements past n hold G = 0
#pragma unroll
                    for (int c = 1; c < 4; ++c) { const uint32_t v = gb[j][c] & 0x7FFFFFFFu; m = v > m ? v : m; }
#pragma unroll
                    for (uint32_t d = 32; d > 0; d >>= 1) { const uint32_t o = __shfl_xor(m, d, 64); m = o > m ? o : m; }
                    if (lane == 0) atomicMax(&s_gmax[bw], m);
                    continue;
                }
            }
        }
        if (SHIFT && f0 < skip) {   // the first slot of a shifted tile: only the elements from skip on are the tile's
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (e0 + uint32_t(c) < n) atomicMax(&s_gmax[bin_of(e0 + c, T, M)], gb[j][c] & 0x7FFFFFFFu);
        } else if (e0 < n) {
            const uint32_t e3 = e0 + 3u < n ? e0 + 3u : n - 1u;
            const uint32_t b0 = bin_of(e0, T, M), b3 = bin_of(e3, T, M);
            if (b0 == b3) {
                uint32_t m = gb[j][0] & 0x7FFFFFFFu;   // elements past n hold G = 0: they never raise a maximum
#pragma unroll
                for (int c = 1; c < 4; ++c) { const uint32_t v = gb[j][c] & 0x7FFFFFFFu; m = v > m ? v : m; }
                atomicMax(&s_gmax[b0], m);
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (e0 + uint32_t(c) < n) atomicMax(&s_gmax[bin_of(e0 + c, T, M)], gb[j][c] & 0x7FFFFFFFu);
            }
        }
    }
    __syncthreads();

    // ---- second loop: the local-max compare.  Sent iff G != 0 and max(|H|, |G|) >= g_max -------
    uint32_t before[J];  // sent elements of this wave's slot row that precede this lane
    uint32_t flags[J];   // bit c: element c of the slot is sent
    uint32_t wtot[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const uint32_t f0 = (uint32_t(j) * WG + tid) * 4u;
        const uint32_t e0 = f0 - skip;
        uint32_t f = 0u;
        if (e0 < n || (SHIFT && f0 < skip)) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t e = e0 + uint32_t(c);
                if (e < n) {
                    const uint32_t gm = s_gmax[bin_of(e, T, M)];
                    // the printed compare alone also sends elements whose G is zero
                    const bool nonzero = (gb[j][c] & 0x7FFFFFFFu) != 0u ||
                                         (VARIANT && a.rule == ADACOMP_RULE_PRINTED_COMPARE);
                    const bool sent = nonzero && (mb[j][c] >= gm);
                    f |= sent ? (1u << c) : 0u;
                }
            }
        }
        flags[j] = f;
        uint32_t acc = 0u, tot = 0u;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint64_t m = __ballot((f >> c) & 1u);
            acc = __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), acc));
            tot += uint32_t(__popcll(m));
        }
        before[j] = acc;
        wtot[j] = tot;
        if (lane == 0) s_wtot[j * WAVES + wave] = tot;
    }
    __syncthreads();

    // element order inside the tile is (j, wave, lane, c): exclusive prefix over the 4 J rows
    const uint32_t row_incl = wave_incl_scan(lane < uint32_t(WAVES * J) ? s_wtot[lane] : 0u);
    const uint32_t tile_total = __shfl(row_incl, WAVES * J - 1, 64);

    // ---- the pack vector of Algorithm 2: a sent element is staged as (tile-local index << 2 | code) --
    uint16_t *__restrict__ stage = stage_all + td.stage_base;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const uint32_t e0 = (uint32_t(j) * WG + tid) * 4u - skip;
        uint32_t pos = __shfl(row_incl, j * WAVES + int(wave), 64) - wtot[j] + before[j];
        const uint32_t f = flags[j];
        if (f) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if ((f >> c) & 1u) {
                    const uint32_t e = e0 + uint32_t(c);
                    const uint32_t code = (gb[j][c] >> 31) ? 3u : 1u;  // ternary value: -scale / +scale
                    stage[pos] = uint16_t((e << 2) | code);
                    ++pos;
                    atomicAdd(&s_cnt[bin_of(e, T, M)], 1u);
                }
            }
        }
    }
    __syncthreads();

    // ---- tile outputs: counts (into the packet), g_max, sum of g_max, chunk prefixes, total ----
    if (ld.word_bytes == 1u) {
        uint8_t *cp = packet + ld.counts_offset + td.first_bin;
        for (uint32_t i = tid; i < nb; i += WG) cp[i] = uint8_t(s_cnt[i]);
    } else {
        uint16_t *cp = reinterpret_cast<uint16_t *>(packet + ld.counts_offset) + td.first_bin;
        for (uint32_t i = tid; i < nb; i += WG) cp[i] = uint16_t(s_cnt[i]);
    }
    double part = 0.0;
    float *gm_out = gmax_out + ld.bin_start + td.first_bin;
    for (uint32_t i = tid; i < nb; i += WG) {
        const float g = __uint_as_float(s_gmax[i]);
        if (a.keep_gmax) gm_out[i] = g;  // diagnostics only: no later kernel reads the g_max vector
        part += double(g);
    }
    // (The pairing of wave_sum_f64, but through the LDS: the longer tail keeps fewer bytes in flight.  In vector registers /
    // here, in us: 16 learners of the 125 M-element table with unpack 4298 / 4256, of 100 M, 12 learners 3880 / 3897.)
#pragma unroll
    for (uint32_t d = 32; d > 0; d >>= 1) part += __shfl_down(part, d, 64);
    if (lane == 0) s_red[wave] = part;
    // running word count at every 64th bin of the layer that falls inside this tile
    const uint32_t t0 = (64u - (td.first_bin & 63u)) & 63u;
    for (uint32_t t = t0 + 64u * wave; t < nb; t += 64u * uint32_t(WAVES)) {
        uint32_t sum = 0u;
        for (uint32_t i = lane; i < t; i += 64u) sum += s_cnt[i];
        sum = wave_sum(sum);
        if (lane == 0) chunk_rel[ld.chunk_start + ((td.first_bin + t) >> 6)] = sum;
    }
    __syncthreads();
    if (tid == 0) {
        TileOut o;
        double sum = s_red[0];
        for (int wv = 1; wv < WAVES; ++wv) sum += s_red[wv];  // fixed order
        o.gmax_sum = sum;
        o.count = tile_total;
        o.base = 0u;  // filled in by k_scan
        tile_out[tile] = o;  // one 16-byte store
    }
}

template <int J, int WAVES, bool VARIANT, bool LAZY, bool SHIFT = false>
__global__ __launch_bounds__(WAVES * 64) void k_fused(const CompressArgs a)
{
    fused_tile<J, WAVES, VARIANT, LAZY, SHIFT>(a);
}
// Those of 1024 threads that the compiler gives 81 scalar registers are held to 80: beyond them one of these workgroups fits a
// compute unit, not two (see k_pack).  Another rule, in us, 81 / 80: 40 M elements, L_T 5000, 1 learner 143 / 101, 4 598 / 416; L_T 5001 143 / 101;
// 20 M, 500 and 8000, 8 594 / 404; 3 M, 200 and 4500, 20 257 / 185.
template <>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_num_sgpr(80))) void k_fused<4, 16, true, false, false>(const CompressArgs a)
{
    fused_tile<4, 16, true, false, false>(a);
}
template <>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_num_sgpr(80))) void k_fused<4, 16, true, false, true>(const CompressArgs a)
{
    fused_tile<4, 16, true, false, true>(a);
}

__device__ __forceinline__ uint64_t pad16_dev(uint64_t x) { return (x + 15u) & ~uint64_t(15); }

// Header, layer records and zero padding of one learner's packet, by one workgroup of WG threads:
// WG layers at a time, word offsets by a block scan of the padded section sizes (all below 2^32: the
// packet bound is).  get(l, layer, words, scale) says what layer l sends; it is called by the thread
// that writes the layer's record.  `first`: the record of layer number threadIdx.x, if there is one.
template <uint32_t WG, class Get>
__device__ __forceinline__ void place_header(const CompressArgs &a, uint8_t *const packet, const LayerDev &first, Get get)
{
    const uint32_t tid = threadIdx.x;
    __shared__ uint32_t s_wtot[WG / 64u];
    const uint32_t lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint64_t carry = a.fixed_bytes, nsel_all = 0;
    for (uint32_t l0 = 0; l0 < a.n_layers; l0 += WG) {
        const uint32_t l = l0 + tid;
        const bool live = l < a.n_layers;
        LayerDev ld = first;
        uint32_t nsel = 0u, bytes = 0u;
        float scale = 0.f;
        if (live) {
            if (l0 != 0u) ld = a.layers[l];
            get(l, ld, nsel, scale);
            bytes = uint32_t(pad16_dev(uint64_t(nsel) * ld.word_bytes));
        }
        const uint32_t incl = wave_incl_scan(bytes);
        uint32_t nsum = wave_sum(nsel);
        __syncthreads();  // previous round's readers of s_wtot are done
        if (lane == 63) s_wtot[wave] = incl;
        __syncthreads();
        uint64_t before = carry;
        for (uint32_t wv = 0; wv < wave; ++wv) before += s_wtot[wv];
        const uint64_t woff = before + incl - bytes;
        for (uint32_t wv = 0; wv < WG / 64u; ++wv) carry += s_wtot[wv];
        if (live) {
            adacomp_packet_layer_t rec;
            rec.elem_offset = ld.elem_offset; rec.n_elems = ld.n_elems;
            rec.L_T = ld.L_T; rec.n_bins = ld.n_bins; rec.word_bits = ld.word_bytes * 8u;
            rec.scale = scale;
            rec.n_selected = nsel;
            rec.counts_offset = ld.counts_offset; rec.chunks_offset = ld.chunks_offset; rec.words_offset = woff;
            reinterpret_cast<adacomp_packet_layer_t *>(packet + sizeof(adacomp_packet_header_t))[l] = rec;
            for (uint64_t b = ld.counts_offset + uint64_t(ld.n_bins) * ld.word_bytes; b < ld.chunks_offset; ++b) packet[b] = 0;
            const uint64_t chunks_end = ld.chunks_offset + 4ull * ld.n_chunks;
            for (uint64_t b = chunks_end; b < pad16_dev(chunks_end); ++b) packet[b] = 0;
            const uint64_t words_end = woff + uint64_t(nsel) * ld.word_bytes;
            for (uint64_t b = words_end; b < pad16_dev(words_end); ++b)
                if (b < a.capacity) packet[b] = 0;
        }
        // total word count: per-wave sums through the same LDS slots
        __syncthreads();
        if (lane == 0) s_wtot[wave] = nsum;
        __syncthreads();
        for (uint32_t wv = 0; wv < WG / 64u; ++wv) nsel_all += s_wtot[wv];
    }
    if (tid == 0) {
        adacomp_packet_header_t h;
        h.magic = ADACOMP_PACKET_MAGIC; h.version = ADACOMP_PACKET_VERSION;
        h.status = carry > a.capacity ? ADACOMP_STATUS_TRUNCATED : ADACOMP_STATUS_COMPLETE;
        h.n_layers = a.n_layers; h.total_bytes = carry; h.n_selected = nsel_all;
        *reinterpret_cast<adacomp_packet_header_t *>(packet) = h;
    }
}

// The thread's first layer record for place_header.
__device__ __forceinline__ LayerDev header_layer(const CompressArgs &a) { return a.layers[threadIdx.x < a.n_layers ? threadIdx.x : 0u]; }

// ==============================================================================================
// The one-launch compress: k_pack does all of Algorithm 2, for tables whose layers are small enough
// that the tiles of a layer are on the GPU together.
//
// What forces a second launch is the layer's scale: it is known when all tiles of the layer have their
// g_max, and the residue and the place of a word in the packet need it (or the word counts, which
// come with it).  Written as two launches the residue is stored, fetched again and corrected; here a
// workgroup keeps its G in registers and its words in LDS, publishes its tile's record (sum of
// g_max, word count), waits until the layer's records are there, and then writes residue and words
// once, in their final form.  ResNet-50's table (25.5 M elements, L_T 50, 8 % of the elements sent)
// moved 12 bytes per element in k_fused and 6 more in the placement.
//
// Who adds up the records:
//   kOneTable   (at most kFoldTiles tiles and kFoldLayers layers) every workgroup reads the records of
//               the whole table: one hop from the last record to everybody, which is what counts
//               where the launch is a few microseconds long.
//   kOneLayers  the workgroup of a layer's last tile reads the layer's records and publishes the scale,
//               the size of the layer's words and every tile's first word; the others wait for those.
//               It does so as soon as its own record is out and before it goes on with its own words, which
//               takes it 3.5 us (ResNet-50's table 62.5 -> 60.2 us, 8 learners with unpack 512 -> 500).  A
//               workgroup per learner that adds up all layers, a wave each in turn, takes 71 and 557: 54 layers
//               at some 3 us each are too many for it.
// Each learner has a workgroup of its own for the packet's header and layer records, the last of its
// workgroups.  (That of the last tile, after its own words, was the end of the launch, by 2 us: 397 k
// elements 8.9 -> 8.2 us, the CIFAR table 10.6 -> 9.9.)
//
// Published words carry their own validity: every 8-byte word holds 32 bits of value and, in the rest,
// the number of the call (the tile's epoch, kept in the exchange area and raised by one by the tile's
// workgroup in every call), and is read and written with relaxed device-scope atomics.  No fence (a
// device-scope release writes back the L2), no counter, nothing to clear between calls, and a call
// replayed from a graph counts on like any other.
//
// No workgroup depends on another one being scheduled.  A wait is bounded (CompressArgs::wait_polls);
// when it runs out, the workgroup works out the missing records itself: a tile's record follows from
// dW and the residue, and the residue of a tile is written only after all records of its layer are
// published, so whoever finds a record missing may read the tile's inputs.  Should the owner have
// moved on while the helper was reading, the helper's compare-and-swap finds the record there (which it
// is before the owner writes the residue: the owner has read it, or see table_records) and drops what
// it computed; otherwise the two hold the same bits, being the same operations in the same order.  So
// two calls on different streams that hold each other's compute units finish, late; those who wait in
// vain share the missing tiles (help_records).
// ==============================================================================================
constexpr int kOneTable = int(kOneLaunchTable), kOneLayers = int(kOneLaunchLayers);

// One element of Algorithm 2: the bits of G = R + dW (sign included) and of what is compared with
// g_max, max(|G|, |H|) with H = G + dW (VARIANT: by the rule and the factor of the call).
template <bool VARIANT>
__device__ __forceinline__ void element_bits(const CompressArgs &a, const float r, const float w, uint32_t &gb, uint32_t &mb)
{
    const float G = r + w;
    float H;
    if (VARIANT) {
        const float extra = a.soft_factor_minus_1 * w;  // residue + f dW = G + (f - 1) dW
        H = G + extra;
    } else {
        H = G + w;
    }
    gb = __float_as_uint(G);
    const uint32_t ag = gb & 0x7FFFFFFFu, ah = __float_as_uint(H) & 0x7FFFFFFFu;
    if (VARIANT && a.rule == ADACOMP_RULE_PRINTED_COMPARE) mb = ah;          // |H| alone
    else if (VARIANT && a.rule == ADACOMP_RULE_LOCAL_SELECTION) mb = ag;     // bin maxima only
    else mb = ag > ah ? ag : ah;
}

// The selection: sent iff G != 0 and max(|H|, |G|) >= g_max; the printed compare alone also sends
// elements whose G is zero.
template <bool VARIANT>
__device__ __forceinline__ bool element_sent(const CompressArgs &a, const uint32_t gb, const uint32_t mb, const uint32_t gm)
{
    const bool nonzero = (gb & 0x7FFFFFFFu) != 0u || (VARIANT && a.rule == ADACOMP_RULE_PRINTED_COMPARE);
    return nonzero && (mb >= gm);
}

struct SyncArea {
    uint64_t *rec;     // 2 per tile: high half of the tile's g_max sum | epoch; low half | word count, epoch (in the order of rec_part)
    uint64_t *tile;    // 4 per tile: scale | epoch; place of its first word in the packet | epoch; words of the layer before it | epoch; unused (kOneTable: see rec_copy)
    uint64_t *layer;   // 4 per layer: scale | epoch; padded bytes of its words | epoch; its words | epoch; unused
    uint32_t *epoch;   // per tile, and for the header's workgroup: number of calls so far, counted up by that workgroup itself
};

// LDS of a workgroup that waits
struct OneShared {
    uint64_t old_rec[2];
    uint32_t w[16];
    double d[16];
    uint32_t any[3][16];
    uint64_t miss[kOneLaunchTiles / 64u];   // bit t: tile t of a layer, or layer t, is not there yet
    uint32_t missing, base, at, bytes;
    float scale;
};

// Whether any thread of the workgroup says so; a barrier.  `slot`: 16 words of LDS that nobody has read since
// the barrier before this one.  (__syncthreads_or does the same with hidden kernel arguments.)
template <uint32_t WG>
__device__ __forceinline__ bool block_any(const bool mine, uint32_t *slot)
{
    const bool in_wave = __builtin_amdgcn_ballot_w64(mine) != 0ull;
    if ((threadIdx.x & 63u) == 0u) slot[threadIdx.x >> 6] = in_wave ? 1u : 0u;
    __syncthreads();
    uint32_t any = 0u;
#pragma unroll
    for (uint32_t wv = 0; wv < WG / 64u; ++wv) any |= slot[wv];
    return any != 0u;
}

__device__ __forceinline__ uint64_t sync_load(const uint64_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void sync_store(uint64_t *p, uint64_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint64_t sync_word(uint32_t value, uint32_t epoch) { return (uint64_t(value) << 32) | epoch; }

// a word count is at most 16384: 15 bits, and 17 for the epoch, which come back after 131072 calls: a low word has to
// be written in every call (see rec_part), so that a stale one is one call old.
constexpr uint32_t kRecEpochMask = (1u << 17) - 1u;
__device__ __forceinline__ uint64_t rec_high(double sum, uint32_t epoch) { return (__builtin_bit_cast(uint64_t, sum) & 0xFFFFFFFF00000000ull) | epoch; }
__device__ __forceinline__ uint64_t rec_low(double sum, uint32_t count, uint32_t epoch)
{
    return (__builtin_bit_cast(uint64_t, sum) << 32) | (count << 17) | (epoch & kRecEpochMask);
}
__device__ __forceinline__ bool rec_valid(uint64_t hi, uint64_t lo, uint32_t epoch)
{
    return uint32_t(hi) == epoch && (uint32_t(lo) & kRecEpochMask) == (epoch & kRecEpochMask);
}
// kOneTable: the records three times, where the other form has what it says about tiles.  Every workgroup reads all
// of them, some hundred times the same lines, and those that publish late wait behind those that already read:
// 298 tiles 9.0 / 8.7 us, 491 tiles 10.0 / 9.8, 205 7.6 / 7.5.
constexpr uint32_t kRecCopies = 3;
constexpr int kWaitVmem = 0x0F70;   // s_waitcnt vmcnt(0): until the wave's loads and stores are done
__device__ __forceinline__ uint64_t *rec_copy(const SyncArea &sy, const uint32_t n_tiles, const uint32_t copy)
{
    return copy == 0u ? sy.rec : sy.tile + 2u * n_tiles * (copy - 1u);
}
// Where in its pair of words a record has its low word (part 1).  kOneLayers: behind the high one.  kOneTable: in every
// second pair before it, so that the low words of the copies stand where kOneLayers has a place or a number of words, in
// the second and third of the four of a tile, and calls of that form replace them too; of the first and the fourth a call
// may leave what is any number of calls old, but a high word says in 32 bits which call it is of.  (A fourth word written by
// kOneLayers instead costs that form 2 %: ResNet-50's table 60.6 / 61.6 us, the character LSTM 70.2 / 71.6.)
template <int ONE>
__device__ __forceinline__ uint32_t rec_part(const uint64_t *pair, const uint32_t part)
{
    return ONE == kOneTable ? ((uint32_t(reinterpret_cast<uintptr_t>(pair)) >> 4) ^ part) & 1u : part;
}
__device__ __forceinline__ double rec_sum(uint64_t hi, uint64_t lo) { return __builtin_bit_cast(double, (hi & 0xFFFFFFFF00000000ull) | (lo >> 32)); }
__device__ __forceinline__ uint32_t rec_count(uint64_t lo) { return uint32_t(lo) >> 17; }

// Sum of a tile's g_max values by a whole workgroup, in the one order that the tile's owner and a
// helper both use; the result is in thread 0.  Has a barrier; `d` is free again after the next one.
template <uint32_t WG>
__device__ __forceinline__ double tile_gmax_sum(const uint32_t *s_gmax, const uint32_t nb, double *d)
{
    const uint32_t tid = threadIdx.x;
    double part = 0.0;
    if ((tid & ~63u) < nb) {   // uniform in a wave
        for (uint32_t i = tid; i < nb; i += WG) part += double(__uint_as_float(s_gmax[i]));
        part = wave_sum_f64(part);
    }
    if ((tid & 63u) == 0u) d[tid >> 6] = part;
    __syncthreads();
    double sum = d[0];
    for (uint32_t wv = 1; wv < WG / 64u; ++wv) sum += d[wv];
    return sum;
}

// LAZY: what the previous call left waiting for a tile: its words' number and its layer's scale, and the words as
// (tile-local index, sign) in the staging area.
struct Waiting {
    uint32_t count;
    float scale;
    const uint2 *entries;   // four to a load; what lies behind the last one is readable
};
__device__ __forceinline__ Waiting waiting_for(const CompressArgs &a, const uint32_t lr, const uint32_t tile, const TileDev &td)
{
    uint8_t *const sb = a.scratch + uint64_t(lr) * a.scratch_stride;
    const TileOut prev = reinterpret_cast<const TileOut *>(sb + a.o_tile_out)[tile];
    return Waiting{prev.count < td.n_elems ? prev.count : td.n_elems, __uint_as_float(prev.base),
                   reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(sb + a.o_stage) + td.stage_base)};
}
// Two bits for every element of the tile, the code of its word, 0 if it has none: sixteen to a word of `map`, and the four
// of a slot in one byte.  By the whole workgroup, `first`: the thread's first four entries; begins and ends with a barrier.
template <uint32_t WG>
__device__ __forceinline__ void fix_map(const Waiting &wait, const uint2 first, const uint32_t n, uint32_t *const map)
{
    const uint32_t tid = threadIdx.x;
    __syncthreads();
    for (uint32_t i = tid; i < (n + 15u) / 16u; i += WG) map[i] = 0u;
    __syncthreads();
    for (uint32_t q = tid; 4u * q < wait.count; q += WG) {
        const uint2 v = q == tid ? first : wait.entries[q];
        const uint32_t entry[4] = {v.x & 0xFFFFu, v.x >> 16, v.y & 0xFFFFu, v.y >> 16};
#pragma unroll
        for (uint32_t i = 0; i < 4u; ++i) {
            const uint32_t e = entry[i] >> 2;
            if (4u * q + i < wait.count && e < n) atomicOr(&map[e >> 4], (entry[i] & 3u) << (2u * (e & 15u)));
        }
    }
    __syncthreads();
}
// residue <- G - Gq of the previous call: the same single float32 operation that the eager placement performs
__device__ __forceinline__ float fixed_residue(const float r, const uint32_t code, const float scale)
{
    return code == 1u ? r - scale : code == 3u ? r + scale : r;
}

// Works out and publishes the record of a tile whose workgroup has not done it, by the whole
// workgroup; does nothing if the record is there.  Begins and ends with a barrier.  s_map (LAZY): LDS for fix_map.
template <uint32_t WG, bool VARIANT, bool LAZY, int ONE>
__device__ __forceinline__ void help_tile(const CompressArgs &a, const SyncArea &sy, const uint32_t lr, const uint32_t tile,
                                          const uint32_t epoch, uint32_t *s_gmax, uint32_t *s_map, OneShared &sh)
{
    const uint32_t tid = threadIdx.x;
    __syncthreads();
    if (tid == 0) {
        const uint64_t *pair = sy.rec + 2u * tile;
        sh.old_rec[0] = sync_load(pair + rec_part<ONE>(pair, 0u));
        sh.old_rec[1] = sync_load(pair + rec_part<ONE>(pair, 1u));
        sh.missing = rec_valid(sh.old_rec[0], sh.old_rec[1], epoch) ? 0u : 1u;
        sh.base = 0u;
    }
    __syncthreads();
    if (sh.missing != 0u) {   // uniform over the workgroup
        const TileDev td = a.tiles[tile];
        const uint32_t n = td.n_elems, T = td.L_T, M = td.magic, nb = td.n_bins;
        const float *gr = a.grad[lr] + td.elem_base, *rs = a.residue[lr] + td.elem_base;
        for (uint32_t i = tid; i < nb; i += WG) s_gmax[i] = 0u;
        float wait_scale = 0.f;
        if (LAZY && a.lazy) {
            const Waiting wait = waiting_for(a, lr, tile, td);
            wait_scale = wait.scale;
            fix_map<WG>(wait, 4u * tid < wait.count ? wait.entries[tid] : make_uint2(0u, 0u), n, s_map);
        }
        auto residue_of = [&](uint32_t e) {
            const float r = rs[e];
            return LAZY && a.lazy ? fixed_residue(r, (s_map[e >> 4] >> (2u * (e & 15u))) & 3u, wait_scale) : r;
        };
        __syncthreads();
        uint32_t gb, mb, count = 0u;
        for (uint32_t e = tid; e < n; e += WG) {
            element_bits<VARIANT>(a, residue_of(e), gr[e], gb, mb);
            atomicMax(&s_gmax[bin_of(e, T, M)], gb & 0x7FFFFFFFu);
        }
        __syncthreads();
        for (uint32_t e = tid; e < n; e += WG) {
            element_bits<VARIANT>(a, residue_of(e), gr[e], gb, mb);
            count += element_sent<VARIANT>(a, gb, mb, s_gmax[bin_of(e, T, M)]) ? 1u : 0u;
        }
        count = wave_sum(count);
        if ((tid & 63u) == 0u) atomicAdd(&sh.base, count);
        const double sum = tile_gmax_sum<WG>(s_gmax, nb, sh.d);
        if (tid == 0) {
            const uint32_t total = sh.base;
            uint64_t *pair = sy.rec + 2u * tile;
            if (uint32_t(sh.old_rec[0]) != epoch)
                __hip_atomic_compare_exchange_strong(pair + rec_part<ONE>(pair, 0u), &sh.old_rec[0], rec_high(sum, epoch), __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((uint32_t(sh.old_rec[1]) & kRecEpochMask) != (epoch & kRecEpochMask))
                __hip_atomic_compare_exchange_strong(pair + rec_part<ONE>(pair, 1u), &sh.old_rec[1], rec_low(sum, total, epoch), __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
}

// One thread's records, tiles ts + tid, ts + tid + WG, ...: HOLD of them.
template <uint32_t HOLD>
struct Records {
    uint64_t hi[HOLD], lo[HOLD];
};

// Polls for the thread's records of tiles ts .. ts + nt - 1; says whether they all came.
template <uint32_t WG, int ONE, uint32_t HOLD>
__device__ __forceinline__ bool poll_records(const SyncArea &sy, const uint32_t ts, const uint32_t nt,
                                             const uint32_t epoch, const uint32_t most_polls, Records<HOLD> &rec)
{
    bool all = true;
#pragma unroll
    for (uint32_t h = 0; h < HOLD; ++h) {
        rec.hi[h] = 0u;
        rec.lo[h] = 0u;
        const uint32_t i = h * WG + threadIdx.x;
        const uint64_t *src = sy.rec + 2u * (ts + i);
        bool ok = i >= nt;
        for (uint32_t polls = 0; !ok && polls <= most_polls; ++polls) {
            if (polls != 0u) __builtin_amdgcn_s_sleep(1);
            rec.hi[h] = sync_load(src + rec_part<ONE>(src, 0u));
            rec.lo[h] = sync_load(src + rec_part<ONE>(src, 1u));
            ok = rec_valid(rec.hi[h], rec.lo[h], epoch);
        }
        all = all && ok;
    }
    return all;
}

// Sees to it that the records of tiles ts .. ts + nt - 1 are there, by the whole workgroup: as long as some are
// missing, works out one of them.  Workgroups that wait in vain do this together, each with its own `seed`, and
// so come upon different ones: those that cannot start are worked out about as fast as if they ran.  (Every
// round adds a record or finds that somebody else did; false after more rounds than there are tiles: another
// call is at work in the same area.)
template <uint32_t WG, uint32_t HOLD, bool VARIANT, bool LAZY, int ONE>
__device__ __forceinline__ bool help_records(const CompressArgs &a, const SyncArea &sy, const uint32_t lr, const uint32_t ts, const uint32_t nt,
                                             const uint32_t epoch, uint32_t seed, uint32_t *s_gmax, uint32_t *s_map, OneShared &sh)
{
    const uint32_t tid = threadIdx.x;
    for (uint32_t round = 0; round <= nt; ++round) {
        __syncthreads();   // nobody reads sh.miss any more
        for (uint32_t h = 0; h < HOLD; ++h) {
            const uint32_t i = h * WG + tid;
            const uint64_t *src = sy.rec + 2u * (ts + i);
            const bool miss = i < nt && !rec_valid(sync_load(src + rec_part<ONE>(src, 0u)), sync_load(src + rec_part<ONE>(src, 1u)), epoch);
            const uint64_t m = __builtin_amdgcn_ballot_w64(miss);
            if ((tid & 63u) == 0u) sh.miss[i >> 6] = m;
        }
        __syncthreads();
        uint32_t n_miss = 0u;
        for (uint32_t w = 0; w < HOLD * WG / 64u; ++w) n_miss += uint32_t(__popcll(sh.miss[w]));
        if (__builtin_amdgcn_readfirstlane(n_miss) == 0u) return true;
        seed = (seed ^ (seed >> 15)) * 0x2C1B3C6Du + 0x9E3779B9u;
        uint32_t k = __umulhi(seed, n_miss), q = 0u;   // the k-th of them
        for (uint32_t w = 0; w < HOLD * WG / 64u; ++w) {
            uint64_t m = sh.miss[w];
            const uint32_t c = uint32_t(__popcll(m));
            if (k < c) {
                for (; k != 0u; --k) m &= m - 1u;
                q = 64u * w + uint32_t(__builtin_ctzll(m));
                break;
            }
            k -= c;
        }
        help_tile<WG, VARIANT, LAZY, ONE>(a, sy, lr, ts + __builtin_amdgcn_readfirstlane(q), epoch, s_gmax, s_map, sh);
    }
    return false;
}

// The first layer below l that has not published its words' size; l if all have.  By the whole workgroup.
template <uint32_t WG>
__device__ __forceinline__ uint32_t first_open_layer(const SyncArea &sy, const uint32_t l, const uint32_t epoch, OneShared &sh)
{
    const uint32_t tid = threadIdx.x;
    __syncthreads();   // nobody reads sh.miss any more
    for (uint32_t m = tid; m < kOneLaunchLayersMax; m += WG) {
        const uint64_t open = __builtin_amdgcn_ballot_w64(m < l && uint32_t(sync_load(sy.layer + 4u * m + 1u)) != epoch);
        if ((tid & 63u) == 0u) sh.miss[m >> 6] = open;
    }
    __syncthreads();
    uint32_t first = l;
    for (uint32_t w = kOneLaunchLayersMax / 64u; w-- > 0u;)
        if (sh.miss[w] != 0ull) first = 64u * w + uint32_t(__builtin_ctzll(sh.miss[w]));
    return __builtin_amdgcn_readfirstlane(first);
}

// before[h]: words of the tiles before the thread's h-th; adds the thread's g_max sums to `part`; returns
// the words of all tiles.  Begins behind a barrier (sh.w is free) and ends with one.
template <uint32_t WG, uint32_t HOLD>
__device__ __forceinline__ uint32_t scan_records(const uint32_t nt, const Records<HOLD> &rec, OneShared &sh, uint32_t (&before)[HOLD], double &part)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t run = 0u;
#pragma unroll
    for (uint32_t h = 0; h < HOLD; ++h) {
        before[h] = 0u;
        if (h != 0u && h * WG >= nt) continue;   // uniform
        const bool live = h * WG + tid < nt;
        const uint32_t count = live ? rec_count(rec.lo[h]) : 0u;
        if (live) part += rec_sum(rec.hi[h], rec.lo[h]);
        const uint32_t incl = wave_incl_scan(count);
        if (lane == 63u) sh.w[wave] = incl;
        __syncthreads();
        before[h] = run + incl - count;
        for (uint32_t wv = 0; wv < WG / 64u; ++wv) {
            const uint32_t t = sh.w[wv];
            before[h] += wv < wave ? t : 0u;
            run += t;
        }
        __syncthreads();
    }
    return run;
}

// One wave: waits for the words of `sy.layer` numbered `first`, first + 4, ... (one per layer) of the
// layers below n_layers and adds up their values; ok: in, whether to wait at all; out, whether all came.
__device__ __forceinline__ uint32_t poll_layer_words(const SyncArea &sy, const uint32_t first, const uint32_t n_layers, const uint32_t epoch,
                                                     const uint32_t most_polls, const uint32_t lane, bool &ok)
{
    uint32_t sum = 0u;
    for (uint32_t m = lane; ok && m < n_layers; m += 64u) {
        uint64_t v = 0u;
        ok = false;
        for (uint32_t polls = 0; !ok && polls <= most_polls; ++polls) {
            if (polls != 0u) __builtin_amdgcn_s_sleep(4);
            v = sync_load(sy.layer + 4u * m + first);
            ok = uint32_t(v) == epoch;
        }
        sum += uint32_t(v >> 32);
    }
    return wave_sum(sum);
}

// Adds up the records of layer l and publishes what its tiles (and the layers behind it) wait for.  Says
// whether everything came in time; HELP: does not wait for records, but works out those that are missing.
template <uint32_t WG, bool VARIANT, bool LAZY, bool HELP>
__device__ __forceinline__ bool complete_layer(const CompressArgs &a, const SyncArea &sy, const uint32_t lr, const uint32_t l,
                                               const uint32_t epoch, const uint32_t seed, uint32_t *s_gmax, uint32_t *s_map, OneShared &sh)
{
    constexpr uint32_t HOLD = (kOneLaunchTiles + WG - 1u) / WG;
    const uint32_t most_polls = HELP ? kWaitPollsKnown : a.wait_polls;   // (the layers before: HELP comes when those are there)
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t ts = a.layers[l].ctile_start, nt = a.layers[l].n_ctiles, wbytes = a.layers[l].word_bytes;
    Records<HOLD> rec;
    if (HELP && !help_records<WG, HOLD, VARIANT, LAZY, kOneLayers>(a, sy, lr, ts, nt, epoch, seed, s_gmax, s_map, sh)) return false;
    if (block_any<WG>(!poll_records<WG, kOneLayers>(sy, ts, nt, epoch, HELP ? 0u : a.wait_polls, rec), sh.any[0])) return false;
    uint32_t before[HOLD];
    double part = 0.0;
    const uint32_t words = scan_records<WG>(nt, rec, sh, before, part);
    part = wave_sum_f64(part);
    if (lane == 0u) sh.d[tid >> 6] = part;
    __syncthreads();
    double total = 0.0;
    for (uint32_t wv = 0; wv < WG / 64u; ++wv) total += sh.d[wv];   // fixed order
    const uint32_t scale = __float_as_uint(float(total / double(a.layers[l].n_bins)));
    if (tid == 0) {
        uint64_t *out = sy.layer + 4u * l;
        sync_store(out + 1, sync_word(uint32_t(pad16_dev(uint64_t(words) * wbytes)), epoch));
        sync_store(out, sync_word(scale, epoch));
        sync_store(out + 2, sync_word(words, epoch));
    }
    bool ok = true;
    if (tid < 64u) {   // the layers before: their words come first in the packet
        const uint32_t bytes = poll_layer_words(sy, 1u, l, epoch, most_polls, lane, ok);
        if (lane == 0u) sh.bytes = bytes;
    }
    if (block_any<WG>(!ok, sh.any[1])) return false;
    const uint32_t woff = uint32_t(a.fixed_bytes) + sh.bytes;   // below 2^32 like the packet
#pragma unroll
    for (uint32_t h = 0; h < HOLD; ++h) {
        if (h * WG + tid < nt) {
            uint64_t *out = sy.tile + 4u * (ts + h * WG + tid);
            sync_store(out, sync_word(scale, epoch));
            sync_store(out + 1, sync_word(woff + before[h] * wbytes, epoch));
            sync_store(out + 2, sync_word(before[h], epoch));
        }
    }
    return true;
}

// scale = average of the layer's g_max values, from the sums of its tiles, by one wave in a fixed order
__device__ __forceinline__ float layer_scale_of(const double *sum, const uint32_t n_ctiles, const uint32_t n_bins, const uint32_t lane)
{
    double s = 0.0;
    for (uint32_t t = lane; t < n_ctiles; t += 64u) s += sum[t];
    return float(wave_sum_f64(s) / double(n_bins));
}

// kOneTable: waits for the records of all tiles and lays them out: s_sum[t] the g_max sum of tile t, s_excl[t] the words
// of the tiles before t in its run of 64, sh.w[r] the words of run r.  By the whole workgroup, behind a barrier;
// ends with one.  helped: this workgroup has worked out records itself.  False: another call is at work in the area.
template <uint32_t WG, bool VARIANT, bool LAZY>
__device__ __forceinline__ bool table_records(const CompressArgs &a, const SyncArea &sy, const uint32_t lr, const uint32_t epoch, const uint32_t seed,
                                              uint32_t *s_gmax, uint32_t *s_map, uint32_t *const s_excl, double *const s_sum, OneShared &sh, bool &helped)
{
    constexpr uint32_t HOLD = (kFoldTiles + WG - 1u) / WG;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Records<HOLD> rec;
    auto lay_out = [&]() {
#pragma unroll
        for (uint32_t h = 0; h < HOLD; ++h) {
            const uint32_t i = h * WG + tid, n = i < a.n_tiles ? rec_count(rec.lo[h]) : 0u;
            const uint32_t incl = wave_incl_scan(n);
            if (i < kFoldTiles) s_excl[i] = incl - n;
            if (i < a.n_tiles) s_sum[i] = rec_sum(rec.hi[h], rec.lo[h]);
            if (lane == 63u) sh.w[WG / 64u * h + wave] = incl;
        }
        if (tid == 0) s_excl[kFoldTiles] = 0u;
    };
    helped = false;
    SyncArea copy = sy;   // (whoever helps publishes in the first copy only, and reads that one)
    copy.rec = rec_copy(sy, a.n_tiles, blockIdx.x % kRecCopies);
    const bool all = poll_records<WG, kOneTable>(copy, 0u, a.n_tiles, epoch, a.wait_polls, rec);
    // Who reads another copy does not learn from it that its own record is in the first one, where a helper that has read the
    // residue after it was written has to find it: the wave that published, the first one, waits for its stores here, and the
    // others for that wave at the barrier, before any of them writes the residue.  (They are done by then: no time.)
    __builtin_amdgcn_s_waitcnt(kWaitVmem);
    lay_out();
    if (__builtin_expect(block_any<WG>(!all, sh.any[0]), false)) {
        const bool there = help_records<WG, HOLD, VARIANT, LAZY, kOneTable>(a, sy, lr, 0u, a.n_tiles, epoch, seed, s_gmax, s_map, sh);
        if (block_any<WG>(!(there && poll_records<WG, kOneTable>(sy, 0u, a.n_tiles, epoch, 0u, rec)), sh.any[1])) return false;
        lay_out();
        __syncthreads();
        helped = true;
    }
    return true;
}
// lane r: the words of all runs of 64 tiles before run r; with it, the words of all tiles before tile t
__device__ __forceinline__ uint32_t words_before_runs(const OneShared &sh, const uint32_t lane)
{
    const uint32_t n = lane < kFoldTiles / 64u ? sh.w[lane] : 0u;
    return wave_incl_scan(n) - n;
}
__device__ __forceinline__ uint32_t words_before(const uint32_t *s_excl, const uint32_t run_at, const uint32_t t)
{
    return s_excl[t] + uint32_t(__shfl(int(run_at), int(t >> 6), 64));
}

// ==============================================================================================
// k_pack: a tile of at most 4096 elements, 256 threads with four 16-byte slots each, or where every workgroup
// reads all records and few are at work, 512 with two (kPackWidePerUnit); a tile of up to 16384 elements, 1024 threads
// with four slots, of which two workgroups fit a compute unit with at most 64 vector and 80 scalar registers (beyond
// 80, waves are given 112 of the 800 that a SIMD has, and seven fit: one workgroup).  Tiles of the
// smaller class start on 16-byte boundaries, those of the larger on 4-byte ones: the buffer accesses of the slots
// need no more.  Bins have at least four elements, so that a slot lies in one bin
// or two.  Bound by HBM at 12 bytes per element plus the packet, and short of that by the wait, about
// 8 us of a workgroup's life of 17 us on ResNet-50's table, which other workgroups have to cover:
// hence eight of them on a compute unit, which takes 64 registers (7 spilled ones cost 10 %) and is why
// several values are worked out anew below instead of being kept.  The lazy form for layers spills 19 at that, and is
// still the faster for it: 8 / 7 / 6 waves, in us, ResNet-50's table, 1 learner 64.5 / 66.5 / 70.8; the character LSTM, 1
// 14.8 / 14.9 / 14.9, 4 35.8 / 36.6 / 40.9; 12 M elements, L_T 50 and 500, 2 60.9 / 64.1 / 67.0; 4 M, 2 22.2 / 27.6 / 28.7.
// Measured, before (k_fused, k_scan, k_place or k_place_tiled) and now, in us: ResNet-50's table
// 98 -> 65, a mini-batch of 8 learners with its unpack 700 -> 524; 23 layers with odd bins, 9.4 M
// elements, 2 learners 71 -> 49; 397 k elements 12.1 -> 9.6; the CIFAR table, 4 learners with unpack,
// 33 -> 23.  (Since then 60, 495, 47, 6.6 and 22: the layer added up early, the header's own workgroup, 512 threads.)
// ==============================================================================================
// values the compiler is not to connect with what they were before
template <int N>
__device__ __forceinline__ void keep_apart(uint32_t (&v)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i]));
}

// max(v, v of the lane CTRL says, 8 or fewer lanes below in the same row of 16), where `from` holds
template <int CTRL>
__device__ __forceinline__ uint32_t take_max_from(const uint32_t v, const bool from)
{
    const uint32_t o = uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, 0xF, 0xF, true));   // 0 past the row's start
    return from && o > v ? o : v;
}

// A pointer that goes through an asm statement, which takes away the compiler's knowledge that a kernel's arguments point to
// global memory: as this type it comes out as one to global memory.  Through a plain one every access behind the statement is a flat one,
// which counts as an access to the LDS too, so that each wait for the LDS waits for it.  Flat / global, us: 397 k elements 6.25 / 6.10, the
// CIFAR table, one learner 8.52 / 8.33, its step of 4 learners 20.33 / 20.25; large tables, where other workgroups cover it, the same.
template <class T>
using global_ptr = __attribute__((address_space(1))) T *;

// What a workgroup needs for its first loads, ahead of the structure (kOneTable).
struct PackFirst {
    const TileDev *tiles;
    uint8_t *sync;
    uint32_t sync_stride, o_epoch, n_tiles, first;
};
// Ahead: the types of PackFirst's members in their order (kOneTable), or none.  (As a function that two kernels call, kOneLayers
// reads back 14 more spilled scalar registers.)
template <bool VARIANT, int ONE, int WAVES, int J, bool LAZY, class... Ahead>
__global__ __launch_bounds__(WAVES * 64, ONE == kOneTable && WAVES == 8 ? 4 : LAZY && WAVES == 4 && ONE == kOneTable ? 6 : 8) __attribute__((amdgpu_num_sgpr(80)))
void k_pack(const Ahead... first_args, const CompressArgs a)
{
    static_assert((ONE == kOneTable) == (sizeof...(Ahead) != 0), "arguments ahead of the structure");
    const PackFirst ahead{first_args...};
    constexpr uint32_t WG = uint32_t(WAVES) * 64u, kRow = WG * 4u;   // J 16-byte slots to a thread: slot j of thread t is number j * WG + t of the tile
    constexpr int P = (J + 1) / 2;   // pairs of rows
    static_assert(WG * uint32_t(J) <= 4096u && J <= 4, "tiles of at most 16384 elements, words counted in 15 bits");
    // Two rounds of scalar loads: arguments, then what they point to.  (Left to the compiler, which fetches what a
    // branch needs behind the branch, there are five, 0.25 us each, before the first load of the tile.)  kOneTable, where the
    // chain is what counts: one, since what the loads of the second need is there when the workgroup starts, in scalar
    // registers (the arguments before the structure, see the build's preload count; as structure / ahead of it, in us: 397 k elements
    // 6.24 / 6.03, the CIFAR table 8.83 / 8.38, 4 learners with unpack 19.98 / 19.79, bins of 800 and 8000 19.95 / 19.39; kOneLayers, ResNet-50's
    // table 58.5 / 59.5, with six more scalar registers spilled).
    constexpr bool kAhead = ONE == kOneTable;
    const TileDev *tiles = ahead.tiles;
    uint8_t *sync = ahead.sync;
    uint64_t sync_stride = ahead.sync_stride;
    uint32_t o_epoch = ahead.o_epoch, n_tiles = ahead.n_tiles, lr = ahead.first, o_rec = 0u, o_tile = 0u, o_layer = 0u;
    const LayerDev *layers = nullptr;
    if constexpr (!kAhead) {
        global_ptr<uint8_t> in_global = (global_ptr<uint8_t>)a.sync;
        tiles = a.tiles; layers = a.layers; sync_stride = a.sync_stride;
        o_rec = a.o_sync_rec; o_tile = a.o_sync_tile; o_layer = a.o_sync_layer; o_epoch = a.o_sync_epoch;
        n_tiles = a.class_count; lr = a.fused_first;
        asm volatile("" : "+s"(tiles), "+s"(layers), "+s"(in_global), "+s"(sync_stride), "+s"(o_rec), "+s"(o_tile), "+s"(o_layer), "+s"(o_epoch), "+s"(n_tiles), "+s"(lr));
        sync = (uint8_t *)in_global;
    }
    // learner-major: one workgroup per tile, within runs of 64 transposed as in k_fused, then the one that writes the header
    uint32_t tile = blockIdx.x;
    const bool heads = tile == n_tiles;
    lr += blockIdx.y;
    if (tile < (n_tiles & ~63u)) tile = (tile & ~63u) | ((tile & 7u) << 3) | ((tile >> 3) & 7u);
    uint8_t *const area = sync + uint64_t(lr) * sync_stride;
    SyncArea sy;
    auto set_sync = [&]() {
        sy.rec = reinterpret_cast<uint64_t *>(area + o_rec);
        sy.tile = reinterpret_cast<uint64_t *>(area + o_tile);
        sy.layer = reinterpret_cast<uint64_t *>(area + o_layer);
    };
    if constexpr (!kAhead) set_sync();
    sy.epoch = reinterpret_cast<uint32_t *>(area + o_epoch);
    vuint8 tile_words = *(const __attribute__((address_space(4))) vuint8 *)(tiles + (heads ? 0u : tile));
    uint32_t epoch = *(const __attribute__((address_space(4))) uint32_t *)(sy.epoch + tile);
    global_ptr<uint8_t> packet_g = (global_ptr<uint8_t>)a.packet[lr];
    global_ptr<float> residue_g = (global_ptr<float>)a.residue[lr];
    global_ptr<const float> grad_g = (global_ptr<const float>)a.grad[lr];
    if constexpr (kAhead) { layers = a.layers; o_rec = a.o_sync_rec; o_tile = a.o_sync_tile; o_layer = a.o_sync_layer; }
    if constexpr (kAhead) asm volatile("" : "+s"(tile_words), "+s"(epoch), "+s"(packet_g), "+s"(residue_g), "+s"(grad_g), "+s"(layers), "+s"(o_rec), "+s"(o_tile), "+s"(o_layer));
    else asm volatile("" : "+s"(tile_words), "+s"(epoch), "+s"(packet_g), "+s"(residue_g), "+s"(grad_g));
    uint8_t *const packet = (uint8_t *)packet_g;
    float *const residue = (float *)residue_g;
    const float *const grad = (const float *)grad_g;
    if constexpr (kAhead) set_sync();
    ++epoch;   // (count_call)
    const TileDev td = __builtin_bit_cast(TileDev, tile_words);

    __shared__ __attribute__((aligned(16))) uint32_t s_gmax[kPackBins];   // bit pattern of max |G| (and of the bins behind the last: pack_bin)
    __shared__ __attribute__((aligned(16))) uint32_t s_cnt[kPackBins];
    __shared__ uint32_t s_words[WG * J * 2u + 4u];  // the tile's words, in their final form, one byte or two each
    __shared__ uint32_t s_rows[WAVES * P * 2];   // words per wave and row, two rows to an entry
    __shared__ uint32_t s_chunk[kMaxTileBins / 64u];
    __shared__ OneShared sh;
    __shared__ uint32_t s_excl[ONE == kOneTable ? kFoldTiles + 1u : 1u];   // kOneTable: words of the tiles before tile t in the same run of 64
    double *const s_sum = reinterpret_cast<double *>(s_gmax);              // kOneTable: g_max sum of tile t, when the tile's own are done with
    static_assert(8u * kFoldTiles <= sizeof(s_gmax), "LDS of the sums");

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    if (heads) {
        const LayerDev first = header_layer(a);
        auto leave = [&](uint32_t m, uint32_t nsel, float sc) {   // LAZY: for whoever applies the corrections later
            if (!LAZY) return;
            uint8_t *const sb = a.scratch + uint64_t(lr) * a.scratch_stride;
            reinterpret_cast<uint32_t *>(sb + a.o_layer_nsel)[m] = nsel;
            reinterpret_cast<float *>(sb + a.o_layer_scale)[m] = sc;
        };
        if (tid == 0) count_call(sy.epoch + a.n_tiles);
        if (ONE == kOneTable) {
            float *const s_lscale = reinterpret_cast<float *>(s_words);
            bool helped;
            if (!table_records<WG, VARIANT, LAZY>(a, sy, lr, epoch, a.n_tiles, s_gmax, s_cnt, s_excl, s_sum, sh, helped)) return;   // nothing to go by
            const uint32_t run_at = words_before_runs(sh, lane);
#pragma unroll
            for (uint32_t i = 0; i < kFoldLayers / uint32_t(WAVES); ++i) {
                const uint32_t m = wave + uint32_t(WAVES) * i;
                if (m >= a.n_layers) continue;   // uniform
                const float sc = layer_scale_of(s_sum + a.layers[m].ctile_start, a.layers[m].n_ctiles, a.layers[m].n_bins, lane);
                if (lane == 0u) s_lscale[m] = sc;
            }
            const uint32_t ts = first.ctile_start, te = ts + first.n_ctiles;
            const uint32_t words = words_before(s_excl, run_at, te) - words_before(s_excl, run_at, ts);
            __syncthreads();
            place_header<WG>(a, packet, first, [&](uint32_t m, const LayerDev &, uint32_t &nsel, float &sc) { nsel = words; sc = s_lscale[m]; leave(m, nsel, sc); });   // (at most kFoldLayers layers: one round)
        } else {
            auto poll_layers = [&](bool ok, const uint32_t most_polls) {   // scale and word count of every layer
                if (wave == 0u) {
                    poll_layer_words(sy, 0u, a.n_layers, epoch, most_polls, lane, ok);
                    poll_layer_words(sy, 2u, a.n_layers, epoch, most_polls, lane, ok);
                }
                return ok;
            };
            if (__builtin_expect(block_any<WG>(!poll_layers(true, a.wait_polls), sh.any[2]), false)) {
                bool ok = true;
                for (uint32_t times = 0; ok; ++times) {   // the layers that are not done
                    const uint32_t m = first_open_layer<WG>(sy, a.n_layers, epoch, sh);
                    if (m == a.n_layers) break;
                    ok = times <= a.n_layers && complete_layer<WG, VARIANT, LAZY, true>(a, sy, lr, m, epoch, a.n_tiles, s_gmax, s_cnt, sh);
                }
                if (block_any<WG>(!poll_layers(ok, kWaitPollsKnown), sh.any[2])) return;   // nothing to go by: store nothing
            }
            place_header<WG>(a, packet, first, [&](uint32_t m, const LayerDev &, uint32_t &nsel, float &sc) {
                nsel = uint32_t(sync_load(sy.layer + 4u * m + 2u) >> 32);
                sc = __uint_as_float(uint32_t(sync_load(sy.layer + 4u * m) >> 32));
                leave(m, nsel, sc);
            });
        }
        return;
    }

    const uint32_t n = td.n_elems, T = td.L_T, M = td.magic, nb = td.n_bins, l = td.layer();
    float *const rs = residue + td.elem_base;
    const float *const gr = grad + td.elem_base;
    // whole slots only: what lies past the tile is read as zero and not stored, without a branch
    const __amdgpu_buffer_rsrc_t r_buf = tile_buffer(rs, n & ~3u), w_buf = tile_buffer(gr, n & ~3u);

    auto skip_row = [&](int j) { return WAVES >= 8 && j != 0 && n <= uint32_t(j) * kRow; };   // (uniform: the small tiles of small tables leave a row empty)
    uint32_t gb[J][4];  // bits of G (sign included)
    uint32_t mb[J][4];  // bits of max(|G|, |H|): what is compared with g_max
    vfloat4 r[J], w[J];
    auto load_slots = [&]() {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            r[j] = buffer_load_slot(r_buf, tid * 16u, uint32_t(j) * kRow * 4u);
            w[j] = buffer_load_slot(w_buf, tid * 16u, uint32_t(j) * kRow * 4u);
        }
        if ((n & 3u) != 0u) {   // the layer's last elements, which do not fill a slot
#pragma unroll
            for (int j = 0; j < J; ++j)
                if (uint32_t(j) * WG + tid == (n >> 2)) {
                    for (uint32_t c = 0; c < (n & 3u); ++c) { r[j][c] = rs[(n & ~3u) + c]; w[j][c] = gr[(n & ~3u) + c]; }
                }
        }
    };
    load_slots();
    asm volatile("" ::: "memory");   // the layer's record, which is not needed before the words, is not waited for together with the tile's
    const LayerDev ld = table_record<vuint16>(layers + l);
    // LAZY: the residue corrections of the learner's previous call are applied to the values in registers first
    auto apply_waiting = [&]() {
        const Waiting wait = waiting_for(a, lr, tile, td);
        fix_map<WG>(wait, 4u * tid < n ? wait.entries[tid] : make_uint2(0u, 0u), n, s_cnt);   // (fetched together with the count)
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if (skip_row(j)) continue;
            const uint32_t codes = uint32_t(j) * kRow + tid * 4u < n ? reinterpret_cast<const uint8_t *>(s_cnt)[uint32_t(j) * WG + tid] : 0u;
#pragma unroll
            for (int c = 0; c < 4; ++c) r[j][c] = fixed_residue(r[j][c], (codes >> (2 * c)) & 3u, wait.scale);
        }
        __syncthreads();
    };
    if (LAZY && a.lazy) apply_waiting();
    for (uint32_t i = tid; i < nb + 2u; i += WG) { s_gmax[i] = 0u; s_cnt[i] = 0u; }
    if (ONE == kOneTable) __builtin_amdgcn_s_setprio(2);   // until the record is out: others wait for it (6 % of a small mini-batch; slower where waves queue for memory)
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) element_bits<VARIANT>(a, r[j][c], w[j][c], gb[j][c], mb[j][c]);
    // (from here on the inputs are not needed again: without this the compiler kept dW and |G| beside G and
    // worked H out later, 16 registers more than eight resident workgroups leave)
#pragma unroll
    for (int j = 0; j < J; ++j) { keep_apart(gb[j]); keep_apart(mb[j]); }
    __syncthreads();

    // ---- first loop of Algorithm 2: g_max(i) per bin.  A slot lies in bin b0, its elements from `left` on in
    // the next one (bins have at least four elements): one division per slot -------------------------
    uint32_t place[J];   // b0 << 16 | left
    const bool whole_slots = (T & 3u) == 0u;   // no slot lies in two bins
    if (whole_slots) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if (skip_row(j)) { place[j] = T; continue; }
            const uint32_t e0 = uint32_t(j) * kRow + tid * 4u;
            const uint32_t b = __umulhi(e0, M), into = e0 - __umul24(b, T), left = T - into, b0 = pack_bin<WAVES == 16>(b, nb);
            place[j] = (b0 << 16) | left;
            uint32_t v = gb[j][0] & 0x7FFFFFFFu;
#pragma unroll
            for (uint32_t c = 1; c < 4u; ++c) { const uint32_t g = gb[j][c] & 0x7FFFFFFFu; v = g > v ? g : v; }
            v = take_max_from<0x111>(v, into >= 4u);   // (as below)
            v = take_max_from<0x112>(v, into >= 8u);
            v = take_max_from<0x114>(v, into >= 16u);
            v = take_max_from<0x118>(v, into >= 32u);
            if ((lane & 15u) == 15u || left < 8u) atomicMax(&s_gmax[b0], v);
        }
    } else
#pragma unroll
    for (int j = 0; j < J; ++j) {
        if (skip_row(j)) { place[j] = T; continue; }
        const uint32_t e0 = uint32_t(j) * kRow + tid * 4u;
        const uint32_t b = __umulhi(e0, M), b0 = pack_bin<WAVES == 16>(b, nb);
        const uint32_t left = T - (e0 - __umul24(b, T));
        place[j] = (b0 << 16) | left;
        uint32_t m0 = gb[j][0] & 0x7FFFFFFFu, m1 = 0u;
#pragma unroll
        for (uint32_t c = 1; c < 4u; ++c) {
            const uint32_t v = gb[j][c] & 0x7FFFFFFFu;
            const uint32_t v0 = c < left ? v : 0u, v1 = c < left ? 0u : v;
            m0 = v0 > m0 ? v0 : m0;
            m1 = v1 > m1 ? v1 : m1;
        }
        // Lanes of a row of 16 whose slots lie in one bin bring one maximum to the LDS: `into` is the start of the
        // slot in its bin, 0 for a slot that begins a new bin on its way (its lane takes nothing over).
        const bool split = left < 4u;
        const uint32_t into = split ? 0u : T - left;
        uint32_t v = split ? m1 : m0;
        v = take_max_from<0x111>(v, into >= 1u);
        v = take_max_from<0x112>(v, into >= 5u);
        v = take_max_from<0x114>(v, into >= 13u);
        v = take_max_from<0x118>(v, into >= 29u);
        if (split) atomicMax(&s_gmax[b0], m0);
        if ((lane & 15u) == 15u || (split ? left + T : left) < 8u) atomicMax(&s_gmax[split ? b0 + 1u : b0], v);
    }
    __syncthreads();

    // (what a pass works out from `place` is worked out anew in the next one: kept, it costs more registers
    // than eight resident workgroups leave)
    keep_apart(place);
#pragma unroll
    for (int j = 0; j < J; ++j) keep_apart(gb[j]);
    // ---- second loop: the local-max compare, and every sent element's place among the tile's words ----
    uint32_t sent_mask = 0u;   // bit 4 j + c: element c of slot j is sent
#pragma unroll
    for (int j = 0; j < J; ++j) {
        if (skip_row(j)) continue;
        const uint32_t b0 = place[j] >> 16, left = place[j] & 0xFFFFu;
        const uint32_t gm0 = s_gmax[b0], gm1 = s_gmax[b0 + 1u];
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c)
            sent_mask |= element_sent<VARIANT>(a, gb[j][c], mb[j][c], c < left ? gm0 : gm1) ? 1u << (4 * j + c) : 0u;
        if (VARIANT) {   // the printed compare sends zeros: not those that stand for what lies past the tile
            const uint32_t e0 = uint32_t(j) * kRow + tid * 4u;
            const uint32_t valid = n > e0 ? (n - e0 < 4u ? n - e0 : 4u) : 0u;
            sent_mask &= ~(0xFu << (4 * j)) | (((1u << valid) - 1u) << (4 * j));
        }
    }
    // words are ordered by (row j, wave, lane, c): counts of two rows to a register, at most 256 each per wave
    uint32_t pre[P];   // words of the wave's rows before this lane
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint32_t c = uint32_t(__popc((sent_mask >> (8 * p)) & 0xFu)) | (uint32_t(__popc((sent_mask >> (8 * p)) & 0xF0u)) << 16);
        const uint32_t incl = wave_incl_scan(c);
        if (lane == 63u) { s_rows[2 * p * WAVES + int(wave)] = incl & 0xFFFFu; s_rows[(2 * p + 1) * WAVES + int(wave)] = incl >> 16; }
        pre[p] = incl - c;
    }
    const double gmax_sum = tile_gmax_sum<WG>(s_gmax, nb, sh.d);   // has the barrier
    const uint32_t row = lane < uint32_t(J * WAVES) ? s_rows[lane] : 0u, rows_incl = wave_incl_scan(row);
    const uint32_t tile_total = uint32_t(__builtin_amdgcn_readlane(int(rows_incl), J * WAVES - 1));
    uint32_t row_at[J];   // words of the rows before the wave's row j
#pragma unroll
    for (int j = 0; j < J; ++j) row_at[j] = uint32_t(__builtin_amdgcn_readlane(int(rows_incl - row), j * WAVES + int(wave)));
    // first thing: others wait for it
    if (tid < (ONE == kOneTable ? 2u * kRecCopies : 2u)) {
        uint64_t *pair = rec_copy(sy, a.n_tiles, tid >> 1) + 2u * tile;
        sync_store(pair + rec_part<ONE>(pair, tid & 1u), (tid & 1u) ? rec_low(gmax_sum, tile_total, epoch) : rec_high(gmax_sum, epoch));
    }
    if (tid == 0) count_call(sy.epoch + tile);
    if (ONE == kOneTable) __builtin_amdgcn_s_setprio(0);
    // A layer's last workgroup adds up its layer, before anything else: all of the layer wait for it.
    bool layer_ok = true;
    if (ONE == kOneLayers && tile == ld.ctile_start + ld.n_ctiles - 1u) layer_ok = complete_layer<WG, VARIANT, LAZY, false>(a, sy, lr, l, epoch, tile, s_gmax, s_cnt, sh);

    // ---- the pack vector of Algorithm 2: the words, and how many each bin sends ----------------------
    const uint32_t wbytes = ld.word_bytes;
    asm volatile("" : "+v"(sent_mask));
    // Where workgroups are many, a lane goes over the bits of its mask, as many rounds as the lane with most of them, which
    // takes fewest instructions; where few are at work and the chain counts, slot by slot, which takes the shortest one.
    // Slots / bits, in us: ResNet-50's table 61.0 / 60.1, bins of 800 and 8000 21.7 / 20.6, but 397 k elements 6.6 / 7.0, the
    // CIFAR table 9.3 / 9.9, 4 learners 21.3 / 23.8.
    if constexpr (ONE == kOneLayers || WAVES == 16) {
        uint32_t signs = 0u;   // bit 4 j + c: G of element c of slot j is negative
#pragma unroll
        for (int k = 4 * J - 1; k >= 0; --k) signs = __builtin_amdgcn_alignbit(signs, gb[k >> 2][k & 3], 31u);
        uint32_t row_start[P];   // place of the lane's first word of each row, two rows to a register
#pragma unroll
        for (int p = 0; p < P; ++p) row_start[p] = pre[p] + (row_at[2 * p] | (2 * p + 1 < J ? row_at[(2 * p + 1) % J] << 16 : 0u));
        for (uint32_t left = sent_mask; left != 0u; left &= left - 1u) {
            const uint32_t k = uint32_t(__builtin_ctz(left)), c = k & 3u;
            const uint32_t e = (k >> 2) * kRow + tid * 4u + c, b = __umulhi(e, M), idx = e - __umul24(b, T);   // idx: inside the bin
            const uint32_t rows = P == 1 || k < 8u ? row_start[0] : row_start[P - 1];
            const uint32_t at = ((rows >> ((k & 4u) * 4u)) & 0xFFFFu) + uint32_t(__popc(__builtin_amdgcn_ubfe(sent_mask, k & 12u, c)));
            const uint32_t word = (idx << 2) | (((signs >> k) & 1u) << 1) | 1u;   // ternary code: 1 +scale, 3 -scale
            if (wbytes == 1u) reinterpret_cast<uint8_t *>(s_words)[at] = uint8_t(word);
            else reinterpret_cast<uint16_t *>(s_words)[at] = uint16_t(word);
            atomicAdd(&s_cnt[b], 1u);
        }
    } else {
        keep_apart(place);
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const uint32_t f = (sent_mask >> (4 * j)) & 0xFu;
            if (f == 0u) continue;
            const uint32_t b0 = place[j] >> 16, left = place[j] & 0xFFFFu;
            uint32_t at = row_at[j] + ((j & 1) ? pre[j / 2] >> 16 : pre[j / 2] & 0xFFFFu);
#pragma unroll
            for (uint32_t c = 0; c < 4u; ++c) {
                if (!((f >> c) & 1u)) continue;
                const uint32_t idx = c < left ? T - left + c : c - left;   // inside the bin
                const uint32_t word = (idx << 2) | ((gb[j][c] >> 31) ? 3u : 1u);   // ternary code: -scale / +scale
                if (wbytes == 1u) reinterpret_cast<uint8_t *>(s_words)[at] = uint8_t(word);
                else reinterpret_cast<uint16_t *>(s_words)[at] = uint16_t(word);
                ++at;
            }
            const uint32_t f1 = left < 4u ? f >> left : 0u;
            const uint32_t k1 = uint32_t(__popc(f1)), k0 = uint32_t(__popc(f)) - k1;
            if (k0) atomicAdd(&s_cnt[b0], k0);
            if (k1) atomicAdd(&s_cnt[b0 + 1u], k1);
        }
    }
    __syncthreads();

    // ---- what does not need the layer: counts per bin, running counts, the optional g_max vector -------
    if (wbytes == 1u) {
        uint8_t *cp = packet + ld.counts_offset + td.first_bin;
        for (uint32_t i = tid; i < nb; i += WG) cp[i] = uint8_t(s_cnt[i]);
    } else {
        uint16_t *cp = reinterpret_cast<uint16_t *>(packet + ld.counts_offset) + td.first_bin;
        for (uint32_t i = tid; i < nb; i += WG) cp[i] = uint16_t(s_cnt[i]);
    }
    if (a.keep_gmax) {
        float *gm_out = reinterpret_cast<float *>(a.scratch + uint64_t(lr) * a.scratch_stride + a.o_gmax) + ld.bin_start + td.first_bin;
        for (uint32_t i = tid; i < nb; i += WG) gm_out[i] = __uint_as_float(s_gmax[i]);
        if (ONE == kOneTable) __syncthreads();   // the records' sums come into their place
    }
    const uint32_t t0 = (64u - (td.first_bin & 63u)) & 63u;   // first bin of the tile that starts a chunk of 64
    for (uint32_t t = t0 + 64u * wave; t < nb; t += WG) {
        uint32_t sum = 0u;
        for (uint32_t i = lane; i < t; i += 64u) sum += s_cnt[i];
        sum = wave_sum(sum);
        if (lane == 0u) s_chunk[t >> 6] = sum;
    }

    // A workgroup that waits in vain (see wait_polls) does all that is missing itself; it then takes its
    // own G from memory again (nobody has written this tile's residue yet) instead of holding sixteen
    // registers through that code.
    auto take_again = [&]() {
        load_slots();
        if (LAZY && a.lazy) apply_waiting();
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) gb[j][c] = __float_as_uint(r[j][c] + w[j][c]);
    };
    // ---- wait for the layer: its scale, the words before this tile --------------------------------------
    uint32_t first_at, base;   // place of the tile's first word in the packet; words of the layer before the tile
    float scale;
    if (ONE == kOneTable) {
        uint32_t l_ts = 0u, l_nt = 0u, l_wb = 0u;   // lane m keeps layer m's tiles and word width
        if (lane < l) { l_ts = a.layers[lane].ctile_start; l_nt = a.layers[lane].n_ctiles; l_wb = a.layers[lane].word_bytes; }   // l < kFoldLayers
        bool helped;
        if (!table_records<WG, VARIANT, LAZY>(a, sy, lr, epoch, tile, s_gmax, s_cnt, s_excl, s_sum, sh, helped)) return;   // nothing to go by: store nothing
        if (__builtin_expect(helped, false)) take_again();
        const uint32_t run_at = words_before_runs(sh, lane);
        base = words_before(s_excl, run_at, tile) - words_before(s_excl, run_at, ld.ctile_start);
        const uint32_t words = words_before(s_excl, run_at, l_ts + l_nt) - words_before(s_excl, run_at, l_ts);
        scale = layer_scale_of(s_sum + ld.ctile_start, ld.n_ctiles, ld.n_bins, lane);
        first_at = uint32_t(a.fixed_bytes) + wave_sum(uint32_t(pad16_dev(uint64_t(words) * l_wb))) + base * wbytes;   // below 2^32 like the packet
    } else {
        auto poll_tile = [&](bool ok, const uint32_t most_polls) {
            if (wave == 0u && lane < 3u) {
                uint64_t v = 0u;
                const uint64_t *src = sy.tile + 4u * tile + lane;
                for (uint32_t polls = 0; ok; ++polls) {
                    v = sync_load(src);
                    if (uint32_t(v) == epoch) break;
                    ok = polls < most_polls;
                    __builtin_amdgcn_s_sleep(8);
                }
                const uint32_t value = uint32_t(v >> 32);
                if (lane == 0u) sh.scale = __uint_as_float(value);
                else if (lane == 1u) sh.at = value;
                else sh.base = value;
            }
            return ok;
        };
        bool ok = layer_ok;
        if (__builtin_expect(block_any<WG>(!poll_tile(ok, a.wait_polls), sh.any[2]), false)) {
            ok = true;
            for (uint32_t times = 0; ok; ++times) {   // the layers before this one that are not done, and this one
                const uint32_t m = first_open_layer<WG>(sy, l, epoch, sh);
                ok = times <= l && complete_layer<WG, VARIANT, LAZY, true>(a, sy, lr, m, epoch, tile, s_gmax, s_cnt, sh);
                if (m == l) break;
            }
            if (block_any<WG>(!poll_tile(ok, kWaitPollsKnown), sh.any[2])) return;   // nothing to go by: store nothing
            take_again();
            __syncthreads();
        }
        base = sh.base;
        scale = sh.scale;
        first_at = sh.at;
    }

    asm volatile("" : "+v"(sent_mask));
    uint32_t tid_r = threadIdx.x;   // (the slots' place is worked out anew, not kept through the wait)
    asm volatile("" : "+v"(tid_r));
    // ---- the residue, in its final form: G - Gq at the sent elements, G elsewhere ---------------------------
    // (LAZY: nothing that a helper reads is written before here: residue, staged words, their number and the scale)
#pragma unroll
    for (int j = 0; j < J; ++j) {
        if (skip_row(j)) continue;
        vfloat4 R;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float G = __uint_as_float(gb[j][c]);
            if (LAZY) { R[c] = G; continue; }   // the corrections wait
            const float corrected = G - __builtin_copysignf(scale, G);
            R[c] = ((sent_mask >> (4 * j + c)) & 1u) ? corrected : G;
        }
        buffer_store_slot(r_buf, tid_r * 16u, uint32_t(j) * kRow * 4u, R);
        if ((n & 3u) != 0u && uint32_t(j) * WG + tid_r == (n >> 2))
            for (uint32_t c = 0; c < (n & 3u); ++c) rs[(n & ~3u) + c] = R[c];
    }
    if (LAZY) {   // the words for the next call, with tile-local indices, at the places worked out before
        uint8_t *const sb = a.scratch + uint64_t(lr) * a.scratch_stride;
        uint16_t *const stage = reinterpret_cast<uint16_t *>(sb + a.o_stage) + td.stage_base;
        const uint32_t row = lane < uint32_t(J * WAVES) ? s_rows[lane] : 0u, rows_before = wave_incl_scan(row) - row;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const uint32_t c2 = uint32_t(__popc((sent_mask >> (8 * p)) & 0xFu)) | (uint32_t(__popc((sent_mask >> (8 * p)) & 0xF0u)) << 16);
            const uint32_t before = wave_incl_scan(c2) - c2;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = 2 * p + h;
                if (j >= J) break;
                uint32_t at = uint32_t(__builtin_amdgcn_readlane(int(rows_before), j * WAVES + int(wave))) + (h ? before >> 16 : before & 0xFFFFu);
#pragma unroll
                for (uint32_t c = 0; c < 4u; ++c)
                    if ((sent_mask >> (4 * j + int(c))) & 1u) stage[at++] = uint16_t(((uint32_t(j) * kRow + tid_r * 4u + c) << 2) | ((gb[j][c] >> 31) ? 3u : 1u));
            }
        }
        if (tid_r == 0u) {
            TileOut o;
            o.gmax_sum = 0.0;
            o.count = tile_total;
            o.base = __float_as_uint(scale);
            reinterpret_cast<TileOut *>(sb + a.o_tile_out)[tile] = o;
        }
    }
    // ---- the words, at their place in the packet, four bytes at a time ---------------------------------------
    const uint32_t n_bytes = tile_total * wbytes, skew = first_at & 3u;
    const uint64_t limit = a.capacity & ~uint64_t(wbytes - 1u);   // no part of a word that does not fit
    for (uint32_t d = tid; 4u * d < skew + n_bytes; d += WG) {
        const uint64_t at = uint64_t(first_at - skew) + 4u * d;
        const uint32_t o = 4u * d - skew;   // first byte of the four among the tile's words; wraps below zero in the first
        if (4u * d >= skew && o + 4u <= n_bytes && at + 4u <= limit) {
            const uint32_t lo = s_words[o >> 2], hi = s_words[(o >> 2) + 1u];
            *reinterpret_cast<uint32_t *>(packet + at) = __builtin_amdgcn_alignbyte(hi, lo, o & 3u);
        } else {
            for (uint32_t c = 0; c < 4u; ++c)
                if (o + c < n_bytes && at + c < limit) packet[at + c] = reinterpret_cast<const uint8_t *>(s_words)[o + c];
        }
    }
    // chunks[c] = words of the layer in bins < 64 c, for the chunk starts inside this tile
    for (uint32_t t = t0 + 64u * tid; t < nb; t += 64u * WG)
        reinterpret_cast<uint32_t *>(packet + ld.chunks_offset)[(td.first_bin + t) >> 6] = base + s_chunk[t >> 6];
}

// ==============================================================================================
// k_scan: per layer, scale = (sum of g_max) / n_bins in float64 rounded once to float32, and the
// exclusive scan of the tiles' word counts.  One workgroup of 1024 threads per layer; a thread
// owns a contiguous run of tiles so that its loads are independent and issue back to back.
// ==============================================================================================
constexpr uint32_t kScanWG = 1024;

__global__ __launch_bounds__(kScanWG) void k_scan(const CompressArgs a)
{
    const uint32_t l = blockIdx.x;
    if (l >= a.n_layers) return;
    // per-learner buffers: blockIdx.y selects the learner of a batched call
    const uint32_t lr = blockIdx.y;
    uint8_t *const sb = a.scratch + uint64_t(lr) * a.scratch_stride;
    TileOut *const tile_out = reinterpret_cast<TileOut *>(sb + a.o_tile_out);
    uint32_t *const layer_nsel = reinterpret_cast<uint32_t *>(sb + a.o_layer_nsel);
    float *const layer_scale = reinterpret_cast<float *>(sb + a.o_layer_scale);
    const LayerDev ld = a.layers[l];
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform across the wave
    const uint32_t nt = ld.n_ctiles, ts = ld.ctile_start;
    const uint32_t per = (nt + kScanWG - 1) / kScanWG;
    const uint32_t lo = tid * per < nt ? tid * per : nt;
    const uint32_t hi = lo + per < nt ? lo + per : nt;

    __shared__ uint32_t s_wsum[16];
    __shared__ double s_dsum[16];

    // a thread's run of tiles is read once into registers when it is short (up to 8 records: layers of
    // up to 8192 tiles), so the kernel costs one memory round trip before the scan and one store after
    constexpr uint32_t kHold = 8;
    uint32_t cnt[kHold];
    uint32_t csum = 0u;
    double dsum = 0.0;
    if (per <= kHold) {
        TileOut rec[kHold];
#pragma unroll
        for (uint32_t i = 0; i < kHold; ++i) {
            rec[i].gmax_sum = 0.0; rec[i].count = 0u;
            if (lo + i < hi) rec[i] = tile_out[ts + lo + i];
        }
#pragma unroll
        for (uint32_t i = 0; i < kHold; ++i) { cnt[i] = rec[i].count; csum += rec[i].count; dsum += rec[i].gmax_sum; }
    } else {
        for (uint32_t i = lo; i < hi; ++i) { const TileOut o = tile_out[ts + i]; csum += o.count; dsum += o.gmax_sum; }
    }

    const uint32_t incl = wave_incl_scan(csum);
    dsum = wave_sum_f64(dsum);
    if (lane == 63) s_wsum[wave] = incl;
    if (lane == 0) s_dsum[wave] = dsum;
    __syncthreads();
    uint32_t wave_base = 0u;
    for (uint32_t wv = 0; wv < wave; ++wv) wave_base += s_wsum[wv];
    uint32_t run = wave_base + incl - csum;
    if (per <= kHold) {
#pragma unroll
        for (uint32_t i = 0; i < kHold; ++i)
            if (lo + i < hi) { tile_out[ts + lo + i].base = run; run += cnt[i]; }
    } else {
        for (uint32_t i = lo; i < hi; ++i) { tile_out[ts + i].base = run; run += tile_out[ts + i].count; }
    }
    if (tid == 0) {
        double total = 0.0;
        uint32_t nsel = 0u;
        for (uint32_t wv = 0; wv < kScanWG / 64u; ++wv) { total += s_dsum[wv]; nsel += s_wsum[wv]; }
        layer_scale[l] = float(total / double(ld.n_bins));
        layer_nsel[l] = nsel;
    }
}

// ==============================================================================================
// k_place: staged entries -> final words; residue <- G - Gq at the sent elements; chunk offsets;
// header, records and padding (last workgroup).  With long bins a tile sends a few dozen words at
// most in steady state, so 16 lanes serve a tile and a workgroup serves 16 tiles; the whole grid
// is resident at once and the kernel costs about three dependent memory round trips.  Its pace is
// set by the scattered read-modify-writes of the residue: a bare kernel that does nothing else
// needs as long for the same number of words.
// ==============================================================================================
// LANES lanes serve a tile: 16 where bins are long and a tile sends a few dozen words, 64 for tables
// with short bins, whose tiles send several hundred (5 % off the compress time of the ResNet-50
// table, 23 % off the small CIFAR table; 64 lanes cost the 125 M-element table half a percent).
// MODE kPlaceEager does all of it.  kPlaceWords leaves the residue alone: the corrections wait in
// the scratch block (staged entries, tile counts, layer scales) and the next lazy k_fused of this
// learner applies them in registers, where they cost next to nothing; until then the residue holds
// G at the sent elements.  kPlaceResidue applies waiting corrections and nothing else.
// FOLD = true (small tables: up to kFoldTiles tiles and kFoldLayers layers; 64 lanes per tile): there
// is no k_scan launch.  Every workgroup scans the word counts of all tiles itself (8 per thread, a
// few kilobytes from L2) and every wave sums the g_max totals of its tile's layer, in one fixed
// order (fold_layer_scale) that the header block uses as well; on tables that take 35-90 us per
// step this is cheaper than a launch of 4 us and the gap before it.
__device__ __forceinline__ float fold_layer_scale(const TileOut *tile_out, const uint32_t ctile_start,
                                                  const uint32_t n_ctiles, const uint32_t n_bins, const uint32_t lane)
{
    double s = 0.0;
    for (uint32_t t = lane; t < n_ctiles; t += 64u) s += tile_out[ctile_start + t].gmax_sum;
    return float(wave_sum_f64(s) / double(n_bins));
}

template <uint32_t LANES, uint32_t MODE, bool FOLD>
__global__ __launch_bounds__(kWG) void k_place(const CompressArgs a)
{
    static_assert(!FOLD || (LANES == 64u && MODE != kPlaceResidue), "the folded scan serves 64-lane placement launches");
    constexpr uint32_t kPlaceLanes = LANES, kPlaceTiles = kWG / LANES;
    const uint32_t tid = threadIdx.x;
    // per-learner buffers: blockIdx.y selects the learner of a batched call
    const uint32_t lr = blockIdx.y;
    uint8_t *const sb = a.scratch + uint64_t(lr) * a.scratch_stride;
    TileOut *const tile_out = reinterpret_cast<TileOut *>(sb + a.o_tile_out);
    uint32_t *const layer_nsel = reinterpret_cast<uint32_t *>(sb + a.o_layer_nsel);
    float *const layer_scale = reinterpret_cast<float *>(sb + a.o_layer_scale);
    uint32_t *const chunk_rel = reinterpret_cast<uint32_t *>(sb + a.o_chunk_rel);
    uint16_t *const stage_all = reinterpret_cast<uint16_t *>(sb + a.o_stage);
    uint8_t *const packet = a.packet[lr];

    // s_excl[t] = words of all tiles before tile t (tile table order: layer after layer)
    __shared__ uint32_t s_excl[FOLD ? kFoldTiles + 1u : 1u];
    if (FOLD) {
        __shared__ uint32_t s_fw[4];
        constexpr uint32_t kPer = kFoldTiles / kWG;
        const uint32_t lane = tid & 63u;
        const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        uint32_t cnt[kPer], sum = 0u;
#pragma unroll
        for (uint32_t i = 0; i < kPer; ++i) {
            const uint32_t t = tid * kPer + i;
            cnt[i] = t < a.n_tiles ? tile_out[t].count : 0u;
            sum += cnt[i];
        }
        const uint32_t incl = wave_incl_scan(sum);
        if (lane == 63u) s_fw[wave] = incl;
        __syncthreads();
        uint32_t run = incl - sum;
        for (uint32_t wv = 0; wv < wave; ++wv) run += s_fw[wv];
#pragma unroll
        for (uint32_t i = 0; i < kPer; ++i) {
            s_excl[tid * kPer + i] = run;
            run += cnt[i];
        }
        if (tid == kWG - 1u) s_excl[kFoldTiles] = run;
        __syncthreads();
    }

    const bool header_block = blockIdx.x == (a.n_tiles + kPlaceTiles - 1u) / kPlaceTiles;   // the last one (gridDim would be a hidden argument)
    if (MODE == kPlaceResidue && header_block) return;
    if (MODE != kPlaceResidue && header_block) {
        if (FOLD) {
            __shared__ float s_fscale[FOLD ? kFoldLayers : 1u];
            const uint32_t lane = tid & 63u;
            const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
            for (uint32_t l = wave; l < a.n_layers; l += 4u) {
                const float sc = fold_layer_scale(tile_out, a.layers[l].ctile_start, a.layers[l].n_ctiles, a.layers[l].n_bins, lane);
                if (lane == 0u) s_fscale[l] = sc;
            }
            __syncthreads();
            place_header<kWG>(a, packet, header_layer(a), [&](uint32_t l, const LayerDev &ld, uint32_t &nsel, float &sc) {
                nsel = s_excl[ld.ctile_start + ld.n_ctiles] - s_excl[ld.ctile_start];
                sc = s_fscale[l];
                layer_nsel[l] = nsel;   // and left in the scratch block for whoever applies the corrections later
                layer_scale[l] = sc;
            });
        } else {
            place_header<kWG>(a, packet, header_layer(a), [&](uint32_t l, const LayerDev &, uint32_t &nsel, float &sc) { nsel = layer_nsel[l]; sc = layer_scale[l]; });
        }
        return;
    }

    const uint32_t sub = tid & (kPlaceLanes - 1u);
    const uint32_t tile = blockIdx.x * kPlaceTiles + (tid / kPlaceLanes);
    if (tile >= a.n_tiles) return;
    const TileDev td = a.tiles[tile];
    const uint32_t l = td.layer();

    // independent loads first: the tile's counters, its first staged entries, the layer's fields
    const TileOut to = tile_out[tile];
    const uint32_t cnt = to.count;
    const uint32_t base = FOLD ? s_excl[tile] - s_excl[a.layers[l].ctile_start] : to.base;
    const uint16_t *__restrict__ stage = stage_all + td.stage_base;
    float *__restrict__ rs = a.residue[lr] + td.elem_base;
    const uint32_t s_first = stage[sub];  // speculative: the staging array has 64 entries of slack
    const float scale = FOLD ? fold_layer_scale(tile_out, a.layers[l].ctile_start, a.layers[l].n_ctiles, a.layers[l].n_bins, sub)
                             : layer_scale[l];
    const uint32_t wbytes = a.layers[l].word_bytes;
    const uint64_t chunks_offset = a.layers[l].chunks_offset;
    const uint32_t chunk_start = a.layers[l].chunk_start;

    // first word of this layer = end of the fixed part + the (padded) word sections before it
    uint64_t woff = 0;
    for (uint32_t m = sub; m < l; m += kPlaceLanes) {
        const uint32_t nsel_m = FOLD ? s_excl[a.layers[m].ctile_start + a.layers[m].n_ctiles] - s_excl[a.layers[m].ctile_start]
                                     : layer_nsel[m];
        woff += pad16_dev(uint64_t(nsel_m) * a.layers[m].word_bytes);
    }
#pragma unroll
    for (uint32_t d = kPlaceLanes / 2; d > 0; d >>= 1) {
        const uint32_t lo = __shfl_xor(uint32_t(woff), d, kPlaceLanes), hi = __shfl_xor(uint32_t(woff >> 32), d, kPlaceLanes);
        woff += (uint64_t(hi) << 32) | lo;
    }
    woff += a.fixed_bytes;

    // Eight words per lane and round, so that a tile with hundreds of words (short bins send several
    // percent of their elements) costs a few memory round trips instead of one per 16 words.
    const uint32_t T = td.L_T, M = td.magic;
    constexpr uint32_t kU = 8;
    for (uint32_t p0 = sub; p0 < cnt; p0 += kPlaceLanes * kU) {
        uint32_t s[kU];
        float g[kU];
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
            const uint32_t p = p0 + kPlaceLanes * u;
            s[u] = p < cnt ? (p == sub ? s_first : uint32_t(stage[p])) : 0u;  // 0: code 0, never a real entry
        }
        // The sent elements' residue update of Algorithm 2: G minus sign(G) * scale; G is what k_fused left in the
        // residue: a read-modify-write, measured at a 64-byte read and a 32-byte write per word.
        // (Keeping G next to the staged entry, so that this becomes a plain store, was built and
        // measured three times: in an array of its own for all layers, for short-bin layers only,
        // and as 8-byte entries in the same staging stretch.  The scattered partial writes, not
        // the reads, set the pace here, and k_fused lost more to the wider staging stores, about
        // 1 %, than this kernel gained.)
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u)
            g[u] = (MODE != kPlaceWords && (s[u] & 1u)) ? rs[s[u] >> 2] : 0.f;
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
            if (!(s[u] & 1u)) continue;  // codes are 1 or 3
            const uint32_t p = p0 + kPlaceLanes * u;
            const uint32_t e = s[u] >> 2, code = s[u] & 3u;
            if (MODE != kPlaceResidue) {
                const uint32_t b = bin_of(e, T, M);
                const uint32_t word = ((e - b * T) << 2) | code;  // index inside the bin, ternary code
                const uint64_t at = woff + uint64_t(base + p) * wbytes;
                if (at + wbytes <= a.capacity) {
                    if (wbytes == 1u) packet[at] = uint8_t(word);
                    else *reinterpret_cast<uint16_t *>(packet + at) = uint16_t(word);
                }
            }
            if (MODE != kPlaceWords) rs[e] = code == 1u ? g[u] - scale : g[u] + scale;
        }
    }
    if (MODE == kPlaceResidue) return;
    if (MODE == kPlaceWords && sub == 0u) tile_out[tile].base = __float_as_uint(scale);   // for the next call, with the count

    // chunks[c] = words of the layer in bins < 64 c, for the chunk starts inside this tile
    const uint32_t t0 = (64u - (td.first_bin & 63u)) & 63u;
    for (uint32_t t = t0 + 64u * sub; t < td.n_bins; t += 64u * kPlaceLanes) {
        const uint32_t c = (td.first_bin + t) >> 6;
        reinterpret_cast<uint32_t *>(packet + chunks_offset)[c] = base + chunk_rel[chunk_start + c];
    }
}

// ==============================================================================================
// k_place_tiled: the eager placement for tables with short bins.  Where L_T <= 64 several percent of
// the elements are sent (7.9 % on the ResNet-50 table) and three quarters of the residue's 64-byte
// lines hold a sent element, so correcting the residue word by word (a scattered read-modify-write
// per word, as k_place does) moves far more than the lines themselves.  Here a workgroup owns one
// compress tile: it places the tile's words, marks the sent elements in an LDS byte map (the
// scheme of the lazy k_fused), and then streams over the tile's residue line by line: a line with a
// mark is loaded whole, corrected with the same single float32 subtraction or addition, and written
// back whole; a line without one is not touched.  Tiles that send only a few words (the fully
// connected layers of such a table) and tiles that are not 16-byte aligned correct word by word.
// ==============================================================================================
constexpr uint32_t kTiledMinWords = 24;  // fewer words than this in a tile: word-by-word corrections

__global__ __launch_bounds__(kWG) void k_place_tiled(const CompressArgs a)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lr = blockIdx.y;   // the learner of a batched call
    uint8_t *const sb = a.scratch + uint64_t(lr) * a.scratch_stride;
    TileOut *const tile_out = reinterpret_cast<TileOut *>(sb + a.o_tile_out);
    uint32_t *const layer_nsel = reinterpret_cast<uint32_t *>(sb + a.o_layer_nsel);
    float *const layer_scale = reinterpret_cast<float *>(sb + a.o_layer_scale);
    const uint32_t *const chunk_rel = reinterpret_cast<const uint32_t *>(sb + a.o_chunk_rel);
    const uint16_t *const stage_all = reinterpret_cast<const uint16_t *>(sb + a.o_stage);
    uint8_t *const packet = a.packet[lr];

    if (blockIdx.x == a.n_tiles) {   // the grid has one workgroup per tile and this one
        place_header<kWG>(a, packet, header_layer(a), [&](uint32_t l, const LayerDev &, uint32_t &nsel, float &sc) { nsel = layer_nsel[l]; sc = layer_scale[l]; });
        return;
    }
    const uint32_t tile = blockIdx.x;   // the grid has one workgroup per tile and one for the header
    const TileDev td = a.tiles[tile];
    const uint32_t l = td.layer();
    const TileOut to = tile_out[tile];
    const uint32_t cnt = to.count, base = to.base;
    const uint32_t n = td.n_elems, T = td.L_T, M = td.magic;
    const float scale = layer_scale[l];
    const uint32_t wbytes = a.layers[l].word_bytes;
    const uint64_t chunks_offset = a.layers[l].chunks_offset;
    const uint32_t chunk_start = a.layers[l].chunk_start;
    const uint16_t *__restrict__ stage = stage_all + td.stage_base;
    float *__restrict__ rs = a.residue[lr] + td.elem_base;
    const bool tiled = td.aligned() && cnt >= kTiledMinWords;   // uniform over the workgroup

    __shared__ __attribute__((aligned(16))) uint8_t s_fix[16384];   // code of the word an element was sent with, or 0
    __shared__ uint64_t s_part[kWG / 64u];
    if (tiled)
        for (uint32_t i = tid; i < (n + 15u) / 16u; i += kWG) reinterpret_cast<uint4 *>(s_fix)[i] = make_uint4(0u, 0u, 0u, 0u);

    // first word of this layer = end of the fixed part + the (padded) word sections before it
    uint64_t part = 0;
    for (uint32_t m = tid; m < l; m += kWG) part += pad16_dev(uint64_t(layer_nsel[m]) * a.layers[m].word_bytes);
#pragma unroll
    for (uint32_t d = 32; d > 0; d >>= 1) {
        const uint32_t lo = __shfl_xor(uint32_t(part), d, 64), hi = __shfl_xor(uint32_t(part >> 32), d, 64);
        part += (uint64_t(hi) << 32) | lo;
    }
    if (lane == 0) s_part[wave] = part;
    __syncthreads();   // the byte map is cleared, the partial sums are there
    uint64_t woff = a.fixed_bytes;
    for (uint32_t wv = 0; wv < kWG / 64u; ++wv) woff += s_part[wv];

    for (uint32_t p = tid; p < cnt; p += kWG) {
        const uint32_t s = stage[p];
        const uint32_t e = s >> 2, code = s & 3u;
        if (!(code & 1u) || e >= n) continue;   // codes are 1 or 3 and indices lie inside the tile
        const uint32_t b = bin_of(e, T, M);
        const uint32_t word = ((e - b * T) << 2) | code;   // index inside the bin, ternary code
        const uint64_t at = woff + uint64_t(base + p) * wbytes;
        if (at + wbytes <= a.capacity) {
            if (wbytes == 1u) packet[at] = uint8_t(word);
            else *reinterpret_cast<uint16_t *>(packet + at) = uint16_t(word);
        }
        if (tiled) s_fix[e] = uint8_t(code);
        else {   // the sent elements' residue update of Algorithm 2, one element at a time
            const float g = rs[e];
            rs[e] = code == 1u ? g - scale : g + scale;
        }
    }

    if (tiled) {
        __syncthreads();   // the byte map is complete
        // Lines of the residue: four consecutive 16-byte slots, the first on a 64-byte boundary.  The
        // tile starts `shift` slots past such a boundary; virtual slot v = shift + (slot in the tile),
        // so that the four lanes v & ~3 .. v | 3 share a line and decide together.
        const uint32_t shift = uint32_t(reinterpret_cast<uintptr_t>(rs) >> 4) & 3u;
        const uint32_t n_virtual = (shift + (n + 3u) / 4u + 3u) & ~3u;
        for (uint32_t v = tid; v < n_virtual; v += kWG) {
            const uint32_t e0 = (v - shift) * 4u;   // wraps to a huge value below the tile's start
            const bool ok = v >= shift && e0 < n;
            const uint32_t codes = ok ? *reinterpret_cast<const uint32_t *>(&s_fix[e0]) : 0u;   // bytes past n are 0
            uint32_t any = codes;
            any |= uint32_t(__shfl_xor(int(any), 1, 64));
            any |= uint32_t(__shfl_xor(int(any), 2, 64));
            if (!ok || any == 0u) continue;
            if (e0 + 4u <= n) {
                const vfloat4 r = load_stream4(rs + e0);
                float g[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint32_t code = (codes >> (8 * c)) & 3u;
                    if (code == 1u) g[c] = g[c] - scale;
                    else if (code == 3u) g[c] = g[c] + scale;
                }
                store_stream4(rs + e0, vfloat4{g[0], g[1], g[2], g[3]});
            } else {   // the layer's last elements: what follows them is not ours to write
                for (uint32_t c = 0; c < 4u && e0 + c < n; ++c) {
                    const uint32_t code = (codes >> (8u * c)) & 3u;
                    if (code == 1u) rs[e0 + c] = rs[e0 + c] - scale;
                    else if (code == 3u) rs[e0 + c] = rs[e0 + c] + scale;
                }
            }
        }
    }

    // chunks[c] = words of the layer in bins < 64 c, for the chunk starts inside this tile
    const uint32_t t0 = (64u - (td.first_bin & 63u)) & 63u;
    for (uint32_t t = t0 + 64u * tid; t < td.n_bins; t += 64u * kWG) {
        const uint32_t c = (td.first_bin + t) >> 6;
        reinterpret_cast<uint32_t *>(packet + chunks_offset)[c] = base + chunk_rel[chunk_start + c];
    }
}

// ==============================================================================================
// k_unpack: dense_out <- sum over learners, in learner order, of the decoded packets.
// A workgroup owns a tile of the output in LDS, and serves a run of up to 8 neighbouring tiles one
// after the other.  Phase 1 gathers, for every (bin, learner) of the run, the word count and the
// position of the first word (one wave per learner, all learners' loads in flight together); with
// up to 16 learners this is done once per run, which is what the runs are for: at L_T = 500 the
// 8 tiles of a 64-bin chunk need the same count lines and the same prefix sums.  Phase 2, per
// tile: a lane group per bin reads the 16 learners' table entries with a few wide LDS loads,
// fetches the words of all 16 learners, and adds +-scale in learner order: with LDS float atomics
// where bins are long and few lanes have a word, with plain LDS loads and stores where bins are
// short (see lds_add).  All adds to one address come from one wave in program order and the LDS
// unit executes a wave's operations in order, so the sum order is fixed: learner 0 first.  (LDS
// float adds round to nearest even and keep denormals, like v_add_f32.)  On the 125 M-element table with 16 learners
// a pass that only clears and writes the tiles takes 88 us, phase 1 per tile added 79 us and
// phase 2 adds 63 us; sharing phase 1 over a run brought the whole launch from 230-250 to 185 us.
// ==============================================================================================
// Row strides of the two LDS tables.  With the natural strides (16 words, 8 words) the 64 lanes of
// phase 1, which write one row each, would hit 2 and 4 of the 32 banks; 20 and 12 words spread
// them over 8 banks and keep the rows 16-byte aligned for the wide reads of phase 2.
template <uint32_t LG>
constexpr uint32_t kOffStride = LG + 4u;  // uint32 per row, LG used
constexpr uint32_t kCntStride = 24;  // uint16 per row, LG used

// What the kernels look up in a packet for one chunk of a layer: the header, where the layer's words begin, how many stand
// before the chunk, the scale.  The same for all threads: scalar loads.  `settle` behind the loads of all packets keeps the
// compiler from waiting for one packet before it asks for the next, as it does where registers or branches suggest it (k_unpack_few,
// 4 packets, 0.4 M elements 4.4 us, one after the other 5.3).
struct PacketChunk {
    vuint4 head;          // magic, version, status, n_layers
    vuint2 total_bytes;
    vuint2 words_offset;
    uint32_t before;
    float scale;
    __device__ __forceinline__ void fetch(const uint8_t *const pk, const uint32_t layer, const uint32_t chunks_offset, const uint32_t chunk)
    {
        const uint8_t *const rec = pk + sizeof(adacomp_packet_header_t) + sizeof(adacomp_packet_layer_t) * layer;
        head = packet_field<vuint4>(pk);
        total_bytes = packet_field<vuint2>(pk + 16);
        words_offset = packet_field<vuint2>(rec + offsetof(adacomp_packet_layer_t, words_offset));
        scale = packet_field<float>(rec + offsetof(adacomp_packet_layer_t, scale));
        before = packet_field<uint32_t>(pk + chunks_offset + 4u * chunk);
    }
    // whether the packet is one that this call can read
    __device__ __forceinline__ bool fits(const UnpackHead &a) const
    {
        return (head.x == ADACOMP_PACKET_MAGIC) & (head.y == ADACOMP_PACKET_VERSION) & (head.z == ADACOMP_STATUS_COMPLETE) & (head.w == a.n_layers) & (total_bytes.y == 0u);
    }
    // words (of `size` bytes each) from the packet's start to the chunk's first one
    __device__ __forceinline__ uint64_t first_word(const uint32_t size) const
    {
        return uint64_t(uint32_t(((uint64_t(words_offset.y) << 32) | words_offset.x) / size)) + before;   // packets stay below 2^32 words (host check)
    }
};
// ... of the headers alone, together with the counts of the lane's bin (which otherwise wait for what says whether they are needed)
template <uint32_t N>
__device__ __forceinline__ void settle_heads(PacketChunk (&p)[N], uint32_t (&c)[N])
{
    static_assert(N == 2 || N == 4, "operands of one statement");
    if constexpr (N == 2)
        asm volatile("" : "+s"(p[0].head), "+s"(p[0].total_bytes), "+s"(p[1].head), "+s"(p[1].total_bytes), "+v"(c[0]), "+v"(c[1]));
    else
        asm volatile("" : "+s"(p[0].head), "+s"(p[0].total_bytes), "+s"(p[1].head), "+s"(p[1].total_bytes), "+s"(p[2].head), "+s"(p[2].total_bytes),
                          "+s"(p[3].head), "+s"(p[3].total_bytes), "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]));
}
template <uint32_t N>
__device__ __forceinline__ void settle(PacketChunk (&p)[N])
{
    static_assert(N == 2 || N == 4, "operands of one statement: what is in flight together");
    asm volatile("" : "+s"(p[0].head), "+s"(p[0].total_bytes), "+s"(p[0].words_offset), "+s"(p[0].before), "+s"(p[0].scale),
                      "+s"(p[1].head), "+s"(p[1].total_bytes), "+s"(p[1].words_offset), "+s"(p[1].before), "+s"(p[1].scale));
    if constexpr (N == 4)
        asm volatile("" : "+s"(p[2].head), "+s"(p[2].total_bytes), "+s"(p[2].words_offset), "+s"(p[2].before), "+s"(p[2].scale),
                          "+s"(p[3].head), "+s"(p[3].total_bytes), "+s"(p[3].words_offset), "+s"(p[3].before), "+s"(p[3].scale));
}

// Phase 1 for learners k0 .. k0 + LG - 1 (LG = 8 or 16) and the bins [row0_bin, scan_end) of one 64-bin chunk: word
// count and position of the first word of every (bin, learner), into the LDS tables (row = bin -
// row0_bin).  The caller has a barrier before (the tables are free) and after (they are filled).
template <bool W8, uint32_t LG, class Args>
__device__ __forceinline__ void unpack_tables(const Args &a, const UTileDev &ut0,
                                              const uint32_t row0_bin, const uint32_t scan_end, const uint32_t k0,
                                              uint32_t (*s_off)[kOffStride<LG>], uint16_t (*s_cnt)[kCntStride],
                                              float *s_scale, uint32_t *s_cmax)
{
    typedef typename std::conditional<W8, uint8_t, uint16_t>::type word_t;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform across the wave
    const uint32_t chunk = row0_bin >> 6;
    const uint32_t b = (chunk << 6) + lane;           // the bin this lane looks up
    const bool in_scan = b < scan_end;                // bins of the chunk up to the end of the group
    const bool in_rows = in_scan && b >= row0_bin;
    constexpr uint32_t kPerWave = LG / 4u;
    const uint32_t nk = a.n_learners - k0 < LG ? a.n_learners - k0 : LG;

    if (tid == 0) *s_cmax = 0u;

    // Wave w serves learners w, w + 4, ...; all their loads are issued first: without a branch around them (learners
    // past nk look at the first one's packet), and what is the same for all bins through scalar loads.
    uint32_t wmax = 0u;
    uint32_t c[kPerWave];
    PacketChunk pc[kPerWave];
#pragma unroll
    for (uint32_t q = 0; q < kPerWave; ++q) {
        const uint32_t kk = wave + 4u * q;
        const uint8_t *const pk = a.packets[k0 + (kk < nk ? kk : 0u)];
        // counts and chunk offsets sit in the fixed part, which every packet buffer holds
        c[q] = reinterpret_cast<const word_t *>(pk + ut0.counts_offset)[in_scan ? b : row0_bin];
        if (LG == 8u) pc[q].fetch(pk, ut0.layer(), ut0.chunks_offset, chunk);
    }
    if constexpr (LG == 8u) settle(pc);
    __syncthreads();   // (s_cmax)
#pragma unroll
    for (uint32_t q = 0; q < kPerWave; ++q) {
        const uint32_t kk = wave + 4u * q;  // < LG; learners past nk get empty entries
        if (LG != 8u) pc[q].fetch(a.packets[k0 + (kk < nk ? kk : 0u)], ut0.layer(), ut0.chunks_offset, chunk);   // (of four at once the registers spill)
        const float sc = pc[q].scale;
        const bool ok = (kk < nk) & pc[q].fits(a);
        const uint32_t limit = pc[q].total_bytes.x / uint32_t(sizeof(word_t));  // words that fit in the packet
        const uint32_t cq = ok && in_scan ? c[q] : 0u;   // a packet that does not match contributes nothing
        const uint32_t incl = wave_incl_scan(cq);
        // A bin whose words would lie past the packet's total_bytes (counts or offsets that do not
        // belong together) contributes nothing: no word is read from outside the packet.
        const uint64_t first = pc[q].first_word(uint32_t(sizeof(word_t))) + (incl - cq);
        const bool inside = first + cq <= limit;
        const uint32_t cw = inside ? cq : 0u;
        if (in_rows) {
            s_off[b - row0_bin][kk] = inside ? uint32_t(first) : 0u;
            s_cnt[b - row0_bin][kk] = uint16_t(cw);
        }
        if (lane == 0) s_scale[kk] = sc;
        wmax = (in_rows && cw > wmax) ? cw : wmax;
    }
    wmax = wave_max(wmax);
    if (lane == 0) atomicMax(s_cmax, wmax);
}

// acc[idx] <- acc[idx] + v as an LDS load, a float add and an LDS store.  The LDS float atomic of
// this GPU works through its active lanes one after the other (3 cycles per lane, measured: a wave
// with all lanes busy holds the unit for 194 cycles, whatever the addresses), which made the adds
// the bottleneck of the short-bin path.  The plain sequence is safe here: the words of one learner
// name different elements, so no two lanes write one address in the same step; steps of different
// learners that do meet on an address come from lanes of one wave in program order, and the LDS
// unit executes a wave's instructions in order.  The accesses are volatile so that the compiler
// keeps that order.  The sum, a single float32 addition per word, is the one the atomic gives.
typedef __attribute__((address_space(3))) float lds_float;  // a float in LDS: ds_read / ds_write, not flat accesses
__device__ __forceinline__ volatile lds_float *lds_volatile(float *p) { return (volatile lds_float *)p; }
__device__ __forceinline__ void lds_add(float *acc, const uint32_t idx, const float v)
{
    volatile lds_float *p = lds_volatile(acc) + idx;
    const float cur = *p;
    *p = cur + v;
}

// Phase 2 for one tile: a lane group owns a bin (table row row0 + bin index inside the tile).
// words_on_their_way: called once by every thread, when the first words that it waits for have been asked for (NoHook: not at all).
struct NoHook {
    __device__ __forceinline__ void operator()() const {}
};
template <bool W8, uint32_t LG, class Hook, class Args>
__device__ __forceinline__ void unpack_adds(const Args &a, const UTileDev &ut, const uint32_t row0, const uint32_t k0,
                                            float *s_acc, uint32_t (*s_off)[kOffStride<LG>],
                                            uint16_t (*s_cnt)[kCntStride], const float *s_scale, const uint32_t *s_cmax, Hook words_on_their_way)
{
    typedef typename std::conditional<W8, uint8_t, uint16_t>::type word_t;
    const uint32_t tid = threadIdx.x;
    const uint32_t n = ut.n_elems, T = ut.L_T, nb = ut.n_bins;
    const uint32_t nk = a.n_learners - k0 < LG ? a.n_learners - k0 : LG;
    constexpr bool kHook = !std::is_same<Hook, NoHook>::value;
    if (W8) {
        // Short bins (8-bit words) send several words each, about 8 % of the elements on the
        // ResNet-50 table.  Four lanes own a bin and lane j fetches the aligned 4 bytes number j of
        // the bin's run of words, for all 16 learners at once (16 words per bin and learner; longer
        // runs are finished with byte loads), then adds learner after learner in program order.
        const uint32_t sub = tid & 3u;
        const bool live = !kHook || (tid >> 2) < nb;   // (the hook is for all threads)
        if (!kHook && (tid >> 2) >= nb) return;
        const uint32_t lb = live ? tid >> 2 : 0u;
        const uint32_t row = row0 + lb;
        const uint32_t span = T < n - lb * T ? T : n - lb * T;  // elements of this bin held by the tile
        float *acc = s_acc + lb * T;
        // 8 learners at a time, to keep the register count (and with it the number of resident
        // workgroups) where the 16-bit path has it
#pragma unroll 1
        for (uint32_t h0 = 0; h0 < LG; h0 += 8u) {
            if (h0 >= nk) break;
            uint32_t cc[8], off[8], packed[8];
            {
                const uint4 t = *reinterpret_cast<const uint4 *>(&s_cnt[row][h0]);
                cc[0] = t.x & 0xFFFFu; cc[1] = t.x >> 16; cc[2] = t.y & 0xFFFFu; cc[3] = t.y >> 16;
                cc[4] = t.z & 0xFFFFu; cc[5] = t.z >> 16; cc[6] = t.w & 0xFFFFu; cc[7] = t.w >> 16;
                const uint4 o0 = *reinterpret_cast<const uint4 *>(&s_off[row][h0]);
                const uint4 o1 = *reinterpret_cast<const uint4 *>(&s_off[row][h0 + 4u]);
                off[0] = o0.x; off[1] = o0.y; off[2] = o0.z; off[3] = o0.w;
                off[4] = o1.x; off[5] = o1.y; off[6] = o1.z; off[7] = o1.w;
            }
#pragma unroll
            for (uint32_t kk = 0; kk < 8u; ++kk) {
                packed[kk] = 0u;
                // word sections start on 16-byte boundaries and are padded to them, so the aligned
                // 4 bytes around any word of the run lie inside the packet
                cc[kk] = live ? cc[kk] : 0u;
                if (cc[kk] != 0u && 4u * sub < (off[kk] & 3u) + cc[kk])
                    packed[kk] = reinterpret_cast<const uint32_t *>(a.packets[k0 + (h0 + kk < nk ? h0 + kk : 0u)])[(off[kk] >> 2) + sub];
            }
            if (h0 == 0u) words_on_their_way();
#pragma unroll
            for (uint32_t kk = 0; kk < 8u; ++kk) {
                __builtin_amdgcn_sched_barrier(0);  // one learner at a time: keeps the register count down
                const uint32_t skew = off[kk] & 3u, cck = cc[kk];
                const float sck = s_scale[h0 + kk];
                // The words of this lane: bytes [beg, end) of its four, moved to the front so that
                // slot j is in use in every lane that has more than j words and a slot that no lane
                // of the wave uses costs nothing.  All loads of the accumulators first, then the
                // stores (one learner's words name different elements).
                volatile lds_float *vacc = lds_volatile(acc);
                const uint32_t lo = 4u * sub, end_all = skew + cck;
                const uint32_t beg = skew > lo ? (skew - lo < 4u ? skew - lo : 4u) : 0u;
                const uint32_t end = end_all > lo ? (end_all - lo < 4u ? end_all - lo : 4u) : 0u;
                const uint32_t nw = end > beg ? end - beg : 0u;
                const uint32_t mine = beg < 4u ? packed[kk] >> (8u * beg) : 0u;
                float cur[4];
                uint32_t at_idx[4];
#pragma unroll
                for (uint32_t j = 0; j < 4u; ++j) {
                    at_idx[j] = 0xFFFFFFFFu;  // all ones: no word
                    cur[j] = 0.f;
                    if (__builtin_amdgcn_ballot_w64(j < nw) != 0ull) {
                        const uint32_t wd = (mine >> (8u * j)) & 0xFFu;
                        const uint32_t idx = wd >> 2, code = wd & 3u;
                        const bool on = j < nw && (code & 1u) && idx < span;
                        if (on) { at_idx[j] = idx | (code << 30); cur[j] = vacc[idx]; }  // code 1 or 3 in the top bits
                    }
                }
#pragma unroll
                for (uint32_t j = 0; j < 4u; ++j)
                    if (at_idx[j] != 0xFFFFFFFFu) vacc[at_idx[j] & 0x3FFFFFFFu] = cur[j] + ((at_idx[j] >> 30) == 1u ? sck : -sck);
                if (skew + cck > 16u) {  // the words of this learner beyond the fetched 16 bytes
                    const word_t *wp = reinterpret_cast<const word_t *>(a.packets[k0 + (h0 + kk < nk ? h0 + kk : 0u)]);
                    for (uint32_t q = 16u - skew + sub; q < cck; q += 4u) {
                        const uint32_t wd = wp[off[kk] + q];
                        const uint32_t idx = wd >> 2, code = wd & 3u;
                        if ((code & 1u) && idx < span) lds_add(acc, idx, code == 1u ? sck : -sck);
                    }
                }
            }
        }
        return;
    }
    // lanes per bin: the smallest power of two that holds the largest word count of the tables,
    // between the layer's default (8 or 16) and the whole wave
    uint32_t glog = ut.group_log2();
    while (glog < 6u && (1u << glog) < *s_cmax) ++glog;
    const uint32_t gsz = 1u << glog;

    const uint32_t slots = nb << glog;
    uint32_t word[LG], cmax;   // of the bin and learners in turn: the lane's word, and how many the bin has at most
    auto fetch = [&](const uint32_t s) {
        const uint32_t row = row0 + (!kHook || s < slots ? s >> glog : 0u), sub = s & (gsz - 1u);
        uint32_t cc[LG], off[LG];
#pragma unroll
        for (uint32_t v = 0; v < LG / 8u; ++v) {
            const uint4 t = *reinterpret_cast<const uint4 *>(&s_cnt[row][8u * v]);
            cc[8 * v] = t.x & 0xFFFFu; cc[8 * v + 1] = t.x >> 16; cc[8 * v + 2] = t.y & 0xFFFFu; cc[8 * v + 3] = t.y >> 16;
            cc[8 * v + 4] = t.z & 0xFFFFu; cc[8 * v + 5] = t.z >> 16; cc[8 * v + 6] = t.w & 0xFFFFu; cc[8 * v + 7] = t.w >> 16;
        }
#pragma unroll
        for (uint32_t v = 0; v < LG / 4u; ++v) {
            const uint4 t = *reinterpret_cast<const uint4 *>(&s_off[row][4u * v]);
            off[4 * v] = t.x; off[4 * v + 1] = t.y; off[4 * v + 2] = t.z; off[4 * v + 3] = t.w;
        }
        cmax = 0u;
#pragma unroll
        for (uint32_t kk = 0; kk < LG; ++kk) {
            cmax = cc[kk] > cmax ? cc[kk] : cmax;
            word[kk] = 0u;
            if ((!kHook || s < slots) && sub < cc[kk]) {
                const word_t *wp = reinterpret_cast<const word_t *>(a.packets[k0 + (kk < nk ? kk : 0u)]);
                word[kk] = wp[off[kk] + sub];
            }
        }
    };
    if (kHook) { fetch(tid); words_on_their_way(); }
    for (uint32_t s = tid; s < slots; s += kWG) {
        if (!kHook || s != tid) fetch(s);
        const uint32_t lb = s >> glog, sub = s & (gsz - 1u);
        const uint32_t row = row0 + lb;
        const uint32_t span = T < n - lb * T ? T : n - lb * T;  // elements of this bin held by the tile
        float *acc = s_acc + lb * T;
        if (cmax <= gsz) {
#pragma unroll
            for (uint32_t kk = 0; kk < LG; ++kk) {
                const uint32_t idx = (word[kk] >> 2) - ut.idx_lo;  // wraps to a huge value below idx_lo
                const uint32_t code = word[kk] & 3u;
                if ((code & 1u) && idx < span) { const float sck = s_scale[kk]; atomicAdd(&acc[idx], code == 1u ? sck : -sck); }
            }
        } else {
            // some learner sends more words from this bin than the group has lanes: plain loops,
            // one learner after the other (same order)
            for (uint32_t kk = 0; kk < nk; ++kk) {
                const word_t *wp = reinterpret_cast<const word_t *>(a.packets[k0 + kk]);
                const uint32_t cck = s_cnt[row][kk], st = s_off[row][kk];
                const float sck = s_scale[kk];
                for (uint32_t jw = sub; jw < cck; jw += gsz) {
                    const uint32_t wd = wp[st + jw];
                    const uint32_t idx = (wd >> 2) - ut.idx_lo;
                    const uint32_t code = wd & 3u;
                    if ((code & 1u) && idx < span) atomicAdd(&acc[idx], code == 1u ? sck : -sck);
                }
            }
        }
    }
}

// averageGradients() and updateWeights() of Algorithm 1 on one element of the finished sum: every
// operation is a separate float32 operation (contraction is off), division and square root are
// the correctly rounded ones.
template <int MODE>
__device__ __forceinline__ void apply_update(const UnpackHead &a, float sum, float &w, float &s1, float &s2)
{
    const float g = sum / a.n_average;
    if (MODE == 1) {  // SGD with momentum: v <- mu v + g; w <- w - lr v
        const float mv = a.p1 * s1;
        const float v = mv + g;
        s1 = v;
        const float step = a.lr * v;
        w = w - step;
    } else {          // Adam
        const float m1 = a.p1 * s1, m2 = a.one_minus_p1 * g;
        const float m = m1 + m2;
        const float g2 = g * g;
        const float v1 = a.p2 * s2, v2 = a.one_minus_p2 * g2;
        const float v = v1 + v2;
        s1 = m;
        s2 = v;
        const float m_hat = m / a.bias1;
        const float v_hat = v / a.bias2;
        const float denom = sqrtf(v_hat) + a.eps;
        const float ratio = m_hat / denom;
        const float step = a.lr * ratio;
        w = w - step;
    }
}

// LDS of a group of 16-bit layers inside k_unpack8 (k_unpack has the same arrays of its own: laid out in a
// structure they cost it 2 %)
template <uint32_t LG>
struct UnpackLds {
    __attribute__((aligned(16))) float acc[kUnpackTileElems];
    __attribute__((aligned(16))) uint32_t off[64][kOffStride<LG>];  // first word of (bin, learner), counted from the packet start
    __attribute__((aligned(16))) uint16_t cnt[64][kCntStride];
    __attribute__((aligned(16))) float scale[LG];
    uint32_t cmax;                                              // largest word count of a (bin, learner) in the tables
};

// Clears the accumulators of a tile of n elements, or loads the partial sum of an earlier launch.
__device__ __forceinline__ void unpack_clear(const UnpackHead &a, const uint32_t n, const bool vec, const float *__restrict__ out, float *const s_acc)
{
    const uint32_t tid = threadIdx.x;
    for (uint32_t i = tid * 4u; i < n; i += kWG * 4u) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (a.accumulate) {
            if (vec && i + 4u <= n) v = *reinterpret_cast<const float4 *>(out + i);
            else {
                v.x = out[i];
                v.y = i + 1u < n ? out[i + 1] : 0.f;
                v.z = i + 2u < n ? out[i + 2] : 0.f;
                v.w = i + 3u < n ? out[i + 3] : 0.f;
            }
        }
        *reinterpret_cast<float4 *>(&s_acc[i]) = v;  // s_acc has room for the rounded-up tail
    }
}

// Writes the finished sum of a tile out.
__device__ __forceinline__ void unpack_write_out(const UnpackHead &a, const UTileDev &ut, float *const s_acc)
{
    const uint32_t tid = threadIdx.x;
    const uint32_t n = ut.n_elems;
    float *__restrict__ out = a.dense + ut.elem_base;
    // The write-out moves 16-byte slots of memory whatever the tile's alignment.  A tile that starts
    // `skip` elements past a 16-byte boundary reads its accumulators from the LDS tile at the matching
    // offset (four 4-byte reads per slot instead of one 16-byte read): slot f (a multiple of 4) holds
    // the elements f - skip .. f + 3 - skip; in the first slot that wraps below zero, and `< n` on the
    // wrapped value tells the elements that are the tile's.  (With 4-byte accesses to memory such
    // tiles were written at 3.1 instead of 5 TB/s.)
    const uint32_t skip = uint32_t(ut.elem_base) & 3u;
    for (uint32_t f = tid * 4u; f < n + skip; f += kWG * 4u) {
        const uint32_t e = f - skip;
        float sum[4];
        if (skip == 0u) {
            const float4 v = *reinterpret_cast<const float4 *>(&s_acc[f]);
            sum[0] = v.x; sum[1] = v.y; sum[2] = v.z; sum[3] = v.w;
        } else {
#pragma unroll
            for (uint32_t c = 0; c < 4u; ++c) sum[c] = e + c < n ? s_acc[e + c] : 0.f;
        }
        if (f >= skip && e + 4u <= n) store_stream4(out + e, vfloat4{sum[0], sum[1], sum[2], sum[3]});
        else {
#pragma unroll
            for (uint32_t c = 0; c < 4u; ++c)
                if (e + c < n) out[e + c] = sum[c];
        }
    }
}

// The optimizer's step on a tile: everything that it reads at once, and the step itself.  Bound by HBM; what it loses is the time
// in which a workgroup adds words and nothing of its own is on the way.  So weights and moments are asked for ahead of the adds
// where that pays (unpack_early_for has the line and both sides of it), and behind them all slots together elsewhere.  One slot
// after the other behind the adds (as before) / all together / ahead, in us: SGD, 25 M elements, L_T 500, 8 packets 78.3 / 73.8 / 70.6, 16
// 79.4 / 78.4 / 72.8, L_T 50, 16 108 / 101 / 122; ResNet-50's table, 8 packets 86.3 / - / 79.5; Adam, 16 packets of the 125 M-element table
// 517 / - / 501.
// Slot j of thread t holds the elements 4 (256 j + t) .. + 3 of the tile; buffer accesses need 4-byte alignment and no more, and
// leave alone what lies past the tile's whole slots.  The layer's last elements, which do not fill one, go one by one.
template <int MODE>
struct TileState {
    static constexpr uint32_t kSlots = kUnpackTileElems / (4u * kWG);
    vfloat4 w[kSlots], s1[kSlots], s2[MODE == 2 ? kSlots : 1u];

    // SKIP: not the slots past the tile, whose loads the hardware drops after they have cost their issue.  Behind the adds of up to two
    // packets, where it pays in tiles of few elements and costs nothing in others; elsewhere the branches spill registers.  All slots /
    // without those past the tile, in us, 25 M elements: L_T 14, Adam, 1 packet 125 / 107.8, 2 133.2 / 112.5; L_T 20, 1 104.8 / 100.8, 2 110.9 /
    // 103.9; 12 M, L_T 20, and 13 M, 65, 2 106.2 / 103.7, with the 16-bit tiles' too 104.4; but 3 packets, L_T 18 123.0 / 129.3, k_unpack, SGD, L_T 33, 8
    // packets 82.0 / 98.1.
    template <bool SKIP>
    __device__ __forceinline__ void fetch(const UnpackHead &a, const UTileDev &ut)
    {
        const uint32_t whole = ut.n_elems & ~3u;
        const __amdgpu_buffer_rsrc_t wb = tile_buffer(a.weights + ut.elem_base, whole), b1 = tile_buffer(a.state1 + ut.elem_base, whole);
        const __amdgpu_buffer_rsrc_t b2 = tile_buffer(MODE == 2 ? a.state2 + ut.elem_base : a.weights, MODE == 2 ? whole : 0u);
#pragma unroll
        for (uint32_t j = 0; j < kSlots; ++j) {
            if (SKIP && j * kWG * 4u >= whole) break;
            w[j] = buffer_load_slot(wb, threadIdx.x * 16u, j * kWG * 16u);
            s1[j] = buffer_load_slot(b1, threadIdx.x * 16u, j * kWG * 16u);
            if (MODE == 2) s2[j] = buffer_load_slot(b2, threadIdx.x * 16u, j * kWG * 16u);
        }
    }
    __device__ __forceinline__ void step(const UnpackHead &a, const UTileDev &ut, const float *const s_acc)
    {
        const uint32_t n = ut.n_elems, whole = n & ~3u;
        const __amdgpu_buffer_rsrc_t wb = tile_buffer(a.weights + ut.elem_base, whole), b1 = tile_buffer(a.state1 + ut.elem_base, whole);
        const __amdgpu_buffer_rsrc_t b2 = tile_buffer(MODE == 2 ? a.state2 + ut.elem_base : a.weights, MODE == 2 ? whole : 0u);
        const __amdgpu_buffer_rsrc_t out = tile_buffer(a.write_dense ? a.dense + ut.elem_base : a.weights, a.write_dense ? whole : 0u);
#pragma unroll
        for (uint32_t j = 0; j < kSlots; ++j) {
            const uint32_t e = (j * kWG + threadIdx.x) * 4u;
            if (e >= whole) break;
            const vfloat4 sum = *reinterpret_cast<const vfloat4 *>(&s_acc[e]);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float wc = w[j][c], s1c = s1[j][c], s2c = MODE == 2 ? s2[j][c] : 0.f;
                apply_update<MODE>(a, sum[c], wc, s1c, s2c);
                w[j][c] = wc; s1[j][c] = s1c;
                if (MODE == 2) s2[j][c] = s2c;
            }
            buffer_store_slot(wb, threadIdx.x * 16u, j * kWG * 16u, w[j]);
            buffer_store_slot(b1, threadIdx.x * 16u, j * kWG * 16u, s1[j]);
            if (MODE == 2) buffer_store_slot(b2, threadIdx.x * 16u, j * kWG * 16u, s2[j]);
            if (a.write_dense) buffer_store_slot(out, threadIdx.x * 16u, j * kWG * 16u, sum);
        }
        if (threadIdx.x < (n & 3u)) {
            const uint64_t e = ut.elem_base + whole + threadIdx.x;
            const float sum = s_acc[whole + threadIdx.x];
            float wc = a.weights[e], s1c = a.state1[e], s2c = MODE == 2 ? a.state2[e] : 0.f;
            apply_update<MODE>(a, sum, wc, s1c, s2c);
            a.weights[e] = wc; a.state1[e] = s1c;
            if (MODE == 2) a.state2[e] = s2c;
            if (a.write_dense) a.dense[e] = sum;
        }
    }
};
template <>
struct TileState<0> {
    template <bool SKIP>
    __device__ __forceinline__ void fetch(const UnpackHead &, const UTileDev &) {}
    __device__ __forceinline__ void step(const UnpackHead &a, const UTileDev &ut, float *const s_acc) { unpack_write_out(a, ut, s_acc); }
};

// Packets of a launch whose tables are for LG of them: 16 do for any number, as many at a time.
template <uint32_t LG>
constexpr uint32_t packets_of = LG <= 8u ? LG : kMaxPacketArgs;

// Group number g of the launch, and its first tile.  Group and tile: a round of scalar loads each, 0.25 us, without one for the
// arguments (see k_pack), and what the packets are asked for stands in the tile's record (so far a round more for the layer's, and
// the compiler fetched the arguments where it used them).  The record is kept whole: taken apart, its short fields come through vector loads.
struct GroupAndTile {
    UGroupDev grp;
    UTileDev tile;
};
__device__ __forceinline__ UTileDev utile_record(const UTileDev *p)
{
    vuint8 v = *(const __attribute__((address_space(4))) vuint8 *)p;
    asm volatile("" : "+s"(v));
    return __builtin_bit_cast(UTileDev, v);
}
__device__ __forceinline__ GroupAndTile first_records(const UTileDev *const tiles, const UGroupDev *const groups, const uint32_t n_groups, const uint32_t g)
{
    GroupAndTile r;
    r.grp = groups == nullptr ? UGroupDev{single_tile(g, n_groups), 1u} : table_record<vuint2>(groups + g);
    r.tile = utile_record(tiles + r.grp.first_tile);
    return r;
}

// MODE 0: dense_out <- sum.  MODE 1 / 2: also (or only) the SGD / Adam step on weights and state.
// KIND 0 / 1: all groups of this launch belong to layers with 16-bit / 8-bit words; 2: either (the
// layer says which), one path after a branch; kUnpackSplitTiles has where one launch for both is taken and where one per kind.
// The single-width kernels are held to 80 registers (6 waves per SIMD, what the LDS tile allows).
// EARLY: weights and moments are asked for ahead of the adds and kept through them, in up to 128 registers.
template <int MODE, bool W8, uint32_t LG, bool EARLY, class Args>
__device__ __forceinline__ void unpack_tiles(const Args &a, const UTileDev *const tiles, const UGroupDev grp, const UTileDev ut0, float *const s_acc,
                                             uint32_t (*const s_off)[kOffStride<LG>], uint16_t (*const s_cnt)[kCntStride], float *const s_scale, uint32_t &s_cmax)
{
    // A workgroup serves a group of consecutive tiles that lie in one 64-bin chunk (or are slices
    // of one long bin).  With up to LG learners the tables of phase 1 are built once for the group.
    const uint32_t row0_bin = ut0.first_bin, chunk_end = (row0_bin & ~63u) + ut0.chunk_bins;
    const uint32_t bins = ut0.L_T > kUnpackTileElems ? 1u : ut0.n_bins * grp.n_tiles;   // (the last tile may have fewer)
    const uint32_t scan_end = row0_bin + bins < chunk_end ? row0_bin + bins : chunk_end;
    const bool tables_once = a.n_learners <= LG;

  for (uint32_t ti = 0; ti < grp.n_tiles; ++ti) {
    const UTileDev ut = ti == 0u ? ut0 : utile_record(tiles + grp.first_tile + ti);
    const uint32_t n = ut.n_elems;
    const bool vec = ut.aligned();
    float *__restrict__ out = a.dense + ut.elem_base;

    __syncthreads();  // the previous tile has been written out and its adds are done with the tables
    unpack_clear(a, n, vec, out, s_acc);

    TileState<MODE> state;
    auto round = [&](const uint32_t k0, auto words_on_their_way) {
        if (!tables_once || ti == 0u) {
            if (k0 != 0u) __syncthreads();  // the adds of the previous learners are done with the tables
            unpack_tables<W8, LG>(a, ut0, row0_bin, scan_end, k0, s_off, s_cnt, s_scale, &s_cmax);
        }
        __syncthreads();  // tables filled, accumulators initialised
        unpack_adds<W8, LG>(a, ut, ut.first_bin - row0_bin, k0, s_acc, s_off, s_cnt, s_scale, &s_cmax, words_on_their_way);
    };
    if constexpr (EARLY) {   // the launch has no more packets than the tables
        round(0u, [&] { state.template fetch<false>(a, ut); });
    } else {
        for (uint32_t k0 = 0; k0 < a.n_learners; k0 += LG) round(k0, NoHook());
        state.template fetch<false>(a, ut);
    }
    __syncthreads();

    state.step(a, ut, s_acc);
  }  // tiles of the group
}

template <int MODE, int KIND, uint32_t LG, bool EARLY, class Args>
__device__ __forceinline__ void unpack_group(const Args &a, const UTileDev *const tiles, const GroupAndTile &first, float *const s_acc, uint32_t (*const s_off)[kOffStride<LG>],
                                             uint16_t (*const s_cnt)[kCntStride], float *const s_scale, uint32_t &s_cmax)
{
    const UGroupDev grp = first.grp;
    const UTileDev ut0 = first.tile;
    if (KIND == 1 || (KIND == 2 && ut0.words8())) unpack_tiles<MODE, true, LG, EARLY>(a, tiles, grp, ut0, s_acc, s_off, s_cnt, s_scale, s_cmax);
    else unpack_tiles<MODE, false, LG, EARLY>(a, tiles, grp, ut0, s_acc, s_off, s_cnt, s_scale, s_cmax);
}

// SGD on 8-bit words with 5 to 8 packets, behind the adds: held to 96 scalar registers, with which a SIMD has room for 7 waves, not 6 (25 M
// elements, L_T 20, 5 packets 100.5 us, so 92.5, 8 packets 112.9 / 104.4; L_T 33, 8 packets 82.0 / 77.2).
template <int MODE, int KIND, uint32_t LG, bool EARLY>
__global__ __launch_bounds__(kWG, (MODE == 1 && KIND == 1 && LG == 8u && !EARLY ? 7 : KIND == 2 || (MODE != 0 && EARLY) ? 4 : 6)) void k_unpack(const UTileDev *const tiles, const UGroupDev *const groups, const uint32_t n_groups,
                                                                                                      const UnpackPackets<packets_of<LG>> a)
{
    __shared__ float s_acc[kUnpackTileElems];
    __shared__ __attribute__((aligned(16))) uint32_t s_off[64][kOffStride<LG>];  // first word of (bin, learner), counted from the packet start
    __shared__ __attribute__((aligned(16))) uint16_t s_cnt[64][kCntStride];
    __shared__ __attribute__((aligned(16))) float s_scale[LG];
    __shared__ uint32_t s_cmax;                                                // largest word count of a (bin, learner) in the tables
    unpack_group<MODE, KIND, LG, EARLY>(a, tiles, first_records(tiles, groups, n_groups, blockIdx.x), s_acc, s_off, s_cnt, s_scale, s_cmax);
}

// ==============================================================================================
// k_unpack_few: up to four learners.  Every wave holds what phase 1 of k_unpack puts into tables in LDS in its registers, lane = bin of the
// chunk, and hands it to the lane groups of its bins with lane permutes: no tables, no barrier between the two phases,
// and the headers come through scalar loads, all in flight together.  Bound by memory on large tables, by the chain
// group, tile, layer, counts, words, adds on small ones.  k_unpack / this kernel, in us: 100 k elements, L_T 500, 1
// packet 5.7 / 4.6; 1 M, Adam, 1 packet 10.8 / 8.2; 8 M, 2 packets 12.3 / 8.9; L_T 133, 4 packets 18.6 / 12.5; ResNet-50's
// table, SGD with 1 packet 84 / 72, Adam with 4 128 / 116.  With 5 to 8 learners it loses: what every wave does for
// itself is then most of its work (8 M, 8 packets: 13.0, k_unpack 10.6).
// ==============================================================================================
constexpr uint32_t kFewLearners = 4;
// In the launch of k_unpack8, where they share the LDS and the registers of its chunks, the groups of the 16-bit layers
// take this form for up to two learners (ResNet-50's table, k_unpack's form / this one: 1 packet 20.3 / 20.0 us, 2 22.1 /
// 20.9, but 4 25.2 / 26.7).
constexpr uint32_t kFewInLaunch8 = 2;
template <int MODE, bool W8, bool MANY, uint32_t NK, class Args>
__device__ __forceinline__ void unpack_group_few(const Args &a, const UTileDev *const tiles, const UGroupDev grp, const UTileDev ut0, float *const s_acc)
{
    typedef typename std::conditional<W8, uint8_t, uint16_t>::type word_t;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    constexpr bool EARLY = MODE != 0 && MANY;
    const uint32_t chunk = ut0.first_bin >> 6;
    const bool in_chunk = lane < ut0.chunk_bins;

    // word count and first word (counted from the packet's start) of the lane's bin, for every learner
    uint32_t c[NK], off[NK];
    float scale[NK];
    PacketChunk pc[NK];
#pragma unroll
    for (uint32_t k = 0; k < NK; ++k) {
        const uint8_t *const pk = a.packets[k < a.n_learners ? k : 0u];
        c[k] = reinterpret_cast<const word_t *>(pk + ut0.counts_offset)[in_chunk ? (chunk << 6) + lane : 0u];
        pc[k].fetch(pk, ut0.layer(), ut0.chunks_offset, chunk);
    }
    if constexpr (W8 || !MANY) settle(pc);
    else settle_heads(pc, c);
#pragma unroll
    for (uint32_t k = 0; k < NK; ++k) {
        scale[k] = pc[k].scale;
        const uint32_t ck = ((k < a.n_learners) & pc[k].fits(a) & in_chunk) ? c[k] : 0u;   // a packet that does not match contributes nothing
        // nor does a bin whose words would lie past the packet's total_bytes
        const uint64_t first = pc[k].first_word(uint32_t(sizeof(word_t))) + (wave_incl_scan(ck) - ck);
        c[k] = first + ck <= pc[k].total_bytes.x / uint32_t(sizeof(word_t)) ? ck : 0u;
        off[k] = uint32_t(first);
    }

    for (uint32_t ti = 0; ti < grp.n_tiles; ++ti) {
        const UTileDev ut = ti == 0u ? ut0 : utile_record(tiles + grp.first_tile + ti);
        const uint32_t n = ut.n_elems, T = ut.L_T, nb = ut.n_bins, bin0 = ut.first_bin & 63u;
        if (ti != 0u) __syncthreads();   // the previous tile has been written out
        TileState<MODE> state;
        unpack_clear(a, n, ut.aligned(), a.dense + ut.elem_base, s_acc);
        __syncthreads();
        if (W8) {
            // Four lanes to a bin, lane j fetches the aligned 4 bytes number j of the bin's run of words (what is
            // beyond these 16 bytes comes byte by byte)
            const uint32_t lb = tid >> 2, sub = tid & 3u;
            const uint32_t span = lb < nb ? (T < n - lb * T ? T : n - lb * T) : 0u;   // elements of this bin
            volatile lds_float *const vacc = lds_volatile(s_acc + lb * T);
            uint32_t cc[NK], at[NK], packed[NK];
#pragma unroll
            for (uint32_t k = 0; k < NK; ++k) {
                cc[k] = uint32_t(__shfl(int(c[k]), int(lb), 64));
                at[k] = uint32_t(__shfl(int(off[k]), int(lb), 64));
                packed[k] = 0u;
                // word sections start on 16-byte boundaries and are padded to them, so the aligned
                // 4 bytes around any word of the run lie inside the packet
                if (cc[k] != 0u && 4u * sub < (at[k] & 3u) + cc[k])
                    packed[k] = reinterpret_cast<const uint32_t *>(a.packets[k < a.n_learners ? k : 0u])[(at[k] >> 2) + sub];
            }
            if (EARLY) state.template fetch<false>(a, ut);
#pragma unroll
            for (uint32_t k = 0; k < NK; ++k) {
                if (k >= a.n_learners) break;   // uniform
                __builtin_amdgcn_sched_barrier(0);   // one learner at a time: keeps the register count down
                // The words of this lane: bytes [beg, end) of its four, moved to the front so that slot j is in use in
                // every lane that has more than j words and a slot that no lane of the wave uses costs nothing.  One
                // learner's words name different elements: all loads of the accumulators, then the stores.
                const uint32_t skew = at[k] & 3u, lo = 4u * sub, end_all = skew + cc[k];
                const uint32_t beg = skew > lo ? (skew - lo < 4u ? skew - lo : 4u) : 0u;
                const uint32_t end = end_all > lo ? (end_all - lo < 4u ? end_all - lo : 4u) : 0u;
                const uint32_t nw = end > beg ? end - beg : 0u;
                const uint32_t mine = beg < 4u ? packed[k] >> (8u * beg) : 0u;
                float cur[4];
                bool on[4];
#pragma unroll
                for (uint32_t j = 0; j < 4u; ++j) {
                    on[j] = false;
                    cur[j] = 0.f;
                    if (__builtin_amdgcn_ballot_w64(j < nw) != 0ull) {
                        const uint32_t w = (mine >> (8u * j)) & 0xFFu;
                        on[j] = j < nw && (w & 1u) && (w >> 2) < span;
                        if (on[j]) cur[j] = vacc[w >> 2];
                    }
                }
#pragma unroll
                for (uint32_t j = 0; j < 4u; ++j) {
                    const uint32_t w = (mine >> (8u * j)) & 0xFFu;
                    if (on[j]) vacc[w >> 2] = cur[j] + ((w & 2u) ? -scale[k] : scale[k]);
                }
                if (end_all > 16u) {   // the words of this learner beyond the fetched 16 bytes
                    const uint8_t *const wp = a.packets[k] + at[k];
                    for (uint32_t q = 16u - skew + sub; q < cc[k]; q += 4u) {
                        const uint32_t w = wp[q];
                        if ((w & 1u) && (w >> 2) < span) vacc[w >> 2] = vacc[w >> 2] + ((w & 2u) ? -scale[k] : scale[k]);
                    }
                }
            }
        } else {
        uint32_t most = 0u;   // words of the lane's bin from the learner that sends most
#pragma unroll
        for (uint32_t k = 0; k < NK; ++k) most = c[k] > most ? c[k] : most;
        // lanes per bin: what makes use of all threads, more if a bin of the tile has more words
        uint32_t glog = nb >= 16u ? 4u : nb >= 8u ? 5u : 6u;
        while (glog < 6u && __builtin_amdgcn_ballot_w64(lane >= bin0 && lane < bin0 + nb && most > (1u << glog)) != 0ull) ++glog;
        const uint32_t gsz = 1u << glog, slots = ((nb << glog) + 63u) & ~63u;   // (whole waves: the permutes need all lanes)
        uint32_t cc[NK], word[NK], cmax;
        auto fetch = [&](const uint32_t s) {
            const uint32_t lb = s >> glog, sub = s & (gsz - 1u), from = (bin0 + lb) & 63u;
            cmax = 0u;
#pragma unroll
            for (uint32_t k = 0; k < NK; ++k) {
                cc[k] = uint32_t(__shfl(int(c[k]), int(from), 64));
                const uint32_t at = uint32_t(__shfl(int(off[k]), int(from), 64)) + sub;
                cmax = cc[k] > cmax ? cc[k] : cmax;
                word[k] = 0u;
                if (lb < nb && sub < cc[k]) word[k] = reinterpret_cast<const word_t *>(a.packets[k < a.n_learners ? k : 0u])[at];
            }
        };
        if (EARLY) { fetch(tid); state.template fetch<false>(a, ut); }
        for (uint32_t s = tid; s < slots; s += kWG) {
            if (!EARLY || s != tid) fetch(s);
            const uint32_t lb = s >> glog, sub = s & (gsz - 1u);
            const uint32_t from = (bin0 + lb) & 63u;
            const bool live = lb < nb;
            const uint32_t span = live ? (T < n - lb * T ? T : n - lb * T) : 0u;   // elements of this bin held by the tile
            float *const acc = s_acc + lb * T;
            if (__builtin_amdgcn_ballot_w64(live && cmax > gsz) == 0ull) {
#pragma unroll
                for (uint32_t k = 0; k < NK; ++k) {
                    const uint32_t idx = (word[k] >> 2) - ut.idx_lo;   // wraps to a huge value below idx_lo
                    if ((word[k] & 1u) && idx < span) atomicAdd(&acc[idx], (word[k] & 2u) ? -scale[k] : scale[k]);
                }
            } else {   // a bin with more words than lanes: one learner after the other
#pragma unroll
                for (uint32_t k = 0; k < NK; ++k) {
                    const word_t *const wp = reinterpret_cast<const word_t *>(a.packets[k < a.n_learners ? k : 0u]) + uint32_t(__shfl(int(off[k]), int(from), 64));
                    for (uint32_t q = sub; live && q < cc[k]; q += gsz) {
                        const uint32_t w = wp[q], idx = (w >> 2) - ut.idx_lo;
                        if ((w & 1u) && idx < span) atomicAdd(&acc[idx], (w & 2u) ? -scale[k] : scale[k]);
                    }
                }
            }
        }
        }
        if (!EARLY) state.template fetch<NK == 2u && (W8 || MODE == 1)>(a, ut);
        __syncthreads();
        state.step(a, ut, s_acc);
    }
}

// KIND as in k_unpack.  MANY: for launches of many workgroups.  With the optimizer's step it asks for weights and moments ahead of the adds
// (unpack_early_for); with 16-bit words it does not insist on all packets' records at once, which shortens the chain of a
// workgroup and costs those that queue for the scalar caches.  Insisting / not, in us, 4 packets, L_T 500: 0.4 M elements 4.6 / 4.8, 2 M
// 5.65 / 5.7, 8 M 10.1 / 9.95, 25 M 24.5 / 24.2, 500 and 9000 24.1 / 23.6; 60 M, 64 and 200 in k_unpack8's launch, 1 packet 51.9 /
// 47.1; 8-bit words, 8 M 13.4 / 15.3, 25 M with 500 28.4 / 30.8.
template <int MODE, int KIND, bool MANY, uint32_t NK>
__global__ __launch_bounds__(kWG, MODE != 0 && MANY ? 4 : 6) void k_unpack_few(const UTileDev *const tiles, const UGroupDev *const groups, const uint32_t n_groups,
                                                                             const UnpackPackets<NK> a)
{
    __shared__ __attribute__((aligned(16))) float s_acc[kUnpackTileElems];
    const GroupAndTile first = first_records(tiles, groups, n_groups, blockIdx.x);
    const UGroupDev grp = first.grp;
    const UTileDev ut0 = first.tile;
    if (KIND == 1 || (KIND == 2 && ut0.words8())) unpack_group_few<MODE, true, MANY, NK>(a, tiles, grp, ut0, s_acc);
    else unpack_group_few<MODE, false, MANY, NK>(a, tiles, grp, ut0, s_acc);
}

// ==============================================================================================
// k_unpack8: layers with 8-bit words (L_T <= 64), several words to a bin.  One wave owns a chunk of 64
// bins, a lane owns a bin: it knows the bin's word count for every learner, a wave scan says where the
// words start, and the lane fetches its words, sixteen bytes at a time, and adds them to the chunk's
// accumulators in LDS, learner after learner.  Nothing is shared between waves, so there are no tables
// and no barriers.  What bounded the scheme before this one (four lanes to a bin, 16 word slots each, of
// which four were in use) was the issue of those slots: without the adds the launch took 20 us, with them
// 33 us for 1 packet of ResNet-50's table and 46 for 8; now 15 and 33, and with the 16-bit layer's groups,
// which ride in the same launch (one of their own cost 7 us), 21 and 39, against 38 and 56 for the two
// launches before.  What bounds it now is the LDS: every word is a load and a store at a random bank.  A
// workgroup is up to four such waves: all workgroups of the launch have the LDS of the chunks, and how many
// of those a workgroup takes decides how many 16-bit groups are resident (unpack8_wg_log).
// All adds to one element come from one lane in program order, and the LDS unit executes a wave's
// operations in order: the sum is taken learner 0 first.
// ==============================================================================================
template <int MODE, class Args>
__device__ __forceinline__ void unpack8_chunk(const Args &a, const UTileDev &ut, float *acc_chunk)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t layer = ut.layer();
    // As numbers of 32 bits: from 16 bits the compiler concludes that the loop of the write-out cannot overflow, and takes what does not
    // fill its unrolled body first, one slot after the other (Adam, 25 M elements, L_T 12, 8 packets 150.7 us, so 143.5).
    uint32_t n = ut.n_elems, T = ut.L_T, nb = ut.n_bins;
    asm volatile("" : "+s"(n), "+s"(T), "+s"(nb));
    float *const out = a.dense + ut.elem_base;
    const uint32_t chunk = ut.first_bin >> 6;

    for (uint32_t e = lane * 4u; e < n; e += 256u) {   // zero, or the partial sum of an earlier launch
        vfloat4 v = {0.f, 0.f, 0.f, 0.f};
        if (a.accumulate)
            for (uint32_t k = 0; k < 4u && e + k < n; ++k) v[k] = out[e + k];
        *reinterpret_cast<vfloat4 *>(&acc_chunk[e]) = v;   // the chunk's LDS has room for the rounded-up tail
    }
    volatile lds_float *const acc = lds_volatile(acc_chunk + lane * T);
    const uint32_t span = lane < nb ? (T < n - lane * T ? T : n - lane * T) : 0u;   // elements of this lane's bin

    constexpr uint32_t kBatch = 8;   // learners whose counts and words are in flight together
    for (uint32_t h0 = 0; h0 < a.n_learners; h0 += kBatch) {
        const uint32_t nk = a.n_learners - h0 < kBatch ? a.n_learners - h0 : kBatch;
        uint32_t c[kBatch], off[kBatch], got[kBatch][4];   // got: the 16 bytes from the aligned 4 that hold the first word on
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            c[k] = 0u;
            if (k < nk && lane < nb) c[k] = (a.packets[h0 + k] + ut.counts_offset)[ut.first_bin + lane];
        }
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            off[k] = got[k][0] = got[k][1] = got[k][2] = got[k][3] = 0u;
            if (k >= nk) continue;   // uniform
            const uint8_t *const pk = a.packets[h0 + k];
            const vuint4 hv = packet_field<vuint4>(pk);        // magic, version, status, n_layers
            const vuint2 tb = packet_field<vuint2>(pk + 16);   // total_bytes
            const bool ok = (hv.x == ADACOMP_PACKET_MAGIC) & (hv.y == ADACOMP_PACKET_VERSION) & (hv.z == ADACOMP_STATUS_COMPLETE) &
                            (hv.w == a.n_layers) & (tb.y == 0u);
            const uint8_t *const rec = pk + sizeof(adacomp_packet_header_t) + sizeof(adacomp_packet_layer_t) * layer;
            const uint32_t words = packet_field<uint32_t>(rec + offsetof(adacomp_packet_layer_t, words_offset));   // packets stay below 2^32 bytes (host check)
            const uint32_t before = packet_field<uint32_t>(pk + ut.chunks_offset + 4u * chunk);
            const uint32_t ck = ok ? c[k] : 0u;   // a packet that does not match contributes nothing
            // a bin whose words would lie past the packet's total_bytes contributes nothing either
            const uint64_t first = uint64_t(words) + before + (wave_incl_scan(ck) - ck);
            const bool inside = first + ck <= tb.x;
            c[k] = inside ? ck : 0u;
            off[k] = uint32_t(first);
            if (c[k] != 0u) {
                // word sections start on 16-byte boundaries and are padded to them, so the aligned 4 bytes
                // around any word of the run lie inside the packet
                const uint32_t *const src = reinterpret_cast<const uint32_t *>(pk) + (off[k] >> 2);
                const uint32_t end = (off[k] & 3u) + c[k];
#pragma unroll
                for (uint32_t i = 0; i < 4u; ++i)
                    if (end > 4u * i) got[k][i] = src[i];
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            if (k >= nk) break;   // uniform
            __builtin_amdgcn_sched_barrier(0);   // one learner at a time: keeps the register count down
            const uint8_t *const pk = a.packets[h0 + k];
            const float scale = packet_field<float>(pk + sizeof(adacomp_packet_header_t) + sizeof(adacomp_packet_layer_t) * layer + offsetof(adacomp_packet_layer_t, scale));
            const uint32_t skew = off[k] & 3u;
#pragma unroll
            for (uint32_t i = 0; i < 4u; ++i) {
                // words 4 i .. 4 i + 3 of the run, as far as they have been fetched
                const uint32_t left = c[k] > 4u * i ? c[k] - 4u * i : 0u;
                const uint32_t here = i < 3u ? left : left < 4u - skew ? left : 4u - skew;
                if (__builtin_amdgcn_ballot_w64(here != 0u) == 0ull) break;
                const uint32_t word = __builtin_amdgcn_alignbyte(i < 3u ? got[k][i < 3u ? i + 1u : 3u] : 0u, got[k][i], skew);
                // one learner's words name different elements: all loads of the accumulators, then the stores
                float cur[4];
                bool on[4];
#pragma unroll
                for (uint32_t j = 0; j < 4u; ++j) {
                    const uint32_t w = (word >> (8u * j)) & 0xFFu;
                    on[j] = j < here && (w & 1u) != 0u && (w >> 2) < span;
                    cur[j] = 0.f;
                    if (on[j]) cur[j] = acc[w >> 2];
                }
#pragma unroll
                for (uint32_t j = 0; j < 4u; ++j) {
                    const uint32_t w = (word >> (8u * j)) & 0xFFu;
                    if (on[j]) acc[w >> 2] = cur[j] + ((w & 2u) ? -scale : scale);
                }
            }
            for (uint32_t q = 16u - skew; q < c[k]; ++q) {   // bins that send more than that
                const uint32_t w = pk[off[k] + q];
                if ((w & 1u) && (w >> 2) < span) acc[w >> 2] = acc[w >> 2] + ((w & 2u) ? -scale : scale);
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");

    const __amdgpu_buffer_rsrc_t w_buf = tile_buffer(MODE != 0 ? a.weights + ut.elem_base : out, MODE != 0 ? n : 0u);
    const __amdgpu_buffer_rsrc_t s1_buf = tile_buffer(MODE != 0 ? a.state1 + ut.elem_base : out, MODE != 0 ? n : 0u);
    const __amdgpu_buffer_rsrc_t s2_buf = tile_buffer(MODE == 2 ? a.state2 + ut.elem_base : out, MODE == 2 ? n : 0u);
#pragma unroll 4
    for (uint32_t e = lane * 4u; e < (n & ~3u); e += 256u) {
        const vfloat4 sum = *reinterpret_cast<const vfloat4 *>(&acc_chunk[e]);
        if (a.write_dense) store_stream4(out + e, sum);
        if (MODE != 0) {
            vfloat4 w = buffer_load_stream4(w_buf, e), s1 = buffer_load_stream4(s1_buf, e), s2 = {0.f, 0.f, 0.f, 0.f};
            if (MODE == 2) s2 = buffer_load_stream4(s2_buf, e);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float wk = w[k], s1k = s1[k], s2k = s2[k];
                apply_update<MODE>(a, sum[k], wk, s1k, s2k);
                w[k] = wk; s1[k] = s1k; s2[k] = s2k;
            }
            buffer_store_stream4(w_buf, e, w);
            buffer_store_stream4(s1_buf, e, s1);
            if (MODE == 2) buffer_store_stream4(s2_buf, e, s2);
        }
    }
    if (lane < (n & 3u)) {   // the layer's last elements
        const uint32_t e = (n & ~3u) + lane;
        const float sum = acc_chunk[e];
        if (a.write_dense) out[e] = sum;
        if (MODE != 0) {
            float w = buffer_load1(w_buf, e), s1 = buffer_load1(s1_buf, e), s2 = 0.f;
            if (MODE == 2) s2 = buffer_load1(s2_buf, e);
            apply_update<MODE>(a, sum, w, s1, s2);
            buffer_store1(w_buf, e, w);
            buffer_store1(s1_buf, e, s1);
            if (MODE == 2) buffer_store1(s2_buf, e, s2);
        }
    }
}

// The first n_groups workgroups take a group of the 16-bit layers each, the others up to four chunks of the
// 8-bit ones.  Dynamic LDS: launch_unpack.  LG: 4 (k_unpack_few), 8 or 16 learners to a group of the former.
// With 3 to 8 packets and the optimizer's step, and with more than 8, it is held to 72 vector registers and 96 scalar ones, with which 7 workgroups are resident: from 97
// scalar ones on a SIMD has room for 6 waves only, from 73 vector ones too.  In us, 106 scalar registers and, Adam, 81 vector ones /
// as it is: 25 M elements, L_T 12, SGD, 8 packets 104.9 / 98.5, Adam 150.7 / 130.4; L_T 16 103.3 / 93.0, 142.3 / 128.5; 30 M, L_T 8, and 30 M, 500
// 213.8 / 202.9, 316.5 / 280.9; 6 M, L_T 8, SGD, 4 25.3 / 22.8; 54 M with 4 M at L_T 16 153.1 / 153.7, 227.7 / 229.2; at the worst 4 M, L_T 16, and
// 4 M, 500, SGD, 4 26.9 / 28.7, where the last workgroups fall into a round of their own.  Sums: 25 M, L_T 8, 16 packets 181.4 / 170.4, 9 110.9 / 104.5;
// 60 M, L_T 16, 24 340.0 / 321.7; 12 M, L_T 16, and 12 M, 500, 16 70.3 / 70.3.
template <int MODE, uint32_t LG>
__global__ __launch_bounds__(kWG, (MODE != 0 && LG == 8u) || LG == 16u ? 7 : 4) void k_unpack8(const UTileDev *const tiles, const UGroupDev *const groups, const uint32_t n_groups,
                                                   const UnpackPackets<(LG == kFewLearners ? kFewInLaunch8 : packets_of<LG>)> a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t s_dyn[];
    if (blockIdx.x < n_groups) {
        if constexpr (LG == kFewLearners) {
            const GroupAndTile first = first_records(tiles, groups, 0u, a.first16 + blockIdx.x);
            unpack_group_few<MODE, false, MODE == 0, kFewInLaunch8>(a, tiles, first.grp, first.tile, reinterpret_cast<float *>(s_dyn));
        } else {
            UnpackLds<LG> &lds = *reinterpret_cast<UnpackLds<LG> *>(s_dyn);
            unpack_group<MODE, 0, LG, false>(a, tiles, first_records(tiles, groups, 0u, a.first16 + blockIdx.x), lds.acc, lds.off, lds.cnt, lds.scale, lds.cmax);
        }
        return;
    }
    uint32_t r = blockIdx.x - n_groups;
    const uint32_t wg_log = a.chunk_lds & 63u, wg_chunks = 1u << wg_log;
    const uint32_t n_runs = (a.n_groups8 + wg_chunks - 1u) >> wg_log;
    if (r < (n_runs & ~63u)) r = (r & ~63u) | ((r & 7u) << 3) | ((r >> 3) & 7u);   // neighbouring chunks share an XCD's L2
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t chunk = (r << wg_log) + wave;
    if (wave < wg_chunks && chunk < a.n_groups8) unpack8_chunk<MODE>(a, first_records(tiles, groups, 0u, chunk).tile, reinterpret_cast<float *>(s_dyn) + wave * (a.chunk_lds & ~63u));
}

// ==============================================================================================
// k_copy: plain float4 copy, the calibration kernel for byte counters and copy bandwidth.
// ==============================================================================================
__global__ __launch_bounds__(kWG) void k_copy(float *__restrict__ dst, const float *__restrict__ src, size_t n)
{
    const size_t n4 = n / 4;
    const size_t stride = size_t(gridDim.x) * kWG;
    for (size_t i = size_t(blockIdx.x) * kWG + threadIdx.x; i < n4; i += stride)
        reinterpret_cast<float4 *>(dst)[i] = reinterpret_cast<const float4 *>(src)[i];
    if (blockIdx.x == 0 && threadIdx.x < n % 4) dst[n4 * 4 + threadIdx.x] = src[n4 * 4 + threadIdx.x];
}

// ==============================================================================================
// k_triad, k_fill: the two streaming ceilings the hot kernels are measured against, with the access
// pattern of k_fused and nothing else.  k_triad: x <- x + y in place, 12 bytes per element (read,
// read, write) in tiles of 4096 elements, 16 per thread, streaming loads and stores, the same
// transposed tile order inside every 64 workgroups.  k_fill: 4 bytes per element written.
// ==============================================================================================
__global__ __launch_bounds__(kWG) void k_triad(float *__restrict__ x, const float *__restrict__ y, uint32_t n_tiles, size_t n)
{
    uint32_t tile = blockIdx.x;
    if (tile < (n_tiles & ~63u)) tile = (tile & ~63u) | ((tile & 7u) << 3) | ((tile >> 3) & 7u);
    const size_t base = size_t(tile) * 4096u;
    if (base + 4096u <= n) {   // a whole tile: eight loads in flight per thread, no branch between them
        vfloat4 a[4], b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const size_t e = base + (uint32_t(j) * kWG + threadIdx.x) * 4u;
            a[j] = load_stream4(x + e);
            b[j] = load_stream4(y + e);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const size_t e = base + (uint32_t(j) * kWG + threadIdx.x) * 4u;
            store_stream4(x + e, a[j] + b[j]);
        }
        return;
    }
    for (int j = 0; j < 4; ++j) {   // the ragged last tile
        const size_t e = base + (uint32_t(j) * kWG + threadIdx.x) * 4u;
        if (e + 4u <= n) store_stream4(x + e, load_stream4(x + e) + load_stream4(y + e));
    }
}

__global__ __launch_bounds__(kWG) void k_fill(float *__restrict__ x, float value, size_t n)
{
    const size_t base = size_t(blockIdx.x) * 4096u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const size_t e = base + (uint32_t(j) * kWG + threadIdx.x) * 4u;
        if (e + 4u <= n) store_stream4(x + e, vfloat4{value, value, value, value});
    }
}

// ---- launchers ---------------------------------------------------------------------------------
static int check_launch() { return hipGetLastError() == hipSuccess ? ADACOMP_OK : ADACOMP_EHIP; }

// a.fused_idle_lds: dynamic LDS that no kernel touches, asked for with the launches of the eager
// 256-thread kernel (the host decides when, adacomp_plan.h says why).
int launch_fused(const CompressArgs &a, int jcode, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    // tiles of the smaller class (up to 4096 elements): 256 threads; of the larger (up to 16384: layers with a bin longer
    // than 4096, and all layers beside those in tables that can go in one launch, of whatever bins): 1024 threads.  Either
    // way a thread holds 16 elements, and a compute unit holds 32 waves of them.  (With 256 threads
    // and 64 elements each the long-bin tiles had two workgroups per compute unit and streamed at
    // 51-55 % of the HBM peak instead of 75-80 %.)
    const dim3 wg(jcode == 0 ? 256 : 1024);
    const bool variant = a.rule != ADACOMP_RULE_ADACOMP || a.soft_factor_minus_1 != 1.0f;
    if (a.one_launch) {   // the host picks it for tables of one tile class whose layers are small
        const bool lazy = a.place_mode == kPlaceWords;
        if (a.class_tiles || a.place_mode == kPlaceResidue || (a.lazy && !lazy) || (lazy && variant)) return ADACOMP_EINVAL;
        const bool table = a.one_launch == kOneLaunchTable;
        if (table && (a.n_tiles > kFoldTiles || a.n_layers > kFoldLayers)) return ADACOMP_EINVAL;
        const dim3 grid(a.class_count + 1u, a.fused_count);   // a learner's tiles and the workgroup that writes the header
        auto method = [&](auto waves, auto slots, auto form) {
            constexpr int W = decltype(waves)::value, J = decltype(slots)::value, F = decltype(form)::value;
            auto go = [&](auto variant_, auto lazy_) {
                constexpr bool V = decltype(variant_)::value, L = decltype(lazy_)::value;
                if constexpr (F == kOneTable)
                    hipLaunchKernelGGL((k_pack<V, F, W, J, L, const TileDev *, uint8_t *, uint32_t, uint32_t, uint32_t, uint32_t>),
                                       grid, dim3(W * 64), 0, s, a.tiles, a.sync, uint32_t(a.sync_stride), a.o_sync_epoch, a.class_count, a.fused_first, a);
                else hipLaunchKernelGGL((k_pack<V, F, W, J, L>), grid, dim3(W * 64), 0, s, a);
            };
            const std::integral_constant<bool, true> yes;
            const std::integral_constant<bool, false> no;
            if (lazy) go(no, yes);
            else if (variant) go(yes, no);
            else go(no, no);
        };
        const std::integral_constant<int, 4> four;
        const std::integral_constant<int, kOneTable> all_records;
        const std::integral_constant<int, kOneLayers> per_layer;
        if (jcode != 0) table ? method(std::integral_constant<int, 16>(), four, all_records) : method(std::integral_constant<int, 16>(), four, per_layer);
        else if (!table) method(four, four, per_layer);
        else if (a.pack_wide) method(std::integral_constant<int, 8>(), std::integral_constant<int, 2>(), all_records);
        else method(four, four, all_records);
        return check_launch();
    }
    const dim3 grid(a.class_count * a.fused_count);
    if (a.lazy) {  // the host offers lazy residues for the default method only
        if (jcode == 0) hipLaunchKernelGGL((k_fused<4, 4, false, true>), grid, wg, 0, s, a);
        else hipLaunchKernelGGL((k_fused<4, 16, false, true>), grid, wg, 0, s, a);
    } else if (!variant) {
        if (jcode == 0) hipLaunchKernelGGL((k_fused<4, 4, false, false>), grid, wg, a.fused_idle_lds, s, a);
        else if (a.shift) hipLaunchKernelGGL((k_fused<4, 16, false, false, true>), grid, wg, 0, s, a);
        else hipLaunchKernelGGL((k_fused<4, 16, false, false>), grid, wg, 0, s, a);
    } else {
        if (jcode == 0) hipLaunchKernelGGL((k_fused<4, 4, true, false>), grid, wg, a.fused_idle_lds, s, a);
        else if (a.shift) hipLaunchKernelGGL((k_fused<4, 16, true, false, true>), grid, wg, 0, s, a);
        else hipLaunchKernelGGL((k_fused<4, 16, true, false>), grid, wg, 0, s, a);
    }
    return check_launch();
}

int launch_scan(const CompressArgs &a, void *stream)
{
    hipLaunchKernelGGL(k_scan, dim3(a.n_layers, a.n_learners), dim3(kScanWG), 0, static_cast<hipStream_t>(stream), a);
    return check_launch();
}

int launch_place(const CompressArgs &a, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    const dim3 wg(kWG);
    if (a.place_tiled) {
        if (a.fold_scan || a.place_mode != kPlaceEager) return ADACOMP_EINVAL;  // the host picks it for eager calls after a k_scan launch only
        hipLaunchKernelGGL(k_place_tiled, dim3(a.n_tiles + 1u, a.n_learners), wg, 0, s, a);
        return check_launch();
    }
    if (a.fold_scan && (a.place_lanes != 64u || a.place_mode == kPlaceResidue || a.n_tiles > kFoldTiles || a.n_layers > kFoldLayers))
        return ADACOMP_EINVAL;  // the host picks the folded scan only where the kernel is built for it
    if (a.place_lanes == 64u) {
        const dim3 grid((a.n_tiles + 3u) / 4u + 1u, a.n_learners);
        if (a.fold_scan) {
            if (a.place_mode == kPlaceWords) hipLaunchKernelGGL((k_place<64, kPlaceWords, true>), grid, wg, 0, s, a);
            else hipLaunchKernelGGL((k_place<64, kPlaceEager, true>), grid, wg, 0, s, a);
        } else if (a.place_mode == kPlaceWords) hipLaunchKernelGGL((k_place<64, kPlaceWords, false>), grid, wg, 0, s, a);
        else if (a.place_mode == kPlaceResidue) hipLaunchKernelGGL((k_place<64, kPlaceResidue, false>), grid, wg, 0, s, a);
        else hipLaunchKernelGGL((k_place<64, kPlaceEager, false>), grid, wg, 0, s, a);
    } else {
        const dim3 grid((a.n_tiles + 15u) / 16u + 1u, a.n_learners);
        if (a.place_mode == kPlaceWords) hipLaunchKernelGGL((k_place<16, kPlaceWords, false>), grid, wg, 0, s, a);
        else if (a.place_mode == kPlaceResidue) hipLaunchKernelGGL((k_place<16, kPlaceResidue, false>), grid, wg, 0, s, a);
        else hipLaunchKernelGGL((k_place<16, kPlaceEager, false>), grid, wg, 0, s, a);
    }
    return check_launch();
}

template <class K>
struct KernelArgs;
template <class A>
struct KernelArgs<void (*)(const UTileDev *, const UGroupDev *, uint32_t, A)> {
    using type = typename std::remove_const<A>::type;
};
// resident: workgroups per compute unit that the launch is held to (5 or 4), or 0.  early: unpack_early_for.
int launch_unpack(const UnpackArgs &a, int kind, uint32_t resident, bool early, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (a.n_groups == 0 && kind != 3) return ADACOMP_OK;
    if (early && (a.mode == 0u || kind == 3 || a.n_learners == 0u || a.n_learners > (kind == 0 ? 16u : 8u))) return ADACOMP_EINVAL;   // the host asks for it where there is a kernel
    const dim3 grid(a.n_groups), wg(kWG);
    uint32_t lds = 0;
    auto launch = [&](const dim3 &workgroups, auto kernel) {
        typename KernelArgs<decltype(kernel)>::type args;
        static_cast<UnpackHead &>(args) = a;
        std::copy_n(a.packets, sizeof(args.packets) / sizeof(args.packets[0]), args.packets);
        hipLaunchKernelGGL(kernel, workgroups, wg, lds, s, a.tiles, a.groups, a.n_groups, args);
    };
    auto with_mode = [&](auto &&go) {
        if (a.mode == 1) go(std::integral_constant<int, 1>());
        else if (a.mode == 2) go(std::integral_constant<int, 2>());
        else go(std::integral_constant<int, 0>());
    };
    const bool few = a.n_learners != 0u && a.n_learners <= kFewLearners, eight = a.n_learners <= 8u;
    // what a workgroup of these kernels has (kind 3: for a group of the 16-bit layers)
    const uint32_t arrays = few ? 4u * kUnpackTileElems : uint32_t(eight ? sizeof(UnpackLds<8>) : sizeof(UnpackLds<16>));
    if (resident != 0u && arrays < kResidentLds[resident == 4u]) lds = kResidentLds[resident == 4u] - arrays;   // LDS that no kernel touches
    if (kind == 3) {
        const uint32_t wg_log = a.chunk_lds & 63u, chunk_elems = a.chunk_lds & ~63u;
        if (a.n_groups8 == 0 || chunk_elems == 0 || chunk_elems > 64u * 64u || wg_log > 2u || (a.mode != 0u && !eight)) return ADACOMP_EINVAL;
        const dim3 both(a.n_groups + ((a.n_groups8 + (1u << wg_log) - 1u) >> wg_log));
        const bool two = a.n_learners != 0u && a.n_learners <= kFewInLaunch8;
        const uint32_t groups = a.n_groups == 0u ? 0u : two ? 4u * kUnpackTileElems : uint32_t(eight ? sizeof(UnpackLds<8>) : sizeof(UnpackLds<16>));
        lds = std::max(groups, 4u * chunk_elems << wg_log);
        with_mode([&](auto mode) {
            constexpr int M = decltype(mode)::value;
            if (two) launch(both, k_unpack8<M, kFewLearners>);
            else if (eight) launch(both, k_unpack8<M, 8>);
            else if constexpr (M == 0) launch(both, k_unpack8<M, 16>);
        });
        return check_launch();
    }
    with_mode([&](auto mode) {
        constexpr int M = decltype(mode)::value;
        auto width = [&](auto k0, auto k1, auto k2) {
            if (kind == 0) launch(grid, k0);
            else if (kind == 1) launch(grid, k1);
            else launch(grid, k2);
        };
        auto kernels = [&](auto how) {
            constexpr bool B = decltype(how)::value, E = M != 0 && B;
            if (few && a.n_learners <= 2u) width(k_unpack_few<M, 0, B, 2>, k_unpack_few<M, 1, E, 2>, k_unpack_few<M, 2, B, 2>);
            else if (few) width(k_unpack_few<M, 0, B, 4>, k_unpack_few<M, 1, E, 4>, k_unpack_few<M, 2, B, 4>);
            else if (eight) width(k_unpack<M, 0, 8, E>, k_unpack<M, 1, 8, E>, k_unpack<M, 2, 8, E>);
            else if constexpr (E) launch(grid, k_unpack<M, 0, 16, E>);
            else width(k_unpack<M, 0, 16, E>, k_unpack<M, 1, 16, E>, k_unpack<M, 2, 16, E>);
        };
        if (M != 0 ? early : a.n_groups > kFewTilesTogether) kernels(std::integral_constant<bool, true>());
        else kernels(std::integral_constant<bool, false>());
    });
    return check_launch();
}

int launch_triad(float *x, const float *y, size_t n, uint32_t resident, void *stream)
{
    const uint32_t n_tiles = uint32_t((n + 4095u) / 4096u);
    // fewer than 8 workgroups per compute unit: each asks for dynamic LDS it never touches, sized so that
    // `resident` of them fit the 160 KB of a compute unit and one more does not
    const uint32_t idle_lds = resident >= 8u ? 0u : 163840u / resident - 1024u;
    hipLaunchKernelGGL(k_triad, dim3(n_tiles), dim3(kWG), idle_lds, static_cast<hipStream_t>(stream), x, y, n_tiles, n);
    return check_launch();
}

int launch_fill(float *x, float value, size_t n, void *stream)
{
    hipLaunchKernelGGL(k_fill, dim3(uint32_t((n + 4095u) / 4096u)), dim3(kWG), 0, static_cast<hipStream_t>(stream), x, value, n);
    return check_launch();
}

int launch_copy(float *dst, const float *src, size_t n, void *stream)
{
    const size_t n4 = n / 4;
    size_t blocks = (n4 + kWG - 1) / kWG;
    if (blocks > 256u * 32u) blocks = 256u * 32u;
    if (blocks == 0) blocks = 1;
    hipLaunchKernelGGL(k_copy, dim3(uint32_t(blocks)), dim3(kWG), 0, static_cast<hipStream_t>(stream), dst, src, n);
    return check_launch();
}

}  // namespace adacomp
