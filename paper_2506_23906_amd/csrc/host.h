// libmmvseg, part of the one translation unit mmvseg.hip (included there, in order).
// Host side: argument checks, workspace layouts, tile plans and the launch sequences behind the C ABI.
#pragma once

namespace {

// ---- host side -------------------------------------------------------------------------------------------------

inline size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }
// Tile plan.  A tile costs one ticket (about 11 ns, serialised), so tiles are as large as the registers
// allow: kMaxCpw chunks of 2048 elements per wave.  Inputs that fit into one round of resident workgroups
// get equal tiles of just the size that gives every workgroup one.  A longer vector starts with groups of
// tiles of 1, 2, ... chunks per wave and ends with groups of ..., 2, 1: started together on full tiles, the
// workgroups of the first round all load, then all compute, then all store (nothing overlaps for a whole
// tile time), and those of the last round would leave most of the chip idle while the last ones finish.
// (Measured on the int8 scan: the time of a launch is a fixed 22 us plus 0.216 ms per 2^28 elements with
// full tiles throughout and one group of short tiles at the end.)
constexpr uint64_t kComputeUnits = 256;   // of an MI355X (not asked from the device: the sizes of workspaces depend on the plans)
constexpr uint64_t kResident = MMV_MIN_TILES;   // workgroups resident at once (2 per compute unit)
#ifndef MMV_HEAD_GROUP
#define MMV_HEAD_GROUP 128   // tiles per length at the start of a long vector (0: full tiles from the start)
#endif
#ifndef MMV_TAIL_GROUP
#define MMV_TAIL_GROUP 64    // tiles per length (2 chunks per wave and more) at the end of a long vector
#endif
#ifndef MMV_TAIL_TILES
#define MMV_TAIL_TILES 128   // tiles of one chunk per wave at the very end (the last of them is ragged)
#endif
// Up to this many tiles the segmented sum and CSR SpMV need no prefix kernel: every wave of the main
// kernel adds up the counts of the tiles before its own, sixteen 128-bit loads per lane at most, four of them under way at a
// time (one load per lane and 64 tiles, waited for one by one, took 5.6 us of a 42 us kernel at 1224 tiles; the prefix
// kernel takes 5 to 6 us of the call).
constexpr uint64_t kCountTiles = 4096;
inline bool is_spmv(mmv_op op) { return op == MMV_OP_SPMV_COO || op == MMV_OP_SPMV_CSR; }
// Most chunks per wave of the tile body that carries its pair from row to row (seg_tile): what the kernel
// instantiation for this operation, type and variant is built with (sums of fp32 values and SpMV have another body).
template <typename TT> inline int row_form_cpw_of(mmv_op op, bool mfma) {
    switch (op) {
        case MMV_OP_SCAN: return mfma ? chunks_per_wave<TT, kPlainScan, true>() : chunks_per_wave<TT, kPlainScan, false>();
        case MMV_OP_SEGSUM: return mfma ? chunks_per_wave<TT, kSum, true>() : chunks_per_wave<TT, kSum, false>();
        default: return mfma ? chunks_per_wave<TT, kScan, true>() : chunks_per_wave<TT, kScan, false>();
    }
}
inline int row_form_cpw(mmv_op op, mmv_dtype dt, bool mfma) {
    switch (dt) {
        case MMV_F32_F32: return op == MMV_OP_SCAN ? lane_cpw<TF32, kPlainScan>() : lane_cpw<TF32, kScan>();   // (lane_tile)
        case MMV_F16_F32: return row_form_cpw_of<TF16>(op, mfma);
        case MMV_BF16_F32: return row_form_cpw_of<TBF16>(op, mfma);
        case MMV_I8_I32: return row_form_cpw_of<TI8>(op, mfma);
        case MMV_U8_XOR: return row_form_cpw_of<TX8>(op, mfma);
        default: break;
    }
    return 1;
}
// Most chunks per wave of the segmented sum that speculates over whole chunks and streams through its spans
// (sum_tile; 0: this operation, type or variant has no such form).
inline int chunk_form_cpw(mmv_op op, mmv_dtype dt, bool mfma) {
    (void)mfma;   // both variants have it
    if (op != MMV_OP_SEGSUM) return 0;
    if (dt == MMV_I8_I32 && chunk_sum_kernel<TI8, kSum, true>()) return sum_cpw<TI8>();
    if (dt == MMV_U8_XOR && chunk_sum_kernel<TX8, kSum, true>()) return sum_cpw<TX8>();
    if (dt == MMV_F16_F32 && chunk_sum_kernel<TF16, kSum, true>()) return sum_cpw<TF16>();
    if (dt == MMV_BF16_F32 && chunk_sum_kernel<TBF16, kSum, true>()) return sum_cpw<TBF16>();
    return 0;
}
// Whether the segmented sum of this type needs its counts of segment starts per wave span too (sum_kernel, whose waves take
// a span of the tile each).  The waves of stream_kernel count inside their tile from its flag words; with a table per span
// beside the one per tile, csr_flags_kernel did its atomic adds twice, and the reset cleared eight times the words (CSR product
// in one step, 3.5 M entries in blocks of 16: 22.2 us before there was one, 24.3 with it, 21.4 without it again).
inline bool segsum_spans(mmv_dtype dt) { return dt != MMV_F32_F32; }
inline int waves_of(mmv_dtype dt) {   // (SpMV has a tile plan of its own)
    switch (dt) {
        case MMV_F32_F32: return TF32::kWaves;
        case MMV_F16_F32: return TF16::kWaves;
        case MMV_BF16_F32: return TBF16::kWaves;
        case MMV_I8_I32: return TI8::kWaves;
        case MMV_U8_XOR: return TX8::kWaves;
        default: break;
    }
    return 1;
}
// Scans of bytes and, in the variant without the matrix cores, of 16-bit values have a form with three workgroups per compute
// unit (OneRound) for vectors whose tiles are all resident at once: more waves hide one another's latencies, and a vector
// of up to 768 chunks per wave no longer needs tiles of two.  Whole calls, two workgroups -> three (us; lengths up to 512 / one
// segment): bytes 5 * 10^6 11.6 / 13.4 -> 10.5 / 12.8, 12 * 10^6 17.1 / 19.0 -> 14.5 / 18.6, 20 * 10^6 24.0 / 26.0 -> 20.1 / 23.9,
// mmv_scan 25.4 -> 23.6; fp16 20 * 10^6 28.2 / 30.3 -> 22.9 / 25.7, 25 * 10^6 30.8 / 34.7 -> 27.4 / 29.4.
// Longer vectors: three workgroups take 5 % more than two (the memory is short of neither, and more tiles are being read and
// written at a time: bytes 2^26 62.2 -> 65.3, 2^28 235 -> 245).  16-bit values: up to 1024 chunks per wave two workgroups are level
// (12 * 10^6 17.0 / 18.5 -> 15.3 / 19.2, 14 * 10^6 18.5 / 20.6 -> 18.5 / 21.6).  On the matrix cores the form spills 20 registers and is
// 20 % slower; segmented scans of that variant take the form in lanes there (lane_kernel.h), whose error is smaller than that of either
// row scan (fp16, lengths up to 512 1.7e-8 against 2.1e-8, one segment 2.5e-8 against 2e-7): 17 * 10^6 26.0 / 29.7 -> 22.8 / 25.1,
// 20 * 10^6 28.5 / 31.4 -> 24.8 / 27.1, 25 * 10^6 31.6 / 35.0 -> 30.2 / 31.3; bf16 25.8 / 29.3 -> 22.0 / 25.1, 27.6 / 31.6 -> 24.7 / 26.6,
// 30.7 / 35.0 -> 29.5 / 31.1.  Not outside this range: 8 * 10^6 12.9 / 15.0 -> 14.4 / 15.7
// (a wave's blocks one after the other), 1.8 * 10^8 181 / 213 -> 188 / 189 (two workgroups per compute unit 186 / 192); and not for
// mmv_scan: tiles of three chunks, 12 * 10^6 19.3 -> 21.2, 5 * 10^7 59.0 -> 57.9, 1.8 * 10^8 195.5 -> 196.5.
template <typename TT, int kOp, bool kMfma> constexpr bool has_round_form() {
    return (kOp == kScan || kOp == kPlainScan) && (TT::kDtype == MMV_I8_I32 || (sizeof(typename TT::in_t) <= 2 && !kMfma) || (kOp == kScan && sizeof(typename TT::in_t) == 2));
}
constexpr uint64_t kRoundTiles = 3 * kComputeUnits;
constexpr bool round_form(mmv_op op, mmv_dtype dt, uint64_t chunks, bool mfma) {   // `chunks`: per wave, of the whole vector
    if ((op != MMV_OP_SEGSCAN && op != MMV_OP_SCAN) || dt == MMV_F32_F32 || chunks > (uint64_t)kRoundCpw * kRoundTiles) return false;
    if (dt == MMV_I8_I32) return true;
    if (dt == MMV_U8_XOR) return !mfma;
    return (!mfma || op == MMV_OP_SEGSCAN) && chunks > (uint64_t)kRoundCpw * kResident;
}
struct TilePlan {
    TileRegions reg;
    uint64_t tiles;        // all tiles (reg.num_tiles holds it when it fits 31 bits)
    uint32_t unit;         // elements that one step of a region's `cpw` stands for: one chunk per wave (stream form: one unit of 1024)
    uint32_t body_elems;   // elements of a tile in the middle of the vector
    bool chunk_form;       // segmented sum: the kernel that streams through long spans (sum_kernel) takes it
    bool round_form;       // scans of 8- and 16-bit values: all tiles resident at once (OneRound, InLanes)
    bool short_form;       // stream form: at most kShortUnits units per tile, which a wave loads at once
};
inline TilePlan tile_plan(mmv_op op, mmv_dtype dt, uint64_t n, bool mfma = true) {
    TilePlan p = {};
    TileRegions &R = p.reg;
    if (is_spmv(op) || (op == MMV_OP_SEGSUM && dt == MMV_F32_F32)) {   // (stream_form)
        // Equal tiles, and as many as a whole number of rounds of resident workgroups takes (or nearly): where every
        // compute unit is busy with gathers all the time, one that holds three tiles when others hold two finishes last
        // (SpMV of 2^25 scattered entries: 683 tiles 0.238 ms, 763 tiles 0.213 ms; shorter tiles for the last 5 to 20 % of
        // the vector make sums and SpMV 1 to 10 % slower).  A tile has at least one unit per wave.
        uint64_t resident = kComputeUnits / 2 * (uint64_t)stream_waves_per_simd(is_spmv(op) ? kSpmv : kSum, mfma);
        const uint64_t units = (n + kUnitElems - 1) / kUnitElems;
        // A short vector gets one workgroup per compute unit as long as the form for short tiles takes that (sums then two):
        // with some of them holding two, it takes longer than with two units for a wave instead of one (CSR SpMV of 2.5 M
        // entries: 306 tiles of 8 units 14.6 us, 245 tiles of 10 units 13.3; sums so short have kernels of their own).
        // SpMV of 5 to 8 M entries in 512 short tiles: from 13 % faster (scattered) to 6 % slower (blocks of 16) than in 768.
        if (units <= kComputeUnits * kShortUnits) resident = kComputeUnits, p.short_form = true;
        else if (!is_spmv(op) && units <= 2 * kComputeUnits * kShortUnits) resident = 2 * kComputeUnits;
        const uint64_t rounds = (units + resident * kMaxUnits - 1) / (resident * kMaxUnits);
        uint64_t c = rounds ? (units + resident * rounds - 1) / (resident * rounds) : 1;
        if (c < kSpans) c = kSpans;
        if (!is_spmv(op) && c <= (uint64_t)kShortUnits) p.short_form = true;
        p.unit = kUnitElems;
        p.body_elems = (uint32_t)(c * kUnitElems);
        R.cpw[0] = (uint32_t)c;
        R.count = 1;
        p.tiles = (units + c - 1) / c;
        R.num_tiles = (uint32_t)(p.tiles < 0x7fffffffull ? p.tiles : 0x7fffffffull);
        return p;
    }
    const uint64_t unit = (uint64_t)waves_of(dt) * kChunkElems;  // one chunk per wave
    const uint64_t chunks = (n + unit - 1) / unit;
    if (round_form(op, dt, chunks, mfma)) {
        // short tiles first, as many long ones behind them as it takes: no compute unit gets more than one chunk per wave more
        p.round_form = true;
        p.unit = (uint32_t)unit;
        const uint64_t longer = chunks > kRoundTiles ? chunks - kRoundTiles : 0, shorter = chunks - 2 * longer;
        p.body_elems = (uint32_t)(longer ? 2 * unit : unit);
        if (shorter) {
            R.cpw[0] = 1;
            R.count = 1;
        }
        if (longer) {
            R.base[R.count] = shorter * unit;
            R.first[R.count] = (uint32_t)shorter;
            R.cpw[R.count] = 2;
            ++R.count;
        }
        p.tiles = shorter + longer;
        R.num_tiles = (uint32_t)p.tiles;
        return p;
    }
    // A sum that fits one round of workgroups is bound by the life of one tile, and the tile that holds all its
    // values, publishes its aggregate and then walks its ends has the shorter life (workload 2, fp16 2^24: 12.4
    // against 15.5 us); longer vectors go to the kernel that streams.
    int cpw = row_form_cpw(op, dt, mfma);
    const int chunk_cpw = chunk_form_cpw(op, dt, mfma);
    p.chunk_form = chunk_cpw > 0 && (MMV_SHORT_SUMS_ROW_FORM == 0 || n > MMV_SHORT_SUMS_ROW_FORM * kResident * unit * (uint64_t)cpw);
    if (p.chunk_form) cpw = chunk_cpw;
    p.unit = (uint32_t)unit;
    uint64_t tiles = 0, at = 0;
    auto add = [&](uint32_t c, uint64_t count) {   // `count` tiles of c chunks per wave from element `at` on
        if (count == 0) return;
        R.base[R.count] = at;
        R.first[R.count] = (uint32_t)tiles;
        R.cpw[R.count] = c;
        ++R.count;
        tiles += count;
        at += count * c * unit;
    };
    // The sum kernel of 8-bit inputs has four workgroups per compute unit, not two: a vector that is too long for
    // one round of 512 workgroups still gets one round, of up to 1024 (n = 2^27: 0.0485 -> 0.0445 ms whole call);
    // shorter ones keep the 512 longer tiles (as fast, and below the number of tiles that needs the prefix kernel).
    const uint64_t resident = p.chunk_form && dt == MMV_I8_I32 && n > kResident * unit * cpw ? 2 * kResident : kResident;
    if (n <= resident * unit * cpw) {
        // one round: equal tiles, as small as gives every resident workgroup at most one
        uint64_t c = (n + resident * unit - 1) / (resident * unit);
        if (c < 1) c = 1;
        if (c > (uint64_t)cpw) c = cpw;
        p.body_elems = (uint32_t)(unit * c);
        add((uint32_t)c, (n + unit * c - 1) / (unit * c));
    } else {
        p.body_elems = (uint32_t)(unit * cpw);
        // lengths of the short tiles: a quarter, a half and three quarters of the full length
        int steps[3], nsteps = 0;
        for (int q = 1; q <= 3; ++q) {
            const int c = cpw * q / 4;
            if (c >= 1 && c < cpw && (nsteps == 0 || steps[nsteps - 1] != c)) steps[nsteps++] = c;
        }
        uint64_t head = 0, tail = (uint64_t)MMV_TAIL_TILES * unit;   // elements in the short tiles of both ends
        for (int i = 0; i < nsteps; ++i) {
            head += (uint64_t)MMV_HEAD_GROUP * steps[i] * unit;
            if (steps[i] >= 2) tail += (uint64_t)MMV_TAIL_GROUP * steps[i] * unit;
        }
        const bool graded = nsteps > 0 && head + tail <= n;
        if (!graded) head = 0, tail = (uint64_t)MMV_TAIL_TILES * unit < n ? (uint64_t)MMV_TAIL_TILES * unit : n;
        if (graded)
            for (int i = 0; i < nsteps; ++i) add((uint32_t)steps[i], MMV_HEAD_GROUP);
        add((uint32_t)cpw, (n - head - tail) / (unit * cpw));
        if (graded)
            for (int i = nsteps - 1; i >= 0; --i)
                if (steps[i] >= 2) add((uint32_t)steps[i], MMV_TAIL_GROUP);
        if (cpw > 1 || R.count == 0) {
            add(1u, (n - at + unit - 1) / unit);          // what is left, the last tile ragged
        } else {
            tiles += (n - at + unit - 1) / unit;          // (tiles of one chunk per wave throughout: one region)
        }
    }
    p.tiles = tiles;
    R.num_tiles = (uint32_t)(tiles < 0x7fffffffull ? tiles : 0x7fffffffull);
    return p;
}
// (for sizing: the variant with the shorter tiles needs more descriptors)
inline uint64_t tiles_for(uint64_t n, mmv_op op, mmv_dtype dt) {
    const uint64_t a = tile_plan(op, dt, n, true).tiles, b = tile_plan(op, dt, n, false).tiles;
    return a > b ? a : b;
}
// Bytes of x where 32-bit offsets reach all of it, else 0.  2^30 entries are one byte more than it can say: loads that check their range
// (buffered_loads) would read 0 for the last entry, so these products take the form for a longer x.
inline uint32_t x_bytes_of(uint64_t n_cols) { return n_cols > (1ull << 30) ? 0u : n_cols == (1ull << 30) ? ~0u : n_cols ? 4u * (uint32_t)n_cols : 1u; }
template <int kOp, bool kShort> constexpr bool narrow_x(uint32_t x_bytes) {
    return kOp == kSum || (x_bytes != 0 && !(x_bytes == ~0u && buffered_loads<kOp, kShort>()));
}
inline bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }
inline bool aligned4(const void *p) { return ((uintptr_t)p & 3u) == 0; }

inline uint64_t short_tiles(uint64_t n) { return (n + kShortTile - 1) / kShortTile; }

struct WsLayout {
    size_t desc_v, desc_c, span_c, packed, total;
};

WsLayout ws_layout(mmv_op op, mmv_dtype dt, mmv_flag_fmt ff, uint64_t n) {
    WsLayout L;
    const uint64_t t = tiles_for(n, op, dt);
    size_t off = kHdrBytes;
    L.desc_v = off;
    off += round256(t * 8);
    L.desc_c = off;   // counts of segment starts: per tile, and (sum_kernel) per wave span
    if (op == MMV_OP_SEGSUM || op == MMV_OP_SPMV_CSR) off += round256(t * 4);
    L.span_c = off;
    if (op == MMV_OP_SEGSUM && segsum_spans(dt)) off += round256(t * 4 * kSpans);
    L.packed = off;
    if (is_spmv(op) || (ff == MMV_FLAGS_U8 && op != MMV_OP_SCAN)) off += round256(((n + 63) / 64) * 8);
    L.total = off;
    // The two launches of a short vector keep one aggregate per tile where the descriptors begin; longer vectors get at least the
    // room for those of a vector of short_max elements.  (The size does not grow with n throughout: where a vector stops
    // fitting one round of workgroups it takes fewer, longer tiles, and fewer descriptors.)
    if (!is_spmv(op)) {
        const size_t aggregates = kHdrBytes + round256(short_tiles(n < short_max(op, dt) ? n : short_max(op, dt)) * 8);
        if (L.total < aggregates) L.total = aggregates;
    }
    return L;
}

// Workspace of COMPRESS: header and one count descriptor per tile, all of it zeroed by every call.
struct CompressLayout {
    size_t desc, total;
    uint64_t tiles;
};
CompressLayout compress_layout(uint64_t n) {
    CompressLayout L;
    L.tiles = (n + compress_tile(n) - 1) / compress_tile(n);
    size_t off = kHdrBytes;
    L.desc = off;
    off += round256(L.tiles * 8);
    L.total = off;
    return L;
}

// Workspaces of the un-fused compositions: the sub-workspaces of the primitives they call and
// their intermediate vectors, one after the other (every offset a multiple of 256).
struct ScdLayout {
    size_t scan_ws, xhat, packed, fminus, compress_ws, w, total;
};
ScdLayout scd_layout(mmv_dtype dt, mmv_flag_fmt ff, uint64_t n, uint64_t cap) {
    ScdLayout L;
    size_t off = 0;
    L.scan_ws = off;
    off += round256(ws_layout(MMV_OP_SCAN, dt, MMV_FLAGS_PACKED32, n).total);
    L.xhat = off;
    off += round256(n * 4);
    L.packed = off;
    if (ff == MMV_FLAGS_U8) off += round256(((n + 63) / 64) * 8);
    L.fminus = off;
    off += round256(((n + 63) / 64) * 8);
    L.compress_ws = off;
    off += round256(compress_layout(n).total);
    L.w = off;
    off += round256((cap < n ? cap : n) * 4 + 16);
    L.total = off;
    return L;
}
struct SscrLayout {
    size_t scan_ws_x, scan_ws_f, fhat, f8, packed, fminus, compress_ws, w, total;
};
SscrLayout sscr_layout(mmv_dtype dt, mmv_flag_fmt ff, uint64_t n) {
    SscrLayout L;
    size_t off = 0;
    L.scan_ws_x = off;
    off += round256(ws_layout(MMV_OP_SCAN, dt, MMV_FLAGS_PACKED32, n).total);
    L.scan_ws_f = off;
    off += round256(ws_layout(MMV_OP_SCAN, MMV_I8_I32, MMV_FLAGS_PACKED32, n).total);
    L.fhat = off;
    off += round256(n * 4);
    L.f8 = off;
    off += round256(n + 16);   // flags as one 0 / 1 byte per element for SCAN(f)
    L.packed = off;
    if (ff == MMV_FLAGS_U8) off += round256(((n + 63) / 64) * 8);
    L.fminus = off;
    off += round256(((n + 63) / 64) * 8);
    L.compress_ws = off;
    off += round256(compress_layout(n).total);
    L.w = off;
    off += round256(n * 4 + 16);   // one entry per segment, at most n
    L.total = off;
    return L;
}
// CSR SpMV: the main kernel's workspace (flags over the non-zeros included), the mask of rows
// with entries, their indices (rowmap) and the workspace of the COMPRESS that makes them.
struct CsrLayout {
    size_t main_ws, rowmask, rowmap, rowcount, compress_ws, total;
};
CsrLayout csr_layout(uint64_t n_rows, uint64_t nnz) {
    CsrLayout L;
    size_t off = 0;
    L.main_ws = off;   // the two workspaces that hold tickets and descriptors lie next to each other:
    off += round256(ws_layout(MMV_OP_SPMV_CSR, MMV_F32_F32, MMV_FLAGS_PACKED32, nnz).total);
    L.compress_ws = off;   // one fill clears both (and the flag words between them)
    off += round256(compress_layout(n_rows).total);
    L.rowmask = off;
    off += round256(((n_rows + 63) / 64) * 8);
    L.rowmap = off;
    off += round256(n_rows * 4 + 16);
    L.rowcount = off;
    off += 256;
    L.total = off;
    return L;
}

// Optional instrumentation (mmv_set_kernel_events): events recorded right before and
// right after the main kernel of a call made by this host thread.
thread_local hipEvent_t tl_ev_start = nullptr, tl_ev_stop = nullptr;

// Workgroups of `kernel` that the current device holds at once (0 when a query fails).  `cache` is the
// caller's table for this kernel, one word per device (0 = not asked yet, else the value + 1): a fixed
// array per kernel instantiation, so nothing grows and nothing is allocated after the library is loaded.
constexpr int kMaxDevices = 64;
uint32_t resident_workgroups(const void *kernel, int threads, std::atomic<uint32_t> (&cache)[kMaxDevices]) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
    const uint32_t known = cache[dev].load(std::memory_order_relaxed);
    if (known) return known - 1u;
    int per_cu = 0, cus = 0;
    uint32_t value = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && per_cu > 0 && cus > 0)
        value = (uint32_t)per_cu * (uint32_t)cus;
    cache[dev].store(value + 1u, std::memory_order_relaxed);   // (two threads asking at once store the same value)
    return value;
}

// Workgroups that take the tile of their own index: those resident from the start, and the first one in any case (the
// number is 0 when the device could not be asked).
constexpr uint32_t first_round_of(uint32_t num_tiles, uint32_t resident) {
    return num_tiles < resident ? num_tiles : resident > 0 ? resident : 1u;
}

template <typename TT, int kOp, bool kMfma> hipError_t launch_variant(Params P, const TilePlan &plan, hipStream_t s) {
    static std::atomic<uint32_t> occupancy[3][kMaxDevices];
    void (*kernel)(Params, const uint32_t *);
    int which = 0;
    if constexpr (stream_form<TT, kOp>()) {
        // (a long x, whatever the matrix: the form for long vectors)
        const bool narrow = plan.short_form ? narrow_x<kOp, true>(P.x_bytes) : narrow_x<kOp, false>(P.x_bytes);
        which = !narrow ? 1 : plan.short_form ? 2 : 0;
        kernel = which == 2 ? stream_kernel<TT, kOp, kMfma, true, true> : stream_kernel<TT, kOp, kMfma, true, false>;
        if constexpr (kOp != kSum) {
            if (!narrow) kernel = stream_kernel<TT, kOp, kMfma, false, false>;
        }
    } else if constexpr (lane_form<TT, kOp>()) {
        kernel = seg_kernel<InLanes<TT>, kOp, false>;   // (both variants)
    } else {
        kernel = seg_kernel<TT, kOp, kMfma>;
        if constexpr (has_round_form<TT, kOp, kMfma>()) {
            which = plan.round_form ? 2 : 0;
            typedef std::conditional_t<sizeof(typename TT::in_t) == 2 && kMfma, InLanes<TT>, OneRound<TT>> Round;
            if (plan.round_form) kernel = seg_kernel<Round, kOp, kMfma && !kInLanes<Round>>;
        }
        if constexpr (chunk_sum_kernel<TT, kOp, kMfma>()) {
            which = plan.chunk_form ? 1 : 0;
            if (plan.chunk_form) kernel = sum_kernel<TT, kMfma>;
        }
    }
    const uint32_t resident = resident_workgroups((const void *)kernel, TT::kWaves * 64, occupancy[which]);
    P.first_round = first_round_of(P.num_tiles, resident);
    kernel<<<P.num_tiles, TT::kWaves * 64, 0, s>>>(P, P.hdr + kHdrHints);
    return hipGetLastError();
}

template <typename TT, int kOp>
hipError_t launch_seg(Params P, mmv_variant v, hipStream_t s) {
    const TilePlan plan = tile_plan((mmv_op)kOp, TT::kDtype, P.n, v == MMV_VARIANT_MFMA);
    if (plan.tiles > 0x7fffffffull) return hipErrorInvalidValue;
    P.num_tiles = (uint32_t)plan.tiles;
    P.reg = plan.reg;
    if (tl_ev_start && hipEventRecord(tl_ev_start, s) != hipSuccess) return hipErrorUnknown;
    if (v == MMV_VARIANT_MFMA) {
        if (launch_variant<TT, kOp, true>(P, plan, s) != hipSuccess) return hipErrorUnknown;
    } else {
        if (launch_variant<TT, kOp, false>(P, plan, s) != hipSuccess) return hipErrorUnknown;
    }
    const hipError_t e = hipGetLastError();
    if (tl_ev_stop && hipEventRecord(tl_ev_stop, s) != hipSuccess) return hipErrorUnknown;
    return e;
}

template <int kOp> hipError_t launch_dt(const Params &P, mmv_dtype dt, mmv_variant v, hipStream_t s) {
    switch (dt) {
        case MMV_F32_F32: return launch_seg<TF32, kOp>(P, v, s);
        case MMV_F16_F32: return launch_seg<TF16, kOp>(P, v, s);
        case MMV_BF16_F32: return launch_seg<TBF16, kOp>(P, v, s);
        case MMV_I8_I32: return launch_seg<TI8, kOp>(P, v, s);
        case MMV_U8_XOR: return launch_seg<TX8, kOp>(P, v, s);
        default: break;
    }
    return hipErrorInvalidValue;
}

inline uint64_t elem_bytes(mmv_dtype dt) { return dt == MMV_F32_F32 ? 4 : dt == MMV_F16_F32 || dt == MMV_BF16_F32 ? 2 : 1; }
inline uint64_t flag_bytes(mmv_flag_fmt ff, uint64_t n) { return ff == MMV_FLAGS_U8 ? n : (n + 31) / 32 * 4; }

// Scans and sums of at most short_max elements on checked arguments (P: where things lie in the workspace).
template <typename TT, int kOp, int kFlags> hipError_t launch_short(const ShortParams &S, bool single, hipStream_t s) {
    const unsigned tiles = (unsigned)short_tiles(S.n);
    // (both launches read the inputs: the events stand around the two)
    if (tl_ev_start && hipEventRecord(tl_ev_start, s) != hipSuccess) return hipErrorUnknown;
    if (!single) {
        short_reduce_kernel<TT, kFlags><<<tiles, kShortThreads, 0, s>>>(S);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const uint64_t bytes = S.n * elem_bytes(TT::kDtype) + (kFlags == kNoFlags ? 0 : flag_bytes(kFlags == kByteFlags ? MMV_FLAGS_U8 : MMV_FLAGS_PACKED32, S.n));
    if (!single) short_kernel<TT, kOp, kFlags, false, kShortThreads><<<tiles, kShortThreads, 0, s>>>(S);
    else if (bytes < many_bytes(TT::kDtype, kFlags)) short_kernel<TT, kOp, kFlags, true, kShortThreads><<<tiles, kShortThreads, 0, s>>>(S);
    else short_kernel<TT, kOp, kFlags, true, kManyThreads><<<tiles, kManyThreads, 0, s>>>(S);
    const hipError_t e = hipGetLastError();
    if (tl_ev_stop && hipEventRecord(tl_ev_stop, s) != hipSuccess) return hipErrorUnknown;
    return e;
}
template <typename TT, int kOp> hipError_t launch_short_flags(const ShortParams &S, mmv_flag_fmt ff, bool single, hipStream_t s) {
    if constexpr (kOp == kPlainScan) return launch_short<TT, kOp, kNoFlags>(S, single, s);
    else return ff == MMV_FLAGS_U8 ? launch_short<TT, kOp, kByteFlags>(S, single, s) : launch_short<TT, kOp, kBitFlags>(S, single, s);
}
inline bool overlap(const void *a, uint64_t a_bytes, const void *b, uint64_t b_bytes) {
    return (uintptr_t)a < (uintptr_t)b + b_bytes && (uintptr_t)b < (uintptr_t)a + a_bytes;
}

// What a scan or sum takes: one launch of short_kernel, two, or the single-pass kernel (always beyond short_max).  In one launch
// every workgroup reads what lies before its tile, so nothing of that may be written meanwhile; in two a workgroup
// still loads the values and flags of its own tile (a sum also the flag behind it), so an output may lie over nothing but a
// scan's own values, each thread's results over its own.  Any other overlap is left to the single-pass kernel, whose
// launches pack byte flags before the first result is written.  (`flags`: nullptr where there are none.)
enum ShortRoute { kSinglePass, kTwoLaunches, kOneLaunch };
inline ShortRoute short_route(mmv_op op, mmv_dtype dt, mmv_flag_fmt ff, uint64_t n, const void *x, const void *flags, const void *out,
                              uint64_t out_bytes) {
    if (n > short_max(op, dt)) return kSinglePass;
    const uint64_t xb = n * elem_bytes(dt), fb = flags ? flag_bytes(ff, n) : 0;
    if (flags && overlap(out, out_bytes, flags, fb)) return kSinglePass;
    if (overlap(out, out_bytes, x, xb)) return op != MMV_OP_SEGSUM && out == x ? kTwoLaunches : kSinglePass;
    return xb + fb <= MMV_SINGLE_BYTES ? kOneLaunch : kTwoLaunches;
}
template <int kOp>
mmv_status short_call(const void *d_x, const void *d_flags, uint64_t n, void *d_z, void *d_out, uint64_t out_cap, uint64_t *d_nseg,
                      bool first_one, mmv_dtype dt, mmv_flag_fmt ff, const Params &P, bool single, hipStream_t s) {
    const ShortParams S = {d_x, d_flags, d_z, d_out, out_cap, d_nseg, P.hdr, P.desc_v, (uint32_t)n, first_one ? 1u : 0u};
    hipError_t e = hipErrorInvalidValue;
    switch (dt) {
        case MMV_F32_F32: e = launch_short_flags<TF32, kOp>(S, ff, single, s); break;
        case MMV_F16_F32: e = launch_short_flags<TF16, kOp>(S, ff, single, s); break;
        case MMV_BF16_F32: e = launch_short_flags<TBF16, kOp>(S, ff, single, s); break;
        case MMV_I8_I32: e = launch_short_flags<TI8, kOp>(S, ff, single, s); break;
        case MMV_U8_XOR: e = launch_short_flags<TX8, kOp>(S, ff, single, s); break;
        default: break;
    }
    return e == hipSuccess ? MMV_OK : MMV_ERR_HIP;
}

int grid_for(uint64_t items_per_thread_total) {
    uint64_t blocks = (items_per_thread_total + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 2048) blocks = 2048;
    return (int)blocks;
}

bool valid_dtype(int dt) { return dt >= 0 && dt <= 4; }
bool valid_ff(int ff) { return ff == 0 || ff == 1; }
bool valid_variant(int v) { return v == 0 || v == 1; }
bool valid_elem(int et) { return et == 0 || et == 1; }
constexpr uint64_t kMaxN = 1ull << 40;

// Common part of scan and sum: checks, which launches follow, workspace reset, flag packing.
mmv_status prepare(mmv_op op, const void *d_x, const void *d_flags, uint64_t n, const void *d_out, uint64_t out_bytes, mmv_dtype dt,
                   mmv_flag_fmt ff, mmv_variant v, void *d_ws, size_t ws_bytes, hipStream_t s, Params &P, ShortRoute &route) {
    if (!valid_dtype(dt) || !valid_ff(ff) || !valid_variant(v) || n > kMaxN) return MMV_ERR_INVALID_ARG;
    if (!d_x || !d_flags) return MMV_ERR_NULL;
    if (!aligned16(d_x) || !aligned16(d_flags)) return MMV_ERR_INVALID_ARG;
    if (!d_ws) return MMV_ERR_NULL;
    const WsLayout L = ws_layout(op, dt, ff, n);
    if (((uintptr_t)d_ws & 255u) != 0 || ws_bytes < L.total) return MMV_ERR_WORKSPACE;
    char *ws = (char *)d_ws;
    P.x = d_x;
    P.n = n;
    P.hdr = (uint32_t *)ws;
    P.desc_v = (uint64_t *)(ws + L.desc_v);
    P.num_tiles = (uint32_t)tiles_for(n, op, dt);
    // header and descriptors zeroed, flags packed if they came as bytes: one launch.  The segmented sum does both in its counting
    // kernel; a short vector needs neither.
    uint32_t *packed = (uint32_t *)(ws + L.packed);
    P.fw = ff == MMV_FLAGS_U8 ? packed : (const uint32_t *)d_flags;
    route = short_route(op, dt, ff, n, d_x, d_flags, d_out, out_bytes);
    if (op == MMV_OP_SEGSUM || route != kSinglePass) return MMV_OK;
    const uint64_t zero_words = L.packed / 4;
    if (ff == MMV_FLAGS_U8) {
        const uint64_t nwords = (n + 31) / 32;
        pack_flags_kernel<<<grid_for(nwords > zero_words ? nwords : zero_words), 256, 0, s>>>((const uint8_t *)d_flags, n, packed, nwords,
                                                                                             (uint32_t *)ws, zero_words);
    } else {
        fill_zero_kernel<<<grid_for(zero_words), 256, 0, s>>>((uint32_t *)ws, zero_words, nullptr, 0);
    }
    if (hipGetLastError() != hipSuccess) return MMV_ERR_HIP;
    return MMV_OK;
}

// Turns timing events off for the sub-calls of a composition (each would re-record them).
struct EventsOff {
    hipEvent_t a, b;
    EventsOff() : a(tl_ev_start), b(tl_ev_stop) { tl_ev_start = tl_ev_stop = nullptr; }
    ~EventsOff() {
        tl_ev_start = a;
        tl_ev_stop = b;
    }
};

// SCAN on an input that is already checked; first_one makes element 0 count as 1 (flag bytes).
mmv_status scan_impl(const void *d_x, uint64_t n, void *d_z, mmv_dtype dt, mmv_variant v, void *d_ws,
                     size_t ws_bytes, hipStream_t s, bool first_one) {
    const WsLayout L = ws_layout(MMV_OP_SCAN, dt, MMV_FLAGS_PACKED32, n);
    if (((uintptr_t)d_ws & 255u) != 0 || ws_bytes < L.total) return MMV_ERR_WORKSPACE;
    char *ws = (char *)d_ws;
    Params P = {};
    P.x = d_x;
    P.n = n;
    P.z = d_z;
    P.hdr = (uint32_t *)ws;
    P.desc_v = (uint64_t *)(ws + L.desc_v);
    P.first_one = first_one ? 1u : 0u;
    const ShortRoute route = short_route(MMV_OP_SCAN, dt, MMV_FLAGS_PACKED32, n, d_x, nullptr, d_z, n * 4);
    if (route != kSinglePass)
        return short_call<kPlainScan>(d_x, nullptr, n, d_z, nullptr, 0, nullptr, first_one, dt, MMV_FLAGS_PACKED32, P, route == kOneLaunch, s);
    const uint64_t zero_words = L.total / 4;
    fill_zero_kernel<<<grid_for(zero_words), 256, 0, s>>>((uint32_t *)ws, zero_words, nullptr, 0);
    if (hipGetLastError() != hipSuccess) return MMV_ERR_HIP;
    return launch_dt<kPlainScan>(P, dt, v, s) == hipSuccess ? MMV_OK : MMV_ERR_HIP;
}

// COMPRESS on checked arguments; d_x == nullptr compresses the positions.
mmv_status compress_impl(const void *d_x, const void *d_mask, uint64_t n, void *d_out, uint64_t out_capacity,
                         uint64_t *d_count, mmv_flag_fmt ff, void *d_ws, size_t ws_bytes, hipStream_t s,
                         bool ws_is_reset = false, const uint32_t *d_needed = nullptr) {
    const CompressLayout L = compress_layout(n);
    if (((uintptr_t)d_ws & 255u) != 0 || ws_bytes < L.total) return MMV_ERR_WORKSPACE;
    if (L.tiles > 0x7fffffffull) return MMV_ERR_INVALID_ARG;
    char *ws = (char *)d_ws;
    // one launch: every workgroup reads the mask before its tile, and none waits for another, so an output over the mask
    // or over x would be written before others have read there
    const uint64_t out_bytes = (out_capacity < n ? out_capacity : n) * 4;
    const bool single = !ws_is_reset && compress_words(n) == 16 && n <= (ff == MMV_FLAGS_U8 ? kCompressSingleBytes : kCompressSingleBits) &&
                        !overlap(d_out, out_bytes, d_mask, flag_bytes(ff, n)) && !(d_x && overlap(d_out, out_bytes, d_x, n * 4));
    if (!ws_is_reset && !single) {
        const uint64_t zero_words = L.total / 4;
        fill_zero_kernel<<<grid_for(zero_words), 256, 0, s>>>((uint32_t *)ws, zero_words, nullptr, 0);
        if (hipGetLastError() != hipSuccess) return MMV_ERR_HIP;
    }
    if (tl_ev_start && hipEventRecord(tl_ev_start, s) != hipSuccess) return MMV_ERR_HIP;
    // the workgroups that are resident from the start take the tile of their own index, the others a ticket
    static std::atomic<uint32_t> occupancy[10][kMaxDevices];
    typedef void (*Kernel)(const uint32_t *, const void *, uint64_t, uint32_t *, uint64_t, uint64_t *, uint32_t *, uint64_t *,
                           uint32_t, const uint32_t *, uint32_t);
    static const Kernel kernels[10] = {compress_kernel<16, 1, false>, compress_kernel<64, 1, false>, compress_kernel<64, 2, false>,
                                       compress_kernel<64, 4, false>, compress_kernel<16, 1, true>,  compress_kernel<64, 1, true>,
                                       compress_kernel<64, 2, true>,  compress_kernel<64, 4, true>,  compress_kernel<16, 1, false, true>,
                                       compress_kernel<16, 1, true, true>};
    const int which = single ? (ff == MMV_FLAGS_U8 ? 9 : 8) :
                      (compress_words(n) == 16 ? 0 : compress_groups(n) == 1 ? 1 : compress_groups(n) == 2 ? 2 : 3) +
                      (ff == MMV_FLAGS_U8 ? 4 : 0);
    const Kernel kernel = kernels[which];
    const uint32_t resident = resident_workgroups((const void *)kernel, kCompressWaves * 64, occupancy[which]);
    const uint32_t first_round = single || (uint32_t)L.tiles < resident ? (uint32_t)L.tiles : resident;   // (no tickets in one launch)
    kernel<<<(unsigned)L.tiles, kCompressWaves * 64, 0, s>>>((const uint32_t *)d_x, d_mask, n, (uint32_t *)d_out, out_capacity,
                                                             d_count, (uint32_t *)ws, (uint64_t *)(ws + L.desc),
                                                             (uint32_t)L.tiles, d_needed, first_round);
    const hipError_t e = hipGetLastError();
    if (tl_ev_stop && hipEventRecord(tl_ev_stop, s) != hipSuccess) return MMV_ERR_HIP;
    return e == hipSuccess ? MMV_OK : MMV_ERR_HIP;
}

// Matrices that csr_plan_kernel prepares tile by tile; the launches over the rows, spread over the chip whatever the rows, are
// left to those with so few entries that a tile holds too many rows.  Products in one step, launches over the rows / tile by
// tile (us), rows with one entry or none, 0.4, 0.25 and 0.06 entries per row: 2^14 rows 31 / 26, 28 / 23, 22 / 22; 2^16 37 / 32,
// 37 / 39, 31 / 54; 2^18 77 / 34, 77 / 41, 72 / 103; 2^20 154 / 44, 175 / 52, 211 / 106.
// Uneven rows, over the rows / tile by tile / with the tiles of many rows shared: 2^18 rows, half of them of 16 entries, then one in
// 20 of one entry in a tile or two, 51 / 59 / 31; 2^25 entries in 200 000 rows, then 2^20 rows, one in 24 of one entry, 369 / 476 / 198;
// a row of 600 000, then 2^20 rows, one in 2048 of one entry, 26 / 38 / 21.
// (A row and two marks share a word of tile_base.)
constexpr bool rows_by_tile(uint64_t n_rows, uint64_t nnz) { return n_rows / 3 <= nnz && n_rows < kPlanByEnd; }
// Most rows of a tile that its workgroup takes alone: two pieces, so many as positions (a shared tile needs a slot for each), or twice
// what a tile has on average, so that the tiles of an even matrix of few entries per row stay whole (2^24 rows, 0.4 entries per row:
// 168 us the call, 194 with its tiles of 23000 rows shared).
constexpr uint64_t plan_share_above(uint64_t n_rows, uint64_t tiles, uint32_t tile_elems) {
    const uint64_t even = 2 * ((n_rows + tiles - 1) / tiles), pieces = 2 * kPlanShare, most = even > pieces ? even : pieces;
    return most > tile_elems ? most : tile_elems;
}
// Workgroups of csr_plan_kernel behind those of the tiles: none where no tile can be shared.
constexpr uint64_t plan_helpers(uint64_t n_rows, uint64_t share_above) {
    return n_rows > share_above ? (n_rows + kPlanShare - 1) / kPlanShare : 0;
}

// What the CSR product needs of the matrix alone, header and descriptors zeroed, and y (nullptr: not).
mmv_status csr_plan(uint64_t n_rows, uint64_t nnz, const int32_t *d_rowptr, uint32_t *d_y, char *ws, const CsrLayout &C, const WsLayout &L,
                    const TilePlan &plan, hipStream_t s) {
    uint32_t *fw = (uint32_t *)(ws + C.main_ws + L.packed);
    uint32_t *tile_count = (uint32_t *)(ws + C.main_ws + L.desc_c);
    if (rows_by_tile(n_rows, nnz)) {
        const uint64_t share_above = plan_share_above(n_rows, plan.tiles, plan.body_elems);
        const unsigned workgroups = (unsigned)(plan.tiles + plan_helpers(n_rows, share_above));
        csr_plan_kernel<<<workgroups, kPlanThreads, 0, s>>>(d_rowptr, (uint32_t)n_rows, (uint32_t)nnz, (uint32_t)plan.tiles,
                                                                      plan.body_elems, (uint32_t)share_above, fw, tile_count, (uint32_t *)(ws + C.rowmap),
                                                                      (uint32_t *)(ws + C.main_ws), L.desc_c / 4, d_y, d_y ? (uint32_t)n_rows : 0u);
        return hipGetLastError() == hipSuccess ? MMV_OK : MMV_ERR_HIP;
    }
    // zero: the main kernel's header, descriptors and flag words, the header and descriptors of COMPRESS; y
    const uint64_t zero_words = (C.compress_ws + compress_layout(n_rows).total) / 4, y_rows = d_y ? n_rows : 0;
    fill_zero_kernel<<<grid_for(zero_words > y_rows ? zero_words : y_rows), 256, 0, s>>>((uint32_t *)ws, zero_words, d_y, y_rows);
    if (hipGetLastError() != hipSuccess) return MMV_ERR_HIP;
    // segment-start flags over the non-zeros, their number per tile of the main kernel, and the mask of
    // rows that have entries
    const uint64_t row_blocks = (n_rows + 255) / 256;
    csr_flags_kernel<<<(unsigned)row_blocks, 256, 0, s>>>(d_rowptr, n_rows, fw, (uint32_t *)(ws + C.rowmask),
                                                          (uint32_t *)(ws + C.main_ws), plan.body_elems, tile_count);
    if (hipGetLastError() != hipSuccess) return MMV_ERR_HIP;
    // rowmap = COMPRESS(0 .. n_rows - 1, rowmask): the k-th segment belongs to row rowmap[k]
    {
        EventsOff quiet;
        const mmv_status st = compress_impl(nullptr, ws + C.rowmask, n_rows, ws + C.rowmap, n_rows,
                                            (uint64_t *)(ws + C.rowcount), MMV_FLAGS_PACKED32, ws + C.compress_ws,
                                            C.rowmask - C.compress_ws, s, true,
                                            (const uint32_t *)(ws + C.main_ws) + kHdrEmptyRows);
        if (st != MMV_OK) return st;
    }
    if (plan.tiles > kCountTiles) {
        scan_counts_kernel<<<1, 1024, 0, s>>>(tile_count, (uint32_t)plan.tiles, (uint64_t *)(ws + C.rowcount));
        if (hipGetLastError() != hipSuccess) return MMV_ERR_HIP;
    }
    return MMV_OK;
}

mmv_status diff_impl(const void *d_x, uint64_t n, void *d_z, mmv_elem et, hipStream_t s,
                     const uint64_t *d_limit = nullptr) {
    const uint64_t blocks = (n + 1023) / 1024;
    if (blocks > 0x7fffffffull) return MMV_ERR_INVALID_ARG;
    if (tl_ev_start && hipEventRecord(tl_ev_start, s) != hipSuccess) return MMV_ERR_HIP;
    if (et == MMV_ELEM_I32)
        diff_kernel<uint32_t><<<(unsigned)blocks, 256, 0, s>>>((const uint32_t *)d_x, n, (uint32_t *)d_z, d_limit);
    else
        diff_kernel<float><<<(unsigned)blocks, 256, 0, s>>>((const uint32_t *)d_x, n, (uint32_t *)d_z, d_limit);
    const hipError_t e = hipGetLastError();
    if (tl_ev_stop && hipEventRecord(tl_ev_stop, s) != hipSuccess) return MMV_ERR_HIP;
    return e == hipSuccess ? MMV_OK : MMV_ERR_HIP;
}

mmv_status revert_impl(const void *d_xhat, const int32_t *d_fhat, const void *d_w, uint64_t n, uint64_t nw,
                       void *d_z, mmv_elem et, hipStream_t s) {
    const uint64_t blocks = (n + 1023) / 1024;
    if (blocks > 0x7fffffffull) return MMV_ERR_INVALID_ARG;
    if (tl_ev_start && hipEventRecord(tl_ev_start, s) != hipSuccess) return MMV_ERR_HIP;
    if (et == MMV_ELEM_I32)
        revert_kernel<uint32_t><<<(unsigned)blocks, 256, 0, s>>>((const uint32_t *)d_xhat, d_fhat, (const uint32_t *)d_w,
                                                                  n, nw, (uint32_t *)d_z);
    else
        revert_kernel<float><<<(unsigned)blocks, 256, 0, s>>>((const uint32_t *)d_xhat, d_fhat, (const uint32_t *)d_w, n,
                                                               nw, (uint32_t *)d_z);
    const hipError_t e = hipGetLastError();
    if (tl_ev_stop && hipEventRecord(tl_ev_stop, s) != hipSuccess) return MMV_ERR_HIP;
    return e == hipSuccess ? MMV_OK : MMV_ERR_HIP;
}

}  // namespace
