// libmmvseg, part of the one translation unit mmvseg.hip (included there, in order).
// The tile body of the segmented sum of 32-bit values and of SpMV (COO and CSR): waves that stream through their spans
// one 32x32 tile of 1024 elements at a time.
#pragma once

namespace {

// ---- segmented sum of 32-bit values, SpMV -------------------------------------------------------------------------
//
// Steps 1 to 6 of the block-recursive scheme as in seg_tile, but an output exists only where a segment ends, so a wave
// is done with a unit of 1024 elements (32 rows of 32) once the ends in it are written, and everything such an end needs
// is in those rows, except for the first end of a unit when its segment began before the unit: that output is kept in LDS,
// with the aggregate of the unit, and written at the end of the tile, when one wave has scanned the aggregates of the
// units and looked back for the carry of the tile.  So a wave keeps one unit in registers and LDS, with the loads of the
// next one under way, however long the tile is.  The units of a tile are dealt to its waves in turn, so that the
// workgroup reads one stretch of memory after the other: with a span of its own for every wave, 6000 spans of the
// arrays were being read at a time (sums of 2^26 values 59 us against 52 now).
// What bounds it: the loads, as far as the tiles are long enough and the ends not too many.  Whole calls, matrix cores /
// without, with one chunk (two) of 2048 elements per wave and tile held in registers as in seg_tile -> now:
//   sum of 10^8 fp32 values, 1 % of them starts    123 / 88 us -> 82 / 73 us (5.1 / 5.7 TB/s)
//   ... 30 % starts                                193 / 143 -> 133 / 133
//   CSR SpMV, sparse attention, 62.8 M entries in blocks of 64 (prepared)     127 -> 103 us (4.9 TB/s)
//   ... 9.5 M entries in blocks of 16                                         37.7 -> 24.9
//   COO SpMV, 33.6 M entries in scattered columns                             239 -> 240 (bound by the gathers)
// Waves per SIMD: SpMV keeps one unit per wave and six waves per SIMD hide the loads (four with two units: 0.128 ms for the
// 62.8 M entries, eight spill); sums on the matrix cores keep two units in flight and four waves (six with one: level).
// Precision is that of seg_tile: speculation within rows of 32 elements, segmented carries from there on.
constexpr int kUnitElems = 1024;   // what a wave handles at a time: 32 rows
constexpr int kUnitRows = 32;

#ifndef MMV_STREAM_CPW
#define MMV_STREAM_CPW 16          // most units per wave and tile (8: 0.118 ms for the 62.8 M entries above, 16: 0.100)
#endif
#ifndef MMV_STREAM_DEPTH_SUM
#define MMV_STREAM_DEPTH_SUM 2     // units of a wave whose loads are under way or waiting in registers, sums
#endif
#ifndef MMV_STREAM_DEPTH_SPMV
#define MMV_STREAM_DEPTH_SPMV 1    // ... SpMV (values and columns)
#endif
#ifndef MMV_STREAM_WPS_SUM
#define MMV_STREAM_WPS_SUM 4       // waves per SIMD the compiler is to leave room for: sums on the matrix cores, ...
#endif
#ifndef MMV_STREAM_WPS_SUM_SHUFFLE
#define MMV_STREAM_WPS_SUM_SHUFFLE 6
#endif
#ifndef MMV_STREAM_WPS_SPMV
#define MMV_STREAM_WPS_SPMV 6
#endif

// Vectors of at most 16 units per tile are bound by the life of one tile, and get a form of their own (kShort): a wave has
// both its units loaded before the first is worked on.  In the other form the loads of its second unit are waited for behind
// the stores of the first (one counter counts both in order, and the number of stores is not known), and the table lookups,
// which stand in branches, ahead of the first value.  Whole calls in a graph, one chunk of 2048 elements per wave as in
// seg_tile / the form for long vectors / this one (sums: matrix cores, 1 % of the values start a segment; up to 3 * 2^20 values they
// come here only with the output over an input, see short_call):
//   sum of 2^22 values   11.3 / 13.0 / 11.7               sum of 2^23          13.3 / 16.0 / 14.1
//                                                         ... 30 % starts      21.7 / 19.5 / 18.2
//   CSR SpMV, prepared, 3.9 M entries in blocks of 4   15.4 / 16.2 / 15.3;  3.5 M in blocks of 16   14.8 / 15.5 / 14.7
// (2^22 and 2^23 fill the rounds of seg_tile exactly; there, with few starts, one chunk per wave in seg_tile was 4 to 6 %
// ahead.)
constexpr int kShortRounds = 2;

template <typename TT, int kOp> constexpr bool stream_form() {
    return kOp == kSpmv || kOp == kSpmvCsr || (kOp == kSum && sizeof(typename TT::in_t) == 4);
}

constexpr int stream_waves_per_simd(int op, bool mfma, bool is_short = false) {
    return is_short ? 4 : op == kSum ? (mfma ? MMV_STREAM_WPS_SUM : MMV_STREAM_WPS_SUM_SHUFFLE) : MMV_STREAM_WPS_SPMV;
}

constexpr int kShortUnits = (int)kSpans * kShortRounds;   // most units of a tile of the form for short vectors
constexpr int kMaxUnits = (int)kSpans * MMV_STREAM_CPW;   // units of a tile: two per lane of a wave
static_assert(kMaxUnits <= 128, "the units of a tile are scanned by one wave, two per lane");

constexpr uint32_t kShortCounts = 3;   // 256 tiles each
static_assert(128 * stream_waves_per_simd(kSum, true) <= 256 * (int)kShortCounts && 128 * stream_waves_per_simd(kSum, false) <= 256 * (int)kShortCounts,
              "tiles of a short vector: one round of workgroups");

template <int kWaves> struct StreamShared {
    __attribute__((aligned(16))) uint32_t rows[kWaves][kUnitRows * kRowStride];
    // per unit: its aggregate and whether it holds a flag, its number of flags, and the one output that needs the sum
    // carried into the unit (its value so far, where it goes, whether there is one)
    __attribute__((aligned(8))) uint32_t unit_v[kMaxUnits], unit_f[kMaxUnits], unit_c[kMaxUnits];
    __attribute__((aligned(8))) uint32_t late_v[kMaxUnits], late_k[kMaxUnits], late_on[kMaxUnits];
    uint32_t tile, ready, arrived;
};

// What a wave holds of one unit while its loads are under way: lane (c, h) the flag word of row c + h, so that both
// halves of the wave can have the words of a row and of the one after it; values and columns striped (word i of lane l =
// elements 256 i + 4 l .. + 3).
template <bool kProduct> struct StreamSlot {
    uint32_t fw;
    v4u raw[4];
    v4u col[kProduct ? 4 : 1];
};
template <bool kProduct>
__device__ __forceinline__ void stream_load(const Params &P, uint64_t unit_base, int lane, StreamSlot<kProduct> &s) {
    const uint64_t rs = unit_base + 32u * ((uint32_t)(lane & 31) + (uint32_t)(lane >> 5));
    const bool full = unit_base + kUnitElems <= P.n;
    s.fw = 0;
    if (rs < P.n) s.fw = __builtin_nontemporal_load(P.fw + (rs >> 5));
    if constexpr (kProduct) {
#pragma unroll
        for (int i = 0; i < 4; ++i) s.col[i] = load128(P.col, unit_base + 256u * i + 4u * lane, P.n, full);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) s.raw[i] = load128((const float *)P.x, unit_base + 256u * i + 4u * lane, P.n, full);
}
// The same by buffer loads: a fixed number of them and no branch, so that the compiler knows how many are behind those that it waits
// for.  Of a unit behind the tile, or of what lies behind the end, nothing is read; columns there are 0.  Sums of 10^8 values, byte flags, 1 %
// starts 103.0 -> 99.5 us the call, 1.5 * 10^8, bits 121.5 -> 116.5; COO product of 3.4 * 10^7 entries in scattered columns, whose first
// gathers go out as their columns arrive, 242 -> 233.  COO products of up to 2.6 * 10^6 entries (kShort: loads of a second unit that
// may not be there) 14.8 -> 15.3, CSR products of 1.15 * 10^7 33.0 -> 33.8, 6.3 * 10^7 level: these keep the branches.
template <int kOp, bool kShort> constexpr bool buffered_loads() { return kOp == kSum || (kOp == kSpmv && !kShort); }
struct StreamArrays {
    __amdgpu_buffer_rsrc_t fw, x, col;
};
template <bool kProduct>
__device__ __forceinline__ void stream_load(const StreamArrays &A, int unit, int lane, StreamSlot<kProduct> &s) {
    s.fw = __builtin_amdgcn_raw_buffer_load_b32(A.fw, 4 * ((lane & 31) + (lane >> 5)) + 128 * unit, 0, kAuxNt);
    const int own = 16 * lane + 4 * kUnitElems * unit;
    if constexpr (kProduct) {
#pragma unroll
        for (int i = 0; i < 4; ++i) s.col[i] = __builtin_amdgcn_raw_buffer_load_b128(A.col, own + 1024 * i, 0, kAuxNt);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) s.raw[i] = __builtin_amdgcn_raw_buffer_load_b128(A.x, own + 1024 * i, 0, kAuxNt);
}

// kNarrow: x has at most 2^30 entries (loads that check their range: fewer, see x_bytes_of), so byte offsets into it fit 32 bits (one register per address, no 64-bit
// additions: SpMV with short rows 8 % faster, with scattered columns 2 %).
template <typename TT, int kOp, bool kMfma, bool kNarrow, bool kShort>
__device__ __forceinline__ void stream_tile(const Params &P, const uint32_t *__restrict__ hints, StreamShared<TT::kWaves> &sm,
                                            const uint32_t tile) {
    constexpr int kWaves = TT::kWaves;
    constexpr bool kProduct = kOp != kSum;
    constexpr bool kCounts = kOp != kSpmv;   // the index of an output is the ordinal of its segment
    constexpr int kDepth = kShort ? kShortRounds : kProduct ? MMV_STREAM_DEPTH_SPMV : MMV_STREAM_DEPTH_SUM;
    constexpr bool kBuffered = buffered_loads<kOp, kShort>();
    static_assert(kWaves == (int)kSpans, "units are dealt to eight waves");

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, h = lane >> 5;
    const uint64_t n = P.n;
    uint32_t *rows = sm.rows[wave];
    const TileSpan span = tile_span(P.reg, tile, kUnitElems);
    const int units = (int)span.cpw, rounds = (units + kWaves - 1) / kWaves;   // unit q = 8 u + wave of the tile in round u

    // Segment starts before each of my units: those before the tile, and those in the units of the tile before mine, from
    // its flag words, eight words per lane.  In a tile of up to 16 units every wave counts for itself; in a longer one
    // each wave counts its part (four threads per unit) and they exchange the counts through LDS.
    // Asked for ahead of the values (loads come back in the order they went out).
    const bool alone = kShort || units <= 16;
    const uint32_t part = alone ? (uint32_t)lane : (uint32_t)tid;   // which eight flag words of the tile I count
    // The first bits of words that do not count are cleared: those beyond n, and position 0, which opens segment 0 whatever
    // its flag says.
    uint32_t count_part = 0;
    v4u fl[2] = {}, tc[kShort ? kShortCounts : 1];
    const bool mine = part < 4u * (uint32_t)units;
    const uint64_t w0 = (span.base >> 5) + 8u * part, words = (n + 31) >> 5;
    auto clear_uncounted = [&] {
        if (kOp == kSum && tile == 0 && part == 0) fl[0][0] &= ~1u;   // (SpMV: a row starts there)
        if (!mine || w0 * 32 + 256u > n) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint64_t e0 = w0 * 32 + 32u * i;
                if (!mine || e0 >= n) fl[i / 4][i % 4] = 0;
                else if (e0 + 32 > n) fl[i / 4][i % 4] &= (1u << (uint32_t)(n - e0)) - 1u;
            }
        }
    };
    if constexpr (kCounts && kShort) {
        // no branch around these loads: what is loaded in a branch is waited for where it ends
        // (a lane with nothing to read reads the first words)
#pragma unroll
        for (uint32_t j = 0; j < kShortCounts; ++j) {
            const uint32_t e = 256u * j + 4u * lane;
            tc[j] = *reinterpret_cast<const v4u *>(P.tile_count + (e < tile ? e : 0u));
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) fl[i] = *reinterpret_cast<const v4u *>(P.fw + (mine && w0 + 4 * i < words ? w0 + 4 * i : 0));
    } else if constexpr (kCounts) {
        if (kOp == kSum || !P.tile_base) count_part = starts_before_part<false>(P, tile, 0, lane);
        if (mine) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (w0 + 4 * i < words) fl[i] = *reinterpret_cast<const v4u *>(P.fw + w0 + 4 * i);   // (the aligned block of the last word is read whole)
            clear_uncounted();
        }
    }
    // CSR: without empty rows (in the tile; in the matrix) the k-th segment is row k and the row map need not be read
    bool rows_dense = false, by_end = false;   // (by_end: the row map goes by the last position of a segment)
    uint32_t tile_base = 0;
    if constexpr (kOp == kSpmvCsr) {
        // (no branch around the load, for the same reason)
        tile_base = *(P.tile_base ? P.tile_base + tile : hints + (kHdrEmptyRows - kHdrHints));
        rows_dense = P.tile_base ? (tile_base & kPlanDense) != 0 : tile_base == 0;
        by_end = P.tile_base && (tile_base & kPlanByEnd) != 0;
        tile_base &= ~(kPlanDense | kPlanByEnd);
    }
    __builtin_amdgcn_sched_barrier(0);
    StreamSlot<kProduct> slot[kDepth];
    StreamArrays arrays;
    __amdgpu_buffer_rsrc_t xv;
    if constexpr (kBuffered) {
        // (the flag word behind the tile says whether its last position ends a segment; the 16-byte block of the last entry is read whole)
        const uint64_t left = n - span.base;
        const uint32_t tile_elems = (uint32_t)units * kUnitElems, entries = left < tile_elems ? (uint32_t)left : tile_elems;
        const uint32_t bytes = (4 * entries + 15) & ~15u;
        arrays.fw = make_rsrc(P.fw + (span.base >> 5), left > tile_elems ? tile_elems / 8 + 4 : (entries + 31) / 32 * 4);
        arrays.x = make_rsrc((const float *)P.x + span.base, bytes);
        if constexpr (kProduct) {
            arrays.col = make_rsrc(P.col + span.base, bytes);
            xv = make_rsrc(P.xv, P.x_bytes);
        }
#pragma unroll
        for (int i = 0; i < kDepth; ++i) stream_load<kProduct>(arrays, kWaves * i + wave, lane, slot[i]);
    } else {
#pragma unroll
        for (int i = 0; i < kDepth; ++i)
            if (kWaves * i + wave < units) stream_load<kProduct>(P, span.base + (uint64_t)(kWaves * i + wave) * kUnitElems, lane, slot[i]);
    }
#if MMV_LOAD_PRIO
    __builtin_amdgcn_s_setprio(0);
#endif
    if (lane < kUnitRows) rows[lane * kRowStride + kSlotZero] = 0;   // x-bar(-1) of every row; nothing overwrites it
    if (lane < MMV_STREAM_CPW) {             // my units
        const int q = kWaves * lane + wave;
        sm.late_on[q] = sm.unit_v[q] = sm.unit_f[q] = 0;
    }
    // starts of the tile: (alone) up to and with my eight words; else before the pair of units 2 lane, 2 lane + 1, and in
    // the first of them
    uint32_t count_carry = 0, starts_upto = 0, starts_even = 0, starts_all = 0;   // (starts_all: of the whole tile, in lane 63)
    if constexpr (kCounts && kShort) {
#pragma unroll
        for (uint32_t j = 0; j < kShortCounts; ++j)
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) count_part += 256u * j + 4u * lane + k < tile ? tc[j][k] : 0u;
        clear_uncounted();
    }
    if constexpr (kCounts) {
        count_carry = wave_sum<uint32_t, true>(count_part);
        // CSR: (the number of starts, or the first row) before the tile, minus 1: the index of the segment that is open there
        if constexpr (kOp == kSpmvCsr) count_carry = P.tile_base ? tile_base - 1u : tile == 0 ? ~0u : count_carry;
        uint32_t s = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) s += __popc(fl[i / 4][i % 4]);
        if (alone) {
            starts_all = starts_upto = wave_inclusive_scan(s);
        } else {
            s += dpp_or_zero<0x111, 0xF>(s);
            s += dpp_or_zero<0x112, 0xF>(s);
            if ((tid & 3) == 3 && tid / 4 < kMaxUnits) sm.unit_c[tid / 4] = s;
            __syncthreads();
            starts_even = 2 * lane < kMaxUnits ? sm.unit_c[2 * lane] : 0u;
            const uint32_t both = starts_even + (2 * lane < kMaxUnits ? sm.unit_c[2 * lane + 1] : 0u);
            starts_all = wave_inclusive_scan(both);
            starts_upto = starts_all - both;
        }
        if (kOp == kSum && !P.count_is_prefix && tile == P.num_tiles - 1 && wave == 0) {   // (else an earlier kernel has written it)
            if (lane == 63) *P.nseg = (uint64_t)count_carry + starts_all + 1u;
        }
    }

    // where the sum of a segment goes: the k-th, whose last element is e of unit q
    auto output_index = [&](uint32_t k, const int32_t *row, uint32_t e, uint32_t q) -> uint32_t {
        if constexpr (kOp == kSpmv) return (uint32_t)row[e];
        else if constexpr (kOp == kSpmvCsr) return rows_dense ? k : P.rowmap[by_end ? tile_base + kUnitElems * q + e : k];
        else return k;
    };
    auto emit = [&](uint32_t at, float v) {
        if constexpr (kOp == kSum) ((float *)P.out)[at] = v;
        else P.y[at] = v;
    };

    if constexpr (kShort) {   // (so that no wait for the second unit stands behind the stores of the first)
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll 1
    for (int u0 = 0; u0 < (kShort ? 1 : rounds); u0 += kDepth) {
#pragma unroll
        for (int i = 0; i < kDepth; ++i) {
            const int u = u0 + i;
            const int q = kWaves * u + wave;
            const uint64_t ub = span.base + (uint64_t)q * kUnitElems;
            if (q < units && ub < n) {
                const bool full = ub + kUnitElems <= n;
                v4u(&raw)[4] = slot[i].raw;
                if constexpr (kProduct) {   // product vector p(i) = val(i) * x(col(i))
                    constexpr int kBatch = kNarrow ? 4 : 1;   // words of columns whose gathers are under way together (64-bit addresses: one, or the registers do not suffice)
                    float xg[kBatch][4];
#pragma unroll
                    for (int j0 = 0; j0 < 4; j0 += kBatch) {
#pragma unroll
                        for (int j = 0; j < kBatch; ++j)
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                // (buffered: columns of what lies behind the end, in the block of the last entry, may be anything; such a
                                // gather reads nothing where it would leave x, or x[0].  Else they were loaded as 0.)
                                const uint32_t at = slot[i].col[j0 + j][k];
                                if constexpr (kBuffered && kNarrow) xg[j][k] = from_bits<float>(__builtin_amdgcn_raw_buffer_load_b32(xv, (int)(at << 2), 0, 0));
                                else if constexpr (kBuffered) xg[j][k] = P.xv[full || ub + 256u * (j0 + j) + 4u * lane + k < n ? at : 0u];
                                else if constexpr (kNarrow) xg[j][k] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(P.xv) + (at << 2));
                                else xg[j][k] = P.xv[at];
                            }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int j = 0; j < kBatch; ++j)
#pragma unroll
                            for (int k = 0; k < 4; ++k) raw[j0 + j][k] = to_bits(from_bits<float>(raw[j0 + j][k]) * xg[j][k]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if (!full) {   // (SpMV: x[0] may be infinite)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (ub + 256u * j + 4u * lane + k >= n) raw[j][k] = 0;
                }
                const Halves w = wave_halves<true>(slot[i].fw, lane);
                uint32_t F = w.lo;                                    // flag word of row c (both halves of the wave)
                uint32_t E = (F >> 1) | (w.hi << 31);                 // bit p: position p + 1 starts a segment, or p is the last
                if (ub == 0 && c == 0) F |= 1u;                       // position 0 starts a segment whatever its flag says
                if (!full || ub + kUnitElems == n) {                  // bits beyond n do not count; element n - 1 ends a segment
                    const uint64_t row_start = ub + 32u * c;
                    if (row_start + 32 > n) F = row_start < n ? (F & ((1u << (uint32_t)(n - row_start)) - 1u)) : 0u;
                    if (row_start >= n) {
                        E = 0;
                    } else if (row_start + 32 >= n) {
                        const uint32_t last = (uint32_t)(n - 1 - row_start);
                        E = (E & ((1u << last) - 1u)) | (1u << last);
                    }
                }
                if (__ballot(E != 0) == 0) {
                    // no segment ends here (one may begin, at the first position): a plain sum
                    float s = 0.0f;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        s += (from_bits<float>(raw[j][0]) + from_bits<float>(raw[j][1])) + (from_bits<float>(raw[j][2]) + from_bits<float>(raw[j][3]));
                    s = wave_sum<float, true>(s);
                    if (lane == 0) {
                        sm.unit_v[q] = to_bits(s);
                        sm.unit_f[q] = F & 1u;
                    }
                } else {
                    // ---- step 1: speculative row scans into the wave's LDS rows ----
                    if constexpr (kMfma) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            *reinterpret_cast<v4u *>(rows + (8 * j + (lane >> 3)) * kRowStride + kRowData + 4 * (lane & 7)) = raw[j];
                        wave_lds_sync();
                        v4u op[4];   // operand layout: positions 16 h + 4 q .. + 3 of row c
#pragma unroll
                        for (int j = 0; j < 4; ++j) op[j] = *reinterpret_cast<const v4u *>(rows + c * kRowStride + kRowData + 16 * h + 4 * j);
                        wave_lds_sync();
                        // (COO: the 0 / 1 operand of the products is made anew for every unit; kept around the loop it makes
                        // one register spill, and its reload waits behind the loads under way)
                        int lane_here = lane;
                        if constexpr (kOp == kSpmv) asm volatile("" : "+v"(lane_here));
                        float acc[16];
                        SpecMfma<TF32>::run(op, lane_here, acc);
                        store_spec_rows(rows, 0, lane, acc);
                    } else {
                        spec_shuffle_tile<TF32, true>(raw, lane, rows, 0);
                    }
                    wave_lds_sync();
                    // ---- steps 2 to 4 for the aggregate of row c (both halves of the wave alike) ----
                    const uint32_t *rp = rows + c * kRowStride + kRowData;
                    const float agg = from_bits<float>(rp[31]) - from_bits<float>(rp[last_flag_pos(F) - 1]);
                    // ---- step 5a: segmented inclusive scan over the 32 rows, and the number of flags up to each ----
                    const uint32_t cnt = __popc(F);
                    float inc_v = agg;
                    uint32_t inc_c = cnt;
#define MMV_SCAN_STEP(CTRL, ROWS)                                                                   \
                    {                                                                               \
                        const float ov = from_bits<float>(dpp_or_zero<CTRL, ROWS>(to_bits(inc_v))); \
                        const uint32_t oc = dpp_or_zero<CTRL, ROWS>(inc_c);                         \
                        if (!inc_c) inc_v = ov + inc_v;                                             \
                        inc_c += oc;                                                                \
                    }
                    MMV_SCAN_STEP(0x111, 0xF)
                    MMV_SCAN_STEP(0x112, 0xF)
                    MMV_SCAN_STEP(0x114, 0xF)
                    MMV_SCAN_STEP(0x118, 0xF)
                    MMV_SCAN_STEP(0x142, 0xA)
#undef MMV_SCAN_STEP
                    const uint32_t ex_c = inc_c - cnt;                                        // flags in the rows before mine
                    float ex_v = from_bits<float>(dpp_or_zero<0x138, 0xF>(to_bits(inc_v)));   // wave_shr 1: carry into row c
                    if (c == 0) ex_v = 0.0f;
                    // segment starts before row c (the one at position 0 is not counted)
                    uint32_t count_base = count_carry + ex_c;
                    if constexpr (kCounts) {
                        if (!alone) {
                            count_base += (uint32_t)__builtin_amdgcn_readlane((int)starts_upto, q >> 1);
                            if (q & 1) count_base += (uint32_t)__builtin_amdgcn_readlane((int)starts_even, q >> 1);
                        } else if (q > 0) {
                            count_base += (uint32_t)__builtin_amdgcn_readlane((int)starts_upto, 4 * q - 1);
                        }
                        if (kOp == kSum && ub == 0) count_base -= 1u;   // position 0 is a flag in F, but counted nowhere else
                    }
                    // ---- steps 2 and 6 at the segment ends: half h of the wave takes the ends in its half of the rows ----
                    uint32_t Eh = E & (h ? 0xFFFF0000u : 0x0000FFFFu);
                    const int32_t *row = kOp == kSpmv ? P.row + ub : nullptr;   // (uniform)
                    while (Eh) {
                        const int e = __builtin_ctz(Eh);
                        Eh &= Eh - 1u;
                        const uint32_t m = F & ((2u << e) - 1u);               // flags at or before the end
                        float v = from_bits<float>(rp[e]) - from_bits<float>(rp[last_flag_pos(m) - 1]);   // REVSPEC: x-bar(e) - x-bar(start - 1)
                        if (!m) v += ex_v;                                     // the segment began before this row
                        const uint32_t k = count_base + __popc(m);
                        const bool kept = kOp == kSpmv || k < P.out_cap;
                        if (!m && ex_c == 0) {                                 // ... before this unit: at most one end
                            sm.late_v[q] = to_bits(v);
                            sm.late_k[q] = kept ? output_index(k, row, 32u * c + e, (uint32_t)q) : 0u;
                            sm.late_on[q] = kept ? 1u : 0u;
                        } else if (kept) {
                            emit(output_index(k, row, 32u * c + e, (uint32_t)q), v);
                        }
                    }
                    if (lane == 31) {
                        sm.unit_v[q] = to_bits(inc_v);
                        sm.unit_f[q] = inc_c;
                    }
                    wave_lds_sync();   // the rows are read before the next unit overwrites them
                }
            }
            if constexpr (kShort) continue;
            // the registers of this unit take the one that many rounds ahead
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (kBuffered && !kProduct) stream_load<kProduct>(arrays, q + kWaves * kDepth, lane, slot[i]);
            else if (q + kWaves * kDepth >= units) slot[i] = StreamSlot<kProduct>{};   // (or the compiler keeps the old columns in registers all the way through)
            else if constexpr (kBuffered) stream_load<kProduct>(arrays, q + kWaves * kDepth, lane, slot[i]);
            else stream_load<kProduct>(P, span.base + (uint64_t)(kWaves * (u + kDepth) + wave) * kUnitElems, lane, slot[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();
    if (wave != 0) return;

    // ---- step 5b: the units of the tile, two per lane: segmented scan of their aggregates ----
    float v[2] = {0.0f, 0.0f};
    uint32_t f[2] = {0, 0}, on[2] = {0, 0}, at[2] = {0, 0};
    float late[2] = {0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (2 * lane + i < kMaxUnits) {
            v[i] = from_bits<float>(sm.unit_v[2 * lane + i]);
            f[i] = sm.unit_f[2 * lane + i];
            on[i] = sm.late_on[2 * lane + i];
            late[i] = from_bits<float>(sm.late_v[2 * lane + i]);
            at[i] = sm.late_k[2 * lane + i];
        }
    float inc_v = f[1] ? v[1] : v[0] + v[1];
    uint32_t inc_f = f[0] | f[1];
#define MMV_SCAN_STEP(CTRL, ROWS)                                                               \
    {                                                                                           \
        const float ov = from_bits<float>(dpp_or_zero<CTRL, ROWS>(to_bits(inc_v)));             \
        const uint32_t of = dpp_or_zero<CTRL, ROWS>(inc_f);                                     \
        if (!inc_f) inc_v = ov + inc_v;                                                         \
        inc_f |= of;                                                                            \
    }
    MMV_SCAN_STEP(0x111, 0xF)
    MMV_SCAN_STEP(0x112, 0xF)
    MMV_SCAN_STEP(0x114, 0xF)
    MMV_SCAN_STEP(0x118, 0xF)
    MMV_SCAN_STEP(0x142, 0xA)
    MMV_SCAN_STEP(0x143, 0xC)
#undef MMV_SCAN_STEP
    float ex_v = from_bits<float>(dpp_or_zero<0x138, 0xF>(to_bits(inc_v)));   // wave_shr 1: lane 0 gets 0
    const uint32_t ex_f = dpp_or_zero<0x138, 0xF>(inc_f);
    const float tagg_v = from_bits<float>((uint32_t)__builtin_amdgcn_readlane((int)to_bits(inc_v), 63));
    const uint32_t tagg_f = (uint32_t)__builtin_amdgcn_readlane((int)inc_f, 63);
    // ---- step 5c: publish the tile, look back for the carry of the tiles before it ----
    const bool final_now = tile == 0 || tagg_f;  // carry out does not depend on predecessors
    if (lane == 0) desc_store(P.desc_v + tile, final_now ? kStatusPrefix : kStatusAggregate, to_bits(tagg_v));
    float tile_carry = 0.0f;
    // (a tile whose carry goes out as it is and whose first open end is none needs no carry in)
    const bool wanted = __ballot((on[0] && !ex_f) || (on[1] && !(ex_f | f[0]))) != 0;
    if (tile > 0 && (wanted || !final_now)) tile_carry = lookback<float, true>(P.desc_v, (int)tile, lane, poll_lanes(P.num_tiles, P.first_round), P.hdr);
    if (lane == 0 && !final_now) desc_store(P.desc_v + tile, kStatusPrefix, to_bits(tile_carry + tagg_v));
    // ---- step 6 for the outputs that were waiting ----
    if (!ex_f) ex_v += tile_carry;
    if (on[0]) emit(at[0], late[0] + ex_v);
    if (on[1]) emit(at[1], late[1] + (f[0] ? v[0] : ex_v + v[0]));
}

}  // namespace
