// libmmvseg, part of the one translation unit mmvseg.hip (included there, in order).
// The single-pass kernel for 8- and 16-bit values: segmented scan, the unsegmented scan, and the segmented sum of vectors of one round of
// workgroups.
#pragma once

namespace {

// ---- the kernel ---------------------------------------------------------------------------------------
//
// One workgroup = one tile = kWaves waves x kCpw chunks x 2048 elements, taken from
// an atomic ticket counter (a tile only ever waits for tiles held by workgroups that
// are already running).  A same-address device-scope atomic costs about 11 ns on
// this chip and they serialise, which is why a ticket covers tens of thousands of
// elements.  Every wave owns a contiguous span of the tile and
//   A. loads all its inputs at once, then for each chunk computes the speculative
//      row scans (matrix cores), the row aggregates and their segmented scan; only
//      a few registers per chunk are kept, the row scans themselves are dropped;
//   -  the wave aggregates are combined and the tile's descriptor is published;
//   B. recomputes the row scans of each chunk from the raw registers (cheaper than
//      holding them: LDS is the scarce resource), reverts the mis-speculation, adds
//      the carries and stores.  Chunks that start after a flag of the tile go first;
//      chunks that continue a segment of an earlier tile go last, after wave 0 has
//      looked back for the carry of the predecessor tiles.
// The chunk loops of the scan kernels are rolled: the per-chunk registers are rotated so that
// the loop body always works on the first slots (unrolled, these kernels spill).

template <typename T, int N> __device__ __forceinline__ void rotate(T (&a)[N]) {
    const T first = a[0];
#pragma unroll
    for (int i = 0; i + 1 < N; ++i) a[i] = a[i + 1];
    a[N - 1] = first;
}
template <int N, int M> __device__ __forceinline__ void rotate_rows(v4u (&a)[N][M]) {
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const v4u first = a[0][m];
#pragma unroll
        for (int i = 0; i + 1 < N; ++i) a[i][m] = a[i + 1][m];
        a[N - 1][m] = first;
    }
}

// LDS of one workgroup: the row buffers of the waves and the words the waves exchange.
template <int kWaves, int kRows> struct SegShared {
    __attribute__((aligned(16))) uint32_t rows[kWaves][kRows * kRowStride];
    uint32_t wave_v[kWaves], wave_f[kWaves], wave_c[kWaves];
    uint32_t early_v[kWaves], early_f[kWaves];   // plain sum and any-flag of every wave's span, written as the loads land
    uint32_t tile, carry_v, carry_c, ready, arrived;
};

// Descriptors that a look-back takes at a time (lookback in lanes.h).  Tiles of bytes hold four times the elements of fp32 ones, so fewer
// of them are in flight and ask for the same lines: without flags, windows of 64 -> 16: 5 * 10^7 bytes 50.6 -> 52.3 us, segmented 52.3 -> 54.9, 10^8
// 90.5 -> 90.6, 2^28 224.8 -> 223.0.  16-bit values, 64 / 32 / 16: segmented, 10^8 115.3 / 111.7 / 111.8, mmv_scan 3 * 10^7 39.1 / 39.6 / 40.4
// (windows of 64 read whole, as before, against these of 32, timed in turn: mmv_scan of 3 * 10^7 fp16 values 38.7 / 38.8, 10^8 111.0 / 108.2, 2^28 285.6 / 279.0).
template <typename TT> __device__ __forceinline__ int seg_poll_lanes(const Params &P) {
    return TT::kOneRound || sizeof(typename TT::in_t) == 1 || P.num_tiles <= P.first_round ? 64 : 32;
}

// One tile, from the loads on.
// In the one-round form LDS holds one 32x32 tile of a wave at a time, half a chunk (37 instead of 74 KB per workgroup).
template <typename TT> constexpr int lds_rows() { return TT::kOneRound ? kS : kRowsPerChunk; }
template <typename TT, int kOp, bool kMfma>
__device__ __forceinline__ void seg_tile(const Params &P, SegShared<TT::kWaves, lds_rows<TT>()> &sm, const uint32_t tile) {
    typedef typename TT::base_t BT;
    typedef typename TT::acc_t A;
    typedef typename TT::in_t In;
    constexpr int kWaves = TT::kWaves;
    constexpr int kCpw = chunks_per_wave<TT, kOp, kMfma>();   // most chunks a wave takes (register arrays)
    constexpr int K = 16 / TT::kEpl;             // 128-bit words per lane and 32x32 tile
    constexpr bool kScanLike = kOp == kScan || kOp == kPlainScan;   // every element is an output
    // The chunk loops are either rolled, with the per-chunk registers rotated so that the body always
    // works on the first slot(s) (about 45 moves per rotation and phase, small code), or unrolled.  Unrolled, the
    // scan kernels spill registers (measured: 100 to 700 bytes per lane) and so does the shuffle-only
    // int8 sum kernel with its four chunks; the other sum kernels do not.
    constexpr bool kUnrollChunks = MMV_UNROLL_CHUNKS != 0 && !kScanLike && (kMfma || kCpw <= 2);
    // chunks per iteration of the chunk loops: all (unrolled), or MMV_ROLL_STEP with the registers
    // rotated by as many slots afterwards (the moves of a rotation do not depend on the distance)
    constexpr int kStep = kUnrollChunks ? kCpw : (kCpw >= 2 * MMV_ROLL_STEP && kCpw % MMV_ROLL_STEP == 0 ? MMV_ROLL_STEP : 1);
    constexpr bool kHalf = lds_rows<TT>() == kS;   // LDS holds the rows of one 32x32 tile
    // lane exchanges through the vector ALU for the sum-type kernels and the 16-bit scans (measured 2 %
    // faster), through the LDS hardware for the int8 scans (0.9 % faster)
    constexpr bool kAluLanes = MMV_DPP_SCAN != 0 && (!kScanLike || TT::kEpl == 8);
    constexpr bool kCounts = kOp == kSum;        // output index = segment ordinal
    // (the count of the segments before the tile comes from tables made by a
    // small kernel before this one, so that no chunk has to wait for it)
    // A tile that holds no flag hands on a plain sum, and its successors cannot finish before they have it.  In the
    // scan kernels such a tile publishes that sum as soon as its loads have landed, ahead of the row scans of
    // phase A (which take several microseconds when all waves of a compute unit are at it): the wave whose loads
    // land last adds up the sums of all waves.  Without this a vector without flags ran 13 % slower than one
    // with a flag in every tile, each tile waiting 6 us for the slowest of the tiles before it.
    // That wave also asks for the descriptors of the tiles before at the end of its phase A and looks at them after the
    // barrier: the look-back takes 3 to 4 us whoever has published what, so it pays to have the poll under way early (looking
    // back at once makes the wave late for the barrier).
    constexpr bool kEarly = kScanLike;

    // the wave index as a scalar: everything derived from it (the wave's span, chunk bases, the
    // "whole chunk inside the vector" tests, base addresses of loads and stores) then lives in scalar
    // registers and costs no vector instructions
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint64_t n = P.n;
    uint32_t *rows = sm.rows[wave];
    // tiles at both ends of a long vector are shorter (fewer chunks per wave)
    const TileSpan span = tile_span(P.reg, tile, kWaves * kChunkElems);
    const int cpw_t = (int)span.cpw;
    const uint64_t tile_base = span.base;
    const uint64_t wave_base = tile_base + (uint64_t)wave * cpw_t * kChunkElems;

    // ---- all inputs of my span: flag word of my row and raw values per chunk ----
    uint32_t F[kCpw];
    v4u raw[kCpw][2 * K];
    // (the flag words go first: a wave knows whether its span holds a flag before the values have landed)
#pragma unroll
    for (int c = 0; c < kCpw; ++c) {
        F[c] = 0;
        if constexpr (kOp != kPlainScan) {
            const uint64_t rs = wave_base + (uint64_t)c * kChunkElems + 32u * lane;
            if (c < cpw_t && rs < n) F[c] = __builtin_nontemporal_load(P.fw + (rs >> 5));
        }
    }
#pragma unroll
    for (int c = 0; c < kCpw; ++c) {
        const uint64_t cb = wave_base + (uint64_t)c * kChunkElems;
        if (c < cpw_t) load_raw<BT, kMfma>((const In *)P.x, cb, n, lane, raw[c]);
    }

#if MMV_LOAD_PRIO
    __builtin_amdgcn_s_setprio(0);
#endif
    if constexpr (kOp == kPlainScan && sizeof(In) == 1) {
        // counting segment starts: position 0 always opens a segment (byte 0 of the first word, both layouts)
        if (P.first_one && tile == 0 && tid == 0) raw[0][0][0] = (raw[0][0][0] & ~0xFFu) | 1u;
    }
    // bits beyond n do not count
    if constexpr (kOp != kPlainScan) {
#pragma unroll
        for (int c = 0; c < kCpw; ++c) {
            const uint64_t rs = wave_base + (uint64_t)c * kChunkElems + 32u * lane;
            if (rs + 32 > n) F[c] = rs < n ? (F[c] & ((1u << (uint32_t)(n - rs)) - 1u)) : 0u;
        }
    }
    bool i_published = false;   // (kEarly) my wave has published the sum of a tile without flags
    if constexpr (kEarly) {
        uint32_t any = 0;
#pragma unroll
        for (int c = 0; c < kCpw; ++c) any |= F[c];
        if (tile == 0) any |= 1u;                       // nobody waits for the first tile's sum ahead of time
        const bool span_flagged = __ballot(any != 0) != 0;
        A s = A(0);
        if (!span_flagged) {
#pragma unroll
            for (int c = 0; c < kCpw; ++c)
                if (c < cpw_t) s += RawSum<BT>::run(raw[c]);
            s = wave_sum<A, kAluLanes>(s);
        }
        uint32_t before = 0;
        if (lane == 0) {
            sm.early_v[wave] = to_bits(s);
            sm.early_f[wave] = span_flagged ? 1u : 0u;
            before = __hip_atomic_fetch_add(&sm.arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (__builtin_amdgcn_readfirstlane(before) == kWaves - 1) {   // my wave's loads landed last
            A total = A(0);
            uint32_t flagged = 0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                total += from_bits<A>(sm.early_v[w]);
                flagged |= sm.early_f[w];
            }
            if (!flagged) {
                i_published = true;
                if (lane == 0) desc_store(P.desc_v + tile, kStatusAggregate, to_bits(total));
            }
        }
    }

    if constexpr (kCounts) {
        // number of segment starts before my tile, while the loads are in flight
        static_assert(kWaves == (int)kSpans, "one span per wave");
        if (wave == 1) {
            const uint32_t c = wave_sum<uint32_t, kAluLanes>(starts_before_part<true>(P, tile, 0, lane));
            if (lane == 0) sm.carry_c = c;
        }
    }

    // per chunk: exclusive segmented prefix of my row inside the chunk, and of the chunk inside
    // my span; run_* = running aggregate of the span
    A ex_v[kCpw], pre_v[kCpw];
    uint32_t ex_f[kCpw], pre_f[kCpw], ex_c[kCpw];
#pragma unroll
    for (int c = 0; c < kCpw; ++c) {
        ex_v[c] = pre_v[c] = A(0);
        ex_f[c] = pre_f[c] = ex_c[c] = 0;
    }
    A run_v = A(0);
    uint32_t run_f = 0, run_c = 0;

    // ================= phase A: aggregates =================
#pragma unroll 1
    for (int c0 = 0; c0 < kCpw; c0 += kStep) {
#pragma unroll
     for (int u = 0; u < kStep; ++u) {
      const int c = c0 + u;
      const int S = kUnrollChunks ? c : u;   // register slot of this chunk
      if (c < cpw_t) {
        const uint64_t cb = wave_base + (uint64_t)c * kChunkElems;
        const uint64_t row_start = cb + 32u * lane;  // first element of the row this lane owns
        // ---- steps 1-4 for the aggregate of my row: last element after the revert, any flag ----
        const uint32_t has_flag = F[S] != 0;
        A agg_v;
        if constexpr (kMfma) {
            static_assert(K == 1 || !kHalf, "a whole chunk passes through LDS on its way into the operand layout");
            if constexpr (K > 1) to_operand_layout<K>(raw[S], rows, lane);
            agg_v = RowAgg<BT>::template run<kAluLanes>(raw[S], F[S], lane);
        } else if constexpr (kHalf) {
            agg_v = A(0);
#pragma unroll
            for (int t = 0; t < 2; ++t) {   // (the lanes of half t own the rows of tile t)
                uint32_t *rp = rows + (lane & 31) * kRowStride;
                spec_shuffle_tile<BT, kAluLanes>(raw[S] + t * K, lane, rows, 0);
                if ((lane >> 5) == t) rp[kSlotZero] = 0;
                wave_lds_sync();
                if ((lane >> 5) == t) agg_v = from_bits<A>(rp[kRowData + 31]) - from_bits<A>(rp[kSlotZero + last_flag_pos(F[S])]);
                wave_lds_sync();
            }
        } else {
#pragma unroll
            for (int t = 0; t < 2; ++t) spec_shuffle_tile<BT, kAluLanes>(raw[S] + t * K, lane, rows, t);
            rows[lane * kRowStride + kSlotZero] = 0;
            wave_lds_sync();
            const A last = from_bits<A>(rows[lane * kRowStride + kRowData + 31]);
            const int slot = kSlotZero + last_flag_pos(F[S]);  // x-bar(start - 1)
            agg_v = last - from_bits<A>(rows[lane * kRowStride + slot]);
            wave_lds_sync();  // the rows are read before the next chunk overwrites them
        }
        // segment starts in my row, position 0 of the whole vector not counted (sum only)
        const uint32_t cnt = __popc(row_start == 0 ? (F[S] & ~1u) : F[S]);

        // ---- step 5a: segmented inclusive scan of (value, flag) over the 64 rows of the chunk ----
        A inc_v = agg_v;
        uint32_t inc_f = has_flag;
        uint32_t inc_c = cnt;
      if constexpr (kAluLanes) {
        // Kogge-Stone inside the rows of 16 lanes (row_shr 1, 2, 4, 8), then the total of a row of lanes
        // to the next one (row_bcast 15 into lane rows 1 and 3) and of the first 32 lanes to the last 32
        // (row_bcast 31 into lane rows 2 and 3).  A lane without a source gets (0, no flag, 0).
#define MMV_SCAN_STEP(CTRL, ROWS)                                                                  \
        {                                                                                          \
            const A ov = from_bits<A>(dpp_or_zero<CTRL, ROWS>(to_bits(inc_v)));                    \
            const uint32_t of = dpp_or_zero<CTRL, ROWS>(inc_f);                                    \
            if (kCounts) inc_c += dpp_or_zero<CTRL, ROWS>(inc_c);                                  \
            if (!inc_f) inc_v = ov + inc_v;                                                        \
            inc_f |= of;                                                                           \
        }
        MMV_SCAN_STEP(0x111, 0xF)
        MMV_SCAN_STEP(0x112, 0xF)
        MMV_SCAN_STEP(0x114, 0xF)
        MMV_SCAN_STEP(0x118, 0xF)
        MMV_SCAN_STEP(0x142, 0xA)
        MMV_SCAN_STEP(0x143, 0xC)
#undef MMV_SCAN_STEP
        ex_v[S] = from_bits<A>(dpp_or_zero<0x138, 0xF>(to_bits(inc_v)));   // wave_shr 1: lane 0 gets 0
        ex_f[S] = dpp_or_zero<0x138, 0xF>(inc_f);
        ex_c[S] = run_c + inc_c - cnt;
        pre_v[S] = run_v;
        pre_f[S] = run_f;
        // chunk aggregate = inclusive value of the last row; fold it into the span's running aggregate
        const A ca_v = from_bits<A>((uint32_t)__builtin_amdgcn_readlane((int)to_bits(inc_v), 63));
        const uint32_t ca_f = (uint32_t)__builtin_amdgcn_readlane((int)inc_f, 63);
        run_v = ca_f ? ca_v : run_v + ca_v;
        run_f |= ca_f;
        if (kCounts) run_c += (uint32_t)__builtin_amdgcn_readlane((int)inc_c, 63);
      } else {
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const A ov = from_bits<A>(__shfl_up(to_bits(inc_v), d));
            const uint32_t of = __shfl_up(inc_f, d);
            if (lane >= d) {
                if (!inc_f) inc_v = ov + inc_v;
                inc_f |= of;
            }
            if (kCounts) {
                const uint32_t oc = __shfl_up(inc_c, d);
                if (lane >= d) inc_c += oc;
            }
        }
        ex_v[S] = from_bits<A>(__shfl_up(to_bits(inc_v), 1));
        ex_f[S] = __shfl_up(inc_f, 1);
        if (lane == 0) {
            ex_v[S] = A(0);
            ex_f[S] = 0;
        }
        ex_c[S] = run_c + inc_c - cnt;
        pre_v[S] = run_v;
        pre_f[S] = run_f;
        // chunk aggregate = inclusive value of the last row; fold it into the span's running aggregate
        const A ca_v = from_bits<A>(__shfl(to_bits(inc_v), 63));
        const uint32_t ca_f = __shfl(inc_f, 63);
        run_v = ca_f ? ca_v : run_v + ca_v;
        run_f |= ca_f;
        if (kCounts) run_c += __shfl(inc_c, 63);
      }
      }
     }
        if constexpr (!kUnrollChunks) {
#pragma unroll
            for (int r = 0; r < kStep; ++r) {
                rotate(F);
                rotate_rows(raw);
                rotate(ex_v);
                rotate(ex_f);
                rotate(pre_v);
                rotate(pre_f);
                if (kCounts) rotate(ex_c);
            }
        }
    }
    // (wave 0) the tile's first element starts a segment: nothing of the tile takes a carry from the tiles before
    // (after the loop the register slots are back in place: slot 0 is the wave's first chunk)
    const bool head_flagged = (__builtin_amdgcn_readfirstlane(F[0]) & 1u) != 0;
    if (lane == 0) {
        sm.wave_v[wave] = to_bits(run_v);
        sm.wave_f[wave] = run_f;
        sm.wave_c[wave] = run_c;
    }
    uint64_t polled = 0;
    if constexpr (kEarly) {
        if (i_published) polled = lookback_poll(P.desc_v, (int)tile, lane, seg_poll_lanes<TT>(P));
    }
    __syncthreads();

    // ---- step 5b: waves of the tile ----
    A wex_v = A(0);
    uint32_t wex_f = 0, wex_c = 0;
    A tagg_v = A(0);
    uint32_t tagg_f = 0, tagg_c = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        if (w == wave) {
            wex_v = tagg_v;
            wex_f = tagg_f;
            wex_c = tagg_c;
        }
        const A wv = from_bits<A>(sm.wave_v[w]);
        const uint32_t wf = sm.wave_f[w];
        tagg_v = wf ? wv : tagg_v + wv;
        tagg_f |= wf;
        tagg_c += sm.wave_c[w];
    }
    wex_f = __builtin_amdgcn_readfirstlane(wex_f);

    if constexpr (kCounts) {
        if (!P.count_is_prefix && tile == P.num_tiles - 1 && tid == 0) *P.nseg = (uint64_t)sm.carry_c + tagg_c + 1u;
    }

    // ---- step 5c, first half: publish this tile ----
    const bool final_now = tile == 0 || tagg_f;  // carry out does not depend on predecessors
    // (a tile without any flag, other than tile 0, has published its aggregate already where kEarly is set)
    if (tid == 0 && (!kEarly || final_now))
        desc_store(P.desc_v + tile, final_now ? kStatusPrefix : kStatusAggregate, to_bits(tagg_v));

    // carry into my span (used only by rows with no flag before them in the tile); the carry of
    // the predecessor tiles is added once it is known
    A span_carry = wex_v;
    uint32_t count_carry = 0;
    if constexpr (kCounts) count_carry = sm.carry_c;

    // ================= phase B: recompute, revert, add carries, store =================
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
        if (pass == 1) {
            // ---- step 5c, second half: carry of the predecessor tiles by decoupled look-back ----
            A tile_carry = A(0);
            // (a tile without flags, other than tile 0, has looked back already where kEarly is set)
            const bool looked_back = kEarly && !final_now;
            if constexpr (kEarly) {
                if (i_published) {
                    tile_carry = lookback<A, kAluLanes, true>(P.desc_v, (int)tile, lane, seg_poll_lanes<TT>(P), P.hdr, polled);
                    if (lane == 0) {
                        desc_store(P.desc_v + tile, kStatusPrefix, to_bits(tile_carry + tagg_v));
                        sm.carry_v = to_bits(tile_carry);
                        __hip_atomic_store(&sm.ready, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
            }
            if (wave == 0 && !looked_back) {
                if (tile > 0 && !head_flagged) tile_carry = lookback<A, kAluLanes>(P.desc_v, (int)tile, lane, seg_poll_lanes<TT>(P), P.hdr);
                if (lane == 0) {
                    if (!final_now) desc_store(P.desc_v + tile, kStatusPrefix, to_bits(tile_carry + tagg_v));
                    sm.carry_v = to_bits(tile_carry);
                    __hip_atomic_store(&sm.ready, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            if ((wave != 0 || looked_back) && !wex_f) {
                // my span starts inside a segment that began in an earlier tile: wait for wave 0
                while (__hip_atomic_load(&sm.ready, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) == 0)
                    __builtin_amdgcn_s_sleep(1);
                tile_carry = from_bits<A>(sm.carry_v);
            }
            if (!wex_f) span_carry = tile_carry + wex_v;
        }
#pragma unroll 1
        for (int c0 = 0; c0 < kCpw; c0 += kStep) {
#pragma unroll
          for (int u = 0; u < kStep; ++u) {
            const int c = c0 + u;
            const int S = kUnrollChunks ? c : u;
            // a chunk is "open" when no flag of the tile precedes it
            const bool chunk_open = !(wex_f || __builtin_amdgcn_readfirstlane(pre_f[S]));
            if (c < cpw_t && chunk_open == (pass == 1)) {
                const uint64_t cb = wave_base + (uint64_t)c * kChunkElems;
                const bool chunk_full = cb + kChunkElems <= n;
                const uint64_t row_start = cb + 32u * lane;
                // sum: end mask of my row, bit p set iff position p + 1 starts a segment or p is
                // the last element; a 32x32 tile none of whose rows holds a segment end needs no x-bar
                uint32_t E = 0;
                uint64_t rows_with_ends = ~0ull;
                if constexpr (!kScanLike) {
                    uint32_t next0 = dpp_or_zero<0x130, 0xF>(F[S]) & 1u;   // wave_shl 1: the word of the next row
                    if (lane == 63) {
                        const uint64_t en = cb + kChunkElems;
                        next0 = 0;
                        if (en < n) next0 = P.fw[en >> 5] & 1u;
                    }
                    E = (F[S] >> 1) | (next0 << 31);
                    if (row_start < n) {
                        if (row_start + 32 >= n) {
                            const uint32_t last = (uint32_t)(n - 1 - row_start);
                            E = (E & ((1u << last) - 1u)) | (1u << last);
                        }
                    } else {
                        E = 0;
                    }
                    rows_with_ends = __ballot(E != 0);
                }
                auto make_rows = [&](int t, int at) {   // the row scans of tile t into the LDS rows of tile `at`
                    if (kMfma) {
                        A acc[16];
                        SpecMfma<BT>::run(raw[S] + t * K, lane, acc);
                        store_spec_rows(rows, at, lane, acc);
                    } else {
                        spec_shuffle_tile<BT, kAluLanes>(raw[S] + t * K, lane, rows, at);
                    }
                };
                if constexpr (!kHalf) {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        if ((rows_with_ends >> (32 * t)) & 0xFFFFFFFFull) make_rows(t, t);
                }
                // ---- step 6: carry into my row ----
                const A carry = ex_f[S] ? ex_v[S] : (pre_f[S] ? pre_v[S] + ex_v[S] : (span_carry + pre_v[S]) + ex_v[S]);
                if constexpr (kScanLike) {
                    const uint64_t row_any = __ballot(F[S] != 0);
#pragma unroll
                    for (int t = 0; t < (kHalf ? 2 : 1); ++t) {   // the tiles one after the other, or both at once
                        if constexpr (kHalf) make_rows(t, 0);
                        // stored negated in the slot before x-bar(-1), so that the revert subtracts it
                        if (!kHalf || (lane >> 5) == t) {
                            uint32_t *mine = rows + (kHalf ? lane & 31 : lane) * kRowStride;
                            mine[kSlotZero] = 0;
                            mine[kSlotF] = F[S];
                            mine[kSlotNegCarry] = to_bits(A(0) - carry);
                        }
                        wave_lds_sync();

                        // ---- steps 2 + 6 on every element, then store; a lane owns 4 consecutive positions ----
#pragma unroll
                        for (int j = kHalf ? 4 * t : 0; j < (kHalf ? 4 * t + 4 : 8); ++j) {
                            const int R = 8 * j + (lane >> 3), p0 = 4 * (lane & 7);
                            const uint32_t *rp = rows + (kHalf ? R & 31 : R) * kRowStride;
                            const v4u xb = *reinterpret_cast<const v4u *>(rp + kRowData + p0);
                            A o[4];
                            if (((row_any >> (8 * j)) & 0xFFull) == 0) {
                                // none of these eight rows has a flag: the speculation stands, only the carry is added
                                const A nc = from_bits<A>(rp[kSlotNegCarry]);
#pragma unroll
                                for (int i = 0; i < 4; ++i) o[i] = from_bits<A>(xb[i]) - nc;
                            } else {
                                const uint32_t Fr = rp[kSlotF];
                                const uint32_t m = Fr & ((2u << p0) - 1u);  // flags at or before my first position
                                const int slot = m ? kSlotZero + (31 - __clz(m)) : kSlotNegCarry;
                                A b = from_bits<A>(rp[slot]);
                                o[0] = from_bits<A>(xb[0]) - b;
#pragma unroll
                                for (int i = 1; i < 4; ++i) {
                                    if ((Fr >> (p0 + i)) & 1u) b = from_bits<A>(xb[i - 1]);
                                    o[i] = from_bits<A>(xb[i]) - b;
                                }
                            }
                            const uint64_t e0 = cb + 256u * j + 4u * lane;
                            A *z = (A *)P.z;
                            if (chunk_full) {
                                v4u w = {to_bits(o[0]), to_bits(o[1]), to_bits(o[2]), to_bits(o[3])};
                                __builtin_nontemporal_store(w, reinterpret_cast<v4u *>(z + e0));
                            } else {
#pragma unroll
                                for (int i = 0; i < 4; ++i)
                                    if (e0 + i < n) z[e0 + i] = o[i];
                            }
                        }
                        if (kHalf && t == 0) wave_lds_sync();   // the rows are read before the next tile overwrites them
                    }
                } else {
                    // ---- sum: only the segment ends produce output; the lane that owns a row
                    // walks the ends of its row (steps 2 + 6 for those positions only) ----
                    wave_lds_sync();
                    const uint32_t *rp = rows + lane * kRowStride + kRowData;
                    const uint32_t Fc = row_start == 0 ? (F[S] & ~1u) : F[S];  // position 0 is not counted
                    const uint64_t count_base = (uint64_t)count_carry + wex_c + ex_c[S];
                    while (E) {
                        const int e = __builtin_ctz(E);
                        E &= E - 1u;
                        const uint32_t m = F[S] & ((2u << e) - 1u);  // flags at or before the end
                        A v = from_bits<A>(rp[e]);
                        if (m) {
                            const int st = 31 - __clz(m);
                            if (st > 0) v -= from_bits<A>(rp[st - 1]);   // REVSPEC: x-bar(e) - x-bar(start - 1)
                        } else {
                            v += carry;                                  // the segment began before this row
                        }
                        const uint64_t k = count_base + __popc(Fc & ((2u << e) - 1u));
                        if (k < P.out_cap) ((A *)P.out)[k] = v;
                    }
                }
                wave_lds_sync();  // the rows are read before the next chunk overwrites them
            }
          }
            if constexpr (!kUnrollChunks) {
#pragma unroll
                for (int r = 0; r < kStep; ++r) {
                    rotate(F);
                    rotate_rows(raw);
                    rotate(ex_v);
                    rotate(ex_f);
                    rotate(pre_v);
                    rotate(pre_f);
                    if (kCounts) rotate(ex_c);
                }
            }
        }
    }
}

}  // namespace
