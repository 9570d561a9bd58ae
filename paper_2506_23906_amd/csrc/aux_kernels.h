// libmmvseg, part of the one translation unit mmvseg.hip (included there, in order).
// The small kernels around the single-pass kernel: workspace reset, per-tile counts, flag packing from
// bytes / COO rows / CSR row pointers, and the benchmark's reference kernels (streaming copy, gather).
#pragma once

namespace {

// ---- auxiliary kernels -------------------------------------------------------------------------------------

// Zero fills two ranges (workspace words and, for SpMV, y) with 32-bit stores.
__global__ __launch_bounds__(256) void fill_zero_kernel(uint32_t *a, uint64_t na, uint32_t *b, uint64_t nb) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < na; i += stride) a[i] = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nb; i += stride) b[i] = 0;
}

// SpMV in two steps, second step: the words of the main kernel's header (but for the hints and the mark of the
// preparing call, words kHdrHints .. 63) and its descriptors are zeroed, and y; a mark that is not the expected one
// is reported through the status word (the main kernel then leaves at once).
__global__ __launch_bounds__(256) void reset_prepared_kernel(uint32_t *ws, uint64_t ws_words, uint32_t *y, uint64_t n_rows,
                                                             uint32_t expected) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool stale = ws[kHdrPrepared] != expected;   // (the word is not written here)
    for (uint64_t i = i0; i < ws_words; i += stride)
        if (i < kHdrHints || i >= 64) ws[i] = (i == kHdrError && stale) ? kErrNotPrepared : 0u;
    for (uint64_t i = i0; i < n_rows; i += stride) y[i] = 0;
}
// SpMV in two steps, first step, last launch: the mark that the second step looks for.
__global__ void mark_prepared_kernel(uint32_t *hdr, uint32_t mark) {
    if (threadIdx.x == 0 && blockIdx.x == 0) hdr[kHdrPrepared] = mark;
}

// 16 flag bytes -> 16 bits (bit set iff the byte is not zero).
__device__ __forceinline__ uint32_t bits_of_16_bytes(v4u w) {
    uint32_t bits = 0;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        // the highest bit of every byte that is not zero, moved to bits 0, 8, 16, 24, and those next to each other
        // (the multiplication puts the bit of byte j at bit 28 + j; no two partial products meet there)
        const uint32_t nz = ((((w[d] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w[d]) >> 7) & 0x01010101u;
        bits |= ((nz * 0x10204080u) >> 28) << (4 * d);
    }
    return bits;
}
// How many of 16 bytes are not zero.
__device__ __forceinline__ uint32_t nonzero_of_16_bytes(v4u w) {
#pragma unroll
    for (int d = 0; d < 4; ++d) w[d] = (((w[d] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w[d]) & 0x80808080u;
    return __popc((w[0] >> 3) | (w[1] >> 2) | (w[2] >> 1) | w[3]);
}
__device__ __forceinline__ uint32_t bits_of_32_bytes(const uint8_t *f, uint64_t e0, uint64_t n) {   // flags e0 .. e0 + 31; 0 beyond n
    const bool full = e0 + 32 <= n;
    const v4u a = load128<uint8_t, false>(f, e0, n, full), b = load128<uint8_t, false>(f, e0 + 16, n, full);
    return bits_of_16_bytes(a) | (bits_of_16_bytes(b) << 16);
}

// Segmented sum, step "scan of the end markers" of COMPRESS (proof of the SCD / SSCR theorem)
// at tile granularity: workgroup t counts the segment starts in tile t and (sum_kernel, whose waves take a span of the tile
// each) in each of its eight spans (position 0 is not counted: it opens segment 0
// whatever its flag says; bits at or beyond n are not counted).  The main kernel adds up what it needs (starts_before_part).
// Flags of one byte per element (kBytes) are packed on the way: the words go to `packed` (10^8 values: packing kernel
// 19.4 us and counting kernel 5.3 us -> 18.2 us together).
// The same launch zeroes the header and the descriptors of the main kernel.
template <bool kBytes>
__global__ __launch_bounds__(512) void count_spans_kernel(uint32_t *zero, uint64_t zero_words, const void *flags,
                                                          uint32_t *packed, uint64_t n, TileRegions reg, uint32_t unit,
                                                          uint32_t *tile_cnt, uint32_t *span_cnt) {
    __shared__ uint32_t s_part[kSpans];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tile = blockIdx.x;
    for (uint64_t i = (uint64_t)tile * 512 + tid; i < zero_words; i += (uint64_t)gridDim.x * 512) zero[i] = 0;
    const TileSpan span = tile_span(reg, tile, unit);
    const uint64_t span_words = (uint64_t)span.cpw * (unit / kSpans / 32);
    // (tiles and spans begin at multiples of four words, which the 128-bit loads below rely on; the smallest unit is that of
    // stream_kernel, 1024 elements for the eight waves together)
    static_assert(kUnitElems / kSpans / 32 % 4 == 0, "128-bit loads of flag words");
    const uint64_t w0 = (span.base >> 5) + wave * span_words;
    const uint64_t last_word = (n + 31) >> 5;
    const uint64_t end = w0 + span_words < last_word ? w0 + span_words : last_word;
    uint32_t sum = 0;
    if constexpr (kBytes) {
#pragma unroll 4
        for (uint64_t w = w0 + lane; w < end; w += 64) {
            const uint32_t v = bits_of_32_bytes((const uint8_t *)flags, w * 32, n);
            packed[w] = v;
            sum += __popc(w == 0 ? v & ~1u : v);
        }
    } else {
        const uint32_t *fw = (const uint32_t *)flags;
#pragma unroll 4
        for (uint64_t w = w0 + 4 * lane; w < end; w += 256) {
            // (the aligned block of the last word is read whole)
            v4u v = *reinterpret_cast<const v4u *>(fw + w);
            if (w == 0) v[0] &= ~1u;
            if ((w + 4) * 32 > n) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint64_t e0 = (w + j) * 32;
                    if (e0 + 32 > n) v[j] = e0 < n ? (v[j] & ((1u << (uint32_t)(n - e0)) - 1u)) : 0u;
                }
            }
            sum += (__popc(v[0]) + __popc(v[1])) + (__popc(v[2]) + __popc(v[3]));
        }
    }
    sum = wave_sum(sum);
    if (lane == 0) {
        if (span_cnt) span_cnt[tile * kSpans + wave] = sum;
        s_part[wave] = sum;
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t all = 0;
#pragma unroll
        for (uint32_t w = 0; w < kSpans; ++w) all += s_part[w];
        tile_cnt[tile] = all;
    }
}

// Exclusive prefix sums of the counts per tile, in place, by one workgroup (only for very long vectors); the total (+ 1
// for segment 0) is the number of segments.
__global__ __launch_bounds__(1024) void scan_counts_kernel(uint32_t *cnt, uint32_t num_tiles, uint64_t *nseg) {
    __shared__ uint32_t s_wave[16];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t running = 0;
    for (uint32_t base = 0; base < num_tiles; base += 1024) {
        const uint32_t i = base + tid;
        const uint32_t v = i < num_tiles ? cnt[i] : 0u;
        uint32_t inc = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl_up(inc, d);
            if (lane >= (uint32_t)d) inc += o;
        }
        if (lane == 63) s_wave[wave] = inc;
        __syncthreads();
        uint32_t before = 0, total = 0;
#pragma unroll
        for (uint32_t w = 0; w < 16; ++w) {
            if (w == wave) before = total;
            total += s_wave[w];
        }
        if (i < num_tiles) cnt[i] = running + before + inc - v;
        running += total;
        __syncthreads();
    }
    if (tid == 0) *nseg = (uint64_t)running + 1u;
}

// One byte per element -> one bit per element; a thread builds one 32-bit word.  The same launch zeroes the words that
// the main kernel needs zeroed (a launch of its own takes 4.6 us of a stream that is never empty).
__global__ __launch_bounds__(256) void pack_flags_kernel(const uint8_t *f, uint64_t n, uint32_t *words, uint64_t nwords,
                                                         uint32_t *zero, uint64_t zero_words) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (uint64_t i = i0; i < zero_words; i += stride) zero[i] = 0;
    for (uint64_t w = i0; w < nwords; w += stride) words[w] = bits_of_32_bytes(f, w * 32, n);
}

// Segment-start flags of a row-sorted COO matrix, f(e) = [e == 0 or row(e) != row(e-1)], bit-packed; the same
// launch zero fills the workspace words (header, descriptors) and y.  A wave takes 2048 entries: every lane reads
// eight times four consecutive indices (all loads in flight at once), compares them with their left neighbours
// (the lane before it holds the one before its first: a DPP move), and eight lanes OR their nibbles into one
// flag word (DPP again; no LDS traffic).
// Bound by the read of the indices (33 million entries: 21 us, 6.4 TB/s).  The loads are plain ones: the main kernel reads
// row[] again at the segment ends and finds it in the memory-side cache as far as it fits.  Whole products, each call on
// another of four matrices (so that nothing is left of the call before), non-temporal loads -> plain ones: 3 million entries
// 27.9 -> 27.0 us, 8 million 47.9 -> 45.9, 16 million 111.7 -> 108.7, 33 million 239.9 -> 239.7.
__global__ __launch_bounds__(256) void row_flags_kernel(const int32_t *row, uint64_t nnz, uint32_t *words,
                                                        uint32_t *ws, uint64_t ws_words, uint32_t *y, uint64_t n_rows) {
    const int lane = threadIdx.x & 63;
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < ws_words; i += stride) ws[i] = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n_rows; i += stride) y[i] = 0;
    const uint64_t wave0 = ((uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 2048;   // eight rounds of 256 entries
    if (wave0 >= nnz) return;
    v4i r[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint64_t e0 = wave0 + 256u * j + 4u * lane;
        r[j] = v4i{0, 0, 0, 0};
        if (e0 + 4 <= nnz) {
            r[j] = *reinterpret_cast<const v4i *>(row + e0);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (e0 + i < nnz) r[j][i] = row[e0 + i];
        }
    }
    int before_first = wave0 > 0 ? row[wave0 - 1] : -1;   // (no row index is negative: entry 0 starts a segment)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint64_t e0 = wave0 + 256u * j + 4u * lane;
        int left = (int)dpp_or_zero<0x138, 0xF>((uint32_t)r[j][3]);   // wave_shr 1: the last index of the lane before
        if (lane == 0) left = before_first;
        const uint32_t nib = (r[j][0] != left ? 1u : 0u) | (r[j][1] != r[j][0] ? 2u : 0u) | (r[j][2] != r[j][1] ? 4u : 0u) |
                             (r[j][3] != r[j][2] ? 8u : 0u);
        const uint32_t valid = e0 >= nnz ? 0u : (nnz - e0 >= 4 ? 0xFu : (1u << (uint32_t)(nnz - e0)) - 1u);
        uint32_t v = (nib & valid) << (4 * (lane & 7));
        v |= dpp_or_zero<0x111, 0xF>(v);   // row_shr 1, 2, 4: lane 8 k + 7 collects the eight nibbles of its row of 32
        v |= dpp_or_zero<0x112, 0xF>(v);
        v |= dpp_or_zero<0x114, 0xF>(v);
        const uint64_t w = ((wave0 + 256u * j) >> 5) + (lane >> 3);
        if ((lane & 7) == 7 && w * 32 < nnz) words[w] = v;
        before_first = __builtin_amdgcn_readlane(r[j][3], 63);
    }
}

// Row pointers of a CSR matrix -> (a) bit-packed segment-start flags over the non-zeros (a row
// with entries sets the bit of its first entry; rows that share a word meet in an atomic OR on
// a zeroed word), (b) the bit-packed mask of rows that have entries (one ballot per 64 rows),
// (c) the number of segment starts inside every tile of the main kernel (as in count_spans_kernel; the tiles are equal
// here, so entry e lies in tile e / tile_elems; the rows of a wave that start in the same tile share one atomic add on a
// zeroed table: adds to one address are served one after the other, about 11 ns each) and (d) the mark that some row is empty.
__global__ __launch_bounds__(256) void csr_flags_kernel(const int32_t *rowptr, uint64_t n_rows, uint32_t *fw,
                                                        uint32_t *rowmask, uint32_t *hdr, uint32_t tile_elems,
                                                        uint32_t *tile_count) {
    const int lane = threadIdx.x & 63;
    const uint64_t r = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    bool nonempty = false;
    uint32_t tile = 0xFFFFFFFFu;   // tile of the first entry of a row that is counted
    if (r < n_rows) {
        const int32_t a = rowptr[r], b = rowptr[r + 1];
        nonempty = b > a;
        if (nonempty) {
            atomicOr(fw + ((uint32_t)a >> 5), 1u << ((uint32_t)a & 31u));
            if (a > 0) tile = (uint32_t)a / tile_elems;
        }
    }
    const uint64_t m = __ballot(nonempty);
    // a matrix none of whose rows is empty needs no row map: segment k is row k
    if (__ballot(r < n_rows && !nonempty) != 0 && lane == 0) hdr[kHdrEmptyRows] = 1u;
    uint64_t todo = __ballot(tile != 0xFFFFFFFFu);
    while (todo) {   // one round per distinct tile among the rows of the wave
        const int first = __ffsll((unsigned long long)todo) - 1;
        const uint32_t t = __shfl(tile, first);
        const uint64_t same = __ballot(tile == t);
        if (lane == first) atomicAdd(tile_count + t, (uint32_t)__popcll((unsigned long long)same));
        todo &= ~same;
    }
    const uint64_t r0 = r - lane;
    if (lane == 0 && r0 < n_rows) {
        rowmask[r0 >> 5] = (uint32_t)m;
        if (r0 + 32 < n_rows) rowmask[(r0 >> 5) + 1] = (uint32_t)(m >> 32);
    }
}

// The same in one launch that needs nothing zeroed first: workgroup t makes all that the product kernel needs for its tile t.
// It finds the rows that start in the tile by a search in the row pointers, all threads probing, sets their bits in LDS and
// stores the words, and leaves
//   tile_base[t]    the first row that starts in the tile (r0), kPlanDense set if none of the tile's rows is empty: then the
//                   j-th start of the tile is row r0 + j, and what is open where it begins is row r0 - 1, the last that starts
//                   before the tile and reaches it;
//   rowmap[r0 - 1 + j]  those rows else.  (The slots of two tiles meet in one alone, which both give the row of its number.)
// A tile may hold nearly all rows (those of one entry or none behind the long ones of a matrix sorted by degree), so one of
// more than share_above rows (see plan_share_above) is shared: tile_base[t] has kPlanByEnd set, and the row whose last entry is
// position e of the tile stands in rowmap[r0 + e], so that nobody needs to know how many rows with entries lie before its own.  The
// workgroups behind those of the tiles have a row each, kPlanShare apart: the first position of that row, rounded up to
// whole 128-bit words of flags, up to that of the next one of them in the tile is theirs, what lies before the tile's own workgroup's.
// They leave at once where no row of another one, half of share_above away, starts in the same tile.
// The same launch zeroes the header and descriptors of the product kernel, and y.
// Bound by its chain of dependent loads: four to five for the two ends of the tile, then one per 2048 rows.  Four waves: eight
// or sixteen start later (blocks of 16, 65536 rows: 33.4 and 38.5 us the call against 31.5).  Products in one step, four
// launches over the rows (reset, csr_flags_kernel, COMPRESS of the row list, product) -> this kernel and the product, us:
//   sparse attention, 65536 rows: 11.5 M entries 34.5 -> 31.4; 63 M 114 -> 106; 8192 rows, 1.4 M 16.5 -> 13.2
//   equal rows of 1, 2, 8, 32 entries, 2^20 rows: 135 -> 35, 98 -> 28, 114 -> 63, 222 -> 209; 65536 rows: 32 -> 24, 28 -> 16,
//   21 -> 13.6, 19.7 -> 17; Zipf lengths, 2^20 rows and 2^25 entries 244 -> 222
// (In the four launches, adds and ORs of many rows meet in the same words, and each launch costs 2.5 to 5.)
constexpr int kPlanThreads = 256, kPlanRows = 8;
constexpr uint32_t kPlanShare = 8192;   // rows of a piece
template <bool kByEnd> struct PlanByEnd {
    static constexpr bool value = kByEnd;
};
__global__ __launch_bounds__(kPlanThreads) void csr_plan_kernel(const int32_t *rowptr, uint32_t n_rows, uint32_t nnz, uint32_t tiles, uint32_t tile_elems, uint32_t share_above,
                                                                uint32_t *fw, uint32_t *tile_base, uint32_t *rowmap, uint32_t *ws,
                                                                uint64_t ws_words, uint32_t *y, uint32_t y_rows) {
    constexpr int kWaves = kPlanThreads / 64;
    __shared__ __attribute__((aligned(16))) uint32_t s_words[kMaxUnits * (kUnitElems / 32)];
    __shared__ uint32_t s_cnt[2][kWaves], s_kept[2][kWaves];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t stride = (uint64_t)gridDim.x * kPlanThreads;
    for (uint64_t i = (uint64_t)blockIdx.x * kPlanThreads + tid; i < ws_words; i += stride) ws[i] = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * kPlanThreads + tid; i < y_rows; i += stride) y[i] = 0;
    const bool helps = blockIdx.x >= tiles;
    const uint32_t my_row = helps ? (blockIdx.x - tiles) * kPlanShare : 0u, my_start = helps ? (uint32_t)rowptr[my_row] : 0u;
    if (helps && my_start >= nnz) return;
    const uint32_t tile = helps ? my_start / tile_elems : blockIdx.x;
    const uint32_t base = tile * tile_elems, end = nnz - base < tile_elems ? nnz : base + tile_elems;
    if (helps) {
        // more than share_above rows are those of share_above / kPlanShare workgroups or more: one that far off at least, before or behind
        const uint32_t off = share_above / kPlanShare / 2 * kPlanShare;
        const bool before = my_row >= off && (uint32_t)rowptr[my_row - off] >= base;
        const bool behind = n_rows - my_row > off && (uint32_t)rowptr[my_row + off] < end;
        if (!before && !behind) return;
    }

    // first index in [lo, hi] whose row pointer is at least the target (hi: none), for two targets at once
    auto search = [&](uint32_t (&lo)[2], uint32_t (&hi)[2], const uint32_t (&target)[2]) {
        while (lo[0] < hi[0] || lo[1] < hi[1]) {
            uint32_t step[2];
            for (int k = 0; k < 2; ++k) {
                step[k] = (hi[k] - lo[k]) / kPlanThreads + 1;
                const uint32_t p = lo[k] + (tid + 1) * step[k] - 1;
                const bool below = p < hi[k] && (uint32_t)rowptr[p] < target[k];
                const uint64_t b = __ballot(below);
                if (lane == 0) s_cnt[k][wave] = (uint32_t)__popcll((unsigned long long)b);
            }
            __syncthreads();
            for (int k = 0; k < 2; ++k) {
                uint32_t c = 0;
                for (int w = 0; w < kWaves; ++w) c += s_cnt[k][w];
                lo[k] += c * step[k];
                hi[k] = hi[k] < lo[k] + step[k] - 1 ? hi[k] : lo[k] + step[k] - 1;
            }
            __syncthreads();
        }
    };
    uint32_t first[2] = {0, 0}, behind[2] = {n_rows, n_rows};
    search(first, behind, {base, end});
    const uint32_t r0 = first[0], r1 = first[1];   // rows that start in the tile
    const bool shared = r1 - r0 > share_above;
    if (helps && !shared) return;
    uint32_t from = base, upto = end, ra = r0, rb = r1;   // the positions that are mine, the rows that start there
    if (shared) {
        auto piece_at = [&](uint32_t start) { return start + 127 < end ? (start + 127) & ~127u : end; };
        const uint32_t next = helps ? my_row + kPlanShare : (r0 + kPlanShare - 1) / kPlanShare * kPlanShare;
        if (helps) from = piece_at(my_start);
        if (next < r1) upto = piece_at((uint32_t)rowptr[next]);
        uint32_t lo[2] = {r0, r0}, hi[2] = {r1, r1};
        search(lo, hi, {from, upto});
        ra = lo[0], rb = lo[1];
    }
    const uint32_t words = (upto - from + 31) / 32;
    for (uint32_t w = tid; w < (words + 3) / 4 * 4; w += kPlanThreads) s_words[w] = 0;
    uint32_t kept = 0;                             // rows with entries so far
    __syncthreads();
    auto store_row = [&](bool by_end, uint32_t slot, uint32_t row) {
        if (!by_end) {
            rowmap[slot] = row;
        } else {
            const uint32_t last = (uint32_t)rowptr[row + 1] - 1u;
            if (last < end) rowmap[r0 + (last - base)] = row;
        }
    };
    // rows found in a round, in their order: masks of 64 candidates each -> where a wave's first one goes
    auto place = [&](const uint64_t (&mask)[kPlanRows], uint32_t odd, uint32_t &total) {
        uint32_t mine = 0;
#pragma unroll
        for (int i = 0; i < kPlanRows; ++i) mine += (uint32_t)__popcll((unsigned long long)mask[i]);
        if (lane == 0) s_kept[odd][wave] = mine;
        __syncthreads();
        uint32_t at = ra + kept;
        total = 0;
        for (int w = 0; w < kWaves; ++w) {
            if (w < (int)wave) at += s_kept[odd][w];
            total += s_kept[odd][w];
        }
        kept += total;
        return at;
    };
    // Row by row.  (Two bodies: a load of the shared one inside the loop would have the other one wait for the next round's pointers,
    // 2^20 rows of 0.4 entries 16.7 us to prepare, 19.0 so.)
    auto row_by_row = [&](auto form) {
        constexpr bool by_end = decltype(form)::value;
        // A round is kPlanRows rows per thread: lane l of a wave takes rows l, l + 64, ... of the wave's share (those from rb on
        // count as empty).  The next round's pointers are under way meanwhile.
        auto load_rows = [&](uint32_t cur, uint32_t (&p)[kPlanRows + 1]) {
            const uint32_t r = cur + 64 * kPlanRows * wave + lane;
#pragma unroll
            for (int i = 0; i <= kPlanRows; ++i) p[i] = (uint32_t)rowptr[r + 64 * i < rb ? r + 64 * i : rb];
        };
        uint32_t p[kPlanRows + 1];
        load_rows(ra, p);
        for (uint32_t cur = ra, odd = 0; cur < rb; odd ^= 1) {
            const uint32_t r = cur + 64 * kPlanRows * wave + lane;
            uint32_t ahead[kPlanRows + 1];
            cur += kPlanThreads * kPlanRows;
            if (cur < rb) load_rows(cur, ahead);
            uint64_t mask[kPlanRows];
#pragma unroll
            for (int i = 0; i < kPlanRows; ++i) {
                // the next row's pointer: the next lane's; of lane 63, the first of the next 64
                const int after = __builtin_amdgcn_readfirstlane((int)p[i + 1]);
                mask[i] = __ballot((uint32_t)__builtin_amdgcn_update_dpp(after, (int)p[i], 0x130, 0xF, 0xF, false) > p[i]);
            }
            uint32_t total, at = place(mask, odd, total);
#pragma unroll
            for (int i = 0; i < kPlanRows; ++i) {
                if (mask[i] == 0) continue;
                if (mask[i] >> lane & 1) {
                    store_row(by_end, at + __popcll((unsigned long long)(mask[i] & ((1ull << lane) - 1))), r + 64 * i);
                    if (p[i] - from < upto - from) atomicOr(s_words + ((p[i] - from) >> 5), 1u << ((p[i] - from) & 31u));
                }
                at += (uint32_t)__popcll((unsigned long long)mask[i]);
            }
            if (cur < rb) {
                if (total == 0) {   // a long run of empty rows: on to the row behind it
                    const uint32_t v = (uint32_t)rowptr[cur];
                    uint32_t lo[2] = {cur, cur}, hi[2] = {rb, cur};
                    search(lo, hi, {v + 1, v + 1});
                    cur = lo[0] - 1;
                    load_rows(cur, p);
                } else {
#pragma unroll
                    for (int i = 0; i <= kPlanRows; ++i) p[i] = ahead[i];
                }
            }
        }
    };
    const uint32_t e0 = ra < rb ? (uint32_t)rowptr[ra] : 0u, starts = ra < rb ? (uint32_t)rowptr[rb - 1] - e0 + 1 : 0u;
    if (rb - ra > kPlanThreads * kPlanRows * 2 && (rb - ra) / 24 > starts) {
        // Many rows, almost all of them empty: a search for every position instead that a row may start at, for the last row
        // that starts up to there.  (2048 positions take about 20 us, 2048 rows 0.9: the two meet at 22 rows per position.)
        uint32_t top = 1u << 31;
        while (top > rb - ra) top >>= 1;
        // Up to 256 positions: one for each thread, all its loads in flight for that one, an eighth of the rows left by each step (2^20
        // rows, one in 2048 of one entry, in one tile: 29 -> 21 us the call).
        const uint32_t cur0 = (e0 - from) & ~63u, behind_last = e0 - from + starts;
        const bool one = behind_last - cur0 <= kPlanThreads;
        for (uint32_t cur = cur0, odd = 0; cur < behind_last; cur += kPlanThreads * kPlanRows, odd ^= 1) {
            const uint32_t at0 = cur + 64 * (one ? 1 : kPlanRows) * wave;   // (in the piece)
            uint32_t row[kPlanRows], start[kPlanRows];
#pragma unroll
            for (int i = 0; i < kPlanRows; ++i) row[i] = ra, start[i] = e0;
            if (one) {
                uint32_t step = 1;
                while (step <= top / 8) step *= 8;
                for (; step; step /= 8) {
                    uint32_t v[kPlanRows - 1], below = 0;
#pragma unroll
                    for (int i = 0; i < kPlanRows - 1; ++i) {
                        const uint64_t next = row[0] + (uint64_t)(i + 1) * step;
                        v[i] = next < rb ? (uint32_t)rowptr[next] : ~0u;
                    }
#pragma unroll
                    for (int i = 0; i < kPlanRows - 1; ++i)
                        if (v[i] <= from + at0 + lane) below = i + 1, start[0] = v[i];
                    row[0] += below * step;
                }
            } else {
                for (uint32_t step = top; step; step >>= 1) {
#pragma unroll
                    for (int i = 0; i < kPlanRows; ++i) {
                        const uint32_t next = row[i] + step < rb ? row[i] + step : row[i], v = (uint32_t)rowptr[next];
                        if (v <= from + at0 + 64 * i + lane) row[i] = next, start[i] = v;
                    }
                }
            }
            uint64_t mask[kPlanRows];
#pragma unroll
            for (int i = 0; i < kPlanRows; ++i) mask[i] = one && i > 0 ? 0 : __ballot(start[i] == from + at0 + 64 * i + lane);
            uint32_t total, at = place(mask, odd, total);
#pragma unroll
            for (int i = 0; i < kPlanRows; ++i) {
                if (mask[i] == 0) continue;
                if (mask[i] >> lane & 1) store_row(shared, at + __popcll((unsigned long long)(mask[i] & ((1ull << lane) - 1))), row[i]);
                if (lane < 2 && at0 + 64 * i + 32 * lane < upto - from) s_words[at0 / 32 + 2 * i + lane] = (uint32_t)(mask[i] >> (32 * lane));
                at += (uint32_t)__popcll((unsigned long long)mask[i]);
            }
        }
    } else if (shared) {
        row_by_row(PlanByEnd<true>());
    } else {
        row_by_row(PlanByEnd<false>());
    }
    __syncthreads();
    if (tid == 0 && !helps) {
        tile_base[tile] = r0 | (shared ? kPlanByEnd : kept == r1 - r0 ? kPlanDense : 0u);
        if (r0 > 0 && !shared) rowmap[r0 - 1] = r0 - 1;
        if (r0 > 0 && shared) {   // (a row that starts before the tile and ends in it)
            const uint32_t last = (uint32_t)rowptr[r0] - 1u;
            if (last >= base && last < end) rowmap[r0 + (last - base)] = r0 - 1;
        }
    }
    v4u *out = reinterpret_cast<v4u *>(fw + from / 32);
    for (uint32_t w = tid; w < (words + 3) / 4; w += kPlanThreads) out[w] = reinterpret_cast<const v4u *>(s_words)[w];
}

// Random-access reference for SpMV: streams val and col with 128-bit loads, gathers x[col] and
// keeps one partial sum per thread: everything the product vector of SpMV costs, and nothing of
// the segmented sum.  A column index at or beyond n_cols reads x[0] instead (no access out of bounds).
constexpr int kGatherRefBlocks = 8192;
__global__ __launch_bounds__(256) void gather_reference_kernel(const v4u *val, const v4u *col, uint64_t quads,
                                                               uint32_t n_cols, const float *x, float *partial) {
    float acc = 0.0f;
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < quads; i += stride) {
        const v4u v = __builtin_nontemporal_load(val + i);
        const v4u c = __builtin_nontemporal_load(col + i);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc += from_bits<float>(v[k]) * x[c[k] < n_cols ? c[k] : 0u];
    }
    partial[(uint64_t)blockIdx.x * 256 + threadIdx.x] = acc;
}

// Streaming reference: 128-bit non-temporal reads and writes, kIn input chunks and kOut
// output chunks per thread, both striped across the workgroup; one workgroup per 256
// units (measured faster than a persistent grid-stride loop on this chip).
template <int kIn, int kOut>
__global__ __launch_bounds__(256) void stream_copy_kernel(const v4u *src, v4u *dst, uint64_t units) {
    const uint64_t u0 = (uint64_t)blockIdx.x * 256;
    v4u acc = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < kIn; ++i) {
        const uint64_t idx = u0 * kIn + (uint64_t)i * 256 + threadIdx.x;
        if (idx < units * kIn) acc ^= __builtin_nontemporal_load(src + idx);
    }
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
        const uint64_t idx = u0 * kOut + (uint64_t)i * 256 + threadIdx.x;
        if (idx < units * kOut) __builtin_nontemporal_store(acc + (unsigned)i, dst + idx);
    }
    if (kOut == 0 && acc[0] == 0x9E3779B9u && acc[1] == 0x7F4A7C15u && acc[2] == 1u && acc[3] == 2u)
        dst[0] = acc;  // keeps the reads alive; practically never taken
}

}  // namespace
