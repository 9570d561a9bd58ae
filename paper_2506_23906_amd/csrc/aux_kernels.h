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
