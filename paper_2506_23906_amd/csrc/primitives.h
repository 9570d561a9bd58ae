// libmmvseg, part of the one translation unit mmvseg.hip (included there, in order).
// The stand-alone primitives of Algorithms SCD and SSCR (Sec. 4.1): COMPRESS, DIFF, REVERT and their helpers.
#pragma once

namespace {

// ---- the stand-alone primitives of Algorithms SCD and SSCR (Sec. 4.1) ------------------------------------
//
// SCAN is the main kernel without a flag vector (kPlainScan).  COMPRESS, DIFF and REVERT follow.
// They exist so that the paper's un-fused compositions (SCD = DIFF o COMPRESS o SCAN, SSCR =
// REVERT o COMPRESS o (SCAN, SCAN)) can be run and timed next to the fused single-pass kernel.

// End markers f^- of Algorithm SCD: f shifted left by one position with a 1 appended, bit-packed.
__global__ __launch_bounds__(256) void end_markers_kernel(const uint32_t *fw, uint64_t n, uint32_t *out,
                                                          uint64_t nwords) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t w = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; w < nwords; w += stride) {
        const uint32_t next = w + 1 < nwords ? fw[w + 1] : 0u;
        uint32_t e = (fw[w] >> 1) | (next << 31);
        if (w == nwords - 1) {
            const uint32_t last = (uint32_t)((n - 1) & 31u);   // position of element n - 1 in this word
            e = (e & ((1u << last) - 1u)) | (1u << last);
        }
        out[w] = e;
    }
}

// Bit-packed flags -> one int8 (0 / 1) per element, for the count scan SCAN(f) of Algorithm SSCR.
__global__ __launch_bounds__(256) void unpack_flags_kernel(const uint32_t *fw, uint64_t n, int8_t *out) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t nquads = (n + 3) / 4;   // a thread writes four bytes; out has room for the padding
    for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nquads; q += stride) {
        const uint32_t bits = (fw[q >> 3] >> (4 * (q & 7))) & 0xFu;
        reinterpret_cast<uint32_t *>(out)[q] = (bits & 1u) | ((bits & 2u) << 7) | ((bits & 4u) << 14) | ((bits & 8u) << 21);
    }
}

// COMPRESS (Sec. 2): out = the 32-bit entries of x whose mask bit is set, in order; with
// x == nullptr the positions themselves are compressed.  The output
// index of an entry is the number of set bits before it (the scan of the mask in the paper's
// COMPRESS), found per tile from popcounts and across tiles by decoupled look-back.
// A wave owns kGroups groups of 64 * kWords consecutive positions (kWords = 64 or 16): lane j < kWords
// holds the 64-bit mask word j of every group.  A mask of one byte per position (kBytes) is read by this kernel itself:
// 16 bytes per lane and load, turned into 16 bits, and the pieces of a word brought together through LDS.
// A wave with few selected entries (at most 1 in 32) lets every lane walk the set bits of its own words: up to
// there most 128-byte lines of x hold at most one of them (n = 2^28, 3 % selected: 0.184 ms; 4 %: 0.175 in pieces, 0.238 walked).  Any other wave takes its positions in pieces of 1024: it
// loads all of x (128 bits per lane, the next piece on its way while one is stored, the first before the look-back), drops
// the selected entries into LDS at their rank, and stores them from there with 128-bit stores.  Bound by the memory;
// n = 2^26 values, 30 % selected by a byte mask: 126 us for packing kernel and a loop over the words of 64 positions (one load and
// one store instruction of 64 lanes each, 30 % of them active), 81 us now (whole calls, with the 5 us of the reset).
// Short masks take the short
// spans: four times the waves, a quarter of the words each wave visits one after the other.  Long masks take
// two or four groups per wave: a tile costs a ticket (11 ns each, one after the other), a barrier and a look-back
// whatever its length, and with one group per wave the tickets alone took 93 us of the 111 us at n = 2^28
// and 0.1 % selected (now 0.048 ms).
// The workgroups that are resident from the start take the tile of their own index, as in the main kernel.
// kSingle: short masks.  Every workgroup counts the set bits before its tile itself, so nothing has to be zeroed and nobody
// waits: one launch instead of two.  Whole calls in a graph, 30 % selected, other inputs every time (the same, in brackets): 3000
// positions 4.6 -> 3.2 us (4.7 -> 3.2), 2^18 bits 6.9 -> 4.7 (6.3 -> 4.0), 2^20 bits 8.3 -> 6.0 (7.8 -> 4.7), 2^21 bits 9.6 -> 7.8 (8.1 -> 5.8),
// 2^16 bytes 6.7 -> 5.9 (6.3 -> 4.6), 2^17 bytes 7.1 -> 6.8 (6.5 -> 5.3; with the loads of the count in a loop of their own latency
// each, and the bytes turned into bits ahead of it, 8.5 and 5.9).  Beyond, the count takes longer than the launch.
constexpr int kCompressWaves = 8;
constexpr uint64_t kCompressSingleBits = 1ull << 21, kCompressSingleBytes = 1ull << 17;   // positions
constexpr uint64_t kCompressShortN = 1ull << 22;   // masks up to this length take 16 words per wave
// masks from 2^26 positions on take two groups of words per wave, from 2^27 on four: the most that still leaves a tile
// for each of the 1024 workgroups that are resident at once (n = 2^27, 1 % selected: 0.054 ms with two groups, 0.039
// with four; n = 2^26, 0.1 % selected: 0.038 ms with one group, 0.015 with two)
inline int compress_words(uint64_t n) { return n <= kCompressShortN ? 16 : 64; }
inline int compress_groups(uint64_t n) { return n >= (1ull << 27) ? 4 : n >= (1ull << 26) ? 2 : 1; }
inline uint64_t compress_tile(uint64_t n) { return (uint64_t)kCompressWaves * 64u * compress_words(n) * compress_groups(n); }

constexpr int kPieceElems = 1024;                  // positions a wave compacts at a time
constexpr int kPieceWords = kPieceElems + 4;       // LDS words of a wave: a piece, shifted by up to three

// One piece of 1024 positions on its way: the values (word i of lane l = positions 256 i + 4 l .. + 3 of the piece) and,
// per word, the rank of the lane's first position among the selected ones of the piece (upper bits) and which of the
// four are selected (lowest four bits).
struct CompressPiece {
    v4u w[4];
    uint32_t rank_sel[4];
};

template <int kWords, int kGroups, bool kBytes, bool kSingle = false>
__global__ __launch_bounds__(kCompressWaves * 64, 8) void compress_kernel(
    const uint32_t *__restrict__ x, const void *__restrict__ mask, uint64_t n, uint32_t *__restrict__ out,
    uint64_t out_cap, uint64_t *__restrict__ count, uint32_t *hdr, uint64_t *desc, uint32_t num_tiles,
    const uint32_t *needed, uint32_t first_round) {
    __shared__ uint32_t s_tile, s_wave[kCompressWaves], s_carry, s_before[kCompressWaves];
    __shared__ __attribute__((aligned(16))) uint32_t s_piece[kCompressWaves][kPieceWords];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (needed && *needed == 0) return;   // CSR SpMV without empty rows: nobody reads the row map
    const bool own_index = blockIdx.x < first_round;
    if (tid == 0 && !own_index)
        s_tile = first_round + __hip_atomic_fetch_add(hdr + kHdrTicket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const uint32_t tile = __builtin_amdgcn_readfirstlane(own_index ? blockIdx.x : s_tile);
    constexpr uint32_t kGroupSpan = 64u * kWords;                                   // positions of one group
    constexpr uint32_t kSpan = kGroupSpan * kGroups;                                // positions of a wave
    const uint64_t span = ((uint64_t)tile * kCompressWaves + wave) * kSpan;          // first position of my wave
    uint32_t *piece_buf = s_piece[wave];
    uint64_t m[kGroups];
    uint32_t before[kGroups];   // selected entries of my wave before my word of group g
    uint32_t wave_cnt = 0;
    if constexpr (kSingle) {   // set bits before the tile (which begins at a multiple of 128 positions)
        const uint64_t start = (uint64_t)tile * kCompressWaves * kSpan;
        // four words under way at a time, also of the last ones (a lane with nothing left reads its first word again)
        const uint32_t words = (uint32_t)(start / (kBytes ? 16 : 128));
        uint32_t cnt = 0;
        for (uint32_t i0 = tid; i0 < words; i0 += 4 * kCompressWaves * 64) {
            v4u w[4];
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) w[j] = ((const v4u *)mask)[i0 + j * kCompressWaves * 64 < words ? i0 + j * kCompressWaves * 64 : i0];
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                const uint32_t c = kBytes ? nonzero_of_16_bytes(w[j]) : (__popc(w[j][0]) + __popc(w[j][1])) + (__popc(w[j][2]) + __popc(w[j][3]));
                cnt += i0 + j * kCompressWaves * 64 < words ? c : 0u;
            }
        }
        cnt = wave_sum(cnt);
        if (lane == 0) s_before[wave] = cnt;
        if (tile == 0 && tid == 0) hdr[kHdrError] = hdr[kHdrPrepared] = 0;
    }
    const uint64_t left = span < n ? n - span : 0;
    const uint32_t positions = left < kSpan ? (uint32_t)left : kSpan;                // of my wave
    if constexpr (kBytes) {
        constexpr int kLoads = kWords / 16;   // 1024 mask bytes of the wave each
        // (the 16-byte block of the last byte is read whole.  All loads under way at once, of four groups all but the last four (60 registers):
        // with the end of the mask looked after by a branch per lane, each was waited for before the next.  2^26 bytes, 30 % selected 81.0 -> 80.5 us the call, 1.3 * 10^7 bits,
        // 8 % 18.6 -> 18.0)
        const auto rsrc = make_rsrc((const uint8_t *)mask + span, (positions + 15) & ~15u);
        v4u b[kGroups][kLoads];
#pragma unroll
        for (int g = 0; g < kGroups; ++g)
#pragma unroll
            for (int i = 0; i < kLoads; ++i) b[g][i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, 16 * lane + (int)(kGroupSpan * g) + 1024 * i, 0, kAuxNt);
        uint16_t *piece16 = reinterpret_cast<uint16_t *>(piece_buf);
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
#pragma unroll
            for (int i = 0; i < kLoads; ++i) piece16[64 * i + lane] = (uint16_t)bits_of_16_bytes(b[g][i]);
            wave_lds_sync();
            m[g] = 0;
            if (lane < kWords) m[g] = *reinterpret_cast<const uint64_t *>(piece_buf + 2 * lane);
            wave_lds_sync();   // read before the next group overwrites it
        }
    } else {
        const auto rsrc = make_rsrc((const uint32_t *)mask + (span >> 5), (positions + 63) / 64 * 8);   // (... of the last word)
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const v2u w = __builtin_amdgcn_raw_buffer_load_b64(rsrc, lane < kWords ? 8 * lane + (int)(kGroupSpan / 8 * g) : -8, 0, 0);   // (-8: beyond every mask)
            m[g] = (uint64_t)w[1] << 32 | w[0];
        }
    }
    if (positions % 64 != 0) {   // (the end of the mask: bits at or beyond n do not count)
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const int valid = (int)positions - (int)(kGroupSpan * g + 64 * lane);
            if (valid < 64) m[g] &= valid > 0 ? (1ull << valid) - 1ull : 0ull;
        }
    }
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        const uint32_t cnt = (uint32_t)__popcll((unsigned long long)m[g]);
        uint32_t inc = cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl_up(inc, d);
            if (lane >= d) inc += o;
        }
        before[g] = wave_cnt + (inc - cnt);
        wave_cnt += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    }
    if (lane == 0) s_wave[wave] = wave_cnt;

    // ---- a wave with many selected entries: its values, piece by piece ----
    const bool dense = wave_cnt > 2u * kWords * kGroups;
    constexpr int kPieces = kGroups * kWords / 16;
    CompressPiece pc;
    const auto x_rsrc = make_rsrc(x + span, x ? (positions * 4 + 15) & ~15u : 0u);   // (the 16-byte block of the last entry is read whole)
    // (c is the same for all lanes: the selects below run on scalar conditions)
    auto load_piece = [&](int c) {
        uint64_t mg = m[0];
        uint32_t bg = before[0];
#pragma unroll
        for (int g = 1; g < kGroups; ++g)
            if (c / (kWords / 16) == g) mg = m[g], bg = before[g];
        const int word0 = 16 * (c % (kWords / 16));   // first of the piece's sixteen mask words
        const uint32_t rank0 = (uint32_t)__builtin_amdgcn_readlane((int)bg, word0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int src = word0 + 4 * i + (lane >> 4);
            const uint64_t word = ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(mg >> 32), src) << 32) | (uint32_t)__shfl((int)(uint32_t)mg, src);
            const uint32_t at = 4u * (lane & 15);
            const uint32_t rank = (uint32_t)__shfl((int)bg, src) - rank0 + (uint32_t)__popcll((unsigned long long)(word & ((1ull << at) - 1ull)));
            const uint32_t sel = (uint32_t)(word >> at) & 0xFu;
            pc.rank_sel[i] = (rank << 4) | sel;
            // (no branch, not even a uniform one: the compiler would wait ahead of each for the loads before it.  A lane without selected
            // entries has nothing to read: its offset lies beyond every x; without x nothing does)
            pc.w[i] = __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, sel ? 4 * (kPieceElems * c + 256 * i + 4 * lane) : -16, 0, kAuxNt);
        }
    };
    if (dense) load_piece(0);
    __syncthreads();
    uint32_t wave_ex = 0, tile_cnt = 0;
#pragma unroll
    for (int w = 0; w < kCompressWaves; ++w) {
        if (w == wave) wave_ex = tile_cnt;
        tile_cnt += s_wave[w];
    }
    uint32_t tile_before = 0;   // selected entries before the tile
    if constexpr (kSingle) {
#pragma unroll
        for (int w = 0; w < kCompressWaves; ++w) tile_before += s_before[w];
        if (tid == 0 && tile == num_tiles - 1) *count = (uint64_t)tile_before + tile_cnt;
    } else {
        if (tid == 0) desc_store(desc + tile, tile == 0 ? kStatusPrefix : kStatusAggregate, tile_cnt);
        if (wave == 0) {
            uint32_t carry = 0;
            if (tile > 0) carry = lookback<uint32_t>(desc, (int)tile, lane, poll_lanes(num_tiles, first_round), hdr);
            if (lane == 0) {
                if (tile > 0) desc_store(desc + tile, kStatusPrefix, carry + tile_cnt);
                s_carry = carry;
                if (tile == num_tiles - 1) *count = (uint64_t)carry + tile_cnt;
            }
        }
        __syncthreads();
        tile_before = s_carry;
    }
    const uint64_t wave_base = (uint64_t)tile_before + wave_ex;   // output index of the first selected entry of my wave
    if (!dense) {
        // few selected entries in my wave's positions: every lane walks the set bits of its own
        // words (a handful of independent loads per lane)
        // Four entries of a word at a time, their loads all under way before the first store: one memory round trip
        // per four entries instead of one per entry.
#pragma unroll 1
        for (int g = 0; g < kGroups; ++g) {
            const uint64_t group0 = span + (uint64_t)g * kGroupSpan;   // (uniform)
            uint64_t mm = m[0];
            uint32_t bg = before[0];
#pragma unroll
            for (int i = 1; i < kGroups; ++i)
                if (g == i) mm = m[i], bg = before[i];
            uint64_t k = wave_base + bg;
            while (mm) {
                uint32_t p[4];
                uint32_t v[4];
                bool on[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    on[i] = mm != 0;
                    p[i] = 64u * lane + (on[i] ? (uint32_t)__builtin_ctzll((unsigned long long)mm) : 0u);
                    mm &= mm - 1;   // (0 stays 0)
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = !on[i] ? 0u : (x ? __builtin_nontemporal_load(x + group0 + p[i]) : (uint32_t)group0 + p[i]);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (on[i] && k + i < out_cap) out[k + i] = v[i];
                k += 4;
            }
        }
        return;
    }
    uint64_t piece_base = wave_base;   // output index of the first selected entry of the piece at hand
#pragma unroll 1
    for (int c = 0; c < kPieces; ++c) {
        // the selected entries into LDS, shifted so that a 16-byte block there is one in `out`
        const uint32_t shift = (uint32_t)piece_base & 3u;
        const uint32_t pos0 = (uint32_t)(span + (uint64_t)c * kPieceElems) + 4u * lane;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t sel = pc.rank_sel[i] & 0xFu;
            const uint32_t at = (pc.rank_sel[i] >> 4) + shift;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if ((sel >> k) & 1u) piece_buf[at + (uint32_t)__popc(sel & ((1u << k) - 1u))] = x ? pc.w[i][k] : pos0 + 256u * i + k;
        }
        // entries of the piece: the rank of the last lane's last position, and that one
        const uint32_t last = pc.rank_sel[3];
        const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)((last >> 4) + (uint32_t)__popc(last & 0xFu)), 63);
        wave_lds_sync();
        if (c + 1 < kPieces) load_piece(c + 1);   // on its way while this one is stored
        const uint64_t out0 = piece_base - shift;   // a multiple of four
        const uint64_t stop = piece_base + cnt < out_cap ? piece_base + cnt : out_cap;
        for (uint32_t q = 4u * lane; q < shift + cnt; q += 256u) {
            const v4u v = *reinterpret_cast<const v4u *>(piece_buf + q);
            const uint64_t k = out0 + q;
            if (k >= piece_base && k + 4 <= stop) {
                *reinterpret_cast<v4u *>(out + k) = v;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (k + j >= piece_base && k + j < stop) out[k + j] = v[j];
            }
        }
        wave_lds_sync();   // read before the next piece overwrites it
        piece_base += cnt;
    }
}

// DIFF (Sec. 4.1): z(i) = x(i) - x(i-1) with x(-1) = 0, on int32 (wrap-around) or fp32.  The
// paper writes it as the product with the bidiagonal matrix D_s plus a vector fix of the block
// borders; here a lane takes four consecutive elements and gets the element before them from
// its neighbour lane (one extra load at the wave border).
// With `limit` the vector ends at min(n, *limit) (a count that an earlier kernel left on the device).
template <typename A>
__global__ __launch_bounds__(256) void diff_kernel(const uint32_t *__restrict__ x, uint64_t n, uint32_t *__restrict__ z,
                                                   const uint64_t *__restrict__ limit) {
    const int lane = threadIdx.x & 63;
    if (limit) {
        const uint64_t m = *limit;
        n = m < n ? m : n;
    }
    const uint64_t e0 = ((uint64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    v4u w = {0, 0, 0, 0};
    if (e0 + 4 <= n) {
        w = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(x + e0));
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (e0 + i < n) w[i] = x[e0 + i];
    }
    uint32_t prev = __shfl_up(w[3], 1);
    if (lane == 0) prev = (e0 > 0 && e0 - 1 < n) ? x[e0 - 1] : 0u;
    v4u o;
    o[0] = to_bits(from_bits<A>(w[0]) - from_bits<A>(prev));
#pragma unroll
    for (int i = 1; i < 4; ++i) o[i] = to_bits(from_bits<A>(w[i]) - from_bits<A>(w[i - 1]));
    if (e0 + 4 <= n) {
        __builtin_nontemporal_store(o, reinterpret_cast<v4u *>(z + e0));
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (e0 + i < n) z[e0 + i] = o[i];
    }
}

// REVERT (Sec. 4.1): z(i) = xhat(i) - w(fhat(i) - 2) where the inclusive count of segment
// starts fhat(i) is at least 2 (the printed index is read shifted by one: the first segment is
// left alone).  A count that points outside w subtracts nothing (there is no workspace to report it through;
// the compositions of this library only ever pass counts that COMPRESS has produced entries for).
template <typename A>
__global__ __launch_bounds__(256) void revert_kernel(const uint32_t *xhat, const int32_t *__restrict__ fhat,
                                                     const uint32_t *__restrict__ w, uint64_t n, uint64_t nw,
                                                     uint32_t *z) {
    const uint64_t e0 = ((uint64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (e0 >= n) return;
    v4u xv = {0, 0, 0, 0};
    v4i kv = {0, 0, 0, 0};
    const bool full = e0 + 4 <= n;
    if (full) {
        xv = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(xhat + e0));
        kv = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(fhat + e0));
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (e0 + i < n) {
                xv[i] = xhat[e0 + i];
                kv[i] = fhat[e0 + i];
            }
    }
    v4u o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        A v = from_bits<A>(xv[i]);
        const int64_t k = kv[i];
        if (k >= 2) {
            if ((uint64_t)(k - 2) < nw) v -= from_bits<A>(w[k - 2]);
        }
        o[i] = to_bits(v);
    }
    if (full) {
        __builtin_nontemporal_store(o, reinterpret_cast<v4u *>(z + e0));
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (e0 + i < n) z[e0 + i] = o[i];
    }
}

}  // namespace
