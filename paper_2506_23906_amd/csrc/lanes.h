// libmmvseg, part of the one translation unit mmvseg.hip (included there, in order).
// Lane-level helpers: bit casts, descriptor loads and stores, lane exchanges (DPP moves, permlane swap,
// shuffles), wave sums, the look-back over tile descriptors.
#pragma once

namespace {

// ---- small helpers -----------------------------------------------------------------------

template <typename T> __device__ __forceinline__ T from_bits(uint32_t b) { return __builtin_bit_cast(T, b); }
template <typename T> __device__ __forceinline__ uint32_t to_bits(T v) { return __builtin_bit_cast(uint32_t, v); }

// Orders LDS traffic between the lanes of one wave (no s_barrier needed: a wave's
// LDS instructions execute in order).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Buffer loads and stores: what lies at or beyond `bytes` reads 0 and is not written, without a branch.  (The whole offset has to be in
// the lane's own one: the scalar offset of these instructions is not part of that check.)  (What is loaded in a branch
// that not all lanes take is waited for before the next one: the branch that a lane does not take sets its registers.)
constexpr int kAuxNt = 2;   // non-temporal
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}

__device__ __forceinline__ uint64_t desc_load(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void desc_store(uint64_t *p, uint64_t status, uint32_t payload) {
    __hip_atomic_store(p, (status << 62) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Data-parallel-primitive move: every lane reads the lane the control word names (row_shr n = 0x110 + n
// inside rows of 16 lanes, row_bcast 15 / 31 = 0x142 / 0x143, wave_shr 1 = 0x138); a lane that has
// no source, or whose row of lanes is not in kRowMask, reads 0.
template <int kCtrl, int kRowMask> __device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, kRowMask, 0xF, false);
}

// Both halves of the wave, each broadcast to all 64 lanes: lo[l] = v[l mod 32], hi[l] = v[32 + l mod 32]
// (one v_permlane32_swap, no LDS hardware).
// Lane exchanges come in two forms: through the vector ALU (DPP moves, v_permlane32_swap) or through
// the LDS hardware (ds_bpermute: what __shfl compiles to).  The ALU form has a tenth of the latency and
// made the segmented sum 10 % faster; the scan kernels, which wait for memory anyway, ran 0.9 % slower
// with it (the extra ALU instructions compete with the address arithmetic of the stores) and keep the
// LDS form.  kAlu selects.
struct Halves {
    uint32_t lo, hi;
};
template <bool kAlu> __device__ __forceinline__ Halves wave_halves(uint32_t v, int lane) {
    if constexpr (kAlu) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return {(uint32_t)r[0], (uint32_t)r[1]};
    } else {
        const uint32_t o = __shfl_xor(v, 32);
        return {lane < 32 ? v : o, lane < 32 ? o : v};
    }
}

// Sum over the 64 lanes, the same value in every lane: DPP adds inside the rows of 16 lanes, row totals
// passed on with row_bcast 15 / 31, the total read from lane 63.
template <typename T, bool kAlu = true> __device__ __forceinline__ T wave_sum(T v) {
    if constexpr (!kAlu) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) v += from_bits<T>(__shfl_xor(to_bits(v), d));
        return v;
    }
    v += from_bits<T>(dpp_or_zero<0x111, 0xF>(to_bits(v)));
    v += from_bits<T>(dpp_or_zero<0x112, 0xF>(to_bits(v)));
    v += from_bits<T>(dpp_or_zero<0x114, 0xF>(to_bits(v)));
    v += from_bits<T>(dpp_or_zero<0x118, 0xF>(to_bits(v)));
    v += from_bits<T>(dpp_or_zero<0x142, 0xA>(to_bits(v)));
    v += from_bits<T>(dpp_or_zero<0x143, 0xC>(to_bits(v)));
    return from_bits<T>((uint32_t)__builtin_amdgcn_readlane((int)to_bits(v), 63));
}

// dpp_or_zero for values of 32 or 64 bits.
template <int kCtrl, int kRowMask, typename V> __device__ __forceinline__ V dpp_value(V v) {
    if constexpr (sizeof(V) == 8) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint64_t lo = dpp_or_zero<kCtrl, kRowMask>((uint32_t)b), hi = dpp_or_zero<kCtrl, kRowMask>((uint32_t)(b >> 32));
        return __builtin_bit_cast(V, (hi << 32) | lo);
    } else {
        return from_bits<V>(dpp_or_zero<kCtrl, kRowMask>(to_bits(v)));
    }
}
template <typename V> __device__ __forceinline__ V wave_last(V v) {   // lane 63's
    if constexpr (sizeof(V) == 8) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
        return __builtin_bit_cast(V, (hi << 32) | lo);
    } else {
        return from_bits<V>((uint32_t)__builtin_amdgcn_readlane((int)to_bits(v), 63));
    }
}

// Sums carried in 64 bits: the descriptor of a tile holds a double without its two last bits.
__device__ __forceinline__ void wide_store(uint64_t *p, uint64_t status, double v) {
    __hip_atomic_store(p, (status << 62) | (__builtin_bit_cast(uint64_t, v) >> 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T> __device__ __forceinline__ T desc_value(uint64_t d) { return from_bits<T>((uint32_t)d); }
template <> __device__ __forceinline__ double desc_value<double>(uint64_t d) { return __builtin_bit_cast(double, d << 2); }
__device__ __forceinline__ double wave_sum_wide(double v) {   // as wave_sum
    v += dpp_value<0x111, 0xF>(v);
    v += dpp_value<0x112, 0xF>(v);
    v += dpp_value<0x114, 0xF>(v);
    v += dpp_value<0x118, 0xF>(v);
    v += dpp_value<0x142, 0xA>(v);
    v += dpp_value<0x143, 0xC>(v);
    return wave_last(v);
}

// Sum of the payloads of the predecessor tiles back to (and including) the first one whose descriptor says "prefix".  Tile -1
// counts as prefix 0, so the loop always ends there at the latest.  The wave takes `lanes` descriptors at a time, and asks again only
// for those of them that are needed and still missing: every such read goes past the L2 to the memory side, where all tiles in
// flight ask for the same few lines, and there it costs more than the round trips that a wide window saves.  Scan of 1.5 * 10^8
// fp32 values: 217 us with windows of 64 asked for whole, 200 (64), 197 (32, 16) and 215 (8) with only the missing ones; without
// any look-back (wrong results) 194.  Segmented sum of 2^28 bytes 69.4 (64, whole), 67.6 (64), 65.5 (16).
// Where all tiles are resident at once they also publish at once, and a tile walks through all those before it: windows of 64 there
// (scan of 5.8 * 10^6 fp16 values 13.7, with windows of 16 15.8).
// The caller may have asked for the first window itself, some time ago (kPolled, lookback_poll).
#ifndef MMV_POLL_LANES
#define MMV_POLL_LANES 16
#endif
__device__ __forceinline__ int poll_lanes(uint32_t num_tiles, uint32_t first_round) { return num_tiles <= first_round ? 64 : MMV_POLL_LANES; }
__device__ __forceinline__ uint64_t lookback_poll(const uint64_t *desc, int tile, int lane, int lanes) {
    const int idx = tile - 1 - lane;
    return idx < 0 ? kStatusPrefix << 62 : lane < lanes ? desc_load(desc + idx) : 0;
}
template <typename T, bool kAlu = true, bool kPolled = false>
__device__ T lookback(const uint64_t *desc, int tile, int lane, int lanes, uint32_t *hdr, uint64_t polled = 0) {
    T carry = T(0);
    uint32_t spins = 0;
    int pos = tile - 1;
    uint64_t d = polled;
    bool ask = !kPolled && lane < lanes;
    while (true) {
        const int idx = pos - lane;
        if (ask) d = idx >= 0 ? desc_load(desc + idx) : kStatusPrefix << 62;
        const uint32_t st = (uint32_t)(d >> 62);
        const uint64_t stop = __ballot(lane < lanes && st == kStatusPrefix);
        const int first_stop = stop ? __ffsll((unsigned long long)stop) - 1 : lanes - 1;
        ask = lane <= first_stop && st == kStatusInvalid;
        if (__ballot(ask) != 0) {
            if (++spins > kMaxSpins) {
                if (lane == 0) __hip_atomic_store(hdr + kHdrError, kErrLookback, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            __builtin_amdgcn_s_sleep(2);
            continue;
        }
        const T v = lane <= first_stop ? desc_value<T>(d) : T(0);
        if constexpr (sizeof(T) == 8) carry += wave_sum_wide(v);
        else carry += wave_sum<T, kAlu>(v);
        if (stop) break;
        pos -= lanes;
        ask = lane < lanes;
    }
    return carry;
}

// Number of segment starts before span `span` of a tile (0: before the tile), from the counts per tile and (kUseSpans, or
// there is no table of them and `span` is 0) per span.  Wave-wide in two halves, so that the loads can go out ahead of others:
// the lane's part, and their sum.  A lane takes eight tiles (two 128-bit loads), so the wave covers 512 tiles before the
// first one of the tile's own group of eight; of that group it takes the spans (or tiles) before its own.
template <bool kUseSpans> __device__ __forceinline__ uint32_t starts_before_part(const Params &P, uint32_t tile, uint32_t span, int lane) {
    const uint32_t g = tile / kGroupTiles;
    uint32_t part = 0;
    if (P.count_is_prefix) {
        if (kUseSpans && lane < (int)span) part = P.span_count[tile * kSpans + lane];
        if (lane == 0) part += P.tile_count[tile];
        return part;
    }
    if constexpr (kUseSpans) {
        if (lane < (int)(tile % kGroupTiles * kSpans + span)) part = P.span_count[g * kGroupSpans + lane];
    } else {
        if (lane < (int)(tile % kGroupTiles)) part = P.tile_count[g * kGroupTiles + lane];
    }
    for (uint32_t i = lane; i < g; i += 128) {   // four loads under way at a time
        v4u a[4] = {};
#pragma unroll
        for (uint32_t j = 0; j < 2; ++j)
            if (i + 64 * j < g) {
                const v4u *t = reinterpret_cast<const v4u *>(P.tile_count + (i + 64 * j) * kGroupTiles);
                a[2 * j] = t[0];
                a[2 * j + 1] = t[1];
            }
#pragma unroll
        for (int j = 0; j < 4; ++j) part += (a[j][0] + a[j][1]) + (a[j][2] + a[j][3]);
    }
    return part;
}

}  // namespace
