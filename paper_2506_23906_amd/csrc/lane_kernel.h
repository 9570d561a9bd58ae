// libmmvseg, part of the one translation unit mmvseg.hip (included there, in order).
// The tile body of the scans of 32-bit values, and of some of 16-bit ones: a tile stays in registers, and its sums go from lane to lane.
#pragma once

namespace {

// ---- scans of 32-bit values ------------------------------------------------------------------------------------------
//
// The roles are those of seg_tile (aggregate, descriptor, look-back, carry, store), but there is no speculation to take back: a wave
// takes 256 elements at a time, four consecutive ones per lane as the 128-bit loads and stores have them, and the segmented pair goes
// from element to element inside a lane and from lane to lane by DPP moves, so a result depends on its own segment alone.
// The aggregate of a wave is the plain sum of what lies behind its last flag (a scalar position), which costs next to nothing, so a
// tile publishes it as soon as its loads have landed, and only then makes its results.  Nothing but the words that the waves exchange
// is in LDS.  (Row scans on the matrix cores need every value split three ways, the operand layout and the results moved
// through LDS, and 112 registers of which a wave's values are 32: they took longer in both variants, which share this kernel.)
// Sums are carried in 64 bits from lane to lane, from block to block and between tiles (wide_store); a result is rounded when the
// carry into a lane is, and when it is added.  Error against 64 bits (2-norms), row scans -> now: 1 of 27 starts 6.8e-8 -> 5.0e-8, no
// flags 2.2e-7 -> 3.9e-8; a start receives its input bit for bit.
// Inside a lane, neighbours may overflow 32 bits where no prefix does (a segment that goes on from -3e38 over 2e38 and 2e38).  A wave that
// holds values that large (LaneRaw::Large, asked while its loads arrive) adds up in 64 throughout, its aggregate a second time.  What
// asking costs: 3 * 10^6 values, 4 % starts 9.5 us the call with and without, 1.5 * 10^8 without flags 204.7 -> 205.1, 2^27 of three kinds of
// segments 178.9 -> 180.9.  (Sums in 64 bits for every wave: 3 * 10^6 values 10.0, 8.2 * 10^6 14.2 -> 15.0.)
// What bounds it: the memory, at its rate for as much read as written (fp32: every byte moved once at 5.9 to 6.2 TB/s, vector pipes 25 to 40 %
// busy; one round of 16-bit values: 5.0 TB/s and 39 %, a wave lives 13.5 us of the kernel's 24.6).  Whole calls, the reset launch of 5 us included, row scans in LDS
// (matrix cores) -> now: 2^27 values, half of them starts, a quarter one segment, the rest in short segments 197 -> 181 us; 1.5 * 10^8 in
// segments of 80 214 -> 196 (6.4 TB/s without the reset), 5.2 * 10^7 without flags 83 -> 72; 8.2 * 10^6 21 -> 17; mmv_scan of 5 * 10^7 77.5 -> 72.7, 1.5 * 10^8 217 -> 199.
// 1.5 * 10^8 starts 193 -> 196: the row scans stored a chunk of starts as it was loaded.
// Tiles: 8 blocks per wave and three workgroups per compute unit (16 and two: lengths up to 2000, 9 * 10^7 127 us against 123; eight
// waves per SIMD: 3 % slower); without flags every tile waits for all those before it, and longer ones pay: 16 blocks (5 * 10^7 72 us; 8: 76, 24: 75).
// Conditions on blocks are made anew in each pass: hoisted, they took a pair of scalar registers each, and 15 to 83 of those spilled.
// 16-bit values (segmented scans that fill 512 to 768 workgroups, round_form in host.h): 64-bit loads, so that a lane's four results are
// one store; their results are rounded once, from 64 bits.  70 to 78 registers, where the form with row scans on the matrix cores needs
// more than the 80 that three workgroups per compute unit leave: fp16 20 * 10^6 28.5 -> 24.8 us the call.

constexpr int kBlockElems = 256;                             // four consecutive elements per lane
constexpr int kChunkBlocks = kChunkElems / kBlockElems;

template <int kWaves> struct LaneShared {
    double wave_v[kWaves], carry;
    uint32_t wave_f[kWaves];
    uint32_t tile, ready, arrived;
};

// Lanes that must not take the value of the lane 1, 2, 4, 8 before them, of lane 15 of the row of lanes before theirs, of lane 31: a
// flagged lane lies between.  (Scalars.)
struct ScanMasks {
    uint64_t shr1, shr2, shr4, shr8, bcast15, bcast31;
};
__device__ __forceinline__ ScanMasks scan_masks(uint64_t m) {   // m: the lanes that hold a flag
    constexpr uint64_t kRow = 0x0001000100010001ull;            // first lanes of the rows of 16
    ScanMasks k;
    k.shr1 = m;
    k.shr2 = k.shr1 | ((k.shr1 << 1) & ~kRow);
    k.shr4 = k.shr2 | ((k.shr2 << 2) & ~(kRow * 0x3));
    k.shr8 = k.shr4 | ((k.shr4 << 4) & ~(kRow * 0xF));
    k.bcast15 = (k.shr8 | ((k.shr8 << 8) & ~(kRow * 0xFF))) | 0x0000FFFF0000FFFFull;   // (rows 0 and 2 take nothing)
    const uint32_t hi = (uint32_t)(m >> 32);
    k.bcast31 = ((uint64_t)(hi ? ~0u << __builtin_ctz(hi) : 0u) << 32) | 0xFFFFFFFFull;
    return k;
}
template <int kCtrl, typename V> __device__ __forceinline__ V dpp_bound(V v) {   // a lane without a source reads 0
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, kCtrl, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), kCtrl, 0xF, 0xF, true);
    return __builtin_bit_cast(V, ((uint64_t)hi << 32) | lo);
}
// (what is left of a double without its upper half is below 2^-1042: nothing, once rounded)
__device__ __forceinline__ double unless(uint64_t blocked, double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t hi = __builtin_amdgcn_inverse_ballot_w64(blocked) ? 0u : (uint32_t)(b >> 32);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | (uint32_t)b);
}
// Inclusive scan over the 64 lanes, restarted at the lanes that hold a flag (kFlagged).
template <bool kFlagged> __device__ __forceinline__ double lane_scan(double v, const ScanMasks &k) {
    constexpr uint64_t kOdd = 0x0000FFFF0000FFFFull, kUpper = 0xFFFFFFFFull;
    double o;
    o = dpp_bound<0x111>(v); v = (kFlagged ? unless(k.shr1, o) : o) + v;
    o = dpp_bound<0x112>(v); v = (kFlagged ? unless(k.shr2, o) : o) + v;
    o = dpp_bound<0x114>(v); v = (kFlagged ? unless(k.shr4, o) : o) + v;
    o = dpp_bound<0x118>(v); v = (kFlagged ? unless(k.shr8, o) : o) + v;
    o = dpp_bound<0x142>(v); v = unless(kFlagged ? k.bcast15 : kOdd, o) + v;
    o = dpp_bound<0x143>(v); v = unless(kFlagged ? k.bcast31 : kUpper, o) + v;
    return v;
}

// The four values of a lane in a block, as loaded, and what lies from `valid` on cleared.
// Large: whether any of the values looked at is 2^125 or more in magnitude (or a NaN).  Four values below that do not overflow 32 bits,
// and fp16 ones never do.  bf16 values are compared as whole numbers: their bits grow with them, those of a negative one as unsigned ones.
template <typename In> struct LaneRaw {
    typedef v2u type;
    typedef int16_t v2i16 __attribute__((ext_vector_type(2)));
    typedef uint16_t v2u16 __attribute__((ext_vector_type(2)));
    static constexpr bool kMayOverflow = std::is_same_v<In, typename TBF16::in_t>;
    struct Large {
        v2i16 up = 0;
        v2u16 down = 0;
        __device__ __forceinline__ void add(const type &w) {
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                up = __builtin_elementwise_max(up, __builtin_bit_cast(v2i16, (uint32_t)w[d]));
                down = __builtin_elementwise_max(down, __builtin_bit_cast(v2u16, (uint32_t)w[d]));
            }
        }
        __device__ __forceinline__ bool any() const { return up.x >= 0x7E00 || up.y >= 0x7E00 || down.x >= 0xFE00 || down.y >= 0xFE00; }
    };
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, int at) { return __builtin_amdgcn_raw_buffer_load_b64(r, at, 0, kAuxNt); }
    static __device__ __forceinline__ void mask(type &w, int valid) {
#pragma unroll
        for (int d = 0; d < 2; ++d) w[d] = valid >= 2 * d + 2 ? w[d] : valid > 2 * d ? w[d] & 0xFFFFu : 0u;
    }
};
template <> struct LaneRaw<float> {
    typedef v4u type;
    static constexpr bool kMayOverflow = true;
    struct Large {
        float m = 0.0f;
        __device__ __forceinline__ void add(const type &w) {
#pragma unroll
            for (int d = 0; d < 4; ++d) m = __builtin_elementwise_maximum(m, fabsf(from_bits<float>(w[d])));
        }
        __device__ __forceinline__ bool any() const { return !(m < 0x1p125f); }   // (a NaN stays one)
    };
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, int at) { return __builtin_amdgcn_raw_buffer_load_b128(r, at, 0, kAuxNt); }
    static __device__ __forceinline__ void mask(type &w, int valid) {
#pragma unroll
        for (int d = 0; d < 4; ++d) w[d] = valid > d ? w[d] : 0u;
    }
};
template <typename TT> __device__ __forceinline__ float lane_value(const typename LaneRaw<typename TT::in_t>::type &w, int i) {
    typedef typename TT::in_t In;
    if constexpr (sizeof(In) == 4) return from_bits<float>(w[i]);
    else return TT::widen(__builtin_bit_cast(In, (uint16_t)(w[i / 2] >> (16 * (i & 1)))));
}
// Carry into a lane plus a sum inside it.  16-bit values, and sums in 64 bits: added in 64 bits, one rounding.
template <typename TT, typename Sum> struct LaneCarry {
    double e;
    __device__ __forceinline__ float plus(Sum p) const { return (float)(e + (double)p); }
};
template <> struct LaneCarry<InLanes<TF32>, float> {
    float e;
    __device__ __forceinline__ explicit LaneCarry(double v) : e((float)v) {}
    __device__ __forceinline__ float plus(float p) const { return e + p; }
};
__device__ __forceinline__ double wave_first(double v) {   // of a value that is the same in all lanes: in scalar registers
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return __builtin_bit_cast(double, (hi << 32) | lo);
}

// One tile.  A wave holds its whole span in registers: block b of lane l = its elements 256 b + 4 l .. + 3.
template <typename TT, int kOp>
__device__ __forceinline__ void lane_tile(const Params &P, LaneShared<TT::kWaves> &sm, const uint32_t tile) {
    typedef typename TT::in_t In;
    constexpr int kWaves = TT::kWaves;
    constexpr int kCpw = lane_cpw<TT, kOp>();
    typedef LaneRaw<In> Raw;
    constexpr int kBlocks = kCpw * kChunkBlocks;
    constexpr bool kFlags = kOp == kScan;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const TileSpan span = tile_span(P.reg, tile, kWaves * kChunkElems);
    const uint32_t span_elems = span.cpw * kChunkElems;
    const uint64_t wave_base = span.base + (uint64_t)wave * span_elems;
    const uint64_t left = wave_base < P.n ? P.n - wave_base : 0;
    const int cnt = left < span_elems ? (int)left : (int)span_elems;      // elements of my span

    // Buffer loads: what lies at or beyond cnt reads 0, without a branch (the 16-byte block of the last element is read whole).
    const auto x_rsrc = make_rsrc((const In *)P.x + wave_base, (uint32_t)((cnt * (int)sizeof(In) + 15) & ~15));
    uint32_t F[kCpw] = {};
    typename Raw::type raw[kBlocks];
    int from_x = 4 * (int)sizeof(In) * lane, own = 16 * lane;   // my byte offsets in a block of values and of results
    asm volatile("" : "+v"(from_x));
    asm volatile("" : "+v"(own));   // (as an unknown, here and at the stores, so that the offset of a block is added by the
                                     // instruction itself and not kept in a register from the start on)
    if constexpr (kFlags) {
        const auto f_rsrc = make_rsrc(P.fw + (wave_base >> 5), (uint32_t)((cnt + 31) / 32 * 4));
#pragma unroll
        for (int c = 0; c < kCpw; ++c) F[c] = __builtin_amdgcn_raw_buffer_load_b32(f_rsrc, 4 * lane + 256 * c, 0, kAuxNt);
    }
#pragma unroll
    for (int b = 0; b < kBlocks; ++b) raw[b] = Raw::load(x_rsrc, from_x + kBlockElems * (int)sizeof(In) * b);
#if MMV_LOAD_PRIO
    __builtin_amdgcn_s_setprio(0);
#endif
    if (cnt % 32 != 0) {   // (the end of the vector)
#pragma unroll
        for (int c = 0; c < kCpw; ++c) {
            const int valid = cnt - kChunkElems * c - 32 * lane;
            if (valid < 32) F[c] = valid > 0 ? F[c] & ((1u << valid) - 1u) : 0u;
        }
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) Raw::mask(raw[b], cnt - kBlockElems * b - 4 * lane);
    }
    // flags of the span: rows of 32 with any, first and last position (scalars)
    uint64_t any[kCpw];
    int first = kBlocks * kBlockElems, last = -1;
#pragma unroll
    for (int c = 0; c < kCpw; ++c) {
        any[c] = kFlags ? __ballot(F[c] != 0) : 0;
        if (any[c]) {
            const int hi = 63 - __builtin_clzll(any[c]);
            last = kChunkElems * c + 32 * hi + 31 - __builtin_clz((uint32_t)__builtin_amdgcn_readlane((int)F[c], hi));
        }
    }
#pragma unroll
    for (int c = kCpw - 1; c >= 0; --c)
        if (any[c]) {
            const int lo = __builtin_ctzll(any[c]);
            first = kChunkElems * c + 32 * lo + __builtin_ctz((uint32_t)__builtin_amdgcn_readlane((int)F[c], lo));
        }

    // ---- aggregate: the sum of the span from its last flag on ----
    double s = 0.0;
    bool large = false;   // sums inside a lane may overflow 32 bits where no prefix does
    if (__builtin_expect(last >= 0, 1)) {
        if constexpr (Raw::kMayOverflow) {
            typename Raw::Large l;
#pragma unroll
            for (int b = 0; b < kBlocks; ++b) l.add(raw[b]);
            large = __ballot(l.any()) != 0;
        }
#pragma unroll
        for (int b = 0; b < kBlocks; ++b)
            if (last < kBlockElems * (b + 1)) {
                const int k = last - kBlockElems * b - 4 * lane;   // my elements from k on count
                float t[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) t[i] = i >= k ? lane_value<TT>(raw[b], i) : 0.0f;
                s += (double)((t[0] + t[1]) + (t[2] + t[3]));
            }
    } else {
#pragma unroll
        for (int b = 0; b < kBlocks; ++b)
            s += (double)((lane_value<TT>(raw[b], 0) + lane_value<TT>(raw[b], 1)) + (lane_value<TT>(raw[b], 2) + lane_value<TT>(raw[b], 3)));
        if constexpr (Raw::kMayOverflow) {
            typename Raw::Large l;
#pragma unroll
            for (int b = 0; b < kBlocks; ++b) l.add(raw[b]);
            large = __ballot(l.any()) != 0;
        }
    }
    s = wave_sum_wide(s);
    if constexpr (Raw::kMayOverflow) {
        if (large) {   // (a second time, in 64 bits)
            s = 0.0;
#pragma unroll
            for (int b = 0; b < kBlocks; ++b) {
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("" : "+v"(raw[b]));
#pragma unroll
                for (int i = 0; i < 4; ++i) s += kBlockElems * b + 4 * lane + i >= last ? (double)lane_value<TT>(raw[b], i) : 0.0;
            }
            s = wave_sum_wide(s);
        }
    }
    if (lane == 0) {
        sm.wave_v[wave] = s;
        sm.wave_f[wave] = last >= 0;
    }
    __syncthreads();
    double wex_v = 0.0, tagg_v = 0.0;
    uint32_t wex_f = 0, tagg_f = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        if (w == wave) {
            wex_v = tagg_v;
            wex_f = tagg_f;
        }
        const double wv = sm.wave_v[w];
        const uint32_t wf = sm.wave_f[w];
        tagg_v = wf ? wv : tagg_v + wv;
        tagg_f |= wf;
    }
    wex_f = __builtin_amdgcn_readfirstlane(wex_f);
    tagg_f = __builtin_amdgcn_readfirstlane(tagg_f);
    if constexpr (sizeof(In) == 2) {   // (two chunks of bf16 values spill without; fp32 ones have the room, and are up to 4 % faster)
        wex_v = wave_first(wex_v);
        tagg_v = wave_first(tagg_v);
    }
    const bool final_now = tile == 0 || tagg_f;   // carry out does not depend on predecessors
    if (tid == 0) wide_store(P.desc_v + tile, final_now ? kStatusPrefix : kStatusAggregate, tagg_v);

    const auto z_rsrc = make_rsrc((float *)P.z + wave_base, 4u * (uint32_t)cnt);
    // ---- results: blocks behind the first flag of the span first, the others once the carry of the tiles before is known ----
    const bool closed = wex_f || tile == 0;       // the carry into the span is known already
    const int first_block = first / kBlockElems;
    double run = wex_v;                           // carry into the block at hand
#pragma unroll 1
    for (int pass = closed ? 1 : 0; pass < 2; ++pass) {
        // (or the compiler makes the sums of every block ahead of the loop, and keeps them)
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) asm volatile("" : "+v"(raw[b]));
        // (... nor the conditions: a pair of scalar registers each, and the scalar registers did not suffice)
        int end = cnt;
        asm volatile("" : "+s"(end));
        uint64_t rows[kCpw];
#pragma unroll
        for (int c = 0; c < kCpw; ++c) {
            rows[c] = any[c];
            asm volatile("" : "+s"(rows[c]));
        }
        int from = 0, upto = closed ? kBlocks : first_block + 1, store_from = 0;
        if (pass == 0) from = first_block, upto = kBlocks, store_from = first_block + 1;   // (of the block of that flag: what it carries on)
        if (pass == 1 && !closed) {
            double tile_carry = 0.0;
            if (wave == 0) {
                if (first != 0 || !final_now) tile_carry = lookback<double>(P.desc_v, (int)tile, lane, poll_lanes(P.num_tiles, P.first_round), P.hdr);
                if (lane == 0) {
                    if (!final_now) wide_store(P.desc_v + tile, kStatusPrefix, tile_carry + tagg_v);
                    sm.carry = tile_carry;
                    __hip_atomic_store(&sm.ready, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            } else {
                while (__hip_atomic_load(&sm.ready, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) == 0)
                    __builtin_amdgcn_s_sleep(1);
                tile_carry = sm.carry;
            }
            run = tile_carry + wex_v;
        }
        auto blocks = [&](auto zero) {
            typedef decltype(zero) Sum;
#pragma unroll
            for (int b = 0; b < kBlocks; ++b) {
                const int c = b / kChunkBlocks, j = b % kChunkBlocks;
                __builtin_amdgcn_sched_barrier(0);
                if (b < from || b >= upto || kBlockElems * b >= end) continue;
                const float x0 = lane_value<TT>(raw[b], 0), x1 = lane_value<TT>(raw[b], 1), x2 = lane_value<TT>(raw[b], 2), x3 = lane_value<TT>(raw[b], 3);
                float o[4];
                if (!kFlags || ((rows[c] >> (8 * j)) & 0xFFull) == 0) {
                    const Sum p0 = x0, p1 = p0 + x1, p2 = p1 + x2, p3 = p2 + x3;
                    const double inc = lane_scan<false>((double)p3, ScanMasks{});
                    const LaneCarry<TT, Sum> ec{run + dpp_bound<0x138>(inc)};   // wave_shr 1: lane 0 gets 0
                    run += wave_last(inc);
                    o[0] = ec.plus(p0);
                    o[1] = ec.plus(p1);
                    o[2] = ec.plus(p2);
                    o[3] = ec.plus(p3);
                } else {
                    // (F[c] holds row l of the chunk in lane l: a lane needs four bits of row 8 j + l / 8)
                    const uint32_t word = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (8 * j + (lane >> 3)), (int)F[c]);
                    const uint32_t nib = (word >> (4 * (lane & 7))) & 0xFu;
                    const Sum p0 = x0, p1 = (nib & 2u) ? (Sum)x1 : p0 + x1, p2 = (nib & 4u) ? (Sum)x2 : p1 + x2, p3 = (nib & 8u) ? (Sum)x3 : p2 + x3;
                    const uint64_t m = __ballot(nib != 0);
                    const double inc = lane_scan<true>((double)p3, scan_masks(m));
                    double e = dpp_bound<0x138>(inc);
                    const uint64_t upto_first = (m & (0 - m)) | ((m & (0 - m)) - 1);   // lanes without a flag in a lane before them
                    e += unless(~upto_first, run);
                    const LaneCarry<TT, Sum> ec{e};
                    run = wave_last(inc);
                    o[0] = (nib & 1u) ? x0 : ec.plus(p0);
                    o[1] = (nib & 3u) ? (float)p1 : ec.plus(p1);
                    o[2] = (nib & 7u) ? (float)p2 : ec.plus(p2);
                    o[3] = nib ? (float)p3 : ec.plus(p3);
                    if constexpr (sizeof(Sum) == 8) {   // (a NaN that starts a segment, bit for bit)
                        o[1] = (nib & 2u) ? x1 : o[1];
                        o[2] = (nib & 4u) ? x2 : o[2];
                        o[3] = (nib & 8u) ? x3 : o[3];
                    }
                }
                if (b >= store_from) {
                    asm volatile("" : "+v"(own));
                    const v4u w = {to_bits(o[0]), to_bits(o[1]), to_bits(o[2]), to_bits(o[3])};
                    if (kBlockElems * (b + 1) <= end) {
                        __builtin_amdgcn_raw_buffer_store_b128(w, z_rsrc, own + 1024 * b, 0, kAuxNt);
                    } else {
                        float *z = (float *)P.z + wave_base;
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (own / 4 + kBlockElems * b + i < end) z[own / 4 + kBlockElems * b + i] = o[i];
                    }
                }
            }
        };
        if (Raw::kMayOverflow && large) blocks(0.0);
        else blocks(0.0f);
    }
}

}  // namespace
