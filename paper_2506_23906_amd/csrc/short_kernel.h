// libmmvseg, part of the one translation unit mmvseg.hip (included there, in order).
// Scans and sums of short vectors: kernels without tickets, look-back or anything that has to be zeroed first.
#pragma once

namespace {

// ---- short vectors ------------------------------------------------------------------------------------------------
//
// A call on a short vector is bound by launches and by the life of one workgroup, not by memory or arithmetic.  The
// single-pass kernels need a launch ahead of them (descriptors have to be zero), and a tile of theirs lives 6 us.
// Here a workgroup takes 2048 elements, eight consecutive ones per thread, and the sum carried into a tile comes
//   from the input itself (kSingle; one launch): every workgroup looks for the last segment start before its tile in the
//     flags, and adds up the values from there on.  All workgroups do that at once, and the L2s serve the reads;
//   from the aggregates of the tiles before it (two launches), which short_reduce_kernel has left: a workgroup reads them
//     all (at most 16 KB).
// The segmented pair is carried from element to element inside a thread and from lane to lane by DPP moves: no speculation,
// so both variants of a call take the same kernels (a 32x32 product and its way through LDS would only add latency), and a
// result depends on its own segment alone.
// Measured, whole calls one after the other, before -> one launch / two (us; before: two launches, or one up to 16384
// elements of a scan with packed flags or none):
//   segmented scan, fp32, byte flags, 1 of 64 set    3000: 8.1 -> 4.4 / 6.5    65536: 8.8 -> 4.4 / 6.3    2^20: 10.0 -> - / 6.6
//   ... no flags, packed                             3000: 5.9 -> 4.2 / 6.3    65536: 7.8 -> 6.2 / 6.5    2^21: 10.8 -> - / 8.2
//   segmented sum, fp16, packed, 1 of 1024 set       3000: 7.3 -> 4.7 / 6.9    131072: 8.0 -> 4.7 / 6.9   2^21: 8.2 -> - / 7.7
//   scan, fp32                                       3000: 7.3 -> 4.0 / 6.3    65536: 10.0 -> 4.7 / 6.1   2^22: 14.2 -> - / 11.9
// Where the lines lie.  One launch: a workgroup alone reads its L2 at some 150 GB/s, so with the whole input before the last
// tile to be read (a vector without flags) one launch takes as long as two from about 320 KB of values and flags on (fp32
// values: 65536 6.2 against 6.5 us, 131072 9.9 against 6.5; with flags every hundred elements one launch takes 4.3 there).
// Two launches: up to 2^21 elements everything gains (segmented scan of bytes 9.9 -> 7.8).  Beyond, where the data read twice
// shows, with the inputs of several calls in turn: scans without flags of 3.3 million and 2^22, fp32 13.5 -> 11.1 and 13.8 -> 13.0,
// bytes 11.6 -> 9.3 and 11.7 -> 11.0, 16-bit 11.5 -> 10.1 and 11.9 -> 12.3; fp32 sums with 1 of 1000 set 10.8 -> 10.8 and 11.3 ->
// 12.0, with 1 of 5 13.0 -> 11.9 and 13.3 -> 13.2: so 16-bit scans and fp32 sums up to 3 * 2^20, the other scans up to 2^22.
// Segmented scans (2^22: 11.6 -> 11.9, bytes 10.8 -> 11.2) and sums of bytes stay at 2^21.  Four elements per thread: level up to 2^19, 10 %
// slower at 2^21; sixteen: 20 % slower there.
constexpr int kShortThreads = 256, kShortWaves = kShortThreads / 64;
constexpr int kShortElems = 8;                                  // consecutive elements of a thread
constexpr uint32_t kShortTile = kShortThreads * kShortElems;
#ifndef MMV_SINGLE_BYTES
#define MMV_SINGLE_BYTES (320u << 10)   // most values and flags, in bytes, of a vector that one launch takes
#endif
#ifndef MMV_SHORT_MAX
#define MMV_SHORT_MAX (1u << 21)        // most elements that two launches take
#endif
constexpr uint64_t short_max(mmv_op op, mmv_dtype dt) {
    const uint64_t n = MMV_SHORT_MAX;
    if (op == MMV_OP_SCAN) return dt == MMV_F16_F32 || dt == MMV_BF16_F32 ? n / 2 * 3 : 2 * n;
    return op == MMV_OP_SEGSUM && dt == MMV_F32_F32 ? n / 2 * 3 : n;
}

enum ShortFlags { kNoFlags = 0, kBitFlags = 1, kByteFlags = 2 };

struct ShortParams {
    const void *x;
    const void *flags;
    void *z;               // scan output, or ...
    void *out;             // ... the sums, their number at most out_cap
    uint64_t out_cap;
    uint64_t *nseg;
    uint32_t *hdr;         // workspace header: the status word and the mark of a plan are cleared
    uint64_t *agg;         // (two launches) one aggregate per tile: sum after the last segment start, number of starts << 32
    uint32_t n;
    uint32_t first_one;    // scan of flag bytes: element 0 counts as 1 whatever it holds
};

// kShortElems consecutive elements from e0 on, as loaded.  The 16-byte block of the last element is not left.
template <typename TT> struct ShortRaw {
    static constexpr int kWords = (kShortElems + TT::kEpl - 1) / TT::kEpl;
    v4u w[kWords];
    __device__ __forceinline__ void load(const void *x, uint32_t e0, uint32_t n) {
        const char *p = (const char *)x + (uint64_t)e0 * sizeof(typename TT::in_t);
#pragma unroll
        for (int j = 0; j < kWords; ++j) w[j] = v4u{0, 0, 0, 0};
        if constexpr (TT::kEpl > kShortElems) {   // bytes: half a block
            if (e0 < n) {
                const v2u v = *(const v2u *)p;
                w[0][0] = v[0];
                w[0][1] = v[1];
            }
        } else {
#pragma unroll
            for (int j = 0; j < kWords; ++j)
                if (e0 + (uint32_t)(TT::kEpl * j) < n) w[j] = *(const v4u *)(p + 16 * j);
        }
    }
    __device__ __forceinline__ typename TT::acc_t elem(int i) const { return raw_elem<TT>(w[i / TT::kEpl], i % TT::kEpl); }
};

// Flags of the elements e0 .. e0 + kShortElems - 1, bit i for element e0 + i; none at or beyond n.
template <int kFlags> __device__ __forceinline__ uint32_t short_flags(const void *flags, uint32_t e0, uint32_t n) {
    uint32_t f = 0;
    if (kFlags == kNoFlags || e0 >= n) return 0;
    if constexpr (kFlags == kBitFlags) {
        f = (((const uint32_t *)flags)[e0 >> 5] >> (e0 & 31u)) & ((1u << kShortElems) - 1u);
    } else if constexpr (kFlags == kByteFlags) {
#pragma unroll
        for (int d = 0; d < kShortElems / 4; ++d) {
            const uint32_t w = ((const uint32_t *)((const uint8_t *)flags + e0))[d];
            const uint32_t nz = ((((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) >> 7) & 0x01010101u;
            f |= ((nz * 0x10204080u) >> 28) << (4 * d);
        }
    }
    if (n - e0 < (uint32_t)kShortElems) f &= (1u << (n - e0)) - 1u;
    return f;
}

// Sums are carried in 64 bits where the results are floats and rounded once, at the end: a vector this short pays nothing for
// it, and the error is that of the last rounding (segmented scan of 65536 values, 1 of 64 a start: 3.0e-8 against 6.5e-8 of the
// row scans in 32 bits; in 32 bits the lanes' scans here would come to 8.1e-8).  The aggregates of the tiles are kept in 32.
template <typename A> struct Wide {
    typedef A type;
};
template <> struct Wide<float> {
    typedef double type;
};
template <int kCtrl, int kRowMask, typename V> __device__ __forceinline__ V dpp_value(V v) {   // dpp_or_zero for 32 or 64 bits
    if constexpr (sizeof(V) == 8) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint64_t lo = dpp_or_zero<kCtrl, kRowMask>((uint32_t)b), hi = dpp_or_zero<kCtrl, kRowMask>((uint32_t)(b >> 32));
        return __builtin_bit_cast(V, (hi << 32) | lo);
    } else {
        return from_bits<V>(dpp_or_zero<kCtrl, kRowMask>(to_bits(v)));
    }
}

// Sum of the elements in one 128-bit word (floats in 64 bits from the first addition on: neighbours may cancel, or overflow 32).
template <typename TT> __device__ __forceinline__ typename Wide<typename TT::acc_t>::type word_sum(const v4u &w) {
    typedef typename TT::acc_t A;
    typedef typename Wide<A>::type V;
    if constexpr (TT::kDtype == MMV_I8_I32) {
        int s = 0;
#pragma unroll
        for (int d = 0; d < 4; ++d) s = __builtin_amdgcn_sdot4((int)w[d], 0x01010101, s, false);
        return A((uint32_t)s);
    } else if constexpr (TT::kDtype == MMV_U8_XOR) {
        uint32_t x = w[0] ^ w[1] ^ w[2] ^ w[3];
        x ^= x >> 16;
        x ^= x >> 8;
        return A(x & 0xFFu);
    } else {
        V s[2] = {V(raw_elem<TT>(w, 0)), V(raw_elem<TT>(w, 1))};
#pragma unroll
        for (int i = 2; i < TT::kEpl; ++i) s[i & 1] += V(raw_elem<TT>(w, i));
        return s[0] + s[1];
    }
}

// Segmented inclusive scan over the 64 lanes of (sum after the last start, number of starts); kFlagged: any starts at all.
template <bool kFlagged, typename V> __device__ __forceinline__ void wave_segmented_scan(V &v, uint32_t &c) {
#define MMV_SCAN_STEP(CTRL, ROWS)                           \
    {                                                       \
        const V ov = dpp_value<CTRL, ROWS>(v);              \
        if (!kFlagged || !c) v = ov + v;                    \
        if (kFlagged) c += dpp_or_zero<CTRL, ROWS>(c);      \
    }
    MMV_SCAN_STEP(0x111, 0xF)
    MMV_SCAN_STEP(0x112, 0xF)
    MMV_SCAN_STEP(0x114, 0xF)
    MMV_SCAN_STEP(0x118, 0xF)
    MMV_SCAN_STEP(0x142, 0xA)
    MMV_SCAN_STEP(0x143, 0xC)
#undef MMV_SCAN_STEP
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#define MMV_MAX_STEP(CTRL, ROWS)                            \
    {                                                       \
        const uint32_t o = dpp_or_zero<CTRL, ROWS>(v);      \
        v = v > o ? v : o;                                  \
    }
    MMV_MAX_STEP(0x111, 0xF)
    MMV_MAX_STEP(0x112, 0xF)
    MMV_MAX_STEP(0x114, 0xF)
    MMV_MAX_STEP(0x118, 0xF)
    MMV_MAX_STEP(0x142, 0xA)
    MMV_MAX_STEP(0x143, 0xC)
#undef MMV_MAX_STEP
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// What a thread knows of its own elements.
template <typename TT> struct ShortOwn {
    typedef typename TT::acc_t A;
    typedef typename Wide<A>::type V;
    V inc[kShortElems];      // running sums inside the thread, restarted at the flags
    uint32_t F, C;           // flags (position 0 of the vector always one); those that are counted (position 0 never)
    V ex_v, tot_v;           // sum carried into the thread inside its wave, aggregate of the wave (lane 63)
    uint32_t ex_c, tot_c;
    template <int kFlags> __device__ __forceinline__ void scan(const ShortRaw<TT> &raw, uint32_t flags, uint32_t e0, uint32_t n, uint32_t first_one) {
        C = e0 == 0 ? flags & ~1u : flags;
        F = e0 == 0 ? flags | 1u : flags;
        V run = V(0);
#pragma unroll
        for (int i = 0; i < kShortElems; ++i) {
            V v = V(raw.elem(i));
            if constexpr (kFlags == kNoFlags && TT::kDtype == MMV_I8_I32) {
                if (i == 0 && e0 == 0 && first_one) v = V(1);
            }
            if (e0 + (uint32_t)i >= n) v = V(0);   // (the rest of the last block that was read)
            run = i == 0 || (kFlags != kNoFlags && ((F >> i) & 1u)) ? v : run + v;
            inc[i] = run;
        }
        tot_v = run;
        tot_c = __popc(C);
        const uint32_t mine = tot_c;
        wave_segmented_scan<kFlags != kNoFlags>(tot_v, tot_c);
        ex_v = dpp_value<0x138, 0xF>(tot_v);   // wave_shr 1: lane 0 gets 0
        ex_c = tot_c - mine;
    }
};

// First of two launches: the aggregate of every tile.
template <typename TT, int kFlags> __global__ __launch_bounds__(kShortThreads) void short_reduce_kernel(ShortParams P) {
    typedef typename TT::acc_t A;
    typedef typename Wide<A>::type V;
    __shared__ V s_v[kShortWaves];
    __shared__ uint32_t s_c[kShortWaves];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, e0 = blockIdx.x * kShortTile + kShortElems * tid;
    const uint32_t flags = short_flags<kFlags>(P.flags, e0, P.n);
    ShortRaw<TT> raw;
    raw.load(P.x, e0, P.n);
    ShortOwn<TT> own;
    own.template scan<kFlags>(raw, flags, e0, P.n, P.first_one);
    if (lane == 63) {
        s_v[wave] = own.tot_v;
        s_c[wave] = own.tot_c;
    }
    __syncthreads();
    if (tid == 0) {
        V v = V(0);
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < kShortWaves; ++w) {
            v = s_c[w] ? s_v[w] : v + s_v[w];
            c += s_c[w];
        }
        P.agg[blockIdx.x] = ((uint64_t)c << 32) | to_bits(A(v));
        if (blockIdx.x == 0) P.hdr[kHdrError] = P.hdr[kHdrPrepared] = 0;
    }
}

// The only launch (kSingle), or the second of two.
template <typename TT, int kOp, int kFlags, bool kSingle>
__global__ __launch_bounds__(kShortThreads) void short_kernel(ShortParams P) {
    typedef typename TT::acc_t A;
    typedef typename Wide<A>::type V;
    constexpr bool kFlagged = kFlags != kNoFlags;
    constexpr uint32_t kEpl = TT::kEpl;
    __shared__ V s_v[kShortWaves], s_pv[kShortWaves];            // of the waves: their aggregates, their part of what lies before the tile
    __shared__ uint32_t s_c[kShortWaves], s_pc[kShortWaves], s_pl[kShortWaves];
    const uint32_t tid = threadIdx.x, lane = tid & 63, tile = blockIdx.x;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t n = P.n, start = tile * kShortTile, e0 = start + kShortElems * tid;

    const uint32_t flags = short_flags<kFlags>(P.flags, e0, n);
    uint32_t next = 0;      // whether the element behind mine starts a segment
    if constexpr (kOp == kSum) next = short_flags<kFlags>(P.flags, e0 + kShortElems, n) & 1u;
    ShortRaw<TT> raw;
    raw.load(P.x, e0, n);

    // ---- what lies before the tile, first part ----
    V part_v = V(0);
    uint32_t part_c = 0, last = 0;   // number of starts, the last of them
    v4u near = {0, 0, 0, 0};         // (kSingle) my 128-bit word of the values that lie right before the tile
    const int32_t near_at = (int32_t)(start / kEpl) - 1 - (int32_t)tid;
    if constexpr (kSingle) {
        if (near_at >= 0) near = ((const v4u *)P.x)[near_at];
        if constexpr (kFlags == kBitFlags) {
#pragma unroll 4
            for (uint32_t i = tid; i < start / 128; i += kShortThreads) {
                v4u f = ((const v4u *)P.flags)[i];
                if (i == 0) f[0] &= ~1u;
#pragma unroll
                for (uint32_t d = 0; d < 4; ++d) {
                    part_c += __popc(f[d]);
                    if (f[d]) last = 128 * i + 32 * d + 31 - __clz((int)f[d]);
                }
            }
        } else if constexpr (kFlags == kByteFlags) {
#pragma unroll 4
            for (uint32_t i = tid; i < start / 16; i += kShortThreads) {
                uint32_t f = bits_of_16_bytes(((const v4u *)P.flags)[i]);
                if (i == 0) f &= ~1u;
                part_c += __popc(f);
                if (f) last = 16 * i + 31 - __clz((int)f);
            }
        }
    } else {
        // the aggregates of the tiles before, a run of them per thread
        const uint32_t run = (tile + kShortThreads - 1) / kShortThreads;
#pragma unroll 4
        for (uint32_t j = 0; j < run; ++j) {
            const uint32_t t = tid * run + j;
            const uint64_t a = t < tile ? P.agg[t] : 0;
            const uint32_t c = (uint32_t)(a >> 32);
            const V v = V(from_bits<A>((uint32_t)a));
            part_v = kFlagged && c ? v : part_v + v;
            part_c += c;
        }
    }

    ShortOwn<TT> own;
    own.template scan<kFlags>(raw, flags, e0, n, P.first_one);
    if (lane == 63) {
        s_v[wave] = own.tot_v;
        s_c[wave] = own.tot_c;
    }
    if constexpr (!kSingle) {
        wave_segmented_scan<kFlagged>(part_v, part_c);
        if (lane == 63) {
            s_pv[wave] = part_v;
            s_pc[wave] = part_c;
        }
    } else if constexpr (kFlagged) {
        part_c = wave_sum(part_c);
        last = wave_max(last);
        if (lane == 0) {
            s_pc[wave] = part_c;
            s_pl[wave] = last;
        }
    }
    if (!kSingle || kFlagged) __syncthreads();

    // ---- second part: the sum carried into the tile, and the starts before it ----
    V before = V(0);
    uint32_t starts = 0;
    if constexpr (!kSingle) {
#pragma unroll
        for (int w = 0; w < kShortWaves; ++w) {
            const uint32_t c = kFlagged ? s_pc[w] : 0u;
            before = c ? s_pv[w] : before + s_pv[w];
            starts += c;
        }
    } else {
        uint32_t from = 0;   // where the segment begins that reaches into the tile
        if constexpr (kFlagged) {
#pragma unroll
            for (int w = 0; w < kShortWaves; ++w) {
                starts += s_pc[w];
                from = from > s_pl[w] ? from : s_pl[w];
            }
        }
        // the words that hold elements from .. start - 1, the nearest ones (there already) first
        const int32_t first_word = (int32_t)(from / kEpl);
        auto add = [&](v4u w, int32_t at) {
            if (at < first_word) return;
            if (at == first_word) {   // elements before `from` do not count
                const uint32_t skip = (from % kEpl) * (uint32_t)sizeof(typename TT::in_t);   // bytes
#pragma unroll
                for (uint32_t d = 0; d < 4; ++d) w[d] = skip >= 4 * d + 4 ? 0u : skip > 4 * d ? w[d] & (~0u << (8 * (skip - 4 * d))) : w[d];
            }
            if constexpr (!kFlagged && TT::kDtype == MMV_I8_I32) {
                if (P.first_one && at == 0) w[0] = (w[0] & ~0xFFu) | 1u;
            }
            part_v += word_sum<TT>(w);
        };
        add(near, near_at);   // (the words before the vector are not added: near_at < 0)
#pragma unroll 4
        for (int32_t at = near_at - kShortThreads; at >= first_word; at -= kShortThreads) add(((const v4u *)P.x)[at], at);
        uint32_t none = 0;
        wave_segmented_scan<false>(part_v, none);
        if (lane == 63) s_pv[wave] = part_v;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kShortWaves; ++w) before += s_pv[w];
    }

    // ---- the waves of the tile before mine ----
    V carry = before;
    uint32_t count = starts, all = starts;
#pragma unroll
    for (int w = 0; w < kShortWaves; ++w) {
        const uint32_t c = kFlagged ? s_c[w] : 0u;
        if (w < (int)wave) {
            carry = c ? s_v[w] : carry + s_v[w];
            count += c;
        }
        all += c;
    }
    carry = own.ex_c ? own.ex_v : carry + own.ex_v;
    count += own.ex_c;

    if (tid == 0 && kSingle && tile == 0) P.hdr[kHdrError] = P.hdr[kHdrPrepared] = 0;
    auto result = [&](int i) { return A(kFlagged && (own.F & ((2u << i) - 1u)) ? own.inc[i] : carry + own.inc[i]); };
    if constexpr (kOp == kSum) {
        if (tid == 0 && tile == gridDim.x - 1) *P.nseg = (uint64_t)all + 1u;
        // an element ends its segment if the next one starts one, or there is none
        uint32_t ends = (own.F >> 1) | (next << (kShortElems - 1));
        if (e0 < n && n - e0 <= (uint32_t)kShortElems) ends = (ends & ((1u << (n - e0 - 1)) - 1u)) | (1u << (n - e0 - 1));
        if (e0 >= n) ends = 0;
#pragma unroll
        for (int i = 0; i < kShortElems; ++i)
            if ((ends >> i) & 1u) {
                const uint64_t k = count + __popc(own.C & ((2u << i) - 1u));
                if (k < P.out_cap) ((A *)P.out)[k] = result(i);
            }
    } else {
        uint32_t o[kShortElems];
#pragma unroll
        for (int i = 0; i < kShortElems; ++i) {
            o[i] = to_bits(result(i));
            if constexpr (kFlagged && sizeof(typename TT::in_t) == 4) {
                if ((own.F >> i) & 1u) o[i] = to_bits(raw.elem(i));   // a start receives its input bit for bit, NaNs too
            }
        }
        uint32_t *z = (uint32_t *)P.z + e0;
        if (e0 < n && n - e0 >= (uint32_t)kShortElems) {
#pragma unroll
            for (int q = 0; q < kShortElems / 4; ++q) *(v4u *)(z + 4 * q) = v4u{o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]};
        } else {
#pragma unroll
            for (int i = 0; i < kShortElems; ++i)
                if (e0 < n && (uint32_t)i < n - e0) z[i] = o[i];
        }
    }
}

}  // namespace
