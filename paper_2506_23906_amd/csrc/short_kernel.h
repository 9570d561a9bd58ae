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
// Measured, whole calls in a graph, on other inputs every time (together beyond every cache) and, in brackets, on the same, the
// single-pass kernel -> one launch / two (us):
//   segmented scan, fp32, byte flags, 1 of 64 set    3000: 8.5 -> 3.2 / 5.2 (7.7 -> 2.9 / 5.0)   65536: 9.3 -> 4.3 / 5.6 (9.2 -> 3.7 / 5.2)
//   ... no flags, packed                             3000: 6.3 -> 3.6 / 5.2 (5.8 -> 3.0 / 4.7)   65536: 9.0 -> 7.4 / 5.4 (8.3 -> 5.8 / 5.0)
//   segmented sum, fp16, packed, 1 of 1000 set       3000: 6.4 -> 3.1 / 4.9 (6.1 -> 3.0 / 4.8)  105000: 8.4 -> 4.7 / 6.0 (8.0 -> 3.8 / 5.3)
//   scan, fp32                                       3000: 7.7 -> 2.8 / 4.2 (7.2 -> 2.4 / 3.9)   65536: 10.4 -> 5.2 / 4.5 (10.0 -> 4.3 / 4.2)
// Where the lines lie (figures on other inputs every time unless said otherwise).
// One launch, MMV_SINGLE_BYTES: with flags anywhere near it is ahead of two (65536 fp32 values, 1 of 1000 set: 4.2 / 5.4); without any
// flag set a workgroup reads all that lies before its tile, and two are ahead from 20000 to 80000 elements on.  The host does
// not know the flags: the line lies where the worst of them come out level with the single-pass kernel (none set, single-pass -> one
// launch: fp32 sum, byte flags, 65536 8.1 -> 7.1; bytes, 160000 8.4 -> 7.0; fp16, packed, 118000 8.6 -> 9.0, 131072 8.4 -> 7.9, 150000
// 8.4 -> 8.4, repeated 8.0 -> 7.9, 8.0 -> 7.1, 8.0 -> 7.7).
// Two launches, short_max: up to 2^21 elements nearly everything gains (350000 to 1.5 million fp32 11 -> 6.5 to 9, segmented scan of bytes, 2^21
// 11.2 -> 9.0).  The least gain have 16-bit segmented scans, whose time in the single-pass kernel is that of whole tiles or
// of a ragged last one: bits, 1 of 1000 set, 1900000 10.1 -> 9.7 (repeated 9.8 -> 8.6), 2080000 10.6 -> 10.0 (9.7 -> 8.7), but 2^21
// 9.1 -> 9.9 (8.9 -> 8.7; none set 10.2 -> 9.8, 10.3 -> 8.7).  Beyond, where the data read twice show: scans without flags of 2^22, fp32 15.0 -> 14.3, bytes 12.1 -> 12.2, 16-bit, 3 * 2^20 12.1 -> 11.0 (2^22 11.9 -> 12.3);
// fp32 sums, 3 * 2^20, 1 of 1000 set 11.9 -> 11.5, 1 of 5 12.4 -> 12.4 (2^22 11.3 -> 12.0).  Segmented scans (2^22: 11.6 -> 11.9, bytes
// 10.8 -> 11.2) and sums of bytes stay at 2^21.  Four elements per thread: level up to 2^19, 10 % slower at 2^21; sixteen: 20 % slower there.
constexpr int kShortThreads = 256, kShortWaves = kShortThreads / 64;
constexpr int kShortElems = 8;                                  // consecutive elements of a thread
constexpr uint32_t kShortTile = kShortThreads * kShortElems;
// Threads of a workgroup of the one launch from so many bytes of values and flags on (many_bytes): those beyond kShortThreads only help with what
// lies before the tile.  Calls as above, on other inputs every time, the single-pass kernel / 256 threads / 1024:
//   segmented scan, fp32, byte flags, 65536: none set 8.8 / 10.0 / 6.8, 1 of 64 9.3 / 5.8 / 4.3;  bits, none set 8.3 / 7.9 / 6.6
//   segmented sum, byte flags, none set: fp32, 65536 8.1 / 10.3 / 7.1; fp16, 105000 8.3 / 11.8 / 7.7; bytes, 160000 8.4 / 12.1 / 7.0
//   scan, fp32, 65536 10.4 / 5.9 / 5.2;  20000 11.4 / 4.4 / 3.9
// With 256 a vector whose segments reach far back took up to 45 % longer than the single-pass kernel.  But sixteen waves start later
// and have more to exchange, 0.1 (bytes) to 0.5 us (fp32), and where a flag is near they bring nothing: segmented scan with bits,
// fp32, 20000, 1 of 64 set, 256 threads / 1024, repeated on the same inputs, 2.9 / 3.5, 65536 3.1 / 3.6; bytes 65536 3.0 / 3.1; with
// byte flags, more of which every workgroup reads, fp32 20000 3.4 / 3.8, 40960 3.7 / 3.8.  So the lines lie where these calls come
// out level, with bits where those without any flag set begin to fall behind the single-pass kernel (segmented sums of none set,
// single-pass / 256: fp32 65536 8.2 / 7.8, 79000 8.6 / 8.8; fp16 105000 8.3 / 8.5, 118000 8.6 / 9.0).  Without flags: where a second or third
// tile begins (scan, 256 threads / 1024, fp16 4096 2.5 / 2.6, 5000 3.1 / 2.7; bytes 6000 2.3 / 2.4, 7000 2.7 / 2.4).
constexpr int kManyThreads = 1024;
#ifndef MMV_SINGLE_BYTES
#define MMV_SINGLE_BYTES (320u << 10)   // most values and flags, in bytes, of a vector that one launch takes
#endif
enum ShortFlags { kNoFlags = 0, kBitFlags = 1, kByteFlags = 2 };
constexpr bool is_16_bit(mmv_dtype dt) { return dt == MMV_F16_F32 || dt == MMV_BF16_F32; }
constexpr uint64_t many_bytes(mmv_dtype dt, int flags) {
    constexpr uint64_t kb[3][3] = {{9, 9, 7}, {288, 240, 96}, {160, 128, 80}};   // no flags, bits, bytes; values of 4, 2, 1 bytes
    return kb[flags][dt == MMV_F32_F32 ? 0 : is_16_bit(dt) ? 1 : 2] << 10;
}
#ifndef MMV_SHORT_MAX
#define MMV_SHORT_MAX (1u << 21)        // most elements that two launches take
#endif
constexpr uint64_t short_max(mmv_op op, mmv_dtype dt) {
    const uint64_t n = MMV_SHORT_MAX;
    if (op == MMV_OP_SCAN) return is_16_bit(dt) ? n / 2 * 3 : 2 * n;
    return op == MMV_OP_SEGSUM && dt == MMV_F32_F32 ? n / 2 * 3 : n;
}

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
// row scans in 32 bits; in 32 bits the lanes' scans here would come to 8.1e-8).  Between two launches the sums of whole tiles are kept
// in 32: a result there is off by the rounding of the tile sums of its segment as well.
template <typename A> struct Wide {
    typedef A type;
};
template <> struct Wide<float> {
    typedef double type;
};
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
template <typename TT, int kOp, int kFlags, bool kSingle, int kThreads>
__global__ __launch_bounds__(kThreads) void short_kernel(ShortParams P) {
    typedef typename TT::acc_t A;
    typedef typename Wide<A>::type V;
    constexpr bool kFlagged = kFlags != kNoFlags;
    constexpr uint32_t kEpl = TT::kEpl;
    constexpr int kWaves = kThreads / 64;
    constexpr bool kMany = kThreads > kShortThreads;
    constexpr int kUnder = kMany ? 8 : 4;   // words of values under way at a time
    static_assert(kSingle || !kMany, "threads that only help with what lies before the tile");
    __shared__ V s_v[kShortWaves], s_pv[kWaves];                 // of the waves: their aggregates, their part of what lies before the tile
    __shared__ uint32_t s_c[kShortWaves], s_pc[kWaves], s_pl[kWaves];
    const uint32_t tid = threadIdx.x, lane = tid & 63, tile = blockIdx.x;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t n = P.n, start = tile * kShortTile, e0 = start + kShortElems * tid;
    const bool owner = !kMany || wave < (uint32_t)kShortWaves;   // (uniform) whether my wave has elements of the tile

    uint32_t flags = 0, next = 0;      // next: whether the element behind mine starts a segment
    ShortRaw<TT> raw;
    if (owner) {
        flags = short_flags<kFlags>(P.flags, e0, n);
        if constexpr (kOp == kSum) next = short_flags<kFlags>(P.flags, e0 + kShortElems, n) & 1u;
        raw.load(P.x, e0, n);
    }

    // ---- what lies before the tile, first part ----
    V part_v = V(0);
    uint32_t part_c = 0, last = 0;   // number of starts (sums), the last of them
    v4u near = {0, 0, 0, 0};         // (kSingle) my 128-bit word of the values that lie right before the tile
    const uint32_t words = start / kEpl;
    const int32_t near_at = (int32_t)words - 1 - (int32_t)tid;
    if constexpr (kSingle) {
        if (near_at >= 0) near = ((const v4u *)P.x)[near_at];
        if constexpr (kFlagged) {
            // the last 128-bit word with a start, its starts, and how many there are
            constexpr uint32_t kPerWord = kFlags == kBitFlags ? 128 : 16;
            const uint32_t flag_words = start / kPerWord;
            v4u hit = {0, 0, 0, 0};
            uint32_t hit_at = 0;
            auto take = [&](v4u f, uint32_t i, bool valid) {   // (selects, no branches: what is loaded in a branch is waited for there)
                if (i == 0) f[0] &= kFlags == kBitFlags ? ~1u : ~0xFFu;
                if constexpr (kFlags == kByteFlags) {
#pragma unroll
                    for (int d = 0; d < 4; ++d) f[d] = (((f[d] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | f[d]) & 0x80808080u;   // the bytes that are not zero
                }
                if constexpr (kOp == kSum) {
                    const uint32_t cnt = kFlags == kByteFlags ? __popc((f[0] >> 3) | (f[1] >> 2) | (f[2] >> 1) | f[3])
                                                              : (__popc(f[0]) + __popc(f[1])) + (__popc(f[2]) + __popc(f[3]));
                    part_c += valid ? cnt : 0u;
                }
                const bool any = valid && ((f[0] | f[1]) | (f[2] | f[3])) != 0;
                hit_at = any ? i : hit_at;
#pragma unroll
                for (int d = 0; d < 4; ++d) hit[d] = any ? f[d] : hit[d];
            };
            if constexpr (kMany) {   // four words under way, also of the last ones
                for (uint32_t i = tid; i < flag_words; i += 4 * kThreads) {
                    v4u f[4];
#pragma unroll
                    for (uint32_t j = 0; j < 4; ++j) f[j] = ((const v4u *)P.flags)[i + j * kThreads < flag_words ? i + j * kThreads : i];
#pragma unroll
                    for (uint32_t j = 0; j < 4; ++j) take(f[j], i + j * kThreads, i + j * kThreads < flag_words);
                }
            } else {
#pragma unroll 4
                for (uint32_t i = tid; i < flag_words; i += kThreads) take(((const v4u *)P.flags)[i], i, true);
            }
            const uint32_t d = hit[3] ? 3 : hit[2] ? 2 : hit[1] ? 1 : 0, bits = hit[3] ? hit[3] : hit[2] ? hit[2] : hit[1] ? hit[1] : hit[0];
            if (bits) last = kPerWord * hit_at + kPerWord / 4 * d + (31 - __clz((int)bits)) / (kFlags == kBitFlags ? 1 : 8);
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
    if (owner) {
        own.template scan<kFlags>(raw, flags, e0, n, P.first_one);
        if (lane == 63) {
            s_v[wave] = own.tot_v;
            s_c[wave] = own.tot_c;
        }
    }
    if constexpr (!kSingle) {
        wave_segmented_scan<kFlagged>(part_v, part_c);
        if (lane == 63) {
            s_pv[wave] = part_v;
            s_pc[wave] = part_c;
        }
    } else if constexpr (kFlagged) {
        if (kOp == kSum) part_c = wave_sum(part_c);
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
            if constexpr (kMany) {
                if (kOp == kSum) starts = wave_sum(lane < kWaves ? s_pc[lane] : 0u);
                from = wave_max(lane < kWaves ? s_pl[lane] : 0u);
            } else {
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    if (kOp == kSum) starts += s_pc[w];
                    from = from > s_pl[w] ? from : s_pl[w];
                }
            }
        }
        // the words that hold elements from .. start - 1: the nearest are there already; the first may hold elements before `from`
        const int32_t first_word = (int32_t)(from / kEpl);
        const bool far = first_word < (int32_t)words - kThreads;      // (nobody holds the first word yet)
        v4u w0 = near;
        if (far && tid == 0) w0 = ((const v4u *)P.x)[first_word];
        if (near_at > first_word) part_v = word_sum<TT>(near);        // (near_at < 0: none)
#pragma unroll kUnder
        for (int32_t at = near_at - kThreads; at > first_word; at -= kThreads) part_v += word_sum<TT>(((const v4u *)P.x)[at]);
        if (near_at == first_word || (far && tid == 0)) {
            const uint32_t skip = (from % kEpl) * (uint32_t)sizeof(typename TT::in_t);   // bytes that do not count
#pragma unroll
            for (uint32_t d = 0; d < 4; ++d) w0[d] = skip >= 4 * d + 4 ? 0u : skip > 4 * d ? w0[d] & (~0u << (8 * (skip - 4 * d))) : w0[d];
            if constexpr (!kFlagged && TT::kDtype == MMV_I8_I32) {
                if (P.first_one) w0[0] = (w0[0] & ~0xFFu) | 1u;
            }
            part_v += word_sum<TT>(w0);
        }
        uint32_t none = 0;
        wave_segmented_scan<false>(part_v, none);
        if (lane == 63) s_pv[wave] = part_v;
        __syncthreads();
        if (!owner) return;
        if constexpr (kMany) {
            before = lane < kWaves ? s_pv[lane] : V(0);
            wave_segmented_scan<false>(before, none);
            before = wave_last(before);
        } else {
#pragma unroll
            for (int w = 0; w < kWaves; ++w) before += s_pv[w];
        }
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
