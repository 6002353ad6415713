// Small products on int8 matrix cores: one wavefront computes one row of four
// 256-coefficient tiles, 4 / TPI instances of TPI tiles each, with no
// workgroup barrier at all.
//   full products:       TPI 1 / 2 / 4 serve up to 32 / 64 / 128 words
//   low product, Poly:   TPI 1 / 2 / 4 serve up to 64 / 128 / 256 words
// What bounds it: at 128 words a product is 28 MFMAs (448 clk of its SIMD),
// 44 KB through the LDS and about 170 vector instructions, all near half of
// the time a product takes, and a third of it in HBM traffic: seven waves per
// SIMD that never wait for each other overlap them.  Measured, full products
// (one workgroup per product before, int8 windows in LDS at 128 words and the
// VALU schoolbook at 32): 65536 x 128 words 83.3 -> 37.1 us (3.6 TB/s),
// 262144 x 32 words 213 -> 33.7 us (4.0 TB/s).
// Full products hold a's chunks in lanes 0..31 and b's in lanes 32..63, so
// both operands are recoded by one carry scan.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "bi_conv.hpp"

namespace bi {

namespace {

using namespace conv;

// Adds R below chunk `nch`, propagates the carries inside each segment of
// CPI lanes and leaves the digits in x.  Returns the carry out of this
// lane's chunk.  `keep` masks the lanes that are not a segment's last.
__device__ __forceinline__ uint32_t recode_lane(uint32_t (&x)[4], bool digits, uint64_t keep, uint32_t lane) {
    const uint32_t R = digits ? kR8 : 0u;
    const uint32_t r4[4] = {R, R, R, R};
    uint32_t s[4];
    const uint32_t g = add_words<4>(x, r4, s);
    const bool p = all_ones<4>(s);
    const WaveCarry wc = wave_carry(ballot(g != 0) & keep, ballot(p) & keep, 0);
    const uint32_t ci = uint32_t(wc.into >> lane) & 1u;
    add_carry_words<4>(s, ci);
#pragma unroll
    for (int t = 0; t < 4; ++t) x[t] = s[t] ^ R;
    return g | (p ? ci : 0u);
}

// The row's words from its accumulators (plus the words of `add`), carries
// cut at instance ends.
template <int TPI, bool ADD>
__device__ __forceinline__ void small_finish(const v4i (&acc)[4], const uint32_t (&add)[4], uint32_t lane,
                                             uint32_t (&s)[4]) {
    const uint32_t co = lane & (16 * TPI - 1);
    uint32_t lo[4], hi[4];
    row_words(acc[0], acc[1], acc[2], acc[3], lo, hi);
    if constexpr (ADD) add_to_words(lo, hi, add);
    uint32_t below = from_below(hi[3], kBelowFirst);
    if (TPI < 4) below = co == 0 ? kBelowFirst : below;
    const uint32_t y[4] = {below, hi[0], hi[1], hi[2]};
    const uint64_t keep = TPI == 4 ? ~(1ull << 63) : TPI == 2 ? ~0x8000000080000000ull : ~0x8000800080008000ull;
    const uint32_t g = add_words<4>(lo, y, s);
    const WaveCarry wc = wave_carry(ballot(g != 0) & keep, ballot(all_ones<4>(s)) & keep, 0);
    add_carry_words<4>(s, uint32_t(wc.into >> lane) & 1u);
}

// Full products of src on this wave: groups first, first + stride, ..; lds
// holds Small<TPI, false>::WAVE bytes.
template <int TPI, class Src>
__device__ __forceinline__ void small_full(const Src &src, uint8_t *lds, uint64_t first, uint64_t stride) {
    using S = Small<TPI, false>;
    const uint32_t lane = lane_id();
    const uint64_t count = src.count();
    const uint64_t groups = (count + S::IPW - 1) / S::IPW;

    // everything but the digits stays zero for the whole launch
    for (uint32_t i = lane; i < S::WAVE / 16; i += 64) *reinterpret_cast<uint4 *>(lds + 16 * i) = make_uint4(0, 0, 0, 0);

    const LaneAddr la = lane_addr();
    const uint8_t *ap = lds + la.a, *bp = lds + S::AB + 16 * S::kPad + la.b;
    const uint32_t co = lane & (16 * TPI - 1), oslot = lane / (16 * TPI);  // output chunk of this lane
    // operand chunk of this lane
    const uint32_t half = lane >> 5, l = lane & 31u;
    const uint32_t slot = l / S::CPI, c = l & (S::CPI - 1);
    const uint64_t keep = TPI == 4 ? ~0x8000000080000000ull : TPI == 2 ? ~0x8000800080008000ull : ~0x8080808080808080ull;
    uint8_t *dst = lds + slot * S::INST + (half ? S::AB + 16 * (S::kPad + c) : kAPad + 16 * c);
    uint32_t *tdst = reinterpret_cast<uint32_t *>(dst + 16 + (half ? 12 : 0));  // digit D of the operand
    auto fetch = [&](uint64_t g, uint32_t (&x)[4], uint32_t &n) {
        const uint64_t inst = g * S::IPW + slot;
        n = 0;
        if (inst < count) {
            const InstRef in = src.get(inst);
            n = in.n;
            load_chunk4(half ? in.b : in.a, in.n, c, x);
        }
    };
    uint32_t xn[4] = {0, 0, 0, 0}, nn = 0;
    uint64_t g = first;
    if (g < groups) fetch(g, xn, nn);
    for (; g < groups; g += stride) {
        uint32_t x[4] = {xn[0], xn[1], xn[2], xn[3]};
        const uint32_t n = nn;
        if (g + stride < groups) fetch(g + stride, xn, nn);
        const bool digits = 4 * c < n;
        if (!digits) { x[0] = x[1] = x[2] = x[3] = 0; }
        const uint32_t t = recode_lane(x, digits, keep, lane);
        wave_lds_fence();
        const uint4 rv = reversed(x);
        *reinterpret_cast<uint4 *>(dst) = half ? rv : make_uint4(x[0], x[1], x[2], x[3]);
        if (c == S::CPI - 1) *tdst = half ? t << 24 : t;
        wave_lds_fence();
        v4i acc[4] = {};
#pragma unroll
        for (int i = 0; i < S::IPW; ++i) small_steps<TPI, false>(ap + i * S::INST, la.sh, bp + i * S::INST, acc + i * TPI);
        uint32_t s[4];
        small_finish<TPI, false>(acc, s, lane, s);
        const uint64_t oi = g * S::IPW + oslot;
        if (oi < count) {
            const InstRef out = src.get(oi);
            store_chunk4(out.c, 2 * out.n, co, s, src.streams());
        }
    }
}

}  // namespace

template <int TPI, int MODE, class Src>
__global__ __launch_bounds__(256, MODE == kPoly ? 4 : MODE == kLow ? 5 : 6) void conv_small_kernel(Src src) {
    constexpr bool LOW = MODE != kFull;
    using S = Small<TPI, LOW>;
    __shared__ __align__(16) uint8_t lds_all[4 * S::WAVE];
    const uint32_t lane = lane_id(), wave = wave_in_block();
    uint8_t *lds = lds_all + wave * S::WAVE;
    if constexpr (!LOW) {
        small_full<TPI>(src, lds, uint64_t(blockIdx.x) * 4 + wave, uint64_t(gridDim.x) * 4);
    } else {
        const uint64_t count = src.count();
        const uint64_t groups = (count + S::IPW - 1) / S::IPW;
        const uint64_t stride = uint64_t(gridDim.x) * 4;
        // everything but the digits stays zero for the whole launch
        for (uint32_t i = lane; i < S::WAVE / 16; i += 64)
            *reinterpret_cast<uint4 *>(lds + 16 * i) = make_uint4(0, 0, 0, 0);
        const LaneAddr la = lane_addr();
        const uint8_t *ap = lds + la.a, *bp = lds + S::AB + 16 * S::kPad + la.b;
        const uint32_t co = lane & (16 * TPI - 1), oslot = lane / (16 * TPI);  // chunk of this lane
        // operand and result chunk of this lane coincide (a top carry digit
        // only reaches coefficients above the low half)
        const uint64_t keep = TPI == 4 ? ~(1ull << 63) : TPI == 2 ? ~0x8000000080000000ull : ~0x8000800080008000ull;
        uint8_t *da = lds + oslot * S::INST + kAPad + 16 * co;
        uint8_t *db = lds + oslot * S::INST + S::AB + 16 * (S::kPad + co);
        auto put_a = [&](const uint32_t (&d)[4]) { *reinterpret_cast<uint4 *>(da) = make_uint4(d[0], d[1], d[2], d[3]); };
        auto put_b = [&](const uint32_t (&d)[4]) { *reinterpret_cast<uint4 *>(db) = reversed(d); };
        auto fetch = [&](uint64_t g, uint32_t (&x)[4], uint32_t (&y)[4], uint32_t &n) {
            const uint64_t inst = g * S::IPW + oslot;
            n = 0;
            if (inst < count) {
                const InstRef in = src.get(inst);
                n = in.n;
                load_chunk4(in.a, in.n, co, x);
                load_chunk4(in.b, in.n, co, y);
            }
        };
        auto steps = [&](v4i (&acc)[4]) {
            wave_lds_fence();
#pragma unroll
            for (int i = 0; i < S::IPW; ++i) small_steps<TPI, LOW>(ap + i * S::INST, la.sh, bp + i * S::INST, acc + i * TPI);
            wave_lds_fence();
        };
        uint32_t xn[4] = {0, 0, 0, 0}, yn[4] = {0, 0, 0, 0}, nn = 0;
        uint64_t g = uint64_t(blockIdx.x) * 4 + wave;
        if (g < groups) fetch(g, xn, yn, nn);
        for (; g < groups; g += stride) {
            uint32_t x[4], y[4], s[4];
            const uint32_t n = nn;
            const bool digits = 4 * co < n;
#pragma unroll
            for (int t = 0; t < 4; ++t) { x[t] = digits ? xn[t] : 0u; y[t] = digits ? yn[t] : 0u; }
            if (g + stride < groups) fetch(g + stride, xn, yn, nn);
            uint32_t b[4] = {y[0], y[1], y[2], y[3]};
            recode_lane(x, digits, keep, lane);
            recode_lane(y, digits, keep, lane);
            put_a(x);
            put_b(y);
            v4i acc[4] = {};
            steps(acc);
            small_finish<TPI, false>(acc, s, lane, s);  // a b
            if constexpr (MODE == kPoly) {
                uint32_t ab[4] = {s[0], s[1], s[2], s[3]}, T[4], V[4];
                auto clear_above = [&](uint32_t (&v)[4]) {  // words at or above n are no part of an operand
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        if (4 * co + t >= n) v[t] = 0;
                };
                put_b(x);
                v4i a2[4] = {};
                steps(a2);
                small_finish<TPI, true>(a2, b, lane, T);  // a a + b
                put_a(y);
                put_b(y);
                v4i b2[4] = {};
                steps(b2);
                small_finish<TPI, true>(b2, b, lane, V);  // b b + b
                clear_above(T);
                clear_above(V);
                recode_lane(T, digits, keep, lane);
                recode_lane(V, digits, keep, lane);
                put_a(T);
                put_b(V);
                v4i c2[4] = {};
                steps(c2);
                small_finish<TPI, true>(c2, ab, lane, s);  // (a a + b)(b b + b) + a b
            }
            const uint64_t oi = g * S::IPW + oslot;
            if (oi < count) {
                const InstRef out = src.get(oi);
                store_chunk4(out.c, n, co, s, src.streams());
            }
        }
    }
}

// The ragged classes of up to 16, 32, 64 and 128 words in one launch: blocks
// first[k] .. first[k + 1] - 1 walk class k's list.
__global__ __launch_bounds__(256, 5) void conv_small_lists_kernel(SmallLists p) {
    __shared__ __align__(16) uint8_t lds_all[4 * Small<1, false>::WAVE];
    static_assert(Small<1, false>::WAVE >= Small<2, false>::WAVE && Small<2, false>::WAVE >= Small<4, false>::WAVE,
                  "one tile per instance takes the most LDS");
    const uint32_t wave = wave_in_block(), blk = blockIdx.x;
    uint8_t *lds = lds_all + wave * Small<1, false>::WAVE;
    const uint32_t k = blk < p.first[1] ? 0 : blk < p.first[2] ? 1 : blk < p.first[3] ? 2 : 3;
    const uint64_t first = uint64_t(blk - p.first[k]) * 4 + wave, stride = uint64_t(p.first[k + 1] - p.first[k]) * 4;
    if (k < 2) small_full<1>(k == 0 ? p.cls[0] : p.cls[1], lds, first, stride);
    else if (k == 2) small_full<2>(p.cls[2], lds, first, stride);
    else small_full<4>(p.cls[3], lds, first, stride);
}

hipError_t launch_conv_small_lists(SmallLists p, const uint64_t (&count)[4], hipStream_t st, int num_cus) {
    // blocks per class, which loop beyond that: one per CU would take 67 us for
    // 20000 products of 1 .. 128 words and 801 for 400000, four take 58 and 578,
    // sixteen 58.5 and 557
    const uint64_t cap = uint64_t(num_cus > 0 ? num_cus : 1) * 4;
    const uint32_t ipw[4] = {4, 4, 2, 1};
    p.first[0] = 0;
    for (int k = 0; k < 4; ++k)
        p.first[k + 1] = p.first[k] + uint32_t(std::min<uint64_t>((count[k] + 4 * ipw[k] - 1) / (4 * ipw[k]), cap));
    if (p.first[4] == 0) return hipSuccess;
    hipLaunchKernelGGL(conv_small_lists_kernel, dim3(p.first[4]), dim3(256), 0, st, p);
    return hipGetLastError();
}

template <int TPI, int MODE, class Src>
static hipError_t launch_small(const Src &src, uint64_t count, hipStream_t st, int num_cus) {
    constexpr int IPW = 4 / TPI;
    static std::atomic<int> occ{0};  // resident workgroups per CU
    int o = occ.load(std::memory_order_relaxed);
    if (o == 0) {
        const void *fn = reinterpret_cast<const void *>(&conv_small_kernel<TPI, MODE, Src>);
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, fn, 256, 0);
        if (e != hipSuccess) return e;
        if (o < 1) o = 1;
        occ.store(o, std::memory_order_relaxed);
    }
    const uint64_t blocks = (count + 4 * IPW - 1) / (4 * IPW);
    const uint64_t cap = uint64_t(num_cus > 0 ? num_cus : 1) * uint64_t(o) * 4;
    const uint32_t grid = uint32_t(std::min(blocks, cap));
    if (grid == 0) return hipSuccess;
    hipLaunchKernelGGL((conv_small_kernel<TPI, MODE, Src>), dim3(grid), dim3(256), 0, st, src);
    return hipGetLastError();
}

template <class Src>
static hipError_t launch_small_full(const Src &src, uint32_t nmax, uint64_t count, hipStream_t st, int num_cus) {
    if (nmax <= 32) return launch_small<1, kFull>(src, count, st, num_cus);
    if (nmax <= 64) return launch_small<2, kFull>(src, count, st, num_cus);
    return launch_small<4, kFull>(src, count, st, num_cus);
}

hipError_t launch_conv_small_full(const UniformInst &src, hipStream_t st, int num_cus) {
    return launch_small_full(src, src.n, src.batch, st, num_cus);
}

hipError_t launch_conv_small_list(const ListInst &src, uint32_t nmax, uint64_t count, hipStream_t st, int num_cus) {
    return launch_small_full(src, nmax, count, st, num_cus);
}

hipError_t launch_conv_small_low(bool poly, const LowInst &src, hipStream_t st, int num_cus) {
    const uint32_t n = src.u.n;
    const uint64_t batch = src.u.batch;
#define BI_SMALL(T) poly ? launch_small<T, kPoly>(src, batch, st, num_cus) : launch_small<T, kLow>(src, batch, st, num_cus)
    if (n <= 64) return BI_SMALL(1);
    if (n <= 128) return BI_SMALL(2);
    return BI_SMALL(4);
#undef BI_SMALL
}

}  // namespace bi
