// Products of up to 8192 words on int8 matrix cores, one workgroup per
// product: full products above 128 words, low products (mod 2^N) and Poly
// above 256.  See bi_conv.hpp for the digits, tiles and operand layout.
//
// A unit is T tiles (T / 4 rows of 256 words), T a multiple of 4.  A wave
// owns UPW units and walks, per residue kappa, the steps m of a unit with the
// T B operands j = t - m of its tiles in registers: one A and one new B
// operand per step of T MFMAs.  Two forms:
//   straight-line (ST): all steps of the largest product unrolled, only the
//     MFMAs inside the band; smaller products are padded with zero digits.
//   loops, for any size: blocks of T steps, straight where every tile is in
//     band and triangles at the ends of the band.
//
// What bounds it.  Random digits hold the chip at about 1.8 GHz (2.05e15
// MAC/s for this MFMA from registers alone, 1.74e15 for 32 x 32 x 32), and the
// LDS reads and vector work beside the MFMAs cost time on top of them: at
// 8192 x 1024 words the MFMAs alone are 73 us of 104, and the loops took 68
// without them.  Hence few operand reads per MFMA (T as large as the registers
// allow where a product fits few units: 2.25 KB per T MFMAs), no MFMA outside
// the band, and small workgroups: a wave that shares nothing waits for
// nothing.  Above 1024 words T = 8 and 128 registers for four waves per SIMD
// (T = 16 at two or three: 2048 words 99 -> 97-103 us, 1500 words 119 ->
// 127-152).  Measured against the kernels before it (32 x 32 x 32 tiles over
// 8-byte windows of a in LDS; three kernels and global scratch above 1024
// words), full products: 16384 x 256 words 51.9 -> 23 us, 8192 x 512 words
// 61.7 -> 30, 4096 x 1024 words 81.4 -> 57, 2048 x 2048 words 198 -> 97, 512 x
// 4096 words 196 -> 90 us.  Up to 64 products of more than 5500 words are
// the exception: each keeps one CU busy for longer than the three kernels,
// which spread it over several, took in all (1 / 32 products of
// 8192 words 91 / 96 -> 128 / 130 us, of 6000 words 69 / 73 -> 74 / 75); the
// default there is Karatsuba (32 and 29 us for one).  Low products and Poly
// against the VALU schoolbook in LDS: 16384 x 512 words 266 -> 35.5 us, 4096 x
// 2048 words (Poly) 3041 -> 375, 128 x 8192 words 657 -> 70 and (Poly) 2631 ->
// 279.
//
// Registers: the bounds of the kernel make the compiler spill in Poly (16 words
// per lane for up to 2048 words, 31 and 33 above, 24 for 769 .. 1024) and in
// full products of two units per wave (17 above 4096 words) and of 641 .. 768
// words (5), and 4 in low products above 2048 words.
#include <algorithm>
#include <atomic>
#include <utility>

#include "bi_conv.hpp"

namespace bi {

namespace {

using namespace conv;

// Order of the units over the waves: cost grows with the unit (low products)
// or peaks in the middle (full ones), and waves w, w + 4, w + 8, .. share a
// SIMD.
template <int NW, bool LOW>
__device__ __forceinline__ uint32_t wave_role(uint32_t wave, uint64_t inst) {
    if constexpr (NW == 1) return 0;
    else if constexpr (NW <= 4) return (wave + uint32_t(inst)) % NW;
    else if constexpr (LOW && NW % 8 == 0) return (wave & 4u) ? (wave ^ 3u) : wave;
    else return wave;
}

// T steps m .. m + T - 1 of a unit from a window w (slot i: B operand
// t0 - m + i), sliding it as they go.  SHAPE: every tile in band (kAll); only
// tiles i <= s of step s (kEntry: the first step takes the last B operand);
// only tiles i >= s (kExit: the last step takes B operand 0).
enum Shape { kAll, kEntry, kExit };
// `a` holds the A operand of the first step, and on return that of step m + T
// (`more`: there is one).  The scheduler is held to this order: operands of
// the next step are requested before the MFMAs of this one and awaited after
// them.
template <int T, int SHAPE>
__device__ __forceinline__ void block_steps(const uint8_t *am, uint32_t sh, const uint8_t *bj, v4i (&w)[T], v4i &a,
                                       bool more, v4i (&acc)[T]) {
#pragma unroll
    for (int s = 0; s < T; ++s) {
        const ARaw next = read_a(s + 1 < T || more ? am + 256 * (s + 1) : am);
        __builtin_amdgcn_sched_barrier(0);
        if (SHAPE != kEntry || s == T - 1) acc[T - 1] = mac64(a, w[(T - 1 - s) & (T - 1)], acc[T - 1]);
        // the window of the next step starts one B operand lower
        if (SHAPE != kExit) w[(T - 1 - s) & (T - 1)] = read_b(bj - 256 * (s + 1));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = T - 2; i >= 1; --i)
            if (SHAPE == kAll || (SHAPE == kEntry ? i <= s : i >= s))
                acc[i] = mac64(a, w[(i - s) & (T - 1)], acc[i]);
        __builtin_amdgcn_sched_barrier(0);
        const v4i an = align_a(next, sh);
        __builtin_amdgcn_sched_barrier(0);
        if (SHAPE != kExit || s == 0) acc[0] = mac64(a, w[(0 - s) & (T - 1)], acc[0]);
        a = an;
    }
}

// Adds the steps of the unit at tile t0 into acc.  U: last step with a
// nonzero A operand; gd: last nonzero group of b.  B operands above J are
// zero, and those below 0 but for -1 at kappa 0.
template <int T>
__device__ __forceinline__ void unit_steps(const uint8_t *ap, uint32_t sh, const uint8_t *bp, int32_t t0, int32_t U,
                                           int32_t gd, v4i (&acc)[T]) {
#pragma unroll 1
    for (int32_t k = 0; k < 4; ++k) {
        const int32_t J = (gd + 4 * k) >> 4, M = (U - k) >> 2;
        const uint8_t *ak = ap + 64 * k, *bk = bp - 64 * k;
        // the unit's band ends inside the steps of a (exit shape), or a ends first
        const bool exits = M >= t0 + T - 1;
        int32_t m = max(0, t0 - J);
        const int32_t end = exits ? t0 : min(M, t0 + T) + 1;
        if (exits || end - m >= T) {
            v4i w[T];
#pragma unroll
            for (int i = 0; i < T; ++i) w[i] = read_b(bk + 256 * min(t0 - m + i, J + 1));
            v4i a = align_a(read_a(ak + 256 * m), sh);
            if (!exits && t0 >= J) {
                block_steps<T, kEntry>(ak + 256 * m, sh, bk + 256 * (t0 - m), w, a, m + T <= M, acc);
                m += T;
            }
#pragma unroll 1
            for (; m + T <= end; m += T)
                block_steps<T, kAll>(ak + 256 * m, sh, bk + 256 * (t0 - m), w, a, m + T <= M, acc);
            if (exits) {
                block_steps<T, kExit>(ak + 256 * m, sh, bk + 256 * (t0 - m), w, a, false, acc);
                m += T;
                if (k == 0) {  // B operand -1 reaches 16 digits of the product below tile m
                    const v4i b = read_b(bk - 256);
#pragma unroll
                    for (int i = 0; i < T; ++i)
                        if (i < T - 1 || m <= M)
                            acc[i] = mac64(align_a(read_a(ak + 256 * (t0 + i + 1)), sh), b, acc[i]);
                }
            }
        }
        if (m < end) {  // fewer than T steps left
            const int32_t least = k == 0 ? -2 : -1, cnt = end - m;
            const uint8_t *am = ak + 256 * m;
            v4i w[T];
#pragma unroll
            for (int i = 0; i < T; ++i) w[i] = read_b(bk + 256 * max(min(t0 - m + i, J + 1), least));
            v4i a = align_a(read_a(am), sh);
#pragma unroll
            for (int s = 0; s < T - 1; ++s) {
                const ARaw next = read_a(am + 256 * min(s + 1, cnt - 1));
                __builtin_amdgcn_sched_barrier(0);
                acc[T - 1] = mac64(a, w[(T - 1 - s) & (T - 1)], acc[T - 1]);
                w[(T - 1 - s) & (T - 1)] = read_b(bk + 256 * max(t0 - m - s - 1, least));
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = T - 2; i >= 1; --i) acc[i] = mac64(a, w[(i - s) & (T - 1)], acc[i]);
                __builtin_amdgcn_sched_barrier(0);
                const v4i an = align_a(next, sh);
                __builtin_amdgcn_sched_barrier(0);
                acc[0] = mac64(a, w[(0 - s) & (T - 1)], acc[0]);
                a = an;
                if (s + 1 >= cnt) break;
            }
        }
    }
}

// One workgroup's view of a product.
template <int NW, int UPW, int MODE, int T, bool ST>
struct Wg {
    static constexpr bool LOW = MODE != kFull;
    static constexpr int NU = NW * UPW;          // units
    static constexpr int RU = T / 4;              // result rows per unit
    static constexpr int NR = RU * UPW;           // result rows per wave
    static constexpr int RW = LOW ? NR : (NR + 1) / 2;  // operand rows per wave
    static constexpr uint32_t LANES = 64 * RW * NW;  // operand chunks the lanes can hold
    static constexpr uint32_t CAP = (LOW ? 16 : 8) * T * NU;  // operand chunks of the largest product
    // ST: straight-line steps for the largest size, smaller ones padded with
    // zero digits
    static constexpr int GD = int(CAP) - (LOW ? 1 : 0), UMAX = (16 * int(CAP) + (LOW ? 62 : 63)) / 64;
    static_assert(!ST || UPW == 1, "straight-line steps take one unit per wave");
    static_assert(!LOW || UPW == 1, "low products take one unit per wave");

    uint8_t *lds;
    uint32_t lane, pw;  // pw: this wave's role
    uint32_t n, nch;
    WgLayout lo;
    LaneAddr la;

    __device__ __forceinline__ uint32_t *sums() const { return reinterpret_cast<uint32_t *>(lds + wg_layout(CAP, CAP).sum); }
    __device__ __forceinline__ uint32_t chunk(int i) const { return 64 * (pw * RW + uint32_t(i)) + lane; }
    // full products: units u and u + NU / 2 of a wave, whose costs add up to
    // the same for every wave
    __device__ __forceinline__ uint32_t unit(int u) const { return pw + uint32_t(u) * NW; }

    // Carry into wave / unit `at` from per-wave (carry out, propagates) words.
    __device__ __forceinline__ uint32_t carry_into(const uint32_t *s, uint32_t count, uint32_t at, uint32_t *out) const {
        const uint32_t v = lane < count ? s[lane] : 0u;
        const WaveCarry wc = wave_carry(ballot((v & 1u) != 0), ballot((v & 2u) != 0), 0);
        if (out) *out = count >= 64 ? wc.out : uint32_t(wc.into >> count) & 1u;
        return uint32_t(wc.into >> at) & 1u;
    }

    // Balanced digits of the operands x and y in place; t[0], t[1]: their
    // top carries.  One barrier.
    __device__ __forceinline__ void recode(uint32_t (&x)[RW][4], uint32_t (&y)[RW][4], uint32_t (&t)[2]) const {
        uint64_t G[2][RW], P[2][RW];
        uint32_t R[RW], out[2] = {0, 0}, all[2] = {1, 1};
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            R[i] = chunk(i) < nch ? kR8 : 0u;
            const uint32_t r4[4] = {R[i], R[i], R[i], R[i]};
            uint32_t s[4];
            G[0][i] = ballot(add_words<4>(x[i], r4, s) != 0);
            P[0][i] = ballot(all_ones<4>(s));
#pragma unroll
            for (int q = 0; q < 4; ++q) x[i][q] = s[q];
            G[1][i] = ballot(add_words<4>(y[i], r4, s) != 0);
            P[1][i] = ballot(all_ones<4>(s));
#pragma unroll
            for (int q = 0; q < 4; ++q) y[i][q] = s[q];
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                out[o] = wave_carry(G[o][i], P[o][i], out[o]).out;
                all[o] &= P[o][i] == ~0ull ? 1u : 0u;
            }
        }
        uint32_t cin[2] = {0, 0};
        if constexpr (NW > 1) {
            uint32_t *s = sums() + kRecodeWords;
            if (lane < 2) s[lane * kRecodeB + pw] = lane == 0 ? out[0] | (all[0] << 1) : out[1] | (all[1] << 1);
            __syncthreads();
            cin[0] = carry_into(s, NW, pw, &t[0]);
            cin[1] = carry_into(s + kRecodeB, NW, pw, &t[1]);
        } else {
            t[0] = out[0];
            t[1] = out[1];
        }
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const WaveCarry ca = wave_carry(G[0][i], P[0][i], cin[0]), cb = wave_carry(G[1][i], P[1][i], cin[1]);
            add_carry_words<4>(x[i], uint32_t(ca.into >> lane) & 1u);
            add_carry_words<4>(y[i], uint32_t(cb.into >> lane) & 1u);
            cin[0] = ca.out;
            cin[1] = cb.out;
#pragma unroll
            for (int q = 0; q < 4; ++q) { x[i][q] ^= R[i]; y[i][q] ^= R[i]; }
        }
    }

    __device__ __forceinline__ bool stored(int i) const {
        if constexpr (ST) return LANES <= CAP || chunk(i) <= CAP;
        else return chunk(i) <= nch;
    }
    // Digits into the area of a or b (the chunk of the top digit included).
    __device__ __forceinline__ void put_a(const uint32_t (&d)[RW][4]) const {
#pragma unroll
        for (int i = 0; i < RW; ++i)
            if (stored(i))
                *reinterpret_cast<uint4 *>(lds + kAPad + 16 * chunk(i)) = make_uint4(d[i][0], d[i][1], d[i][2], d[i][3]);
    }
    __device__ __forceinline__ void put_b(const uint32_t (&d)[RW][4]) const {
#pragma unroll
        for (int i = 0; i < RW; ++i)
            if (stored(i)) *reinterpret_cast<uint4 *>(lds + lo.b + 16 * (kBPad + chunk(i))) = reversed(d[i]);
    }
    // The top digits where no lane holds their chunk.  ST: for every product,
    // since its steps read the chunk whatever its size and a longer product may
    // have left a digit there (t is 0 for a product with fewer chunks than lanes).
    __device__ __forceinline__ void put_top(const uint32_t (&t)[2]) const {
        if ((ST ? LANES == CAP : nch == LANES) && threadIdx.x == 0) {
            *reinterpret_cast<uint4 *>(lds + kAPad + 16 * LANES) = make_uint4(t[0], 0, 0, 0);
            *reinterpret_cast<uint4 *>(lds + lo.b + 16 * (kBPad + LANES)) = make_uint4(0, 0, 0, t[1] << 24);
        }
    }

    // The straight-line steps of this wave's unit.
    template <int... Q>
    __device__ __forceinline__ void unit_static(std::integer_sequence<int, Q...>, v4i (&acc)[T]) const {
        const uint8_t *ap = lds + la.a, *bp = lds + lo.b + 16 * kBPad + la.b;
        ((pw == uint32_t(Q) ? static_steps<Q * T, T, GD, UMAX>(ap, la.sh, bp, acc) : void()), ...);
    }

    // The product of the digits in LDS plus the words `add`: on return
    // s[RU u + i] holds chunk `lane` of row RU unit(u) + i.  Two barriers; the
    // digit areas are free after the first.
    template <bool ADD>
    __device__ __forceinline__ void product(const uint32_t (&add)[RW][4], uint32_t (&s)[NR][4]) const {
        uint32_t x[NR][4], hv[NR][4];
        const int32_t gd = LOW ? int32_t(nch) - 1 : int32_t(nch);
        const int32_t U = (16 * int32_t(nch) + (LOW ? 62 : 63)) >> 6;
        const int32_t tiles = LOW ? int32_t(nch + 15) >> 4 : int32_t(nch + 7) >> 3;
        uint32_t *bnd = sums() + kBoundaryWords, *cs = sums() + kCarryWords;
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            v4i acc[T] = {};
            const int32_t t0 = T * int32_t(unit(u));
            if constexpr (ST) unit_static(std::make_integer_sequence<int, NU>{}, acc);
            else if (t0 < tiles) unit_steps<T>(lds + la.a, la.sh, lds + lo.b + 16 * kBPad + la.b, t0, U, gd, acc);
#pragma unroll
            for (int i = 0; i < RU; ++i) {
                const int r = RU * u + i;
                row_words(acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3], x[r], hv[r]);
                if constexpr (ADD) add_to_words(x[r], hv[r], add[r]);
            }
            if (lane == 63) bnd[unit(u)] = hv[RU * u + RU - 1][3];
        }
        __syncthreads();
        uint64_t G[NR], P[NR];
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            const uint32_t un = unit(u);
            uint32_t out = 0, all = 1;
#pragma unroll
            for (int i = 0; i < RU; ++i) {
                const int r = RU * u + i;
                const uint32_t first = i ? uint32_t(__builtin_amdgcn_readlane(hv[r - 1][3], 63))
                                         : un ? bnd[un - 1] : kBelowFirst;
                const uint32_t y[4] = {from_below(hv[r][3], first), hv[r][0], hv[r][1], hv[r][2]};
                const uint32_t g = add_words<4>(x[r], y, s[r]);
                G[r] = ballot(g != 0);
                P[r] = ballot(all_ones<4>(s[r]));
                out = wave_carry(G[r], P[r], out).out;
                all &= P[r] == ~0ull ? 1u : 0u;
            }
            if (NU > 1 && lane == 0) cs[un] = out | (all << 1);
        }
        if constexpr (NU > 1) __syncthreads();
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            uint32_t cin = NU > 1 ? carry_into(cs, NU, unit(u), nullptr) : 0u;
#pragma unroll
            for (int i = 0; i < RU; ++i) {
                const int r = RU * u + i;
                const WaveCarry wc = wave_carry(G[r], P[r], cin);
                add_carry_words<4>(s[r], uint32_t(wc.into >> lane) & 1u);
                cin = wc.out;
            }
        }
    }

    __device__ __forceinline__ void fetch(const InstRef &in, uint32_t (&x)[RW][4], uint32_t (&y)[RW][4]) const {
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            load_chunk4(in.a, in.n, chunk(i), x[i]);
            load_chunk4(in.b, in.n, chunk(i), y[i]);
        }
    }
};

}  // namespace

template <int NW, int UPW, int MODE, int T, bool ST, class Src>
__global__ __launch_bounds__(64 * NW, T >= 16 || (T > 8 && MODE == kPoly) ? 2 : T > 8 || (MODE == kPoly && NW < 4) ? 3 : 4) void conv_wg_kernel(Src src) {
    extern __shared__ __align__(16) uint8_t lds[];
    using W = Wg<NW, UPW, MODE, T, ST>;
    constexpr bool LOW = W::LOW;
    constexpr int RW = W::RW;
    const uint32_t wave = wave_in_block();
    const uint64_t count = src.count();
    W w;
    w.lds = lds;
    w.lane = lane_id();
    w.la = lane_addr();
    uint32_t x[RW][4], y[RW][4];
    uint64_t inst = blockIdx.x;
    uint32_t zeros_for = 0;  // chunks whose layout's zeros the LDS holds
    InstRef in{};
    if (inst < count) {
        in = src.get(inst);
        w.pw = wave_role<NW, LOW>(wave, inst);
        w.fetch(in, x, y);
    }
    for (; inst < count; inst += gridDim.x) {
        uint32_t *outp = in.c;
        w.pw = wave_role<NW, LOW>(wave, inst);
        w.n = in.n;
        w.nch = (in.n + 3) / 4;
        w.lo = wg_layout(ST ? W::CAP : w.nch, W::CAP);
        uint32_t t[2];
        uint32_t b[RW][4];  // Poly: the words of b
        if constexpr (MODE == kPoly) {
#pragma unroll
            for (int i = 0; i < RW; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) b[i][q] = y[i][q];
        }
        w.recode(x, y, t);
        const uint32_t held = ST ? W::CAP : w.nch;  // chunks of each digit area
        if (held != zeros_for) {  // uniform: the zero bytes around both digit areas
            zeros_for = held;
            const uint32_t za = kAPad / 16, zt = kATail, zb = kBPad, zu = kBTail;
            for (uint32_t i = threadIdx.x; i < za + zt + zb + zu; i += 64 * NW) {
                uint32_t at;
                if (i < za) at = 16 * i;
                else if (i < za + zt) at = kAPad + 16 * held + 16 * (i - za);
                else if (i < za + zt + zb) at = w.lo.b + 16 * (i - za - zt);
                else at = w.lo.b + 16 * (kBPad + held + (i - za - zt - zb));
                *reinterpret_cast<uint4 *>(lds + at) = make_uint4(0, 0, 0, 0);
            }
            __syncthreads();  // before the top digits overwrite their zeros
        }
        w.put_a(x);
        w.put_b(y);
        if constexpr (!LOW) w.put_top(t);
        __syncthreads();
        uint32_t s[W::NR][4];
        const uint64_t nxt = inst + gridDim.x;
        uint32_t da[RW][4], db[RW][4];
        if constexpr (MODE == kPoly) {
#pragma unroll
            for (int i = 0; i < RW; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) { da[i][q] = x[i][q]; db[i][q] = y[i][q]; }
        }
        auto prefetch = [&]() {
            if (nxt < count) {
                in = src.get(nxt);
                const uint32_t pw = w.pw;
                w.pw = wave_role<NW, LOW>(wave, nxt);
                w.fetch(in, x, y);
                w.pw = pw;
            }
        };
        if constexpr (MODE == kPoly) {
            uint32_t ab[RW][4], u[RW][4], v[RW][4];
            w.template product<false>(b, ab);  // a b
            w.put_b(da);
            __syncthreads();
            w.template product<true>(b, u);  // a a + b
            w.put_a(db);
            w.put_b(db);
            __syncthreads();
            w.template product<true>(b, v);  // b b + b
#pragma unroll
            for (int i = 0; i < RW; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (4 * w.chunk(i) + q >= w.n) { u[i][q] = 0; v[i][q] = 0; }
            w.recode(u, v, t);
            w.put_a(u);
            w.put_b(v);
            __syncthreads();
            prefetch();
            w.template product<true>(ab, s);  // (a a + b)(b b + b) + a b
        } else {
            prefetch();
            w.template product<false>(x, s);
        }
        const uint32_t nout = LOW ? w.n : 2 * w.n;
#pragma unroll
        for (int u = 0; u < UPW; ++u)
#pragma unroll
            for (int i = 0; i < W::RU; ++i)
                store_chunk4(outp, nout, 64 * (W::RU * w.unit(u) + uint32_t(i)) + w.lane, s[W::RU * u + i],
                             src.streams());
    }
}

template <int NW, int UPW, int MODE, int T, bool ST, class Src>
static hipError_t launch_wg(const Src &src, uint32_t nmax, uint64_t count, hipStream_t st, int num_cus) {
    using W = Wg<NW, UPW, MODE, T, ST>;
    if (nmax > 4 * W::CAP) return hipErrorInvalidValue;
    constexpr uint32_t lds_bytes = wg_layout(W::CAP, W::CAP).total;
    const void *fn = reinterpret_cast<const void *>(&conv_wg_kernel<NW, UPW, MODE, T, ST, Src>);
    static std::atomic<uint64_t> lds_set{0};
    static std::atomic<int> occ{0};  // resident workgroups per CU
    hipError_t e = lds_limit_once(fn, lds_set);
    if (e != hipSuccess) return e;
    int o = occ.load(std::memory_order_relaxed);
    if (o == 0) {
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, fn, 64 * NW, lds_bytes);
        if (e != hipSuccess) return e;
        if (o < 1) o = 1;
        occ.store(o, std::memory_order_relaxed);
    }
    const uint64_t cap = uint64_t(o) * uint64_t(num_cus > 0 ? num_cus : 1) * 8;
    const uint32_t grid = uint32_t(std::min(count, cap));
    if (grid == 0) return hipSuccess;
    hipLaunchKernelGGL((conv_wg_kernel<NW, UPW, MODE, T, ST, Src>), dim3(grid), dim3(64 * NW), lds_bytes, st, src);
    return hipGetLastError();
}

// Full products by size: one straight-line wave while its T = 4 tiles per 128
// words fit the registers (up to 640 words: batches of 2^24 words, but at most
// 2^33 products of words, of 300 / 512 / 600 words take 121 / 110 / 122 us, in
// loops over two or three units 186 / 142 / 190), two of them up to 768 words
// and above 896 (768 / 1024 words 111 / 104 us, loops 140 / 111; between the two
// the padding to 1024 costs more than it saves: 800 words 160, loops 143), else
// loops over one unit of 256 words per wave.
template <class Src>
static hipError_t launch_full(const Src &src, uint32_t nmax, uint64_t count, hipStream_t st, int num_cus) {
    if (nmax <= 256) return launch_wg<1, 1, kFull, 8, true>(src, nmax, count, st, num_cus);
    if (nmax <= 384) return launch_wg<1, 1, kFull, 12, true>(src, nmax, count, st, num_cus);
    if (nmax <= 512) return launch_wg<1, 1, kFull, 16, true>(src, nmax, count, st, num_cus);
    if (nmax <= 640) return launch_wg<1, 1, kFull, 20, true>(src, nmax, count, st, num_cus);
    if (nmax <= 768) return launch_wg<2, 1, kFull, 12, true>(src, nmax, count, st, num_cus);
    if (nmax > 896 && nmax <= 1024) return launch_wg<2, 1, kFull, 16, true>(src, nmax, count, st, num_cus);
    if (nmax <= 1024) return launch_wg<4, 1, kFull, 8, false>(src, nmax, count, st, num_cus);
    if (nmax <= 2048) return launch_wg<8, 1, kFull, 8, false>(src, nmax, count, st, num_cus);
    if (nmax <= 4096) return launch_wg<16, 1, kFull, 8, false>(src, nmax, count, st, num_cus);
    return launch_wg<16, 2, kFull, 8, false>(src, nmax, count, st, num_cus);
}

hipError_t launch_bigmul_mfma(const uint32_t *a, const uint32_t *b, uint32_t *c, uint32_t n32, uint64_t batch,
                              hipStream_t st, int num_cus) {
    if (batch == 0) return hipSuccess;
    if (n32 > kMaxLimbs32) return hipErrorInvalidValue;
    const UniformInst src{a, b, c, n32, batch, streamed_results(8 * uint64_t(n32) * batch)};
    if (n32 <= kConvSmallMax) return launch_conv_small_full(src, st, num_cus);
    return launch_full(src, n32, batch, st, num_cus);
}

hipError_t launch_bigmul_mfma_list(const ListInst &src, uint32_t nmax, uint64_t count_max, hipStream_t st,
                                   int num_cus) {
    if (nmax > kMaxLimbs32) return hipErrorInvalidValue;
    if (nmax <= kConvSmallMax) return launch_conv_small_list(src, nmax, count_max, st, num_cus);
    return launch_full(src, nmax, count_max, st, num_cus);
}

hipError_t launch_conv_fused(bool poly, const uint32_t *a, const uint32_t *b, uint32_t *c, uint32_t n, uint64_t batch,
                             hipStream_t st, int num_cus) {
    if (batch == 0) return hipSuccess;
    if (n > kMaxLimbs32) return hipErrorInvalidValue;
    const LowInst src{{a, b, c, n, batch, streamed_results(4 * uint64_t(n) * batch)}};
    if (n <= kConvSmallLowMax) return launch_conv_small_low(poly, src, st, num_cus);
    // Up to 1024 words one straight-line wave (the same batches of 600 / 768 /
    // 1024 words: 90 / 58 / 54 us, Poly 335 / 236 / 197; in loops over units of
    // 512 words 142 / 101 / 62 and 546 / 393 / 236), above it a wave per unit.
#define BI_WG(W, ST)                                                 \
    poly ? launch_wg<W, 1, kPoly, 8, ST>(src, n, batch, st, num_cus) \
         : launch_wg<W, 1, kLow, 8, ST>(src, n, batch, st, num_cus)
    if (n <= 512) return BI_WG(1, true);
    if (poly && n <= 768) return launch_wg<1, 1, kPoly, 12, true>(src, n, batch, st, num_cus);
    if (poly && n <= 1024) return launch_wg<1, 1, kPoly, 16, true>(src, n, batch, st, num_cus);
    if (!poly && n <= 768) return launch_wg<1, 1, kLow, 12, true>(src, n, batch, st, num_cus);
    if (!poly && n <= 1024) return launch_wg<1, 1, kLow, 16, true>(src, n, batch, st, num_cus);
    if (poly && n <= 1536) return launch_wg<3, 1, kPoly, 8, false>(src, n, batch, st, num_cus);
    if (n <= 2048) return BI_WG(4, false);
    if (n <= 4096) return BI_WG(8, false);
    return BI_WG(16, false);
#undef BI_WG
}

}  // namespace bi
