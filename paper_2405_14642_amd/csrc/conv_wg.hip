// Products of up to 8192 words on int8 matrix cores, one workgroup per
// product: full products above 128 words, low products (mod 2^N) and Poly
// above 256.  See bi_conv.hpp for the digits, tiles and operand layout.
//
// A unit is eight tiles (two rows of 256 words).  A wave owns UPW units and
// walks, per residue kappa, the steps m of a unit with the eight B operands
// j = t - m of its tiles in registers: one A and one new B operand per step
// of eight MFMAs.  Steps where every tile is in band run straight; at the
// ends of a band straight-line triangles leave out the MFMAs whose operand
// is zero.  Products of one unit run straight-line altogether.
//
// What bounds it: the matrix cores from 1024 words up (at 1024 words a
// product is 1120 MFMAs of 16 clk, 1024 of them inside the band: 17.9k clk
// of one SIMD), the chain recode - steps - carries below, which four waves
// per SIMD of several workgroups overlap.  Eight tiles per unit: the LDS
// traffic per MFMA falls with the tiles (2.25 KB per step), the registers
// grow (four accumulators and four B words per tile and lane); eight leave
// 128 registers for four waves per SIMD.  Measured against the kernel before
// it (32 x 32 x 32 tiles over 8-byte windows of a in LDS; three kernels and
// global scratch above 1024 words): 4096 x 1024 words 81.4 -> 62.1 us (2.2e15
// int8 ops/s), 8192 x 512 words 61.7 -> 40.7, 16384 x 256 words 51.9 -> 24.5,
// 2048 x 2048 words 198 -> 102, 512 x 4096 words 196 -> 91 us.  Low products
// and Poly against the VALU schoolbook in LDS: 16384 x 512 words 266 -> 40.5
// us, 4096 x 2048 words (Poly) 3041 -> 408, 128 x 8192 words 657 -> 78 and
// (Poly) 2631 -> 303.
#include <algorithm>
#include <atomic>

#include "bi_conv.hpp"

namespace bi {

namespace {

using namespace conv;

constexpr int kT = 8;            // tiles per unit
constexpr uint32_t kATail = 7;   // 16-byte pieces after a's digits (steps read up to 83 bytes past them)
constexpr uint32_t kBPad = 32;   // zero groups below group 0 of b: B operand -2 at kappa 0, -1 above
constexpr uint32_t kBTail = 35;  // groups from the top digit's on: B operand J + 1

// Byte offsets of the dynamic LDS block of products of nch chunks.
struct WgLayout {
    uint32_t b, sum, total;
};
__host__ __device__ inline WgLayout wg_layout(uint32_t nch) {
    WgLayout l;
    l.b = kAPad + 16 * (nch + kATail);              // a: digits, the top digit, zeros
    l.sum = l.b + 16 * (kBPad + nch + kBTail);      // b: groups, the top digit, zeros
    l.total = l.sum + 4 * 4 * 64;                // recode, boundary and carry words
    return l;
}

// Order of the units over the waves: cost grows with the unit (low products)
// or peaks in the middle (full ones), and waves w, w + 4, w + 8, .. share a
// SIMD.
template <int NW, bool LOW>
__device__ __forceinline__ uint32_t wave_role(uint32_t wave, uint64_t inst) {
    if constexpr (NW == 1) return 0;
    else if constexpr (NW <= 4) return (wave + uint32_t(inst)) % NW;
    else if constexpr (LOW) return (wave & 4u) ? (wave ^ 3u) : wave;
    else return wave;
}

// Eight steps m .. m + 7 of a unit from a window w (slot i: B operand
// t0 - m + i), sliding it as they go.  SHAPE: every tile in band (kAll); only
// tiles i <= s of step s (kEntry: the first step takes the last B operand);
// only tiles i >= s (kExit: the last step takes B operand 0).
enum Shape { kAll, kEntry, kExit };
template <int SHAPE>
__device__ __forceinline__ void block8(const uint8_t *am, uint32_t sh, const uint8_t *bj, v4i (&w)[kT],
                                       v4i (&acc)[kT]) {
    ARaw next = read_a(am);
#pragma unroll
    for (int s = 0; s < kT; ++s) {
        const v4i a = align_a(next, sh);
        if (s + 1 < kT) next = read_a(am + 256 * (s + 1));
#pragma unroll
        for (int i = kT - 1; i >= 0; --i)
            if (SHAPE == kAll || (SHAPE == kEntry ? i <= s : i >= s))
                acc[i] = mac64(a, w[(i - s) & (kT - 1)], acc[i]);
        // the window of the next step starts one B operand lower
        if (SHAPE != kExit) w[(kT - 1 - s) & (kT - 1)] = read_b(bj - 256 * (s + 1));
    }
}

// Adds the steps of the unit at tile t0 into acc.  U: last step with a
// nonzero A operand; gd: last nonzero group of b.  B operands above J are
// zero, and those below 0 but for -1 at kappa 0.
__device__ __forceinline__ void unit_steps(const uint8_t *ap, uint32_t sh, const uint8_t *bp, int32_t t0, int32_t U,
                                           int32_t gd, v4i (&acc)[kT]) {
#pragma unroll 1
    for (int32_t k = 0; k < 4; ++k) {
        const int32_t J = (gd + 4 * k) >> 4, M = (U - k) >> 2;
        const uint8_t *ak = ap + 64 * k, *bk = bp - 64 * k;
        // the unit's band ends inside the steps of a (exit shape), or a ends first
        const bool exits = M >= t0 + kT - 1;
        int32_t m = max(0, t0 - J);
        const int32_t end = exits ? t0 : min(M, t0 + kT) + 1;
        if (exits || end - m >= kT) {
            v4i w[kT];
#pragma unroll
            for (int i = 0; i < kT; ++i) w[i] = read_b(bk + 256 * min(t0 - m + i, J + 1));
            if (!exits && t0 >= J) {
                block8<kEntry>(ak + 256 * m, sh, bk + 256 * (t0 - m), w, acc);
                m += kT;
            }
#pragma unroll 1
            for (; m + kT <= end; m += kT) block8<kAll>(ak + 256 * m, sh, bk + 256 * (t0 - m), w, acc);
            if (exits) {
                block8<kExit>(ak + 256 * m, sh, bk + 256 * (t0 - m), w, acc);
                m += kT;
                if (k == 0) {  // B operand -1 reaches 16 digits of the product below tile m
                    const v4i b = read_b(bk - 256);
#pragma unroll
                    for (int i = 0; i < kT; ++i)
                        if (i < kT - 1 || m <= M)
                            acc[i] = mac64(align_a(read_a(ak + 256 * (t0 + i + 1)), sh), b, acc[i]);
                }
            }
        }
if (m < end) {  // fewer than eight steps left
            const int32_t least = k == 0 ? -2 : -1, cnt = end - m;
            const uint8_t *am = ak + 256 * m;
            v4i w[kT];
#pragma unroll
            for (int i = 0; i < kT; ++i) w[i] = read_b(bk + 256 * max(min(t0 - m + i, J + 1), least));
            ARaw next = read_a(am);
#pragma unroll
            for (int s = 0; s < kT - 1; ++s) {
                const v4i a = align_a(next, sh);
                next = read_a(am + 256 * min(s + 1, cnt - 1));
#pragma unroll
                for (int i = kT - 1; i >= 0; --i) acc[i] = mac64(a, w[(i - s) & (kT - 1)], acc[i]);
                w[(kT - 1 - s) & (kT - 1)] = read_b(bk + 256 * max(t0 - m - s - 1, least));
                if (s + 1 >= cnt) break;
            }
        }
    }
}

// One workgroup's view of a product.
template <int NW, int UPW, int MODE>
struct Wg {
    static constexpr bool LOW = MODE != kFull;
    static constexpr int NU = NW * UPW;          // units
    static constexpr int RW = LOW ? 2 * UPW : UPW;  // operand rows per wave
    static constexpr uint32_t CAP = 64 * RW * NW;   // operand chunks held by the workgroup
    // one unit holds the whole product: straight-line steps for the largest
    // size, smaller ones padded with zero digits
    static constexpr bool ONE = NU == 1;
    static_assert(!LOW || UPW == 1, "low products take one unit per wave");

    uint8_t *lds;
    uint32_t lane, pw;  // pw: this wave's role
    uint32_t n, nch;
    WgLayout lo;
    LaneAddr la;

    __device__ __forceinline__ uint32_t *sums() const { return reinterpret_cast<uint32_t *>(lds + lo.sum); }
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
            uint32_t *s = sums();
            if (lane < 2) s[32 * lane + pw] = lane == 0 ? out[0] | (all[0] << 1) : out[1] | (all[1] << 1);
            __syncthreads();
            cin[0] = carry_into(s, NW, pw, &t[0]);
            cin[1] = carry_into(s + 32, NW, pw, &t[1]);
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

    // Digits into the area of a or b (the chunk of the top digit included).
    __device__ __forceinline__ void put_a(const uint32_t (&d)[RW][4]) const {
#pragma unroll
        for (int i = 0; i < RW; ++i)
            if (ONE || chunk(i) <= nch)
                *reinterpret_cast<uint4 *>(lds + kAPad + 16 * chunk(i)) = make_uint4(d[i][0], d[i][1], d[i][2], d[i][3]);
    }
    __device__ __forceinline__ void put_b(const uint32_t (&d)[RW][4]) const {
#pragma unroll
        for (int i = 0; i < RW; ++i)
            if (ONE || chunk(i) <= nch) *reinterpret_cast<uint4 *>(lds + lo.b + 16 * (kBPad + chunk(i))) = reversed(d[i]);
    }
    // The top digits where no lane holds their chunk.
    __device__ __forceinline__ void put_top(const uint32_t (&t)[2]) const {
        if (nch == CAP && threadIdx.x == 0) {
            *reinterpret_cast<uint4 *>(lds + kAPad + 16 * nch) = make_uint4(t[0], 0, 0, 0);
            *reinterpret_cast<uint4 *>(lds + lo.b + 16 * (kBPad + nch)) = make_uint4(0, 0, 0, t[1] << 24);
        }
    }

    // The product of the digits in LDS plus the words `add`: on return
    // s[2 u + i] holds chunk `lane` of row 2 unit(u) + i.  Two barriers; the
    // digit areas are free after the first.
    template <bool ADD>
    __device__ __forceinline__ void product(const uint32_t (&add)[RW][4], uint32_t (&s)[2 * UPW][4]) const {
        uint32_t x[2 * UPW][4], hv[2 * UPW][4];
        const int32_t gd = LOW ? int32_t(nch) - 1 : int32_t(nch);
        const int32_t U = (16 * int32_t(nch) + (LOW ? 62 : 63)) >> 6;
        const int32_t tiles = LOW ? int32_t(nch + 15) >> 4 : int32_t(nch + 7) >> 3;
        uint32_t *bnd = sums() + 64, *cs = sums() + 128;
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            v4i acc[kT] = {};
            const int32_t t0 = kT * int32_t(unit(u));
            if constexpr (ONE) small_steps<kT, LOW>(lds + la.a, la.sh, lds + lo.b + 16 * kBPad + la.b, acc);
            else if (t0 < tiles) unit_steps(lds + la.a, la.sh, lds + lo.b + 16 * kBPad + la.b, t0, U, gd, acc);
            row_words(acc[0], acc[1], acc[2], acc[3], x[2 * u], hv[2 * u]);
            row_words(acc[4], acc[5], acc[6], acc[7], x[2 * u + 1], hv[2 * u + 1]);
            if constexpr (ADD) {
                add_to_words(x[2 * u], hv[2 * u], add[2 * u]);
                add_to_words(x[2 * u + 1], hv[2 * u + 1], add[2 * u + 1]);
            }
            if (lane == 63) bnd[unit(u)] = hv[2 * u + 1][3];
        }
        __syncthreads();
        uint64_t G[2 * UPW], P[2 * UPW];
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            const uint32_t un = unit(u);
            uint32_t out = 0, all = 1;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = 2 * u + i;
                const uint32_t first = i ? uint32_t(__builtin_amdgcn_readlane(hv[2 * u][3], 63))
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
            for (int i = 0; i < 2; ++i) {
                const int r = 2 * u + i;
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

template <int NW, int UPW, int MODE, class Src>
__global__ __launch_bounds__(64 * NW, MODE == kPoly && NW < 16 ? 3 : 4) void conv_wg_kernel(Src src) {
    extern __shared__ __align__(16) uint8_t lds[];
    using W = Wg<NW, UPW, MODE>;
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
        w.lo = wg_layout(W::ONE ? W::CAP : w.nch);
        uint32_t t[2];
        uint32_t b[RW][4];  // Poly: the words of b
        if constexpr (MODE == kPoly) {
#pragma unroll
            for (int i = 0; i < RW; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) b[i][q] = y[i][q];
        }
        w.recode(x, y, t);
        const uint32_t held = W::ONE ? W::CAP : w.nch;  // chunks of each digit area
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
        uint32_t s[2 * UPW][4];
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
            uint32_t ab[RW][4], T[RW][4], V[RW][4];
            w.template product<false>(b, ab);  // a b
            w.put_b(da);
            __syncthreads();
            w.template product<true>(b, T);  // a a + b
            w.put_a(db);
            w.put_b(db);
            __syncthreads();
            w.template product<true>(b, V);  // b b + b
#pragma unroll
            for (int i = 0; i < RW; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (4 * w.chunk(i) + q >= w.n) { T[i][q] = 0; V[i][q] = 0; }
            w.recode(T, V, t);
            w.put_a(T);
            w.put_b(V);
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
            for (int i = 0; i < 2; ++i) store_chunk4(outp, nout, 64 * (2 * w.unit(u) + uint32_t(i)) + w.lane, s[2 * u + i]);
    }
}

template <int NW, int UPW, int MODE, class Src>
static hipError_t launch_wg(const Src &src, uint32_t nmax, uint64_t count, hipStream_t st, int num_cus) {
    using W = Wg<NW, UPW, MODE>;
    const uint32_t lds_bytes = wg_layout(W::ONE ? W::CAP : (nmax + 3) / 4).total;
    const void *fn = reinterpret_cast<const void *>(&conv_wg_kernel<NW, UPW, MODE, Src>);
    // (LDS bytes << 32 | resident workgroups per CU) of the last launch shape
    static std::atomic<uint64_t> occ{0}, lds_set{0};
    hipError_t e = lds_limit_once(fn, lds_set);
    if (e != hipSuccess) return e;
    uint64_t o = occ.load(std::memory_order_relaxed);
    if ((o >> 32) != lds_bytes) {
        int nblk = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nblk, fn, 64 * NW, lds_bytes);
        if (e != hipSuccess) return e;
        o = (uint64_t(lds_bytes) << 32) | uint32_t(nblk < 1 ? 1 : nblk);
        occ.store(o, std::memory_order_relaxed);
    }
    const uint64_t cap = uint64_t(uint32_t(o)) * uint64_t(num_cus > 0 ? num_cus : 1);
    const uint32_t grid = uint32_t(std::min(count, cap));
    if (grid == 0) return hipSuccess;
    hipLaunchKernelGGL((conv_wg_kernel<NW, UPW, MODE, Src>), dim3(grid), dim3(64 * NW), lds_bytes, st, src);
    return hipGetLastError();
}

template <class Src>
static hipError_t launch_full(const Src &src, uint32_t nmax, uint64_t count, hipStream_t st, int num_cus) {
    if (nmax <= 256) return launch_wg<1, 1, kFull>(src, nmax, count, st, num_cus);
    if (nmax <= 512) return launch_wg<2, 1, kFull>(src, nmax, count, st, num_cus);
    if (nmax <= 1024) return launch_wg<4, 1, kFull>(src, nmax, count, st, num_cus);
    if (nmax <= 2048) return launch_wg<8, 1, kFull>(src, nmax, count, st, num_cus);
    if (nmax <= 4096) return launch_wg<16, 1, kFull>(src, nmax, count, st, num_cus);
    return launch_wg<16, 2, kFull>(src, nmax, count, st, num_cus);
}

hipError_t launch_bigmul_mfma(const uint32_t *a, const uint32_t *b, uint32_t *c, uint32_t n32, uint64_t batch,
                              hipStream_t st, int num_cus) {
    if (batch == 0) return hipSuccess;
    if (n32 > kMaxLimbs32) return hipErrorInvalidValue;
    const UniformInst src{a, b, c, n32, batch};
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
    const LowInst src{{a, b, c, n, batch}};
    if (n <= kConvSmallLowMax) return launch_conv_small_low(poly, src, st, num_cus);
#define BI_WG(W)                                              \
    poly ? launch_wg<W, 1, kPoly>(src, n, batch, st, num_cus) \
         : launch_wg<W, 1, kLow>(src, n, batch, st, num_cus)
    if (n <= 512) return BI_WG(1);
    if (n <= 1024) return BI_WG(2);
    if (n <= 2048) return BI_WG(4);
    if (n <= 4096) return BI_WG(8);
    return BI_WG(16);
#undef BI_WG
}

}  // namespace bi
