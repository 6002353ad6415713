// Integer products as int8 convolutions on v_mfma_i32_16x16x64_i8: the device
// parts shared by the small-product and the workgroup kernels.
//
// Digits.  An operand padded to whole 16-byte chunks is D bytes.  Adding
// R = 0x8080..80 (one carry scan) and flipping the top bit of every byte
// gives balanced digits in [-128, 127]; the carry out t in {0, 1} of that
// addition is digit D, one more digit of the convolution, so the digits
// represent the operand exactly.  |c_k| <= (D + 1) 2^14 < 2^30 for D <= 2^15:
// int32 accumulation cannot overflow.
//
// Tiles.  A tile is 256 coefficients = 16 blocks of 16 (64 product words):
//   C[256 t + 16 c + r] = sum_u sum_{s<64} a[64 u + r - s] b[256 t + 16 c - 64 u + s]
// so step u of tile t is one MFMA with A operand T_u[r][s] = a[64 u + r - s]
// and B operand columns b[16 (16 t - 4 u + c) + s].  Within each 16-byte part
// both operands run through s in reverse, so lane (r, h) reads the 16
// ascending bytes a[64 u + r - 16 h - 15 ..] and lane (c, h) the 16-digit
// group 16 t - 4 u + c + h of b, stored byte-reversed.
//
// A operands come straight from the digit bytes: a lane's 16 bytes start at a
// byte offset whose low two bits depend on the lane alone, so it reads the
// five aligned words that cover them and shifts (four v_alignbyte).  Lanes
// share those words (the LDS broadcasts them): no conflicts, and no shifted
// copies of a to build and hold.
//
// B of tile t + 1 at step u + 4 is B of tile t at step u.  With the residue
// kappa = u mod 4 outer and m = u / 4 inner, tile t at m takes B operand
// j = t - m: a wave that owns consecutive tiles keeps one B operand per tile
// in registers and reads one A and one new B per step of all its tiles.
//
// A lane's four accumulators of a tile are one product word, and a 4 x 4
// exchange between tiles and 16-lane groups leaves every lane with the four
// words of one 16-byte chunk, in lane order.
#pragma once

#include "bi_common.hpp"
#include "bi_internal.hpp"
#include "conv_layout.hpp"

namespace bi {
namespace conv {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef u32x4 __attribute__((aligned(4))) u32x4_a4;  // 16 bytes at any word address

enum Mode { kFull = 0, kLow = 1, kPoly = 2 };

constexpr uint32_t kR8 = 0x80808080u;

// The four words of chunk c of an n-word operand (zero at or above n).
__device__ __forceinline__ void load_chunk4(const uint32_t *p, uint32_t n, uint32_t c, uint32_t (&x)[4]) {
    const uint32_t base = 4 * c;
    if (base + 4 <= n) {
        const u32x4 v = *reinterpret_cast<const u32x4_a4 *>(p + base);
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) x[t] = base + t < n ? p[base + t] : 0u;
    }
}

// Stores the words of chunk c that lie below n (`stream`, uniform: past the
// caches).
__device__ __forceinline__ void store_chunk4(uint32_t *p, uint32_t n, uint32_t c, const uint32_t (&x)[4], bool stream) {
    const uint32_t base = 4 * c;
    if (base + 4 <= n) {
        const u32x4 v = {x[0], x[1], x[2], x[3]};
        u32x4_a4 *q = reinterpret_cast<u32x4_a4 *>(p + base);
        if (stream) {
            // kept apart from the other store: merged, it would lose the hint
            asm volatile("" ::: "memory");
            __builtin_nontemporal_store(v, q);
            asm volatile("" ::: "memory");
        } else {
            *q = v;
        }
    } else {
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (base + t < n) p[base + t] = x[t];
    }
}

// The digit words of a chunk with its bytes in reverse order (a B group).
__device__ __forceinline__ uint4 reversed(const uint32_t (&d)[4]) {
    return make_uint4(__builtin_bswap32(d[3]), __builtin_bswap32(d[2]), __builtin_bswap32(d[1]),
                      __builtin_bswap32(d[0]));
}

// Bytes an area of a needs so that step u <= umax stays inside it.
__host__ __device__ constexpr uint32_t a_bytes(uint32_t umax) { return (64 * umax + 84 + 15) & ~15u; }

// Operand addresses of a lane, relative to an area of a (kAPad zero bytes
// before digit 0) and to group 0 of an area of b.
struct LaneAddr {
    uint32_t a, sh, b;
};
__device__ __forceinline__ LaneAddr lane_addr() {
    const uint32_t r = lane_id() & 15u, h = lane_id() >> 4;
    const uint32_t p = kAPad - 15 + r;
    return LaneAddr{(p & ~3u) - 16 * h, p & 3u, 16 * (r + h)};
}

struct ARaw {
    uint32_t w[5];
};
__device__ __forceinline__ ARaw read_a(const uint8_t *p) {
    const uint32_t *q = reinterpret_cast<const uint32_t *>(p);
    return ARaw{{q[0], q[1], q[2], q[3], q[4]}};
}
__device__ __forceinline__ v4i align_a(const ARaw &x, uint32_t sh) {
    return v4i{int(__builtin_amdgcn_alignbyte(x.w[1], x.w[0], sh)), int(__builtin_amdgcn_alignbyte(x.w[2], x.w[1], sh)),
               int(__builtin_amdgcn_alignbyte(x.w[3], x.w[2], sh)), int(__builtin_amdgcn_alignbyte(x.w[4], x.w[3], sh))};
}
__device__ __forceinline__ v4i read_b(const uint8_t *p) { return *reinterpret_cast<const v4i *>(p); }

__device__ __forceinline__ v4i mac64(v4i a, v4i b, v4i c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// A product of at most TPI tiles: the sizes of its digit areas.  Full
// products have half as many operand chunks as result chunks and a top digit
// each; low products (mod 2^N) as many, and their top carries reach no
// coefficient below 2^N.
template <int TPI, bool LOW>
struct Small {
    static constexpr uint32_t kPad = 16;                  // zero groups below group 0 of b
    static constexpr int IPW = TPI < 4 ? 4 / TPI : 1;      // instances per wave
    static constexpr int CPI = LOW ? 16 * TPI : 8 * TPI;   // operand chunks per instance
    static constexpr int GD = LOW ? CPI - 1 : CPI;         // last 16-digit group that may be nonzero
    static constexpr int U = (16 * CPI - (LOW ? 1 : 0) + 63) / 64;  // last step
    static constexpr uint32_t AB = a_bytes(U);
    static constexpr int JMAX = GD / 16 < TPI - 1 ? GD / 16 : TPI - 1;  // at kappa 0, which reaches highest
    static constexpr uint32_t BB = 16 * (kPad + 16 * JMAX + 19);
    static constexpr uint32_t INST = AB + BB;
    static constexpr uint32_t WAVE = IPW * INST;  // LDS bytes per wave
    static_assert(kAPad + 16 * CPI + (LOW ? 0 : 16) <= AB, "digits of a fit their area");
    static_assert(16 * (kPad + CPI + (LOW ? 0 : 1)) <= BB, "digits of b fit their area");
};

// All steps of one instance of at most TPI tiles, straight-line.  ap / bp: this lane's operand addresses.
template <int TPI, bool LOW>
__device__ __forceinline__ void small_steps(const uint8_t *ap, uint32_t sh, const uint8_t *bp, v4i *acc) {
    using S = Small<TPI, LOW>;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int J = (S::GD + 4 * k) / 16 < TPI - 1 ? (S::GD + 4 * k) / 16 : TPI - 1;
        const int j0 = k == 0 ? -1 : 0;
        const int M = (S::U - k) / 4;
        v4i w[TPI + 1];
#pragma unroll
        for (int j = j0; j <= J; ++j) w[j - j0] = read_b(bp + 256 * j - 64 * k);
#pragma unroll
        for (int m = 0; m <= M; ++m) {
            if (k + 4 * m > S::U) continue;
            const v4i a = align_a(read_a(ap + 64 * (k + 4 * m)), sh);
#pragma unroll
            for (int t = 0; t < TPI; ++t) {
                const int j = t - m;
                if (j >= j0 && j <= J) acc[t] = mac64(a, w[j - j0], acc[t]);
            }
        }
    }
}

// The steps of tiles T0 .. T0 + T - 1 of a product with groups 0 .. GD of b
// and steps up to U of a, straight-line: only MFMAs inside the band, the
// operands of each step requested before the MFMAs of the one before it.
template <int T0, int T, int GD, int U>
__device__ __forceinline__ void static_steps(const uint8_t *ap, uint32_t sh, const uint8_t *bp, v4i (&acc)[T]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int J = (GD + 4 * k) / 16, j0 = k == 0 ? -1 : 0, M = (U - k) / 4;
        const int mlo = T0 > J ? T0 - J : 0, mhi = M < T0 + T - 1 - j0 ? M : T0 + T - 1 - j0;
        v4i w[(GD + 12) / 16 + 2];  // B operand j at j + 1
#pragma unroll
        for (int j = j0; j <= J; ++j)
            if (j >= T0 - mlo && j <= T0 - mlo + T - 1) w[j + 1] = read_b(bp + 256 * j - 64 * k);
        v4i a = align_a(read_a(ap + 64 * k + 256 * mlo), sh);
#pragma unroll
        for (int m = mlo; m <= mhi; ++m) {
            ARaw next;
            if (m < mhi) {
                next = read_a(ap + 64 * k + 256 * (m + 1));
                const int j = T0 - m - 1;
                if (j >= j0 && j <= J) w[j + 1] = read_b(bp + 256 * j - 64 * k);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = T - 1; i >= 0; --i) {
                const int j = T0 + i - m;
                if (j >= j0 && j <= J) acc[i] = mac64(a, w[j + 1], acc[i]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (m < mhi) a = align_a(next, sh);
        }
    }
}

// LDS written by this wave is read by its other lanes: the LDS serves one
// wave's instructions in order, so only the compiler has to keep them.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Word values of a row of four tiles, lo[w] and hi[w] of words 4 lane + w.
// V = sum_e c_e 2^(8e) + 2^63 - 2^31 lies in [0, 2^64); the bias 2^63 of a
// word and -2^31 of the next cancel, so the words below the first one of a
// product count as hi = 2^31 (kBelowFirst) and 2^63 stays above the last.
constexpr uint32_t kBelowFirst = 0x80000000u;

// The factors are opaque to the compiler so that each term is one
// v_mad_i64_i32 instead of a sign extension, a 64-bit shift and an add.  (Not
// inline asm: the compiler inserts the wait states between an MFMA and a read
// of its result only for instructions it knows.)
struct WordScale {
    int32_t f[4] = {1, 1 << 8, 1 << 16, 1 << 24};
    __device__ __forceinline__ WordScale() {
#pragma unroll
        for (int e = 0; e < 4; ++e) asm("" : "+s"(f[e]));
    }
};

__device__ __forceinline__ uint64_t word_value(const v4i &c, const WordScale &k) {
    int64_t v = int64_t((1ull << 63) - (1ull << 31));
#pragma unroll
    for (int e = 0; e < 4; ++e) v = int64_t(uint64_t(v) + uint64_t(int64_t(c[e]) * int64_t(k.f[e])));
    return uint64_t(v);
}

// (register q, lane group h) <-> (register h, lane group q)
__device__ __forceinline__ void exchange4(uint32_t (&v)[4]) {
    const auto s02 = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
    const auto s13 = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
    const auto s01 = __builtin_amdgcn_permlane16_swap(s02[0], s13[0], false, false);
    const auto s23 = __builtin_amdgcn_permlane16_swap(s02[1], s13[1], false, false);
    v[0] = s01[0]; v[1] = s01[1]; v[2] = s23[0]; v[3] = s23[1];
}

__device__ __forceinline__ void row_words(const v4i &c0, const v4i &c1, const v4i &c2, const v4i &c3,
                                          uint32_t (&lo)[4], uint32_t (&hi)[4]) {
    const WordScale k;
    const uint64_t v[4] = {word_value(c0, k), word_value(c1, k), word_value(c2, k), word_value(c3, k)};
#pragma unroll
    for (int q = 0; q < 4; ++q) { lo[q] = uint32_t(v[q]); hi[q] = uint32_t(v[q] >> 32); }
    exchange4(lo);
    exchange4(hi);
}

// Adds the words y into (lo, hi): V + y stays below 2^64.
__device__ __forceinline__ void add_to_words(uint32_t (&lo)[4], uint32_t (&hi)[4], const uint32_t (&y)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t c;
        lo[q] = __builtin_addc(lo[q], y[q], 0u, &c);
        hi[q] += c;
    }
}

// hi[3] of the lane below; lane 0 takes `first`.
__device__ __forceinline__ uint32_t from_below(uint32_t v, uint32_t first) {
    return uint32_t(__builtin_amdgcn_update_dpp(int(first), int(v), 0x138 /* wave_shr:1 */, 0xf, 0xf, false));
}

}  // namespace conv
}  // namespace bi
