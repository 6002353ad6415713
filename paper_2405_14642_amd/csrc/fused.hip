// Fused multi-operation programs (Section 6.1): several same-length
// operations per instance in one kernel, the intermediates kept in registers
// and LDS, the operands read from HBM once and the result written once.
//
//   BI_PROG_ADD6  six additions, a + b, then + a, + b, + a, + b, + a in turn:
//                 4 a + 3 b mod 2^N (the paper names only "six additions";
//                 this alternating chain is the reading taken).
//   BI_PROG_POLY  (a a + b) (b b + b) + a b mod 2^N: four same-length products
//                 (the low n limbs of eq. (1)) and three additions.
//   BI_PROG_MUL_LOW  a b mod 2^N alone: the paper's same-length product of
//                 Figs. 4-5 (only the coefficients below n are formed).
//
// The six additions keep every operand in registers: each lane holds the
// same 4-word chunks of a, b and the running sum throughout.  Instances of up
// to 256 words are packed several to a wave (a segmented ballot-adder: the
// last chunk of an instance neither generates nor propagates into the next),
// larger ones take a workgroup whose waves exchange one carry summary per
// addition.
//
// Products and Poly above 32 words run on the matrix cores (launch_conv_fused).
// Shorter instances share wavefronts on the VALU (fused_packed_kernel): an
// instance takes a segment of lanes, its operands sit in the wavefront's own
// LDS areas and each lane accumulates its output words over a sliding window
// (Section 3), the (high, carry) pair moves to the next lane by a lane shuffle
// and the segment's chunks are added with one ballot-adder step, so Poly's
// intermediates stay in registers but for the two factors of its last product.
#include <algorithm>
#include <atomic>

#include "bi_common.hpp"
#include "bi_internal.hpp"
#include "bi_valu.hpp"

namespace bi {

constexpr int kPackedQ = 2;  // output words per lane of the packed kernels

namespace {

typedef u32x4 __attribute__((aligned(4))) u32x4_word;  // 16 bytes at any word address

// A lane's 4-word chunk c of an n-word operand in two steps, so that all of a
// lane's loads are in flight before the first is used (a branch for the ragged
// chunk at each load made every load wait for the one before it): the 16 bytes
// at the chunk, or the operand's last 16 where the chunk ends past it (n >= 4),
// then the words moved into place, zero past n or when not valid.
template <bool NT>
__device__ __forceinline__ u32x4 load_raw(const uint32_t *p, uint32_t n, uint32_t c) {
    const u32x4_word *q = reinterpret_cast<const u32x4_word *>(p + min(4 * c, n - 4));
    return NT ? __builtin_nontemporal_load(q) : *q;
}
__device__ __forceinline__ void place_words(const u32x4 &v, uint32_t n, uint32_t c, bool valid, uint32_t (&x)[4]) {
    x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    if (n & 3u) {
        const uint32_t s = 4 * c + 4 > n ? 4 * c + 4 - n : 0u;  // words of the chunk past n
        if (s & 1u) { x[0] = x[1]; x[1] = x[2]; x[2] = x[3]; x[3] = 0; }
        if (s & 2u) { x[0] = x[2]; x[1] = x[3]; x[2] = 0; x[3] = 0; }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) x[t] = valid ? x[t] : 0u;
}

// Operands of fewer than 4 words.
__device__ __forceinline__ void load_short(const uint32_t *p, uint32_t n, bool valid, uint32_t (&x)[4]) {
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) x[t] = valid && t < n ? p[t] : 0u;
}

// Stores the words of chunk c below n when valid.
template <bool NT>
__device__ __forceinline__ void store_chunk(uint32_t *p, uint32_t n, uint32_t c, bool valid, const uint32_t (&x)[4]) {
    if (!valid) return;
    const uint32_t base = 4 * c;
    if (base + 4 <= n) {
        const u32x4 v = {x[0], x[1], x[2], x[3]};
        u32x4_word *q = reinterpret_cast<u32x4_word *>(p + base);
        if (NT) __builtin_nontemporal_store(v, q); else *q = v;
    } else {
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (base + t < n) p[base + t] = x[t];
    }
}

}  // namespace

// Instances of up to 256 words (64 chunks): 64 / 2^seg_log instances per row,
// ROWS rows per wave, lane j of segment s holding chunk j of instance s.
// `keep` masks the lanes whose carry may reach the next lane: not an
// instance's last chunk (its carry out is dropped, mod 2^N) and not past the
// instance's end.
template <int ROWS, bool NTL, bool NTS>
__global__ __launch_bounds__(256) void fused_add6_packed_kernel(const uint32_t *__restrict__ a,
                                                                const uint32_t *__restrict__ b,
                                                                uint32_t *__restrict__ out, uint32_t n,
                                                                uint64_t batch, uint32_t seg_log) {
    const uint32_t lane = lane_id(), wave = wave_in_block();
    const uint32_t nchunks = (n + 3) / 4, ipw = 64u >> seg_log;
    const uint32_t j = lane & ((1u << seg_log) - 1u);
    for (uint64_t g = uint64_t(blockIdx.x) * 4 + wave; g * ipw * ROWS < batch; g += uint64_t(gridDim.x) * 4) {
        const uint64_t inst0 = g * ipw * ROWS + (lane >> seg_log);
        uint32_t A[ROWS][4], B[ROWS][4], X[ROWS][4];
        bool valid[ROWS];
        if (n >= 4) {
            u32x4 va[ROWS], vb[ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const uint64_t at = min(inst0 + r * ipw, batch - 1) * n;
                va[r] = load_raw<NTL>(a + at, n, j);
                vb[r] = load_raw<NTL>(b + at, n, j);
            }
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                valid[r] = inst0 + r * ipw < batch && j < nchunks;
                place_words(va[r], n, j, valid[r], A[r]);
                place_words(vb[r], n, j, valid[r], B[r]);
            }
        } else {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                valid[r] = inst0 + r * ipw < batch && j < nchunks;
                load_short(a + (inst0 + r * ipw) * n, n, valid[r], A[r]);
                load_short(b + (inst0 + r * ipw) * n, n, valid[r], B[r]);
            }
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const uint64_t keep = ballot(valid[r] && j + 1 < nchunks);
            auto add = [&](const uint32_t (&y)[4]) {
                uint32_t s[4];
                const uint32_t gen = add_words<4>(X[r], y, s);
                const uint64_t G = ballot(gen != 0) & keep, P = ballot(all_ones<4>(s)) & keep;
                add_carry_words<4>(s, uint32_t(wave_carry(G, P, 0).into >> lane) & 1u);
#pragma unroll
                for (int t = 0; t < 4; ++t) X[r][t] = s[t];
            };
#pragma unroll
            for (int t = 0; t < 4; ++t) X[r][t] = A[r][t];
            add(B[r]);
            add(A[r]);
            add(B[r]);
            add(A[r]);
            add(B[r]);
            add(A[r]);
            store_chunk<NTS>(out + (inst0 + r * ipw) * n, n, j, valid[r], X[r]);
        }
    }
}

// Instances above 256 words: one workgroup of NW waves, wave w holding rows
// w R .. w R + R - 1 (64 chunks each) in registers.  Per addition each wave
// scans its rows, publishes (carry out, all-propagate) in one LDS word,
// and after one barrier applies the carry from the waves below; the summary
// words alternate between two arrays so one barrier per addition suffices.
template <int NW, int R, bool NTL, bool NTS>
__global__ __launch_bounds__(64 * NW) void fused_add6_rows_kernel(const uint32_t *__restrict__ a,
                                                                  const uint32_t *__restrict__ b,
                                                                  uint32_t *__restrict__ out, uint32_t n,
                                                                  uint64_t batch) {
    __shared__ uint32_t summary[2][NW];
    const uint32_t lane = lane_id(), w = wave_in_block();
    const uint32_t nchunks = (n + 3) / 4;
    for (uint64_t q = blockIdx.x; q < batch; q += gridDim.x) {
        uint32_t A[R][4], B[R][4], X[R][4];
        uint64_t vmask[R];
        u32x4 va[R], vb[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t row = w * R + r, c = row * 64 + lane;
            va[r] = load_raw<NTL>(a + q * n, n, c);
            vb[r] = load_raw<NTL>(b + q * n, n, c);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t c = (w * R + r) * 64 + lane;
            const bool valid = c < nchunks;
            place_words(va[r], n, c, valid, A[r]);
            place_words(vb[r], n, c, valid, B[r]);
            vmask[r] = ballot(valid);
#pragma unroll
            for (int t = 0; t < 4; ++t) X[r][t] = A[r][t];
        }
        uint32_t par = 0;
        auto add = [&](const uint32_t (&y)[R][4]) {
            uint32_t s[R][4];
            uint64_t G[R], P[R];
            uint32_t cin = 0, allp = 1;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t gen = add_words<4>(X[r], y[r], s[r]);
                G[r] = ballot(gen != 0) & vmask[r];
                P[r] = ballot(all_ones<4>(s[r])) & vmask[r];
                cin = wave_carry(G[r], P[r], cin).out;  // past the last chunk: dropped (mod 2^N)
                allp &= P[r] == vmask[r] ? 1u : 0u;
            }
            if (lane == 0) summary[par][w] = cin | (allp << 1);
            __syncthreads();
            cin = 0;
#pragma unroll
            for (int v = 0; v < NW; ++v) {
                const uint32_t sv = summary[par][v];
                if (v < int(w)) cin = (sv & 1u) | ((sv >> 1) & cin);
            }
            par ^= 1u;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const WaveCarry wc = wave_carry(G[r], P[r], cin);
                add_carry_words<4>(s[r], uint32_t(wc.into >> lane) & 1u);
                cin = wc.out;
#pragma unroll
                for (int t = 0; t < 4; ++t) X[r][t] = s[r][t];
            }
        };
        add(B);
        add(A);
        add(B);
        add(A);
        add(B);
        add(A);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t c = (w * R + r) * 64 + lane;
            store_chunk<NTS>(out + q * n, n, c, c < nchunks, X[r]);
        }
    }
}

namespace {

// ---- Packed small instances (n <= 64 Q words): several per wavefront ----
//
// An instance takes a segment of S = 2^seg_log lanes (S Q >= n); lane j of it
// owns output words Q j .. Q j + Q - 1.  The operands of a product sit in the
// wavefront's own LDS areas, each with at least n + 4 zero words below word 0
// and zeros from word n up to S Q + 4, so the sliding window of the
// multiplicand never needs a bounds check.  Carries between a lane and the
// next one of its segment come from one ballot-adder step (the lanes of an
// instance's last chunk, and lanes past it, neither generate nor propagate).

// Adds y into the lane's Q-word chunk x with carries across the segment.
template <int Q>
__device__ __forceinline__ void seg_add(uint32_t (&x)[Q], const uint32_t (&y)[Q], uint64_t keep, uint32_t lane) {
    uint32_t s[Q];
    const uint32_t g = add_words<Q>(x, y, s);
    const uint64_t G = ballot(g != 0) & keep, P = ballot(all_ones<Q>(s)) & keep;
    add_carry_words<Q>(s, uint32_t(wave_carry(G, P, 0).into >> lane) & 1u);
#pragma unroll
    for (int q = 0; q < Q; ++q) x[q] = s[q];
}

// Four words of V from `at`.
__device__ __forceinline__ void seg_window(const uint32_t *V, int32_t at, uint32_t (&x)[4]) {
    const uint2 v0 = *reinterpret_cast<const uint2 *>(V + at);
    const uint2 v1 = *reinterpret_cast<const uint2 *>(V + at + 2);
    x[0] = v0.x; x[1] = v0.y; x[2] = v1.x; x[3] = v1.y;
}

// Z = this lane's chunk of (U V) mod 2^(32 n), U and V the LDS areas of the
// lane's instance.  Each lane accumulates its Q coefficients over every step
// i < n (steps above a coefficient read the zeros below V), folds them into
// Q low words and a (high, carry) pair that belongs to the next lane's first
// two words, and the chunks are then added across the segment.
template <int Q>
__device__ __forceinline__ void seg_mul_low(const uint32_t *U, const uint32_t *V, uint32_t n, uint32_t j,
                                            uint64_t keep, uint32_t lane, uint32_t (&Z)[Q]) {
    const uint32_t kl = Q * j;
    uint64_t acc[Q];
    uint32_t cnt[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) { acc[q] = 0; cnt[q] = 0; }
    uint32_t w[4];  // V[kl .. kl + 3]
    seg_window(V, int32_t(kl), w);
    for (uint32_t i = 0; i < n; i += 4) {
        uint32_t x[4];  // V[kl - i - 4 .. kl - i - 1]
        seg_window(V, int32_t(kl) - int32_t(i) - 4, x);
        const uint4 a4 = *reinterpret_cast<const uint4 *>(U + i);
        const uint32_t av[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int t = q - u + 4;
                mac_v(acc[q], cnt[q], av[u], t >= 4 ? w[t - 4] : x[t]);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = x[q];
    }
    uint32_t R[Q + 2];
    uint64_t carry = 0;
#pragma unroll
    for (int p = 0; p < Q + 2; ++p) {
        uint64_t s = carry;
        if (p < Q) s += uint32_t(acc[p]);
        if (p >= 1 && p <= Q) s += uint32_t(acc[p - 1] >> 32);
        if (p >= 2) s += cnt[p - 2];
        R[p] = uint32_t(s);
        carry = s >> 32;
    }
    uint32_t h0 = __shfl_up(R[Q], 1), h1 = __shfl_up(R[Q + 1], 1);
    if (j == 0) { h0 = 0; h1 = 0; }
    uint32_t y[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) { Z[q] = R[q]; y[q] = q == 0 ? h0 : q == 1 ? h1 : 0u; }
    seg_add<Q>(Z, y, keep, lane);
}

// Words Q j .. Q j + Q - 1 of an n-word operand (zero past n or when invalid).
template <int Q>
__device__ __forceinline__ void load_q(const uint32_t *p, uint32_t n, uint32_t j, bool valid, uint32_t (&x)[Q]) {
#pragma unroll
    for (int q = 0; q < Q; ++q) x[q] = (valid && Q * j + q < n) ? p[Q * j + q] : 0u;
}

template <int Q>
__device__ __forceinline__ void store_q(uint32_t *p, uint32_t n, uint32_t j, bool valid, const uint32_t (&x)[Q]) {
    if (!valid) return;
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (Q * j + q < n) p[Q * j + q] = x[q];
}

// Words per LDS operand area: the zeros below (>= n + 4, a multiple of 4)
// and S Q + 4 words from word 0, rounded to a multiple of 4.
__host__ __device__ inline uint32_t packed_pad(uint32_t n) { return (n + 7) & ~3u; }
__host__ __device__ inline uint32_t packed_area(uint32_t n, uint32_t sq) { return packed_pad(n) + ((sq + 7) & ~3u); }

}  // namespace

constexpr int kPackedFull = 0;  // the full product, 2 n words
typedef u32x2 __attribute__((aligned(4))) u32x2_a4;  // 8 bytes at any word address

// Full product (PROG = kPackedFull), same-length product (BI_PROG_MUL_LOW) or
// Poly (BI_PROG_POLY) of instances whose result has at most 64 Q words,
// 64 / 2^seg_log per wavefront, one wavefront per workgroup.  LDS: per instance 2 (product) or 4 (Poly)
// operand areas.  Poly keeps a b in registers, forms a a + b and b b + b in
// registers and stores them as the operands of the last product.
// What bounds it: per group of products a chain of one load, one LDS round
// trip and n / 4 window steps, overlapped by eight waves per SIMD.  Full
// products of 4 / 16 words (2^22 words in all, 13 us of HBM traffic at copy
// rate): 15.6 / 21.2 us, one workgroup per product 430 / 140, the int8
// tiles 97 / 29.  Loading the next group ahead measured 5-25 % slower at odd
// sizes (the extra registers buy nothing that eight waves do not hide).
template <int PROG>
__global__ __launch_bounds__(64) void fused_packed_kernel(const uint32_t *__restrict__ a,
                                                          const uint32_t *__restrict__ b, uint32_t *__restrict__ out,
                                                          uint32_t n, uint64_t batch, uint32_t seg_log) {
    extern __shared__ __align__(16) uint32_t lds[];
    constexpr int Q = kPackedQ;
    constexpr uint32_t NA = PROG == BI_PROG_POLY ? 4 : 2;
    const uint32_t lane = lane_id(), S = 1u << seg_log, ipw = 64u >> seg_log;
    const uint32_t j = lane & (S - 1u), slot = lane >> seg_log;
    const uint32_t nr = PROG == kPackedFull ? 2 * n : n;  // words of a result
    const uint32_t nq = (nr + Q - 1) / Q;                 // chunks per instance
    const uint32_t aw = packed_area(n, S * Q);
    for (uint32_t t = lane; t < ipw * NA * aw; t += 64) lds[t] = 0;
    __syncthreads();
    uint32_t *area[NA];
#pragma unroll
    for (uint32_t k = 0; k < NA; ++k) area[k] = lds + (slot * NA + k) * aw + packed_pad(n);
    for (uint64_t g = blockIdx.x; g * ipw < batch; g += gridDim.x) {
        const uint64_t inst = g * ipw + slot;
        const bool valid = inst < batch && j < nq;
        const uint64_t keep = ballot(valid && j + 1 < nq);
        uint32_t A[Q], Bv[Q], Z[Q];
        load_q<Q>(a + inst * n, n, j, valid, A);
        load_q<Q>(b + inst * n, n, j, valid, Bv);
        store_q<Q>(area[0], n, j, valid, A);
        store_q<Q>(area[1], n, j, valid, Bv);
        __syncthreads();
        seg_mul_low<Q>(area[0], area[1], n, j, keep, lane, Z);  // a b
        if constexpr (PROG == BI_PROG_POLY) {
            uint32_t T[Q], U2[Q], R[Q];
            seg_mul_low<Q>(area[0], area[0], n, j, keep, lane, T);  // a a
            seg_add<Q>(T, Bv, keep, lane);                          // a a + b
            seg_mul_low<Q>(area[1], area[1], n, j, keep, lane, U2);  // b b
            seg_add<Q>(U2, Bv, keep, lane);                          // b b + b
            store_q<Q>(area[2], n, j, valid, T);
            store_q<Q>(area[3], n, j, valid, U2);
            __syncthreads();
            seg_mul_low<Q>(area[2], area[3], n, j, keep, lane, R);  // (a a + b)(b b + b)
            seg_add<Q>(R, Z, keep, lane);                           // + a b
#pragma unroll
            for (int q = 0; q < Q; ++q) Z[q] = R[q];
        }
        if constexpr (PROG == kPackedFull) {  // 2 n words: whole chunks of Q = 2
            if (valid) *reinterpret_cast<u32x2_a4 *>(out + inst * nr + Q * j) = u32x2{Z[0], Z[1]};
        } else {
            store_q<Q>(out + inst * nr, nr, j, valid, Z);
        }
        __syncthreads();  // the areas are rewritten by the next group
    }
}

namespace {

// log2 of the lanes an instance with results of nr words takes.
uint32_t packed_seg_log(uint32_t nr) {
    const uint32_t lanes = (nr + kPackedQ - 1) / kPackedQ;
    uint32_t seg_log = 0;
    while ((1u << seg_log) < lanes) ++seg_log;
    return seg_log;
}
size_t packed_lds_bytes(bool poly, uint32_t n, uint32_t seg_log) {
    return 4ull * (64u >> seg_log) * (poly ? 4 : 2) * packed_area(n, kPackedQ << seg_log);
}

// Persistent grid of resident workgroups (each loops over instances).  One
// instantiation per kernel, so each keeps its own occupancy record.
// Grids of up to 64 times the resident workgroups: equal persistent shares
// finish unevenly (2^27 words of 512 / 1024 / 8192 words 299 / 299 / 294 ->
// 246 / 256 / 282 us; at 8 times 264 / 266 / 295).
using FusedKernel = void (*)(const uint32_t *, const uint32_t *, uint32_t *, uint32_t, uint64_t);
template <FusedKernel kernel>
hipError_t launch_persistent(uint32_t threads, const uint32_t *a, const uint32_t *b, uint32_t *c, uint32_t n,
                             uint64_t batch, hipStream_t st, int num_cus) {
    static std::atomic<int> occ{0};  // resident workgroups per CU (0: not asked yet)
    int o = occ.load(std::memory_order_relaxed);
    if (o == 0) {
        const hipError_t e =
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, reinterpret_cast<const void *>(kernel), int(threads), 0);
        if (e != hipSuccess) return e;
        if (o < 1) o = 1;
        occ.store(o, std::memory_order_relaxed);
    }
    const uint64_t cap = uint64_t(o) * uint64_t(num_cus > 0 ? num_cus : 1) * 64;
    const uint32_t grid = uint32_t(batch < cap ? batch : cap);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, a, b, c, n, batch);
    return hipGetLastError();
}

template <int PROG>
hipError_t launch_packed(const uint32_t *a, const uint32_t *b, uint32_t *c, uint32_t n, uint64_t batch, hipStream_t st,
                         int num_cus) {
    const uint32_t seg_log = packed_seg_log(PROG == kPackedFull ? 2 * n : n);
    const size_t lds = packed_lds_bytes(PROG == BI_PROG_POLY, n, seg_log);
    const uint64_t waves = (batch + (64u >> seg_log) - 1) / (64u >> seg_log);
    const uint32_t grid = uint32_t(std::min<uint64_t>(waves, uint64_t(num_cus > 0 ? num_cus : 1) * 32));
    hipLaunchKernelGGL((fused_packed_kernel<PROG>), dim3(grid), dim3(64), lds, st, a, b, c, n, batch, seg_log);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_packed_full(const uint32_t *a, const uint32_t *b, uint32_t *c, uint32_t n, uint64_t batch,
                              hipStream_t st, int num_cus) {
    if (n == 0 || n > kPackedMaxWords) return hipErrorInvalidValue;
    if (batch == 0) return hipSuccess;
    return launch_packed<kPackedFull>(a, b, c, n, batch, st, num_cus);
}

hipError_t launch_fused(int program, const uint32_t *a, const uint32_t *b, uint32_t *c, uint32_t n, uint64_t batch,
                        hipStream_t st, int num_cus) {
    if (batch == 0) return hipSuccess;
    if (program == BI_PROG_ADD6) {
        // Bound by HBM.  Results go past the caches as for products (2^25 words
        // of 128: 72 -> 57 us), unless short odd instances would write partial
        // lines (2^27 words of 31: 424 -> 495).  Operands beyond twice the
        // 256 MiB memory-side cache are read past it too (2^27 words of 128:
        // 329 -> 285; below that 2^25 words 57 -> 64), in aligned rows (257
        // words 366 -> 394), and from 768 MiB four rows per wavefront are in
        // flight (2^27 words 269 -> 244, 2^26 words 132 -> 137).  Operands
        // beyond the cache also run on finer grids (2^27 words of 255: 340 ->
        // 280; 2^24 words of one 53 -> 63).
        const uint64_t words = uint64_t(n) * batch;
        const bool nts = streamed_results(4 * words) && (n % 4 == 0 || n >= 48);
        const bool ntl = nts && n % 4 == 0 && 8 * words > (uint64_t(512) << 20);
        const uint32_t nchunks = (n + 3) / 4, rows = (nchunks + 63) / 64;
        if (rows == 1) {
            uint32_t seg_log = 0;
            while ((1u << seg_log) < nchunks) ++seg_log;
            const uint32_t per_wave = ntl && 8 * words > (uint64_t(768) << 20) ? 4 : 1;
            const uint64_t ipw = per_wave * (64u >> seg_log), waves = (batch + ipw - 1) / ipw;
            const uint64_t cap = uint64_t(num_cus > 0 ? num_cus : 1) * (8 * words > (uint64_t(256) << 20) ? 256 : 32);
            const uint32_t grid = uint32_t(std::min((waves + 3) / 4, cap));
            const auto kernel = per_wave == 4 ? fused_add6_packed_kernel<4, true, true>
                                : ntl ? fused_add6_packed_kernel<1, true, true>
                                : nts ? fused_add6_packed_kernel<1, false, true>
                                      : fused_add6_packed_kernel<1, false, false>;
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, st, a, b, c, n, batch, seg_log);
            return hipGetLastError();
        }
        // up to 4 rows per lane group: fewer waves per instance, more
        // instances resident per CU to hide the per-addition barrier
        uint32_t nw = 1;
        while (4 * nw < rows) nw *= 2;
        const uint32_t r = (rows + nw - 1) / nw;
#define BI_ADD6_CASE(W, RR) \
    if (nw == W && r == RR)                                                                                     \
        return ntl   ? launch_persistent<&fused_add6_rows_kernel<W, RR, true, true>>(64 * W, a, b, c, n, batch, st, num_cus)  \
               : nts ? launch_persistent<&fused_add6_rows_kernel<W, RR, false, true>>(64 * W, a, b, c, n, batch, st, num_cus) \
                     : launch_persistent<&fused_add6_rows_kernel<W, RR, false, false>>(64 * W, a, b, c, n, batch, st, num_cus);
        BI_ADD6_CASE(1, 2) BI_ADD6_CASE(1, 3) BI_ADD6_CASE(1, 4) BI_ADD6_CASE(2, 3) BI_ADD6_CASE(2, 4)
        BI_ADD6_CASE(4, 3) BI_ADD6_CASE(4, 4) BI_ADD6_CASE(8, 3) BI_ADD6_CASE(8, 4)
#undef BI_ADD6_CASE
        return hipErrorInvalidValue;
    }
    const bool poly = program == BI_PROG_POLY;
    // Small instances: the VALU schoolbook packed several to a wavefront is
    // faster up to 32 words (2^22 words of 16 / 32 / 33 words, low product:
    // 13.3 / 18.0 / 32.0 us against 47.5 / 27.0 / 26.0 on the matrix cores,
    // whose tiles hold 64 words; Poly 51 / 55 / 107 against 161 / 85 / 84).
    // So does Poly of up to 36 words in batches that leave most of the chip idle
    // (2 / 500 instances of 36 words 5.9 / 6.4 us, 6.4 / 7.1 on the matrix cores;
    // 2000 equal).
    const bool packed = n <= kPackedMaxWords || (poly && n <= 36 && batch <= 1000);
    if (!packed) return launch_conv_fused(poly, a, b, c, n, batch, st, num_cus);
    return poly ? launch_packed<BI_PROG_POLY>(a, b, c, n, batch, st, num_cus)
                : launch_packed<BI_PROG_MUL_LOW>(a, b, c, n, batch, st, num_cus);
}

}  // namespace bi
