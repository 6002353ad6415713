// LDS layout of the one-workgroup-per-product convolution kernels
// (conv_wg.hip).  No device code, so that a host compiler can check it.
#pragma once

#include <stdint.h>

#ifndef __HIP__
#define __host__
#define __device__
#endif

namespace bi {
namespace conv {

constexpr uint32_t kAPad = 64;   // zero bytes before digit 0 of a
constexpr uint32_t kATail = 7;   // 16-byte pieces after a's digits (steps read up to 83 bytes past them)
constexpr uint32_t kBPad = 32;   // zero groups below group 0 of b: B operand -2 at kappa 0, -1 above
constexpr uint32_t kBTail = 35;  // groups from the top digit's on: B operand J + 1

// Words that the waves exchange: (carry out, propagates) of each wave's digits
// of a and of b, each unit's last high word, (carry out, propagates) of each
// unit's result.
constexpr uint32_t kRecodeWords = 0, kRecodeB = 32, kBoundaryWords = 64, kCarryWords = 128, kSumWords = 256;

// Byte offsets of the dynamic LDS block of products of nch chunks in a kernel
// for up to cap chunks.  The exchanged words follow the largest product's
// digits, at the same place for every size: a workgroup that takes products of
// different sizes in turn has no barrier between the last reads of one's
// carries and the first writes of the next one's.
struct WgLayout {
    uint32_t b, sum, total;
};
__host__ __device__ constexpr uint32_t wg_a_bytes(uint32_t nch) { return kAPad + 16 * (nch + kATail); }
__host__ __device__ constexpr uint32_t wg_b_bytes(uint32_t nch) { return 16 * (kBPad + nch + kBTail); }
__host__ __device__ constexpr WgLayout wg_layout(uint32_t nch, uint32_t cap) {
    const uint32_t sum = wg_a_bytes(cap) + wg_b_bytes(cap);
    return WgLayout{wg_a_bytes(nch), sum, sum + 4 * kSumWords};  // a: zeros, digits, the top digit, zeros; then b alike
}

}  // namespace conv
}  // namespace bi
