// The carry-less forms of the hash: the Toeplitz product computed over
// GF(2) itself, on packed bits, instead of through integer residues.
//
//   direct  the m x n product as a binary matrix product on the matrix
//           cores (one launch, or two when the key is cut into slices);
//   split   the cyclic product of T = 3^k chunks of M = (T/3) g 32-bit
//           words each: the chunks are coefficients in the ring
//           GF(2)[X] / (X^(64 M) + X^(32 M) + 1), in which X^32 has order
//           3 M, so that a length-T transform multiplies by word rotations
//           only.  Each of the T products in that ring is again split, by
//           2 * 3^a points in the ring of 2 M2 words (M2 = M / 3^a), and
//           those are multiplied on the matrix cores.
//
// Both are exact: every value is a bit, or the count of fewer than 2^23 ones
// in an fp32 accumulator.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pa_internal.h"

namespace pa {

enum GfForm { kGfNone = 0, kGfDirect = 1, kGfSplit = 2 };

// How a launch sequence computes its products (kGfNone: number-theoretic
// transform).  Results do not depend on the choice.
struct GfChoice {
    int form = kGfNone;
    // direct: tiles of 256 outputs per workgroup, slices of the key
    int nt = 0, slices = 0;
    // split: T = 3^k chunks, word unit g, log3 of the half point count a,
    // leaf half length M2 (words)
    int T = 0, g = 0, a = 0, M2 = 0;
    // largest output length (bits) of the launch's jobs: the grid's extent
    uint32_t max_m = 0;
    int chunk_words() const { return T / 3 * g; }                             // M
    uint64_t cyclic_bits() const { return 32ull * T * (uint64_t)chunk_words(); }
    uint64_t spectrum_words() const { return 2ull * T * chunk_words(); }      // X and the seed's spectrum
    uint64_t work_words() const { return 6ull * T * chunk_words(); }          // X, then the products (4 T M)
};

// Bits by which the split form's product can be shifted: a key that starts
// inside its buffer (modified Toeplitz) is taken from a whole 64-bit word on.
constexpr uint64_t kGfLead = 63;

// Split of a cyclic product of at least `bits` bits whose work area fits in
// `words` 32-bit words; form kGfNone if there is none.
GfChoice gf_split_for(uint64_t bits, uint64_t words);

// What a split product stands in for: blocks with a seed each (one launch
// sequence), or keys against a spectrum that is there already, of a plan, of a
// server's seed or of a batch's shared seed.
enum GfUse { kGfBlocks, kGfPlan, kGfServed, kGfShared };

// The most outputs of a block for which the split product is faster than the
// transform of length L (0: never; UINT64_MAX: always).
uint64_t gf_split_limit(const GfChoice &split, uint64_t L, GfUse use, int njobs);

// Form for njobs blocks of one launch sequence, none longer than n bits, m
// outputs or a cyclic product of `bits` bits, where L is the transform length
// otherwise; form kGfNone if the transform is faster.  captured: the launches
// of a graph, among which one more costs little.
GfChoice gf_plain_for(uint64_t L, uint64_t n, uint64_t m, uint64_t bits, uint64_t words, int njobs,
                      GfUse use = kGfBlocks, bool captured = false);

// Words of a direct launch's partial results per block (0: one slice).
inline uint64_t gf_direct_words(const GfChoice &c) {
    return c.slices > 1 ? (uint64_t)c.slices * ((c.max_m + 255u) / 256u * 8u) : 0u;
}

// Launchers.  jobs: as the number-theoretic passes (JobArgs); s: stream;
// e0, e1: timing events or null.
hipError_t launch_gf_direct(const GfChoice &c, const JobArgs &ja, int njobs, hipStream_t s, hipEvent_t e0,
                            hipEvent_t e1);
hipError_t launch_gf_parts(const GfChoice &c, const JobArgs &ja, int njobs, hipStream_t s, hipEvent_t e0,
                           hipEvent_t e1);
hipError_t launch_gf_fwd(const GfChoice &c, int nsrc, const JobArgs &ja, int njobs, hipStream_t s, hipEvent_t e0,
                         hipEvent_t e1);
// resident: the second factor is job.Shat (a spectrum), else job.S.
hipError_t launch_gf_mul(const GfChoice &c, bool resident, const JobArgs &ja, int njobs, hipStream_t s, hipEvent_t e0,
                         hipEvent_t e1);
hipError_t launch_gf_inv(const GfChoice &c, const JobArgs &ja, int njobs, hipStream_t s, hipEvent_t e0, hipEvent_t e1);

}  // namespace pa
