// gfx950 kernels of the carry-less forms (see pa_gf2.h).  Included by
// pa_kernels.hip, whose buffer and job helpers they use.
#pragma once

#include "pa_gf2.h"

namespace pa {

typedef int gf_v4i __attribute__((ext_vector_type(4)));
typedef int gf_v8i __attribute__((ext_vector_type(8)));
typedef float gf_v4f __attribute__((ext_vector_type(4)));

// 32 bits from bit `sh` (0..31) of the 64-bit value (hi, lo).
__device__ __forceinline__ uint32_t funnel(uint32_t hi, uint32_t lo, uint32_t sh) {
    return __builtin_amdgcn_alignbit(hi, lo, sh);
}

// Load at a byte offset that may be negative (out of range: 0).  The offset
// is made opaque: the compiler would otherwise form it as a register, which
// can be negative for a neighbouring load of the same code, plus a positive
// instruction offset, and a negative register is out of range whatever is
// added to it.
__device__ __forceinline__ uint32_t ld32_any(rsrc_t r, int o) {
    asm("" : "+v"(o));
    return (uint32_t)ld32(r, o);
}

// What lanes of a wave have written to LDS, handed to its other lanes.  The
// hardware keeps a wave's LDS operations in order; the fences keep the
// compiler from moving loads over stores whose address, or type (halfwords,
// words and word pairs of one area), differs from theirs.  No instruction.
__device__ __forceinline__ void wave_handoff() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// One 16 x 16 x 128 binary product on the matrix cores: the operands hold
// one bit per fp4 element, ones as 0.5 in one operand where they are 1.0 in
// the other, so a common one adds 0.5.  Accumulators start at 2^22, whose
// last place is 0.5: with fewer than 2^23 common ones (kGfOnes) sums are exact
// and the lowest mantissa bit is the parity.  Lane l holds 32 consecutive k of row (column)
// l & 15 from k = 32 (l >> 4), as one 32-bit window; the order of k inside
// the four registers is free as long as both operands share it.
constexpr float kGfBias = 4194304.0f;  // 2^22
constexpr uint64_t kGfOnes = 1u << 23;
__device__ __forceinline__ gf_v4f bit_mfma(gf_v4i a, gf_v4i b, gf_v4f c) {
    const gf_v8i A = {a[0], a[1], a[2], a[3], 0, 0, 0, 0}, B = {b[0], b[1], b[2], b[3], 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A, B, c, 4, 4, 0, 0, 0, 0);
}
// One operand expanded in LDS in units of 16 bits (8 bytes each, so that a
// window at any multiple of 16 bits is 16 consecutive bytes): a unit holds
// its bits 0, 4, 8, 12 and 1, 5, 9, 13 in the nibbles of the low and high
// half of its first word, 2, 6, .. and 3, 7, .. in its second.  The even
// bits are 1.0 and the odd ones 0.5 here, and the reverse in the window.
__device__ __forceinline__ gf_v4i expand_units(uint32_t w) {
    const uint32_t l = ((w << 1) & 0xFFFFu) | ((w << 15) & 0xFFFF0000u);
    const uint32_t h = ((w >> 15) & 0xFFFEu) | ((w >> 1) & 0xFFFF0000u);
    gf_v4i r = {(int)(l & 0x11112222u), (int)((l >> 2) & 0x11112222u), (int)(h & 0x11112222u),
                (int)((h >> 2) & 0x11112222u)};
    return r;
}
__device__ __forceinline__ gf_v4i expand_window(uint32_t w) {
    const uint32_t l = __builtin_amdgcn_perm(w, w, 0x01000100u), h = __builtin_amdgcn_perm(w, w, 0x03020302u);
    gf_v4i r = {(int)(l & 0x22221111u), (int)((l >> 2) & 0x22221111u), (int)(h & 0x22221111u),
                (int)((h >> 2) & 0x22221111u)};
    return r;
}

// The units of a word whose window is read in the other direction: each
// 16-bit half bit-reversed, in place; the window's halves change places.
__device__ __forceinline__ gf_v4i expand_units_reversed(uint32_t w) {
    const gf_v4i r = expand_units(__builtin_bitreverse32(w));
    return gf_v4i{r[2], r[3], r[0], r[1]};
}
__device__ __forceinline__ gf_v4i expand_window_swapped(uint32_t w) {
    const gf_v4i r = expand_window(w);
    return gf_v4i{r[2], r[3], r[0], r[1]};
}

// The parities of NT <= 8 tiles whose accumulator v in lane l is output bit
// 16 (l & 15) + 4 (l >> 4) + v: lane l < 32 gets tiles 4 (l >> 4) .. + 3 as
// 16-bit fields of row l & 15 (tiles 0, 1 in a, 2, 3 in b of lanes 0 .. 15).
template <int NT>
__device__ __forceinline__ uint2 tile_halfwords(const gf_v4f (&acc)[NT]) {
    static_assert(NT <= 8, "eight nibbles a lane");
    uint32_t x = 0;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) x = funnel(__float_as_uint(acc[t][v]), x, 1);
    x >>= 32 - 4 * NT;  // nibble t: bits 4 (l >> 4) .. + 3 of row l & 15, tile t
    const uint32_t s = (threadIdx.x & 16u);  // odd rows of 16 lanes take tiles 4 ..
    const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    auto bytes = [&](uint32_t v) PA_INLINE {  // four nibbles to four bytes
        v = (v >> s) & 0xFFFFu;
        v = (v | (v << 8)) & 0x00FF00FFu;
        return (v | (v << 4)) & 0x0F0F0F0Fu;
    };
    const uint32_t y = bytes(p[0]) | (bytes(p[1]) << 4);
    const auto q = __builtin_amdgcn_permlane32_swap(y, y, false, false);
    return make_uint2(__builtin_amdgcn_perm(q[1], q[0], 0x05010400u), __builtin_amdgcn_perm(q[1], q[0], 0x07030602u));
}

// Word w of the job's output: bits past m cleared, the head of the key
// XORed in (modified Toeplitz), words past the last 64-bit word dropped.
struct OutWords {
    rsrc_t out, head;
    uint32_t m;
    __device__ __forceinline__ OutWords(const JobDesc &job)
        : out(make_rsrc(job.out, (uint32_t)((job.m + 63) / 64 * 8))),
          head(make_rsrc(job.xor_src, job.xor_src ? (uint32_t)((job.m + 31) / 32 * 4) : 0u)),
          m(job.m) {}
    __device__ __forceinline__ void put(uint32_t w, uint32_t v) const {
        v ^= (uint32_t)ld32(head, (int)(w * 4));
        const int keep = (int)m - (int)(w * 32);
        if (keep < 32) v = keep > 0 ? v & ((1u << keep) - 1u) : 0u;
        st32(out, (int)(w * 4), (int)v);
    }
};

// ------------------------------------------------------------------- direct
//
// y[i] = sum_j s[i - j + n - 1] x[j].  With xr the reversed key and
// i = 256 t + 16 r + q this is sum_k s[256 t + 16 r + k] xr[k - q]: a matrix
// product whose row operand starts at a multiple of 16 bits of the seed and
// whose column operand is the key shifted by its column.  A workgroup
// computes NT tiles of 256 outputs; its waves (and the launch's slices)
// share k.
//
// A wave goes through k in chunks of ST steps of 128: the chunk's seed words
// are expanded once into LDS, so that a row fragment is 16 bytes read at
// 8-byte alignment, and its key words are copied there; the next chunk's
// words are loaded meanwhile.  The row operand depends on k + 256 t only:
// a step needs one new row fragment for all NT tiles (the others are those
// of earlier steps, kept in 2 NT rotating registers) and one column window,
// expanded in nine operations.  So with NT = 4 the matrix cores (64 clocks a
// step) bound it, with NT = 2 vector issue does.  The reversal is the
// seed's: its words are expanded bit-reversed, and the two halves of a
// window change places.  (Windows of both operands fetched from the caches
// and expanded in registers, 27 vector operations a step: 32 blocks of 10^5
// bits to 20,000 in 57 us, now 34.)
template <int NT, int ST, int NW, bool PARTS>
__global__ void __launch_bounds__(64 * NW) k_gf_direct(JobArgs ja) {
    constexpr int U = 2 * NT, SW = 4 * ST + 8 * NT, KW = 4 * ST + 2;  // a chunk's seed and key words
    static_assert(kMaxLen / NW + 2 * 128 * ST < kGfOnes, "a wave's whole chunks of the longest key");
    const JobDesc job = job_of(ja, uni(blockIdx.z));
    const int n = (int)job.n, R0 = (int)blockIdx.x * NT;
    if ((uint32_t)R0 * 256u >= job.m) return;
    const int lane = threadIdx.x & 63, wave = (int)uni(threadIdx.x >> 6);
    const int q = lane & 15, kb = lane >> 4;
    constexpr int nw = NW;
    const int chunks = (n + 15 + 128 * ST - 1) / (128 * ST);
    const int share = (int)gridDim.y * nw, per = (chunks + share - 1) / share;
    const int c0 = min(chunks, ((int)blockIdx.y * nw + wave) * per), c1 = min(chunks, c0 + per);

    const rsrc_t sb = make_rsrc(job.seed, (uint32_t)((job.seed_bits + 31) / 32 * 4));
    const int ko = (int)(job.key_off & 31u), last = (ko + n - 1) >> 5;
    const rsrc_t xb = make_rsrc((const uint32_t *)job.key + (job.key_off >> 5), (uint32_t)(last + 1) * 4);
    const uint32_t first_mask = ~0u << ko, last_mask = ~0u >> (31 - ((ko + n - 1) & 31));

    __shared__ __attribute__((aligned(16))) uint32_t rows_lds[nw][SW * 4];
    __shared__ uint32_t keys_lds[nw][KW];
    uint32_t *rows = rows_lds[wave], *keys = keys_lds[wave];
    // the key window of step k starts at bit x0 + q - 128 k - 32 kb of the
    // key's words; chunk c needs the words from top + 3 - 4 ST (c + 1)
    const int x0 = n + ko - 32, top = x0 >> 5;
    const uint32_t ksh = (uint32_t)(x0 + q) & 31u;
    const uint32_t *kwin = keys + (3 - kb + (((x0 + q) >> 5) - top));
    const uint32_t *rwin = rows + (q + 2 * kb) * 2;

    auto key_word = [&](int w) PA_INLINE {
        uint32_t v = ld32_any(xb, w * 4);
        if (w == 0) v &= first_mask;
        if (w == last) v &= last_mask;
        return v;
    };
    uint32_t s0 = 0, s1 = 0, k0 = 0, k1 = 0;
    auto fetch = [&](int c) PA_INLINE {
        const int sw = R0 * 8 + c * (4 * ST), kw = top + 1 - 4 * ST * (c + 1);
        if (lane < SW) s0 = (uint32_t)ld32(sb, (sw + lane) * 4);
        if (lane < SW - 64) s1 = (uint32_t)ld32(sb, (sw + 64 + lane) * 4);
        if (lane < KW) k0 = key_word(kw + lane);
        if (lane < KW - 64) k1 = key_word(kw + 64 + lane);
    };
    typedef gf_v4i __attribute__((aligned(8))) gf_v4i_a8;
    auto fragment = [&](int f) PA_INLINE { return *(const gf_v4i_a8 *)(rwin + f * 16); };

    gf_v4f acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = gf_v4f{kGfBias, kGfBias, kGfBias, kGfBias};
    if (c0 < c1) fetch(c0);
    for (int c = c0; c < c1; ++c) {
        // the chunk before is read (at the end of the loop the same fence makes
        // a schedule 3% slower: 262,144 bits to 65,536 in 12.4 us, here 12.0)
        wave_handoff();
        if (lane < SW) ((gf_v4i *)rows)[lane] = expand_units_reversed(s0);
        if (lane < SW - 64) ((gf_v4i *)rows)[64 + lane] = expand_units_reversed(s1);
        if (lane < KW) keys[lane] = k0;
        if (lane < KW - 64) keys[64 + lane] = k1;
        wave_handoff();
        if (c + 1 < c1) fetch(c + 1);
        gf_v4i row[ST + U - 2];
#pragma unroll
        for (int f = 0; f < U - 2; ++f) row[f] = fragment(f);
#pragma unroll
        for (int k = 0; k < ST; ++k) {
            row[k + U - 2] = fragment(k + U - 2);
            const gf_v4i b = expand_window_swapped(funnel(kwin[4 * (ST - 1 - k) + 1], kwin[4 * (ST - 1 - k)], ksh));
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] = bit_mfma(b, row[k + 2 * t], acc[t]);
        }
    }
    // XOR of the waves' parities, 8 NT words per workgroup
    __shared__ uint32_t red[nw][8 * NT];
    {
        const uint2 hw = tile_halfwords<NT>(acc);
        uint16_t *o = (uint16_t *)red[wave];
        const int at = 64 * (lane >> 4) + q;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (lane < 32 && 4 * (lane >> 4) + i < NT)
                o[at + 16 * i] = (uint16_t)((i & 2 ? hw.y : hw.x) >> (16 * (i & 1)));
    }
    __syncthreads();
    if (threadIdx.x < 8 * NT) {
        uint32_t v = 0;
#pragma unroll
        for (int w = 0; w < nw; ++w) v ^= red[w][threadIdx.x];
        const uint32_t wd = (uint32_t)R0 * 8u + threadIdx.x;
        if constexpr (PARTS) {
            const uint32_t stride = (job.m + 255u) / 256u * 8u;
            if (wd < stride) ((uint32_t *)job.A)[(size_t)blockIdx.y * stride + wd] = v;
        } else {
            OutWords(job).put(wd, v);
        }
    }
}

// XOR of the slices' partial words into the output.
__global__ void __launch_bounds__(256) k_gf_parts(JobArgs ja, int slices) {
    const JobDesc job = job_of(ja, uni(blockIdx.y));
    const uint32_t w = blockIdx.x * 256u + threadIdx.x, stride = (job.m + 255u) / 256u * 8u;
    if (w >= stride) return;
    uint32_t v = 0;
    for (int i = 0; i < slices; ++i) v ^= ((const uint32_t *)job.A)[(size_t)i * stride + w];
    OutWords(job).put(w, v);
}

// -------------------------------------------------------------------- split
//
// Ring elements.  In GF(2)[v] / (v^(2M) + v^M + 1), v = X^32, v has order
// 3 M.  An element (lo, hi) of 2 M words is also the periodic sequence
// beta = (lo, lo + hi, hi) of 3 M words, and multiplying by v^s rotates
// beta by s: sums of rotated elements need no reduction.  Two of the three
// thirds determine the element; a table of five thirds (one period and two
// more) gives lo and hi of a rotation at a linear index.

__device__ __forceinline__ unsigned long long ld64(rsrc_t r, int voff, int soff) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    return (unsigned long long)v[1] << 32 | v[0];
}

// a - b (mod n) for 0 <= a, b < n as one subtraction, one addition and an
// unsigned minimum.
__device__ __forceinline__ uint32_t sub_mod(uint32_t a, uint32_t b, uint32_t n) {
    const uint32_t d = a - b;
    return min(d, d + n);
}
__device__ __forceinline__ uint32_t add_mod(uint32_t a, uint32_t b, uint32_t n) {
    const uint32_t d = a + b;
    return min(d, d - n);
}

// P1: forward transform of the chunks a_t (M words each, t < T = P Q) at
// the T-th root v^G:  X_tau = sum_t v^(G tau t) a_t.  With tau = rho + Q
// sigma and t = t0 + P t1 the inner sums over t1 are formed by scattering
// every chunk, rotated, into tile t0, and a length-P transform over t0
// follows.  Word positions split into classes modulo Cm = G P that no
// rotation of the second step leaves; a workgroup takes one rho and F
// classes (F divides Cm), so its tile is P x Q x F words.
//
// The rotations cost no vector operation: a chunk's target row is its first row plus rho t1 (mod
// Q), the chunks are taken in the order that makes rho t1 = D k for k = 0,
// 1, .. (D = gcd(rho, Q); D chunks share each target and are added first),
// a scalar row offset, and tiles have 2 Q rows, so that rows never wrap and
// D k is an immediate offset.  The same in the second step: every wave has
// one sigma, so a tile's rotation is a scalar.  Everything but rho is a
// constant.  Then the loads bound it (address units busy 77% of the
// time), so with whole classes (F = Cm, the words of a chunk in order) a
// workgroup can take R = 2 values of rho that read the same words: rho and
// Q - rho, whose targets are the same rows in the other direction.  With G
// even, words go in pairs.  256 blocks of 10^6 bits: 341 us with per-word
// rotations, 277 with scalar ones, 207 with two rho a workgroup.
// Grid: (Q Cm / F, or (Q / 2 + 1) Cm / F with two rho, sources, jobs), 9
// waves.  Wave w owns tiles t0 = w, w + 9, ...: nothing else writes them
// before the barrier.
constexpr int kGfWaves = 9;

// Bits before the source in its first 64-bit word.
__device__ __forceinline__ uint32_t gf_lead_bits(const JobDesc &job, bool src) { return src ? 0u : job.key_off & 63u; }

template <int Q, int P, int G, int F, int R>
__global__ void __launch_bounds__(64 * kGfWaves) k_gf_fwd(JobArgs ja) {
    constexpr int T = P * Q, Q3 = Q / 3, M = T / 3 * G, Cm = G * P, NF = Cm / F;
    static_assert(P % kGfWaves == 0 && (Q == 9 || Q == 27) && Cm % F == 0, "tiles are dealt to 9 waves");
    static_assert(R == 1 || F == Cm, "a pair of rho reads the same words");
    constexpr int third = Q3 * F, period = Q * F, trow = 2 * period;  // words of a tile: two periods
    // words a lane handles together: every rotation is a multiple of G, so
    // with G even pairs stay pairs (half the loads, LDS operations and
    // addresses)
    constexpr int V = G % 2 == 0 && F % 2 == 0 ? 2 : 1;
    typedef typename std::conditional<V == 2, unsigned long long, uint32_t>::type Wv;
    const bool src = blockIdx.y != 0;
    const JobDesc job = job_of(ja, uni(blockIdx.z));
    const int rho0 = (int)blockIdx.x / NF, f0 = ((int)blockIdx.x - rho0 * NF) * F;
    const int nr = R == 2 && rho0 ? 2 : 1;  // values of rho: rho0 and Q - rho0
    uint32_t *tile = (uint32_t *)pa_lds;    // [R][P][2 Q][F]
    const int lane = threadIdx.x & 63, wave = (int)uni(threadIdx.x >> 6);

    // A source that starts at bit `off` of its buffer is taken from the
    // 64-bit word of that bit on, with the `rem` bits before it as zeros: the
    // product is then shifted by rem, which the inverse pass allows for.  The
    // words before and after the source are whole 64-bit words of its buffer.
    const uint32_t off = src ? 0u : job.key_off;
    const int rem = (int)gf_lead_bits(job, src), nbits = (int)(src ? job.seed_bits : job.n) + rem;
    const rsrc_t in = make_rsrc((src ? job.seed : job.key) + (off >> 6), ((uint32_t)nbits + 63) / 64 * 8);
    const int last = (nbits - 1) >> 5;

    // the Q chunks of a tile in the order of their targets: slot k D + b is
    // chunk t1 = (k inv mod K) + K b, K = Q / D, inv = (rho / D)^-1 mod K (the
    // 17th power: the orders of the units mod 27, 9 and 3 divide 18).  Each
    // lane finds one slot's offset; loads take them as scalars.
    const int D = rho0 % 3 ? 1 : rho0 % 9 ? 3 : Q == 9 || rho0 % 27 ? 9 : Q;
    int slot;
    {
        const uint32_t K = (uint32_t)(Q / D), r = (uint32_t)(rho0 / D) % K, k = (uint32_t)(lane / D);
        uint32_t inv = r * r % K;
        inv = inv * inv % K;
        inv = inv * inv % K;
        inv = inv * inv % K * r % K;
        slot = (int)(k * inv % K + K * (uint32_t)(lane - (int)k * D)) * (P * M * 4);
    }

    for (int t0 = wave; t0 < P; t0 += kGfWaves) {
        uint32_t *tl = tile + t0 * trow;
        for (int r = 0; r < nr; ++r)
            for (int i = lane; i < trow / V; i += 64) ((Wv *)(tl + r * P * trow))[i] = 0;
        wave_handoff();
        const int s0 = G * ((rho0 * t0) % T), sc = s0 % Cm, si = s0 / Cm;
        const int s1 = G * (((Q - rho0) * t0) % T);  // (a pair's second)
        int off_k[Q];
#pragma unroll
        for (int k = 0; k < Q; ++k) off_k[k] = __builtin_amdgcn_readlane(slot, k);
        for (int l = lane * V; l < third; l += 64 * V) {
            // source word e of the chunks and its target for t1 = 0 (of two
            // periods, in the first)
            int e, to;
            if constexpr (F == Cm) {
                e = l;
                to = si * F + sc + l;
            } else {
                const int i1 = l / F, f = l - i1 * F;
                int c = f0 + f - sc;
                const int wrap = c < 0 ? 1 : 0;
                c += wrap ? Cm : 0;
                e = c + Cm * i1;
                to = (i1 + wrap + si) * F + f;
            }
            to -= to >= period ? period : 0;
            uint32_t *dst = tl + to, *dst1 = nullptr;
            if constexpr (R == 2) {
                to = s1 + l;
                to -= to >= period ? period : 0;
                dst1 = tl + P * trow + to;
            }
            const int at = (t0 * M + e) * 4;
            // NB loads in flight a lane (pairs: 9, for the registers)
            constexpr int NB = V == 2 ? 9 : Q;
#pragma unroll
            for (int g = 0; g < Q; g += NB) {
                Wv w[NB];
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    if constexpr (V == 2) w[k] = ld64(in, at, off_k[g + k]);
                    else w[k] = (Wv)__builtin_amdgcn_raw_buffer_load_b32(in, at, off_k[g + k], 0);
                }
                auto scatter = [&](auto d) PA_INLINE {
                    constexpr int DD = decltype(d)::value, C = DD < NB ? DD : NB;
#pragma unroll
                    for (int k = 0; k < NB / C; ++k) {
                        Wv x = w[k * C];
#pragma unroll
                        for (int b = 1; b < C; ++b) x ^= w[k * C + b];
                        atomicXor((Wv *)(dst + (g / DD + k) * (DD * F)), x);
                        // the other rho's targets go the other way round
                        if (R == 2 && DD < Q)
                            atomicXor((Wv *)(dst1 + (Q / DD - g / DD - k) % (Q / DD) * (DD * F)), x);
                    }
                };
                if (D == 1) scatter(std::integral_constant<int, 1>{});
                else if (D == 3) scatter(std::integral_constant<int, 3>{});
                else if (D == 9) scatter(std::integral_constant<int, 9>{});
                else scatter(std::integral_constant<int, Q>{});
            }
            // take back what lies past the source's last bit (the rest of its
            // last word and the word after) and before its first
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int W = d < 2 ? last + d : d - 2, t = W / M, ew = W - t * M - e;
                if (d >= 2 && 32 * (d - 2) >= rem) break;
                if (t % P == t0 && ew >= 0 && ew < V && t < T) {
                    const uint32_t tail = d ? ~0u : ~(~0u >> (31 - ((nbits - 1) & 31)));
                    const uint32_t head = rem >= 32 * (d - 1) ? ~0u : (1u << (rem & 31)) - 1u;
                    const uint32_t x = (uint32_t)ld32(in, W * 4) & (d < 2 ? tail : head);
                    atomicXor(dst + ew + rho0 * (t / P) % Q * F, x);
                    if (R == 2 && nr == 2) atomicXor(dst1 + ew + (Q - rho0) * (t / P) % Q * F, x);
                }
            }
        }
        wave_handoff();
        // to periodic form, two periods
        for (int r = 0; r < nr; ++r)
        for (int l = lane; l < third / V; l += 64) {
            Wv *x = (Wv *)(tl + r * P * trow) + l;
            constexpr int th = third / V, pe = period / V;
            const Wv a = x[0] ^ x[pe], b = x[th] ^ x[th + pe], c = x[2 * th] ^ x[2 * th + pe];
            x[0] = x[pe] = a ^ c;
            x[th] = x[th + pe] = a ^ b;
            x[2 * th] = x[2 * th + pe] = b ^ c;
        }
    }
    __syncthreads();
    const rsrc_t xo = make_rsrc(src ? job.S : job.A, (uint32_t)(2 * T * M * 4));
    for (int r = 0; r < nr; ++r)
    for (int sg = wave; sg < P; sg += kGfWaves) {
        const int rho = r ? Q - rho0 : rho0;
        const uint32_t *tr = tile + r * P * trow;
        // tile t0 rotated by (Q / P) sigma t0 rows, as a word offset
        const int turn = lane * trow + (Q - Q / P * sg * lane % Q) * F;
        int off_t[P];
#pragma unroll
        for (int t0 = 0; t0 < P; ++t0) off_t[t0] = __builtin_amdgcn_readlane(turn, t0);
        for (int l = lane * V; l < third; l += 64 * V) {
            const int i = l / F, f = l - i * F;
            Wv lo = 0, hi = 0;
#pragma unroll
            for (int t0 = 0; t0 < P; ++t0) {
                lo ^= *(const Wv *)(tr + off_t[t0] + l);
                hi ^= *(const Wv *)(tr + off_t[t0] + l + 2 * third);
            }
            const int at = ((rho + Q * sg) * (2 * M) + i * Cm + f0 + f) * 4;
            if constexpr (V == 2) {
                st64(xo, at, lo);
                st64(xo, at + M * 4, hi);
            } else {
                st32(xo, at, (int)lo);
                st32(xo, at + M * 4, (int)hi);
            }
        }
    }
}

// P2: the product of X_tau and S_tau in the ring of 2 M words, and its
// combination with the next chunk's overlap, one workgroup per (tau, job).
// An element is a polynomial of 2 * 3^a coefficients of M2 words; its values
// at the points z = u^i, u = v^(M2 / 3^a) of order 3^(a+1), i not a multiple
// of 3, in the ring of 2 M2 words are sums of rotated coefficients.  The
// 2 * 3^a products there are binary Toeplitz products on the matrix cores:
// with the periodic sequence of one factor, output x is the plain
// correlation at x for 0 <= x < 64 M2, so no reduction follows.
//
// Vector issue and the matrix cores bound it: they hardly overlap (256
// blocks of 10^6 bits: 850 us, 290 of it without the leaf products, 700 with
// a fifth of their matrix instructions).  So the leaf loop expands each
// column window once for all tiles, its outputs go to their places at
// immediate offsets, and the transforms of both factors run one after the
// other so that the row operands can take the first one's place: two
// workgroups a CU up to M2 = 45 (blocks of 2.5 10^6 bits: 427 us for eight
// with one, 330 with two).
template <int A, int M2, int W>
struct GfMul {
    static constexpr int NA = A == 1 ? 3 : A == 2 ? 9 : 27;
    static constexpr int NP = 2 * NA, M = NA * M2, U = M2 / NA;
    static_assert(M2 % NA == 0, "the unit rotation is a whole number of words");
    static_assert(64 * M2 + 128 < kGfOnes, "a leaf product's counts");
    static constexpr int tiles = (64 * M2 + 255) / 256, steps = (64 * M2 + 16 + 127) / 128;
    // tiles of one sweep over k (their row fragments stay in registers)
    static constexpr int sweeps = (tiles + 6) / 7, nt = (tiles + sweeps - 1) / sweeps;
    static constexpr int waves = W;
    // LDS (words): area A, the five-third table of X, then the expanded row
    // operands (two words per 16 bits of 128 M2), then the product; area B,
    // the table of S, then that of the products; and the reversed column
    // operands, then the inverse transform's output
    static constexpr int table = (NP * 5 * M2 + 3) / 4 * 4;
    static constexpr int row = 16 * M2, over = 16 * (2 * nt * sweeps + steps);  // a fragment may end past its row
    static constexpr int col = 4 * steps + 2, cols = NP * col > 4 * M ? NP * col : 4 * M;
    static constexpr int area = NP * row + over;
    static_assert(area >= table && area >= 3 * M, "area A");
    static constexpr int off_b = area, off_col = area + table;
    static constexpr int lds_words = off_col + cols;
};

template <int A, int M2, int W>
__global__ void __launch_bounds__(64 * W) k_gf_mul(JobArgs ja, int T, int g, int resident) {
    using G = GfMul<A, M2, W>;
    constexpr int NA = G::NA, NP = G::NP, M = G::M, U = G::U, NTH = 64 * G::waves;
    const JobDesc job = job_of(ja, uni(blockIdx.y));
    const int tau = (int)blockIdx.x, tid = threadIdx.x;
    const int lane = tid & 63, wave = (int)uni((uint32_t)tid >> 6);
    uint32_t *lds = (uint32_t *)pa_lds;
    uint32_t *tx = lds, *rw = lds, *ts = lds + G::off_b, *va = lds + G::off_col;
    const int32_t *S = resident ? job.Shat : job.S;
    const rsrc_t xr = make_rsrc(job.A + (size_t)tau * 2 * M, 2 * M * 4);
    const rsrc_t sr = make_rsrc(S + (size_t)tau * 2 * M, 2 * M * 4);

    // coefficients c of B_r(z) = element mod (z^NA - v^(r M2)), r = 1, 2, in
    // five thirds: (lo, lo+hi, hi, ...) and (lo+hi, lo, hi, ...)
    for (int i = tid; i < 2 * M; i += NTH) {
        const bool second = i >= M;
        const int p = second ? i - M : i, c = p / M2, o = p - c * M2;
        const uint32_t lo = (uint32_t)ld32(second ? sr : xr, p * 4), hi = (uint32_t)ld32(second ? sr : xr, (M + p) * 4);
        uint32_t *t = (second ? ts : tx) + c * 5 * M2 + o;
        t[0] = lo;
        t[M2] = lo ^ hi;
        t[2 * M2] = hi;
        t[3 * M2] = lo;
        t[4 * M2] = lo ^ hi;
        t += NA * 5 * M2;
        t[0] = lo ^ hi;
        t[M2] = lo;
        t[2 * M2] = hi;
        t[3 * M2] = lo ^ hi;
        t[4 * M2] = lo;
    }
    // the column operands' words before and after the element
    for (int i = tid; i < NP * (G::col - 2 * M2); i += NTH) {
        const int pt = i / (G::col - 2 * M2), j = i - pt * (G::col - 2 * M2);
        va[pt * G::col + (j ? 2 * M2 + j : 0)] = 0;
    }
    __syncthreads();
    // value at the point u^(3 i + r), pt = (r - 1) NA + i: the sum of
    // coefficients rotated by (3 i + r) c U; words p0 of both halves
    auto value = [&](const uint32_t *t, int pt, int p0, uint32_t &b0, uint32_t &b1) PA_INLINE {
        const int r = pt >= NA ? 2 : 1;
        const uint32_t step = (uint32_t)(U * (3 * (pt - (r - 1) * NA) + r));
        t += (r - 1) * NA * 5 * M2;
        uint32_t qq = (uint32_t)p0;
        b0 = b1 = 0;
#pragma unroll
        for (int c = 0; c < NA; c += 3) {
            uint32_t w[3][2];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                w[i][0] = t[(c + i) * 5 * M2 + qq];
                w[i][1] = t[(c + i) * 5 * M2 + qq + 2 * M2];
                qq = sub_mod(qq, step, 3 * M2);
            }
            b0 = xor3(b0, w[0][0], w[1][0]) ^ w[2][0];
            b1 = xor3(b1, w[0][1], w[1][1]) ^ w[2][1];
        }
    };
    for (int k = tid; k < NP * M2; k += NTH) {
        const int pt = k / M2, p0 = k - pt * M2;
        uint32_t b0, b1;
        value(tx, pt, p0, b0, b1);
        // bit-reversed as a whole, after one word of zeros
        uint32_t *o = va + pt * G::col;
        o[2 * M2 - p0] = __builtin_bitreverse32(b0);
        o[M2 - p0] = __builtin_bitreverse32(b1);
    }
    __syncthreads();
    for (int k = tid; k < NP * M2; k += NTH) {
        const int pt = k / M2, p0 = k - pt * M2;
        uint32_t b0, b1;
        value(ts, pt, p0, b0, b1);
        // the periodic sequence (b0, b0 + b1, b1, b0), expanded
        gf_v4i *o = (gf_v4i *)(rw + pt * G::row) + p0;
        const gf_v4i e0 = expand_units(b0), e1 = expand_units(b1);
        o[0] = e0;
        o[M2] = e0 ^ e1;
        o[2 * M2] = e1;
        o[3 * M2] = e0;
    }
    __syncthreads();
    // leaf products.  out[x] = sum_k row[x + k] col[k - q - 1] over the row
    // operand's bits and the reversed column operand, x = 256 t + 16 r + q,
    // as in the direct form.  Fragment k + 2 t of the row operand serves
    // step k of tile t and later ones.
    {
        typedef gf_v4i __attribute__((aligned(8))) gf_v4i_a8;
        const int q = lane & 15, kb = lane >> 4;
        // the waves that take one product more are on other SIMDs in other
        // workgroups
        static_assert(G::waves % 4 == 0, "waves are spread evenly over the SIMDs");
        for (int pt = (int)((uint32_t)(wave + (tau & 3)) % (uint32_t)G::waves); pt < NP; pt += G::waves) {
            const uint32_t *cl = va + pt * G::col + kb;
            const uint32_t *rx = rw + pt * G::row + (q + 2 * kb) * 2;
            uint32_t *to = ts + pt * 5 * M2;
#pragma unroll 1
            for (int sw = 0; sw < G::sweeps; ++sw, rx += G::nt * 32) {
                constexpr int NT = G::nt, ST = G::steps;
                gf_v4f acc[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = gf_v4f{kGfBias, kGfBias, kGfBias, kGfBias};
                gf_v4i af[ST + 2 * NT - 2];
#pragma unroll
                for (int k = 0; k < ST; ++k) {
                    const gf_v4i b = expand_window(funnel(cl[4 * k + 1], cl[4 * k], (uint32_t)(31 - q)));
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        if (k < 2 || t == NT - 1) af[k + 2 * t] = *(const gf_v4i_a8 *)(rx + (k + 2 * t) * 16);
                        acc[t] = bit_mfma(b, af[k + 2 * t], acc[t]);
                    }
                }
                // output halfwords 0 .. 2 M2 - 1 are the element's high part,
                // the next 2 M2 its low part: thirds 2 and 3 of the table
                // (tiles may end in the last third, written below)
                static_assert(32 * G::sweeps * NT <= 20 * M2 - 8 * M2, "tiles end in the point's table");
                const uint2 hw = tile_halfwords<NT>(acc);
                uint16_t *o = (uint16_t *)(to + 2 * M2) + 16 * (sw * NT + 4 * kb) + q;
                auto put = [&](int i) PA_INLINE { o[16 * i] = (uint16_t)((i & 2 ? hw.y : hw.x) >> (16 * (i & 1))); };
                constexpr int two = NT > 4 ? NT - 4 : 0;  // fields that lanes 16 .. 31 hold too
                if (lane < 32) {
#pragma unroll
                    for (int i = 0; i < two; ++i) put(i);
                }
                if (lane < 16) {
#pragma unroll
                    for (int i = two; i < (NT < 4 ? NT : 4); ++i) put(i);
                }
            }
            wave_handoff();
            if (lane < M2) {
                static_assert(M2 <= 64, "a lane a word");
                uint32_t *o = to + lane;
                const uint32_t lo = o[3 * M2], v = lo ^ o[2 * M2];
                o[0] = lo;
                o[M2] = v;
                o[4 * M2] = v;
            }
        }
    }
    __syncthreads();
    // inverse: coefficient c modulo z^NA - v^(r M2)
    for (int tk = tid; tk < 2 * M; tk += NTH) {
        const int r = tk >= M ? 2 : 1, k = tk - (r - 1) * M;
        const int c = k / M2, p0 = k - c * M2;
        const uint32_t *t = ts + (r - 1) * NA * 5 * M2;
        uint32_t b0 = 0, b1 = 0;
        const uint32_t step = (uint32_t)(3 * U * c);  // < 3 M2, as is U r c
        uint32_t qq = add_mod((uint32_t)p0, (uint32_t)(U * r * c), 3 * M2);
#pragma unroll
        for (int i = 0; i < NA; i += 3) {
            uint32_t w[3][2];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                w[j][0] = t[(i + j) * 5 * M2 + qq];
                w[j][1] = t[(i + j) * 5 * M2 + qq + 2 * M2];
                qq = add_mod(qq, step, 3 * M2);
            }
            b0 = xor3(b0, w[0][0], w[1][0]) ^ w[2][0];
            b1 = xor3(b1, w[0][1], w[1][1]) ^ w[2][1];
        }
        va[tk] = b0;          // [r][c][p0], low halves, then high halves
        va[2 * M + tk] = b1;
    }
    __syncthreads();
    // the coefficients C_c (2 M2 words each) overlap by M2: block b of the
    // product is C_b low + C_(b-1) high, and v^(2M) = v^M + 1
    {
        const uint32_t *l1 = va, *l2 = va + M, *h1 = va + 2 * M, *h2 = va + 3 * M;
        auto lo_of = [&](int c, int o) PA_INLINE { return l1[c * M2 + o] ^ h1[c * M2 + o] ^ h2[c * M2 + o]; };
        auto hi_of = [&](int c, int o) PA_INLINE { return l1[c * M2 + o] ^ l2[c * M2 + o] ^ h2[c * M2 + o]; };
        auto lo2_of = [&](int c, int o) PA_INLINE { return l1[c * M2 + o] ^ l2[c * M2 + o]; };
        auto hi2_of = [&](int c, int o) PA_INLINE { return h1[c * M2 + o] ^ h2[c * M2 + o]; };
        for (int p = tid; p < M; p += NTH) {
            const int c = p / M2, o = p - c * M2;
            uint32_t c0 = lo_of(c, o), c1 = lo2_of(c, o);
            if (c > 0) {
                c0 ^= hi_of(c - 1, o);
                c1 ^= hi2_of(c - 1, o);
            } else {
                const uint32_t top = hi2_of(NA - 1, o);
                c0 ^= top;
                c1 ^= hi_of(NA - 1, o) ^ top;
            }
            tx[p] = c0;
            tx[M + p] = c0 ^ c1;
            tx[2 * M + p] = c1;
        }
    }
    __syncthreads();
    // with the overlap of the chunk before: beta[p] + beta[p + 2M - g tau],
    // one period and its first third again
    {
        const rsrc_t ho = make_rsrc(job.A + (size_t)T * 2 * M + (size_t)tau * 4 * M, 4 * M * 4);
        const int d = (2 * M + 3 * M - (g * tau) % (3 * M)) % (3 * M);
        for (int p = tid; p < 3 * M; p += NTH) {
            int k = p + d;
            if (k >= 3 * M) k -= 3 * M;
            const int v = (int)(tx[p] ^ tx[k]);
            st32(ho, p * 4, v);
            if (p < M) st32(ho, (p + 3 * M) * 4, v);
        }
    }
}

// P3: word W = t M + e of the cyclic product is the sum over tau of word
// e + g t tau (modulo 3 M) of product tau (whose rows hold 4 M words, so
// that e needs no wrap).  A workgroup takes 64 consecutive words of one t
// from word 63 s; its waves share tau, and each lane finds one product's
// offset, which the loads take as a scalar.  The output starts at bit
// n - 1 (further on by the bits before the key in its first word), so each
// word also takes bits of the next one and 64 words give 63; in a row's last
// segment the word after the row belongs to t + 1, and the offsets are formed
// by lane.  The reads (address units, 88% busy with many blocks) bound it.
// Grid: (segments of 63 words of each t that the output can meet, jobs).
template <int T>
__global__ void __launch_bounds__(64 * kGfWaves) k_gf_inv(JobArgs ja, int g) {
    static_assert(T % kGfWaves == 0, "waves share tau evenly");
    constexpr int K = T / kGfWaves;
    const JobDesc job = job_of(ja, uni(blockIdx.y));
    const int M = T / 3 * g, segs = (M + 62) / 63;
    const uint32_t start = job.n + gf_lead_bits(job, false) - 1u;  // bit of the product where the output starts
    const int words = (int)((job.m + 63u) / 64u * 2u), W0 = (int)(start / 32u);
    const int row = (int)blockIdx.x / segs, t = W0 / M + row, e0 = ((int)blockIdx.x - row * segs) * 63;
    const int w0 = t * M + e0 - W0;  // output word of lane 0
    if (w0 >= words || w0 + 63 <= 0 || t >= T) return;
    const int lane = threadIdx.x & 63, wave = (int)uni(threadIdx.x >> 6);
    const rsrc_t h = make_rsrc(job.A + (size_t)T * 2 * M, (uint32_t)(T * 4 * M * 4));
    const int first = wave * K;  // the wave's products
    uint32_t acc = 0;
    if (e0 + 63 < M) {
#pragma unroll
        for (int b = 0; b < K; b += 27) {
            constexpr int N = K < 27 ? K : 27;
            const int tau = first + b + lane;
            const int at = (tau * 4 * M + g * ((t * tau) % T) + e0) * 4;
#pragma unroll
            for (int k = 0; k < N; ++k)
                acc ^= (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(h, lane * 4, __builtin_amdgcn_readlane(at, k), 0);
        }
    } else {
        const int e = e0 + lane, tl = e < M ? t : t + 1 < T ? t + 1 : 0, el = e < M ? e : 0;
        const uint32_t step = (uint32_t)(4 * g * tl), period = (uint32_t)(12 * M);
        uint32_t p = (uint32_t)(4 * g * ((tl * first) % T));
#pragma unroll 27
        for (int k = 0; k < K; ++k) {
            acc ^= (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(h, (int)p + el * 4, (first + k) * (16 * M), 0);
            p = add_mod(p, step, period);
        }
    }
    __shared__ uint32_t red[kGfWaves][64];
    red[wave][lane] = acc;
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int i = 1; i < kGfWaves; ++i) acc ^= red[i][lane];
        red[0][lane] = acc;
        wave_handoff();
        const int w = w0 + lane;
        if (lane < 63 && e0 + lane < M && w >= 0 && w < words)
            OutWords(job).put((uint32_t)w, funnel(red[0][lane + 1], acc, start & 31u));
    }
}

// P3 for launches over many jobs.  There the reads of k_gf_inv bound it: every
// output word reads one word of each of the T products, through L2 (256
// blocks of 10^6 bits: 1.6 GB in 165 us).  Here a workgroup accumulates
// 1024 K V consecutive words in registers and the products pass through
// LDS, nine at a time and once each, so that a word read from memory serves
// as many outputs as the workgroup has rows of 3 M words (17 at that size);
// word pairs for even G, whose rotations keep them.  Bound by the LDS reads
// and the three operations that step an offset modulo 3 M: 53 us.  (64
// blocks, four ranges each: 41 us, 21.7 staged, 19.8 with a job's ranges on
// one XCD.)
// Grid: (ranges of 1024 K V - 2 output words, jobs), 16 waves.
template <int T, int G, int K>
struct GfInvMany {
    static constexpr int M = T / 3 * G, V = G % 2 == 0 ? 2 : 1, NTH = 1024;
    static constexpr int cover = NTH * K * V, step = cover - 2;  // words held, words written
    static constexpr int stage = 9 * 3 * M;                     // words of nine products
    static constexpr size_t lds = (size_t)(2 * stage > cover ? 2 * stage : cover) * 4;
};
template <int T, int G, int K>
__global__ void __launch_bounds__(1024) k_gf_inv_many(JobArgs ja) {
    using I = GfInvMany<T, G, K>;
    constexpr int M = I::M, V = I::V, NTH = I::NTH, PE = 3 * M, NL = (9 * PE / V + NTH - 1) / NTH;
    static_assert(T % 9 == 0 && PE % V == 0, "nine products a stage");
    typedef typename std::conditional<V == 2, unsigned long long, uint32_t>::type Wv;
    // workgroups go to the eight XCDs in turn, each with an L2 of its own: all
    // ranges of a job to one (jobs past a multiple of eight: as they come)
    uint32_t range = blockIdx.x, of = blockIdx.y;
    if (of < (gridDim.y & ~7u)) {
        const uint32_t id = range + gridDim.x * of, slot = id >> 3, set = slot / gridDim.x;
        range = slot - set * gridDim.x;
        of = set * 8 + (id & 7u);
    }
    const JobDesc job = job_of(ja, uni(of));
    const int tid = threadIdx.x;
    const uint32_t first = job.n + gf_lead_bits(job, false) - 1u;  // bit of the product where the output starts
    const int words = (int)((job.m + 63u) / 64u * 2u), W0 = (int)(first / 32u);
    // cyclic word of the range's first (V = 2: even, so that pairs lie in a row)
    const int base = (W0 & ~(V - 1)) + (int)range * I::step;
    if (base - W0 >= words) return;
    const rsrc_t h = make_rsrc(job.A + (size_t)T * 2 * M, (uint32_t)(T * 4 * M * 4));
    uint32_t *lds = (uint32_t *)pa_lds;
    uint32_t at[K], step[K];  // bytes: offset in the next product, and what the following ones add
    Wv acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int W = base + (tid + NTH * k) * V;
        W -= W >= T * M ? T * M : 0;
        W = W < T * M ? W : 0;  // (words past the last output)
        const int t = W / M;
        at[k] = (uint32_t)(W - t * M) * 4;
        step[k] = (uint32_t)(G * t) * 4;
        acc[k] = 0;
    }
    Wv w[NL];
    auto load = [&](int c) PA_INLINE {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int f = (tid + NTH * i) * V, r = f / PE;
            const int o = (r * 4 * M + f - r * PE) * 4;
            if ((i + 1) * NTH * V <= 9 * PE || f < 9 * PE) {
                if constexpr (V == 2) w[i] = ld64(h, o, c * (9 * 4 * M * 4));
                else w[i] = (Wv)__builtin_amdgcn_raw_buffer_load_b32(h, o, c * (9 * 4 * M * 4), 0);
            }
        }
    };
    auto store = [&](int buf) PA_INLINE {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int f = (tid + NTH * i) * V;
            if ((i + 1) * NTH * V <= 9 * PE || f < 9 * PE) *(Wv *)(lds + buf * I::stage + f) = w[i];
        }
    };
    auto add = [&](int buf) PA_INLINE {
        const char *b = (const char *)(lds + buf * I::stage);
#pragma unroll
        for (int r = 0; r < 9; ++r)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                acc[k] ^= *(const Wv *)(b + at[k] + r * (PE * 4));
                at[k] = add_mod(at[k], step[k], (uint32_t)(PE * 4));
            }
    };
    load(0);
    store(0);
    __syncthreads();
    // products 9 c .. 9 c + 8 in buffer c & 1; the next nine are loaded meanwhile
#pragma unroll 1
    for (int c = 0; c < T / 9; c += 2) {
        if (c + 1 < T / 9) load(c + 1);
        add(0);
        if (c + 1 < T / 9) {
            store(1);
            __syncthreads();
            if (c + 2 < T / 9) load(c + 2);
            add(1);
            if (c + 2 < T / 9) store(0);
        }
        __syncthreads();
    }
    // the output starts at bit n - 1 of the product: each word takes bits of
    // the next one too
#pragma unroll
    for (int k = 0; k < K; ++k) *(Wv *)(lds + (tid + NTH * k) * V) = acc[k];
    __syncthreads();
    const OutWords out(job);
    const uint32_t sh = first & 31u;
    for (int f = tid; f < I::step; f += NTH) {
        const int w = base + f - W0;
        if (w >= 0 && w < words) out.put((uint32_t)w, funnel(lds[f + 1], lds[f], sh));
    }
}

// ---------------------------------------------------------------- launchers

static hipError_t set_lds_limits(int *limit);  // once per device, with gf_set_lds_limits

static hipError_t gf_launch(const void *fn, dim3 grid, int threads, void **args, size_t lds, hipStream_t s,
                            hipEvent_t e0, hipEvent_t e1) {
    if (!fn || grid.x == 0 || grid.y == 0 || grid.z == 0 || grid.y > 65535 || grid.z > 65535)
        return hipErrorInvalidConfiguration;
    int limit = 0;
    const hipError_t e = set_lds_limits(&limit);
    if (e != hipSuccess) return e;
    if (lds > (size_t)limit) return hipErrorInvalidConfiguration;
    return hipExtLaunchKernel(fn, grid, dim3((unsigned)threads), args, lds, s, e0, e1, 0);
}

hipError_t launch_gf_direct(const GfChoice &c, const JobArgs &ja, int njobs, hipStream_t s, hipEvent_t e0,
                            hipEvent_t e1) {
    const void *fn = nullptr;
    const bool parts = c.slices > 1;
    // few tiles a workgroup, so few workgroups: 16 waves that share the key
    // in finer chunks
    const int nw = c.nt == 4 ? 8 : 16;
    if (c.nt == 1 && !parts) fn = (const void *)k_gf_direct<1, 8, 16, false>;
    if (c.nt == 2 && !parts) fn = (const void *)k_gf_direct<2, 8, 16, false>;
    if (c.nt == 4) fn = parts ? (const void *)k_gf_direct<4, 16, 8, true> : (const void *)k_gf_direct<4, 16, 8, false>;
    if (c.form != kGfDirect || ja.seg || c.slices < 1) return hipErrorInvalidConfiguration;
    void *args[] = {(void *)&ja};
    const uint32_t per = 256u * (uint32_t)c.nt;
    return gf_launch(fn, dim3((c.max_m + per - 1) / per, (unsigned)c.slices, (unsigned)njobs), 64 * nw, args, 0, s, e0, e1);
}

hipError_t launch_gf_parts(const GfChoice &c, const JobArgs &ja, int njobs, hipStream_t s, hipEvent_t e0,
                           hipEvent_t e1) {
    if (c.form != kGfDirect || ja.seg) return hipErrorInvalidConfiguration;
    int slices = c.slices;
    void *args[] = {(void *)&ja, (void *)&slices};
    const uint32_t words = (c.max_m + 255) / 256 * 8;
    return gf_launch((const void *)k_gf_parts, dim3((words + 255) / 256, (unsigned)njobs), 256, args, 0, s, e0, e1);
}

// The forward kernels that exist, by (T, g): the classes per workgroup of
// launches over many jobs (whole chunks in order, and two rho a workgroup
// where its LDS leaves room for another workgroup) and of a few jobs (more
// workgroups).
struct GfFwdFn {
    int T, g, F;
    bool many;
    const void *fn;
    unsigned wgs;
    size_t lds;
};
template <int Q, int P, int G, int F, int R = 1>
static GfFwdFn gf_fwd_fn(bool many) {
    return {P * Q, G, F, many, (const void *)k_gf_fwd<Q, P, G, F, R>, (unsigned)((R == 2 ? Q / 2 + 1 : Q) * (G * P / F)),
            (size_t)R * P * 2 * Q * F * 4};
}
static const GfFwdFn *gf_fwd_table(int *count) {
    static const GfFwdFn table[] = {
        gf_fwd_fn<9, 9, 1, 9, 2>(true),  gf_fwd_fn<9, 9, 2, 18, 2>(true), gf_fwd_fn<9, 9, 3, 27, 2>(true),
        gf_fwd_fn<27, 9, 1, 9, 2>(true), gf_fwd_fn<27, 9, 2, 18, 2>(true), gf_fwd_fn<27, 9, 3, 27>(true),
        gf_fwd_fn<27, 9, 4, 36>(true),   gf_fwd_fn<27, 9, 5, 45>(true),  gf_fwd_fn<27, 27, 1, 27>(true),
        gf_fwd_fn<27, 27, 3, 27>(true),  gf_fwd_fn<27, 9, 1, 3>(false),  gf_fwd_fn<27, 9, 2, 6>(false),
        gf_fwd_fn<27, 9, 3, 9>(false),   gf_fwd_fn<27, 9, 4, 12>(false), gf_fwd_fn<27, 9, 5, 5>(false),
        gf_fwd_fn<27, 27, 1, 9>(false),  gf_fwd_fn<27, 27, 3, 9>(false)};
    *count = (int)(sizeof(table) / sizeof(table[0]));
    return table;
}

hipError_t launch_gf_fwd(const GfChoice &c, int nsrc, const JobArgs &ja, int njobs, hipStream_t s, hipEvent_t e0,
                         hipEvent_t e1) {
    if (c.form != kGfSplit || ja.seg) return hipErrorInvalidConfiguration;
    int n = 0;
    const GfFwdFn *t = gf_fwd_table(&n), *best = nullptr;
    for (int i = 0; i < n; ++i)
        if (t[i].T == c.T && t[i].g == c.g && (!best || t[i].many == (njobs > 4))) best = &t[i];
    if (!best) return hipErrorInvalidConfiguration;
    void *args[] = {(void *)&ja};
    return gf_launch(best->fn, dim3(best->wgs, (unsigned)nsrc, (unsigned)njobs), 64 * kGfWaves, args, best->lds, s, e0,
                     e1);
}

// The product kernels that exist: (a, M2), waves, and their LDS.  Launches
// of a few jobs have at most three workgroups a CU and take more waves each:
// 12 for 18 points (two rounds of leaf products, even over the SIMDs).
struct GfMulFn {
    int a, M2;
    bool many;
    const void *fn;
    int threads;
    size_t lds;
};
template <int A, int M2, int W>
static GfMulFn gf_mul_fn(bool many) {
    using G = GfMul<A, M2, W>;
    static_assert(G::lds_words * 4 <= 160 * 1024, "a workgroup's LDS");
    return {A, M2, many, (const void *)k_gf_mul<A, M2, W>, 64 * W, (size_t)G::lds_words * 4};
}
static const GfMulFn *gf_mul_table(int *count) {
    static const GfMulFn table[] = {
        gf_mul_fn<1, 9, 4>(true),   gf_mul_fn<1, 18, 4>(true),  gf_mul_fn<1, 27, 4>(true),  gf_mul_fn<2, 9, 8>(true),
        gf_mul_fn<2, 18, 8>(true),  gf_mul_fn<2, 27, 8>(true),  gf_mul_fn<2, 36, 8>(true),  gf_mul_fn<2, 45, 8>(true),
        gf_mul_fn<3, 27, 16>(true), gf_mul_fn<2, 9, 12>(false), gf_mul_fn<2, 18, 12>(false), gf_mul_fn<2, 27, 12>(false),
        gf_mul_fn<2, 36, 12>(false), gf_mul_fn<2, 45, 12>(false)};
    *count = (int)(sizeof(table) / sizeof(table[0]));
    return table;
}

// The inverse kernels for many jobs: K ascending.  With g = 5 the products are
// so long that ranges of 1024 and 2048 words stage more than k_gf_inv reads
// (10 keys of 3.1 10^6 bits to a third on one seed: 276 us with them, 249).
struct GfInvFn {
    int T, g, step;
    const void *fn;
    size_t lds;
};
template <int T, int G, int K>
static GfInvFn gf_inv_fn() {
    using I = GfInvMany<T, G, K>;
    return {T, G, I::step, (const void *)k_gf_inv_many<T, G, K>, I::lds};
}
static const GfInvFn *gf_inv_table(int *count) {
    static const GfInvFn table[] = {
        gf_inv_fn<243, 1, 1>(), gf_inv_fn<243, 1, 2>(), gf_inv_fn<243, 1, 4>(), gf_inv_fn<243, 2, 1>(),
        gf_inv_fn<243, 2, 2>(), gf_inv_fn<243, 2, 4>(), gf_inv_fn<243, 3, 1>(), gf_inv_fn<243, 3, 2>(),
        gf_inv_fn<243, 3, 4>(), gf_inv_fn<243, 4, 1>(), gf_inv_fn<243, 4, 2>(), gf_inv_fn<243, 4, 4>(),
        gf_inv_fn<243, 5, 4>()};
    *count = (int)(sizeof(table) / sizeof(table[0]));
    return table;
}

// Kernels whose workgroups use more than the default LDS.
static hipError_t gf_set_lds_limits(int maxb) {
    int n = 0;
    const GfMulFn *t = gf_mul_table(&n);
    hipError_t e = hipSuccess;
    for (int i = 0; i < n && e == hipSuccess; ++i)
        e = hipFuncSetAttribute(t[i].fn, hipFuncAttributeMaxDynamicSharedMemorySize, maxb);
    const GfFwdFn *f = gf_fwd_table(&n);
    for (int i = 0; i < n && e == hipSuccess; ++i)
        e = hipFuncSetAttribute(f[i].fn, hipFuncAttributeMaxDynamicSharedMemorySize, maxb);
    const GfInvFn *v = gf_inv_table(&n);
    for (int i = 0; i < n && e == hipSuccess; ++i)
        e = hipFuncSetAttribute(v[i].fn, hipFuncAttributeMaxDynamicSharedMemorySize, maxb);
    return e;
}

hipError_t launch_gf_mul(const GfChoice &c, bool resident, const JobArgs &ja, int njobs, hipStream_t s, hipEvent_t e0,
                         hipEvent_t e1) {
    if (c.form != kGfSplit || ja.seg) return hipErrorInvalidConfiguration;
    int n = 0, T = c.T, g = c.g, r = resident ? 1 : 0;
    const GfMulFn *t = gf_mul_table(&n);
    void *args[] = {(void *)&ja, (void *)&T, (void *)&g, (void *)&r};
    const GfMulFn *best = nullptr;
    for (int i = 0; i < n; ++i)
        if (t[i].a == c.a && t[i].M2 == c.M2 && (!best || t[i].many == (T * njobs > 768))) best = &t[i];
    if (!best) return hipErrorInvalidConfiguration;
    return gf_launch(best->fn, dim3((unsigned)T, (unsigned)njobs), best->threads, args, best->lds, s, e0, e1);
}

// Ranges of `step` words that hold a job's output words and one before.
static unsigned inv_ranges(const GfChoice &c, int step) {
    return ((c.max_m + 63) / 64 * 2 + 1 + (unsigned)step - 1) / (unsigned)step;
}

hipError_t launch_gf_inv(const GfChoice &c, const JobArgs &ja, int njobs, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    const void *fn = nullptr;
    if (c.T == 81) fn = (const void *)k_gf_inv<81>;
    if (c.T == 243) fn = (const void *)k_gf_inv<243>;
    if (c.T == 729) fn = (const void *)k_gf_inv<729>;
    if (c.form != kGfSplit || ja.seg) return hipErrorInvalidConfiguration;
    // many jobs: the widest ranges that still give every CU a workgroup
    int n = 0;
    const GfInvFn *v = gf_inv_table(&n), *best = nullptr;
    for (int i = 0; i < n; ++i)
        if (v[i].T == c.T && v[i].g == c.g && (uint64_t)inv_ranges(c, v[i].step) * (uint64_t)njobs >= 256) best = &v[i];
    if (best) {
        void *many[] = {(void *)&ja};
        return gf_launch(best->fn, dim3(inv_ranges(c, best->step), (unsigned)njobs), 1024, many, best->lds, s, e0, e1);
    }
    int g = c.g;
    void *args[] = {(void *)&ja, (void *)&g};
    // output words can begin anywhere in a row of M
    const unsigned M = (unsigned)c.chunk_words(), words = (c.max_m + 63) / 64 * 2;
    return gf_launch(fn, dim3(((words + M - 2) / M + 1) * ((M + 62) / 63), (unsigned)njobs), 64 * kGfWaves, args, 0, s,
                     e0, e1);
}

}  // namespace pa
