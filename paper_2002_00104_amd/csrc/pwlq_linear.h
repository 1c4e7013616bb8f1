// k_linear: inner products of 8-bit activations with bit-packed PWLQ weights on
// the integer matrix cores (Section 4).  k_linear_wsum: the per-channel constants.
//
// For output channel n with steps s1 = p/L, s2 = (m-p)/L and activations
// X_hat = s_x X_q + z_x, Section 4 splits the inner product by region:
//   P1 = C2 <X_q, W_q1>_R1 + C3,   P2 = C4 <X_q, W_q2>_R2 + C5 <X_q, sigma>_R2 + C6,
// three integer accumulators per output (sigma: the sign of a tail weight, which
// the offset p carries).  On the matrix cores these are three int8 products of the
// same activation tile with three operand planes decoded from the packed codes:
//   plane 0: signed code where the region bit is 0, else 0
//   plane 1: signed code where the region bit is 1, else 0
//   plane 2: sign (+1 / -1) where the region bit is 1, else 0
// The planes exist only in LDS; memory holds b + 1 bits per weight.
//
// A caller that wants y alone does not need the second and third sum apart:
// C5 = C2 L (the offset p is L steps of the centre), so
//   C2 A1 + C5 A3 = C2 (A1 + L A3),
// and L sigma fits an int8 like any code.  The folded form keeps two planes,
//   plane 0: signed code where the region bit is 0, else L sigma
//   plane 1: signed code where the region bit is 1, else 0
// two matrix products per weight instead of three, with the same bound on the
// integer sums (|entry| <= L in both planes).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace pwlq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kLinWM = 2;          // wavefronts along the rows; 2 along the channels
constexpr int kLinBN = 64;        // output channels per workgroup
constexpr int kLinBK = 64;        // reduction elements per step
constexpr int kLinStride = 64;    // bytes per LDS row; the four 16-byte chunks of a row are swizzled
constexpr int kLinWG = 128 * kLinWM;   // wavefronts kLinWM (rows) x 2 (channels), each 32*kMT x 32 outputs

// kMT: 32-row tiles per wavefront.  The accumulators of a wavefront are
// kMT * planes * 16 registers: 3 tiles with three planes (1, 2, 4 measured
// slower), 4 tiles with two.
constexpr int lin_mt(int planes) { return planes == 3 ? 3 : 4; }
constexpr int lin_bm(int planes) { return kLinWM * 32 * lin_mt(planes); }   // activation rows per workgroup
constexpr int lin_avec(int planes) { return lin_bm(planes) * kLinBK / 16 / kLinWG; }   // 16-byte activation loads per thread

// Thread of a group of four wavefronts (k_linear_split has two groups).
__device__ inline int lin_thread() { return threadIdx.x & (kLinWG - 1); }

// LDS rows hold 64 reduction bytes as four 16-byte chunks; chunk c of row r is
// stored at position c ^ swz(r), swz(r) = (r >> 3) & 3.  A 16-byte LDS read of a
// wavefront is served 16 lanes per cycle over 64 banks, and the lanes of a cycle
// are not consecutive: measured on this chip, lanes 0-3, 12-15, 20-23 and 24-27
// go together (of the eight groups of four lanes in each half of the wavefront,
// those whose index has even parity, then those with odd parity).  The fragment
// reads of the matrix cores (lane = row, same chunk) therefore need the four
// groups {0, 3, 5, 6} and {1, 2, 4, 7} of four rows on different chunk
// positions, which r >> 3 gives; a swizzle that spreads consecutive rows
// instead costs 6.9 cycles per read against 3.6.  The 16-byte writes of the
// staging threads (four lanes = the four chunks of one row) are indifferent to it.
__device__ inline int lin_swz(int row) { return (row >> 3) & 3; }

// 16 consecutive b-bit codes of a stream (sign-magnitude: bit b-1 is the sign)
// starting at element index e0 (a multiple of 16) occupy 2b bytes that start
// 2-byte aligned (4-byte aligned for even b, 8 for b = 4, 16 for b = 8).
// load_raw16 only issues the loads; unpack16 turns the raw bytes into 16 bytes,
// one code in the low bits of each byte, in order.  Keeping the two apart lets the loads of a later
// step fly while the matrix cores work on the current one.
template <int kBits>
struct RawCodes {
    uint32_t w[(2 * kBits + 3) / 4];
};

template <int kBits>
__device__ inline void load_raw16(const uint8_t *__restrict__ stream, long long e0,
                                  RawCodes<kBits> &raw)
{
    const uint8_t *src = stream + (e0 >> 4) * (2 * kBits);
    if (kBits == 4) {
        const uint2 v = *reinterpret_cast<const uint2 *>(src);
        raw.w[0] = v.x;
        raw.w[1] = v.y;
    } else if (kBits == 8) {
        const uint4 v = *reinterpret_cast<const uint4 *>(src);
        raw.w[0] = v.x; raw.w[1] = v.y; raw.w[2] = v.z; raw.w[3] = v.w;
    } else if (kBits % 2 == 0) {
#pragma unroll
        for (int i = 0; i < kBits / 2; ++i) raw.w[i] = reinterpret_cast<const uint32_t *>(src)[i];
    } else {
        const uint16_t *s16 = reinterpret_cast<const uint16_t *>(src);
#pragma unroll
        for (int i = 0; i < (2 * kBits + 3) / 4; ++i) raw.w[i] = 0;
#pragma unroll
        for (int i = 0; i < kBits; ++i) raw.w[i / 2] |= (uint32_t)s16[i] << (16 * (i & 1));
    }
}

template <int kBits>
__device__ inline void zero_raw16(RawCodes<kBits> &raw)
{
#pragma unroll
    for (int i = 0; i < (2 * kBits + 3) / 4; ++i) raw.w[i] = 0;
}

template <int kBits>
__device__ inline void unpack16(const RawCodes<kBits> &raw, uint32_t (&out)[4])
{
    if (kBits == 4) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t ev = raw.w[h];                        // elements 0,2,4,6 of this half in the low nibbles
            const uint32_t od = raw.w[h] >> 4;                   // elements 1,3,5,7
            // interleave bytes: (e0,o0,e1,o1) and (e2,o2,e3,o3)
            out[2 * h] = __builtin_amdgcn_perm(od, ev, 0x05010400u);
            out[2 * h + 1] = __builtin_amdgcn_perm(od, ev, 0x07030602u);
        }
    } else if (kBits == 8) {
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = raw.w[i];
    } else {
        constexpr uint32_t mask = (1u << kBits) - 1u;
#pragma unroll
        for (int wd = 0; wd < 4; ++wd) {
            uint32_t word = 0;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int pos = (wd * 4 + x) * kBits;       // compile-time after unrolling
                const int wi = pos >> 5, sh = pos & 31;
                uint32_t v = raw.w[wi] >> sh;
                if (sh + kBits > 32) v |= raw.w[wi + 1] << (32 - sh);
                word |= (v & mask) << (8 * x);
            }
            out[wd] = word;
        }
    }
}

// Four sign-magnitude codes (one per byte; bits above the code are ignored) and their four
// region bits (low nibble of f) -> the operand planes, four int8 each.  Two forms with the same
// results.  By borrows: a byte mask is a subtraction and an exclusive or.  `bits` is an int or a
// std::integral_constant: the latter lets the compiler fold the masks before it sees the kernel around
// them, which schedules some kernels 1-4 % faster and others 1-4 % slower (see weight_planes).
template <typename Bits>
__device__ inline void planes4(uint32_t codes, uint32_t f, Bits bits, uint32_t &w1, uint32_t &w2, uint32_t &w3)
{
    const uint32_t magmask = ((1u << (bits - 1)) - 1u) * 0x01010101u;
    const uint32_t mag = codes & magmask;
    const uint32_t sgn = (codes >> (bits - 1)) & 0x01010101u;
    // 0xff in the bytes that hold 1 (written so that it stays two full-rate
    // instructions: x * 0xff would be a quarter-rate 32-bit multiply)
    const uint32_t smask = (0x80808080u - sgn) ^ 0x80808080u;          // negative codes
    const uint32_t neg = (0x80808080u - mag) ^ 0x80808080u;            // -mag per byte (mag <= 127)
    const uint32_t val = (neg & smask) | (mag & ~smask);
    const uint32_t f01 = __umul24(f & 0xfu, 0x00204081u) & 0x01010101u;   // region bit of each byte (24-bit multiply: full rate)
    const uint32_t fm = (0x80808080u - f01) ^ 0x80808080u;             // tail bytes
    w1 = val & ~fm;
    w2 = val & fm;
    w3 = (smask | 0x01010101u) & fm;
}

// The folded form: plane 0 holds L sigma in the tail bytes, plane 1 as above.
template <typename Bits>
__device__ inline void planes4_folded(uint32_t codes, uint32_t f, Bits bits, uint32_t &w1, uint32_t &w2)
{
    const uint32_t magmask = ((1u << (bits - 1)) - 1u) * 0x01010101u;      // L in every byte
    const uint32_t mag = codes & magmask;
    const uint32_t sgn = (codes >> (bits - 1)) & 0x01010101u;
    const uint32_t smask = (0x80808080u - sgn) ^ 0x80808080u;
    const uint32_t f01 = __umul24(f & 0xfu, 0x00204081u) & 0x01010101u;
    const uint32_t fm = (0x80808080u - f01) ^ 0x80808080u;
    const uint32_t neg = (0x80808080u - mag) ^ 0x80808080u;
    const uint32_t val = (neg & smask) | (mag & ~smask);                   // signed code
    const uint32_t negl = (0x80808080u - magmask) ^ 0x80808080u;           // -L in every byte
    const uint32_t lsig = (negl & smask) | (magmask & ~smask);             // L sigma
    w1 = (lsig & fm) | (val & ~fm);
    w2 = val & fm;
}

// By look-ups: byte masks and values of small codes with v_perm_b32, one instruction for four: a selector
// 0..3 takes a byte of its second source, 4..7 of its first, 8 the sign of the second's byte 1 in every bit, 13 and
// above 0xff.  In the folded form 12 instructions for four codes at b = 4, 17 by borrows.
template <int kBits>
struct SignedCodes {
    uint32_t val, smask, lsig;         // signed codes; 0xff in the bytes of negative ones; L with the code's sign
};
template <int kBits>
__device__ inline SignedCodes<kBits> signed_codes(uint32_t codes)
{
    SignedCodes<kBits> r;
    if constexpr (kBits <= 3) {        // a whole code is a selector
        const uint32_t c = codes & ((1u << kBits) - 1u) * 0x01010101u;
        r.val = __builtin_amdgcn_perm(0xfdfeff00u, kBits == 2 ? 0xff000100u : 0x03020100u, c);
        r.smask = __builtin_amdgcn_perm(0xffffffffu, kBits == 2 ? 0xffff0000u : 0u, c);
        r.lsig = __builtin_amdgcn_perm(0xfdfdfdfdu, kBits == 2 ? 0xffff0101u : 0x03030303u, c);
    } else {
        constexpr uint32_t L4 = ((1u << (kBits - 1)) - 1u) * 0x01010101u;      // L in every byte
        constexpr uint32_t negL4 = (0x80808080u - L4) ^ 0x80808080u;
        r.smask = __builtin_amdgcn_perm(0u, kBits == 4 ? 0x00008000u : 0u, codes & ((1u << (kBits - 1)) * 0x01010101u));
        const uint32_t mag = codes & L4;
        // -mag: from a table, or by a borrow (mag <= 127)
        const uint32_t neg = kBits == 4 ? __builtin_amdgcn_perm(0xf9fafbfcu, 0xfdfeff00u, mag)
                                        : (0x80808080u - mag) ^ 0x80808080u;
        r.val = (neg & r.smask) | (mag & ~r.smask);
        r.lsig = (negL4 & r.smask) | (L4 & ~r.smask);
    }
    return r;
}
// 0xff in the tail bytes
__device__ inline uint32_t tail_mask(uint32_t f)
{
    return __builtin_amdgcn_perm(0u, 0x0000ff00u, __umul24(f & 0xfu, 0x00204081u) & 0x01010101u);
}

// The form a kernel takes, the faster one in 34 calls of 1 to 4096 rows (best of four runs in turn, us).  To
// four bits look-ups: 8x4096x11008, b = 2, 11.8/9.5, b = 4 10.8/10.3; 4096^3 162.7/152.6, 159.9/153.8.  From five
// on a code's unpacking is the longer part:
//  - k_linear gains with the sums apart (4096^3, b = 5 -4 %, b = 6 -2 %) and at 8 bits, and loses in
//    the folded form at five to seven (2048x1024x2048, b = 7, 22.8/23.8; 600x1040x3000, b = 5, 21.5/22.1);
//  - k_linear_rows gains in 15 rows by 16 channels (8x4096x11008, b = 7, 16.3/15.2, b = 8, three sums, 14.8/13.7), and
//    at 8 bits but for 63 rows with the sums apart (63x4096x11008 41.0/42.6); elsewhere look-ups take 20 to 40 registers more,
//    and may take a workgroup per CU (31x1024x5000, b = 6, three sums, 6.2/7.0).
enum Decode { kBorrows, kBorrowsConst, kLookUps };        // (kBorrowsConst: `bits` an integral_constant)
constexpr Decode linear_decode(int bits, int planes) { return bits <= 4 || bits == 8 || planes == 3 ? kLookUps : kBorrows; }
constexpr Decode rows_decode(int bits, int planes, int tile, int mt)
{
    const bool row15 = tile == 16 && mt == 1, row31 = tile == 16 && mt == 2, row63 = tile == 32 && mt == 2;
    if (bits <= 4) return kLookUps;
    if (bits == 8) return row63 && planes == 3 ? kBorrows : kLookUps;      // (planes == 2: see kRows63BorrowsK)
    if (planes == 2 && row15) return kLookUps;
    // b = 5, 6, 7, 31x4096x11008: kBorrows 20.7/21.6/23.2, kBorrowsConst 21.3/21.1/23.0, kLookUps 20.9/20.7/22.7;
    // 24x512x11008: 6.7/6.9/7.0, 6.7/6.9/6.8, 6.5/6.6/7.1; 31x1024x5000: 5.9/6.3/6.1, 6.1/6.4/6.0, 6.0/6.2/6.2
    if (planes == 2 && row31) return bits == 5 ? kBorrows : bits == 6 ? kLookUps : kBorrowsConst;
    // 63x4096x1500, b = 5, 11.5 with kBorrows, 11.1 with kBorrowsConst
    return row15 || row31 || row63 ? kBorrows : kBorrowsConst;
}

// Four weights of each of kPlanes planes (three, or two in the folded form).
template <int kBits, int kPlanes, Decode kDecode>
__device__ inline void weight_planes(uint32_t codes, uint32_t f, uint32_t &w1, uint32_t &w2, uint32_t &w3)
{
    if constexpr (kDecode == kLookUps) {
        const SignedCodes<kBits> c = signed_codes<kBits>(codes);
        const uint32_t fm = tail_mask(f);
        w1 = kPlanes == 3 ? c.val & ~fm : (c.lsig & fm) | (c.val & ~fm);
        w2 = c.val & fm;
        if (kPlanes == 3) w3 = (c.smask | 0x01010101u) & fm;
    } else if constexpr (kDecode == kBorrowsConst) {
        if constexpr (kPlanes == 3) planes4(codes, f, std::integral_constant<int, kBits>(), w1, w2, w3);
        else planes4_folded(codes, f, std::integral_constant<int, kBits>(), w1, w2);
    } else {
        if constexpr (kPlanes == 3) planes4(codes, f, kBits, w1, w2, w3);
        else planes4_folded(codes, f, kBits, w1, w2);
    }
}

// ---------------------------------------------------------------- constants
// s1 * sum_R1 w_q + s2 * sum_R2 w_q + p * sum_R2 sigma (binary64, rounded to
// binary32): multiplied by z_x it is C3 + C6 of Section 4.  `sums` are those of the
// weights in each plane.  The folded form has the first and third as one sum and p / L
// for both.  Every kernel forms a channel's constant here, so that a row of y is the
// same whichever kernel the number of rows chooses.
template <int kPlanes>
__device__ inline float lin_constant(const int (&sums)[kPlanes], float pn, float s1, float s2, float Lf)
{
    if (kPlanes == 3)
        return (float)((double)s1 * (double)sums[0] + (double)s2 * (double)sums[1] +
                       (double)pn * (double)sums[kPlanes - 1]);
    return (float)((double)pn / (double)Lf * (double)sums[0] + (double)s2 * (double)sums[1]);
}

// wconst[n]: the constant of channel n.  One wavefront per channel.
__device__ inline int add_bytes(uint32_t w, int sum)
{
    return __builtin_amdgcn_sdot4((int)w, 0x01010101, sum, false);
}

template <int kBits, int kPlanes>
__global__ __launch_bounds__(kLinWG) void k_linear_wsum(const uint8_t *__restrict__ pcodes,
                                                        const uint8_t *__restrict__ pflags,
                                                        long long N, long long K,
                                                        const float *__restrict__ p,
                                                        const float *__restrict__ m,
                                                        float *__restrict__ wconst)
{
    const long long n = (long long)blockIdx.x * (kLinWG / 64) + (threadIdx.x >> 6);
    if (n >= N) return;
    const int lane = threadIdx.x & 63;
    int sums[kPlanes] = {};
    constexpr int kStep = 16 * 64, kAhead = 4;
    // kCount runs of 16 codes, all loads in flight first: a channel's wavefront waits for memory
    // and little else (b = 4, us: K = 4096, 4096 channels 6.1 -> 4.8; K = 11008 11.6 -> 9.6).  A lane's last
    // runs, up to three, are waited for one by one: up to K = 3072 that is all of them.
    const auto runs = [&](long long k0, auto count) {
        constexpr int kCount = decltype(count)::value;
        RawCodes<kBits> raw[kCount];
        uint32_t f[kCount];
#pragma unroll
        for (int i = 0; i < kCount; ++i) {
            const long long e0 = n * K + k0 + i * kStep;
            load_raw16<kBits>(pcodes, e0, raw[i]);
            f[i] = *reinterpret_cast<const uint16_t *>(pflags + (e0 >> 3));
        }
#pragma unroll
        for (int i = 0; i < kCount; ++i) {
            uint32_t c[4];
            unpack16<kBits>(raw[i], c);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                uint32_t w[3];
                weight_planes<kBits, kPlanes, linear_decode(kBits, kPlanes)>(c[x], f[i] >> (4 * x), w[0], w[1], w[2]);
#pragma unroll
                for (int pl = 0; pl < kPlanes; ++pl) sums[pl] = add_bytes(w[pl], sums[pl]);
            }
        }
    };
    long long k0 = 16LL * lane;
    for (; k0 + (kAhead - 1) * kStep < K; k0 += kAhead * kStep) runs(k0, std::integral_constant<int, kAhead>());
    for (; k0 < K; k0 += kStep) runs(k0, std::integral_constant<int, 1>());
    for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
        for (int pl = 0; pl < kPlanes; ++pl) sums[pl] += __shfl_xor(sums[pl], off, 64);
    }
    if (lane == 0) {
        const float Lf = (float)((1 << (kBits - 1)) - 1);
        const float pn = p[n], mn = m[n];
        const float s1 = pn / Lf;
        const float width = mn - pn;
        const float s2 = width / Lf;
        wconst[n] = lin_constant<kPlanes>(sums, pn, s1, s2, Lf);
    }
}

// -------------------------------------------------------------------- linear
template <int kBits, int kAVec>
struct LinStage {
    v4i a[kAVec];       // activation bytes: vector v of thread t is piece t + v*kLinWG of the tile
    RawCodes<kBits> codes; // 16 packed weight codes
    uint32_t flags;        // their 16 region bits
};

// Issues the loads of one reduction step and nothing else.  Rows past M and
// channels past N read the last valid row / channel instead (their products are
// never written), so no load sits under a branch and the compiler can count the
// outstanding loads exactly.
// kvalid: how many of the step's four 16-element pieces lie below K (4 except in
// the last step when K is not a multiple of 64); the others read the step's first
// piece instead and are zeroed when the step is written to LDS.
template <int kBits, int kAVec>
__device__ inline void lin_load(LinStage<kBits, kAVec> &st, const int8_t *__restrict__ xq, long long M,
                                long long K, const uint8_t *__restrict__ pcodes,
                                const uint8_t *__restrict__ pflags, long long N, long long row0,
                                long long col0, long long k0, int kvalid)
{
    static_assert(kLinWG == 4 * kLinBN, "every thread carries 16 weights of the tile");
    const int t = lin_thread();
    const int c = ((t & 3) < kvalid) ? (t & 3) : 0;     // piece & 3 == t & 3: kLinWG is a multiple of 4
#pragma unroll
    for (int v = 0; v < kAVec; ++v) {
        const int piece = t + v * kLinWG;              // 4 pieces of 16 bytes per row
        long long r = row0 + (piece >> 2);
        r = r < M ? r : M - 1;
        st.a[v] = *reinterpret_cast<const v4i *>(xq + r * K + k0 + c * 16);
    }
    long long n = col0 + (t >> 2);
    n = n < N ? n : N - 1;
    const long long e0 = n * K + k0 + c * 16;
    load_raw16<kBits>(pcodes, e0, st.codes);
    st.flags = *reinterpret_cast<const uint16_t *>(pflags + (e0 >> 3));
}

// The same loads for a step that lies wholly below K, from addresses split into
// a base that is the same in every lane and changes from step to step (scalar
// arithmetic) and a 32-bit offset per thread that never changes (computed once,
// before the loop): no vector address arithmetic per step.
template <int kBits, int kAVec>
struct LinOffsets {
    unsigned a[kAVec];      // from xq + row0*K + k0
    unsigned codes, flags;     // from the streams at element col0*K + k0
};

template <int kBits, int kAVec>
__device__ inline LinOffsets<kBits, kAVec> lin_offsets(long long M, long long K, long long N,
                                                long long row0, long long col0)
{
    LinOffsets<kBits, kAVec> o;
    const int t = lin_thread();
#pragma unroll
    for (int v = 0; v < kAVec; ++v) {
        const int piece = t + v * kLinWG;
        long long r = row0 + (piece >> 2);
        r = r < M ? r : M - 1;
        o.a[v] = (unsigned)((r - row0) * K) + (unsigned)((t & 3) * 16);     // < 256 * 2^22 + 64
    }
    long long n = col0 + (t >> 2);
    n = n < N ? n : N - 1;
    const unsigned piece16 = (unsigned)((n - col0) * (K >> 4)) + (unsigned)(t & 3);   // in runs of 16 elements
    o.codes = piece16 * (2 * kBits);
    o.flags = piece16 * 2;
    return o;
}

template <int kBits, int kAVec>
__device__ inline void lin_load_whole(LinStage<kBits, kAVec> &st, const LinOffsets<kBits, kAVec> &o,
                                      const int8_t *__restrict__ a_base,
                                      const uint8_t *__restrict__ code_base,
                                      const uint8_t *__restrict__ flag_base)
{
#pragma unroll
    for (int v = 0; v < kAVec; ++v)
        st.a[v] = *reinterpret_cast<const v4i *>(a_base + o.a[v]);
    load_raw16<kBits>(code_base + o.codes, 0, st.codes);
    st.flags = *reinterpret_cast<const uint16_t *>(flag_base + o.flags);
}

// Writes one step into LDS: activations as they are, weights decoded into the
// operand planes (three, or two in the folded form).
template <int kBits, int kPlanes, Decode kDecode, int kAVec>
__device__ inline void lin_store(const LinStage<kBits, kAVec> &st, int8_t *__restrict__ sA,
                                 int8_t *__restrict__ sB, int kvalid)
{
    const int t = lin_thread();
    const int keep = ((t & 3) < kvalid) ? -1 : 0;       // all ones for a piece below K
#pragma unroll
    for (int v = 0; v < kAVec; ++v) {
        const int piece = t + v * kLinWG;
        v4i a = st.a[v];
        a[0] &= keep; a[1] &= keep; a[2] &= keep; a[3] &= keep;
        *reinterpret_cast<v4i *>(sA + (piece >> 2) * kLinStride +
                                 (((piece & 3) ^ lin_swz(piece >> 2)) * 16)) = a;
    }
    uint32_t c[4];
    unpack16<kBits>(st.codes, c);
    v4i w1, w2, w3;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        uint32_t a, b, d = 0;
        weight_planes<kBits, kPlanes, kDecode>(c[x], st.flags >> (4 * x), a, b, d);
        w1[x] = (int)a & keep;
        w2[x] = (int)b & keep;
        w3[x] = (int)d & keep;
    }
    const int off = (t >> 2) * kLinStride + (((t & 3) ^ lin_swz(t >> 2)) * 16);
    *reinterpret_cast<v4i *>(sB + off) = w1;
    *reinterpret_cast<v4i *>(sB + kLinBN * kLinStride + off) = w2;
    if (kPlanes == 3) *reinterpret_cast<v4i *>(sB + 2 * kLinBN * kLinStride + off) = w3;
}

// One reduction step of a wavefront: fragments of LDS buffer `buf`, the next
// step decoded into the other buffer (kStore), 2 * kMT * kPlanes matrix
// instructions, one barrier.
template <int kBits, int kPlanes, Decode kDecode, bool kStore, int kMT, int kAVec>
__device__ inline void lin_step(v16i (&acc)[kMT][kPlanes],
                                const LinStage<kBits, kAVec> &next, int kvalid_next,
                                const int8_t *a_lane, const int8_t *b_lane, int swz, int half,
                                int8_t *sA0, int8_t *sB0, int buf)
{
    constexpr int kABuf = kLinWM * 32 * kMT * kLinStride, kBBuf = kPlanes * kLinBN * kLinStride;
    const int8_t *a_base = a_lane + buf * kABuf;
    const int8_t *b_base = b_lane + buf * kBBuf;
    v4i bf[kLinBK / 32][kPlanes], af[kLinBK / 32][kMT];
#pragma unroll
    for (int ks = 0; ks < kLinBK / 32; ++ks) {
        const int chunk = ((2 * ks + half) ^ swz) * 16;
#pragma unroll
        for (int pl = 0; pl < kPlanes; ++pl)
            bf[ks][pl] = *reinterpret_cast<const v4i *>(b_base + pl * kLinBN * kLinStride + chunk);
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt)
            af[ks][mt] = *reinterpret_cast<const v4i *>(a_base + mt * 32 * kLinStride + chunk);
    }
    if (kStore)
        lin_store<kBits, kPlanes, kDecode, kAVec>(next, sA0 + (buf ^ 1) * kABuf, sB0 + (buf ^ 1) * kBBuf, kvalid_next);
#pragma unroll
    for (int ks = 0; ks < kLinBK / 32; ++ks)
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
            for (int pl = 0; pl < kPlanes; ++pl)
                acc[mt][pl] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[ks][mt], bf[ks][pl],
                                                                    acc[mt][pl], 0, 0, 0);
    __syncthreads();
}

// Workgroup ids are dealt round-robin to the 8 XCDs.  Each XCD takes a
// contiguous eighth of the channel tiles (their packed weights, about 1 MB,
// stay in its L2) and walks them for one row tile before the next row tile, so
// that the workgroups in flight on an XCD share a few activation tiles: every
// XCD then reads the activations once instead of once per channel tile.
//
// Pipeline of a step kt: the loads of step kt+2 are issued, the fragments of
// step kt are read from LDS buffer kt&1, step kt+1 (loaded one step ago) is
// decoded into the other buffer, the matrix cores run, one barrier.
//
// kPlanes = 3: the three sums of Section 4 apart (acc_out may receive them);
// kPlanes = 2: the folded form, y only.
template <int kBits, int kPlanes>
__global__ __launch_bounds__(kLinWG, 2) void k_linear(const int8_t *__restrict__ xq, long long M,
                                                   long long K, float s_x, float z_x,
                                                   const uint8_t *__restrict__ pcodes,
                                                   const uint8_t *__restrict__ pflags,
                                                   long long N,
                                                   const float *__restrict__ p,
                                                   const float *__restrict__ m,
                                                   const float *__restrict__ wconst,
                                                   float *__restrict__ y, int *__restrict__ acc_out,
                                                   int tiles_m, int tiles_n, int tn_per_xcd)
{
    constexpr int kMT = lin_mt(kPlanes), kBM = lin_bm(kPlanes), kAVec = lin_avec(kPlanes);
    constexpr Decode kDecode = linear_decode(kBits, kPlanes);
    __shared__ __attribute__((aligned(16))) int8_t sA[2][kBM * kLinStride];
    __shared__ __attribute__((aligned(16))) int8_t sB[2][kPlanes * kLinBN * kLinStride];

    const int xcd = blockIdx.x & 7;
    const int slot = blockIdx.x >> 3;
    const int bn = xcd * tn_per_xcd + slot % tn_per_xcd;
    const int bm = slot / tn_per_xcd;
    if (bm >= tiles_m || bn >= tiles_n) return;
    const long long row0 = (long long)bm * kBM, col0 = (long long)bn * kLinBN;

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;        // wm in [0, kLinWM)

    v16i acc[kMT][kPlanes];
#pragma unroll
    for (int a = 0; a < kMT; ++a)
#pragma unroll
        for (int b = 0; b < kPlanes; ++b)
#pragma unroll
            for (int c = 0; c < 16; ++c) acc[a][b][c] = 0;

    // K is a multiple of 16; the last step holds 1 to 4 pieces of 16 elements
    const int steps = (int)((K + kLinBK - 1) / kLinBK);
    const int last_valid = (int)((K - (long long)(steps - 1) * kLinBK) / 16);
    auto valid = [&](int step) { return step == steps - 1 ? last_valid : 4; };
    LinStage<kBits, kAVec> near, far;
    lin_load<kBits, kAVec>(near, xq, M, K, pcodes, pflags, N, row0, col0, 0, valid(0));
    lin_store<kBits, kPlanes, kDecode, kAVec>(near, sA[0], sB[0], valid(0));
    if (steps > 1) lin_load<kBits, kAVec>(near, xq, M, K, pcodes, pflags, N, row0, col0, kLinBK, valid(1));
    __syncthreads();
    // row of this lane's fragments (every 32-row tile of a wavefront has the same
    // swizzle: tiles start at multiples of 32 rows) and its chunk swizzle
    const int8_t *a_lane = sA[0] + (wm * 32 * kMT + (lane & 31)) * kLinStride;
    const int8_t *b_lane = sB[0] + (wn * 32 + (lane & 31)) * kLinStride;
    const int swz = lin_swz(lane & 31), half = lane >> 5;
    // the last two steps have nothing left to load / to decode: peeled, so that
    // the steady-state body is free of branches
    int kt = 0;
    // Steady state, two steps per trip so that the two register stages swap roles
    // instead of being copied; every step loaded here lies wholly below K.
    const LinOffsets<kBits, kAVec> offs = lin_offsets<kBits, kAVec>(M, K, N, row0, col0);
    const int8_t *a_base = xq + row0 * K;                                   // + k0
    const uint8_t *code_base = pcodes + ((col0 * K) >> 4) * (2 * kBits);    // + (k0 / 16) * 2b
    const uint8_t *flag_base = pflags + ((col0 * K) >> 3);                  // + k0 / 8
    for (; kt + 4 < steps; kt += 2) {
        const long long k2 = (long long)(kt + 2) * kLinBK, k3 = k2 + kLinBK;
        lin_load_whole<kBits, kAVec>(far, offs, a_base + k2, code_base + (k2 >> 4) * (2 * kBits), flag_base + (k2 >> 3));
        lin_step<kBits, kPlanes, kDecode, true>(acc, near, 4, a_lane, b_lane, swz, half, sA[0], sB[0], 0);
        lin_load_whole<kBits, kAVec>(near, offs, a_base + k3, code_base + (k3 >> 4) * (2 * kBits), flag_base + (k3 >> 3));
        lin_step<kBits, kPlanes, kDecode, true>(acc, far, 4, a_lane, b_lane, swz, half, sA[0], sB[0], 1);
    }
    for (; kt + 2 < steps; ++kt) {
        lin_load<kBits, kAVec>(far, xq, M, K, pcodes, pflags, N, row0, col0, (long long)(kt + 2) * kLinBK,
                               valid(kt + 2));
        lin_step<kBits, kPlanes, kDecode, true>(acc, near, valid(kt + 1), a_lane, b_lane, swz, half, sA[0], sB[0], kt & 1);
        near = far;
    }
    if (kt + 1 < steps) {
        lin_step<kBits, kPlanes, kDecode, true>(acc, near, valid(kt + 1), a_lane, b_lane, swz, half, sA[0], sB[0], kt & 1);
        ++kt;
    }
    lin_step<kBits, kPlanes, kDecode, false>(acc, near, 4, a_lane, b_lane, swz, half, sA[0], sB[0], kt & 1);

    // epilogue: C2 A1 + C4 A2 + C5 A3 + (C3 + C6), per output channel
    const long long n = col0 + wn * 32 + (lane & 31);
    if (n >= N) return;
    const float Lf = (float)((1 << (kBits - 1)) - 1);
    const float pn = p[n], mn = m[n];
    const float s1 = pn / Lf;
    const float width = mn - pn;
    const float s2 = width / Lf;
    const float cst = z_x * wconst[n];
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const long long row = row0 + wm * 32 * kMT + mt * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
            if (row < M) {
                if (kPlanes == 3) {
                    const int a1 = acc[mt][0][r], a2 = acc[mt][1][r], a3 = acc[mt][2][r];
                    float t = s1 * (float)a1;
                    t = __builtin_fmaf(s2, (float)a2, t);
                    t = __builtin_fmaf(pn, (float)a3, t);
                    y[row * N + n] = __builtin_fmaf(s_x, t, cst);
                    if (acc_out) {
                        acc_out[(0 * M + row) * N + n] = a1;
                        acc_out[(1 * M + row) * N + n] = a2;
                        acc_out[(2 * M + row) * N + n] = a3;
                    }
                } else {
                    // acc[mt][0] = A1 + L A3
                    float t = s1 * (float)acc[mt][0][r];
                    t = __builtin_fmaf(s2, (float)acc[mt][1][r], t);
                    y[row * N + n] = __builtin_fmaf(s_x, t, cst);
                }
            }
        }
    }
}

// ------------------------------------------------------- half the reduction each
// k_linear_split: the folded form for calls whose tiles do not fill the chip.  One
// workgroup of k_linear per CU is one wavefront per SIMD, which issues an instruction
// every eight or nine cycles and waits out every barrier and LDS read alone.  Here the
// tile is 128 rows instead of 256 and a workgroup has two groups of four wavefronts,
// each with LDS buffers of its own and half of the reduction; their whole-number sums are
// exchanged through LDS, each group finishing half of the rows.  The sums are whole
// numbers, so the split changes no result.  Bound by the latency of a step (LDS write,
// barrier, fragment reads, matrix instructions): K = 4096, b = 4, k_linear against this
// kernel, whole call in us: 512x4096 50.8/33.3, 128x11008 55.6/37.7; K = 8192 90.7/58.5;
// K = 512, 1024x2048 15.7/12.6; K = 1024, 2048x1024 20.5/15.2.
constexpr int kSplitMT = 2, kSplitBM = kLinWM * 32 * kSplitMT;
constexpr int kSplitAVec = kSplitBM * kLinBK / 16 / kLinWG;
constexpr int kSplitMaxWgs = 384;      // the rule stands where it is applied
constexpr int kSplitMinK = 512;        // K is a multiple of 128: whole steps, as many in both halves
// At 8 bits the look-ups spill 18 registers, the borrows 8, all outside the loop over the steps, where the
// look-ups are the faster ones (us, borrows / look-ups: 768x512x4096 14.9/15.8, 900x1024x2000 14.0/14.4,
// 700x1536x3000 24.2/24.1, 300x3072x5000 28.2/27.8, 31x4096x11008 35.9/34.3).
constexpr int kSplitBorrowsMaxK = 1024;

template <int kBits, Decode kDecode>
__global__ __launch_bounds__(2 * kLinWG, 4) void k_linear_split(const int8_t *__restrict__ xq, long long M, long long K,
                                                         float s_x, float z_x, const uint8_t *__restrict__ pcodes,
                                                         const uint8_t *__restrict__ pflags, long long N,
                                                         const float *__restrict__ p, const float *__restrict__ m,
                                                         const float *__restrict__ wconst, float *__restrict__ y,
                                                         int tiles_m, int tiles_n, int tn_per_xcd)
{
    constexpr int kMT = kSplitMT, kAVec = kSplitAVec;
    __shared__ __attribute__((aligned(16))) int8_t sA[2][2 * kSplitBM * kLinStride];         // [group][two buffers]
    __shared__ __attribute__((aligned(16))) int8_t sB[2][2 * 2 * kLinBN * kLinStride];

    const int xcd = blockIdx.x & 7;
    const int slot = blockIdx.x >> 3;
    const int bn = xcd * tn_per_xcd + slot % tn_per_xcd;
    const int bm = slot / tn_per_xcd;
    if (bm >= tiles_m || bn >= tiles_n) return;
    const long long row0 = (long long)bm * kSplitBM, col0 = (long long)bn * kLinBN;
    const int lane = threadIdx.x & 63;
    const int group = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);
    const int wm = wave >> 1, wn = wave & 1;

    v16i acc[kMT][2];
#pragma unroll
    for (int a = 0; a < kMT; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int c = 0; c < 16; ++c) acc[a][b][c] = 0;

    const int steps = (int)(K / (2 * kLinBK));                      // of this group; at least four
    const long long kb = (long long)group * steps * kLinBK;         // where its half begins
    LinStage<kBits, kAVec> near, far;
    const LinOffsets<kBits, kAVec> offs = lin_offsets<kBits, kAVec>(M, K, N, row0, col0);
    const int8_t *a_base = xq + row0 * K + kb;
    const uint8_t *code_base = pcodes + ((col0 * K + kb) >> 4) * (2 * kBits);
    const uint8_t *flag_base = pflags + ((col0 * K + kb) >> 3);
    auto load = [&](LinStage<kBits, kAVec> &st, int step) {
        const long long k0 = (long long)step * kLinBK;
        lin_load_whole<kBits, kAVec>(st, offs, a_base + k0, code_base + (k0 >> 4) * (2 * kBits), flag_base + (k0 >> 3));
    };
    load(near, 0);
    lin_store<kBits, 2, kDecode, kAVec>(near, sA[group], sB[group], 4);
    load(near, 1);
    __syncthreads();
    const int8_t *a_lane = sA[group] + (wm * 32 * kMT + (lane & 31)) * kLinStride;
    const int8_t *b_lane = sB[group] + (wn * 32 + (lane & 31)) * kLinStride;
    const int swz = lin_swz(lane & 31), half = lane >> 5;
    int kt = 0;
    for (; kt + 3 < steps; kt += 2) {
        load(far, kt + 2);
        lin_step<kBits, 2, kDecode, true>(acc, near, 4, a_lane, b_lane, swz, half, sA[group], sB[group], 0);
        load(near, kt + 3);
        lin_step<kBits, 2, kDecode, true>(acc, far, 4, a_lane, b_lane, swz, half, sA[group], sB[group], 1);
    }
    if (kt + 2 < steps) {
        load(far, kt + 2);
        lin_step<kBits, 2, kDecode, true>(acc, near, 4, a_lane, b_lane, swz, half, sA[group], sB[group], 0);
        near = far;
        ++kt;
    }
    lin_step<kBits, 2, kDecode, true>(acc, near, 4, a_lane, b_lane, swz, half, sA[group], sB[group], kt & 1);
    lin_step<kBits, 2, kDecode, false>(acc, near, 4, a_lane, b_lane, swz, half, sA[group], sB[group], (kt + 1) & 1);

    // the last step's barrier has ended every fragment read, so the buffers are free:
    // group g finishes the rows of its g-th 32-row tile: the other's sums of them come through LDS
    static_assert(kMT == 2 && sizeof(sA) >= 2 * 16 * kLinWG * sizeof(int) && sizeof(sB) >= 2 * 16 * kLinWG * sizeof(int),
                  "one array per group");
    int *mine = reinterpret_cast<int *>(group ? &sB[0][0] : &sA[0][0]);
    const int *theirs = reinterpret_cast<const int *>(group ? &sA[0][0] : &sB[0][0]);
    const int t = lin_thread();
    v16i sum[2];
#pragma unroll
    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            mine[(pl * 16 + r) * kLinWG + t] = group ? acc[0][pl][r] : acc[1][pl][r];
            sum[pl][r] = group ? acc[1][pl][r] : acc[0][pl][r];
        }
    __syncthreads();
#pragma unroll
    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[pl][r] += theirs[(pl * 16 + r) * kLinWG + t];

    const long long n = col0 + wn * 32 + (lane & 31);
    if (n >= N) return;
    const float Lf = (float)((1 << (kBits - 1)) - 1);
    const float pn = p[n], mn = m[n];
    const float s1 = pn / Lf;
    const float width = mn - pn;
    const float s2 = width / Lf;
    const float cst = z_x * wconst[n];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const long long row = row0 + wm * 32 * kMT + group * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        if (row < M) {
            float t1 = s1 * (float)sum[0][r];
            t1 = __builtin_fmaf(s2, (float)sum[1][r], t1);
            y[row * N + n] = __builtin_fmaf(s_x, t1, cst);
        }
    }
}

// -------------------------------------------------------------- few rows
// k_linear_rows: the same sums where the tiles of k_linear would leave the chip
// idle (few rows of activations, or few channels).  Nothing goes through LDS on
// the way in: in the B fragment of a matrix instruction a lane holds 16
// consecutive weights of one channel, i.e. a run of its packed codes, which it
// loads and decodes itself.  The eight wavefronts of a workgroup share 16 or 32
// channels and take every eighth piece of their rows, so that together they read
// whole lines of every row; their integer sums meet in LDS and are added there
// (exact, whatever the split).  One row of the activation tile is all ones: its
// sums are those of the weights themselves, which the offset z_x multiplies, so
// no other pass reads the weights.  Bound by the packed weights' bytes for a few
// rows, then by the decoding, paid again by every tile of rows (80 vector instructions per 16
// weights of a lane in all at 8 rows, b = 4; 218 with three planes at 250 rows, b = 6).
constexpr int kRowWaves = 8;
constexpr int kRowLane = 64;           // weights of a lane per step

// kTile x kTile outputs of one matrix instruction: 16 (64 deep) or 32 (32 deep).
template <int kTile>
struct RowTile {
    static constexpr int kGroups = 64 / kTile;             // groups of lanes along the reduction
    static constexpr int kRun = kRowLane * kGroups;        // weights of a channel per step
    static constexpr int kRegs = kTile * kTile / 64;       // accumulators of a lane
    typedef int Acc __attribute__((ext_vector_type(kRegs)));
    __device__ static inline Acc mfma(const v4i &a, const v4i &b, const Acc &c)
    {
        if constexpr (kTile == 16) return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
    }
    // row of the tile that register r of a lane in group g holds
    __device__ static inline int row(int r, int g) { return kTile == 16 ? g * 4 + r : (r >> 2) * 8 + g * 4 + (r & 3); }
};

template <int kBits>
struct RowStage {
    uint32_t codes[2 * kBits];         // 64 packed codes
    uint32_t flags[2];
};

// Unaligned loads: a run of 16 codes starts 2-byte aligned.
template <int kWords>
__device__ inline void load_words2(uint32_t (&out)[kWords], const uint8_t *__restrict__ src)
{
    struct __attribute__((packed, aligned(2))) Words { uint32_t w[kWords]; };
    const Words v = *reinterpret_cast<const Words *>(src);
#pragma unroll
    for (int i = 0; i < kWords; ++i) out[i] = v.w[i];
}

// Codes and region bits of elements e0 .. e0+63 of the streams.
template <int kBits>
__device__ inline void row_load(RowStage<kBits> &st, const uint8_t *__restrict__ pcodes,
                                const uint8_t *__restrict__ pflags, long long e0)
{
    load_words2<2 * kBits>(st.codes, pcodes + (e0 >> 4) * (2 * kBits));
    load_words2<2>(st.flags, pflags + (e0 >> 3));
}

// The same where only `pieces` runs of 16 exist; the others read as code 0 in the
// centre, which adds nothing.
template <int kBits>
__device__ inline void row_load_part(RowStage<kBits> &st, const uint8_t *__restrict__ pcodes,
                                     const uint8_t *__restrict__ pflags, long long e0, int pieces)
{
    const uint16_t *c = reinterpret_cast<const uint16_t *>(pcodes + (e0 >> 4) * (2 * kBits));
    const uint16_t *f = reinterpret_cast<const uint16_t *>(pflags + (e0 >> 3));
#pragma unroll
    for (int i = 0; i < 2 * kBits; ++i) st.codes[i] = 0;
    st.flags[0] = st.flags[1] = 0;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        if (p < pieces) {
#pragma unroll
            for (int i = 0; i < kBits; ++i) {          // half-words
                const int at = p * kBits + i;
                st.codes[at >> 1] |= (uint32_t)c[at] << (16 * (at & 1));
            }
            st.flags[p >> 1] |= (uint32_t)f[p] << (16 * (p & 1));
        }
    }
}

// 63 rows by 32 channels at 8 bits, y alone: past one workgroup per CU and this K, where the memory they share is what
// they wait for, borrows (us, borrows / look-ups: 1245x4160x448, 280 workgroups, 34.5/35.6; 63x4160x11008, 344, 34.9/37.3;
// but 41x2080x5106, 160, 10.2/9.8; 1245x4160x256, 160, 22.6/21.5; 126x1536x5106, 320, 14.0/14.1).
constexpr int kRows63BorrowsK = 2048;
// 31 rows by 16 channels at 4 bits, three planes: by itself the compiler takes 87 registers, two workgroups per CU.  Past
// those, 80 and three (us, 87 / 80: 24x512x11008, 688 workgroups, 6.5/5.4; 16x2080x8566, 536, 9.6/8.3; but 16x8192x2500, 157, 10.4/11.2).
constexpr int kRows31Waves = 6, kRows31WavesWgs = 512;

// The operand planes of run p (0..3, 16 weights) of a stage.
template <int kBits, int kPlanes, Decode kDecode>
__device__ inline void row_planes(const RowStage<kBits> &st, int p, v4i (&b)[kPlanes])
{
    RawCodes<kBits> raw;
#pragma unroll
    for (int i = 0; i < (2 * kBits + 3) / 4; ++i) {
        const int at = p * kBits + 2 * i;              // in half-words
        uint32_t v = st.codes[at >> 1];
        if (at & 1) {
            v >>= 16;
            if ((at >> 1) + 1 < 2 * kBits) v |= st.codes[(at >> 1) + 1] << 16;
        }
        raw.w[i] = v;
    }
    uint32_t c[4];
    unpack16<kBits>(raw, c);
    const uint32_t f = st.flags[p >> 1] >> (16 * (p & 1));
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        uint32_t w1, w2, w3 = 0;
        // (kBorrows here, not a call further in: the constant has to come after the inlining)
        if constexpr (kDecode == kBorrows && kPlanes == 3) planes4(c[x], f >> (4 * x), kBits, w1, w2, w3);
        else weight_planes<kBits, kPlanes, kDecode>(c[x], f >> (4 * x), w1, w2, w3);
        b[0][x] = (int)w1;
        b[1][x] = (int)w2;
        if (kPlanes == 3) b[kPlanes - 1][x] = (int)w3;
    }
}

// A workgroup's rows: [row0, row0 + rows), rows < kTile kMT; row `rows` of its tile is
// the row of ones.
// kWaves: wavefronts per SIMD that the registers have to leave room for.
template <int kBits, int kPlanes, int kTile, int kMT, Decode kDecode = rows_decode(kBits, kPlanes, kTile, kMT), int kWaves = 1>
__global__ __launch_bounds__(64 * kRowWaves, kWaves) void k_linear_rows(
    const int8_t *__restrict__ xq, long long M, long long K, float s_x, float z_x,
    const uint8_t *__restrict__ pcodes, const uint8_t *__restrict__ pflags, long long N,
    const float *__restrict__ p, const float *__restrict__ m, float *__restrict__ y,
    int *__restrict__ acc_out, int rows_per_tile)
{
    typedef RowTile<kTile> T;
    typedef typename T::Acc Acc;
    __shared__ int row_sums[kPlanes][kTile * kMT][kTile];        // [plane][row][channel]
    constexpr int kSums = kPlanes * kTile * kMT * kTile;
    for (int i = threadIdx.x; i < kSums; i += 64 * kRowWaves) (&row_sums[0][0][0])[i] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = lane / kTile, col = lane % kTile;
    const long long col0 = (long long)blockIdx.x * kTile;
    const long long row0 = (long long)blockIdx.y * rows_per_tile;
    const int rows = (int)(M - row0 < rows_per_tile ? M - row0 : rows_per_tile);

    long long n = col0 + col;
    n = n < N ? n : N - 1;
    const long long e_lane = n * K + group * kRowLane;
    const int8_t *a_lane[kMT];
    bool ones[kMT];
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt) {
        const int r = mt * kTile + col;
        ones[mt] = r == rows;
        a_lane[mt] = xq + (row0 + (r < rows ? r : rows - 1)) * K + group * kRowLane;
    }

    Acc acc[kMT][kPlanes];
#pragma unroll
    for (int a = 0; a < kMT; ++a)
#pragma unroll
        for (int b = 0; b < kPlanes; ++b)
#pragma unroll
            for (int c = 0; c < T::kRegs; ++c) acc[a][b][c] = 0;

    v4i a[kMT][4];
    auto products = [&](const RowStage<kBits> &st, int s) {
        v4i b[kPlanes];
        row_planes<kBits, kPlanes, kDecode>(st, s, b);
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt) {
            v4i x = a[mt][s];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = ones[mt] ? 0x01010101 : x[i];
#pragma unroll
            for (int pl = 0; pl < kPlanes; ++pl) acc[mt][pl] = T::mfma(x, b[pl], acc[mt][pl]);
        }
    };
    auto load_a = [&](long long k0, int s) {
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt) a[mt][s] = *reinterpret_cast<const v4i *>(a_lane[mt] + k0 + s * 16);
    };

    // whole runs; the next run's codes are in flight while this one is decoded, and a
    // fragment of activations is loaded again as soon as it has been used
    const int runs = (int)(K / T::kRun);
    RowStage<kBits> cur, next;
    if (wave < runs) {
        row_load<kBits>(cur, pcodes, pflags, e_lane + (long long)wave * T::kRun);
#pragma unroll
        for (int s = 0; s < 4; ++s) load_a((long long)wave * T::kRun, s);
        for (int run = wave; run < runs; run += kRowWaves) {
            // after the wavefront's last run: that run again, unused
            const long long k1 = (long long)(run + kRowWaves < runs ? run + kRowWaves : run) * T::kRun;
            row_load<kBits>(next, pcodes, pflags, e_lane + k1);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                products(cur, s);
                load_a(k1, s);
            }
            cur = next;
        }
    }
    // what is left of the rows, in runs of 16: the first groups of lanes have four of them
    if (K % T::kRun && wave == runs % kRowWaves) {
        const long long k0 = (long long)runs * T::kRun;
        const int left = (int)((K - k0) / 16) - 4 * group;
        const int pieces = left > 4 ? 4 : left < 0 ? 0 : left;
        row_load_part<kBits>(cur, pcodes, pflags, e_lane + k0, pieces);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            // weights that do not exist are 0: their activations are the row's first
            load_a(s < pieces ? k0 : -(long long)(group * kRowLane + s * 16), s);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) products(cur, s);
    }

    // the wavefronts' sums, rows 0 .. rows (ones) only; whole numbers, so the order is free
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
        for (int r = 0; r < T::kRegs; ++r) {
            const int row = mt * kTile + T::row(r, group);
            if (row <= rows) {
#pragma unroll
                for (int pl = 0; pl < kPlanes; ++pl) atomicAdd(&row_sums[pl][row][col], acc[mt][pl][r]);
            }
        }
    __syncthreads();

    // C2 A1 + C4 A2 + C5 A3 + (C3 + C6), per output channel
    const float Lf = (float)((1 << (kBits - 1)) - 1);
    for (int i = threadIdx.x; i < rows * kTile; i += 64 * kRowWaves) {
        const int row = i / kTile, c = i % kTile;
        const long long nn = col0 + c;
        if (nn >= N) continue;
        const float pn = p[nn], mn = m[nn];
        const float s1 = pn / Lf;
        const float width = mn - pn;
        const float s2 = width / Lf;
        int sum[kPlanes], wsum[kPlanes];
#pragma unroll
        for (int pl = 0; pl < kPlanes; ++pl) {
            sum[pl] = row_sums[pl][row][c];
            wsum[pl] = row_sums[pl][rows][c];
        }
        const float w = lin_constant<kPlanes>(wsum, pn, s1, s2, Lf);
        float t = s1 * (float)sum[0];
        t = __builtin_fmaf(s2, (float)sum[1], t);
        if (kPlanes == 3) t = __builtin_fmaf(pn, (float)sum[kPlanes - 1], t);
        const long long at = (row0 + row) * N + nn;
        y[at] = __builtin_fmaf(s_x, t, z_x * w);
        if (kPlanes == 3 && acc_out) {
#pragma unroll
            for (int pl = 0; pl < kPlanes; ++pl) acc_out[pl * M * N + at] = sum[pl];
        }
    }
}

} // namespace pwlq
