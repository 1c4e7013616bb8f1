// k_linear_wide: the folded form (y alone) of the inner product for calls of many tiles.
//
// What bounds a large call is cycles in which the matrix cores wait, for LDS, decoding, loads and the barrier: they are busy in
// 47 % of them ([4096]^3, b = 4), one workgroup of eight wavefronts to a CU.  The clock is the smaller part: with operands that are
// all zero, which toggle nothing, the same 0.27 million cycles pass at 2.48 instead of 2.23 GHz (110 us instead of 124, counted by
// GRBM_GUI_ACTIVE).  So the tile is large (256 rows by 128 channels, eight wavefronts of 64 x
// 64 outputs), which halves what is read from L2 and decoded per product against
// k_linear's 256 x 64, and the instruction is the 16 x 16 x 64 one, whose 32-bit accumulators are read and
// written half as often per product (random operands, in registers only: 4.1 POP/s against 3.4-3.6 of 32 x 32 x 32).
// Calls back to back, until the chip has its sustained clock, k_linear with k_linear_wsum before it / this kernel, us: [4096]^3, b = 4,
// 153/122 (2.25 POP/s; first calls and calls with others between them 131 to 136), b = 2 151/120, b = 6 172/142, b = 8 159/127;
// 8192 x 4096 x 11008 811/662.  When it was written: with 32 x 32 x 32 130, with the
// weights' sums on the matrix cores 122 where it took 117.  (A library product of the same int8 work, 4096 x 4096 x 8192, takes 121-137 here.)
// Measured and no faster: tiles taken by resident workgroups with the next one's loads in flight across the epilogue, wave
// priorities, other places for the decoding in a step.  With the sums apart (192 rows, 96 KB of
// planes) it gained 9 % at [4096]^3 and lost 2-15 % at two passes over the chip: k_linear keeps those calls.
#pragma once

#include "pwlq_linear.h"

namespace pwlq {

constexpr int kLinWideBN = 128, kLinWideBK = 128;    // channels, reduction elements per step
constexpr int kLinWideWG = 512;                   // 4 (rows) x 2 (channels) wavefronts
constexpr int kLinWideNT = 4;                     // 16-channel tiles of a wavefront
constexpr int kLinWideMT = 4, kLinWideBM = 64 * kLinWideMT;     // 16-row tiles of a wavefront; rows
constexpr int kLinWideMaxTiles = 1 << 22;         // of a launch: indices of tiles are 32-bit numbers

// Weights are decoded by look-ups at every width ([4096]^3, us, borrows / look-ups: b = 2, 136/121, b = 4, 128/119, b = 6,
// 142/137, b = 8, 124/122).

// LDS rows hold 128 reduction bytes as eight 16-byte chunks; chunk c of row r is stored at position
// c ^ lin_wide_swz(r): the sixteen lanes that a cycle of a 16-byte read serves (see lin_swz) then lie in
// different banks, whether they hold one chunk of sixteen rows or two of eight.  The writes of weights do not: eight lanes
// write four chunks of each of two rows with one swizzle, two to a bank (SQ_LDS_BANK_CONFLICT 2^22 at [4096]^3, 16 % of the LDS cycles).
__device__ inline int lin_wide_swz(int row) { return (row >> 1) & 7; }

// What a thread loads for one step: activation rows (t >> 3) + 64 v, chunk t & 7; of channel
// t >> 2 the 32 codes and region bits from element 32 (t & 3) on.
template <int kBits>
struct LinWideStage {
    v4i a[kLinWideMT];
    uint32_t codes[kBits], flags;
};

// Tiles in the order in which the XCDs take them, an eighth each: groups of `cols` channel tiles,
// whose packed weights stay in an L2, walked for one row tile before the next.
struct LinWideTiles {
    int rows, chans, cols;
    __device__ inline void at(int i, int &row, int &chan) const
    {
        const int g = i / (cols * rows), r = i - g * cols * rows;
        const int width = chans - g * cols < cols ? chans - g * cols : cols;
        row = r / width;
        chan = g * cols + r - row * width;
    }
};

template <int kBits>
__global__ __launch_bounds__(kLinWideWG, 2) void k_linear_wide(const int8_t *__restrict__ xq, long long M, long long K,
                                                        float s_x, float z_x, const uint8_t *__restrict__ pcodes,
                                                        const uint8_t *__restrict__ pflags, long long N,
                                                        const float *__restrict__ p, const float *__restrict__ m,
                                                        float *__restrict__ y, LinWideTiles tiles)
{
    constexpr int kABytes = kLinWideBM * kLinWideBK, kPlane = kLinWideBN * kLinWideBK, kBuf = kABytes + 2 * kPlane;
    __shared__ __attribute__((aligned(256))) int8_t lds[2 * kBuf];
    __shared__ float chan_s1[kLinWideBN], chan_s2[kLinWideBN], chan_p[kLinWideBN], chan_cst[kLinWideBN];

    int bm, bn;
    {
        const long long xcd = blockIdx.x & 7, all = (long long)tiles.rows * tiles.chans;
        const int i = (int)(all * xcd / 8) + (int)(blockIdx.x >> 3);
        if (i >= (int)(all * (xcd + 1) / 8)) return;
        tiles.at(i, bm, bn);
    }
    const long long row0 = (long long)bm * kLinWideBM, col0 = (long long)bn * kLinWideBN;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), wm = wave >> 1, wn = wave & 1;

    // K is a multiple of 16: the last step may hold 1 to 7 pieces of 16
    const int whole = (int)(K / kLinWideBK), left = (int)(K % kLinWideBK) / 16;

    // Offsets of a thread's loads from bases that are the same in every lane.  Rows past M and
    // channels past N read the last one.
    unsigned off_a[kLinWideMT];
#pragma unroll
    for (int v = 0; v < kLinWideMT; ++v) {
        long long r = row0 + (t >> 3) + 64 * v;
        r = r < M ? r : M - 1;
        off_a[v] = (unsigned)((r - row0) * K) + (unsigned)((t & 7) * 16);          // < 256 * 2^22 + 128
    }
    long long n0 = col0 + (t >> 2);
    n0 = n0 < N ? n0 : N - 1;
    const unsigned run = (unsigned)((n0 - col0) * (K >> 4)) + 2u * (unsigned)(t & 3);      // in runs of 16 elements
    const unsigned off_c = run * (2 * kBits), off_f = run * 2;
    const int8_t *a_base = xq + row0 * K;
    const uint8_t *code_base = pcodes + ((col0 * K) >> 4) * (2 * kBits);
    const uint8_t *flag_base = pflags + ((col0 * K) >> 3);

    typedef LinWideStage<kBits> Stage;
    auto load = [&](Stage &st, int step) {
        const long long k0 = (long long)step * kLinWideBK;
        const int8_t *a = a_base + k0;
        const uint8_t *c = code_base + (k0 >> 4) * (2 * kBits), *f = flag_base + (k0 >> 3);
#pragma unroll
        for (int v = 0; v < kLinWideMT; ++v) st.a[v] = *reinterpret_cast<const v4i *>(a + off_a[v]);
        load_words2<kBits>(st.codes, c + off_c);
        uint32_t f1[1];
        load_words2<1>(f1, f + off_f);
        st.flags = f1[0];
    };
    // The last step where K ends in it.  Past K activations are 0, weights code 0 in the centre.
    auto load_part = [&](Stage &st) {
        const long long k0 = (long long)whole * kLinWideBK;
        const int8_t *a = a_base + k0;
        const bool in = (t & 7) < left;
        const int keep = in ? -1 : 0;
#pragma unroll
        for (int v = 0; v < kLinWideMT; ++v) {
            v4i x = *reinterpret_cast<const v4i *>(a + off_a[v] - (in ? 0 : (t & 7) * 16));
            x[0] &= keep; x[1] &= keep; x[2] &= keep; x[3] &= keep;
            st.a[v] = x;
        }
        const int runs = left - 2 * (t & 3);                   // of this thread's two
        const uint16_t *c = reinterpret_cast<const uint16_t *>(code_base + (k0 >> 4) * (2 * kBits) + off_c);
        const uint16_t *f = reinterpret_cast<const uint16_t *>(flag_base + (k0 >> 3) + off_f);
#pragma unroll
        for (int i = 0; i < kBits; ++i) st.codes[i] = 0;
        st.flags = 0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (q < runs) {
#pragma unroll
                for (int i = 0; i < kBits; ++i) {              // half-words
                    const int at = q * kBits + i;
                    st.codes[at >> 1] |= (uint32_t)c[at] << (16 * (at & 1));
                }
                st.flags |= (uint32_t)f[q] << (16 * q);
            }
        }
    };

    // where a thread's pieces go in LDS; the sums of its weights in each plane
    const int ra = t >> 3, rb = t >> 2;
    int8_t *to_a = lds + ra * kLinWideBK + (((t & 7) ^ lin_wide_swz(ra)) * 16);           // row ra + 64 v has the same swizzle
    int8_t *to_b[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) to_b[q] = lds + kABytes + rb * kLinWideBK + (((2 * (t & 3) + q) ^ lin_wide_swz(rb)) * 16);
    uint32_t sums[2] = {};
    // The sums by bytes without a sign (a weight plus 2^(b-1)), as many words together as fit: a dot product of bytes, one
    // instruction a word, takes six cycles of the matrix cores ([4096]^3, b = 4: 122 us, 117 so).
    constexpr uint32_t kSumBias = 1u << (kBits - 1);
    constexpr int kSumWords = kBits <= 6 ? 4 : kBits == 7 ? 2 : 1;
    auto store_a = [&](const Stage &st, int buf) {
#pragma unroll
        for (int v = 0; v < kLinWideMT; ++v) *reinterpret_cast<v4i *>(to_a + buf + v * 64 * kLinWideBK) = st.a[v];
    };
    auto store_b = [&](const Stage &st, int buf, int q) {
        RawCodes<kBits> raw;
#pragma unroll
        for (int i = 0; i < (2 * kBits + 3) / 4; ++i) {
            const int at = q * kBits + 2 * i;                  // in half-words
            uint32_t v = st.codes[at >> 1];
            if (at & 1) {
                v >>= 16;
                if ((at >> 1) + 1 < kBits) v |= st.codes[(at >> 1) + 1] << 16;
            }
            raw.w[i] = v;
        }
        uint32_t c[4];
        unpack16<kBits>(raw, c);
        v4i w[2];
        uint32_t bytes[2];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            uint32_t u[3];
            weight_planes<kBits, 2, kLookUps>(c[x], st.flags >> (16 * q + 4 * x), u[0], u[1], u[2]);
#pragma unroll
            for (int pl = 0; pl < 2; ++pl) {
                w[pl][x] = (int)u[pl];
                const uint32_t up = (u[pl] & (2 * kSumBias - 1) * 0x01010101u) ^ kSumBias * 0x01010101u;
                bytes[pl] = x % kSumWords ? bytes[pl] + up : up;
                if (x % kSumWords == kSumWords - 1) sums[pl] = __builtin_amdgcn_sad_u8(bytes[pl], 0u, sums[pl]);
            }
        }
#pragma unroll
        for (int pl = 0; pl < 2; ++pl) *reinterpret_cast<v4i *>(to_b[q] + buf + pl * kPlane) = w[pl];
    };

    // fragments: lane = row or channel (16), a piece of 16 for each of four groups of lanes; half a step per instruction
    const int fr = lane & 15, quarter = lane >> 4, swz = lin_wide_swz(fr);
    const int8_t *a_lane = lds + (wm * 16 * kLinWideMT + fr) * kLinWideBK;
    const int8_t *b_lane = lds + kABytes + (wn * 16 * kLinWideNT + fr) * kLinWideBK;
    v4i fa[2][kLinWideMT], fb[2][2];
    auto frag_a = [&](int half, int mt, int buf) {
        fa[half][mt] = *reinterpret_cast<const v4i *>(a_lane + ((4 * half + quarter) ^ swz) * 16 + buf + mt * 16 * kLinWideBK);
    };
    auto frag_b = [&](int half, int nt, int buf) {
#pragma unroll
        for (int pl = 0; pl < 2; ++pl)
            fb[nt & 1][pl] = *reinterpret_cast<const v4i *>(b_lane + ((4 * half + quarter) ^ swz) * 16 + buf + pl * kPlane +
                                                            nt * 16 * kLinWideBK);
    };
    v4i acc[kLinWideMT][kLinWideNT][2];
#pragma unroll
    for (int a = 0; a < kLinWideMT; ++a)
#pragma unroll
        for (int b = 0; b < kLinWideNT; ++b)
#pragma unroll
            for (int pl = 0; pl < 2; ++pl) acc[a][b][pl] = v4i{0, 0, 0, 0};

    auto products = [&](int half, int nt) {
#pragma unroll
        for (int mt = 0; mt < kLinWideMT; ++mt)
#pragma unroll
            for (int pl = 0; pl < 2; ++pl)
                acc[mt][nt][pl] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[nt & 1][pl], fa[half][mt], acc[mt][nt][pl], 0, 0, 0);
    };

    int buf = 0;
    Stage st;
    {
        Stage first;
        if (whole) {
            load(first, 0);
            load(st, whole > 1 ? 1 : 0);
        } else
            load_part(first);
        store_a(first, 0);
        store_b(first, 0, 0);
        store_b(first, 0, 1);
    }
    if (t < kLinWideBN) {                                         // the channels' parameters
        long long n = col0 + t;
        n = n < N ? n : N - 1;
        const float Lf = (float)((1 << (kBits - 1)) - 1);
        const float pn = p[n], width = m[n] - pn;
        chan_p[t] = pn;
        chan_s1[t] = pn / Lf;
        chan_s2[t] = width / Lf;
    }
    __syncthreads();
    // One step: the stage (the next step) is decoded into the other buffer and loaded again (the step after) while the
    // matrix cores work on this one, sixteen channels and half of the step at a time.  The one barrier
    // stands before the last of these products; the next step's first fragments are read behind it.
    // The last whole step is loaded again where there is no step after: not used.
    if (whole > 1) {
#pragma unroll
        for (int mt = 0; mt < kLinWideMT; ++mt) frag_a(0, mt, 0);
        frag_b(0, 0, 0);
    }
    for (int s = 2; s <= whole; ++s) {
#pragma unroll
        for (int part = 0; part < 2 * kLinWideNT; ++part) {
            if (part == 2 * kLinWideNT - 1) {
                __builtin_amdgcn_sched_barrier(0);
                __syncthreads();
                buf = kBuf - buf;
#pragma unroll
                for (int mt = 0; mt < kLinWideMT; ++mt) frag_a(0, mt, buf);
                frag_b(0, 0, buf);
            } else {
                frag_b((part + 1) / kLinWideNT, (part + 1) % kLinWideNT, buf);
                if (part < kLinWideMT) frag_a(1, part, buf);
            }
            if (part == 0) store_b(st, kBuf - buf, 0);
            if (part == 2) store_b(st, kBuf - buf, 1);
            if (part == kLinWideNT) {
                store_a(st, kBuf - buf);
                load(st, s < whole ? s : whole - 1);
            }
            products(part / kLinWideNT, part % kLinWideNT);
        }
    }
    // the last whole step, and what is left of K
    bool more = whole && left;
    if (more) load_part(st);
    for (;;) {
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int nt = 0; nt < kLinWideNT; ++nt) {
                if (nt == 0) {
#pragma unroll
                    for (int mt = 0; mt < kLinWideMT; ++mt) frag_a(half, mt, buf);
                }
                frag_b(half, nt, buf);
                products(half, nt);
            }
        if (!more) break;
        more = false;
        store_a(st, kBuf - buf);
        store_b(st, kBuf - buf, 0);
        store_b(st, kBuf - buf, 1);
        buf = kBuf - buf;
        __syncthreads();
    }

    // the channels' constants; a channel's weights are summed in four threads
    int total[2];
#pragma unroll
    for (int pl = 0; pl < 2; ++pl) {
        total[pl] = (int)sums[pl] - (int)kSumBias * 32 * (whole + (left ? 1 : 0));
        total[pl] += __shfl_xor(total[pl], 1, 64);
        total[pl] += __shfl_xor(total[pl], 2, 64);
    }
    if ((t & 3) == 0) {
        const float Lf = (float)((1 << (kBits - 1)) - 1);
        chan_cst[rb] = z_x * lin_constant<2>(total, chan_p[rb], chan_s1[rb], chan_s2[rb], Lf);
    }
    __syncthreads();

    // A lane holds four channels of one row per tile, 64 bytes of a line per instruction: the
    // wavefront's outputs go through LDS instead (its part of the buffers, which are free) and out in whole
    // lines.  16-byte chunk c of row r is at c ^ (r & 15).  Only this wavefront reads what it writes.
    float *mine = reinterpret_cast<float *>(lds) + wave * (16 * kLinWideMT * 64);
    const long long rw = row0 + wm * 16 * kLinWideMT, nw = col0 + wn * 64;
#pragma unroll
    for (int nt = 0; nt < kLinWideNT; ++nt) {
        float s1[4], s2[4], cst[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = wn * 64 + nt * 16 + quarter * 4 + r;
            s1[r] = chan_s1[c];
            s2[r] = chan_s2[c];
            cst[r] = chan_cst[c];
        }
        auto value = [&](int mt, int r) {
            float v = s1[r] * (float)acc[mt][nt][0][r];        // acc[..][0] = A1 + L A3
            v = __builtin_fmaf(s2[r], (float)acc[mt][nt][1][r], v);
            return __builtin_fmaf(s_x, v, cst[r]);
        };
#pragma unroll
        for (int mt = 0; mt < kLinWideMT; ++mt)
            *reinterpret_cast<float4 *>(mine + (mt * 16 + fr) * 64 + ((nt * 4 + quarter) ^ fr) * 4) =
                make_float4(value(mt, 0), value(mt, 1), value(mt, 2), value(mt, 3));
    }
    if ((N & 3) == 0 && ((uintptr_t)y & 15) == 0) {
        const long long n = nw + fr * 4;
#pragma unroll
        for (int i = 0; i < 4 * kLinWideMT; ++i) {
            const int r = i * 4 + quarter;
            const float4 o = *reinterpret_cast<const float4 *>(mine + r * 64 + (fr ^ (r & 15)) * 4);
            if (rw + r < M && n < N) *reinterpret_cast<float4 *>(y + (rw + r) * N + n) = o;
        }
    } else {
        const long long n = nw + lane;
#pragma unroll 16
        for (int r = 0; r < 16 * kLinWideMT; ++r) {
            const float o = mine[r * 64 + ((lane >> 2) ^ (r & 15)) * 4 + (lane & 3)];
            if (rw + r < M && n < N) y[(rw + r) * N + n] = o;
        }
    }
}

} // namespace pwlq
