// Implicit-GEMM convolution for the deep layers (bf16, 3x3x3; v_mfma_f32_32x32x16_bf16, fp32 accumulation): stride-1
// forward and data gradient on volumes too small to fill the chip with planes, stride-2 forward with more than 32 input channels,
// stride-2 data gradient with more than 64 output channels, and channel counts in multiples of 8 that 32 does not divide.
//
// One product: out[m, j] = sum over taps t and contracted channels c of w[m, t, c] * in[is j + delta_t, c].  Positions j are
// numbered through all samples, so a tile of positions is full whatever the extents of the volume (the plane-streaming
// kernels cover a 12 x 12 plane with a 12 x 32 patch).  The stride-2 data gradient is eight such products, one per parity
// class of the output voxel, each with the 1, 2, 4 or 8 taps that hit it.  Where the tiles leave CUs idle the steps of the
// contraction are split and fp32 partial sums are added in index order by ig_sum_kernel.
//
// A workgroup (4 waves, two workgroups per CU) owns 128 m x 128 j (or 64 x 256, 32 x 256), a wave 64 x 64; a step contracts 64
// channels of one tap: rows of 128 bytes of weights and activations are fetched with direct-to-LDS loads (the range check
// of the buffer supplies the zero padding), double buffered.  The piece a lane fetches is permuted inside its row so
// that the 16-byte fragment reads of neighbouring rows fall into different banks.
//
// Bound: 1 KB of fragment reads per MFMA is what the LDS delivers at 64 % of the MFMA rate; on the smallest volumes the
// weights' way from HBM and the launches.  Forward / data gradient with their packing and summing launches, former
// chunked kernels -> this one: 128->256 at 48^3, stride 2, N = 2 112 / 301 -> 62 / 70 us (794 / 698 TFLOP/s), 64->128 at
// 96^3, stride 2, N = 2 260 / 551 -> 142 / 204, 320->320 at 12^3 74 / 74 -> 30 / 30, 256->256 at 24^3 101 / 101 -> 69 / 69.
// Measured and left out: a ring of 32-channel steps (rows of 64 bytes; 48^3 60 -> 67, 12^3 30 -> 35), deeper rings, fragments read a
// product ahead, and 128 x 256 tiles on eight waves (no change): fragment reads and the loads' way into LDS are the bound.
#include <cstdio>

#include "ig_common.h"
#include "mi3d_internal.h"

namespace mi3d {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef unsigned u32x2 __attribute__((__vector_size__(2 * sizeof(unsigned))));
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr unsigned OOB = 0x80000000u;   // buffer offset of a piece that must read as zero
constexpr int BK = 64;                  // contracted channels of a step

struct IgClass {      // one product: a parity class of the output voxels (stride-2 data gradient) or everything
    Div jD, jH, jW;   // extents of the position space of a sample
    int J, PT, tile0; // positions of all samples, tiles of them, first tile in the grid
    int od0, oh0, ow0;
    int tap0, ntap;
};
struct IgParams {
    const uint16_t *in, *in_hi;   // two halves along the channels (virtual concatenation), or the tensor and itself
    const uint16_t* w;            // [M][T][C]
    uint16_t *out, *out_hi;
    const uint16_t *add, *ref;    // optional operands of the epilogue, of the output's shape
    float* part;                  // [split][voxel][M] fp32 partial sums, or null: the kernel finishes the output itself
    float slope;
    int C, csplit, pitch, M;      // contracted channels, first of those in in_hi, channels per voxel of in / in_hi; output channels
    int T, is, os;                // taps of a weight row; strides of the input and the output per position
    int iD, iH, iW, oD, oH, oW;
    int MT, splits, ncls, tiles;
    long long in_bytes;           // of one of in / in_hi
    long long out_elems;
    IgClass cls[8];
    Div Cdiv;                     // contracted channels
    uint32_t taps[27];
    long long slack;              // voxels by which a position can lie before an earlier one of its tile (max_span)
};

// the bytes of a tensor from byte `at` on (before it or behind its end too), 2^31 at most
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_from(const uint16_t* p, long long at, long long bytes) {
    const long long left = bytes - at;
    return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p + at), 0, left > 0x7fffffffll ? 0x7fffffff : left < 0 ? 0 : (int)left, 0x00020000);
}
// 16 bytes per lane from buffer r at byte offset off (zeros beyond its range) to the wave's 1 KB at l
__device__ __forceinline__ void load_lds(__amdgpu_buffer_rsrc_t r, char* l, unsigned off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)l, 16, (int)off, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ uint32_t cvt2(float a, float b) {
    typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
    f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float lo_f(uint32_t v) { return __builtin_bit_cast(float, v << 16); }
__device__ __forceinline__ float hi_f(uint32_t v) { return __builtin_bit_cast(float, v & 0xFFFF0000u); }

// WN = waves along the positions, MA = blocks of 32 channels of a wave: 2, 2 (128 x 128), 4, 2 (64 x 256) or 4, 1 (32 x 256).
// TR: the weights are read as they are, w[contracted][T][M] (the data gradient's): rows of the tile's channels per contracted one,
// which the fragments are read from transposed (ds_read_b64_tr_b16).  FLAT: the contraction runs over (tap, channel) pairs, 64 of them per step whatever the number of channels; without it a step is
// 64 channels of one tap, which is the same where the channels come in multiples of 64.  WIDE: planes too large for 32-bit offsets from a plane to
// all that a tile and its taps touch (narrow_planes); the buffers move with the tap then, which costs 2 % (48^3 128->256,
// stride 2, N = 2: 225 -> 231 us for the three passes).
template <int WN, int MA, bool WIDE, bool FLAT, bool TR = false>
__global__ void __launch_bounds__(256, 2) ig_kernel(const IgParams P) {
    static_assert(!(WIDE && FLAT) && !(TR && (WIDE || FLAT)), "");
    constexpr int BM = 128 / WN * MA, BN = 64 * WN, NA = BM / 32, NB = BN / 32;
    constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);

    // block -> (split, class, tile of positions, tile of channels); the blocks of an XCD (every eighth) get neighbouring
    // tiles of a class, channels fastest, so that they share the positions' rows and the weights of a split in its L2
    int id = blockIdx.x;
    const int split = id / P.tiles;
    id -= split * P.tiles;
    int ci = 0;
    while (ci + 1 < P.ncls && id >= P.cls[ci + 1].tile0) ++ci;
    const IgClass& K = P.cls[ci];
    {
        const int n = K.PT * P.MT, l = id - K.tile0, x = l & 7, q = l >> 3;
        id = x * (n >> 3) + ((n & 7) < x ? (n & 7) : x) + q;
    }
    const int pt = id / P.MT, mt = id - pt * P.MT;

    auto decode = [&](int j, int& n, int& d, int& h, int& w) {
        int r = divide(j, K.jW);
        w = j - r * (int)K.jW.d;
        int r2 = divide(r, K.jH);
        h = r - r2 * (int)K.jH.d;
        n = divide(r2, K.jD);
        d = r2 - n * (int)K.jD.d;
    };

    // the rows this thread fetches: row 32 i + 8 wave + lane / 8 of either operand, the same 8-channel piece of each
    const int rl = 8 * wave + (lane >> 3), piece = (lane & 7) ^ (lane >> 3) ^ (wave & 1);
    // 32-bit offsets are relative to the plane two below the first position's (a tile spans few planes).  WIDE: to the first
    // position's own voxel, and a tap moves the buffer (its voxel may lie before or behind the tensor: lanes that would
    // read there are masked).
    long long base;
    {
        int n, d, h, w;
        decode(pt * BN, n, d, h, w);
        if (WIDE) {
            base = (((long long)n * P.iD + P.is * d) * P.iH + P.is * h) * P.iW + P.is * w - P.slack;
        } else {
            const long long v = ((long long)n * P.iD + P.is * d - 2) * P.iH * P.iW;
            base = v > 0 ? v : 0;
        }
    }
    const int nch = (P.C + BK - 1) / BK, steps = FLAT ? (K.ntap * P.C + BK - 1) / BK : K.ntap * nch;
    const int s0 = (int)((unsigned)(steps * split) / (unsigned)P.splits), s1 = (int)((unsigned)(steps * (split + 1)) / (unsigned)P.splits);
    int tap = s0 / nch, chunk = s0 - tap * nch;   // of the next step to be fetched
    // lane k keeps tap k: reading it from there costs no memory latency between two steps
    const int tapv = lane < K.ntap ? (int)P.taps[K.tap0 + lane] : 0;
    int rowb[NB];
    uint32_t mask[NB];   // bit k: tap k of this split's steps reads inside the volume
    {
        int dd[NB], hh[NB], ww[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int j = pt * BN + 32 * i + rl;
            int n, d, h, w;
            decode(j, n, d, h, w);
            d *= P.is; h *= P.is; w *= P.is;
            rowb[i] = (int)(((((long long)n * P.iD + d) * P.iH + h) * P.iW + w - base) * P.pitch * 2) + piece * 16;
            mask[i] = 0;
            dd[i] = j < K.J ? d : -1000000; hh[i] = h; ww[i] = w;
        }
        for (int k = FLAT ? 0 : tap; FLAT ? k < K.ntap : k * nch < s1; ++k) {
            const IgTap a(__builtin_amdgcn_readlane(tapv, k));
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const bool ok = ((unsigned)(dd[i] + a.dd) < (unsigned)P.iD) & ((unsigned)(hh[i] + a.dh) < (unsigned)P.iH) & ((unsigned)(ww[i] + a.dw) < (unsigned)P.iW);
                mask[i] |= (ok ? 1u : 0u) << k;
            }
        }
    }
    // TR: this lane's row (contracted channel) and piece of it; all its rows are a multiple of four apart and permuted alike
    constexpr int RA = BM * 2, LA = 64 / (RA / 16);
    auto swz_a = [](int row) { return RA == 256 ? 4 * (row & 3) : RA == 128 ? 2 * (row & 2) : 0; };
    const int ra = wave * LA + lane / (RA / 16), ma = mt * BM + 8 * (lane % (RA / 16) ^ swz_a(ra));
    const unsigned row_w = (unsigned)(P.T * P.M) * 2, offa = ma < P.M ? (unsigned)ra * row_w + (unsigned)ma * 2 : OOB;
    int rowa[NA];
    unsigned oka[NA];
#pragma unroll
    for (int i = 0; i < NA && !TR; ++i) {
        const int m = mt * BM + 32 * i + rl;
        oka[i] = m < P.M;
        rowa[i] = m * P.T * P.C * 2 + piece * 16;
    }
    const long long base_b = base * P.pitch * 2, left = P.in_bytes - base_b;
    const int range = left > 0x7fffffffll ? 0x7fffffff : (int)left;
    __amdgpu_buffer_rsrc_t r_in = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)P.in + base_b), 0, range, 0x00020000);
    __amdgpu_buffer_rsrc_t r_hi = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)P.in_hi + base_b), 0, range, 0x00020000);
    __amdgpu_buffer_rsrc_t r_w = __builtin_amdgcn_make_buffer_rsrc((void*)P.w, 0, P.M * P.T * P.C * 2, 0x00020000);

    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_ptr)lds);
    auto fetch_flat = [&](int buf, int s) {
        const int k = s * BK + piece * 8, tp = divide(k, P.Cdiv), c = k - tp * P.C;   // this lane's tap and channels
        const bool in = tp < K.ntap;
        const IgTap a((uint32_t)__shfl(tapv, tp & 31));
        const int ua = (a.wt * P.C + c) * 2 - piece * 16, ub = (((a.dd * P.iH + a.dh) * P.iW + a.dw) * P.pitch + c) * 2 - piece * 16;
        const uint32_t bit = in ? 1u << (tp & 31) : 0u;
        char* l = lds + buf * STAGE + wave * 1024;
#pragma unroll
        for (int i = 0; i < NA; ++i) load_lds(r_w, l + i * 4096, oka[i] & (in ? 1u : 0u) ? rowa[i] + ua : OOB);
        l += A_BYTES;
#pragma unroll
        for (int i = 0; i < NB; ++i) load_lds(r_in, l + i * 4096, mask[i] & bit ? rowb[i] + ub : OOB);
    };
    auto fetch = [&](int buf, int s) {
        if constexpr (FLAT) return fetch_flat(buf, s);
        const IgTap a(__builtin_amdgcn_readlane(tapv, tap));
        const int c = chunk * BK + piece * 8;     // this lane's channels
        const unsigned okc = c < P.C;
        int ub = 0;
        if (WIDE) {
            const long long at = (base + (a.dd * P.iH + a.dh) * P.iW + a.dw) * P.pitch * 2 + chunk * (BK * 2);
            r_in = buffer_from(P.in, at, P.in_bytes);
            r_hi = buffer_from(P.in_hi, at - P.csplit * 2, P.in_bytes);
        } else {
            ub = ((a.dd * P.iH + a.dh) * P.iW + a.dw) * P.pitch * 2 + chunk * BK * 2;
        }
        const int ua = (a.wt * P.C + chunk * BK) * 2;
        char* l = lds + buf * STAGE + wave * 1024;
        const unsigned la = lds0 + buf * STAGE + wave * 1024;
        auto to_lds = [&](__amdgpu_buffer_rsrc_t r, int at, unsigned off) {
            if constexpr (TR) load_lds_asm(r, la + at, off);
            else load_lds(r, l + at, off);
        };
        if constexpr (TR) {   // (contracted channels behind the last one lie behind the end of w)
            const unsigned u = (unsigned)(chunk * BK) * row_w + (unsigned)(a.wt * P.M) * 2;
#pragma unroll
            for (int i = 0; i < NA; ++i) to_lds(r_w, i * 4096, offa == OOB ? OOB : offa + u + (unsigned)(i * 4 * LA) * row_w);
        } else {
#pragma unroll
            for (int i = 0; i < NA; ++i) to_lds(r_w, i * 4096, oka[i] & okc ? rowa[i] + ua : OOB);
        }
        // (a step may begin in one half of a virtual concatenation and end in the other: inactive lanes write nothing)
        if (c < P.csplit) {
#pragma unroll
            for (int i = 0; i < NB; ++i) to_lds(r_in, A_BYTES + i * 4096, okc & (mask[i] >> tap) ? rowb[i] + ub : OOB);
            asm volatile("; low half");   // keeps the branches apart: merged, their last loads run in a loop over the resources
        } else {
#pragma unroll
            for (int i = 0; i < NB; ++i) to_lds(r_hi, A_BYTES + i * 4096, okc & (mask[i] >> tap) ? rowb[i] + ub - (WIDE ? 0 : P.csplit * 2) : OOB);
        }
        if (++chunk == nch) { chunk = 0; ++tap; }
    };

    f32x16 acc[MA][2];
#pragma unroll
    for (int a = 0; a < MA; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

    const int r32 = lane & 31, half = lane >> 5, swz = (r32 & 7) ^ (r32 >> 3 & 1);
    const int wm = WN == 2 ? wave >> 1 : 0, wn = WN == 2 ? wave & 1 : wave;
    int frag[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) frag[k] = r32 * 128 + ((2 * k + half) ^ swz) * 16;
    // TR: a group of 16 lanes reads four rows of 16 channels; groups 0, 1 rows 0 .. 7 of channels 0 .. 15 and 16 .. 31 of a block of 32,
    // groups 2, 3 rows 8 .. 15
    int fraga[MA];
    if constexpr (TR) {
        const int g = lane >> 4, row = 8 * (g >> 1) + (lane >> 2 & 3), c8 = lane & 3;
#pragma unroll
        for (int a = 0; a < MA; ++a) {
            const int at = (wm * 64 + 32 * a + 16 * (g & 1)) / 8 + (c8 >> 1);
            fraga[a] = row * RA + (at ^ swz_a(row)) * 16 + (c8 & 1) * 8;
        }
    }

    if (s0 < s1) {
        fetch(0, s0);
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        for (int s = s0; s < s1; ++s) {
            const int buf = (s - s0) & 1;
            if (s + 1 < s1) fetch(1 - buf, s + 1);
            const char* la = lds + buf * STAGE + (TR ? 0 : wm * 64 * 128);
            const char* lb = lds + buf * STAGE + A_BYTES + wn * 64 * 128;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                bf16x8 fa[MA], fb[2];
#pragma unroll
                for (int a = 0; a < MA; ++a) fa[a] = TR ? tr_frag(la + fraga[a] + k * 16 * RA, RA) : *(const bf16x8*)(la + a * 4096 + frag[k]);
#pragma unroll
                for (int b = 0; b < 2; ++b) fb[b] = *(const bf16x8*)(lb + b * 4096 + frag[k]);
#pragma unroll
                for (int a = 0; a < MA; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) acc[a][b] = mfma(fa[a], fb[b], acc[a][b]);
            }
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
    }

    // lane (voxel r32, half): register 4 g + i of a block is channel 8 g + 4 half + i of its 32
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int j = pt * BN + wn * 64 + b * 32 + r32;
        if (j >= K.J) continue;
        int n, d, h, w;
        decode(j, n, d, h, w);
        const long long vox = (((long long)n * P.oD + P.os * d + K.od0) * P.oH + P.os * h + K.oh0) * P.oW + P.os * w + K.ow0;
#pragma unroll
        for (int a = 0; a < MA; ++a) {
            const int m0 = mt * BM + wm * 64 + a * 32;
            if (m0 >= P.M) continue;
            const int groups = (P.M - m0 - 4 * half + 7) >> 3;     // (channels in fours: a last block may end early)
            if (P.part) {
                float* p = P.part + (long long)split * P.out_elems + vox * P.M + m0 + 4 * half;
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    if (g < groups) *(float4*)(p + 8 * g) = float4{acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2], acc[a][b][4 * g + 3]};
                continue;
            }
            const long long e = vox * P.M + m0 + 4 * half;
            const bool high = P.out_hi && m0 >= (P.M >> 1);
            uint16_t* o = P.out_hi ? (high ? P.out_hi - (P.M >> 1) : P.out) + vox * (P.M >> 1) + m0 + 4 * half : P.out + e;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (g >= groups) break;
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = acc[a][b][4 * g + i];
                if (P.add) {   // the stored (rounded) result of the plain pass plus the second gradient
                    const uint2 q = *(const uint2*)(P.add + e + 8 * g);
                    const uint32_t x = cvt2(v[0], v[1]), y = cvt2(v[2], v[3]);
                    v[0] = lo_f(x) + lo_f(q.x); v[1] = hi_f(x) + hi_f(q.x);
                    v[2] = lo_f(y) + lo_f(q.y); v[3] = hi_f(y) + hi_f(q.y);
                }
                if (P.ref) {
                    const uint2 q = *(const uint2*)(P.ref + e + 8 * g);
                    if (!((int)(q.x << 16) > 0)) v[0] *= P.slope;
                    if (!((int)(q.x & 0xFFFF0000u) > 0)) v[1] *= P.slope;
                    if (!((int)(q.y << 16) > 0)) v[2] *= P.slope;
                    if (!((int)(q.y & 0xFFFF0000u) > 0)) v[3] *= P.slope;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], P.slope * v[i]);
                }
                *(uint2*)(o + 8 * g) = uint2{cvt2(v[0], v[1]), cvt2(v[2], v[3])};
            }
        }
    }
}

// wt[ci][tap][co] = w[co][tap][ci]: the data gradient's weights with the contracted channels contiguous.  64 x 64 blocks
// through LDS, 16-byte accesses on both sides; block (tap, ci block, co block).  flags (null: none): one word per block, 1 where it
// met an infinity or a NaN.
__device__ __forceinline__ bool odd_bf16(uint32_t v) { return (v & 0x7F80u) == 0x7F80u || (v & 0x7F800000u) == 0x7F800000u; }
__global__ void __launch_bounds__(256) ig_transpose_kernel(const uint16_t* __restrict__ w, uint16_t* __restrict__ wt, int T, int Cin, int Cout,
                                                           uint32_t* __restrict__ flags) {
    __shared__ uint16_t tile[64][72];
    const int tap = blockIdx.x, ci0 = blockIdx.y * 64, co0 = blockIdx.z * 64, t = threadIdx.x;
    bool odd = false;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = (t >> 3) + 32 * i, c = (t & 7) * 8;
        if (co0 + r < Cout && ci0 + c < Cin) {
            const uint4 v = *(const uint4*)(w + ((long long)(co0 + r) * T + tap) * Cin + ci0 + c);
            *(uint4*)&tile[r][c] = v;
            odd = odd || odd_bf16(v.x) || odd_bf16(v.y) || odd_bf16(v.z) || odd_bf16(v.w);
        }
    }
    const int any = __syncthreads_or(odd);
    if (flags && t == 0) flags[tap + T * (blockIdx.y + gridDim.y * blockIdx.z)] = any ? 1u : 0u;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        // lanes run over ci, so that the column reads of a wave are 2 bytes apart
        const int r = t & 63, c = ((t >> 6) + 4 * i) * 8;
        if (ci0 + r < Cin && co0 + c < Cout) {
            uint32_t o[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = tile[c + 2 * j][r] | (uint32_t)tile[c + 2 * j + 1][r] << 16;
            *(uint4*)(wt + ((long long)(ci0 + r) * T + tap) * Cout + co0 + c) = uint4{o[0], o[1], o[2], o[3]};
        }
    }
}

// y = bf16(act(sum over chunks of part[chunk])), chunks added in index order; 8 outputs per thread.
// act: LeakyReLU with `slope` (1 = none) if ref is null; otherwise the factor of element i is 1 where
// ref[i] > 0 and `slope` elsewhere (LeakyReLU derivative taken from the activated tensor ref).
__global__ void __launch_bounds__(256) ig_sum_kernel(const float* __restrict__ part, uint16_t* __restrict__ y, long long n8, long long n, int nch,
                                                              float slope, const uint16_t* __restrict__ ref, uint16_t* __restrict__ y_hi, int cout,
                                                              const uint16_t* __restrict__ add) {
    typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2_;
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n8; i += (long long)gridDim.x * 256) {
        float a[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] = 0.f;
#pragma unroll 4
        for (int c = 0; c < nch; ++c) {
            const float4 lo = *(const float4*)(part + c * n + 8 * i), hi = *(const float4*)(part + c * n + 8 * i + 4);
            a[0] += lo.x; a[1] += lo.y; a[2] += lo.z; a[3] += lo.w; a[4] += hi.x; a[5] += hi.y; a[6] += hi.z; a[7] += hi.w;
        }
        if (add) {   // skip connection: the sum as the plain pass would store it (bf16), plus the second gradient
            const uint4 a4 = *(const uint4*)(add + 8 * i);
            const uint32_t aw[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x2_ v = {a[2 * j], a[2 * j + 1]};
                const uint32_t r = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_));
                a[2 * j] = __builtin_bit_cast(float, r << 16) + __builtin_bit_cast(float, aw[j] << 16);
                a[2 * j + 1] = __builtin_bit_cast(float, r & 0xFFFF0000u) + __builtin_bit_cast(float, aw[j] & 0xFFFF0000u);
            }
        }
        if (ref) {
            const uint4 m4 = *(const uint4*)(ref + 8 * i);
            const uint32_t m[4] = {m4.x, m4.y, m4.z, m4.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!((int)(m[j] << 16) > 0)) a[2 * j] *= slope;
                if (!((int)(m[j] & 0xFFFF0000u) > 0)) a[2 * j + 1] *= slope;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) a[j] = fmaxf(a[j], slope * a[j]);
        }
        uint32_t o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f32x2_ v = {a[2 * j], a[2 * j + 1]};
            o[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_));
        }
        uint16_t* dst = y + 8 * i;
        if (y_hi) {   // output in two halves of cout / 2 channels per voxel
            const long long vox = 8 * i / cout;
            const int c = (int)(8 * i - vox * cout), half = cout >> 1;
            dst = (c >= half ? y_hi - half : y) + vox * half + c;
        }
        *(uint4*)dst = uint4{o[0], o[1], o[2], o[3]};
    }
}

// Tile shape and splits of the contraction, by a model of the time: a round of two workgroups per CU takes STEP_US per
// step, partial sums are written and read at PART_BYTES_PER_US.
struct IgPlan {
    int v, splits, MT, ncls, tiles;   // v: 0 128 x 128, 1 64 x 256, 2 32 x 256
    size_t out_elems;
};
constexpr int BMS[3] = {128, 64, 32}, BNS[3] = {128, 256, 256};
constexpr double STEP_US[3] = {0.75, 0.75, 0.5}, START_US = 3.0, PART_BYTES_PER_US = 3e6;

size_t weight_bytes(const Geom& g) { return ((size_t)g.w_elems() * 2 + 255) & ~(size_t)255; }

// The planes that a tile of 256 positions and its taps touch, with room to spare, within 2 GiB
bool narrow_planes(const Geom& g, int pass) {
    const bool flip = pass == MI3D_PASS_DGRAD;
    const long long plane = flip ? (long long)g.Ho * g.Wo * g.Cout * 2 : (long long)g.H * g.W * g.Cin * 2;
    const int os = flip ? g.sD : 1;
    const long long rows = flip ? (long long)(g.H > 1 ? g.H / os : 1) * (g.W > 1 ? g.W / os : 1) : (long long)g.Ho * g.Wo;
    return plane * (16 + 6 * (255 / rows + 2)) < (1ll << 31);
}

// Steps of (tap, channel) pairs: where steps of 64 channels would be partly empty.  48->48 at 37 x 50 x 61: 27 steps -> 21,
// 16 channels: 27 -> 7.  (Not for the classes of a strided data gradient with channels in multiples of 32, 96 and more: a quarter
// at most.)
bool is_flat(const Geom& g, int pass) {
    const int C = pass == MI3D_PASS_DGRAD ? g.Cout : g.Cin;
    return C % BK != 0 && (C % 32 != 0 || g.sD == 1) && narrow_planes(g, pass);   // (halves of an input come in 32s: C is a multiple of 64)
}

// Weights of the data gradient read as they are (TR) rather than from a transposed copy.  Ragged channels keep the copy: their
// repair of non-finite weights takes its flags from it.
bool reads_tr(const Geom& g, int pass) {
    return pass == MI3D_PASS_DGRAD && g.Cin % 32 == 0 && g.Cout % 32 == 0 && narrow_planes(g, pass) && !is_flat(g, pass);
}
size_t copy_bytes(const Geom& g, int pass) { return pass == MI3D_PASS_DGRAD && !reads_tr(g, pass) ? weight_bytes(g) : 0; }

// Tiles of all classes for tiles of bm x bn, the steps of all of them, and of the longest
long long count_tiles(const Geom& g, int pass, int bm, int bn, long long* work, int* most) {
    const bool flip = pass == MI3D_PASS_DGRAD, classes = flip && g.sD == 2;
    const int M = flip ? g.Cin : g.Cout, C = flip ? g.Cout : g.Cin, nch = (C + BK - 1) / BK, MT = (M + bm - 1) / bm;
    const bool flat = is_flat(g, pass);
    long long tiles = 0;
    *work = 0; *most = 0;
    for (int c = 0; c < (classes ? 8 : 1); ++c) {
        const int a = c >> 2, b = c >> 1 & 1, d = c & 1;
        const long long J = classes ? (long long)g.N * ((g.D - a + 1) / 2) * ((g.H - b + 1) / 2) * ((g.W - d + 1) / 2) : (flip ? g.in_voxels() : g.out_voxels());
        const int ntap = classes ? (g.pD ? (1 << (a + b + d)) : (1 << (3 - a - b - d))) : 27;
        const long long n = (J + bn - 1) / bn * MT;
        tiles += n;
        const int steps = flat ? (ntap * C + BK - 1) / BK : ntap * nch;
        *work += n * steps;
        if (J && steps > *most) *most = steps;
    }
    return tiles;
}
constexpr long long MAX_TILES = 1ll << 26;   // (of a grid; no volume whose planes are this small has more)

// (with less workspace than the best plan wants: fewer splits, down to whole contractions, which need none)
IgPlan plan_for(const Geom& g, int pass, size_t ws_bytes) {
    const bool flip = pass == MI3D_PASS_DGRAD, classes = flip && g.sD == 2;
    const int M = flip ? g.Cin : g.Cout, slots = 2 * cu_count();
    IgPlan best{};
    double best_us = 1e30;
    // (tiles of 32 channels where there are no more and the positions are not few: two tiles of 512 would need more splits)
    const bool narrow = M <= 32 && (flip ? g.in_voxels() : g.out_voxels()) >= 1024;
    for (int v = 0; v < (narrow ? 3 : 2); ++v) {
        const int bm = BMS[v], MT = (M + bm - 1) / bm;
        long long work;          // in tile steps
        int most;
        const long long tiles = count_tiles(g, pass, bm, BNS[v], &work, &most);
        if (tiles > MAX_TILES) continue;
        const size_t out_elems = (size_t)(flip ? g.in_voxels() * g.Cin : g.out_voxels() * g.Cout);
        for (const int S : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 40, 48, 64}) {
            if (S > most) break;
            if (S > 1 && (S * out_elems * 4 > ((size_t)64 << 20) || tiles * S > 4 * slots)) break;
            if (S > 1 && S * out_elems * 4 + copy_bytes(g, pass) > ws_bytes) break;
            // (classes of one to eight taps fill each other's rounds, but none is over before its longest workgroup: 320->256 of
            // the data gradient at 16^3, stride 2, whole 42 us, in four parts 28; with 16 steps or fewer splitting gives what it costs)
            double rounds = classes ? (double)work / most * S / slots + 0.5 : (double)((tiles * S + slots - 1) / slots);
            if (rounds < 1.0 && most > 16) rounds = 1.0;
            const double us = rounds * ((most + S - 1) / S) * STEP_US[v] + START_US + (S > 1 ? START_US + S * (double)out_elems * 8 / PART_BYTES_PER_US : 0.0);
            if (us < best_us) {
                best_us = us;
                best = IgPlan{v, S, MT, classes ? 8 : 1, (int)tiles, out_elems};
            }
        }
    }
    return best;
}
IgPlan make_plan(const Geom& g, int pass, size_t ws_bytes) { return kept_plan<IgPlan>(g, pass, ws_bytes, [&] { return plan_for(g, pass, ws_bytes); }); }

// Bytes from the first to the last voxel at the positions of a tile (256 of them at most), and the voxels by which a position
// can lie before an earlier one: positions beyond the volume they read from (it is the smaller one where a data gradient
// has little padding) run into the next row, plane and sample.  A position's voxel itself is at is * (d, h, w).
long long max_span(const Geom& g, int pass, long long* slack) {
    const bool flip = pass == MI3D_PASS_DGRAD;
    const long long is = flip ? 1 : g.sD, os = flip ? g.sD : 1;
    const long long C = flip ? g.Cout : g.Cin, iD = flip ? g.Do : g.D, iH = flip ? g.Ho : g.H, iW = flip ? g.Wo : g.W, plane = iH * iW;
    const long long oD = flip ? g.D : g.Do, oH = flip ? g.H : g.Ho, oW = flip ? g.W : g.Wo;
    long long most = 0, back = 0;
    for (int c = 0; c < (os == 2 ? 8 : 1); ++c) {
        const long long jD = (oD - (c >> 2) + os - 1) / os, jH = (oH - (c >> 1 & 1) + os - 1) / os, jW = (oW - (c & 1) + os - 1) / os;
        if (jD <= 0 || jH <= 0 || jW <= 0) continue;
        const long long xD = is * (jD - 1) - (iD - 1), xH = is * (jH - 1) - (iH - 1), xW = is * (jW - 1) - (iW - 1);   // beyond the volume
        const long long b = (g.N > 1 && xD > 0 ? (xD + 1) * plane : 0) + (xH > 0 ? (xH + 1) * iW : 0) + (xW > 0 ? xW + 1 : 0);
        if (b > back) back = b;
        // planes from a plane of positions to the next one, in the same sample or across its end
        const long long across = iD - is * (jD - 1), step = g.N > 1 && across > is ? across : is, rows = jH * jW;
        long long v;
        if (rows >= 256) {   // at most one change of plane, with the end of one plane and the beginning of the next
            const long long tail = iH - is * jH > 0 ? iH - is * jH : 0;
            v = (g.N * jD > 1 ? (step - 1) * plane : 0) + (tail + is * (2 * (255 / jW) + 4)) * iW;
        } else {
            const long long extent = is * (jH - 1) * iW + is * (jW - 1) + 1;
            v = (254 / rows + 1) * step * plane + (extent > plane ? extent : plane);
        }
        if (v > most) most = v;
    }
    if (slack) *slack = back;
    return (most + back) * C * 2 + 256;
}

}  // namespace

bool ig_supported(const Geom& g, int pass) { return g.Cin % 32 == 0 && g.Cout % 32 == 0 && ig_takes(g, pass); }

// (channels in eights: rows of whole 16-byte pieces)
bool ig_takes(const Geom& g, int pass) {
    if (g.dtype != MI3D_BF16 || pass == MI3D_PASS_WGRAD || g.kD != 3 || g.kH != 3 || g.kW != 3) return false;
    if (g.sD != g.sH || g.sD != g.sW || g.sD > 2 || g.Cin % 8 || g.Cout % 8) return false;
    if (g.sD == 1 ? (g.pD > 2 || g.pH > 2 || g.pW > 2) : (g.pD > 1 || g.pH > 1 || g.pW > 1)) return false;
    if (pass == MI3D_PASS_DGRAD && g.sD == 2 && (g.pD != g.pH || g.pD != g.pW)) return false;
    const bool flip = pass == MI3D_PASS_DGRAD;
    if ((flip ? g.H * (long long)g.W : g.Ho * (long long)g.Wo) >= (1ll << 31) || g.w_elems() * 2 >= (1ll << 31)) return false;
    // (stride-1 layers have the plane kernels for larger planes; ragged channels need steps of (tap, channel) pairs)
    if (!narrow_planes(g, pass) && (g.sD == 1 || g.Cin % 32 || g.Cout % 32 || max_span(g, pass, nullptr) >= (1ll << 31))) return false;
    long long work;
    int most;
    return g.in_voxels() < (1ll << 31) - 1024 && g.out_voxels() < (1ll << 31) - 1024 &&
           (count_tiles(g, pass, 128, 128, &work, &most) <= MAX_TILES || count_tiles(g, pass, 64, 256, &work, &most) <= MAX_TILES);
}

size_t ig_min_workspace_bytes(const Geom& g, int pass) { return copy_bytes(g, pass); }
size_t ig_workspace_bytes(const Geom& g, int pass) {
    const IgPlan p = make_plan(g, pass, ~(size_t)0);
    return copy_bytes(g, pass) + (p.splits > 1 ? p.splits * p.out_elems * sizeof(float) : 0);
}

void ig_describe(const Geom& g, int pass, size_t ws_bytes, char* buf, size_t len) {
    const IgPlan p = make_plan(g, pass, ws_bytes);
    snprintf(buf, len, "implicit_gemm_%dx%d%s parts %d", BMS[p.v], BNS[p.v], narrow_planes(g, pass) ? "" : "_wide", p.splits);
}

// in: activations read (x of the forward pass, dy of the data gradient); out: y or dx
// wflags: see ig_transpose_kernel (27 words per 64 x 64 block of channels; the forward pass writes none)
int ig_conv(const Geom& g, int pass, const void* in, const void* w, void* out, void* ws, size_t ws_bytes, hipStream_t s, uint32_t* wflags) {
    if (ws_bytes < ig_min_workspace_bytes(g, pass)) return MI3D_ERR_WORKSPACE;
    const bool flip = pass == MI3D_PASS_DGRAD;
    const IgPlan plan = make_plan(g, pass, ws_bytes);
    if (g.hi && g.Cin % 64) return MI3D_ERR_UNSUPPORTED;
    int st = MI3D_OK;
    const bool tr = reads_tr(g, pass);
    if (flip && !tr) {
        ig_transpose_kernel<<<dim3(27, (g.Cin + 63) / 64, (g.Cout + 63) / 64), 256, 0, s>>>((const uint16_t*)w, (uint16_t*)ws, 27, g.Cin, g.Cout, wflags);
        if ((st = check_launch())) return st;
    }
    IgParams P{};
    P.in = P.in_hi = (const uint16_t*)in;
    P.w = (const uint16_t*)(flip && !tr ? ws : w);
    P.out = (uint16_t*)out;
    P.add = (const uint16_t*)g.add; P.ref = (const uint16_t*)g.ref; P.slope = g.slope;
    P.part = plan.splits > 1 ? (float*)((char*)ws + copy_bytes(g, pass)) : nullptr;
    P.T = 27; P.splits = plan.splits; P.MT = plan.MT; P.ncls = plan.ncls; P.tiles = plan.tiles; P.out_elems = (long long)plan.out_elems;
    P.is = flip ? 1 : g.sD; P.os = flip ? g.sD : 1;
    if (!flip) {
        P.C = g.Cin; P.M = g.Cout; P.iD = g.D; P.iH = g.H; P.iW = g.W; P.oD = g.Do; P.oH = g.Ho; P.oW = g.Wo;
    } else {
        P.C = g.Cout; P.M = g.Cin; P.iD = g.Do; P.iH = g.Ho; P.iW = g.Wo; P.oD = g.D; P.oH = g.H; P.oW = g.W;
    }
    P.csplit = P.pitch = P.C;
    if (g.hi && !flip) { P.in_hi = (const uint16_t*)g.hi; P.csplit = P.pitch = P.C / 2; }
    if (g.hi && flip) P.out_hi = (uint16_t*)g.hi;
    P.in_bytes = (long long)g.N * P.iD * P.iH * P.iW * P.pitch * 2;
    max_span(g, pass, &P.slack);
    P.Cdiv = make_div(P.C);
    const int bn = BNS[plan.v], pads[3] = {g.pD, g.pH, g.pW};
    int tile = 0, ntap = 0;
    for (int q = 0; q < plan.ncls; ++q) {
        // classes with the most taps first, so that the long workgroups do not start last
        const int c = plan.ncls == 8 && g.pD ? 7 - q : q;
        const int par[3] = {c >> 2, c >> 1 & 1, c & 1};
        IgClass& K = P.cls[q];
        const int ext[3] = {P.oD, P.oH, P.oW};
        int j[3];
        for (int a = 0; a < 3; ++a) j[a] = plan.ncls == 8 ? (ext[a] - par[a] + 1) / 2 : ext[a];
        K.od0 = plan.ncls == 8 ? par[0] : 0; K.oh0 = plan.ncls == 8 ? par[1] : 0; K.ow0 = plan.ncls == 8 ? par[2] : 0;
        K.J = g.N * j[0] * j[1] * j[2];
        K.PT = (K.J + bn - 1) / bn;
        for (int a = 0; a < 3; ++a) j[a] = j[a] > 0 ? j[a] : 1;   // (an empty class has no tile)
        K.jD = make_div(j[0]); K.jH = make_div(j[1]); K.jW = make_div(j[2]);
        K.tile0 = tile;
        tile += K.PT * plan.MT;
        K.tap0 = ntap;
        for (int k = 0; k < 27; ++k) {
            const int kk[3] = {k / 9, k / 3 % 3, k % 3};
            int delta[3];
            bool hit = true;
            for (int a = 0; a < 3; ++a) {
                if (!flip) delta[a] = kk[a] - pads[a];
                else if (plan.ncls == 1) delta[a] = pads[a] - kk[a];
                else {   // output 2 j + par receives dy at (2 j + par + p - k) / 2
                    const int v = par[a] + pads[a] - kk[a];
                    hit = hit && (v & 1) == 0;
                    delta[a] = v / 2;
                }
            }
            if (!hit) continue;
            P.taps[ntap++] = tap_word(delta[0], delta[1], delta[2], k);
        }
        K.ntap = ntap - K.tap0;
    }
    const bool wide = !narrow_planes(g, pass), flat = is_flat(g, pass);
    typedef void (*Kernel)(IgParams);
    static const Kernel kernels[3][4] = {{ig_kernel<2, 2, false, false>, ig_kernel<2, 2, true, false>, ig_kernel<2, 2, false, true>, ig_kernel<2, 2, false, false, true>},
                                         {ig_kernel<4, 2, false, false>, ig_kernel<4, 2, true, false>, ig_kernel<4, 2, false, true>, ig_kernel<4, 2, false, false, true>},
                                         {ig_kernel<4, 1, false, false>, ig_kernel<4, 1, true, false>, ig_kernel<4, 1, false, true>, ig_kernel<4, 1, false, false, true>}};
    auto lds = [](int v) { return (size_t)2 * (BMS[v] + BNS[v]) * 128; };
    static std::atomic<bool> attr_set{false};   // set once per process; a second thread racing here repeats an idempotent call
    if (!attr_set) {
        for (int v = 0; v < 3; ++v)
            for (Kernel f : kernels[v]) {
                hipError_t e = hipFuncSetAttribute((const void*)f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds(v));
                if (e != hipSuccess) { note_hip_error(e); return MI3D_ERR_HIP; }
            }
        attr_set = true;
    }
    kernels[plan.v][wide ? 1 : flat ? 2 : tr ? 3 : 0]<<<(unsigned)(plan.tiles * plan.splits), 256, lds(plan.v), s>>>(P);
    st = check_launch();
    if (st || plan.splits == 1) return st;
    const long long n = P.out_elems;
    long long blocks = (n / 8 + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    ig_sum_kernel<<<(unsigned)blocks, 256, 0, s>>>(P.part, (uint16_t*)out, n / 8, n, plan.splits, g.slope, (const uint16_t*)g.ref,
                                                            (uint16_t*)(flip ? g.hi : nullptr), P.M, (const uint16_t*)g.add);
    return check_launch();
}

}  // namespace mi3d
