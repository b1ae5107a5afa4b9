// fp32 convolution over numbered positions (implicit GEMM), its products formed by bf16 matrix instructions: forward pass and
// data gradient of any layer with kernel extents up to 3 and strides up to 2 whose contracted channels come in fours.
// Each operand is taken apart into three bf16 numbers and six of the nine products are added in fp32 (conv_f32.hip has the
// bound of what is left out).
//
//   out[os j + par, m] = sum over taps t and contracted channels c of  in[is j + delta_t, c] * w[m, t, c]
//
// Positions j are numbered through all samples.  The contraction runs over (tap, channel) pairs in steps of 32, whatever the
// number of channels is.  A strided data gradient is one product per parity class of the output voxel, all in
// one launch; where the taps do not overlap (kernel extent = stride) the classes read the same voxel, so they are
// output channels of a single product: m = (tap, channel).  Where the tiles leave CUs idle the steps are split and fp32
// partial sums are added in index order by igf_sum_kernel.
//
// A workgroup (4 waves) owns 128 positions x 128, 64 or 32 channels.  The step after next is requested from memory into
// registers, the next one is taken apart on its way to LDS ([part][position][32], 16-byte pieces permuted so that 16
// neighbouring rows cover all banks) between the MFMAs of this one.  Weights are packed in fragment order by
// igf_pack_kernel and read from there half a step ahead.  A lane ends with one channel of 16 positions, so that 32 lanes
// store 128 contiguous bytes.
//
// Bound: with 128 channels and many steps the matrix cores at the power limit (128->128 at 32^3, N = 2: 1.0 PFLOP/s of bf16
// products, a library product of 8192^2 matrices 1.15); with fewer channels per tile the conversion, which a tile repeats for
// each tap; with few steps the beginning and the end of a workgroup.  conv_f32.hip has the times beside the dispatch rule.
//
// A value outside the range of the split (split_f32.h; infinities and NaN among them) sends its step through
// v_mfma_f32_32x32x2_f32 on operands read straight from memory; where a weight is not finite, position by position for those
// whose tap lies inside the volume: it meets no zero that is not there.
#include <cstdio>

#include "ig_common.h"
#include "mi3d_internal.h"
#include "split_f32.h"

namespace mi3d {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef unsigned u32x4 __attribute__((__vector_size__(4 * sizeof(unsigned))));

constexpr int BN = 128, BK = 32, ROWS = BN / 32;   // positions of a tile, (tap, channel) pairs of a step, rows a thread fetches
constexpr int PART = BN * BK * 2, STAGE = 3 * PART;
constexpr unsigned OOB = 0xFFFFFFF0u;              // buffer offset of a piece that must read as zero
constexpr long long MAX_BYTES = 0xFFFFFF00ll;      // of a tensor whose pieces are addressed with 32-bit offsets
constexpr int MAX_STEPS = 2048;                    // of a workgroup: a bit for each that the parts cannot hold

struct IgfClass {
    Div jD, jH, jW;          // extents of the position space of a sample
    int J, PT, tile0;        // positions of all samples, tiles of them, first tile in the grid
    int od0, oh0, ow0;
    int tap0, ntap, steps;
    int frag0;               // first half step of the class among the packed weights
};
struct IgfParams {
    const float *in, *in_hi;     // two halves along the channels (virtual concatenation), or the tensor and itself
    const float* w;              // the layer's own weights: element (m, tap, c) at m * w_m + tap * w_t + c * w_c
    long long w_m, w_t, w_c;
    const uint16_t* wsplit;      // [half step][MB][3 parts][64 lanes][8]
    const uint32_t* wflag;       // [half step][MB]: a value of this fragment cannot be split
    float *out, *out_hi;
    const float *add, *ref;      // optional operands of the epilogue, of the output's shape
    float* part;                 // [split][output element] partial sums, or null: the kernel finishes the output itself
    float slope;
    Div C;                       // contracted channels
    int csplit, pitch;           // first channel in in_hi, channels per voxel of in / in_hi
    int M, MB, MT;               // output channels, blocks of 32 of them, tiles
    int isd, ish, isw, osd, osh, osw;
    int iD, iH, iW, oD, oH, oW;
    int out_pitch, out_split;    // channels per voxel of out / out_hi, first channel in out_hi
    int scatter, kH, kW;         // 1: m = (tap, channel) and the tap moves the output voxel
    Div sC;                      // scatter: channels of a tap
    int splits, ncls, tiles;
    long long out_elems;
    uint32_t in_bytes;           // of one of in / in_hi
    IgfClass cls[8];
    uint32_t taps[27];
};
static_assert(sizeof(IgfParams) <= 4096, "kernel arguments");

__device__ __forceinline__ f32x16 mfma16(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x16 mfma2(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ float4 load16(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}
__device__ __forceinline__ float load4(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}

__device__ __forceinline__ void decode(const IgfClass& K, int j, int& n, int& d, int& h, int& w) {
    const int r = divide(j, K.jW);
    w = j - r * (int)K.jW.d;
    const int r2 = divide(r, K.jH);
    h = r - r2 * (int)K.jH.d;
    n = divide(r2, K.jD);
    d = r2 - n * (int)K.jD.d;
}

struct Tables {            // of a workgroup, behind the stages in LDS
    long long out[BN];     // element of channel 0 of the position's output voxel, or -1
    uint32_t row[BN];      // byte of its input voxel (modulo 2^32)
    uint32_t mask[BN];     // bit k: tap k of the class reads inside the volume; from bit 27 on: the next voxel along w, h, d exists
    uint32_t tap[32];      // byte offset of each tap
    uint32_t bad[MAX_STEPS / 32];
};
static_assert(sizeof(Tables) % 16 == 0, "");

// WP = waves along the positions, PB / CB = blocks of 32 positions / channels of a wave.  DEEP: weights are held half a step
// ahead; otherwise they are requested behind their last use, which makes room for a third workgroup per CU: with few steps
// a workgroup's beginning and end count for more (64->128, 2x2x2 at 96^3 data gradient, 4 steps, 199 -> 169 us; with 108
// steps 338 -> 344).
template <int WP, int PB, int CB, bool DEEP>
__global__ void __launch_bounds__(256, DEEP ? 2 : 3) igf_kernel(const IgfParams P) {
    static_assert(WP * PB * 32 == BN, "");
    constexpr int WC = 4 / WP, BM = 32 * WC * CB;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    Tables& L = *(Tables*)(lds + 2 * STAGE);
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int ln = lane & 31, half = lane >> 5;
    const int wp = wave % WP, wc = wave / WP;

    // block -> (split, class, tile of positions, tile of channels); the blocks of an XCD (every eighth) get neighbouring
    // tiles of a class, channels fastest, so that they share the positions' rows in its L2
    int id = blockIdx.x;
    const int split = id / P.tiles;
    id -= split * P.tiles;
    int ci = 0;
    while (ci + 1 < P.ncls && id >= P.cls[ci + 1].tile0) ++ci;
    const IgfClass& K = P.cls[ci];
    {
        const int n = K.PT * P.MT, l = id - K.tile0, x = l & 7, q = l >> 3;
        id = x * (n >> 3) + ((n & 7) < x ? (n & 7) : x) + q;
    }
    const int pt = id / P.MT, mt = id - pt * P.MT;
    const int s0 = (int)((long long)K.steps * split / P.splits), s1 = (int)((long long)K.steps * (split + 1) / P.splits);
    const int mb0 = mt * (BM / 32) + wc * CB;

    // lane k keeps tap k: reading it from there costs no memory latency
    const int tapv = lane < K.ntap ? (int)P.taps[K.tap0 + lane] : 0;
    if (t < BN) {
        const int j = pt * BN + t;
        int n, d, h, w;
        decode(K, j, n, d, h, w);
        const int od = P.osd * d + K.od0, oh = P.osh * h + K.oh0, ow = P.osw * w + K.ow0;
        const long long vox = (((long long)n * P.oD + od) * P.oH + oh) * P.oW + ow;
        L.out[t] = j < K.J ? vox * P.out_pitch : -1;
        d *= P.isd; h *= P.ish; w *= P.isw;
        L.row[t] = (((uint32_t)(n * P.iD + d) * P.iH + h) * P.iW + w) * P.pitch * 4;
        uint32_t m = 0;
        for (int k = 0; k < K.ntap; ++k) {
            const IgTap a(__builtin_amdgcn_readlane(tapv, k));
            const bool ok = ((unsigned)(d + a.dd) < (unsigned)P.iD) & ((unsigned)(h + a.dh) < (unsigned)P.iH) & ((unsigned)(w + a.dw) < (unsigned)P.iW);
            m |= (ok ? 1u : 0u) << k;
        }
        if (j >= K.J) m = 0;
        m |= (ow + 1 < P.oW ? 1u : 0u) << 27 | (oh + 1 < P.oH ? 1u : 0u) << 28 | (od + 1 < P.oD ? 1u : 0u) << 29;
        L.mask[t] = m;
    } else if (t < BN + 32) {
        const int k = t - BN;     // (= lane)
        uint32_t o = 0;
        if (k < K.ntap) {
            const IgTap a((uint32_t)tapv);
            o = (uint32_t)((a.dd * P.iH + a.dh) * P.iW + a.dw) * P.pitch * 4;
        }
        L.tap[k] = o;
    } else if (t < BN + 32 + MAX_STEPS / 32) {
        L.bad[t - BN - 32] = 0;
    }
    __syncthreads();
    auto set_bad = [&](int s) { atomicOr(&L.bad[(s - s0) >> 5], 1u << ((s - s0) & 31)); };
    auto is_bad = [&](int s) { return __builtin_amdgcn_readfirstlane(L.bad[(s - s0) >> 5] >> ((s - s0) & 31) & 1) != 0; };
    const __amdgpu_buffer_rsrc_t r_in = __builtin_amdgcn_make_buffer_rsrc((void*)P.in, 0, (int)P.in_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t r_hi = __builtin_amdgcn_make_buffer_rsrc((void*)P.in_hi, 0, (int)P.in_bytes, 0x00020000);
    // the rows this thread fetches: t / 8 + 32 i, four (tap, channel) pairs of each
    uint32_t row[ROWS], mask[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) { row[i] = L.row[(t >> 3) + 32 * i]; mask[i] = L.mask[(t >> 3) + 32 * i] & 0x7FFFFFFu; }
    float4 px[ROWS];
    auto request = [&](int s) {
        const int k = s * BK + 4 * (t & 7), tap = divide(k, P.C), c = k - tap * (int)P.C.d;
        const uint32_t off = L.tap[tap & 31] + 4 * c, bit = tap < K.ntap ? 1u << tap : 0u;
        // (a step lies in one half of a virtual concatenation: both are multiples of 32 channels)
        if (__builtin_amdgcn_readfirstlane(c) < P.csplit) {
#pragma unroll
            for (int i = 0; i < ROWS; ++i) px[i] = load16(r_in, mask[i] & bit ? row[i] + off : OOB);
            asm volatile("; low half");   // keeps the branches apart: merged, their loads run in a loop over the resources
        } else {
#pragma unroll
            for (int i = 0; i < ROWS; ++i) px[i] = load16(r_hi, mask[i] & bit ? row[i] + off - P.csplit * 4 : OOB);
        }
    };
    const int wr = (t >> 3) * 64 + ((((t & 7) >> 1) ^ (t >> 5)) & 3) * 16 + (t & 1) * 8;   // (row + 32 i: the same permutation)
    auto stage = [&](int s) {   // px -> parts of step s
        char* d = lds + ((s - s0) & 1) * STAGE + wr;
        SplitRangeNumbers range;
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            range.add(px[i]);
            uint32_t lo[3], hi[3];
            split2(px[i].x, px[i].y, lo);
            split2(px[i].z, px[i].w, hi);
#pragma unroll
            for (int p = 0; p < 3; ++p) *(uint2*)(d + p * PART + i * 32 * 64) = uint2{lo[p], hi[p]};
        }
        if (__any(range.exceeded()) && lane == 0) set_bad(s);
    };
    bf16x8 wf[DEEP ? 2 : 1][CB][3];
    auto weights = [&](int f, bf16x8 (&v)[CB][3]) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            // (blocks beyond the last one read that again and are not stored)
            const int mb = mb0 + cb < P.MB ? mb0 + cb : P.MB - 1;
            const uint16_t* q = P.wsplit + ((long long)(K.frag0 + f) * P.MB + mb) * (3 * 512) + lane * 8;
#pragma unroll
            for (int p = 0; p < 3; ++p) v[cb][p] = *(const bf16x8*)(q + p * 512);
        }
    };

    f32x16 acc[PB][CB];
#pragma unroll
    for (int a = 0; a < PB; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

    const int rd = (wp * PB * 32 + ln) * 64, swz = (ln >> 2) & 3;
    auto products = [&](int s, int hs) {   // half step hs
        const char* b = lds + ((s - s0) & 1) * STAGE + rd + (((2 * hs + half) ^ swz) & 3) * 16;
        bf16x8 xf[PB][3];
#pragma unroll
        for (int a = 0; a < PB; ++a)
#pragma unroll
            for (int p = 0; p < 3; ++p) xf[a][p] = *(const bf16x8*)(b + p * PART + a * 32 * 64);
        constexpr int PW[6] = {2, 0, 1, 1, 0, 0}, PX[6] = {0, 2, 1, 0, 1, 0};   // small products first
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int b2 = 0; b2 < CB; ++b2)
#pragma unroll
                for (int a = 0; a < PB; ++a) acc[a][b2] = mfma16(xf[a][PX[q]], wf[DEEP ? hs : 0][b2][PW[q]], acc[a][b2]);
    };
    if (s0 < s1) {
        request(s0);
        weights(2 * s0, wf[0]);
        for (int e = t; e < 2 * (s1 - s0) * (BM / 32); e += 256) {
            const int f = 2 * s0 + e / (BM / 32), mb = mt * (BM / 32) + e % (BM / 32);
            if (mb < P.MB && P.wflag[(long long)(K.frag0 + f) * P.MB + mb]) set_bad(f / 2);
        }
        stage(s0);
        if (s0 + 1 < s1) request(s0 + 1);
        __syncthreads();
        for (int s = s0; s < s1; ++s) {
            const bool bad = is_bad(s);
            if (DEEP) weights(2 * s + 1, wf[DEEP ? 1 : 0]);
            if (!bad) products(s, 0);
            if (!DEEP) weights(2 * s + 1, wf[0]);
            if (s + 1 < s1) {
                if (DEEP) weights(2 * s + 2, wf[0]);
                stage(s + 1);
                if (s + 2 < s1) request(s + 2);
            }
            if (!bad) products(s, 1);
            if (!DEEP && s + 1 < s1) weights(2 * s + 2, wf[0]);
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // (requests stay under way)
        }
    }
    // the steps left out, on the values themselves (a loop of its own: inside the other one it costs that 80 registers)
    for (int s = s0; s < s1; ++s) {
        if (!is_bad(s)) continue;
#pragma unroll 1
        for (int kk = 0; kk < BK; kk += 2) {
            float xv[PB];
            const int k = s * BK + kk + half, tap = divide(k, P.C), c = k - tap * (int)P.C.d;
            const bool in = tap < K.ntap, hi = c >= P.csplit;
            const uint32_t off = L.tap[tap & 31] + 4 * (hi ? c - P.csplit : c);
#pragma unroll
            for (int a = 0; a < PB; ++a) {
                const int r = wp * PB * 32 + a * 32 + ln;
                const uint32_t o = in && (L.mask[r] >> tap & 1) ? L.row[r] + off : OOB;
                const float lo = load4(r_in, hi ? OOB : o), up = load4(r_hi, hi ? o : OOB);
                xv[a] = hi ? up : lo;
            }
            const long long wt = in ? (P.taps[K.tap0 + tap] >> 24) * P.w_t + c * P.w_c : 0;
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                const int m = (mb0 + b) * 32 + ln;
                const float wv = in && m < P.M ? P.w[m * P.w_m + wt] : 0.f;
                const bool odd = !(fabsf(wv) < __builtin_inff());
                if (!__any(odd)) {
#pragma unroll
                    for (int a = 0; a < PB; ++a) acc[a][b] = mfma2(xv[a], wv, acc[a][b]);
                    continue;
                }
#pragma unroll 1
                for (int h = 0; h < 2; ++h) {   // the two pairs of this instruction, one after the other
                    const float w1 = __shfl(wv, ln + 32 * h);
                    const int tap1 = __shfl(in ? tap : 31, 32 * h);
#pragma unroll
                    for (int a = 0; a < PB; ++a)
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const int r = 8 * (i >> 2) + 4 * half + (i & 3);
                            const float x1 = __shfl(xv[a], r + 32 * h);
                            if ((L.mask[wp * PB * 32 + a * 32 + r] & 0x7FFFFFFu) >> tap1 & 1) acc[a][b][i] += x1 * w1;
                            asm volatile("" ::: "memory");   // (one table read at a time: together they would take the registers)
                        }
                }
            }
        }
    }

    // lane (channel ln, half): register i of a block is position 8 (i / 4) + 4 half + i % 4 of its 32
    long long mo[CB];     // of the lane's channels, from the voxel's first one on
    uint32_t need[CB];    // neighbours of the voxel that have to exist
    float* dst[CB];
#pragma unroll
    for (int b = 0; b < CB; ++b) {
        const int m = (mb0 + b) * 32 + ln;
        int c = m;            // channel of its output voxel
        mo[b] = m;
        need[b] = m < P.M ? 0u : 1u << 31;
        if (P.scatter) {
            const int tap = divide(m, P.sC), kw = tap % P.kW, kh = tap / P.kW % P.kH, kd = tap / P.kW / P.kH;
            c = m - tap * (int)P.sC.d;
            mo[b] = ((long long)(kd * P.oH + kh) * P.oW + kw) * P.out_pitch + c;
            need[b] |= (uint32_t)kw << 27 | (uint32_t)kh << 28 | (uint32_t)kd << 29;
        }
        dst[b] = (P.part ? P.part + split * P.out_elems : c >= P.out_split ? P.out_hi - P.out_split : P.out) + mo[b];
    }
#pragma unroll
    for (int a = 0; a < PB; ++a)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = wp * PB * 32 + a * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
            const long long o = L.out[r];
            const uint32_t have = L.mask[r];
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                if (o < 0 || (need[b] & ~have)) continue;
                float v = acc[a][b][i];
                if (!P.part) {
                    if (P.add) v += P.add[o + mo[b]];
                    v = (P.ref ? P.ref[o + mo[b]] : v) > 0.f ? v : P.slope * v;
                }
                dst[b][o] = v;
            }
            if ((i & 3) == 3) asm volatile("" ::: "memory");   // (all table reads at once would take the registers)
        }
}

// One wave per fragment of half a step: 16 (tap, channel) pairs of a class x 32 output channels.  Zero beyond either.
__global__ void __launch_bounds__(256) igf_pack_kernel(const IgfParams P, uint16_t* __restrict__ out, uint32_t* __restrict__ flag, int frags) {
    const int lane = threadIdx.x & 63, f = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (f >= frags) return;
    const int mb = f % P.MB, hs = f / P.MB;
    int ci = 0;
    while (ci + 1 < P.ncls && hs >= P.cls[ci + 1].frag0) ++ci;
    const IgfClass& K = P.cls[ci];
    const int m = mb * 32 + (lane & 31), k0 = (hs - K.frag0) * 16 + 8 * (lane >> 5);
    float v[8];
    SplitRange range;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int tap = divide(k0 + i, P.C), c = k0 + i - tap * (int)P.C.d;
        v[i] = m < P.M && tap < K.ntap ? P.w[m * P.w_m + (P.taps[K.tap0 + tap] >> 24) * P.w_t + c * P.w_c] : 0.f;
        range.add(v[i]);
    }
    uint32_t o[4][3];
#pragma unroll
    for (int i = 0; i < 4; ++i) split2(v[2 * i], v[2 * i + 1], o[i]);
#pragma unroll
    for (int p = 0; p < 3; ++p) *(uint4*)(out + (((long long)f * 3 + p) * 64 + lane) * 8) = uint4{o[0][p], o[1][p], o[2][p], o[3][p]};
    const bool any = __any(range.exceeded());
    if (lane == 0) flag[f] = any ? 1u : 0u;
}

// out = epilogue(sum of the parts in index order), one element per thread and turn (the parts are at most a few MB)
__global__ void __launch_bounds__(256) igf_sum_kernel(const float* __restrict__ part, long long n, int splits, int M, int out_split, float* __restrict__ out,
                                                      float* __restrict__ out_hi, const float* __restrict__ add, const float* __restrict__ ref, float slope) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
        float v = 0.f;
#pragma unroll 8
        for (int p = 0; p < splits; ++p) v += part[p * n + i];
        if (add) v += add[i];
        v = (ref ? ref[i] : v) > 0.f ? v : slope * v;
        if (out_split < M) {   // output in two halves along the channels
            const long long vox = i / M;
            const int c = (int)(i - vox * M);
            if (c < out_split) out[vox * out_split + c] = v;
            else out_hi[vox * (M - out_split) + c - out_split] = v;
        } else {
            out[i] = v;
        }
    }
}

// Tile shape and splits of the contraction, by a model of the time: steps of a workgroup times what a step takes with that
// many workgroups on its CU (measured: 320->320 at 8^3, N = 2, whose 24 to 160 workgroups are alone on theirs, and 128->128 at
// 32^3, 64->64 at 64^3, 64->32 at 45 x 75 x 91, which fill them), what a workgroup needs before and after, and the way of the
// partial sums.
struct IgfPlan {
    int v;                 // 0: 128 channels, 1: 64, 2: 32
    int splits, MT, most;  // most: steps of the longest class
    long long tiles, frags;
    long long out_elems;
    double us;
};
constexpr int BMS[3] = {128, 64, 32}, RES[3] = {2, 3, 3};
constexpr double STEP_US[3][3] = {{1.95, 3.1, 3.1}, {1.5, 2.0, 2.6}, {1.25, 1.5, 1.9}};
constexpr double START_US[3] = {4.0, 3.0, 2.5}, LAUNCH_US = 4.0, PART_BYTES_PER_US = 3.5e6;
constexpr long long MAX_TILES = 1ll << 26;

bool one_voxel(const Geom& g, int pass) {   // data gradient whose classes read one voxel each, the same one
    return pass == MI3D_PASS_DGRAD && g.kD == g.sD && g.kH == g.sH && g.kW == g.sW && !g.pD && !g.pH && !g.pW && g.taps() > 1;
}

// Classes, their positions, taps and packed weights
// (returns the half steps of all classes)
int make_classes(const Geom& g, int pass, IgfParams* P, long long* J, int* most) {
    const bool dgrad = pass == MI3D_PASS_DGRAD, scatter = one_voxel(g, pass);
    const int C = dgrad ? g.Cout : g.Cin;
    const int sD = dgrad ? g.sD : 1, sH = dgrad ? g.sH : 1, sW = dgrad ? g.sW : 1;
    const int eD = dgrad ? g.D : g.Do, eH = dgrad ? g.H : g.Ho, eW = dgrad ? g.W : g.Wo;
    P->ncls = 0;
    int ntap = 0, frag = 0;
    *most = 0;
    struct Par { int d, h, w, n; } par[8];
    int np = 0;
    for (int a = 0; a < (scatter ? 1 : sD); ++a)
        for (int b = 0; b < (scatter ? 1 : sH); ++b)
            for (int c = 0; c < (scatter ? 1 : sW); ++c)
                par[np++] = Par{a, b, c, scatter ? 1 : axis_taps(g.kD, g.sD, g.pD, dgrad, a).n * axis_taps(g.kH, g.sH, g.pH, dgrad, b).n * axis_taps(g.kW, g.sW, g.pW, dgrad, c).n};
    // classes with the most taps first, so that the long workgroups do not start last
    for (int i = 0; i < np; ++i)
        for (int k = i + 1; k < np; ++k)
            if (par[k].n > par[i].n) { const Par q = par[i]; par[i] = par[k]; par[k] = q; }
    for (int i = 0; i < np; ++i) {
        const Par& r = par[i];
        const int j[3] = {(eD - r.d + sD - 1) / sD, (eH - r.h + sH - 1) / sH, (eW - r.w + sW - 1) / sW};
        if (j[0] <= 0 || j[1] <= 0 || j[2] <= 0) continue;
        IgfClass& K = P->cls[P->ncls];
        J[P->ncls++] = (long long)g.N * j[0] * j[1] * j[2];
        K.jD = make_div(j[0]); K.jH = make_div(j[1]); K.jW = make_div(j[2]);
        K.od0 = r.d; K.oh0 = r.h; K.ow0 = r.w;
        K.tap0 = ntap;
        if (scatter) {
            P->taps[ntap++] = tap_word(0, 0, 0, 0);
        } else {
            const AxisTaps ad = axis_taps(g.kD, g.sD, g.pD, dgrad, r.d), ah = axis_taps(g.kH, g.sH, g.pH, dgrad, r.h), aw = axis_taps(g.kW, g.sW, g.pW, dgrad, r.w);
            for (int a = 0; a < ad.n; ++a)
                for (int b = 0; b < ah.n; ++b)
                    for (int c = 0; c < aw.n; ++c)
                        // stride-1 data gradient: axis_taps has delta = pad - t
                        P->taps[ntap++] = tap_word(ad.d[a], ah.d[b], aw.d[c], (ad.t[a] * g.kH + ah.t[b]) * g.kW + aw.t[c]);
        }
        K.ntap = ntap - K.tap0;
        K.steps = (K.ntap * C + BK - 1) / BK;
        K.frag0 = frag;
        frag += 2 * K.steps;
        if (K.steps > *most) *most = K.steps;
    }
    const int M = scatter ? (int)g.taps() * g.Cin : dgrad ? g.Cin : g.Cout;
    P->M = M;
    P->MB = (M + 31) / 32;
    return frag;
}

size_t flags_at(long long frags) { return (size_t)frags * (3 * 512 * 2); }
size_t pack_bytes(long long frags) { return (flags_at(frags) + (size_t)frags * 4 + 255) & ~(size_t)255; }

// Workgroups of `mean` steps each (the longest: most): full rounds of RES per CU, and what is left over
double plan_us(int v, int cus, long long wgs, double most, double mean) {
    const long long full = wgs / ((long long)RES[v] * cus), rest = wgs - full * RES[v] * cus;
    const int k = (int)((rest + cus - 1) / cus);
    auto round = [&](int n, double steps) { return steps * STEP_US[v][n - 1] + START_US[v] * n; };
    const double us = full * round(RES[v], mean) + (k ? round(k, mean < most ? 0.5 * (mean + most) : mean) : 0.0);
    // (uneven workgroups: the longest have company for about half of their time)
    const double longest = mean < most && wgs > cus ? 0.5 * (round(1, most) + round(RES[v], most)) : round(1, most);
    return us > longest ? us : longest;
}

// (with less workspace than the best plan wants: fewer splits, down to whole contractions, which need the packed weights alone)
IgfPlan plan_for(const Geom& g, int pass, size_t ws_bytes) {
    IgfParams P;
    long long J[8];
    int most;
    const long long half_steps = make_classes(g, pass, &P, J, &most);
    const int cus = cu_count();
    const long long out_elems = pass == MI3D_PASS_DGRAD ? g.in_voxels() * g.Cin : g.out_voxels() * g.Cout;
    IgfPlan best{-1, 1, 0, most, 0, half_steps * P.MB, out_elems, 1e30};
    for (int v = 0; v < 3; ++v) {
        const int MT = (P.M + BMS[v] - 1) / BMS[v];
        long long tiles = 0;
        double work = 0;
        for (int c = 0; c < P.ncls; ++c) {
            const long long n = (J[c] + BN - 1) / BN * MT;
            tiles += n;
            work += (double)n * P.cls[c].steps;
        }
        if (tiles > MAX_TILES) continue;
        for (const int S : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 40, 48, 64}) {
            if (most > S * (long long)MAX_STEPS) continue;
            if (S > 1 && (S > most || S * out_elems * 4 > (32ll << 20) || tiles * S > 8 * cus)) break;
            if (S > 1 && S * (size_t)out_elems * 4 + pack_bytes(best.frags) > ws_bytes) break;
            const double us = plan_us(v, cus, tiles * S, (most + S - 1) / S, work / (tiles ? tiles : 1) / S) + (S > 1 ? LAUNCH_US + S * (double)out_elems * 8 / PART_BYTES_PER_US : 0.0);
            if (us < best.us) {
                best.us = us;
                best.v = v; best.splits = S; best.MT = MT; best.tiles = tiles;
            }
        }
    }
    return best;
}
IgfPlan make_plan(const Geom& g, int pass, size_t ws_bytes) { return kept_plan<IgfPlan>(g, pass, ws_bytes, [&] { return plan_for(g, pass, ws_bytes); }); }

}  // namespace

bool igf_supported(const Geom& g, int pass) {
    if (g.dtype != MI3D_F32 || pass == MI3D_PASS_WGRAD) return false;
    if (g.kD > 3 || g.kH > 3 || g.kW > 3 || g.sD > 2 || g.sH > 2 || g.sW > 2 || g.pD > 2 || g.pH > 2 || g.pW > 2) return false;
    const bool dgrad = pass == MI3D_PASS_DGRAD;
    if ((dgrad ? g.Cout : g.Cin) % 4) return false;
    const long long in = dgrad ? g.out_voxels() * g.Cout : g.in_voxels() * g.Cin;
    if (in * 4 > MAX_BYTES || g.in_voxels() >= (1ll << 31) - 1024 || g.out_voxels() >= (1ll << 31) - 1024 || g.w_elems() >= (1ll << 28)) return false;
    return make_plan(g, pass, 0).v >= 0;   // (whole contractions: whether there is a tile shape)
}

double igf_us(const Geom& g, int pass) { return LAUNCH_US + make_plan(g, pass, ~(size_t)0).us; }
size_t igf_min_workspace_bytes(const Geom& g, int pass) { return pack_bytes(make_plan(g, pass, 0).frags); }
size_t igf_workspace_bytes(const Geom& g, int pass) {
    const IgfPlan p = make_plan(g, pass, ~(size_t)0);
    return pack_bytes(p.frags) + (p.splits > 1 ? (size_t)p.splits * p.out_elems * sizeof(float) : 0);
}
void igf_describe(const Geom& g, int pass, size_t ws_bytes, char* buf, size_t len) {
    const IgfPlan p = make_plan(g, pass, ws_bytes);
    snprintf(buf, len, "f32_implicit_gemm_%dx%d_parts_%d_from_bf16_parts", BMS[p.v], BN, p.splits);
}

// in: activations read (x of the forward pass, dy of the data gradient); out: y or dx
int igf_conv(const Geom& g, int pass, const void* in, const void* w, void* out, void* ws, size_t ws_bytes, hipStream_t s) {
    const bool dgrad = pass == MI3D_PASS_DGRAD;
    const IgfPlan plan = make_plan(g, pass, ws_bytes);
    if (plan.v < 0) return MI3D_ERR_UNSUPPORTED;
    if (ws_bytes < pack_bytes(plan.frags)) return MI3D_ERR_WORKSPACE;
    if (g.hi && g.Cin % 64) return MI3D_ERR_UNSUPPORTED;
    IgfParams P{};
    long long J[8];
    int most;
    make_classes(g, pass, &P, J, &most);
    const int C = dgrad ? g.Cout : g.Cin, T = (int)g.taps();
    P.scatter = one_voxel(g, pass);
    P.in = P.in_hi = (const float*)in;
    P.w = (const float*)w;
    P.wsplit = (const uint16_t*)ws;
    P.wflag = (const uint32_t*)((const char*)ws + flags_at(plan.frags));
    if (!dgrad) { P.w_m = (long long)T * g.Cin; P.w_t = g.Cin; P.w_c = 1; }
    else if (P.scatter) { P.w_m = 1; P.w_t = 0; P.w_c = (long long)T * g.Cin; }
    else { P.w_m = 1; P.w_t = g.Cin; P.w_c = (long long)T * g.Cin; }
    P.out = P.out_hi = (float*)out;
    P.add = (const float*)g.add; P.ref = (const float*)g.ref; P.slope = g.slope;
    P.part = plan.splits > 1 ? (float*)((char*)ws + pack_bytes(plan.frags)) : nullptr;
    P.C = make_div(C);
    P.csplit = P.pitch = C;
    const int M = dgrad ? g.Cin : g.Cout;
    P.out_pitch = M; P.out_split = 1 << 30;
    if (!dgrad) {
        P.isd = g.sD; P.ish = g.sH; P.isw = g.sW; P.osd = P.osh = P.osw = 1;
        P.iD = g.D; P.iH = g.H; P.iW = g.W; P.oD = g.Do; P.oH = g.Ho; P.oW = g.Wo;
        if (g.hi) { P.in_hi = (const float*)g.hi; P.csplit = P.pitch = C / 2; }
    } else {
        P.isd = P.ish = P.isw = 1; P.osd = g.sD; P.osh = g.sH; P.osw = g.sW;
        P.iD = g.Do; P.iH = g.Ho; P.iW = g.Wo; P.oD = g.D; P.oH = g.H; P.oW = g.W;
        if (g.hi) P.out_hi = (float*)g.hi;
        if (g.hi && plan.splits == 1) P.out_pitch = P.out_split = M / 2;   // (partial sums keep the channels of both halves together)
    }
    P.in_bytes = (uint32_t)((long long)g.N * P.iD * P.iH * P.iW * P.pitch * 4);
    P.kH = g.kH; P.kW = g.kW;
    P.sC = make_div(g.Cin);
    P.splits = plan.splits; P.MT = plan.MT; P.tiles = (int)plan.tiles; P.out_elems = plan.out_elems;
    int tile = 0;
    for (int c = 0; c < P.ncls; ++c) {
        P.cls[c].J = (int)J[c];
        P.cls[c].PT = (int)((J[c] + BN - 1) / BN);
        P.cls[c].tile0 = tile;
        tile += P.cls[c].PT * plan.MT;
    }
    const size_t lds = 2 * STAGE + sizeof(Tables);
    static std::atomic<bool> attr_set{false};   // set once per process; a second thread racing here repeats an idempotent call
    if (!attr_set) {
        for (const void* f : {(const void*)igf_kernel<2, 2, 2, true>, (const void*)igf_kernel<2, 2, 2, false>, (const void*)igf_kernel<2, 2, 1, true>,
                              (const void*)igf_kernel<4, 1, 1, true>}) {
            hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) { note_hip_error(e); return MI3D_ERR_HIP; }
        }
        attr_set = true;
    }
    if (plan.frags) igf_pack_kernel<<<(unsigned)((plan.frags + 3) / 4), 256, 0, s>>>(P, (uint16_t*)ws, (uint32_t*)((char*)ws + flags_at(plan.frags)), (int)plan.frags);
    int st = check_launch();
    if (st) return st;
    const unsigned grid = (unsigned)(plan.tiles * plan.splits);
    if (plan.v == 0 && plan.most > 8 * plan.splits) igf_kernel<2, 2, 2, true><<<grid, 256, lds, s>>>(P);
    else if (plan.v == 0) igf_kernel<2, 2, 2, false><<<grid, 256, lds, s>>>(P);
    else if (plan.v == 1) igf_kernel<2, 2, 1, true><<<grid, 256, lds, s>>>(P);
    else igf_kernel<4, 1, 1, true><<<grid, 256, lds, s>>>(P);
    st = check_launch();
    if (st || plan.splits == 1) return st;
    long long blocks = (plan.out_elems + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    igf_sum_kernel<<<(unsigned)blocks, 256, 0, s>>>(P.part, plan.out_elems, plan.splits, M, dgrad && g.hi ? M / 2 : M, (float*)out, (float*)(dgrad ? g.hi : nullptr),
                                                    P.add, P.ref, P.slope);
    return check_launch();
}

}  // namespace mi3d
