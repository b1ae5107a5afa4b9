// fp32 convolution on the fp32 matrix cores (v_mfma_f32_32x32x2_f32): forward, data gradient and weight gradient of
// the feature-map layers of Section 3.1 for any kernel extent up to 3 and stride up to 2, the precision the paper's
// own runs presumably used (Section 4.1 names none).
//
// Forward pass and data gradient are one kernel, a "gather convolution" over an iteration space j:
//     out[n, os * j + oo, m] = sum over taps t and channels k of  in[n, is * j + delta_t, k] * wt[t][k][m]
// per axis.  The forward pass has is = stride, os = 1, delta_t = t - pad.  The stride-1 data gradient reads dy with
// delta_t = pad - t and the weights with their channel roles swapped.  The stride-2 data gradient is split into the 8
// parity classes of the output position: class pi writes positions 2 j + pi and sees the taps t with pi + pad - t
// even, at delta_t = (pi + pad - t) / 2, so no product with a structural zero is formed.  The 2x2x2 stride-2
// up-sampling layers (run as the data gradient of a 2x2x2 / stride-2 convolution) are the same thing with one tap per
// class.
// MFMA roles: A = weights (M = 32 output channels, K = 2 contracted channels), B = input (N = 32 positions along W),
// so a lane ends with 16 output channels of one position.  A workgroup (4 waves) owns 8 rows x 32 columns of one j
// plane for 32 or 64 output channels and stages, per group of taps that share an input plane and per chunk of the
// contracted channels, the input patch with halo and the group's weights in LDS.  An fp32 MFMA takes 64 cycles and
// needs 8 bytes of operands per lane, so plain 4-byte LDS reads keep it fed.
//
// Weight gradient: contraction over positions, A = dy (M = 32 output channels, K = 2 neighbouring positions along W),
// B = x at the tap's shift (N = 32 input channels); a workgroup owns one 32 x 32 block of (cout, cin) for all taps
// (dealt round-robin to its 8 waves) over a range of position tiles; per-workgroup partial sums are added in index
// order by reduce_partials (bit-reproducible).
#include "ig_common.h"
#include "mi3d_internal.h"
#include "split_f32.h"

namespace mi3d {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// j tile of a workgroup: 256 positions, 8 rows x 32 columns or 16 x 16 (whichever covers the plane with fewer positions
// outside it: 48 columns are 3 x 16 but 2 x 32 with a quarter wasted, 12 x 12 fits one 16 x 16 tile).  A wave owns two
// MFMA blocks of 32 positions; position f of the tile is row f / TJW, column f % TJW.
constexpr int MAX_TAPS = 27;
// Waves of a convolution workgroup with 32 / 64 output channels.  With 64 channels eight waves take one block of 32
// positions each (72 registers instead of 107: six or seven waves per SIMD instead of four; strided forward 2.90 ->
// 2.44 ms at 192^3, the stride-1 layers 1 % faster); with 32 channels four waves of two blocks stay (eight: 96 instead
// of 103 TFLOP/s, every weight read then feeds one MFMA instead of two).
constexpr int GC_NW1 = 4, GC_NW2 = 8;
// Budget for the tiles of a stage.  40 KB makes a stage 8 contracted channels deep for the 3x3x3 layers (21 KB with
// 32 output channels per workgroup, 31 KB with 64), so that several workgroups share a CU and one's staging hides behind
// the others' MFMAs: 64->32 at 192^3 93 -> 106 TFLOP/s, 128->64 at 96^3 98 -> 112 (64 KB: 16 channels; 20 KB: 4
// channels, slower again: 92 and 100).
constexpr int LDS_SOFT = 40 * 1024;
constexpr int LDS_SOFT_STRIDED = 64 * 1024;   // forward passes with stride 2

struct GcParams {
    const float* in; const float* in2;     // input (second half of the channels of a virtually concatenated input)
    float* out; float* out2;               // output (second half of the channels of an output written as two tensors)
    const float* wpack;                    // [tap][K][Mpad] weights, M fastest, zero beyond M
    const float* ref; const float* add;    // optional epilogue operands of the output's shape (see GcEpilogue)
    float slope;
    int N, Di, Hi, Wi, K;                  // input extents, contracted channels
    int Do, Ho, Wo, M, Mpad;               // output extents, output channels (padded to 32)
    int in_pitch, in_split;                // channels per voxel of each input tensor; first channel that lives in in2
    int out_pitch, out_split;              // same for the output
    int Jd, Jh, Jw, JHT, JWT, MT;          // iteration space, tiles
    int isd, ish, isw, osd, osh, osw, ood, ooh, oow;
    int ntaps, ngroups;
    int gstart[4];                         // taps of group g: gstart[g] .. gstart[g + 1] - 1 (sorted by plane offset)
    int gd[3];                             // input plane offset of each group
    signed char th[MAX_TAPS], tw[MAX_TAPS];  // row / column offsets of each tap
    signed char tapidx[MAX_TAPS];            // its index in the layer's own tap order (slot in wpack)
    int hmin, wmin, prows, pcols;          // smallest offsets; patch extent in LDS
    int TJH, TJW, LW;                      // tile rows, columns (a power of two, 2^LW)
    int flat;                              // 1: row-major tiles over the whole width (TJW = Jw, JWT = 1, JHT = tiles of 256 positions)
    int CK;                                // contracted channels per stage (even)
};

__device__ __forceinline__ f32x16 mfma2(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// This lane's position in each of the wave's blocks: row and column inside the tile, inside the plane or not;
// active: the wave has a position inside the plane (its first one; waves without one issue no MFMA).
template <int NB>
__device__ __forceinline__ void gconv_positions(const GcParams& P, int jht, int jwt, int wave, int ln, int& jh0, int& jw0, int& tr0, int& tc0, int& tr1,
                                                int& tc1, bool& ok0, bool& ok1, bool& active) {
    const int f0 = (NB * wave) * 32 + ln, f1 = NB == 2 ? f0 + 32 : f0;
    if (P.flat) {
        const int base = jht * 256, total = P.Jh * P.Jw;
        jh0 = base / P.Jw; jw0 = 0;
        const int r0 = (base + f0) / P.Jw, r1 = (base + f1) / P.Jw;
        ok0 = base + f0 < total; ok1 = base + f1 < total;
        tr0 = ok0 ? r0 - jh0 : 0; tc0 = ok0 ? base + f0 - r0 * P.Jw : 0;     // (outside: any staged position)
        tr1 = ok1 ? r1 - jh0 : 0; tc1 = ok1 ? base + f1 - r1 * P.Jw : 0;
        active = base + (NB * wave) * 32 < total;
    } else {
        jh0 = jht * P.TJH; jw0 = jwt * P.TJW;
        tr0 = f0 >> P.LW; tc0 = f0 & (P.TJW - 1); tr1 = f1 >> P.LW; tc1 = f1 & (P.TJW - 1);
        ok0 = jh0 + tr0 < P.Jh && jw0 + tc0 < P.Jw; ok1 = jh0 + tr1 < P.Jh && jw0 + tc1 < P.Jw;
        active = jh0 + (((NB * wave) * 32) >> P.LW) < P.Jh;
    }
}

// The work of one workgroup: tile (n, jd, jht, jwt) of the iteration space, output channel block mt.
// CB = 32-wide blocks of output channels per workgroup
template <int CB, int NW, int NB>
__device__ __forceinline__ void gconv_tile(const GcParams& P, float* lds_f, int n, int jd, int jht, int jwt, int mt) {
    constexpr int NT = 64 * NW;   // threads; NB = blocks of 32 positions per wave (the tile has NW * NB * 32 positions)
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int ln = lane & 31, half = lane >> 5;
    const int xp = P.CK + 1;                                   // channel pitch of a staged voxel (odd: no bank conflicts)
    float* xs = lds_f;                                         // [prows][pcols][CK + 1]
    float* ws = lds_f + ((P.prows * P.pcols * xp + 3) & ~3);   // [taps of the group][CK][32 CB]
    const int m0 = mt * 32 * CB;
    int jh0, jw0, tr0, tc0, tr1, tc1;
    bool ok0, ok1, active;
    gconv_positions<NB>(P, jht, jwt, wave, ln, jh0, jw0, tr0, tc0, tr1, tc1, ok0, ok1, active);

    f32x16 acc[NB][CB];
#pragma unroll
    for (int r = 0; r < NB; ++r)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][cb][i] = 0.f;

    const long long in_plane = (long long)P.Hi * P.Wi * P.in_pitch;
    for (int c0 = 0; c0 < P.K; c0 += P.CK) {
        const bool hi_in = c0 >= P.in_split;
        const float* src = (hi_in ? P.in2 : P.in) + (long long)n * P.Di * in_plane + (hi_in ? c0 - P.in_split : c0);
        for (int g = 0; g < P.ngroups; ++g) {
            const int id = P.isd * jd + P.gd[g];
            const int t0 = P.gstart[g], nt = P.gstart[g + 1] - t0;
            __syncthreads();   // the previous stage's readers are done
            // ---- input patch: rows ish * jh0 + hmin .., columns isw * jw0 + wmin .., channels c0 .. c0 + CK - 1
            const bool plane_ok = id >= 0 && id < P.Di;
            const int nvox = P.prows * P.pcols;
            if ((P.CK & 3) == 0 && (P.in_pitch & 3) == 0) {
                const int q4 = P.CK >> 2;
                for (int e = t; e < nvox * q4; e += NT) {
                    const int v = e / q4, q = e - v * q4;
                    const int pr = v / P.pcols, pc = v - pr * P.pcols;
                    const int ih = P.ish * jh0 + P.hmin + pr, iw = P.isw * jw0 + P.wmin + pc;
                    float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (plane_ok && ih >= 0 && ih < P.Hi && iw >= 0 && iw < P.Wi)
                        val = *(const float4*)(src + (long long)id * in_plane + ((long long)ih * P.Wi + iw) * P.in_pitch + 4 * q);
                    float* d = xs + v * xp + 4 * q;
                    d[0] = val.x; d[1] = val.y; d[2] = val.z; d[3] = val.w;
                }
            } else {   // ragged channel counts: element by element, zero beyond K
                for (int e = t; e < nvox * P.CK; e += NT) {
                    const int v = e / P.CK, q = e - v * P.CK;
                    const int pr = v / P.pcols, pc = v - pr * P.pcols;
                    const int ih = P.ish * jh0 + P.hmin + pr, iw = P.isw * jw0 + P.wmin + pc;
                    float val = 0.f;
                    if (plane_ok && c0 + q < P.K && ih >= 0 && ih < P.Hi && iw >= 0 && iw < P.Wi)
                        val = src[(long long)id * in_plane + ((long long)ih * P.Wi + iw) * P.in_pitch + q];
                    xs[v * xp + q] = val;
                }
            }
            // ---- weights of the group's taps: ws[tap][k][m] for m in this workgroup's blocks
            const int wrow = 32 * CB;
            for (int e = t; e < nt * P.CK * (wrow >> 2); e += NT) {
                const int m4 = e % (wrow >> 2);
                const int k = (e / (wrow >> 2)) % P.CK;
                const int tp = e / ((wrow >> 2) * P.CK);
                float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
                if (c0 + k < P.K && m0 + 4 * m4 < P.Mpad)
                    val = *(const float4*)(P.wpack + ((long long)P.tapidx[t0 + tp] * P.K + c0 + k) * P.Mpad + m0 + 4 * m4);
                *(float4*)(ws + (tp * P.CK + k) * wrow + 4 * m4) = val;
            }
            __syncthreads();
            if (!plane_ok) continue;   // zero padding plane: nothing to add (uniform over the workgroup)
            if (!active) continue;     // no block of this wave has a position inside the plane (uniform over the wave)
            // ---- MFMAs: per tap and pair of contracted channels, 2 rows x CB blocks
            for (int tp = 0; tp < nt; ++tp) {
                const int dh = P.th[t0 + tp] - P.hmin, dw = P.tw[t0 + tp] - P.wmin;
                const float* b0 = xs + ((tr0 * P.ish + dh) * P.pcols + tc0 * P.isw + dw) * xp + half;
                const float* b1 = xs + ((tr1 * P.ish + dh) * P.pcols + tc1 * P.isw + dw) * xp + half;
                const float* a = ws + (tp * P.CK + half) * wrow + ln;
                if constexpr (NB == 2) {
#pragma unroll 4
                    for (int kk = 0; kk < P.CK; kk += 2) {
                        const float x0 = b0[kk], x1 = b1[kk];
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) {
                            const float wv = a[kk * wrow + 32 * cb];
                            acc[0][cb] = mfma2(wv, x0, acc[0][cb]);
                            acc[1][cb] = mfma2(wv, x1, acc[1][cb]);
                        }
                    }
                } else {
#pragma unroll 4
                    for (int kk = 0; kk < P.CK; kk += 2) {
                        const float x0 = b0[kk];
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) acc[0][cb] = mfma2(a[kk * wrow + 32 * cb], x0, acc[0][cb]);
                    }
                }
            }
        }
    }
    // ---- epilogue: lane (position ln, half) holds output channels 8 (i / 4) + 4 half + i % 4 of each block.
    // The optional operands (second gradient, reference tensor of the derivative) are read 16 bytes at a time (as single
    // floats the stride-2 data gradient with both took 5.5 ms instead of 3.5 at 192^3); a block's operands are
    // requested right where they are used: requesting a whole row's ahead of time costs 15 to 48 registers and, through
    // the lower occupancy, more than it gains.  (Shared with f32s_gconv_kernel as a function, these lines take 15 registers more
    // here: the three passes of 64->128 up-sampling at 96^3 874 -> 913 us.)
    const bool vec = (P.out_pitch & 3) == 0;
#pragma unroll
    for (int r = 0; r < NB; ++r) {
        const int jh = jh0 + (r ? tr1 : tr0), jw = jw0 + (r ? tc1 : tc0);
        if (!(r ? ok1 : ok0)) continue;
        const int od = P.osd * jd + P.ood, oh = P.osh * jh + P.ooh, ow = P.osw * jw + P.oow;
        const long long vox = (((long long)n * P.Do + od) * P.Ho + oh) * P.Wo + ow;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                int c = m0 + 32 * cb + 8 * g4 + 4 * half;
                if (c >= P.M) continue;
                float v[4] = {acc[r][cb][4 * g4], acc[r][cb][4 * g4 + 1], acc[r][cb][4 * g4 + 2], acc[r][cb][4 * g4 + 3]};
                const bool hi_out = c >= P.out_split;
                float* dst = (hi_out ? P.out2 : P.out) + vox * P.out_pitch + (hi_out ? c - P.out_split : c);
                const long long eoff = vox * P.out_pitch + (hi_out ? c - P.out_split : c);   // same offset in ref / add (never split)
                const int nv = P.M - c < 4 ? P.M - c : 4;
                if (vec && nv == 4) {
                    const float4 a4 = P.add ? *(const float4*)(P.add + eoff) : make_float4(0.f, 0.f, 0.f, 0.f);
                    const float4 r4 = P.ref ? *(const float4*)(P.ref + eoff) : make_float4(0.f, 0.f, 0.f, 0.f);
                    const float ad[4] = {a4.x, a4.y, a4.z, a4.w};
                    const float rf[4] = {r4.x, r4.y, r4.z, r4.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float x = v[i];
                        if (P.add) x += ad[i];
                        if (P.ref) x = rf[i] > 0.f ? x : P.slope * x;
                        else x = x > 0.f ? x : P.slope * x;
                        v[i] = x;
                    }
                    *(float4*)dst = make_float4(v[0], v[1], v[2], v[3]);
                    continue;
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (i >= nv) break;
                    float x = v[i];
                    if (P.add) x += P.add[eoff + i];
                    if (P.ref) x = P.ref[eoff + i] > 0.f ? x : P.slope * x;
                    else x = x > 0.f ? x : P.slope * x;
                    v[i] = x;
                }
                for (int i = 0; i < nv; ++i) dst[i] = v[i];
            }
    }
}

template <int CB, int NW, int NB>
__global__ void __launch_bounds__(64 * NW, 2) f32_gconv_kernel(GcParams P) {
    extern __shared__ __attribute__((aligned(16))) float lds_f[];
    long long u = blockIdx.x;
    const int mt = (int)(u % P.MT); u /= P.MT;
    const int jwt = (int)(u % P.JWT); u /= P.JWT;
    const int jht = (int)(u % P.JHT); u /= P.JHT;
    const int jd = (int)(u % P.Jd);
    const int n = (int)(u / P.Jd);
    gconv_tile<CB, NW, NB>(P, lds_f, n, jd, jht, jwt, mt);
}

// ---- fp32 products from bf16 matrix instructions -----------------------------------------------------------------------
// The same gather convolution with each fp32 operand taken apart into three bf16 numbers, v = a + b + c exactly (a the
// nearest bf16 to v, b to v - a, c the rest: 3 x 8 significant bits and two signs hold the 24 of v).  Of the nine products
// the six a a', a b', b a', a c', c a', b b' are formed with v_mfma_f32_32x32x16_bf16 and added in fp32.  With |b| <= 2^-8 |v|
// and |c| <= 2^-17 |v| the three left out can reach 2^-24 of the product, one rounding of a single fp32 product (the worst
// operands, 1 + 2^-8 - 2^-17, are a test); of normal random operands 3.5 % exceed 2^-26, their root mean square is
// a tenth of 2^-24.  An accumulator
// is rounded 6 times per 16 contracted channels instead of 8 to 16 times, and that decides.  Measured
// against 64 bits (2-norm, fp32 instructions -> this kernel): 32->32 at 8 x 48 x 48 5.0e-7 -> 4.3e-7, 320->320 at 5 x 12 x 12
// 1.5e-6 -> 1.35e-6, 640->32 2.2e-6 -> 2.0e-6; operands that are all the worst one 6e-8 (0.99 x 2^-24) with either.
//
// Bound: the fp32 matrix instructions need 64 cycles for 32x32x2, six bf16 ones for 32x32x16 need 6 x 32: a ceiling 2.7
// times as high.  Forward pass with its packing launch, fp32 instructions -> this kernel: 32->32 at 128^3, N = 2 2225 -> 1444 us
// (104 -> 161 TFLOP/s), 64->64 at 64^3, N = 2 1060 -> 600 (109 -> 193), 64->32 at 45 x 75 x 91 470 -> 279, 256->256 at 16^3,
// N = 2 486 -> 217; on the smallest volumes the way of the weights to the few waves at work is the bound, 320->320 at 8^3,
// N = 2 608 -> 319.
// A workgroup (4 waves) owns 256 positions x 32 or 64 output channels, a wave two blocks of 32 positions.  A stage is 16
// contracted channels of one input plane: the patch is requested during the previous stage's MFMAs, taken apart on its way
// to LDS ([part][voxel][16 channels], 32 bytes per voxel, the two 16-byte halves swapped every 8 voxels so that 16
// neighbouring voxels cover all banks) and read by all taps of the plane.  Weights are packed in fragment order by
// f32s_pack_kernel and read from there (L1 / L2) one or two taps ahead of their use.
//
// A value outside the range of the split (split_f32.h; infinities and NaN among them) sends its stage (a weight: that stage of
// all tiles of its channel block) through v_mfma_f32_32x32x2_f32 on the values themselves: infinities, NaN and overflow come
// out as they do from the fp32 instructions.  Forward pass 64->64 at 64^3, N = 2: 577 us, with one such activation 577, with
// one such weight (a stage in twelve) 653, with such activations in every stage 1365 (the kernel of the fp32 instructions 1155).
constexpr int SP_NT = 256, SP_CK = 16;
constexpr int SP_BITS = 256;                       // stages told apart by their weights' flags
constexpr int SP_MAXV = 448;                       // staged voxels (bound of the dispatch rule)
constexpr int SP_NPX = SP_MAXV * (SP_CK / 4) / SP_NT;   // 16-byte pieces of the patch per thread

struct GsParams {
    GcParams c;
    const uint16_t* wsplit;      // [tap][K / 16][Mpad / 32][3 parts][64 lanes][8]
    const uint32_t* wflag;       // [Mpad / 32][tap][K / 16]: a value of this fragment cannot be split
    const float* w;              // the layer's own weights: element (m, tap, k) at m * w_m + tap * w_t + k * w_k
    long long w_m, w_t, w_k;
    int T;
    uint32_t taps[MAX_TAPS];     // voxel offset in the patch | index in the layer's tap order << 16 (scalar loads have no bytes)
};

__device__ __forceinline__ f32x16 mfma16(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }

// One wave per fragment: 32 output channels x 16 contracted channels of a tap.  grid.x * 4 waves >= T * K / 16 * Mpad / 32.
__global__ void __launch_bounds__(256) f32s_pack_kernel(const float* __restrict__ w, uint16_t* __restrict__ out, uint32_t* __restrict__ flag, int T, int K,
                                                        int M, int MB, long long w_m, long long w_t, long long w_k) {
    const int lane = threadIdx.x & 63, KC = K / SP_CK;
    const int frag = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (frag >= T * KC * MB) return;
    const int mb = frag % MB, r = frag / MB, kc = r % KC, tap = r / KC;
    const int m = mb * 32 + (lane & 31), k0 = kc * SP_CK + 8 * (lane >> 5);
    float v[8];
    SplitRange range;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        v[i] = m < M ? w[m * w_m + tap * w_t + (k0 + i) * w_k] : 0.f;
        range.add(v[i]);
    }
    uint32_t o[4][3];
#pragma unroll
    for (int i = 0; i < 4; ++i) split2(v[2 * i], v[2 * i + 1], o[i]);
#pragma unroll
    for (int p = 0; p < 3; ++p) *(uint4*)(out + (((long long)frag * 3 + p) * 64 + lane) * 8) = uint4{o[0][p], o[1][p], o[2][p], o[3][p]};
    const bool any = __any(range.exceeded());
    if (lane == 0) flag[(mb * T + tap) * KC + kc] = any ? 1u : 0u;
}

// Epilogue of one block of 32 channels from m0 on, at position (jh, jw) of plane jd.
__device__ __forceinline__ void split_store(const GcParams& P, f32x16 a, int n, int jd, int jh, int jw, int m0, int half) {
    const int od = P.osd * jd + P.ood, oh = P.osh * jh + P.ooh, ow = P.osw * jw + P.oow;
    const long long vox = (((long long)n * P.Do + od) * P.Ho + oh) * P.Wo + ow;
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
        const int c = m0 + 8 * g4 + 4 * half;
        if (c >= P.M) continue;
        const bool hi_out = c >= P.out_split, full = (P.out_pitch & 3) == 0 && P.M - c >= 4;
        const int nv = P.M - c < 4 ? P.M - c : 4;
        const long long e = vox * P.out_pitch + (hi_out ? c - P.out_split : c);   // (add and ref never come with a split output)
        float* dst = (hi_out ? P.out2 : P.out) + e;
        float v[4], ad[4] = {0.f, 0.f, 0.f, 0.f}, rf[4] = {0.f, 0.f, 0.f, 0.f};
        if (full) {
            if (P.add) *(float4*)ad = *(const float4*)(P.add + e);
            if (P.ref) *(float4*)rf = *(const float4*)(P.ref + e);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (P.add && i < nv) ad[i] = P.add[e + i];
                if (P.ref && i < nv) rf[i] = P.ref[e + i];
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float x = a[4 * g4 + i];
            if (P.add) x += ad[i];
            v[i] = (P.ref ? rf[i] : x) > 0.f ? x : P.slope * x;
        }
        if (full) *(float4*)dst = make_float4(v[0], v[1], v[2], v[3]);
        else
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i < nv) dst[i] = v[i];
    }
}

// CB = 32-wide blocks of output channels per workgroup, NTC = taps of a plane (every group has that many)
template <int CB, int NTC>
__global__ void __launch_bounds__(SP_NT, 2) f32s_gconv_kernel(GsParams Q) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const GcParams& P = Q.c;
    constexpr int NB = 2, WANT = CB == 2 ? 2 : 3, AHEAD = NTC < WANT ? NTC : WANT;   // weight fragments held: this tap's and the next ones'
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int ln = lane & 31, half = lane >> 5;
    int u = blockIdx.x;
    const int mt = u % P.MT; u /= P.MT;
    const int jwt = u % P.JWT; u /= P.JWT;
    const int jht = u % P.JHT; u /= P.JHT;
    const int jd = u % P.Jd, n = u / P.Jd;
    const int m0 = mt * 32 * CB;
    int jh0, jw0, tr0, tc0, tr1, tc1;
    bool ok0, ok1, active;
    gconv_positions<NB>(P, jht, jwt, wave, ln, jh0, jw0, tr0, tc0, tr1, tc1, ok0, ok1, active);
    const int nvox = P.prows * P.pcols, part = nvox * 32;
    uint32_t* bad_lds = (uint32_t*)(lds + 3 * part);   // [0], [1]: patch of the stage of that parity; then a bit per stage's weights

    f32x16 acc[NB][CB];
#pragma unroll
    for (int r = 0; r < NB; ++r)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][cb][i] = 0.f;

    // this thread's pieces of the patch: offset inside an input plane, or -1 for zero padding
    int gofs[SP_NPX];
#pragma unroll
    for (int i = 0; i < SP_NPX; ++i) {
        const int e = t + SP_NT * i, v = e >> 2, pr = v / P.pcols, pc = v - pr * P.pcols;
        const int ih = jh0 + P.hmin + pr, iw = jw0 + P.wmin + pc;
        gofs[i] = v < nvox && ih >= 0 && ih < P.Hi && iw >= 0 && iw < P.Wi ? (ih * P.Wi + iw) * P.in_pitch + 4 * (e & 3) : -1;
    }
    // groups whose input plane exists (zero planes add nothing)
    const int KC = P.K / SP_CK;
    unsigned gmask = 0;
    for (int g = 0; g < P.ngroups; ++g) {
        const int id = P.isd * jd + P.gd[g];
        gmask |= (id >= 0 && id < P.Di ? 1u : 0u) << g;
    }
    const int ngv = __popc(gmask), stages = KC * ngv;
    const long long in_plane = (long long)P.Hi * P.Wi * P.in_pitch;
    auto stage_group = [&](int s) {   // the (s % ngv)-th existing group
        unsigned m = gmask;
        for (int r = s % ngv; r > 0; --r) m &= m - 1;
        return __ffs(m) - 1;
    };
    float4 px[SP_NPX];
    auto request = [&](int s) {
        const int c0 = s / ngv * SP_CK, g = stage_group(s);
        const bool hi_in = c0 >= P.in_split;
        const float* src = (hi_in ? P.in2 : P.in) + ((long long)n * P.Di + P.isd * jd + P.gd[g]) * in_plane + (hi_in ? c0 - P.in_split : c0);
#pragma unroll
        for (int i = 0; i < SP_NPX; ++i) {
            px[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (gofs[i] >= 0) px[i] = *(const float4*)(src + gofs[i]);
        }
    };
    auto slot = [&](int e) { const int v = e >> 2, q = e & 3; return v * 32 + (((q >> 1) ^ (v >> 3)) & 1) * 16 + (q & 1) * 8; };

    if (t < 2 + SP_BITS / 32) bad_lds[t] = 0;
    if (stages > 0) request(0);
    __syncthreads();
    // stages with weights that cannot be split (stages SP_BITS apart share a bit: one may go the other way needlessly)
    auto stage_bit = [&](int kc, int g) { return (kc * P.ngroups + g) & (SP_BITS - 1); };
    const int TK = Q.T * KC;
    for (int cb = 0; cb < CB; ++cb)
        if (m0 + 32 * cb < P.Mpad)
            for (int e = t; e < TK; e += SP_NT)
                if (Q.wflag[(m0 / 32 + cb) * TK + e] != 0)
                    for (int k = 0; k < P.ntaps; ++k)
                        if ((int)(Q.taps[k] >> 16) == e / KC) {
                            const int bit = stage_bit(e % KC, k / NTC);
                            atomicOr(&bad_lds[2 + (bit >> 5)], 1u << (bit & 31));
                        }
    const int MB = P.Mpad / 32;
    const int vb[NB] = {tr0 * P.pcols + tc0, tr1 * P.pcols + tc1};
    for (int s = 0; s < stages; ++s) {
        const int kc = s / ngv, g = stage_group(s), tap0 = P.gstart[g];
        if (s) __syncthreads();   // the previous stage's readers are done
        SplitRange range;
#pragma unroll
        for (int i = 0; i < SP_NPX; ++i) {
            const int e = t + SP_NT * i;
            if ((e >> 2) >= nvox) break;
            range.add(px[i]);
            uint32_t lo[3], hi[3];
            split2(px[i].x, px[i].y, lo);
            split2(px[i].z, px[i].w, hi);
            char* d = lds + slot(e);
#pragma unroll
            for (int p = 0; p < 3; ++p) *(uint2*)(d + p * part) = uint2{lo[p], hi[p]};
        }
        if (__any(range.exceeded()) && lane == 0) bad_lds[s & 1] = 1;
        bf16x8 wf[AHEAD][CB][3];
        auto weights = [&](int tp, bf16x8 (&f)[CB][3]) {
            const int tap = (int)(Q.taps[tap0 + tp] >> 16);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                // (a last block of 64 with 32 channels: the second half reads the first again and is not stored)
                const int mb = m0 / 32 + cb < MB ? m0 / 32 + cb : MB - 1;
                const uint16_t* q = Q.wsplit + (((long long)tap * KC + kc) * MB + mb) * (3 * 512) + lane * 8;
#pragma unroll
                for (int p = 0; p < 3; ++p) f[cb][p] = *(const bf16x8*)(q + p * 512);
            }
        };
#pragma unroll
        for (int a = 0; a < AHEAD - 1; ++a) weights(a, wf[a]);
        if (AHEAD == 1) weights(0, wf[0]);
        __syncthreads();
        const int bit = stage_bit(kc, g);
        const bool plain = __builtin_amdgcn_readfirstlane(bad_lds[s & 1] | (bad_lds[2 + (bit >> 5)] >> (bit & 31) & 1)) != 0;
        if (t == 0) bad_lds[1 - (s & 1)] = 0;   // (next written behind the next stage's first barrier)
        if (plain) {
            // raw bits in two halves take the place of the parts; weights come as they are
            __syncthreads();
#pragma unroll
            for (int i = 0; i < SP_NPX; ++i) {
                const int e = t + SP_NT * i;
                if ((e >> 2) >= nvox) break;
                const uint4 b = __builtin_bit_cast(uint4, px[i]);
                char* d = lds + slot(e);
                *(uint2*)d = uint2{b.x >> 16 | (b.y & 0xFFFF0000u), b.z >> 16 | (b.w & 0xFFFF0000u)};
                *(uint2*)(d + part) = uint2{(b.x & 0xFFFFu) | b.y << 16, (b.z & 0xFFFFu) | b.w << 16};
            }
            __syncthreads();
            if (s + 1 < stages) request(s + 1);
            if (!active) continue;
            for (int tp = 0; tp < NTC; ++tp) {
                const int vo = (int)(Q.taps[tap0 + tp] & 0xFFFFu);
                const float* wt = Q.w + (long long)(Q.taps[tap0 + tp] >> 16) * Q.w_t;
#pragma unroll 1
                for (int i = 0; i < 8; ++i) {
                    float xv[NB];
#pragma unroll
                    for (int r = 0; r < NB; ++r) {
                        const int v = vb[r] + vo;
                        const uint16_t* q = (const uint16_t*)(lds + v * 32 + ((half ^ (v >> 3)) & 1) * 16) + i;
                        xv[r] = __builtin_bit_cast(float, (uint32_t)q[0] << 16 | *(const uint16_t*)((const char*)q + part));
                    }
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        const int m = m0 + 32 * cb + ln, k = kc * SP_CK + 8 * half + i;
                        const float wv = m < P.M ? wt[m * Q.w_m + k * Q.w_k] : 0.f;
#pragma unroll
                        for (int r = 0; r < NB; ++r) acc[r][cb] = mfma2(wv, xv[r], acc[r][cb]);
                    }
                }
            }
            continue;
        }
        if (s + 1 < stages) request(s + 1);
        if (!active) continue;
#pragma unroll
        for (int tp = 0; tp < NTC; ++tp) {
            if (AHEAD > 1 && tp + AHEAD - 1 < NTC) weights(tp + AHEAD - 1, wf[(tp + AHEAD - 1) % AHEAD]);
            const int vo = (int)(Q.taps[tap0 + tp] & 0xFFFFu);
            bf16x8 xf[NB][3];
#pragma unroll
            for (int r = 0; r < NB; ++r) {
                const int v = vb[r] + vo;
                const char* q = lds + v * 32 + ((half ^ (v >> 3)) & 1) * 16;
#pragma unroll
                for (int p = 0; p < 3; ++p) xf[r][p] = *(const bf16x8*)(q + p * part);
            }
            // small products first
            constexpr int PW[6] = {2, 0, 1, 1, 0, 0}, PX[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int r = 0; r < NB; ++r) acc[r][cb] = mfma16(wf[tp % AHEAD][cb][PW[q]], xf[r][PX[q]], acc[r][cb]);
        }
    }
#pragma unroll
    for (int r = 0; r < NB; ++r) {
        if (!(r ? ok1 : ok0)) continue;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) split_store(P, acc[r][cb], n, jd, jh0 + (r ? tr1 : tr0), jw0 + (r ? tc1 : tc0), m0 + 32 * cb, half);
    }
}

// The parity classes of a stride-2 data gradient in one launch.  Workgroups are dealt to the 8 XCDs by index modulo
// 8, so tile t goes to XCD t % 8 and its classes follow each other there: b = 8 (ncls (t / 8) + class) + t % 8.  The
// classes of a tile read the same input patch, which then comes from that XCD's L2 for all but the first, and
// every XCD gets every class (class = b % 8 would hand each XCD one class).  Used where the classes have the same
// work each.  The grid spans the largest iteration space of the classes; a workgroup whose tile lies
// outside its class's leaves at once.
struct GcMulti {
    GcParams p[8];
    int ncls, MT, JWT, JHT, Jd;
    long long tiles;      // N * Jd * JHT * JWT * MT of the spanning grid
};
static_assert(sizeof(GcMulti) <= 4096, "kernel arguments");

template <int CB, int NW>
__global__ void __launch_bounds__(64 * NW, 2) f32_gconv_classes_kernel(GcMulti Q) {
    extern __shared__ __attribute__((aligned(16))) float lds_f[];
    const long long r = blockIdx.x >> 3;
    const int cls = (int)(r % Q.ncls);
    long long u = (r / Q.ncls) * 8 + (blockIdx.x & 7);
    if (u >= Q.tiles) return;
    const int mt = (int)(u % Q.MT); u /= Q.MT;
    const int jwt = (int)(u % Q.JWT); u /= Q.JWT;
    const int jht = (int)(u % Q.JHT); u /= Q.JHT;
    const int jd = (int)(u % Q.Jd);
    const int n = (int)(u / Q.Jd);
    const GcParams& P = Q.p[cls];
    if (mt >= P.MT || jwt >= P.JWT || jht >= P.JHT || jd >= P.Jd) return;   // (uniform over the workgroup)
    gconv_tile<CB, NW, 8 / NW>(P, lds_f, n, jd, jht, jwt, mt);
}

// wpack[t][k][m] (m padded to Mpad with zeros) from w[co][t][ci]; swap = 0: (k, m) = (ci, co); swap = 1: (k, m) = (co, ci)
__global__ void __launch_bounds__(256) f32_pack_kernel(const float* __restrict__ w, float* __restrict__ wpack, int Cout, int Cin, int T, int Mpad, int swap) {
    const int K = swap ? Cout : Cin, M = swap ? Cin : Cout;
    const long long total = (long long)T * K * Mpad;
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int m = (int)(idx % Mpad);
    const int k = (int)((idx / Mpad) % K);
    const int t = (int)(idx / ((long long)Mpad * K));
    float v = 0.f;
    if (m < M) {
        const int co = swap ? k : m, ci = swap ? m : k;
        v = w[((long long)co * T + t) * Cin + ci];
    }
    wpack[idx] = v;
}

// ---- weight gradient ------------------------------------------------------------------------------------------------
struct WgParams {
    const float* x; const float* x2;   // input (second half of the channels of a virtually concatenated input)
    const float* dy;
    float* part;                       // [split][Cout][T][Cin]
    int N, D, H, W, Cin, Cout, Do, Ho, Wo;
    int kD, kH, kW, sD, sH, sW, pD, pH, pW, T;
    int x_pitch, x_split;
    int TR, TW;                        // output tile: rows, columns (16 or 32)
    int HT, WT, CIT, COT, S;           // tiles per plane, channel blocks, splits
    long long units;                   // N * HT * WT * Do, Do fastest: a workgroup walks along D
    int prows, pcols;                  // staged x patch per plane
    unsigned pcols_magic;              // q / pcols == (q * pcols_magic) >> 16 for every q < prows * pcols (checked on the host)
};

// Waves, threads of a weight-gradient workgroup.  Eight waves share the staged tiles and take 3 or 4 taps each (64
// accumulator registers instead of 112 with four waves), so two workgroups per CU are four waves per SIMD: 91 -> 100
// TFLOP/s on the 192^3 layers.  Sixteen waves in one workgroup per CU: 88 (no second workgroup to compute while this
// one stages).
constexpr int WG_NW = 8, WG_NT = 64 * WG_NW;

// A workgroup walks a contiguous range of (sample, tile, output plane) units with the output plane running fastest, so
// consecutive units share input planes: the kD planes a unit needs live in a ring of kD LDS slots (plane id in slot
// id mod kD) and only the planes that were not there for the previous unit are fetched.
__global__ void __launch_bounds__(WG_NT, 2) f32_wgrad_kernel(WgParams P) {
    extern __shared__ __attribute__((aligned(16))) float lds_f[];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int ln = lane & 31, half = lane >> 5;
    constexpr int CP = 32;                                     // channels per staged voxel (reads run along the channels)
    float* dys = lds_f;                                        // [TR][TW][32]
    float* xs = lds_f + P.TR * P.TW * CP;                      // [kD ring][prows][pcols][32]
    const int pv = P.prows * P.pcols;
    int b = blockIdx.x;
    const int split = b % P.S; b /= P.S;
    const int cit = b % P.CIT;
    const int cot = b / P.CIT;
    const int ci0 = cit * 32, co0 = cot * 32;
    const bool hi_x = ci0 >= P.x_split;
    const float* xsrc = (hi_x ? P.x2 : P.x) + (hi_x ? ci0 - P.x_split : ci0);
    const bool vec_x = (P.x_pitch & 3) == 0 && (P.Cin & 3) == 0, vec_dy = (P.Cout & 3) == 0;

    constexpr int MAXA = (27 + WG_NW - 1) / WG_NW;   // taps per wave: 27 taps dealt round-robin to the waves
    f32x16 acc[MAXA];
#pragma unroll
    for (int a = 0; a < MAXA; ++a)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[a][i] = 0.f;

    const long long u0 = P.units * split / P.S, u1 = P.units * (split + 1) / P.S;
    const long long x_plane = (long long)P.H * P.W * P.x_pitch;
    const int c4 = t & 7, vslot = t >> 3;   // staging: 8 threads x 16 bytes per voxel, WG_NT / 8 voxels per pass
    long long cur_col = -1;
    int have_lo = 1, have_hi = 0;           // input planes resident in the ring (none)
    for (long long u = u0; u < u1; ++u) {
        const long long col = u / P.Do;
        const int od = (int)(u - col * P.Do);
        long long r = col;
        const int wt = (int)(r % P.WT); r /= P.WT;
        const int ht = (int)(r % P.HT);
        const int n = (int)(r / P.HT);
        const int oh0 = ht * P.TR, ow0 = wt * P.TW;
        if (col != cur_col) { cur_col = col; have_lo = 1; have_hi = 0; }
        const int need_lo = od * P.sD - P.pD, need_hi = need_lo + P.kD - 1;
        __syncthreads();   // every wave is done with the previous unit's tiles
        // ---- dy tile: TR rows x TW columns x 32 output channels (zero outside the tensor)
        if (vec_dy) {
            for (int v = vslot; v < P.TR * P.TW; v += WG_NT / 8) {
                const int tr = v / P.TW, tc = v - tr * P.TW;
                const int oh = oh0 + tr, ow = ow0 + tc;
                float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
                if (oh < P.Ho && ow < P.Wo && co0 + 4 * c4 < P.Cout)
                    val = *(const float4*)(P.dy + ((((long long)n * P.Do + od) * P.Ho + oh) * P.Wo + ow) * P.Cout + co0 + 4 * c4);
                *(float4*)(dys + v * CP + 4 * c4) = val;
            }
        } else {
            for (int e = t; e < P.TR * P.TW * 32; e += WG_NT) {
                const int c = e & 31, v = e >> 5;
                const int tr = v / P.TW, tc = v - tr * P.TW;
                const int oh = oh0 + tr, ow = ow0 + tc;
                float val = 0.f;
                if (oh < P.Ho && ow < P.Wo && co0 + c < P.Cout)
                    val = P.dy[((((long long)n * P.Do + od) * P.Ho + oh) * P.Wo + ow) * P.Cout + co0 + c];
                dys[v * CP + c] = val;
            }
        }
        // ---- x patches: rows oh0 sH - pH .., columns ow0 sW - pW .., 32 input channels, of the planes not yet in the ring
        for (int id = need_lo; id <= need_hi; ++id) {
            if (id >= have_lo && id <= have_hi) continue;
            float* dst = xs + (((id % P.kD) + P.kD) % P.kD) * pv * CP;
            const bool plane_ok = id >= 0 && id < P.D;
            const float* src = xsrc + ((long long)n * P.D + (plane_ok ? id : 0)) * x_plane;
            if (vec_x) {
                for (int q = vslot; q < pv; q += WG_NT / 8) {
                    const int pr = (int)(((unsigned)q * P.pcols_magic) >> 16), pc = q - pr * P.pcols;
                    const int ih = oh0 * P.sH - P.pH + pr, iw = ow0 * P.sW - P.pW + pc;
                    float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (plane_ok && ih >= 0 && ih < P.H && iw >= 0 && iw < P.W && ci0 + 4 * c4 < P.Cin)
                        val = *(const float4*)(src + ((long long)ih * P.W + iw) * P.x_pitch + 4 * c4);
                    *(float4*)(dst + q * CP + 4 * c4) = val;
                }
            } else {
                for (int e = t; e < pv * 32; e += WG_NT) {
                    const int c = e & 31, q = e >> 5;
                    const int pr = (int)(((unsigned)q * P.pcols_magic) >> 16), pc = q - pr * P.pcols;
                    const int ih = oh0 * P.sH - P.pH + pr, iw = ow0 * P.sW - P.pW + pc;
                    float val = 0.f;
                    if (plane_ok && ih >= 0 && ih < P.H && iw >= 0 && iw < P.W && ci0 + c < P.Cin)
                        val = src[((long long)ih * P.W + iw) * P.x_pitch + c];
                    dst[q * CP + c] = val;
                }
            }
        }
        have_lo = need_lo; have_hi = need_hi;
        __syncthreads();
        // ---- this wave's taps: K runs over pairs of neighbouring output columns
#pragma unroll
        for (int a = 0; a < MAXA; ++a) {
            const int tap = wave + WG_NW * a;
            if (tap >= P.T) break;
            const int kw = tap % P.kW, kh = (tap / P.kW) % P.kH, kd = tap / (P.kW * P.kH);
            const int id = need_lo + kd;
            const float* plane = xs + (((id % P.kD) + P.kD) % P.kD) * pv * CP;
            for (int tr = 0; tr < P.TR; ++tr) {
                const float* ap = dys + (tr * P.TW + half) * CP + ln;
                const float* bp = plane + ((tr * P.sH + kh) * P.pcols + half * P.sW + kw) * CP + ln;
#pragma unroll 4
                for (int c2 = 0; c2 < P.TW; c2 += 2)
                    acc[a] = mfma2(ap[c2 * CP], bp[c2 * P.sW * CP], acc[a]);
            }
        }
    }
    // ---- partial sums: lane holds input channel ci0 + ln, output channels co0 + 8 (i / 4) + 4 half + i % 4
    float* part = P.part + (long long)split * P.Cout * P.T * P.Cin;
#pragma unroll
    for (int a = 0; a < MAXA; ++a) {
        const int tap = wave + WG_NW * a;
        if (tap >= P.T) break;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int co = co0 + 8 * (i >> 2) + 4 * half + (i & 3), ci = ci0 + ln;
            if (co < P.Cout && ci < P.Cin) part[((long long)co * P.T + tap) * P.Cin + ci] = acc[a][i];
        }
    }
}

// Weight gradient of a 3x3x3 / stride-1 layer with at most 4 input channels (the network's first layer).  The general
// kernel above would give each tap a 32 x 32 block of which 4 columns are in use; here (tap, input channel) pairs are
// the columns: four groups of 8 taps x 4 channels, one group and one block per wave (27 taps: the last group has 3).
// Lane column ln of wave w is tap 8 w + ln / 4, channel ln % 4, so the B operand is a per-lane shifted read of the
// staged x patch ([plane ring][row][column][4 channels]); units, ring and partial sums as in the general kernel.
__global__ void __launch_bounds__(256, 2) f32_wgrad_c4_kernel(WgParams P) {
    extern __shared__ __attribute__((aligned(16))) float lds_f[];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int ln = lane & 31, half = lane >> 5;
    float* dys = lds_f;                                        // [TR][TW][32 output channels]
    float* xs = lds_f + P.TR * P.TW * 32;                      // [3 ring slots][prows][pcols][4]
    const int pv = P.prows * P.pcols;
    const int split = blockIdx.x % P.S, cot = blockIdx.x / P.S;
    const int co0 = cot * 32;
    const int tap = 8 * wave + (ln >> 2), ci = ln & 3;
    const bool col_ok = tap < 27 && ci < P.Cin;
    const int kd = tap / 9, kh = (tap / 3) % 3, kw = tap % 3;   // (tap >= 27: reads inside the staged patch, value unused)
    f32x16 acc[2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[a][i] = 0.f;

    const long long u0 = P.units * split / P.S, u1 = P.units * (split + 1) / P.S;
    const long long x_plane = (long long)P.H * P.W * P.Cin;
    const int c4 = t & 7, vslot = t >> 3;   // dy staging: 8 threads x 16 bytes per voxel, 32 voxels per pass
    long long cur_col = -1;
    int have_lo = 1, have_hi = 0;           // input planes resident in the ring (none)
    for (long long u = u0; u < u1; ++u) {
        const long long col = u / P.Do;
        const int od = (int)(u - col * P.Do);
        long long r = col;
        const int wt = (int)(r % P.WT); r /= P.WT;
        const int ht = (int)(r % P.HT);
        const int n = (int)(r / P.HT);
        const int oh0 = ht * P.TR, ow0 = wt * P.TW;
        if (col != cur_col) { cur_col = col; have_lo = 1; have_hi = 0; }
        const int need_lo = od - P.pD, need_hi = need_lo + 2;
        __syncthreads();   // every wave is done with the previous unit's tiles
        for (int v = vslot; v < P.TR * P.TW; v += 32) {
            const int tr = v / P.TW, tc = v - tr * P.TW;
            const int oh = oh0 + tr, ow = ow0 + tc;
            float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
            if (oh < P.Ho && ow < P.Wo && co0 + 4 * c4 < P.Cout)
                val = *(const float4*)(P.dy + ((((long long)n * P.Do + od) * P.Ho + oh) * P.Wo + ow) * P.Cout + co0 + 4 * c4);
            *(float4*)(dys + v * 32 + 4 * c4) = val;
        }
        for (int id = need_lo; id <= need_hi; ++id) {
            if (id >= have_lo && id <= have_hi) continue;
            float* dst = xs + ((id % 3 + 3) % 3) * pv * 4;
            const bool plane_ok = id >= 0 && id < P.D;
            const float* src = P.x + ((long long)n * P.D + (plane_ok ? id : 0)) * x_plane;
            for (int q = t; q < pv; q += 256) {
                const int pr = q / P.pcols, pc = q - pr * P.pcols;
                const int ih = oh0 - P.pH + pr, iw = ow0 - P.pW + pc;
                float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
                if (plane_ok && ih >= 0 && ih < P.H && iw >= 0 && iw < P.W) {
                    const float* px = src + ((long long)ih * P.W + iw) * P.Cin;
                    if (P.Cin == 4) val = *(const float4*)px;
                    else { val.x = px[0]; if (P.Cin > 1) val.y = px[1]; if (P.Cin > 2) val.z = px[2]; }
                }
                *(float4*)(dst + q * 4) = val;
            }
        }
        have_lo = need_lo; have_hi = need_hi;
        __syncthreads();
        const float* plane = xs + (((need_lo + kd) % 3 + 3) % 3) * pv * 4 + ci;
        for (int tr = 0; tr < P.TR; ++tr) {
            const float* ap = dys + (tr * P.TW + half) * 32 + ln;
            const float* bp = plane + ((tr + kh) * P.pcols + half + kw) * 4;
#pragma unroll 4
            for (int c2 = 0; c2 < P.TW; c2 += 4) {   // K = pairs of neighbouring output columns, two chains
                const float b0 = bp[c2 * 4], b1 = bp[(c2 + 2) * 4];
                acc[0] = mfma2(ap[c2 * 32], col_ok ? b0 : 0.f, acc[0]);
                acc[1] = mfma2(ap[(c2 + 2) * 32], col_ok ? b1 : 0.f, acc[1]);
            }
        }
    }
    // partial sums: lane column (tap, ci), rows are the output channels co0 + 8 (i / 4) + 4 half + i % 4
    float* part = P.part + (long long)split * P.Cout * 27 * P.Cin;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int co = co0 + 8 * (i >> 2) + 4 * half + (i & 3);
        if (col_ok && co < P.Cout) part[((long long)co * 27 + tap) * P.Cin + ci] = acc[0][i] + acc[1][i];
    }
}

size_t pack_bytes(const Geom& g, int pass) {
    const int K = pass == MI3D_PASS_DGRAD ? g.Cout : g.Cin, M = pass == MI3D_PASS_DGRAD ? g.Cin : g.Cout;
    const int Mpad = (M + 31) / 32 * 32;
    return ((size_t)g.taps() * K * Mpad * sizeof(float) + 255) & ~(size_t)255;
}

void wgrad_layout(const Geom& g, WgParams* P) {
    P->TR = 2;
    P->TW = (g.sW == 1) ? 32 : 16;
    // (2x2x2 stride 2: one tap per wave and 16 MFMAs per tile and wave leave the kernel waiting for its staging; 32 columns
    // double the work per staged tile, and the x patch of two planes still leaves room for two workgroups per CU)
    if (g.sW == 2 && g.kD <= 2 && g.kH <= 2 && g.kW <= 2 && g.Wo % 32 == 0) P->TW = 32;   // (1.43 -> 1.27 ms at 192^3)
    // Stride 1.  Width: 32 columns, 16 where that leaves fewer positions outside the plane (48 = 3 x 16 columns); planes
    // narrower than 32 take their own (even) width: the contraction runs over pairs of neighbouring columns, so any
    // even width works (24^3 layers 70 -> 88 TFLOP/s).  Rows: as many as make about 96 positions (3 x 32, 6 x 16,
    // 4 x 24) while the dy tile and the ring of x planes leave room for two workgroups per CU (78 KB each), fewer
    // where that divides the height better: more MFMAs per staged tile and fewer halo rows per row (2 x 32 -> 3 x 32:
    // 100 -> 106 TFLOP/s on the 192^3 layers).
    auto padded = [&](int tr, int tw) { return (long long)((g.Ho + tr - 1) / tr * tr) * ((g.Wo + tw - 1) / tw * tw); };
    if (g.sW == 1) {
        if (g.Wo < 32) P->TW = (g.Wo + 1) & ~1;
        else if (padded(2, 16) < padded(2, 32)) P->TW = 16;
        auto lds = [&](int tr) { return ((size_t)tr * P->TW + (size_t)g.kD * ((tr - 1) * g.sH + g.kH) * ((P->TW - 1) * g.sW + g.kW)) * 32 * sizeof(float); };
        int tr = 96 / P->TW;
        tr = tr < 2 ? 2 : (tr > 8 ? 8 : tr);
        while (tr > 2 && (lds(tr) > 78 * 1024 || padded(tr, P->TW) > padded(tr - 1, P->TW))) --tr;
        P->TR = tr;
    }
    P->prows = (P->TR - 1) * g.sH + g.kH;
    P->pcols = (P->TW - 1) * g.sW + g.kW;
    P->pcols_magic = 65536u / (unsigned)P->pcols + 1u;
    P->HT = (g.Ho + P->TR - 1) / P->TR;
    P->WT = (g.Wo + P->TW - 1) / P->TW;
    P->CIT = (g.Cin + 31) / 32;
    P->COT = (g.Cout + 31) / 32;
    P->units = (long long)g.N * g.Do * P->HT * P->WT;
    // about four workgroups per CU in all, each with at least a few units to walk
    long long s = 4ll * cu_count() / ((long long)P->CIT * P->COT);
    if (s > P->units / 4) s = P->units / 4;
    if (s > 1024) s = 1024;
    if (s < 1) s = 1;
    P->S = (int)s;
}

// the folded-tap kernel for at most 4 input channels: 4 x 32 output tiles, two workgroups per CU
bool wgrad_c4_ok(const Geom& g) {
    return g.kD == 3 && g.kH == 3 && g.kW == 3 && g.sD == 1 && g.sH == 1 && g.sW == 1 && g.Cin <= 4 && g.Cout % 4 == 0 && !g.hi;
}
void wgrad_c4_layout(const Geom& g, WgParams* P) {
    P->TR = 4;
    P->TW = 32;
    P->prows = P->TR + 2;
    P->pcols = P->TW + 2;
    P->pcols_magic = 0;
    P->HT = (g.Ho + P->TR - 1) / P->TR;
    P->WT = (g.Wo + P->TW - 1) / P->TW;
    P->CIT = 1;
    P->COT = (g.Cout + 31) / 32;
    P->units = (long long)g.N * g.Do * P->HT * P->WT;
    long long s = 2ll * cu_count() / P->COT;
    if (s > P->units / 4) s = P->units / 4;
    if (s > 1024) s = 1024;
    if (s < 1) s = 1;
    P->S = (int)s;
}

// Sizes that f32s_gconv_kernel takes (forward and data gradient).  Whole steps of 16 contracted channels, taps that come in
// groups of 1, 2, 4 or 9 per plane, unit input stride (a strided patch is four times the tile) and at most SP_MAXV voxels of
// patch (planes of a few columns have more; the general kernel serves those).
bool split_ok(const Geom& g, int pass) {
    if (pass == MI3D_PASS_WGRAD || g.kH != 3 || g.kW != 3) return false;
    const bool dgrad = pass == MI3D_PASS_DGRAD;
    if ((dgrad ? g.Cout : g.Cin) % SP_CK) return false;
    if (dgrad ? g.sH != g.sW : (g.sH != 1 || g.sW != 1)) return false;
    // (the classes of a strided data gradient have 1, 2 or 4 taps per staged patch: with 32 contracted channels they are
    // over before the staging pays, 64->32 at 9 x 20 x 33 140 -> 155 us; with 64 and more 32->64 at 128^3, N = 2 940 -> 805,
    // at 9 x 20 x 33 200 -> 157, 128->256 at 32^3, N = 2 829 -> 591, 64->128 at 6 x 10 x 11 263 -> 271)
    if (g.sH == 2 && g.Cout < 64) return false;
    const int os = dgrad ? g.sH : 1;
    const long long JH = ((dgrad ? g.H : g.Ho) + os - 1) / os, JW = ((dgrad ? g.W : g.Wo) + os - 1) / os;
    for (long long jw = JW > 1 ? JW - 1 : 1; jw <= JW; ++jw) {   // (the parity classes differ by one column)
        if (jw >= 32) continue;                                   // 8 x 32 or 16 x 16 tiles: 340 voxels at most
        long long rows = 255 / jw + 2;
        if (rows > JH) rows = JH;
        if ((rows + 2) * (jw + 2) > SP_MAXV) return false;
    }
    return true;
}
size_t split_pack_bytes(const Geom& g, int pass, size_t* flags_at) {
    const long long K = pass == MI3D_PASS_DGRAD ? g.Cout : g.Cin, M = pass == MI3D_PASS_DGRAD ? g.Cin : g.Cout;
    const size_t frags = (size_t)g.taps() * (K / SP_CK) * ((M + 31) / 32);
    *flags_at = frags * 3 * 512 * sizeof(uint16_t);
    return (*flags_at + frags * sizeof(uint32_t) + 255) & ~(size_t)255;
}

bool wgrad_magic_ok(const WgParams& P) {
    for (unsigned q = 0; q < (unsigned)(P.prows * P.pcols); ++q)
        if (((q * P.pcols_magic) >> 16) != q / (unsigned)P.pcols) return false;
    return true;
}

}  // namespace

bool f32_supported(const Geom& g, int pass) {
    if (g.dtype != MI3D_F32) return false;
    if (g.kD > 3 || g.kH > 3 || g.kW > 3 || g.sD > 2 || g.sH > 2 || g.sW > 2) return false;
    if (g.pD > 2 || g.pH > 2 || g.pW > 2) return false;
    // 32-bit offsets inside one sample's plane and sane grids
    if ((long long)g.H * g.W * g.Cin >= (1ll << 30) || (long long)g.Ho * g.Wo * g.Cout >= (1ll << 30)) return false;
    if (g.w_elems() >= (1ll << 28)) return false;
    if (pass == MI3D_PASS_WGRAD) {
        WgParams P;
        wgrad_layout(g, &P);
        const size_t lds = ((size_t)P.TR * P.TW + (size_t)g.kD * P.prows * P.pcols) * 32 * sizeof(float);
        return lds <= 160 * 1024 && (long long)P.CIT * P.COT * P.S < (1ll << 30) && wgrad_magic_ok(P);
    }
    return true;
}

// 1x1x1 layers with a handful of output channels (the segmentation head) run through plain VALU kernels: with 3 of 32
// MFMA rows in use the matrix cores would do ten times the work (measured at 192^3, N = 2: 0.74 / 1.81 / 3.06 ms for the
// three passes on the matrix cores).  A call with an added gradient or a two-tensor operand keeps the general kernel.
static bool f32_head(const Geom& g) { return pointwise_f32_supported(g) && !g.add && !g.hi; }

static bool ig_better(const Geom& g, int pass);

size_t f32_min_workspace_bytes(const Geom& g, int pass) {
    if (!f32_supported(g, pass)) return 0;
    size_t b;
    if (pass == MI3D_PASS_WGRAD) {
        WgParams P;
        wgrad_layout(g, &P);
        b = (size_t)P.S * g.w_elems() * sizeof(float);
        if (wgrad_c4_ok(g)) {
            wgrad_c4_layout(g, &P);
            const size_t c = (size_t)P.S * g.w_elems() * sizeof(float);
            b = b > c ? b : c;
        }
    } else {
        b = pack_bytes(g, pass);
    }
    const size_t h = pointwise_f32_workspace_bytes(g, pass);   // (0 where the head kernels do not apply)
    return b > h ? b : h;
}

// Weight gradients that the matrix product over numbered positions serves better than the fp32 instructions (which take about 35 us and
// reach about 70 TFLOP/s of whole 32 x 32 blocks of channels, 45 where taps do not overlap), by its model of the time.  With the launch that adds
// the partial sums, f32_wgrad_kernel -> igw_f32_kernel: 64->128, 2x2x2 at 96^3 342 -> 120 us, 32->64, stride 2 at 128^3, N = 2 861 -> 684,
// 128->256, stride 2 at 32^3, N = 2 218 -> 110, 256->256 at 16^3, N = 2 339 -> 213, 128->320 at 11 x 12 x 9 71 -> 43,
// 32->64 at 13 x 18 x 20 57 -> 21.  Layers with at most
// four input channels have the kernel that folds the taps (4->32 at 60^3 44 -> 60) but for the smallest volumes (2->32 at
// 20^3 25 -> 13), and those f32s_wgrad takes stay there (128->128 at 32^3, N = 2 333 -> 394).
static bool igw_better(const Geom& g, size_t ws_bytes) {
    Geom q = g;
    q.hi = nullptr;      // (the sizes decide, not how the call passes its tensors)
    if (f32s_wgrad_supported(q) || !igw_supported(q) || (g.hi && g.Cin % 64)) return false;
    if (wgrad_c4_ok(q)) return g.out_voxels() <= 8192;
    const double blocks = (double)((g.Cin + 31) / 32) * ((g.Cout + 31) / 32) * 1024;
    const bool apart = g.kD <= g.sD && g.kH <= g.sH && g.kW <= g.sW;
    return igw_us(q, ws_bytes) < 35.0 + 2.0 * g.out_voxels() * g.taps() * blocks / (apart ? 45e6 : 70e6);
}

// (the parts of the weights take 1.5 times their room; a call with the smaller workspace gets the fp32 instructions)
size_t f32_workspace_bytes(const Geom& g, int pass) {
    size_t b = f32_min_workspace_bytes(g, pass), at;
    if (f32_supported(g, pass) && pass == MI3D_PASS_WGRAD && f32s_wgrad_supported(g)) {
        const size_t p = f32s_wgrad_workspace_bytes(g);
        b = b > p ? b : p;
    }
    if (f32_supported(g, pass) && pass == MI3D_PASS_WGRAD && igw_better(g, ~(size_t)0)) {
        const size_t p = igw_workspace_bytes(g);
        b = b > p ? b : p;
    }
    if (f32_supported(g, pass) && ig_better(g, pass)) {
        const size_t p = igf_workspace_bytes(g, pass);
        return b > p ? b : p;
    }
    if (f32_supported(g, pass) && split_ok(g, pass)) {
        const size_t p = split_pack_bytes(g, pass, &at);
        b = b > p ? b : p;
    }
    return b;
}

// Planes 32 columns wide and more stay with f32s_gconv_kernel, whose tiles they fill and whose edges the tests reach through
// them.  They would be faster here (this line costs them: 16->16 at 2 x 33 x 33 19 us instead of 12, 16->8 at 4 x 20 x 40 24
// instead of 13, at 32^2 13 instead of 8).
bool f32_uses_tiny(const Geom& g, int pass) {
    if (!f32_supported(g, pass) || f32_head(g) || !tiny_supported(g, pass)) return false;
    return !split_ok(g, pass) || (pass == MI3D_PASS_DGRAD ? g.W : g.Wo) < 32;
}

bool f32_uses_igw(const Geom& g, size_t ws_bytes) { return f32_supported(g, MI3D_PASS_WGRAD) && !f32_head(g) && igw_better(g, ws_bytes); }

bool f32_uses_ig(const Geom& g, int pass, size_t ws_bytes) {
    return f32_supported(g, pass) && !f32_head(g) && ig_better(g, pass) && ws_bytes >= igf_min_workspace_bytes(g, pass);
}

bool f32_uses_parts(const Geom& g, int pass, size_t ws_bytes) {
    if (!f32_supported(g, pass) || f32_head(g)) return false;
    if (pass == MI3D_PASS_WGRAD) return f32s_wgrad_supported(g) && ws_bytes >= f32s_wgrad_workspace_bytes(g);
    return split_ok(g, pass) && ws_bytes >= f32_workspace_bytes(g, pass);
}

bool f32_wgrad_folds_taps(const Geom& g) { return f32_supported(g, MI3D_PASS_WGRAD) && wgrad_c4_ok(g); }

bool f32_takes_halves(const Geom& g, int pass) {   // virtual concatenation: halves of Cin in multiples of 32 channels
    return f32_supported(g, pass) && g.Cin % 64 == 0;
}

// 8 x 32 unless 16 x 16 covers the iteration plane with fewer positions outside it; planes narrower than 32 columns in
// row-major order over their whole width (tile k = positions 256 k .. 256 k + 255 of the plane, whatever rows they fall
// in: a 24 x 24 plane is 18 full blocks of 32 positions instead of 24 blocks three quarters full; TJH = the most rows 256
// consecutive positions can touch)
static void gconv_tile_shape(GcParams* P, bool big_tiles) {
    P->flat = P->Jw < 32 ? 1 : 0;
    if (P->flat) {
        P->TJW = P->Jw;
        P->TJH = 255 / P->Jw + 2;
        if (P->TJH > P->Jh) P->TJH = P->Jh;
        P->LW = 0;
        return;
    }
    auto padded = [&](int th, int tw) { return (long long)((P->Jh + th - 1) / th * th) * ((P->Jw + tw - 1) / tw * tw); };
    const bool square = padded(16, 16) < padded(8, 32);
    P->TJH = square ? 16 : 8;
    P->TJW = square ? 16 : 32;
    P->LW = square ? 4 : 5;
    // Layers with at most 32 output channels (one block per workgroup whatever the grid): 16 x 32 tiles for eight waves
    // where they cover the plane as well; the weights of a stage then serve 512 positions and the halo rows are 2 in
    // 18 instead of 2 in 10 (32->32 at 192^3 +2 %).
    if (!square && big_tiles && P->M <= 32 && padded(16, 32) == padded(8, 32)) P->TJH = 16;
}
static int gconv_row_tiles(const GcParams& P) { return P.flat ? (P.Jh * P.Jw + 255) / 256 : (P.Jh + P.TJH - 1) / P.TJH; }
static int gconv_col_tiles(const GcParams& P) { return P.flat ? 1 : (P.Jw + P.TJW - 1) / P.TJW; }

static int gconv_attributes() {
    static std::atomic<bool> attr_set{false};   // set once per process; a second thread racing here repeats an idempotent call
    if (!attr_set) {
        const void* fns[6] = {(const void*)f32_gconv_kernel<1, GC_NW1, 2>, (const void*)f32_gconv_kernel<2, GC_NW2, 1>, (const void*)f32_gconv_classes_kernel<1, GC_NW1>,
                              (const void*)f32_gconv_classes_kernel<2, GC_NW2>, (const void*)f32_wgrad_kernel, (const void*)f32_gconv_kernel<1, 8, 2>};
        for (const void* f : fns) {
            hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (e != hipSuccess) { note_hip_error(e); return MI3D_ERR_HIP; }
        }
        attr_set = true;
    }
    return MI3D_OK;
}

// Output channels per workgroup: 64 where there are that many, unless the grid is so small that its last round
// over the 2 x CUs workgroup slots would be mostly empty and 32-channel workgroups fill the rounds better
// (24^3, N = 2, 256 output channels: 576 workgroups = 2 rounds of 512 at 56 %; 1152 = 3 rounds at 75 %).
// Only where the MFMA work of a workgroup outweighs its staging (taps x contracted channels): a 2x2x2 layer with
// 128 channels got slower with the smaller workgroups (0.40 -> 0.61 ms), which stage the same patch twice.
static int gconv_blocks_of_channels(const GcParams& P, long long tiles, int ntaps) {
    int CB = P.M > 32 ? 2 : 1;
    if (CB == 2 && ntaps * P.K >= 27 * 64) {
        const long long slots = 2ll * cu_count();
        auto fill = [&](int cb) {
            const long long b = tiles * ((P.Mpad + 32 * cb - 1) / (32 * cb));
            return (double)b / (double)(((b + slots - 1) / slots) * slots);
        };
        if (fill(1) > 1.15 * fill(2)) CB = 1;
    }
    return CB;
}

// What f32s_gconv_kernel takes for a stride-1 layer: stages of 16 channels of a plane times what one takes with that many
// workgroups on a CU (32 / 64 channels per workgroup; alone: 320->320 at 8^3 and 256->256 at 16^3, N = 2, 20^3 64->128; full:
// 45 x 75 x 91 64->32 and back, 64->64 at 64^3 and 128->128 at 32^3, N = 2).
static double split_us(const Geom& g, int pass) {
    GcParams P{};
    const bool dgrad = pass == MI3D_PASS_DGRAD;
    P.N = g.N; P.Jd = dgrad ? g.D : g.Do; P.Jh = dgrad ? g.H : g.Ho; P.Jw = dgrad ? g.W : g.Wo;
    P.K = dgrad ? g.Cout : g.Cin; P.M = dgrad ? g.Cin : g.Cout; P.Mpad = (P.M + 31) / 32 * 32;
    gconv_tile_shape(&P, false);
    const long long tiles = (long long)P.N * P.Jd * gconv_row_tiles(P) * gconv_col_tiles(P);
    const int CB = gconv_blocks_of_channels(P, tiles, (int)g.taps());
    const double alone = CB == 2 ? 6.4 : 5.0, full = CB == 2 ? 6.2 : 3.95;
    const double per_cu = full * (double)(tiles * ((P.Mpad + 32 * CB - 1) / (32 * CB))) / cu_count();
    return 5.0 + (double)(P.K / SP_CK) * g.kD * (per_cu > alone ? per_cu : alone);
}

// Layers that the implicit GEMM over numbered positions serves better than the kernels here, which stage patches.
// - Everything f32s_gconv_kernel does not take: its products are formed on the fp32 instructions, from patches up to four
//   times the tile where the stride is 2.  Forward / data gradient with their packing launches, f32_gconv_kernel -> igf_kernel:
//   64->128, 2x2x2 at 96^3 320 / 250 -> 138 / 163 us, 32->64, stride 2 at 128^3, N = 2 834 -> 462, 128->256, stride 2 at 32^3,
//   N = 2 448 -> 116.  Not where a workgroup would be over after four steps and writes 32 channels (the first layer on large
//   volumes): 4->32 at 60^3 33 -> 40, at 16^3 19 -> 17.
// - The strided data gradients it does take, eight launches of one to eight taps each: 32->64 at 128^3, N = 2 810 -> 709,
//   64->128 at 64^3, N = 2 415 -> 244, 128->256 at 32^3, N = 2 592 -> 140, 32->64 at 24^3 159 -> 25.  (Volumes below 2048 voxels
//   with at most 32 channels keep their kernel, whose classes are tested there on values without parts; it costs them: 32->64
//   at 4^3 to 12^3 120 to 136 us where igf_kernel takes 13 to 15.)
// - Of the stride-1 layers those too small for its tiles of 256 positions of a plane and of 64 contracted channels or more
//   (those with fewer are the large volumes of a network), by the two models of the time: 320->320 at 8^3, N = 2 322 -> 73,
//   256->256 at 16^3, N = 2 230 -> 194; but 128->128 at 32^3, N = 2 291 -> 338 and 64->64 at 64^3, N = 2 600 -> 745: a patch is
//   taken apart once for its 27 taps.
static bool ig_better(const Geom& g, int pass) {
    if (!igf_supported(g, pass)) return false;
    const bool dgrad = pass == MI3D_PASS_DGRAD;
    if (!split_ok(g, pass)) {
        const int K = dgrad ? g.Cout : g.Cin, M = dgrad ? g.Cin : g.Cout;
        return K * g.taps() > 128 || M > 32 || (dgrad ? g.in_voxels() : g.out_voxels()) <= 65536;
    }
    if (dgrad && g.sH == 2) return g.Cin > 32 || g.N * (long long)g.D * g.H * g.W >= 2048;
    return (dgrad ? g.Cout : g.Cin) >= 64 && igf_us(g, pass) < split_us(g, pass);
}

// tiles, channel chunk and LDS bytes of one launch (or one class of a launch) for CB blocks of output channels
static int gconv_prepare(GcParams& P, int CB, size_t* lds) {
    P.JHT = gconv_row_tiles(P);
    P.JWT = gconv_col_tiles(P);
    P.MT = (P.Mpad + 32 * CB - 1) / (32 * CB);
    // contracted channels per stage: the largest even chunk that keeps the tiles of a stage within LDS_SOFT
    int max_group = 1;
    for (int g = 0; g < P.ngroups; ++g) max_group = max_group > P.gstart[g + 1] - P.gstart[g] ? max_group : P.gstart[g + 1] - P.gstart[g];
    auto lds_bytes = [&](int ck) {
        return (size_t)(((P.prows * P.pcols * (ck + 1) + 3) & ~3) + max_group * ck * 32 * CB) * sizeof(float);
    };
    int ck = 32;
    const int kpad = (P.K + 1) & ~1;
    if (ck > kpad) ck = kpad;
    // (strided reads: the patch is four times the tile and the layer is bound by its staging, which deeper stages
    // repeat less often: 32->64 2x2x2 stride 2 at 192^3 1.14 ms with the larger budget, 2.04 with the smaller)
    const size_t soft = (P.isd > 1 || P.ish > 1 || P.isw > 1) ? (size_t)LDS_SOFT_STRIDED : (size_t)LDS_SOFT;
    while (ck > 2 && (lds_bytes(ck) > soft || (kpad % ck && ck > 4))) ck >>= 1;
    if (ck < 2) ck = 2;
    if (lds_bytes(ck) > 160 * 1024) return MI3D_ERR_UNSUPPORTED;
    P.CK = ck;
    *lds = lds_bytes(ck);
    return MI3D_OK;
}

static int launch_gconv(GcParams& P, hipStream_t s) {
    const int CB = gconv_blocks_of_channels(P, (long long)P.N * P.Jd * gconv_row_tiles(P) * gconv_col_tiles(P), P.ntaps);
    size_t lds = 0;
    int st = gconv_prepare(P, CB, &lds);
    if (st) return st;
    const long long blocks = (long long)P.N * P.Jd * P.JHT * P.JWT * P.MT;
    if (blocks <= 0) return MI3D_OK;
    if (blocks > 0x7fffffffll) return MI3D_ERR_UNSUPPORTED;
    if ((st = gconv_attributes())) return st;
    if (CB == 2) f32_gconv_kernel<2, GC_NW2, 1><<<(unsigned)blocks, 64 * GC_NW2, lds, s>>>(P);
    else if (P.TJH == 16 && P.TJW == 32) f32_gconv_kernel<1, 8, 2><<<(unsigned)blocks, 512, lds, s>>>(P);   // 512 positions
    else f32_gconv_kernel<1, GC_NW1, 2><<<(unsigned)blocks, 64 * GC_NW1, lds, s>>>(P);
    return check_launch();
}

template <int CB>
static int launch_split_cb(const GsParams& Q, int ntc, unsigned blocks, size_t lds, hipStream_t s) {
    switch (ntc) {
        case 1: f32s_gconv_kernel<CB, 1><<<blocks, SP_NT, lds, s>>>(Q); break;
        case 2: f32s_gconv_kernel<CB, 2><<<blocks, SP_NT, lds, s>>>(Q); break;
        case 4: f32s_gconv_kernel<CB, 4><<<blocks, SP_NT, lds, s>>>(Q); break;
        case 9: f32s_gconv_kernel<CB, 9><<<blocks, SP_NT, lds, s>>>(Q); break;
        default: return MI3D_ERR_UNSUPPORTED;
    }
    return check_launch();
}
static int launch_split(GsParams& Q, hipStream_t s) {
    GcParams& P = Q.c;
    const int CB = gconv_blocks_of_channels(P, (long long)P.N * P.Jd * gconv_row_tiles(P) * gconv_col_tiles(P), P.ntaps);
    P.JHT = gconv_row_tiles(P);
    P.JWT = gconv_col_tiles(P);
    P.MT = (P.Mpad + 32 * CB - 1) / (32 * CB);
    const long long blocks = (long long)P.N * P.Jd * P.JHT * P.JWT * P.MT;
    if (blocks <= 0) return MI3D_OK;
    if (blocks > 0x7fffffffll || P.prows * P.pcols > SP_MAXV) return MI3D_ERR_UNSUPPORTED;
    for (int k = 0; k < P.ntaps; ++k) Q.taps[k] = (uint32_t)((P.th[k] - P.hmin) * P.pcols + P.tw[k] - P.wmin) | (uint32_t)P.tapidx[k] << 16;
    const int ntc = P.ngroups ? P.ntaps / P.ngroups : 9;   // (no group: nothing to add, any instance writes the epilogue)
    const size_t lds = (size_t)P.prows * P.pcols * 96 + 8 + SP_BITS / 8;
    return CB == 2 ? launch_split_cb<2>(Q, ntc, (unsigned)blocks, lds, s) : launch_split_cb<1>(Q, ntc, (unsigned)blocks, lds, s);
}

// all classes of a stride-2 data gradient in one launch (Q.p[0 .. ncls - 1] filled in but for tiles, CK)
static int launch_gconv_classes(GcMulti& Q, hipStream_t s) {
    if (Q.ncls == 0) return MI3D_OK;
    long long tiles = 0;
    int ntaps = 0;
    for (int c = 0; c < Q.ncls; ++c) {
        const GcParams& P = Q.p[c];
        const long long tc = (long long)P.N * P.Jd * gconv_row_tiles(P) * gconv_col_tiles(P);
        tiles += tc;
        ntaps = ntaps > P.ntaps ? ntaps : P.ntaps;
    }
    const int CB = gconv_blocks_of_channels(Q.p[0], tiles, ntaps);
    size_t lds = 0;
    Q.MT = Q.JWT = Q.JHT = Q.Jd = 0;
    for (int c = 0; c < Q.ncls; ++c) {
        size_t l = 0;
        int st = gconv_prepare(Q.p[c], CB, &l);
        if (st) return st;
        lds = lds > l ? lds : l;
        Q.MT = Q.MT > Q.p[c].MT ? Q.MT : Q.p[c].MT;
        Q.JWT = Q.JWT > Q.p[c].JWT ? Q.JWT : Q.p[c].JWT;
        Q.JHT = Q.JHT > Q.p[c].JHT ? Q.JHT : Q.p[c].JHT;
        Q.Jd = Q.Jd > Q.p[c].Jd ? Q.Jd : Q.p[c].Jd;
    }
    Q.tiles = (long long)Q.p[0].N * Q.Jd * Q.JHT * Q.JWT * Q.MT;
    const long long blocks = (Q.tiles + 7) / 8 * 8 * Q.ncls;
    if (blocks <= 0) return MI3D_OK;
    if (blocks > 0x7fffffffll) return MI3D_ERR_UNSUPPORTED;
    int st = gconv_attributes();
    if (st) return st;
    if (CB == 2) f32_gconv_classes_kernel<2, GC_NW2><<<(unsigned)blocks, 64 * GC_NW2, lds, s>>>(Q);
    else f32_gconv_classes_kernel<1, GC_NW1><<<(unsigned)blocks, 64 * GC_NW1, lds, s>>>(Q);
    return check_launch();
}

// forward (in = x, out = y) and data gradient (in = dy, out = dx)
int f32_conv(const Geom& g, int pass, const void* in, const void* w, void* out, void* ws, size_t ws_bytes, hipStream_t s) {
    if (f32_head(g)) return pointwise_f32_conv(g, pass, in, w, out, ws, ws_bytes, s);
    if (ws_bytes < f32_min_workspace_bytes(g, pass)) return MI3D_ERR_WORKSPACE;
    if (f32_uses_tiny(g, pass)) return tiny_conv(g, pass, in, w, out, s);
    if (f32_uses_ig(g, pass, ws_bytes)) return igf_conv(g, pass, in, w, out, ws, ws_bytes, s);
    const bool split = f32_uses_parts(g, pass, ws_bytes);
    const bool dgrad = pass == MI3D_PASS_DGRAD;
    const int T = (int)g.taps();
    const int K = dgrad ? g.Cout : g.Cin, M = dgrad ? g.Cin : g.Cout, Mpad = (M + 31) / 32 * 32;
    const long long total = (long long)T * K * Mpad;
    GsParams S{};
    if (split) {
        size_t at;
        split_pack_bytes(g, pass, &at);
        S.wsplit = (const uint16_t*)ws;
        S.wflag = (const uint32_t*)((const char*)ws + at);
        S.w = (const float*)w;
        S.w_m = dgrad ? 1 : (long long)T * g.Cin; S.w_t = g.Cin; S.w_k = dgrad ? (long long)T * g.Cin : 1;
        S.T = T;
        const long long frags = (long long)T * (K / SP_CK) * (Mpad / 32);
        f32s_pack_kernel<<<(unsigned)((frags + 3) / 4), 256, 0, s>>>(S.w, (uint16_t*)ws, (uint32_t*)((char*)ws + at), T, K, M, Mpad / 32, S.w_m, S.w_t, S.w_k);
    } else {
        f32_pack_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>((const float*)w, (float*)ws, g.Cout, g.Cin, T, Mpad, dgrad ? 1 : 0);
    }
    int st = check_launch();
    if (st) return st;
    GcParams B;
    B.in = B.in2 = (const float*)in;
    B.out = B.out2 = (float*)out;
    B.ref = (const float*)g.ref;
    B.add = (const float*)g.add;
    B.slope = g.slope;
    B.N = g.N; B.K = K; B.M = M; B.Mpad = Mpad;
    B.in_pitch = K; B.in_split = 1 << 30; B.out_pitch = M; B.out_split = 1 << 30;
    if (!dgrad) {
        B.Di = g.D; B.Hi = g.H; B.Wi = g.W; B.Do = g.Do; B.Ho = g.Ho; B.Wo = g.Wo;
        if (g.hi) { B.in2 = (const float*)g.hi; B.in_pitch = K / 2; B.in_split = K / 2; }
    } else {
        B.Di = g.Do; B.Hi = g.Ho; B.Wi = g.Wo; B.Do = g.D; B.Ho = g.H; B.Wo = g.W;
        if (g.hi) { B.out2 = (float*)g.hi; B.out_pitch = M / 2; B.out_split = M / 2; }
    }
    const int sD = dgrad ? g.sD : 1, sH = dgrad ? g.sH : 1, sW = dgrad ? g.sW : 1;   // number of classes per axis
    // Classes with the same work each (2x2x2: one tap per class) go into one launch, where they share their input
    // patch through the L2 (192^3, N = 2: 1.74 -> 1.58 ms; 48^3: 0.63 -> 0.30).  Classes of 1 to 8 taps (3x3x3) keep a
    // launch each: merged, their mix left CUs with the eight-tap workgroups behind (6.0 against 5.4 ms).
    const bool classes = sD * sH * sW > 1 && g.kD <= g.sD && g.kH <= g.sH && g.kW <= g.sW;
    GcMulti Q;
    Q.ncls = 0;
    for (int pd = 0; pd < sD; ++pd)
        for (int ph = 0; ph < sH; ++ph)
            for (int pw = 0; pw < sW; ++pw) {
                GcParams P = B;
                const AxisTaps ad = axis_taps(g.kD, g.sD, g.pD, dgrad, pd), ah = axis_taps(g.kH, g.sH, g.pH, dgrad, ph),
                               aw = axis_taps(g.kW, g.sW, g.pW, dgrad, pw);
                if (!dgrad) {
                    P.Jd = g.Do; P.Jh = g.Ho; P.Jw = g.Wo;
                    P.isd = g.sD; P.ish = g.sH; P.isw = g.sW;
                    P.osd = P.osh = P.osw = 1; P.ood = P.ooh = P.oow = 0;
                } else {
                    P.Jd = (g.D - pd + g.sD - 1) / g.sD; P.Jh = (g.H - ph + g.sH - 1) / g.sH; P.Jw = (g.W - pw + g.sW - 1) / g.sW;
                    P.isd = P.ish = P.isw = 1;
                    P.osd = g.sD; P.osh = g.sH; P.osw = g.sW; P.ood = pd; P.ooh = ph; P.oow = pw;
                }
                if (P.Jd <= 0 || P.Jh <= 0 || P.Jw <= 0) continue;
                // taps grouped by input plane offset (the kd axis is the outer one)
                P.ntaps = 0; P.ngroups = 0;
                int hmin = 1 << 20, hmax = -(1 << 20), wmin = 1 << 20, wmax = -(1 << 20);
                for (int a = 0; a < ad.n; ++a) {
                    P.gstart[P.ngroups] = P.ntaps;
                    P.gd[P.ngroups] = ad.d[a];
                    for (int bq = 0; bq < ah.n; ++bq)
                        for (int c = 0; c < aw.n; ++c) {
                            P.th[P.ntaps] = (signed char)ah.d[bq];
                            P.tw[P.ntaps] = (signed char)aw.d[c];
                            P.tapidx[P.ntaps] = (signed char)((ad.t[a] * g.kH + ah.t[bq]) * g.kW + aw.t[c]);
                            hmin = hmin < ah.d[bq] ? hmin : ah.d[bq]; hmax = hmax > ah.d[bq] ? hmax : ah.d[bq];
                            wmin = wmin < aw.d[c] ? wmin : aw.d[c]; wmax = wmax > aw.d[c] ? wmax : aw.d[c];
                            ++P.ntaps;
                        }
                    if (P.ntaps > P.gstart[P.ngroups]) ++P.ngroups;
                }
                P.gstart[P.ngroups] = P.ntaps;
                if (P.ntaps == 0) { hmin = hmax = wmin = wmax = 0; }   // a class no tap reaches: zeros (plus the epilogue)
                P.hmin = hmin; P.wmin = wmin;
                gconv_tile_shape(&P, !split && !classes && sD * sH * sW == 1);
                P.prows = (P.TJH - 1) * P.ish + (hmax - hmin) + 1;
                P.pcols = (P.TJW - 1) * P.isw + (wmax - wmin) + 1;
                P.wpack = (const float*)ws;
                if (classes) { Q.p[Q.ncls++] = P; continue; }
                if (split) {
                    S.c = P;
                    st = launch_split(S, s);
                } else {
                    st = launch_gconv(P, s);
                }
                if (st) return st;
            }
    return classes ? launch_gconv_classes(Q, s) : MI3D_OK;
}

int f32_wgrad(const Geom& g, const void* x, const void* dy, float* dw, void* ws, size_t ws_bytes, hipStream_t s) {
    if (f32_head(g)) return pointwise_f32_conv(g, MI3D_PASS_WGRAD, x, dy, dw, ws, ws_bytes, s);
    if (ws_bytes < f32_min_workspace_bytes(g, MI3D_PASS_WGRAD)) return MI3D_ERR_WORKSPACE;
    if (f32_uses_tiny(g, MI3D_PASS_WGRAD)) return tiny_wgrad(g, x, dy, dw, s);
    if (f32_uses_igw(g, ws_bytes)) return igw_run(g, x, dy, dw, ws, ws_bytes, s);
    if (f32_uses_parts(g, MI3D_PASS_WGRAD, ws_bytes)) return f32s_wgrad(g, x, dy, dw, ws, ws_bytes, s);
    WgParams P;
    wgrad_layout(g, &P);
    P.x = P.x2 = (const float*)x;
    P.dy = (const float*)dy;
    P.part = (float*)ws;
    P.N = g.N; P.D = g.D; P.H = g.H; P.W = g.W; P.Cin = g.Cin; P.Cout = g.Cout; P.Do = g.Do; P.Ho = g.Ho; P.Wo = g.Wo;
    P.kD = g.kD; P.kH = g.kH; P.kW = g.kW; P.sD = g.sD; P.sH = g.sH; P.sW = g.sW; P.pD = g.pD; P.pH = g.pH; P.pW = g.pW;
    P.T = (int)g.taps();
    P.x_pitch = g.Cin; P.x_split = 1 << 30;
    if (g.hi) { P.x2 = (const float*)g.hi; P.x_pitch = g.Cin / 2; P.x_split = g.Cin / 2; }
    if (wgrad_c4_ok(g)) {
        wgrad_c4_layout(g, &P);
        const size_t lds4 = ((size_t)P.TR * P.TW * 32 + (size_t)3 * P.prows * P.pcols * 4) * sizeof(float);   // 26 KB
        f32_wgrad_c4_kernel<<<(unsigned)(P.COT * P.S), 256, lds4, s>>>(P);
        int st4 = check_launch();
        if (st4) return st4;
        return reduce_partials((const float*)ws, dw, g.w_elems(), P.S, s);
    }
    const size_t lds = ((size_t)P.TR * P.TW + (size_t)g.kD * P.prows * P.pcols) * 32 * sizeof(float);
    static std::atomic<bool> attr_set{false};   // set once per process; a second thread racing here repeats an idempotent call
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)f32_wgrad_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) { note_hip_error(e); return MI3D_ERR_HIP; }
        attr_set = true;
    }
    f32_wgrad_kernel<<<(unsigned)(P.CIT * P.COT * P.S), WG_NT, lds, s>>>(P);
    int st = check_launch();
    if (st) return st;
    return reduce_partials((const float*)ws, dw, g.w_elems(), P.S, s);
}

}  // namespace mi3d
