// fp32 weight gradient of 3x3x3 / stride-1 layers with channels in multiples of 32, its products formed by bf16 matrix
// instructions (v_mfma_f32_16x16x32_bf16): each fp32 operand is taken apart into three bf16 numbers, v = a + b + c exactly,
// and six of the nine products are added in fp32; the three left out are at most about 2^-24 of the product
// (see conv_f32.hip).  The five small ones are summed apart and added once, so that an accumulator is rounded twice per 32 positions (the fp32 instructions: 16 times).
// Errors against 64 bits (2-norm, fp32 instructions -> this kernel): 32->32 at 40 x 96 x 96,
// N = 2 5.0e-7 -> 3.8e-7, 64->64 at 24 x 64 x 64 3.6e-7 -> 2.7e-7.
//
//   dw[co,t,ci] = sum_{n,o} dy[n,o,co] * x[n, o - p + t, ci]
//
// Work decomposition as in the bf16 kernel: a workgroup owns a pair of 32-channel tiles and walks x planes along D of
// patches of 4 rows x 32 columns of dy, keeping a ring of three dy planes; each of the 4 waves owns a 16 x 16 quadrant
// for all 27 taps; an x fragment (one per kw) meets the 3 x 3 window of dy fragments (kd, kh) held in registers.  The parts
// are stored as [part][16-channel slab][voxel] and fetched with the transposing ds_read_b64_tr_b16.  Partial sums per
// workgroup are added in slot order by reduce_partials (bit-reproducible).
//
// Bound: with four rows per plane a wave issues 648 MFMAs (10 400 cycles) against 10 16-byte loads, their conversion and
// 31 LDS writes per thread; LDS (113 KB: three parts of an x patch and three dy patches) leaves one workgroup per CU, so the
// conversion is not hidden.  fp32 instructions -> this kernel: 32->32 at 128^3, N = 2 2343 -> 1260 us (99 -> 184 TFLOP/s),
// 64->64 at 64^3, N = 2 1173 -> 642, 64->32 at 45 x 75 x 91 397 -> 255.
//
// A value outside the range of the split (split_f32.h; infinities and NaN among them) sends its step through
// v_mfma_f32_16x16x4_f32 on operands read straight from memory, both zero where either lies outside its volume, so that a
// value at a border meets no zero that is not there.  Such a step takes nine times as long (64->64 at 64^3, N = 2: one value
// 747 -> 835 us, values in every patch 6.6 ms); a row's loads requested together take half of that, but cost the
// ordinary steps 40 % through the registers they spill.
#include "mi3d_internal.h"
#include "split_f32.h"

namespace mi3d {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int TH = 4, TW = 32, XR = TH + 2, XC = TW + 2;
constexpr int X_SLAB = XR * XC * 32, X_PART = 2 * X_SLAB;           // bytes
constexpr int DY_SLAB = TH * TW * 32, DY_PART = 2 * DY_SLAB;
constexpr int X_BYTES = 3 * X_PART, DY_BYTES = 3 * DY_PART;
constexpr int LDS_BYTES = X_BYTES + 3 * DY_BYTES + 16;
constexpr int XPIECES = XR * XC * 8, NX = (XPIECES + 255) / 256, NDY = TH * TW * 8 / 256;   // 16-byte pieces (4 channels)
static_assert(NX + NDY <= 2 * XR && NDY * 256 == TH * TW * 8, "two global loads per x row cover both patches");

struct Params {
    const float* x;
    const float* x2;        // cin tiles >= xsplit (virtual concatenation)
    const float* dy;
    float* part;            // [slots][Cout][27][Cin]
    int N, D, H, W, Cin, Cout, Do, Ho, Wo, pD, pH, pW;
    int HT, WT, CiT, slots;
    int xpitch, xsplit;
    long long units;        // per pair: N * HT * WT * D
};

__device__ __forceinline__ bf16x8 tr_frag(const char* p) {   // 32 voxels of this lane group's 16 channels
    typedef __attribute__((address_space(3))) s16x4* lptr;
    s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr)(p));
    s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr)(p + 16 * 32));
    s16x8 c = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, c);
}
__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

typedef bf16x8 Frag[3];   // the three parts

// x row R of the patch against the dy rows R - kh (window slot = dy row mod 3: row R + 1 takes the place of row R - 2 once
// that has met this x row; a fourth slot costs 36 registers, which spill)
template <int R, class Hook>
__device__ __forceinline__ void rows_from(f32x4 (&acc)[3][3][3], Frag (&dyw)[3][3], Frag (&xf)[3], Frag (&xn)[3], const char* x_lane,
                                          const char* const (&dy_lane)[3], Hook&& hook) {
    if constexpr (R < XR) {
        hook(R);
        if (R + 1 < XR) {
#pragma unroll
            for (int kw = 0; kw < 3; ++kw)
#pragma unroll
                for (int p = 0; p < 3; ++p) xn[kw][p] = tr_frag(x_lane + p * X_PART + ((R + 1) * XC + kw) * 32);
        }
#pragma unroll
        for (int kh = 2; kh >= 0; --kh) {
            const int dr = R - kh;
            if (dr >= 0 && dr < TH) {
                constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
#pragma unroll
                for (int kd = 0; kd < 3; ++kd) {
                    f32x4 low[3];
#pragma unroll
                    for (int q = 0; q < 5; ++q)
#pragma unroll
                        for (int kw = 0; kw < 3; ++kw)
                            low[kw] = mfma(dyw[kd][dr % 3][PA[q]], xf[kw][PB[q]], q ? low[kw] : f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                    for (int kw = 0; kw < 3; ++kw) acc[kd][kh][kw] = mfma(dyw[kd][dr % 3][0], xf[kw][0], acc[kd][kh][kw]);
#pragma unroll
                    for (int kw = 0; kw < 3; ++kw)
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[kd][kh][kw][i] += low[kw][i];
                }
            }
            if (kh == 2 && R + 1 < TH) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int kd = 0; kd < 3; ++kd)
#pragma unroll
                    for (int p = 0; p < 3; ++p) dyw[kd][(R + 1) % 3][p] = tr_frag(dy_lane[kd] + p * DY_PART + (R + 1) * TW * 32);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        rows_from<R + 1>(acc, dyw, xn, xf, x_lane, dy_lane, hook);
    }
}

__global__ void __launch_bounds__(256, 1) f32s_wgrad_kernel(Params P) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char* x_lds = lds;
    char* dy_lds = lds + X_BYTES;                            // ring of three planes
    int* bad_lds = (int*)(lds + X_BYTES + 3 * DY_BYTES);     // stamp of the last plane with a value the parts cannot hold: dy ring slots, x

    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int coh = wave >> 1, cih = wave & 1;
    const int pair = blockIdx.y, slot = blockIdx.x;
    const int cot = pair / P.CiT, cit = pair % P.CiT;
    long long u0 = P.units * slot / P.slots;
    const long long u1 = P.units * (slot + 1) / P.slots;
    const int g = lane >> 4, s = lane & 15;
    const int lane_off = (4 * g + (s >> 2)) * 32 + (s & 3) * 8;
    const char* x_lane = x_lds + cih * X_SLAB + lane_off;

    f32x4 acc[3][3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[a][b][c] = f32x4{0.f, 0.f, 0.f, 0.f};

    const long long x_plane = (long long)P.H * P.W * P.xpitch, dy_plane = (long long)P.Ho * P.Wo * P.Cout;
    const bool x_high = cit >= P.xsplit;
    const int xc0 = (x_high ? cit - P.xsplit : cit) * 32, yc0 = cot * 32;
    if (t < 4) bad_lds[t] = -1;
    // Stamp of the current step: its x plane carries it, the dy plane of tap kd carries stamp - kd and sits in ring slot
    // (stamp - kd) % 3; every segment begins three further on.
    int stamp = 0;

    while (u0 < u1) {
        const long long column = u0 / P.D;
        const int id_start = (int)(u0 - column * P.D);
        const long long left = u1 - u0;
        const int id_end = id_start + (int)(left < (long long)(P.D - id_start) ? left : (long long)(P.D - id_start));
        u0 += id_end - id_start;
        const int wt = (int)(column % P.WT), ht = (int)(column / P.WT % P.HT), n = (int)(column / P.WT / P.HT);
        const int h0 = ht * TH, w0 = wt * TW;
        int gx[NX], gdy[NDY];
        unsigned vx = 0, vdy = 0;
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int q = t + 256 * i, v = q >> 3, c = q & 7, row = v / XC, col = v - row * XC;
            const int gh = h0 - P.pH + row, gw = w0 - P.pW + col;
            const bool ok = q < XPIECES && gh >= 0 && gh < P.H && gw >= 0 && gw < P.W;
            gx[i] = ok ? (gh * P.W + gw) * P.xpitch + xc0 + c * 4 : 0;
            vx |= (ok ? 1u : 0u) << i;
        }
#pragma unroll
        for (int i = 0; i < NDY; ++i) {
            const int q = t + 256 * i, v = q >> 3, c = q & 7, row = v >> 5, col = v & 31;
            const int gh = h0 + row, gw = w0 + col;
            const bool ok = gh < P.Ho && gw < P.Wo;
            gdy[i] = ok ? (gh * P.Wo + gw) * P.Cout + yc0 + c * 4 : 0;
            vdy |= (ok ? 1u : 0u) << i;
        }
        const float* xn = (x_high ? P.x2 : P.x) + (long long)n * P.D * x_plane;
        const float* dyn = P.dy + (long long)n * P.Do * dy_plane;

        float4 px[NX], pdy[NDY];
        unsigned mx = 0, mdy = 0;
        const float *bx = xn, *bdy = dyn;
        auto begin_x = [&](int id) {
            const bool in = id >= 0 && id < P.D;
            bx = xn + (long long)(in ? id : 0) * x_plane;
            mx = in ? vx : 0u;
        };
        auto begin_dy = [&](int od) {
            const bool in = od >= 0 && od < P.Do;
            bdy = dyn + (long long)(in ? od : 0) * dy_plane;
            mdy = in ? vdy : 0u;
        };
        // one piece, zero where it lies outside, to the three parts at d
        auto store = [&](const float4& v, bool ok, char* d, int part, SplitRange& range) {
            const float4 w = ok ? v : make_float4(0.f, 0.f, 0.f, 0.f);
            uint32_t lo[3], hi[3];
            split2(w.x, w.y, lo);
            split2(w.z, w.w, hi);
#pragma unroll
            for (int p = 0; p < 3; ++p) *(uint2*)(d + p * part) = uint2{lo[p], hi[p]};
            range.add(w);
        };
        auto write_x = [&](int st) {
            SplitRange range;
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                const int q = t + 256 * i, v = q >> 3, c = q & 7;
                if (q < XPIECES) store(px[i], (mx >> i) & 1, x_lds + (c >> 2) * X_SLAB + v * 32 + (c & 3) * 8, X_PART, range);
            }
            if (__any(range.exceeded()) && lane == 0) bad_lds[3] = st;
        };
        auto write_dy = [&](int st) {
            const int ring = st % 3;
            SplitRange range;
#pragma unroll
            for (int i = 0; i < NDY; ++i) {
                const int q = t + 256 * i, v = q >> 3, c = q & 7;
                store(pdy[i], (mdy >> i) & 1, dy_lds + ring * DY_BYTES + (c >> 2) * DY_SLAB + v * 32 + (c & 3) * 8, DY_PART, range);
            }
            if (__any(range.exceeded()) && lane == 0) bad_lds[ring] = st;
        };

        stamp += 3;
        __syncthreads();   // the previous segment's readers are done with the LDS
        begin_x(id_start);
#pragma unroll
        for (int i = 0; i < NX; ++i) px[i] = *(const float4*)(bx + gx[i]);
        write_x(stamp);
        for (int kd = 0; kd < 3; ++kd) {
            begin_dy(id_start + P.pD - kd);
#pragma unroll
            for (int i = 0; i < NDY; ++i) pdy[i] = *(const float4*)(bdy + gdy[i]);
            write_dy(stamp - kd);
        }
        __syncthreads();

        for (int id = id_start; id < id_end; ++id, ++stamp) {
            begin_x(id + 1);
            begin_dy(id + 1 + P.pD);   // the plane that enters the ring for the next step
            bool plain = bad_lds[3] == stamp;
#pragma unroll
            for (int kd = 0; kd < 3; ++kd) plain |= bad_lds[(stamp - kd) % 3] == stamp - kd;
            if (__builtin_amdgcn_readfirstlane(plain)) {
                const float* bxn = xn + (long long)id * x_plane + xc0 + cih * 16 + s;
                const float* byn = dyn + yc0 + coh * 16 + s;
#pragma unroll
                for (int kd = 0; kd < 3; ++kd) {
                    const int od = id + P.pD - kd;
                    if (od < 0 || od >= P.Do) continue;
#pragma unroll
                    for (int kh = 0; kh < 3; ++kh)
#pragma unroll
                        for (int kw = 0; kw < 3; ++kw)
#pragma unroll 1
                            for (int e = 0; e < TH * TW / 4; ++e) {   // four columns at a time
                                const int oh = h0 + e / (TW / 4), ow = w0 + e % (TW / 4) * 4 + g;
                                const int ih = oh - P.pH + kh, iw = ow - P.pW + kw;
                                const bool ok = oh < P.Ho && ow < P.Wo && ih >= 0 && ih < P.H && iw >= 0 && iw < P.W;
                                const float a = ok ? byn[od * dy_plane + ((long long)oh * P.Wo + ow) * P.Cout] : 0.f;
                                const float b = ok ? bxn[((long long)ih * P.W + iw) * P.xpitch] : 0.f;
                                acc[kd][kh][kw] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[kd][kh][kw], 0, 0, 0);
                            }
                }
#pragma unroll
                for (int i = 0; i < NX; ++i) px[i] = *(const float4*)(bx + gx[i]);
#pragma unroll
                for (int i = 0; i < NDY; ++i) pdy[i] = *(const float4*)(bdy + gdy[i]);
            } else {
                const char* dy_lane[3];
#pragma unroll
                for (int kd = 0; kd < 3; ++kd) dy_lane[kd] = dy_lds + (stamp - kd) % 3 * DY_BYTES + coh * DY_SLAB + lane_off;
                const char* const dyl[3] = {dy_lane[0], dy_lane[1], dy_lane[2]};
                Frag dyw[3][3], xa[3], xb[3];
#pragma unroll
                for (int kd = 0; kd < 3; ++kd)
#pragma unroll
                    for (int p = 0; p < 3; ++p) dyw[kd][0][p] = tr_frag(dyl[kd] + p * DY_PART);
#pragma unroll
                for (int kw = 0; kw < 3; ++kw)
#pragma unroll
                    for (int p = 0; p < 3; ++p) xa[kw][p] = tr_frag(x_lane + p * X_PART + kw * 32);
                // two global loads per x row.  They and the LDS writes below are unconditional (the step after the last of a
                // segment fetches a valid plane that is not used), so that each load is paired with its consumer.
                rows_from<0>(acc, dyw, xa, xb, x_lane, dyl, [&](int r) {
#pragma unroll
                    for (int j = 2 * r; j < 2 * r + 2; ++j) {
                        if (j < NX) px[j] = *(const float4*)(bx + gx[j]);
                        else if (j - NX < NDY) pdy[j - NX] = *(const float4*)(bdy + gdy[j - NX]);
                    }
                });
            }
            __syncthreads();   // everyone is done reading the x patch and the oldest dy patch
            write_x(stamp + 1);
            write_dy(stamp + 1);
            __syncthreads();
        }
    }

    // acc register v of lane l is (co = 4 (l / 16) + v, ci = l % 16) of the quadrant
    float* out = P.part + (long long)slot * ((long long)P.Cout * 27 * P.Cin);
#pragma unroll
    for (int kd = 0; kd < 3; ++kd)
#pragma unroll
        for (int kh = 0; kh < 3; ++kh)
#pragma unroll
            for (int kw = 0; kw < 3; ++kw)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int co = cot * 32 + coh * 16 + 4 * (lane >> 4) + v, ci = cit * 32 + cih * 16 + (lane & 15);
                    out[((long long)co * 27 + (kd * 3 + kh) * 3 + kw) * P.Cin + ci] = acc[kd][kh][kw][v];
                }
}

long long columns(const Geom& g) { return (long long)g.N * ((g.Ho + TH - 1) / TH) * ((g.Wo + TW - 1) / TW); }
int slots_of(const Geom& g) {
    const long long pairs = (long long)(g.Cin / 32) * (g.Cout / 32), units = columns(g) * g.D;
    long long slots = (cu_count() + pairs - 1) / pairs;   // one workgroup per CU in total
    if (slots > units) slots = units;
    return (int)(slots < 1 ? 1 : slots);
}

}  // namespace

bool f32s_wgrad_supported(const Geom& g) {
    if (g.dtype != MI3D_F32 || g.kD != 3 || g.kH != 3 || g.kW != 3 || g.sD != 1 || g.sH != 1 || g.sW != 1) return false;
    if (g.pD > 2 || g.pH > 2 || g.pW > 2 || g.Cin % 32 || g.Cout % 32) return false;
    if ((long long)g.H * g.W * g.Cin >= (1ll << 30) || (long long)g.Ho * g.Wo * g.Cout >= (1ll << 30)) return false;
    if ((long long)(g.Cin / 32) * (g.Cout / 32) > 65535) return false;
    // Planes that 4 x 32 patches cover to 60 % and more, and eight or more of them per workgroup: the fp32 kernel takes narrower
    // tiles and a quarter of the units per workgroup (64->64 at 24 x 64 x 64, 12 patches each: 261 -> 158 us; 640->32 at
    // 6 x 20 x 40, 5 each: 114 -> 126; 64->96 at 8 x 24 x 24, N = 2, 2 each: 75 -> 80).
    const double share = (double)g.Ho * g.Wo / ((double)((g.Ho + TH - 1) / TH * TH) * ((g.Wo + TW - 1) / TW * TW));
    const long long pairs = (long long)(g.Cin / 32) * (g.Cout / 32);
    return share >= 0.6 && columns(g) * g.D * pairs >= 8ll * cu_count();
}

size_t f32s_wgrad_workspace_bytes(const Geom& g) { return (size_t)slots_of(g) * g.w_elems() * sizeof(float); }

int f32s_wgrad(const Geom& g, const void* x, const void* dy, float* dw, void* ws, size_t ws_bytes, hipStream_t s) {
    if (ws_bytes < f32s_wgrad_workspace_bytes(g)) return MI3D_ERR_WORKSPACE;
    Params P{};
    P.x = P.x2 = (const float*)x; P.dy = (const float*)dy; P.part = (float*)ws;
    P.N = g.N; P.D = g.D; P.H = g.H; P.W = g.W; P.Cin = g.Cin; P.Cout = g.Cout; P.Do = g.Do; P.Ho = g.Ho; P.Wo = g.Wo;
    P.pD = g.pD; P.pH = g.pH; P.pW = g.pW;
    P.HT = (g.Ho + TH - 1) / TH; P.WT = (g.Wo + TW - 1) / TW; P.CiT = g.Cin / 32;
    P.slots = slots_of(g);
    P.xpitch = g.Cin; P.xsplit = P.CiT;
    P.units = columns(g) * g.D;
    if (g.hi) {
        if (g.Cin % 64) return MI3D_ERR_UNSUPPORTED;
        P.x2 = (const float*)g.hi; P.xpitch = g.Cin / 2; P.xsplit = P.CiT / 2;
    }
    static std::atomic<bool> attr_set{false};   // set once per process; a second thread racing here repeats an idempotent call
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)f32s_wgrad_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) { note_hip_error(e); return MI3D_ERR_HIP; }
        attr_set = true;
    }
    f32s_wgrad_kernel<<<dim3((unsigned)P.slots, (unsigned)(P.CiT * (g.Cout / 32))), 256, LDS_BYTES, s>>>(P);
    const int st = check_launch();
    return st ? st : reduce_partials((const float*)ws, dw, g.w_elems(), P.slots, s);
}

}  // namespace mi3d
