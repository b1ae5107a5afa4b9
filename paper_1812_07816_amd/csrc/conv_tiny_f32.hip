// The smallest fp32 layers in one launch a pass (forward, data gradient, weight gradient; plain fp32 multiply-adds).
//
// Bound: latency.  A layer of a few million multiply-adds takes the other kernels two or three launches of 4 to 12 us (weights
// taken apart, products, partial sums added), each a trip or two to memory and several us of host work; here a thread has
// its whole sum, or a workgroup the whole sum of its weights.  Errors against fp64 are half those of the fp32 matrix instructions (4->8 at 16^3 9.8e-8 to 1.8e-7: four sums side by side).
#include "ig_common.h"
#include "mi3d_internal.h"

namespace mi3d {
namespace {

struct TinyParams {
    const float *in, *w, *add, *ref;   // activations read (x, or dy of the data gradient; x of the weight gradient)
    const float* dy;                   // weight gradient only
    float* out;
    float slope;
    int K, M, T, row;                  // contracted and output channels, taps, floats between two rows of weights in LDS
    int iD, iH, iW, outputs, dgrad;
    int k[3], s[3], p[3];
    Div oD, oH, oW, Md, TKd, TMd;      // extents of the positions; output channels, T * K, T * M
};

// coordinate read along an axis by position o at tap t, -1: none
__device__ __forceinline__ int source(const TinyParams& P, int a, int o, int t, int extent) {
    if (t >= P.k[a]) return -1;
    int v = P.dgrad ? o + P.p[a] - t : o * P.s[a] - P.p[a] + t;
    if (P.dgrad && P.s[a] == 2) v = v & 1 ? -1 : v >> 1;
    return (unsigned)v < (unsigned)extent ? v : -1;
}

// Thread = (position, output channel), channels fastest.  The weights lie in LDS as [output channel][tap][contracted channel];
// nine taps of VEC channels are requested at a time.
template <int VEC>
__global__ void __launch_bounds__(256) tiny_conv_kernel(const TinyParams P) {
    typedef float vec __attribute__((__vector_size__(VEC * sizeof(float))));
    extern __shared__ __attribute__((aligned(16))) float wl[];
    const int n_w = P.M * P.T * P.K;
    for (int i = threadIdx.x; i < n_w; i += 256) {
        int m, tk;
        if (P.dgrad) {   // w[contracted][tap][output]
            const int k = divide(i, P.TMd), r = i - k * (int)P.TMd.d, t = divide(r, P.Md);
            m = r - t * P.M;
            tk = t * P.K + k;
        } else {
            m = divide(i, P.TKd);
            tk = i - m * (int)P.TKd.d;
        }
        wl[m * P.row + tk] = P.w[i];
    }
    __syncthreads();
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= P.outputs) return;
    int r = divide(idx, P.Md);
    const float* wm = wl + (idx - r * P.M) * P.row;
    int q = divide(r, P.oW);
    const int ow = r - q * (int)P.oW.d;
    r = divide(q, P.oH);
    const int oh = q - r * (int)P.oH.d, n = divide(r, P.oD), od = r - n * (int)P.oD.d;
    int d[3], h[3], w[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        d[t] = source(P, 0, od, t, P.iD);
        h[t] = source(P, 1, oh, t, P.iH);
        w[t] = source(P, 2, ow, t, P.iW);
    }
    float acc[4] = {0.f, 0.f, 0.f, 0.f};   // four sums side by side: of every fourth channel, or of every fourth tap
    for (int c = 0; c < P.K; c += VEC) {
#pragma unroll
        for (int td = 0; td < 3; ++td) {
            if (d[td] < 0) continue;
            vec v[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const int th = i / 3, tw = i % 3;
                const long long at = (((long long)n * P.iD + d[td]) * P.iH + h[th]) * P.iW + w[tw];
                v[i] = *(const vec*)(P.in + ((h[th] | w[tw]) >= 0 ? at * P.K + c : 0));
            }
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const int th = i / 3, tw = i % 3;
                if ((h[th] | w[tw]) < 0) continue;   // (not a product with zero: weights may be infinite)
                const vec f = *(const vec*)(wm + ((td * P.k[1] + th) * P.k[2] + tw) * P.K + c);
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[VEC == 4 ? e : (td * 9 + i) & 3] = fmaf(v[i][e], f[e], acc[VEC == 4 ? e : (td * 9 + i) & 3]);
            }
        }
    }
    float v = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    if (P.add) v += P.add[idx];
    P.out[idx] = (P.ref ? P.ref[idx] : v) > 0.f ? v : P.slope * v;
}

constexpr int MAX_W = 12288;     // weights in LDS, with the padding of their rows: 48 KB
constexpr int TM = 8, TK = 4;   // weights of a workgroup: output channels x input channels of one tap

// Workgroup = (tap, TM x TK weights); its threads share the positions, and the sums go from lane to lane (a lane gives away half
// of those it holds in each step), then from wave to wave, in a fixed order.
template <bool VEC>
__global__ void __launch_bounds__(1024) tiny_wgrad_kernel(const TinyParams P) {
    __shared__ float red[16][TM * TK];
    const int t = threadIdx.x, lane = t & 63, KT = (P.K + TK - 1) / TK, MT = (P.M + TM - 1) / TM;
    int b = blockIdx.x;
    const int tap = b / (KT * MT);
    b -= tap * KT * MT;
    const int m0 = b / KT * TM, k0 = b % KT * TK;
    const int td = tap / (P.k[1] * P.k[2]), th = tap / P.k[2] % P.k[1], tw = tap % P.k[2];
    float s[TM * TK];
#pragma unroll
    for (int i = 0; i < TM * TK; ++i) s[i] = 0.f;
#pragma unroll 2
    for (int j = t; j < P.outputs; j += (int)blockDim.x) {
        int q = divide(j, P.oW);
        const int w = source(P, 2, j - q * (int)P.oW.d, tw, P.iW);
        const int r = divide(q, P.oH), h = source(P, 1, q - r * (int)P.oH.d, th, P.iH);
        const int n = divide(r, P.oD), d = source(P, 0, r - n * (int)P.oD.d, td, P.iD);
        if ((d | h | w) < 0) continue;
        const float* x = P.in + ((((long long)n * P.iD + d) * P.iH + h) * P.iW + w) * P.K + k0;
        const float* y = P.dy + (long long)j * P.M + m0;
        float xv[TK], yv[TM];
        if (VEC) {
            const float4 a = *(const float4*)x, c = *(const float4*)y, e = m0 + 4 < P.M ? *(const float4*)(y + 4) : float4{0.f, 0.f, 0.f, 0.f};
            xv[0] = a.x; xv[1] = a.y; xv[2] = a.z; xv[3] = a.w;
            yv[0] = c.x; yv[1] = c.y; yv[2] = c.z; yv[3] = c.w; yv[4] = e.x; yv[5] = e.y; yv[6] = e.z; yv[7] = e.w;
        } else {
#pragma unroll
            for (int i = 0; i < TK; ++i) xv[i] = k0 + i < P.K ? x[i] : 0.f;
#pragma unroll
            for (int i = 0; i < TM; ++i) yv[i] = m0 + i < P.M ? y[i] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < TM * TK; ++i) s[i] = fmaf(yv[i / TK], xv[i % TK], s[i]);
    }
#pragma unroll
    for (int w = TM * TK / 2; w >= 1; w >>= 1) {
        const unsigned up = lane & w * 2 ? ~0u : 0u;   // (selects by mask: a conditional over an array's elements becomes compares)
#pragma unroll
        for (int i = 0; i < w; ++i) {
            const unsigned lo = __builtin_bit_cast(unsigned, s[i]), hi = __builtin_bit_cast(unsigned, s[i + w]);
            const int give = (int)((lo & up) | (hi & ~up));
            s[i] = __builtin_bit_cast(float, (hi & up) | (lo & ~up)) +
                   __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((lane ^ w * 2) * 4, give));
        }
    }
    s[0] += __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((lane ^ 1) * 4, __builtin_bit_cast(int, s[0])));
    if ((lane & 1) == 0) red[t >> 6][lane >> 1] = s[0];
    __syncthreads();
    if (t >= TM * TK) return;
    float v = 0.f;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) v += red[w][t];
    const int m = m0 + t / TK, k = k0 + t % TK;
    if (m < P.M && k < P.K) P.out[((long long)m * P.T + tap) * P.K + k] = v;
}

// floats from one row of weights to the next: lanes of different output channels read different banks
int lds_row(int T, int K) { return K % 4 ? T * K | 1 : 4 * (T * K / 4 | 1); }

TinyParams params(const Geom& g, int pass) {
    TinyParams P{};
    const bool dgrad = pass == MI3D_PASS_DGRAD, wgrad = pass == MI3D_PASS_WGRAD;
    P.add = (const float*)g.add; P.ref = (const float*)g.ref; P.slope = g.slope;
    P.K = dgrad ? g.Cout : g.Cin; P.M = dgrad ? g.Cin : g.Cout; P.T = (int)g.taps(); P.row = lds_row(P.T, P.K);
    P.iD = dgrad ? g.Do : g.D; P.iH = dgrad ? g.Ho : g.H; P.iW = dgrad ? g.Wo : g.W;
    P.oD = make_div(dgrad ? g.D : g.Do); P.oH = make_div(dgrad ? g.H : g.Ho); P.oW = make_div(dgrad ? g.W : g.Wo);
    P.Md = make_div(P.M); P.TKd = make_div(P.T * P.K); P.TMd = make_div(P.T * P.M);
    P.k[0] = g.kD; P.k[1] = g.kH; P.k[2] = g.kW; P.s[0] = g.sD; P.s[1] = g.sH; P.s[2] = g.sW; P.p[0] = g.pD; P.p[1] = g.pH; P.p[2] = g.pW;
    P.dgrad = dgrad;
    P.outputs = (int)((dgrad ? g.in_voxels() : g.out_voxels()) * (wgrad ? 1 : P.M));
    return P;
}

}  // namespace

// Measured on the device alone, with all launches, former kernels -> this one (forward, data gradient, weight gradient):
//   4->8 at 16^3         17.0 -> 6.5, 17.0 -> 8.0, 10.4 -> 7.2 us (and two, two and one launch of host time)
//   4->32 at 14^3        16.7 -> 8.1, 39.7 -> 22.2, 11.2 -> 7.0
//   8->16 at 16^3        17.0 -> 9.7, 25.0 -> 13.9, 11.3 -> 8.0
//   8->16, 2x2x2 at 16^3 13.0 -> 5.9, 12.2 -> 5.5, 8.3 -> 4.5
// The lines: weights of a workgroup within 48 KB, copied by each; 2^24 multiply-adds (14 M: 9.7 us) and sums of 864
// (1080: 17.7 -> 28.3, 648: 17.5 -> 19.4 with a launch less): one thread's chain; weight gradients to 8192 positions (10.5 us),
// 4096 where channels come one at a time (8000: 12.6 -> 33), and of those that igw_f32_kernel takes the ones for which wgrad_us
// expects less than that (5 us below its model at these sizes): a workgroup fetches whole lines for 16 and 32 bytes of a voxel's channels
// (igw_f32_kernel / this one, 2x2x2 32->64: 729 positions 10.4 / 7.8, 1728 11.2 / 14.0, 8000 15.6 / 48.8; 16->16 at 20^3 15.8 / 11.9;
// 1x1x1 32->32 at 16^3 9.6 / 9.3, at 20^3 11.5 / 14.8).  Not halves of an input, nor the whole tensors of layers that have
// them: both ways give the same bits.
static double wgrad_us(const Geom& g, long long groups) {
    const double V = (double)g.out_voxels();
    const int x = 4 * g.Cin * g.sW, y = 4 * g.Cout, line = 128, bytes = (x < line ? x : line) + (y < line ? y : line);   // per position
    const double us[3] = {0.85 * V / 1024, V * bytes / 150e3, groups * V * bytes / 20e6};    // trips of a thread, one CU's rate, what the L2s deliver
    return 2.5 + (us[0] > us[1] ? us[0] > us[2] ? us[0] : us[2] : us[1] > us[2] ? us[1] : us[2]);
}
bool tiny_supported(const Geom& g, int pass) {
    if (g.dtype != MI3D_F32 || g.Cin % 64 == 0 || g.kD > 3 || g.kH > 3 || g.kW > 3 || g.sD > 2 || g.sH > 2 || g.sW > 2) return false;
    const long long T = g.taps(), V = pass == MI3D_PASS_DGRAD ? g.in_voxels() : g.out_voxels();
    const long long K = pass == MI3D_PASS_DGRAD ? g.Cout : g.Cin, M = pass == MI3D_PASS_DGRAD ? g.Cin : g.Cout;
    if (pass == MI3D_PASS_WGRAD) {
        const long long groups = T * ((K + TK - 1) / TK) * ((M + TM - 1) / TM);
        if (V > (K % 4 || M % 4 ? 4096 : 8192) || groups > 512) return false;
        const double us = wgrad_us(g, groups);
        return us < 9.0 || !igw_supported(g) || us < igw_us(g, ~(size_t)0) - 5.0;    // (that model is never below 14)
    }
    return M * lds_row((int)T, (int)K) <= MAX_W && T * K <= 864 && V * M * T * K <= (16ll << 20);
}

int tiny_conv(const Geom& g, int pass, const void* in, const void* w, void* out, hipStream_t s) {
    TinyParams P = params(g, pass);
    P.in = (const float*)in; P.w = (const float*)w; P.out = (float*)out;
    const unsigned grid = (unsigned)((P.outputs + 255) / 256);
    const size_t lds = (size_t)P.M * P.row * sizeof(float);
    if (P.K % 4 == 0) tiny_conv_kernel<4><<<grid, 256, lds, s>>>(P);
    else tiny_conv_kernel<1><<<grid, 256, lds, s>>>(P);
    return check_launch();
}

int tiny_wgrad(const Geom& g, const void* x, const void* dy, float* dw, hipStream_t s) {
    TinyParams P = params(g, MI3D_PASS_WGRAD);
    P.in = (const float*)x; P.dy = (const float*)dy; P.out = dw;
    const unsigned grid = (unsigned)(P.T * ((P.K + TK - 1) / TK) * ((P.M + TM - 1) / TM));
    const unsigned threads = P.outputs >= 1024 ? 1024u : (unsigned)((P.outputs + 63) / 64 * 64);
    if (P.K % 4 == 0 && P.M % 4 == 0) tiny_wgrad_kernel<true><<<grid, threads, 0, s>>>(P);
    else tiny_wgrad_kernel<false><<<grid, threads, 0, s>>>(P);
    return check_launch();
}

}  // namespace mi3d
