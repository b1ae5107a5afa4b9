// Sums over exactly the window of one result, a product at a time in fp32: the plain kernels are made of them, and results
// of a padded layer that came out as NaN are formed again with them.
#pragma once
#include "mi3d_internal.h"

namespace mi3d {

template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ float load(const float* p) { return *p; }
    static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct Elem<uint16_t> {
    static __device__ __forceinline__ float load(const uint16_t* p) { return bf16_to_f32(*p); }
    static __device__ __forceinline__ void store(uint16_t* p, float v) { *p = f32_to_bf16_rne(v); }
};

// y[idx].  STOP: returns as soon as the sum is NaN (it stays one).
template <typename T, bool STOP = false>
__device__ __forceinline__ float fwd_sum(const Geom& g, const T* __restrict__ x, const T* __restrict__ w, long long idx) {
    int co = (int)(idx % g.Cout);
    long long v = idx / g.Cout;
    int ow = (int)(v % g.Wo); v /= g.Wo;
    int oh = (int)(v % g.Ho); v /= g.Ho;
    int od = (int)(v % g.Do);
    int n = (int)(v / g.Do);
    float acc = 0.f;
    for (int kd = 0; kd < g.kD; ++kd) {
        int id = od * g.sD - g.pD + kd;
        if (id < 0 || id >= g.D) continue;
        for (int kh = 0; kh < g.kH; ++kh) {
            int ih = oh * g.sH - g.pH + kh;
            if (ih < 0 || ih >= g.H) continue;
            for (int kw = 0; kw < g.kW; ++kw) {
                int iw = ow * g.sW - g.pW + kw;
                if (iw < 0 || iw >= g.W) continue;
                const T* xp = x + ((((long long)n * g.D + id) * g.H + ih) * g.W + iw) * g.Cin;
                const T* wp = w + ((((long long)co * g.kD + kd) * g.kH + kh) * g.kW + kw) * g.Cin;
                for (int ci = 0; ci < g.Cin; ++ci) acc = fmaf(Elem<T>::load(xp + ci), Elem<T>::load(wp + ci), acc);
                if (STOP && acc != acc) return acc;
            }
        }
    }
    return acc;
}

// dx[idx]
template <typename T, bool STOP = false>
__device__ __forceinline__ float dgrad_sum(const Geom& g, const T* __restrict__ dy, const T* __restrict__ w, long long idx) {
    int ci = (int)(idx % g.Cin);
    long long v = idx / g.Cin;
    int iw = (int)(v % g.W); v /= g.W;
    int ih = (int)(v % g.H); v /= g.H;
    int id = (int)(v % g.D);
    int n = (int)(v / g.D);
    float acc = 0.f;
    for (int kd = 0; kd < g.kD; ++kd) {
        int nd = id + g.pD - kd;
        if (nd < 0 || nd % g.sD) continue;
        int od = nd / g.sD;
        if (od >= g.Do) continue;
        for (int kh = 0; kh < g.kH; ++kh) {
            int nh = ih + g.pH - kh;
            if (nh < 0 || nh % g.sH) continue;
            int oh = nh / g.sH;
            if (oh >= g.Ho) continue;
            for (int kw = 0; kw < g.kW; ++kw) {
                int nw = iw + g.pW - kw;
                if (nw < 0 || nw % g.sW) continue;
                int ow = nw / g.sW;
                if (ow >= g.Wo) continue;
                const T* gp = dy + ((((long long)n * g.Do + od) * g.Ho + oh) * g.Wo + ow) * g.Cout;
                const T* wp = w + (((long long)kd * g.kH + kh) * g.kW + kw) * g.Cin + ci;
                long long wstride = g.taps() * g.Cin;
                for (int co = 0; co < g.Cout; ++co) acc = fmaf(Elem<T>::load(gp + co), Elem<T>::load(wp + co * wstride), acc);
                if (STOP && acc != acc) return acc;
            }
        }
    }
    return acc;
}

// One output voxel's product of dw[co][t][ci], added to acc (unchanged where the tap lies outside the volume).
template <typename T>
__device__ __forceinline__ float wgrad_add(const Geom& g, const T* __restrict__ x, const T* __restrict__ dy, int co, int kd, int kh, int kw, int ci,
                                           long long v, float acc) {
    long long r = v;
    int ow = (int)(r % g.Wo); r /= g.Wo;
    int oh = (int)(r % g.Ho); r /= g.Ho;
    int od = (int)(r % g.Do);
    int n = (int)(r / g.Do);
    int id = od * g.sD - g.pD + kd, ih = oh * g.sH - g.pH + kh, iw = ow * g.sW - g.pW + kw;
    if (id < 0 || id >= g.D || ih < 0 || ih >= g.H || iw < 0 || iw >= g.W) return acc;
    float a = Elem<T>::load(dy + v * g.Cout + co);
    float b = Elem<T>::load(x + ((((long long)n * g.D + id) * g.H + ih) * g.W + iw) * g.Cin + ci);
    return fmaf(a, b, acc);
}

}  // namespace mi3d
