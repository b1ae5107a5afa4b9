// What the kernels over numbered positions (implicit GEMM) share: division of position numbers by the extents of the volume,
// taps in one word, and the parity classes of a strided data gradient.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include "mi3d_internal.h"

namespace mi3d {

// make(): the plan for these sizes and this workspace.  A call asks for its plan up to five times (kernel choice, least
// workspace, models of the time, run) and one takes 1 to 3 us, a tenth of what the smallest layers take in all; so a thread keeps the
// last ones, by everything that make() may look at (the pointers of the geometry only as being there or not).
template <class Plan, class Make>
inline Plan kept_plan(const Geom& g, int pass, size_t ws_bytes, Make make) {
    struct Key {
        int sizes[19], pass, halves, cus;
        size_t ws_bytes;
    };
    struct Slot {
        Key key;
        Plan plan;
    };
    static_assert(offsetof(Geom, dtype) == 18 * sizeof(int), "the sizes are the first members of Geom");
    static thread_local Slot slots[32];       // (a key of zeros is that of no layer)
    Key k;
    memset(&k, 0, sizeof(k));
    memcpy(k.sizes, &g, sizeof(k.sizes));
    k.pass = pass; k.halves = g.hi ? 1 : 0; k.cus = cu_count(); k.ws_bytes = ws_bytes;
    uint64_t h = k.pass + 3 * k.ws_bytes;
    for (int v : k.sizes) h = h * 0x9E3779B97F4A7C15ull + (uint32_t)v;
    Slot& s = slots[h >> 59];
    if (memcmp(&s.key, &k, sizeof(k))) {
        s.plan = make();
        s.key = k;
    }
    return s.plan;
}

// x / d for 0 <= x < 2^31 by multiplication (Granlund and Montgomery, "Division by Invariant Integers using
// Multiplication", PLDI 1994): s = ceil(log2 d), m = floor(2^32 (2^s - d) / d) + 1
struct Div {
    uint32_t m, s, d;
};
inline Div make_div(uint32_t d) {
    uint32_t s = 0;
    while ((1ull << s) < d) ++s;
    return Div{(uint32_t)(((1ull << 32) * ((1ull << s) - d)) / d + 1), s, d};
}
__device__ __forceinline__ int divide(int x, const Div& v) {
    const uint64_t t = (uint64_t)__umulhi(v.m, (uint32_t)x) + (uint32_t)x;
    return (int)(t >> v.s);
}

// A tap in one word (scalar loads have no bytes): delta_t + 8 along d, h, w and the tap's index in the weights.
__host__ __device__ __forceinline__ uint32_t tap_word(int dd, int dh, int dw, int wt) { return (dd + 8) | (dh + 8) << 8 | (dw + 8) << 16 | (uint32_t)wt << 24; }
struct IgTap {
    int dd, dh, dw, wt;
    __device__ __forceinline__ IgTap(uint32_t v) : dd((int)(v & 255) - 8), dh((int)(v >> 8 & 255) - 8), dw((int)(v >> 16 & 255) - 8), wt((int)(v >> 24)) {}
};

// The taps of one axis for outputs of parity class par of the data gradient (out = s j + par reads in = j + delta), or of
// the forward pass (in = s j + delta): weight indices and deltas.  v / s is exact.
struct AxisTaps {
    int n, t[3], d[3];
};
inline AxisTaps axis_taps(int k, int s, int p, bool dgrad, int par) {
    AxisTaps a{0, {0, 0, 0}, {0, 0, 0}};
    for (int t = 0; t < k; ++t) {
        if (!dgrad) { a.t[a.n] = t; a.d[a.n++] = t - p; continue; }
        const int v = par + p - t;
        if (v % s) continue;
        a.t[a.n] = t; a.d[a.n++] = v / s;
    }
    return a;
}

// Fragment of v_mfma_f32_32x32x16_bf16 from rows of LDS that run along its other axis: rows 0 to 3 and 4 to 7 behind p, of this
// lane's column (a group of 16 lanes reads four rows of 16 columns and gets them transposed)
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
__device__ __forceinline__ bf16x8 tr_frag(const char* p, int row_bytes) {
    typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
    typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
    typedef __attribute__((address_space(3))) s16x4* lptr;
    s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr)(p));
    s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr)(p + 4 * row_bytes));
    s16x8 c = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, c);
}

// 16 bytes per lane from buffer r at byte offset off (zeros beyond its range) to the wave's 1 KB at LDS byte l.  Inline assembly:
// behind the builtin the compiler waits for all loads before every transposing LDS read.  A load to LDS takes M0 one wait state after
// a scalar instruction has written it: the compiler puts that in behind its builtin, inside an asm block nobody does.
__device__ __forceinline__ void load_lds_asm(__amdgpu_buffer_rsrc_t r, unsigned l, unsigned off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(l), "v"(off), "s"(r) : "memory", "m0");
}

}  // namespace mi3d
