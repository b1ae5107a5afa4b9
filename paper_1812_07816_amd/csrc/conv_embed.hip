// Layers no tuned kernel covers on the MFMA kernels.  Ragged channel counts that come in eights run as they are on the kernels
// over numbered positions where that is faster (ragged_*: 3x3x3); everything else embeds its operands:
//   - channel counts that are not multiples of 32: operands are zero-padded, results
//     sliced back;
//   - strided layers: the forward pass is the stride-1 result subsampled;
//     for the gradients dy is spread onto the stride-1 output grid (zeros in
//     between), after which dx and dw are exactly the stride-1 gradients.
// They trade extra MFMA work and one extra pass over a tensor for not falling
// back to the plain kernels; dedicated kernels replace them where it matters.
#include "conv_window.h"

namespace mi3d {
namespace {

// Zero-padding of channel rows: dst[v][0..CP) = src[v][0..C) followed by zeros for v < rows, all zeros for the rows up to
// rows_p.  Two independent jobs share a launch (the activations and the weights of a pass): these passes take a few
// microseconds each, about what a launch costs.  One thread per 8 channels of dst; rows whose length is a multiple of 8
// are read 16 bytes at a time.  wflag (null: none): one word per block of the job `weights` (0 or 1), 1 where the block
// met an infinity or a NaN.
struct PadJob {
    const uint16_t* src;
    uint16_t* dst;
    long long rows, rows_p;
    int C, CP;
    __host__ __device__ long long threads() const { return rows_p * (CP / 8); }
};
__device__ __forceinline__ bool bf16_nonfinite(uint32_t v) { return (v & 0x7F80u) == 0x7F80u; }
__device__ __forceinline__ bool pair_nonfinite(uint32_t v) { return bf16_nonfinite(v) | bf16_nonfinite(v >> 16); }
__global__ void __launch_bounds__(256) pad_channels_kernel(PadJob a, PadJob b, uint32_t* __restrict__ wflag, int weights) {
    long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    const bool second = idx >= a.threads();
    if (second) idx -= a.threads();
    const PadJob& J = second ? b : a;
    uint4 out = {0, 0, 0, 0};
    if (idx < J.threads()) {
        const int per = J.CP / 8;
        const long long v = idx / per;
        const int c0 = (int)(idx - v * per) * 8;
        if (v < J.rows) {
            const uint16_t* src = J.src + v * J.C + c0;
            if (J.C % 8 == 0) {
                if (c0 < J.C) out = *(const uint4*)src;
            } else {
                uint32_t o[4] = {0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (c0 + j < J.C) o[j >> 1] |= (uint32_t)src[j] << (16 * (j & 1));
                out = uint4{o[0], o[1], o[2], o[3]};
            }
        }
        *(uint4*)(J.dst + v * J.CP + c0) = out;
    }
    if (!wflag) return;
    const int first = weights ? (int)(a.threads() / 256) : 0;   // block in which the weights begin
    if ((int)blockIdx.x < first) return;
    const bool bad = second == (weights == 1) && (pair_nonfinite(out.x) | pair_nonfinite(out.y) | pair_nonfinite(out.z) | pair_nonfinite(out.w));
    const int any = __syncthreads_or(bad);
    if (threadIdx.x == 0) wflag[blockIdx.x - first] = any ? 1u : 0u;
}
// the same with rows padded to 4 channels (inputs with fewer than 4 channels): one thread per row
__global__ void __launch_bounds__(256) pad_to4_kernel(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, long long rows, long long rows_p, int C,
                                                      uint32_t* __restrict__ wflag) {
    const long long v = (long long)blockIdx.x * 256 + threadIdx.x;
    uint32_t o[2] = {0, 0};
    if (v < rows)
        for (int j = 0; j < C; ++j) o[j >> 1] |= (uint32_t)src[v * C + j] << (16 * (j & 1));
    if (v < rows_p) *(uint2*)(dst + v * 4) = uint2{o[0], o[1]};
    if (!wflag) return;
    const int any = __syncthreads_or(pair_nonfinite(o[0]) | pair_nonfinite(o[1]));
    if (threadIdx.x == 0) wflag[blockIdx.x] = any ? 1u : 0u;
}

// ---- results of the padded layer ----
// The matrix-core kernels add zeros where a window or a patch leaves the volume, and 0 x inf is NaN: a NaN of theirs need
// not be one.  Whatever comes out as NaN is formed again as the sum over its window alone; other values cannot have met
// such a zero.  Looking for them costs nothing where results are sliced and a launch where they are not (padded 48 -> 48 at
// 37 x 50 x 61 222.9 -> 223.9 us, 40 -> 96 forward at 64^3 126 -> 130), as in layers that are read as they are; with nothing
// but NaN in all operands a pass costs about what the plain kernels take (48 -> 48 weight gradient 43 ms).

// y or dx, channels [0, C) of CP-channel rows; V elements per thread (16 bytes, or one where C is not a multiple of 8)
__device__ __forceinline__ uint16_t exact_bf16(const Geom& g, int pass, const uint16_t* in, const uint16_t* w, long long e) {
    return f32_to_bf16_rne(pass == MI3D_PASS_FWD ? fwd_sum<uint16_t, true>(g, in, w, e) : dgrad_sum<uint16_t, true>(g, in, w, e));
}
__device__ __forceinline__ bool bf16_nan(uint32_t v) { return (v & 0x7FFFu) > 0x7F80u; }
__device__ __forceinline__ bool pair_nan(uint32_t v) { return bf16_nan(v) | bf16_nan(v >> 16); }
__device__ __forceinline__ uint32_t exact_pair(const Geom& g, int pass, const uint16_t* in, const uint16_t* w, long long e, uint32_t v) {
    if (bf16_nan(v)) v = (v & 0xFFFF0000u) | exact_bf16(g, pass, in, w, e);
    if (bf16_nan(v >> 16)) v = (v & 0xFFFFu) | (uint32_t)exact_bf16(g, pass, in, w, e + 1) << 16;
    return v;
}
template <int V>
__global__ void __launch_bounds__(256) slice_channels_kernel(Geom g, int pass, const uint16_t* __restrict__ in, const uint16_t* __restrict__ w,
                                                             const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, long long voxels, int C, int CP) {
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    const int per = C / V;
    if (idx >= voxels * per) return;
    const long long v = idx / per;
    const int c = (int)(idx - v * per) * V;
    if constexpr (V == 1) {
        uint16_t o = src[v * CP + c];
        if (bf16_nan(o)) o = exact_bf16(g, pass, in, w, idx);
        dst[idx] = o;
    } else {
        uint4 o = *(const uint4*)(src + v * CP + c);
        if (pair_nan(o.x) | pair_nan(o.y) | pair_nan(o.z) | pair_nan(o.w)) {
            uint32_t q[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) q[j] = exact_pair(g, pass, in, w, idx * 8 + 2 * j, q[j]);
            o = uint4{q[0], q[1], q[2], q[3]};
        }
        *(uint4*)(dst + idx * 8) = o;
    }
}

// One word per block of 256 x 8 weights: 1 where the block met an infinity or a NaN (n a multiple of 8)
__global__ void __launch_bounds__(256) weight_flags_kernel(const uint16_t* __restrict__ w, long long n8, uint32_t* __restrict__ flags) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    uint4 v = {0, 0, 0, 0};
    if (i < n8) v = *(const uint4*)(w + 8 * i);
    const int any = __syncthreads_or(pair_nonfinite(v.x) | pair_nonfinite(v.y) | pair_nonfinite(v.z) | pair_nonfinite(v.w));
    if (threadIdx.x == 0) flags[blockIdx.x] = any ? 1u : 0u;
}

// The same in place, for results that need no slicing (a multiple of 4 elements): only where a weight is not finite (flags
// of the padding kernel; the kernels keep to the window of an activation), or, with flags null, on any NaN.
__global__ void __launch_bounds__(256) exact_in_place_kernel(Geom g, int pass, const uint16_t* __restrict__ in, const uint16_t* __restrict__ w,
                                                             uint16_t* __restrict__ out, long long n4, const uint32_t* __restrict__ flags, int nflags) {
    if (flags) {
        uint32_t f = 0;
        for (int i = threadIdx.x; i < nflags; i += 256) f |= flags[i];
        if (!__syncthreads_or((int)f)) return;
    }
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n4; i += (long long)gridDim.x * 256) {
        const uint2 o = *(const uint2*)(out + 4 * i);
        if (pair_nan(o.x) | pair_nan(o.y))
            *(uint2*)(out + 4 * i) = uint2{exact_pair(g, pass, in, w, 4 * i, o.x), exact_pair(g, pass, in, w, 4 * i + 2, o.y)};
    }
}

// dw, V elements per thread (src may be dst: nothing to slice).  The NaN of a block are formed again one after the other by all its threads: partial sums
// over every 256th voxel, added in a fixed order.
template <int V>
__global__ void __launch_bounds__(256) slice_dw_kernel(Geom g, const uint16_t* __restrict__ x, const uint16_t* __restrict__ dy, const float* src,
                                                       float* dst, int CP) {
    const int t = threadIdx.x;
    const long long idx = (long long)blockIdx.x * 256 + t, rows = g.taps() * g.Cout;
    const int C = g.Cin, per = C / V;
    bool nan = false;
    if (idx < rows * per) {
        const long long v = idx / per;
        const int c = (int)(idx - v * per) * V;
        if constexpr (V == 1) {
            const float o = dst[idx] = src[v * CP + c];
            nan = o != o;
        } else {
            const float4 o = *(float4*)(dst + 4 * idx) = *(const float4*)(src + v * CP + c);
            nan = (o.x != o.x) | (o.y != o.y) | (o.z != o.z) | (o.w != o.w);
        }
    }
    if (!__syncthreads_or(nan)) return;
    __shared__ float red[256];
    const long long first = (long long)blockIdx.x * 256 * V, last = first + 256 * V < rows * C ? first + 256 * V : rows * C, vox = g.out_voxels();
    for (long long e = first; e < last; ++e) {
        const float now = dst[e];      // (each element is written by this block alone, before the barrier above or at the end of its turn)
        if (!__syncthreads_or(now != now)) continue;
        const int ci = (int)(e % C);
        const long long r = e / C;
        const int tap = (int)(r % g.taps()), co = (int)(r / g.taps());
        const int kd = tap / (g.kH * g.kW), kh = tap / g.kW % g.kH, kw = tap % g.kW;
        float acc = 0.f;
        for (long long v0 = 0; v0 < vox; v0 += 256 * 64) {
            const long long v1 = v0 + 256 * 64 < vox ? v0 + 256 * 64 : vox;
            for (long long v = v0 + t; v < v1; v += 256) acc = wgrad_add(g, x, dy, co, kd, kh, kw, ci, v, acc);
            if (__syncthreads_or(acc != acc)) break;       // NaN it stays
        }
        red[t] = acc;
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if (t < h) red[t] += red[t + h];
            __syncthreads();
        }
        if (t == 0) dst[e] = red[0];
        __syncthreads();
    }
}

// up[n][s*od][s*oh][s*ow][:] = dy[n][od][oh][ow][:], zero elsewhere; up has extents (Du,Hu,Wu).
// One thread per 16 bytes of up.
__global__ void __launch_bounds__(256) spread_kernel(const uint16_t* __restrict__ dy, uint16_t* __restrict__ up, int N, int Do, int Ho,
                                                     int Wo, int Du, int Hu, int Wu, int C, int sD, int sH, int sW) {
    const int per = C / 8;
    long long total = (long long)N * Du * Hu * Wu * per;
    long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    int c8 = (int)(idx % per);
    long long v = idx / per;
    int w = (int)(v % Wu); v /= Wu;
    int h = (int)(v % Hu); v /= Hu;
    int d = (int)(v % Du);
    int n = (int)(v / Du);
    uint4 val = {0, 0, 0, 0};
    if (d % sD == 0 && h % sH == 0 && w % sW == 0) {
        int od = d / sD, oh = h / sH, ow = w / sW;
        if (od < Do && oh < Ho && ow < Wo)
            val = *(const uint4*)(dy + ((((long long)n * Do + od) * Ho + oh) * Wo + ow) * C + c8 * 8);
    }
    *(uint4*)(up + idx * 8) = val;
}

// y[n][od][oh][ow][:] = full[n][s*od][s*oh][s*ow][:]; one thread per 16 bytes of y
__global__ void __launch_bounds__(256) subsample_kernel(const uint16_t* __restrict__ full, uint16_t* __restrict__ y, int N, int Do, int Ho,
                                                        int Wo, int Du, int Hu, int Wu, int C, int sD, int sH, int sW) {
    const int per = C / 8;
    long long total = (long long)N * Do * Ho * Wo * per;
    long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    int c8 = (int)(idx % per);
    long long v = idx / per;
    int ow = (int)(v % Wo); v /= Wo;
    int oh = (int)(v % Ho); v /= Ho;
    int od = (int)(v % Do);
    int n = (int)(v / Do);
    *(uint4*)(y + idx * 8) = *(const uint4*)(full + ((((long long)n * Du + od * sD) * Hu + oh * sH) * Wu + ow * sW) * C + c8 * 8);
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

unsigned blocks_for(long long n) { return (unsigned)((n + 255) / 256); }

}  // namespace

// ---- channel counts that no MFMA kernel takes --------------------------------
// The padded layer: channels rounded up to multiples of 32, or input channels to 4 where the first-layer kernels then apply.
// 2x2x2 layers get multiples of 64: the kernel for them takes those, the embedding into 3x3x3 reads voxels outside the
// window, times zero, and does 27/8 of the work (24->24 at 30^3, N = 2, padded to 32 / to 64: 28.7 / 18.8, 22.4 / 18.4, 32.4 / 22.2 us
// for the three passes; 64->96 at 48^3 embedded / padded to 128: 47 / 26, 81 / 20, 40 / 27).  Layers of 32 output channels that
// need no padding otherwise stay with the embedding (32->32 at 96^3 31 / 27, 32 / 36, 31 / 45).
static Geom padded_geom(const Geom& g, int pass) {
    Geom p = g;
    p.Cout = (g.Cout + 31) / 32 * 32;
    if (g.Cin <= 4) {
        p.Cin = 4;
        if (pass == MI3D_PASS_FWD ? c4_fwd_supported(p) : pass == MI3D_PASS_DGRAD ? c4_dgrad_supported(p) : c4_wgrad_supported(p)) return p;
    }
    p.Cin = (g.Cin + 31) / 32 * 32;
    const bool ragged = p.Cin != g.Cin || p.Cout != g.Cout;
    if (g.kD == 2 && (ragged || p.Cout > 32)) p.Cout = (p.Cout + 63) / 64 * 64;
    return p;
}

// bytes of the padded operands and result in the workspace: x-shaped, y-shaped, weight-shaped tensors, flags of the
// weights (0: not needed)
struct EmbedC {
    Geom p;
    size_t xb, yb, wb, fb;
};
static long long weight_threads(const Geom& p) { return p.taps() * p.Cout * (p.Cin % 8 ? 1 : p.Cin / 8); }   // of the padding kernels
static EmbedC embed_c_layout(const Geom& g, int pass) {
    EmbedC e{padded_geom(g, pass), 0, 0, 0, 0};
    const bool ci = e.p.Cin != g.Cin, co = e.p.Cout != g.Cout;
    if (ci) e.xb = align256((size_t)g.in_voxels() * e.p.Cin * 2);
    if (co) e.yb = align256((size_t)g.out_voxels() * e.p.Cout * 2);
    if (ci || co) e.wb = align256((size_t)e.p.w_elems() * (pass == MI3D_PASS_WGRAD ? 4 : 2));
    if (e.wb && (pass == MI3D_PASS_FWD ? !co : pass == MI3D_PASS_DGRAD && !ci)) e.fb = align256((size_t)(weight_threads(e.p) / 256 + 2) * 4);
    return e;
}

bool embed_c_supported(const Geom& g, int pass) {
    if (g.dtype != MI3D_BF16) return false;
    const EmbedC e = embed_c_layout(g, pass);
    if (!e.wb || e.xb + e.yb > (16ull << 30)) return false;   // (copies of more than 16 GiB: the plain kernels need none)
    return auto_is_mfma(e.p, pass);
}

size_t embed_c_workspace_bytes(const Geom& g, int pass) {
    if (!embed_c_supported(g, pass)) return 0;
    const EmbedC e = embed_c_layout(g, pass);
    return e.xb + e.yb + e.wb + e.fb + align256(auto_workspace_bytes(e.p, pass));
}

size_t embed_c_min_workspace_bytes(const Geom& g, int pass) {
    if (!embed_c_supported(g, pass)) return 0;
    const EmbedC e = embed_c_layout(g, pass);
    return e.xb + e.yb + e.wb + auto_min_workspace_bytes(e.p, pass);
}

// ---- channel counts in eights that 32 does not divide ------------------------
// 3x3x3 layers that the kernels over numbered positions take as they are, without copies of the operands (padded -> as they
// are, 48 -> 48 at 37 x 50 x 61: 225 -> 124 us for the three passes); smaller volumes are padded.
//
// Where padding serves them better, from about 500 layers measured both ways (padded / as they are, us).  A tensor whose
// channels 32 divides needs no copy, and on large volumes the kernels behind the padding, which read a voxel once for all of its
// taps, beat those that read it for each.
// - Unit stride, contracted channels a multiple of 32, more than one round of 512 tiles of 256 positions: forward 96->16 at
//   288144 voxels 92 / 126, 160->8 at 905760 257 / 604, data gradient 16->160 at 254016 101 / 240 (below: 96->16 at 102131 55 / 48,
//   128->48 at 88560 70 / 65).  The exceptions: 128->40 at 303030 200 / 176.  (Not where the implicit GEMM runs behind the
//   padding as well: 128->8 at 155288 103 / 87.)
// - Unit stride, outputs a multiple of 32: steps of so few channels pay only where tiles of outputs are badly filled (24 channels: 24->96
//   at 687792 153 / 179, 24->32 at 913140 110 / 133; 16->32 at 864270 104 / 115, 8->160 at 905760 253 / 317, but 16->64 at
//   909455 142 / 129 and 40->96 at 313000 155 / 122).
// - Stride 2, forward: only 32 channels have a kernel of their own behind the padding (32->48 at 300300 80 / 125, at 36704 29 / 37;
//   64->24 at 110880 55 / 51).  Data gradient: up to 64 contracted channels have one, which wins on large volumes (64->24 at
//   859473 voxels 55 / 64, 48->32 at 2365860 113 / 136, 24->64 at 17 M 684 / 1353; 64->48 at 9.5 M 777 / 840, at 254040 42 / 29).
// - Weight gradient: by the models of the time of both, padding at 2 TB/s (0.3 % above the better way over 570 layers, 20 % at
//   most): 64->16 at 1044576 168 / 446, 128->24 at 499824 121 / 405, 104->8 at 304732 146 / 200; but 48->48 at
//   37 x 50 x 61 as it is.
static bool padding_better(const Geom& g, const Geom& p, int pass) {
    const bool ci = p.Cin != g.Cin, co = p.Cout != g.Cout;
    if (pass == MI3D_PASS_WGRAD) {
        const bool s1 = wgrad_mfma_supported(p);
        if (s1 ? wgrad_mfma_uses_igw(p, ~(size_t)0) : !wgrad_s2_supported(p) || wgrad_s2_uses_igw(p, ~(size_t)0)) return false;   // (the same kernel, or one behind further copies)
        const double bytes = (ci ? g.in_voxels() * 2.0 * (g.Cin + p.Cin) : 0.0) + (co ? g.out_voxels() * 2.0 * (g.Cout + p.Cout) : 0.0);
        return igw_us(g, ~(size_t)0) > (s1 ? wgrad_mfma_patches_us(p) : wgrad_s2_patches_us(p)) + 8.0 + bytes / 2e6;
    }
    const bool dgrad = pass == MI3D_PASS_DGRAD, k_whole = dgrad ? !co : !ci, m_whole = dgrad ? !ci : !co;
    const int K = dgrad ? g.Cout : g.Cin, M = dgrad ? g.Cin : g.Cout;
    const long long voxels = dgrad ? g.in_voxels() : g.out_voxels();
    if ((!k_whole && !m_whole) || (sp_supported(p, pass) && sp_uses_ig(p, pass))) return false;
    if (g.sD == 1) return k_whole ? voxels > 512 * 256 : K <= 24 && voxels > (1 << 18) && (K == 24 || M == 32 || (M > 128 && M % 64 == 32));
    if (!dgrad) return K == 32 && voxels > (1 << 15);
    return p.Cout <= 64 && voxels > (!k_whole || M <= 32 ? 1 << 19 : 1 << 22);
}

bool ragged_supported(const Geom& g, int pass) {
    if (g.dtype != MI3D_BF16 || g.Cin % 8 || g.Cout % 8 || g.kD != 3 || g.kH != 3 || g.kW != 3) return false;
    const Geom p = padded_geom(g, pass);
    if ((p.Cin == g.Cin && p.Cout == g.Cout) || !auto_is_mfma(p, pass)) return false;
    if (pass == MI3D_PASS_WGRAD) return igw_supported(g);
    return ig_takes(g, pass) && g.out_voxels() >= 1024;
}
bool ragged_better(const Geom& g, int pass) { return !embed_c_supported(g, pass) || !padding_better(g, padded_geom(g, pass), pass); }
static int weight_flag_words(const Geom& g, int pass) {
    return pass == MI3D_PASS_FWD ? (int)((g.w_elems() / 8 + 255) / 256) : 27 * ((g.Cin + 63) / 64) * ((g.Cout + 63) / 64);
}

static size_t weight_flag_bytes(const Geom& g, int pass) { return pass == MI3D_PASS_WGRAD ? 0 : align256((size_t)weight_flag_words(g, pass) * 4); }

size_t ragged_min_workspace_bytes(const Geom& g, int pass) { return pass == MI3D_PASS_WGRAD ? 0 : ig_min_workspace_bytes(g, pass); }
size_t ragged_workspace_bytes(const Geom& g, int pass) { return pass == MI3D_PASS_WGRAD ? igw_workspace_bytes(g) : weight_flag_bytes(g, pass) + ig_workspace_bytes(g, pass); }
// (less than the flags want on top of the least: every result is looked at)
static size_t ragged_flags_within(const Geom& g, int pass, size_t ws_bytes) {
    const size_t fb = weight_flag_bytes(g, pass);
    return ws_bytes >= fb + ragged_min_workspace_bytes(g, pass) ? fb : 0;
}
void ragged_describe(const Geom& g, int pass, size_t ws_bytes, char* buf, size_t len) {
    if (pass == MI3D_PASS_WGRAD) igw_describe(g, ws_bytes, buf, len);
    else ig_describe(g, pass, ws_bytes - ragged_flags_within(g, pass, ws_bytes), buf, len);
}

// Its NaN are formed again like those of a padded layer
int ragged_conv(const Geom& g, int pass, const void* a, const void* b, void* out, void* ws, size_t ws_bytes, hipStream_t s) {
    int st;
    if (pass == MI3D_PASS_WGRAD) {
        if ((st = igw_run(g, a, b, (float*)out, ws, ws_bytes, s))) return st;
        slice_dw_kernel<4><<<blocks_for(g.w_elems() / 4), 256, 0, s>>>(g, (const uint16_t*)a, (const uint16_t*)b, (const float*)out, (float*)out, g.Cin);
        return check_launch();
    }
    const int nflags = weight_flag_words(g, pass);
    const size_t fb = ragged_flags_within(g, pass, ws_bytes);
    uint32_t* flags = fb ? (uint32_t*)ws : nullptr;
    if (flags && pass == MI3D_PASS_FWD) {
        weight_flags_kernel<<<(unsigned)nflags, 256, 0, s>>>((const uint16_t*)b, g.w_elems() / 8, flags);
        if ((st = check_launch())) return st;
    }
    if ((st = ig_conv(g, pass, a, b, out, (char*)ws + fb, ws_bytes - fb, s, flags))) return st;
    const long long n4 = (pass == MI3D_PASS_FWD ? g.out_voxels() * g.Cout : g.in_voxels() * g.Cin) / 4;
    exact_in_place_kernel<<<(unsigned)(n4 < 256 * 256 ? (n4 + 255) / 256 : 256), 256, 0, s>>>(g, pass, (const uint16_t*)a, (const uint16_t*)b, (uint16_t*)out, n4, flags, nflags);
    return check_launch();
}

Geom embed_c_inner(const Geom& g, int pass, size_t ws_bytes, size_t* rest) {
    EmbedC e = embed_c_layout(g, pass);
    if (ws_bytes < embed_c_workspace_bytes(g, pass)) e.fb = 0;
    *rest = ws_bytes - e.xb - e.yb - e.wb - e.fb;
    return e.p;
}

// Bound: the copies are a pass over each operand and one more launch, the plain kernels do one product at a time per thread.
// The three passes, plain kernels -> padded: 48 -> 48 channels at 37 x 50 x 61 34.5 -> 0.22 ms (as it is: 0.12), 8 -> 16 at 6^3
// 0.140 -> 0.061, 40 -> 48 at 12^3 0.98 -> 0.084, 24 -> 48 at 10^3 with stride 2 0.171 -> 0.064: the padded layer wins at every
// size, so the plain kernels are left with the geometries no matrix-core kernel takes.
int embed_c_conv(const Geom& g, int pass, const void* a, const void* b, void* out, void* ws, size_t ws_bytes, hipStream_t s) {
    if (ws_bytes < embed_c_min_workspace_bytes(g, pass)) return MI3D_ERR_WORKSPACE;
    EmbedC e = embed_c_layout(g, pass);
    if (ws_bytes < embed_c_workspace_bytes(g, pass)) e.fb = 0;      // no room for flags: every result is looked at
    const Geom& p = e.p;
    uint16_t* xp = (uint16_t*)ws;
    uint16_t* yp = (uint16_t*)((char*)ws + e.xb);
    void* wp = (char*)ws + e.xb + e.yb;
    uint32_t* flags = e.fb ? (uint32_t*)((char*)wp + e.wb) : nullptr;
    void* rest = (char*)wp + e.wb + e.fb;
    const size_t rest_bytes = ws_bytes - e.xb - e.yb - e.wb - e.fb;
    const long long T = g.taps();
    int st = MI3D_OK;
    // operands: the activations that are read (x, dy) and the weights, in one launch
    PadJob jobs[2] = {};
    int n = 0, nflags = 0;
    auto add = [&](const void* src, void* dst, long long rows, long long rows_p, int C, int CP, uint32_t* f) {
        if (CP % 8 == 0) { jobs[n++] = PadJob{(const uint16_t*)src, (uint16_t*)dst, rows, rows_p, C, CP}; return; }
        pad_to4_kernel<<<blocks_for(rows_p), 256, 0, s>>>((const uint16_t*)src, (uint16_t*)dst, rows, rows_p, C, f);   // (4 channels)
        if (f) nflags = (int)blocks_for(rows_p);
        st = check_launch();
    };
    const void* x = pass == MI3D_PASS_DGRAD ? nullptr : a;
    const void* dy = pass == MI3D_PASS_DGRAD ? a : (pass == MI3D_PASS_WGRAD ? b : nullptr);
    if (x && e.xb) { add(x, xp, g.in_voxels(), g.in_voxels(), g.Cin, p.Cin, nullptr); x = xp; }
    if (st) return st;
    if (dy && e.yb) { add(dy, yp, g.out_voxels(), g.out_voxels(), g.Cout, p.Cout, nullptr); dy = yp; }
    if (pass != MI3D_PASS_WGRAD) add(b, wp, T * g.Cout, T * p.Cout, g.Cin, p.Cin, flags);
    if (st) return st;
    if (n) {
        const unsigned blocks = blocks_for(jobs[0].threads() + (n > 1 ? jobs[1].threads() : 0));
        uint32_t* f = p.Cin % 8 ? nullptr : flags;     // (weights of 4 channels have had their launch)
        if (f) nflags = (int)blocks - (n > 1 ? (int)(jobs[0].threads() / 256) : 0);
        pad_channels_kernel<<<blocks, 256, 0, s>>>(jobs[0], jobs[1], f, n - 1);
        if ((st = check_launch())) return st;
    }
    // the padded layer, then the channels that were asked for
    if (pass == MI3D_PASS_WGRAD) {
        if ((st = auto_conv(p, pass, x, dy, wp, rest, rest_bytes, s))) return st;
        const long long rows = T * g.Cout;
        if (g.Cin % 4 == 0) slice_dw_kernel<4><<<blocks_for(rows * (g.Cin / 4)), 256, 0, s>>>(g, (const uint16_t*)a, (const uint16_t*)b, (const float*)wp, (float*)out, p.Cin);
        else slice_dw_kernel<1><<<blocks_for(rows * g.Cin), 256, 0, s>>>(g, (const uint16_t*)a, (const uint16_t*)b, (const float*)wp, (float*)out, p.Cin);
        return check_launch();
    }
    const bool fwd = pass == MI3D_PASS_FWD;
    const int C = fwd ? g.Cout : g.Cin, CP = fwd ? p.Cout : p.Cin;
    uint16_t* padded_out = C != CP ? (fwd ? yp : xp) : (uint16_t*)out;
    if ((st = auto_conv(p, pass, fwd ? x : dy, wp, padded_out, rest, rest_bytes, s))) return st;
    const long long rows = fwd ? g.out_voxels() : g.in_voxels();
    const uint16_t *in = (const uint16_t*)a, *w = (const uint16_t*)b;
    if (C == CP) {
        // (the 3x3x3 embedding of a 2x2x2 layer reads beyond the window; the data gradient of 4 channels adds zero rows)
        const bool any = (g.kD == 2 && !k2_supported(p, pass)) || C == 4;
        const long long n4 = rows * C / 4;
        exact_in_place_kernel<<<(unsigned)(n4 < 256 * 256 ? (n4 + 255) / 256 : 256), 256, 0, s>>>(g, pass, in, w, (uint16_t*)out, n4, any ? nullptr : flags, nflags);
    } else if (C % 8 == 0) {
        slice_channels_kernel<8><<<blocks_for(rows * (C / 8)), 256, 0, s>>>(g, pass, in, w, padded_out, (uint16_t*)out, rows, C, CP);
    } else {
        slice_channels_kernel<1><<<blocks_for(rows * C), 256, 0, s>>>(g, pass, in, w, padded_out, (uint16_t*)out, rows, C, CP);
    }
    return check_launch();
}

// ---- stride > 1 gradients through the stride-1 kernels -------------------
static Geom unit_stride_geom(const Geom& g) {
    Geom u = g;
    u.sD = u.sH = u.sW = 1;
    u.Do = g.D + 2 * g.pD - g.kD + 1;
    u.Ho = g.H + 2 * g.pH - g.kH + 1;
    u.Wo = g.W + 2 * g.pW - g.kW + 1;
    return u;
}

bool embed_s_supported(const Geom& g, int pass) {
    if (g.dtype != MI3D_BF16 || (g.sD == 1 && g.sH == 1 && g.sW == 1)) return false;
    if (g.Cout % 8) return false;
    Geom u = unit_stride_geom(g);
    if (pass == MI3D_PASS_WGRAD) return wgrad_mfma_supported(u);
    return sp_supported(u, pass);   // forward: full-resolution output, then subsampled
}

static size_t embed_s_bytes(const Geom& g, int pass, bool least) {
    if (!embed_s_supported(g, pass)) return 0;
    Geom u = unit_stride_geom(g);
    size_t up = align256((size_t)u.out_voxels() * g.Cout * 2);
    if (pass == MI3D_PASS_WGRAD) return up + (least ? wgrad_mfma_min_workspace_bytes(u) : align256(wgrad_mfma_workspace_bytes(u)));
    return up + (least ? sp_min_workspace_bytes(u, pass) : align256(sp_workspace_bytes(u, pass)));
}
size_t embed_s_workspace_bytes(const Geom& g, int pass) { return embed_s_bytes(g, pass, false); }
size_t embed_s_min_workspace_bytes(const Geom& g, int pass) { return embed_s_bytes(g, pass, true); }

Geom embed_s_inner(const Geom& g, size_t ws_bytes, size_t* rest) {
    const Geom u = unit_stride_geom(g);
    *rest = ws_bytes - align256((size_t)u.out_voxels() * g.Cout * 2);
    return u;
}

// fwd: a = x, b = w, out = y.  dgrad: a = dy, b = w, out = dx.  wgrad: a = x, b = dy, out = dw.
int embed_s_conv(const Geom& g, int pass, const void* a, const void* b, void* out, void* ws, size_t ws_bytes, hipStream_t s) {
    if (ws_bytes < embed_s_min_workspace_bytes(g, pass)) return MI3D_ERR_WORKSPACE;
    Geom u = unit_stride_geom(g);
    const size_t upb = align256((size_t)u.out_voxels() * g.Cout * 2);
    uint16_t* up = (uint16_t*)ws;
    void* rest = (char*)ws + upb;
    if (pass == MI3D_PASS_FWD) {  // 7/8 of the stride-1 outputs are thrown away
        int st = sp_conv(u, MI3D_PASS_FWD, a, b, up, rest, ws_bytes - upb, s);
        if (st) return st;
        subsample_kernel<<<blocks_for(g.out_voxels() * (g.Cout / 8)), 256, 0, s>>>(up, (uint16_t*)out, g.N, g.Do, g.Ho, g.Wo, u.Do, u.Ho, u.Wo,
                                                                               g.Cout, g.sD, g.sH, g.sW);
        return check_launch();
    }
    const uint16_t* dy = (const uint16_t*)(pass == MI3D_PASS_DGRAD ? a : b);
    spread_kernel<<<blocks_for(u.out_voxels() * (g.Cout / 8)), 256, 0, s>>>(dy, up, g.N, g.Do, g.Ho, g.Wo, u.Do, u.Ho, u.Wo, g.Cout,
                                                                          g.sD, g.sH, g.sW);
    int st = check_launch();
    if (st) return st;
    if (pass == MI3D_PASS_DGRAD) return sp_conv(u, MI3D_PASS_DGRAD, up, b, out, rest, ws_bytes - upb, s);
    return wgrad_mfma(u, a, up, (float*)out, rest, ws_bytes - upb, s);
}

// ---- 2x2x2 / stride 2 / pad 0 as 3x3x3 / stride 2 / pad 1 --------------------
// input index 2 o + t2 (t2 in {0,1}) == 2 o - 1 + t3 with t3 = t2 + 1: the same layer with its
// weights at taps {1,2}^3 of a 3x3x3 kernel and zeros at the 19 other taps.
namespace {
__global__ void __launch_bounds__(256) k2_to_k3_weights_kernel(const uint16_t* __restrict__ w2, uint16_t* __restrict__ w3, int Cout, int Cin) {
    long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long long)Cout * 27 * Cin) return;
    int ci = (int)(idx % Cin);
    long long r = idx / Cin;
    int t3 = (int)(r % 27);
    int co = (int)(r / 27);
    int kd = t3 / 9, kh = (t3 / 3) % 3, kw = t3 % 3;
    uint16_t v = 0;
    if (kd && kh && kw) v = w2[((long long)co * 8 + ((kd - 1) * 2 + (kh - 1)) * 2 + (kw - 1)) * Cin + ci];
    w3[idx] = v;
}
__global__ void __launch_bounds__(256) k3_to_k2_dw_kernel(const float* __restrict__ dw3, float* __restrict__ dw2, int Cout, int Cin) {
    long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long long)Cout * 8 * Cin) return;
    int ci = (int)(idx % Cin);
    long long r = idx / Cin;
    int t2 = (int)(r % 8);
    int co = (int)(r / 8);
    int t3 = ((t2 >> 2) + 1) * 9 + (((t2 >> 1) & 1) + 1) * 3 + (t2 & 1) + 1;
    dw2[idx] = dw3[((long long)co * 27 + t3) * Cin + ci];
}
Geom k3_geom(const Geom& g) {
    Geom e = g;
    e.kD = e.kH = e.kW = 3;
    e.pD = e.pH = e.pW = 1;
    return e;   // Do = (D + 2 - 3) / 2 + 1 = D / 2 for even D: unchanged
}
}  // namespace

bool embed_k2_supported(const Geom& g, int pass) {
    (void)pass;
    if (g.dtype != MI3D_BF16 || g.kD != 2 || g.kH != 2 || g.kW != 2) return false;
    if (g.sD != 2 || g.sH != 2 || g.sW != 2 || g.pD || g.pH || g.pW) return false;
    if ((g.D | g.H | g.W) & 1) return false;
    return g.Cin % 32 == 0 && g.Cout % 32 == 0;
}

static size_t embed_k2_bytes(const Geom& g, int pass, bool least) {
    if (!embed_k2_supported(g, pass)) return 0;
    Geom e = k3_geom(g);
    size_t first = pass == MI3D_PASS_WGRAD ? align256((size_t)e.w_elems() * 4) : align256((size_t)e.w_elems() * 2);
    return first + (least ? auto_min_workspace_bytes(e, pass) : align256(auto_workspace_bytes(e, pass)));
}
size_t embed_k2_workspace_bytes(const Geom& g, int pass) { return embed_k2_bytes(g, pass, false); }
size_t embed_k2_min_workspace_bytes(const Geom& g, int pass) { return embed_k2_bytes(g, pass, true); }

Geom embed_k2_inner(const Geom& g, int pass, size_t ws_bytes, size_t* rest) {
    const Geom e = k3_geom(g);
    *rest = ws_bytes - align256((size_t)e.w_elems() * (pass == MI3D_PASS_WGRAD ? 4 : 2));
    return e;
}

int embed_k2_conv(const Geom& g, int pass, const void* a, const void* b, void* out, void* ws, size_t ws_bytes, hipStream_t s) {
    if (ws_bytes < embed_k2_min_workspace_bytes(g, pass)) return MI3D_ERR_WORKSPACE;
    Geom e = k3_geom(g);
    int st;
    if (pass == MI3D_PASS_WGRAD) {
        const size_t first = align256((size_t)e.w_elems() * 4);
        float* dw3 = (float*)ws;
        if ((st = auto_conv(e, pass, a, b, dw3, (char*)ws + first, ws_bytes - first, s))) return st;
        k3_to_k2_dw_kernel<<<blocks_for(g.w_elems()), 256, 0, s>>>(dw3, (float*)out, g.Cout, g.Cin);
        return check_launch();
    }
    const size_t first = align256((size_t)e.w_elems() * 2);
    uint16_t* w3 = (uint16_t*)ws;
    k2_to_k3_weights_kernel<<<blocks_for(e.w_elems()), 256, 0, s>>>((const uint16_t*)b, w3, g.Cout, g.Cin);
    if ((st = check_launch())) return st;
    return auto_conv(e, pass, a, w3, out, (char*)ws + first, ws_bytes - first, s);
}

}  // namespace mi3d
