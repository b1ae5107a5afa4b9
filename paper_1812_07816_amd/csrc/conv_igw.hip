// Weight gradient as a matrix product over numbered positions (bf16, and fp32 with its products formed by bf16 matrix
// instructions):
//
//   dw[co, t, ci] = sum over positions o of  dy[o, co] * x[s o - p + t, ci]
//
// Rows are output channels, columns the (tap, channel) pairs in the order of dw, and the contraction runs over the positions
// of all samples in steps of 32, so nothing is lost at the edges of small, odd or narrow volumes, whose planes the
// patch kernels cover with patches of 4 to 16 x 32.  A workgroup (4 waves) owns 128 or 64 rows x 128 columns and a range of
// steps; where tiles leave CUs idle several share a tile, and reduce_partials adds their sums in index order.  A table of the
// next positions' voxels and of the taps that lie inside the volume is kept in LDS.
//
// bf16: rows of positions go to LDS as they are in memory (direct-to-LDS loads, three steps ahead; the range check of the buffer
// supplies the zero padding; 16-byte pieces permuted inside a row so that the four rows of a transposing read fall into
// different banks) and are fetched with ds_read_b64_tr_b16.  v_mfma_f32_32x32x16_bf16, fp32 accumulation.
//
// fp32: each operand is taken apart into three bf16 numbers and six of the nine products are added in fp32 (conv_f32.hip has
// the bound of what is left out).  A thread holds eight positions of two channels, so that the transposition happens in
// its registers: [part][8 positions][channel][8] in LDS, even channels before odd ones.  A value outside the
// range of the split (split_f32.h; infinities and NaN among them) sends its step through v_mfma_f32_32x32x2_f32 on operands read
// straight from memory; where an element of dy is not finite, pair by pair for the columns whose voxel lies inside the volume: it
// meets no zero that is not there.
#include <cstdio>
#include <utility>

#include "ig_common.h"
#include "mi3d_internal.h"
#include "split_f32.h"

namespace mi3d {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((address_space(3))) char* lds_char;

constexpr int BN = 128;                            // columns of a tile
constexpr unsigned OOB = 0xFFFFFFF0u;              // buffer offset of a piece that must read as zero
constexpr long long MAX_BYTES = 0xFFFFFF00ll;      // of a tensor whose pieces are addressed with 32-bit offsets
constexpr int MAX_STEPS = 2048;                    // of an fp32 workgroup: a bit for each that the parts cannot hold
constexpr int STEP = 32;                           // positions of a step

struct IgwParams {
    const void *x, *x_hi;      // two halves along the channels (virtual concatenation), or the tensor and nothing
    const void* dy;
    float* out;                // [split][Cout][T * Cin]
    Div oD, oH, oW;            // extents of the positions of a sample
    Div C;                     // channels per voxel of x (of one half)
    int sD, sH, sW, pD, pH, pW, iD, iH, iW;
    int kH, kW, T, Cout, Cin;
    int NT, MT;                // tiles of columns (of one half), of rows
    long long J, steps;        // positions, steps of them
    int splits, tiles;
    uint32_t x_bytes, dy_bytes;
};

// Voxel of position j at tap 0 in bytes (modulo 2^32), and the taps of each axis that lie inside the volume: kw in bits 0 to 2, kh in 3 to 5, kd in 6 to 8
__device__ __forceinline__ uint2 position(const IgwParams& P, long long j, int esize) {
    if (j >= P.J) return uint2{0, 0};
    const int r = divide((int)j, P.oW), w = ((int)j - r * (int)P.oW.d) * P.sW - P.pW;
    const int r2 = divide(r, P.oH), h = (r - r2 * (int)P.oH.d) * P.sH - P.pH;
    const int n = divide(r2, P.oD), d = (r2 - n * (int)P.oD.d) * P.sD - P.pD;
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        m |= ((unsigned)(w + k) < (unsigned)P.iW ? 1u << k : 0u) | ((unsigned)(h + k) < (unsigned)P.iH ? 8u << k : 0u) | ((unsigned)(d + k) < (unsigned)P.iD ? 64u << k : 0u);
    return uint2{(((uint32_t)(n * P.iD + d) * P.iH + h) * P.iW + w) * P.C.d * esize, m};
}
// A column (of one half): bytes from tap 0 of a position on, the table's bits it needs (one that is never set beyond the last
// column), and its place in a row of dw
struct Column {
    uint32_t off, need;
    int at;
};
__device__ __forceinline__ Column column(const IgwParams& P, int c, bool hi, int esize) {
    const int tap = divide(c, P.C), ci = c - tap * (int)P.C.d;
    const int kw = tap % P.kW, kh = tap / P.kW % P.kH, kd = tap / P.kW / P.kH;
    Column q;
    q.off = (uint32_t)(((kd * P.iH + kh) * P.iW + kw) * (int)P.C.d + ci) * esize;
    q.need = tap < P.T ? 1u << kw | 8u << kh | 64u << kd : 1u << 31;
    q.at = tap * P.Cin + (hi ? (int)P.C.d : 0) + ci;
    return q;
}

// block -> (split, tile of columns, tile of rows); the blocks of an XCD (every eighth) get neighbouring splits of all tiles, which
// read the same positions
struct Work {
    int split, mt, nt;
    bool hi;
    long long s0, s1;
};
__device__ __forceinline__ Work work_of(const IgwParams& P) {
    const int n = P.tiles * P.splits, l = blockIdx.x, x = l & 7, q = l >> 3;
    const int id = x * (n >> 3) + ((n & 7) < x ? (n & 7) : x) + q;
    Work w;
    w.split = id / P.tiles;
    const int tile = id - w.split * P.tiles;
    w.mt = tile % P.MT;
    w.nt = tile / P.MT;
    w.hi = w.nt >= P.NT;
    if (w.hi) w.nt -= P.NT;
    w.s0 = P.steps * w.split / P.splits;
    w.s1 = P.steps * (w.split + 1) / P.splits;
    return w;
}

__device__ __forceinline__ f32x16 mfma16(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x16 mfma2(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// lane (column ln, half): register i of a block is row 8 (i / 4) + 4 half + i % 4 of its 32
template <int AB>
__device__ __forceinline__ void store(const IgwParams& P, const Work& w, const f32x16 (&acc)[AB][2], int m0, int n0, int lane) {
    const int ln = lane & 31, half = lane >> 5, row = P.T * P.Cin;
    float* out = P.out + (long long)w.split * P.Cout * row;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const Column q = column(P, n0 + 32 * b + ln, w.hi, 1);
        if (q.need >> 31) continue;
#pragma unroll
        for (int a = 0; a < AB; ++a)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int co = m0 + 32 * a + 8 * (i >> 2) + 4 * half + (i & 3);
                if (co < P.Cout) out[(long long)co * row + q.at] = acc[a][b][i];
            }
    }
}

// ---- bf16 ----------------------------------------------------------------------------------------------------------------

// BM = rows of a tile: 128 (waves 2 x 2 of 64 x 64) or 64 (2 x 2 of 32 x 64)
template <int BM>
__global__ void __launch_bounds__(256, 2) igw_kernel(const IgwParams P) {
    constexpr int AB = BM / 64, KP = STEP;
    constexpr int RA = BM * 2, RB = BN * 2;                                // bytes of a row of positions
    constexpr int A_BYTES = KP * RA, STAGE = A_BYTES + KP * RB;
    constexpr int LA = 64 / (RA / 16), LB = 64 / (RB / 16);                // rows a wave fetches with one load
    constexpr int NA = KP / (4 * LA), NB = KP / (4 * LB), RING = 4;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    uint2* tab = (uint2*)(lds + RING * STAGE);                             // [2][256]: eight steps' positions
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const Work w = work_of(P);
    const int m0 = w.mt * BM, n0 = w.nt * BN;

    const __amdgpu_buffer_rsrc_t r_x = __builtin_amdgcn_make_buffer_rsrc((void*)(w.hi ? P.x_hi : P.x), 0, (int)P.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t r_dy = __builtin_amdgcn_make_buffer_rsrc((void*)P.dy, 0, (int)P.dy_bytes, 0x00020000);
    // the pieces this lane fetches: place in the row and row, one permutation for all its rows (16 rows apart)
    const int la = lane % (RA / 16), ra = wave * LA + lane / (RA / 16);
    const int lb = lane % (RB / 16), rb = wave * LB + lane / (RB / 16);
    auto swz = [](int row, int row_bytes) { return row_bytes == 256 ? 4 * (row & 3) : 2 * (row & 2); };   // (the same four rows further)
    const int co = m0 + 8 * (la ^ swz(ra, RA));
    const uint32_t offa = co < P.Cout ? (uint32_t)(ra * P.Cout + co) * 2 : OOB;
    const Column col = column(P, n0 + 8 * (lb ^ swz(rb, RB)), w.hi, 2);
    const uint32_t rowa = (uint32_t)P.Cout * 2;

    auto fill = [&](long long s) {   // table of steps s .. s + 7, s - s0 a multiple of 8
        tab[((s - w.s0) & 8 ? 256 : 0) + t] = position(P, s * KP + t, 2);
    };
    const unsigned lds_wave = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_char)lds) + wave * 1024;
    auto fetch = [&](long long s) {
        const unsigned l = lds_wave + (unsigned)((s - w.s0) & (RING - 1)) * STAGE;
        const uint32_t base = (uint32_t)(s * KP) * rowa;
        uint2 v[NB];
        const uint2* q = tab + ((s - w.s0) & 15) * KP + rb;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            v[i] = q[i * 4 * LB];
            asm volatile("" : "+v"(v[i].x), "+v"(v[i].y));   // (read whole, at once)
        }
#pragma unroll
        for (int i = 0; i < NA; ++i)
            load_lds_asm(r_dy, l + i * 4096, offa == OOB ? OOB : offa + base + (uint32_t)(i * 4 * LA) * rowa);   // (behind the last position: the end of dy)
#pragma unroll
        for (int i = 0; i < NB; ++i) load_lds_asm(r_x, l + A_BYTES + i * 4096, (v[i].y & col.need) == col.need ? v[i].x + col.off : OOB);
    };

    f32x16 acc[AB][2];
#pragma unroll
    for (int a = 0; a < AB; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

    // transposing reads: a group of 16 lanes reads four rows of 16 channels; groups 0, 1 rows 0 .. 7 of channels 0 .. 15 and 16 .. 31 of a
    // block, groups 2, 3 rows 8 .. 15
    const int wm = (wave & 1) * (BM / 2), wn = (wave >> 1) * 64;
    const int g = lane >> 4, row = 8 * (g >> 1) + (lane >> 2 & 3), c8 = lane & 3;
    auto place = [&](int ch, int row_bytes) {
        const int piece = (ch + 16 * (g & 1)) / 8 + (c8 >> 1);
        return row * row_bytes + (piece ^ swz(row, row_bytes)) * 16 + (c8 & 1) * 8;
    };
    int fa[AB], fb[2];
#pragma unroll
    for (int a = 0; a < AB; ++a) fa[a] = place(wm + 32 * a, RA);
#pragma unroll
    for (int b = 0; b < 2; ++b) fb[b] = A_BYTES + place(wn + 32 * b, RB);

    if (w.s0 < w.s1) {
        fill(w.s0);
        __syncthreads();
        // three steps under way: a step's loads are waited for with those of the next two still out
#pragma unroll
        for (int i = 0; i < RING - 1; ++i)
            if (w.s0 + i < w.s1) fetch(w.s0 + i);
        for (long long s = w.s0; s < w.s1; ++s) {
            if (s + 2 < w.s1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * (NA + NB)) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (((s - w.s0) & 7) == 0 && s + 8 < w.s1) fill(s + 8);   // (its place was last read for step s - 1)
            if (s + RING - 1 < w.s1) fetch(s + RING - 1);             // (takes the place of step s - 1)
            const char* l = lds + ((s - w.s0) & (RING - 1)) * STAGE;
#pragma unroll
            for (int k = 0; k < KP / 16; ++k) {
                bf16x8 va[AB], vb[2];
#pragma unroll
                for (int a = 0; a < AB; ++a) va[a] = tr_frag(l + fa[a] + k * 16 * RA, RA);
#pragma unroll
                for (int b = 0; b < 2; ++b) vb[b] = tr_frag(l + fb[b] + k * 16 * RB, RB);
#pragma unroll
                for (int a = 0; a < AB; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) acc[a][b] = mfma16(va[a], vb[b], acc[a][b]);
            }
        }
    }
    store<AB>(P, w, acc, m0 + wm, n0 + wn, lane);
}

// ---- fp32 ----------------------------------------------------------------------------------------------------------------

template <int CH> constexpr int K8 = CH * 16 + 128;     // bytes of eight positions of CH channels of a part
template <int CH> __device__ __forceinline__ int slot(int ch) { return (ch >> 1) * 16 + (ch & 1) * (CH * 8 + 128); }

template <int BM>
__global__ void __launch_bounds__(256, 2) igw_f32_kernel(const IgwParams P) {
    constexpr int AB = BM / 64, KP = STEP;
    constexpr int A_PART = 4 * K8<BM>, B_PART = 4 * K8<BN>, A_BYTES = 3 * A_PART, STAGE = A_BYTES + 3 * B_PART;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    uint2* tab = (uint2*)(lds + STAGE);                // [2][128]: four steps' positions
    uint32_t* bad = (uint32_t*)(tab + 256);            // [MAX_STEPS / 32]
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int ln = lane & 31, half = lane >> 5;
    const Work w = work_of(P);
    const int m0 = w.mt * BM, n0 = w.nt * BN;

    const __amdgpu_buffer_rsrc_t r_x = __builtin_amdgcn_make_buffer_rsrc((void*)(w.hi ? P.x_hi : P.x), 0, (int)P.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t r_dy = __builtin_amdgcn_make_buffer_rsrc((void*)P.dy, 0, (int)P.dy_bytes, 0x00020000);
    // this thread's two channels of dy (BM = 64: half of the threads have some) and two columns of x, eight positions of each
    const int ca = 2 * (BM == 128 ? lane : ln), ka = BM == 128 ? wave : 2 * wave + half;
    const bool has_a = ka < 4 && m0 + ca < P.Cout;
    const uint32_t rowa = (uint32_t)P.Cout * 4, offa = (uint32_t)(8 * ka) * rowa + (uint32_t)(m0 + ca) * 4;
    const Column col = column(P, n0 + 2 * lane, w.hi, 4);

    if (t < MAX_STEPS / 32) bad[t] = 0;
    auto set_bad = [&](long long s) { atomicOr(&bad[(s - w.s0) >> 5], 1u << ((s - w.s0) & 31)); };
    auto is_bad = [&](long long s) { return __builtin_amdgcn_readfirstlane(bad[(s - w.s0) >> 5] >> ((s - w.s0) & 31) & 1) != 0; };
    auto fill = [&](long long s) {   // table of steps s .. s + 3, s - s0 a multiple of 4
        if (t < 128) tab[((s - w.s0) & 4 ? 128 : 0) + t] = position(P, s * KP + t, 4);
    };
    float2 pa[8], pb[8];
    auto load8 = [](__amdgpu_buffer_rsrc_t r, uint32_t off) { return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0)); };
    auto request = [&](long long s) {
        const uint32_t base = offa + (uint32_t)(s * KP) * rowa;
        const uint4* q = (const uint4*)(tab + ((s - w.s0) & 7) * KP + 8 * wave);
        uint4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = q[j];
            asm volatile("" : "+v"(v[j].x), "+v"(v[j].y), "+v"(v[j].z), "+v"(v[j].w));   // (read whole, at once)
        }
        // (positions behind the last one lie behind the end of dy)
        if (BM == 128 || wave < 2) {
#pragma unroll
            for (int j = 0; j < 8; ++j) pa[j] = load8(r_dy, has_a ? base + (uint32_t)j * rowa : OOB);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t at = j & 1 ? v[j / 2].z : v[j / 2].x, have = j & 1 ? v[j / 2].w : v[j / 2].y;
            pb[j] = load8(r_x, (have & col.need) == col.need ? at + col.off : OOB);
        }
    };
    auto put = [&](auto& range, const float2 (&v)[8], char* d, int ch, int channels_half, int part) {   // eight positions of channels ch, ch + 1
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            uint32_t o[4][3];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float x = c ? v[2 * j].y : v[2 * j].x, y = c ? v[2 * j + 1].y : v[2 * j + 1].x;
                range.add2(x, y);
                split2(x, y, o[j]);
            }
            char* q = d + (ch >> 1) * 16 + c * channels_half;
#pragma unroll
            for (int p = 0; p < 3; ++p) *(uint4*)(q + p * part) = uint4{o[0][p], o[1][p], o[2][p], o[3][p]};
        }
    };

    f32x16 acc[AB][2];
#pragma unroll
    for (int a = 0; a < AB; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

    const int wm = (wave & 1) * (BM / 2), wn = (wave >> 1) * 64;
    if (w.s0 < w.s1) {
        fill(w.s0);
        __syncthreads();
        request(w.s0);
        for (long long s = w.s0; s < w.s1; ++s) {
            if (((s - w.s0) & 3) == 0 && s + 4 < w.s1) fill(s + 4);   // (its place was last read for step s - 1)
            SplitRange range_a;            // (a NaN of dy must not meet the zeros of voxels outside the volume)
            SplitRangeNumbers range_b;
            if (BM == 128 || wave < 2) put(range_a, pa, lds + ka * K8<BM>, ca, BM * 8 + 128, A_PART);
            put(range_b, pb, lds + A_BYTES + wave * K8<BN>, 2 * lane, BN * 8 + 128, B_PART);
            if (__any(range_a.exceeded() || range_b.exceeded()) && lane == 0) set_bad(s);
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (s + 1 < w.s1) request(s + 1);
            if (!is_bad(s)) {
                // the small products of two blocks at a time apart: an accumulator is rounded three times per 32 positions
                constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
                bf16x8 vb[2][2][3];
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int p = 0; p < 3; ++p) vb[k][b][p] = *(const bf16x8*)(lds + A_BYTES + p * B_PART + (2 * k + half) * K8<BN> + slot<BN>(wn + 32 * b + ln));
#pragma unroll
                for (int a = 0; a < AB; ++a) {
                    f32x16 low[2];
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int i = 0; i < 16; ++i) low[b][i] = 0.f;
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        bf16x8 va[3];
#pragma unroll
                        for (int p = 0; p < 3; ++p) va[p] = *(const bf16x8*)(lds + p * A_PART + (2 * k + half) * K8<BM> + slot<BM>(wm + 32 * a + ln));
#pragma unroll
                        for (int q = 0; q < 5; ++q)
#pragma unroll
                            for (int b = 0; b < 2; ++b) low[b] = mfma16(va[PA[q]], vb[k][b][PB[q]], low[b]);
#pragma unroll
                        for (int b = 0; b < 2; ++b) acc[a][b] = mfma16(va[0], vb[k][b][0], acc[a][b]);
                    }
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[a][b][i] += low[b][i];
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // readers are done (requests stay under way)
        }
    }
    // the steps left out, on the values themselves
    for (long long s = w.s0; s < w.s1; ++s) {
        if (!is_bad(s)) continue;
#pragma unroll 1
        for (int kk = 0; kk < KP; kk += 2) {
            const long long j = s * KP + kk + half;
            const uint2 v = position(P, j, 4);
            float da[AB], xb[2];
            int ok[2];
            bool odd = false;
#pragma unroll
            for (int a = 0; a < AB; ++a) {
                const int co = m0 + wm + 32 * a + ln;
                da[a] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r_dy, (int)(co < P.Cout && j < P.J ? (uint32_t)j * rowa + co * 4 : OOB), 0, 0));
                odd |= !(fabsf(da[a]) < __builtin_inff());
            }
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const Column q = column(P, n0 + wn + 32 * b + ln, w.hi, 4);
                ok[b] = (v.y & q.need) == q.need;
                xb[b] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r_x, (int)(ok[b] ? v.x + q.off : OOB), 0, 0));
            }
            if (!__any(odd)) {
#pragma unroll
                for (int a = 0; a < AB; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) acc[a][b] = mfma2(da[a], xb[b], acc[a][b]);
                continue;
            }
#pragma unroll 1
            for (int h = 0; h < 2; ++h)   // the two positions of this instruction, one after the other
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const float x1 = __shfl(xb[b], ln + 32 * h);
                    const int ok1 = __shfl(ok[b], ln + 32 * h);
#pragma unroll
                    for (int a = 0; a < AB; ++a)
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const float d1 = __shfl(da[a], 8 * (i >> 2) + 4 * half + (i & 3) + 32 * h);
                            if (ok1) acc[a][b][i] += d1 * x1;
                        }
                }
        }
    }
    store<AB>(P, w, acc, m0 + wm, n0 + wn, lane);
}

// Tile shape and splits of the positions, by a model of the time (see plan_us)
struct IgwPlan {
    int bm, splits, MT, NT, halves;
    long long steps;
    double us;
};
// What a step takes with one, two, three workgroups on a CU, [fp32][BM = 64] (320->320 at 12^3 and 128->256, stride 2 at 48^3, N = 2;
// fp32 64->128, 2x2x2 at 64^3, N = 2, with 64 to 512 workgroups)
constexpr int RES[2] = {2, 3};
constexpr double STEP_US[2][2][3] = {{{0.38, 0.52, 0.52}, {0.30, 0.38, 0.49}}, {{2.45, 3.6, 3.6}, {2.05, 2.9, 3.9}}};
constexpr double START_US = 4.0, LAUNCH_US = 4.0, PART_BYTES_PER_US = 3.5e6, READ_BYTES_PER_US = 13e6;   // (what all CUs read from the L2s)

IgwPlan plan_for(const Geom& g, size_t ws_bytes) {
    const bool f32 = g.dtype == MI3D_F32;
    const int cus = cu_count(), C = g.hi ? g.Cin / 2 : g.Cin;
    IgwPlan best{0, 1, 0, 0, g.hi ? 2 : 1, 0, 1e30};
    const long long J = g.out_voxels();
    best.steps = (J + STEP - 1) / STEP;
    best.NT = (int)((g.taps() * C + BN - 1) / BN);
    for (int bm = 128; bm >= 64; bm -= 64) {
        const long long MT = (g.Cout + bm - 1) / bm, tiles = MT * best.NT * best.halves;
        for (long long S = 1; S <= best.steps; S = S < 16 ? S + 1 : S + S / 8) {
            if (f32 && best.steps > S * MAX_STEPS) continue;
            if (S > 1 && S * (size_t)g.w_elems() * 4 > ws_bytes) break;
            if (S > 1 && (S * (size_t)g.w_elems() * 4 > ((size_t)48 << 20) || tiles * S > 6ll * cus)) break;
            if (tiles * S > (1ll << 30)) break;
            const double each = (double)((best.steps + S - 1) / S);
            const int res = RES[bm == 64];
            const long long full = tiles * S / ((long long)res * cus), rest = tiles * S - full * res * cus;
            const int k = (int)((rest + cus - 1) / cus);
            auto round = [&](int n) { return each * STEP_US[f32][bm == 64][n - 1] + START_US * n; };
            double us = full * round(res) + (k ? round(k) : 0.0);
            const double read = START_US + (double)tiles * g.out_voxels() * (bm + BN) * (double)g.esize() / READ_BYTES_PER_US;
            if (us < read) us = read;
            us += (S > 1 ? LAUNCH_US + (double)S * g.w_elems() * 8 / PART_BYTES_PER_US : 0.0);
            if (us < best.us) { best.us = us; best.bm = bm; best.splits = (int)S; best.MT = (int)MT; }
        }
    }
    return best;
}
IgwPlan make_plan(const Geom& g, size_t ws_bytes) { return kept_plan<IgwPlan>(g, MI3D_PASS_WGRAD, ws_bytes, [&] { return plan_for(g, ws_bytes); }); }

}  // namespace

bool igw_supported(const Geom& g) {
    if (g.kD > 3 || g.kH > 3 || g.kW > 3) return false;
    const int unit = g.dtype == MI3D_F32 ? 2 : 8;
    if (g.Cin % unit || g.Cout % unit) return false;
    const long long e = (long long)g.esize(), J = g.out_voxels();
    if (g.in_voxels() * g.Cin * e > MAX_BYTES || (J + STEP) * g.Cout * e > MAX_BYTES || J >= (1ll << 31) - 4096 || g.in_voxels() >= (1ll << 31)) return false;
    if (g.taps() * g.Cin >= (1ll << 30)) return false;
    return true;
}
double igw_us(const Geom& g, size_t ws_bytes) { return LAUNCH_US + make_plan(g, ws_bytes).us; }
size_t igw_workspace_bytes(const Geom& g) {
    const IgwPlan p = make_plan(g, ~(size_t)0);
    return p.splits > 1 ? (size_t)p.splits * g.w_elems() * sizeof(float) : 0;
}
void igw_describe(const Geom& g, size_t ws_bytes, char* buf, size_t len) {
    const IgwPlan p = make_plan(g, ws_bytes);
    snprintf(buf, len, "%swgrad_implicit_gemm_%dx%d parts %d", g.dtype == MI3D_F32 ? "f32_" : "", p.bm, BN, p.splits);
}

int igw_run(const Geom& g, const void* x, const void* dy, float* dw, void* ws, size_t ws_bytes, hipStream_t s) {
    const IgwPlan p = make_plan(g, ws_bytes);
    const bool f32 = g.dtype == MI3D_F32;
    if (!p.bm) return MI3D_ERR_WORKSPACE;
    if (g.hi && g.Cin % 64) return MI3D_ERR_UNSUPPORTED;
    IgwParams P{};
    P.x = x; P.x_hi = g.hi; P.dy = dy;
    P.out = p.splits > 1 ? (float*)ws : dw;
    P.oD = make_div(g.Do); P.oH = make_div(g.Ho); P.oW = make_div(g.Wo);
    P.C = make_div(g.Cin / p.halves);
    P.sD = g.sD; P.sH = g.sH; P.sW = g.sW; P.pD = g.pD; P.pH = g.pH; P.pW = g.pW;
    P.iD = g.D; P.iH = g.H; P.iW = g.W;
    P.kH = g.kH; P.kW = g.kW; P.T = (int)g.taps(); P.Cout = g.Cout; P.Cin = g.Cin;
    P.NT = p.NT; P.MT = p.MT;
    P.J = g.out_voxels(); P.steps = p.steps;
    P.splits = p.splits; P.tiles = p.MT * p.NT * p.halves;
    P.x_bytes = (uint32_t)(g.in_voxels() * (g.Cin / p.halves) * (long long)g.esize());
    P.dy_bytes = (uint32_t)(P.J * g.Cout * (long long)g.esize());
    const auto lds_bf16 = [](int bm) { return 4 * STEP * (bm + BN) * 2 + 512 * 8; };
    const auto lds_f32 = [](int bm) { return 3 * 4 * (bm * 16 + 128 + BN * 16 + 128) + 256 * 8 + MAX_STEPS / 8; };
    static std::atomic<bool> attr_set{false};   // set once per process; a second thread racing here repeats an idempotent call
    if (!attr_set) {
        const std::pair<const void*, int> fns[4] = {{(const void*)igw_kernel<128>, lds_bf16(128)}, {(const void*)igw_kernel<64>, lds_bf16(64)},
                                                    {(const void*)igw_f32_kernel<128>, lds_f32(128)}, {(const void*)igw_f32_kernel<64>, lds_f32(64)}};
        for (const auto& f : fns) {
            hipError_t e = hipFuncSetAttribute(f.first, hipFuncAttributeMaxDynamicSharedMemorySize, f.second);
            if (e != hipSuccess) { note_hip_error(e); return MI3D_ERR_HIP; }
        }
        attr_set = true;
    }
    const unsigned grid = (unsigned)(P.tiles * P.splits);
    if (f32 && p.bm == 128) igw_f32_kernel<128><<<grid, 256, lds_f32(128), s>>>(P);
    else if (f32) igw_f32_kernel<64><<<grid, 256, lds_f32(64), s>>>(P);
    else if (p.bm == 128) igw_kernel<128><<<grid, 256, lds_bf16(128), s>>>(P);
    else igw_kernel<64><<<grid, 256, lds_bf16(64), s>>>(P);
    const int st = check_launch();
    return st || p.splits == 1 ? st : reduce_partials((const float*)ws, dw, g.w_elems(), p.splits, s);
}

}  // namespace mi3d
