// gfx950 kernels of the learned surrogate: a residual network of 3x3
// convolutions over (phi, u_x, u_y, T) frames that advances the lattice state
// by a fixed number of time steps.  Activations and weights are BF16, all
// products accumulate in FP32 on the matrix cores (v_mfma_f32_32x32x16_bf16).
//
// Layouts: activations NHWC with C = 32 channels (the 4-channel network input
// is padded to C = 8), weights [co = 32][tap = 9][ci] (rows beyond the layer's
// real output channels are zero), taps ordered (dy, dx) = (-1..1, -1..1) with
// tap = 3 (dy + 1) + (dx + 1).  Frames are periodic in x and zero-padded in y
// (x is the periodic direction of the lattices the surrogate stands in for).
//
// Convolution as an implicit GEMM: one wave computes a 32-pixel x 32-channel
// output block; the reduction runs over K = 9 Cin in blocks of 16, where each
// lane's 8 consecutive K entries are 8 consecutive channels of one tap, i.e.
// one 16-byte load from NHWC memory and one from the weights.
// MFMA 32x32x16 operand layout (checked on the device): lane l holds
// A[l % 32][8 (l / 32) + j] and B[8 (l / 32) + j][l % 32], j = 0..7; the
// accumulator element i of lane l is C[8 (i / 4) + 4 (l / 32) + i % 4][l % 32].
#include "sur_internal.hpp"
#include <mutex>
#include <type_traits>

namespace sur {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ inline bf16x8 load8(const bf16* p)
{
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}

typedef __bf16 bf16x8_u __attribute__((ext_vector_type(8), aligned(2)));

// Eight BF16 values at any alignment a BF16 array may have.
__device__ inline bf16x8 load8u(const bf16* p) { return *reinterpret_cast<const bf16x8_u*>(p); }

typedef short s16x8 __attribute__((ext_vector_type(8)));

// max(v, 0) of 8 BF16 values as packed 16-bit integer maxima: a BF16 value
// with its sign bit set is a negative 16-bit integer and a positive one a
// positive integer, so the integer maximum with 0 is the ReLU (-0 becomes +0)
// at four packed instructions instead of eight conversions and selects.
__device__ inline bf16x8 relu8(bf16x8 v)
{
    const s16x8 s = __builtin_bit_cast(s16x8, v);
    return __builtin_bit_cast(bf16x8, __builtin_elementwise_max(s, (s16x8)(short)0));
}

__device__ inline float to_f(bf16 v) { return (float)v; }

// Workgroups are dealt round-robin to the 8 XCDs: renumbers them so that each
// XCD gets a contiguous run of numbers.
__device__ inline int xcd_contiguous(int b, int n)
{
    const int x = b % 8, per = n / 8, rem = n % 8;
    return x * per + (x < rem ? x : rem) + b / 8;
}

// Run b of n that share nitems in order (n at most 2^15).  The longer runs are
// spread evenly: at the front of the order they would all lie on the first XCDs
// (580 items on 512 workgroups, 2 x 456 x 160: 10.5 us a layer, 9.6 spread).
struct Run {
    int first, n;
};
__device__ inline Run run_of(unsigned b, unsigned n, unsigned nitems)
{
    const unsigned per = nitems / n, rem = nitems - per * n;
    if (!rem) return {(int)__builtin_amdgcn_readfirstlane(b * per), (int)__builtin_amdgcn_readfirstlane(per)};
    const unsigned lo = b * rem / n, more = b * rem - lo * n + rem >= n;
    return {(int)__builtin_amdgcn_readfirstlane(b * per + lo), (int)__builtin_amdgcn_readfirstlane(per + more)};
}

// Most products take the weights as the first operand and the pixels as the
// second: lane l of the accumulator then holds 16 channels of one pixel (pixel
// l % 32 of the segment).  The rows of the weight operand are permuted so that
// these are the consecutive channels 16 (l / 32) ... + 15, and an epilogue
// loads and stores 16 bytes at a time: 2 instead of 16 memory instructions per
// BF16 tensor and segment.  Row m of the weight operand holds channel
// weight_row(m).
__device__ constexpr int weight_row(int m) { return 16 * ((m / 4) % 2) + 4 * (m / 8) + m % 4; }

// Rows of 64-byte pixels in LDS, unpadded: the four 16-byte chunks of a pixel
// are rotated by its number, so that lanes reading one chunk of consecutive
// pixels meet distinct banks.  Element offset of chunk c of pixel p.
__device__ inline int swz(int p, int c) { return p * 32 + 8 * (c ^ ((p >> 2) & 3)); }

// Orders a wave's LDS writes before its lanes read what other lanes wrote.
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Epilogue inputs of one pixel: mask and residual of the lane's 16 channels.
struct Extra {
    bf16x8 mask[2], res[2];
};

// Loads them (element offset `o` of the lane's first channel).
template <bool OUTF32, bool RES, bool MASK>
__device__ inline void load_extra(Extra& e, const void* __restrict__ res, const bf16* __restrict__ mask, long long o)
{
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (MASK) e.mask[j] = load8u(mask + o + 8 * j);
        if (RES && !OUTF32) e.res[j] = load8(static_cast<const bf16*>(res) + o + 8 * j);
    }
}

// acc + bias, zero where mask <= 0, + residual, stored as FP32 or BF16 through
// the wave's tile of 32 pixels (2 KB), from which 4 (FP32: 8) lanes store a
// whole pixel: with 16 bytes per lane at a 64-byte stride straight from the
// accumulator a hidden layer took 0.7 us more and an FP32 layer 4 us more
// (256 x 1024).  `o` is the element offset of the segment's first pixel, npx its
// pixels inside the row.
template <bool OUTF32, bool RES, bool MASK>
__device__ inline void conv_store(const f32x16& acc, const float* __restrict__ bias, const Extra& e,
                                  const void* __restrict__ res, bf16* tile, void* __restrict__ out, long long o, int npx,
                                  int lane)
{
    const int m = lane % 32, kh = lane / 32;
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        v[i] = acc[i] + bias[16 * kh + i];
        if (MASK) v[i] = to_f(e.mask[i / 8][i % 8]) > 0.f ? v[i] : 0.f;
    }
    if constexpr (OUTF32) {
        float* ft = reinterpret_cast<float*>(tile);  // half a segment: 16 pixels x 32 channels
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (m / 16 == h) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    *reinterpret_cast<float4*>(ft + (m % 16) * 32 + 4 * ((4 * kh + j) ^ (m % 8))) =
                        make_float4(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]);
            }
            wave_sync();
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int p = 8 * j + lane / 8, c = lane % 8;
                float4 q = *reinterpret_cast<const float4*>(ft + p * 32 + 4 * (c ^ (p % 8)));
                if (16 * h + p < npx) {
                    const long long at = o + (16 * h + p) * 32 + 4 * c;
                    if (RES) {
                        const float4 r = *reinterpret_cast<const float4*>(static_cast<const float*>(res) + at);
                        q = make_float4(q.x + r.x, q.y + r.y, q.z + r.z, q.w + r.w);
                    }
                    *reinterpret_cast<float4*>(static_cast<float*>(out) + at) = q;
                }
            }
            wave_sync();
        }
    } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            bf16x8 q;
#pragma unroll
            for (int i = 0; i < 8; ++i) q[i] = (bf16)(RES ? v[8 * j + i] + to_f(e.res[j][i]) : v[8 * j + i]);
            *reinterpret_cast<bf16x8*>(tile + swz(m, 2 * kh + j)) = q;
        }
        wave_sync();
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int p = 16 * j + lane / 4, c = lane % 4;
            if (p < npx)
                *reinterpret_cast<bf16x8*>(static_cast<bf16*>(out) + o + p * 32 + 8 * c) =
                    *reinterpret_cast<const bf16x8*>(tile + swz(p, c));
        }
        wave_sync();
    }
}

// Layers without residual or mask that store FP32 or have 8 input channels take
// the pixels as the first operand and the weights, not permuted, as the second:
// element i of the accumulator is pixel 8 (i / 4) + 4 (l / 32) + i % 4 of the
// segment, channel l % 32, and half a wave stores the 32 channels of a pixel,
// whole lines in FP32, without the pass through LDS.  FP32 layer of 256 x 1024
// 13.4 -> 12.4 us, of 64 x 64 5.3 -> 4.9.
template <int CIN, bool OUTF32, bool RES, bool MASK>
constexpr bool pixels_first() { return (OUTF32 || CIN == 8) && !RES && !MASK; }

// acc + the product of a block of weights and a block of pixels, in either order.
template <bool PF>
__device__ inline f32x16 product(bf16x8 w, bf16x8 a, const f32x16& acc)
{
    return PF ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, w, acc, 0, 0, 0)
              : __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, a, acc, 0, 0, 0);
}

// Their epilogue: acc + the channel's bias bv.
template <bool OUTF32>
__device__ inline void store_channels(const f32x16& acc, float bv, void* __restrict__ out, long long o, int npx, int lane)
{
    const int p0 = 4 * (lane / 32);
    const long long o0 = o + p0 * 32 + lane % 32;
    auto one = [&](int i) {
        const long long at = o0 + (8 * (i / 4) + i % 4) * 32;
        if (OUTF32) static_cast<float*>(out)[at] = acc[i] + bv;
        else static_cast<bf16*>(out)[at] = (bf16)(acc[i] + bv);
    };
    if (npx >= 32) {
#pragma unroll
        for (int i = 0; i < 16; ++i) one(i);
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (p0 + 8 * (i / 4) + i % 4 < npx) one(i);
    }
}

// One 32-pixel segment of a 32-channel layer (row y of frame n, pixels x0 ..
// x0 + 31).  K block q is tap q / 2, channels 16 (q % 2) + 8 kh ... + 7: the
// three tap rows (clamped to the frame) and the three tap columns (periodic)
// are computed once per segment, and all 18 operands are loaded before the
// first matrix-core op.  A tap row outside the frame contributes nothing: its
// K blocks take their weight operands from the all-zero block sB[18] (a
// scalar choice of LDS address per block; the clamped row's activations are
// finite, so the products are exact zeros, as if the inputs were zeroed by a
// select per operand register).
template <bool RELU, bool PF = false>
__device__ __forceinline__ f32x16 conv_seg32(const bf16* __restrict__ in, const bf16x8 (*__restrict__ sB)[64], int lz,
                                             int dil, int H, int W, int n, int y, int x0, int m, int kh)
{
    constexpr int CIN = 32, NKB = 18;
    const int xm = x0 + m < W ? x0 + m : W - 1;
    const bf16* rowp[3];
    bool rok[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int yy = y + (r - 1) * dil;
        rok[r] = yy >= 0 && yy < H;
        rowp[r] = in + ((long long)n * H + (rok[r] ? yy : y)) * W * CIN + 8 * kh;
    }
    long long xc[3];  // a row may hold 2^31 elements and more
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int xx = xm + (c - 1) * dil;  // |offset| <= W, so one wrap suffices
        xc[c] = (long long)(xx < 0 ? xx + W : (xx >= W ? xx - W : xx)) * CIN;
    }
    bf16x8 a[NKB];
#pragma unroll
    for (int q = 0; q < NKB; ++q) {
        const int tap = q >> 1;
        a[q] = load8(rowp[tap / 3] + xc[tap % 3] + 16 * (q & 1));
    }
    f32x16 acc = {};
#pragma unroll
    for (int q = 0; q < NKB; ++q)
        acc = product<PF>(sB[rok[(q >> 1) / 3] ? q : NKB][lz], RELU ? relu8(a[q]) : a[q], acc);
    return acc;
}

// Stages the weight operands of a 32-channel layer in LDS, in the order the
// lanes read them, followed by an all-zero block (every work-item calls it).
template <int CIN, bool PF = false>
__device__ inline void stage_weights(const bf16* __restrict__ w, bf16x8 (*sB)[64])
{
    constexpr int K = 9 * CIN, NKB = (K + 15) / 16;
    for (int e = threadIdx.x; e < (NKB + 1) * 64; e += blockDim.x) {
        const int q = e / 64, l = e % 64;
        const int kk = q * 16 + 8 * (l / 32);
        bf16x8 v = bf16x8{};
        if (kk < K) v = load8(w + ((long long)(PF ? l % 32 : weight_row(l % 32)) * 9 + kk / CIN) * CIN + kk % CIN);
        sB[q][l] = v;
    }
    __syncthreads();
}

// out[n][y][x][co] = epilogue( sum_{tap, ci} A(n, y + d dy, x + d dx, ci) W[co][tap][ci] )
// with dilation d; A = relu(in) if RELU.  Epilogue: + bias[co] (if bias);
// then, if MASK, zero where mask <= 0; then, if RES, + res.  The output is
// FP32 if OUTF32, else BF16.  Per 32-pixel segment all K / 16 input operands
// are loaded before the first matrix-core op (rows outside the frame load a
// clamped row and are zeroed), so the loads of a wave are in flight together.
// A row of W pixels takes ceil(W / 32) segments; in the last one the pixels
// beyond the row repeat its last pixel and are not stored.  Segment indices
// are 32-bit (the host keeps N H ceil(W / 32) below 2^31): 64-bit divisions
// took ~250 scalar instructions per segment.
// The plain first layer always runs here, its waves taking every segment in
// turn: with five products per segment it spends more on staging its rows, or
// on runs of segments per XCD and stores through LDS, than it saves (256 x 1024
// 7.0 us, by columns 8.0; 2 x 456 x 160 5.4 and 6.9; 64 x 64 3.0 and 3.65).
template <int CIN, bool RELU, bool OUTF32, bool RES, bool MASK>
__global__ __launch_bounds__(256) void k_conv(const bf16* __restrict__ in, const bf16* __restrict__ w,
                                              const float* __restrict__ bias, const void* __restrict__ res,
                                              const bf16* __restrict__ mask, void* __restrict__ out, int dil, int N,
                                              int H, int W)
{
    constexpr int K = 9 * CIN, NKB = (K + 15) / 16;
    const int lane = threadIdx.x % 64;
    const int segs_per_row = (W + 31) / 32;
    const int nseg = N * H * segs_per_row;
    // the segment index is the same for every lane of a wave: kept scalar, so
    // that everything derived from it (row, frame, validity of tap rows) is
    // scalar too
    constexpr bool PF = pixels_first<CIN, OUTF32, RES, MASK>(), TURNS = CIN == 8 && PF;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
    int seg0 = (int)blockIdx.x * 4, seg1 = nseg;
    if constexpr (!TURNS) {
        // a contiguous run of segments per workgroup, runs in XCD order (bands of
        // rows, as in the column kernel)
        const int b = xcd_contiguous(blockIdx.x, gridDim.x);
        const int per = (unsigned)nseg / gridDim.x, rem = nseg - per * gridDim.x;
        seg0 = b * per + (b < rem ? b : rem);
        seg1 = seg0 + per + (b < rem ? 1 : 0);
    }
    const int m = lane % 32, kh = lane / 32;
    // the weight operands of the whole K loop are staged once per workgroup
    __shared__ bf16x8 sB[NKB + 1][64];
    __shared__ __attribute__((aligned(16))) float sBias[32];
    __shared__ __attribute__((aligned(16))) bf16 sO[PF ? 1 : 4][32 * 32];
    if (!PF && threadIdx.x < 32) sBias[threadIdx.x] = bias ? bias[threadIdx.x] : 0.f;
    stage_weights<CIN, PF>(w, sB);
    const float bv = PF && bias ? bias[m] : 0.f;
    for (int seg = seg0 + wave; seg < seg1; seg += TURNS ? 4 * (int)gridDim.x : 4) {
        // an index the compiler cannot hoist: the weight operands are read from
        // LDS per segment instead of being held in 72 registers
        const int lz = lane + 64 * __builtin_amdgcn_readfirstlane((int)((unsigned)seg >> 31));
        const int x0 = (seg % segs_per_row) * 32;
        const int ny = seg / segs_per_row;
        const int y = ny % H, n = ny / H;
        f32x16 acc = {};
        if constexpr (CIN == 32) {
            acc = conv_seg32<RELU, PF>(in, sB, lz, dil, H, W, n, y, x0, m, kh);
        } else {
            const int xm = x0 + m < W ? x0 + m : W - 1;
            bf16x8 a[NKB];
#pragma unroll
            for (int q = 0; q < NKB; ++q) {
                const int kk = q * 16 + 8 * kh;
                const bool kv = kk < K;
                const int kc = kv ? kk : 0;
                const int tap = kc / CIN, ci = kc % CIN;
                const int yy = y + (tap / 3 - 1) * dil;
                int xx = xm + (tap % 3 - 1) * dil;  // |offset| <= W, so one wrap suffices
                xx = xx < 0 ? xx + W : (xx >= W ? xx - W : xx);
                const bool ok = kv && yy >= 0 && yy < H;
                const int yc = ok ? yy : y;
                a[q] = load8(in + (((long long)n * H + yc) * W + xx) * CIN + ci);
                if (!ok) a[q] = bf16x8{};
            }
#pragma unroll
            for (int q = 0; q < NKB; ++q)
                acc = product<PF>(sB[q][lz], RELU ? relu8(a[q]) : a[q], acc);
        }
        const long long o = (((long long)n * H + y) * W + x0) * 32;
        if constexpr (PF) {
            store_channels<OUTF32>(acc, bv, out, o, W - x0, lane);
        } else {
            Extra e = {};
            if (x0 + m < W) load_extra<OUTF32, RES, MASK>(e, res, mask, o + 32 * m + 16 * kh);
            conv_store<OUTF32, RES, MASK>(acc, sBias, e, res, sO[threadIdx.x / 64], out, o, W - x0, lane);
        }
    }
}

// Work item of a column kernel: frame n, group g of kColRW rows of a residue
// class of the rows mod the dilation, that class r, column sx, in this order of
// significance: any run of items then lies in a band of rows, so an XCD's part
// of the items is a band, the same one in every layer, and a layer finds in
// the XCD's L2 what the layer before left there (with the residue class
// outermost the layers with dilation 8 and 16 took 15.6 us of a network block
// instead of 12.3).  A workgroup takes a contiguous run of items, located once
// (integer divisions cost ~20 vector instructions each) and stepped by counting.
struct Item {
    int n, r, g, sx;
    // R = min(dilation, H) residue classes
    __device__ void locate(unsigned t, unsigned R, unsigned G, unsigned SC)
    {
        const unsigned u = t / SC, v = u / R;
        sx = (int)__builtin_amdgcn_readfirstlane(t - u * SC);
        r = (int)__builtin_amdgcn_readfirstlane(u - v * R);
        n = (int)__builtin_amdgcn_readfirstlane(v / G);
        g = (int)__builtin_amdgcn_readfirstlane(v % G);
    }
    __device__ void next(int R, int G, int SC)
    {
        if (++sx < SC) return;
        sx = 0;
        if (++r < R) return;
        r = 0;
        if (++g < G) return;
        g = 0;
        ++n;
    }
};

// A uniform row base plus a 32-bit byte offset per lane, as one address.
template <typename T>
using gptr = __attribute__((address_space(1))) T*;
template <typename T>
__device__ inline gptr<T> at(T* base, unsigned bytes)
{
    typedef typename std::conditional<std::is_const<T>::value, const char, char>::type byte;
    return (gptr<T>)((gptr<byte>)base + bytes);
}

// Network input of one pixel of row y: 8 BF16 channels (see k_pack).
__device__ inline bf16x8 pack_pixel(float phi, float ux, float uy, float T, float p, float y, const Scales& sc)
{
    bf16x8 o;
    o[0] = (bf16)phi;
    o[1] = (bf16)(ux / sc.u);
    o[2] = (bf16)(uy / sc.u);
    o[3] = (bf16)((T - (sc.t_a + sc.t_b * y)) / sc.dT);
    o[4] = (bf16)sc.c4;
    o[5] = (bf16)sc.c5;
    o[6] = (bf16)((p - sc.P * 0.5f * (1.f - phi)) / sc.P);
    o[7] = (bf16)0.f;
    return o;
}

// Five fields of the state advanced by the increments of one pixel (channels
// 0 .. 4, the first of lane half 0).
__device__ inline void advance_pixel(const f32x16& acc, const float* __restrict__ bv, const float (&old)[5], const State5& f,
                                     const Scales& sc, long long p, float& phi)
{
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        const float nv = old[c] + (acc[c] + bv[c]) * sc.inc[c];
        const_cast<float*>(f.v[c])[p] = nv;
        if (c == 0) phi = nv;
    }
}

// A 32-channel layer with dilation d <= 16 by columns: a workgroup of kColRW / SEG
// waves computes the output rows y0, y0 + d, ..., y0 + (kColRW - 1) d of one
// 32-pixel column (wave k: SEG rows from y0 + SEG k d).  The kColRW + 2 input rows they read
// (y0 - d ... y0 + kColRW d; rows outside the frame as zeros) are staged once
// in LDS over the column's window of 32 + 2d pixels (periodic in x), with the
// ReLU applied as they are staged, and the 18 operands of each segment are read
// from there: each input pixel is loaded ~1.25 times per segment instead of 9.
// The next item's rows are loaded into registers while the current one is
// multiplied; the residual and mask are loaded before them, so that the
// epilogue waits for neither.  The products and their order are those of k_conv.
// The staged window holds up to kColPix pixels (dilation <= 16), or
// kColPixNarrow for dilation <= 4 (fewer idle lanes as it is staged).
// Bound by latency and by its phases: two workgroups per CU load, multiply and
// store nearly in step.  Without the stores a hidden layer took 3 us less,
// without the products 2 (256 x 1024, timing only).  The weight operands in
// registers spill at 4 waves per SIMD.  Residuals taken from the staged rows
// instead of memory: no gain, and 5% slower at 8 x 256 x 192.  Hidden layer in
// a network block at 256 x 1024 13.2 -> 12.3 us, with mask and residual at
// 8 x 256 x 192 24 -> 16 us.
constexpr int kColPix = 64, kColPixNarrow = 40;
// Output rows per workgroup.
constexpr int kColRW = 8;
constexpr int kColRows = kColRW + 2;

// ADV: the output layer of inference, whose epilogue adds the increment to the
// five state fields f (as k_conv_advance; N = 1).  VOL (with ADV): the
// epilogue also sums the light-phase volume (1 - phi) / 2 of the updated phi
// in FP64, per workgroup in a fixed order, into vpart[8 blockIdx.x] (the
// partials layout of k_frame_sums, which k_frame_final sums).  A last
// workgroup that sums the partials after an atomic ticket needs agent-scope
// fences (an L2 write-back per workgroup): measured slower than the separate
// final kernel.
constexpr int kVolParts = kVolPartsApi;  // at least the column kernel's grid (<= 256 * 2)
// MSE: the output layer of training, whose epilogue compares the increment's
// five channels with the target (5 FP32 channels per pixel) and stores only the
// gradient 2 (delta - target) mse_scale as BF16 (zero beyond channel 5) and the
// workgroup's sum of squares into lpart[blockIdx.x]; at 8 x 256 x 192 the 50 MB
// of FP32 increments took 18 us to write and, with a kernel of its own, 89 us
// to compare.
// CIN = 8 (the network's first layer): a lane half's 8 K entries are the 8
// channels of one tap.  PACK: the input is packed from the five state fields f
// as it is staged (N = 1), without a pass over the frame of its own.
// SEG: output rows per wave.  With two, a wave holds the weight operands of a
// tap row for the second row and reads 42 operands from LDS instead of 72, and
// three workgroups of half the waves fit into a CU (narrow windows), but fewer
// waves hide each other's phases: for item counts that three per CU serve in
// fewer rounds than two.
template <int CIN, bool RELU, bool OUTF32, bool RES, bool MASK, bool ADV = false, int PIX = kColPix, bool VOL = false,
          bool PACK = false, bool MSE = false, int SEG = 1>
__global__ __launch_bounds__(64 * kColRW / SEG, SEG == 1 ? 4 : 3) void k_conv_col(const bf16* __restrict__ in, const bf16* __restrict__ w,
                                                          const float* __restrict__ bias, const void* __restrict__ res,
                                                          const bf16* __restrict__ mask, void* __restrict__ out,
                                                          int dil, int N, int H, int W, State5 f, Scales sc,
                                                          double* __restrict__ vpart = nullptr,
                                                          const float* __restrict__ target = nullptr,
                                                          float mse_scale = 0.f, float* __restrict__ lpart = nullptr)
{
    static_assert(!MSE || (CIN == 32 && !OUTF32 && !RES && !MASK && !ADV), "the output layer of training");
    static_assert(!VOL || ADV, "the volume is summed in the state update's epilogue");
    static_assert(!PACK || (CIN == 8 && !ADV), "only the network's input is packed");
    static_assert(SEG == 1 || CIN == 32, "the first layers have one row per wave");
    constexpr int RW = kColRW, WV = kColRW / SEG, S = SEG, K = 9 * CIN, NKB = (K + 15) / 16;
    constexpr bool PF = OUTF32 && !ADV && pixels_first<CIN, OUTF32, RES, MASK>();
    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
    const int m = lane % 32, kh = lane / 32;
    __shared__ bf16x8 sB[NKB][64];
    __shared__ __attribute__((aligned(16))) float sBias[32];
    __shared__ __attribute__((aligned(16))) bf16 sX[kColRows][PIX * CIN];
    // each wave's output segment on its way to memory
    __shared__ __attribute__((aligned(16))) bf16 sO[ADV || MSE || PF ? 1 : WV][32 * 32];
    const int SC = (W + 31) / 32;
    const int G = ((H + dil - 1) / dil + RW - 1) / RW;  // groups of RW rows per residue class of y mod d
    const int R = dil < H ? dil : H;
    const int nitems = N * R * G * SC;
    const int win = 32 + 2 * dil;
    // 64 pixels of CIN / 8 chunks of 8 channels, RP rows per pass: work-item t
    // takes chunk c of window pixel i of row jr of the pass (win <= PIX <= 64)
    constexpr int CH = CIN / 8, RP = WV / CH, NPASS = (kColRows + RP - 1) / RP;
    const int c = threadIdx.x % CH, i = (threadIdx.x % (64 * CH)) / CH;
    const int jr = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / (64 * CH)));
    bf16x8 v[NPASS];
    float raw[PACK ? NPASS : 1][5], rawy[PACK ? NPASS : 1];
    unsigned inframe = 0;  // bit k: the row of pass k lies in the frame
    // runs of items numbered so that each XCD has a contiguous part of them:
    // what neighbouring items share of the window is fetched into one L2
    const int b = xcd_contiguous(blockIdx.x, gridDim.x);
    const Run run = run_of(b, gridDim.x, nitems);
    int left = run.n;
    Item it;
    it.locate(run.first, R, G, SC);
    int y0 = it.r + RW * it.g * dil;
    // passes over items whose rows lie beyond the frame (a residue class with fewer rows)
    auto settle = [&]() {
        while (left > 0 && (y0 = it.r + RW * it.g * dil) >= H) {
            it.next(R, G, SC);
            --left;
        }
    };
    auto fetch = [&]() {
        inframe = 0;
        if (i < win) {
            int xx = it.sx * 32 - dil + i;
            while (xx < 0) xx += W;
            while (xx >= W) xx -= W;
#pragma unroll
            for (int k = 0; k < NPASS; ++k) {
                const int yy = y0 + (k * RP + jr - 1) * dil;
                if (k * RP + jr < kColRows && yy >= 0 && yy < H) inframe |= 1u << k;
                const int yc = yy < 0 ? 0 : (yy < H ? yy : H - 1);
                if constexpr (PACK) {
#pragma unroll
                    for (int q = 0; q < 5; ++q) raw[k][q] = *at(f.v[q] + (long long)yc * W, 4u * xx);
                    rawy[k] = (float)yc;
                } else {
                    v[k] = __builtin_bit_cast(bf16x8, *(gptr<const uint4>)at(in + ((long long)it.n * H + yc) * W * CIN,
                                                                           (unsigned)xx * (2u * CIN) + 16u * c));
                }
            }
        }
    };
    settle();
    if (left > 0) fetch();
    // the weight operands in the order the lanes read them, all loaded at once
    // behind the first item's rows (one memory round trip for everything; block
    // by block through LDS took 0.1 to 0.3 us more)
    constexpr int WPW = (NKB + WV - 1) / WV;
    bf16x8 wv[WPW];
#pragma unroll
    for (int k = 0; k < WPW; ++k) {
        const int kk = 16 * (k * WV + wave) + 8 * kh;
        wv[k] = kk < K ? load8(w + ((PF ? m : weight_row(m)) * 9 + kk / CIN) * CIN + kk % CIN) : bf16x8{};
    }
    if (threadIdx.x < 32) sBias[threadIdx.x] = bias ? bias[threadIdx.x] : 0.f;
#pragma unroll
    for (int k = 0; k < WPW; ++k)
        if (k * WV + wave < NKB) sB[k * WV + wave][lane] = wv[k];
    double vacc = 0.0;  // VOL: this lane's share of the light-phase volume
    float lacc = 0.f;   // MSE: this lane's share of the squared error
    for (bool later = false; left > 0; later = true) {
        if (later) __syncthreads();  // every wave is done with the previous item's rows
        if (i < win) {
#pragma unroll
            for (int k = 0; k < NPASS; ++k) {
                const int j = k * RP + jr;
                if (CIN == 8 && j >= kColRows) break;
                if constexpr (PACK)
                    v[k] = pack_pixel(raw[k][0], raw[k][1], raw[k][2], raw[k][3], raw[k][4], rawy[k], sc);
                if (!(inframe >> k & 1)) v[k] = bf16x8{};
                *reinterpret_cast<bf16x8*>(&sX[j][CIN == 32 ? swz(i, c) : 8 * i]) = RELU ? relu8(v[k]) : v[k];
            }
        }
        __syncthreads();
        const int ya = y0 + S * wave * dil, x0 = it.sx * 32, npx = W - x0;
        const long long pa = ((long long)it.n * H + ya) * W + x0;  // the first segment's first pixel
        Extra e[S] = {};
        float old[S][5];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const long long p = pa + (long long)s * dil * W;
            if (ya + s * dil >= H || m >= npx) continue;
            if constexpr (ADV) {
                if (kh == 0) {
#pragma unroll
                    for (int q = 0; q < 5; ++q) old[s][q] = *at(f.v[q] + p, 4u * m);
                }
            } else if constexpr (MSE) {
                if (kh == 0) {
#pragma unroll
                    for (int q = 0; q < 5; ++q) old[s][q] = *at(target + 5 * p, 4u * (5 * m + q));
                }
            } else if constexpr (!PF) {
                load_extra<OUTF32, RES, MASK>(e[s], res, mask, p * 32 + 32 * m + 16 * kh);
            }
        }
        // the next item's rows
        it.next(R, G, SC);
        --left;
        settle();
        if (left > 0) fetch();
        if (ya >= H) continue;
        f32x16 acc[S] = {};
        if constexpr (S > 1) {
            // window row r is tap row r - s of segment s
            bf16x8 wr[3][6];
#pragma unroll
            for (int r = 0; r < S + 2; ++r) {
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    if (r < 3) wr[r][q] = sB[6 * r + q][lane];
                    const bf16x8 a =
                        *reinterpret_cast<const bf16x8*>(&sX[S * wave + r][swz(m + (q >> 1) * dil, 2 * (q & 1) + kh)]);
#pragma unroll
                    for (int s = 0; s < S; ++s)
                        if (r >= s && r - s < 3)
                            acc[s] = product<PF>(wr[r - s][q], a, acc[s]);
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < NKB; ++q) {
                bf16x8 a;
                if constexpr (CIN == 32) {
                    const int tap = q >> 1, tr = tap / 3, tc = tap % 3;
                    a = *reinterpret_cast<const bf16x8*>(&sX[wave + tr][swz(m + tc * dil, 2 * (q & 1) + kh)]);
                } else {
                    const int tap = 2 * q + kh < 9 ? 2 * q + kh : 8;
                    a = *reinterpret_cast<const bf16x8*>(&sX[wave + tap / 3][8 * (m + tap % 3 * dil)]);
                    if (2 * q + 1 >= 9 && kh) a = bf16x8{};
                }
                acc[0] = product<PF>(sB[q][lane], a, acc[0]);
            }
        }
        // keeps the epilogue's LDS reads behind the products: hoisted above them
        // they cost the registers of a wave per SIMD or spills
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (ya + s * dil >= H) break;
            const long long p = pa + (long long)s * dil * W, o = p * 32;
            const bool here = m < npx;
            if constexpr (ADV) {
                if (here && kh == 0) {
                    float phi;
                    advance_pixel(acc[s], sBias, old[s], f, sc, p + m, phi);
                    if (VOL) vacc += 0.5 * (1.0 - (double)phi);
                }
            } else if constexpr (MSE) {
                bf16x8 gr = {};
                if (here && kh == 0) {
#pragma unroll
                    for (int q = 0; q < 5; ++q) {
                        const float err = acc[s][q] + sBias[q] - old[s][q];
                        lacc += err * err;
                        gr[q] = (bf16)(2.f * err * mse_scale);
                    }
                }
                // 16 bytes per lane, 4 lanes a pixel: chunk 0 from the pixel's lane, the others zero
                const uint4 g4 = __builtin_bit_cast(uint4, gr);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int px = 16 * j + lane / 4;
                    uint4 q = {(unsigned)__shfl((int)g4.x, px), (unsigned)__shfl((int)g4.y, px),
                               (unsigned)__shfl((int)g4.z, px), 0u};
                    if (lane % 4) q = uint4{0u, 0u, 0u, 0u};
                    if (px < npx) *reinterpret_cast<uint4*>(static_cast<bf16*>(out) + o + px * 32 + 8 * (lane % 4)) = q;
                }
            } else if constexpr (PF) {
                store_channels<OUTF32>(acc[s], sBias[m], out, o, npx, lane);
            } else {
                conv_store<OUTF32, RES, MASK>(acc[s], sBias, e[s], res, sO[wave], out, o, npx, lane);
            }
        }
    }
    if constexpr (MSE) {
        // as the volume below; the first workgroup clears the entries without one
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) lacc += __shfl_xor(lacc, o);
        __shared__ float sL[WV];
        if (lane == 0) sL[wave] = lacc;
        __syncthreads();
        if (threadIdx.x == 0) {
            float s = 0.f;
            for (int k = 0; k < WV; ++k) s += sL[k];
            lpart[blockIdx.x] = s;
        }
        if (blockIdx.x == 0)
            for (int k = gridDim.x + threadIdx.x; k < kLossParts; k += blockDim.x) lpart[k] = 0.f;
    }
    if constexpr (VOL) {
        // the wave's sum (butterfly: every lane ends with the same value), then the
        // workgroup's in wave order into vpart[8 blockIdx.x]
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) vacc += __shfl_xor(vacc, o);
        __shared__ double sV[WV];
        if (lane == 0) sV[wave] = vacc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double s = 0.0;
            for (int k = 0; k < WV; ++k) s += sV[k];
            vpart[8 * blockIdx.x] = s;
        }
    }
}

// The network's last layer with the state update fused into its epilogue,
// on one frame: f_c += (conv(A, w) + bias)_c inc[c] for the five state fields
// c < 5 (A = relu(in) if RELU; 32 input channels).  Equal to k_conv with an
// FP32 output followed by k_advance (the same sums, the same roundings), but
// the 32 FP32 channels of the increment are never written or read back.
template <bool RELU>
__global__ __launch_bounds__(256) void k_conv_advance(const bf16* __restrict__ in, const bf16* __restrict__ w,
                                                      const float* __restrict__ bias, State5 f, Scales sc, int dil,
                                                      int H, int W)
{
    constexpr int NKB = 18;
    const int lane = threadIdx.x % 64;
    const int segs_per_row = (W + 31) / 32;
    const int nseg = H * segs_per_row;
    const int wave0 = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
    const int nwaves = (int)gridDim.x * 4;
    const int m = lane % 32, kh = lane / 32;
    __shared__ bf16x8 sB[NKB + 1][64];
    __shared__ float sBias[32];
    if (threadIdx.x < 32) sBias[threadIdx.x] = bias ? bias[threadIdx.x] : 0.f;
    stage_weights<32>(w, sB);
    for (int seg = wave0; seg < nseg; seg += nwaves) {
        const int lz = lane + 64 * __builtin_amdgcn_readfirstlane((int)((unsigned)seg >> 31));
        const int x0 = (seg % segs_per_row) * 32;
        const int y = seg / segs_per_row;
        const f32x16 acc = conv_seg32<RELU>(in, sB, lz, dil, H, W, 0, y, x0, m, kh);
        if (kh == 0 && x0 + m < W) {
            const long long p = (long long)y * W + x0 + m;
            float old[5], phi;
#pragma unroll
            for (int c = 0; c < 5; ++c) old[c] = f.v[c][p];
            advance_pixel(acc, sBias, old, f, sc, p, phi);
        }
    }
}

// Weights of the adjoint convolution: wt[ci][8 - tap][co] = w[co][tap][ci]
// (channels swapped, taps mirrored).  wt has cin_t = 32 input channels and
// cout rows; rows ci >= cin of w stay zero.
// Workgroups with the same blockIdx.y work on one layer.
__global__ void k_adjoint_weights(AdjointLayers L)
{
    const bf16* __restrict__ w = L.w[blockIdx.y];
    bf16* __restrict__ wt = L.wt[blockIdx.y];
    const int cin = L.cin[blockIdx.y];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;  // over 32 x 9 x 32
    if (i >= 32 * 9 * 32) return;
    const int co = i % 32, tap = (i / 32) % 9, ci = i / (32 * 9);
    wt[((long long)ci * 9 + (8 - tap)) * 32 + co] = ci < cin ? w[((long long)co * 9 + tap) * cin + ci] : (bf16)0.f;
}

// ---- weight and bias gradients ----

typedef short s16x4 __attribute__((ext_vector_type(4)));
// v > 0 ? v : 0 of 8 BF16 values (NaN becomes 0) in packed 16-bit integers:
// positive NaNs are the positive integers above the infinity's.
__device__ inline bf16x8 relu8_nan(bf16x8 v)
{
    s16x8 s = __builtin_elementwise_max(__builtin_bit_cast(s16x8, v), (s16x8)(short)0);
    s &= ~(((s16x8)(short)0x7F80 - s) >> (s16x8)(short)15);
    return __builtin_bit_cast(bf16x8, s);
}

// Bits of the first n of 8 BF16 values, and the values they keep.
__device__ inline uint4 first_of(int n)
{
    auto word = [&](int i) { return n >= 2 * i + 2 ? ~0u : (n == 2 * i + 1 ? 0xffffu : 0u); };
    return {word(0), word(1), word(2), word(3)};
}
__device__ inline bf16x8 keep(bf16x8 v, const uint4& bits)
{
    const uint4 u = __builtin_bit_cast(uint4, v);
    return __builtin_bit_cast(bf16x8, uint4{u.x & bits.x, u.y & bits.y, u.z & bits.z, u.w & bits.w});
}

// Transposed operand of a matrix-core product from pixel-major LDS rows: the
// 16 lanes of a group hand in 4 pixels x 16 channels (lane i: pixel i / 4,
// channels 4 (i % 4) ..) and lane i receives channel i of the 4 pixels; two
// reads give 8 pixels.  `p` is this lane's address for the first four, and
// `step` the elements from a pixel to the one 4 further on.
__device__ inline bf16x8 read_tr(const bf16* p, int step)
{
    typedef __attribute__((address_space(3))) s16x4* lptr;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr)(p + step));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Weight gradient partials: part[g][co][kk] = sum over the workgroup's pixels
// of dy[p][co] * A(p + d off(tap))[ci], kk = tap * CIN + ci, A = relu(in) if
// relu_in, dilation d.  As a matrix product M = co, N = (tap, ci), K = pixels:
// both operands are wanted with 8 pixels of one channel per lane, the
// transpose of the NHWC rows, which the LDS transpose reads deliver from rows
// stored as they come.
// A work item is 8 rows y0, y0 + d, ... of one 64-pixel column: 8 rows of dy
// and the 10 input rows they meet, over 64 + 2 min(d, 64) pixels (periodic in
// x; for d > 64 the three tap columns' 64 pixels each), rows outside the frame
// and dy beyond the row as zeros.  Twelve waves: wave (ty, k) takes the tap
// row ty and pixels 16 k ... of every row, 3 products (one per tap column) to
// one dy operand: 8 LDS reads of 512 bytes per 3 products, 48 accumulators.
// All nine taps in one wave read less (20 per 9) but hold 144 accumulators and
// have three times as many to add up over waves at the end.  CIN = 8: the 32
// columns of one product are the 8 channels of the three taps (the last 8 are
// dropped).  The next item's rows are loaded into registers while the current
// one is multiplied.  One workgroup per partial sum.
// Bound by the latency of an item's loads (three items per workgroup at 8 x 256
// x 192, 256 partial sums) and then by the bytes of dy and in.  On 8 x 256 x 192
// pixels, CIN = 32, with the bias:
// 18.7 us (2.7 TB/s of the 50 MB it cannot do without; 21.5 with items located
// by 64-bit divisions and the residue class outermost); by segments with 2-byte
// LDS transposes 609 us without the bias.
constexpr int kWgRW = 8, kWgRows = kWgRW + 2, kWgCol = 64, kWgThreads = 768;
// BIAS: also the bias gradient's partial sums, 32 values behind the weights'
// in part[g], added up by the work-items that stage dy (a kernel of its own
// reads dy again: 7 us per layer at 8 x 256 x 192).
// RAGGED (W not whole in 16): in the K block that holds the row's end dy is zero
// behind it, but the window holds other pixels there (x is periodic), and an
// infinite one times zero is no zero: the inputs are masked too, which costs 2
// to 5% (8 x 256 x 201 22.5 -> 23.6 us; a second loop for that block spills).
template <int CIN, int PIX, bool BIAS, bool RAGGED>
__global__ __launch_bounds__(kWgThreads) void k_wgrad(const bf16* __restrict__ dy, const bf16* __restrict__ in,
                                                      int relu_in, int dil, int N, int H, int W,
                                                      float* __restrict__ part)
{
    constexpr int CH = CIN / 8, UR = PIX * CH;           // 16-byte units per staged input row
    constexpr int RP = kWgThreads / UR;                  // input rows per pass
    constexpr int NP = (kWgRows + RP - 1) / RP;
    constexpr int NPD = (kWgRW + 2) / 3;                 // dy: 3 rows of 64 x 4 units per pass
    constexpr int NT = CIN == 32 ? 3 : 1;                // products per K block
    constexpr int K = 9 * CIN;
    struct Stage {
        bf16 a[kWgRows][PIX * CIN];
        bf16 d[kWgRW][kWgCol * 32];
    };
    union LDS {
        Stage s;
        float red[2][3][NT][16][64];
        float bias[kWgThreads / 4][33];
    };
    __shared__ __attribute__((aligned(16))) LDS L;
    static_assert(kWgThreads % UR == 0 && kWgThreads == 3 * kWgCol * 4, "whole rows per pass");
    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int ty = wave % 3, kg = wave / 3;
    const int SC = (W + kWgCol - 1) / kWgCol;
    const int G = ((H + dil - 1) / dil + kWgRW - 1) / kWgRW, R = dil < H ? dil : H;
    const unsigned nitems = (unsigned)N * R * G * SC;
    // a contiguous run of items per workgroup, runs in XCD order (bands of rows,
    // as in the convolutions that wrote dy and in); workgroups beyond the items
    // have none and write zeros
    const unsigned used = nitems < gridDim.x ? nitems : gridDim.x;
    const unsigned b = xcd_contiguous(blockIdx.x, gridDim.x);
    const unsigned per = nitems / used, rem = nitems - per * used;
    int left = b < used ? (int)__builtin_amdgcn_readfirstlane(per + (b < rem ? 1 : 0)) : 0;
    Item it;
    it.locate(left ? b * per + (b < rem ? b : rem) : 0, R, G, SC);
    const int sd = dil < kWgCol ? dil : kWgCol;          // window pixels from a tap column to the next
    // this work-item's unit of each pass: row ja of the pass, window pixel ia, channels 8 ca ..
    const int ja = tid / UR, ia = (tid % UR) / CH, ca = tid % CH;
    const bool useda = ia < kWgCol + 2 * sd;
    const int xrel = dil <= kWgCol ? ia - dil : (ia / kWgCol - 1) * dil + ia % kWgCol;
    const int jd = tid / (kWgCol * 4), id = (tid % (kWgCol * 4)) / 4, cd = tid % 4;

    bf16x8 va[NP], vd[NPD];
    // first row of the item `it`; passes over items whose rows lie beyond the frame
    long long y0 = 0;
    auto settle = [&]() {
        while (left > 0 && (y0 = it.r + (long long)it.g * kWgRW * dil) >= H) {
            it.next(R, G, SC);
            --left;
        }
    };
    auto fetch = [&]() {
        const int x0 = it.sx * kWgCol;
        long long xx = (long long)x0 + xrel;
        while (xx < 0) xx += W;
        while (xx >= W) xx -= W;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int j = k * RP + ja;
            const long long y = y0 + (long long)(j - 1) * dil;
            va[k] = bf16x8{};
            if (j < kWgRows && useda && y >= 0 && y < H)
                va[k] = load8u(in + (((long long)it.n * H + y) * W + xx) * CIN + 8 * ca);
        }
#pragma unroll
        for (int k = 0; k < NPD; ++k) {
            const int j = 3 * k + jd;
            const long long y = y0 + (long long)j * dil;
            vd[k] = bf16x8{};
            if (j < kWgRW && y < H && x0 + id < W) vd[k] = load8u(dy + (((long long)it.n * H + y) * W + x0 + id) * 32 + 8 * cd);
        }
    };
    // operand addresses of this lane: pixel (within a K block) and channels of its group's read
    const int pl = 16 * kg + 8 * (lane / 32) + (lane % 16) / 4, c4 = 16 * ((lane / 16) % 2) + 4 * (lane % 4);
    const int tx8 = c4 / 8 < 2 ? c4 / 8 : 2;             // CIN = 8: the tap column of the lane's channels
    f32x16 acc[NT] = {};
    float bsum[8] = {};
    settle();
    if (left > 0) fetch();
    while (left > 0) {
        __syncthreads();  // every wave is done with the previous item
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int j = k * RP + ja;
            if (j < kWgRows && useda) *reinterpret_cast<bf16x8*>(&L.s.a[j][ia * CIN + 8 * ca]) = relu_in ? relu8_nan(va[k]) : va[k];
        }
#pragma unroll
        for (int k = 0; k < NPD; ++k) {
            if (3 * k + jd < kWgRW) *reinterpret_cast<bf16x8*>(&L.s.d[3 * k + jd][id * 32 + 8 * cd]) = vd[k];
            if constexpr (BIAS) {  // zeros beyond the rows and the frame
#pragma unroll
                for (int j = 0; j < 8; ++j) bsum[j] += to_f(vd[k][j]);
            }
        }
        const int last = (int)(H - 1 - y0);  // rows of the frame below y0
        const int npx = W - it.sx * kWgCol;  // pixels of the row from the column's first
        const bool mine = 16 * kg < npx;
        uint4 real = {};
        if constexpr (RAGGED) real = first_of(npx - (16 * kg + 8 * (lane / 32)));
        __syncthreads();
        it.next(R, G, SC);
        --left;
        settle();
        if (left > 0) fetch();
        if (!mine) continue;
        for (int k = 0; k < kWgRW && k * (long long)dil <= last; ++k) {
            const bf16x8 a = read_tr(&L.s.d[k][pl * 32 + c4], 4 * 32);
            if constexpr (CIN == 32) {
#pragma unroll
                for (int tx = 0; tx < 3; ++tx) {
                    bf16x8 b = read_tr(&L.s.a[k + ty][(pl + tx * sd) * 32 + c4], 4 * 32);
                    if constexpr (RAGGED) b = keep(b, real);
                    acc[tx] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[tx], 0, 0, 0);
                }
            } else {
                bf16x8 b = read_tr(&L.s.a[k + ty][(pl + tx8 * sd) * 8 + c4 % 8], 4 * 8);
                if constexpr (RAGGED) b = keep(b, real);
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[0], 0, 0, 0);
            }
        }
    }
    // the four waves of a tap row add up: 2 and 3 into 0 and 1, then 1 into 0
#pragma unroll
    for (int half = 2; half >= 1; half /= 2) {
        __syncthreads();
        if (kg >= half && kg < 2 * half) {
#pragma unroll
            for (int q = 0; q < NT; ++q)
#pragma unroll
                for (int i = 0; i < 16; ++i) L.red[kg - half][ty][q][i][lane] = acc[q][i];
        }
        __syncthreads();
        if (kg < half) {
#pragma unroll
            for (int q = 0; q < NT; ++q)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[q][i] += L.red[kg][ty][q][i][lane];
        }
    }
    constexpr long long WIDTH = 32LL * K + (BIAS ? 32 : 0);
    part += b * WIDTH;
    if constexpr (BIAS) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; ++j) L.bias[tid / 4][8 * cd + j] = bsum[j];
        __syncthreads();
        // 768 = 24 x 32: slice s of 24 adds 8 rows, then one work-item the slices in order
        const int co = tid % 32, sl = tid / 32;
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) v += L.bias[8 * sl + q][co];
        __syncthreads();
        L.bias[sl][co] = v;
        __syncthreads();
        if (tid < 32) {
            float t = 0.f;
            for (int q = 0; q < kWgThreads / 32; ++q) t += L.bias[q][tid];
            part[32 * K + tid] = t;
        }
    }
    if (kg == 0) {
        const int m = lane % 32;
        if (CIN == 8 && m >= 24) return;
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const int kk = CIN == 32 ? (3 * ty + q) * 32 + m : 3 * ty * 8 + m;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int co = 8 * (i / 4) + 4 * (lane / 32) + (i % 4);
                part[co * K + kk] = acc[q][i];
            }
        }
    }
}

// Bias gradient partials: part[g][co] = sum over the workgroup's pixels of
// dy[p][co]; 64 pixels of 16-byte units per pass, four passes in flight.
// Bound by the bytes of dy: 6.9 us on 8 x 256 x 192 pixels (25 MB; 45 us with
// 2-byte loads, one in flight per work-item).
__global__ __launch_bounds__(256) void k_bgrad(const bf16* __restrict__ dy, long long npix, float* __restrict__ part)
{
    __shared__ float red[64][33];
    const int c = threadIdx.x % 4, r = threadIdx.x / 4;
    const long long p0 = (long long)blockIdx.x * npix / gridDim.x, p1 = (long long)(blockIdx.x + 1) * npix / gridDim.x;
    float s[8] = {};
#pragma unroll 4
    for (long long p = p0 + r; p < p1; p += 64) {
        const bf16x8 v = load8u(dy + p * 32 + 8 * c);
#pragma unroll
        for (int j = 0; j < 8; ++j) s[j] += to_f(v[j]);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) red[r][8 * c + j] = s[j];
    __syncthreads();
    if (threadIdx.x < 32) {
        float t = 0.f;
        for (int q = 0; q < 64; ++q) t += red[q][threadIdx.x];
        part[(long long)blockIdx.x * 32 + threadIdx.x] = t;
    }
}

// out[j] = sum_g part[g][j] in a fixed order (deterministic): a workgroup takes
// 64 columns, wave s of 16 the groups s, s + 16, ... in turn, then the 16 sums
// in order.  4 us for 256 groups of 9216 columns; one work-item per column and
// all groups in turn has too few loads in flight (60 us).
__global__ __launch_bounds__(1024) void k_reduce(const float* __restrict__ part, int ngroups, long long width,
                                                 float* __restrict__ out)
{
    __shared__ float red[16][64];
    const int lane = threadIdx.x % 64, s = threadIdx.x / 64;
    const long long j = (long long)blockIdx.x * 64 + lane;
    float v = 0.f;
    if (j < width) {
#pragma unroll 8
        for (int g = s; g < ngroups; g += 16) v += part[(long long)g * width + j];
    }
    red[s][lane] = v;
    __syncthreads();
    if (s == 0 && j < width) {
        float t = 0.f;
#pragma unroll
        for (int q = 0; q < 16; ++q) t += red[q][lane];
        out[j] = t;
    }
}

// One Adam update of a master value; returns it.
__device__ inline float adam_value(float& p, float g, float& m1, float& m2, float lr, float b1, float b2, float eps,
                                   float c1, float c2)
{
    const float a = b1 * m1 + (1.f - b1) * g;
    const float b = b2 * m2 + (1.f - b2) * g * g;
    m1 = a;
    m2 = b;
    return p -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

// Adam on FP32 master weights; writes the BF16 copy used by the convolutions.
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ gr, float* __restrict__ m1,
                       float* __restrict__ m2, bf16* __restrict__ pb, long long n, float lr, float b1, float b2,
                       float eps, float c1, float c2)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    pb[i] = (bf16)adam_value(p[i], gr[i], m1[i], m2[i], lr, b1, b2, eps, c1, c2);
}

// Adam for every layer of a network straight from the gradients' partial sums
// (sur_layer_grads: part[g] = 32 * 9 * cin weights, then 32 biases), each summed
// as k_reduce does: workgroup = 64 columns of one layer, the layers' workgroups
// one after another.  One launch instead of 24; the first workgroup also adds
// up the loss.
__global__ __launch_bounds__(1024) void k_adam_layers(AdamLayers L, float lr, float b1, float b2, float eps, float c1,
                                                      float c2, const float* __restrict__ lpart,
                                                      float* __restrict__ loss)
{
    __shared__ float red[16][64];
    const int lane = threadIdx.x % 64, s = threadIdx.x / 64;
    int b = blockIdx.x, q = 0;
    while (q + 1 < L.n && b >= L.blocks[q]) b -= L.blocks[q++];
    const AdamLayer A = L.l[q];
    const int nw = 32 * 9 * A.cin, width = nw + 32, j = 64 * b + lane;
    float v = 0.f;
    if (j < width) {
#pragma unroll 8
        for (int g = s; g < A.groups; g += 16) v += A.part[(long long)g * width + j];
    }
    red[s][lane] = v;
    __syncthreads();
    if (s == 0 && j < width) {
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < 16; ++k) t += red[k][lane];
        if (j < nw) A.Wb[j] = (bf16)adam_value(A.W[j], t, A.mW1[j], A.mW2[j], lr, b1, b2, eps, c1, c2);
        else adam_value(A.b[j - nw], t, A.mb1[j - nw], A.mb2[j - nw], lr, b1, b2, eps, c1, c2);
    }
    if (blockIdx.x == 0) {
        __syncthreads();
        float e = 0.f;
        for (int k = threadIdx.x; k < kLossParts; k += 1024) e += lpart[k];
        for (int o = 32; o > 0; o >>= 1) e += __shfl_xor(e, o);
        if (lane == 0) red[0][s] = e;
        __syncthreads();
        if (threadIdx.x == 0) {
            float t = 0.f;
            for (int k = 0; k < 16; ++k) t += red[0][k];
            *loss = t;
        }
    }
}

// Squared error of the predicted increment delta (channels 0..nout-1) against
// the target increment (nout channels): per-workgroup partial sums, and the
// gradient 2 (delta - target) * scale as BF16 (channels >= nout zero).
__global__ __launch_bounds__(256) void k_mse(const float* __restrict__ delta /*C=32*/,
                                             const float* __restrict__ target /*C=nout*/, long long npix, int nout,
                                             float scale, bf16* __restrict__ grad /*C=32*/, float* __restrict__ part)
{
    __shared__ float red[256];
    float s = 0.f;
    for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < npix * 32;
         q += (long long)gridDim.x * blockDim.x) {
        const long long p = q / 32;
        const int c = (int)(q % 32);
        float g = 0.f;
        if (c < nout) {
            const float e = delta[q] - target[p * nout + c];
            s += e * e;
            g = 2.f * e * scale;
        }
        grad[q] = (bf16)g;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// Network input from the five FP32 state fields of one frame (x fastest):
// channels (phi, ux / U, uy / U, (T - T_rest(y)) / dT, c4, c5,
// (p - P (1 - phi) / 2) / P, 0), BF16: the pressure enters less its
// Young-Laplace part, so the small dynamic pressure keeps BF16's relative precision.
__global__ void k_pack(State5 f, long long npix, int w, Scales sc, bf16* __restrict__ x)
{
    const long long p = (long long)xcd_contiguous(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (p >= npix) return;
    *reinterpret_cast<bf16x8_u*>(x + p * 8) =
        pack_pixel(f.v[0][p], f.v[1][p], f.v[2][p], f.v[3][p], f.v[4][p], (float)(p / w), sc);
}

// Target increment between two states, channel c in units of inc[c]: FP32, C = 5.
__global__ void k_pack_target(State5 f0, State5 f1, long long npix, Scales sc, float* __restrict__ t)
{
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npix) return;
#pragma unroll
    for (int c = 0; c < 5; ++c) t[p * 5 + c] = (f1.v[c][p] - f0.v[c][p]) / sc.inc[c];
}

// Advances the five FP32 state fields in place: f_c += delta_c inc[c].
__global__ void k_advance(const float* __restrict__ delta, long long npix, Scales sc, State5 f)
{
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npix) return;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        float* v = const_cast<float*>(f.v[c]);
        v[p] = v[p] + delta[p * 32 + c] * sc.inc[c];
    }
}

// Per-workgroup FP64 partial sums over one frame: the light-phase volume
// sum (1 - phi) / 2 if b is null, else, for the channels phi, ux, uy, T,
// sum (a - b)^2 and sum (b - rest)^2 with rest = (1, 0, 0, T_rest(y)).
__global__ __launch_bounds__(256) void k_frame_sums(State5 a, State5 b, int has_b, long long npix, int w, Scales sc,
                                                    double* __restrict__ part)
{
    __shared__ double red[8][256];
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < npix;
         p += (long long)gridDim.x * blockDim.x) {
        if (!has_b) {
            acc[0] += 0.5 * (1.0 - (double)a.v[0][p]);
            continue;
        }
        const double rest[4] = {1.0, 0.0, 0.0, (double)sc.t_a + (double)sc.t_b * (double)(p / w)};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const double bv = b.v[c][p];
            const double d = (double)a.v[c][p] - bv, r = bv - rest[c];
            acc[2 * c] += d * d;
            acc[2 * c + 1] += r * r;
        }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) red[k][threadIdx.x] = acc[k];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o)
#pragma unroll
            for (int k = 0; k < 8; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x < 8) part[blockIdx.x * 8 + threadIdx.x] = red[threadIdx.x][0];
}

// Sums the partials of k_frame_sums over workgroups in a fixed order: each
// of 256 threads adds the groups g = t, t + 256, ... in turn, then a tree over
// the threads; one pass for each of the first nout quantities.
__global__ __launch_bounds__(256) void k_frame_final(const double* __restrict__ part, int groups, int nout,
                                                     double* __restrict__ out)
{
    __shared__ double red[256];
    const int t = threadIdx.x;
    for (int k = 0; k < nout; ++k) {
        double s = 0.0;
        for (int g = t; g < groups; g += 256) s += part[g * 8 + k];
        red[t] = s;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if (t < o) red[t] += red[t + o];
            __syncthreads();
        }
        if (t == 0) out[k] = red[0];
        __syncthreads();
    }
}

// ---- launchers ----

// Whether the byte offsets within a row fit the 32 bits the column kernels give
// them; the kernels by segments take longer rows.
static bool row_fits(int cin, int W) { return W <= (1LL << 32) / (2 * cin); }

// Work items of a column-kernel launch: every column's group of kColRW rows of
// one residue class of y mod dil.
static long long col_items(int dil, int N, int H, int W)
{
    return (long long)N * (dil < H ? dil : H) * (((H + dil - 1) / dil + kColRW - 1) / kColRW) * ((W + 31) / 32);
}

// Its workgroups where each leaves a partial sum: those resident, two per CU.
static unsigned resident_groups(int dil, int N, int H, int W)
{
    const long long items = col_items(dil, N, H, W);
    return (unsigned)(items < 512 ? items : 512);
}

// Elsewhere up to three items per CU get a workgroup each, and the items of the
// last third start as others end, wherever that is: runs of one and two items
// take longer (580 items of 2 x 456 x 160 at dilation 8: 10.4 us a layer in
// runs, 9.5 so).  Beyond, runs are better for the item fetched ahead (832 items,
// 2 x 405 x 242: 10.6 and 11.3; 2 x 1024 x 240: 19.6 and 21.4).
static unsigned col_groups(int dil, int N, int H, int W)
{
    const long long items = col_items(dil, N, H, W);
    return (unsigned)(items <= 768 ? items : 512);
}

// Narrow windows: whether waves of two rows and three workgroups per CU take
// the items in fewer rounds: 768 in one (3 x 256 CUs; 256 wide, dilation 2:
// 528 items 9.4 -> 8.4 us a layer, 768 9.6 -> 9.1), 1025 to 1280 in two, the
// second one not full (1088 items 14.4 -> 12.9, 1280 14.2 -> 13.1).  Elsewhere
// single rows are better or within 3% (512 items 7.4 and 7.3, 896 10.7 and 11.6, 1024 11.4
// and 12.0, 1536 15.0 and 14.6, 1920 18.5 and 18.8).
static bool two_rows(int dil, int N, int H, int W)
{
    const long long items = col_items(dil, N, H, W);
    return (items > 512 && items <= 768) || (items > 1024 && items <= 1280);
}

// By columns (dilation <= 16): workgroups walk the columns' groups of rows, with
// the narrow window up to dilation 4.
template <int CIN, bool RELU, bool OUTF32, bool RES, bool MASK>
static void conv_columns(const bf16* in, const bf16* w, const float* bias, const void* res, const bf16* mask, void* out,
                         int dil, int N, int H, int W, hipStream_t s)
{
    const dim3 grid(col_groups(dil, N, H, W)), block(64 * kColRW);
    if (dil > 4) {
        hipLaunchKernelGGL((k_conv_col<CIN, RELU, OUTF32, RES, MASK>), grid, block, 0, s, in, w, bias, res, mask, out, dil,
                           N, H, W, State5{}, Scales{});
        return;
    }
    if constexpr (CIN == 32) {
        if (two_rows(dil, N, H, W)) {
            const long long items = col_items(dil, N, H, W);
            hipLaunchKernelGGL((k_conv_col<CIN, RELU, OUTF32, RES, MASK, false, kColPixNarrow, false, false, false, 2>),
                               dim3((unsigned)(items < 768 ? items : 768)), dim3(64 * kColRW / 2), 0, s, in, w, bias,
                               res, mask, out, dil, N, H, W, State5{}, Scales{});
            return;
        }
    }
    hipLaunchKernelGGL((k_conv_col<CIN, RELU, OUTF32, RES, MASK, false, kColPixNarrow>), grid, block, 0, s, in, w, bias, res,
                       mask, out, dil, N, H, W, State5{}, Scales{});
}

template <int CIN, bool RELU, bool OUTF32, bool RES, bool MASK>
static void conv_t(const bf16* in, const bf16* w, const float* bias, const void* res, const bf16* mask, void* out,
                   int dil, int N, int H, int W, hipStream_t s)
{
    if constexpr (CIN == 32 || RES || MASK) {  // the plain first layer: see k_conv
        if (dil <= 16 && row_fits(CIN, W)) {
            conv_columns<CIN, RELU, OUTF32, RES, MASK>(in, w, bias, res, mask, out, dil, N, H, W, s);
            return;
        }
    }
    // a resident grid walks the segments, so each workgroup stages the weights once
    const long long segs = (long long)N * H * ((W + 31) / 32);
    long long groups = (segs + 3) / 4;
    if (groups > 1536) groups = 1536;
    hipLaunchKernelGGL((k_conv<CIN, RELU, OUTF32, RES, MASK>), dim3((unsigned)groups), dim3(256), 0, s, in, w, bias, res,
                       mask, out, dil, N, H, W);
}

template <int CIN, bool RELU, bool OUTF32>
static void conv_rm(const bf16* in, const bf16* w, const float* bias, const void* res, const bf16* mask, void* out,
                    int dil, int N, int H, int W, hipStream_t s)
{
    if (res && mask) conv_t<CIN, RELU, OUTF32, true, true>(in, w, bias, res, mask, out, dil, N, H, W, s);
    else if (res) conv_t<CIN, RELU, OUTF32, true, false>(in, w, bias, res, mask, out, dil, N, H, W, s);
    else if (mask) conv_t<CIN, RELU, OUTF32, false, true>(in, w, bias, res, mask, out, dil, N, H, W, s);
    else conv_t<CIN, RELU, OUTF32, false, false>(in, w, bias, res, mask, out, dil, N, H, W, s);
}

template <int CIN>
static void conv_c(const bf16* in, const bf16* w, const float* bias, const void* res, const bf16* mask, void* out,
                   int out_f32, int relu_in, int dil, int N, int H, int W, hipStream_t s)
{
    if (relu_in && out_f32) conv_rm<CIN, true, true>(in, w, bias, res, mask, out, dil, N, H, W, s);
    else if (relu_in) conv_rm<CIN, true, false>(in, w, bias, res, mask, out, dil, N, H, W, s);
    else if (out_f32) conv_rm<CIN, false, true>(in, w, bias, res, mask, out, dil, N, H, W, s);
    else conv_rm<CIN, false, false>(in, w, bias, res, mask, out, dil, N, H, W, s);
}

hipError_t conv(const bf16* in, int cin, const bf16* w, const float* bias, const void* res, const bf16* mask,
                void* out, int out_f32, int relu_in, int dil, int N, int H, int W, hipStream_t s)
{
    if (cin == 8) conv_c<8>(in, w, bias, res, mask, out, out_f32, relu_in, dil, N, H, W, s);
    else conv_c<32>(in, w, bias, res, mask, out, out_f32, relu_in, dil, N, H, W, s);
    return hipGetLastError();
}

hipError_t conv_packed(const State5& f, const Scales& sc, const bf16* w, const float* bias, bf16* out, int dil, int H,
                       int W, hipStream_t s)
{
    if (dil > 16) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_conv_col<8, false, false, false, false, false, kColPix, false, true>),
                       dim3(col_groups(dil, 1, H, W)), dim3(64 * kColRW), 0, s, nullptr, w, bias, nullptr, nullptr,
                       out, dil, 1, H, W, f, sc, nullptr);
    return hipGetLastError();
}

// The output layer by columns (dilation <= 16), always with the wide window:
// 10.2 us in a network block at 256 x 1024 (12.0 with the increment passed
// through LDS; here a lane has the five channels of its pixel).
template <bool RELU, bool VOL>
static void col_advance(const bf16* in, const bf16* w, const float* bias, int dil, int H, int W, const Scales& sc,
                        const State5& f, double* vpart, hipStream_t s)
{
    hipLaunchKernelGGL((k_conv_col<32, RELU, false, false, false, true, kColPix, VOL>), dim3(resident_groups(dil, 1, H, W)),
                       dim3(64 * kColRW), 0, s, in, w, bias, nullptr, nullptr, nullptr, dil, 1, H, W, f, sc, vpart);
}

hipError_t conv_advance_volume(const bf16* in, const bf16* w, const float* bias, int relu_in, int dil, int H, int W,
                               const Scales& sc, const State5& f, double* vpart, double* vout, hipStream_t s)
{
    if (dil > 16 || resident_groups(dil, 1, H, W) > (unsigned)kVolParts) return hipErrorInvalidValue;
    if (!row_fits(32, W)) {
        const hipError_t e = conv_advance(in, w, bias, relu_in, dil, H, W, sc, f, s);
        return e != hipSuccess ? e : frame_sums(f, nullptr, (long long)H * W, W, sc, vpart, kVolParts, vout, s);
    }
    if (relu_in) col_advance<true, true>(in, w, bias, dil, H, W, sc, f, vpart, s);
    else col_advance<false, true>(in, w, bias, dil, H, W, sc, f, vpart, s);
    hipLaunchKernelGGL(k_frame_final, dim3(1), dim3(256), 0, s, vpart, (int)resident_groups(dil, 1, H, W), 1, vout);
    return hipGetLastError();
}

hipError_t conv_advance(const bf16* in, const bf16* w, const float* bias, int relu_in, int dil, int H, int W,
                        const Scales& sc, const State5& f, hipStream_t s)
{
    if (dil <= 16 && row_fits(32, W)) {
        if (relu_in) col_advance<true, false>(in, w, bias, dil, H, W, sc, f, nullptr, s);
        else col_advance<false, false>(in, w, bias, dil, H, W, sc, f, nullptr, s);
        return hipGetLastError();
    }
    const long long segs = (long long)H * ((W + 31) / 32);
    long long groups = (segs + 3) / 4;
    if (groups > 1536) groups = 1536;
    if (relu_in)
        hipLaunchKernelGGL(k_conv_advance<true>, dim3((unsigned)groups), dim3(256), 0, s, in, w, bias, f, sc, dil, H, W);
    else
        hipLaunchKernelGGL(k_conv_advance<false>, dim3((unsigned)groups), dim3(256), 0, s, in, w, bias, f, sc, dil, H,
                           W);
    return hipGetLastError();
}

hipError_t adjoint_weights(const AdjointLayers& L, hipStream_t s)
{
    hipLaunchKernelGGL(k_adjoint_weights, dim3((32 * 9 * 32 + 255) / 256, L.n), dim3(256), 0, s, L);
    return hipGetLastError();
}

static hipError_t reduce(const float* part, int groups, long long width, float* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_reduce, dim3((unsigned)((width + 63) / 64)), dim3(1024), 0, s, part, groups, width, out);
    return hipGetLastError();
}

// The window of 96 pixels holds dilations up to 16 (47 or 94 KB of LDS); wider
// ones take 192 (up to 156 KB).  One workgroup per CU either way: a partial
// sum costs 36 KB of memory, and its caller sets how many there may be.
template <int CIN, bool BIAS, bool RAGGED>
static void wgrad_w(const bf16* dy, const bf16* in, int relu_in, int dil, int N, int H, int W, float* part, int groups,
                    hipStream_t s)
{
    if (dil <= 16)
        hipLaunchKernelGGL((k_wgrad<CIN, 96, BIAS, RAGGED>), dim3(groups), dim3(kWgThreads), 0, s, dy, in, relu_in, dil, N, H,
                           W, part);
    else
        hipLaunchKernelGGL((k_wgrad<CIN, 192, BIAS, RAGGED>), dim3(groups), dim3(kWgThreads), 0, s, dy, in, relu_in, dil, N,
                           H, W, part);
}
template <int CIN, bool BIAS>
static void wgrad_t(const bf16* dy, const bf16* in, int relu_in, int dil, int N, int H, int W, float* part, int groups,
                    hipStream_t s)
{
    if (W % 16) wgrad_w<CIN, BIAS, true>(dy, in, relu_in, dil, N, H, W, part, groups, s);
    else wgrad_w<CIN, BIAS, false>(dy, in, relu_in, dil, N, H, W, part, groups, s);
}

hipError_t wgrad(const bf16* dy, const bf16* in, int cin, int relu_in, int dil, int N, int H, int W, float* part,
                 int groups, float* out, hipStream_t s)
{
    const long long items = (long long)N * ((W + kWgCol - 1) / kWgCol) * (dil < H ? dil : H) * (((H + dil - 1) / dil + kWgRW - 1) / kWgRW);
    if (groups > items) groups = (int)items;
    if (cin == 8) wgrad_t<8, false>(dy, in, relu_in, dil, N, H, W, part, groups, s);
    else wgrad_t<32, false>(dy, in, relu_in, dil, N, H, W, part, groups, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return reduce(part, groups, 32LL * 9 * cin, out, s);
}

hipError_t layer_grads(const bf16* dy, const bf16* in, int cin, int relu_in, int dil, int N, int H, int W, float* part,
                       int groups, hipStream_t s)
{
    if (cin == 8) wgrad_t<8, true>(dy, in, relu_in, dil, N, H, W, part, groups, s);
    else wgrad_t<32, true>(dy, in, relu_in, dil, N, H, W, part, groups, s);
    return hipGetLastError();
}

hipError_t adam_layers(AdamLayers& L, float lr, float b1, float b2, float eps, int t, const float* lpart, float* loss,
                       hipStream_t s)
{
    const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
    unsigned total = 0;
    for (int q = 0; q < L.n; ++q) total += (unsigned)(L.blocks[q] = (32 * 9 * L.l[q].cin + 32 + 63) / 64);
    hipLaunchKernelGGL(k_adam_layers, dim3(total), dim3(1024), 0, s, L, lr, b1, b2, eps, c1, c2, lpart, loss);
    return hipGetLastError();
}

hipError_t conv_mse(const bf16* in, const bf16* w, const float* bias, int relu_in, int dil, int N, int H, int W,
                    const float* target, float scale, bf16* grad, float* lpart, hipStream_t s)
{
    if (dil > 16) return hipErrorInvalidValue;
    static_assert(kLossParts >= 512, "a loss partial per workgroup");
    const dim3 grid(resident_groups(dil, N, H, W)), block(64 * kColRW);
    if (relu_in)
        hipLaunchKernelGGL((k_conv_col<32, true, false, false, false, false, kColPix, false, false, true>), grid, block, 0,
                           s, in, w, bias, nullptr, nullptr, grad, dil, N, H, W, State5{}, Scales{}, nullptr, target,
                           scale, lpart);
    else
        hipLaunchKernelGGL((k_conv_col<32, false, false, false, false, false, kColPix, false, false, true>), grid, block,
                           0, s, in, w, bias, nullptr, nullptr, grad, dil, N, H, W, State5{}, Scales{}, nullptr, target,
                           scale, lpart);
    return hipGetLastError();
}

hipError_t bgrad(const bf16* dy, long long npix, float* part, int groups, float* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_bgrad, dim3(groups), dim3(256), 0, s, dy, npix, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return reduce(part, groups, 32, out, s);
}

hipError_t adam(float* p, const float* g, float* m1, float* m2, bf16* pb, long long n, float lr, float b1, float b2,
                float eps, int t, hipStream_t s)
{
    const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, g, m1, m2, pb, n, lr, b1, b2,
                       eps, c1, c2);
    return hipGetLastError();
}

hipError_t mse(const float* delta, const float* target, long long npix, int nout, float scale, bf16* grad,
               float* part, int groups, hipStream_t s)
{
    hipLaunchKernelGGL(k_mse, dim3(groups), dim3(256), 0, s, delta, target, npix, nout, scale, grad, part);
    return hipGetLastError();
}

static dim3 pix_grid(long long npix) { return dim3((unsigned)((npix + 255) / 256)); }

hipError_t pack(const State5& f, long long npix, int w, const Scales& sc, bf16* x, hipStream_t s)
{
    hipLaunchKernelGGL(k_pack, pix_grid(npix), dim3(256), 0, s, f, npix, w, sc, x);
    return hipGetLastError();
}

hipError_t pack_target(const State5& f0, const State5& f1, long long npix, const Scales& sc, float* t, hipStream_t s)
{
    hipLaunchKernelGGL(k_pack_target, pix_grid(npix), dim3(256), 0, s, f0, f1, npix, sc, t);
    return hipGetLastError();
}

hipError_t advance(const float* delta, long long npix, const Scales& sc, const State5& f, hipStream_t s)
{
    hipLaunchKernelGGL(k_advance, pix_grid(npix), dim3(256), 0, s, delta, npix, sc, f);
    return hipGetLastError();
}

// Partial sums of the judge for callers that cannot allocate device memory:
// a file-scope array of kJudgeMaxGroups * 8 doubles per GPU, held until the
// process ends.  In host code `scratch` names a host-side stand-in, not
// device memory: its device address is taken once per device with
// hipGetSymbolAddress (the device current at that call) and only that address
// is passed to kernels.
static __device__ __align__(256) double scratch[kJudgeMaxGroups * 8];

namespace {
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t judge_scratch_ptr(double** out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = static_cast<double*>(p);
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

hipError_t frame_sums(const State5& a, const State5* b, long long npix, int w, const Scales& sc, double* part,
                      int groups, double* out, hipStream_t s)
{
    const State5 bb = b ? *b : a;
    hipLaunchKernelGGL(k_frame_sums, dim3(groups), dim3(256), 0, s, a, bb, b != nullptr, npix, w, sc, part);
    hipLaunchKernelGGL(k_frame_final, dim3(1), dim3(256), 0, s, part, groups, b ? 8 : 1, out);
    return hipGetLastError();
}

}  // namespace sur
